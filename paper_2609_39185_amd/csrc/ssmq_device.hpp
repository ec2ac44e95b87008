// ssmq_device.hpp -- device primitives of the quantized state update (gfx950).
//
// Formats, thresholds and the dithered rounding of eq. (dither) (Section 2).
//
// The rule. Write |x| = s (K + F) on the local grid of the format (K integer,
// F in [0, 1)), u = U / 2^24 with U the 24-bit threshold. Eq. (dither) is a
// signed floor, s floor(x/s + u): a positive x rounds up iff u >= 1 - F, a
// negative x rounds away from zero iff u < F. With R the k dropped fraction
// bits, for k <= 24 both read "R + (U_e >> (24 - k)) >= 2^k" where U_e = U for
// x >= 0 and U_e = 2^24 - 1 - U for x < 0, i.e. the magnitude is rounded up
// iff adding U_e's top k bits to it carries. In a 32-bit threshold word thr
// (U = thr >> 8), U_e is the top 24 bits of thr ^ signmask(x).
//
// Fast paths (the gfx950 conversions, checked on the device against the exact
// rule): v_cvt_sr_{bf16,f16,fp8}_f32(x, r) round |x| up iff the top 24 bits of
// r, added as above, carry; fed r = thr ^ signmask they implement eq. (dither)
// wherever k <= 24. The plain casts and v_cvt_pk_fp8_f32 are round-to-nearest-
// even. What they do not cover goes to the exact software path below, inside a
// branch that is taken by a wave only when one of its lanes needs it:
//   bf16  nothing (k = 16 everywhere; NaN and Inf come out canonical);
//   fp16  the subnormal range |x| < 2^-14 (the conversion is not exact there);
//   E4M3  NaN (the conversion loses its sign) and |q| < 2^-10, where k > 24.
// E4M3 values are clamped to +-448 (saturation) before the stochastic
// conversions, which do not saturate.
//
// INT8 / INT4 (symmetric, block scale, Appendix B "Formats") round q = h / s
// on the integer lattice. With q24 = h * (2^24 / s) (exactly q * 2^24 whenever
// q is a normal float), X = floor(q24) and U the 24-bit threshold,
// floor(q + U / 2^24) = (X + U) >> 24 exactly: only the top 24 fraction bits of
// q can decide the comparison with a multiple of 2^-24. The low byte (nibble)
// of X + U shifted right by 24 is the stored code. Values saturate at +-qmax
// (see quantize_int_chunk); NaN and |q| < 2^-126 (q24 then differs from q * 2^24)
// take the exact path.
//
// Exact software path. Normal ranges use the carry rule on the magnitude bits.
// Below the smallest normal of fp16 and E4M3 the grid step is fixed, |x| / step
// has an exact fp32 integer part I and fraction F, and the rule is the exact
// fp32 comparison F >= 1 - u (x >= 0) or F > u (x < 0).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ssmq_launch.hpp"

namespace ssmq {

enum Fmt : int { kFP16 = 0, kBF16 = 1, kE4M3 = 2, kFP32 = 3, kINT8 = 4, kINT4 = 5 };
enum Rule : int { kRTN = 0, kSR = 1, kWEYL = 2, kPHILOX = 3 };

// Weyl accumulator (Appendix B "Dithers", hardware form): 2^32 times
// 0.7548776662, 0.5698402910, 0.1234567, 0.3141592, rounded to nearest, and the
// 32-bit golden increment (Section 6.4 "Three silent pitfalls").
constexpr uint32_t kWeylA = 0xC13FA9A9u;
constexpr uint32_t kWeylB = 0x91E10DA6u;
constexpr uint32_t kWeylL = 0x1F9ADBB9u;
constexpr uint32_t kWeylS = 0x506CBCC2u;
constexpr uint32_t kWeylPhi = 0x9E3779B9u;
// Hash SR multipliers: entry and step (Appendix B "Decode regime"), layer.
constexpr uint32_t kSrEntry = 0x9E3779B1u;
constexpr uint32_t kSrStep = 0x85EBCA77u;
constexpr uint32_t kSrLayer = 0xC2B2AE3Du;

// MurmurHash3 32-bit finalizer.
__host__ __device__ inline uint32_t fmix32(uint32_t h) {
  h ^= h >> 16;
  h *= 0x85EBCA6Bu;
  h ^= h >> 13;
  h *= 0xC2B2AE35u;
  h ^= h >> 16;
  return h;
}

// Per-step threshold keys (host and device). Weyl: the entry-independent part
// A + B + L layer + S seed + Phi t of the accumulator; hash SR: the chained key
// fmix32(fmix32(fmix32(seed) ^ layer * kSrLayer) ^ t * kSrStep).
__host__ __device__ inline uint32_t weyl_step_key(uint32_t seed, uint32_t layer, uint32_t step) {
  return kWeylA + kWeylB + kWeylL * layer + kWeylS * seed + kWeylPhi * step;
}
__host__ __device__ inline uint32_t sr_seed_key(uint32_t seed, uint32_t layer) {
  return fmix32(fmix32(seed) ^ (layer * kSrLayer));
}
__host__ __device__ inline uint32_t sr_step_key(uint32_t seed_key, uint32_t step) {
  return fmix32(seed_key ^ (step * kSrStep));
}

// A chunk is the unit one lane loads and stores: V entries in CB bytes (16, or
// 8 for INT4). Scaled formats keep one fp32 scale per group of entries;
// qmax is the value the group maximum is mapped to.
template <int F> struct Traits;
template <> struct Traits<kFP16> { static constexpr int V = 8, CB = 16; static constexpr bool scaled = false; };
template <> struct Traits<kBF16> { static constexpr int V = 8, CB = 16; static constexpr bool scaled = false; };
template <> struct Traits<kFP32> { static constexpr int V = 4, CB = 16; static constexpr bool scaled = false; };
// zh = fl32(1 / qmax) and zl = fl32(1 / qmax - zh) serve the group-scale division.
template <> struct Traits<kE4M3> {
  static constexpr int V = 16, CB = 16; static constexpr bool scaled = true;
  static constexpr float qmax = 448.0f, zh = 0x1.24924ap-9f, zl = -0x1.b6db6ep-34f;
};
template <> struct Traits<kINT8> {
  static constexpr int V = 16, CB = 16; static constexpr bool scaled = true;
  static constexpr float qmax = 127.0f, zh = 0x1.020408p-7f, zl = 0x1.020408p-35f;
};
template <> struct Traits<kINT4> {
  static constexpr int V = 16, CB = 8; static constexpr bool scaled = true;
  static constexpr float qmax = 7.0f, zh = 0x1.24924ap-3f, zl = -0x1.b6db6ep-28f;
};
template <int F> constexpr bool is_int_fmt = (F == kINT8 || F == kINT4);

template <int CB> struct ChunkOf;
template <> struct ChunkOf<16> { using type = uint4; };
template <> struct ChunkOf<8> { using type = uint2; };
template <int F> using chunk_t = typename ChunkOf<Traits<F>::CB>::type;

// Byte offset of the chunk that starts at entry e (a multiple of V).
template <int F, typename I>
__host__ __device__ constexpr I chunk_bytes_at(I e) {
  return e / static_cast<I>(Traits<F>::V) * static_cast<I>(Traits<F>::CB);
}

typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Thresholds. A chunk is V consecutive entries starting at a flat index e0 that
// is a multiple of V; entry k of the chunk uses thr_word(base(e0), off[k]) with
// off[k] precomputed on the host (Weyl: A (k >> lb) + B (k & (block-1)); SR:
// k * 0x9E3779B1).
// ---------------------------------------------------------------------------
template <int R>
__device__ inline uint32_t thr_base(uint64_t e0, const Thr& th) {
  if constexpr (R == kWEYL) {
    const uint32_t r = static_cast<uint32_t>(e0 >> th.lb);
    const uint32_t c = static_cast<uint32_t>(e0) & ((1u << th.lb) - 1u);
    return kWeylA * r + kWeylB * c + th.key;
  } else if constexpr (R == kSR) {
    return static_cast<uint32_t>(e0) * kSrEntry + th.key;
  } else {
    return 0u;
  }
}
template <int R>
__device__ inline uint32_t thr_word(uint32_t base, uint32_t off) {
  if constexpr (R == kWEYL) return base + off;
  else if constexpr (R == kSR) return fmix32(base + off);
  else return 0x80000000u;
}

// Philox4x32-10 (Salmon et al., SC 2011): ten rounds of two 32x32->64-bit
// products on a four-word counter, key advanced by the Weyl increments.
__device__ inline void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                     uint32_t k0, uint32_t k1, uint32_t (&out)[4]) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t p0 = static_cast<uint64_t>(0xD2511F53u) * c0;
    const uint64_t p1 = static_cast<uint64_t>(0xCD9E8D57u) * c2;
    // three-input XORs in one v_bitop3_b32 each (truth table 0x96)
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p1 >> 32), c1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32(static_cast<uint32_t>(p0 >> 32), c3, k1, 0x96);
    c1 = static_cast<uint32_t>(p1);
    c3 = static_cast<uint32_t>(p0);
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// Thresholds of one chunk of N entries whose first flat index is e0: tg(k) is
// the 32-bit word of entry k (U = word >> 8). Weyl and hash SR derive it from
// a per-chunk base and the per-position offsets; Philox SR draws word
// (e0 + k) mod 4 of the block with counter ((e0 + k) / 4, step, 0) and key
// (seed, layer).
template <int R, int N>
struct ChunkThr {
  uint32_t base;
  const uint32_t* off;
  __device__ uint32_t operator()(int k) const { return thr_word<R>(base, off[k]); }
};
template <int N>
struct ChunkThr<kPHILOX, N> {
  uint32_t w[N];
  __device__ uint32_t operator()(int k) const { return w[k]; }
};

// The 32-bit threshold word of one entry with global flat index i.
template <int R>
__device__ inline uint32_t entry_thr(uint64_t i, const Thr& th) {
  if constexpr (R == kPHILOX) {
    const uint64_t q = i >> 2;
    uint32_t o[4];
    philox4x32_10(static_cast<uint32_t>(q), static_cast<uint32_t>(q >> 32), th.step, 0u, th.seed,
                  th.layer, o);
    const uint32_t j = static_cast<uint32_t>(i) & 3u;
    return j == 0 ? o[0] : (j == 1 ? o[1] : (j == 2 ? o[2] : o[3]));
  } else {
    return thr_word<R>(thr_base<R>(i, th), 0u);
  }
}

template <int R, int N>
__device__ inline ChunkThr<R, N> chunk_thr(uint64_t e0, const Thr& th, uint32_t base,
                                           const uint32_t* off) {
  if constexpr (R == kPHILOX) {
    static_assert(N % 4 == 0, "Philox blocks cover four entries");
    ChunkThr<R, N> t;
    const uint64_t q0 = e0 >> 2;
#pragma unroll
    for (int g = 0; g < N / 4; ++g) {
      const uint64_t q = q0 + static_cast<uint64_t>(g);
      uint32_t o[4];
      philox4x32_10(static_cast<uint32_t>(q), static_cast<uint32_t>(q >> 32), th.step, 0u,
                    th.seed, th.layer, o);
#pragma unroll
      for (int i = 0; i < 4; ++i) t.w[4 * g + i] = o[i];
    }
    return t;
  } else {
    return ChunkThr<R, N>{base, off};
  }
}

// thr ^ signmask(x) in the top 24 bits (the low byte is don't-care).
__device__ inline uint32_t signed_thr(uint32_t thr, float x) {
  return thr ^ static_cast<uint32_t>(static_cast<int32_t>(__float_as_uint(x)) >> 24);
}

// ---------------------------------------------------------------------------
// Exact software rounding fp32 -> code.
// ---------------------------------------------------------------------------
template <bool RTN>
__device__ inline uint32_t round_fixed_step(float T, uint32_t neg, uint32_t thr) {
  const float I = floorf(T);
  const float F = T - I;  // exact
  bool up;
  if constexpr (RTN) {
    up = (F > 0.5f) || (F == 0.5f && (static_cast<uint32_t>(I) & 1u));
  } else {
    const uint32_t U = thr >> 8;
    up = neg ? (F > static_cast<float>(U) * 0x1p-24f)
             : (F >= static_cast<float>(0x1000000u - U) * 0x1p-24f);
  }
  return static_cast<uint32_t>(I) + (up ? 1u : 0u);
}

template <bool RTN>
__device__ inline uint32_t round_bf16(float x, uint32_t thr) {
  const uint32_t b = __float_as_uint(x);
  uint32_t add;
  if constexpr (RTN) {
    add = 0x7FFFu + ((b >> 16) & 1u);
  } else {
    const uint32_t sm = static_cast<uint32_t>(static_cast<int32_t>(b) >> 31);
    add = (thr ^ sm) >> 16;
  }
  uint32_t c = (b + add) >> 16;
  if ((b & 0x7FFFFFFFu) > 0x7F800000u) c = ((b >> 16) & 0x8000u) | 0x7FC0u;
  return c;
}

template <bool RTN>
__device__ inline uint32_t round_fp16(float x, uint32_t thr) {
  const uint32_t b = __float_as_uint(x);
  const uint32_t sign = (b >> 16) & 0x8000u;
  const uint32_t m = b & 0x7FFFFFFFu;
  uint32_t c;
  if (m >= 0x38800000u) {  // |x| >= 2^-14: normal range (k = 13) or overflow
    uint32_t add;
    if constexpr (RTN) {
      add = 0xFFFu + ((m >> 13) & 1u);
    } else {
      const uint32_t sm = static_cast<uint32_t>(static_cast<int32_t>(b) >> 31);
      add = (thr ^ sm) >> 19;
    }
    c = min(((m + add) >> 13) - (112u << 10), 0x7C00u);
  } else {                 // subnormal grid, step 2^-24
    c = round_fixed_step<RTN>(__uint_as_float(m) * 16777216.0f, sign, thr);
  }
  if (m > 0x7F800000u) c = 0x7E00u;
  return c | sign;
}

template <bool RTN>
__device__ inline uint32_t round_e4m3(float q, uint32_t thr) {
  const uint32_t b = __float_as_uint(q);
  const uint32_t sign = (b >> 24) & 0x80u;
  uint32_t m = b & 0x7FFFFFFFu;
  if (m > 0x7F800000u) return 0x7Fu | sign;  // NaN
  m = min(m, 0x43E00000u);                   // saturate at 448
  uint32_t c;
  if (m >= 0x3C800000u) {  // |q| >= 2^-6: normal range (k = 20)
    uint32_t add;
    if constexpr (RTN) {
      add = 0x7FFFFu + ((m >> 20) & 1u);
    } else {
      const uint32_t sm = static_cast<uint32_t>(static_cast<int32_t>(b) >> 31);
      add = (thr ^ sm) >> 12;
    }
    c = ((m + add) >> 20) - 960u;
  } else {                 // subnormal grid, step 2^-9
    c = round_fixed_step<RTN>(__uint_as_float(m) * 512.0f, sign, thr);
  }
  return c | sign;
}

// INT lattice, exact: q = h / s clamped to [-qmax, qmax], then floor(q + u)
// via the exact fp32 fraction (RTN: nearest, ties to even); NaN -> 0. Returns
// the two's complement code in the low bits.
template <bool RTN>
__device__ inline uint32_t round_int(float q, uint32_t thr, float qmax) {
  if (q != q) return 0u;
  q = fminf(fmaxf(q, -qmax), qmax);
  int k;
  if constexpr (RTN) {
    k = static_cast<int>(__builtin_rintf(q));
  } else {
    const float I = floorf(q);
    const float Fr = q - I;  // exact
    const uint32_t U = thr >> 8;
    k = static_cast<int>(I) + (Fr >= static_cast<float>(0x1000000u - U) * 0x1p-24f ? 1 : 0);
  }
  return static_cast<uint32_t>(k);
}

template <int F, int R>
__device__ inline uint32_t round_code(float x, uint32_t thr) {
  constexpr bool rtn = (R == kRTN);
  if constexpr (F == kBF16) return round_bf16<rtn>(x, thr);
  else if constexpr (F == kFP16) return round_fp16<rtn>(x, thr);
  else if constexpr (F == kE4M3) return round_e4m3<rtn>(x, thr);
  else if constexpr (F == kINT8) return round_int<rtn>(x, thr, 127.0f) & 0xFFu;
  else if constexpr (F == kINT4) return round_int<rtn>(x, thr, 7.0f) & 0xFu;
  else return __float_as_uint(x);
}

// ---------------------------------------------------------------------------
// Chunk quantizers: one chunk of fp32 values -> its codes, fast path plus the
// exact path for rare entries (the unscaled float formats here, E4M3 and the
// integer formats, which also take the group's 1 / s, further below).
// ---------------------------------------------------------------------------
template <int F>
__device__ inline void patch_code(uint32_t (&w)[4], int k, uint32_t c) {
  constexpr int bits = Traits<F>::CB * 8 / Traits<F>::V;  // code width
  if constexpr (bits == 32) {
    w[k] = c;
  } else {
    constexpr int per = 32 / bits;
    const int i = k / per, sh = (k % per) * bits;
    const uint32_t mask = ((1u << bits) - 1u) << sh;
    w[i] = (w[i] & ~mask) | ((c << sh) & mask);
  }
}

template <int F, int R>
__device__ inline bool needs_exact_path(float v) {
  if constexpr (F == kE4M3) {
    if constexpr (R == kRTN) return v != v;                            // NaN
    else return !(__builtin_fabsf(v) >= 0x1p-10f);                     // NaN or k > 24
  } else if constexpr (F == kFP16) {
    if constexpr (R == kRTN) return false;
    else return __builtin_fabsf(v) < 0x1p-14f;                         // subnormal range
  } else {
    return false;
  }
}

// Does any value of the chunk need the exact path (fp16 below its normal range)?
// The small-magnitude test uses the chunk minimum (fminf ignores NaN).
template <int F, int R, int V>
__device__ inline bool chunk_is_rare(const float (&v)[V]) {
  if constexpr (F != kFP16 || R == kRTN) {
    return false;
  } else {
    float mn = __builtin_fabsf(v[0]);
#pragma unroll
    for (int k = 1; k < V; ++k) mn = fminf(mn, __builtin_fabsf(v[k]));
    return mn < 0x1p-14f;
  }
}

// Whether any of the chunk's values is NaN, for callers without a cheaper test.
template <int V>
__device__ inline bool chunk_has_nan(const float (&v)[V]) {
  bool n = false;
#pragma unroll
  for (int k = 0; k < V; k += 2) n |= __builtin_isunordered(v[k], v[k + 1]);
  return n;
}

// The unscaled float formats need no NaN test: their conversions give the
// canonical NaN (maybe_nan is accepted for a uniform interface).
template <int F, int R, typename TG>
__device__ inline uint4 quantize_chunk(const float (&v)[Traits<F>::V], const TG& tg,
                                       bool /*maybe_nan*/) {
  static_assert(F == kBF16 || F == kFP16 || F == kFP32, "unscaled float formats");
  uint32_t w[4];
  if constexpr (F == kFP32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = __float_as_uint(v[i]);
    return make_uint4(w[0], w[1], w[2], w[3]);
  }
  if constexpr (F == kBF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v2bf p;
      if constexpr (R == kRTN) {
        p = (v2bf){static_cast<__bf16>(v[2 * i]), static_cast<__bf16>(v[2 * i + 1])};
      } else {
        // Both halves are written, so the destination's previous contents are
        // don't-care: it starts as the first threshold, which dies here.
        const uint32_t t0 = signed_thr(tg(2 * i), v[2 * i]);
        p = __builtin_amdgcn_cvt_sr_bf16_f32(__builtin_bit_cast(v2bf, t0), v[2 * i], t0, false);
        p = __builtin_amdgcn_cvt_sr_bf16_f32(
            p, v[2 * i + 1], signed_thr(tg(2 * i + 1), v[2 * i + 1]), true);
      }
      w[i] = __builtin_bit_cast(uint32_t, p);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v2h p;
      if constexpr (R == kRTN) {
        p = (v2h){static_cast<_Float16>(v[2 * i]), static_cast<_Float16>(v[2 * i + 1])};
      } else {
        const uint32_t t0 = signed_thr(tg(2 * i), v[2 * i]);
        p = __builtin_amdgcn_cvt_sr_f16_f32(__builtin_bit_cast(v2h, t0), v[2 * i], t0, false);
        p = __builtin_amdgcn_cvt_sr_f16_f32(
            p, v[2 * i + 1], signed_thr(tg(2 * i + 1), v[2 * i + 1]), true);
      }
      w[i] = __builtin_bit_cast(uint32_t, p);
    }
  }
  if (__builtin_amdgcn_ballot_w64(chunk_is_rare<F, R, Traits<F>::V>(v)) != 0) {
#pragma unroll
    for (int k = 0; k < Traits<F>::V; ++k) {
      if (needs_exact_path<F, R>(v[k])) patch_code<F>(w, k, round_code<F, R>(v[k], tg(k)));
    }
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// E4M3 chunk of 16 entries: h the fp32 values, r = fl32(1 / s) of their group.
// Values q = fl32(h r) exceed 448 only by the scale's own rounding (the scale
// maps the group maximum to 448): the stochastic conversions, which do not
// saturate, get q clamped with v_med3_f32 (clamping first is eq. (dither) on
// the saturated grid) unless the caller knows that no q of the group passes 448
// (clamp = false, wave-uniform: fl32(max|h| r) <= 448, rounding is monotonic);
// round-to-nearest needs no clamp below 464, which a scaled value never
// reaches. The exact path takes NaN (maybe_nan: a NaN may be among h) and
// |q| < 2^-10; since fl32(x r) is monotonic in x, the smallest |q| is
// fl32(min|h| r), one product per chunk.
template <int R, typename TG>
__device__ inline uint4 quantize_e4m3_chunk(const float (&h)[16], float r, const TG& tg,
                                            bool maybe_nan, bool clamp) {
  float q[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) q[k] = h[k] * r;
  // Philox SR always clamps: its generator already fills the registers that a
  // second code path would need.
  if (R != kRTN && (R == kPHILOX || clamp)) {
#pragma unroll
    for (int k = 0; k < 16; ++k) q[k] = __builtin_amdgcn_fmed3f(q[k], -448.0f, 448.0f);
  }
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int k = 4 * i;
    int d;  // all four bytes are written: the previous contents are don't-care
    if constexpr (R == kRTN) {
      d = __builtin_amdgcn_cvt_pk_fp8_f32(q[k], q[k + 1], static_cast<int>(__float_as_uint(q[k])), false);
      d = __builtin_amdgcn_cvt_pk_fp8_f32(q[k + 2], q[k + 3], d, true);
    } else {
      const uint32_t t0 = signed_thr(tg(k), q[k]);  // dies here
      d = __builtin_amdgcn_cvt_sr_fp8_f32(q[k], t0, static_cast<int>(t0), 0);
      d = __builtin_amdgcn_cvt_sr_fp8_f32(q[k + 1], signed_thr(tg(k + 1), q[k + 1]), d, 1);
      d = __builtin_amdgcn_cvt_sr_fp8_f32(q[k + 2], signed_thr(tg(k + 2), q[k + 2]), d, 2);
      d = __builtin_amdgcn_cvt_sr_fp8_f32(q[k + 3], signed_thr(tg(k + 3), q[k + 3]), d, 3);
    }
    w[i] = static_cast<uint32_t>(d);
  }
  bool rare = maybe_nan;
  if constexpr (R != kRTN) {
    // Started from +infinity, the chain is eight v_min3 with |h| as source
    // modifiers (from |h[0]| the compiler first canonicalises two values). A NaN in
    // h is caught by maybe_nan: it reaches the row's y.
    float mn = __builtin_inff();
#pragma unroll
    for (int k = 0; k < 16; ++k) mn = fminf(mn, __builtin_fabsf(h[k]));
    rare = rare || !(mn * r >= 0x1p-10f);
  }
  if (__builtin_amdgcn_ballot_w64(rare) != 0) {
    // The products are formed again here (r passed through an empty asm so that
    // they are not shared with q): q then needs no copy to survive the clamp.
    float rr = r;
    asm volatile("" : "+v"(rr));
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float v = h[k] * rr;
      if (needs_exact_path<kE4M3, R>(v)) patch_code<kE4M3>(w, k, round_code<kE4M3, R>(v, tg(k)));
    }
  }
  return make_uint4(w[0], w[1], w[2], w[3]);
}

// Byte `b` of each of four words, packed little-end first (v_perm_b32).
template <int B>
__device__ inline uint32_t pack_bytes(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3) {
  constexpr uint32_t lo = (0x0C0Cu << 16) | ((4u + B) << 8) | B;  // {w0.b, w1.b, 0, 0}
  const uint32_t p01 = __builtin_amdgcn_perm(w1, w0, lo);
  const uint32_t p23 = __builtin_amdgcn_perm(w3, w2, lo);
  return __builtin_amdgcn_perm(p23, p01, 0x05040100u);
}

// INT8 / INT4 chunk of 16 entries. h: the fp32 values, r = fl32(1 / s) and
// r24 = 2^24 r of their group (r24 is infinite when 2^24 r overflows);
// maybe_nan: a NaN may be among h. Saturation: the group's scale maps its maximum to
// qmax, so q passes qmax only by rounding, by at most qmax 2^-22.
//   Round to nearest needs no clamp: such a q still rounds to qmax.
//   Dithers clamp to +-qmax before the floor (CLAMP: v_med3_f32, one instruction per
//   entry; the bounds are lattice points, so this is the exact saturation).
//   INT8 dithers can do without (CLAMP = false): X + U then leaves the range of the codes
//   -127 .. 127 only if U lies within 2^9 of an end of its range, and a sum that has
//   done so reads, as a signed word, less than -127 2^24. The chunk's smallest sum
//   (half an instruction per entry) sends those to the exact path. It takes registers, so
//   it is left to the kernels where it pays: blocks with two chunks per thread, and
//   Mamba-1's. Elsewhere, 21M to 42M entries, Weyl, from a graph, without / with the clamp:
//   64x128 heads, one scale each (two spills more) 23.0 / 21.8 us; 64x64 heads, blocks of
//   16 (one chunk per thread, 74 / 66 registers) 13.5 / 13.1; rows of 48x128 heads 25.1 / 23.9.
// One layer of 268M entries in blocks of 128, against a clamp everywhere: INT8 Weyl
// 119.8 -> 118.1 us, INT8 RTN 97.7 -> 93.9 us, INT4 RTN 81.8 -> 77.6 us.
constexpr int32_t kInt8Low = -127 * (1 << 24);
template <int F, int R, bool CLAMP, typename TG>
__device__ inline chunk_t<F> quantize_int_chunk(const float (&h)[16], float r, float r24,
                                               const TG& tg, bool maybe_nan) {
  constexpr float qmax = Traits<F>::qmax;
  uint32_t S[16];
  bool rare = maybe_nan;
  if constexpr (R == kRTN) {
    // Adding 1.5 * 2^23 rounds q to an integer, ties to even (the sum's ulp is 1),
    // and leaves that integer's two's complement in the low bits of the sum's
    // encoding. (NaN, from an infinite group maximum, leaves 0.)
#pragma unroll
    for (int k = 0; k < 16; ++k) S[k] = __float_as_uint(h[k] * r + 0x1.8p23f);
  } else {
    float mn = __builtin_inff();
    int32_t low = 0;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float q24 = h[k] * r24;
      mn = fminf(mn, __builtin_fabsf(q24));
      float c24 = q24;
      if constexpr (CLAMP) c24 = __builtin_amdgcn_fmed3f(q24, -qmax * 0x1p24f, qmax * 0x1p24f);
      int X;  // floor
      asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(X) : "v"(c24));
      S[k] = static_cast<uint32_t>(X) + (tg(k) >> 8);
      if constexpr (!CLAMP) low = min(low, static_cast<int32_t>(S[k]));
    }
    rare = rare || !(mn >= 0x1p-102f) || !(r24 < __builtin_inff()) || low < kInt8Low;
  }
  constexpr int B = (R == kRTN) ? 0 : 3;  // the byte that holds the code
  uint32_t w[4];
  if constexpr (F == kINT8) {
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = pack_bytes<B>(S[4 * i], S[4 * i + 1], S[4 * i + 2], S[4 * i + 3]);
  } else {
    // even entries' bytes in one word, odd entries' in another, then nibble-interleave
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = 8 * i;
      const uint32_t ev = pack_bytes<B>(S[k], S[k + 2], S[k + 4], S[k + 6]);
      const uint32_t od = pack_bytes<B>(S[k + 1], S[k + 3], S[k + 5], S[k + 7]);
      w[i] = (ev & 0x0F0F0F0Fu) | ((od << 4) & 0xF0F0F0F0u);
    }
    w[2] = w[3] = 0u;
  }
  if (__builtin_amdgcn_ballot_w64(rare) != 0) {
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      bool exact;
      if constexpr (R == kRTN) {
        exact = h[k] != h[k];
      } else {
        // NaN, q below the normal range (q24 then differs from q 2^24), r24 overflowed, or
        // an unclamped sum out of the codes' range
        exact = !(__builtin_fabsf(h[k] * r24) >= 0x1p-102f) || !(r24 < __builtin_inff()) ||
                (!CLAMP && static_cast<int32_t>(S[k]) < kInt8Low);
      }
      if (exact) patch_code<F>(w, k, round_code<F, R>(h[k] * r, tg(k)));
    }
  }
  if constexpr (F == kINT8) return make_uint4(w[0], w[1], w[2], w[3]);
  else return make_uint2(w[0], w[1]);
}

// One chunk of fp32 values h -> codes, for every format: r = 1 / s of the
// chunk's group (ignored by unscaled formats). INT_CLAMP: the integer formats' dithers
// clamp (see quantize_int_chunk).
template <int F, int R, bool INT_CLAMP = true, typename TG>
__device__ inline chunk_t<F> quantize_any(const float (&h)[Traits<F>::V], float r, const TG& tg,
                                         bool maybe_nan, bool clamp = true) {
  if constexpr (is_int_fmt<F>) {
    return quantize_int_chunk<F, R, INT_CLAMP>(h, r, r * 0x1p24f, tg, maybe_nan);
  } else if constexpr (F == kE4M3) {
    return quantize_e4m3_chunk<R>(h, r, tg, maybe_nan, clamp);
  } else {
    return quantize_chunk<F, R>(h, tg, maybe_nan);
  }
}

// The exact fp32 value of one code (E4M3 and INT without the group scale).
template <int F>
__device__ inline float code_value(uint32_t c) {
  if constexpr (F == kBF16) return __uint_as_float(c << 16);
  else if constexpr (F == kFP16) return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(c)));
  else if constexpr (F == kE4M3) return __builtin_amdgcn_cvt_f32_fp8(static_cast<int>(c), 0);
  else if constexpr (F == kINT8) return static_cast<float>(static_cast<int32_t>(c << 24) >> 24);
  else if constexpr (F == kINT4) return static_cast<float>(static_cast<int32_t>(c << 28) >> 28);
  else return __uint_as_float(c);
}

// ---------------------------------------------------------------------------
// Decoding code -> its exact value as fp32 (E4M3 without the group scale, via
// v_cvt_pk_f32_fp8, which decodes OCP E4M3 exactly).
// ---------------------------------------------------------------------------
template <int F>
__device__ inline void decode_chunk(const uint2& raw, float (&out)[Traits<F>::V]) {
  static_assert(F == kINT4, "8-byte chunks hold INT4 codes");
  const uint32_t w[2] = {raw.x, raw.y};
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
      out[8 * i + j] = static_cast<float>(static_cast<int32_t>(w[i] << (28 - 4 * j)) >> 28);
}

template <int F>
__device__ inline void decode_chunk(const uint4& raw, float (&out)[Traits<F>::V]) {
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (F == kBF16) {
      out[2 * i] = __uint_as_float(w[i] << 16);
      out[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    } else if constexpr (F == kFP16) {
      const v2h p = __builtin_bit_cast(v2h, w[i]);
      out[2 * i] = static_cast<float>(p.x);
      out[2 * i + 1] = static_cast<float>(p.y);
    } else if constexpr (F == kE4M3) {
      const v2f lo = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(w[i]), false);
      const v2f hi = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(w[i]), true);
      out[4 * i] = lo.x;
      out[4 * i + 1] = lo.y;
      out[4 * i + 2] = hi.x;
      out[4 * i + 3] = hi.y;
    } else if constexpr (F == kINT8) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        out[4 * i + j] = static_cast<float>(static_cast<int8_t>(w[i] >> (8 * j)));
    } else {
      out[i] = __uint_as_float(w[i]);
    }
  }
}

// Group scale of a scaled format: s = fl32(m / qmax), flushed to zero below
// 2^-126. For m in [2^-112, FLT_MAX], fma(m, zh, fl32(m zl)) is the correctly
// rounded quotient (Brisebarre, Muller and Raina, "Accelerating correctly rounded
// floating-point division when the divisor is known in advance", 2004; checked
// here for every such fp32 m and qmax = 7, 127, 448); smaller or infinite m
// divide (a wave-uniform branch, taken only by waves that hold such a group).
template <int F>
__device__ inline float group_scale(float m) {
  float s = fmaf(m, Traits<F>::zh, m * Traits<F>::zl);
  const bool slow = !(m >= 0x1p-112f && m <= 3.40282347e38f);
  if (__builtin_amdgcn_ballot_w64(slow) != 0) {
    // The empty asm keeps the division inside the branch: hoisted out of it
    // (the compiler's choice for a cheap-looking fdiv), every group pays for it.
    float mm = m;
    asm volatile("" : "+v"(mm));
    if (slow) s = mm / Traits<F>::qmax;
  }
  return (s >= 1.17549435e-38f) ? s : 0.0f;
}

// r = fl32(1 / s) for a group scale s: 0 for s = 0 or s infinite; otherwise
// s lies in [2^-126, 2^126), where one Newton step from v_rcp_f32,
// fma(fma(-s, y0, 1), y0, y0), is the correctly rounded reciprocal (checked on
// the device for every fp32 value in that range).
__device__ inline float recip_scale(float s) {
  const float y0 = __builtin_amdgcn_rcpf(s);
  const float r = fmaf(fmaf(-s, y0, 1.0f), y0, y0);
  return (s > 0.0f && s < __builtin_inff()) ? r : 0.0f;
}

// ---------------------------------------------------------------------------
// fl32(exp(z)), correctly rounded: exp in double, one rounding to fp32. For every fp32
// argument the results are those of (float)exp((double)z) (checked on the device).
// Two forms, both without a branch but for |z| > 700, where the double's exponent
// would wrap (the result is 0 or infinity there):
//   exp_values        k = rint(z log2 e), r = z - k ln 2 (ln 2 in two doubles), exp(r)
//                     on |r| <= ln 2 / 2 by a degree-11 minimax polynomial (Remez
//                     exchange, relative error 2^-53.7): 17 double operations, for
//                     lanes that take several.
//   exp_values_table  k = rint(z 256 / ln 2), 2^(k mod 256 / 256) from a table in LDS
//                     and exp(r) - 1 on |r| <= ln 2 / 512 by its Taylor polynomial of
//                     degree 4 (relative error 2^-54.5): 11 double operations, for
//                     workgroups that take several thousand.
// A double operation issues in as many cycles as a three-operand fp32 one (4.7 at a
// nominal 2.4 GHz), and the library's exp takes about 20 and branches.
// ---------------------------------------------------------------------------
// p with k << shift added to its upper word (one instruction; written out, the
// compiler makes a 64-bit addition of it).
template <int SHIFT>
__device__ inline double add_exponent(double p, uint32_t k) {
  typedef unsigned int words __attribute__((ext_vector_type(2)));
  words w = __builtin_bit_cast(words, p);
  uint32_t hi = w.y;
  asm("v_lshl_add_u32 %0, %1, %2, %0" : "+v"(hi) : "v"(k), "n"(SHIFT));
  w.y = hi;
  return __builtin_bit_cast(double, w);
}
constexpr float kExpRange = 700.0f;
template <int N>
__device__ inline void exp_out_of_range(const float (&z)[N], float (&out)[N]) {
  float m = 0.0f;  // ignores NaN, which the common path keeps
#pragma unroll
  for (int i = 0; i < N; ++i) m = fmaxf(m, __builtin_fabsf(z[i]));
  if (__builtin_amdgcn_ballot_w64(m > kExpRange) != 0) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (z[i] > kExpRange) out[i] = __builtin_inff();
      if (z[i] < -kExpRange) out[i] = 0.0f;
    }
  }
}
__device__ inline float exp_in_range(float zf) {
  const double z = static_cast<double>(zf);
  const double t = __builtin_fma(z, 0x1.71547652b82fep+0, 0x1.8p52);  // k in the low bits
  const uint32_t k = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, t));
  const double kd = t - 0x1.8p52;
  double r = __builtin_fma(kd, -0x1.62e42fefa39efp-1, z);
  r = __builtin_fma(kd, -0x1.abc9e3b39803fp-56, r);
  double p = __builtin_fma(r, 0x1.8ad0f40784e9dp-26, 0x1.28a2c68333593p-22);
  p = __builtin_fma(p, r, 0x1.71f6152e4b934p-19);
  p = __builtin_fma(p, r, 0x1.a019a66a00698p-16);
  p = __builtin_fma(p, r, 0x1.a019f62058ba4p-13);
  p = __builtin_fma(p, r, 0x1.6c16c17f41b14p-10);
  p = __builtin_fma(p, r, 0x1.111111137ba72p-7);
  p = __builtin_fma(p, r, 0x1.55555555520c1p-5);
  p = __builtin_fma(p, r, 0x1.555555555481ap-3);
  p = __builtin_fma(p, r, 0x1.0000000000005p-1);
  p = __builtin_fma(p, r, 0x1.0000000000003p+0);
  p = __builtin_fma(p, r, 1.0);
  return static_cast<float>(add_exponent<20>(p, k));
}
// N of them in one stretch of code, so that their chains overlap, with one test of the
// range: a branch for each left every chain of 17 operations to itself. Row kernel, E4M3 RTN,
// 2048 channels of 64 states, from a graph: one sequence 4.01 -> 3.45 us (with the library's
// exp 3.45), 64 sequences 11.9 -> 10.3 us (11.3).
template <int N>
__device__ inline void exp_values(const float (&z)[N], float (&out)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) out[i] = exp_in_range(z[i]);
  exp_out_of_range<N>(z, out);
}
// One alone, as the exhaustive check takes it too.
__device__ inline float exp_value(float zf) {
  const float z[1] = {zf};
  float out[1];
  exp_values<1>(z, out);
  return out[0];
}

// 2^(j/256) with j 2^-8 taken off the exponent field in advance, so that adding
// k 2^-8 (k = 256 n + j) leaves the exponent n.
constexpr int kExpTable = 256;
__device__ const uint64_t kExpTableBits[kExpTable] = {
    0x3ff0000000000000ull, 0x3feffb1afa5abcbfull, 0x3feff63da9fb3335ull, 0x3feff168143b0281ull, 0x3fefec9a3e778061ull,
    0x3fefe7d42e11bbccull, 0x3fefe315e86e7f85ull, 0x3fefde5f72f654b1ull, 0x3fefd9b0d3158574ull, 0x3fefd50a0e3c1f89ull,
    0x3fefd06b29ddf6deull, 0x3fefcbd42b72a836ull, 0x3fefc74518759bc8ull, 0x3fefc2bdf66607e0ull, 0x3fefbe3ecac6f383ull,
    0x3fefb9c79b1f3919ull, 0x3fefb5586cf9890full, 0x3fefb0f145e46c85ull, 0x3fefac922b7247f7ull, 0x3fefa83b23395decull,
    0x3fefa3ec32d3d1a2ull, 0x3fef9fa55fdfa9c5ull, 0x3fef9b66affed31bull, 0x3fef973028d7233eull, 0x3fef9301d0125b51ull,
    0x3fef8edbab5e2ab6ull, 0x3fef8abdc06c31ccull, 0x3fef86a814f204abull, 0x3fef829aaea92de0ull, 0x3fef7e95934f312eull,
    0x3fef7a98c8a58e51ull, 0x3fef76a45471c3c2ull, 0x3fef72b83c7d517bull, 0x3fef6ed48695bbc0ull, 0x3fef6af9388c8deaull,
    0x3fef672658375d2full, 0x3fef635beb6fcb75ull, 0x3fef5f99f8138a1cull, 0x3fef5be084045cd4ull, 0x3fef582f95281c6bull,
    0x3fef54873168b9aaull, 0x3fef50e75eb44027ull, 0x3fef4d5022fcd91dull, 0x3fef49c18438ce4dull, 0x3fef463b88628cd6ull,
    0x3fef42be3578a819ull, 0x3fef3f49917ddc96ull, 0x3fef3bdda27912d1ull, 0x3fef387a6e756238ull, 0x3fef351ffb82140aull,
    0x3fef31ce4fb2a63full, 0x3fef2e85711ece75ull, 0x3fef2b4565e27cddull, 0x3fef280e341ddf29ull, 0x3fef24dfe1f56381ull,
    0x3fef21ba7591bb70ull, 0x3fef1e9df51fdee1ull, 0x3fef1b8a66d10f13ull, 0x3fef187fd0dad990ull, 0x3fef157e39771b2full,
    0x3fef1285a6e4030bull, 0x3fef0f961f641589ull, 0x3fef0cafa93e2f56ull, 0x3fef09d24abd886bull, 0x3fef06fe0a31b715ull,
    0x3fef0432edeeb2fdull, 0x3fef0170fc4cd831ull, 0x3feefeb83ba8ea32ull, 0x3feefc08b26416ffull, 0x3feef96266e3fa2dull,
    0x3feef6c55f929ff1ull, 0x3feef431a2de883bull, 0x3feef1a7373aa9cbull, 0x3feeef26231e754aull, 0x3feeecae6d05d866ull,
    0x3feeea401b7140efull, 0x3feee7db34e59ff7ull, 0x3feee57fbfec6cf4ull, 0x3feee32dc313a8e5ull, 0x3feee0e544ede173ull,
    0x3feedea64c123422ull, 0x3feedc70df1c5175ull, 0x3feeda4504ac801cull, 0x3feed822c367a024ull, 0x3feed60a21f72e2aull,
    0x3feed3fb2709468aull, 0x3feed1f5d950a897ull, 0x3feecffa3f84b9d4ull, 0x3feece086061892dull, 0x3feecc2042a7d232ull,
    0x3feeca41ed1d0057ull, 0x3feec86d668b3237ull, 0x3feec6a2b5c13cd0ull, 0x3feec4e1e192aed2ull, 0x3feec32af0d7d3deull,
    0x3feec17dea6db7d7ull, 0x3feebfdad5362a27ull, 0x3feebe41b817c114ull, 0x3feebcb299fddd0dull, 0x3feebb2d81d8abffull,
    0x3feeb9b2769d2ca7ull, 0x3feeb8417f4531eeull, 0x3feeb6daa2cf6642ull, 0x3feeb57de83f4eefull, 0x3feeb42b569d4f82ull,
    0x3feeb2e2f4f6ad27ull, 0x3feeb1a4ca5d920full, 0x3feeb070dde910d2ull, 0x3feeaf4736b527daull, 0x3feeae27dbe2c4cfull,
    0x3feead12d497c7fdull, 0x3feeac0827ff07ccull, 0x3feeab07dd485429ull, 0x3feeaa11fba87a03ull, 0x3feea9268a5946b7ull,
    0x3feea84590998b93ull, 0x3feea76f15ad2148ull, 0x3feea6a320dceb71ull, 0x3feea5e1b976dc09ull, 0x3feea52ae6cdf6f4ull,
    0x3feea47eb03a5585ull, 0x3feea3dd1d1929fdull, 0x3feea34634ccc320ull, 0x3feea2b9febc8fb7ull, 0x3feea23882552225ull,
    0x3feea1c1c70833f6ull, 0x3feea155d44ca973ull, 0x3feea0f4b19e9538ull, 0x3feea09e667f3bcdull, 0x3feea052fa75173eull,
    0x3feea012750bdabfull, 0x3fee9fdcddd47645ull, 0x3fee9fb23c651a2full, 0x3fee9f9298593ae5ull, 0x3fee9f7df9519484ull,
    0x3fee9f7466f42e87ull, 0x3fee9f75e8ec5f74ull, 0x3fee9f8286ead08aull, 0x3fee9f9a48a58174ull, 0x3fee9fbd35d7cbfdull,
    0x3fee9feb564267c9ull, 0x3feea024b1ab6e09ull, 0x3feea0694fde5d3full, 0x3feea0b938ac1cf6ull, 0x3feea11473eb0187ull,
    0x3feea17b0976cfdbull, 0x3feea1ed0130c132ull, 0x3feea26a62ff86f0ull, 0x3feea2f336cf4e62ull, 0x3feea3878491c491ull,
    0x3feea427543e1a12ull, 0x3feea4d2add106d9ull, 0x3feea589994cce13ull, 0x3feea64c1eb941f7ull, 0x3feea71a4623c7adull,
    0x3feea7f4179f5b21ull, 0x3feea8d99b4492edull, 0x3feea9cad931a436ull, 0x3feeaac7d98a6699ull, 0x3feeabd0a478580full,
    0x3feeace5422aa0dbull, 0x3feeae05bad61778ull, 0x3feeaf3216b5448cull, 0x3feeb06a5e0866d9ull, 0x3feeb1ae99157736ull,
    0x3feeb2fed0282c8aull, 0x3feeb45b0b91ffc6ull, 0x3feeb5c353aa2fe2ull, 0x3feeb737b0cdc5e5ull, 0x3feeb8b82b5f98e5ull,
    0x3feeba44cbc8520full, 0x3feebbdd9a7670b3ull, 0x3feebd829fde4e50ull, 0x3feebf33e47a22a2ull, 0x3feec0f170ca07baull,
    0x3feec2bb4d53fe0dull, 0x3feec49182a3f090ull, 0x3feec674194bb8d5ull, 0x3feec86319e32323ull, 0x3feeca5e8d07f29eull,
    0x3feecc667b5de565ull, 0x3feece7aed8eb8bbull, 0x3feed09bec4a2d33ull, 0x3feed2c980460ad8ull, 0x3feed503b23e255dull,
    0x3feed74a8af46052ull, 0x3feed99e1330b358ull, 0x3feedbfe53c12e59ull, 0x3feede6b5579fdbfull, 0x3feee0e521356ebaull,
    0x3feee36bbfd3f37aull, 0x3feee5ff3a3c2774ull, 0x3feee89f995ad3adull, 0x3feeeb4ce622f2ffull, 0x3feeee07298db666ull,
    0x3feef0ce6c9a8952ull, 0x3feef3a2b84f15fbull, 0x3feef68415b749b1ull, 0x3feef9728de5593aull, 0x3feefc6e29f1c52aull,
    0x3feeff76f2fb5e47ull, 0x3fef028cf22749e4ull, 0x3fef05b030a1064aull, 0x3fef08e0b79a6f1full, 0x3fef0c1e904bc1d2ull,
    0x3fef0f69c3f3a207ull, 0x3fef12c25bd71e09ull, 0x3fef16286141b33dull, 0x3fef199bdd85529cull, 0x3fef1d1cd9fa652cull,
    0x3fef20ab5fffd07aull, 0x3fef244778fafb22ull, 0x3fef27f12e57d14bull, 0x3fef2ba88988c933ull, 0x3fef2f6d9406e7b5ull,
    0x3fef33405751c4dbull, 0x3fef3720dcef9069ull, 0x3fef3b0f2e6d1675ull, 0x3fef3f0b555dc3faull, 0x3fef43155b5bab74ull,
    0x3fef472d4a07897cull, 0x3fef4b532b08c968ull, 0x3fef4f87080d89f2ull, 0x3fef53c8eacaa1d6ull, 0x3fef5818dcfba487ull,
    0x3fef5c76e862e6d3ull, 0x3fef60e316c98398ull, 0x3fef655d71ff6075ull, 0x3fef69e603db3285ull, 0x3fef6e7cd63a8315ull,
    0x3fef7321f301b460ull, 0x3fef77d5641c0658ull, 0x3fef7c97337b9b5full, 0x3fef81676b197d17ull, 0x3fef864614f5a129ull,
    0x3fef8b333b16ee12ull, 0x3fef902ee78b3ff6ull, 0x3fef953924676d76ull, 0x3fef9a51fbc74c83ull, 0x3fef9f7977cdb740ull,
    0x3fefa4afa2a490daull, 0x3fefa9f4867cca6eull, 0x3fefaf482d8e67f1ull, 0x3fefb4aaa2188510ull, 0x3fefba1bee615a27ull,
    0x3fefbf9c1cb6412aull, 0x3fefc52b376bba97ull, 0x3fefcac948dd7274ull, 0x3fefd0765b6e4540ull, 0x3fefd632798844f8ull,
    0x3fefdbfdad9cbe14ull, 0x3fefe1d802243c89ull, 0x3fefe7c1819e90d8ull, 0x3fefedba3692d514ull, 0x3feff3c22b8f71f1ull,
    0x3feff9d96b2a23d9ull,
};
// Copies the table to LDS (a barrier of the caller's has to follow).
__device__ inline void stage_exp_table(double* tab, int t, int threads) {
  for (int i = t; i < kExpTable; i += threads) tab[i] = __builtin_bit_cast(double, kExpTableBits[i]);
}
// p = fma(p, r, c), c in a scalar register pair: left to itself the compiler takes the
// two-operand form, which overwrites its addend, and copies c into vector registers
// for every term.
__device__ inline double fma_s(double p, double r, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(p), "v"(r), "s"(c));
  return d;
}
template <int N>
__device__ inline void exp_values_table(const double* tab, const float (&z)[N], float (&out)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double zd = static_cast<double>(z[i]);
    const double t = __builtin_fma(zd, 0x1.71547652b82fep+8, 0x1.8p52);
    const uint32_t k = static_cast<uint32_t>(__builtin_bit_cast(uint64_t, t));
    const double T = add_exponent<12>(tab[k & (kExpTable - 1)], k);
    const double kd = t - 0x1.8p52;
    double r = __builtin_fma(kd, -0x1.62e42fefa39efp-9, zd);
    r = __builtin_fma(kd, -0x1.abc9e3b39803fp-64, r);
    double p = fma_s(r, 0x1.5555555555555p-5, 0x1.5555555555555p-3);
    p = __builtin_fma(p, r, 0.5);
    p = __builtin_fma(p, r, 1.0);
    out[i] = static_cast<float>(__builtin_fma(p, T * r, T));
  }
  exp_out_of_range<N>(z, out);
}

// ---------------------------------------------------------------------------
// Cross-lane reductions over aligned groups of `width` lanes (a power of two
// <= 64): DPP within 16-lane rows, then swizzles across rows.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ inline float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                               CTRL, 0xF, 0xF, false));
}
constexpr int kQuadXor1 = 0xB1;     // quad_perm [1,0,3,2]
constexpr int kQuadXor2 = 0x4E;     // quad_perm [2,3,0,1]
constexpr int kHalfMirror = 0x141;  // lane i <-> 7 - i within 8
constexpr int kRowMirror = 0x140;   // lane i <-> 15 - i within 16

__device__ inline float lane_sum(float v, int width) {
  if (width >= 2) v += dpp_f<kQuadXor1>(v);
  if (width >= 4) v += dpp_f<kQuadXor2>(v);
  if (width >= 8) v += dpp_f<kHalfMirror>(v);
  if (width >= 16) v += dpp_f<kRowMirror>(v);
  if (width >= 32) v += __shfl_xor(v, 16, 64);
  if (width >= 64) v += __shfl_xor(v, 32, 64);
  return v;
}
template <int CTRL>
__device__ inline uint32_t dpp_u(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, false));
}
// Maximum of unsigned words (bit patterns of non-negative, non-NaN floats).
__device__ inline uint32_t lane_umax(uint32_t v, int width) {
  if (width >= 2) v = max(v, dpp_u<kQuadXor1>(v));
  if (width >= 4) v = max(v, dpp_u<kQuadXor2>(v));
  if (width >= 8) v = max(v, dpp_u<kHalfMirror>(v));
  if (width >= 16) v = max(v, dpp_u<kRowMirror>(v));
  if (width >= 32) v = max(v, static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 16, 64)));
  if (width >= 64) v = max(v, static_cast<uint32_t>(__shfl_xor(static_cast<int>(v), 32, 64)));
  return v;
}

// Streaming (nontemporal) 16- and 8-byte accesses for the state.
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
template <typename C>
__device__ inline C load_stream(const void* p);
template <>
__device__ inline uint4 load_stream<uint4>(const void* p) {
  const v4u v = __builtin_nontemporal_load(static_cast<const v4u*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
template <>
__device__ inline uint2 load_stream<uint2>(const void* p) {
  const v2u v = __builtin_nontemporal_load(static_cast<const v2u*>(p));
  return make_uint2(v.x, v.y);
}
__device__ inline void store_stream(void* p, const uint4& v) {
  const v4u w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, static_cast<v4u*>(p));
}
__device__ inline void store_stream(void* p, const uint2& v) {
  const v2u w = {v.x, v.y};
  __builtin_nontemporal_store(w, static_cast<v2u*>(p));
}

}  // namespace ssmq
