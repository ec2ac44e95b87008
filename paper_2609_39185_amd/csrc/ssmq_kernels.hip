// ssmq_kernels.hip -- HIP kernels of the quantized selective-state update (gfx950).
//
// Kernels:
//   k_update_slab  Mamba-2 heads (scalar A per head): a workgroup updates a slab
//                  of rows of one (batch, head) tile: dequantize -> exp(dt A) ->
//                  FMA recurrence -> y = C h + D x -> (E4M3 group scale) ->
//                  threshold -> round -> store, in registers, so the state
//                  crosses HBM once each way (Section 2 eq. (rec) and eq.
//                  (dither); Appendix B "Runners", "Formats", "Dithers").
//   k_update_channels  the same step for large batches of Mamba-1 layers (heads of one
//                  row of 16 entries, A per (channel, n)): a workgroup takes a tile of
//                  channels through several sequences.
//   k_update_rows  the same step for any other row layout (Mamba-2 heads smaller
//                  than a slab, A per (head, n) with other rows or several B/C groups), and the
//                  checkpoint write on an fp32 state.
//   k_requant      fp32 -> codes for fp16 / bf16 / fp32, one chunk per thread.
//   k_requant_scaled fp32 -> E4M3 / INT8 / INT4 codes with group scales.
//   k_dither_fill  the 24-bit thresholds themselves.
//   k_conv1d_update the causal depthwise convolution's decode step.
//   k_replay       open-loop replay of recorded decays and writes: a reference
//                  and a stored trajectory per entry, iterated in registers.
//
// Layout. A chunk is the codes of V consecutive entries of one state row: 16
// bytes holding 8 fp16 / bf16, 16 E4M3 / INT8 or 4 fp32 entries, or 8 bytes
// holding 16 INT4 entries. The LR = dstate / V chunks of a row sit in LR
// consecutive lanes of one wave, so a lane's slice of B and C is fixed and C.h
// is an LR-lane reduction. Each thread owns CPT chunks (one row per pass); the
// state moves with nontemporal 16- or 8-byte accesses (each byte is touched once
// per step, so nothing is gained by keeping it in the caches).
#include "ssmq_device.hpp"

namespace ssmq {

template <int V>
__device__ inline void load_floats(const float* p, float (&out)[V]) {
#pragma unroll
  for (int i = 0; i < V; i += 4) {
    const float4 v = *reinterpret_cast<const float4*>(p + i);
    out[i] = v.x; out[i + 1] = v.y; out[i + 2] = v.z; out[i + 3] = v.w;
  }
}

// dA = fl32(exp(fl32(dt A))), correctly rounded. One per lane or per head: the library's exp,
// rounded once, is no slower there than the forms of ssmq_device.hpp (same bits), which serve
// lanes that take many.
__device__ inline float decay(float dtv, float a) {
  return static_cast<float>(exp(static_cast<double>(dtv * a)));
}
template <int N>
__device__ inline void decays(float dtv, const float (&a)[N], float (&dA)[N]) {
  float z[N];
#pragma unroll
  for (int k = 0; k < N; ++k) z[k] = dtv * a[k];
  exp_values<N>(z, dA);
}

// The step size the update uses: dt, plus dt_bias[head] when given, through
// softplus(v) = log(1 + e^v) (double, one rounding; v itself above 20) when asked.
__device__ inline float step_bias(const UpdateArgs& a, int head) {
  return a.dt_bias ? a.dt_bias[head] : 0.0f;
}
__device__ inline float step_size(const UpdateArgs& a, float dtv, float bias) {
  if (a.dt_bias) dtv = dtv + bias;
  if (a.dt_softplus && !(dtv > 20.0f)) dtv = static_cast<float>(log1p(exp(static_cast<double>(dtv))));
  return dtv;
}

__device__ inline float silu(float v) { return v / (1.0f + expf(-v)); }

// ---------------------------------------------------------------------------
// Mamba-2 head slabs: NT threads x CPT chunks = a run of whole rows of one head.
// ---------------------------------------------------------------------------
// The whole-head configurations of the scaled formats (four chunks per thread,
// up to 128 threads) hold 64 state values per thread and sit near the
// 128-register line; they are held to it (four waves per SIMD) instead of
// dropping to three waves.
//
// LR > 0: a row is LR lanes and a scale group LG lanes (one row, or one lane) or the whole
// head, so the lanes per row and per group are compile-time constants: the reductions lose their runtime
// width tests. 44M entries, one group per row: 64x256 heads INT8 Weyl 25.6 -> 22.6 us, RTN
// 22.1 -> 18.3 us; 32x256 INT4 RTN 18.0 -> 14.3 us; 128x64 INT8 Weyl 23.9 -> 21.7 us.
// A group per lane (blocks of 16), 44M entries: INT8 Weyl 24.9 -> 23.0 us, RTN 22.8 -> 20.5 us, INT4 RTN
// 20.4 -> 17.0 us, E4M3 RTN 22.5 -> 21.5 us.
constexpr int log2c(int v) { return v <= 1 ? 0 : 1 + log2c(v / 2); }

template <int F, int R, int NT, int CPT, int LR = 0, int LG = LR>
__global__ __launch_bounds__(NT, (Traits<F>::scaled && CPT == 4 && NT <= 128) ? 4 : 1)
void k_update_slab(UpdateArgs a) {
  constexpr int V = Traits<F>::V;
  constexpr int NW = NT / 64;
  const int lanes_per_row = LR ? LR : a.lanes_per_row;
  const int lr_shift = LR ? log2c(LR) : a.lr_shift;
  const int lanes_per_group = LR ? LG : a.lanes_per_group;  // when not the whole head
  const int t = threadIdx.x;
  const uint32_t blk = blockIdx.x;
  const uint32_t tile32 = a.div_slabs.div(blk);  // b * nheads + h
  const uint32_t slab = blk - tile32 * static_cast<uint32_t>(a.slabs_per_head);
  const uint32_t b32 = a.div_nheads.div(tile32);
  const int hh = static_cast<int>(tile32 - b32 * static_cast<uint32_t>(a.nheads));
  const int g = static_cast<int>(a.div_hpg.div(static_cast<uint32_t>(hh)));
  const int64_t tile = tile32, b = b32;
  const int cc = t & (lanes_per_row - 1);
  const int n0 = cc * V;
  const int rows_per_pass = NT >> lr_shift;
  const int r0 = (t >> lr_shift) + static_cast<int>(slab) * rows_per_pass * CPT;
  const int64_t tile_base = tile * a.head_size;
  // Uniform bases plus 32-bit lane offsets (a head holds fewer than 2^31 bytes).
  uint8_t* const hstate = static_cast<uint8_t*>(a.state) + chunk_bytes_at<F>(tile_base);
  const float* const hx = a.x + tile * a.headdim;
  float* const hy = a.y + tile * a.headdim;
  const uint32_t l0 = static_cast<uint32_t>(r0 * a.dstate + n0);  // lane's first entry in the head
  const uint32_t pass = static_cast<uint32_t>(rows_per_pass * a.dstate);  // entries per pass
  const int64_t e0 = tile_base + l0;

  // Per-head values are staged once per workgroup in LDS while the state loads
  // are in flight: B and C of the head's group (one float4 per thread, loaded
  // before the state so that staging them waits for them alone), and exp(dt A),
  // evaluated by the first wave in double with one final rounding.
  __shared__ float4 sBC[kMaxDstate / 2];
  __shared__ float sh[4];
  // y of the slab is staged here and written back as whole lines (the integer
  // formats, whose kernels measure 2-3 % slower that way, store it directly).
  constexpr bool kStageY = !(F == kINT8 || F == kINT4);
  __shared__ float sY[kStageY ? NT * CPT : 1];
  __shared__ uint32_t sDone;  // waves whose rows of y are in sY
  const int nq = a.dstate >> 2;  // float4 per vector
  const float* Bg = a.B + (b * a.ngroups + g) * a.dstate;
  const float* Cg = a.C + (b * a.ngroups + g) * a.dstate;
  const bool bc_one = 2 * nq <= NT;  // one float4 of B or C per thread at most
  float4 bc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (bc_one && t < 2 * nq)
    bc = (t < nq) ? reinterpret_cast<const float4*>(Bg)[t] : reinterpret_cast<const float4*>(Cg)[t - nq];

  chunk_t<F> raw[CPT];
  float xv[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    raw[j] = load_stream<chunk_t<F>>(hstate + chunk_bytes_at<F>(l0 + j * pass));
    xv[j] = hx[r0 + j * rows_per_pass];
  }
  const float dt_in = a.dt[tile];
  const float Dv = a.D ? a.D[hh] : 0.0f;

  if (t < 64) {
    const float dte = step_size(a, dt_in, step_bias(a, hh));
    const float d = decay(dte, a.A[hh]);
    if (t == 0) { sh[0] = d; sh[2] = dte; sDone = 0; }
  }
  if (bc_one) {
    if (t < 2 * nq) sBC[t] = bc;
  } else {
    for (int i = t; i < 2 * nq; i += NT)
      sBC[i] = (i < nq) ? reinterpret_cast<const float4*>(Bg)[i]
                        : reinterpret_cast<const float4*>(Cg)[i - nq];
  }
  __syncthreads();
  const float dA = sh[0];
  const float dtv = sh[2];

  float h[CPT][V];
  bool bad[CPT];  // a NaN or infinity reached this chunk's partial of y
  float yo[CPT];  // rows' y, for kernels that store it directly
  // Scaled formats store fl32(v * s_old); dA * h_prev is evaluated as
  // fma(fl32(dA * s_old), v, w), one rounding of the scaled decay per group in
  // place of one rounding of v * s_old per entry (it saves a multiply per entry;
  // h_new moves by about an ulp at most). E4M3, and the four-chunk configurations (one
  // scale per head), read their scales before the loop (read inside it, each
  // load is issued after the previous chunk's y store and waited for at once);
  // the block-scaled INT kernels measure faster with one select-addressed load
  // per chunk.
  constexpr bool kScalesFirst = (F == kE4M3) || (is_int_fmt<F> && CPT >= 4);
  float dAs[CPT];
#pragma unroll
  for (int j = 0; j < CPT; ++j) dAs[j] = dA;
  if constexpr (kScalesFirst) {
    if (a.lanes_per_group == 0) {
      const float d = dA * a.scale[tile];
#pragma unroll
      for (int j = 0; j < CPT; ++j) dAs[j] = d;
    } else {
#pragma unroll
      for (int j = 0; j < CPT; ++j) dAs[j] = dA * a.scale[(e0 + j * pass) >> a.group_shift];
    }
  }
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    float dAj = dAs[j];
    if constexpr (is_int_fmt<F> && !kScalesFirst)
      dAj = dA * ((a.lanes_per_group == 0) ? a.scale[tile] : a.scale[(e0 + j * pass) >> a.group_shift]);
    float hp[V];
    decode_chunk<F>(raw[j], hp);
    const float dx = dtv * xv[j];
    // The lane's part of y: INT8 round-to-nearest, whose rounding is short enough
    // for the chain of dependent fmas to set the pace, sums in four interleaved
    // partial sums (4 % faster); elsewhere they measure no gain (the dithered
    // rules) or a loss (E4M3 and INT4 round-to-nearest, 1.5 and 3 %).
    constexpr int kYP = (F == kINT8 && R == kRTN) ? 4 : 1;
    float yp[kYP];
#pragma unroll
    for (int u = 0; u < kYP; ++u) yp[u] = 0.0f;
    // B and C come from LDS four at a time, so they are not held in registers
    // across passes.
#pragma unroll
    for (int i = 0; i < V / 4; ++i) {
      const float4 bq = sBC[(n0 >> 2) + i];
      const float4 cq = sBC[nq + (n0 >> 2) + i];
      const float bk[4] = {bq.x, bq.y, bq.z, bq.w};
      const float ck[4] = {cq.x, cq.y, cq.z, cq.w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 4 * i + u;
        const float w = dx * bk[u];
        h[j][k] = fmaf(dAj, hp[k], w);
        yp[u % kYP] = fmaf(ck[u], h[j][k], yp[u % kYP]);
      }
    }
    float ys = yp[0];
    if constexpr (kYP == 4) ys = (yp[0] + yp[1]) + (yp[2] + yp[3]);
    // (a finite overflow of a partial sum only sends the chunk down the exact path)
    bad[j] = !__builtin_isfinite(ys);
    ys = lane_sum(ys, lanes_per_row);
    if constexpr (kStageY) {
      if (cc == 0) sY[(t >> lr_shift) + j * rows_per_pass] = ys + Dv * xv[j];
    } else {
      yo[j] = ys + Dv * xv[j];
    }
  }
  if constexpr (!kStageY) {
    // Stored after the loop, so no chunk's scale load waits behind a y store.
    if (cc == 0) {
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        float yv = yo[j];
        if (a.z) yv = yv * silu(a.z[tile * a.headdim + r0 + j * rows_per_pass]);
        hy[r0 + j * rows_per_pass] = yv;
      }
    }
  }

  float r[CPT];  // scaled formats: 1 / s of each chunk's group
  bool clamp = true;  // E4M3 dithers: some value may exceed 448 after scaling
#pragma unroll
  for (int j = 0; j < CPT; ++j) r[j] = 1.0f;
  if constexpr (Traits<F>::scaled) {
    // Lane maxima of |h| ignore NaN and are >= 0, so the cross-lane maximum can
    // compare bit patterns as unsigned integers.
    uint32_t m[CPT];
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      float mj = 0.0f;
#pragma unroll
      for (int k = 0; k < V; ++k) mj = fmaxf(mj, __builtin_fabsf(h[j][k]));
      m[j] = __float_as_uint(mj);
    }
    if (a.lanes_per_group == 0) {  // one scale for the whole head, which is this workgroup
      __shared__ uint32_t red[NW];
      uint32_t mm = m[0];
#pragma unroll
      for (int j = 1; j < CPT; ++j) mm = max(mm, m[j]);
      mm = lane_umax(mm, 64);
      if ((t & 63) == 0) red[t >> 6] = mm;
      __syncthreads();
      if (t < 64) {  // the first wave turns the maximum into the scale and its reciprocal
        uint32_t w = red[0];
#pragma unroll
        for (int i = 1; i < NW; ++i) w = max(w, red[i]);
        const float s = group_scale<F>(__uint_as_float(w));
        const float rs = recip_scale(s);
        if (t == 0) {
          sh[0] = s;
          sh[1] = rs;
          sh[3] = (__uint_as_float(w) * rs <= 448.0f) ? 0.0f : 1.0f;  // E4M3: clamp needed
          a.scale[tile] = s;
        }
      }
      __syncthreads();
      const float rs = sh[1];
      // A per-head scale whose own rounding leaves max|h| r <= 448 (about four
      // heads in five) needs the E4M3 clamp nowhere in the head.
      clamp = __builtin_amdgcn_readfirstlane(__float_as_uint(sh[3])) != 0u;
#pragma unroll
      for (int j = 0; j < CPT; ++j) r[j] = rs;
    } else if (CPT % 2 == 0 && lanes_per_group >= 2) {
      // Lanes t and t ^ 1 share their group in every chunk, so each computes one
      // scale of a pair of chunks (even lanes chunk j, odd lanes chunk j + 1) and
      // takes the other reciprocal from its neighbour: half the divisions and
      // reciprocals (INT8 about 2 % faster).
      const bool odd = (t & 1) != 0;
      const int lg = t & (lanes_per_group - 1);
#pragma unroll
      for (int j = 0; j < CPT; j += 2) {
        const uint32_t m0 = lane_umax(m[j], lanes_per_group);
        const uint32_t m1 = lane_umax(m[j + 1], lanes_per_group);
        const float s = group_scale<F>(__uint_as_float(odd ? m1 : m0));
        const float rs = recip_scale(s);
        const float other = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, rs), kQuadXor1, 0xF, 0xF, true));
        r[j] = odd ? other : rs;
        r[j + 1] = odd ? rs : other;
        if (lg == 0) a.scale[(e0 + j * pass) >> a.group_shift] = s;
        if (lg == 1) a.scale[(e0 + (j + 1) * pass) >> a.group_shift] = s;
      }
    } else {  // groups of lanes_per_group consecutive lanes of one pass
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const float s = group_scale<F>(__uint_as_float(lane_umax(m[j], lanes_per_group)));
        r[j] = recip_scale(s);
        if ((t & (lanes_per_group - 1)) == 0) a.scale[(e0 + j * pass) >> a.group_shift] = s;
      }
    }
  }

  // See quantize_int_chunk for what the clamp costs and saves.
  constexpr bool kClamp = F == kINT4 || CPT == 1 || (CPT == 4 && NT <= 128);
  // Threshold bases of the chunks: one pass of NT chunks apart, a constant
  // step when the pass spans whole dither blocks. The direct form is kept
  // inside its branch by the empty asm: if-converted, its two 32-bit
  // multiplies would run for every chunk.
  uint32_t bases[CPT];
  bases[0] = thr_base<R>(a.entry_base + static_cast<uint64_t>(e0), a.thr);
  if (a.pass_thr_ok) {
#pragma unroll
    for (int j = 1; j < CPT; ++j) bases[j] = bases[0] + static_cast<uint32_t>(j) * a.pass_thr_inc;
  } else {
    uint64_t eb = a.entry_base + static_cast<uint64_t>(e0);
    asm volatile("" : "+v"(eb));
#pragma unroll
    for (int j = 1; j < CPT; ++j) bases[j] = thr_base<R>(eb + static_cast<uint64_t>(j) * pass, a.thr);
  }
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int64_t e = e0 + static_cast<int64_t>(j) * pass;
    const uint32_t base = bases[j];
    const chunk_t<F> out = quantize_any<F, R, kClamp>(
        h[j], r[j], chunk_thr<R, V>(a.entry_base + static_cast<uint64_t>(e), a.thr, base, a.toff),
        bad[j], clamp);
    store_stream(hstate + chunk_bytes_at<F>(l0 + j * pass), out);
  }

  // y leaves as whole lines rather than one float per row from every wave: each
  // wave counts itself in after its rows are in sY, and the last one to arrive
  // writes the slab's rows (the others exit; nothing waits).
  if constexpr (!kStageY) return;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  uint32_t arrived = 0;
  if ((t & 63) == 0) arrived = atomicAdd(&sDone, 1u);
  arrived = __shfl(arrived, 0);
  if (arrived == NW - 1) {
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    const int rows_slab = rows_per_pass * CPT;
    const int row0 = static_cast<int>(slab) * rows_slab;
    for (int i = t & 63; i < rows_slab; i += 64) {
      float yv = sY[i];
      if (a.z) yv = yv * silu(a.z[tile * a.headdim + row0 + i]);
      hy[row0 + i] = yv;
    }
  }
}

// ---------------------------------------------------------------------------
// Row kernel: any layout whose rows are LR = dstate / V chunks; one chunk per
// thread, chunk q = blockIdx * 256 + t.
// ---------------------------------------------------------------------------
// One wave's span of an fp32 state: lane L owns the V entries L V .. L V + V - 1 of
// the span, S = V / 4 units of 16 bytes. Unit u of the span moves between global
// memory and LDS by lane u mod 64, so an instruction covers 1 KiB without gaps. In
// LDS the units of a lane are rotated by an XOR with bits of the lane number, which
// spreads the owners' 16-byte accesses (32 or 64 bytes apart) over all banks.
template <int V>
struct FpSpan {
  static constexpr int S = V / 4;
  uint4* lds;       // the wave's 64 * S units
  uint8_t* state;
  int64_t first;    // the wave's first unit
  int64_t units;    // units of the state from that one on (<= 0: a wave past its end)
  int lane;
  __device__ FpSpan(uint4* block_lds, void* state, int64_t first_unit, int64_t end_unit, int t)
      : lds(block_lds + (t >> 6) * 64 * S), state(static_cast<uint8_t*>(state)), first(first_unit),
        units(end_unit - first_unit), lane(t & 63) {}
  __device__ FpSpan(uint4* block_lds, const UpdateArgs& a, int t)
      : FpSpan(block_lds, a.state, (static_cast<int64_t>(blockIdx.x) * 256 + (t & ~63)) * S,
               a.n_chunks * S, t) {}
  __device__ static int at(int owner, int k) {
    return owner * S + (k ^ ((owner >> (S == 4 ? 1 : 2)) & (S - 1)));
  }
  // LDS is written and read by lanes of one wave: the fences only keep the compiler
  // from moving one lane's reads above another's writes.
  __device__ static void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __device__ void fetch(uint4 (&u)[S]) const {
#pragma unroll
    for (int i = 0; i < S; ++i) {  // past the end (a ragged last block) the state's first unit is read
      const int n = i * 64 + lane;
      u[i] = load_stream<uint4>(state + (n < units ? (first + n) * 16 : 0));
    }
  }
  __device__ void load(float (&v)[V]) {
    uint4 u[S];
    fetch(u);
    distribute(u, v);
  }
  __device__ void distribute(const uint4 (&u)[S], float (&v)[V]) {
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int n = i * 64 + lane;
      lds[at(n / S, n % S)] = u[i];
    }
    wave_sync();
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const uint4 w = lds[at(lane, i)];
      v[4 * i] = __uint_as_float(w.x); v[4 * i + 1] = __uint_as_float(w.y);
      v[4 * i + 2] = __uint_as_float(w.z); v[4 * i + 3] = __uint_as_float(w.w);
    }
  }
  __device__ void store(const float (&v)[V]) {
#pragma unroll
    for (int i = 0; i < S; ++i)  // over the lane's own units, which it has read
      lds[at(lane, i)] = make_uint4(__float_as_uint(v[4 * i]), __float_as_uint(v[4 * i + 1]),
                                    __float_as_uint(v[4 * i + 2]), __float_as_uint(v[4 * i + 3]));
    wave_sync();
#pragma unroll
    for (int i = 0; i < S; ++i) {
      const int n = i * 64 + lane;
      if (n < units) store_stream(state + (first + n) * 16, lds[at(n / S, n % S)]);
    }
  }
};

// FP32_STATE: a checkpoint write on an fp32 state. The stored values are fp32
// (read as they are, no scale fold); each new value is rounded onto F's grid
// and written back as the fp32 value of its code (times the group scale for
// the scaled formats, whose scales are written only when a.scale is set).
// A lane still owns V consecutive entries, 32 or 64 bytes of fp32, but moves them
// through LDS: read directly, each 16-byte load of a wave would touch 2 or 4 KiB in
// pieces of 16 bytes, and the step is paced by those partial lines (INT8 blocks of
// 128, 67M entries, 545 MB: 210 us, 2.6 TB/s). Each wave copies its own span, whole
// lines per instruction, and only its own lanes read it, so no barrier is needed:
// 94 us, 5.8 TB/s, bound by HBM.
template <int F, int R, bool A_PER_STATE, bool FP32_STATE>
__global__ __launch_bounds__(256) void k_update_rows(UpdateArgs a) {
  constexpr int V = Traits<F>::V;
  const int t = threadIdx.x;
  __shared__ uint4 sState[FP32_STATE ? 256 * (V / 4) : 1];
  FpSpan<V> span(sState, a, t);
  const int cc = t & (a.lanes_per_row - 1);
  const int n0 = cc * V;
  const int64_t q = static_cast<int64_t>(blockIdx.x) * 256 + t;
  const bool live = q < a.n_chunks;  // whole rows (and groups) are live or dead together
  const int64_t e = (live ? q : 0) * V;
  const uint32_t row = static_cast<uint32_t>(e >> a.dstate_shift);  // rows < 2^32 (checked on host)
  const uint32_t bh = a.div_headdim.div(row);                        // b * nheads + h
  const uint32_t b = a.div_nheads.div(bh);
  const int hh = static_cast<int>(bh - b * static_cast<uint32_t>(a.nheads));
  const int g = static_cast<int>(a.div_hpg.div(static_cast<uint32_t>(hh)));
  uint8_t* const state = static_cast<uint8_t*>(a.state);
  float hp[V], h[V];
  if constexpr (FP32_STATE) {
    span.load(hp);
  } else {
    decode_chunk<F>(load_stream<chunk_t<F>>(state + chunk_bytes_at<F>(e)), hp);
  }
  const float xv = a.x[row];
  const float dtv = step_size(a, a.dt[bh], step_bias(a, hh));
  const float Dv = a.D ? a.D[hh] : 0.0f;
  float Bv[V], Cv[V], dA[V];
  load_floats<V>(a.B + (static_cast<int64_t>(b) * a.ngroups + g) * a.dstate + n0, Bv);
  load_floats<V>(a.C + (static_cast<int64_t>(b) * a.ngroups + g) * a.dstate + n0, Cv);
  if constexpr (A_PER_STATE) {
    float Av[V];
    load_floats<V>(a.A + static_cast<int64_t>(hh) * a.dstate + n0, Av);
    decays<V>(dtv, Av, dA);
  } else {
    const float d = decay(dtv, a.A[hh]);
#pragma unroll
    for (int k = 0; k < V; ++k) dA[k] = d;
  }
  if constexpr (Traits<F>::scaled && !FP32_STATE) {  // fold the old group scale into the decay (see k_update_slab)
    const float s_old = a.scale[e >> a.group_shift];
#pragma unroll
    for (int k = 0; k < V; ++k) dA[k] = dA[k] * s_old;
  }
  const float dx = dtv * xv;
  float ys = 0.0f;
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const float w = dx * Bv[k];
    h[k] = fmaf(dA[k], hp[k], w);
    ys = fmaf(Cv[k], h[k], ys);
  }
  const bool bad = !__builtin_isfinite(ys);
  ys = lane_sum(ys, a.lanes_per_row);
  if (live && cc == 0) a.y[row] = a.z ? (ys + Dv * xv) * silu(a.z[row]) : ys + Dv * xv;
  float rs = 1.0f, s = 1.0f;
  if constexpr (Traits<F>::scaled) {
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < V; ++k) m = fmaxf(m, __builtin_fabsf(h[k]));
    s = group_scale<F>(__uint_as_float(lane_umax(__float_as_uint(m), a.lanes_per_group)));
    rs = recip_scale(s);
    if (live && a.scale && (t & (a.lanes_per_group - 1)) == 0) a.scale[e >> a.group_shift] = s;
  }
  const uint64_t ge = a.entry_base + static_cast<uint64_t>(e);
  const chunk_t<F> out = quantize_any<F, R, F == kINT4 || !A_PER_STATE>(
      h, rs, chunk_thr<R, V>(ge, a.thr, thr_base<R>(ge, a.thr), a.toff), bad);
  if constexpr (FP32_STATE) {
    float v[V];
    decode_chunk<F>(out, v);
#pragma unroll
    for (int k = 0; k < V; ++k)
      if constexpr (Traits<F>::scaled) v[k] = v[k] * s;
    span.store(v);
  } else {
    if (live) store_stream(state + chunk_bytes_at<F>(e), out);
  }
}

// ---------------------------------------------------------------------------
// Mamba-1 layers: heads of one row of 16 entries (headdim 1, dstate 16), A per
// (channel, n), B and C shared by all channels of a sequence.
// ---------------------------------------------------------------------------
// A workgroup takes a tile of channels (256 chunks, one per lane) through
// batch_per_wg sequences or one more. Vector issue bounds the step (15 of the 21.4 us below,
// beside the set-up, which all workgroups run at once): of 32 instructions per INT8 entry
// about 15 are its own exp(dt A), so that takes the short table form. A and D
// stay in registers, B and C of the workgroup's sequences are staged in LDS, and the
// next sequence's state and x load while the current one is computed (one chunk per
// lane and launch reads A anew for every sequence, 4 bytes per entry against 2 of INT8
// state, and waits for three rounds of loads one after another). 5120 channels, batch
// 225, INT8 blocks of 16, Weyl, from a graph: row kernel 22.5 us, this one 21.4.
// Four waves per SIMD: at the 128 registers of that bound only INT8 hash SR spills (two; four
// without its clamp).
template <int F, int R>
__global__ __launch_bounds__(256, 4) void k_update_channels(UpdateArgs a) {
  constexpr int V = Traits<F>::V;
  const int t = threadIdx.x;
  constexpr int N = kChannelN, LR = N / V;  // lanes per row: 1 or 2; a scaled row is one group
  const int cc = t & (LR - 1);
  const int n0 = cc * V;
  const int tile = static_cast<int>(blockIdx.x) * (256 / LR) + t / LR;
  const bool live = tile < a.nheads;  // whole rows (and groups) are live or dead together
  const int ch = live ? tile : 0;
  const int part = static_cast<int>(blockIdx.y);  // the first batch_rem parts take one more
  const int64_t b0 = static_cast<int64_t>(part) * a.batch_per_wg + min(part, a.batch_rem);
  const int nb = a.batch_per_wg + (part < a.batch_rem ? 1 : 0);

  __shared__ float4 sBC[kChannelBatch * 2 * N / 4];  // per sequence: B, then C
  __shared__ double sExp[kExpTable];
  stage_exp_table(sExp, t, 256);
  constexpr int NQ = N / 4;
  static_assert(kChannelBatch * 2 * NQ <= 256, "one float4 of B or C per thread");
  const bool has_bc = t < nb * 2 * NQ;
  float4 bc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (has_bc) {  // before the state: its staging waits for it alone
    const int j = t & (2 * NQ - 1);
    const float* v = (j < NQ ? a.B : a.C) + (b0 + t / (2 * NQ)) * N;
    bc = reinterpret_cast<const float4*>(v)[j & (NQ - 1)];
  }

  struct Row {
    chunk_t<F> raw;
    float x, s, z;
  };
  uint8_t* const state = static_cast<uint8_t*>(a.state);
  const int64_t row0 = b0 * a.nheads + ch;
  auto fetch = [&](int i) {
    const int64_t row = row0 + static_cast<int64_t>(i) * a.nheads;
    const int64_t e = row * N + n0;
    Row r;
    r.raw = load_stream<chunk_t<F>>(state + chunk_bytes_at<F>(e));
    r.x = a.x[row];
    r.s = 1.0f;
    if constexpr (Traits<F>::scaled) r.s = a.scale[row];
    r.z = a.z ? a.z[row] : 0.0f;
    return r;
  };
  Row next = fetch(0);
  float Av[V];
  load_floats<V>(a.A + static_cast<int64_t>(ch) * N + n0, Av);
  const float Dv = a.D ? a.D[ch] : 0.0f;
  if (has_bc) sBC[t] = bc;
  // The lane's own step sizes, ahead of the loop: inside it, the softplus's double
  // constants would stay in some thirty registers.
  __shared__ float sDt[kChannelBatch][256];
  {
    const float bias = step_bias(a, ch);
#pragma unroll 1
    for (int i = 0; i < nb; ++i)
      sDt[i][t] = step_size(a, a.dt[row0 + static_cast<int64_t>(i) * a.nheads], bias);
  }
  __syncthreads();

#pragma unroll 1
  for (int i = 0; i < nb; ++i) {
    const Row cur = next;
    if (i + 1 < nb) next = fetch(i + 1);
    const int64_t row = row0 + static_cast<int64_t>(i) * a.nheads;
    const int64_t e = row * N + n0;
    const float dtv = sDt[i][t];
    float hp[V], h[V];
    decode_chunk<F>(cur.raw, hp);
    const float dx = dtv * cur.x;
    const float4* const Bq = sBC + i * 2 * NQ + n0 / 4;
    float ys = 0.0f;
#pragma unroll
    for (int j = 0; j < V / 4; ++j) {
      float z[4], dA[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) z[u] = dtv * Av[4 * j + u];
      exp_values_table<4>(sExp, z, dA);
      const float4 bq = Bq[j], cq = Bq[NQ + j];
      const float bk[4] = {bq.x, bq.y, bq.z, bq.w};
      const float ck[4] = {cq.x, cq.y, cq.z, cq.w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int k = 4 * j + u;
        if constexpr (Traits<F>::scaled) dA[u] = dA[u] * cur.s;  // the old scale folded into the decay
        h[k] = fmaf(dA[u], hp[k], dx * bk[u]);
        ys = fmaf(ck[u], h[k], ys);
      }
      // Four exponentials in flight: with all of a lane's the registers allow three
      // waves per SIMD instead of five.
      __builtin_amdgcn_sched_barrier(0);
    }
    const bool bad = !__builtin_isfinite(ys);
    ys = lane_sum(ys, LR);
    if (live && cc == 0) a.y[row] = a.z ? (ys + Dv * cur.x) * silu(cur.z) : ys + Dv * cur.x;
    float rs = 1.0f;
    if constexpr (Traits<F>::scaled) {
      float m = 0.0f;
#pragma unroll
      for (int k = 0; k < V; ++k) m = fmaxf(m, __builtin_fabsf(h[k]));
      const float s = group_scale<F>(m);
      rs = recip_scale(s);
      if (live) a.scale[row] = s;
    }
    const uint64_t ge = a.entry_base + static_cast<uint64_t>(e);
    const chunk_t<F> out =
        quantize_any<F, R, F == kINT4 || R == kSR>(h, rs, chunk_thr<R, V>(ge, a.thr, thr_base<R>(ge, a.thr), a.toff), bad);
    if (live) store_stream(state + chunk_bytes_at<F>(e), out);
  }
}

// ---------------------------------------------------------------------------
// Requantize without scale: one chunk of V entries per thread; the entries
// after the last whole chunk one by one.
// ---------------------------------------------------------------------------
template <int F>
__device__ inline void store_code(void* codes, int64_t k, uint32_t c) {
  constexpr int bytes = Traits<F>::CB / Traits<F>::V;
  if constexpr (bytes == 2) static_cast<uint16_t*>(codes)[k] = static_cast<uint16_t>(c);
  else if constexpr (bytes == 4) static_cast<uint32_t*>(codes)[k] = c;
  else static_cast<uint8_t*>(codes)[k] = static_cast<uint8_t>(c);
}

// STREAM (see kRequantStream; 16-bit formats): the fp32 entries come past the caches, through
// LDS in whole lines (see FpSpan). bf16 Weyl, from a graph, without / with it: 63M entries of
// one buffer 64.0 / 56.1 us, of three in turn 64.6 / 62.2; 15M of one 14.4 / 16.6.
template <int F, int R, bool STREAM>
__global__ __launch_bounds__(256) void k_requant(RequantArgs a) {
  constexpr int V = Traits<F>::V;
  const int64_t q = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t e = q * V;
  float h[V];
  if constexpr (STREAM) {
    // Units up to the last whole one: a lane with a whole chunk has all of its own.
    __shared__ uint4 sSpan[256 * (V / 4)];
    FpSpan<V> span(sSpan, const_cast<float*>(a.h), (q & ~int64_t{63}) * (V / 4), a.n / 4, threadIdx.x);
    span.load(h);
  }
  if (e >= a.n) return;
  const uint64_t ge = a.entry_base + static_cast<uint64_t>(e);
  if (e + V <= a.n) {
    if constexpr (!STREAM) load_floats<V>(a.h + e, h);
    const uint4 out = quantize_chunk<F, R>(h, chunk_thr<R, V>(ge, a.thr, thr_base<R>(ge, a.thr), a.toff),
                                           chunk_has_nan<V>(h));
    *reinterpret_cast<chunk_t<F>*>(static_cast<uint8_t*>(a.codes) + chunk_bytes_at<F>(e)) = out;
  } else {
    for (int64_t k = e; k < a.n; ++k) {
      const uint64_t gk = a.entry_base + static_cast<uint64_t>(k);
      store_code<F>(a.codes, k, round_code<F, R>(a.h[k], entry_thr<R>(gk, a.thr)));
    }
  }
}

// ---------------------------------------------------------------------------
// Requantize to a scaled format (E4M3, INT8, INT4) with group scales.
// ---------------------------------------------------------------------------
// Groups that fit neither a wave's chunks nor a workgroup's (48, 1536, 65536 entries): one
// wave per group loops over its 16-entry chunks twice, for the maximum and for the rounding.
template <int F, int R>
__global__ __launch_bounds__(256) void k_requant_scaled(RequantArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t chunks_per_group = a.group / 16;
  const int64_t n_groups = a.n / a.group;
  const int64_t wave = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int64_t nwaves = static_cast<int64_t>(gridDim.x) * 4;
  for (int64_t grp = wave; grp < n_groups; grp += nwaves) {
    float m = 0.0f;
    for (int64_t c = lane; c < chunks_per_group; c += 64) {
      float h[16];
      load_floats<16>(a.h + grp * a.group + c * 16, h);
#pragma unroll
      for (int k = 0; k < 16; ++k) m = fmaxf(m, __builtin_fabsf(h[k]));
    }
    const float s = group_scale<F>(__uint_as_float(lane_umax(__float_as_uint(m), 64)));
    const float rs = recip_scale(s);
    if (lane == 0) a.scale[grp] = s;
    for (int64_t c0 = 0; c0 < chunks_per_group; c0 += 64) {  // uniform trip count
      const bool live = c0 + lane < chunks_per_group;
      const int64_t e = grp * a.group + (live ? c0 + lane : 0) * 16;
      float h[16];
      load_floats<16>(a.h + e, h);
      const uint64_t ge = a.entry_base + static_cast<uint64_t>(e);
      const chunk_t<F> out = quantize_any<F, R>(h, rs, chunk_thr<R, 16>(ge, a.thr, thr_base<R>(ge, a.thr), a.toff),
                                                chunk_has_nan<16>(h));
      if (live) *reinterpret_cast<chunk_t<F>*>(static_cast<uint8_t*>(a.codes) + chunk_bytes_at<F>(e)) = out;
    }
  }
}

// Groups of up to 64 chunks (a power of two): one chunk per lane, held in registers
// between the maximum and the rounding, so the fp32 input is read once. Against two reads,
// E4M3 hash SR, blocks of 128, from a graph: 31M entries of one buffer 30.3 -> 24.2 us, 63M of
// three in turn (STREAM, see kRequantStream) 64.7 -> 50.3.
template <int F, int R, bool STREAM>
__global__ __launch_bounds__(256) void k_requant_chunks(RequantArgs a) {
  const int t = threadIdx.x;
  const int64_t q = static_cast<int64_t>(blockIdx.x) * 256 + t;
  const bool live = q * 16 < a.n;  // whole groups are live or dead together
  const int64_t e = live ? q * 16 : 0;
  float h[16];
  if constexpr (STREAM) {
    __shared__ uint4 sSpan[256 * 4];
    FpSpan<16> span(sSpan, const_cast<float*>(a.h), (q & ~int64_t{63}) * 4, a.n / 4, t);
    span.load(h);
  } else {
    load_floats<16>(a.h + e, h);
  }
  float m = 0.0f;
#pragma unroll
  for (int k = 0; k < 16; ++k) m = fmaxf(m, __builtin_fabsf(h[k]));
  const float s = group_scale<F>(__uint_as_float(lane_umax(__float_as_uint(m), a.lanes_per_group)));
  const float rs = recip_scale(s);
  if (live && (t & (a.lanes_per_group - 1)) == 0) a.scale[q >> a.lpg_shift] = s;
  const uint64_t ge = a.entry_base + static_cast<uint64_t>(e);
  const chunk_t<F> out = quantize_any<F, R>(
      h, rs, chunk_thr<R, 16>(ge, a.thr, thr_base<R>(ge, a.thr), a.toff), chunk_has_nan<16>(h));
  if (live) *reinterpret_cast<chunk_t<F>*>(static_cast<uint8_t*>(a.codes) + chunk_bytes_at<F>(e)) = out;
}

// Groups of NT * 16 * CPT entries (e.g. one scale per 64x128 head): one workgroup per
// group, its values held in registers between the maximum and the rounding. With STREAM
// (see kRequantStream) each load of a wave covers 1 KiB without gaps and reaches its lane
// through LDS: bound by HBM, 63M entries of E4M3 (315 MB) in heads of 8192, three buffers in
// turn, 55.8 -> 50.7 us. Heads of 16384, which one wave each read twice, 99.2 -> 51.6 us.
template <int F, int R, int NT, int CPT, bool STREAM>
__global__ __launch_bounds__(NT) void k_requant_group_wg(RequantArgs a) {
  const int t = threadIdx.x;
  const int64_t c0 = static_cast<int64_t>(blockIdx.x) * (NT * CPT);  // the group's first chunk
  const int64_t e0 = c0 * 16;
  float h[CPT][16];
  if constexpr (STREAM) {
    __shared__ uint4 sSpan[NT * 4];
    FpSpan<16> span(sSpan, const_cast<float*>(a.h), (c0 + (t & ~63)) * 4, a.n / 4, t);
    uint4 u[CPT][4];
#pragma unroll
    for (int j = 0; j < CPT; ++j, span.first += NT * 4, span.units -= NT * 4) span.fetch(u[j]);
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      span.distribute(u[j], h[j]);
      if (j + 1 < CPT) span.wave_sync();  // its units have been read before the next ones replace them
    }
  } else {
#pragma unroll
    for (int j = 0; j < CPT; ++j) load_floats<16>(a.h + e0 + (static_cast<int64_t>(j) * NT + t) * 16, h[j]);
  }
  float m = 0.0f;
#pragma unroll
  for (int j = 0; j < CPT; ++j)
#pragma unroll
    for (int k = 0; k < 16; ++k) m = fmaxf(m, __builtin_fabsf(h[j][k]));
  constexpr int NW = NT / 64;
  __shared__ uint32_t red[NW];
  const uint32_t mw = lane_umax(__float_as_uint(m), 64);
  if ((t & 63) == 0) red[t >> 6] = mw;
  __syncthreads();
  uint32_t w = red[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) w = max(w, red[i]);
  const float s = group_scale<F>(__uint_as_float(w));
  const float rs = recip_scale(s);
  if (t == 0) a.scale[blockIdx.x] = s;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    const int64_t e = e0 + (static_cast<int64_t>(j) * NT + t) * 16;
    const uint64_t ge = a.entry_base + static_cast<uint64_t>(e);
    const chunk_t<F> out = quantize_any<F, R>(
        h[j], rs, chunk_thr<R, 16>(ge, a.thr, thr_base<R>(ge, a.thr), a.toff), chunk_has_nan<16>(h[j]));
    *reinterpret_cast<chunk_t<F>*>(static_cast<uint8_t*>(a.codes) + chunk_bytes_at<F>(e)) = out;
  }
}

template <int R>
__global__ __launch_bounds__(256) void k_dither_fill(DitherArgs a) {
  const int64_t q = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t e = q * 4;
  if (e >= a.n) return;
  const uint64_t ge = a.entry_base + static_cast<uint64_t>(e);
  if (a.n - e >= 4 && (reinterpret_cast<uintptr_t>(a.out) & 15u) == 0) {
    // Four whole words to a 16-byte aligned address: one 16-byte store, and one
    // Philox block when the four entries are the words of one block.
    uint32_t w[4];
    if constexpr (R == kPHILOX) {
      if ((ge & 3u) == 0) {
        const uint64_t blk = ge >> 2;
        philox4x32_10(static_cast<uint32_t>(blk), static_cast<uint32_t>(blk >> 32), a.thr.step, 0u,
                      a.thr.seed, a.thr.layer, w);
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] >>= 8;
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = entry_thr<R>(ge + k, a.thr) >> 8;
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = (R == kRTN) ? (1u << 23) : (entry_thr<R>(ge + k, a.thr) >> 8);
    }
    store_stream(a.out + e, make_uint4(w[0], w[1], w[2], w[3]));
    return;
  }
  const int64_t lim = (a.n - e < 4) ? (a.n - e) : 4;
  for (int64_t k = 0; k < lim; ++k)
    a.out[e + k] = (R == kRTN) ? (1u << 23) : (entry_thr<R>(ge + static_cast<uint64_t>(k), a.thr) >> 8);
}

// ---------------------------------------------------------------------------
// Open-loop replay. Thread q owns entries E q .. E q + E - 1 for all steps: the fp32
// reference h and the stored value hq stay in registers, so the only traffic is
// the trace (a and w, 8 bytes per entry and step, nontemporal, the rows of the next
// AHEAD steps loaded while the current one is rounded) and the error sums per block.
// Each step rounds fma(a, hq, w) with the exact software rounding of the
// format (the per-entry functions of the fused kernels' exact path); the
// scaled formats first reduce max|x| over the group's lanes. Lanes past n
// (the grid's ragged end) run on the first entries and store nothing, so the group
// reductions always see whole groups.
//
// Four entries per thread and one step ahead stream a long state at the rate of HBM (1.3M
// entries, 256 steps: 485 us, 5.7 TB/s; two or four steps ahead, with more rows open at
// once, 505 and 530 us). A state below kReplayShort entries then has less than two waves
// per SIMD, and the steps' own chain of dependent operations and loads sets the pace:
// two entries per thread, four steps ahead, in workgroups of one wave give it twice the
// waves on more CUs. INT8, 12k entries 145 -> 99 us; fp16, 147k 139 -> 88 us; INT8, 328k
// (300 steps) 214 -> 169 us; bf16, 655k 300 -> 295 us, but INT8, 983k 372 -> 408 us.
// ---------------------------------------------------------------------------
constexpr int64_t kReplayShort = 1 << 19;

// Two or four 32-bit words in one access.
template <int E>
__device__ inline void load_words(const float* p, float (&v)[E]) {
  typedef unsigned int words __attribute__((ext_vector_type(E)));
  const words w = __builtin_nontemporal_load(reinterpret_cast<const words*>(p));
#pragma unroll
  for (int k = 0; k < E; ++k) v[k] = __uint_as_float(w[k]);
}
template <int W>
__device__ inline void store_words(uint32_t* p, const uint32_t (&v)[W]) {
  typedef unsigned int words __attribute__((ext_vector_type(W)));
  words w;
#pragma unroll
  for (int k = 0; k < W; ++k) w[k] = v[k];
  *reinterpret_cast<words*>(p) = w;
}

template <int F, int R, int E>
__device__ inline void replay_round(const ReplayArgs& a, uint64_t e0, uint32_t step,
                                    const float (&x)[E], float (&hq)[E], uint32_t (&code)[E],
                                    float& scale) {
  Thr th = a.thr;
  th.step = step;
  if constexpr (R == kWEYL) th.key = a.weyl_key0 + kWeylPhi * (step - a.step0);
  else if constexpr (R == kSR) th.key = sr_step_key(a.sr_key0, step);
  uint32_t thr[E];
  if constexpr (R == kPHILOX) {
    const ChunkThr<R, 4> t4 = chunk_thr<R, 4>(e0, th, 0u, nullptr);
    const bool upper = E == 2 && (e0 & 2u) != 0;  // entries 2 and 3 of the block of four
#pragma unroll
    for (int k = 0; k < E; ++k) thr[k] = upper ? t4(k + 4 - E) : t4(k);
  } else {
#pragma unroll
    for (int k = 0; k < E; ++k) thr[k] = entry_thr<R>(e0 + k, th);
  }
  if constexpr (Traits<F>::scaled) {
    float m = 0.0f;
#pragma unroll
    for (int k = 0; k < E; ++k) m = fmaxf(m, __builtin_fabsf(x[k]));
    const float s = group_scale<F>(__uint_as_float(lane_umax(__float_as_uint(m), a.lanes_per_group)));
    const float r = recip_scale(s);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      code[k] = round_code<F, R>(x[k] * r, thr[k]);
      hq[k] = code_value<F>(code[k]) * s;
    }
    scale = s;
  } else {
#pragma unroll
    for (int k = 0; k < E; ++k) {
      code[k] = round_code<F, R>(x[k], thr[k]);
      hq[k] = code_value<F>(code[k]);
    }
  }
}

template <int F, int R, int E, int AHEAD>
__global__ __launch_bounds__(256) void k_replay(ReplayArgs a) {
  const int64_t q = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const bool live = q * E < a.n;
  const int64_t i0 = live ? q * E : 0;
  const uint64_t e0 = a.entry_base + static_cast<uint64_t>(i0);
  float h[E];
  load_words(a.h0 + i0, h);
  float hq[E];
  uint32_t code[E];
  float scale = 0.0f;
  replay_round<F, R, E>(a, e0, a.step0, h, hq, code, scale);

  double err[E] = {}, ref[E] = {};
  float an[AHEAD][E] = {}, wn[AHEAD][E] = {};
  const uint32_t steps = static_cast<uint32_t>(a.steps);
  auto fetch = [&](uint32_t t, int u) {
    const int64_t off = static_cast<int64_t>(t) * a.n + i0;
    load_words(a.a + off, an[u]);
    load_words(a.w + off, wn[u]);
  };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u)
    if (static_cast<uint32_t>(u) < steps) fetch(u, u);
  int32_t left = a.block_steps;  // steps until the block's sums are stored
  int64_t out = i0;
  auto step = [&](uint32_t t, int u) {  // step t + 1, whose row is in slot u
    float at[E], wt[E];
#pragma unroll
    for (int k = 0; k < E; ++k) { at[k] = an[u][k]; wt[k] = wn[u][k]; }
    if (t + AHEAD < steps) fetch(t + AHEAD, u);  // in flight while this step rounds
    float x[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
      h[k] = fmaf(at[k], h[k], wt[k]);
      x[k] = fmaf(at[k], hq[k], wt[k]);
    }
    replay_round<F, R, E>(a, e0, a.step0 + t + 1u, x, hq, code, scale);
#pragma unroll
    for (int k = 0; k < E; ++k) {
      const double d = static_cast<double>(hq[k]) - static_cast<double>(h[k]);
      err[k] += d * d;
      ref[k] += static_cast<double>(h[k]) * static_cast<double>(h[k]);
    }
    if (--left == 0 || t + 1 == steps) {
      if (live) {
#pragma unroll
        for (int k = 0; k < E; k += 2) {
          *reinterpret_cast<double2*>(a.err + out + k) = make_double2(err[k], err[k + 1]);
          if (a.ref) *reinterpret_cast<double2*>(a.ref + out + k) = make_double2(ref[k], ref[k + 1]);
        }
      }
      out += a.n;
      left = a.block_steps;
#pragma unroll
      for (int k = 0; k < E; ++k) { err[k] = 0.0; ref[k] = 0.0; }
    }
  };
#pragma unroll 1
  for (uint32_t t = 0; t < steps; t += AHEAD) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u)
      if (t + u < steps) step(t + u, u);
  }
  if (!live) return;
  if (a.codes) {
    constexpr int bits = Traits<F>::CB * 8 / Traits<F>::V;  // code width
    if constexpr (bits * E >= 32) {
      uint32_t w[bits * E / 32] = {};
#pragma unroll
      for (int k = 0; k < E; ++k) w[k * bits / 32] |= code[k] << (k * bits % 32);
      store_words(static_cast<uint32_t*>(a.codes) + i0 / E * (bits * E / 32), w);
    } else {
      uint32_t w = 0;
#pragma unroll
      for (int k = 0; k < E; ++k) w |= code[k] << (k * bits);
      if constexpr (bits * E == 16) static_cast<uint16_t*>(a.codes)[i0 / E] = static_cast<uint16_t>(w);
      else static_cast<uint8_t*>(a.codes)[i0 / E] = static_cast<uint8_t>(w);
    }
  }
  if constexpr (Traits<F>::scaled) {
    if (a.scale && (threadIdx.x & (a.lanes_per_group - 1)) == 0)
      a.scale[static_cast<int64_t>(e0 - a.entry_base) >> a.group_shift] = scale;
  }
  if (a.h_final) {
    uint32_t w[E];
#pragma unroll
    for (int k = 0; k < E; ++k) w[k] = __float_as_uint(h[k]);
    store_words(reinterpret_cast<uint32_t*>(a.h_final) + i0, w);
  }
}

// ---------------------------------------------------------------------------
// Causal depthwise conv1d decode update: thread i = b * channels + c shifts its
// channel's window by one, appends x[i] and writes
// out[i] = (silu)(bias[c] + sum_k window[k] * weight[c][k]).
// ---------------------------------------------------------------------------
// With four taps and 16-byte aligned buffers (Mamba's width) the window and the weights
// are one 16-byte access each, so a wave moves whole lines; word by word each of its
// eight accesses touches 1 KiB to use a quarter of it. 64 x 10240 channels (26 MB):
// 10.4 -> 6.0 us.
__global__ __launch_bounds__(256) void k_conv1d_update4(ConvArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= a.n) return;
  const uint32_t c = static_cast<uint32_t>(i) - a.div_channels.div(static_cast<uint32_t>(i)) * a.channels;
  const uint4 raw = load_stream<uint4>(a.state + i * 4);
  const float4 w = reinterpret_cast<const float4*>(a.weight)[c];
  const float x = a.x[i];
  float acc = a.bias ? a.bias[c] : 0.0f;
  acc = fmaf(__uint_as_float(raw.y), w.x, acc);
  acc = fmaf(__uint_as_float(raw.z), w.y, acc);
  acc = fmaf(__uint_as_float(raw.w), w.z, acc);
  acc = fmaf(x, w.w, acc);
  store_stream(a.state + i * 4, make_uint4(raw.y, raw.z, raw.w, __float_as_uint(x)));
  a.out[i] = a.act ? silu(acc) : acc;
}

__global__ __launch_bounds__(256) void k_conv1d_update(ConvArgs a) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= a.n) return;
  const uint32_t c = static_cast<uint32_t>(i) - a.div_channels.div(static_cast<uint32_t>(i)) * a.channels;
  float* const st = a.state + i * a.width;
  const float* const w = a.weight + static_cast<int64_t>(c) * a.width;
  float acc = a.bias ? a.bias[c] : 0.0f;
  for (int k = 0; k < a.width; ++k) {
    const float v = (k + 1 < a.width) ? st[k + 1] : a.x[i];
    st[k] = v;
    acc = fmaf(v, w[k], acc);
  }
  a.out[i] = a.act ? silu(acc) : acc;
}

// ---------------------------------------------------------------------------
// Launchers.
// ---------------------------------------------------------------------------
template <int F, int R, int NT, int CPT, int LR = 0, int LG = LR>
static hipError_t launch_slab(const UpdateArgs& a, hipStream_t s) {
  const int64_t blocks = a.batch * a.nheads * a.slabs_per_head;
  hipLaunchKernelGGL((k_update_slab<F, R, NT, CPT, LR, LG>), dim3(static_cast<unsigned>(blocks)),
                     dim3(NT), 0, s, a);
  return hipGetLastError();
}

// The instances for rows of a.const_lanes lanes, of the configurations that have them.
template <int F, int R, int NT, int CPT>
static hipError_t launch_slab_lanes(const UpdateArgs& a, hipStream_t s) {
  if constexpr (F == kE4M3 || (is_int_fmt<F> && CPT == 2)) {  // the block configurations
    if (a.lanes_per_group == 1) {
      if (a.const_lanes == 4) return launch_slab<F, R, NT, CPT, 4, 1>(a, s);
      if (a.const_lanes == 8) return launch_slab<F, R, NT, CPT, 8, 1>(a, s);
      if (a.const_lanes == 16) return launch_slab<F, R, NT, CPT, 16, 1>(a, s);
      return launch_slab<F, R, NT, CPT>(a, s);
    }
  }
  if constexpr (Traits<F>::scaled) {
    if (a.const_lanes == 4) return launch_slab<F, R, NT, CPT, 4>(a, s);
    if (a.const_lanes == 8) return launch_slab<F, R, NT, CPT, 8>(a, s);
    if (a.const_lanes == 16) return launch_slab<F, R, NT, CPT, 16>(a, s);
  } else {
    if (a.const_lanes != 0) return launch_slab<F, R, NT, CPT, 128 / Traits<F>::V>(a, s);
  }
  return launch_slab<F, R, NT, CPT>(a, s);
}

template <int F, int R>
static hipError_t launch_slab_cfg(const UpdateArgs& a, int cfg, hipStream_t s) {
  if (cfg == kSlab256x1) return launch_slab<F, R, 256, 1>(a, s);
  if constexpr (!Traits<F>::scaled) {
    if (cfg == kSlab256x2) return launch_slab<F, R, 256, 2>(a, s);
    if (cfg == kSlab512x2) return launch_slab_lanes<F, R, 512, 2>(a, s);
  } else {
    if constexpr (F != kE4M3) {
      if (cfg == kSlab256x2) return launch_slab_lanes<F, R, 256, 2>(a, s);
    }
    switch (cfg) {  // four chunks per thread: one scale per head, and E4M3 blocks
      case kSlab64x4: return launch_slab<F, R, 64, 4>(a, s);
      case kSlab128x4: return launch_slab_lanes<F, R, 128, 4>(a, s);
      case kSlab256x4: return launch_slab<F, R, 256, 4>(a, s);
      case kSlab512x4: return launch_slab<F, R, 512, 4>(a, s);
      case kSlab1024x4: return launch_slab<F, R, 1024, 4>(a, s);
      case kSlab1024x8: return launch_slab<F, R, 1024, 8>(a, s);
      default: break;
    }
  }
  return hipErrorInvalidValue;
}

template <int F, int R>
static hipError_t launch_rows(const UpdateArgs& a, bool a_per_state, hipStream_t s) {
  const unsigned grid = static_cast<unsigned>((a.n_chunks + 255) / 256);
  if (a.fp32_state) {
    if constexpr (F != kFP32) {
      if (a_per_state)
        hipLaunchKernelGGL((k_update_rows<F, R, true, true>), dim3(grid), dim3(256), 0, s, a);
      else
        hipLaunchKernelGGL((k_update_rows<F, R, false, true>), dim3(grid), dim3(256), 0, s, a);
    } else {
      return hipErrorInvalidValue;
    }
  } else if (a_per_state) {
    hipLaunchKernelGGL((k_update_rows<F, R, true, false>), dim3(grid), dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((k_update_rows<F, R, false, false>), dim3(grid), dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

template <int F, int R>
static hipError_t launch_channels(const UpdateArgs& a, hipStream_t s) {
  const unsigned tiles = static_cast<unsigned>((static_cast<int64_t>(a.nheads) * kChannelN / Traits<F>::V + 255) / 256);
  const unsigned parts = static_cast<unsigned>((a.batch - a.batch_rem) / a.batch_per_wg);
  hipLaunchKernelGGL((k_update_channels<F, R>), dim3(tiles, parts), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int F, int R>
static hipError_t launch_update_fr(const UpdateArgs& a, int cfg, bool aps, hipStream_t s) {
  if constexpr (F != kFP32) {
    if (cfg == kChannelKernel) return launch_channels<F, R>(a, s);
  }
  return cfg == kRowKernel ? launch_rows<F, R>(a, aps, s) : launch_slab_cfg<F, R>(a, cfg, s);
}

template <int F>
static hipError_t launch_update_f(const UpdateArgs& a, int rule, int cfg, bool aps, hipStream_t s) {
  switch (rule) {
    case kRTN: return launch_update_fr<F, kRTN>(a, cfg, aps, s);
    case kSR: return launch_update_fr<F, kSR>(a, cfg, aps, s);
    case kPHILOX: return launch_update_fr<F, kPHILOX>(a, cfg, aps, s);
    default: return launch_update_fr<F, kWEYL>(a, cfg, aps, s);
  }
}

hipError_t launch_update(const UpdateArgs& a, int format, int rule, int cfg, bool a_per_state,
                         hipStream_t s) {
  switch (format) {
    case kFP16: return launch_update_f<kFP16>(a, rule, cfg, a_per_state, s);
    case kBF16: return launch_update_f<kBF16>(a, rule, cfg, a_per_state, s);
    case kE4M3: return launch_update_f<kE4M3>(a, rule, cfg, a_per_state, s);
    case kINT8: return launch_update_f<kINT8>(a, rule, cfg, a_per_state, s);
    case kINT4: return launch_update_f<kINT4>(a, rule, cfg, a_per_state, s);
    default: return launch_update_f<kFP32>(a, rule, cfg, a_per_state, s);
  }
}

template <int F, bool STREAM>
static hipError_t launch_requant_f(const RequantArgs& a, int rule, hipStream_t s) {
  constexpr int V = Traits<F>::V;
  const int64_t chunks = (a.n + V - 1) / V;
  const unsigned grid = static_cast<unsigned>((chunks + 255) / 256);
  switch (rule) {
    case kRTN: hipLaunchKernelGGL((k_requant<F, kRTN, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
    case kSR: hipLaunchKernelGGL((k_requant<F, kSR, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
    case kPHILOX: hipLaunchKernelGGL((k_requant<F, kPHILOX, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_requant<F, kWEYL, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

template <int F, int NT, int CPT, bool STREAM>
static hipError_t launch_requant_group_wg(const RequantArgs& a, int rule, hipStream_t s) {
  const dim3 grid(static_cast<unsigned>(a.n / a.group));
  switch (rule) {
    case kRTN: hipLaunchKernelGGL((k_requant_group_wg<F, kRTN, NT, CPT, STREAM>), grid, dim3(NT), 0, s, a); break;
    case kSR: hipLaunchKernelGGL((k_requant_group_wg<F, kSR, NT, CPT, STREAM>), grid, dim3(NT), 0, s, a); break;
    case kPHILOX: hipLaunchKernelGGL((k_requant_group_wg<F, kPHILOX, NT, CPT, STREAM>), grid, dim3(NT), 0, s, a); break;
    default: hipLaunchKernelGGL((k_requant_group_wg<F, kWEYL, NT, CPT, STREAM>), grid, dim3(NT), 0, s, a); break;
  }
  return hipGetLastError();
}

template <int F, bool STREAM>
static hipError_t launch_requant_chunks(const RequantArgs& a, int rule, hipStream_t s) {
  const unsigned grid = static_cast<unsigned>((a.n / 16 + 255) / 256);
  switch (rule) {
    case kRTN: hipLaunchKernelGGL((k_requant_chunks<F, kRTN, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
    case kSR: hipLaunchKernelGGL((k_requant_chunks<F, kSR, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
    case kPHILOX: hipLaunchKernelGGL((k_requant_chunks<F, kPHILOX, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_requant_chunks<F, kWEYL, STREAM>), dim3(grid), dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

// One read of the input, where a group fits a wave or a workgroup; hipErrorNotSupported for
// the other groups.
template <int F, bool STREAM>
static hipError_t launch_requant_once(const RequantArgs& a, int rule, hipStream_t s) {
  if (a.group <= 1024 && a.lanes_per_group * 16 == a.group) return launch_requant_chunks<F, STREAM>(a, rule, s);
  switch (a.group) {
    case 2048: return launch_requant_group_wg<F, 128, 1, STREAM>(a, rule, s);
    case 4096: return launch_requant_group_wg<F, 256, 1, STREAM>(a, rule, s);
    case 8192: return launch_requant_group_wg<F, 256, 2, STREAM>(a, rule, s);
    case 16384: return launch_requant_group_wg<F, 256, 4, STREAM>(a, rule, s);
    case 32768: return launch_requant_group_wg<F, 512, 4, STREAM>(a, rule, s);
    default: return hipErrorNotSupported;
  }
}

template <int F>
static hipError_t launch_requant_scaled(const RequantArgs& a, int rule, hipStream_t s) {
  const int64_t n_groups = a.n / a.group;
  // Launches of 2^32 threads or more take the loop over groups.
  if (a.n / 16 < 0xFFFFFF00LL) {
    const hipError_t e = a.n >= kRequantStream ? launch_requant_once<F, true>(a, rule, s)
                                               : launch_requant_once<F, false>(a, rule, s);
    if (e != hipErrorNotSupported) return e;
  }
  int64_t blocks = (n_groups + 3) / 4;
  if (blocks > 65536) blocks = 65536;
  const unsigned grid = static_cast<unsigned>(blocks);
  switch (rule) {
    case kRTN: hipLaunchKernelGGL((k_requant_scaled<F, kRTN>), dim3(grid), dim3(256), 0, s, a); break;
    case kSR: hipLaunchKernelGGL((k_requant_scaled<F, kSR>), dim3(grid), dim3(256), 0, s, a); break;
    case kPHILOX: hipLaunchKernelGGL((k_requant_scaled<F, kPHILOX>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_requant_scaled<F, kWEYL>), dim3(grid), dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

template <int F>
static hipError_t launch_requant_16(const RequantArgs& a, int rule, hipStream_t s) {
  return a.n >= kRequantStream ? launch_requant_f<F, true>(a, rule, s) : launch_requant_f<F, false>(a, rule, s);
}

hipError_t launch_requant(const RequantArgs& a, int format, int rule, hipStream_t s) {
  switch (format) {
    case kFP16: return launch_requant_16<kFP16>(a, rule, s);
    case kBF16: return launch_requant_16<kBF16>(a, rule, s);
    case kE4M3: return launch_requant_scaled<kE4M3>(a, rule, s);
    case kINT8: return launch_requant_scaled<kINT8>(a, rule, s);
    case kINT4: return launch_requant_scaled<kINT4>(a, rule, s);
    default: return launch_requant_f<kFP32, false>(a, rule, s);
  }
}

hipError_t launch_dither(const DitherArgs& a, int rule, hipStream_t s) {
  const int64_t chunks = (a.n + 3) / 4;
  const unsigned grid = static_cast<unsigned>((chunks + 255) / 256);
  switch (rule) {
    case kRTN: hipLaunchKernelGGL((k_dither_fill<kRTN>), dim3(grid), dim3(256), 0, s, a); break;
    case kSR: hipLaunchKernelGGL((k_dither_fill<kSR>), dim3(grid), dim3(256), 0, s, a); break;
    case kPHILOX: hipLaunchKernelGGL((k_dither_fill<kPHILOX>), dim3(grid), dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((k_dither_fill<kWEYL>), dim3(grid), dim3(256), 0, s, a); break;
  }
  return hipGetLastError();
}

template <int F, int E, int AHEAD>
static hipError_t launch_replay_e(const ReplayArgs& a, int rule, int threads, hipStream_t s) {
  const unsigned grid = static_cast<unsigned>((a.n / E + threads - 1) / threads);
  switch (rule) {
    case kRTN: hipLaunchKernelGGL((k_replay<F, kRTN, E, AHEAD>), dim3(grid), dim3(threads), 0, s, a); break;
    case kSR: hipLaunchKernelGGL((k_replay<F, kSR, E, AHEAD>), dim3(grid), dim3(threads), 0, s, a); break;
    case kPHILOX: hipLaunchKernelGGL((k_replay<F, kPHILOX, E, AHEAD>), dim3(grid), dim3(threads), 0, s, a); break;
    default: hipLaunchKernelGGL((k_replay<F, kWEYL, E, AHEAD>), dim3(grid), dim3(threads), 0, s, a); break;
  }
  return hipGetLastError();
}

template <int F>
static hipError_t launch_replay_f(const ReplayArgs& a, int rule, hipStream_t s) {
  // Groups of 256 entries need four per lane. Philox makes its thresholds for four entries at a
  // time, twice the work for two per lane: INT8 and INT4, whose rounding is short enough for that
  // to show, take the short form only up to half that size (INT8 blocks of 128, 64 steps: 262k
  // entries 49.7 us with four, 48.3 with two; 400k 62.9 and 69.9).
  const int64_t most = rule == kPHILOX && is_int_fmt<F> ? kReplayShort / 2 : kReplayShort - 1;
  if (a.n <= most && a.lanes_per_group <= 32) {
    ReplayArgs b = a;
    if (Traits<F>::scaled) b.lanes_per_group *= 2;
    return launch_replay_e<F, 2, 4>(b, rule, 64, s);
  }
  return launch_replay_e<F, 4, 1>(a, rule, 256, s);
}

hipError_t launch_replay(const ReplayArgs& a, int format, int rule, hipStream_t s) {
  switch (format) {
    case kFP16: return launch_replay_f<kFP16>(a, rule, s);
    case kBF16: return launch_replay_f<kBF16>(a, rule, s);
    case kE4M3: return launch_replay_f<kE4M3>(a, rule, s);
    case kINT8: return launch_replay_f<kINT8>(a, rule, s);
    case kINT4: return launch_replay_f<kINT4>(a, rule, s);
    default: return launch_replay_f<kFP32>(a, rule, s);
  }
}

hipError_t launch_conv1d(const ConvArgs& a, hipStream_t s) {
  const unsigned grid = static_cast<unsigned>((a.n + 255) / 256);
  const uintptr_t both = reinterpret_cast<uintptr_t>(a.state) | reinterpret_cast<uintptr_t>(a.weight);
  if (a.width == 4 && (both & 15u) == 0)
    hipLaunchKernelGGL(k_conv1d_update4, dim3(grid), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(k_conv1d_update, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace ssmq
