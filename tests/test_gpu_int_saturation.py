"""Saturation of the integer formats, where the kernels do without a clamp: groups whose
maximum rounds above qmax after scaling, with thresholds at both ends of their range,
against the oracle bit for bit through ssmq_requantize."""
import numpy as np
import pytest
import torch

import oracle

from ._parity import DEV, Bar

pytestmark = pytest.mark.gpu
QMAX = {"int8": 127, "int4": 7}


@pytest.fixture(scope="module")
def ssmq():
    import paper_2609_39185_amd as m
    m.library()
    return m


def _above(qmax, n):
    """n fp32 maxima m with fl32(m fl32(1 / fl32(m / qmax))) > qmax."""
    m = np.linspace(1.0, 3.9, 40 * n, dtype=np.float32)
    s = (m / np.float32(qmax)).astype(np.float32)
    q = (m * (np.float32(1) / s).astype(np.float32)).astype(np.float32)
    m = m[q > qmax]
    assert m.size >= n
    return m[:n]


def _extreme_steps(group):
    """Weyl steps whose thresholds of the entries of one group come within 2^12 of an end."""
    t = np.arange(1 << 18, dtype=np.uint64)
    phi, a, b = 2654435769, 0xC13FA9A9, 0x91E10DA6
    found = []
    for k in range(group):
        u = ((a + b * (k + 1) + phi * t) & 0xFFFFFFFF) >> 8
        for hit in (np.nonzero(u < 1 << 6)[0], np.nonzero(u >= (1 << 24) - (1 << 6))[0]):
            found += [(k, int(v)) for v in hit[:1]]
    return found


@pytest.mark.parametrize("fmt", ["int8", "int4"])
def test_saturation_without_clamp(ssmq, fmt):
    group, qmax = 16, QMAX[fmt]
    maxima = _above(qmax, 64)
    hits = _extreme_steps(group)
    assert len(hits) >= 8
    rng = np.random.default_rng(3)
    for k, step in hits + [(0, 1), (15, 2)]:
        # every group has +-its maximum at entry k, whose threshold is the extreme one in
        # group 0; the group index moves the others'
        h = (rng.uniform(-1, 1, (64, group)) * maxima[:, None]).astype(np.float32)
        h[:, k] = maxima * np.where(np.arange(64) % 2, -1, 1)
        h[0] = maxima[0] * (1 if step % 2 else -1)
        for rule in ("weyl", "rtn", "sr"):
            codes = torch.zeros(h.size // (2 if fmt == "int4" else 1), dtype=torch.uint8, device=DEV)
            scale = torch.zeros(64, device=DEV)
            ssmq.requantize(torch.from_numpy(h.ravel()).to(DEV), codes, scale, rule=rule, fmt=fmt,
                            scale_group=group, step=step)
            torch.cuda.synchronize()
            want, wsc = oracle.requantize(fmt, rule, h.ravel(), group=group, step=step)
            assert np.array_equal(scale.cpu().numpy(), wsc)
            assert np.array_equal(codes.cpu().numpy(), np.asarray(want).ravel()), (fmt, rule, k, step)


# the step kernels that clamp and those that test the smallest sum instead: heads of one, two
# and four chunks per thread, rows, Mamba-1 rows; every value of a group is its maximum, so
# every code is at an end of the range, and a third of the heads hold infinities or NaN
@pytest.mark.parametrize("rule", ["weyl", "sr", "rtn"])
@pytest.mark.parametrize("headdim,dstate,group,family,b,h", [
    (64, 128, 128, "mamba2", 2, 6), (64, 128, 0, "mamba2", 2, 6), (64, 64, 16, "mamba2", 2, 6),
    (128, 256, 0, "mamba2", 1, 6), (3, 128, 128, "mamba2", 2, 6), (1, 16, 16, "mamba1", 3, 300)])
@pytest.mark.parametrize("fmt", ["int8", "int4"])
def test_step_saturation(ssmq, fmt, rule, headdim, dstate, group, family, b, h):
    from paper_2609_39185_amd import workloads as wl

    qmax, size = QMAX[fmt], group or headdim * dstate
    A, D = wl.layer_params(family, h, dstate, 31)
    x, dt, B, C = wl.step_inputs(b, h, headdim, dstate, 1, 32)
    x.zero_()  # h_new = dA h_prev: every group keeps one magnitude (per row where A is per state)
    if family == "mamba1":
        A = A[:, :1].expand(h, dstate).contiguous()
    n = b * h * headdim * dstate
    codes = torch.where(torch.arange(n) % 3 == 0, -qmax, qmax).view(b, h, headdim, dstate)
    per = 2 if fmt == "int4" else 1
    packed = codes.to(torch.uint8) if per == 1 else (
        (codes[..., 0::2] & 15) | ((codes[..., 1::2] & 15) << 4)).to(torch.uint8)
    maxima = torch.from_numpy(np.resize(_above(qmax, 64), n // size).astype(np.float32))
    scale = (maxima / qmax).contiguous()
    scale[::3] = torch.tensor([float("inf"), float("nan"), 1e-39]).repeat(n // size // 9 + 1)[:scale[::3].numel()]
    print(f"case step saturation {fmt} {rule} {headdim}x{dstate} g{group} {family}", flush=True)
    st, sc, y = packed.to(DEV), scale.to(DEV), torch.zeros((b, h, headdim), device=DEV)
    ssmq.state_update(st, sc, *(v.to(DEV) for v in (x, dt, A, B, C, D)), y, rule=rule, fmt=fmt,
                      scale_group=group, step=77, layer=1)
    torch.cuda.synchronize()
    want, wsc, _, _ = oracle.state_update(
        fmt, rule, wl.to_numpy_codes(fmt, packed), scale.numpy(), x.numpy(), dt.numpy(), A.numpy(),
        B.numpy(), C.numpy(), D.numpy(), step=77, layer=1, block=16, group=group)
    g, w = sc.cpu().numpy(), np.asarray(wsc)
    fin = np.isfinite(w)
    assert np.array_equal(np.isfinite(g), fin)
    # the scale folded into the decay may move h_new, and so the scale, by an ulp or two
    assert np.all(np.abs(g[fin] - w[fin]) <= 2.0 ** -21 * w[fin])
    # that ulp moves q = +-qmax by at most 2^-21 qmax: an entry takes the neighbouring code if its
    # threshold is that close to an end, one in 2^21 / qmax (the stated bar: one code, 1e-4 of them);
    # a sum past the range that wrapped round would be off by the whole range
    Bar(fmt, f"step saturation {fmt} {rule}").codes(wl.to_numpy_codes(fmt, st), np.asarray(want)).check()
