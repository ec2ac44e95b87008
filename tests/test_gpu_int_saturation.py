"""Saturation of the integer formats, where the kernels do without a clamp: groups whose
maximum rounds above qmax after scaling, with thresholds at both ends of their range,
against the oracle bit for bit through ssmq_requantize."""
import numpy as np
import pytest
import torch

import oracle

from ._parity import DEV

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
