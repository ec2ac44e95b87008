"""The C++ marshalling of the per-token calls against the ctypes path: what it leaves to
that path (CPU), and that both paths give the same bits and the same errors (GPU)."""
import numpy as np
import pytest
import torch

from paper_2609_39185_amd import workloads as wl

N = 16


@pytest.fixture(scope="module")
def binding():
    import paper_2609_39185_amd  # noqa: F401
    from paper_2609_39185_amd import _binding
    _binding.library()
    return _binding


class Sub(torch.Tensor):
    pass


def test_unhandled_calls_are_left_to_ctypes(binding):
    """CPU tensors, subclasses, wrapped tensors, wrong types and argument counts."""
    n = binding._load_native()
    t = torch.zeros(1, 2, 3, N)
    ints = [0, 3, 16, 0, 0, 0, 0, 0]

    def call(first):
        return n.state_update(first, None, t, t, t, t, t, t, t, *ints, False, None, False, None, None)

    assert call(t) is None and call(t.as_subclass(Sub)) is None
    assert call(None) is None and call(3) is None and call(np.zeros(4)) is None
    assert n.state_update(t) is None and n.conv1d_update() is None and n.requantize(t, t) is None
    seen = []
    torch.vmap(lambda v: seen.append(call(v)) or v)(torch.zeros(2, 1, 2, 3, N))
    torch.func.grad(lambda v: (seen.append(call(v)), v.sum())[1])(t)
    assert seen == [None, None]


class Off:
    """A stand-in for the C++ module that leaves every call."""
    state_update = conv1d_update = requantize = staticmethod(lambda *a: None)


def _both(binding, monkeypatch, make):
    """make()'s result through the C++ path and through ctypes: (outcome, outcome)."""
    out = []
    for module in (binding._load_native(), Off):
        monkeypatch.setattr(binding, "_native", module)
        try:
            out.append(make())
        except Exception as e:  # the error itself is compared
            out.append((type(e), str(e)))
        torch.cuda.synchronize()
    monkeypatch.undo()
    return out


STEPS = [("bf16", 0, {}), ("int4", 16, {"dt_softplus": True}), ("e4m3", 16, {"z": True, "dt_bias": True}),
         ("int8", 16, {"fp32_state": True}), ("fp32", 0, {"stream": True}),
         # left to ctypes or refused there
         ("fp16", 0, {"seed": np.uint32(7)}), ("fp16", 0, {"strided": True}), ("fp16", 0, {"wide": True}),
         ("fp16", 0, {"layer": -1, "step": 2 ** 40 + 3}), ("fp16", 0, {"entry_base": 3}),
         ("fp16", 0, {"rule": "none"}), ("int8", 48, {}), ("fp16", 0, {"odd": True})]


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,group,how", STEPS)
def test_step_same_as_ctypes(binding, monkeypatch, fmt, group, how):
    dev, b, h, p = torch.device("cuda:0"), 3, 4, 8
    how = dict(how)
    A, D = (v.to(dev) for v in wl.layer_params("mamba2", h, N, 1))
    x, dt, B, C = (v.to(dev) for v in wl.step_inputs(b, h, p, N, 2, 2))
    kw = {"rule": how.pop("rule", "weyl"), "fmt": fmt, "scale_group": group, "seed": 5, "layer": 1, "step": 9}
    strided, wide, odd = how.pop("strided", False), how.pop("wide", False), how.pop("odd", False)
    if how.pop("z", False):
        kw["z"] = torch.ones_like(x)
    if how.pop("dt_bias", False):
        kw["dt_bias"] = torch.full((h,), 0.1, device=dev)
    if how.pop("stream", False):
        kw["stream"] = torch.cuda.Stream()
    kw.update(how)
    torch.cuda.synchronize()

    def make():
        codes, scale = wl.initial_state(fmt, b, h, p, N, 3, group=16 if group else 0)
        if kw.get("fp32_state"):
            codes = torch.linspace(-1, 1, b * h * p * N).view(b, h, p, N)
        st, sc = codes.to(dev), None if scale is None else scale.to(dev)
        if strided:
            st = st.transpose(0, 1)
        if wide:
            st = st.to(torch.int32)
        if odd:  # two bytes off the 16-byte alignment
            room = torch.zeros(st.numel() + 8, dtype=st.dtype, device=dev)
            st = room[1:1 + st.numel()].view(st.shape)
        y = torch.zeros((b, h, p), device=dev)
        torch.cuda.synchronize()
        binding.state_update(st, sc, x, dt, A, B, C, D, y, **kw)
        torch.cuda.synchronize()
        return [v.cpu().numpy().tobytes() for v in (st, y) + (() if sc is None else (sc,))]

    print(f"case native step {fmt} {group} {how}", flush=True)
    got, want = _both(binding, monkeypatch, make)
    assert got == want


@pytest.mark.gpu
@pytest.mark.parametrize("case", ["conv", "conv_no_bias", "requant", "requant_group", "requant_size", "requant_cpu"])
def test_other_calls_same_as_ctypes(binding, monkeypatch, case):
    dev = torch.device("cuda:0")

    def make():
        if case.startswith("conv"):
            st, w = (torch.from_numpy(np.random.default_rng(8).standard_normal(s).astype(np.float32)).to(dev)
                     for s in ((2, 5, 4), (5, 4)))
            x, out = torch.ones((2, 5), device=dev), torch.zeros((2, 5), device=dev)
            binding.conv1d_update(st, x, w, None if case == "conv_no_bias" else torch.ones(5, device=dev), out)
            res = (st, out)
        else:
            hh = torch.linspace(-2, 3, 512, device="cpu" if case == "requant_cpu" else dev)
            codes = torch.zeros(500 if case == "requant_size" else 512, dtype=torch.uint8, device=dev)
            sc = torch.zeros(512 // 32, device=dev)
            kw = {"scale_group": 32} if case == "requant_group" else {"head_size": 32}
            binding.requantize(hh, codes, sc, rule="sr", fmt="e4m3", seed=1, step=4, **kw)
            res = (codes, sc)
        torch.cuda.synchronize()
        return [v.cpu().numpy().tobytes() for v in res]

    print(f"case native {case}", flush=True)
    got, want = _both(binding, monkeypatch, make)
    assert got == want


@pytest.mark.parametrize("why", ["missing", "other torch", "no version"])
def test_ctypes_takes_over_without_the_module(binding, monkeypatch, why):
    """Where the module cannot be loaded, or was built for another torch, calls reach the
    ctypes path (here its refusal of CPU tensors), with one warning per process."""
    import sys
    import types

    name = "paper_2609_39185_amd._native"
    fake = types.ModuleType(name)  # an older module: taking a call would be a mistake
    fake.state_update = fake.conv1d_update = fake.requantize = lambda *a: 0
    if why == "other torch":
        fake.BUILT_FOR = "torch 1.0, Python 3.10"
    monkeypatch.setitem(sys.modules, name, None if why == "missing" else fake)
    if why != "missing":
        monkeypatch.setattr(sys.modules["paper_2609_39185_amd"], "_native", fake, raising=False)
    else:
        monkeypatch.delattr(sys.modules["paper_2609_39185_amd"], "_native", raising=False)
    monkeypatch.setattr(binding, "_native", None)
    t = torch.zeros(1, 2, 4)
    with pytest.warns(RuntimeWarning, match="ctypes"):
        with pytest.raises(ValueError, match="GPU memory"):
            binding.conv1d_update(t, t[0], t[0], None, t[0])
    import warnings
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        with pytest.raises(ValueError, match="GPU memory"):
            binding.requantize(t, torch.zeros(8, dtype=torch.int16), None, rule="rtn", fmt="bf16")


@pytest.mark.gpu
def test_step_without_the_module(binding, monkeypatch):
    """The same bits through the stand-in that serves calls where the module is missing."""
    dev = torch.device("cuda:0")
    codes = torch.linspace(-2, 2, 4 * N, device=dev)

    def make():
        out = torch.zeros(4 * N, dtype=torch.int16, device=dev)
        binding.requantize(codes, out, None, rule="weyl", fmt="bf16", step=3)
        torch.cuda.synchronize()
        return out.cpu().numpy().tobytes()

    assert binding._load_native() is not binding._CtypesOnly, "run __graft_entry__.build()"
    want = make()
    monkeypatch.setattr(binding, "_native", binding._CtypesOnly)
    print("case native stand-in", flush=True)
    assert make() == want
