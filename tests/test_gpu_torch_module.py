"""The C++ module behind the binding's calls: the plain case gives what the binding's own way gives, bit for bit, and everything
else is left to the binding, which takes or refuses it as it does by itself."""
import numpy as np
import pytest
import torch

from paper_2605_24058_amd import binding


def test_what_is_not_plain_is_left_to_the_binding():
    # CPU tensors, other types, wrong argument counts: None, for every function and without a device
    m = binding._load_torch_module()
    t = torch.zeros(2, 2, dtype=torch.float16)
    for name, n in (("forward", 9), ("forward_multi", 9), ("forward_batched", 10), ("forward_batched_multi", 10), ("pack_latents", 4),
                    ("forward_save_t", 8), ("forward_multi_save_t", 8), ("backward", 15), ("backward_multi", 15)):
        f = getattr(m, name)
        assert f(*[t] * n) is None and f(*[None] * n) is None and f(*["x"] * n) is None and f(t) is None, name


def _case(ell, pool, T=5, d_in=64, d_out=48, r=8, n=3):
    g = torch.Generator().manual_seed(3)
    half = lambda *s: torch.randn(s, generator=g).half().cuda()
    lead = ((n,) if pool else ()) + ((ell,) if ell > 1 else ())
    word = lambda rows, cols: torch.randint(-2**31, 2**31 - 1, ((n,) if pool else ()) + ((rows * cols + 31) // 32,), generator=g,
                                            dtype=torch.int32).cuda()
    p = [half(T, d_in), word(r, d_in), word(d_out, r), half(*lead, d_in), half(*lead, r), half(*lead, d_out)]
    if pool:
        p.append(torch.tensor([0, 2, -1, 2, 1], dtype=torch.int32).cuda())
    return p + [half(T, d_out)]


def _both(monkeypatch, call):
    """The call through the module and the binding's own way: (result or exception type) of each."""
    got = []
    for plain in (True, False):
        with monkeypatch.context() as mp:
            if not plain:
                mp.setattr(binding, "_plain_call", lambda *a: None)
            try:
                got.append(call())
                if torch.cuda.is_available():
                    torch.cuda.synchronize()
            except Exception as e:  # noqa: BLE001 - the type is what is compared
                got.append(type(e))
    return got


def _same(a, b):
    if isinstance(a, dict):
        return a.keys() == b.keys() and all(_same(a[k], b[k]) for k in a)
    if isinstance(a, (tuple, list)):
        return len(a) == len(b) and all(_same(u, v) for u, v in zip(a, b))
    if isinstance(a, torch.Tensor):
        if not isinstance(b, torch.Tensor) or a.dtype != b.dtype or a.shape != b.shape:
            return False
        bits = {torch.float16: torch.int16, torch.float32: torch.int32}.get(a.dtype, a.dtype)
        return torch.equal(a.view(bits), b.view(bits))
    return a is b


def test_the_comparison_is_by_bits():
    a, b = torch.tensor([1.0, float("nan")]).half(), torch.tensor([1.0, 0.0]).half()
    assert _same(a, a.clone()) and not _same(a, b) and not _same(b, -b) and not _same(a, None) and not _same(a, a.float())


@pytest.mark.gpu
@pytest.mark.parametrize("name,ell,pool", [("lordba_forward", 1, False), ("lordba_forward_multi", 2, False),
                                           ("lordba_forward_batched", 1, True), ("lordba_forward_batched_multi", 2, True)])
def test_forward_calls(monkeypatch, name, ell, pool):
    f, p = getattr(binding, name), _case(ell, pool)
    side = torch.cuda.Stream()
    for kw in ({}, {"y_out": None}, {"stream": side}, {"stream": side.cuda_stream}):
        a, b = _both(monkeypatch, lambda: f(*p, **({"y_out": torch.empty_like(p[-1])} if "y_out" in kw else kw)))
        assert _same(a, b), (name, kw)
    y = p[-1].clone()
    assert f(*p[:-1], y, y_out=y) is y   # in place
    # one argument at a time: another type, not contiguous, on the CPU, shorter, one more dimension, not a tensor
    spoil = (lambda t: t.double(), lambda t: torch.stack((t, t), -1)[..., 0], lambda t: t.cpu(), lambda t: t[..., :-1].contiguous(),
             lambda t: t[None], lambda t: None)
    for k in range(len(p)):
        for s in spoil:
            q = list(p)
            q[k] = s(p[k])
            a, b = _both(monkeypatch, lambda: f(*q))
            assert _same(a, b), (name, k)


@pytest.mark.gpu
@pytest.mark.parametrize("ell", [1, 2])
def test_training_calls(monkeypatch, ell):
    T, d_in, d_out, r = 37, 96, 64, 8
    g = torch.Generator().manual_seed(4)
    half = lambda *s: torch.randn(s, generator=g).half().cuda()
    lead = (ell,) if ell > 1 else ()
    x, gy, yb, dxb = half(T, d_in), half(T, d_out), half(T, d_out), half(T, d_in)
    latA, latB = torch.randn(r, d_in, generator=g).cuda(), torch.randn(d_out, r, generator=g).cuda()
    s = half(*lead, d_in), half(*lead, r), half(*lead, d_out)
    for transposed in (True, False):
        a, b = _both(monkeypatch, lambda: binding.lordba_pack_latents(latA, latB, transposed=transposed))
        assert _same(a, b)
    pA, pB, pAt, pBt = binding.lordba_pack_latents(latA, latB)
    save = binding.lordba_forward_save_t if ell == 1 else binding.lordba_forward_multi_save_t
    back = binding.lordba_backward if ell == 1 else binding.lordba_backward_multi
    a, b = _both(monkeypatch, lambda: tuple(v[..., :T].clone() if v.dtype == torch.float32 else v for v in save(x, pA, pB, *s, y_base=yb)))
    assert _same(a, b)
    t = save(x, pA, pB, *s, y_base=yb)[1]
    need = (binding.lordba_backward_workspace_bytes(T, d_in, d_out, r) if ell == 1
            else binding.lordba_backward_multi_workspace_bytes(T, d_in, d_out, r, ell))
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    for lat in ((latA, latB), (None, None)):
        for kw in ({}, {"dx_base": dxb}, {"dx_base": dxb, "t_saved": t, "workspace": ws}, {"workspace": ws[:16]}):   # (the last: refused)
            a, b = _both(monkeypatch, lambda: back(x, gy, pA, pAt, pBt, *s, *lat, 100.0, **kw))
            assert _same(a, b), kw.keys()
    assert isinstance(_both(monkeypatch, lambda: back(x, gy, pA, pAt, pBt, *s, latA, latB, 100, dx_base=dxb))[0], dict)   # an int kappa


@pytest.mark.gpu
def test_tensors_that_refuse_their_pointer(monkeypatch):
    # The exception rises where the call is about to give the interpreter's lock away; for every call
    def refusing(t):
        t = t.clone()
        torch._C._set_throw_on_mutable_data_ptr(t)
        return t

    for name, ell, pool in (("lordba_forward", 1, False), ("lordba_forward_multi", 2, False), ("lordba_forward_batched", 1, True),
                            ("lordba_forward_batched_multi", 2, True)):
        p = _case(ell, pool)
        for k in range(len(p)):
            q = p[:k] + [refusing(p[k])] + p[k + 1:]
            assert _both(monkeypatch, lambda: getattr(binding, name)(*q)) == [RuntimeError, RuntimeError], (name, k)
        assert _both(monkeypatch, lambda: getattr(binding, name)(*p, y_out=refusing(p[-1]))) == [RuntimeError, RuntimeError], name
    x, pA, pB, si, sr, so, yb = _case(1, False)
    assert _both(monkeypatch, lambda: binding.lordba_forward_save_t(x, pA, refusing(pB), si, sr, so, y_base=yb)) == [RuntimeError] * 2
    lat = torch.ones(8, 64).cuda(), torch.ones(48, 8).cuda()
    assert _both(monkeypatch, lambda: binding.lordba_pack_latents(lat[0], refusing(lat[1]))) == [RuntimeError] * 2
    args = [x, yb, pA, pA, pB, si, sr, so, *lat, 100.0]
    for k in range(10):
        q = args[:k] + [refusing(args[k])] + args[k + 1:]
        assert _both(monkeypatch, lambda: binding.lordba_backward(*q, dx_base=x.clone())) == [RuntimeError] * 2, k


@pytest.mark.gpu
def test_modes_that_see_torchs_functions_get_the_bindings_own_way():
    from torch._subclasses.fake_tensor import FakeTensorMode
    from torch.utils._python_dispatch import TorchDispatchMode

    class Watch(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    m, p = binding._load_torch_module(), _case(1, False)
    assert isinstance(m.forward(*p, None, None), torch.Tensor)
    with Watch():
        assert m.forward(*p, None, None) is None
        under = binding.lordba_forward(*p)
    assert _same(under, binding.lordba_forward(*p))
    with FakeTensorMode(allow_non_fake_inputs=True):
        assert m.forward(*p, None, None) is None   # (its output would have no memory)


@pytest.mark.gpu
def test_default_devices_and_whole_numbers_are_the_plain_case(monkeypatch):
    from torch.overrides import TorchFunctionMode
    from torch.utils._device import DeviceContext

    class Watch(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    m, p = binding._load_torch_module(), _case(1, False)
    want = m.forward(*p, None, None)
    with torch.device("cpu"), torch.device("cuda"):
        assert _same(m.forward(*p, None, None), want)
    torch.set_default_device("cpu")
    try:
        assert _same(m.forward(*p, None, None), want)
        with Watch():
            assert m.forward(*p, None, None) is None
    finally:
        torch.set_default_device(None)
    with Watch(), torch.device("cpu"):
        assert m.forward(*p, None, None) is None
    with type("Other", (DeviceContext,), {})(torch.device("cpu")):
        assert m.forward(*p, None, None) is None

    x, pA, pB, si, sr, so, yb = p
    lat = torch.ones(8, 64).cuda(), torch.ones(48, 8).cuda()
    back = lambda kappa: m.backward(x, yb, pA, pA, pB, si, sr, so, *lat, kappa, None, None, None, None)
    for kappa in (100, 100.0, True, np.float64(25.0), 10**400, np.float32(3.0), "100", None):
        got = back(kappa)
        plain = isinstance(kappa, float) or (isinstance(kappa, int) and kappa < 10**300)
        assert (got is not None) == plain, kappa
        if plain:
            assert _same(got, back(float(kappa))), kappa
