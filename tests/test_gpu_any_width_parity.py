"""GPU parity of the matrix-core variants for element-aligned tensors of any width: every forward entry point against the fp64
oracle, on widths that are no multiples of 32 / 8, and on tensors that start at odd elements.  The bar is that of the other
forward tests: per token row ||y_gpu - y||_2 / ||y||_2 <= 1e-3, also with y_base = 0."""
import numpy as np
import pytest

import oracle
from paper_2605_24058_amd import binding, inputs

pytestmark = pytest.mark.gpu

TOL = 1e-3
A_AUTO, A_GEN = 0, 1


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.load_library()
    return torch


def place(torch, a, shift):
    """`a` on the GPU, its first element `shift` elements behind a 16-byte boundary, NaN (or all ones) around it."""
    t = torch.from_numpy(np.ascontiguousarray(a))
    fill = float("nan") if t.dtype == torch.float16 else -1
    big = torch.full((t.numel() + 64,), fill, dtype=t.dtype, device="cuda:0")
    v = big[16 + shift:16 + shift + t.numel()].view(t.shape)
    v.copy_(t)
    return v


# (T, d_in, d_out, r): widths one below, at and one above the edges of groups (8), words (32), chunks and blocks (128) and of the
# one-shot x pipeline (2048); every rank-block count; one row, a ragged tile,
# more tiles than are split; an aligned shape (four envelopes at r = 64 take the general kernel)
SHAPES = [(1, 8, 8, 5), (3, 9, 15, 64), (5, 33, 17, 3), (9, 127, 129, 16), (8, 129, 127, 8), (17, 136, 250, 17), (300, 1000, 3001, 12),
          (261, 2047, 513, 33), (12, 2049, 1030, 64), (11, 512, 640, 64), (7, 3999, 640, 16), (2, 40, 4097, 48)]


def lifted(d):
    """With few input channels the branch alone would land among the subnormals of fp16: lift it out."""
    if d["x"].shape[1] < 256:
        d["s_out"] = (d["s_out"].astype(np.float32) * 2.0 ** 8).astype(np.float16)
    return d


def pools(d):
    packed = [binding.lordba_pack_signs(a, b) for a, b in zip(d["signsA"], d["signsB"])]
    return np.stack([p[0] for p in packed]).view(np.int32), np.stack([p[1] for p in packed]).view(np.int32)


@pytest.mark.parametrize("ell", [1, 2, 3, 4])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "T%d_%dx%d_r%d" % s)
def test_odd_widths(torch_cuda, shape, ell):
    torch = torch_cuda
    T, d_in, d_out, r = shape
    d = lifted(inputs.make_inputs_multi(31, T, d_in, d_out, r, ell))
    for y_base in (d["y_base"], np.zeros_like(d["y_base"])):
        want = oracle.forward_multi(d["x"], d["signsA"], d["signsB"], d["s_in"], d["s_rank"], d["s_out"], y_base)
        pA, pB = binding.lordba_pack_signs(d["signsA"], d["signsB"])
        for shift in (0, 1):
            args = [place(torch, v, shift) for v in (d["x"], pA.view(np.int32), pB.view(np.int32), d["s_in"], d["s_rank"], d["s_out"])]
            out = place(torch, np.full((T, d_out), np.nan, np.float16), 3 * shift)
            binding.lordba_forward_multi(*args, place(torch, y_base, shift), y_out=out)
            torch.cuda.synchronize()
            around = out._base.cpu().numpy()
            at = 16 + 3 * shift
            assert np.isnan(around[:at]).all() and np.isnan(around[at + T * d_out:]).all(), "write outside y_out"
            got = out.cpu().numpy()
            err = oracle.row_rel_l2(got.astype(np.float64), want).max()
            assert err <= TOL, (shape, ell, shift, err)
            # in place, and the training forward with its t (fp32 sums of d_in terms: at most about sqrt(d_in) 2^-24)
            inout = place(torch, y_base, shift)
            binding.lordba_forward_multi(*args, inout, y_out=inout)
            t_out = torch.full((ell, r, binding.saved_t_stride(T)), float("nan"), dtype=torch.float32, device="cuda:0")
            y2, _ = binding.lordba_forward_multi_save_t(*args, y_base=place(torch, y_base, shift), t_out=t_out)
            torch.cuda.synchronize()
            assert np.array_equal(inout.cpu().numpy(), got) and np.array_equal(y2.cpu().numpy(), got)
            t_got = t_out.cpu().numpy()
            assert np.isnan(t_got[:, :, T:]).all()
            for e in range(ell):
                assert oracle.rel_l2(t_got[e, :, :T].T, oracle.rank_intermediate(d["x"], d["signsA"], d["s_in"][e])) <= 1e-5


@pytest.mark.parametrize("ell", [1, 2, 4])
@pytest.mark.parametrize("case", [(21, 100, 61, 5, 3, "mixed"), (21, 512, 384, 64, 3, "mixed"), (14, 2050, 90, 50, 3, "mixed"), (300, 2055, 1001, 16, 4, "segments"), (9, 1000, 3001, 33, 5, "decode")],
                         ids=lambda c: "T%d_%dx%d_r%d_n%d_%s" % c)
def test_odd_widths_of_a_pool(torch_cuda, case, ell):
    torch = torch_cuda
    T, d_in, d_out, r, n, pattern = case
    d = inputs.make_adapter_pool_multi(32, d_in, d_out, r, n, ell)
    d.update(inputs.make_activations(32, T, d_in, d_out))
    ids = inputs.make_adapter_ids(32, T, n, pattern)
    d = lifted(d)
    want = oracle.forward_batched_multi(d["x"], d["signsA"], d["signsB"], d["s_in"], d["s_rank"], d["s_out"], ids, d["y_base"])
    pA, pB = pools(d)
    args = [place(torch, v, 1) for v in (d["x"], pA, pB, d["s_in"], d["s_rank"], d["s_out"], ids)]
    for algo in (A_AUTO, A_GEN):
        y = place(torch, d["y_base"], 1)
        binding.lordba_forward_batched_multi(*args, y, y_out=y, algo=algo)
        torch.cuda.synchronize()
        got = y.cpu().numpy()
        assert oracle.row_rel_l2(got.astype(np.float64), want).max() <= TOL, (case, ell, algo)
        none = (ids < 0) | (ids >= n)
        assert np.array_equal(got[none], d["y_base"][none])


def test_a_row_of_nan_stays_in_its_row(torch_cuda):
    """Groups that reach past the end of a row must not let the next row's values in."""
    torch = torch_cuda
    d = inputs.make_inputs(33, 6, 203, 77, 16)
    clean = binding.to_device(d)
    y0 = binding.lordba_forward(clean["x"], clean["packedA"], clean["packedB"], clean["s_in"], clean["s_rank"], clean["s_out"], clean["y_base"])
    x, yb = clean["x"].clone(), clean["y_base"].clone()
    x[3] = float("nan")
    yb[4] = float("inf")
    y = binding.lordba_forward(x, clean["packedA"], clean["packedB"], clean["s_in"], clean["s_rank"], clean["s_out"], yb)
    torch.cuda.synchronize()
    y, y0 = y.cpu().numpy(), y0.cpu().numpy()
    for row in (0, 1, 2, 5):
        assert np.array_equal(y[row], y0[row]), row
    assert np.isnan(y[3]).all() and np.isinf(y[4]).all()


def same_with_infinities(got, want, label):
    """Infinities of the same sign and NaN in the same places; finite values within one rounding to fp16."""
    with np.errstate(over="ignore"):
        w16 = want.astype(np.float16)
    assert np.array_equal(np.isnan(got), np.isnan(w16)), label
    assert np.array_equal(np.isposinf(got), np.isposinf(w16)) and np.array_equal(np.isneginf(got), np.isneginf(w16)), label
    ok = np.isfinite(w16)
    # half a unit of fp16 and the fp32 sums
    assert np.abs(got[ok].astype(np.float64) - want[ok]).max(initial=0.0) <= 2.0 ** -10 * max(np.abs(want[ok]).max(initial=0.0), 2.0 ** -14), label


@pytest.mark.parametrize("ell", [1, 2, 3])
@pytest.mark.parametrize("r", [1, 5, 16, 17, 50])
@pytest.mark.parametrize("where", ["x", "x_end", "s_in", "s_rank", "s_out"])
def test_infinities(torch_cuda, where, r, ell):
    """An infinite input gives infinities where IEEE arithmetic does (one rank, or all ranks' signs agree) and NaN only where
    infinities of both signs meet."""
    torch = torch_cuda
    d = inputs.make_inputs_multi(34, 6, 203, 77, r, ell)
    place_of = {"x": ("x", (2, 3)), "x_end": ("x", (2, 202)), "s_in": ("s_in", (ell - 1, 7)), "s_rank": ("s_rank", (0, r // 2)), "s_out": ("s_out", (0, 75))}
    name, index = place_of[where]
    d[name][index] = np.inf
    with np.errstate(invalid="ignore"):
        want = oracle.forward_multi(d["x"], d["signsA"], d["signsB"], d["s_in"], d["s_rank"], d["s_out"], d["y_base"])
    dev = binding.to_device(d)
    args = [dev[k] for k in ("x", "packedA", "packedB", "s_in", "s_rank", "s_out", "y_base")]
    for algo in (A_GEN, A_AUTO):
        got = binding.lordba_forward_multi(*args, algo=algo).cpu().numpy()
        same_with_infinities(got, want, (where, r, ell, algo))
    # one adapter of a pool, whose other rows stay finite
    ids = torch.tensor([0, 0, 1, 1, 0, 1], dtype=torch.int32, device="cuda")
    clean = binding.to_device(inputs.make_inputs_multi(35, 6, 203, 77, r, ell))
    pool = [torch.stack([clean[k], dev[k]]) for k in ("packedA", "packedB", "s_in", "s_rank", "s_out")]
    got = binding.lordba_forward_batched_multi(dev["x"], *pool, ids, dev["y_base"]).cpu().numpy()
    rows = [2, 3, 5]
    same_with_infinities(got[rows], want[rows], (where, r, ell, "pool"))
    assert np.isfinite(got[[0, 1, 4]]).all()


def backward_both_ways(torch, d):
    """The parameter gradients and dx by the element-aligned matrix-core kernels (kept t in rows of the padded token count) and by
    the general kernel (rows of T, no multiple of 128), from the same t."""
    T = d["x"].shape[0]
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    w = lambda a: cu(a.view(np.int32))
    pA, pB = map(w, binding.lordba_pack_signs(d["signsA"], d["signsB"]))
    pAt, pBt = map(w, binding.lordba_pack_transposed(d["signsA"], d["signsB"]))
    x, scales = cu(d["x"]), tuple(cu(d[k]) for k in ("s_in", "s_rank", "s_out"))
    _, t = binding.lordba_forward_save_t(x, pA, pB, *scales)
    out = []
    for t_saved in (t, t[:, :T].contiguous()):
        got = binding.lordba_backward(x, cu(d["g"]), pA, pAt, pBt, *scales, cu(d["latA"]), cu(d["latB"]), 100.0,
                                      dx_base=cu(d["dx_base"]), t_saved=t_saved)
        out.append({k: v.cpu().numpy() for k, v in got.items()})
    return out


# (the last row and column: what a ragged group or a padded row repeats; a rank scale of zero; g, whose du is then infinite)
@pytest.mark.parametrize("r", [1, 5, 17, 50])
@pytest.mark.parametrize("where", [("x", (3, 7)), ("x", (44, 56)), ("g", (2, 32)), ("g", (44, 1)), ("s_rank", (0,)), ("s_out", (4,))],
                         ids=lambda w: "%s_%s" % (w[0], "_".join(map(str, w[1]))))
def test_infinities_in_the_backward(torch_cuda, where, r):
    """Infinite and NaN gradients where the general kernel, which adds up each column by itself, has them; the rest as it has them
    (fp32 sums of 45 terms in another order: 45 half units of 2^-24 of the largest partial sum, taken as 1e-5 of the norm)."""
    d = inputs.make_backward_inputs(36, 45, 57, 33, r)
    d[where[0]][where[1]] = np.inf
    d["s_rank"][r // 2] = 0 if where[0] != "s_rank" else d["s_rank"][r // 2]
    any_, general = backward_both_ways(torch_cuda, d)
    for k in general:
        a, b = any_[k].astype(np.float64), general[k].astype(np.float64)
        assert np.array_equal(np.isnan(a), np.isnan(b)), (k, where, r)
        assert np.array_equal(np.isposinf(a), np.isposinf(b)) and np.array_equal(np.isneginf(a), np.isneginf(b)), (k, where, r)
        ok = np.isfinite(b)
        assert np.linalg.norm(a[ok] - b[ok]) <= 1e-5 * np.linalg.norm(b[ok]), (k, where, r)


@pytest.mark.parametrize("shape", [(57, 33, 50), (129, 200, 33), (1000, 77, 64)], ids=lambda s: "%dx%d_r%d" % s)
def test_gradients_keep_24_bits(torch_cuda, shape):
    """One row of x and g that holds powers of two: a latent gradient is then alpha * dt * smooth-sign factor with exact products
    by 2^n, and the fp32 dt must come through whole, as in the general kernel."""
    d_in, d_out, r = shape
    d = inputs.make_backward_inputs(37, 1, d_in, d_out, r)
    rng = np.random.default_rng(38)
    for k in ("x", "g"):
        d[k] = np.ldexp(np.where(rng.random(d[k].shape) < 0.5, -1.0, 1.0), rng.integers(-3, 4, d[k].shape)).astype(np.float16)
    any_, general = backward_both_ways(torch_cuda, d)
    for k in ("d_latentA", "d_latentB"):
        assert general[k].any() and np.array_equal(any_[k], general[k]), k
