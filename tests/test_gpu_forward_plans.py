"""GPU parity of the plans that the forward dispatch chooses between for few tiles, wide inputs and narrow outputs, against the
fp64 oracle: per token row ||y_gpu - y||_2 / ||y||_2 <= 1e-3, also with y_base = 0, and nothing written outside y_out."""
import numpy as np
import pytest

import oracle
from paper_2605_24058_amd import binding, inputs

pytestmark = pytest.mark.gpu

TOL = 1e-3


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    binding.load_library()
    return torch


def guarded(torch, T, d_out):
    """An output whose surroundings are NaN, 16-byte aligned."""
    big = torch.full((T * d_out + 128,), float("nan"), dtype=torch.float16, device="cuda:0")
    return big, big[64:64 + T * d_out].view(T, d_out)


def check(torch, call, want, T, d_out, label):
    big, out = guarded(torch, T, d_out)
    call(out)
    torch.cuda.synchronize()
    around = big.cpu().numpy()
    assert np.isnan(around[:64]).all() and np.isnan(around[64 + T * d_out:]).all(), (label, "write outside y_out")
    err = oracle.row_rel_l2(out.cpu().numpy().astype(np.float64), want).max()
    assert err <= TOL, (label, err)


# (T, d_in, d_out, r, envelopes), each with a ragged last tile or a ragged last chunk somewhere in its group
PLANS = [
    # twelve x slots per wave on 8 waves (three and four rank blocks, whole and ragged carrier words), and the loop beside them
    (9, 11008, 640, 48, 1), (8, 11008, 4096, 64, 1), (11, 9760, 512, 50, 1), (10, 9760, 384, 41, 1), (300, 12288, 1024, 64, 1),
    (9, 8480, 512, 64, 1), (9, 8320, 256, 64, 1), (9, 8480, 256, 48, 1),
    # fourteen slots on 8 waves and seven on 16 (97 to 112 chunks, the last one whole or ragged; on 8 waves 97 only where it is whole), and the
    # loop from 113 chunks on
    (9, 12416, 640, 48, 1), (1, 12416, 512, 64, 1), (8, 12384, 520, 41, 1),
    (9, 12320, 640, 48, 1), (8, 13824, 5120, 64, 1), (1, 14336, 136, 41, 1), (300, 14336, 520, 64, 1), (9, 14368, 512, 64, 1),
    (9, 12320, 640, 16, 1), (8, 13824, 5120, 32, 1), (1, 14336, 136, 12, 1), (300, 14304, 520, 24, 1), (9, 14368, 512, 16, 1),
    # every wave with two chunks on 16 waves, with and without a chip full of workgroups, and one wave short of it
    (2040, 4096, 264, 16, 1), (1601, 4096, 264, 8, 1), (2040, 3968, 264, 16, 1), (2040, 4064, 264, 30, 1),
    # eight slots, and the loop
    (9, 4640, 640, 48, 1), (8, 5120, 4096, 64, 1), (13, 8192, 136, 57, 1), (1000, 4608, 512, 33, 1), (9, 4480, 256, 48, 1), (9, 4256, 512, 64, 1),
    # six slots on 16 waves, and the loop
    (9, 9760, 640, 16, 1), (300, 11008, 512, 12, 1), (9, 8480, 512, 32, 1), (9, 9600, 512, 16, 1), (9, 8352, 512, 8, 1),
    # a tile's blocks split over workgroups with more than one block per wave, on 16 and on 8 waves; all of them in one workgroup
    (264, 96, 11008, 16, 1), (401, 160, 4096, 16, 1), (643, 96, 2048, 16, 1), (1, 160, 28680, 16, 1),
    (601, 512, 11008, 16, 1), (1000, 512, 4224, 64, 1), (601, 96, 11008, 33, 1), (1021, 160, 4168, 24, 1), (1029, 512, 4224, 64, 1),
    # fewer blocks than waves at three and four rank blocks behind few chunks
    (8, 512, 512, 64, 1), (3, 128, 5120, 48, 1), (16, 256, 1032, 33, 1), (1, 64, 128, 64, 1),
    # a general rank on more than 128 tiles: up to one block per wave (16 and 8 waves), and one block more
    (1031, 96, 2048, 2, 1), (1030, 96, 2056, 20, 1), (2055, 160, 1024, 30, 1), (2051, 160, 1032, 50, 1), (5001, 96, 1000, 12, 1),
    # three slots on 16 waves and six on 8 (40 to 48 chunks, the last one whole or ragged), and the plans beside them
    (1033, 5120, 512, 16, 1), (2047, 6144, 264, 8, 1), (1033, 5088, 2056, 12, 1), (2049, 5120, 136, 32, 1), (1029, 6144, 1032, 50, 1),
    (1027, 5088, 512, 64, 1), (2051, 5120, 512, 20, 1), (1025, 4992, 512, 32, 1), (1030, 6176, 512, 48, 1),
    # two envelopes on 16 waves, and on 8 beyond one tile per compute unit and beyond four chunks per wave
    (1033, 3072, 3080, 30, 2), (2048, 3104, 3072, 16, 2), (1025, 5120, 3072, 32, 2), (2049, 3072, 3072, 32, 2),
    (1027, 8192, 3072, 20, 2), (1029, 8224, 3080, 32, 2), (1026, 8352, 3080, 5, 2),
    # several envelopes at a general rank: up to one block per wave, and one block more
    (1100, 256, 256, 30, 3), (1031, 96, 1024, 2, 4), (1029, 160, 1032, 20, 3), (5, 160, 136, 30, 4), (1027, 64, 72, 1, 3), (300, 256, 2056, 44, 3),
]


@pytest.mark.parametrize("plan", PLANS, ids=lambda s: "T%d_%dx%d_r%d_ell%d" % s)
def test_plan(torch_cuda, plan):
    torch = torch_cuda
    T, d_in, d_out, r, ell = plan
    d = inputs.make_inputs_multi(51, T, d_in, d_out, r, ell)
    if d_in < 256:  # with few input channels the branch alone would land among the subnormals of fp16
        d["s_out"] = (d["s_out"].astype(np.float32) * 2.0 ** 8).astype(np.float16)
    dev = binding.to_device(d)
    args = [dev[k] for k in ("x", "packedA", "packedB", "s_in", "s_rank", "s_out")]
    for base in (d["y_base"], np.zeros_like(d["y_base"])):
        want = oracle.forward_multi(d["x"], d["signsA"], d["signsB"], d["s_in"], d["s_rank"], d["s_out"], base, nthreads=8)
        yb = torch.from_numpy(base).cuda()
        check(torch, lambda out: binding.lordba_forward_multi(*args, yb, y_out=out), want, T, d_out, plan)
    # the training forward keeps t, and a call for t alone gives the same (no block is then split)
    y, t = binding.lordba_forward_multi_save_t(*args, y_base=dev["y_base"])
    _, t_only = binding.lordba_forward_multi_save_t(*args)
    torch.cuda.synchronize()
    want = oracle.forward_multi(d["x"], d["signsA"], d["signsB"], d["s_in"], d["s_rank"], d["s_out"], d["y_base"], nthreads=8)
    assert oracle.row_rel_l2(y.cpu().numpy().astype(np.float64), want).max() <= TOL
    t, t_only = t.cpu().numpy(), t_only.cpu().numpy()
    for e in range(ell):
        assert oracle.rel_l2(t[e, :, :T].T, oracle.rank_intermediate(d["x"], d["signsA"], d["s_in"][e])) <= 1e-5
    assert np.array_equal(t[:, :, :T], t_only[:, :, :T])


# (T, d_in, d_out, r, adapters, pattern): the six-slot kernel and the loop on pools; pools of odd widths with a workgroup per run
# (up to 128 tiles) and with two workgroups per tile, every row its own run, few runs, rows without an adapter
POOLS = [
    (61, 11008, 640, 16, 3, "decode"), (61, 11008, 640, 16, 3, "mixed"), (61, 11008, 512, 16, 3, "decode"), (9, 9760, 1024, 8, 2, "mixed"),
    (250, 12288, 1152, 16, 4, "segments"),
    (61, 13824, 640, 16, 3, "decode"), (9, 12320, 1024, 8, 2, "mixed"), (61, 14336, 512, 32, 3, "mixed"), (9, 14368, 512, 16, 2, "decode"),
    (289, 353, 140, 2, 16, "decode"), (1021, 99, 77, 17, 5, "decode"), (300, 130, 205, 40, 3, "mixed"), (1030, 99, 77, 17, 5, "decode"),
    (1033, 353, 140, 8, 4, "segments"),
]


@pytest.mark.parametrize("case", POOLS, ids=lambda c: "T%d_%dx%d_r%d_n%d_%s" % c)
def test_pool_plan(torch_cuda, case):
    torch = torch_cuda
    T, d_in, d_out, r, n, pattern = case
    d = inputs.make_adapter_pool(52, d_in, d_out, r, n)
    d.update(inputs.make_activations(52, T, d_in, d_out))
    if d_in < 256:
        d["s_out"] = (d["s_out"].astype(np.float32) * 2.0 ** 8).astype(np.float16)
    ids = inputs.make_adapter_ids(52, T, n, pattern)
    packed = [binding.lordba_pack_signs(a, b) for a, b in zip(d["signsA"], d["signsB"])]
    cu = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    pool = [cu(np.stack([p[k] for p in packed]).view(np.int32)) for k in (0, 1)]
    args = [cu(d["x"])] + pool + [cu(d[k]) for k in ("s_in", "s_rank", "s_out")] + [cu(ids)]
    want = oracle.forward_batched(d["x"], d["signsA"], d["signsB"], d["s_in"], d["s_rank"], d["s_out"], ids, d["y_base"])
    yb = cu(d["y_base"])
    check(torch, lambda out: binding.lordba_forward_batched(*args, yb, y_out=out), want, T, d_out, case)
