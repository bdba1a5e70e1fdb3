"""The calls by which the speed of this library is measured, over the range of its entry points.

A case is a dict of plain values; `prepare` makes on the GPU what a program has in hand before the call, `run` is one pass
through the entry points of `paper_2605_24058_amd.binding`, `exact` is the same result in 64 bits.  Kinds of pass ("path"):

  forward   one adapted projection: lordba_forward, lordba_forward_multi (ell > 1)
  pool      one projection of a batch that is served by a pool of adapters: lordba_forward_batched(_multi)
  layer     the seven adapted projections of one decoder layer (q, k, v, o, gate, up, down), captured once into a HIP graph
            and replayed, as a serving loop runs its decode or prefill step; adapters > 0: each through a pool
  train     one training step of a projection: sign and pack the latents, forward that keeps t, backward
  train4    the training steps of the four square projections of a layer, captured once into a HIP graph
  ptq       post-training quantisation of one low-rank update into an adapter

Activations and gradients are N(0, 1) in fp16, scales lognormal(-3, 0.5) in fp16, carriers the signs of latents N(0, 1/d): what
the benchmark and the tests of this repository use.  No weights or datasets are involved, only their shapes.
"""
import math

import numpy as np
import torch

from paper_2605_24058_amd import binding

KAPPA = 100.0  # temperature of the smooth sign, as training uses it


# ------------------------------------------------------------------------------------------------ cases ----
def _case(path, T, d_in, d_out, r, ell=1, adapters=0, pattern="none"):
    return dict(path=path, T=T, d_in=d_in, d_out=d_out, r=r, ell=ell, adapters=adapters, pattern=pattern)


def listed():
    return [
        # One token through one projection, called by itself: a first decode step, or a program without graphs.
        dict(_case("forward", 1, 4096, 4096, 16), name="decode_call"),
        # A decode step of eight sequences through a layer with adapters of the highest rank.
        dict(_case("layer", 8, 4096, 11008, 64), name="decode_layer_r64"),
        # A decode step of 64 sequences, each with an adapter of its own out of a resident pool.
        dict(_case("layer", 64, 4096, 11008, 16, adapters=64, pattern="decode"), name="decode_layer_pool"),
        # Prefill of 2048 tokens through a layer at the usual rank.
        dict(_case("layer", 2048, 4096, 11008, 16), name="prefill_layer"),
        # Prefill through the wide projection of a layer with high-rank adapters.
        dict(_case("forward", 4096, 4096, 11008, 64), name="prefill_r64"),
        # Prefill with two scale envelopes per adapter.
        dict(_case("forward", 4096, 4096, 11008, 16, ell=2), name="prefill_two_envelopes"),
        # Prefill of sixteen requests, each with its adapter, in one batch sorted by request.
        dict(_case("pool", 8192, 5120, 5120, 16, adapters=16, pattern="segments"), name="prefill_pool"),
        # A head with an odd number of outputs behind features that are no multiple of 32, at a rank that is no multiple of 16.
        dict(_case("forward", 1500, 1000, 3001, 12), name="odd_sizes"),
        # Training of the square projections of a layer, launch costs taken out by a graph.
        dict(_case("train4", 2048, 4096, 4096, 16), name="train_square"),
        # Training of the largest projection on a long batch.
        dict(_case("train", 8192, 13824, 5120, 16), name="train_large"),
        # Training with two envelopes at rank 32.
        dict(_case("train", 2048, 5120, 5120, 32, ell=2), name="train_two_envelopes"),
        # Quantisation of one fp16 update of rank 16.
        dict(_case("ptq", 0, 4096, 4096, 16), name="ptq"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, odd):
    d = _log_uniform(rng, lo, hi)
    step = rng.choice((128, 128, 32))
    return d if odd else max(step, d // step * step)


_LARGEST = 2 * 8192 * (13824 + 2 * 5120)  # activation bytes of the largest listed projection


def draw(rng):
    path = rng.choice(("forward", "forward", "forward", "pool", "layer", "train", "train", "ptq"))
    if path == "ptq":
        return _case("ptq", 0, _log_uniform(rng, 400, 4096), _log_uniform(rng, 400, 4096), rng.randint(4, 16))
    T = _log_uniform(rng, 1, 8192)
    r = rng.choice((4, 8, 16, 16, 16, 32, 64, rng.randint(1, 64)))
    ell = rng.choice((1, 1, 1, 2, 3, 4)) if path != "layer" else 1
    odd = path != "layer" and rng.random() < 0.25
    if path == "layer":
        d_in, d_out = rng.choice(((2048, 5632), (4096, 11008), (5120, 13824)))
        T = min(T, 2048)
    else:
        d_in, d_out = _width(rng, 512, 13824, odd), _width(rng, 512, 13824, odd)
    adapters, pattern = 0, "none"
    if path == "pool" or (path == "layer" and rng.random() < 0.4):
        pattern = rng.choice(("segments", "decode", "mixed"))
        T = min(T, 256) if pattern == "decode" else T
        adapters = min(rng.choice((2, 8, 16, 64)), 16 if path == "layer" or ell > 1 else 64)
    if odd and path == "train":
        T = min(T, 600)
    if odd:  # these run far from the streams' speed
        T = min(T, 2048)
    T = max(1, min(T, _LARGEST // (2 * ell * (2 if path == "train" else 1) * (d_in + 2 * d_out))))
    return _case(path, T, d_in, d_out, r, ell, adapters, pattern)


def _projections(case):
    """(d_in, d_out) of the projections of one pass."""
    h, f = case["d_in"], case["d_out"]
    if case["path"] == "layer":
        return [(h, h)] * 4 + [(h, f)] * 2 + [(f, h)]
    return [(h, f)] * (4 if case["path"] == "train4" else 1)


# ----------------------------------------------------------------------------------------------- inputs ----
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, dtype=torch.float16, scale=1.0):
    return (torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) * scale).to(dtype)


def _scales(g, shape):
    return torch.exp(0.5 * torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) - 3.0).half()


def _adapter_of_row(g, case):
    T, n, pattern = case["T"], case["adapters"], case["pattern"]
    if pattern == "decode":
        return torch.randint(0, n, (T,), generator=g, device="cuda", dtype=torch.int32)
    cuts = torch.sort(torch.randint(0, T + 1, (n - 1,), generator=g, device="cuda")).values
    ids = torch.searchsorted(cuts, torch.arange(T, device="cuda"), right=True).to(torch.int32)
    if pattern == "mixed":  # one row in eight has no adapter
        ids[torch.rand(T, generator=g, device="cuda") < 0.125] = -1
    return ids


def _inputs(case, seed):
    """The tensors of every projection of a pass, from the seed alone (plain torch)."""
    g = _generator(seed)
    T, r, ell, n, train = case["T"], case["r"], case["ell"], case["adapters"], case["path"].startswith("train")
    lead = ((n,) if n else ()) + ((ell,) if ell > 1 else ())
    out = []
    for d_in, d_out in _projections(case):
        p = {"x": _normal(g, (T, d_in)), "y_base": _normal(g, (T, d_out))}
        stack = (n,) if n else ()
        p["latA"] = _normal(g, stack + (r, d_in), torch.float32, 1 / math.sqrt(d_in))
        p["latB"] = _normal(g, stack + (d_out, r), torch.float32, 1 / math.sqrt(d_out))
        p["s_in"], p["s_rank"], p["s_out"] = (_scales(g, lead + (d,)) for d in (d_in, r, d_out))
        if ell > 1:  # further envelopes partly cancel the first
            flip = torch.randint(0, 2, p["s_rank"].shape, generator=g, device="cuda").half() * 2 - 1
            flip.select(-2, 0).fill_(1)
            p["s_rank"] *= flip
        if n:
            p["ids"] = _adapter_of_row(g, case)
        if train:
            p["g"], p["dx_base"] = _normal(g, (T, d_out)), _normal(g, (T, d_in))
        out.append(p)
    return out


def _ptq_inputs(case, seed):
    """fp16 factors of an update whose singular spectrum decays as a trained one's does."""
    g = _generator(seed)
    r = case["r"]
    damp = 0.85 ** torch.arange(r, device="cuda", dtype=torch.float32)
    a = torch.randn((case["d_in"], r), generator=g, device="cuda") * 0.05 * damp
    b = torch.randn((case["d_out"], r), generator=g, device="cuda") * 0.05
    return a.half(), b.half()


# ----------------------------------------------------------------------------------------------- passes ----
def _forward(p, ell, y_out=None):
    if "ids" in p:
        f = binding.lordba_forward_batched if ell == 1 else binding.lordba_forward_batched_multi
        return f(p["x"], p["pA"], p["pB"], p["s_in"], p["s_rank"], p["s_out"], p["ids"], p["y_base"], y_out=y_out)
    f = binding.lordba_forward if ell == 1 else binding.lordba_forward_multi
    return f(p["x"], p["pA"], p["pB"], p["s_in"], p["s_rank"], p["s_out"], p["y_base"], y_out=y_out)


def _train(p, ell):
    pA, pB, pAt, pBt = binding.lordba_pack_latents(p["latA"], p["latB"])
    scales = (p["s_in"], p["s_rank"], p["s_out"])
    save_t = binding.lordba_forward_save_t if ell == 1 else binding.lordba_forward_multi_save_t
    y, t = save_t(p["x"], pA, pB, *scales, y_base=p["y_base"])
    backward = binding.lordba_backward if ell == 1 else binding.lordba_backward_multi
    grads = backward(p["x"], p["g"], pA, pAt, pBt, *scales, p["latA"], p["latB"], KAPPA, dx_base=p["dx_base"],
                     workspace=p["workspace"], t_saved=t)
    return {"y": y, **grads}


def _captured(state, body):
    """Runs `body` once by itself, then captures it into a HIP graph whose outputs stay where they are."""
    body()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        state["out"] = body()
    state["graph"] = graph


def prepare(case, seed):
    if case["path"] == "ptq":
        a, b = _ptq_inputs(case, seed)
        return {"case": case, "a": a, "b": b}
    ell = case["ell"]
    state = {"case": case, "p": _inputs(case, seed)}
    for p in state["p"]:
        if case["path"].startswith("train"):  # packed anew in every step; the workspace is kept between steps
            size = (case["T"], p["x"].shape[1], p["g"].shape[1], case["r"])
            need = (binding.lordba_backward_workspace_bytes(*size) if ell == 1
                    else binding.lordba_backward_multi_workspace_bytes(*size, ell))
            p["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
            continue
        if case["adapters"]:
            packed = [binding.lordba_pack_latents(a, b, transposed=False)[:2] for a, b in zip(p["latA"], p["latB"])]
            p["pA"], p["pB"] = (torch.stack(w) for w in zip(*packed))
        else:
            p["pA"], p["pB"] = binding.lordba_pack_latents(p["latA"], p["latB"], transposed=False)[:2]
        del p["latA"], p["latB"]  # a serving program holds the packed carriers only
    if case["path"] == "layer":
        outs = [torch.empty_like(p["y_base"]) for p in state["p"]]
        _captured(state, lambda: [_forward(p, ell, y) for p, y in zip(state["p"], outs)])
    elif case["path"] == "train4":
        _captured(state, lambda: [_train(p, ell) for p in state["p"]])
    return state


def run(state):
    case = state["case"]
    if "graph" in state:
        state["graph"].replay()
        return state["out"]
    if case["path"] == "ptq":
        out = binding.lordba_ptq(state["a"], state["b"], case["r"])
        return {k: v for k, v in out.items() if k != "workspace"}
    return (_train if case["path"] == "train" else _forward)(state["p"][0], case["ell"])


# ---------------------------------------------------------------------------------------- what is needed ----
def work(case):
    T, r, ell, n = case["T"], case["r"], case["ell"], max(case["adapters"], 1)
    if case["path"] == "ptq":
        N, M = case["d_in"], case["d_out"]
        outputs = (N + M) * (8 + 2 + r * 8) + r * (N + M) / 8  # scales in 64 and 16 bits, iterates, carriers
        # about twenty sweeps, each with two solves of an r x r system per row, their right-hand sides and Gram matrices
        return {"bytes": 2 * r * (N + M) + outputs, "flops": 20.0 * (N + M) * (r ** 3 / 3 + 14 * r * r)}
    total, flops = 0, 0
    for d_in, d_out in _projections(case):
        n_used = min(n, T)
        carriers, scales = r * (d_in + d_out) / 8, 2 * ell * (d_in + r + d_out)
        total += 2 * T * (d_in + 2 * d_out) + n_used * scales
        flops += 2 * T * r * ell * (d_in + d_out)
        if case["path"].startswith("train"):  # latents in and gradients out; g, dx_base, dx
            total += 8 * r * (d_in + d_out) + 4 * ell * (d_in + r + d_out) + 2 * T * (d_out + 2 * d_in)
            flops += 4 * T * r * ell * (d_in + d_out)
        else:
            total += n_used * carriers + (4 * T if case["adapters"] else 0)
    return {"bytes": total, "flops": flops}


def tolerance(case):
    if case["path"] == "ptq":  # 64-bit arithmetic whose decisions (signs, number of sweeps) are the same in any order of sums
        return {"rel": 1e-8, "max": 1e-6, "differ": 0.0}
    # fp16 results with one rounding: 2.2e-4 against the exact result (2-norm), half a unit in the last place at most
    return {"rel": 9e-4, "max": 2e-3}


# -------------------------------------------------------------------------------------- exact, in 64 bits ----
def _sign(latent):
    return torch.where(latent < 0, -1.0, 1.0).double()


def _branch(x, SA, SB, s_in, s_rank, s_out):
    return ((x * s_in) @ SA.t() * s_rank) @ SB.t() * s_out


def _exact_forward(p, ell):
    x, y = p["x"].double(), p["y_base"].double()
    many = lambda s: s.double().reshape(ell, -1)
    if "ids" in p:
        for a in range(p["latA"].shape[0]):
            rows = torch.nonzero(p["ids"] == a).squeeze(1)
            if rows.numel():
                SA, SB = _sign(p["latA"][a]), _sign(p["latB"][a])
                for s in zip(many(p["s_in"][a]), many(p["s_rank"][a]), many(p["s_out"][a])):
                    y[rows] += _branch(x[rows], SA, SB, *s)
        return y
    SA, SB = _sign(p["latA"]), _sign(p["latB"])
    for s in zip(many(p["s_in"]), many(p["s_rank"]), many(p["s_out"])):
        y += _branch(x, SA, SB, *s)
    return y


def _exact_train(p, ell):
    x, g, dx = p["x"].double(), p["g"].double(), p["dx_base"].double()
    latA, latB = p["latA"].double(), p["latB"].double()
    SA, SB = _sign(p["latA"]), _sign(p["latB"])
    smooth = lambda u: KAPPA / torch.cosh(KAPPA * u) ** 2
    d_in_s, d_rank_s, d_out_s = [], [], []
    dA, dB = torch.zeros_like(latA), torch.zeros_like(latB)
    for e in range(ell):
        si, sr, so = (p[k].double().reshape(ell, -1)[e] for k in ("s_in", "s_rank", "s_out"))
        t, du = (x * si) @ SA.t(), (g * so) @ SB
        dx += (du * sr) @ SA * si
        Q, P = (du * sr).t() @ x, (t * sr).t() @ g  # [r, d_in], [r, d_out]
        d_in_s.append((SA * Q).sum(0))
        d_out_s.append((SB.t() * P).sum(0))
        d_rank_s.append((du * t).sum(0))
        dA += si * Q
        dB += (so * P).t()
    pick = lambda v: v[0] if ell == 1 else torch.stack(v)
    return {"y": _exact_forward(p, ell), "dx": dx, "d_s_in": pick(d_in_s), "d_s_rank": pick(d_rank_s), "d_s_out": pick(d_out_s),
            "d_latentA": dA * smooth(latA), "d_latentB": dB * smooth(latB)}


def _exact_ptq(case, seed, K=100, tau=2.0, mu=10.0):
    """The consensus ADMM on the factors of the update; carriers and iterates are defined up to the signs of their pairs, so
    only the scales are given."""
    A, B = (v.double().cpu().numpy() for v in _ptq_inputs(case, seed))
    r = case["r"]
    sgn = lambda v: np.where(v < 0, -1.0, 1.0)
    (Qa, Ra), (Qb, Rb) = np.linalg.qr(A), np.linalg.qr(B)
    u, s, vt = np.linalg.svd(Ra @ Rb.T)
    U1, U2 = sgn(Qa @ u[:, :r]), sgn(vt[:r] @ Qb.T)  # [N, r], [r, M]
    beta, gamma = s[:r].copy(), np.ones(B.shape[0])

    def ratio(num, den):
        return np.where(den > 0, num / np.where(den > 0, den, 1.0), 0.0)

    def alpha_of():
        C = beta[:, None] * U2 * gamma
        return ratio(((A @ (B.T @ C.T)) * U1).sum(1), ((U1 @ (C @ C.T)) * U1).sum(1))

    def gamma_of():
        C = alpha[:, None] * U1 * beta
        return ratio(((C.T @ A) @ B.T * U2).sum(0), ((C.T @ C) @ U2 * U2).sum(0))

    alpha = alpha_of()
    gamma = gamma_of()
    M1, M2, Y1, Y2 = U1.copy(), U2.copy(), np.zeros_like(U1), np.zeros_like(U2)
    n1, n2 = U1.size, U2.size
    rho = float(((A.T @ A) * (B.T @ B)).sum()) / (n1 + n2)
    eye = np.eye(r)
    for t in range(K):
        C = beta[:, None] * U2 * gamma
        H = (alpha ** 2)[:, None, None] * (C @ C.T) + rho / n1 * eye
        U1 = np.linalg.solve(H, (alpha[:, None] * (A @ (B.T @ C.T)) + rho / n1 * (M1 - Y1))[..., None])[..., 0]
        C = alpha[:, None] * U1 * beta
        H = (gamma ** 2)[:, None, None] * (C.T @ C) + rho / n2 * eye
        U2 = np.linalg.solve(H, (gamma * ((C.T @ A) @ B.T) + rho / n2 * (M2 - Y2)).T[..., None])[..., 0].T
        alpha = alpha_of()
        gamma = gamma_of()
        P, Q = alpha[:, None] * U1, U2 * gamma
        beta = np.linalg.pinv((P.T @ P) * (Q @ Q.T), hermitian=True) @ (((P.T @ A) * (Q @ B)).sum(1))
        N1, N2 = sgn(U1 + Y1), sgn(U2 + Y2)
        Y1, Y2 = Y1 + U1 - N1, Y2 + U2 - N2
        same = np.array_equal(N1, M1) and np.array_equal(N2, M2)
        if 2 * t < K:
            primal = math.sqrt(((U1 - N1) ** 2).sum() + ((U2 - N2) ** 2).sum())
            dual = math.sqrt((rho / n1) ** 2 * ((N1 - M1) ** 2).sum() + (rho / n2) ** 2 * ((N2 - M2) ** 2).sum())
            f = tau if primal > mu * dual else 1 / tau if dual > mu * primal else 1.0
            rho, Y1, Y2 = rho * f, Y1 / f, Y2 / f
        M1, M2 = N1, N2
        if same:
            break
    return {"packedA": None, "packedB": None, "alpha": alpha, "beta": beta, "gamma": gamma, "s_in": alpha, "s_rank": beta,
            "s_out": gamma, "info": None, "U1": None, "U2t": None}


def exact(case, seed):
    if case["path"] == "ptq":
        return _exact_ptq(case, seed)
    one = _exact_train if case["path"].startswith("train") else _exact_forward
    outs = [one(p, case["ell"]) for p in _inputs(case, seed)]
    return outs if case["path"] in ("layer", "train4") else outs[0]
