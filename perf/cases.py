"""What a program does with this library, as cases that can be timed and compared.

Online: the linear layers of a pruned model, from one token (decoding) over small batches to prompts of a few
thousand tokens, with 2:4 and 4:8 weights, the dense product of a layer that was left unpruned, and several
layers that read the same hidden state in one call.  Offline: pruning one matrix (from calibration features, or
with channel scores that the program has already) and compressing it.

Every product goes through the library's own choice of kernel (variant -1) without a search before it, as a
program that loads a model and serves it does.  Shapes are those of the workloads in workloads.py, ragged ones
beside them; weights are N(0, K^-1/2) and activations normal with a log-normal scale per channel and a few
outlier channels, as that module makes them.
"""
import math

import numpy as np
import torch

import paper_2310_15929_amd as esp

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


# ---- the cases ------------------------------------------------------------------------------------
def listed():
    return [
        # smallest call: one 512 x 512 layer on 16 tokens (launches and staging count, nothing else)
        dict(name="small_linear", kind="spmm", M=16, N=512, K=512, n=2, m=4, dtype="f16"),
        # decoding one sequence: q, k and v of a 7B layer in one call
        dict(name="decode_qkv", kind="group", count=3, M=1, N=4096, K=4096, n=2, m=4, dtype="f16"),
        # decoding eight sequences: the seven linears of a 7B layer (q/k/v and gate/up as groups)
        dict(name="decode_layer", kind="layer", M=8, H=4096, F=11008, n=2, m=4, dtype="f16"),
        # a large decoding batch on the gate matrix of a 65B layer
        dict(name="decode_batch", kind="spmm", M=128, N=22016, K=8192, n=2, m=4, dtype="bf16"),
        # decoding 16 sequences with the less restrictive pattern
        dict(name="decode_4_8", kind="spmm", M=16, N=9216, K=9216, n=4, m=8, dtype="f16"),
        # a short prompt through a layer whose sizes are no multiple of any tile
        dict(name="prompt_ragged", kind="spmm", M=333, N=5003, K=3020, n=2, m=4, dtype="bf16"),
        # a long prompt through the gate matrix of a 13B layer
        dict(name="prefill", kind="spmm", M=2048, N=13824, K=5120, n=2, m=4, dtype="f16"),
        # a prompt through a 4:8 layer
        dict(name="prefill_4_8", kind="spmm", M=512, N=5120, K=13824, n=4, m=8, dtype="bf16"),
        # a prompt through a layer that was left dense
        dict(name="prompt_dense", kind="dense", M=512, N=5120, K=5120, dtype="f16"),
        # offline: one 7B attention matrix pruned from 128 x 2048 calibration tokens
        dict(name="prune_layer", kind="prune", T=262144, N=4096, K=4096, block=64, n=2, m=4, dtype="f16", scores=False),
        # offline: a 13B matrix pruned to 4:8, the channel scores at hand (layers that share an input share them)
        dict(name="prune_4_8", kind="prune", T=0, N=5120, K=5120, block=64, n=4, m=8, dtype="bf16", scores=True),
        # offline: compression of a pruned 7B gate matrix, canonical and kernel-native form
        dict(name="compress", kind="compress", N=11008, K=4096, n=2, m=4, dtype="f16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, ragged_to):
    """A layer size: half the time a multiple of 256, else one of `ragged_to` only."""
    v = _log_int(rng, lo, hi)
    q = 256 if rng.random() < 0.5 else ragged_to
    return max(q, v // q * q)


def draw(rng):
    kind = rng.choice(["spmm", "spmm", "spmm", "spmm", "group", "layer", "dense", "prune", "prune", "compress"])
    n, m = (4, 8) if rng.random() < 0.25 else (2, 4)
    dtype = rng.choice(["f16", "bf16"])
    if kind == "spmm":
        M = _log_int(rng, 1, 2048)
        N, K = _size(rng, 512, 22016, 1), _size(rng, 512, 13824, m)
        while 2 * M * N * K > 2 * 2048 * 13824 * 5120:
            N = max(512, N // 2)
        return dict(kind=kind, M=M, N=N, K=K, n=n, m=m, dtype=dtype)
    if kind == "group":
        return dict(kind=kind, count=rng.choice([2, 3, 4]), M=_log_int(rng, 1, 64), N=_size(rng, 1024, 11008, 1),
                    K=_size(rng, 1024, 8192, m), n=n, m=m, dtype=dtype)
    if kind == "layer":
        H = 256 * rng.randint(4, 20)
        return dict(kind=kind, M=_log_int(rng, 1, 64), H=H, F=_size(rng, 2 * H, 3 * H, 16), n=n, m=m, dtype=dtype)
    if kind == "dense":
        return dict(kind=kind, M=_log_int(rng, 1, 1024), N=_size(rng, 512, 13824, 1), K=_size(rng, 512, 8192, 4), dtype=dtype)
    if kind == "prune":
        block, scores = rng.choice([32, 64]), rng.random() < 0.3
        return dict(kind=kind, T=0 if scores else _log_int(rng, 2048, 262144), N=_size(rng, 1024, 4096, 1),
                    K=block * rng.randint(1024 // block, 4096 // block), block=block, n=n, m=m, dtype=dtype, scores=scores)
    return dict(kind=kind, N=_size(rng, 1024, 13824, 1), K=_size(rng, 1024, 13824, m), n=n, m=m, dtype=dtype)


# ---- inputs ---------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _weights(g, N, K, dtype):
    return (torch.randn(N, K, device="cuda", generator=g) * K ** -0.5).to(dtype)


def _channel_scales(g, K):
    s = torch.exp(torch.randn(K, device="cuda", generator=g))
    few = torch.randperm(K, device="cuda", generator=g)[: max(1, round(0.005 * K))]
    s[few] *= 30.0
    return s


def _features(g, T, K, dtype):
    s = _channel_scales(g, K)
    out = torch.empty(T, K, dtype=dtype, device="cuda")
    for lo in range(0, T, 32768):
        hi = min(T, lo + 32768)
        out[lo:hi] = (torch.randn(hi - lo, K, device="cuda", generator=g) * s).clamp_(-60000, 60000).to(dtype)
    return out


def _perm(g, K):
    return torch.randperm(K, device="cuda", generator=g).to(torch.int32)


def _mask(W, perm, n, m):
    """The n largest magnitudes of every m re-ordered channels, one byte per weight in re-ordered order."""
    a = W[:, perm.long()].abs().reshape(W.shape[0], -1, m)
    kept = torch.zeros(a.shape, dtype=torch.uint8, device="cuda")
    kept.scatter_(2, torch.argsort(a, dim=2, descending=True, stable=True)[:, :, :n], 1)
    return kept.reshape(W.shape)


def _matrices(case):
    """(N, K) of each weight matrix, grouped by call; the members of a call share their input."""
    if case["kind"] == "layer":
        H, F = case["H"], case["F"]
        return [[(H, H)] * 3, [(H, H)], [(F, H)] * 2, [(H, F)]]
    return [[(case["N"], case["K"])] * case.get("count", 1)]


def _linear_inputs(case, seed):
    """Per call: X, and (W, perm, mask) of each member."""
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    calls = []
    for shapes in _matrices(case):
        X = _features(g, case["M"], shapes[0][1], dt)
        members = []
        for N, K in shapes:
            W, perm = _weights(g, N, K, dt), _perm(g, K)
            members.append((W, perm, _mask(W, perm, case["n"], case["m"])))
        calls.append((X, members))
    return calls


def _prune_inputs(case, seed):
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    W = _weights(g, case["N"], case["K"], dt)
    if case["scores"]:
        s = _channel_scales(g, case["K"]).double().cpu().numpy()
        return W, None, 2.5 + s
    return W, _features(g, case["T"], case["K"], dt), None


def prepare(case, seed):
    kind = case["kind"]
    state = dict(kind=kind, ctx=esp.Context(0))
    if kind in ("spmm", "group", "layer"):
        calls = []
        for X, members in _linear_inputs(case, seed):
            comps = [state["ctx"].compress(W, mask, perm, case["n"], case["m"], canonical=False) for W, perm, mask in members]
            calls.append((X, comps, [perm for _, perm, _ in members]))
        state["calls"] = calls
    elif kind == "dense":
        g, dt = _gen(seed), DTYPES[case["dtype"]]
        state["X"] = _features(g, case["M"], case["K"], dt)
        state["N"] = case["N"]
        state["packed"] = state["ctx"].dense_pack(_weights(g, case["N"], case["K"], dt))
    elif kind == "prune":
        state["W"], state["calib"], state["score"] = _prune_inputs(case, seed)
        alpha = 1.0 / math.sqrt(case["T"]) if case["T"] else 1.0
        state["opts"] = esp.PruneOpts(n_keep=case["n"], m_group=case["m"], block=case["block"], bins=100, alpha=alpha)
    else:
        g = _gen(seed)
        W = _weights(g, case["N"], case["K"], DTYPES[case["dtype"]])
        perm = _perm(g, case["K"])
        state.update(W=W, perm=perm, mask=_mask(W, perm, case["n"], case["m"]), n=case["n"], m=case["m"])
    return state


def run(state):
    ctx, kind = state["ctx"], state["kind"]
    if kind in ("spmm", "group", "layer"):
        outs = []
        for X, comps, perms in state["calls"]:
            if len(comps) == 1:
                outs.append(ctx.spmm(X, comps[0], perms[0]))
            else:
                outs.extend(ctx.spmm_group([X] * len(comps), comps, perms))
        return outs
    if kind == "dense":
        return ctx.dense_gemm(state["X"], state["packed"], state["N"])
    if kind == "prune":
        r = ctx.prune(state["calib"], state["W"], state["opts"], score=state["score"], want_retained=True)
        return dict(perm=r.perm, mask=r.mask, score=r.score, swaps=r.swaps, retained=r.retained)
    c = ctx.compress(state["W"], state["mask"], state["perm"], state["n"], state["m"])
    return dict(values=c.values, meta=c.meta, native=c.native)


# ---- what a pass cannot do without ----------------------------------------------------------------
def work(case):
    kind = case["kind"]
    if kind in ("spmm", "group", "layer"):
        M, by, fl = case["M"], 0, 0
        for shapes in _matrices(case):
            by += 2 * M * shapes[0][1]
            for N, K in shapes:
                # kept values (half of 2 bytes) and 2 bits of index for each, the permutation, the output
                by += N * K + N * K // 8 + 4 * K + 2 * M * N
                fl += M * N * K  # 2 M N K over the kept half
        return {"bytes": by, "flops": fl}
    N, K = case["N"], case["K"]
    if kind == "dense":
        return {"bytes": 2 * (N * K + case["M"] * (N + K)), "flops": 2 * case["M"] * N * K}
    if kind == "prune":
        # features and weights read, mask and permutation written; the first table of a block's exchanges:
        # every group with each member replaced by each channel of the block, four operations a row
        return {"bytes": 2 * case["T"] * K + 3 * N * K + 4 * K, "flops": 4 * N * K * case["block"]}
    # weights, mask, permutation read; kept values and indices written in both forms
    return {"bytes": 3 * N * K + 4 * K + 2 * (N * K + N * K // 8), "flops": 0}


def tolerance(case):
    kind = case["kind"]
    if kind in ("spmm", "group", "layer", "dense"):
        # fp32 sums rounded once to 16 bits: half a unit in the last place, 2^-12 / 2^-9 of a value at most
        return {"rel": 8e-4, "max": 4e-3} if case["dtype"] == "f16" else {"rel": 7e-3, "max": 3e-2}
    if kind == "prune":
        # permutation, mask and exchange counts the same; the retained metric is a float64 sum whose order is free
        return {"rel": 1e-12, "max": 1e-12}
    return "exact"


# ---- the same in 64 bits --------------------------------------------------------------------------
def _scores(calib, bins, alpha):
    T, K = calib.shape
    out = np.empty(K)
    for lo in range(0, K, 64):
        x = calib[:, lo:lo + 64].double()
        c = x.shape[1]
        low, high = x.amin(0), x.amax(0)
        b = torch.floor((x - low) * bins / (high - low)).clamp_(max=bins - 1).long()
        b += torch.arange(c, device="cuda") * bins
        p = torch.bincount(b.flatten(), minlength=c * bins).reshape(c, bins).double() / T
        ent = -torch.special.xlogy(p, p).sum(1)
        out[lo:lo + 64] = (ent + alpha * x.square().sum(0).sqrt()).cpu().numpy()
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("spmm", "group", "layer"):
        outs = []
        for X, members in _linear_inputs(case, seed):
            for W, perm, mask in members:
                order = perm.long()
                outs.append(X.double()[:, order] @ (W[:, order] * mask).double().t())
        return outs
    if kind == "dense":
        g, dt = _gen(seed), DTYPES[case["dtype"]]
        X = _features(g, case["M"], case["K"], dt)
        return X.double() @ _weights(g, case["N"], case["K"], dt).double().t()
    if kind == "prune":
        # the exchanges are a greedy search: integers, compared as such; the scores are computed numbers
        _, calib, score = _prune_inputs(case, seed)
        if calib is not None:
            score = _scores(calib, 100, 1.0 / math.sqrt(case["T"]))
        return dict(perm=None, mask=None, score=score, swaps=None, retained=None)
    return None
