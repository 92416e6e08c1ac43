"""GPU parity: every stage of the HIP path against the CPU oracle, through the C ABI.

Bar: permutation, mask, statistics, compressed values and metadata bit-exact; products within a
normwise relative error per output row of 2e-3 (fp16) / 1e-2 (bf16).
"""
import ctypes as C
import hashlib
import json
import math
import os

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import esparse_oracle as orc

pytestmark = pytest.mark.gpu

TOL = {torch.float16: 2e-3, torch.bfloat16: 1e-2}


@pytest.fixture(scope="module")
def esp():
    import paper_2310_15929_amd as esp
    esp.load_library()
    return esp


@pytest.fixture(scope="module")
def ctx(esp):
    assert torch.cuda.is_available()
    return esp.Context(0)


def _np(t: torch.Tensor) -> np.ndarray:
    t = t.detach().cpu()
    if t.dtype == torch.bfloat16:
        return t.float().numpy()
    return t.numpy()


def _bits(t: torch.Tensor) -> np.ndarray:
    return t.detach().cpu().contiguous().view(torch.int16).numpy().view(np.uint16)


def _rand(shape, dtype, seed, scale=1.0, col_scale=None):
    return wl.normal_matrix(shape[0], shape[1], wl.stream_id("test", seed), scale=scale, col_scale=col_scale,
                            dtype=dtype)


def _sha(a):
    return hashlib.sha256(np.ascontiguousarray(a).tobytes()).hexdigest()


# ---------------------------------------------------------------- channel statistics
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("T,K", [(256, 512), (1000, 70), (37, 2)])
def test_channel_stats_bit_exact(ctx, dtype, T, K):
    scales = np.exp(np.random.default_rng(T + K).standard_normal(K) * 2.0)
    Xc = _rand((T, K), dtype, 11, col_scale=scales)
    if K >= 4:
        Xc[:, 1] = 0.75          # constant channel
        Xc[:, 3] = 0.0           # all-zero channel
    print(f"stats T={T} K={K} {dtype}", flush=True)
    ir, am = ctx.channel_stats(Xc.cuda(), 100)
    x = _np(Xc)
    assert (ir == orc.channel_entropy(x, 100)).all()
    assert (am == orc.channel_amplitude(x)).all()


def test_channel_stats_other_bin_counts(ctx):
    Xc = _rand((512, 16), torch.float16, 12)
    for bins in (1, 7, 256):
        ir, _ = ctx.channel_stats(Xc.cuda(), bins)
        assert (ir == orc.channel_entropy(_np(Xc), bins)).all()


# several channels' bins to a wave, with lanes left over, up to one channel to a wave; channels that end within a workgroup and within a wave's share
@pytest.mark.parametrize("K", [300, 302])
def test_channel_stats_few_bins_of_many_channels(ctx, K):
    Xc = _rand((600, K), torch.float16, 13)
    for bins in (2, 3, 10, 30, 32, 33, 63, 64, 65):
        ir, _ = ctx.channel_stats(Xc.cuda(), bins)
        assert (ir == orc.channel_entropy(_np(Xc), bins)).all(), bins


# every value on the edge of a bin, and one unit beside it
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("bins", [1, 64, 100, 256])
def test_channel_entropy_values_on_bin_edges(ctx, dtype, bins):
    g = torch.Generator().manual_seed(bins)
    x = torch.randint(0, bins + 1, (700, 24), generator=g).float()
    x[:, 8:16] += 1.0 / 64 * torch.randint(-1, 2, (700, 8), generator=g)
    x[:, 16:] = x[:, 16:] * 0.37 - 11.0
    Xc = x.to(dtype)
    ir, _ = ctx.channel_stats(Xc.cuda(), bins)
    assert (ir == orc.channel_entropy(_np(Xc), bins)).all()


# so many channels that a lane adds up more than 256 rows: the largest and the smallest squares, alone and together
def test_channel_amplitude_many_rows_per_lane(ctx):
    T, K = 9000, 131072
    Xc = torch.empty(T, K, dtype=torch.float16, device="cuda").normal_(generator=torch.Generator(device="cuda").manual_seed(1))
    tiny = 2.0 ** -24
    cols = {0: torch.full((T,), 65504.0), 5: torch.full((T,), tiny), 130: torch.where(torch.arange(T) % 3 == 0, 65504.0, tiny),
            131071: torch.where(torch.arange(T) % 2 == 0, -0.015625, 3 * tiny)}
    for c, v in cols.items():
        Xc[:, c] = v.to(torch.float16).cuda()
    _, am = ctx.channel_stats(Xc, 10)
    pick = list(cols) + [1, 2, 77777]
    assert (am[pick] == orc.channel_amplitude(_np(Xc[:, pick].cpu()))).all()


# ---------------------------------------------------------------- prune
def _prune_case(esp, ctx, N, K, T, B, n, m, dtype, flags, seed, max_swaps=0):
    scales = wl.channel_scales("lognormal", K, wl.stream_id("ps", seed))
    W = _rand((N, K), dtype, seed, scale=K ** -0.5)
    Xc = _rand((T, K), dtype, seed + 1, col_scale=scales)
    alpha = wl.default_alpha(T)
    opts = esp.PruneOpts(n_keep=n, m_group=m, block=B, bins=100, alpha=alpha, flags=flags, max_swaps=max_swaps)
    print(f"prune N={N} K={K} T={T} B={B} {n}:{m} {dtype} flags={flags} max_swaps={max_swaps}", flush=True)
    res = ctx.prune(Xc.cuda(), W.cuda(), opts, want_retained=True)
    torch.cuda.synchronize()
    theta, mask, s, swaps = orc.prune(_np(Xc), _np(W), n, m, B, alpha, 100,
                                      use_entropy=bool(flags & esp.USE_ENTROPY), use_norm=bool(flags & esp.USE_NORM),
                                      use_gns=bool(flags & esp.USE_GNS), use_lbs=bool(flags & esp.USE_LBS),
                                      max_swaps=max_swaps)
    assert (res.score == s).all(), "scores differ"
    assert (res.perm.cpu().numpy() == theta).all(), "theta differs"
    if flags & esp.USE_LBS:
        assert (res.swaps == swaps).all(), "swap counts differ"
    assert (res.mask.cpu().numpy() == mask).all(), "mask differs"
    # a float64 sum of N * K / m terms: the device adds them in its own order (eq. 5 fixes none)
    assert res.retained == pytest.approx(orc.retained_metric(_np(W), s, theta, n, m), rel=1e-12)
    return res, W, Xc, theta, mask, s


@pytest.mark.parametrize("n,m,B", [(2, 4, 32), (2, 4, 64), (4, 8, 32)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_prune_bit_exact(esp, ctx, n, m, B, dtype):
    _prune_case(esp, ctx, 96, 128, 200, B, n, m, dtype, esp.USE_ALL, 21)


# scores on the device and, with many tokens of few channels (4096 of 24, 4097 of 24) or a negative weight of the norm, on the host: constant
# channels (all tokens in one bin), few and many bins, each term alone
@pytest.mark.parametrize("T,K,bins,alpha,which", [(512, 8, 100, 0.3, 3), (513, 8, 100, 0.3, 3), (300, 24, 1, 0.1, 3), (700, 40, 256, 0.0, 3),
                                                  (700, 40, 100, -0.2, 3), (1, 16, 7, 1.0, 3), (90, 36, 33, 1.0, 1), (90, 36, 33, 0.7, 2),
                                                  (4096, 24, 100, 0.1, 3), (4097, 24, 100, 0.1, 3), (4097, 760, 100, 0.1, 3), (50000, 768, 100, 0.1, 3)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_prune_scores_bit_exact(esp, ctx, T, K, bins, alpha, which, dtype):
    Xc = _rand((T, K), dtype, T + K, col_scale=np.exp(np.random.default_rng(K).standard_normal(K)))
    Xc[:, 1] = 0.75
    Xc[:, 3] = 0.0
    W = _rand((24, K), dtype, 3)
    opts = esp.PruneOpts(n_keep=2, m_group=4, block=8, bins=bins, alpha=alpha, flags=which | esp.USE_GNS)
    x, want = _np(Xc), np.zeros(K)
    if which & esp.USE_ENTROPY:
        want = want + orc.channel_entropy(x, bins)
    if which & esp.USE_NORM:
        want = want + alpha * orc.channel_amplitude(x)
    assert (ctx.prune(Xc.cuda(), W.cuda(), opts).score == want).all()


def test_prune_ablation_switches(esp, ctx):
    for flags in (esp.USE_NORM, esp.USE_NORM | esp.USE_ENTROPY, esp.USE_NORM | esp.USE_ENTROPY | esp.USE_GNS,
                  esp.USE_ENTROPY | esp.USE_LBS):
        _prune_case(esp, ctx, 64, 64, 128, 32, 2, 4, torch.float16, flags, 22)


def test_prune_max_swaps_and_ties(esp, ctx):
    _prune_case(esp, ctx, 48, 64, 64, 32, 2, 4, torch.float16, esp.USE_ALL, 23, max_swaps=3)
    # heavy ties: weights on a coarse grid, scores given
    N, K, B = 40, 64, 32
    rng = np.random.default_rng(5)
    W = torch.tensor(rng.integers(-3, 4, size=(N, K)) * 0.25, dtype=torch.float16)
    s = rng.integers(1, 4, size=K).astype(np.float64)
    opts = esp.PruneOpts(block=B, alpha=1.0)
    res = ctx.prune(None, W.cuda(), opts, score=s)
    theta0 = orc.global_naive_shuffle(W.numpy(), s, 4)
    theta, swaps = orc.local_block_shuffle_vectorised(W.numpy(), s, theta0, 2, 4, B)
    assert (res.perm.cpu().numpy() == theta).all() and (res.swaps == swaps).all()
    assert (res.mask.cpu().numpy() == orc.nm_mask(W.numpy(), s, theta, 2, 4)).all()


def _check_block_shuffle(esp, ctx, W, s, n, m, B, max_swaps=0):
    """The exchanges against the oracle's with the rows added in the device's order (16 interleaved sub-sums)."""
    print(f"lbs N={W.shape[0]} K={W.shape[1]} B={B} {n}:{m} {W.dtype}", flush=True)
    res = ctx.prune(None, W.cuda(), esp.PruneOpts(n_keep=n, m_group=m, block=B, max_swaps=max_swaps), score=s, want_retained=True)
    Wn = _np(W)
    theta, swaps = orc.local_block_shuffle_vectorised(Wn, s, orc.global_naive_shuffle(Wn, s, m), n, m, B, max_swaps,
                                                      order=("lanes", 16))
    assert (res.swaps == swaps).all() and (res.perm.cpu().numpy() == theta).all()
    assert (res.mask.cpu().numpy() == orc.nm_mask_vectorised(Wn, s, theta, n, m)).all()
    assert res.retained == pytest.approx(orc.retained_metric(Wn, s, theta, n, m), rel=1e-12)
    return swaps


# sizes at the edges of the evaluation kernel: fewer rows than a wave's 32, one more than a batch of rows, more than
# one batch per wave; blocks of fewer columns than a lane group, of an odd number of groups, of more than 64 columns
@pytest.mark.parametrize("n,m,B,N", [(2, 4, 8, 1), (2, 4, 12, 33), (2, 4, 36, 257), (2, 4, 64, 1100), (2, 4, 100, 300), (2, 4, 256, 31),
                                     (4, 8, 16, 7), (4, 8, 24, 257), (4, 8, 40, 530), (4, 8, 72, 64), (4, 8, 128, 300)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_block_shuffle_edges_of_the_evaluation_kernel(esp, ctx, n, m, B, N, dtype):
    W = _rand((N, 2 * B), dtype, 31 + N, scale=(2 * B) ** -0.5)
    s = np.random.default_rng(N + B).lognormal(size=2 * B)
    _check_block_shuffle(esp, ctx, W, s, n, m, B, max_swaps=6 if B > 64 else 0)


# all rounds of a block by a team of workgroups: one block; blocks that leave XCDs without a last one; more blocks than are resident at
# once; one workgroup per team and 16; rows that leave the last waves short or empty; and so many rows of few blocks that there are no teams
@pytest.mark.parametrize("n,m,B,nblk,N", [(2, 4, 64, 1, 4000), (2, 4, 8, 600, 40), (2, 4, 32, 9, 1025), (2, 4, 64, 20, 515), (4, 8, 64, 1, 3900),
                                          (4, 8, 16, 530, 33), (4, 8, 32, 17, 771), (4, 8, 64, 10, 1300), (4, 8, 40, 2, 13700), (2, 4, 16, 1, 44100)])
def test_block_shuffle_teams(esp, ctx, n, m, B, nblk, N):
    K = B * nblk
    W = _rand((N, K), torch.bfloat16 if N % 2 else torch.float16, 5 + N, scale=K ** -0.5)
    s = np.random.default_rng(N + B).lognormal(size=K)
    assert _check_block_shuffle(esp, ctx, W, s, n, m, B, max_swaps=3).max() > 1


# teams to the last exchange, so that each of the three buffers of their sums comes round many times: 2 to 16 workgroups per team
@pytest.mark.parametrize("n,m,B,nblk,N", [(2, 4, 16, 40, 700), (2, 4, 32, 6, 1030), (2, 4, 64, 1, 700), (4, 8, 16, 30, 520), (4, 8, 32, 10, 600),
                                          (4, 8, 32, 2, 4000), (4, 8, 64, 1, 520)])
def test_block_shuffle_teams_to_the_end(esp, ctx, n, m, B, nblk, N):
    W = _rand((N, B * nblk), torch.float16 if N % 8 else torch.bfloat16, 6 + N, scale=(B * nblk) ** -0.5)
    s = np.random.default_rng(N + B + 1).lognormal(size=B * nblk)
    assert _check_block_shuffle(esp, ctx, W, s, n, m, B).max() > 4


# Teams that stop waiting: at once, or sooner or later for some of the blocks.  The launches that take over go on from the first
# table and lead to the same exchanges, mask and retained metric (whose sums have taken the place of the panel by columns by then);
# with equal columns in every second block (no global shuffle then) some blocks are left to the exact table meanwhile
@pytest.mark.parametrize("n,m,B,nblk,N", [(2, 4, 64, 2, 520), (2, 4, 32, 12, 300), (4, 8, 64, 2, 270), (4, 8, 32, 5, 520)])
@pytest.mark.parametrize("ties", [False, True])
def test_block_shuffle_teams_that_give_up(esp, n, m, B, nblk, N, ties):
    K = B * nblk
    W = _rand((N, K), torch.float16, 41 + N, scale=K ** -0.5)
    s = np.random.default_rng(N + B).lognormal(size=K)
    if ties:
        tied = np.arange(K) // B % 2 == 0
        s[tied] = 1.0
        W[:, torch.tensor(tied)] = W[:, :1]
    opts = esp.PruneOpts(n_keep=n, m_group=m, block=B, max_swaps=6, flags=esp.USE_NORM | esp.USE_LBS | (0 if ties else esp.USE_GNS))
    Wn = _np(W)
    theta0 = np.arange(K) if ties else orc.global_naive_shuffle(Wn, s, m)
    theta, swaps = orc.local_block_shuffle_vectorised(Wn, s, theta0, n, m, B, 6, order=("lanes", 16))
    mask, retained = orc.nm_mask_vectorised(Wn, s, theta, n, m), orc.retained_metric(Wn, s, theta, n, m)
    c = esp.Context(0)
    team_wait = c._lib._Z13esp_team_waitP11esparse_ctxy
    team_wait.argtypes, team_wait.restype = [C.c_void_p, C.c_ulonglong], C.c_int
    left = 0
    for wait in (0, 30, 100, 300, 1000, 0):
        before = team_wait(c._h, wait)
        print(f"teams that give up: {n}:{m} B={B} nblk={nblk} N={N} ties={ties} wait={wait}", flush=True)
        res = c.prune(None, W.cuda(), opts, score=s, want_retained=True)
        assert (res.swaps == swaps).all() and (res.perm.cpu().numpy() == theta).all()
        assert (res.mask.cpu().numpy() == mask).all() and res.retained == pytest.approx(retained, rel=1e-12)
        left = team_wait(c._h, wait)
        assert left == before + 1 or wait > 0
    print("given up", left)
    c.close()


# exchanges that the cheaper table cannot decide: equal columns (ties), columns without weights and channels kept in every
# row (exchanges that change nothing but the rounding), negative scores
@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
@pytest.mark.parametrize("what", ["equal", "zero", "dominant", "negative"])
def test_block_shuffle_undecided_exchanges(esp, ctx, n, m, what):
    N, K, B = 90, 128, 64
    W = _rand((N, K), torch.float16, 77, scale=K ** -0.5)
    rng = np.random.default_rng(7)
    s = rng.lognormal(size=K)
    some = rng.permutation(K)[:24]
    if what == "equal":
        W[:, some] = W[:, some[:1]]
        s[some] = s[some[0]]
    elif what == "zero":
        W[:, some] = 0
    elif what == "dominant":
        W[:, some] += 8
        s[some] *= 100
    else:
        s[some] *= -1
    assert _check_block_shuffle(esp, ctx, W, s, n, m, B).sum() > 0


# an infinite weight or score (in one column: equal means are another test) sends every block to the exact table in its first
# round; all that is finite about the result is the oracle's, the retained metric is infinite
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
@pytest.mark.parametrize("what", ["weight", "score"])
def test_block_shuffle_infinite_values(esp, ctx, what, n, m, dtype):
    N, K, B = 90, 192, 64
    W = _rand((N, K), dtype, 79, scale=K ** -0.5)
    s = np.random.default_rng(9).lognormal(size=K)
    if what == "score":
        assert (W[:, 11] != 0).all()
        s[11] = np.inf
    else:
        W[7, 11] = float("inf")
        W[40, 11] = float("-inf")
    assert _check_block_shuffle(esp, ctx, W, s, n, m, B).sum() > 0


def _kept_of_network(v, n):
    """The n largest of the last axis as a network of fmax / fmin selects them: of a value and a NaN it makes the value twice."""
    v = np.moveaxis(v, -1, 0).copy()
    for a in range(n):
        for b in range(v.shape[0] - 1, a, -1):
            v[b - 1], v[b] = np.fmax(v[b - 1], v[b]), np.fmin(v[b - 1], v[b])
    return v[:n].sum(axis=0)


# weights that are no numbers: a column's mean leaves them out, they stand behind no weight of their group (kept), and the retained
# metric does not become NaN - the same with and without the block shuffle (4:8 only: the exact 2:4 table makes no sense of a NaN,
# the exchanges do not come to an end and the call reports that)
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
def test_prune_weights_that_are_not_numbers(esp, ctx, n, m, dtype):
    N, K, B = 90, 192, 64
    W = _rand((N, K), dtype, 83, scale=K ** -0.5)
    s = np.random.default_rng(11).lognormal(size=K)
    for j, c in ((5, 3), (17, 70), (17, 71), (60, 150)):
        W[j, c] = float("nan")
    Wn = _np(W).astype(np.float64)
    for flags in ((esp.USE_ALL,) if m == 8 else ()) + (esp.USE_ALL & ~esp.USE_LBS,):
        print(f"nan {n}:{m} {dtype} flags {flags}", flush=True)
        res = ctx.prune(None, W.cuda(), esp.PruneOpts(n_keep=n, m_group=m, block=B, flags=flags), score=s, want_retained=True)
        theta = res.perm.cpu().numpy()
        assert (np.sort(theta) == np.arange(K)).all()
        if not flags & esp.USE_LBS:
            assert (theta == orc.global_naive_shuffle(np.nan_to_num(Wn), s, m)).all()
        xi = (np.abs(Wn) * s)[:, theta].reshape(N, K // m, m)
        pos = np.arange(m)
        ahead = ((xi[..., None, :] > xi[..., :, None]) | ((xi[..., None, :] == xi[..., :, None]) & (pos[None, :] < pos[:, None]))).sum(axis=-1)
        assert (res.mask.cpu().numpy() == (ahead < n).reshape(N, K)).all()
        assert res.retained == pytest.approx(_kept_of_network(xi, n).sum(), rel=1e-12)


# column sums and ranks: fewer rows than a row lane's batch and a remainder, channels past a workgroup's 128 (16), values
# over the whole range of the type with zeros and subnormal ones, equal means
@pytest.mark.parametrize("N,K", [(1, 36), (7, 132), (70, 264), (129, 40)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_naive_shuffle_over_the_range_of_the_type(esp, ctx, N, K, dtype):
    rng = np.random.default_rng(N + K)
    bits = rng.integers(0, 0x7c00 if dtype == torch.float16 else 0x7f80, size=(N, K)).astype(np.int16)
    bits[:, 3] = bits[:, 9]
    bits[:, 5] = 0
    W = torch.from_numpy(bits).view(dtype)
    s = rng.lognormal(size=K)
    s[3] = s[9]
    print(f"gns N={N} K={K} {dtype}", flush=True)
    res = ctx.prune(None, W.cuda(), esp.PruneOpts(block=K, flags=esp.USE_NORM | esp.USE_GNS), score=s)
    assert (res.perm.cpu().numpy() == orc.global_naive_shuffle(_np(W), s, 4)).all()


# the ranks are counted on the device up to 3 x 2^16 channels and sorted on the host beyond: both sides of the line, equal means and
# scores that are no numbers (behind all others, lower channel first); the last needs more staging memory than a context pins
@pytest.mark.parametrize("K", [64, 3 << 16, (3 << 16) + 64, 1 << 22])
def test_naive_shuffle_ranks(esp, ctx, K):
    W = _rand((3, K), torch.float16, 37, scale=0.02)
    rng = np.random.default_rng(K)
    s = rng.lognormal(size=K)
    same, nan = rng.permutation(K)[:40].reshape(2, 20)
    W[:, same] = W[:, same[:1]]
    s[same] = s[same[0]]
    s[nan] = np.nan
    for m in (4, 8):
        print(f"ranks K={K} m={m}", flush=True)
        res = ctx.prune(None, W.cuda(), esp.PruneOpts(n_keep=m // 2, m_group=m, block=64, flags=esp.USE_NORM | esp.USE_GNS), score=s)
        order = np.argsort(-((s * np.abs(_np(W).astype(np.float64)).sum(axis=0)) / 3), kind="stable")
        theta = np.empty(K, dtype=np.int64)
        theta[(np.arange(K) % (K // m)) * m + np.arange(K) // (K // m)] = order
        assert (res.perm.cpu().numpy() == theta).all()
    if K > 3 << 16:  # and the scores in that order reach the block shuffle
        s[nan] = 0.5
        opts = esp.PruneOpts(block=64, max_swaps=1)
        res = ctx.prune(None, W.cuda(), opts, score=s)
        theta, swaps = orc.local_block_shuffle_vectorised(_np(W), s, orc.global_naive_shuffle(_np(W), s, 4), 2, 4, 64, 1,
                                                          blocks=[0, 7, K // 64 - 1], order=("lanes", 16))
        for b in (0, 7, K // 64 - 1):
            assert (res.perm.cpu().numpy()[64 * b:64 * b + 64] == theta[64 * b:64 * b + 64]).all() and res.swaps[b] == swaps[b]


# where the device has room for one panel but not for the two of the cheaper table, the exact table works alone: same result.
# All but 3.25 GiB of the card are taken; the panel of 32768 x 32768 weights needs 2 GiB
def test_prune_with_room_for_one_panel(esp):
    N = K = 32768
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    W = torch.randn(N, K, device="cuda", generator=g, dtype=torch.float16) * 2 ** -7
    s = np.random.default_rng(5).lognormal(size=K)
    opts = esp.PruneOpts(block=64, max_swaps=1)
    first = esp.Context(0)
    want = first.prune(None, W, opts, score=s, want_retained=True)
    first.close()
    mask = torch.empty_like(want.mask)  # the call's own outputs come from what torch keeps
    del mask
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    print(f"free {free >> 20} MiB", flush=True)
    hold = torch.empty(free - (13 << 28), dtype=torch.uint8, device="cuda")
    try:
        ctx = esp.Context(0)
        got = ctx.prune(None, W, opts, score=s, want_retained=True)
        ctx.close()
    finally:
        del hold
        torch.cuda.empty_cache()
    assert torch.equal(got.perm, want.perm) and torch.equal(got.mask, want.mask) and (got.swaps == want.swaps).all()
    assert got.retained == pytest.approx(want.retained, rel=1e-12) and want.swaps.sum() == K // 64


def test_prune_scratch_is_shared_by_calls_and_streams(esp, ctx):
    """One context, shapes that grow and shrink, two streams in turn: every call as on a context of its own."""
    rng = np.random.default_rng(3)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for i, (N, K, B, n, m) in enumerate([(64, 256, 64, 2, 4), (300, 512, 32, 4, 8), (64, 256, 64, 2, 4), (40, 128, 64, 2, 4)]):
        W, s = _rand((N, K), torch.float16, 90 + N).cuda(), rng.lognormal(size=K)
        Xc = _rand((200, K), torch.float16, 91 + K).cuda()
        torch.cuda.synchronize()
        opts = esp.PruneOpts(n_keep=n, m_group=m, block=B)
        with torch.cuda.stream(streams[i % 2]):
            a = ctx.prune(None, W, opts, score=s)
            ca = ctx.compress(W, a.mask, a.perm, n, m)
            b = ctx.prune(Xc, W, opts)
        own = esp.Context(0)
        a2, b2 = own.prune(None, W, opts, score=s), own.prune(Xc, W, opts)
        cb = own.compress(W, a2.mask, a2.perm, n, m)
        own.close()
        for x, y in ((a, a2), (b, b2)):
            assert torch.equal(x.perm, y.perm) and torch.equal(x.mask, y.mask) and (x.score == y.score).all()
        assert torch.equal(ca.native, cb.native)


def test_config1_against_stored_oracle_results(esp, ctx):
    """Workload configuration 1, complete, against results the oracle wrote to tests/golden."""
    gold = json.load(open(os.path.join(os.path.dirname(__file__), "golden", "cfg1_oracle.json")))
    W = wl.weights(1, "linear")
    Xc = wl.calibration(1, "linear")
    X = wl.activations(1, "linear", 16)
    assert _sha(W.numpy()) == gold["inputs_sha256"]["W"] and _sha(Xc.numpy()) == gold["inputs_sha256"]["Xc"]
    opts = esp.PruneOpts(block=64, alpha=gold["alpha"])
    print("config 1 prune", flush=True)
    res = ctx.prune(Xc.cuda(), W.cuda(), opts, want_retained=True)
    assert res.perm.cpu().tolist() == gold["theta"]
    assert res.swaps.tolist() == gold["swaps"]
    assert _sha(res.score) == gold["score_sha256"]
    assert _sha(res.mask.cpu().numpy()) == gold["mask_sha256"]
    assert res.retained == pytest.approx(gold["retained"], rel=1e-12)
    comp = ctx.compress(W.cuda(), res.mask, res.perm)
    assert _sha(_bits(comp.values)) == gold["values_sha256"]
    assert _sha(comp.meta.cpu().numpy()) == gold["meta_sha256"]
    Np_Kp = 512 * 512
    nat = comp.native.cpu().numpy()
    assert _sha(nat[:Np_Kp]) == gold["native_values_sha256"] and _sha(nat[Np_Kp:]) == gold["native_meta_sha256"]
    theta = np.array(gold["theta"])
    mask = res.mask.cpu().numpy()
    Yref = orc.spmm_ref(X.numpy(), W.numpy(), theta, mask)
    for v in range(esp.num_variants()):
        try:
            Y = ctx.spmm(X.cuda(), comp, res.perm, variant=v)
        except esp.EsparseError as e:
            assert e.code == -2                      # variant not applicable to this M
            continue
        err = orc.rowwise_rel_error(_np(Y), Yref)
        assert err.max() <= 2e-3, (esp.variant_name(v), err.max())


# ---------------------------------------------------------------- compression
@pytest.mark.parametrize("N,K", [(24, 320), (16, 256), (5, 36), (130, 1040), (33, 36864), (3, 81920)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_compress_2_4_bit_exact(esp, ctx, N, K, dtype):
    W = _rand((N, K), dtype, 31)
    rng = np.random.default_rng(N * K)
    s = np.abs(rng.standard_normal(K)) + 0.1
    theta = rng.permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), s, theta, 2, 4)
    print(f"compress N={N} K={K} {dtype}", flush=True)
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), torch.tensor(theta, dtype=torch.int32).cuda())
    Wb = _bits(W).reshape(N, K)
    values, meta = orc.compress_vectorised(Wb, theta, mask, 2, 4)        # on raw 16-bit patterns
    assert (_bits(comp.values).reshape(values.shape) == values).all()
    assert (comp.meta.cpu().numpy().view(np.uint32).reshape(meta.shape) == meta).all()
    nv, nm = orc.native_tiling(values, meta, N, K)
    nat = comp.native.cpu().numpy()
    assert nat.size == esp.compressed_size(N, K, 2, 4)[2]
    assert (nat[:nv.nbytes].view(np.uint16) == nv).all()
    assert (nat[nv.nbytes:].view(np.uint16) == nm).all()


# rows and channels that end inside a tile, a 64-channel step, a mask or index word; rows that fill the LDS, rows that do
# not fit it; identity order; a permutation that is none leaves the outputs as they are
@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
@pytest.mark.parametrize("N,K", [(17, 8), (33, 264), (16, 320), (50, 1064), (7, 36872), (3, 81920)])
def test_compress_edges_of_the_row_kernel(esp, ctx, N, K, n, m):
    W = _rand((N, K), torch.float16, 33)
    rng = np.random.default_rng(N + K)
    s = np.abs(rng.standard_normal(K)) + 0.1
    theta = rng.permutation(K) if K != 320 else np.arange(K)
    mask = orc.nm_mask_vectorised(_np(W), s, theta, n, m)
    th = None if K == 320 else torch.tensor(theta, dtype=torch.int32).cuda()
    print(f"compress N={N} K={K} {n}:{m}", flush=True)
    mk = torch.tensor(mask).cuda()
    comp = ctx.compress(W.cuda(), mk, th, n, m)
    values, meta = orc.compress_vectorised(_bits(W).reshape(N, K), theta, mask, n, m)
    assert (_bits(comp.values).reshape(values.shape) == values).all()
    assert (comp.meta.cpu().numpy().view(meta.dtype).reshape(meta.shape) == meta).all()
    nv, nm = (orc.native_tiling if m == 4 else orc.native_tiling_4_8)(values, meta, N, K)
    nat = comp.native.cpu().numpy()
    assert nat.size == esp.compressed_size(N, K, n, m)[2] == nv.nbytes + nm.nbytes
    assert (nat[:nv.nbytes].view(nv.dtype) == nv).all() and (nat[nv.nbytes:].view(nm.dtype) == nm).all()
    assert torch.equal(ctx.compress(W.cuda(), mk, th, n, m, canonical=False).native, comp.native)
    assert torch.equal(ctx.compress(W.cuda(), mk, th, n, m, native=False).values, comp.values)
    if th is not None:
        bad = th.clone()
        bad[0] = K
        before = comp.native.clone()
        Wd = W.cuda()
        rc = ctx._lib.esparse_compress(ctx._h, Wd.data_ptr(), mk.data_ptr(), bad.data_ptr(), N, K, 0, n, m, None, None, comp.native.data_ptr())
        assert rc == -6 and torch.equal(before, comp.native)


def _kept_in_order(W, mask, n):
    """The kept values of each group of a matrix of one or two groups, in position order, and their positions (torch)."""
    N, K = W.shape
    m = 2 * n
    pos = torch.arange(m, device="cuda", dtype=torch.uint8)
    at = torch.where(mask.reshape(N, K // m, m) != 0, pos, pos + m).sort(dim=2).values[:, :, :n].long()
    return W.reshape(N, K // m, m).gather(2, at).reshape(N, -1), at


# so many rows that a launch of a few rows per workgroup has more threads than a launch can have (2^32)
@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
def test_compress_and_prune_very_many_rows(esp, ctx, n, m):
    N, K = (1 << 27) + 1000, 8
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    W = torch.empty(N, K, dtype=torch.float16, device="cuda").normal_(generator=g)
    s = np.array([1.0, 3.0, 0.5, 2.0, 1.5, 0.25, 2.5, 0.75])
    print(f"rows {N} {n}:{m}", flush=True)
    res = ctx.prune(None, W, esp.PruneOpts(n_keep=n, m_group=m, block=8, max_swaps=1, flags=esp.USE_ALL if m == 4 else esp.USE_ALL & ~esp.USE_LBS), score=s)
    perm = res.perm.long()
    sc = torch.tensor(s, device="cuda")[perm]
    comp = ctx.compress(W, res.mask, res.perm, n, m, native=False)
    for lo in range(0, N, 1 << 24):
        Wp = W[lo:lo + (1 << 24)][:, perm]
        mask = res.mask[lo:lo + (1 << 24)]
        xi = (Wp.double().abs() * sc).reshape(-1, K // m, m)
        keep = torch.zeros(xi.shape, dtype=torch.uint8, device="cuda").scatter_(2, xi.argsort(dim=2, descending=True, stable=True)[:, :, :n], 1)
        assert torch.equal(keep.reshape(mask.shape), mask), lo
        values, at = _kept_in_order(Wp, mask, n)
        assert torch.equal(comp.values[lo:lo + (1 << 24)], values), lo
        rows = values.shape[0]
        meta = comp.meta[lo * 4 if m == 4 else lo:][:rows * 4 if m == 4 else rows]
        if m == 4:
            want = sum(at.reshape(rows, 4)[:, f] << (2 * f) for f in range(4))
            assert torch.equal(meta.view(torch.int32).long(), want), lo
        else:
            assert torch.equal(meta.long(), (1 << at.reshape(rows, 4)).sum(dim=1)), lo


def test_compress_4_8_and_derived_mask_and_errors(esp, ctx):
    N, K = 20, 64
    W = _rand((N, K), torch.float16, 32)
    rng = np.random.default_rng(9)
    s = np.abs(rng.standard_normal(K)) + 0.1
    theta = rng.permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), s, theta, 4, 8)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, 4, 8)
    values, meta = orc.compress_vectorised(_bits(W).reshape(N, K), theta, mask, 4, 8)
    assert (_bits(comp.values).reshape(values.shape) == values).all()
    assert (comp.meta.cpu().numpy().reshape(meta.shape) == meta).all()
    nv, nm = orc.native_tiling_4_8(values, meta, N, K)
    nat = comp.native.cpu().numpy()
    assert nat.size == esp.compressed_size(N, K, 4, 8)[2] == nv.nbytes + nm.nbytes
    assert (nat[:nv.nbytes].view(np.uint16) == nv).all() and (nat[nv.nbytes:] == nm).all()
    # mask = NULL: the mask is read off the zeros of an already pruned weight
    for n, m in ((2, 4), (4, 8)):
        mk = orc.nm_mask_vectorised(_np(W), s, theta, n, m)
        Wz = torch.tensor(_np(W) * orc.mask_to_original_order(mk, theta), dtype=torch.float16)
        comp = ctx.compress(Wz.cuda(), None, th, n, m)
        values, meta = orc.compress_vectorised(_bits(Wz).reshape(N, K), theta, mk, n, m)
        assert (_bits(comp.values).reshape(values.shape) == values).all()
        assert (comp.meta.cpu().numpy().view(meta.dtype).reshape(meta.shape) == meta).all()
    # a dense weight has more than n non-zeros per group
    with pytest.raises(esp.EsparseError) as e:
        ctx.compress(W.cuda(), None, th, 2, 4)
    assert e.value.code == -5
    bad = mask.copy()
    bad[3, 8:16] = 1
    with pytest.raises(esp.EsparseError) as e:
        ctx.compress(W.cuda(), torch.tensor(bad).cuda(), th, 4, 8)
    assert e.value.code == -5
    th_bad = th.clone()
    th_bad[5] = th_bad[6]
    with pytest.raises(esp.EsparseError) as e:
        ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th_bad, 4, 8)
    assert e.value.code == -6


# ---------------------------------------------------------------- products
def _spmm_case(esp, ctx, M, N, K, dtype, seed, use_perm=True):
    rng = np.random.default_rng(seed)
    scales = wl.channel_scales("lognormal", K, wl.stream_id("xs", seed))
    W = _rand((N, K), dtype, seed, scale=K ** -0.5)
    X = _rand((M, K), dtype, seed + 7, col_scale=scales)
    s = np.abs(rng.standard_normal(K)) + 0.1
    theta = rng.permutation(K) if use_perm else np.arange(K)
    mask = orc.nm_mask_vectorised(_np(W), s, theta, 2, 4)
    th = torch.tensor(theta, dtype=torch.int32).cuda() if use_perm else None
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, canonical=False)
    Yref = orc.spmm_ref(_np(X), _np(W), theta, mask)
    Ydref = orc.dense_ref(_np(X), _np(W))
    packed = ctx.dense_pack(W.cuda())
    Xd = X.cuda()
    for v in range(esp.num_variants()):
        print(f"spmm M={M} N={N} K={K} {dtype} perm={use_perm} variant={esp.variant_name(v)}", flush=True)
        try:
            Y = ctx.spmm(Xd, comp, th, variant=v)
            torch.cuda.synchronize()
            err = orc.rowwise_rel_error(_np(Y), Yref)
            assert err.max() <= TOL[dtype], ("sparse", esp.variant_name(v), err.max())
        except esp.EsparseError as e:
            assert e.code == -2                      # not for this shape, or a variant of the dense product only
        try:
            Yd = ctx.dense_gemm(Xd, packed, N, variant=v)
            torch.cuda.synchronize()
            err = orc.rowwise_rel_error(_np(Yd), Ydref)
            assert err.max() <= TOL[dtype], ("dense", esp.variant_name(v), err.max())
        except esp.EsparseError as e:
            assert e.code == -2                      # not for this shape, or a variant of the 2:4 product only
    # default variant
    Y = ctx.spmm(Xd, comp, th)
    assert orc.rowwise_rel_error(_np(Y), Yref).max() <= TOL[dtype]


def test_workspace_of_no_bytes(esp):
    c = esp.Context(0)
    assert c.workspace(0).numel() == 0 and c.workspace(0).data_ptr() % 256 == 0 and c.workspace(300).numel() == 300
    c.close()


def _aligned(nbytes):
    ws = torch.zeros(nbytes + 256, dtype=torch.uint8, device="cuda")
    return ws[(-ws.data_ptr()) % 256:]


def _device_case(ctx, M, N, K, n, m, seed, dtype=torch.float16):
    """A case made on the device (sizes the CPU oracle would take seconds for): X, theta, compressed weights, float64 reference."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    X = torch.randn(M, K, device="cuda", generator=g).to(dtype)
    W = (torch.randn(N, K, device="cuda", generator=g) * K ** -0.5).to(dtype)
    perm = torch.randperm(K, device="cuda", generator=g).to(torch.int32)
    Wp = W[:, perm.long()]
    top = Wp.abs().reshape(N, -1, m).argsort(dim=2, descending=True, stable=True)[:, :, :n]
    mask = torch.zeros(N, K // m, m, dtype=torch.uint8, device="cuda").scatter_(2, top, 1).reshape(N, K)
    comp = ctx.compress(W, mask, perm, n, m, canonical=False)
    ref = X.double()[:, perm.long()] @ (Wp * mask).double().t().contiguous()
    return X, perm, comp, ref.cpu().numpy()


@pytest.mark.parametrize("M", [1, 8, 16, 33, 130])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_spmm_small_ragged(esp, ctx, M, dtype):
    _spmm_case(esp, ctx, M, 72, 576, dtype, 41)


@pytest.mark.parametrize("M", [2, 3, 5, 9, 15, 17])
def test_spmm_few_tokens_compact_staging(esp, ctx, M):
    """Up to 16 tokens the decode kernels read the compact copy of the staged activations (token count rounded up
    to a power of two, the padding tokens zero); 17 is the first size that does not."""
    _spmm_case(esp, ctx, M, 88, 832, torch.float16, 46 + M)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_spmm_decode_step_pairs(esp, ctx, dtype):
    """K = 2048: 16 step pairs divide among 8 and 16 waves, so the decode kernels with two or four token tiles take
    the steps pairwise and read one index word per pair."""
    _spmm_case(esp, ctx, 33, 80, 2048, dtype, 52)
    _spmm_case(esp, ctx, 20, 48, 2048, dtype, 53)


def test_spmm_stream_spans(esp, ctx):
    """Stream kernels cut the steps of all row blocks into equal spans: a span inside one row block (partial
    pieces), a span across a row block boundary, and spans holding several whole row blocks (stored directly)."""
    _spmm_case(esp, ctx, 70, 400, 768, torch.float16, 44)        # 12 steps per row block, spans of 8
    _spmm_case(esp, ctx, 40, 65536 + 48, 256, torch.bfloat16, 45)  # 4 steps per row block, spans of 8 or more


def test_spmm_identity_perm_and_multi_tile(esp, ctx):
    _spmm_case(esp, ctx, 16, 512, 2048, torch.float16, 42, use_perm=False)
    _spmm_case(esp, ctx, 200, 272, 1280, torch.float16, 43)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_spmm_k_split_over_workgroups(esp, ctx, dtype):
    # K long enough (64 stages of 64 channels) for the split-K variants to really split; ragged M and N
    _spmm_case(esp, ctx, 100, 300, 4096, dtype, 49)
    _spmm_case(esp, ctx, 64, 144, 2304, dtype, 50)
    _spmm_case(esp, ctx, 300, 272, 4096, dtype, 51)   # 128 < M <= 512: up to four splits


def test_spmm_many_tokens_row_staging(esp, ctx):
    """Long inputs are staged by workgroups that hold 2 to 16 whole rows of X; the workgroups of one token tile are
    numbered 8 apart.  8 and 16 rows per workgroup need thousands of tokens; the tile counts (257, 513) are not
    multiples of 8 and the last tile is ragged."""
    _spmm_case(esp, ctx, 4100, 32, 512, torch.float16, 54)
    _spmm_case(esp, ctx, 8200, 32, 320, torch.bfloat16, 55)


def test_spmm_banded_tile_order(esp, ctx):
    """More than 8 token blocks per row block: the tile kernels number their macro tiles in bands of 8 row blocks
    (token blocks outermost within a band).  11 row blocks of 256 (22 of 128) leave a ragged last band; 2400 tokens are
    10 blocks of 256 (19 of 128), the last one ragged."""
    _spmm_case(esp, ctx, 2400, 2816, 256, torch.float16, 56)


def test_stacked_matrices_share_one_theta(esp, ctx):
    """Matrices that read the same input (q/k/v, gate/up) pruned as one stacked matrix: one theta, one mask;
    the product of the stack is the concatenation of the products of its slices (bitwise: rows are independent)
    and matches the oracle on the stack."""
    K, T, M = 256, 128, 20
    Ws = [_rand((n, K), torch.float16, 60 + i, scale=K ** -0.5) for i, n in enumerate((48, 32, 80))]
    Wcat = torch.cat(Ws, dim=0)
    Xc = _rand((T, K), torch.float16, 63, col_scale=wl.channel_scales("lognormal", K, wl.stream_id("st", 1)))
    X = _rand((M, K), torch.float16, 64)
    alpha = wl.default_alpha(T)
    res = ctx.prune(Xc.cuda(), Wcat.cuda(), esp.PruneOpts(block=64, alpha=alpha))
    theta, mask, s, _ = orc.prune(_np(Xc), _np(Wcat), 2, 4, 64, alpha, 100)
    assert (res.perm.cpu().numpy() == theta).all() and (res.mask.cpu().numpy() == mask).all()
    comp = ctx.compress(Wcat.cuda(), res.mask, res.perm, canonical=False)
    Y = ctx.spmm(X.cuda(), comp, res.perm)
    assert orc.rowwise_rel_error(_np(Y), orc.spmm_ref(_np(X), _np(Wcat), theta, mask)).max() <= 2e-3
    lo = 0
    for W in Ws:
        n = W.shape[0]
        part = ctx.compress(W.cuda(), res.mask[lo:lo + n].contiguous(), res.perm, canonical=False)
        Yp = ctx.spmm(X.cuda(), part, res.perm)
        assert (_bits(Yp) == _bits(Y[:, lo:lo + n])).all()
        lo += n


def test_spmm_one_hot_reads_back_weights_through_theta(esp, ctx):
    N, K = 48, 256
    rng = np.random.default_rng(3)
    W = _rand((N, K), torch.float16, 44)
    s = np.abs(rng.standard_normal(K)) + 0.1
    theta = rng.permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), s, theta, 2, 4)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th)
    X = torch.eye(K, dtype=torch.float16)
    Y = ctx.spmm(X.cuda(), comp, th)                      # [K, N]: row c = masked W[:, c]
    ref = (_np(W) * orc.mask_to_original_order(mask, theta)).T
    assert (_np(Y) == ref).all()
    ones = torch.ones((1, K), dtype=torch.float16)
    Y1 = ctx.spmm(ones.cuda(), comp, th)
    assert np.allclose(_np(Y1)[0], ref.sum(axis=0), rtol=2e-3, atol=1e-3)


def test_spmm_repeat_is_bitwise_identical_and_m0(esp, ctx):
    N, K, M = 64, 1024, 24
    W = _rand((N, K), torch.float16, 45, scale=K ** -0.5)
    X = _rand((M, K), torch.float16, 46)
    theta = np.random.default_rng(1).permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), np.ones(K), theta, 2, 4)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, canonical=False)
    for v in range(esp.num_variants()):
        try:
            a = _bits(ctx.spmm(X.cuda(), comp, th, variant=v))
        except esp.EsparseError as e:
            assert e.code == -2                      # variant not applicable to this M
            continue
        b = _bits(ctx.spmm(X.cuda(), comp, th, variant=v))
        assert (a == b).all()
    Y0 = ctx.spmm(X[:0].cuda(), comp, th)
    assert Y0.shape == (0, N)


@pytest.mark.parametrize("M,K", [(1, 832), (2, 832), (1, 11008), (2, 4096), (1, 36864), (3, 832)])
def test_spmm_theta_gathered_in_the_kernel_equals_staged(esp, ctx, M, K):
    """With one or two tokens the decode kernels apply the channel re-ordering themselves (no staged copy, no staging
    launch) where the gathered row fits the LDS; the result is bitwise the one of the two-step path (activations staged
    through theta by a launch of their own, then multiplied) and within tolerance of the oracle.  K = 36864 at one token
     (and 11008) and three tokens are beyond what is gathered in the kernel (both calls then take the staged path)."""
    N = 80
    rng = np.random.default_rng(M * 7 + K)
    W = _rand((N, K), torch.float16, 61, scale=K ** -0.5)
    X = _rand((M, K), torch.float16, 62, col_scale=wl.channel_scales("lognormal", K, wl.stream_id("xs", 62)))
    theta = rng.permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), np.abs(rng.standard_normal(K)) + 0.1, theta, 2, 4)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, canonical=False)
    Yref = orc.spmm_ref(_np(X), _np(W), theta, mask)
    Xd = X.cuda()
    ran = 0
    for perm in (th, None):
        ref = Yref if perm is not None else orc.spmm_ref(_np(X), _np(W[:, theta]), np.arange(K), mask)
        comp_p = comp if perm is not None else ctx.compress(W[:, theta].contiguous().cuda(), torch.tensor(mask).cuda(), None, canonical=False)
        for v in range(esp.num_variants()):
            print(f"fold M={M} K={K} perm={'theta' if perm is not None else 'identity'} variant={esp.variant_name(v)}", flush=True)
            try:
                Y = ctx.spmm(Xd, comp_p, perm, variant=v)
            except esp.EsparseError as e:
                assert e.code == -2
                continue
            ws = ctx.stage_activations(Xd, perm, N)
            Y2 = torch.empty_like(Y)
            ctx.spmm_staged(M, comp_p, ws, Y2, variant=v)
            torch.cuda.synchronize()
            assert (_bits(Y) == _bits(Y2)).all(), esp.variant_name(v)
            assert orc.rowwise_rel_error(_np(Y), ref).max() <= 2e-3
            ran += 1
    assert ran > 4


# up to 16 tokens of few channels are gathered inside the decode kernel as well: token counts that are no power of two, channels
# that end inside a unit, waves without a step of their own, groups, each pattern and the dense product
@pytest.mark.parametrize("M,K", [(3, 64), (4, 2304), (5, 1004), (9, 640), (16, 512), (16, 640), (7, 1280)])
@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
def test_few_tokens_gathered_in_the_kernel_equal_staged(esp, ctx, M, K, n, m):
    K = K // m * m
    N, count = 72, 3
    rng = np.random.default_rng(M + K)
    X = _rand((M, K), torch.float16, 61).cuda()
    comps, perms = [], []
    for i in range(count):
        W = _rand((N, K), torch.float16, 62 + i, scale=K ** -0.5)
        theta = rng.permutation(K)
        mask = orc.nm_mask_vectorised(_np(W), np.ones(K), theta, n, m)
        perms.append(torch.tensor(theta, dtype=torch.int32).cuda())
        comps.append(ctx.compress(W.cuda(), torch.tensor(mask).cuda(), perms[-1], n, m))
        ref = orc.spmm_ref(_np(X), _np(W), theta, mask)
        # every decode kernel that keeps K inside the workgroup takes these shapes: an error of any kind is a failure
        decode = [v for v in range(esp.num_variants()) if esp.variant_name(v).startswith("ksplit") and "_k" not in esp.variant_name(v)]
        assert len(decode) >= 12
        for v in [-1] + decode:
            Y = ctx.spmm(X, comps[-1], perms[-1], variant=v)
            assert orc.rowwise_rel_error(_np(Y).astype(np.float64), ref).max() <= TOL[torch.float16]
            ws = torch.zeros(esp.spmm_workspace(M, N, K) + 256, dtype=torch.uint8, device="cuda")
            ws = ws[(-ws.data_ptr()) % 256:]
            ctx.stage_activations(X, perms[-1], N, ws=ws)
            assert torch.equal(ctx.spmm_staged(M, comps[-1], ws, torch.empty_like(Y), variant=v), Y)
    for v in decode:
        for Y, comp, perm in zip(ctx.spmm_group([X] * count, comps, perms, variant=v), comps, perms):
            assert torch.equal(Y, ctx.spmm(X, comp, perm, variant=v))


# Tokens' rows kept by the decode kernels, at the edges: the first token of the second tile, K that ends within a unit of 8 channels, the
# longest rows that the LDS holds and the first that it does not, no re-ordering, dense weights; 4:8 rows that stay below 64 KiB of dynamic LDS
# only without the table of selectors beside them.  The sums are the staged product's in
# the same order: equal bit by bit, for each kernel and for the built-in choice, alone and in a group
@pytest.mark.parametrize("M,K,n,m", [(3, 4, 2, 4), (9, 1036, 2, 4), (5, 264, 4, 8), (8, 8960, 2, 4), (8, 8964, 2, 4), (3, 8960, 4, 8), (16, 4744, 2, 4),
                                     (16, 4748, 2, 4), (9, 4744, 4, 8), (8, 8960, 0, 0), (16, 4744, 0, 0), (4, 1036, 0, 0),
                                     (8, 3600, 4, 8), (16, 1904, 4, 8)])
def test_tokens_rows_kept_by_the_decode_kernels(esp, ctx, M, K, n, m):
    N = 40
    decode = [v for v in range(esp.num_variants()) if esp.variant_name(v).startswith("ksplit") and "_k" not in esp.variant_name(v)]
    if m:
        X, perm, comp, ref = _device_case(ctx, M, N, K, n, m, 71, torch.bfloat16)
        ordered = X[:, perm.long()].contiguous()
        calls = [(lambda v: ctx.spmm(X, comp, perm, variant=v)), (lambda v: ctx.spmm(ordered, comp, None, variant=v)),
                 (lambda v: ctx.spmm_group([X, ordered], [comp] * 2, [perm, None], variant=v)[1])]
        ws = _aligned(esp.spmm_workspace(M, N, K))
        ctx.stage_activations(X, perm, N, ws=ws)
        staged = lambda v: ctx.spmm_staged(M, comp, ws, torch.empty(M, N, dtype=X.dtype, device="cuda"), variant=v)
    else:
        g = torch.Generator(device="cuda").manual_seed(71)
        X = torch.randn(M, K, device="cuda", generator=g).bfloat16()
        W = (torch.randn(N, K, device="cuda", generator=g) * K ** -0.5).bfloat16()
        packed, ref = ctx.dense_pack(W), (X.double() @ W.double().t().contiguous()).cpu().numpy()
        calls = [(lambda v: ctx.dense_gemm(X, packed, N, variant=v)), (lambda v: ctx.dense_gemm_group([X, X], [packed] * 2, N, variant=v)[1])]
        ws = _aligned(esp.spmm_workspace(M, N, K))
        ctx.stage_activations(X, None, N, ws=ws)
        staged = lambda v: ctx.dense_gemm_staged(M, packed, N, K, ws, torch.empty(M, N, dtype=X.dtype, device="cuda"), variant=v)
        decode = [v for v in decode if "_q" not in esp.variant_name(v)]
    for v in [-1] + decode:
        want = staged(v)
        assert orc.rowwise_rel_error(_np(want).astype(np.float64), ref).max() <= TOL[torch.bfloat16], v
        for i, call in enumerate(calls):
            assert (_bits(call(v)) == _bits(want)).all(), (v, i)


# the pairs kernel: fewer pairs of stages than its ring holds, one more, two more and a multiple; one row tile, a macro tile and one row more; the last
# token tile and token of a macro tile; rows of Y that are no multiple of 8 values; some rows and all tokens beyond one XCD's share
@pytest.mark.parametrize("M,N,K", [(64, 16, 64), (65, 129, 512), (100, 128, 772), (79, 8, 1024), (512, 1031, 1280), (333, 1000, 2304), (1024, 2048, 256), (96, 4099, 516)])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_pairs_of_stages(esp, ctx, M, N, K, dtype):
    X, perm, comp, ref = _device_case(ctx, M, N, K, 2, 4, 81, dtype)
    v = [esp.variant_name(i) for i in range(esp.num_variants())].index("pairs_w8_r128_t64")
    guard = 4096
    buf = torch.full((M * N + 2 * guard,), 7.0, dtype=dtype, device="cuda")
    Y = ctx.spmm(X, comp, perm, variant=v, out=buf[guard:guard + M * N].view(M, N))
    assert orc.rowwise_rel_error(_np(Y).astype(np.float64), ref).max() <= TOL[dtype]
    assert (buf[:guard] == 7.0).all() and (buf[guard + M * N:] == 7.0).all()
    assert torch.equal(ctx.spmm(X, comp, perm, variant=v), Y)


# a square layer applied in place, whole and overlapping by some rows, alone and in a group whose members share an input
@pytest.mark.parametrize("M", [2, 4, 8])
def test_outputs_that_overlap_the_input(esp, ctx, M):
    N = K = 512
    cases = [_device_case(ctx, M, N, K, 2, 4, 51 + i) for i in range(3)]
    X = cases[0][0]
    apart = [ctx.spmm(X, c[2], c[1]) for c in cases]
    print(f"in place M={M}", flush=True)
    for shift in (0, M // 2, -(M // 2), M):
        buf = torch.zeros(3 * M, K, dtype=X.dtype, device="cuda")
        Xi = buf[M:2 * M]
        Xi.copy_(X)
        Y = buf[M + shift:2 * M + shift]
        ctx.spmm(Xi, cases[0][2], cases[0][1], out=Y)
        assert (_bits(Y) == _bits(apart[0])).all(), shift
        Xi.copy_(X)
        outs = [torch.empty_like(X), Y, torch.empty_like(X)]
        named = [esp.variant_name(v) for v in range(esp.num_variants())].index("ksplit_w8_r1")
        ctx.spmm_group([Xi] * 3, [c[2] for c in cases], [c[1] for c in cases], variant=named, outs=outs)
        for o, c in zip(outs, cases):
            assert (_bits(o) == _bits(ctx.spmm(X, c[2], c[1], variant=named))).all(), shift


# row lengths of Y that are no multiple of 8 outputs leave the tile kernels word by word: odd, 2 and 4 modulo 8, a last tile of
# one output, fewer outputs than a wave owns; a guard behind Y and every kernel that takes the shape
@pytest.mark.parametrize("N", [1, 30, 129, 260, 321])
@pytest.mark.parametrize("mode", ["2:4", "4:8", "dense"])
def test_tile_kernels_store_rows_of_any_length(esp, ctx, N, mode):
    M, K = 150, 512
    n, m = (4, 8) if mode == "4:8" else (2, 4)
    W, X = _rand((N, K), torch.float16, 81, scale=K ** -0.5), _rand((M, K), torch.float16, 82)
    theta = np.random.default_rng(N).permutation(K) if mode != "dense" else np.arange(K)
    if mode == "dense":
        ref = orc.dense_ref(_np(X), _np(W))
        packed = ctx.dense_pack(W.cuda())
    else:
        mask = orc.nm_mask_vectorised(_np(W), np.ones(K), theta, n, m)
        ref = orc.spmm_ref(_np(X), _np(W), theta, mask)
        th = torch.tensor(theta, dtype=torch.int32).cuda()
        comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, n, m)
    Xd, ran = X.cuda(), 0
    for v in range(esp.num_variants()):
        if not esp.variant_name(v).startswith("tile"):
            continue
        buf = torch.full((M * N + 64,), 7.0, dtype=torch.float16, device="cuda")
        Y = buf[:M * N].view(M, N)
        try:
            ctx.dense_gemm(Xd, packed, N, variant=v, out=Y) if mode == "dense" else ctx.spmm(Xd, comp, th, variant=v, out=Y)
        except esp.EsparseError as e:
            assert e.code == -2, (esp.variant_name(v), e)  # a kernel for other weights
            continue
        ran += 1
        assert orc.rowwise_rel_error(_np(Y), ref).max() <= TOL[torch.float16], esp.variant_name(v)
        assert (buf[M * N:] == 7.0).all(), esp.variant_name(v)
    other = {"2:4": ("tile48", "_h"), "4:8": ("tile_", "tile32"), "dense": ("tile48", "tile32")}[mode]
    tiles = [esp.variant_name(v) for v in range(esp.num_variants()) if esp.variant_name(v).startswith("tile")]
    assert ran == sum(not any(o in name for o in other) for name in tiles)


# rows of X that are a multiple of 8 but not of 16 bytes go through the row staging 8 bytes at a time
@pytest.mark.parametrize("M,K", [(64, 4), (65, 68), (130, 3020), (600, 516)])
@pytest.mark.parametrize("with_perm", [True, False])
def test_row_staging_of_odd_row_lengths(esp, ctx, M, K, with_perm):
    N = 48
    W, X = _rand((N, K), torch.bfloat16, 71, scale=K ** -0.5), _rand((M, K), torch.bfloat16, 72)
    theta = np.random.default_rng(K).permutation(K) if with_perm else np.arange(K)
    mask = orc.nm_mask_vectorised(_np(W), np.ones(K), theta, 2, 4)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, 2, 4)
    Y = ctx.spmm(X.cuda(), comp, th if with_perm else None)
    assert orc.rowwise_rel_error(_np(Y), orc.spmm_ref(_np(X), _np(W), theta, mask)).max() <= TOL[torch.bfloat16]


@pytest.mark.parametrize("M", [8, 100, 300])
def test_spmm_replayed_from_a_hip_graph(esp, ctx, M):
    """The calls enqueue kernels only (no allocation, no memset, no synchronisation), so a caller may capture them
    into a HIP graph: every variant, staging included, captured once on a side stream and replayed three times with
    new activations and eager work of the same context between the replays, must reproduce the eager result bit
    for bit (decode, K-split, stream and tile kernels with their reduction launches)."""
    N, K = 272, 2048
    W = _rand((N, K), torch.float16, 61, scale=K ** -0.5)
    theta = np.random.default_rng(2).permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), np.ones(K), theta, 2, 4)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, canonical=False)
    Xs = [_rand((M, K), torch.float16, 62 + i).cuda() for i in range(3)]
    other = _rand((M + 5, K), torch.float16, 70).cuda()
    side = torch.cuda.Stream()
    for v in range(esp.num_variants()):
        try:
            eager = [_bits(ctx.spmm(x, comp, th, variant=v)) for x in Xs]
        except esp.EsparseError as e:
            assert e.code == -2
            continue
        print(f"graph replay M={M} variant={esp.variant_name(v)}", flush=True)
        xin = Xs[0].clone()
        yout = torch.zeros((M, N), dtype=torch.float16, device="cuda")
        ws = torch.empty(esp.spmm_workspace(M, N, K) + 256, dtype=torch.uint8, device="cuda")
        ws = ws[(-ws.data_ptr()) % 256:]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            ctx.stage_activations(xin, th, N, ws)
            ctx.spmm_staged(M, comp, ws, yout, variant=v)       # warm-up on the side stream
            torch.cuda.synchronize()
            with torch.cuda.graph(g, stream=side):
                ctx.stage_activations(xin, th, N, ws)
                ctx.spmm_staged(M, comp, ws, yout, variant=v)
        torch.cuda.synchronize()
        for i in (1, 2, 0):
            xin.copy_(Xs[i])
            yout.zero_()
            ctx.spmm(other, comp, th, variant=v)                # eager work between the replays (own workspace)
            torch.cuda.synchronize()
            g.replay()
            torch.cuda.synchronize()
            assert (_bits(yout) == eager[i]).all(), (esp.variant_name(v), i)
        del g


def test_workspace_too_small_and_bad_variant(esp, ctx):
    import ctypes as C
    N, K, M = 32, 256, 4
    W = _rand((N, K), torch.float16, 47)
    comp = ctx.compress(torch.tensor(_np(W) * np.tile([1, 1, 0, 0], (N, K // 4)), dtype=torch.float16).cuda(), None, None)
    X = _rand((M, K), torch.float16, 48).cuda()
    Y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    ws = ctx.workspace(1024)
    lib = esp.load_library()
    rc = lib.esparse_spmm(ctx._h, X.data_ptr(), M, comp.native.data_ptr(), None, N, K, 0, 2, 4, Y.data_ptr(),
                          ws.data_ptr(), 1024, -1)
    assert rc == -7
    with pytest.raises(esp.EsparseError) as e:
        ctx.spmm(X, comp, None, variant=999)
    assert e.value.code == -1


@pytest.mark.parametrize("M,N,K", [(33, 80, 2048), (130, 272, 1024), (600, 528, 768)])
def test_named_variant_stays_inside_the_workspace_size_reported_for_it(esp, ctx, M, N, K):
    # esparse_spmm_workspace(M, N, K, variant): a call naming that variant accepts exactly that many bytes, touches
    # nothing behind them (a guard pattern follows the workspace) and gives the product of the full-size workspace
    W = _rand((N, K), torch.float16, 81)
    comp = ctx.compress(torch.tensor(_np(W) * np.tile([1, 0, 1, 0], (N, K // 4)), dtype=torch.float16).cuda(), None, None)
    X = _rand((M, K), torch.float16, 82).cuda()
    th = torch.tensor(np.random.default_rng(83).permutation(K), dtype=torch.int32).cuda()
    lib = esp.load_library()
    guard = 1 << 20
    for v in range(esp.num_variants()):
        try:
            ref = _bits(ctx.spmm(X, comp, th, variant=v))
        except esp.EsparseError as e:
            assert e.code == -2
            continue
        need = esp.spmm_workspace(M, N, K, v)
        assert need <= esp.spmm_workspace(M, N, K)
        buf = torch.full((need + guard + 256,), 0xA5, dtype=torch.uint8, device="cuda")
        off = (-buf.data_ptr()) % 256
        Y = torch.zeros((M, N), dtype=torch.float16, device="cuda")
        print(f"workspace of variant {esp.variant_name(v)}: {need} bytes", flush=True)
        rc = lib.esparse_spmm(ctx._h, X.data_ptr(), M, comp.native.data_ptr(), th.data_ptr(), N, K, 0, 2, 4, Y.data_ptr(),
                              buf.data_ptr() + off, need, v)
        assert rc == 0, (esp.variant_name(v), lib.esparse_last_error(ctx._h).decode())
        torch.cuda.synchronize()
        assert (_bits(Y) == ref).all(), esp.variant_name(v)
        assert bool((buf[off + need:] == 0xA5).all()), esp.variant_name(v)
        rc = lib.esparse_spmm(ctx._h, X.data_ptr(), M, comp.native.data_ptr(), th.data_ptr(), N, K, 0, 2, 4, Y.data_ptr(),
                              buf.data_ptr() + off, need - 256, v)
        assert rc == -7


def test_matrix_rate_is_plausible(esp, ctx):
    # register-resident operands: below the published peaks (5.0 PFLOP/s effective for 2:4, 2.5 dense; 3 % for the
    # clock's tolerance), well above what any product kernel reaches, zeros not slower than random data, and the 2:4
    # instruction about twice the dense one
    sr = ctx.matrix_rate(True, esp.F16, True)
    sz = ctx.matrix_rate(True, esp.F16, False)
    dr = ctx.matrix_rate(False, esp.F16, True)
    br = ctx.matrix_rate(True, esp.BF16, True)
    m1 = ctx.matrix_rate(True, esp.F16, True, mix=1)
    m2 = ctx.matrix_rate(True, esp.F16, True, mix=2)
    print(f"matrix rate TFLOP/s: 2:4 fp16 random {sr:.0f}, zeros {sz:.0f}, bf16 random {br:.0f}, dense fp16 random {dr:.0f}; "
          f"with a stage's LDS reads {m1:.0f}, and its DMA, wait and barrier {m2:.0f}", flush=True)
    assert 1500 < sr <= 5150 and 1500 < br <= 5150 and sr * 0.95 <= sz <= 5150
    assert 750 < dr <= 2575 and 1.6 < sr / dr < 2.4
    assert 1000 < m2 <= m1 * 1.05 and m1 <= sr * 1.05


def test_read_rate_is_plausible(esp, ctx):
    # cold plain reads: below the published 8 TB/s, rising with the bytes per launch (launch, ramp-up and drain are fixed)
    small, mid, big = ctx.read_rate(16 << 20), ctx.read_rate(100 << 20), ctx.read_rate(1 << 30)
    print(f"plain read GB/s: 16 MiB {small:.0f}, 100 MiB {mid:.0f}, 1 GiB {big:.0f}", flush=True)
    assert 1000 < small < mid < big * 1.05 and big < 8000


def test_tune_picks_a_variant_and_persists(esp, ctx, tmp_path):
    best, ms = ctx.tune(16, 512, 1024, esp.F16, sparse=True)
    assert 0 <= best < esp.num_variants() and ms > 0
    p = str(tmp_path / "tuned.txt")
    ctx.tune_save(p)
    c2 = esp.Context(0)
    c2.tune_load(p)
    assert esp.variant_name(best) in open(p).read()
    # a choice for launches of three products of the shape is kept beside the single one and survives the file
    bg, msg = ctx.tune_group(3, 16, 512, 1024, esp.F16, sparse=True)
    assert 0 <= bg < esp.num_variants() and msg > 0
    ctx.tune_save(p)
    lines = [l.split() for l in open(p).read().splitlines() if not l.startswith("#")]
    assert ["1", "0", "16", "512", "1024", esp.variant_name(best)] in lines
    assert ["1", "0", "16", "512", "1024", esp.variant_name(bg), "3"] in lines
    c3 = esp.Context(0)
    c3.tune_load(p)
    q = str(tmp_path / "again.txt")
    c3.tune_save(q)
    assert sorted(open(q).read().splitlines()) == sorted(open(p).read().splitlines())


# ---------------------------------------------------------------- eq. 4 report
def test_output_error_report_for_the_ablation_settings(esp, ctx):
    """Relative output error of eq. (4) on held-out activations for the four settings of the paper's ablation
    (norm; + entropy; + global shuffle; + local block shuffle), device against oracle."""
    N, K, T, M = 96, 128, 200, 64
    scales = wl.channel_scales("lognormal", K, wl.stream_id("oe", 1))
    W = _rand((N, K), torch.float16, 70, scale=K ** -0.5)
    Xc = _rand((T, K), torch.float16, 71, col_scale=scales)
    X = _rand((M, K), torch.float16, 72, col_scale=scales)
    alpha = wl.default_alpha(T)
    packed = ctx.dense_pack(W.cuda())
    Yd = ctx.dense_gemm(X.cuda(), packed, N)
    for flags in (esp.USE_NORM, esp.USE_NORM | esp.USE_ENTROPY, esp.USE_NORM | esp.USE_ENTROPY | esp.USE_GNS, esp.USE_ALL):
        res = ctx.prune(Xc.cuda(), W.cuda(), esp.PruneOpts(block=32, alpha=alpha, flags=flags))
        comp = ctx.compress(W.cuda(), res.mask, res.perm, canonical=False)
        Ys = ctx.spmm(X.cuda(), comp, res.perm)
        num, den = ctx.output_error(Yd, Ys)
        # the entry point itself, against float64 numpy on the same two outputs
        a, b = _np(Yd).astype(np.float64), _np(Ys).astype(np.float64)
        assert abs(num - ((a - b) ** 2).sum()) <= 1e-12 * num and abs(den - (a ** 2).sum()) <= 1e-12 * den
        # the report, against the oracle's eq. (4) on exact products (the device outputs are rounded to 16 bits)
        theta, mask, _, _ = orc.prune(_np(Xc), _np(W), 2, 4, 32, alpha, 100, use_entropy=bool(flags & esp.USE_ENTROPY),
                                      use_norm=True, use_gns=bool(flags & esp.USE_GNS), use_lbs=bool(flags & esp.USE_LBS))
        ref = orc.output_error(_np(X), _np(W), theta, mask)
        assert abs(num / den - ref) <= 1e-2 * ref, (flags, num / den, ref)
    n0, d0 = ctx.output_error(Yd[:0], Yd[:0])
    assert (n0, d0) == (0.0, 0.0)


# ---------------------------------------------------------------- 4:8 product (bitmaps expanded in registers)
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("M,N,K", [(1, 72, 576), (8, 40, 256), (33, 72, 576), (40, 72, 1024), (64, 144, 2304), (150, 48, 512),
                                   (300, 520, 768), (200, 100, 264)])
def test_spmm_4_8(esp, ctx, M, N, K, dtype):
    rng = np.random.default_rng(M * N + K)
    scales = wl.channel_scales("lognormal", K, wl.stream_id("x48", M))
    W = _rand((N, K), dtype, 80, scale=K ** -0.5)
    X = _rand((M, K), dtype, 81, col_scale=scales)
    s = np.abs(rng.standard_normal(K)) + 0.1
    theta = rng.permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), s, theta, 4, 8)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, 4, 8)
    values, meta = orc.compress_vectorised(_bits(W).reshape(N, K), theta, mask, 4, 8)
    nv, nm = orc.native_tiling_4_8(values, meta, N, K)
    nat = comp.native.cpu().numpy()
    assert (nat[:nv.nbytes].view(np.uint16) == nv).all() and (nat[nv.nbytes:] == nm).all()
    Yref = orc.spmm_ref(_np(X), _np(W), theta, mask)
    ran = 0
    for v in [-1] + list(range(esp.num_variants())):
        print(f"4:8 spmm M={M} N={N} K={K} {dtype} variant={v}", flush=True)
        try:
            Y = ctx.spmm(X.cuda(), comp, th, variant=v)
        except esp.EsparseError as e:
            assert e.code == -2 and v >= 0          # not a decode, four-slot stream or 4:8 tile kernel, or not for this M
            continue
        torch.cuda.synchronize()
        err = orc.rowwise_rel_error(_np(Y), Yref)
        assert err.max() <= TOL[dtype], (v, err.max())
        ran += 1
    assert ran >= 3


def test_products_on_seeded_random_shapes(esp, ctx):
    """Shapes drawn from a seeded generator (ragged tails in every dimension, token counts on both sides of every
    kernel family's boundary), both weight formats and the dense product, each through the kernel the library
    chooses by itself, against the oracle."""
    rng = np.random.default_rng(20231015)
    boundaries = [1, 2, 3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257, 300]
    for case in range(18):
        M = int(boundaries[case])
        N = int(rng.integers(1, 700))
        K = int(rng.integers(1, 200)) * 8
        dtype = torch.float16 if case % 3 else torch.bfloat16
        W = _rand((N, K), dtype, 300 + case, scale=K ** -0.5)
        X = _rand((M, K), dtype, 400 + case, col_scale=wl.channel_scales("lognormal", K, wl.stream_id("rs", case)))
        s = np.abs(rng.standard_normal(K)) + 0.1
        theta = rng.permutation(K)
        th = torch.tensor(theta, dtype=torch.int32).cuda()
        print(f"random shape {case}: M={M} N={N} K={K} {dtype}", flush=True)
        for n, m in ((2, 4), (4, 8)):
            mask = orc.nm_mask_vectorised(_np(W), s, theta, n, m)
            comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, n, m, canonical=False)
            Y = ctx.spmm(X.cuda(), comp, th)
            torch.cuda.synchronize()
            err = orc.rowwise_rel_error(_np(Y), orc.spmm_ref(_np(X), _np(W), theta, mask))
            assert err.max() <= TOL[dtype], (case, n, m, err.max())
        Yd = ctx.dense_gemm(X.cuda(), ctx.dense_pack(W.cuda()), N)
        torch.cuda.synchronize()
        assert orc.rowwise_rel_error(_np(Yd), orc.dense_ref(_np(X), _np(W))).max() <= TOL[dtype], case


def test_spmm_4_8_one_hot_reads_back_weights(esp, ctx):
    N, K = 32, 256
    rng = np.random.default_rng(48)
    W = _rand((N, K), torch.float16, 82)
    s = np.abs(rng.standard_normal(K)) + 0.1
    theta = rng.permutation(K)
    mask = orc.nm_mask_vectorised(_np(W), s, theta, 4, 8)
    th = torch.tensor(theta, dtype=torch.int32).cuda()
    comp = ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, 4, 8, canonical=False)
    Y = ctx.spmm(torch.eye(K, dtype=torch.float16).cuda(), comp, th)         # [K, N]: row c = masked W[:, c]
    assert (_np(Y) == (_np(W) * orc.mask_to_original_order(mask, theta)).T).all()


# ---------------------------------------------------------------- several products of one shape in one call
# a group of one at shapes where a single product's built-in choice is no decode kernel: the halves exist all the same
@pytest.mark.parametrize("M,N,K,n,m", [(24, 4096, 11008, 2, 4), (27, 1172, 13928, 2, 4), (16, 5120, 13824, 4, 8)])
def test_halves_of_a_group_of_one(esp, ctx, M, N, K, n, m):
    print(f"halves M={M} N={N} K={K} {n}:{m}", flush=True)
    X, perm, comp, ref = _device_case(ctx, M, N, K, n, m, 41)
    whole = ctx.spmm_group([X], [comp], [perm])[0]
    ws = torch.zeros(esp.spmm_workspace(M, N, K) + 256, dtype=torch.uint8, device="cuda")
    ws = ws[(-ws.data_ptr()) % 256:]
    out = torch.empty_like(whole)
    ctx.stage_activations_group([X], [perm], comp, ws)
    ctx.spmm_group_staged(M, [comp], ws, [out])
    assert orc.rowwise_rel_error(_np(out), ref).max() <= TOL[X.dtype]
    assert (_bits(out) == _bits(whole)).all()


# the built-in choice knows how many products share the launch, so a group may run another kernel than a single product (at this
# shape it does): the same product within the tolerance, bit for bit with the same named variant
def test_group_and_single_product_choose_for_themselves(esp, ctx):
    M, N, K = 8, 4096, 4096
    cases = [_device_case(ctx, M, N, K, 2, 4, 45 + i) for i in range(3)]
    for v in (-1, [esp.variant_name(v) for v in range(esp.num_variants())].index("ksplit_w8_r4")):
        Ys = ctx.spmm_group([c[0] for c in cases], [c[2] for c in cases], [c[1] for c in cases], variant=v)
        for Y, (X, perm, comp, ref) in zip(Ys, cases):
            single = ctx.spmm(X, comp, perm, variant=v)
            assert orc.rowwise_rel_error(_np(Y), ref).max() <= TOL[X.dtype]
            assert orc.rowwise_rel_error(_np(single), ref).max() <= TOL[X.dtype]
            assert v < 0 or torch.equal(Y, single)


@pytest.mark.parametrize("n,m", [(2, 4), (4, 8)])
@pytest.mark.parametrize("M", [1, 20, 64, 100])
def test_spmm_group_equals_single_products(esp, ctx, M, n, m):
    N, K = 80, 512
    rng = np.random.default_rng(M + n)
    X = _rand((M, K), torch.float16, 90).cuda()
    X2 = _rand((M, K), torch.float16, 91).cuda()
    comps, perms, refs = [], [], []
    for i in range(3):
        W = _rand((N, K), torch.float16, 92 + i, scale=K ** -0.5)
        s = np.abs(rng.standard_normal(K)) + 0.1
        theta = rng.permutation(K)
        mask = orc.nm_mask_vectorised(_np(W), s, theta, n, m)
        th = torch.tensor(theta, dtype=torch.int32).cuda()
        comps.append(ctx.compress(W.cuda(), torch.tensor(mask).cuda(), th, n, m, canonical=False))
        perms.append(th)
        refs.append(orc.spmm_ref(_np(X2 if i == 2 else X), _np(W), theta, mask))
    Xs = [X, X, X2]                                   # two members share their input, like q/k/v
    print(f"group M={M} {n}:{m}", flush=True)
    Ys = ctx.spmm_group(Xs, comps, perms)
    torch.cuda.synchronize()
    for i in range(3):
        assert orc.rowwise_rel_error(_np(Ys[i]), refs[i]).max() <= 2e-3
        single = ctx.spmm(Xs[i], comps[i], perms[i])
        assert (_bits(single) == _bits(Ys[i])).all()
    if n == 2:
        Ws = [_rand((N, K), torch.float16, 92 + i, scale=K ** -0.5).cuda() for i in range(3)]
        packed = [ctx.dense_pack(W) for W in Ws]
        Yd = ctx.dense_gemm_group(Xs, packed, N)
        for i in range(3):
            assert (_bits(Yd[i]) == _bits(ctx.dense_gemm(Xs[i], packed[i], N))).all()
            assert orc.rowwise_rel_error(_np(Yd[i]), orc.dense_ref(_np(Xs[i]), _np(Ws[i]))).max() <= 2e-3
    if M <= 32:
        # the two halves as separate calls (they exist where a decode kernel is the default: M <= 32)
        ws = ctx.workspace(4 * esp.spmm_workspace(M, N, K))
        ctx.stage_activations_group(Xs, perms, comps[0], ws)
        outs = [torch.empty_like(y) for y in Ys]
        ctx.spmm_group_staged(M, comps, ws, outs)
        for i in range(3):
            assert (_bits(outs[i]) == _bits(Ys[i])).all()
    # identity permutation for all members, one member only
    Y1 = ctx.spmm_group([X], comps[:1], None)
    assert (_bits(Y1[0]) == _bits(ctx.spmm(X, comps[0], None))).all()
