"""Host-side checks that need no GPU: the C-ABI library loads, exports every declared symbol,
answers its closed-form size queries and rejects bad arguments before touching the GPU."""
import ctypes as C
import os
import random
import re
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2310_15929_amd as esp
from paper_2310_15929_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    lib = esp.load_library()
    header = open(os.path.join(ROOT, "include", "esparse.h")).read()
    declared = set(re.findall(r"\b(esparse_[a-z_]+)\s*\(", header))
    declared -= {"esparse_ctx", "esparse_status", "esparse_dtype", "esparse_prune_opts"}
    assert declared == set(binding.EXPORTED)
    for name in declared:
        assert hasattr(lib, name), name
    assert lib.esparse_version().startswith(b"esparse")


def test_size_queries_closed_form():
    for N, K in [(512, 512), (4096, 11008), (24, 320)]:
        vb, mb, nb = esp.compressed_size(N, K, 2, 4)
        assert vb == N * K and mb == N * ((K // 2 + 15) // 16) * 4
        Np, Kp = -(-N // 16) * 16, -(-K // 256) * 256
        assert nb == Np * Kp * 9 // 8
        vb8, mb8, nb8 = esp.compressed_size(N, K - K % 8, 4, 8)
        Kp8 = -(-(K - K % 8) // 256) * 256
        assert vb8 == N * (K - K % 8) and mb8 == N * (K - K % 8) // 8 and nb8 == Np * Kp8 * 9 // 8
    vb, mb, _ = esp.compressed_size(4096, 4096, 2, 4)
    assert (vb + mb) / (2 * 4096 * 4096) == 0.5625
    assert esp.dense_packed_size(24, 320) == 32 * 512 * 2
    assert esp.spmm_workspace(16, 512, 512) >= 16 * 512 * 2
    # the size for a named variant never exceeds the size that serves every variant, covers the staged activations,
    # and only variants that split K over workgroups ask for fp32 partial tiles
    for M, N, K in [(1, 4096, 4096), (33, 80, 2048), (128, 22016, 8192), (2048, 13824, 5120)]:
        every = esp.spmm_workspace(M, N, K)
        assert every == esp.spmm_workspace(M, N, K, -1)
        Mp = -(-M // 16) * 16
        for v in range(esp.num_variants()):
            one = esp.spmm_workspace(M, N, K, v)
            assert Mp * K * 2 <= one <= every, esp.variant_name(v)
            splits = "splitk" in esp.variant_name(v) or "stream" in esp.variant_name(v) or "_k" in esp.variant_name(v)
            if not splits:
                assert one < Mp * K * 2 * 2 + 4096, esp.variant_name(v)
    with pytest.raises(esp.EsparseError):
        esp.spmm_workspace(16, 512, 512, esp.num_variants())
    with pytest.raises(esp.EsparseError):
        esp.compressed_size(8, 8, 1, 4)


def test_argument_errors_need_no_gpu():
    ctx = esp.Context(0)
    W = torch.zeros(8, 16, dtype=torch.float16)
    Xc = torch.zeros(4, 16, dtype=torch.float16)

    def code(fn):
        with pytest.raises(esp.EsparseError) as e:
            fn()
        return e.value.code

    assert code(lambda: ctx.compress(W, None, None, 3, 4)) == -2
    assert code(lambda: ctx.compress(torch.zeros(8, 18, dtype=torch.float16), None, None, 2, 4)) == -1
    assert code(lambda: ctx.prune(Xc, W, esp.PruneOpts(block=24))) == -1          # 16 % 24
    assert code(lambda: ctx.prune(Xc, W, esp.PruneOpts(block=6))) == -1           # block % m
    assert code(lambda: ctx.prune(Xc, W, esp.PruneOpts(n_keep=1, m_group=4, block=8))) == -2
    assert code(lambda: ctx.prune(Xc, W, esp.PruneOpts(block=8, bins=0))) == -1
    assert code(lambda: ctx.prune(Xc, W, esp.PruneOpts(block=8, flags=esp.USE_GNS))) == -1
    assert code(lambda: ctx.prune(Xc, W, esp.PruneOpts(block=8, max_swaps=-1))) == -1
    lib = esp.load_library()
    assert lib.esparse_spmm(ctx._h, None, 4, None, None, 8, 16, 0, 1, 4, None, None, 0, -1) == -2   # no 1:4 product
    assert lib.esparse_spmm(ctx._h, None, 4, None, None, 8, 16, 0, 4, 8, None, None, 0, -1) == -1   # 4:8: null pointers
    assert lib.esparse_spmm(ctx._h, None, 4, None, None, 8, 16, 0, 2, 4, None, None, 0, -1) == -1
    assert b"null" in lib.esparse_last_error(ctx._h)
    assert lib.esparse_spmm(ctx._h, None, 0, None, None, 8, 16, 0, 2, 4, None, None, 0, -1) == 0   # M = 0
    assert lib.esparse_channel_stats(ctx._h, None, 4, 16, 0, 100, None, None) == -1
    assert lib.esparse_create(None, 0, None) == -1
    assert lib.esparse_output_error(ctx._h, None, None, 4, 4, 0, None, None) == -1      # null result pointers
    assert lib.esparse_spmm_group(ctx._h, 0, None, 4, None, None, 8, 16, 0, 2, 4, None, None, 0, -1) == -1   # count
    assert lib.esparse_spmm_group(ctx._h, 5, None, 4, None, None, 8, 16, 0, 2, 4, None, None, 0, -1) == -1
    assert lib.esparse_spmm_group(ctx._h, 2, None, 4, None, None, 8, 16, 0, 2, 4, None, None, 0, -1) == -1   # null arrays
    assert lib.esparse_spmm_group(ctx._h, 2, None, 4, None, None, 8, 16, 0, 3, 4, None, None, 0, -1) == -2   # no 3:4
    import ctypes as C
    nb = C.c_size_t(0)
    assert lib.esparse_spmm_group_workspace(3, 8, 512, 512, C.byref(nb)) == 0 and nb.value >= 65536 + 3 * 16 * 512 * 2
    assert lib.esparse_spmm_group_workspace(0, 8, 512, 512, C.byref(nb)) == -1
    assert lib.esparse_output_error(None, None, None, 4, 4, 0, None, None) == -1        # null context
    assert lib.esparse_tune_group(ctx._h, 0, 16, 512, 512, 0, 1, None, None) == -1       # count outside 1..4
    assert lib.esparse_tune_group(ctx._h, 5, 16, 512, 512, 0, 1, None, None) == -1
    assert lib.esparse_matrix_rate(ctx._h, 1, 0, 1, 0, None) == -1                       # null result pointer
    rate = C.c_double(0.0)
    assert lib.esparse_matrix_rate(ctx._h, 2, 0, 1, 0, C.byref(rate)) == -1              # sparse is 0 or 1
    assert lib.esparse_matrix_rate(ctx._h, 1, 7, 1, 0, C.byref(rate)) == -2              # no such dtype
    assert lib.esparse_matrix_rate(ctx._h, 1, 0, 1, 3, C.byref(rate)) == -1              # mix is 0, 1 or 2
    assert lib.esparse_matrix_rate(ctx._h, 0, 0, 1, 2, C.byref(rate)) == -2              # the stage mixes are 2:4 only
    # which kernel variants serve which weights is decided on the host, before any GPU call (the pointers are never used)
    vs = {esp.variant_name(v): v for v in range(esp.num_variants())}
    fake = C.c_void_p(1 << 20)

    def spmm_code(M, n, m, name):
        return lib.esparse_spmm(ctx._h, fake, M, fake, None, 512, 512, 0, n, m, fake, fake, 1 << 30, vs[name])

    assert spmm_code(256, 4, 8, "tile32_w8_t256") == -2       # the 32x32x32 kernel multiplies 2:4 weights only
    assert spmm_code(256, 2, 4, "tile48_w8_t128") == -2       # the tile48 kernels 4:8 weights only
    assert spmm_code(32, 4, 8, "tile48_w8_t128") == -2        # ... and 64 tokens or more
    assert spmm_code(64, 4, 8, "stream_w8_r1_d7") == -2       # 4:8 through the stream kernels: rings of four slots only
    assert spmm_code(256, 4, 8, "stream_w8_r1_d3") == -2      # ... and at most 128 tokens
    assert spmm_code(32, 4, 8, "ksplit_w8_r1_q") == -2        # one metadata load per four steps: at most 16 tokens
    assert spmm_code(256, 2, 4, "tile_w8_t256_h") == -2       # dense weights only
    assert b"variant" in lib.esparse_last_error(ctx._h)
    assert lib.esparse_read_rate(ctx._h, 1 << 20, None) == -1                             # null result pointer
    assert lib.esparse_read_rate(ctx._h, 16, C.byref(rate)) == -1                         # fewer than 4 KiB


def test_halves_of_a_group_up_to_32_tokens_have_a_decode_kernel():
    """Whatever the shape and the count, the built-in choice for the halves of a group call of at most 32 tokens is a kernel
    that has halves.  The context names a device that does not exist: an accepted call ends there (EHIP), before any launch."""
    lib = esp.load_library()
    ctx = esp.Context(1000)
    fake = C.c_void_p(1 << 20)
    for M in (1, 2, 7, 16, 17, 24, 32):
        for N in (16, 512, 1172, 4096, 5120, 11008, 36864):
            for K in (64, 512, 4096, 9216, 13928, 22016):
                for count in (1, 2, 3, 4):
                    a = (C.c_void_p * count)(*[fake] * count)
                    for n, m in ((2, 4), (4, 8)):
                        args = (M, N, K, count, n)
                        assert lib.esparse_stage_activations_group(ctx._h, count, a, M, None, N, K, 0, n, m, fake, 1 << 40, -1) == -4, args
                        assert lib.esparse_spmm_group_staged(ctx._h, count, M, a, N, K, 0, n, m, a, fake, 1 << 40, -1) == -4, args
    a = (C.c_void_p * 1)(fake)
    assert lib.esparse_stage_activations_group(ctx._h, 1, a, 33, None, 4096, 4096, 0, 2, 4, fake, 1 << 40, -1) == -2


def test_sizes_refuse_the_same_arguments_again():
    """Arguments that the library's size queries refuse stay refused after a call with equal ones of the right type, also where a call
    looks a size up again."""
    known = [(esp.spmm_workspace, (16, 512, 512)), (binding._known_workspace, (16, 512, 512)), (esp.compressed_size, (8, 512, 2, 4)),
             (binding._known_size, (8, 512, 2, 4)), (binding._known_group_workspace, (2, 16, 512, 512))]
    for f, args in known:
        assert f(*args) == f(*args)
        for i in range(len(args)):
            with pytest.raises(C.ArgumentError):
                f(*args[:i], float(args[i]), *args[i + 1:])
    assert binding._known_workspace(16, 512, 512) == esp.spmm_workspace(16, 512, 512)


def test_built_in_choices_can_run():
    """Over all sizes: the built-in choice is a kernel that takes the shape; a group of at most 32 tokens gets one with a grouped
    form; where no partial tiles fit, it is one that keeps none."""
    lib = esp.load_library()
    ll, i, b = C.c_longlong, C.c_int, C.c_bool
    pick, without, fits = lib._Z19esp_default_variantxxxiib, lib._Z36esp_default_variant_without_partialsxxxi, lib._Z22esp_variant_applicableixxxi
    pick.argtypes, without.argtypes, fits.argtypes, fits.restype = [ll, ll, ll, i, i, b], [ll, ll, ll, i], [i, ll, ll, ll, i], b
    names = [esp.variant_name(v) for v in range(esp.num_variants())]
    rng = random.Random(5)
    for _ in range(4000):
        M, N, K = int(2 ** rng.uniform(0, 20)), int(2 ** rng.uniform(0, 18)), 8 * int(2 ** rng.uniform(0, 14))
        for sparse in (0, 1, 2):
            for count in (1, 2, 4):
                for grouped in (False, True):
                    v = pick(M, N, K, sparse, count, grouped)
                    assert 0 <= v < len(names) and fits(v, M, N, K, sparse), (M, N, K, sparse, count)
                    if grouped and M <= 32:
                        assert names[v].startswith("ksplit") and "_k" not in names[v]
            v = without(M, N, K, sparse)
            assert fits(v, M, N, K, sparse) and not any(p in names[v] for p in ("splitk", "stream", "_k")), (M, N, K, sparse, names[v])


def test_scores_stay_on_the_device_where_that_is_faster():
    """Sizes at which one of the two ways was measured faster by a fifth and more; negative scores and more channels than are ranked
    there never stay on the device, scores without a logarithm always do."""
    on = esp.load_library()._Z20esp_scores_on_devicexxibbd
    on.argtypes, on.restype = [C.c_longlong, C.c_longlong, C.c_int, C.c_bool, C.c_bool, C.c_double], C.c_bool
    for T, K, bins in [(512, 256, 100), (2048, 64, 256), (4096, 384, 100), (6000, 640, 256), (6000, 256, 256), (16384, 640, 256), (32768, 1024, 100),
                       (131072, 1024, 100), (131072, 1536, 256), (524288, 640, 100), (262144, 3072, 100), (262144, 4096, 100), (1 << 22, 4096, 100)]:
        assert on(T, K, bins, True, True, 0.5) and on(T, K, bins, True, False, -1.0) and not on(T, K, bins, True, True, -1e-9), (T, K, bins)
    for T, K, bins in [(8192, 128, 100), (16384, 256, 10), (16384, 256, 100), (32768, 768, 10), (131072, 512, 10), (524288, 64, 256)]:
        assert not on(T, K, bins, True, True, 0.5) and on(T, K, bins, False, True, 0.5), (T, K, bins)
    assert not on(512, 196612, 100, True, True, 1.0) and not on(512, 196612, 100, False, True, 1.0)


def test_block_shuffle_teams_can_end():
    """Teams only where the device has 8 XCDs of 64 places; no more workgroups than an XCD has places for its share of the blocks, and so
    few per team that parts of the teams of four launches never fill the places of an XCD; none for many rows of few blocks."""
    team = esp.load_library()._Z12esp_lbs_teamxxiii
    team.argtypes = [C.c_longlong, C.c_longlong, C.c_int, C.c_int, C.c_int]
    rng, largest = random.Random(7), 0
    for _ in range(5000):
        N, nblk, m = int(2 ** rng.uniform(0, 24)), int(2 ** rng.uniform(0, 16)), rng.choice([4, 8])
        B = m * rng.randint(2, 256 // m)
        for cus in (32, 64, 128, 255):
            assert team(N, nblk, B, m, cus) == 0
        t = team(N, nblk, B, m, 256)
        if B > 64 or (N > 44000 and nblk <= 8):
            assert t == 0
            continue
        if t == 0:
            assert (nblk <= 16 and N > 13600 and m == 8 and B > 32) or (17 <= nblk <= 24 and N > 24000 and B > 32)
            continue
        assert 4 * (t - 1) < 64
        assert t == 1 or (t * -(-nblk // 8) <= 64 and (t - 1) * 256 < N)
        largest = max(largest, t)
    assert largest == 16
    assert team(13600, 8, 64, 8, 256) == 16 and team(13601, 8, 64, 8, 256) == 0 and team(19200, 9, 64, 8, 256) == 16 and team(19201, 9, 64, 8, 256) == 0
    assert team(24000, 17, 64, 4, 256) == 16 and team(24001, 24, 64, 4, 256) == 0 and team(1 << 20, 25, 64, 8, 256) == 16 and team(1 << 20, 9, 64, 4, 256) == 16


@pytest.mark.parametrize("room_mib", [64, 1])
def test_entropies_without_threads_or_memory(room_mib):
    """The host part of the channel statistics on 8 threads, and where the address space has no room for another thread's
    stack (std::thread then throws): same values."""
    code = f"""
import ctypes as C, resource, numpy as np, sys
lib = C.CDLL({binding._LIB_PATH!r})
f = lib._Z13esp_entropiesPKjxixPd
f.argtypes = [C.c_void_p, C.c_longlong, C.c_int, C.c_longlong, C.c_void_p]; f.restype = None
K, bins, T = 6000, 100, 40000
hist = np.random.default_rng(1).multinomial(T, np.full(bins, 1 / bins), size=K).astype(np.uint32)
hist[0] = 0; hist[0, 5] = T
p = hist / T
want = -np.where(hist > 0, p * np.log(np.where(hist > 0, p, 1.0)), 0.0).sum(axis=1)
out = np.full(K, 7.0)
now = int(open('/proc/self/statm').read().split()[0]) * 4096
resource.setrlimit(resource.RLIMIT_AS, (now + ({room_mib} << 20), resource.RLIM_INFINITY))
f(hist.ctypes.data, K, bins, T, out.ctypes.data)
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
sys.exit(0 if np.abs(out - want).max() < 1e-13 else 3)
"""
    assert subprocess.run([sys.executable, "-c", code], timeout=60).returncode == 0


def test_tune_table_text_roundtrip(tmp_path):
    ctx = esp.Context(0)
    p = tmp_path / "t.txt"
    p.write_text("# comment\n1 0 16 512 512 %s\n" % esp.variant_name(1))
    ctx.tune_load(str(p))
    q = tmp_path / "u.txt"
    ctx.tune_save(str(q))
    assert "1 0 16 512 512 " + esp.variant_name(1) in q.read_text()
    # a trailing count marks a choice for group launches; lines without it are for single products
    p.write_text("1 0 16 512 512 %s 3\n1 0 16 512 512 %s\n" % (esp.variant_name(4), esp.variant_name(1)))
    c2 = esp.Context(0)
    c2.tune_load(str(p))
    c2.tune_save(str(q))
    body = [l for l in q.read_text().splitlines() if not l.startswith("#")]
    assert sorted(body) == sorted(["1 0 16 512 512 %s 3" % esp.variant_name(4), "1 0 16 512 512 %s" % esp.variant_name(1)])


def test_missing_library_fails_loudly(monkeypatch):
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_LIB_PATH", "/nonexistent/libesparse.so")
    with pytest.raises(FileNotFoundError):
        binding.load_library()


def test_traffic_profile_rows_parse_and_name_existing_variants():
    """bench.py looks roofline.traffic up in profiles/product_kernels_hbm_traffic.txt by shape and kernel variant: every
    row must parse, name a variant the library has, and carry counter bytes of at least the algorithmic bytes."""
    names = {esp.variant_name(v) for v in range(esp.num_variants())}
    rows = [l for l in open(os.path.join(ROOT, "profiles", "product_kernels_hbm_traffic.txt")) if l.startswith("traffic ")]
    assert len(rows) >= 10
    seen = set()
    for line in rows:
        f = dict(kv.split("=", 1) for kv in line.split()[1:])
        assert f["variant"] in names, f["variant"]
        key = (f["members"], f["M"], f["N"], f["K"], f["variant"])
        assert key not in seen
        seen.add(key)
        moved = int(f["fetch_bytes"]) + int(f["write_bytes"])
        assert moved >= 0.98 * int(f["algorithmic_bytes"])


def test_constants_of_the_kernel_choice_come_from_their_times():
    """The fits that profiles/kernel_choice_fit.py makes of the times beside it are the constants in the source, to their printed digits."""
    run = subprocess.run([sys.executable, os.path.join(ROOT, "profiles", "kernel_choice_fit.py")], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr
    off = [float(x) for x in re.findall(r"refit within ([0-9.]+) % of a time", run.stdout)]
    assert len(off) == 3 + 2 + 3 and max(off) < 0.3, run.stdout
