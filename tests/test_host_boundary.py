"""Host-side checks that need no GPU: the C-ABI library loads, exports every symbol the
header declares, validates descriptors, and its chunk store matches the oracle's model."""
import os
import re

import numpy as np
import pytest

import oracle.hcache_oracle as oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def hc():
    import paper_2410_05004_amd as hc
    return hc


def header_symbols():
    text = open(os.path.join(ROOT, "include", "hcache.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(hc_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol(hc):
    syms = header_symbols()
    assert len(syms) >= 18
    for s in syms:
        assert hasattr(hc.lib, s), f"{s} declared in hcache.h but not exported"
    from paper_2410_05004_amd.binding import EXPORTED
    assert sorted(EXPORTED) == syms, "binding and header disagree on the entry points"


def test_version_and_error_string(hc):
    assert hc.version().startswith("hcache-mi355x")
    assert hc.lib.hc_last_error() is not None


def good_desc(hc, **over):
    kw = dict(n_layers=2, d_model=256, n_q_heads=4, n_kv_heads=4, head_dim=64, block_size=16,
              max_position=128, rope_style=0, rope_theta=10000.0, rms_eps=1e-5, norm_kind=0)
    kw.update(over)
    return hc.ModelDesc(*[kw[k] for k in ("n_layers", "d_model", "n_q_heads", "n_kv_heads",
                                           "head_dim", "block_size", "max_position", "rope_style",
                                           "rope_theta", "rms_eps", "norm_kind")])


def test_desc_validation(hc):
    hc.validate_desc(good_desc(hc))
    hc.validate_desc(good_desc(hc, rope_style=2, norm_kind=1))
    bad = [dict(n_layers=0), dict(d_model=100), dict(head_dim=48), dict(n_q_heads=6, n_kv_heads=4),
           dict(block_size=12), dict(max_position=0), dict(rope_style=3), dict(rope_theta=0.0),
           dict(norm_kind=2),
           dict(rms_eps=-1.0), dict(n_kv_heads=0)]
    for over in bad:
        with pytest.raises(hc.HCacheError) as e:
            hc.validate_desc(good_desc(hc, **over))
        assert e.value.status == hc.HC_EINVAL, over
        assert str(e.value)


def read_chunk(store, seq, layer, c, d):
    import ctypes
    ptr, rows = store.chunk(seq, layer, c)
    buf = (ctypes.c_uint16 * (rows * d)).from_address(ptr)
    return np.frombuffer(buf, dtype=np.uint16).reshape(rows, d).copy()


def test_store_matches_oracle_model(hc):
    L, d, CT, T = 3, 16, 4, 11
    st = hc.Store(L, d, CT, capacity_chunks=64, pinned=False)
    ref = oracle.ChunkStore(L, d, CT)
    rng = np.random.default_rng(1)
    full = rng.integers(0, 65536, size=(L, T, d), dtype=np.uint16)
    # generation order: prefill of 5 tokens, then token by token, layer by layer
    steps = [(0, 5)] + [(t, t + 1) for t in range(5, T)]
    for a, b in steps:
        for l in range(L):
            rows = np.ascontiguousarray(full[l, a:b])
            st.append(7, l, rows, b - a)
            ref.append(7, l, rows)
    for l in range(L):
        assert st.tokens(7, l) == T == ref.n_tokens(7, l)
        for c in range(ref.n_chunks(7, l)):
            assert np.array_equal(read_chunk(st, 7, l, c, d), ref.chunk(7, l, c))
        with pytest.raises(hc.HCacheError) as e:
            st.chunk(7, l, ref.n_chunks(7, l))
        assert e.value.status == hc.HC_ERANGE
    # Figure 6: 2nd token, 2nd layer -> chunk (layer 1, 0), row 1
    assert np.array_equal(read_chunk(st, 7, 1, 0, d)[1], full[1, 1])
    # the arena is cut into rows of L chunk slots: chunk index c of every layer shares a row
    # (layer l at slot l of it), and a context's rows are consecutive while nothing interferes,
    # so a layer's chunks are exactly L slots apart -- one strided transfer per layer
    chunk_bytes = CT * d * 2
    p = [[st.chunk(7, l, c)[0] for c in range(3)] for l in range(L)]
    for c in range(3):
        assert p[1][c] - p[0][c] == chunk_bytes and p[2][c] - p[1][c] == chunk_bytes
    for l in range(L):
        assert p[l][1] - p[l][0] == L * chunk_bytes and p[l][2] - p[l][1] == L * chunk_bytes
    st.destroy()


def test_store_errors_and_reuse(hc):
    L, d, CT = 2, 8, 4
    st = hc.Store(L, d, CT, capacity_chunks=4, pinned=False)
    rows = np.zeros((8, d), dtype=np.uint16)
    with pytest.raises(hc.HCacheError) as e:        # layer 1 before layer 0
        st.append(1, 1, rows, 1)
    assert e.value.status == hc.HC_ESTATE
    with pytest.raises(hc.HCacheError) as e:
        st.append(1, 2, rows, 1)
    assert e.value.status == hc.HC_ERANGE
    st.append(1, 0, rows, 8)                        # 2 chunks
    st.append(1, 1, rows, 8)                        # 2 chunks -> arena full
    with pytest.raises(hc.HCacheError) as e:
        st.append(2, 0, rows, 1)
    assert e.value.status == hc.HC_ERANGE
    assert st.tokens(2, 0) == 0
    with pytest.raises(hc.HCacheError):
        st.drop(99)
    st.drop(1)
    assert st.tokens(1, 0) == 0
    st.append(2, 0, rows, 5)                        # reuses freed chunks
    assert st.tokens(2, 0) == 5
    assert st.chunk(2, 0, 1)[1] == 1                # tail chunk holds one row
    st.append(2, 0, rows, 0)                        # empty append is a no-op
    st.destroy()


def test_store_rows_stay_regular_under_interleaving_and_reuse(hc):
    """Four contexts appended in decode order (a few tokens at a time, taking turns), two of
    them dropped, two new ones appended into the holes: every context's chunks of a layer stay
    L slots apart in long runs (the spacing the strided loader needs), and every byte reads back."""
    L, d, CT, T = 4, 8, 4, 96
    n_idx = T // CT
    st = hc.Store(L, d, CT, capacity_chunks=L * (4 * n_idx + 8), pinned=False)
    rng = np.random.default_rng(4)
    data = {s: rng.integers(0, 65536, size=(L, T, d), dtype=np.uint16) for s in (1, 2, 3, 4, 5, 6)}

    def feed(ids):
        for a in range(0, T, 3):
            for s in ids:
                for l in range(L):
                    st.append(s, l, np.ascontiguousarray(data[s][l, a:a + 3]), 3)

    def runs(s, l):
        slots = [(st.chunk(s, l, c)[0] - st.chunk(1, 0, 0)[0]) // (CT * d * 2) for c in range(n_idx)]
        gaps = np.diff(slots)
        assert all((slots[c] - l) % L == 0 for c in range(n_idx))       # slot l of a row
        return 1 + int(np.sum(gaps != L))

    feed((1, 2, 3, 4))
    for s in (1, 2, 3, 4):
        assert max(runs(s, l) for l in range(L)) <= 3, "interleaved arrivals broke a context into many runs"
    st.drop(2)
    st.drop(4)
    feed((5, 6))
    for s in (1, 3, 5, 6):
        assert max(runs(s, l) for l in range(L)) <= 4
        for l in range(L):
            got = np.concatenate([read_chunk(st, s, l, c, d) for c in range(n_idx)])
            assert np.array_equal(got, data[s][l])
    st.destroy()


def test_store_bad_arguments(hc):
    for args in [(0, 8, 4, 4), (2, 0, 4, 4), (2, 8, 0, 4), (2, 8, 4, 0), (2, 12, 4, 4)]:
        with pytest.raises(hc.HCacheError) as e:
            hc.Store(*args, pinned=False)
        assert e.value.status == hc.HC_EINVAL


def test_create_fails_loudly_without_gpu(hc):
    import torch
    if torch.cuda.is_available():
        pytest.skip("a GPU is present")
    with pytest.raises(hc.HCacheError) as e:
        hc.Context(good_desc(hc))
    assert e.value.status == hc.HC_EHIP


def test_partition_matches_oracle(hc):
    """The library's closed-form layer partition against the oracle (which is itself pinned to
    the brute-force optimum and to the schedules the paper prints)."""
    rng = np.random.default_rng(8)
    for _ in range(500):
        n = int(rng.integers(1, 129))
        io_h, c_h = float(rng.uniform(0.1, 3)), float(rng.uniform(0.1, 3))
        io_kv, c_tok = io_h * float(rng.uniform(1.01, 6)), c_h * float(rng.uniform(1.01, 20))
        l_h, l_o, comp = hc.partition_layers(n, io_h, io_kv, c_h, c_tok)
        want = oracle.partition_layers(n, io_h, io_kv, c_h, c_tok)
        assert (l_h, l_o, "kv" if comp == 0 else "re") == want
    assert hc.partition_layers(32, 1.0, 2.0, 1.1, 10.0) == (31, 1, 0)
    # the ceiling is the plain one: a quotient 8.4e-10 above 9 gives 10 layers, on both sides
    for c_h, want in ((2.0, 9), (2.0 - 2.0 ** -30, 10), (2.0 + 2.0 ** -30, 9)):
        assert hc.partition_layers(10, 1.0, 9.0, c_h, 50.0) == (want, 10 - want, 0)
        assert oracle.partition_layers(10, 1.0, 9.0, c_h, 50.0) == (want, 10 - want, "kv")
    for bad in [(0, 1, 1, 1, 1), (4, 0, 1, 1, 1), (4, 1, -1, 1, 1), (4, 1, 1, 0, 1), (4, 1, 1, 1, float("nan")),
                (4, 2, 1, 3, 9), (4, 1, 2, 3, 2)]:
        with pytest.raises(hc.HCacheError) as e:
            hc.partition_layers(*bad)
        assert e.value.status == hc.HC_EINVAL


def test_bench_refuses_more_than_one_gpu():
    """This build runs on one GPU; asking the benchmark for more must say so and fail."""
    import subprocess
    import sys
    res = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                         capture_output=True, text=True, timeout=120)
    assert res.returncode != 0
    assert "one GPU" in res.stderr
    assert res.stdout.strip() == ""


def test_header_is_plain_c_and_links(hc, tmp_path):
    """include/hcache.h compiles as pedantic C99 and a C program can call the library."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler")
    libdir = os.path.dirname(hc.lib_path())
    exe = str(tmp_path / "cabi_smoke")
    rocm_lib = "/opt/rocm/lib"
    cmd = [gcc, "-std=c99", "-pedantic", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"),
           os.path.join(ROOT, "tests", "cabi_smoke.c"), "-o", exe, "-L", libdir, "-lhcache",
           f"-Wl,-rpath,{libdir}", f"-Wl,-rpath,{rocm_lib}"]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, (res.returncode, res.stdout, res.stderr)
    assert "hcache-mi355x" in res.stdout


def test_store_index_is_safe_across_threads(hc):
    """Appends, queries and drops of different contexts from several host threads at once."""
    import threading
    L, d, CT, per_ctx = 2, 64, 4, 40
    n_threads, rounds = 6, 30
    st = hc.Store(L, d, CT, capacity_chunks=n_threads * L * (per_ctx // CT) + 8, pinned=False)
    errors = []

    def worker(tid):
        try:
            rng = np.random.default_rng(tid)
            for r in range(rounds):
                sid = tid * 1000 + r
                rows = rng.integers(0, 65536, size=(per_ctx, d), dtype=np.uint16)
                for a in range(0, per_ctx, 10):
                    for l in range(L):
                        st.append(sid, l, np.ascontiguousarray(rows[a:a + 10]), 10)
                    st.tokens((tid + 1) % n_threads * 1000 + r, 0)      # someone else's context
                for l in range(L):
                    assert st.tokens(sid, l) == per_ctx
                    got = np.concatenate([read_chunk(st, sid, l, c, d) for c in range(per_ctx // CT)])
                    assert np.array_equal(got, rows)
                st.drop(sid)
        except Exception as e:                               # noqa: BLE001 - reported below
            errors.append((tid, repr(e)))

    threads = [threading.Thread(target=worker, args=(t,)) for t in range(n_threads)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    st.destroy()


def test_tile_map_covers_every_tile_once_and_balances_the_xcds(hc):
    """The kernel's slot -> tile map (the same function the kernel compiles, evaluated on the
    host): for a range of layer shapes and launch depths every tile of every layer belongs to
    exactly one slot, a slot's workgroup stays inside its XCD's super tiles (slot % 8), and over
    an eight-layer launch the XCDs differ by at most one super tile's worth of tiles."""
    import numpy as np
    shapes = [(1024, 8192), (4096, 2048), (7168, 2048), (5120, 1536), (5120, 1600), (192, 257),
              (128, 1), (640, 600), (1024, 32768), (384, 280)]
    for d_kv, n_tok in shapes:
        for n_layers in (1, 3, 8):
            shape, tiles = hc.diag_tile_map(d_kv, n_tok, n_layers)
            nf, nt, slots = shape["nf"], shape["nt"], shape["slots"]
            assert slots % 8 == 0 and shape["gf"] * shape["gt"] <= 32
            assert nf == 2 * (-(-d_kv // 128) * 128) // 256 and nt == -(-n_tok // 256)
            per_xcd = np.zeros(8, dtype=np.int64)
            for l in range(n_layers):
                t = tiles[l]
                real = t[:, 0] >= 0
                assert ((t[real, 0] < nf) & (t[real, 1] < nt)).all()
                flat = t[real, 0].astype(np.int64) * nt + t[real, 1]
                assert flat.size == nf * nt and np.unique(flat).size == nf * nt, (d_kv, n_tok, n_layers, l)
                # workgroup l * slots + w runs on XCD (l * slots + w) % 8 = w % 8
                per_xcd += np.bincount(np.nonzero(real)[0] % 8, minlength=8)
                # the tiles an XCD works on in one layer come from whole super tiles
                for x in range(8):
                    tx = t[real & (np.arange(slots) % 8 == x)]
                    supers = {(int(a) // shape["gf"], int(b) // shape["gt"]) for a, b in tx}
                    assert len(tx) <= len(supers) * shape["gf"] * shape["gt"]
            if n_layers == 8:
                assert per_xcd.max() - per_xcd.min() <= shape["gf"] * shape["gt"], (d_kv, n_tok, per_xcd)
    # a single-layer launch applies no rotation: slot w of layer 0 is the same in both
    one = hc.diag_tile_map(7168, 2048, 1)[1]
    many = hc.diag_tile_map(7168, 2048, 8)[1]
    assert (one[0] == many[0]).all() and not (many[1] == many[0]).all()


def test_split_plan_invariants(hc):
    """hc_diag_split_plan (host logic only).  Whenever a launch is split: its last round of 256
    workgroups would be at most half full; the whole tiles are the whole rows of token tiles
    that fit the full rounds and their slot grid is the one an unsplit launch of that many
    tokens gets; every share of a split loop is at least 8 x 64 channels; the workspace holds
    one slot per split workgroup (256 at most).  Mode 1 splits a subset of what mode 2 splits,
    in the same way, and only where its cost model (1.5 x the 64-channel steps of a whole tile against
    steps / ways + 0.143 x tiles x ways + 15) says so; mode 0 never splits."""
    for d_model in (256, 1024, 2048, 4096, 5120, 7168, 8192):
        nm = d_model // 64
        for d_kv in (64, 640, 1024, 5120, 7168):
            for n_tok in list(range(1, 4500, 173)) + [256, 1536, 1600, 2048, 8192, 16384]:
                p0, p1, p = (hc.diag_split_plan(d_model, d_kv, n_tok, m) for m in (0, 1, 2))
                nf, nt = p["nf"], p["nt"]
                assert nf == 2 * (-(-d_kv // 128) * 128) // 256 and nt == -(-n_tok // 256)
                unsplit = dict(p, split=0, nt_main=nt, n_tail=0, n_split=1, main_slots=0, fixup_workgroups=0)
                assert p0 == unsplit and p1 in (unsplit, p)
                if not p["split"]:
                    assert p == unsplit
                    continue
                rem = nf * nt % 256
                assert 0 < rem <= 128
                assert nf * p["nt_main"] <= nf * nt - rem                   # whole tiles stay within the full rounds
                assert nf * (p["nt_main"] + 1) > nf * nt - rem              # ... and no further row would
                assert p["n_tail"] == nf * (nt - p["nt_main"]) > 0
                assert 2 <= p["n_split"] <= 16 and p["n_tail"] * p["n_split"] <= 256
                assert nm // p["n_split"] >= 8
                assert p["fixup_workgroups"] == 4 * p["n_tail"]
                if p["nt_main"]:
                    assert p["main_slots"] == hc.diag_tile_map(d_kv, 256 * p["nt_main"], 1)[0]["slots"]
                else:
                    assert p["main_slots"] == 0
                cost = nm / p["n_split"] + 0.143 * p["n_tail"] * p["n_split"] + 15
                if abs(cost - 1.5 * nm) > 1e-3:
                    assert p1["split"] == (cost < 1.5 * nm), (d_model, d_kv, n_tok, cost)
    p = hc.diag_split_plan(5120, 5120, 1600)                                # 40 x 7 tiles
    assert (p["split"], p["nt_main"], p["n_tail"], p["n_split"], p["main_slots"]) == (1, 6, 40, 4, 256)
    assert hc.diag_split_plan(4096, 1024, 8192, 2)["split"] == 0            # 8 x 32 tiles: exactly one round
    assert hc.diag_split_plan(5120, 5120, 1536, 2)["split"] == 0            # 240 of 256: full enough
    assert hc.diag_split_plan(1024, 640, 600)["split"] == 0                 # narrow model: does not pay
    assert hc.diag_split_plan(1024, 640, 600, 2)["n_split"] == 2
    with pytest.raises(hc.HCacheError):
        hc.diag_split_plan(100, 64, 10)
    with pytest.raises(hc.HCacheError):
        hc.diag_split_plan(1024, 64, 10, 3)


def test_route_invariants(hc):
    """hc_diag_route (host logic only).  A context that asks for split launches gets the 256 x 256 tiles in
    every call, split as the plan says in single-layer ones; with splitting off no launch sums in another order (no split
    tiles, no few-token kernel); several layers never split and never take the few-token kernel."""
    for d_model in (64, 256, 1024, 4096, 8192):
        for d_kv in (64, 192, 1024, 7168):
            for n_tok in (1, 16, 65, 300, 1000, 2501, 16384):
                for norm in (hc.HC_NORM_RMS, hc.HC_NORM_LAYER):
                    for mode in (0, 1, 2):
                        kernel, blocks, ways, layers = hc.diag_route(d_model, d_kv, n_tok, 0, norm, mode)
                        plan = hc.diag_split_plan(d_model, d_kv, n_tok, mode)
                        where = (d_model, d_kv, n_tok, norm, mode, kernel, blocks, ways)
                        assert layers == 1 and ways == (plan["n_split"] if kernel == "tiles" else 1), where
                        assert blocks in {"tiles": (0,), "few": (1, 2, 3, 4), "rows128": (1, 2, 3, 4, 5)}[kernel], where
                        assert mode != 2 or kernel == "tiles", where
                        assert kernel != "few" or (mode == 1 and d_model >= 1024), where
                        assert blocks < 5 or norm == hc.HC_NORM_RMS, where
                        for n_layers in (1, 3, 8, 40):
                            kernel, blocks, ways, layers = hc.diag_route(d_model, d_kv, n_tok, n_layers, norm, mode)
                            assert kernel != "few" and ways == 1 and min(n_layers, 8) <= layers <= min(n_layers, 32)
                            assert mode != 2 or kernel == "tiles", (d_model, d_kv, n_tok, n_layers, norm)
    for bad in ((100, 64, 10), (1024, 60, 10), (1024, 64, 0), (1024, 64, 10, -1), (1024, 64, 10, 0, 2), (1024, 64, 10, 0, 0, 3)):
        with pytest.raises(hc.HCacheError):
            hc.diag_route(*bad)


# Measured on MI355X: (d_model, d_kv, tokens, us of the few-token kernel, us of the 256 x 256 tiles, whole or split)
FEW_TOKEN_TIMES = [
    (1024, 64, 400, 5.2, 26.4), (1024, 64, 6000, 36.5, 25.7), (1024, 64, 9000, 53.7, 26.4), (2048, 64, 1700, 15.2, 29.9),
    (2048, 64, 6000, 51.2, 34.9), (4096, 64, 2600, 38.5, 36.2), (4096, 64, 4000, 47.8, 39.8), (4096, 64, 6000, 76.0, 42.7),
    (4096, 128, 2600, 41.2, 37.2), (4096, 128, 4000, 51.1, 41.0), (8192, 128, 700, 25.2, 39.0), (8192, 128, 2600, 68.0, 46.9),
    (8192, 128, 4000, 96.4, 50.8), (4096, 1024, 40, 9.9, 26.8), (4096, 1024, 128, 12.1, 29.6), (8192, 1024, 40, 16.3, 30.6),
]


def test_few_token_kernel_only_where_it_was_measured_faster(hc):
    """The launch rule against measured times, narrow K/V parts and long contexts included (few row groups lie on few
    of the XCDs): a layer never goes to the few-token kernel where that took longer than the large tiles."""
    for d_model, d_kv, n_tok, few_us, tiles_us in FEW_TOKEN_TIMES:
        kernel = hc.diag_route(d_model, d_kv, n_tok)[0]
        assert kernel != "few" or few_us < tiles_us, (d_model, d_kv, n_tok, few_us, tiles_us)
    for d_model, d_kv, n_tok in ((4096, 1024, 40), (4096, 1024, 128), (8192, 1024, 40), (2048, 64, 400)):
        assert hc.diag_route(d_model, d_kv, n_tok)[0] == "few"


# Measured on MI355X: (d_model, d_kv, tokens, LayerNorm, {kernel: (us with the weights from memory, from the caches)}); "stream": tiles of
# 64 tokens with loader waves, "rows": the best of the tiles of 128 rows x 64 n tokens
FEW_OR_TILES_TIMES = [
    (1664, 8064, 35, 0, dict(few=(19.92, 15.64), stream=(17.61, 11.76), rows=(20.46, 13.27))),
    (1408, 1152, 322, 0, dict(few=(13.93, 12.75), stream=(9.97, 9.24), rows=(12.03, 11.19))),
    (1344, 3264, 125, 0, dict(few=(15.4, 11.51), stream=(13.7, 8.8), rows=(14.53, 10.28))),
    (1280, 256, 1607, 1, dict(few=(14.03, 13.58), stream=(10.05, 9.43), rows=(12.29, 11.19))),
    (5376, 7808, 63, 0, dict(few=(44.54, 33.91), stream=(43.64, 28.19), rows=(46.06, 29.46))),
    (1856, 6656, 64, 1, dict(few=(22.39, 16.12), stream=(20.45, 13.28), rows=(22.74, 14.92))),
    (1920, 256, 2036, 0, dict(few=(18.75, 17.4), stream=(15.87, 12.79), rows=(17.19, 14.44))),
]


def test_few_token_kernel_only_where_no_tiles_are_estimated_faster(hc):
    """Shapes whose tiles of 64 tokens, with and without loader waves, are both faster than the few-token kernel: the margin
    that one of them gives it does not carry it past the other."""
    for d_model, d_kv, n_tok, norm, us in FEW_OR_TILES_TIMES:
        kernel = "few" if hc.diag_route(d_model, d_kv, n_tok, 0, norm)[0] == "few" else "stream" if hc.diag_tile(d_model, d_kv, n_tok, 0, norm)[2] else "rows"
        where = (d_model, d_kv, n_tok, norm, kernel, us)
        assert all(a <= 1.05 * b for k in us for a, b in zip(us[kernel], us[k])), where
    assert hc.diag_route(5120, 5120, 41)[0] == "few"       # 27.4 us, 32.6 on tiles with loader waves


# Measured on MI355X: (d_model, d_kv, tokens, layers, {layers in the first launch: us of the call}), 256 x 256 tiles
LAYERS_PER_LAUNCH_TIMES = [
    (640, 2816, 239, 10, {8: 56.8, 10: 36.8}), (256, 2688, 173, 10, {8: 32.0, 10: 23.5}),
    (256, 3456, 72, 9, {8: 30.3, 9: 22.3}), (128, 768, 271, 20, {16: 36.2, 20: 27.1}),
    (1344, 256, 2179, 10, {8: 132.5, 10: 101.0}), (5056, 2496, 1, 9, {8: 205.6, 9: 100.5}),
    (4672, 3008, 32, 9, {8: 203.5, 9: 111.4}), (1152, 1152, 529, 9, {8: 92.6, 9: 71.8}),
    (4096, 1024, 600, 32, {8: 381.0, 10: 578.0}),
]


def test_layers_per_launch_against_measured_times(hc):
    """How many layers of a short context go into a launch: the count that was measured fastest."""
    for d_model, d_kv, n_tok, n_layers, us in LAYERS_PER_LAUNCH_TIMES:
        n = hc.diag_route(d_model, d_kv, n_tok, n_layers, mode=2)[3]
        assert n in us and us[n] == min(us.values()), (d_model, d_kv, n_tok, n_layers, n, us)
    # 256 tiles or more a layer: eight; never more than 32; a call of at most eight layers is one launch
    assert hc.diag_route(4096, 1024, 8192, 32)[3] == 8 and hc.diag_route(256, 128, 20, 100)[3] <= 32
    assert hc.diag_route(4096, 1024, 600, 8)[3] == 8


def test_chip_load_matches_the_tile_map(hc, tmp_path):
    """ChipLoad (the closed form the launch rules use) against a count over the tile map, which the kernels
    compile: the workgroup of slot w of layer l runs on XCD (l slots + w) % 8, and the ids of an XCD go round its four
    engines."""
    import shutil
    import subprocess
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    src = tmp_path / "load.cpp"
    src.write_text("""
#include <cstdio>
#include "hcache_internal.h"
using namespace hc;
int main() {
  int bad = 0, n = 0;
  for (int nf : {1, 2, 3, 5, 8, 9, 10, 18, 40, 80, 112})
    for (int nt : {1, 2, 3, 5, 7, 16, 33})
      for (int live = nf > 1 ? nf - 1 : 1; live <= nf; ++live) {
        TileGrid g;
        const int slots = choose_tile_grid(nf, nt, g);
        const ChipLoad load(g, slots, live);
        int count[32] = {};
        for (int l = 0; l < 33; ++l) {
          int most = 0;
          for (int c : count) most = c > most ? c : most;
          bad += load.busiest(l) != most;
          ++n;
          for (int w = 0; w < slots; ++w) {
            int f, t;
            const int id = l * slots + w;
            if (slot_to_tile(g, w, l, f, t) && f < live) ++count[(id & 7) * 4 + (id >> 3 & 3)];
          }
        }
      }
  std::printf("%d of %d differ\\n", bad, n);
  return bad != 0;
}
""")
    inc = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2410_05004_amd", "csrc")]
    exe = tmp_path / "load"
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", inc[0], "-I", inc[1],
                    str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_rows_of_tiles_with_loader_waves(tmp_path):
    """tile_base_row and tile_row, as the kernel uses them: live rows are the tile's own, the others lie within the tokens, none is
    read much more often than the rest, and byte offsets fit 32 bits (a tile of 192 rows alone allows d_model of 10 million)."""
    import shutil
    import subprocess
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    src = tmp_path / "rows.cpp"
    src.write_text("""
#include <cstdio>
#include <vector>
#include "hcache_internal.h"
using namespace hc;
int main() {
  long bad = 0, n = 0;
  for (int T = 64; T <= 192; T += 32)
    for (int n_tok = 1; n_tok <= 3 * T + 1; ++n_tok)
      for (int d : {1088, 7168, 1 << 22, (1 << 22) + 64, 10 << 20})
        for (int t0 = 0; t0 < n_tok; t0 += T) {
          const int base = tile_base_row(t0, n_tok, T, d), live = n_tok - t0 < T ? n_tok - t0 : T;
          std::vector<int> reads(n_tok);
          bad += base < 0 || (t0 > 0 && live < 8 && d <= 1 << 22) != (base < t0);
          for (int r = 0; r < T; ++r, ++n) {
            const int off = tile_row(r, t0, base, n_tok), row = base + off;
            if (off < 0 || row < 0 || row >= n_tok) { ++bad; continue; }
            bad += r < live && row != t0 + r;
            bad += (unsigned long long)off * d * 2 + 128 > 0xffffffffull;
            bad += ++reads[row] > (base < t0 ? (T + 15) / 16 : (T + live - 1) / live);
          }
        }
  std::printf("%ld of %ld\\n", bad, n);
  return bad != 0;
}
""")
    inc = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2410_05004_amd", "csrc")]
    exe = tmp_path / "rows"
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", inc[0], "-I", inc[1],
                    str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_layers_per_launch_prices_the_last_launch(hc, tmp_path):
    """plan_layers over layer counts that leave a remainder: by the rule's own estimates, the whole call (full launches and
    the last one, which goes its own way) takes no longer than with any other count it weighs, and a launch on the tiles of
    288 or 320 tokens fills at most one round."""
    import shutil
    import subprocess
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    src = tmp_path / "plan.cpp"
    src.write_text("""
#include <cstdio>
#include "hcache_internal.h"
using namespace hc;
int main() {
  int bad = 0, n_all = 0, n_wide = 0;
  const int widths[][2] = {{4096, 1024}, {8192, 1024}, {2112, 320}, {5120, 640}, {4096, 4096}, {5120, 5120}};
  for (auto& w : widths)
    for (int layers : {9, 16, 20, 24, 33, 40, 48, 80})
      for (int tok : {250, 257, 270, 288, 289, 300, 320, 321, 577, 600, 1100, 1153, 1601}) {
        RestoreArgs a{};
        a.d_model = w[0];
        a.d_kv = w[1];
        a.d_kv_pad = round_up(w[1], kPartAlign);
        a.n_tok = tok;
        set_split_rule(a, 1, nullptr, true);
        Route route;
        const int n = plan_layers(a, layers, route);
        auto call_us = [&](float us, int per) { return us * (layers / per) + (layers % per ? restore_route(a, layers % per).us : 0.f); };
        const float us = call_us(route.us, n);
        int per = layers_per_launch(2 * a.d_kv_pad / kTileF, (tok + kTileT - 1) / kTileT, layers);
        if (per > layers) per = layers;
        float least = call_us(restore_route(a, per).us, per);
        for (int b = 9; b <= 10; ++b) {
          int nb = b;
          const int wide = wide_layers_per_launch(a.d_kv, tok, nb, layers);
          if (wide <= per) continue;
          const float t = call_us(kWideCallPromise * wide_us(a.d_kv, a.d_model, tok, wide, nb), wide);
          if (t < least) least = t;
        }
        const int tiles = 2 * a.d_kv_pad / kTileF * ((tok + 32 * route.nb - 1) / (32 * (route.nb > 0 ? route.nb : 1)));
        const bool over = route.kind == Route::kWide && n > per && tiles * n > kChipCUs;
        if (us > 1.0001f * least || over) {
          ++bad;
          std::printf("%d onto %d, %d layers of %d: %d a launch, kernel %d x %d, %.1f us, least %.1f\\n", w[0], 2 * w[1], layers, tok, n, route.kind, route.nb, us, least);
        }
        ++n_all;
        n_wide += n > per;
      }
  std::printf("%d of %d\\n", bad, n_all);
  return bad != 0 || n_wide < 20;
}
""")
    inc = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2410_05004_amd", "csrc")]
    exe = tmp_path / "plan"
    subprocess.run([hipcc, "-x", "hip", "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", inc[0], "-I", inc[1],
                    str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


# Measured on MI355X, one call over and over: (d_model, d_kv, tokens, layers in the call, {layers in the first launch: us}), the 256-token
# tiles or those of 64 n tokens up to 16 layers, those of 288 or 320 tokens beyond, or where they fill a round with fewer
WHOLE_CALL_TIMES = [
    (4096, 1024, 257, 20, {20: 125.1, 16: 157.5}), (4096, 1024, 320, 20, {20: 136.2, 16: 163.8}),
    (8192, 1024, 288, 20, {20: 232.5, 16: 294.7}), (8192, 1024, 320, 20, {20: 256.9, 16: 300.2}),
    (4096, 1024, 320, 24, {24: 151.4, 16: 185.7}), (8192, 1024, 300, 24, {24: 275.7, 16: 333.0}),
    (8192, 1024, 257, 33, {16: 477.4, 32: 337.3}), (4096, 1024, 300, 40, {16: 306.5, 32: 247.3}),
    (8192, 1024, 289, 80, {16: 1123.1, 32: 896.6}), (5120, 640, 257, 48, {16: 356.2, 32: 283.7}),
    (5120, 640, 289, 33, {24: 227.7, 32: 211.6}), (4096, 1024, 600, 16, {8: 192.7, 16: 158.4}),
    (8192, 1024, 577, 80, {8: 1846.0, 16: 1463.4}), (5120, 640, 1153, 20, {10: 560.0, 12: 434.3}),
    (2112, 320, 1153, 20, {20: 117.5, 16: 111.1}), (2112, 320, 577, 33, {24: 120.5, 32: 102.5}),
]


def test_whole_calls_against_measured_times(hc):
    """Layers in the first launch of calls that leave a remainder: the count that was measured fastest."""
    for d_model, d_kv, n_tok, n_layers, us in WHOLE_CALL_TIMES:
        n = hc.diag_route(d_model, d_kv, n_tok, n_layers)[3]
        assert n in us and us[n] == min(us.values()), (d_model, d_kv, n_tok, n_layers, n, us)


# Measured on MI355X, weights not lately read: (d_model, d_kv, tokens, layers in the call or 0 for a single-layer call,
# LayerNorm, us on the 256 x 256 tiles (whole or split), [us on tiles of 128 rows x 64, 128, .. 320 tokens])
ROWS128_TIMES = [
    (4096, 1024, 11650, 0, 0, 196.5, [298.8, 263.7, 231.2, 214.6, 301.4]),
    (4096, 1024, 12286, 0, 0, 205.5, [307.3, 267.5, 233.4, 214.5, 304.6]),
    (7872, 64, 8627, 0, 0, 65.36, [107.52, 79.21, 97.24, 117.34, 183.67]),
    (5312, 2304, 217, 6, 1, 112.76, [154.88, 151.82, 183.74, 165.87, 233.05]),
    (192, 192, 13144, 0, 1, 14.6, [14.24, 16.59, 21.33, 14.81, 16.77]),
    (64, 1280, 455, 4, 1, 13.63, [12.87, 15.06, 18.84, 14.84, 16.46]),
    (768, 576, 6802, 0, 0, 27.53, [31.73, 37.22, 33.3, 37.91, 26.06]),
    (4096, 1024, 179, 20, 0, 99.33, [136.33, 127.88, 119.94, 133.79, 199.46]),
    (7168, 576, 226, 20, 1, 160.41, [208.39, 198.08, 222.4, 214.1, 316.01]),
    (1088, 576, 714, 3, 0, 27.65, [20.74, 36.49, 31.65, 35.74, 41.33]),
    (8192, 1024, 138, 20, 1, 200.49, [259.18, 242.33, 212.47, 245.01, 344.6]),
    (4800, 576, 765, 3, 0, 88.8, [65.64, 114.52, 93.85, 109.44, 132.34]),
    (8192, 1024, 616, 5, 1, 171.16, [192.78, 204.72, 183.28, 219.97, 145.78]),
    (4096, 1024, 144, 20, 0, 103.69, [132.68, 123.67, 115.17, 127.99, 190.78]),
    (8192, 1024, 395, 9, 1, 175.8, [220.66, 217.69, 200.11, 232.66, 333.92]),
    (8192, 1024, 637, 6, 0, 165.17, [208.2, 203.96, 183.15, 206.23, 170.66]),
    (192, 64, 89, 9, 0, 13.89, [8.35, 11.54, 12.8, 14.04, 15.38]),
    (1600, 768, 5, 4, 0, 32.29, [14.85, 16.54, 18.81, 21.57, 25.35]),
    (1088, 960, 1, 2, 0, 23.64, [11.4, 12.19, 13.95, 15.87, 18.29]),
    (128, 192, 558, 13, 0, 18.5, [12.02, 14.86, 15.43, 16.38, 16.73]),
    (64, 256, 80, 0, 0, 8.98, [4.9, 6.77, 8.15, 8.81, 10.06]),
    (192, 448, 117, 0, 0, 11.02, [5.02, 6.83, 8.03, 9.13, 9.92]),
    (256, 256, 147, 0, 0, 11.97, [6.11, 8.39, 10.53, 12.01, 13.45]),
    (5504, 256, 47, 24, 0, 104.65, [46.86, 54.36, 61.98, 72.49, 85.54]),
]


def test_tiles_of_128_rows_only_where_they_were_measured_faster(hc):
    """The launch rule against measured times: launches whose busiest XCD or shader engine needs a round more than
    the chip as a whole would, and some that the tiles of 128 rows are there for.  The chosen kernel takes at
    most 1.05 of the large tiles' time, and at most 1.1 of the fastest's where that is 128-row tiles by far."""
    for d_model, d_kv, n_tok, n_layers, norm, tiles_us, rows_us in ROWS128_TIMES:
        kernel, blocks, _, _ = hc.diag_route(d_model, d_kv, n_tok, n_layers, norm)
        assert kernel != "few"
        rows, tokens, loaders, _ = hc.diag_tile(d_model, d_kv, n_tok, n_layers, norm)
        if loaders or (rows, tokens) in ((256, 288), (256, 320)):   # kernels of their own: with their times in TILE_TIMES
            assert (d_model, d_kv, n_tok, n_layers, norm) in [r[:5] for r in TILE_TIMES]
            continue
        assert (rows, tokens) == ((256, 256) if kernel == "tiles" else (128, 64 * blocks))
        us = tiles_us if kernel == "tiles" else rows_us[blocks - 1]
        where = (d_model, d_kv, n_tok, n_layers, norm, kernel, blocks, us, tiles_us, rows_us)
        assert us <= 1.05 * tiles_us, where
        assert min(rows_us) > 0.7 * tiles_us or us <= 1.1 * min(rows_us), where


# Measured on MI355X: (d_model, d_kv, tokens, layers in the call or 0, LayerNorm, {(rows, tokens, loader waves) of a tile: us}), the kernels of
# a row on one machine; 256 x 256 tiles whole or split; a single layer mostly with the weights from memory, several mostly over and over
TILE_TIMES = [
    (4224, 3584, 853, 0, 0, {(128, 96, 4): 86.8, (128, 256, 0): 66.9}),      # nine token tiles: the weights into the L2s nine times
    (4864, 2816, 993, 0, 0, {(128, 96, 4): 97.7, (128, 256, 0): 81.4}),
    (3072, 3328, 803, 0, 0, {(128, 96, 4): 63.2, (128, 256, 0): 51.4}),
    (7872, 4608, 615, 0, 1, {(128, 96, 4): 155.5, (256, 256, 0): 129.4}),
    (1728, 1344, 2182, 0, 0, {(128, 96, 4): 38.4, (128, 256, 0): 32.2}),
    (5120, 5120, 346, 0, 1, {(128, 128, 4): 56.5, (128, 128, 0): 62.7}),     # both bound by that
    (3136, 896, 3216, 0, 1, {(128, 192, 4): 44.5, (128, 192, 0): 51.7}),
    (7168, 7168, 191, 4, 1, {(128, 192, 4): 220.5, (256, 256, 0): 191.5}),   # second rounds from memory
    (5120, 5120, 173, 4, 0, {(128, 192, 4): 136.0, (256, 256, 0): 120.0}),
    (5120, 5120, 161, 3, 0, {(128, 192, 4): 118.5, (256, 256, 0): 106.0}),
    (5120, 5120, 120, 4, 0, {(128, 128, 4): 120.1, (128, 128, 0): 128.8}),
    (4096, 1024, 2501, 0, 0, {(128, 160, 4): 48.1, (128, 192, 0): 54.4}),
    (4800, 576, 765, 3, 0, {(128, 64, 4): 74.4, (128, 64, 0): 76.7, (256, 256, 0): 92.9}),
    (1600, 768, 5, 4, 0, {(128, 64, 4): 14.3, (128, 64, 0): 20.95, (256, 256, 0): 33.3}),
    (5120, 5120, 1601, 0, 0, {(256, 288, 0): 147.5, (256, 256, 0): 163.5}),
    (4096, 1024, 300, 32, 0, {(256, 320, 0): 185.0, (256, 256, 0): 247.0}),
    (4096, 4096, 277, 8, 0, {(256, 288, 0): 148.0, (256, 256, 0): 213.4, (128, 160, 4): 203.0}),
    (4096, 1024, 1128, 8, 0, {(256, 288, 0): 139.5, (128, 192, 4): 137.0, (256, 256, 0): 178.4}),
]


def test_tiles_with_loader_waves_only_where_they_were_measured_faster(hc):
    """The launch rule against measured times of tiles with and without loader waves and of the large ones: the tile
    chosen takes at most 1.05 of the fastest of those measured."""
    for d_model, d_kv, n_tok, n_layers, norm, us in TILE_TIMES:
        tile = hc.diag_tile(d_model, d_kv, n_tok, n_layers, norm)[:3]
        best = min(us.values())
        assert tile not in us or us[tile] <= 1.05 * best, (d_model, d_kv, n_tok, n_layers, norm, tile, us)
        assert tile in us or tile[2] == 0, (d_model, d_kv, n_tok, n_layers, norm, tile, us)


def test_token_sweep_names_the_tile_of_a_launch(hc):
    """sweep_tokens prints the tile that runs: 128 rows with and without loader waves, 256 rows of more than 256 tokens."""
    from paper_2410_05004_amd.sweep_tokens import kernel_name
    for shape, name in (((4096, 1024, 37, 0), "few tokens, 16"), ((4096, 1024, 2501, 0), "128 rows x 160, loader waves"),
                        ((5120, 5120, 1601, 0), "256 rows x 288"), ((704, 576, 1601, 0), "128 rows x 128"),
                        ((4096, 1024, 8192, 0), "whole tiles")):
        assert kernel_name(hc, *shape) == name, (shape, kernel_name(hc, *shape))
