"""GPU parity: the HIP restoration path, called through the C ABI, against the fp64 oracle
on the same seeded inputs.  Indexing (which page/slot is written) must match exactly;
values must agree within 2e-2 x the oracle's per-head RMS (bf16 inputs, fp32 accumulation,
one bf16 rounding of the output)."""
import numpy as np
import pytest

import synthetic as syn
import oracle.hcache_oracle as oracle
import gpu_harness as gh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    import paper_2410_05004_amd as hc
    return hc


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


def run_single(hc, torch, case, desc, positions, block_table, num_pages, layer=0, split=None):
    """One hc_restore_kv call under split mode `split` (None: the default), or, "whole", on whole 256 x 256 tiles."""
    ctx = hc.Context(desc)
    if split not in (None, "whole"):
        ctx.set_split(split)
    pool = gh.new_pool(num_pages, desc.block_size, desc.n_kv_heads, desc.head_dim)
    s = gh.stream_handle()
    d_w, d_g = gh.to_dev_bf16(case.wkv_bits), gh.to_dev_bf16(case.gamma_bits)
    ctx.set_layer_weights(layer, d_w, d_g, s)
    ctx.set_kv_pool(layer, pool, num_pages)
    d_x = gh.to_dev_bf16(case.x_bits) if len(case.x_bits) else None
    d_pos, d_bt = gh.to_dev_i32(positions), gh.to_dev_i32(block_table)
    if split == "whole":
        gh.restore_whole_tiles(ctx, layer, d_x, d_pos, len(positions), d_bt, len(block_table), s)
    else:
        ctx.restore_kv(layer, d_x, d_pos, len(positions), d_bt, len(block_table), s)
    flags = ctx.poll_device_error(s)
    bits = gh.pool_bits(pool)
    ctx.destroy()
    return bits, flags


def oracle_single(case, desc, positions, block_table, num_pages):
    pool = np.full((num_pages, 2, desc.block_size, desc.n_kv_heads, desc.head_dim), np.nan)
    oracle.restore_kv(pool, case.x, case.gamma, case.wkv, positions, block_table,
                      **gh.oracle_kw(desc))
    return pool


# ---------------------------------------------------------------------------------------
def test_tiny_workload_all_layers(hc, torch):
    """Workload 0 (2 layers, d=256, 4 KV heads of 64, T=128), every element."""
    w = syn.WORKLOADS[0]
    desc = gh.desc_of_workload(hc, w)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    bt, num_pages = syn.block_table(w, w.tokens)
    pos = np.arange(w.tokens, dtype=np.int32)
    d_pos, d_bt = gh.to_dev_i32(pos), gh.to_dev_i32(bt)
    keep = []
    for l in range(w.n_layers):
        wkv, gamma = syn.layer_weights(w, l)
        x = syn.layer_hidden(w, l)
        pool = gh.new_pool(num_pages, w.block_size, w.n_kv_heads, w.head_dim)
        d_w, d_g, d_x = gh.to_dev_bf16(wkv), gh.to_dev_bf16(gamma), gh.to_dev_bf16(x)
        keep += [d_w, d_g, d_x]
        ctx.set_layer_weights(l, d_w, d_g, s)
        ctx.set_kv_pool(l, pool, num_pages)
        ctx.restore_kv(l, d_x, d_pos, w.tokens, d_bt, len(bt), s)
        assert ctx.poll_device_error(s) == 0
        ora = np.full((num_pages, 2, w.block_size, w.n_kv_heads, w.head_dim), np.nan)
        oracle.restore_kv(ora, syn.bf16_bits_to_f64(x), syn.bf16_bits_to_f64(gamma),
                          syn.bf16_bits_to_f64(wkv), pos, bt, **gh.oracle_kw(desc))
        worst = gh.compare_pool(gh.pool_bits(pool), ora)
        print(f"layer {l}: worst err = {worst * gh.TOL:.3e} x RMS_head")
    ctx.destroy()


SHAPES = [
    # d_model, n_kv, hd, n_tok, style   (several token tiles + ragged tail; padded feature tiles)
    (1024, 6, 128, 600, 0),
    (512, 3, 64, 257, 0),      # d_kv = 192 -> part padded to 256 rows
    (512, 3, 64, 300, 1),      # interleaved RoPE
    (1024, 4, 128, 513, 1),
    (256, 1, 64, 1, 0),        # a single token, a single head
    (2048, 2, 128, 255, 0),
    (64, 1, 64, 70, 0),        # fewer d_model steps (2) than the weight ring is deep (4)
    (128, 2, 64, 300, 1),      # 4 steps: the ring is filled exactly once
    (192, 1, 64, 33, 0),
    # head dimensions other than 64 and 128: a tile's two pair groups are half a head (256) or
    # straddle heads (192), which the epilogue's write-out order has to follow
    (1024, 2, 256, 300, 0),
    (512, 2, 256, 100, 1),
    (1024, 2, 192, 280, 0),    # d_kv = 384: three pair groups per head, padded to 512 rows
    (512, 1, 192, 131, 1),
]


def shape_inputs(d_model, n_kv, hd, n_tok, style):
    """Seeded inputs of one SHAPES case (also read by the CPU feasibility test)."""
    rng = np.random.default_rng([11, d_model, n_kv, hd, n_tok, style])
    case = gh.LayerCase(rng, d_model, n_kv, hd, n_tok)
    B = 16
    offset = 1000                                   # starts mid-page: 1000 = 62*16 + 8
    n_blocks = (offset + n_tok + B - 1) // B
    num_pages = n_blocks + 7
    bt = rng.permutation(num_pages)[:n_blocks].astype(np.int32)
    # tokens in scrambled order: positions drive RoPE and the slot, not the row index
    pos = (offset + rng.permutation(n_tok)).astype(np.int32)
    return case, pos, bt, num_pages, offset


@pytest.mark.parametrize("d_model,n_kv,hd,n_tok,style", SHAPES)
def test_shapes_against_oracle(hc, torch, d_model, n_kv, hd, n_tok, style):
    case, pos, bt, num_pages, offset = shape_inputs(d_model, n_kv, hd, n_tok, style)
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv * 2, n_kv_heads=n_kv,
                        head_dim=hd, block_size=16, max_position=offset + n_tok, rope_style=style,
                        rope_theta=500000.0)
    ora = oracle_single(case, desc, pos, bt, num_pages)
    model = gh.model_pool(desc, case.x, case.gamma, case.wkv, pos, bt, num_pages)
    # as the library launches it by default and without another order of sums (mode 0); on whole 256 x 256 tiles;
    # where the shape allows it, with the d_model loops of these tiles split (mode 2)
    modes = [None, 0, "whole"] + ([2] if hc.diag_split_plan(d_model, n_kv * hd, n_tok, 2)["split"] else [])
    for split in modes:
        bits, flags = run_single(hc, torch, case, desc, pos, bt, num_pages, split=split)
        assert flags == 0
        worst = gh.compare_pool(bits, ora)
        equal = gh.assert_close_to_model(bits, model)
        print(f"split mode {split}: worst err = {worst * gh.TOL:.3e} x RMS_head; {equal:.5f} of the outputs "
              f"equal the two-rounding arithmetic model")


SPLIT_SHAPES = [
    # d_model, n_kv, hd, n_tok, style, expected (token tiles computed whole, split tiles, workgroups per split tile)
    (2048, 2, 128, 700, 1, (0, 6, 4)),       # 2 x 3 tiles, every one split four ways
    (4096, 1, 64, 100, 0, (0, 1, 8)),        # one ragged tile, eight shares of 512 channels
]


@pytest.mark.parametrize("d_model,n_kv,hd,n_tok,style,expect", SPLIT_SHAPES)
def test_split_launch_against_oracle(hc, torch, d_model, n_kv, hd, n_tok, style, expect):
    """Launches that split the d_model loop of their tiles (split workgroups, then the finishing
    launch), every element against the oracle; the same on whole tiles, and in the other split modes, where
    the few-token kernel and the tiles of 128 rows take these shapes.  A launch with whole tiles and split
    tiles in one grid needs more than 256 tiles: tests/test_gpu_fullsize.py."""
    plan = hc.diag_split_plan(d_model, n_kv * hd, n_tok, 2)
    assert plan["split"] == 1 and (plan["nt_main"], plan["n_tail"], plan["n_split"]) == expect, plan
    case, pos, bt, num_pages, offset = shape_inputs(d_model, n_kv, hd, n_tok, style)
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv * 2, n_kv_heads=n_kv,
                        head_dim=hd, block_size=16, max_position=offset + n_tok, rope_style=style,
                        rope_theta=500000.0)
    ora = oracle_single(case, desc, pos, bt, num_pages)
    assert [hc.diag_route(d_model, n_kv * hd, n_tok, mode=m)[0] for m in (2, 1, 0)] == ["tiles", "few", "rows128"]
    for split in (2, "whole", 1, 0):
        bits, flags = run_single(hc, torch, case, desc, pos, bt, num_pages, split=split)
        assert flags == 0
        worst = gh.compare_pool(bits, ora)
        print(f"split={split}: worst err = {worst * gh.TOL:.3e} x RMS_head", flush=True)


def test_split_and_unsplit_launches_agree_on_random_shapes(hc, torch):
    """Twenty seeded shapes (odd numbers of feature tiles, padded K/V parts, ragged token tiles,
    one to twelve tiles split two to sixteen ways, all three RoPE styles): the split launch
    writes exactly the cache elements the unsplit launch writes, and every value within one
    bf16 step of it, or, for values that are small because their terms cancel, within 2^-9 of
    the RMS of all values (the two differ only in the order of fp32 additions).  The unsplit launch
    computes whole 256 x 256 tiles, which test_shapes_against_oracle holds against the oracle."""
    rng = np.random.default_rng(2024)
    done = 0
    while done < 20:
        d_model = int(rng.choice([1024, 2048, 4096, 8192]))
        hd = int(rng.choice([64, 128]))
        n_kv = int(rng.integers(1, 7))
        n_tok = int(rng.integers(1, 900))
        style = int(rng.integers(0, 3))
        plan = hc.diag_split_plan(d_model, n_kv * hd, n_tok, 2)
        if not plan["split"]:
            continue
        done += 1
        case = gh.LayerCase(rng, d_model, n_kv, hd, n_tok)
        B = 16
        offset = int(rng.integers(0, 64))
        n_blocks = (offset + n_tok + B - 1) // B
        num_pages = n_blocks + 3
        bt = rng.permutation(num_pages)[:n_blocks].astype(np.int32)
        pos = (offset + rng.permutation(n_tok)).astype(np.int32)
        desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd,
                            block_size=B, max_position=offset + n_tok, rope_style=style)
        got = []
        for split in (2, "whole"):
            bits, flags = run_single(hc, torch, case, desc, pos, bt, num_pages, split=split)
            assert flags == 0
            got.append(bits)
        a, b = got
        m = gh.assert_same_but_for_order(a, b)
        assert m.sum() == 2 * n_tok * n_kv * hd, (d_model, n_kv, hd, n_tok, style)
        print(f"d_model {d_model} heads {n_kv} x {hd} tokens {n_tok} style {style}: {plan['n_tail']} tiles x "
              f"{plan['n_split']}; {np.mean(a[m] == b[m]):.4f} of the values bit-identical", flush=True)


@pytest.mark.parametrize("d_model,n_kv,hd,n_tok,style,norm,blocks", [
    (1024, 2, 64, 1, 0, 0, 1),     # one token; two supersteps of the loop per wave
    (1088, 3, 64, 16, 1, 0, 1),    # 17 supersteps over eight waves; padded K/V parts
    (4096, 8, 128, 17, 0, 0, 1),
    (1600, 2, 192, 33, 1, 0, 1),   # pair groups that straddle the tile's heads
    (2048, 16, 128, 49, 0, 0, 2),
    (1024, 40, 128, 50, 2, 0, 2),  # several workgroups per CU
    (2048, 1, 256, 130, 0, 0, 1),
    (1088, 32, 128, 33, 0, 0, 3),
    (4096, 8, 128, 201, 0, 0, 4),  # four blocks of tokens per workgroup, ragged last one
    (1472, 5, 128, 47, 0, 1, 1),   # LayerNorm
    (4096, 4, 64, 240, 2, 1, 1),
])
def test_few_tokens(hc, torch, d_model, n_kv, hd, n_tok, style, norm, blocks):
    """Layers that the few-token kernel takes, at the edges of its token blocks and loop shares:
    against the CPU model of the arithmetic (RMSNorm), and against whole 256 x 256 tiles but for the order of the
    fp32 additions."""
    assert hc.diag_route(d_model, n_kv * hd, n_tok, 0, norm)[:2] == ("few", blocks)
    rng = np.random.default_rng([77, d_model, n_kv, hd, n_tok, style, norm])
    case = gh.LayerCase(rng, d_model, n_kv, hd, n_tok)
    B, offset = 16, 40
    n_blocks = (offset + n_tok + B - 1) // B
    num_pages = n_blocks + 3
    bt = rng.permutation(num_pages)[:n_blocks].astype(np.int32)
    pos = (offset + rng.permutation(n_tok)).astype(np.int32)
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd,
                        block_size=B, max_position=offset + n_tok, rope_style=style, norm_kind=norm)
    bits, flags = run_single(hc, torch, case, desc, pos, bt, num_pages)
    whole, flags0 = run_single(hc, torch, case, desc, pos, bt, num_pages, split="whole")
    assert flags == 0 and flags0 == 0
    if norm == 0:
        gh.assert_close_to_model(bits, gh.model_pool(desc, case.x, case.gamma, case.wkv, pos, bt, num_pages))
    m = gh.assert_same_but_for_order(bits, whole)
    assert m.sum() == 2 * n_tok * n_kv * hd


@pytest.mark.parametrize("d_model,n_kv,hd,n_tok,style,norm,blocks", [
    (1024, 1, 64, 17, 2, "layer", 1),
    (1472, 5, 128, 47, 1, "bias", 1),
    (1024, 5, 64, 201, 0, "layer", 2),
    (1024, 5, 64, 201, 1, "bias", 2),
    (1088, 32, 128, 33, 1, "layer", 3),
    (1088, 32, 128, 33, 2, "bias", 3),
    (1024, 8, 128, 201, 2, "layer", 4),
    (1024, 16, 64, 201, 0, "bias", 4),
])
def test_few_tokens_variants_and_bad_rows(hc, torch, d_model, n_kv, hd, n_tok, style, norm, blocks):
    """The few-token kernel's other epilogues (LayerNorm with shift and bias, RMSNorm with a K/V bias) for every count
    of token blocks, with a row whose position lies past max_position and the rows of a page that the pool does not have:
    flags and written elements of whole 256 x 256 tiles, values but for the order of the sums, and as a
    ragged batch of two contexts the same bits again."""
    layer_norm = norm == "layer"
    assert hc.diag_route(d_model, n_kv * hd, n_tok, 0, layer_norm)[:2] == ("few", blocks)
    torch.manual_seed(d_model * 7919 + n_tok)
    rows, B, offset = 2 * n_kv * hd, 16, 40
    n_blocks = (offset + n_tok + B - 1) // B
    num_pages = n_blocks + 3
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd, block_size=B,
                        max_position=offset + n_tok, rope_style=style, norm_kind=int(layer_norm))
    ctx, s = hc.Context(desc), gh.stream_handle()
    bf = dict(dtype=torch.bfloat16, device="cuda")
    w, gain = torch.randn((rows, d_model), **bf) * 0.05, 1 + 0.1 * torch.randn(d_model, **bf)
    shift = 0.1 * torch.randn(d_model, **bf) if layer_norm else None
    bias = 0.1 * torch.randn(rows, **bf)
    ctx.set_layer_weights_affine(0, w, gain, shift, bias, s)
    x = torch.randn((n_tok, d_model), **bf) + 0.25
    pos = torch.arange(offset, offset + n_tok, dtype=torch.int32, device="cuda")
    pos[n_tok // 2] = offset + n_tok
    table = torch.randperm(num_pages, device="cuda")[:n_blocks].to(torch.int32)
    table[-1] = num_pages
    cu = torch.tensor([0, n_tok // 3, n_tok], dtype=torch.int32, device="cuda")
    tables = torch.stack([table, table])

    def outcome(call):
        pool = gh.new_pool(num_pages, B, n_kv, hd)
        ctx.set_kv_pool(0, pool, num_pages)
        ctx.set_split(1)
        call()
        return ctx.poll_device_error(s), gh.pool_bits(pool)

    flags, few = outcome(lambda: ctx.restore_kv(0, x, pos, n_tok, table, n_blocks, s))
    whole_flags, whole = outcome(lambda: gh.restore_whole_tiles(ctx, 0, x, pos, n_tok, table, n_blocks, s))
    ragged_flags, ragged = outcome(lambda: ctx.restore_kv_ragged(0, x, pos, n_tok, cu, 2, tables, n_blocks, s))
    assert flags == whole_flags == ragged_flags == (hc.HC_DEV_BAD_POSITION | hc.HC_DEV_BAD_PAGE)
    at = torch.arange(offset, offset + n_tok, device="cuda")
    bad = (at // B == n_blocks - 1) | (at == offset + n_tok // 2)
    m = gh.assert_same_but_for_order(few, whole)
    assert m.sum() == int((~bad).sum()) * rows
    assert np.array_equal(ragged, few)
    ctx.destroy()


@pytest.mark.parametrize("d_model,n_kv,hd,n_tok,layers,style,norm,alone,together", [
    # alone, together: token blocks per wave of a single-layer call and of the launch over all layers
    (64, 1, 64, 1, 2, 0, "rms", 1, 1),           # one token, one superstep of the loop, one workgroup
    (256, 4, 64, 65, 3, 1, "rms", 1, 1),         # one token in the second tile
    (576, 3, 192, 130, 2, 0, "bias", 1, 1),      # padded K/V parts, pair groups that straddle the packed tile's halves
    (640, 43, 128, 140, 1, 0, "rms", 1, 1),      # two workgroups on a CU
    (128, 42, 128, 193, 1, 1, "layer", 1, 1),
    (704, 9, 64, 1601, 1, 2, "rms", 2, 2),
    (704, 5, 192, 1025, 1, 1, "layer", 2, 2),    # one token in the ninth tile
    (64, 103, 64, 257, 1, 2, "bias", 3, 3),
    (64, 86, 64, 321, 1, 0, "layer", 3, 3),
    (192, 33, 128, 577, 1, 0, "layer", 4, 4),
    (256, 51, 64, 769, 1, 1, "bias", 4, 4),      # one token in the fourth tile
    (1024, 25, 64, 2501, 1, 0, "rms", 5, 5),
    (704, 5, 64, 385, 3, 0, "layer", 1, 2),      # several layers: one token in the fourth tile
    (704, 3, 64, 641, 3, 1, "bias", 1, 2),
    (448, 8, 64, 513, 3, 1, "rms", 1, 3),
    (448, 4, 64, 1025, 3, 2, "layer", 1, 3),
    (640, 5, 128, 387, 3, 0, "bias", 1, 4),
    (640, 5, 64, 900, 3, 1, "layer", 1, 4),
])
def test_mid_tiles_equal_whole_tiles(hc, torch, d_model, n_kv, hd, n_tok, layers, style, norm, alone, together):
    """Shapes that go to tiles of 128 rows x 64..320 tokens, at the edges of the tiles and rings: layer
    by layer, all layers at once and as a ragged batch, with two rows whose position and page are
    invalid, bit for bit the 256 x 256 tiles' results and flags (a context that asks for split launches gets whole
    tiles at these shapes: nothing can be split)."""
    layer_norm = norm == "layer"
    for mode in (0, 1):
        assert hc.diag_route(d_model, n_kv * hd, n_tok, 0, layer_norm, mode)[:2] == ("rows128", alone)
        assert hc.diag_route(d_model, n_kv * hd, n_tok, layers, layer_norm, mode)[::3] == ("rows128", layers)
        assert hc.diag_route(d_model, n_kv * hd, n_tok, layers, layer_norm, mode)[1] == together
    assert hc.diag_route(d_model, n_kv * hd, n_tok, 0, layer_norm, 2)[::2] == ("tiles", 1)
    torch.manual_seed(d_model * 7919 + n_tok)
    rows, B, offset = 2 * n_kv * hd, 16, 40
    desc = gh.make_desc(hc, n_layers=layers, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd, block_size=B,
                        max_position=offset + n_tok, rope_style=style, norm_kind=1 if norm == "layer" else 0)
    ctx, s = hc.Context(desc), gh.stream_handle()
    bf = dict(dtype=torch.bfloat16, device="cuda")
    n_blocks = (offset + n_tok + B - 1) // B
    num_pages = n_blocks + 3
    keep, pools, xs = [], [], []
    for l in range(layers):
        w, gain = torch.randn((rows, d_model), **bf) * 0.05, 1 + 0.1 * torch.randn(d_model, **bf)
        shift = 0.1 * torch.randn(d_model, **bf) if norm == "layer" else None
        bias = 0.1 * torch.randn(rows, **bf) if norm != "rms" else None
        keep += [w, gain, shift, bias]
        if norm == "rms":
            ctx.set_layer_weights(l, w, gain, s)
        else:
            ctx.set_layer_weights_affine(l, w, gain, shift, bias, s)
        pools.append(gh.new_pool(num_pages, B, n_kv, hd))
        ctx.set_kv_pool(l, pools[l], num_pages)
        xs.append(torch.randn((n_tok, d_model), **bf) + 0.25)
    pos = torch.arange(offset, offset + n_tok, dtype=torch.int32, device="cuda")
    table = torch.randperm(num_pages, device="cuda")[:n_blocks].to(torch.int32)
    if n_tok > 2:
        pos[n_tok // 2] = offset + n_tok                  # past max_position
        table[-1] = num_pages                             # not a page of the pool
    cut = n_tok // 3
    cu = torch.tensor([0, cut, n_tok], dtype=torch.int32, device="cuda")
    tables = torch.stack([table, table])

    def ragged(l):
        ctx.restore_kv_ragged(l, xs[l], pos, n_tok, cu, 2, tables, n_blocks, s)

    def single(l):
        ctx.restore_kv(l, xs[l], pos, n_tok, table, n_blocks, s)

    def outcome(mode, call):
        ctx.set_split(mode)
        for p in pools:
            p.view(torch.int16).fill_(np.array(gh.SENTINEL, dtype=np.uint16).view(np.int16).item())
        if call is None:
            ctx.restore_kv_layers(0, xs, pos, n_tok, table, n_blocks, s)
        else:
            for l in range(layers):
                call(l)
        flags = ctx.poll_device_error(s)
        return flags, [gh.pool_bits(p) for p in pools]

    flags, want = outcome(2, single)
    assert (flags != 0) == (n_tok > 2)
    assert all(0 < (b != gh.SENTINEL).sum() <= n_tok * rows for b in want)
    for mode, call in ((1, single), (0, single), (1, None), (1, ragged), (2, ragged)):
        got_flags, got = outcome(mode, call)
        assert got_flags == flags
        for g, b in zip(got, want):
            assert np.array_equal(g, b)
    ctx.destroy()


def test_block_sizes(hc, torch):
    for B in (8, 32):
        rng = np.random.default_rng([5, B])
        case = gh.LayerCase(rng, 512, 2, 128, 100)
        n_blocks = (100 + B - 1) // B
        bt = rng.permutation(n_blocks + 3)[:n_blocks].astype(np.int32)
        pos = np.arange(100, dtype=np.int32)
        desc = gh.make_desc(hc, n_layers=1, d_model=512, n_q_heads=2, n_kv_heads=2, head_dim=128,
                            block_size=B, max_position=128)
        bits, flags = run_single(hc, torch, case, desc, pos, bt, n_blocks + 3)
        assert flags == 0
        gh.compare_pool(bits, oracle_single(case, desc, pos, bt, n_blocks + 3))


def test_ragged_batch(hc, torch):
    rng = np.random.default_rng(17)
    d_model, n_kv, hd, B = 512, 2, 128, 16
    lens = np.array([37, 260, 1, 129, 300], dtype=np.int32)     # crosses token tiles mid-context
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    case = gh.LayerCase(rng, d_model, n_kv, hd, T)
    pos = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
    nblk = (lens + B - 1) // B
    num_pages = int(nblk.sum()) + 9
    perm = rng.permutation(num_pages).astype(np.int32)
    tables = np.full((len(lens), int(nblk.max())), -1, dtype=np.int32)
    at = 0
    for s, n in enumerate(nblk):
        tables[s, :n] = perm[at:at + n]
        at += n
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv,
                        head_dim=hd, block_size=B, max_position=512)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    pool = gh.new_pool(num_pages, B, n_kv, hd)
    d_w, d_g, d_x = gh.to_dev_bf16(case.wkv_bits), gh.to_dev_bf16(case.gamma_bits), gh.to_dev_bf16(case.x_bits)
    ctx.set_layer_weights(0, d_w, d_g, s)
    ctx.set_kv_pool(0, pool, num_pages)
    d_pos, d_cu, d_tab = gh.to_dev_i32(pos), gh.to_dev_i32(cu), gh.to_dev_i32(tables)
    ctx.restore_kv_ragged(0, d_x, d_pos, T, d_cu, len(lens), d_tab, tables.shape[1], s)
    assert ctx.poll_device_error(s) == 0
    ora = np.full((num_pages, 2, B, n_kv, hd), np.nan)
    oracle.restore_kv_ragged(ora, case.x, case.gamma, case.wkv, pos, cu, tables, **gh.oracle_kw(desc))
    gh.compare_pool(gh.pool_bits(pool), ora)
    ctx.destroy()


def test_ragged_batch_split_launch_with_bad_rows(hc, torch):
    """The ragged batch at d_model 2048 with the d_model loops split four ways (mode 2), so that
    the per-token lookups (context by row offset, page by block table) run in the workgroups of
    the finishing launch; one context's table has an unmapped block and one position lies past
    the table: those rows are skipped and flagged, the rest matches the oracle.  Then on the few-token kernel (mode
    1) and on the tiles of 128 rows (mode 0)."""
    rng = np.random.default_rng(29)
    d_model, n_kv, hd, B = 2048, 2, 128, 16
    lens = np.array([37, 260, 1, 129, 300], dtype=np.int32)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T = int(cu[-1])
    assert hc.diag_split_plan(d_model, n_kv * hd, T, 2)["n_split"] == 4
    case = gh.LayerCase(rng, d_model, n_kv, hd, T)
    pos = np.concatenate([rng.permutation(n) for n in lens]).astype(np.int32)
    nblk = (lens + B - 1) // B
    num_pages = int(nblk.sum()) + 9
    perm = rng.permutation(num_pages).astype(np.int32)
    tables = np.full((len(lens), int(nblk.max())), -1, dtype=np.int32)
    at = 0
    for i, n in enumerate(nblk):
        tables[i, :n] = perm[at:at + n]
        at += n
    tables[1, 3] = -1                                 # context 1: positions 48..63 unmapped
    pos[cu[4] + 7] = 400                              # context 4: block 25 is past its table
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv,
                        head_dim=hd, block_size=B, max_position=512)
    good = np.ones(T, dtype=bool)
    for i in range(len(lens)):
        for t in range(cu[i], cu[i + 1]):
            blk = pos[t] // B
            good[t] = blk < tables.shape[1] and tables[i, blk] >= 0
    assert (~good).sum() == 17
    ora = np.full((num_pages, 2, B, n_kv, hd), np.nan)
    seq_of = np.repeat(np.arange(len(lens)), lens)
    keep = np.nonzero(good)[0]
    cu_good = np.concatenate([[0], np.cumsum([good[cu[i]:cu[i + 1]].sum() for i in range(len(lens))])]).astype(np.int32)
    oracle.restore_kv_ragged(ora, case.x[keep], case.gamma, case.wkv, pos[keep], cu_good, tables, **gh.oracle_kw(desc))
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    d_w, d_g, d_x = gh.to_dev_bf16(case.wkv_bits), gh.to_dev_bf16(case.gamma_bits), gh.to_dev_bf16(case.x_bits)
    ctx.set_layer_weights(0, d_w, d_g, s)
    d_pos, d_cu, d_tab = gh.to_dev_i32(pos), gh.to_dev_i32(cu), gh.to_dev_i32(tables)
    for split, kernel in ((2, "tiles"), (1, "few"), (0, "rows128")):
        assert hc.diag_route(d_model, n_kv * hd, T, mode=split)[0] == kernel
        ctx.set_split(split)
        pool = gh.new_pool(num_pages, B, n_kv, hd)
        ctx.set_kv_pool(0, pool, num_pages)
        ctx.restore_kv_ragged(0, d_x, d_pos, T, d_cu, len(lens), d_tab, tables.shape[1], s)
        assert ctx.poll_device_error(s) == (hc.HC_DEV_BAD_POSITION | hc.HC_DEV_BAD_PAGE)
        gh.compare_pool(gh.pool_bits(pool), ora)
    ctx.destroy()


def test_bad_rows_are_skipped_and_flagged(hc, torch):
    rng = np.random.default_rng(23)
    d_model, n_kv, hd, B, T = 256, 1, 64, 16, 40
    case = gh.LayerCase(rng, d_model, n_kv, hd, T)
    bt = np.array([3, -1, 1, 9], dtype=np.int32)     # block 1 unmapped, block 3 -> page outside pool
    num_pages = 5
    pos = np.arange(T, dtype=np.int32)               # 0..39 : blocks 0,1,2
    pos[5] = 70                                      # beyond the block table (block 4)
    pos[6] = -3
    pos[7] = 48                                      # block 3 -> page 9 >= num_pages
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=1, n_kv_heads=1, head_dim=hd,
                        block_size=B, max_position=128)
    bits, flags = run_single(hc, torch, case, desc, pos, bt, num_pages)
    assert flags == (hc.HC_DEV_BAD_POSITION | hc.HC_DEV_BAD_PAGE)
    good = np.array([p >= 0 and p // B < 4 and 0 <= bt[p // B] < num_pages for p in pos])
    ora = np.full((num_pages, 2, B, n_kv, hd), np.nan)
    oracle.restore_kv(ora, case.x[good], case.gamma, case.wkv, pos[good], bt, **gh.oracle_kw(desc))
    gh.compare_pool(bits, ora)
    # position >= max_position is refused even when the table would cover it
    desc2 = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=1, n_kv_heads=1, head_dim=hd,
                         block_size=B, max_position=16)
    bits, flags = run_single(hc, torch, case, desc2, np.arange(T, dtype=np.int32),
                             np.array([0, 1, 2], dtype=np.int32), num_pages)
    assert flags == hc.HC_DEV_BAD_POSITION
    assert np.all(bits[1:] == gh.SENTINEL) and np.all(bits[0] != gh.SENTINEL)


def test_host_side_errors(hc, torch):
    desc = gh.make_desc(hc, n_layers=2, d_model=256, n_q_heads=1, n_kv_heads=1, head_dim=64)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    x = torch.zeros(64, 256, dtype=torch.bfloat16, device="cuda")
    pos = torch.zeros(64, dtype=torch.int32, device="cuda")
    bt = torch.zeros(8, dtype=torch.int32, device="cuda")

    def status(fn, *a):
        with pytest.raises(hc.HCacheError) as e:
            fn(*a)
        return e.value.status

    assert status(ctx.restore_kv, 5, x, pos, 64, bt, 8, s) == hc.HC_ERANGE
    assert status(ctx.restore_kv, 0, x, pos, 64, bt, 8, s) == hc.HC_ESTATE      # no weights yet
    w = torch.zeros(128, 256, dtype=torch.bfloat16, device="cuda")
    g = torch.ones(256, dtype=torch.bfloat16, device="cuda")
    ctx.set_layer_weights(0, w, g, s)
    assert status(ctx.restore_kv, 0, x, pos, 64, bt, 8, s) == hc.HC_ESTATE      # no pool yet
    pool = gh.new_pool(4, 16, 1, 64)
    ctx.set_kv_pool(0, pool, 4)
    assert status(ctx.restore_kv, 0, None, pos, 64, bt, 8, s) == hc.HC_EINVAL
    assert status(ctx.restore_kv, 0, x.data_ptr() + 2, pos, 63, bt, 8, s) == hc.HC_EALIGN
    assert status(ctx.restore_kv, 0, x, pos, -1, bt, 8, s) == hc.HC_EINVAL
    assert status(ctx.set_kv_pool, 0, pool, 0) == hc.HC_ERANGE
    assert status(ctx.set_layer_weights, 0, None, g, s) == hc.HC_EINVAL
    ctx.restore_kv(0, x, pos, 0, bt, 8, s)                                      # empty: no-op
    assert ctx.poll_device_error(s) == 0
    assert np.all(gh.pool_bits(pool) == gh.SENTINEL)
    ctx.destroy()


@pytest.mark.parametrize("pinned,loader,d_model", [(True, 0, 512), (True, 1, 512), (False, 0, 512), (True, 0, 2048)],
                         ids=["copy-engines", "gather-kernel", "pageable-store", "few-token-kernel"])
def test_restore_context_from_store(hc, torch, pinned, loader, d_model):
    """Whole-context pipelined restore from the chunk store: all layers, a token range that
    starts and ends inside chunks, positions offset so the first page is part filled; with
    the gather-kernel loader, the hipMemcpyAsync loader, and a store in pageable memory; at d_model 512 on the
    tiles of 128 rows, at 2048 on the few-token kernel."""
    rng = np.random.default_rng(31)
    L, n_kv, hd, B, CT = 5, 2, 128, 16, 64
    assert hc.diag_route(d_model, n_kv * hd, 650)[0] == ("few" if d_model == 2048 else "rows128")
    T_stored, tok_begin, n_tok, pos_offset = 700, 30, 650, 1000
    desc = gh.make_desc(hc, n_layers=L, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv,
                        head_dim=hd, block_size=B, max_position=pos_offset + T_stored)
    cases = [gh.LayerCase(np.random.default_rng([31, l]), d_model, n_kv, hd, T_stored) for l in range(L)]
    store = hc.Store(L, d_model, CT, capacity_chunks=L * ((T_stored + CT - 1) // CT) + 2, pinned=pinned)
    # save order: a 512-token prefill, then smaller appends, layer by layer each time
    cuts = [0, 512, 600, 601, 700]
    for a, b in zip(cuts[:-1], cuts[1:]):
        for l in range(L):
            store.append(3, l, np.ascontiguousarray(cases[l].x_bits[a:b]), b - a)
    n_blocks = (pos_offset + T_stored + B - 1) // B
    num_pages = n_blocks + 5
    bt = rng.permutation(num_pages)[:n_blocks].astype(np.int32)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    copy_stream = torch.cuda.Stream()
    pools, keep = [], []
    for l in range(L):
        d_w, d_g = gh.to_dev_bf16(cases[l].wkv_bits), gh.to_dev_bf16(cases[l].gamma_bits)
        keep += [d_w, d_g]
        ctx.set_layer_weights(l, d_w, d_g, s)
        pools.append(gh.new_pool(num_pages, B, n_kv, hd))
        ctx.set_kv_pool(l, pools[l], num_pages)
    d_bt = gh.to_dev_i32(bt)
    ctx.set_loader(loader)
    torch.cuda.synchronize()
    for rep in range(2):                                # second call reuses the staging buffers
        ctx.restore_context(store, 3, tok_begin, n_tok, pos_offset, d_bt, n_blocks, s,
                            copy_stream.cuda_stream)
    assert ctx.poll_device_error(s) == 0
    torch.cuda.synchronize()
    pos = (pos_offset + tok_begin + np.arange(n_tok)).astype(np.int32)
    for l in range(L):
        ora = np.full((num_pages, 2, B, n_kv, hd), np.nan)
        c = cases[l]
        oracle.restore_kv(ora, c.x[tok_begin:tok_begin + n_tok], c.gamma, c.wkv, pos, bt,
                          **gh.oracle_kw(desc))
        gh.compare_pool(gh.pool_bits(pools[l]), ora)
    # errors
    with pytest.raises(hc.HCacheError) as e:
        ctx.restore_context(store, 3, 100, 700, 0, d_bt, n_blocks, s, copy_stream.cuda_stream)
    assert e.value.status == hc.HC_ERANGE
    with pytest.raises(hc.HCacheError) as e:
        ctx.restore_context(store, 3, 0, 10, 0, d_bt, n_blocks, s, s)
    assert e.value.status == hc.HC_EINVAL
    ctx.destroy()
    store.destroy()


def test_restore_context_from_store_split(hc, torch, monkeypatch):
    """The same with split launches asked for: every layer's launch is one (six tiles, four shares each, then the
    finishing launch), so the loader's events interleave with two kernels per layer that share the
    context's workspace."""
    assert hc.diag_route(2048, 256, 650, mode=2) == ("tiles", 0, 4, 1)
    plain = hc.Context

    def split_context(desc):
        ctx = plain(desc)
        ctx.set_split(2)
        return ctx

    monkeypatch.setattr(hc, "Context", split_context)
    test_restore_context_from_store(hc, torch, True, 0, 2048)


SEVERAL_LENGTHS = np.array([200, 0, 1, 333, 64], dtype=np.int32)
SEVERAL_STORED = SEVERAL_LENGTHS + np.array([10, 5, 0, 0, 7])     # the store may hold more than is restored


def several_contexts_cases(seed=69, L=3, d_model=512, n_kv=2, hd=128):
    """cases[context][layer]; the seed is one for which the prescribed bf16 arithmetic itself
    stays inside the tolerance at this narrow width (tests/test_tolerance_model.py)."""
    return [[gh.LayerCase(np.random.default_rng([seed, i, l]), d_model, n_kv, hd, int(SEVERAL_STORED[i]))
             for l in range(L)] for i in range(len(SEVERAL_LENGTHS))]


def test_restore_several_contexts_from_store(hc, torch):
    """hc_restore_contexts: five stored contexts (one of them empty, one a single token) restored
    together, one ragged launch per layer, positions implied by the row offsets; against the
    oracle's ragged restore and against restoring each context on its own."""
    rng = np.random.default_rng(63)
    L, d_model, n_kv, hd, B, CT = 3, 512, 2, 128, 16, 64
    lengths, stored = SEVERAL_LENGTHS, SEVERAL_STORED
    ids = np.array([11, 5, 42, 7, 1000], dtype=np.int64)
    desc = gh.make_desc(hc, n_layers=L, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd,
                        block_size=B, max_position=512)
    cases = several_contexts_cases()
    store = hc.Store(L, d_model, CT, capacity_chunks=int(sum(-(-int(n) // CT) for n in stored)) * L + 4)
    # interleaved arrival: contexts take turns, 50 tokens at a time, layer by layer
    done = np.zeros(len(ids), dtype=int)
    while np.any(done < stored):
        for i in range(len(ids)):
            n = int(min(50, stored[i] - done[i]))
            if n > 0:
                for l in range(L):
                    store.append(int(ids[i]), l, np.ascontiguousarray(cases[i][l].x_bits[done[i]:done[i] + n]), n)
                done[i] += n
    max_blocks = 24
    num_pages = len(ids) * max_blocks + 3
    perm = rng.permutation(num_pages).astype(np.int32)
    tables = np.full((len(ids), max_blocks), -1, dtype=np.int32)
    at = 0
    for i, n in enumerate(lengths):
        nb = (int(n) + B - 1) // B
        tables[i, :nb] = perm[at:at + nb]
        at += nb
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    copy_stream = torch.cuda.Stream()
    keep, pools = [], []
    # all contexts of a layer share the layer's weights: take context 0's
    for l in range(L):
        d_w, d_g = gh.to_dev_bf16(cases[0][l].wkv_bits), gh.to_dev_bf16(cases[0][l].gamma_bits)
        keep += [d_w, d_g]
        ctx.set_layer_weights(l, d_w, d_g, s)
        pools.append(gh.new_pool(num_pages, B, n_kv, hd))
        ctx.set_kv_pool(l, pools[l], num_pages)
    d_tables = gh.to_dev_i32(tables)
    for rep in range(2):
        ctx.restore_contexts(store, ids, lengths, d_tables, max_blocks, s, copy_stream.cuda_stream)
    assert ctx.poll_device_error(s) == 0
    torch.cuda.synchronize()
    cu = np.concatenate([[0], np.cumsum(lengths)])
    pos = np.concatenate([np.arange(n) for n in lengths]).astype(np.int32)
    for l in range(L):
        x = np.concatenate([cases[i][l].x[:lengths[i]] for i in range(len(ids))])
        ora = np.full((num_pages, 2, B, n_kv, hd), np.nan)
        oracle.restore_kv_ragged(ora, x, cases[0][l].gamma, cases[0][l].wkv, pos, cu, tables,
                                 **gh.oracle_kw(desc))
        gh.compare_pool(gh.pool_bits(pools[l]), ora)
    # bit for bit what restoring each context alone writes
    alone = [gh.new_pool(num_pages, B, n_kv, hd) for _ in range(L)]
    for l in range(L):
        ctx.set_kv_pool(l, alone[l], num_pages)
    for i, n in enumerate(lengths):
        if n:
            ctx.restore_context(store, int(ids[i]), 0, int(n), 0, gh.to_dev_i32(tables[i]), max_blocks, s,
                                copy_stream.cuda_stream)
    torch.cuda.synchronize()
    for l in range(L):
        assert np.array_equal(gh.pool_bits(alone[l]), gh.pool_bits(pools[l]))
    # errors
    def status(*a):
        with pytest.raises(hc.HCacheError) as e:
            ctx.restore_contexts(*a)
        return e.value.status
    cs = copy_stream.cuda_stream
    assert status(store, [11, 99], [10, 10], d_tables, max_blocks, s, cs) == hc.HC_ERANGE     # unknown context
    assert status(store, [11], [500], d_tables, max_blocks, s, cs) == hc.HC_ERANGE             # more than stored
    assert status(store, [11], [-1], d_tables, max_blocks, s, cs) == hc.HC_EINVAL
    assert status(store, [11], [10], d_tables, max_blocks, s, s) == hc.HC_EINVAL
    ctx.restore_contexts(store, [], [], d_tables, max_blocks, s, cs)                           # nothing to do
    ctx.destroy()
    store.destroy()
