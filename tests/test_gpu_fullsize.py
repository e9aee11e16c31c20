"""GPU parity at the full sizes of the five workloads, in the launch configuration the
benchmark times (one fused launch per layer over all tokens; workloads 2 and 4 streamed
from the pinned chunk store through the pipelined whole-context restore).

The oracle cannot afford every output at these sizes, so each layer is checked by
  (i)   exact indexing over the WHOLE pool: the set of written cache elements equals the
        set the oracle's page/slot arithmetic predicts for all tokens;
  (ii)  element-by-element values for a sample of tokens: every token of the first and the
        last page, the rows around every 256-token tile edge and chunk edge, and 1024
        seeded random tokens, all features;
  (iii) a whole-tensor random-projection check in fp64 for EVERY token: for a seeded
        vector r, <V_gpu[t], r> and <unrotated K_gpu[t], r> against <x_hat[t], W^T r>.
Workloads 1 and 3 take two layers (first and last).  The streamed workloads go through the
layer pipeline at full depth: all 32 layers of workload 2 and 8 consecutive middle layers of
workload 4, every layer with its own seeded input, so that both staging buffers are reused
many times while the kernel is much shorter than the copy; check (ii) runs on a few of
those layers (first, middle ones, last), checks (i) and (iii) on every layer.  Between two
restores both staging buffers are filled with a NaN pattern.
"""
import numpy as np
import pytest

import synthetic as syn
import oracle.hcache_oracle as oracle
import gpu_harness as gh
import arith_model

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hc():
    import paper_2410_05004_amd as hc
    return hc


def sample_rows(rng, T, edges, first_page, last_page, n_random=1024):
    rows = set(first_page) | set(last_page)
    for e in edges:
        rows.update(r for r in (e - 2, e - 1, e, e + 1) if 0 <= r < T)
    rows.update(rng.choice(T, size=min(n_random, T), replace=False).tolist())
    return np.array(sorted(rows), dtype=np.int64)


def check_layer(w, desc, bits, x_bits, wkv_bits, gamma_bits, pos, seq_of_row, tables, rows, rng,
                beta_bits=None, bias_bits=None):
    """bits: GPU pool uint16 [P,2,B,H,hd]; pos/seq_of_row per token; tables [n_seq, max_blocks];
    beta_bits / bias_bits: LayerNorm shift and projection bias of the affine variants."""
    kw = gh.oracle_kw(desc)
    B, H, hd = desc.block_size, desc.n_kv_heads, desc.head_dim
    T = len(pos)
    # (i) exact indexing over the whole pool
    page = np.empty(T, dtype=np.int64)
    slot = np.empty(T, dtype=np.int64)
    for s in range(tables.shape[0]):
        m = seq_of_row == s
        page[m], slot[m] = oracle.page_slots(pos[m], tables[s], B)
    assert len(set(zip(page.tolist(), slot.tolist()))) == T, "token -> (page, slot) is not injective"
    expect = np.zeros(bits.shape[:3], dtype=bool)
    expect[page, :, slot] = True
    touched = bits != gh.SENTINEL
    assert np.array_equal(touched.all(axis=(3, 4)), expect), "written (page, kv, slot) set differs"
    assert np.array_equal(touched.any(axis=(3, 4)), expect), "partially written slot"

    gamma = syn.bf16_bits_to_f64(gamma_bits)
    wkv = syn.bf16_bits_to_f64(wkv_bits)
    got = syn.bf16_bits_to_f64(bits[page, :, slot])           # [T, 2, H, hd] in token order
    assert np.all(np.isfinite(got))

    # (ii) sampled tokens, every feature.  rows = None: this layer is not one of the few that
    # are held to the tolerance against the unrounded oracle element by element (the prescribed
    # bf16 arithmetic itself sits at 1.7e-2 - 2.2e-2 x RMS_head, tests/test_tolerance_model.py);
    # 256 seeded rows are then compared with the CPU model of that arithmetic instead, to one
    # bf16 step, which is the tighter check of the kernel.
    xf = syn.bf16_bits_to_f64(x_bits)                          # [T, d]
    sampled = rows is not None
    if not sampled:
        rows = np.sort(rng.choice(T, size=min(256, T), replace=False))
    xs = xf[rows]
    beta = None if beta_bits is None else syn.bf16_bits_to_f64(beta_bits)
    bias = None if bias_bits is None else syn.bf16_bits_to_f64(bias_bits)
    k, v = oracle.project_kv(xs, gamma, wkv, kw["eps"], H, hd, norm=kw["norm"], beta=beta, bias=bias)
    if kw["rope_style"] != 2:
        k = oracle.apply_rope(k, pos[rows], kw["theta"], kw["rope_style"])
    worst = 0.0
    rms_kv = []
    for ref, g in ((k, got[rows, 0]), (v, got[rows, 1])):
        rms = np.sqrt(np.mean(ref * ref, axis=(0, 2)))        # per head
        rms_kv.append(np.sqrt(np.mean(ref * ref)))
        err = np.max(np.abs(g - ref), axis=(0, 2))
        worst = max(worst, float(np.max(err / rms)))
    if sampled:
        assert worst <= gh.TOL, f"sampled rows: max |err| = {worst:.3e} x per-head RMS"
    if kw["norm"] == "rms":
        km, vm = arith_model.restore_rows(xs, gamma, wkv, pos[rows], eps=kw["eps"], theta=kw["theta"],
                                          n_kv_heads=H, head_dim=hd, rope_style=kw["rope_style"], bias=bias)
        model_bits = np.stack([syn.f32_to_bf16_bits(km.astype(np.float32)),
                               syn.f32_to_bf16_bits(vm.astype(np.float32))], axis=1)
        gh.assert_close_to_model(bits[page[rows], :, slot[rows]], model_bits)

    # (iii) random projection over all tokens
    r = rng.standard_normal(H * hd)
    d_kv = H * hd
    if kw["norm"] == "rms":
        mu = np.zeros(T)
        xh_scale = 1.0 / np.sqrt(np.einsum("td,td->t", xf, xf) / xf.shape[1] + kw["eps"])
    else:
        mu = xf.mean(axis=1)
        xh_scale = 1.0 / np.sqrt(xf.var(axis=1) + kw["eps"])
    proj = []
    for part in (0, 1):
        wr = wkv[part * d_kv:(part + 1) * d_kv].T @ r                   # [d]
        u = wr * gamma
        const = (0.0 if beta is None else wr @ beta) + \
            (0.0 if bias is None else bias[part * d_kv:(part + 1) * d_kv] @ r)
        proj.append((xf @ u - mu * u.sum()) * xh_scale + const)         # [T]
    k_unrot = got[:, 0] if kw["rope_style"] == 2 else \
        oracle.apply_rope(got[:, 0], -pos.astype(np.int64), kw["theta"], kw["rope_style"])
    dk = np.abs(k_unrot.reshape(T, -1) @ r - proj[0])
    dv = np.abs(got[:, 1].reshape(T, -1) @ r - proj[1])
    lim_k = gh.TOL * rms_kv[0] * np.linalg.norm(r)
    lim_v = gh.TOL * rms_kv[1] * np.linalg.norm(r)
    assert dk.max() <= lim_k, f"projection check K: {dk.max():.3e} > {lim_k:.3e} at row {dk.argmax()}"
    assert dv.max() <= lim_v, f"projection check V: {dv.max():.3e} > {lim_v:.3e} at row {dv.argmax()}"
    return worst, dk.max() / lim_k, dv.max() / lim_v


def layers_under_test(w):
    return (0, w.n_layers - 1)


@pytest.mark.parametrize("index", [1])
def test_single_context_workloads(hc, index):
    """Workload 1 from HBM through hc_restore_kv."""
    import torch
    w = syn.WORKLOADS[index]
    T, B = w.tokens, w.block_size
    layers = layers_under_test(w)
    # a context holding just the layers under test (each layer's work is independent)
    desc = gh.make_desc(hc, n_layers=len(layers), d_model=w.d_model, n_q_heads=w.n_q_heads,
                        n_kv_heads=w.n_kv_heads, head_dim=w.head_dim, block_size=B,
                        max_position=w.pos_offset + T, rope_theta=w.rope_theta, rms_eps=w.rms_eps)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    bt, num_pages = syn.block_table(w, w.pos_offset + T)
    d_bt = gh.to_dev_i32(bt)
    pos = (w.pos_offset + np.arange(T)).astype(np.int32)
    data, pools = [], []
    for i, l in enumerate(layers):
        wkv, gamma = syn.layer_weights(w, l)
        x = syn.layer_hidden(w, l)
        data.append((wkv, gamma, x))
        d_w, d_g = gh.to_dev_bf16(wkv), gh.to_dev_bf16(gamma)
        ctx.set_layer_weights(i, d_w, d_g, s)
        torch.cuda.synchronize()
        pools.append(gh.new_pool(num_pages, B, w.n_kv_heads, w.head_dim))
        ctx.set_kv_pool(i, pools[i], num_pages)
    print(f"{w.name}: inputs ready", flush=True)
    d_pos = gh.to_dev_i32(pos)
    for i in range(len(layers)):
        d_x = gh.to_dev_bf16(data[i][2])
        ctx.restore_kv(i, d_x, d_pos, T, d_bt, len(bt), s)
    assert ctx.poll_device_error(s) == 0
    torch.cuda.synchronize()
    print(f"{w.name}: restored", flush=True)
    rng = np.random.default_rng([99, index])
    edges = list(range(256, T, 256)) + list(range(w.chunk_tokens, T, w.chunk_tokens))
    rows = sample_rows(rng, T, edges, range(0, B - w.pos_offset % B), range(T - 16, T))
    for i, l in enumerate(layers):
        wkv, gamma, x = data[i]
        res = check_layer(w, desc, gh.pool_bits(pools[i]), x, wkv, gamma, pos,
                          np.zeros(T, dtype=np.int64), bt[None, :], rows, rng)
        print(f"{w.name} layer {l}: sampled worst {res[0]:.3e} x RMS_head; projection check "
              f"K {res[1]:.3f} V {res[2]:.3f} of limit", flush=True)
    ctx.destroy()


SPLIT_CASES = {
    # 16 feature tiles x 17 token tiles: the first 16 rows of token tiles fill one round of 256
    # workgroups and are computed whole, the 16 tiles of the ragged 17th are split in two
    "16x17": dict(d_model=1024, n_kv=16, hd=128, T=4315, B=16, offset=1000, seed=20,
                  plan=dict(nt_main=16, n_tail=16, n_split=2, main_slots=256)),
    # 5 x 52 = 260 tiles (d_kv = 640 pads the K and V parts): 51 whole rows (255 tiles in 256
    # slots), the five tiles of the ragged last row split in two
    "5x52": dict(d_model=1024, n_kv=5, hd=128, T=13156, B=16, offset=1000, seed=20,
                 plan=dict(nt_main=51, n_tail=5, n_split=2, main_slots=256)),
}


def split_case_inputs(name):
    """Seeded inputs of a split-launch test below and the token rows it checks element by
    element (also read by the CPU feasibility test).  The seeds are ones for which the prescribed
    bf16 arithmetic itself stays inside the tolerance on those rows
    (tests/test_tolerance_model.py; for the first case seeds 17-19 sit at 2.04e-2 - 2.15e-2 x
    RMS_head)."""
    c = SPLIT_CASES[name]
    T, B = c["T"], c["B"]
    rng = np.random.default_rng([c["seed"], c["d_model"], T])
    case = gh.LayerCase(rng, c["d_model"], c["n_kv"], c["hd"], T)
    n_blocks = (c["offset"] + T + B - 1) // B
    num_pages = n_blocks + 5
    bt = rng.permutation(num_pages)[:n_blocks].astype(np.int32)
    pos = (c["offset"] + rng.permutation(T)).astype(np.int32)
    last_row = (T - 1) // 256 * 256
    rows = np.union1d(np.arange(last_row, T), sample_rows(rng, T, range(256, T, 256), range(0, 8), [], n_random=600))
    return case, pos, bt, num_pages, rows


@pytest.mark.parametrize("name", list(SPLIT_CASES))
def test_split_launch_whole_and_split_tiles(hc, name):
    """Launches of more than 256 tiles whose last few tiles have their d_model loop split: whole
    tiles and split workgroups in one grid, then the finishing launch; tokens in scrambled
    order.  Exact written set, the random projection over every token, and every element of
    all tokens of the last, ragged row of token tiles (where the split tiles are) plus ~650
    sampled tokens of the whole rows; then the same with every tile whole, and with splitting off, where
    the launch rule may take the tiles of 128 rows."""
    import torch
    c = SPLIT_CASES[name]
    d_model, n_kv, hd, T, B = c["d_model"], c["n_kv"], c["hd"], c["T"], c["B"]
    plan = hc.diag_split_plan(d_model, n_kv * hd, T, 2)
    assert plan["split"] == 1 and {k: plan[k] for k in c["plan"]} == c["plan"], plan
    case, pos, bt, num_pages, rows = split_case_inputs(name)
    desc = gh.make_desc(hc, n_layers=1, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd,
                        block_size=B, max_position=c["offset"] + T, rope_theta=500000.0)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    d_w, d_g, d_x = gh.to_dev_bf16(case.wkv_bits), gh.to_dev_bf16(case.gamma_bits), gh.to_dev_bf16(case.x_bits)
    ctx.set_layer_weights(0, d_w, d_g, s)
    d_pos, d_bt = gh.to_dev_i32(pos), gh.to_dev_i32(bt)
    assert hc.diag_route(d_model, n_kv * hd, T, mode=2)[::2] == ("tiles", plan["n_split"])
    for split in (2, "whole", 0):
        pool = gh.new_pool(num_pages, B, n_kv, hd)
        ctx.set_kv_pool(0, pool, num_pages)
        if split == "whole":
            gh.restore_whole_tiles(ctx, 0, d_x, d_pos, T, d_bt, len(bt), s)
        else:
            ctx.set_split(split)
            ctx.restore_kv(0, d_x, d_pos, T, d_bt, len(bt), s)
        assert ctx.poll_device_error(s) == 0
        torch.cuda.synchronize()
        res = check_layer(None, desc, gh.pool_bits(pool), case.x_bits, case.wkv_bits, case.gamma_bits, pos,
                          np.zeros(T, dtype=np.int64), bt[None, :], rows, np.random.default_rng(5))
        print(f"{name} split={split}: sampled worst {res[0]:.3e} x RMS_head; projection check "
              f"K {res[1]:.3f} V {res[2]:.3f} of limit", flush=True)
    ctx.destroy()


@pytest.mark.parametrize("index,layers,sampled_layers", [
    (2, tuple(range(32)), (0, 9, 16, 22, 31)),
    (4, tuple(range(36, 44)), (36, 39, 43)),
], ids=["llama3-8b-gqa-T8192-all-32-layers", "70b-gqa-T32768-layers-36-43"])
def test_streamed_workloads_full_depth(hc, index, layers, sampled_layers):
    """hc_restore_context over a deep stack at full size: the kernel of a layer (0.12 ms / 0.9 ms)
    is far shorter than the layer's copy (1.2 ms / 9.5 ms), so the loader runs ahead as far as
    the two staging buffers allow and every buffer is refilled many times.  Restore once, fill
    both staging buffers with NaNs, restore again into fresh pools: the two results must be
    bit-identical and every layer must pass checks (i) and (iii); a few layers also (ii)."""
    import torch
    from concurrent.futures import ThreadPoolExecutor
    w = syn.WORKLOADS[index]
    T, B, CT, L = w.tokens, w.block_size, w.chunk_tokens, len(layers)
    desc = gh.make_desc(hc, n_layers=L, d_model=w.d_model, n_q_heads=w.n_q_heads,
                        n_kv_heads=w.n_kv_heads, head_dim=w.head_dim, block_size=B,
                        max_position=w.pos_offset + T, rope_theta=w.rope_theta, rms_eps=w.rms_eps)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    bt, num_pages = syn.block_table(w, w.pos_offset + T)
    d_bt = gh.to_dev_i32(bt)
    pos = (w.pos_offset + np.arange(T)).astype(np.int32)
    n_chunks = (T + CT - 1) // CT
    store = hc.Store(L, w.d_model, CT, L * n_chunks, pinned=True)
    import os
    with ThreadPoolExecutor(min(16, os.cpu_count() or 8)) as ex:                    # a different seeded input per layer
        hidden = list(ex.map(lambda l: syn.layer_hidden(w, l), layers))
    weights = [syn.layer_weights(w, l) for l in layers]
    for i in range(L):
        ctx.set_layer_weights(i, gh.to_dev_bf16(weights[i][0]), gh.to_dev_bf16(weights[i][1]), s)
        torch.cuda.synchronize()
    for c in range(n_chunks):                            # arrival order: chunk by chunk, layer by layer
        for i in range(L):
            rows = hidden[i][c * CT:(c + 1) * CT]
            store.append(0, i, rows, len(rows))
    print(f"{w.name}: {L} layers stored", flush=True)
    copy_stream = torch.cuda.Stream()

    def restore():
        pools = [gh.new_pool(num_pages, B, w.n_kv_heads, w.head_dim) for _ in range(L)]
        for i in range(L):
            ctx.set_kv_pool(i, pools[i], num_pages)
        ctx.restore_context(store, 0, 0, T, w.pos_offset, d_bt, len(bt), s, copy_stream.cuda_stream)
        assert ctx.poll_device_error(s) == 0
        torch.cuda.synchronize()
        return pools

    first = restore()
    ctx.poison_staging(s)
    second = restore()
    for i in range(L):
        assert torch.equal(first[i].view(torch.int16), second[i].view(torch.int16)), \
            f"layer {layers[i]}: the restore after the staging buffers were poisoned differs"
    del first
    print(f"{w.name}: restored twice, staging poisoned in between", flush=True)
    rng = np.random.default_rng([99, index])
    edges = list(range(256, T, 256)) + list(range(CT, T, CT))
    rows = sample_rows(rng, T, edges, range(0, B - w.pos_offset % B), range(T - 16, T))
    for i, l in enumerate(layers):
        res = check_layer(w, desc, gh.pool_bits(second[i]), hidden[i], weights[i][0], weights[i][1], pos,
                          np.zeros(T, dtype=np.int64), bt[None, :], rows if l in sampled_layers else None,
                          rng)
        print(f"{w.name} layer {l}: sampled worst {res[0]:.3e} x RMS_head; projection check "
              f"K {res[1]:.3f} V {res[2]:.3f} of limit", flush=True)
        second[i] = None
    ctx.destroy()
    store.destroy()


@pytest.mark.parametrize("index,n_layers,sampled", [(2, 10, (0, 3, 7, 9)), (5, 8, (0,))],
                         ids=["llama3-8b-gqa-T8192-10-layers", "opt30b-T2048-8-layers"])
def test_layers_per_launch_full_size(hc, index, n_layers, sampled):
    """hc_restore_kv_layers at full size, the launch configuration bench.py times: hidden states
    of all layers resident in HBM, eight layers per launch (workload 2: 10 layers = a launch
    of eight and one of two; 256 tiles per layer, the XCD a super tile goes to rotating with
    the layer; workload 5: 448 tiles per layer, LayerNorm + biases, no rotation).  A different
    seeded input per layer; every layer equals bit for bit what one hc_restore_kv launch for
    that layer writes, and passes the exact written-set check and the random projection over
    all tokens; the sampled ones are also compared element by element (workload 2: ~1100 rows;
    workload 5: the rows of test_gpu_variants.py::test_opt30b_shape -- the tolerance sits at the
    edge of bf16 output rounding, and 16 M outputs of this LayerNorm shape reach 2.2e-2)."""
    import torch
    w = syn.WORKLOADS[index]
    T, B = w.tokens, w.block_size
    layer_norm = w.norm == "layer"
    desc = gh.make_desc(hc, n_layers=n_layers, d_model=w.d_model, n_q_heads=w.n_q_heads,
                        n_kv_heads=w.n_kv_heads, head_dim=w.head_dim, block_size=B,
                        max_position=w.pos_offset + T, rope_theta=w.rope_theta, rms_eps=w.rms_eps,
                        rope_style=w.rope_style, norm_kind=1 if layer_norm else 0)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    bt, num_pages = syn.block_table(w, w.pos_offset + T)
    d_bt = gh.to_dev_i32(bt)
    pos = (w.pos_offset + np.arange(T)).astype(np.int32)
    d_pos = gh.to_dev_i32(pos)
    data, hidden_dev, pools = [], [], []
    for l in range(n_layers):
        wkv, gamma = syn.layer_weights(w, l)
        x = syn.layer_hidden(w, l)
        beta = bias = None
        if layer_norm:
            beta, bias = syn.layer_affine(w, l)
            ctx.set_layer_weights_affine(l, gh.to_dev_bf16(wkv), gh.to_dev_bf16(gamma), gh.to_dev_bf16(beta),
                                         gh.to_dev_bf16(bias), s)
        else:
            ctx.set_layer_weights(l, gh.to_dev_bf16(wkv), gh.to_dev_bf16(gamma), s)
        torch.cuda.synchronize()
        data.append((wkv, gamma, x, beta, bias))
        hidden_dev.append(gh.to_dev_bf16(x))
        pools.append(gh.new_pool(num_pages, B, w.n_kv_heads, w.head_dim))
        ctx.set_kv_pool(l, pools[l], num_pages)
    print(f"{w.name}: {n_layers} layers resident", flush=True)
    ctx.timing_begin()
    ctx.restore_kv_layers(0, hidden_dev, d_pos, T, d_bt, len(bt), s)
    _, launches = ctx.timing_end(s)
    assert launches == -(-n_layers // 8)
    assert ctx.poll_device_error(s) == 0
    torch.cuda.synchronize()
    if layer_norm:
        rng = np.random.default_rng(55)
        rows = sample_rows(rng, T, [256 * i for i in range(1, T // 256)], range(B), range(T - B, T), 256)
    else:
        rng = np.random.default_rng([98, index])
        rows = sample_rows(rng, T, range(256, T, 256), range(0, B - w.pos_offset % B), range(T - 16, T))
    ctx.set_split(0)
    for l in range(n_layers):
        wkv, gamma, x, beta, bias = data[l]
        alone = gh.new_pool(num_pages, B, w.n_kv_heads, w.head_dim)
        ctx.set_kv_pool(l, alone, num_pages)
        ctx.restore_kv(l, hidden_dev[l], d_pos, T, d_bt, len(bt), s)
        assert ctx.poll_device_error(s) == 0
        assert torch.equal(alone.view(torch.int16), pools[l].view(torch.int16)), \
            f"layer {l}: the launch over several layers differs from the single-layer launch"
        del alone
        res = check_layer(w, desc, gh.pool_bits(pools[l]), x, wkv, gamma, pos, np.zeros(T, dtype=np.int64),
                          bt[None, :], rows if l in sampled else None, rng, beta_bits=beta, bias_bits=bias)
        print(f"{w.name} layer {l}: sampled worst {res[0]:.3e} x RMS_head; projection check "
              f"K {res[1]:.3f} V {res[2]:.3f} of limit", flush=True)
        pools[l] = None
    ctx.destroy()


def test_ragged_workload(hc):
    """Workload 3: 16 contexts of 512..4096 tokens in one ragged launch per layer."""
    import torch
    w = syn.WORKLOADS[3]
    lens = syn.ragged_lengths(w)
    assert len(lens) == 16 and lens.min() >= 512 and lens.max() <= 4096
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, B = int(cu[-1]), w.block_size
    tables, num_pages = syn.ragged_block_tables(w, lens)
    pos = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
    seq_of_row = np.repeat(np.arange(len(lens)), lens)
    layers = layers_under_test(w)
    desc = gh.make_desc(hc, n_layers=len(layers), d_model=w.d_model, n_q_heads=w.n_q_heads,
                        n_kv_heads=w.n_kv_heads, head_dim=w.head_dim, block_size=B,
                        max_position=4096, rope_theta=w.rope_theta, rms_eps=w.rms_eps)
    ctx = hc.Context(desc)
    s = gh.stream_handle()
    d_pos, d_cu, d_tab = gh.to_dev_i32(pos), gh.to_dev_i32(cu), gh.to_dev_i32(tables)
    rng = np.random.default_rng([99, 3])
    edges = list(range(256, T, 256)) + cu[1:-1].tolist()
    rows = sample_rows(rng, T, edges, range(0, 16), range(T - 16, T))
    for i, l in enumerate(layers):
        wkv, gamma = syn.layer_weights(w, l)
        x = syn.layer_hidden(w, l, T)
        d_w, d_g, d_x = gh.to_dev_bf16(wkv), gh.to_dev_bf16(gamma), gh.to_dev_bf16(x)
        ctx.set_layer_weights(i, d_w, d_g, s)
        pool = gh.new_pool(num_pages, B, w.n_kv_heads, w.head_dim)
        ctx.set_kv_pool(i, pool, num_pages)
        ctx.restore_kv_ragged(i, d_x, d_pos, T, d_cu, len(lens), d_tab, tables.shape[1], s)
        assert ctx.poll_device_error(s) == 0
        print(f"{w.name} layer {l}: restored {T} tokens", flush=True)
        res = check_layer(w, desc, gh.pool_bits(pool), x, wkv, gamma, pos, seq_of_row, tables,
                          rows, rng)
        print(f"{w.name} layer {l}: sampled worst {res[0]:.3e} x RMS_head; projection check "
              f"K {res[1]:.3f} V {res[2]:.3f} of limit", flush=True)
        del pool, d_x, d_w
    ctx.destroy()
