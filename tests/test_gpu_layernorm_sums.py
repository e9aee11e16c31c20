"""LayerNorm's sums worked out ahead of the 256 x 256 tiles: bit for bit the results of the sums in the tiles, in calls in a
row that use more slots than there are, on two streams, and under capture, where the tiles work them out."""
import numpy as np
import pytest

import gpu_harness as gh

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,n_kv,n_tok,layers,style", [
    (2048, 64, 8190, 1, 2),        # 15 tokens of the last 16-token block, no rotation
    (2048, 64, 4097, 2, 0),        # one token in the last tile and block
    (2112, 64, 4097, 2, 1),        # 66 steps: the unrolled loop of the sums ends inside its last round
])
def test_sums_ahead_equal_sums_in_the_tiles(d_model, n_kv, n_tok, layers, style):
    import torch
    import paper_2410_05004_amd as hc
    hd, B = 128, 16
    assert hc.diag_tile(d_model, n_kv * hd, n_tok, layers if layers > 1 else 0, hc.HC_NORM_LAYER) == (256, 256, 0, 1)
    torch.manual_seed(n_tok + d_model)
    desc = gh.make_desc(hc, n_layers=layers, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd, block_size=B,
                        max_position=n_tok, rope_style=style, norm_kind=1)
    ctx, s = hc.Context(desc), gh.stream_handle()
    bf = dict(dtype=torch.bfloat16, device="cuda")
    n_blocks = -(-n_tok // B)
    pos = torch.arange(n_tok, dtype=torch.int32, device="cuda")
    table = torch.randperm(n_blocks + 2, device="cuda")[:n_blocks].to(torch.int32)
    xs, pools = [], []
    for l in range(layers):
        w, gain, shift = torch.randn((2 * n_kv * hd, d_model), **bf) * 0.05, 1 + 0.1 * torch.randn(d_model, **bf), 0.1 * torch.randn(d_model, **bf)
        ctx.set_layer_weights_affine(l, w, gain, shift, None, s)
        torch.cuda.synchronize()
        xs.append(torch.randn((n_tok, d_model), **bf) + 0.25)
        pools.append(torch.zeros((n_blocks + 2, 2, B, n_kv, hd), **bf))
        ctx.set_kv_pool(l, pools[l], n_blocks + 2)

    def call(stream):
        if layers == 1:
            ctx.restore_kv(0, xs[0], pos, n_tok, table, n_blocks, stream)
        else:
            ctx.restore_kv_layers(0, xs, pos, n_tok, table, n_blocks, stream)

    for l in range(layers):
        gh.restore_whole_tiles(ctx, l, xs[l], pos, n_tok, table, n_blocks, s)
    torch.cuda.synchronize()
    want = [p.clone() for p in pools]
    ctx.set_split(1)

    def check():
        torch.cuda.synchronize()
        for p, v in zip(pools, want):
            assert torch.equal(p.view(torch.int16), v.view(torch.int16))
            p.zero_()
        torch.cuda.synchronize()

    for p in pools:
        p.zero_()
    for _ in range(6):
        call(s)
    check()
    side = torch.cuda.Stream()
    for _ in range(3):
        call(s)
        call(side.cuda_stream)
    check()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        graph.replay()
        check()
        call(s)
        check()
    assert ctx.poll_device_error(s) == 0
    ctx.destroy()


def _context(hc, d_model, n_kv, n_tok, layers, norm_kind):
    import torch
    hd, B = 128, 16
    ctx, s = hc.Context(gh.make_desc(hc, n_layers=layers, d_model=d_model, n_q_heads=n_kv, n_kv_heads=n_kv, head_dim=hd, block_size=B,
                                     max_position=n_tok, rope_style=0, norm_kind=norm_kind)), gh.stream_handle()
    bf = dict(dtype=torch.bfloat16, device="cuda")
    n_blocks, pools = -(-n_tok // B), []
    w, gain = torch.randn((2 * n_kv * hd, d_model), **bf) * 0.05, 1 + 0.1 * torch.randn(d_model, **bf)
    for l in range(layers):
        if norm_kind:
            ctx.set_layer_weights_affine(l, w, gain, 0.1 * gain, None, s)
        else:
            ctx.set_layer_weights(l, w, gain, s)
        pools.append(torch.zeros((n_blocks + 2, 2, B, n_kv, hd), **bf))
        ctx.set_kv_pool(l, pools[l], n_blocks + 2)
    pos = torch.arange(n_tok, dtype=torch.int32, device="cuda")
    table = torch.randperm(n_blocks + 2, device="cuda")[:n_blocks].to(torch.int32)
    torch.cuda.synchronize()
    return ctx, pools, pos, table, n_blocks


@pytest.mark.parametrize("d_model,n_kv,n_tok,norm_kind,mode,what", [
    (2048, 64, 8190, 1, 1, "sums"),        # the slots of the sums
    (4096, 8, 300, 0, 2, "split"),         # the workspace of split launches
])
def test_timing_leaves_out_the_wait_for_another_stream(d_model, n_kv, n_tok, norm_kind, mode, what):
    """The time of a launch that waits on the GPU for launches of the same context on another stream: at most that of the
    launches which may share the chip with it (four and itself), not of the whole queue."""
    import torch
    import paper_2410_05004_amd as hc
    assert hc.diag_tile(d_model, n_kv * 128, n_tok, 0, norm_kind, mode)[3] == (what == "sums")
    assert (hc.diag_route(d_model, n_kv * 128, n_tok, 0, norm_kind, mode)[2] > 1) == (what == "split")
    torch.manual_seed(1)
    ctx, pools, pos, table, n_blocks = _context(hc, d_model, n_kv, n_tok, 1, norm_kind)
    ctx.set_split(mode)
    x = torch.randn((n_tok, d_model), dtype=torch.bfloat16, device="cuda")
    main, side = gh.stream_handle(), torch.cuda.Stream()
    call = lambda stream: ctx.restore_kv(0, x, pos, n_tok, table, n_blocks, stream)
    for _ in range(20):
        call(main)
    torch.cuda.synchronize()
    ctx.timing_begin()
    for _ in range(20):
        call(main)
    alone = ctx.timing_end_stats(main)[2]
    torch.cuda.synchronize()
    for _ in range(60):
        call(side.cuda_stream)
    ctx.timing_begin()
    call(main)
    behind, launches = ctx.timing_end(main)
    torch.cuda.synchronize()
    assert launches == 1
    assert behind < 8 * alone, (behind, alone)
    ctx.destroy()


def test_slots_of_the_sums_hold_until_their_readers_are_done():
    """Sixteen calls in flight on two streams, four times as many as there are slots, each with hidden states, a layer and a pool of
    its own: every pool gets its own call's results.  The inputs differ in scale and offset, so another call's sums would show
    in every value."""
    import torch
    import paper_2410_05004_amd as hc
    d_model, n_kv, n_tok, layers = 2048, 64, 8190, 8
    assert hc.diag_tile(d_model, n_kv * 128, n_tok, 0, 1)[3] == 1
    torch.manual_seed(2)
    ctx, pools, pos, table, n_blocks = _context(hc, d_model, n_kv, n_tok, layers, 1)
    xs = [(torch.randn((n_tok, d_model), device="cuda") * (1 + 0.5 * l) + 0.25 * l).to(torch.bfloat16) for l in range(layers)]
    for l in range(layers):
        gh.restore_whole_tiles(ctx, l, xs[l], pos, n_tok, table, n_blocks, gh.stream_handle())
    torch.cuda.synchronize()
    want = [p.clone() for p in pools]
    sums = [(x.double().square().sum(1), x.double().sum(1)) for x in xs]
    for l in range(1, layers):                             # another call's sums are others by far, for nearly every token
        assert all(((a - b).abs() > 0.05 * b.abs().mean()).float().mean() > 0.8 for a, b in zip(sums[l], sums[l - 1]))
        assert not torch.equal(want[l], want[l - 1])
    ctx.set_split(1)
    streams = [torch.cuda.current_stream(), torch.cuda.Stream()]
    for _ in range(3):
        for p in pools:
            p.zero_()
        torch.cuda.synchronize()
        for i in range(2 * layers):                        # a layer stays on its stream
            l = i % layers
            ctx.restore_kv(l, xs[l], pos, n_tok, table, n_blocks, streams[l % 2].cuda_stream)
        torch.cuda.synchronize()
        for l in range(layers):
            assert torch.equal(pools[l].view(torch.int16), want[l].view(torch.int16)), l
    assert ctx.poll_device_error(gh.stream_handle()) == 0
    ctx.destroy()
