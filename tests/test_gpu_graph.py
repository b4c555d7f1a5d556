"""The entry points allocate nothing, keep no per-call state and never touch the host after
validation, so a decode step (kv_quant_write of the newest tokens + paged_decode_attn) can be
captured in a HIP graph once and replayed: the sequence lengths, tables, queries and new rows
are read on the device at every replay.  Each replay is checked bit for bit against the same
calls made eagerly on the same inputs, with eager work and synchronisations in between."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2605_29639_amd import workloads as W
from helpers import bits_to_bf16_tensor, gpu_fill


@pytest.mark.parametrize("mode", [W.MODE_INT8, W.MODE_FP8])
def test_a_captured_decode_step_replays_like_eager_calls(mode):
    import torch
    from paper_2605_29639_amd import kvq
    wl = W.custom("graph", mode, [200, 77, 1030, 64, 513], 1, 8, 2, 128, 16, seed=5)
    B, Hq, D, H = wl.batch, wl.num_q_heads, wl.head_dim, wl.num_kv_heads
    max_len = int(wl.seq_lens.max())
    bt = torch.from_numpy(wl.block_tables).cuda()
    rng = np.random.default_rng(77)

    def fresh_inputs(lens):
        """q, the newest token's k and v (random bf16) and its slot, for the given lengths."""
        q = W.to_bf16_bits(rng.standard_normal((B, Hq, D), dtype=np.float32))
        k = W.to_bf16_bits(rng.standard_normal((B, H, D), dtype=np.float32))
        v = W.to_bf16_bits(rng.standard_normal((B, H, D), dtype=np.float32))
        slots = np.array([wl.slots(b, int(lens[b]) - 1, int(lens[b]))[0] for b in range(B)], np.int64)
        return (bits_to_bf16_tensor(q), bits_to_bf16_tensor(k), bits_to_bf16_tensor(v),
                torch.from_numpy(slots).cuda(), torch.from_numpy(lens.astype(np.int32)).cuda())

    def step(cache, scales, desc, ins, out, ws):
        q, k, v, slots, sl = ins
        kvq.kv_quant_write(k, v, slots, cache, scales, desc)
        kvq.paged_decode_attn(q, cache, scales, desc, bt, sl, 1, max_len, wl.sm_scale, out, ws)

    # two identical caches: one for the graph, one for the eager calls
    cache_g, scales_g, desc = gpu_fill(wl)
    cache_e, scales_e = cache_g.clone(), scales_g.clone()
    ws_g = kvq.alloc_workspace(desc, B, 1, Hq, max_len, 0)
    ws_e = kvq.alloc_workspace(desc, B, 1, Hq, max_len, 0)
    out_g = torch.zeros((B, Hq, D), dtype=torch.float32, device="cuda")
    out_e = torch.zeros_like(out_g)

    static = fresh_inputs(wl.seq_lens)              # the tensors the graph reads
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                   # warm-up on the capture stream
        step(cache_g, scales_g, desc, static, out_g, ws_g)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    cache_g.copy_(cache_e), scales_g.copy_(scales_e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(cache_g, scales_g, desc, static, out_g, ws_g)
    cache_g.copy_(cache_e), scales_g.copy_(scales_e)   # (capturing runs nothing, but be sure)

    lens = wl.seq_lens.copy()
    for replay in range(4):
        if replay == 2:      # another decode position for two of the sequences
            lens[0] -= 37
            lens[2] -= 500
        new = fresh_inputs(lens)
        for dst, src in zip(static, new):
            dst.copy_(src)
        torch.cuda.synchronize()
        graph.replay()
        step(cache_e, scales_e, desc, new, out_e, ws_e)   # eager, same inputs
        torch.cuda.synchronize()
        assert torch.equal(out_g, out_e), "replay %d differs from the eager calls" % replay
        assert torch.equal(cache_g, cache_e) and torch.equal(scales_g, scales_e), replay
        assert torch.isfinite(out_g).all()


def test_a_captured_verify_step_with_a_shared_prefix_replays_like_eager_calls():
    """The same for paged_decode_attn_prefix (prefix kernel, streaming kernel, reduce): whether
    the prefix is used is decided on the device at every replay, so a replay in which one
    sequence has become shorter than the prefix falls back by itself."""
    import torch
    from paper_2605_29639_amd import kvq
    q_len, prefix = 2, 2048
    wl = W.custom("graph_prefix", W.MODE_INT8, [2100 + 7 * (i % 9) for i in range(260)], q_len, 4, 2, 128, 16,
                  seed=6, shared_prefix=prefix)
    B, Hq, D, H = wl.batch, wl.num_q_heads, wl.head_dim, wl.num_kv_heads
    max_len = int(wl.seq_lens.max())
    bt = torch.from_numpy(wl.block_tables).cuda()
    rng = np.random.default_rng(78)

    def fresh_inputs(lens):
        q = W.to_bf16_bits(rng.standard_normal((B * q_len, Hq, D), dtype=np.float32))
        k = W.to_bf16_bits(rng.standard_normal((B * q_len, H, D), dtype=np.float32))
        v = W.to_bf16_bits(rng.standard_normal((B * q_len, H, D), dtype=np.float32))
        slots = np.concatenate([wl.slots(b, int(lens[b]) - q_len, int(lens[b])) for b in range(B)])
        return (bits_to_bf16_tensor(q), bits_to_bf16_tensor(k), bits_to_bf16_tensor(v),
                torch.from_numpy(slots.astype(np.int64)).cuda(),
                torch.from_numpy(lens.astype(np.int32)).cuda())

    def step(cache, scales, desc, ins, out, ws):
        q, k, v, slots, sl = ins
        kvq.kv_quant_write(k, v, slots, cache, scales, desc)
        kvq.paged_decode_attn(q, cache, scales, desc, bt, sl, q_len, max_len, wl.sm_scale, out, ws,
                              shared_prefix_tokens=prefix)

    cache_g, scales_g, desc = gpu_fill(wl)
    assert kvq.prof_lib().kvq_profile_prefix_pieces(C.byref(desc), B, q_len, Hq, max_len, 0, prefix) > 1
    cache_e, scales_e = cache_g.clone(), scales_g.clone()
    ws_g = kvq.alloc_workspace(desc, B, q_len, Hq, max_len, 0, shared_prefix_tokens=prefix)
    ws_e = kvq.alloc_workspace(desc, B, q_len, Hq, max_len, 0, shared_prefix_tokens=prefix)
    out_g = torch.zeros((B * q_len, Hq, D), dtype=torch.float32, device="cuda")
    out_e = torch.zeros_like(out_g)

    static = fresh_inputs(wl.seq_lens)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(cache_g, scales_g, desc, static, out_g, ws_g)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    cache_g.copy_(cache_e), scales_g.copy_(scales_e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(cache_g, scales_g, desc, static, out_g, ws_g)
    cache_g.copy_(cache_e), scales_g.copy_(scales_e)

    lens = wl.seq_lens.copy()
    for replay in range(4):
        if replay == 1:      # other decode positions, every sequence still holds the prefix
            lens[0] -= 37
            lens[2] -= 50
        if replay == 2:      # sequence 3 shorter than the prefix: the prefix is not used
            lens[3] = 1000
        if replay == 3:
            lens[3] = 2048   # exactly the prefix: nothing but shared positions
        new = fresh_inputs(lens)
        for dst, src in zip(static, new):
            dst.copy_(src)
        torch.cuda.synchronize()
        graph.replay()
        step(cache_e, scales_e, desc, new, out_e, ws_e)
        torch.cuda.synchronize()
        assert torch.equal(out_g, out_e), "replay %d differs from the eager calls" % replay
        assert torch.equal(cache_g, cache_e) and torch.equal(scales_g, scales_e), replay
        assert torch.isfinite(out_g).all()


@pytest.mark.parametrize("mode,D,q_len", [(W.MODE_INT8, 128, 40), (W.MODE_BF16, 64, 13)])
def test_a_captured_many_row_call_cuts_the_contexts_of_each_replay(mode, D, q_len):
    """How the contexts are cut is worked out on the device from the lengths of the moment: a graph
    captured with one long sequence replays with another long one, with none, and with all of them
    long, bit for bit like eager calls."""
    import torch
    from paper_2605_29639_amd import kvq
    wl = W.custom("graph_cut", mode, [2500, 2300, 2400], q_len, 16, 2, D, 16, seed=9)
    bt = torch.from_numpy(wl.block_tables).cuda()
    cache, scales, desc = gpu_fill(wl)
    bound = int(wl.seq_lens.max())
    q = bits_to_bf16_tensor(wl.q)
    ws = [kvq.alloc_workspace(desc, wl.batch, q_len, 16, bound, 0) for _ in range(2)]
    out = [torch.zeros(q.shape, dtype=torch.float32, device="cuda") for _ in range(2)]
    static = torch.tensor([2500, 60, 50], dtype=torch.int32, device="cuda")

    def call(lens, i):
        kvq.paged_decode_attn(q, cache, scales, desc, bt, lens, q_len, bound, wl.sm_scale, out[i], ws[i])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call(static, 0)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(static, 0)
    for lens in ([2500, 60, 50], [41, 2300, 700], [64, 65, 40], [2500, 2300, 2400], [60, 40, 2400]):
        new = torch.tensor(lens, dtype=torch.int32, device="cuda")
        static.copy_(new)
        ws[0].fill_(0xFF)
        out[0].fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        call(new, 1)
        torch.cuda.synchronize()
        assert torch.equal(out[0], out[1]), lens
        assert torch.isfinite(out[0]).all()


@pytest.mark.parametrize("to_packed", [True, False], ids=["export", "import"])
@pytest.mark.parametrize("host", [False, True], ids=["device", "pinned_host"])
def test_a_captured_block_move_replays_like_an_eager_one(host, to_packed):
    """Moves of more pieces than a move from or to host memory has in flight, which ask where the packed area
    lies: a capture takes that like any other call, and every replay moves what is there at the time."""
    import torch
    from paper_2605_29639_amd import kvq
    num = 300                                   # 8 pieces of 4 KiB a block
    desc = kvq.make_desc(W.MODE_INT8, num + 50, 16, 8, 128)
    cache, scales = kvq.alloc_cache(desc)
    nbytes, nscales = kvq.packed_sizes(desc, num)
    where = dict(pin_memory=True) if host else dict(device="cuda")
    pc, ps = torch.zeros(nbytes, dtype=torch.uint8, **where), torch.zeros(nscales, **where)
    ids = torch.randperm(num + 50, device="cuda")[:num].to(torch.int32)
    codes, floats = cache.view(torch.uint8).view(num + 50, -1), scales.view(num + 50, -1)

    def move():
        if to_packed:
            kvq.blocks_export(cache, scales, desc, ids, pc, ps)
        else:
            kvq.blocks_import(pc, ps, desc, ids, cache, scales)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        move()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        move()
    for replay in range(3):
        g = torch.Generator(device="cuda").manual_seed(replay)
        ids.copy_(torch.randperm(num + 50, generator=g, device="cuda")[:num])
        codes.copy_(torch.randint(0, 256, codes.shape, generator=g, device="cuda", dtype=torch.uint8))
        floats.copy_(torch.rand(floats.shape, generator=g, device="cuda"))
        pc.copy_(torch.randint(0, 256, pc.shape, generator=g, device="cuda", dtype=torch.uint8))
        ps.copy_(torch.rand(ps.shape, generator=g, device="cuda"))
        want_c, want_s = (codes[ids.long()], floats[ids.long()]) if to_packed else (pc.cuda(), ps.cuda())
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got_c, got_s = (pc.cuda(), ps.cuda()) if to_packed else (codes[ids.long()], floats[ids.long()])
        assert torch.equal(got_c.view(num, -1), want_c.view(num, -1)), replay
        assert torch.equal(got_s.view(num, -1), want_s.view(num, -1)), replay
