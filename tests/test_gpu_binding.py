"""The binding's native route takes what it accepts to the same library calls as the route through
ctypes, and leaves everything else, errors included, to that one."""
from types import SimpleNamespace

import pytest

pytestmark = pytest.mark.gpu

from paper_2605_29639_amd import workloads as W

LONG_WAY = SimpleNamespace(write=lambda *a: None, attn=lambda *a: None, move=lambda *a: None)


@pytest.fixture
def routes(monkeypatch):
    """(set a route by its module, [the ctypes route, the native one])."""
    from paper_2605_29639_amd import kvq
    return lambda m: monkeypatch.setattr(kvq, "_fast_module", m), [LONG_WAY, kvq._fast()]


def outcome(call):
    try:
        return call()
    except Exception as e:
        return type(e).__name__, str(e)


@pytest.mark.parametrize("mode", [W.MODE_INT8, W.MODE_FP8_TENSOR, W.MODE_BF16])
def test_both_routes_give_the_same(mode, routes):
    import torch
    from paper_2605_29639_amd import kvq
    choose, modules = routes
    desc = kvq.make_desc(mode, 40, 16, 2, 128)
    g = torch.Generator(device="cuda").manual_seed(mode)
    k, v, q = (torch.randn((n, h, 128), generator=g, device="cuda").to(torch.bfloat16)
               for n, h in ((300, 2), (300, 2), (3, 8)))
    slots = torch.randperm(640, generator=g, device="cuda")[:300].sort().values
    tables = torch.arange(39, dtype=torch.int32, device="cuda").view(3, 13).contiguous()
    lens = torch.tensor([200, 33, 1], dtype=torch.int32, device="cuda")
    ids = torch.tensor([7, 3], dtype=torch.int32, device="cuda")
    ws = kvq.alloc_workspace(desc, 3, 1, 8, 208, shared_prefix_tokens=64)
    wrong = {  # call -> (position, value) of one argument that is not as it should be
        "write": [(0, k[:, :, :64]), (0, k.half()), (1, v.cpu()), (2, slots.int()), (2, slots[:-1]), (5, None), (5, bytes(desc))],
        "attn": [(0, q[:, :, ::2]), (3, bytes(desc)), (4, tables.long()), (5, lens[:-1]), (6, 2), (7, -1), (7, True), (7, 209),
                 (9, q), (10, ws[:8]), (11, 63), (11, -64)],
        "move": [(2, bytes(desc)), (3, ids.long()), (3, ids[:0]), (4, torch.zeros(8, dtype=torch.uint8)), (5, None)],
    }
    seen = []
    for module in modules:
        choose(module)
        cache, scales = kvq.alloc_cache(desc)
        if mode == W.MODE_FP8_TENSOR:
            scales.copy_(torch.tensor(W.STATIC_SCALES))
        out = torch.zeros((3, 8, 128), device="cuda")
        packed = [torch.zeros(n, dtype=t, device="cuda") for n, t in zip(kvq.packed_sizes(desc, 2), (torch.uint8, torch.float32))]
        write = [k, v, slots, cache, scales, desc]
        attn = [q, cache, scales, desc, tables, lens, 1, 208, 0.09, out, ws, 0]
        move = [cache, scales, desc, ids, *packed]
        kvq.kv_quant_write(*write)
        for prefix in (0, 64):
            kvq.paged_decode_attn(*attn, shared_prefix_tokens=prefix)
        kvq.blocks_export(*move)
        kvq.blocks_import(*packed, desc, ids.flip(0).contiguous(), cache, scales)
        state = [t.clone() for t in (cache, scales, out, *packed)]
        if module is not LONG_WAY:   # (and it was this route that did it)
            assert module.write(*write, None) == 0 and module.attn(*attn, None, 0) == 0
            assert module.move(True, *move, torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        errors = []
        for call, args in (("write", write), ("attn", attn), ("move", move)):
            f = {"write": kvq.kv_quant_write, "attn": kvq.paged_decode_attn, "move": kvq.blocks_export}[call]
            for at, value in wrong[call]:
                errors.append(outcome(lambda: f(*[value if i == at else a for i, a in enumerate(args)])))
        torch.cuda.synchronize()
        seen.append((state, errors))
    assert all(torch.equal(a, b) for a, b in zip(seen[0][0], seen[1][0]))
    assert seen[0][1] == seen[1][1] and sum(e is not None for e in seen[0][1]) >= 21
