"""The binding's native route, without a GPU: what it answers, and what becomes of that."""
from types import SimpleNamespace

import pytest

from paper_2605_29639_amd import kvq

CALLS = {
    "write": lambda desc: kvq.kv_quant_write(None, None, None, None, None, desc),
    "attn": lambda desc: kvq.paged_decode_attn(None, None, None, desc, None, None, 1, 1, 0.1, None, None),
    "prefix": lambda desc: kvq.paged_decode_attn(None, None, None, desc, None, None, 1, 1, 0.1, None, None, shared_prefix_tokens=64),
    "export": lambda desc: kvq.blocks_export(None, None, desc, None, None, None),
    "import": lambda desc: kvq.blocks_import(None, None, desc, None, None, None),
}


@pytest.mark.parametrize("code", [kvq.E_HIP, kvq.E_BAD_INDEX])
@pytest.mark.parametrize("call", sorted(CALLS))
def test_a_call_that_reached_the_device_is_not_made_again(call, code, monkeypatch):
    """The library has launched, or asked the device, by the time it answers these: the error is raised, and
    the route through ctypes, where a second attempt might pass and hide it, is not taken."""
    message = kvq.strerror(code)
    monkeypatch.setattr(kvq, "_fast_module", SimpleNamespace(**dict.fromkeys(("write", "attn", "move"), lambda *a: code)))
    monkeypatch.setattr(kvq, "strerror", lambda c: message)
    monkeypatch.setattr(kvq, "lib", lambda: pytest.fail("the call was made a second time"))
    with pytest.raises(kvq.KvqError) as e:
        CALLS[call](kvq.make_desc(0, 8, 16, 2, 64))
    assert e.value.code == code and message in str(e.value)


@pytest.mark.parametrize("why", ["not built", "does not load"])
def test_without_the_native_module_calls_go_through_ctypes(why, tmp_path, monkeypatch):
    """libkvq.so alone does: the module saves time and nothing else.  (CPU tensors of the right shapes get as far
    as the device check of the route through ctypes.)"""
    import sys
    import torch
    desc = kvq.make_desc(0, 4, 16, 2, 64)
    cache, scales = kvq.alloc_cache(desc, device="cpu")
    k, slots = torch.zeros((3, 2, 64), dtype=torch.bfloat16), torch.zeros(3, dtype=torch.int64)
    monkeypatch.setattr(kvq, "_fast_module", None)
    if why == "not built":
        monkeypatch.setattr(kvq, "FAST_PATH", str(tmp_path / "_kvq_fast.so"))
    else:
        monkeypatch.delattr("paper_2605_29639_amd._kvq_fast", raising=False)
        monkeypatch.setitem(sys.modules, "paper_2605_29639_amd._kvq_fast", None)
    with pytest.warns(RuntimeWarning, match="_kvq_fast"), pytest.raises(TypeError, match="device tensor"):
        kvq.kv_quant_write(k, k, slots, cache, scales, desc)
