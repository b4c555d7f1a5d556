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
