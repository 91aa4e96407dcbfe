"""Call sequences of the runtime on the CPU (tests/host_runtime.cpp): what a
call that fails leaves behind never reaches a later one."""
from dataclasses import replace

import numpy as np
import pytest

import synth
from tests.host_lib import host, host_lib  # noqa: F401  (fixtures)

CFG = replace(synth.get_config("tiny_bf16"), name="host", n_layers=2, hidden=64, n_q_heads=2, n_kv_heads=1, ffn=64,
              vocab=200, readout_layers=(1,))
_W = {}


def make(max_seq, chunk=None, persistent=None):
    from paper_2609_14144_amd import Engine
    if not _W:
        _W.update(synth.generate_weights(CFG))
    e = Engine(CFG, max_seq, page_size=4)
    e.ee_load_weights(_W)
    if chunk is not None:
        e.ee_set_prefill_chunk(chunk)
    if persistent is not None:
        e.ee_set_persistent(persistent)
    return e


def entries(e, layer=1):
    return [int(e.ee_read_kv(layer, t)[0][0]) for t in range(e.ee_position())]


def refused(call, *args, **kw):
    from paper_2609_14144_amd import EEError
    with pytest.raises(EEError) as x:
        call(*args, **kw)
    return x.value.code


EINVAL, ENOMEM, ECAPACITY = -1, -3, -5


@pytest.mark.parametrize("persistent", [True, False], ids=["persistent", "per_op"])
@pytest.mark.parametrize("chunk", [0, None], ids=["stepwise", "batched"])
@pytest.mark.parametrize("call", ["prefill", "decode", "decode_grown"])
def test_refused_call_leaves_no_inputs(host, chunk, persistent, call):  # noqa: F811
    """A prompt or imposed steps beyond the capacity are refused; the refresh
    and the steps after it read the sequence's own tokens."""
    e = make(12, chunk, persistent)
    prompt = np.arange(50, 58, dtype=np.int32)
    e.ee_prefill(prompt)
    bad = np.full(40 if call == "decode_grown" else 6, 7, np.int32)
    if call == "prefill":
        assert refused(e.ee_prefill, bad) == ECAPACITY
    else:
        assert refused(e.ee_decode_n_ex, 0.5, 1, len(bad), force_tokens=bad, force_exit=np.ones(len(bad), np.int32)) == ECAPACITY
    e.ee_refresh(8)
    assert entries(e) == list(prompt)
    tok, exited, _, _ = e.ee_decode_n_ex(0.5, 1, 2)
    assert list(tok) == [59, 60] and not exited.any()
    assert entries(e) == list(prompt) + [58, 59]
    e.ee_refresh(3)
    assert entries(e) == list(prompt) + [58, 59]
    e.close()
