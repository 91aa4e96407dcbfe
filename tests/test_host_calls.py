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


def check_calls(host, e, prompt):  # noqa: F811
    """Every kind of call on a context, with the values the stand-in decoder gives."""
    import ctypes as C

    import paper_2609_14144_amd._binding as B
    n = len(prompt)
    e.ee_reset()
    assert e.ee_prefill(prompt) == (prompt[-1] + 1) % CFG.vocab
    e.ee_refresh(n)
    d = [C.c_void_p() for _ in range(3)]
    for p in d:
        assert host.hipMalloc(C.byref(p), C.c_size_t(8)) == 0
    e._check(B.lib.ee_decode_n_noalloc(e._ctx, 0.5, 1, 2, *d))
    assert (C.c_int32 * 2).from_address(d[0].value)[:] == [prompt[-1] + 2, prompt[-1] + 3]
    for p in d:
        host.hipFree(p)
    assert list(e.ee_decode_n(0.5, 1, 1)[0]) == [prompt[-1] + 4]
    assert entries(e) == list(prompt) + [prompt[-1] + 1 + i for i in range(3)]


@pytest.mark.parametrize("kind", [0, 1], ids=["pinned", "device"])
@pytest.mark.parametrize("nth", [1, 2])
def test_results_that_find_no_memory(host, kind, nth):  # noqa: F811
    """Calls whose results need more memory than there is are refused; the
    calls after them work, and so do they once there is memory."""
    e = make(4000)
    prompt = np.arange(90, 94, dtype=np.int32)
    x = np.full(CFG.hidden, 9.0, np.float32)
    e.ee_prefill(prompt)
    for call in (lambda: e.ee_head_eval(0, x), lambda: e.ee_decode_step_ex(0.5, 1, 5, 0),
                 lambda: e.ee_decode_n(0.5, 1, 2000), lambda: e.ee_decode_n(0.5, 1, 3900)):
        host.host_fail_alloc(kind, nth)
        try:
            call()
        except RuntimeError as err:
            assert err.code == ENOMEM
        host.host_fail_alloc(kind, 0)
        check_calls(host, e, prompt)
    e.ee_reset()
    e.ee_prefill(prompt)
    d = e.ee_decode_step_ex(0.5, 1, 5, 0)
    assert d["token"] == 6 and d["logits_full"][6] == 1.0 and d["logits_readout"].sum() == 1.0
    assert e.ee_head_eval(0, x)[0] == 10
    assert len(e.ee_decode_n(0.5, 1, 3900)[0]) == 3900
    e.close()


def test_first_calls_pin_no_memory(host):  # noqa: F811
    """A new context has the pinned memory that its first calls need; only
    more steps at once than it has room for allocate."""
    e = make(4000)
    n = host.host_pinned_allocs()
    e.ee_prefill(np.arange(50, 58, dtype=np.int32))
    e.ee_decode_step_ex(0.5, 1, 5, 0)
    e.ee_head_eval(0, np.ones(CFG.hidden, np.float32))
    e.ee_decode_n(0.5, 1, 1000)
    e.ee_decode_n_ex(0.5, 1, 1000, force_tokens=np.full(1000, 7, np.int32), force_exit=np.zeros(1000, np.int32))
    assert host.host_pinned_allocs() == n
    e.ee_decode_n(0.5, 1, 1900)
    assert host.host_pinned_allocs() == n + 1
    e.close()


def context_bytes(host):  # noqa: F811
    """Device bytes of a context with room for everything, its copies included, and of one with its weights loaded."""
    before = host.host_device_bytes()
    e = make(200)
    n = host.host_device_bytes() - before
    e.close()
    assert host.host_device_bytes() == before
    return before, n


@pytest.mark.parametrize("short", [16, 4096, 0], ids=lambda s: "short_%d" % s)
def test_context_without_room_for_the_tiled_copies(host, short):  # noqa: F811
    """The prompt pass's copies of the weights are what a context goes without
    when memory is short: it is made, and its passes make one copy at a time."""
    before, need = context_bytes(host)
    host.host_device_limit(before + need - short)
    e = make(200)
    tilings = host.host_tilings()
    prompt = np.arange(90, 94, dtype=np.int32)
    e.ee_prefill(prompt)
    e.ee_refresh(4)
    assert entries(e) == list(prompt)
    made = host.host_tilings() - tilings
    assert made == (2 * 4 * CFG.n_layers if short else 0)
    w = {"layers.1.wo": 2 * _W["layers.1.wo"] + 1}
    e.ee_load_weights(w)
    e.ee_prefill(prompt)
    e.close()


def test_copies_make_room_for_later_buffers(host):  # noqa: F811
    """A call that finds no memory gives the copies back and goes on."""
    before, need = context_bytes(host)
    e = make(200)
    prompt = np.arange(90, 94, dtype=np.int32)
    e.ee_prefill(prompt)
    host.host_device_limit(host.host_device_bytes() + 16)
    e.ee_decode_n(0.5, 1, 100)     # the ring buffers
    d = e.ee_decode_step_ex(0.5, 1, 5, 0)
    assert d["token"] == 6 and d["logits_full"][6] == 1.0
    tilings = host.host_tilings()
    e.ee_reset()
    e.ee_prefill(prompt)
    assert entries(e) == list(prompt) and host.host_tilings() > tilings
    e.ee_load_weights(_W)
    e.ee_prefill(prompt)
    # a buffer larger than the copies does not cost them
    e2_limit = host.host_device_bytes() + need
    host.host_device_limit(e2_limit)
    f = make(200)
    f.ee_prefill(prompt)
    host.host_device_limit(host.host_device_bytes())
    assert refused(f.ee_stream_probe, 1 << 30) == ENOMEM
    tilings = host.host_tilings()
    f.ee_prefill(prompt)
    assert host.host_tilings() == tilings
    f.close()
    e.close()
    assert host.host_device_bytes() == before


@pytest.mark.parametrize("per_cu", [1, 2, 3, 4])
def test_every_grid_has_its_partial_records(host, per_cu):  # noqa: F811
    """Each workgroup of a grid that can be selected has its head partial record."""
    host.host_max_wgs(4)
    e = make(64)
    e.ee_prefill(np.arange(50, 58, dtype=np.int32))
    for select, grid in ((lambda: e.ee_set_persistent(per_cu), 256 * per_cu),
                         (lambda: e.ee_set_persistent_grid(256 * per_cu - 3), 256 * per_cu - 3)):
        select()
        assert list(e.ee_decode_n_ex(0.5, 1, 2, force_tokens=[4, 5])[0]) == [5, 6]
        assert host.host_last_grid() == grid
    assert refused(e.ee_set_persistent, 5) == EINVAL
    assert refused(e.ee_set_persistent_grid, 4 * 256 + 1) == EINVAL
    e.close()


def test_grid_selection(host):  # noqa: F811
    """A new context's grid follows its shape; a negative count selects as
    many workgroups as can be co-resident, as the header says."""
    host.host_max_wgs(2)
    e = make(64)
    step = lambda: e.ee_decode_n_ex(0.5, 1, 1, force_tokens=[4])
    step()
    assert 1 <= host.host_last_grid() < 256
    for select in (-1, True):
        e.ee_set_persistent(0)
        e.ee_set_persistent(select)
        step()
        assert host.host_last_grid() == 512
    e.close()


@pytest.mark.parametrize("chunk", [0, None], ids=["stepwise", "batched"])
@pytest.mark.parametrize("how", ["grown", "given_back"])
def test_new_buffers_are_cleared_before_they_are_written(host, chunk, how):  # noqa: F811
    """The clearing of a buffer that a call allocates is over before the
    call's own kernels and copies write to it: longer prompts and imposed steps
    than a new context has room for, a refresh of all of them, and a pass
    whose room for one matrix had to be found again."""
    n = 9000
    e = make(n + 64, chunk)
    prompt = (np.arange(n) % 190 + 1).astype(np.int32)
    if how == "given_back":
        host.host_fail_alloc(1, 1)   # no room for one matrix either
        assert host.ee_test_give_back_tiled(e._ctx) != 0
        prompt = prompt[:8]
    assert e.ee_prefill(prompt) == prompt[-1] + 1
    forced = np.full(5, 9, np.int32)
    assert list(e.ee_decode_n_ex(0.5, 1, 5, force_tokens=forced)[0]) == [10] * 5
    e.ee_refresh(len(prompt) + 5)
    assert [int(e.ee_read_kv(1, t)[0][0]) for t in (0, 1, 7, len(prompt) - 1, len(prompt) + 4)] == \
        [int(prompt[t]) for t in (0, 1, 7, len(prompt) - 1)] + [9]
    e.close()
