"""Call boundaries: imposed inputs, results and the step record move through
pinned buffers that grow with the calls and are shared by all of them."""
import numpy as np
import pytest

import synth
from paper_2609_14144_amd import EEError
from tests.gpu_helpers import engine

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("persistent", [True, False], ids=["persistent", "per_op"])
def test_mixed_calls_equal_single_steps(persistent):
    """Calls of growing and shrinking sizes with imposed inputs, head
    evaluations, debug steps and a refresh between them give what one step per
    call gives; a head evaluation and a refresh leave the next input alone."""
    cfg = synth.get_config("tiny_bf16")
    prompt = synth.prompts(cfg, 1, 70)
    toks = synth.prompts(cfg, 2, 60)
    fe = np.resize(np.array([-1, 1, 0, -1, 1], np.int32), 60)
    a, b = engine("tiny_bf16", 256, persistent, page_size=16), engine("tiny_bf16", 256, persistent, page_size=16)
    a.ee_prefill(prompt[:40])
    b.ee_prefill(prompt[:40])
    x = np.random.default_rng(0).standard_normal(cfg.hidden).astype(np.float32)
    h0 = a.ee_head_eval(2, x)
    at = 0
    got, want = [], []
    for n in (3, 50, 2, 5):
        r = a.ee_decode_n_ex(0.3, 2, n, force_tokens=toks[at:at + n], force_exit=fe[at:at + n])
        got.append(np.stack([r[0], r[1], r[2], r[3]]))
        for i in range(at, at + n):
            s = b.ee_decode_n_ex(0.3, 2, 1, force_tokens=toks[i:i + 1], force_exit=fe[i:i + 1])
            want.append(np.stack([s[0], s[1], s[2], s[3]]))
        at += n
        h1 = a.ee_head_eval(2, x)
        assert h1[0] == h0[0] and h1[1] == h0[1]
        np.testing.assert_array_equal(h1[2], h0[2])
        a.ee_refresh(1)
        b.ee_refresh(1)
    np.testing.assert_array_equal(np.concatenate(got, 1), np.concatenate(want, 1))
    # the free-running continuation starts from the last emitted token on both
    ra, rb = a.ee_decode_n(0.3, 2, 4), b.ee_decode_n(0.3, 2, 4)
    for u, v in zip(ra, rb):
        np.testing.assert_array_equal(u, v)
    # a reset sequence starts over, a prompt in two parts equals the parts' positions
    a.ee_reset()
    a.ee_prefill(prompt[:40])
    a.ee_prefill(prompt[40:])
    assert a.ee_position() == 70
    d = a.ee_decode_step_ex(0.3, 2, 7, 0)
    b.ee_reset()
    b.ee_prefill(prompt[:40])
    b.ee_prefill(prompt[40:])
    e = b.ee_decode_step_ex(0.3, 2, 7, 0)
    for k in ("h_exit", "h_final", "logits_readout", "logits_full"):
        np.testing.assert_array_equal(d[k], e[k])
    a.close()
    b.close()


@pytest.mark.parametrize("chunk", [0, 16], ids=["stepwise", "batched"])
def test_refused_call_leaves_no_inputs(chunk):
    """A prompt and imposed steps beyond the capacity are refused; the refresh
    after them recomputes the same cache as in a context that made no such call."""
    cfg = synth.get_config("tiny_bf16")
    prompt = synth.prompts(cfg, 4, 40)
    toks = synth.prompts(cfg, 5, 60)
    kept = []
    for disturb in (False, True):
        e = engine("tiny_bf16", 48, page_size=16)
        e.ee_set_prefill_chunk(chunk)
        e.ee_prefill(prompt)
        if disturb:
            with pytest.raises(EEError):
                e.ee_prefill(toks)
            with pytest.raises(EEError):
                e.ee_decode_n_ex(0.3, 2, 60, force_tokens=toks, force_exit=np.ones(60, np.int32))
        e.ee_refresh(40)
        kv = [np.concatenate(e.ee_read_kv(l, t)) for l in range(cfg.n_layers) for t in range(40)]
        kept.append((np.stack(kv), *e.ee_decode_n(0.3, 2, 4)))
        e.close()
    for a, b in zip(*kept):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("name", ["tiny", "tiny_bf16"])
def test_default_grid_equals_the_full_one(name):
    """A new engine's own grid (small models: fewer workgroups) gives the cache
    bits and tokens of the full one; confidences differ by the order in which
    the head's partial sums (at most two per unit, positive terms) are added:
    512 roundings of 2^-24."""
    from paper_2609_14144_amd import Engine
    from tests.conftest import weights_for
    cfg = synth.get_config(name)
    prompt, toks = synth.prompts(cfg, 6, 30), synth.prompts(cfg, 7, 12)
    runs = []
    for full in (False, True):
        e = Engine(cfg, 64, page_size=16)
        e.ee_load_weights(weights_for(name))
        if full:
            e.ee_set_persistent(-1)
        e.ee_set_prefill_chunk(0)
        e.ee_prefill(prompt)
        r = e.ee_decode_n_ex(0.3, 2, 12, force_tokens=toks, force_exit=np.resize([0, 1, 1, 0], 12))
        kv = np.stack([np.concatenate(e.ee_read_kv(l, t)) for l in range(cfg.n_layers) for t in range(42)])
        runs.append((kv, r))
        e.close()
    (kva, a), (kvb, b) = runs
    np.testing.assert_array_equal(kva, kvb)
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_allclose(a[2], b[2], rtol=512 * 2.0 ** -24)
