"""The batched full-depth pass at the edges of its tiles, against the CPU
oracle. Tolerances are those of tests/gpu_helpers.py."""
from dataclasses import replace

import numpy as np
import pytest

import synth
from tests import tile_shapes
from tests.gpu_helpers import MARGIN, check_kv, engine, lockstep, oracle_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# Widths that fill no tile: K of 200 and 328 (32- and 64-wide steps with a
# remainder), 320 QKV rows, 656 gate/up rows; three query heads per KV head.
RAGGED = replace(synth.get_config("tiny_bf16"), name="ragged_bf16", n_layers=2, hidden=200, n_q_heads=3, n_kv_heads=1,
                 ffn=328, vocab=600, readout_layers=(1,))
_W = {}


def ragged_weights(seed=0):
    if seed not in _W:
        _W[seed] = synth.generate_weights(RAGGED, seed=seed)
    return _W[seed]


def check_prompt(e, o, cfg, prompt, exit_layer, page_positions):
    P = len(prompt)
    g0 = o.prefill(prompt)
    g = e.ee_prefill(prompt)
    if o.last_prefill_stats[2] > MARGIN:
        assert g == g0, (P, g, g0)
    check_kv(e, o, cfg, range(cfg.n_layers), page_positions)
    lockstep(e, o, g0, 0.5, exit_layer, 2, force_tokens=synth.prompts(cfg, 3 + P, 2), force_exit=[0, 1])


@pytest.mark.parametrize("P", [1, 2, 15, 16, 17, 31, 33, 48, 49, 63, 64, 65, 97, 129, 257, 300])
def test_ragged_widths_and_positions(P):
    w = ragged_weights()
    o = oracle_for(RAGGED.name, P + 2, cfg=RAGGED, weights=w)
    e = engine(RAGGED.name, P + 2, page_size=16, cfg=RAGGED, weights=w)
    check_prompt(e, o, RAGGED, synth.prompts(RAGGED, 70 + P, P), 1, sorted({0, P // 2, max(P - 2, 0), P - 1}))
    e.close()


def test_positions_of_another_chunk_leave_no_trace():
    """A long chunk, then short prompts on the same context: what the long
    one left in the padded operands does not reach the short ones."""
    w = ragged_weights()
    e = engine(RAGGED.name, 304, page_size=16, cfg=RAGGED, weights=w)
    e.ee_prefill(synth.prompts(RAGGED, 5, 300))
    for P in (1, 18, 70):
        e.ee_reset()
        o = oracle_for(RAGGED.name, P + 2, cfg=RAGGED, weights=w)
        check_prompt(e, o, RAGGED, synth.prompts(RAGGED, 170 + P, P), 1, [0, P - 1])
    e.close()


def test_replaced_weights_reach_the_prompt_pass():
    """A later ee_load_weights of some tensors: the prompt pass uses them."""
    w = dict(ragged_weights())
    e = engine(RAGGED.name, 64, page_size=16, cfg=RAGGED, weights=w)
    prompt = synth.prompts(RAGGED, 9, 40)
    e.ee_prefill(prompt)
    other = ragged_weights(1)
    for leaf in ("layers.0.wk", "layers.1.w_up", "layers.0.wo", "layers.0.w_down"):
        w[leaf] = other[leaf]
        e.ee_load_weights({leaf: other[leaf]})
        e.ee_reset()
        o = oracle_for(RAGGED.name, 64, cfg=RAGGED, weights=w)
        check_prompt(e, o, RAGGED, prompt, 1, [0, 17, 39])
    e.close()


def test_pass_is_deterministic_over_k_slices():
    """Two passes give the same cache bits and logits: K slices are added in
    order (17 positions at the 0.5B widths split K over many workgroups)."""
    cfg = replace(synth.get_config("d0p5b"), n_layers=2, vocab=4096, readout_layers=(1,))
    w = synth.generate_weights(cfg)
    prompt = synth.prompts(cfg, 13, 17)
    runs = []
    for _ in range(2):
        e = engine("d0p5b", 32, cfg=cfg, weights=w)
        g = e.ee_prefill(prompt)
        kv = np.concatenate([np.concatenate(e.ee_read_kv(l, t)) for l in range(2) for t in range(17)])
        d = e.ee_decode_step_ex(0.5, 1, 7, 0)
        runs.append((g, kv, d["logits_full"]))
        e.close()
    assert runs[0][0] == runs[1][0]
    np.testing.assert_array_equal(runs[0][1], runs[1][1])
    np.testing.assert_array_equal(runs[0][2], runs[1][2])


# Query heads per KV head 1..8 and both head sizes: the waves of a workgroup,
# its blocks of query positions and the staging of key tiles follow from them.
HEADS = [(1, 1, 64), (2, 1, 128), (6, 2, 64), (4, 1, 64), (5, 1, 128), (6, 1, 128), (7, 1, 64), (16, 2, 128)]


@pytest.mark.parametrize("heads", HEADS, ids=lambda h: "A%d_K%d_D%d" % h)
def test_attention_head_groups(heads):
    """Prompts about the edges of the 16-position query blocks and 64-key
    tiles, in one chunk and in chunks of 48 (later chunks attend to the
    earlier ones through the cache)."""
    A, K, D = heads
    cfg = replace(synth.get_config("tiny_bf16"), name="heads", n_layers=2, hidden=max(128, A * D), n_q_heads=A,
                  n_kv_heads=K, head_dim=D, ffn=256, vocab=512, readout_layers=(1,))
    w = synth.generate_weights(cfg)
    for P, chunk in ((3, None), (64, None), (65, 48), (97, 48), (130, 48), (197, None)):
        o = oracle_for(cfg.name, P + 2, cfg=cfg, weights=w)
        e = engine(cfg.name, P + 2, page_size=16, cfg=cfg, weights=w)
        if chunk:
            e.ee_set_prefill_chunk(chunk)
        check_prompt(e, o, cfg, synth.prompts(cfg, 90 + P, P), 1, sorted({0, 15, 16, 63, 64, P // 2, P - 2, P - 1} & set(range(P))))
        e.close()


def test_attention_key_splits():
    """1500 positions: a second chunk whose query blocks take several key
    splits, merged in split order; later cache entries match the oracle's."""
    cfg = replace(synth.get_config("tiny_bf16"), name="splits", n_layers=2, hidden=128, n_q_heads=2, n_kv_heads=1,
                  ffn=256, vocab=512, readout_layers=(1,))
    w = synth.generate_weights(cfg)
    P = 1500
    o = oracle_for(cfg.name, P + 2, cfg=cfg, weights=w)
    e = engine(cfg.name, P + 2, page_size=64, cfg=cfg, weights=w)
    check_prompt(e, o, cfg, synth.prompts(cfg, 91, P), 1, [0, 1023, 1024, 1100, 1279, 1280, 1498, 1499])
    e.close()


@pytest.mark.parametrize("name", ["tiny", "tiny_bf16"])
def test_copies_made_per_product_give_the_same(name):
    """A context that has given its weight copies back makes them one at a time: the same cache bits and logits,
    over chunks, a refresh and replaced weights."""
    from paper_2609_14144_amd import lib
    cfg = replace(synth.get_config(name), n_layers=3, vocab=600, readout_layers=(1,))
    w = synth.generate_weights(cfg)
    prompt = synth.prompts(cfg, 14, 90)
    other = {"layers.1.w_down": synth.generate_weights(cfg, seed=1)["layers.1.w_down"]}
    runs = []
    for give_back in (False, True):
        e = engine(name, 128, page_size=16, cfg=cfg, weights=w)
        e.ee_set_prefill_chunk(48)
        if give_back:
            assert lib.ee_test_give_back_tiled(e._ctx) == 0
        got = [e.ee_prefill(prompt)]
        e.ee_decode_n_ex(0.5, 1, 4, force_tokens=prompt[:4], force_exit=np.ones(4, np.int32))
        e.ee_refresh(20)
        e.ee_load_weights(other)
        e.ee_refresh(7)
        got.append(np.stack([np.concatenate(e.ee_read_kv(l, t)) for l in range(3) for t in range(94)]))
        got.append(e.ee_decode_step_ex(0.5, 1, 7, 0)["logits_full"])
        runs.append(got)
        e.close()
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("shape", tile_shapes.SHAPES, ids=lambda s: "%s_H%d_A%d_K%d_F%d" % s[:5])
def test_every_tile(shape):
    """Shapes whose products take every tile of the table in turn (the list is checked against the choice itself on
    the CPU), with remainders of rows, positions and K."""
    cfg = tile_shapes.config(shape)
    w = synth.generate_weights(cfg)
    for P in shape[-1]:
        o = oracle_for(cfg.name, P + 2, cfg=cfg, weights=w)
        e = engine(cfg.name, P + 2, page_size=16, cfg=cfg, weights=w)
        check_prompt(e, o, cfg, synth.prompts(cfg, 110 + P, P), 1, sorted({0, P // 3, P // 2, max(P - 17, 0), max(P - 2, 0), P - 1}))
        e.close()


@pytest.mark.parametrize("G", range(1, 9))
def test_attention_head_groups_f32(G):
    """fp32 caches: every number of query heads per KV head, over two KV heads, about the edges of query blocks and
    key tiles, in one chunk and in several; K padding (104 of 128) in the products."""
    cfg = replace(synth.get_config("tiny"), name="heads_f32", n_layers=2, hidden=104, n_q_heads=2 * G, n_kv_heads=2,
                  head_dim=64, ffn=152, vocab=512, readout_layers=(1,))
    w = synth.generate_weights(cfg)
    for P, chunk in ((3, None), (64, None), (97, 48), (197, None)):
        o = oracle_for(cfg.name, P + 2, cfg=cfg, weights=w)
        e = engine(cfg.name, P + 2, page_size=16, cfg=cfg, weights=w)
        if chunk:
            e.ee_set_prefill_chunk(chunk)
        check_prompt(e, o, cfg, synth.prompts(cfg, 120 + P, P), 1, sorted({0, 15, 16, 63, 64, P // 2, P - 2, P - 1} & set(range(P))))
        e.close()


def test_attention_key_splits_f32():
    """As test_attention_key_splits over an fp32 cache."""
    cfg = replace(synth.get_config("tiny"), name="splits_f32", n_layers=2, hidden=128, n_q_heads=2, n_kv_heads=1,
                  ffn=256, vocab=512, readout_layers=(1,))
    w = synth.generate_weights(cfg)
    P = 1500
    o = oracle_for(cfg.name, P + 2, cfg=cfg, weights=w)
    e = engine(cfg.name, P + 2, page_size=64, cfg=cfg, weights=w)
    check_prompt(e, o, cfg, synth.prompts(cfg, 91, P), 1, [0, 1023, 1024, 1100, 1279, 1280, 1498, 1499])
    e.close()
