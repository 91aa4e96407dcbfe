"""Decoders whose heads are wider together than the residual stream
(A * D > H): a row of W_o then has more 16-byte chunks per lane than a row of
any H-wide matrix. Against the CPU oracle, with the tolerances of
tests/gpu_helpers.py."""
from dataclasses import replace

import pytest

import synth
from tests.gpu_helpers import MARGIN, check_kv, engine, lockstep, oracle_for

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# (storage, H, A, K, D): chunks per lane of H-wide rows and of W_o's are 1 and
# 2, 1 and 4, 2 and 3, 1 and 2; the last three have more than any program has (6, 9 and 3)
SHAPES = [("tiny_bf16", 128, 10, 2, 64), ("tiny_bf16", 64, 16, 2, 128), ("tiny_bf16", 520, 10, 2, 128),
          ("tiny", 256, 8, 2, 64), ("tiny_bf16", 64, 24, 3, 128), ("tiny_bf16", 1000, 33, 11, 128),
          ("tiny", 256, 12, 2, 64)]


@pytest.mark.parametrize("persistent", [True, False], ids=["persistent", "per_op"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "%s_H%d_A%d_K%d_D%d" % s)
def test_heads_wider_than_the_stream(shape, persistent):
    name, H, A, K, D = shape
    cfg = replace(synth.get_config(name), name="wide_heads", n_layers=2, hidden=H, n_q_heads=A, n_kv_heads=K,
                  head_dim=D, ffn=256, vocab=512, readout_layers=(1,))
    w = synth.generate_weights(cfg)
    prompt = synth.prompts(cfg, 31, 21)
    for chunk in (0, 16):
        o = oracle_for(cfg.name, 32, cfg=cfg, weights=w)
        e = engine(cfg.name, 32, persistent, page_size=16, cfg=cfg, weights=w)
        e.ee_set_prefill_chunk(chunk)
        g0, g = o.prefill(prompt), e.ee_prefill(prompt)
        if o.last_prefill_stats[2] > MARGIN:
            assert g == g0
        check_kv(e, o, cfg, range(2), [0, 15, 16, 20])
        lockstep(e, o, g0, 0.5, 1, 3, force_tokens=synth.prompts(cfg, 32, 3), force_exit=[0, 1, 0])
        e.close()
