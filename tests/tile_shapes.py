"""Two-layer decoders and prompt lengths whose products between them take
every tile of csrc/ee_tiles.h, with a remainder of rows, positions or K in
most (tests/test_tile_choice.py holds the list to that;
tests/test_gpu_batched_pass.py runs it)."""
from dataclasses import replace

import synth

# storage, H, A, K, F, positions; D = 64
SHAPES = [
    ("bf16", 72, 2, 1, 104, (5, 17)),
    ("bf16", 520, 2, 1, 104, (5, 20)),
    ("bf16", 520, 16, 2, 104, (5, 257)),
    ("bf16", 72, 2, 1, 15200, (33, 97)),
    ("bf16", 72, 3, 1, 4800, (130,)),
    ("bf16", 72, 1, 1, 12000, (70, 240)),
    ("bf16", 200, 4, 2, 2000, (477,)),
    ("bf16", 776, 7, 1, 4800, (300,)),
    ("f32", 72, 3, 1, 104, (5, 50)),
    ("f32", 456, 6, 1, 200, (9, 33)),
    ("f32", 72, 2, 1, 12000, (600,)),
]


def config(shape):
    dt, H, A, K, F, _ = shape
    return replace(synth.get_config("tiny_bf16" if dt == "bf16" else "tiny"), name="tiles", n_layers=2, hidden=H,
                   n_q_heads=A, n_kv_heads=K, head_dim=64, ffn=F, vocab=520, readout_layers=(1,))


def products(shape, P):
    """(bytes, resid, qkv, P, N, K, workspace floats, compute units) of the first layer's four products."""
    dt, H, A, K, F, _ = shape
    w, qkv, ad = (2 if dt == "bf16" else 4), (A + 2 * K) * 64, A * 64
    room = min(8 << 20, 32 * min(1024, P + 2) * max(qkv, 2 * F, H))
    return [(w, int(resid), int(is_qkv), P, N, k, room, 256)
            for resid, is_qkv, N, k in ((0, 1, qkv, H), (1, 0, H, ad), (0, 0, 2 * F, H), (1, 0, H, F))]
