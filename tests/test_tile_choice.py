"""The choice of the products' tiles (csrc/ee_tiles.h), compiled for the CPU."""
import os
import random
import shutil
import subprocess

import pytest

from tests.conftest import ROOT
from tests.tile_shapes import SHAPES, products


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    exe = str(tmp_path_factory.mktemp("tiles") / "tile_choice")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2609_14144_amd", "csrc"), os.path.join(ROOT, "tests", "tile_choice.cpp"),
                    "-o", exe], check=True)

    def ask(queries):
        r = subprocess.run([exe], input="\n".join(" ".join(map(str, q)) for q in queries), text=True, check=True,
                           capture_output=True).stdout.split("\n")
        return tuple(map(int, r[0].split())), [tuple(map(int, l.split())) for l in r[1:1 + len(queries)]]
    return ask


def test_the_tested_shapes_take_every_tile(choose):
    q = [p for s in SHAPES for P in s[-1] for p in products(s, P)]
    counts, got = choose(q)
    for w, n in zip((2, 4), counts):
        assert {t for p, (t, _) in zip(q, got) if p[0] == w} == set(range(n)), w
    # K slices too, of products of both kinds of position tile
    assert {p[3] <= 16 for p, (_, s) in zip(q, got) if s > 1} == {True, False}


def test_slices_fit_the_workspace_and_the_rows_of_k(choose):
    r = random.Random(3)
    q = []
    for _ in range(4000):
        w = r.choice([2, 4])
        P, K = r.randint(1, 1024), 8 * r.randint(1, 1376 if w == 2 else 128)
        N = 8 * r.randint(1, 256)
        q.append((w, 1, 0, P, N, K, r.choice([P * N, 3 * P * N + 1, 8 << 20]), 256))
    for p, (tile, splits) in zip(q, choose(q)[1]):
        assert 1 <= splits <= 16 and splits * p[3] * p[4] <= p[6]
        assert splits == 1 or (p[5] + 63) // 64 // splits >= 4
    # no room for one slice: refused
    assert choose([(2, 1, 0, 100, 64, 64, 100 * 64 - 1, 256)])[1] == [(0, 0)]
