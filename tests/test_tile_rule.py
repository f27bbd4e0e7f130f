"""The rule that chooses the tile shape of the large-tile kernel's bf16 products:
its bounds over many shapes, and the choices that were measured."""
import math
import random

import pytest

from host_rules import run_program

BODY = """
    int N, work, T, k, ncol, K, part, bn0;
    std::cin >> N >> work >> T >> k >> ncol >> K >> part >> bn0;
    const lx::TilePick p = lx::pick_tile(N, work, T, k, ncol, K, part, bn0);
    std::printf("%d %d %d %.9g %.9g\\n", p.bm, p.bn, (int)p.base, p.us, p.base_us);
"""
SHAPES = {(256, 256), (256, 128), (256, 64), (128, 128), (128, 64)}


def _pick(tmp_path, cases):
    return [(int(a), int(b), int(c), float(d), float(e)) for a, b, c, d, e in run_program(tmp_path, "lx_tiles.h", BODY, cases)]


def _products(E, C, d, f, r):
    """(N, work, ncol, K, part_cols, bn0) of a flat layer's six products."""
    M = E - C
    return {"gate_up": (C, C, 2 * f, d, 0, 256), "down": (C, C, d, 2 * f, 0, 256),
            "low_in": (E, M, 2 * r, d, 0, 128 if 2 * r <= 128 else 256),
            "low_out": (E, M, 2 * f, 2 * r, f, 256 if f % 256 == 0 else 128 if f % 128 == 0 else 64),
            "down_in": (E, M, r, 2 * f, 0, 64 if r <= 64 else 128), "down_out": (E, M, d, 2 * r, 0, 256)}


def test_bounds(tmp_path):
    rng = random.Random(11)
    cases = []
    while len(cases) < 1500:
        C = rng.choice((1, 2, 4, 16, 64, 128))
        E = C * rng.choice((1, 2, 8))
        if E == C:
            E = 2 * C
        d, f, r = 64 * rng.randint(1, 64), 64 * rng.randint(1, 32), rng.choice((32, 64, 96, 128))
        T, k = int(round(math.exp(rng.uniform(0, math.log(200000))))), rng.randint(1, min(8, E))
        for N, work, ncol, K, part, bn0 in _products(E, C, d, f, r).values():
            cases.append((N, work, T, k, ncol, K, part, bn0))
    kept = changed = 0
    for (N, work, T, k, ncol, K, part, bn0), (bm, bn, base, us, base_us) in zip(cases, _pick(tmp_path, cases)):
        assert (bm, bn) in SHAPES and bn <= bn0 and (part == 0 or part % bn == 0)
        assert bool(base) == ((bm, bn) == (256, bn0))
        assert math.isfinite(us) and 0 < us <= base_us and (base or us < 0.9 * base_us)
        mean = T * (1 - (1 - 1 / N) ** k)
        # at least one tile, and at least rows / 256, per node
        if work * max(1.0, mean / 256) * -(-ncol // bn0) >= 256:
            assert base, (N, work, T, k, ncol, K, part, bn0)
            kept += 1
        changed += not base
    assert kept > 300 and changed > 100


# measured, us: 256 x 256, 256 x 128, 256 x 64, 128 x 128, 128 x 64 (d = 2048, k = 8)
@pytest.mark.parametrize("E,C,f,r,T,product,want,us", [
    (128, 16, 768, 64, 237, "gate_up", (128, 128), (53.9, 36.9, 61.5, 31.7, 44.0)),
    (128, 16, 768, 64, 400, "gate_up", (256, 128), (55.2, 35.3, 60.1, 55.0, 60.6)),
    (128, 16, 768, 64, 700, "gate_up", (256, 256), (57.0, 67.6, 87.1, 77.8, 96.2)),
    (128, 16, 768, 64, 237, "down", (128, 128), (43.7, 31.4, 48.6, 26.9, 36.0)),
    (128, 16, 704, 64, 8192, "low_in", (256, 128), (117.2, 76.2, 93.6, 61.8, 81.6)),
    (128, 16, 704, 64, 8192, "down_in", (256, 64), (97.3, 76.9, 71.8, 59.8, 55.0)),
    (128, 16, 704, 64, 4096, "low_out", (256, 64), (None, None, 71.3, None, 80.7)),
    (256, 64, 1280, 32, 200, "low_in", (128, 64), (55.0, 34.8, 32.9, 30.0, 23.5)),
    (256, 64, 1280, 32, 200, "down_in", (128, 64), (64.7, 40.5, 38.1, 34.4, 27.2)),
    (256, 64, 1280, 32, 200, "low_out", (256, 256), (41.1, 47.3, 92.0, 48.2, 73.1)),
])
def test_measured_choices(tmp_path, E, C, f, r, T, product, want, us):
    N, work, ncol, K, part, bn0 = _products(E, C, 2048, f, r)[product]
    (bm, bn, *_), = _pick(tmp_path, [(N, work, T, 8, ncol, K, part, bn0)])
    assert (bm, bn) == want
    t = dict(zip(((256, 256), (256, 128), (256, 64), (128, 128), (128, 64)), us))
    assert t[want] <= t[(256, bn0)]
