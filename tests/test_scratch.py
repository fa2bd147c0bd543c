"""Scratch sizes of the MFMA path."""
import os
import random

import plans
from paper_2306_15799_amd import binding as fb

HERE = os.path.dirname(os.path.abspath(__file__))


def _up(x):
    return -(-x // 256) * 256


def _partial_bytes(p):
    tile = 128 if p.fine else 256
    return 0 if p.splits == 1 else 2 * p.splits * p.tilesM * p.tilesN * tile * tile * 4


def test_the_elu_backward_asks_for_what_its_kernels_use():
    """dK', dV' images, dS and dz of every query range and summed, split partials of dE, dF; two numbers per query row at
    head size 128, none at 64."""
    rng = random.Random(5)
    shapes = [(4, 16, 16384, 64, 256), (1, 1, 32, 64, 1), (1, 2, 8192, 128, 100)]
    shapes += [(rng.choice([1, 2, 4, 8]), rng.randint(1, 16), 32 * rng.randint(1, 300), rng.choice([64, 128]), rng.randint(1, 600))
               for _ in range(300)]
    for (B, H, n, d, k), p in zip(shapes, plans.grad(shapes)):
        BH, kp = B * H, -(-k // 64) * 64
        # ranges of all heads together: two rounds of workgroups, or as many as leave at most a tenth of a round empty
        ranges = max(BH, 2 * plans.CUS) if d == 128 else BH + 10 * plans.CUS
        bound = 2 * _up(4 * BH * kp * d) + _up(4 * ranges * d * d) + _up(4 * ranges * d) + _up(4 * BH * d * d) + _up(4 * BH * d)
        bound += _up(_partial_bytes(p)) + (2 * _up(4 * BH * n) if d == 128 else 0)
        got = fb.workspace_bytes(B, H, n, d, k, d, fb.BF16, "elu1", fb.PASS_BWD, "fast")
        assert 0 < got <= bound, ((B, H, n, d, k), got, bound)


def test_no_shape_asks_for_more_than_it_used_to():
    """Buffers that a caller sized once stay large enough: recorded sizes of 200 shapes, 80 of which smaller tiles with
    more splits of dE, dF had outgrown."""
    with open(os.path.join(HERE, "golden", "scratch_bytes.txt")) as f:
        rows = [[int(x) for x in line.split()] for line in f if not line.startswith("#")]
    assert len(rows) == 200
    for B, H, n, d, k, m, phi, *bytes_ in rows:
        for pass_, was in zip((fb.PASS_FWD, fb.PASS_BWD), bytes_):
            assert 0 < fb.workspace_bytes(B, H, n, d, k, m, fb.BF16, phi, pass_, "fast") <= was, (B, H, n, d, k, m, phi, pass_)
