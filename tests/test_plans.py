"""Which tile and split the sequence-length GEMMs run with."""
import random

import plans


def _draws(count):
    rng = random.Random(4)
    out = []
    while len(out) < count:
        B, H, d = rng.choice([1, 2, 3, 4, 8]), rng.choice([1, 2, 3, 4, 6, 7, 8, 12, 16]), rng.choice([64, 128])
        n, k = 8 * rng.randint(8, 4096), int(round(32 * 64 ** rng.random()))
        if B * H * n * d < 1 << 27:
            out.append((B, H, n, d, k))
    return out


def test_a_split_does_not_cost_a_second_round_of_workgroups():
    """Ids are padded to a multiple of 8 per row tile: a split that fills the chip with items may hand out more ids than
    there are compute units, and the launch then takes two rounds (k 675, n 14624, 6 heads of 128: 128 x 256 tiles in 7
    splits, 252 items with 288 ids, took 56 us, in 8 splits of 256 x 256 ones 46, 128 x 128 in 3 splits 45)."""
    shapes = [(3, 2, 14624, 128, 675)] + _draws(3000)
    for s, p in zip(shapes, plans.proj(shapes)):
        if (p.tm, p.tn) != (256, 256) and p.splits > 1:
            assert plans.ids(p) <= plans.CUS, (s, p)


def test_long_reductions_keep_the_large_tile_where_it_leaves_some_of_the_chip_idle():
    """256 x 256 tiles on 192 to 240 of 256 compute units against 128 x 256 ones, forward passes: 185 and 193 us, 195
    and 204, 215 and 225, 285 and 296."""
    shapes = [(4, 8, 8192, 128, 768), (4, 12, 8192, 64, 1024), (3, 8, 9952, 128, 994), (3, 8, 13280, 128, 1129)]
    assert all((p.tm, p.tn) == (256, 256) for p in plans.proj(shapes))


def test_short_reductions_take_the_small_tiles():
    """Encoder inference 82 us with 128 x 128 tiles, 97 with 256 x 256; a small training step with 64 x 128."""
    a, b = plans.proj([(8, 8, 4096, 64, 256), (2, 2, 512, 64, 64)])
    assert (a.tm, a.tn) == (128, 128) and (b.tm, b.tn) == (64, 128)
