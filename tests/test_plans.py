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


def _tile(p):
    return p.tm, p.tn


TILES = [(64, 128), (128, 128), (128, 256), (256, 256)]


def test_the_projection_is_tested_with_every_tile():
    """At both head sizes: a ragged last reduction step, ragged keys, a ragged column tile where heads can leave one, a
    split reduction, and (the tiles that stream) more ids than workgroups, some of them past the last tile."""
    import test_gpu_tiles
    seen = set()
    for s, p in zip(test_gpu_tiles.SHAPES, plans.proj(test_gpu_tiles.SHAPES)):
        B, H, n, d, k = s
        if n % 64 and k % p.tm:
            seen.add((_tile(p), d, "ragged rows"))
            if B * H * d % p.tn:
                seen.add((_tile(p), d, "ragged columns"))
            if p.splits > 1:
                seen.add((_tile(p), d, "split"))
        if plans.ids(p) > plans.CUS and p.splits * p.tilesN * 2 % 8:
            seen.add((_tile(p), d, "ids past the end"))
    want = {(t, d, x) for t in TILES for d in (64, 128) for x in ("ragged rows", "ragged columns", "split", "ids past the end")}
    want -= {(t, 128, "ragged columns") for t in TILES if t[1] == 128}          # a head is a whole column tile
    want -= {((256, 256), d, "ids past the end") for d in (64, 128)}            # ids of that tile are not padded here
    assert want <= seen, sorted(want - seen)


def test_the_paper_order_products_are_tested_with_every_tile():
    import test_gpu_paper_order as t
    shapes = [s[:5] + (s[6],) for s in t.SHAPES] + t.TILE_SHAPES
    seen = [set(), set()]
    for s, both in zip(shapes, plans.fused(shapes)):
        B, H, n, d, k, dm = s
        for i, p in enumerate(both):
            if k % p.tm:
                seen[i].add(_tile(p))
                if B > 1:
                    seen[i].add((_tile(p), "batches"))
                if i == 0 and n % 64 and dm % p.tn:
                    seen[i].add((_tile(p), "ragged"))
    assert {x for t_ in TILES for x in (t_, (t_, "batches"), (t_, "ragged"))} <= seen[0]
    assert {x for t_ in TILES for x in (t_, (t_, "batches"))} <= seen[1]


def test_the_gradient_products_are_tested_with_both_tiles_whole_and_split():
    import test_gpu_tiles
    shapes = test_gpu_tiles.GRAD_SHAPES
    seen = {(p.fine, p.splits > 1, s[3]) for s, p in zip(shapes, plans.grad(shapes))
            if s[2] % (128 if p.fine else 256) and s[4] % 64}
    assert seen == {(fine, split, d) for fine in (False, True) for split in (False, True) for d in (64, 128)}


def test_a_plan_does_not_depend_on_the_ones_before_it():
    """Each thread keeps its last plans by their sizes: every shape alone, among many, and again in another order."""
    shapes = _draws(40) + [(2, 2, 512, 64, 64), (2, 2, 512, 64, 65), (2, 2, 520, 64, 64), (2, 2, 512, 128, 64), (1, 4, 512, 64, 64)]
    for ask in (plans.proj, plans.grad):
        once = ask(shapes)
        assert ask([s for s in shapes for _ in range(2)]) == [p for p in once for _ in range(2)]
        assert ask(shapes[::-1] + shapes) == once[::-1] + once
    for s, p in list(zip(shapes, plans.proj(shapes)))[-5:]:
        assert plans.proj([s]) == [p]
