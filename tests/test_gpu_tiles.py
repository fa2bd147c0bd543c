"""Tiled contractions over the sequence at the edges of their tiles: the projected keys and values that the forward
leaves in ctx (fp32 sums of bf16 products) against float64."""
import numpy as np
import pytest
import torch

from paper_2306_15799_amd import binding as fb
from paper_2306_15799_amd import inputs
from paper_2306_15799_amd.inputs import Workload, PHI_ELU1, PHI_PERFORMER

import gpu_util as gu

pytestmark = pytest.mark.gpu

# (B, H, n, d, k): key counts around the 64-, 128- and 256-row tiles, head counts that leave a column tile ragged, one
# reduction step and a last one of 8 to 56 positions, one split and many, more tiles than compute units (in a number that
# is no multiple of 8: ids past the last tile).  test_plans.py holds the list to every tile at both head sizes, each with
# ragged edges, a split reduction and several tiles to a workgroup.
SHAPES = [
    # 64 x 128 tiles
    (1, 1, 8, 64, 1), (1, 3, 56, 64, 63), (1, 3, 64, 128, 64), (1, 5, 72, 64, 65), (2, 3, 1000, 64, 100),
    (1, 1, 2048, 128, 127), (1, 7, 520, 64, 128), (1, 3, 2056, 128, 129), (2, 8, 2000, 64, 257), (1, 16, 1032, 128, 300),
    (8, 80, 136, 64, 33), (1, 2, 8200, 64, 20), (7, 37, 72, 64, 33), (1, 33, 40, 128, 304),
    # 128 x 128
    (4, 8, 4096, 64, 255), (4, 4, 4104, 128, 256), (1, 42, 24, 64, 853), (5, 5, 200, 64, 514), (3, 3, 856, 64, 746),
    (1, 17, 8, 64, 1376), (3, 1, 920, 128, 1036), (1, 13, 8, 128, 1405),
    # 128 x 256
    (7, 22, 72, 64, 618), (9, 9, 136, 128, 609), (1, 41, 72, 128, 377), (2, 7, 2280, 64, 1044), (2, 53, 8, 64, 875),
    (1, 13, 2184, 128, 526), (5, 29, 8, 128, 373),
    # 256 x 256
    (4, 24, 200, 128, 400), (1, 17, 2352, 64, 1460), (1, 47, 8, 64, 1496), (3, 3, 2400, 128, 1421), (1, 77, 8, 128, 456)]


@pytest.mark.parametrize("shape", SHAPES)
def test_projected_keys_and_values(shape):
    B, H, n, d, k = shape
    w = Workload("tiles", B, H, n, d, k, d, "bf16", PHI_ELU1, False)
    t = inputs.make_inputs(w, 3)
    if H > 1:
        # what lies behind a head's last position in memory must not reach that head
        t["K"][:, 1, 0, :] = np.inf
        t["V"][:, 1, 0, :] = np.inf
    g = gu.to_device(t, "bf16")
    _, ctx = fb.flurka_attn_fwd(g["Q"], g["K"], g["V"], g["E"], g["F"], g["omega"], phi=w.phi, algo="fast")
    torch.cuda.synchronize()
    v = fb.ctx_views(ctx, B, H, n, d, k, d, fb.BF16, w.phi)
    heads = [h for h in range(H) if h != 1]
    for name, x, e in (("Kp", t["K"], t["E"]), ("Vp", t["V"], t["F"])):
        ref = np.matmul(e.astype(np.float64), x[:, heads].astype(np.float64))
        got = gu.to_host(v[name]).astype(np.float64)[:, heads]
        # n products are exact in fp32 and added in an order of their own: each partial sum rounds by 2^-24 of
        # itself, and a random walk of n such errors stays within sqrt(n) 2^-24 of the norm
        bar = 2.0 * np.sqrt(n) * 2.0 ** -24
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(shape, name, f"{err:.2e} of {bar:.2e}")
        assert err <= bar
        # no element far off (a wrong row, column or split), by the same walk: its terms have unit variance
        # times that of one product
        assert np.abs(got - ref).max() <= 8 * bar * np.sqrt((ref ** 2).mean())


# (B, H, n, d, k, m): position and slot counts around the 128- and 256-wide tiles of the gradient products, the
# reduction over (head, coordinate) whole, split a few ways and split into many, tiles that cross a head.  test_plans.py
# holds the list to both tile sizes, whole and split, at both head sizes.
GRAD_SHAPES = [
    # 128 x 128 tiles
    (1, 1, 32, 64, 9, 32), (1, 3, 160, 64, 63, 32), (2, 2, 96, 128, 127, 64), (2, 5, 416, 64, 129, 64),
    (6, 12, 288, 64, 65, 32), (1, 7, 1056, 64, 128, 64), (2, 8, 544, 128, 300, 64), (16, 8, 128, 64, 40, 32),
    (1, 2, 4128, 64, 256, 64), (1, 2, 96, 128, 70, 32),
    # 256 x 256
    (5, 1, 5152, 64, 262, 32), (2, 1, 8352, 128, 204, 32), (3, 32, 160, 64, 699, 32), (3, 17, 192, 128, 693, 32)]


@pytest.mark.parametrize("shape", GRAD_SHAPES)
def test_gradients(shape):
    B, H, n, d, k, m = shape
    w = Workload("tiles", B, H, n, d, k, m, "bf16", PHI_PERFORMER, True)
    print(shape, gu.check_forward_backward(w, seed=5, algo="fast"))


# elu map at head size 64 (dQ, dS and dz in one pass): one query tile, fewer tiles than wavefronts, ranges that leave some
# wavefronts a tile short, one head over many ranges, more heads than compute units
@pytest.mark.parametrize("shape", [(1, 1, 32, 64, 16), (1, 3, 288, 64, 40), (2, 5, 1056, 64, 100), (1, 1, 8224, 64, 64),
                                   (9, 30, 64, 64, 33)])
def test_elu_gradients(shape):
    B, H, n, d, k = shape
    w = Workload("tiles", B, H, n, d, k, d, "bf16", PHI_ELU1, True)
    print(shape, gu.check_forward_backward(w, seed=6, algo="fast"))


# the first key tile, the second and the last ones: one tile per wavefront, two, three and four, several
@pytest.mark.parametrize("far", [slice(0, 32), slice(32, 64), slice(-40, None)], ids=["first", "second", "last"])
@pytest.mark.parametrize("B,H,n,d,k,m", [(1, 2, 64, 64, 64, 64), (1, 2, 96, 128, 96, 40), (1, 2, 640, 64, 600, 32),
                                         (1, 1, 1024, 64, 1000, 40), (3, 80, 128, 64, 128, 64), (1, 1, 1088, 64, 1056, 32)])
def test_keys_too_long_for_their_squared_norm(B, H, n, d, k, m, far):
    """Whole tiles of projected keys with |k'|^2 beyond float32: exponents of -inf, weights of 0."""
    w = Workload("far_keys", B, H, n, d, k, m, "bf16", PHI_PERFORMER, True)
    t = inputs.make_inputs(w, 3)
    t["E"][far] *= np.float32(2.0 ** 66)
    print((B, H, n, d, k, m), far, flush=True)
    g, out, ctx = gu.run_forward(w, t, "fast")
    grads = gu.run_backward(w, g, out, ctx, "fast")
    errs = {"out": gu.rel_err(gu.to_host(out), gu.oracle_forward(w, t))}
    for name, a, b in zip(("dQ", "dK", "dV", "dE", "dF"), grads, gu.oracle_backward(w, t)):
        errs[name] = gu.rel_err(gu.to_host(a), b)
    print({x: f"{v:.2e}" for x, v in errs.items()})
    assert all(v <= gu.TOL["bf16"] for v in errs.values()), errs
