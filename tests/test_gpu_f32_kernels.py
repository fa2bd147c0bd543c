"""GPU parity of the fp32-arithmetic kernels at the sizes where their tiling can go wrong: one element
below, at and above the 32-, 64- and 128-wide tiles, odd row lengths (element-aligned loads), reductions
split over workgroups, head sizes between and above the padded ones."""
import pytest

from paper_2306_15799_amd.inputs import Workload, PHI_ELU1, PHI_PERFORMER

import gpu_util as gu

pytestmark = pytest.mark.gpu

# (B, H, n, d, k, m)
SHAPES = [
    (1, 2, 127, 31, 63, 33),
    (1, 2, 128, 32, 64, 32),
    (2, 1, 129, 33, 65, 31),
    (1, 1, 2049, 64, 130, 65),        # one head: the projection's reduction is split
    (2, 2, 515, 96, 129, 127),
    (1, 2, 321, 128, 40, 129),
    (1, 1, 260, 136, 50, 200),        # above the largest padded head size
    (3, 40, 70, 64, 33, 40),          # many heads: the larger tiles
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("phi", [PHI_PERFORMER, PHI_ELU1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_tile_edges(shape, phi, dtype):
    B, H, n, d, k, m = shape
    w = Workload("f32_edges", B, H, n, d, k, d if phi == PHI_ELU1 else m, dtype, phi, True)
    errs = gu.check_forward_backward(w, seed=n + d, algo="generic")
    print(shape, phi, dtype, {x: f"{v:.2e}" for x, v in errs.items() if ":" not in x})


# (B, H, n, d, k, m): reductions of dE, dF over many heads split over workgroups (bf16 storage) and summed 4
# results at a time with 0 to 3 left over; reductions one group short of, at and past a 32-deep step; head
# sizes whose heads do not end on a step
@pytest.mark.parametrize("shape", [(4, 8, 301, 64, 70, 40), (4, 8, 303, 64, 71, 40), (2, 8, 129, 80, 33, 24),
                                   (1, 6, 257, 128, 28, 33), (1, 3, 200, 12, 36, 16)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_split_gradients_and_short_reductions(shape, dtype):
    B, H, n, d, k, m = shape
    errs = gu.check_forward_backward(Workload("f32_split", B, H, n, d, k, m, dtype, PHI_PERFORMER, True), seed=n + k,
                                     algo="generic")
    print(shape, dtype, {x: f"{v:.2e}" for x, v in errs.items() if ":" not in x})
