"""Which kernels a fp32 linear step takes: the sizes of test_gpu_linear_f32.py reach what they are there for, and the rule's edges.  Host only."""
import pytest

pytest.importorskip("torch")

from paper_2401_11504_amd import api  # noqa: E402
from test_gpu_linear_f32 import CASES, DIRECT16, DIRECT32, SHORT, SPLIT  # noqa: E402

D16, D32, F64, S128, S256 = "direct-16x16", "direct-32x32", "64x64", "split-128x128", "split-256x128"


@pytest.mark.parametrize("sizes,main", list(zip(CASES, [D16] * 6 + [D32] + [F64] * 4 + [S128] * 3 + [S256] * 2)) +
                         list(zip(SPLIT, [S256] + [S128] * 3)) + [(c, D16) for c in DIRECT16] + [(c, D32) for c in DIRECT32] +
                         [((2, (1 << 22) + 3, 3, 2), "wide-64x64"), ((3, 5, (1 << 22) + 1, 4), "wide-64x64"), ((70, (1 << 22) + 6, 2, 1), "wide-64x64")])
def test_sizes_reach_the_kernel_they_are_for(sizes, main):
    assert api.tl_k_linear_step_plan(*sizes)[1] == main


@pytest.mark.parametrize("sizes", CASES + SPLIT + DIRECT16 + DIRECT32)
def test_low_rank_products_are_small_tiles(sizes):
    assert api.tl_k_linear_step_plan(*sizes)[0] == D16


# where an output shares memory with an input, each product is a launch of its own: H, Y, dH, dX, dA, dB
@pytest.mark.parametrize("sizes,launch,kernel", [((700, 1200, 1111, 37), 1, F64), ((700, 1200, 1111, 37), 3, F64), ((8192, 63, 4096, 3), 1, S256),
                                                 ((1027, 4096, 2050, 64), 4, D32), ((2, (1 << 22) + 3, 3, 2), 0, "wide-32x32")] +
                         [(c, 1 if c[1] < c[2] else 3, ("direct", F64) if min(c[1:3]) < 32 else S128) for c in SHORT])
def test_products_one_by_one(sizes, launch, kernel):
    assert api.tl_k_linear_step_plan(*sizes, one_by_one=True)[launch].startswith(kernel)


def test_what_the_split_kernel_leaves_to_the_others():
    sizes = (1024, 4096, 4096, 64)
    assert api.tl_k_linear_step_plan(*sizes)[1] == S256
    for s in (0.0, 2.0 ** -20, 2.0 ** 20, -1.5):                     # scales of the low-rank term
        assert api.tl_k_linear_step_plan(*sizes, s=s)[1] == S256
    for s in (2.0 ** -21, 2.0 ** 21, float("inf"), float("nan")):
        assert api.tl_k_linear_step_plan(*sizes, s=s)[1] == F64
    for short in ((8192, 31, 8192, 4), (8192, 8192, 31, 4), (31, 8192, 8192, 4)):     # contractions of less than a tile
        assert not any(k.startswith("split") for k in api.tl_k_linear_step_plan(*short))


def test_bad_sizes_are_refused():
    with pytest.raises(api.TlError):
        api.tl_k_linear_step_plan(0, 1, 1, 1)
