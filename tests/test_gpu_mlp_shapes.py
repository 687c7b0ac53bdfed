"""GPU: the perceptron's gradient at the sizes where its kernels change form: fp64 products through LDS rings or, for
contractions shorter than 64, straight from memory, 128- or 32-bit copies, contractions that are no multiple of a stage or
shorter than the wavefronts' shares, few and many tiles, many classes (column sums and loss inside the GEMMs)."""
import pytest

from test_gpu_parity import test_mlp2_gradient_single_step as gradient_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [
    dict(d_in=260, d_hidden=72, d_out=20, B_loc=21, K=3),       # 32 x 32 tiles; shares without a stage; rows 16-byte aligned
    dict(d_in=64, d_hidden=1000, d_out=4, B_loc=70, K=8),       # 64 x 64 tiles, 128-bit copies of the weights, four stages
    # one, four and two groups per tile, by the number of tiles and the length of the contraction.  With this many hidden
    # units the sizes are ones where none lies within 2e-6 of zero: the draws agree with the oracle's to a few ulp, so a
    # unit at 2e-8 (516 features, 700 units, 180 samples, worker 6) is on in one and off in the other, 6e-4 in a gradient
    dict(d_in=68, d_hidden=1000, d_out=4, B_loc=250, K=8),
    dict(d_in=524, d_hidden=700, d_out=4, B_loc=180, K=8),
    dict(d_in=508, d_hidden=760, d_out=4, B_loc=180, K=6),
    dict(d_in=68, d_hidden=1000, d_out=5, B_loc=70, K=8),       # 32-bit copies, a last stage of four
    dict(d_in=67, d_hidden=1000, d_out=5, B_loc=70, K=8),       # 32-bit copies, padded rows, a last stage of three
    dict(d_in=333, d_hidden=50, d_out=100, B_loc=5, K=2),       # the same, few tiles, contractions of 333 and 50 (straight from memory)
    # straight from memory on 64 x 64 tiles, 264 of them (no hidden unit within 8e-6 of zero)
    dict(d_in=43, d_hidden=650, d_out=5, B_loc=190, K=8),
    dict(d_in=32, d_hidden=64, d_out=1024, B_loc=9, K=1),       # the most classes
    dict(d_in=48, d_hidden=17, d_out=65, B_loc=130, K=2),       # one class beyond a wavefront's lanes
])
def test_gradient_where_the_kernels_change(dims):
    gradient_case(dims)
