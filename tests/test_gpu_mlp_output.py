"""GPU: the perceptron's output layer for at most 16 classes at the edges of what a workgroup takes: samples in sixteens (logits) and
hundreds and twenty-eights (backward), hidden units in sixteens, sixteen wavefronts' shares of them (eight beyond 256 workgroups), some without
any, and, backward, in thirty-twos up to 256 workgroups and in sixty-fours beyond; one, two and sixteen classes."""
import pytest

from test_gpu_parity import test_mlp2_gradient_single_step as gradient_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [
    dict(d_in=70, d_hidden=1, d_out=2, B_loc=1, K=2),
    dict(d_in=70, d_hidden=31, d_out=16, B_loc=15, K=1),
    dict(d_in=70, d_hidden=33, d_out=3, B_loc=17, K=3),
    dict(d_in=70, d_hidden=64, d_out=16, B_loc=127, K=1),
    dict(d_in=70, d_hidden=257, d_out=10, B_loc=16, K=2),
    dict(d_in=70, d_hidden=65, d_out=7, B_loc=129, K=2),
    dict(d_in=70, d_hidden=40, d_out=2, B_loc=260, K=1),
    dict(d_in=70, d_hidden=50, d_out=9, B_loc=512, K=8),        # 256 workgroups of sixteen wavefronts
    dict(d_in=70, d_hidden=130, d_out=16, B_loc=513, K=8),      # 264 of eight, the last of a worker with one sample; three of them without units
    dict(d_in=70, d_hidden=50, d_out=2, B_loc=1100, K=4),       # 276 of eight, four of them without units
    dict(d_in=10, d_hidden=1024, d_out=10, B_loc=20, K=8),      # 256 workgroups of 32 units
    dict(d_in=10, d_hidden=1025, d_out=10, B_loc=129, K=8),     # 136 of 64, the last with one unit
    dict(d_in=10, d_hidden=1983, d_out=16, B_loc=33, K=5),      # 155 of 64, the last one unit short
])
def test_output_layer(dims):
    gradient_case(dims)
