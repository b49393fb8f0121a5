"""Causal launches whose workgroups are more than the CUs and all start at once, where the order of the blocks folds back behind the first
workgroup of every CU: one block more than the CUs hold singly and the most they hold, heads x sequences that do and do not divide the number
of CUs, a last block of one row.  bf16: the forward pass in every launch shape that fits twice; fp32: the backward pass in one launch."""
import pytest

from test_gpu_attention_f32_launches import test_backward_on_both_sides_of_the_launch_rule as fp32
from test_gpu_attention_one_launch import test_backward_on_both_sides_of_the_launch_rule as bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [16, 32, 48, 64])
@pytest.mark.parametrize("b,s,a", [(1, 513, 8), (2, 512, 8), (1, 450, 16), (3, 161, 11), (1, 512, 16), (1, 1025, 7)])
def test_fp32_backward(dh, b, s, a):
    fp32(dh, b, s, a, 1)


@pytest.mark.parametrize("dh", [32, 64, 24])
@pytest.mark.parametrize("b,s,a", [(4, 1024, 16), (5, 513, 11), (8, 300, 17), (9, 1025, 13), (3, 1153, 12), (2, 2048, 24)])
def test_bf16_forward(dh, b, s, a):
    bf16(dh, b, s, a, 1)


@pytest.mark.parametrize("dh", [16, 32, 48, 64])
@pytest.mark.parametrize("b,s,a", [(4, 138, 8), (1, 286, 16), (1, 537, 8), (4, 77, 16), (2, 128, 24), (2, 224, 11), (1, 150, 30), (2, 128, 26)])
def test_fp32_backward_with_one_two_and_three_positions_turned(dh, b, s, a):
    """Two positions stay as they are where blocks take more than one step and heads x sequences divides the CUs (the first three), and are
    turned elsewhere; one and three."""
    fp32(dh, b, s, a, 1)
