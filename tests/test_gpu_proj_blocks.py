"""The projections' backward at the edges of its token blocks (32, 64 and 128
tokens per workgroup, the last one partly empty), of its stages of 64 features
(odd numbers of 32-feature halves, projections that end inside a stage) and of
the gradient sums (one and several token chunks), against the fp64 oracle with
the bounds of the shape tests."""
import pytest
import torch

from paper_2404_11068_amd import workloads as W
from tests.test_gpu_proj import run_bwd, test_linear_forward_backward as linear_case

pytestmark = pytest.mark.gpu

LN = [
    # R, C, HD, P, bias
    (31, 256, 32, 1, True), (33, 256, 96, 3, True), (8193, 256, 32, 1, False),   # 32 tokens a block
    (16385, 256, 64, 1, True), (32801, 256, 32, 2, True),                         # 64, 128 tokens
    (65, 128, 32, 3, True), (16447, 128, 64, 1, False),
    (127, 64, 96, 1, True), (129, 64, 32, 3, True), (40001, 64, 64, 2, True),
]


@pytest.mark.parametrize("case", LN, ids=lambda c: "R%d_C%d_HD%d_P%d_b%d" % c)
def test_layernorm_backward(case):
    R, C, HD, P, bias = case
    w = W.ProjWorkload("adhoc", R, C, HD, n_proj=P, bias=bias, seed=R + 5 * C + HD)
    run_bwd(w, W.generate_proj(w), str(case), seed=R + 1)


PLAIN = [(1, 128, 32, 1, True), (63, 128, 160, 1, True), (8191, 256, 128, 1, True), (257, 64, 96, 2, False),
         (33, 256, 288, 1, True)]


@pytest.mark.parametrize("case", PLAIN, ids=lambda c: "R%d_C%d_HD%d_P%d_b%d" % c)
def test_plain_backward(case):
    linear_case(case)
    torch.cuda.synchronize()
