"""The bf16 contraction's ragged tiles: sides of one to four 64-row units, in
the plain (256-row grid, short last tile) and the transposed operand order
(units spread evenly), the same sums bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_14806_amd import trimul as T
from tests.gpu_util import host, make_layer, needs_gpu, say

pytestmark = [pytest.mark.gpu, needs_gpu]
CHANNELS = [0, 77, 127]


# one tile of 1, 2, 3 units; 5 = 4 + 1 | 3 + 2, 7 = 4 + 3, 9 = 4 + 4 + 1 | 3 + 3 + 3, 10 = 4 + 4 + 2 | 4 + 3 + 3 units
@pytest.mark.parametrize("N", [33, 66, 130, 290, 449, 513, 639])
def test_ragged_tiles_exact_on_integers(N):
    say(f"ragged tiles N={N}")
    layer, _ = make_layer("bf16")
    g = torch.Generator().manual_seed(N)
    A, B = (torch.randint(-4, 5, (128, N, N), generator=g).to(torch.bfloat16) for _ in range(2))
    ref = oracle.block_contract([host(A[CHANNELS])], [host(B[CHANNELS])], [np.ones(N)])
    plain = layer.contract(T.dense_to_panel(A).cuda(), T.dense_to_panel(B).cuda(), N)
    turned = layer.contract_transposed(*(T.dense_to_panel(X.transpose(1, 2).contiguous()).cuda() for X in (A, B)), N)
    torch.cuda.synchronize()
    a, b = (T.result_to_dense(C, N) for C in (plain, turned))
    np.testing.assert_array_equal(host(a[CHANNELS]).transpose(1, 2, 0), ref)
    assert torch.equal(a, b)
