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


# one tile of 1, 2, 3 units; 5 = 4 + 1 | 3 + 2, 7 = 4 + 3, 8 = whole tiles with a ragged edge,
# 9 = 4 + 4 + 1 | 3 + 3 + 3, 10 = 4 + 4 + 2 | 4 + 3 + 3 units
@pytest.mark.parametrize("N", [33, 66, 130, 290, 447, 449, 513, 639])
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


def _panel(X):
    """Dense [c][rows][K] -> flat blocked panel, its padding NaN."""
    c, rows, K = X.shape
    t, s = -(-rows // 256), -(-K // 32)
    P = torch.full((c, t * 256, s * 32), float("nan"), dtype=X.dtype)
    P[:, :rows, :K] = X
    return P.reshape(c, t, 256, s, 32).permute(0, 1, 3, 2, 4).contiguous().reshape(-1).cuda()


# units of the rows x units of the columns: one tile each way, then more
@pytest.mark.parametrize("rows,cols,klen", [(60, 100, 33), (40, 190, 70), (100, 170, 31), (190, 64, 45), (250, 130, 64),
                                            (300, 190, 40), (447, 65, 70), (130, 570, 33)])
def test_ragged_rectangles_exact_on_integers(rows, cols, klen):
    """Two ring steps into one packed accumulator, in both operand orders:
    exact sums of small integers, with NaN in all of the panels' padding."""
    say(f"ragged rectangle {rows} x {cols} x {klen}")
    layer, _ = make_layer("bf16")
    g = torch.Generator().manual_seed(rows * cols)
    n = max(rows, cols) + 2 * klen
    ld = -(-klen // 8) * 8
    views = [T.BlockView(n, 0, 0, rows, cols, k * klen, klen, ld, ld, k, 3) for k in range(2)]   # a third step would run the epilogue
    accs = [torch.full((layer.block_accumulator_size(views[0]) // 4,), float("nan"), device="cuda") for _ in range(2)]
    ref = 0
    for v in views:
        A, B = (torch.randint(-4, 5, (128, m, klen), generator=g).to(torch.bfloat16) for m in (rows, cols))
        layer.block_accumulate_blocked(v, _panel(A), _panel(B), accs[0])
        layer.block_accumulate_transposed(v, *(_panel(X.transpose(1, 2).contiguous()) for X in (A, B)), accs[1])
        ref = ref + oracle.block_contract([host(A[CHANNELS])], [host(B[CHANNELS])], [np.ones(klen)])
    torch.cuda.synchronize()
    plain, turned = (T.result_to_dense(a, rows, cols=cols) for a in accs)
    np.testing.assert_array_equal(host(plain[CHANNELS]).transpose(1, 2, 0), ref)
    assert torch.equal(plain, turned)
