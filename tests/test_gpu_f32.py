"""fp32 storage path: the matrix-core contraction at the edges of its tiles
(64 and 128 wide) and steps (32 k), with NaN in everything that must not count."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_14806_amd import trimul as T
from tests.gpu_util import host, make_layer, needs_gpu, say

pytestmark = [pytest.mark.gpu, needs_gpu]
CHANNELS = [0, 63, 127]   # the addressing is the same in every channel apart from its offset


def _tile(M, N):
    return T.check_contract_tile("f32", M, N, cus=torch.cuda.get_device_properties(0).multi_processor_count)


def _ints(shape, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(-4, 5, shape, generator=g).float()


@pytest.mark.parametrize("N,tile", [(1, 64), (31, 64), (64, 64), (97, 64), (769, 64), (705, 128)])
def test_contract_f32_exact_with_nan_padding(N, tile):
    """Small integers are exact in fp32 in any order of the sums; the panels'
    padding rows and k hold NaN."""
    assert _tile(N, N) == tile
    say(f"f32 contract exact N={N}")
    layer, _ = make_layer("f32")
    A, B = _ints((128, N, N), N), _ints((128, N, N), N + 1)
    dense = torch.zeros((128, N, N))
    hole = T.dense_to_panel(dense + 1) == 0            # True on padding
    panels = []
    for X in (A, B):
        P = T.dense_to_panel(X)
        P[hole] = float("nan")
        panels.append(P.cuda())
    C = layer.contract(panels[0], panels[1], N)
    torch.cuda.synchronize()
    ref = oracle.block_contract([host(A[CHANNELS])], [host(B[CHANNELS])], [np.ones(N)])
    np.testing.assert_array_equal(host(T.result_to_dense(C, N)[CHANNELS]).transpose(1, 2, 0), ref)


@pytest.mark.parametrize("rows,cols,klen,tile", [(1, 130, 33, 64), (100, 65, 70, 64), (900, 770, 45, 64), (833, 705, 45, 128)])
def test_block_accumulate_f32_row_major_exact(rows, cols, klen, tile):
    """Row-major panels over two steps into one accumulator: NaN past klen in
    the row padding and at masked k, exact sums elsewhere."""
    assert _tile(rows, cols) == tile
    say(f"f32 block accumulate exact {rows} x {cols} x {klen}")
    layer, _ = make_layer("f32")
    ld = -(-klen // 8) * 8 + 8
    n = max(rows, cols) + 2 * klen
    mask = (torch.rand(n, generator=torch.Generator().manual_seed(klen)) < 0.7).to(torch.uint8)
    acc = torch.full((128, rows, cols), float("nan"), device="cuda")
    ref = 0
    for step in range(2):
        k0 = step * klen
        dead = torch.ones(ld, dtype=torch.bool)
        dead[:klen] = mask[k0:k0 + klen] == 0
        A, B = _ints((128, rows, ld), 7 + step), _ints((128, cols, ld), 17 + step)
        A[:, :, dead] = float("nan")
        B[:, :, dead] = float("nan")
        view = T.BlockView(n, 0, 0, rows, cols, k0, klen, ld, ld, step, 3)   # a third step, never sent, would run the epilogue
        layer.block_accumulate(view, A.cuda(), B.cuda(), acc, mask.cuda())
        a, b = (torch.nan_to_num(x[CHANNELS, :, :klen]) for x in (A, B))
        ref = ref + oracle.block_contract([host(a)], [host(b)], [mask[k0:k0 + klen].numpy()])
    torch.cuda.synchronize()
    np.testing.assert_array_equal(host(acc[CHANNELS]).transpose(1, 2, 0), ref)
