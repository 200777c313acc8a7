"""Calls without a mask run kernels that load none: bit for bit the calls with
a mask of any non-zero bytes (which the other tests hold to the oracle), from
one line of pairs to several per work-group, full updates and device tiles."""
import pytest
import torch

from paper_2603_14806_amd import synth
from paper_2603_14806_amd import trimul as T
from tests.gpu_util import make_layer, needs_gpu, say

pytestmark = [pytest.mark.gpu, needs_gpu]


@pytest.mark.parametrize("out_dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N", [1, 33, 100, 257, 400])   # 400: 5200 lines and units, ten and more per work-group
def test_update_without_mask_is_the_all_real_mask(N, out_dtype):
    say(f"no mask, update N={N} out={out_dtype}")
    layer, _ = make_layer("bf16", out_dtype, affine=True)
    z = synth.pair_tensor(N, dtype="bf16", seed=N, device="cuda")
    ones = torch.full((N,), 0x80, dtype=torch.uint8, device="cuda")
    ones[::2] = 1
    for direction in ("outgoing", "incoming"):
        got, ref = layer(z, None, direction), layer(z, ones, direction)
        torch.cuda.synchronize()
        assert torch.isfinite(got).all()
        assert torch.equal(got, ref), direction


@pytest.mark.parametrize("rows,cols", [(40, 100), (300, 33)])
def test_tile_without_mask_is_the_all_real_mask(rows, cols):
    say(f"no mask, tile {rows} x {cols}")
    layer, _ = make_layer("bf16")
    n, row0, col0 = 500, 150, 7
    z = synth.pair_tensor(n, dtype="bf16", seed=rows, device="cuda", shape=(rows, cols, 128))
    ones = torch.full((n,), 3, dtype=torch.uint8, device="cuda")
    klen = 65
    ld = -(-klen // 8) * 8
    view = T.BlockView(n, row0, col0, rows, cols, 11, klen, ld, ld, 0, 1)
    gen = torch.Generator(device="cuda").manual_seed(cols)
    at, bt = (torch.randn(layer.block_panel_size(klen, m) // 2, generator=gen, device="cuda").to(torch.bfloat16) for m in (rows, cols))
    acc = torch.empty(layer.block_accumulator_size(view) // 4, device="cuda")
    outs, panels = [], []
    for mask in (None, ones):
        out = torch.full((rows, cols, 128), float("nan"), device="cuda")
        layer.block_accumulate_transposed(view, at, bt, acc, mask, z, out)
        outs.append(out)
        for direction in ("outgoing", "incoming"):
            K, M = (cols, rows) if direction == "outgoing" else (rows, cols)
            a, b = layer.block_project(z, mask, n, row0, col0, direction)
            # past M the panels are not written
            panels.append([T.panel_to_dense(x, M, klen=K) for x in (a, b)])
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])
    for got, ref in zip(panels[:2], panels[2:]):
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
