"""Workspace of the layer backward: no size needs more than the layout in
which the epilogue's weight operands travelled as unit blocks did, and a call
with exactly the reported bytes writes nothing past them."""
import pytest
import torch

from paper_2603_14806_amd import synth
from paper_2603_14806_amd import trimul as T
from tests.gpu_util import make_layer, needs_gpu, say

pytestmark = [pytest.mark.gpu, needs_gpu]


def unit_block_layout_bytes(N, cus):
    """Three panels, three results, dx_g, nine unit blocks, the LayerNorm
    partials of one work-group per compute unit, the partials of one weight
    from two per compute unit and those of four weights from one."""
    def up(x):
        return -(-x // 256) * 256
    J = -(-N // 32)
    units = N * J
    one, two = min(units, cus), min(units, 2 * cus)
    return (3 * up(128 * -(-N // 256) * J * 256 * 32 * 2) + 3 * up(N * J * 32 * 128 * 4) + up(N * N * 128 * 4) +
            9 * up(units * 128 * 32 * 2) + 2 * up(one * 2 * 128 * 4) + up(two * 128 * 128 * 4) + up(4 * one * 128 * 128 * 4))


def test_no_size_needs_more_than_the_unit_block_layout():
    say("backward workspace sizes")
    layer, _ = make_layer("bf16")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for N in list(range(1, 400)) + [512, 1024, 1300, 2048, 4096]:
        assert T.tri_mul_backward_workspace_size(layer.h, N) <= unit_block_layout_bytes(N, cus), N


@pytest.mark.parametrize("saved", [False, True])
@pytest.mark.parametrize("N", [1, 33, 257])   # the four weights' partials outgrow dA, dB and dx_g up to N = 201, not at 257
def test_exact_workspace_is_enough(N, saved):
    say(f"backward with its exact workspace N={N} saved={saved}")
    layer, _ = make_layer("bf16", affine=True)
    z = synth.pair_tensor(N, dtype="bf16", device="cuda")
    dout = synth.pair_tensor(N, dtype="f32", device="cuda", name="dout")
    mask = synth.token_mask(N, N // 10, device="cuda")
    need = T.tri_mul_backward_workspace_size(layer.h, N)
    guard = 1 << 20
    ws = torch.full((need + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    dz = torch.empty_like(z)
    grads = {k: torch.empty(s, dtype=torch.float32, device="cuda") for k, s in T.WEIGHT_SHAPES.items()}
    if saved:
        A, B = layer.project(z, mask, "incoming")
        state = (A, B, layer.contract_transposed(A, B, N))
        T.tri_mul_layer_backward_saved(layer.h, "outgoing", z, mask, N, *state, dout, dz, grads, ws, need)
    else:
        T.tri_mul_layer_backward(layer.h, "outgoing", z, mask, N, dout, dz, grads, ws, need)
    ref_dz, ref = layer.backward(z, dout, mask, "outgoing")
    torch.cuda.synchronize()
    assert (ws[need:] == 0xA5).all()
    assert torch.equal(dz, ref_dz)
    for k in ref:
        assert torch.equal(grads[k], ref[k]), k
        assert torch.isfinite(ref[k]).all(), k
    with pytest.raises(T.TriMulError) as e:   # one byte less is refused on the host
        T.tri_mul_layer_backward(layer.h, "outgoing", z, mask, N, dout, dz, grads, ws, need - 1)
    assert e.value.code == T.TRI_MUL_ENOMEM
