"""What the calls accept and refuse on their way into the library (the binding's functions and the layer objects)."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from gpu_util import dev, oracle_condensed
from paper_2305_02299_amd import binding as B_

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("packed", [False, True])
@pytest.mark.parametrize("bits", [32, 16])
def test_negative_sizes_are_refused(bits, packed):
    L = si.make_layer(64, 12, 5, 3, seed=45)
    W_c, idx, _ = oracle_condensed(L)
    x, W, ix = dev(L.x), dev(W_c), dev(idx if bits == 32 else idx.astype(np.uint16))
    y = torch.full((3, 12), 7.0, device="cuda")
    for B, d_in, n, K, d_out in ((-1, 64, 12, 5, 12), (-2**31, 64, 12, 5, 12), (3, -64, 12, 5, 12), (3, 64, -1, 5, 12), (3, 64, 12, -5, 12), (3, 64, 12, 5, -12)):
        with pytest.raises(B_.SriglError) as e:
            B_.srigl_condensed_linear_fwd(x, B, d_in, W, ix, None, n, K, None, d_out, y, packed=torch.zeros(1024, dtype=torch.uint8, device="cuda") if packed and bits == 32 else None)
        assert e.value.status == B_.ERR_INVALID_ARG
    assert (y == 7.0).all()


@pytest.mark.parametrize("given", ["hidden", "both", "none"])
def test_block_runs_the_rows_of_its_input(given):
    """Both layers of a block run on as many rows as x has: buffers of a larger batch are filled as far as x goes, and x may have any shape of that many rows."""
    from paper_2305_02299_amd import condense_layer, fold_mlp
    L1, L2 = si.make_layer(96, 200, 10, 8, ablate_frac=0.3, seed=1), si.make_layer(200, 96, 20, 8, seed=2)
    block = fold_mlp(condense_layer(dev(L1.W), dev(L1.mask), 10, dev(L1.bias)), condense_layer(dev(L2.W), dev(L2.mask), 20, dev(L2.bias)), B_.ACT_GELU)
    x = dev(L1.x)
    want = block.forward(x)
    hidden = torch.full((8, block.first.d_out), 5.0, device="cuda") if given != "none" else None
    room = torch.full((8, 96), 7.0, device="cuda")
    y = block.forward(x[:3].reshape(3, 1, 96), room if given == "both" else None, hidden)
    if given == "both":
        assert y is room and (room[3:] == 7.0).all()
    else:
        assert y.shape == (3, 96)
    np.testing.assert_allclose(y[:3].cpu(), want[:3].cpu(), rtol=0, atol=1e-5)
    assert hidden is None or (hidden[3:] == 5.0).all()


def test_sizes_in_any_form_that_int_takes():
    L = si.make_layer(64, 12, 5, 3, seed=45)
    W_c, idx, _ = oracle_condensed(L)
    x, W, ix = dev(L.x), dev(W_c), dev(idx)
    want, y = torch.empty((3, 12), device="cuda"), torch.empty((3, 12), device="cuda")
    B_.srigl_condensed_linear_fwd(x, 3, 64, W, ix, None, 12, 5, None, 12, want)
    for form in (float, np.int64, np.float32, torch.tensor):
        B_.srigl_condensed_linear_fwd(x, form(3), form(64), W, ix, None, form(12), form(5), None, form(12), y.fill_(0))
        assert torch.equal(y, want)
    for wrong in (None, "many", [3]):
        with pytest.raises((TypeError, ValueError)):
            B_.srigl_condensed_linear_fwd(x, 3, 64, W, ix, None, 12, wrong, None, 12, y)
    Wm, mask, g = dev(np.where(L.mask != 0, L.W, 0).astype(np.float32)), dev(L.mask), dev(L.W)
    ws = torch.empty(B_.srigl_mask_update_workspace_bytes(12, 64), dtype=torch.uint8, device="cuda")
    outs = []
    for form in (int, float, np.int32):
        mo, Wo, rep = torch.empty_like(mask), torch.empty_like(Wm), torch.empty(4, dtype=torch.int64, device="cuda")
        B_.srigl_mask_update(Wm, mask, g, form(12), form(64), form(5), form(0.3 * 60), form(30), form(60), mo, Wo, ws, rep)
        outs.append((mo, Wo, rep))
    for other in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(outs[0], other))


def test_condensing_refuses_a_captured_stream():
    """The call waits for its report: under capture it says so, before it has put anything into the graph."""
    from paper_2305_02299_amd import condense_layer
    L = si.make_layer(64, 12, 5, 3, seed=45)
    W, mask = dev(L.W), dev(L.mask)
    y = torch.zeros(4, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        y.add_(1)
        with pytest.raises(RuntimeError, match="captured"):
            condense_layer(W, mask, 5)
    for _ in range(3):
        graph.replay()
    torch.cuda.synchronize()
    assert (y == 3).all() and condense_layer(W, mask, 5).n_active == 12
