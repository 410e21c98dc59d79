"""The matrix-core form of the condensed forward call (srigl_block_terms + srigl_blocked_linear_fwd, bf16 storage) against the CPU
oracle, at the edges of its tiles, pieces of 64 columns, lists and output ranges."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from gpu_util import TOL_BF16, dev, gate, host, oracle_condensed, oracle_seg
from paper_2305_02299_amd import binding as B_
from paper_2305_02299_amd import condense_layer

pytestmark = pytest.mark.gpu

TILES = {64: B_.BLOCKED_64, 128: B_.BLOCKED_128, 256: B_.BLOCKED_256, 192: B_.BLOCKED_192}
SHAPES = [   # d_in, d_out, K, B, ablated
    (64, 33, 5, 3, 0.0), (8, 40, 8, 65, 0.0), (65, 1, 4, 1, 0.0), (129, 300, 30, 64, 0.3), (1000, 257, 50, 129, 0.1), (546, 130, 98, 257, 0.0),
    (768, 513, 8, 70, 0.98), (4160, 70, 300, 66, 0.2), (200, 96, 200, 33, 0.5), (9000, 64, 40, 40, 0.0), (1024, 1500, 11, 20, 0.995)]


def blocked(W_c, idx, seg, d_in):
    out = torch.full((B_.srigl_blocked_bytes(W_c.shape[0], W_c.shape[1], d_in),), 255, dtype=torch.uint8, device="cuda")
    B_.srigl_block_terms(W_c, idx, seg, W_c.shape[0], W_c.shape[1], d_in, out)
    return out


@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("bits", [32, 16])
@pytest.mark.parametrize("d_in,d_out,K,B,abl", SHAPES)
def test_blocked_forward(d_in, d_out, K, B, abl, bits, tile):
    L = si.make_layer(d_in, d_out, K, B, ablate_frac=abl, dtype="bf16", seed=d_in + B, idx_dist="clustered" if d_in > 512 else "uniform")
    W_c, idx, active = oracle_condensed(L)
    n = len(active)
    y_ref, S = oracle.fwd(L.x_bf16, W_c, idx, active, L.bias, d_out, want_scale=True)
    ix = dev(idx if bits == 32 else idx.astype(np.uint16))
    Wd, act = dev(W_c), dev(active) if n < d_out else None
    blk = blocked(Wd, ix, dev(oracle_seg(idx, d_in)), d_in)
    y = torch.full((B, d_out), float("nan"), device="cuda")
    B_.srigl_blocked_linear_fwd(dev(L.x_bf16), B, d_in, blk, Wd, ix, act, n, K, dev(L.bias), d_out, y, tile=TILES[tile])
    yh = host(y)
    gate(yh, y_ref, S, 2e-6)   # exact products, fp32 sums
    ablated = np.setdiff1d(np.arange(d_out), active)
    assert np.array_equal(yh[:, ablated].view(np.uint32), np.tile(L.bias[ablated], (B, 1)).view(np.uint32))


@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("d_in", [768, 770])
def test_non_finite_activations_reach_only_the_neurons_that_name_them(tile, d_in):
    L = si.make_layer(d_in, 300, 20, 70, ablate_frac=0.1, dtype="bf16", seed=5)
    W_c, idx, active = oracle_condensed(L)
    n, cols = len(active), np.array([0, 100, d_in - 1])
    x = L.x_bf16.copy()
    x[3, cols], x[69, cols] = 0x7f80, 0x7fc0   # +inf, NaN
    ix, Wd = dev(idx), dev(W_c)
    y = torch.full((70, 300), float("nan"), device="cuda")
    B_.srigl_blocked_linear_fwd(dev(x), 70, d_in, blocked(Wd, ix, dev(oracle_seg(idx, d_in)), d_in), Wd, ix, dev(active), n, 20, None, 300, y,
                                tile=TILES[tile])
    yh = host(y)[:, active]
    named = np.isin(idx, cols).any(axis=1)
    y_ref, S = oracle.fwd(L.x_bf16, W_c, idx, active, None, 300, want_scale=True)
    assert named.any() and not np.isfinite(yh[[3, 69]][:, named]).any()
    clean = np.ones((70, n), bool)
    clean[3, named] = clean[69, named] = False
    gate(np.where(clean, yh, 0), np.where(clean, y_ref[:, active], 0), S[:, active], TOL_BF16)


def test_layer_object_keeps_the_copy_and_renews_it():
    """The layer's own call takes the matrix cores where the library expects them faster, in eager calls and in captured ones, and
    follows weights that are written in place."""
    d_in, d_out, K, B = 512, 2048, 100, 1024
    assert B_.srigl_blocked_tile(B, d_in, d_out, K, d_out) != 0 and B_.srigl_blocked_tile(1, d_in, d_out, K, d_out) == 0
    L = si.make_layer(d_in, d_out, K, B, dtype="bf16", seed=9)
    W_c, idx, active = oracle_condensed(L)
    y_ref, S = oracle.fwd(L.x_bf16, W_c, idx, active, L.bias, d_out, want_scale=True)
    layer = condense_layer(dev(L.W_bf16).view(torch.bfloat16), dev(L.mask), K, dev(L.bias))
    x = dev(L.x_bf16).view(torch.bfloat16)
    y = torch.empty((B, d_out), device="cuda")
    layer.forward(x[:1])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):      # no copy yet: the captured call takes a form that needs none
        layer.forward(x, y)
    assert layer._blocked is None
    gate(host(layer.forward(x)), y_ref, S, TOL_BF16)
    kept = layer._blocked
    assert kept is not None
    with torch.cuda.graph(graph2 := torch.cuda.CUDAGraph()):
        layer.forward(x, y)
    for g in (graph, graph2, graph, graph2):
        y.fill_(float("nan"))
        g.replay()
        gate(host(y), y_ref, S, TOL_BF16)
        assert layer._blocked is kept and torch.isfinite(layer.narrow().forward(x)).all()
    layer.W_c.mul_(2)
    gate(host(layer.forward(x)), (y_ref - L.bias) * 2 + L.bias, 2 * S, TOL_BF16)
    assert layer._blocked is not kept


@pytest.mark.parametrize("first,second,columns", [(B_.BLOCKED_256, B_.BLOCKED_192, 2), (B_.BLOCKED_192, B_.BLOCKED_64, 3), (B_.BLOCKED_64, B_.BLOCKED_256, 1),
                                                  (B_.BLOCKED_128, B_.BLOCKED_128, 4)])
@pytest.mark.parametrize("abl", [0.0, 0.3])
def test_split_rows(first, second, columns, abl):
    """Stored rows in two launches of different tile shapes: every column written once, ablated ones at the seam included."""
    d_in, d_out, K, B = 200, 900, 30, 300
    L = si.make_layer(d_in, d_out, K, B, ablate_frac=abl, dtype="bf16", seed=columns)
    W_c, idx, active = oracle_condensed(L)
    n = len(active)
    y_ref, S = oracle.fwd(L.x_bf16, W_c, idx, active, L.bias, d_out, want_scale=True)
    Wd, ix, act = dev(W_c), dev(idx), dev(active) if n < d_out else None
    blk = blocked(Wd, ix, dev(oracle_seg(idx, d_in)), d_in)
    y = torch.full((B, d_out), float("nan"), device="cuda")
    args = (dev(L.x_bf16), B, d_in, blk, Wd, ix, act, n, K, dev(L.bias), d_out, y)
    B_.srigl_blocked_linear_fwd(*args, tile=first | second << 4 | columns << 8)
    yh = host(y)
    gate(yh, y_ref, S, TOL_BF16)
    gone = np.setdiff1d(np.arange(d_out), active)
    assert np.array_equal(yh[:, gone].view(np.uint32), np.tile(L.bias[gone], (B, 1)).view(np.uint32))
    for bad in (first | second << 4, first | second << 4 | 100 << 8, first | columns << 8, 5):
        with pytest.raises(B_.SriglError):
            B_.srigl_blocked_linear_fwd(*args, tile=bad)
