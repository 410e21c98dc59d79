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


D_IN, D_OUT, K_, B_ROWS = 512, 2048, 100, 1024   # the layer's own call takes the matrix cores here


def bf16_layer(seed):
    """A synthetic layer, its arrays as the layer object takes them, and the oracle's result and scale."""
    L = si.make_layer(D_IN, D_OUT, K_, B_ROWS, dtype="bf16", seed=seed)
    W_c, idx, active = oracle_condensed(L)
    return L, dev(L.W_bf16).view(torch.bfloat16), dev(L.mask), *oracle.fwd(L.x_bf16, W_c, idx, active, L.bias, D_OUT, want_scale=True)


def test_layer_call_takes_the_matrix_cores_and_reads_what_the_arrays_hold():
    """Every way of changing a layer in place shows in the next call: writes through torch, condensing again into the same buffers (raw
    pointers, no version counter), inference tensors (which have none)."""
    assert B_.srigl_blocked_tile_with_copy(B_ROWS, D_IN, D_OUT, K_, D_OUT) != 0 and B_.srigl_blocked_tile_with_copy(1, D_IN, D_OUT, K_, D_OUT) == 0
    L, W, mask, y_ref, S = bf16_layer(9)
    layer = condense_layer(W, mask, K_, dev(L.bias))
    x = dev(L.x_bf16).view(torch.bfloat16)
    first = layer.forward(x)
    gate(host(first), y_ref, S, 2e-6)
    assert torch.equal(layer.forward(x), first) and torch.equal(layer.narrow().forward(x), first)
    forced = torch.empty_like(first)     # the same form with a copy made by hand
    B_.srigl_blocked_linear_fwd(x, B_ROWS, D_IN, blocked(layer.W_c, layer.idx, layer.seg, D_IN), layer.W_c, layer.idx, None, D_OUT, K_, layer.bias, D_OUT, forced)
    assert torch.equal(forced, first)
    layer.W_c.mul_(2)
    gate(host(layer.forward(x)), (y_ref - L.bias) * 2 + L.bias, 2 * S, 2e-6)
    L2, W2, mask2, y2_ref, S2 = bf16_layer(10)
    y2_ref, S2 = oracle.fwd(L.x_bf16, *oracle_condensed(L2), L.bias, D_OUT, want_scale=True)
    B_.srigl_condense(W2, mask2, D_OUT, D_IN, K_, D_OUT, layer.W_c, layer.idx, torch.empty(D_OUT, dtype=torch.int32, device="cuda"), layer.seg,
                      B_.new_workspace(D_OUT), B_.new_report(), packed=layer.packed)
    gate(host(layer.forward(x)), y2_ref, S2, 2e-6)
    with torch.inference_mode():
        inferred = condense_layer(W.clone(), mask, K_, dev(L.bias))
        assert inferred.W_c.is_inference()
        gate(host(inferred.forward(x)), y_ref, S, 2e-6)
        inferred.W_c.mul_(2)
        gate(host(inferred.forward(x)), (y_ref - L.bias) * 2 + L.bias, 2 * S, 2e-6)


@pytest.mark.parametrize("prepared", [False, True])
def test_captured_layer_calls(prepared):
    """A call captured before any other runs the same kernels as the eager one; replays follow weights that are written in place, with eager calls
    and other allocations between them."""
    L, W, mask, y_ref, S = bf16_layer(9)
    layer = condense_layer(W, mask, K_, dev(L.bias))
    if prepared:
        at = layer.prepare().blocked.data_ptr()
    x = dev(L.x_bf16).view(torch.bfloat16)
    y = torch.empty((B_ROWS, D_OUT), device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        layer.forward(x, y)
    eager = layer.forward(x)
    gate(host(eager), y_ref, S, 2e-6)
    for turn in range(6):
        if turn == 3:
            layer.W_c.mul_(2)
            y_ref, S = (y_ref - L.bias) * 2 + L.bias, 2 * S
            if prepared:
                assert layer.prepare().blocked.data_ptr() == at
        y.fill_(float("nan"))
        junk = [torch.full((4 << 20,), -1, dtype=torch.int32, device="cuda") for _ in range(3)]
        graph.replay()
        torch.cuda.synchronize()
        del junk
        gate(host(y), y_ref, S, 2e-6)
        assert torch.equal(layer.forward(x), y)
        torch.cuda.synchronize()


@pytest.mark.parametrize("prepared", [False, True])
def test_first_calls_from_several_threads_and_streams(prepared):
    import threading
    L, W, mask, y_ref, S = bf16_layer(9)
    layer = condense_layer(W, mask, K_, dev(L.bias))
    if prepared:
        layer.prepare()
    x = dev(L.x_bf16).view(torch.bfloat16)
    torch.cuda.synchronize()
    results, start = [None] * 4, threading.Barrier(4)

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            start.wait()
            results[i] = [layer.forward(x) for _ in range(8)]
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    gate(host(results[0][0]), y_ref, S, 2e-6)
    assert all(torch.equal(y, results[0][0]) for r in results for y in r)


def test_prepare_is_what_the_call_reads_and_other_layers_need_none():
    L, W, mask, y_ref, S = bf16_layer(9)
    layer = condense_layer(W, mask, K_, dev(L.bias))
    x = dev(L.x_bf16).view(torch.bfloat16)
    want = layer.forward(x)
    assert torch.equal(layer.prepare().forward(x), want) and layer.narrow().blocked is layer.blocked
    assert layer.blocked.numel() == B_.srigl_blocked_bytes(D_OUT, K_, D_IN)
    layer.blocked = layer.blocked[:-16].clone()
    with pytest.raises(ValueError):
        layer.forward(x)
    assert torch.equal(layer.prepare().forward(x), want) and layer.blocked.numel() == B_.srigl_blocked_bytes(D_OUT, K_, D_IN)
    plain = condense_layer(dev(L.W), mask, K_)      # fp32
    assert plain.prepare().blocked is None and condense_layer(W, mask, K_, want_seg=False).prepare().blocked is None


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


@pytest.mark.parametrize("tile", list(TILES))
@pytest.mark.parametrize("d_in,d_out,K,B,abl", [(768, 300, 20, 300, 0.1), (770, 70, 300, 70, 0.0), (9001, 200, 130, 40, 0.2), (64, 700, 5, 9, 0.0)])
def test_rows_with_sums_that_are_not_finite(d_in, d_out, K, B, abl, tile):
    """Infinities of either sign, NaN, stored zeros and infinite weights, from one row to all of them: every sum is what its own terms give in
    64 bits (the same infinity or a NaN, or the finite sum), others untouched; also behind an activation."""
    L = si.make_layer(d_in, d_out, K, B, ablate_frac=abl, dtype="bf16", seed=d_in + 1)
    W_c, idx, active = oracle_condensed(L)
    n = len(active)
    rng = np.random.default_rng(K)
    W_c = W_c.copy()
    W_c[rng.integers(0, n, 6), rng.integers(0, K, 6)] = [0, 0x8000, 0, 0x7f80, 0xff80, 0x7fc0]
    W_c[-1, :] = 0
    ix, Wd, act = dev(idx.astype(np.uint16)) if d_in == 768 else dev(idx), dev(W_c), dev(active) if n < d_out else None
    blk = blocked(Wd, ix, dev(oracle_seg(idx, d_in)), d_in)
    wide = lambda bits: (bits.astype(np.uint32) << 16).view(np.float32).astype(np.float64)   # noqa: E731
    w64 = wide(W_c)
    for name in ("one", "nine rows", "a column", "every value", "none"):
        x = L.x_bf16.copy()
        bad = np.array([0x7f80, 0xff80, 0x7fc0, 0x7f80], np.uint16)
        if name == "one":
            x[B - 1, d_in // 2] = 0x7f80
        elif name == "nine rows":
            for r in range(0, min(B, 9)):
                x[r * (B // 9), rng.integers(0, d_in, 4)] = bad
        elif name == "a column":
            x[:, idx[0, 0]] = 0x7f80
        elif name == "every value":
            x[:] = np.where(rng.random(x.shape) < 0.01, 0x7fc0, 0x7f80)
        x64 = wide(x)
        with np.errstate(all="ignore"):
            want = np.stack([(w64[s] * x64[:, idx[s]]).sum(axis=1) for s in range(n)], axis=1) + L.bias[active].astype(np.float64)
            scale = np.stack([np.abs(np.where(np.isfinite(w64[s] * x64[:, idx[s]]), w64[s] * x64[:, idx[s]], 0)).sum(axis=1) for s in range(n)], axis=1) + 1
        for fn in (B_.ACT_NONE, B_.ACT_RELU):
            y = torch.full((B, d_out), 5.0, device="cuda")
            B_.srigl_blocked_linear_fwd(dev(x), B, d_in, blk, Wd, ix, act, n, K, dev(L.bias), d_out, y, act=fn, tile=TILES[tile])
            yh = host(y).astype(np.float64)
            ref = want if fn == B_.ACT_NONE else np.fmax(want, 0)   # (the activation of a NaN is 0)
            got = yh[:, active]
            assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref)), (name, fn)
            assert (np.sign(got[np.isinf(ref)]) == np.sign(ref[np.isinf(ref)])).all()
            ok = np.isfinite(ref)
            assert (np.abs(got[ok] - ref[ok]) <= 2e-6 * scale[ok]).all()   # exact products, fp32 sums of at most 300
            gone = np.setdiff1d(np.arange(d_out), active)
            flat = L.bias[gone] if fn == B_.ACT_NONE else np.maximum(L.bias[gone], 0)
            assert np.array_equal(host(y)[:, gone], np.tile(flat, (B, 1)))


def test_layer_call_without_memory_for_the_copy():
    """The layer's call needs 4 bytes per stored weight for itself where it takes the matrix cores; with no memory to be had it takes the kernel that
    needs none."""
    d_in, d_out, K, B = 1024, 8192, 200, 512
    assert B_.srigl_blocked_tile_with_copy(B, d_in, d_out, K, d_out) != 0
    L = si.make_layer(d_in, d_out, K, 8, dtype="bf16", seed=3)
    layer = condense_layer(dev(L.W_bf16).view(torch.bfloat16), dev(L.mask), K, dev(L.bias))
    x = dev(L.x_bf16).view(torch.bfloat16).repeat(B // 8, 1)
    y, want = torch.empty((B, d_out), device="cuda"), layer.forward(x)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    eaten = []
    try:
        torch.cuda.set_per_process_memory_fraction(torch.cuda.memory_reserved() / total)
        for size in (8 << 20, 1 << 20, 1 << 18):
            while True:
                try:
                    eaten.append(torch.empty((size,), dtype=torch.uint8, device="cuda"))
                except torch.cuda.OutOfMemoryError:
                    break
        with pytest.raises(torch.cuda.OutOfMemoryError):
            torch.empty((B_.srigl_blocked_bytes(d_out, K, d_in),), dtype=torch.uint8, device="cuda")
        layer.forward(x, y)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
        del eaten
    y_ref, S = oracle.fwd(L.x_bf16, *oracle_condensed(L), L.bias, d_out, want_scale=True)
    gate(host(y[:8]), y_ref, S, TOL_BF16)
    gate(host(y), host(want), np.tile(S, (B // 8, 1)), 4e-6)
