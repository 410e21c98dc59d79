"""GPU parity of the whole-input batched kernel in every tile it runs in (8, 16, 32 and 64 batch rows): rows of every number of steps it
has code for, rows of any length and alignment, last tiles and groups that are not full, both index widths."""
import numpy as np
import pytest
import torch

import oracle
import synth_inputs as si
from gpu_util import TOL_BF16, TOL_F32, dev, gate, oracle_condensed, oracle_seg
from paper_2305_02299_amd import binding as B_

pytestmark = pytest.mark.gpu
WIDEST = {8: 4096, 16: 2528, 32: 1248, 64: 608}     # columns (whole units) with which 16 result rows still fit the LDS, or that the kernel takes at most
GUARD = 1 << 12


def run_tile(L, tile_rows, rows_per_wave=0, xcd_order=0, narrow=False, x=None, offset=0, act=0):
    W_c, idx, active = oracle_condensed(L)
    xs = dev(L.x_bf16 if L.dtype == "bf16" else L.x) if x is None else dev(x)
    if offset:    # the same rows at an address that is a multiple of the element size only
        flat = torch.zeros((xs.numel() + offset,), dtype=xs.dtype, device="cuda")
        flat[offset:] = xs.flatten()
        xs = flat[offset:].view(xs.shape)
    idx_d = dev(idx)
    if narrow:
        idx16 = torch.empty(idx_d.shape, dtype=torch.int16, device="cuda")
        B_.srigl_narrow_idx(idx_d, L.d_in, idx16)
        idx_d = idx16
    Bn = xs.shape[0]
    flat = torch.full((Bn * L.d_out + 2 * GUARD,), 777.0, dtype=torch.float32, device="cuda")
    y = flat[GUARD:GUARD + Bn * L.d_out].view(Bn, L.d_out)
    B_.srigl_condensed_linear_fwd_tile(xs, Bn, L.d_in, dev(W_c), idx_d, None if len(active) == L.d_out else dev(active), len(active), L.K, dev(L.bias),
                                       L.d_out, y, act=act, tile_rows=tile_rows, rows_per_wave=rows_per_wave, xcd_order=xcd_order)
    torch.cuda.synchronize()
    out = flat.cpu().numpy()
    assert (out[:GUARD] == 777.0).all() and (out[GUARD + Bn * L.d_out:] == 777.0).all(), "write outside y"
    return out[GUARD:GUARD + Bn * L.d_out].reshape(Bn, L.d_out).copy()


def check(L, tile_rows, **kw):
    W_c, idx, active = oracle_condensed(L)
    y_ref, S = oracle.fwd(L.x_bf16 if L.dtype == "bf16" else L.x, W_c, idx, active, L.bias, L.d_out, want_scale=True)
    y = run_tile(L, tile_rows, **kw)
    # sums of at most 600 fp32 terms in 16 or more partial sums: well inside 2e-6 of the summed magnitudes, whatever the storage type
    assert gate(y, y_ref, S, TOL_BF16 if L.dtype == "bf16" else TOL_F32) < 2e-6
    return y


@pytest.mark.parametrize("tile_rows", [8, 16, 32, 64])
@pytest.mark.parametrize("K", [1, 15, 16, 17, 33, 63, 64, 65, 77, 96, 112, 113, 128, 129, 144, 177, 200, 240, 241, 256, 257, 320, 333, 600])
def test_rows_of_every_number_of_steps(tile_rows, K):
    d_in = 605 if K % 2 else 608                    # rows of whole 16-column units, and others
    L = si.make_layer(d_in, 75, K, tile_rows + 3, dtype="bf16" if K % 3 == 0 else "f32", ablate_frac=0.2 if K % 4 else 0.0, seed=300 + K)
    check(L, tile_rows)


@pytest.mark.parametrize("tile_rows", [8, 16, 32, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_widths_alignments_and_index_types(tile_rows, dtype):
    for d_in, B, abl, offset, rows_per_wave in ((16, 1, 0.0, 0, 0), (17, 2, 0.3, 1, 1), (31, tile_rows, 0.0, 3, 2), (33, tile_rows - 1, 0.5, 0, 0),
                                                (100, 2 * tile_rows + 1, 0.0, 1, 3), (255, 5, 0.9, 2, 1), (WIDEST[tile_rows], 40, 0.1, 0, 1),
                                                (WIDEST[tile_rows] - 7, 40, 0.0, 1, 1)):
        L = si.make_layer(d_in, 133, max(1, d_in // 9), B, dtype=dtype, ablate_frac=abl, seed=400 + d_in)
        wide = check(L, tile_rows, rows_per_wave=rows_per_wave, offset=offset, xcd_order=1 + d_in % 2)
        narrow = check(L, tile_rows, rows_per_wave=rows_per_wave, offset=offset, narrow=True)
        assert np.array_equal(wide.view(np.uint32), narrow.view(np.uint32))


@pytest.mark.parametrize("tile_rows", [8, 16, 32, 64])
def test_columns_no_row_names_do_not_matter(tile_rows):
    """NaN and infinities in columns that no stored row reads (padding terms point at an all-zero column of the tile), at the end of rows
    whose length is not a multiple of 16 among them."""
    for d_in, K in ((600, 70), (208, 5)):
        L = si.make_layer(d_in, 60, K, tile_rows + 5, seed=500 + K)
        mask = L.mask.copy()
        keep = np.setdiff1d(np.arange(d_in), [0, 7, 16, d_in - 1])
        rng = np.random.RandomState(3)
        mask[:] = 0
        for r in range(mask.shape[0]):
            mask[r, rng.choice(keep, K, replace=False)] = 1
        L.mask = mask
        L.W = np.where(mask > 0, rng.randn(*mask.shape).astype(np.float32), 0).astype(np.float32)
        clean = run_tile(L, tile_rows)
        x = L.x.copy()
        x[:, 0], x[:, 7], x[:, 16], x[:, d_in - 1] = np.nan, np.inf, -np.inf, np.nan
        assert np.array_equal(run_tile(L, tile_rows, x=x).view(np.uint32), clean.view(np.uint32))
        # a named column carries its non-finite value into exactly the neurons that read it
        c = int(keep[3])
        x = L.x.copy()
        x[2, c] = np.inf
        y = run_tile(L, tile_rows, x=x)
        hit = np.zeros(y.shape, bool)
        hit[2, mask[:, c] > 0] = True
        assert np.array_equal(~np.isfinite(y), hit)


def test_what_does_not_fit_is_refused():
    for tile_rows, d_in in ((8, 4112), (16, 2560), (32, 1280), (64, 640), (16, 15)):
        L = si.make_layer(d_in, 40, 5, 20, seed=600)
        with pytest.raises(B_.SriglError) as e:
            run_tile(L, tile_rows)
        assert e.value.status == B_.ERR_UNSUPPORTED, (tile_rows, d_in)
    L = si.make_layer(256, 40, 5, 20, seed=600)
    for kw in (dict(tile_rows=4), dict(tile_rows=16, rows_per_wave=-1), dict(tile_rows=16, xcd_order=3)):
        with pytest.raises(B_.SriglError):
            run_tile(L, **kw)


@pytest.mark.parametrize("act", [B_.ACT_RELU, B_.ACT_GELU])
def test_activation_in_the_epilogue(act):
    L = si.make_layer(300, 90, 25, 37, ablate_frac=0.3, seed=700)
    plain = run_tile(L, 16).astype(np.float64)
    got = run_tile(L, 16, act=act)
    want = np.maximum(plain, 0) if act == B_.ACT_RELU else torch.nn.functional.gelu(torch.from_numpy(plain)).numpy()
    assert np.abs(got - want).max() <= 2e-6 * max(1.0, np.abs(want).max())    # the activation of the same fp32 sums


@pytest.mark.parametrize("B,n,d_in,ablated,tile", [
    (520, 12001, 136, 57, B_.TILE_256x192), (520, 12001, 72, 57, B_.TILE_256x192), (1500, 5401, 264, 57, B_.TILE_256x192),
    (520, 16121, 520, 0, B_.TILE_256x192),                                     # 256 x 192 tiles: rows, columns and depth end inside a tile
    (520, 16121, 136, 0, B_.TILE_256x256), (1000, 8200, 72, 333, B_.TILE_256x256),
])
def test_structured_library_choice(B, n, d_in, ablated, tile):
    """The shape that only the library's own choice takes, and its neighbour, against float64: two orders of one fp32 sum of d_in products differ by at most
    d_in * 2^-23 of the sum of the magnitudes (bf16 products are exact in fp32)."""
    assert B_.srigl_structured_tile_query(B, d_in, n, n + ablated, B_.BF16) == tile
    g = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randn(B, d_in, device="cuda", generator=g).bfloat16()
    Wd = torch.randn(n, d_in, device="cuda", generator=g).bfloat16()
    d_out = n + ablated
    bias = torch.randn(d_out, device="cuda", generator=g)
    active = torch.sort(torch.randperm(d_out, device="cuda", generator=g)[:n]).values
    flat = torch.full((B * d_out + 2 * GUARD,), 777.0, device="cuda")
    y = flat[GUARD:GUARD + B * d_out].view(B, d_out)
    B_.srigl_structured_linear_fwd(x.view(torch.int16), B, d_in, Wd.view(torch.int16), active.int() if ablated else None, n, bias, d_out, y)
    ref = bias.double().repeat(B, 1)
    ref[:, active] += x.double() @ Wd.double().t()
    bound = bias.abs().repeat(B, 1)
    bound[:, active] += x.float().abs() @ Wd.float().abs().t()
    worst = ((y - ref).abs() / (bound * (d_in + 1) * 2.0 ** -23)).max().item()
    assert worst <= 1, worst
    assert (flat[:GUARD] == 777.0).all() and (flat[GUARD + B * d_out:] == 777.0).all()


@pytest.mark.parametrize("tile", [B_.BLOCKED_64, B_.BLOCKED_128, B_.BLOCKED_192, B_.BLOCKED_256])
@pytest.mark.parametrize("d_in,K", [(8, 3), (72, 20), (136, 70), (776, 60), (4104, 90), (8328, 500)])
def test_blocked_rows_that_end_inside_a_piece(d_in, K, tile):
    """Rows of whole 16-byte pieces that end inside a piece of 64 columns (the rest of it comes from the row's last columns and meets zero
    weights), one to more than 64 iterations, lists of more and of fewer terms than are fetched ahead; the last columns of one row are not
    finite and no neuron reads them."""
    B, d_out = 70, 300
    rng = np.random.default_rng(d_in)
    used = max(K, d_in - 8)
    idx = np.sort(np.argsort(rng.random((d_out, used)), axis=1)[:, :K], axis=1).astype(np.int32)
    Wf, xf = rng.standard_normal((d_out, K)).astype(np.float32), rng.standard_normal((B, d_in)).astype(np.float32)
    W, x = torch.from_numpy(Wf).bfloat16().cuda(), torch.from_numpy(xf).bfloat16().cuda()
    if d_in > 8:
        x[B - 1, -8:] = float("nan")
    idx_d = torch.from_numpy(idx).cuda()
    seg = dev(oracle_seg(idx, d_in))
    blk = torch.empty(B_.srigl_blocked_bytes(d_out, K, d_in), dtype=torch.uint8, device="cuda")
    B_.srigl_block_terms(W, idx_d, seg, d_out, K, d_in, blk)
    y = torch.full((B, d_out), float("nan"), device="cuda")
    B_.srigl_blocked_linear_fwd(x, B, d_in, blk, W, idx_d, None, d_out, K, None, d_out, y, tile=tile)
    xd, Wd = x.double().cpu().numpy(), W.double().cpu().numpy()
    want = np.stack([(Wd[s] * xd[:, idx[s]]).sum(axis=1) for s in range(d_out)], axis=1)
    scale = np.stack([np.abs(Wd[s] * xd[:, idx[s]]).sum(axis=1) for s in range(d_out)], axis=1)
    assert (np.abs(y.cpu().numpy() - want) <= scale * (K + 1) * 2.0 ** -23).all()   # exact products, fp32 sums of K of them


@pytest.mark.parametrize("activation", [B_.ACT_NONE, B_.ACT_RELU])
@pytest.mark.parametrize("d_in,d_out,n,K,B,dtype,narrow,streamed", [
    (1501, 9000, 8201, 290, 1, "f32", False, True), (1200, 8200, 8200, 500, 1, "bf16", True, True), (4096, 16384, 13108, 205, 1, "bf16", True, True),
    (3999, 5440, 5440, 143, 3, "f32", True, True), (3072, 768, 538, 307, 16, "f32", False, True), (700, 400, 255, 256, 63, "bf16", False, True),
    (2200, 3000, 1601, 683, 3, "bf16", False, True), (3700, 5000, 4001, 683, 1, "f32", False, True),       # three chunks, the last one not full
    (4000, 4096, 4090, 768, 1, "bf16", True, True), (3000, 3000, 2303, 1030, 2, "f32", True, True),        # three whole ones; five
    (2200, 3000, 1601, 683, 8, "bf16", False, False),      # (taken by the whole-input batched kernel)
])
def test_streamed_terms_against_the_general_kernel(d_in, d_out, n, K, B, dtype, narrow, streamed, activation):
    """The small-batch kernel for layers whose terms are streamed, at sizes where the library's own choice takes it (asked of the plan query): rows of
    one to five chunks of 256 terms that end inside a lane's four, wavefronts and workgroups with fewer rows than they have room for, both types and
    index widths, ablated neurons in front, between and behind; activations that are not finite in a column no row reads."""
    p = B_.srigl_fwd_plan_query(B, d_in, n, K, d_out, B_.F32 if dtype == "f32" else B_.BF16, has_active=n < d_out, has_seg=False)
    assert (p["algo"] == B_.FWD_KLANE and p["waves"] == 8) == streamed, p
    if streamed:     # (the query above means 32-bit indices)
        assert B_.srigl_fwd_tile_query(B, d_in, n, K, d_out, B_.F32 if dtype == "f32" else B_.BF16, 16 if narrow else 32, n < d_out, False) == (0, 0)
    rng = np.random.default_rng(K)
    active = np.sort(rng.permutation(d_out - (2 if n < d_out else 0))[:n] + (1 if n < d_out else 0)).astype(np.int32)
    idx = np.sort(np.argsort(rng.random((n, d_in - 1)), axis=1)[:, :K], axis=1).astype(np.int32)     # (nobody reads the last column)
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    W, x = torch.from_numpy(rng.standard_normal((n, K)).astype(np.float32)).to(t).cuda(), torch.from_numpy(rng.standard_normal((B, d_in)).astype(np.float32)).to(t).cuda()
    x[:, -1] = float("nan")
    bias, act = torch.from_numpy(rng.standard_normal(d_out).astype(np.float32)).cuda(), dev(active) if n < d_out else None
    ix = torch.from_numpy(idx).cuda()
    got = torch.full((B + 2, d_out), 777.0, device="cuda")
    want = torch.full((B, d_out), 777.0, device="cuda")
    B_.srigl_condensed_linear_fwd(x, B, d_in, W, ix.to(torch.int16) if narrow else ix, act, n, K, bias, d_out, got[1:B + 1], act=activation)
    B_.srigl_condensed_linear_fwd(x, B, d_in, W, ix, act, n, K, bias, d_out, want, act=activation, algo=B_.FWD_GENERIC)
    scale = torch.full((B, d_out), 1.0, device="cuda") + bias.abs()
    rows = torch.from_numpy(active).cuda().long()
    for b in range(B):
        scale[b, rows] += (W.float().abs() * x[b].float().abs()[ix.long()]).sum(1)
    assert ((got[1:B + 1] - want).abs() <= scale * (K + 1) * 2.0 ** -23).all()       # two orders of one fp32 sum of K products
    assert (got[0] == 777.0).all() and (got[B + 1] == 777.0).all()


@pytest.mark.parametrize("n,activation,with_bias", [(1100, B_.ACT_NONE, True), (1101, B_.ACT_RELU, True), (1103, B_.ACT_NONE, False)])
def test_streamed_terms_beside_long_runs_of_ablated_columns(n, activation, with_bias):
    """Neighbours ablated together: runs of 0 to 700 columns in front of each of a wavefront's four rows, around the ends of wavefronts and workgroups,
    and behind the last row; every ablated column is its bias (bits), the others as the general kernel has them."""
    d_in, K, B = 2000, 300, 5
    runs = {0: 700, 1: 15, 2: 16, 3: 17, 4: 80, 6: 81, 9: 272, 31: 33, 32: 273, 33: 1, 500: 64, n - 1: 300}
    active = (np.arange(n) + np.cumsum([runs.get(s, 0) for s in range(n)])).astype(np.int32)
    d_out = int(active[-1]) + 1 + 517
    p = B_.srigl_fwd_plan_query(B, d_in, n, K, d_out, B_.F32, has_active=True, has_seg=False)
    assert p["algo"] == B_.FWD_KLANE and p["waves"] == 8, p
    rng = np.random.default_rng(n)
    idx = dev(np.sort(np.argsort(rng.random((n, d_in)), axis=1)[:, :K], axis=1).astype(np.int32))
    W, x = dev(rng.standard_normal((n, K)).astype(np.float32)), dev(rng.standard_normal((B, d_in)).astype(np.float32))
    bias = dev(rng.standard_normal(d_out).astype(np.float32)) if with_bias else None
    got, want = torch.full((B + 2, d_out), 777.0, device="cuda"), torch.full((B, d_out), 777.0, device="cuda")
    B_.srigl_condensed_linear_fwd(x, B, d_in, W, idx, dev(active), n, K, bias, d_out, got[1:B + 1], act=activation)
    B_.srigl_condensed_linear_fwd(x, B, d_in, W, idx, dev(active), n, K, bias, d_out, want, act=activation, algo=B_.FWD_GENERIC)
    stored = torch.zeros(d_out, dtype=torch.bool, device="cuda")
    stored[dev(active).long()] = True
    assert torch.equal(got[1:B + 1, ~stored], want[:, ~stored])
    scale = torch.zeros((B, d_out), device="cuda") + (bias.abs() if with_bias else 0)
    for b in range(B):
        scale[b, stored] += (W.abs() * x[b].abs()[idx.long()]).sum(1)
    assert ((got[1:B + 1] - want).abs() <= scale * (K + 1) * 2.0 ** -23).all()       # two orders of one fp32 sum of K products
    assert (got[0] == 777.0).all() and (got[B + 1] == 777.0).all()
