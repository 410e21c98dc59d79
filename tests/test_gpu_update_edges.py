"""Connectivity update against the oracle at the edges of its row kernels (one wavefront per row up to 1024 columns, four beyond) and
of the per-neuron counts that come with the layer-wide passes (rows shorter and longer than a wavefront's 256 elements, rows that
share four elements, lists that do not fit).  Everything must match exactly."""
import numpy as np
import pytest

import synth_inputs as si
from paper_2305_02299_amd import binding as B_
from test_gpu_update import check

pytestmark = pytest.mark.gpu


def layer(d_in, d_out, k, seed, ablated=0.25):
    L = si.make_layer(d_in, d_out, k, 1, ablate_frac=ablated, seed=seed)
    return np.where(L.mask != 0, L.W, 0).astype(np.float32), L.mask, np.random.default_rng(seed).normal(size=L.W.shape).astype(np.float32)


@pytest.mark.parametrize("d_in", [1, 2, 3, 4, 5, 63, 64, 65, 66, 67, 255, 257, 768, 1024, 1025, 1028, 2048, 2049, 3073, 4097, 6145, 8192])
@pytest.mark.parametrize("gamma", [0, 60, 95])
def test_row_lengths(d_in, gamma):
    d_out = 5 if d_in >= 1024 else 131
    k = max(1, d_in // 9)
    W, mask, g = layer(d_in, d_out, k, d_in)
    kept = int(mask.sum())
    g *= np.linspace(0.1, 1.0, d_out, dtype=np.float32)[:, None]   # rows differ in what is salient: some go at 60 and 95 %
    check(B_, W, mask, g, k, int(0.3 * kept), gamma)
    check(B_, np.sign(W), mask, np.ones_like(g), k, int(0.3 * kept), gamma)   # positions alone decide


@pytest.mark.parametrize("K_upd", [0, 1, 300, 10**6])
@pytest.mark.parametrize("levels", [1, 3, 40])
def test_finished_thresholds_count_the_same_neurons(K_upd, levels):
    """Few distinct magnitudes: thresholds that are final after the first digit, inside the list, or over a list that does not fit."""
    W, mask, g = layer(300, 400, 30, levels, 0.1)
    q = np.float32(1.0 / levels)
    W = np.where(mask != 0, np.sign(W) * (np.floor(np.abs(W) * 7 / q) % levels + 1) * q, 0).astype(np.float32)
    g = (np.floor(np.abs(g) / q) % levels + 1).astype(np.float32) * q
    check(B_, W, mask, g, 30, K_upd, 50)


def few_magnitudes(kind, rng, shape):
    """Contents whose threshold's first digit (exponent and four mantissa bits) is shared by more keys than a list holds."""
    ulps = {"one": 1, "last bits": 100, "second digit": 40000}.get(kind)
    if ulps is not None:    # 1.0 and the numbers behind it: apart in the last 7 bits of the magnitude, or in the 12 above them too
        mag = (np.uint32(0x3f800000) + rng.integers(0, ulps, shape).astype(np.uint32)).view(np.float32)
    elif kind == "zero":
        mag = np.zeros(shape, np.float32)
    else:                   # "mostly one": a few elements are smaller or larger
        mag = np.where(rng.random(shape) < 0.05, rng.random(shape) * 2, 1.0).astype(np.float32)
    return np.where(rng.random(shape) < 0.5, -mag, mag)


@pytest.mark.parametrize("shape", [(65, 64), (41, 100), (300, 401), (2049, 255), (777, 1000)])   # 4160, 4100: two parts of the layer
@pytest.mark.parametrize("kinds", [("one", "zero"), ("one", "one"), ("last bits", "real"), ("real", "last bits"), ("second digit", "second digit"),
                                   ("mostly one", "mostly one"), ("zero", "mostly one")])
def test_selections_without_a_list(shape, kinds):
    d_out, d_in = shape
    rng = np.random.default_rng(d_out)
    k = d_in // 2     # (as many kept weights as free positions: both sides exceed the list)
    L = si.make_layer(d_in, d_out, k, 1, ablate_frac=0.1, seed=d_in)
    W, g = (rng.normal(size=shape).astype(np.float32) if kind == "real" else few_magnitudes(kind, rng, shape) for kind in kinds)
    W = np.where(L.mask != 0, W, 0).astype(np.float32)
    kept = int(L.mask.sum())
    for K_upd in (1, kept // 3, kept - 1, kept):
        for gamma in (0, 60, 95):     # (none, some and most neurons ablated: step 6 ranks what remains)
            check(B_, W, L.mask, g, k, K_upd, gamma)


def test_selections_without_a_list_on_a_layer_of_256_parts():
    d_out, d_in, k = 4097, 4096, 410
    rng = np.random.default_rng(1)
    mask = np.zeros((d_out, d_in), np.uint8)
    for r in range(d_out):
        mask[r, rng.choice(d_in, k, replace=False)] = 1
    W = np.where(mask != 0, few_magnitudes("mostly one", rng, mask.shape), 0).astype(np.float32)
    info = check(B_, W, mask, np.zeros_like(W), k, d_out * k // 2, 50)
    assert info["n_ablated_now"] > 0


@pytest.mark.parametrize("d_out,d_in", [(8191, 1024), (8193, 1024), (32800, 256), (16400, 512), (10930, 768), (4100, 2048), (2735, 3072), (2049, 4097), (1030, 8192)])
def test_rows_that_do_not_stay_on_either_side_of_8_m_elements(d_out, d_in):
    """Up to 2^23 elements the last launch requests a row beside the flag that says whether it stays, beyond behind it (every number of columns a lane holds)."""
    k = d_in // 20
    W, mask, g = layer(d_in, d_out, k, d_out, 0.2)
    g *= np.linspace(0.1, 1.0, d_out, dtype=np.float32)[:, None]
    check(B_, W, mask, g, k, int(0.3 * mask.sum()), 60)
