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
