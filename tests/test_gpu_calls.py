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
