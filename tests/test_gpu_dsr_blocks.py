"""gs_dsr at the edges of its split into blocks, against the oracle: one scale
short of and past a chunk of 2048 scales, several chunks, a last chunk of a
few scales, and more chunks than the 1024 blocks (two chunks a block, some
with none left to prefetch).

The oracle's exponentials are the same bits, so the sets and their counts are
equal; sums of m < 4.3e6 doubles in any order differ by at most m 2^-53 <
5e-10 relative, and typically by sqrt(m) 2^-53 < 3e-13: 1e-10, the existing
parity bound.  The gradient is one float32 rounding of the sum: 1e-6 of its
largest value.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_27781_amd import raster

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 682, 683, 1366, 20_000, 699_050, 699_052, 1_400_001])
@pytest.mark.parametrize("spread", [0.0, 0.4])
def test_dsr_blocks(n, spread):
    rng = np.random.default_rng(n)
    ls = (-4.5 + spread * rng.standard_normal((3, n))).astype(np.float32)
    if n > 100:
        k = n // 200
        ls[0, :k] = -1.0
        ls[2, -k:] = -9.0
    ref, gref = oracle.dsr(ls, float(np.float32(0.01)), float(np.float32(0.001)))
    grad = torch.zeros(3, n, device="cuda")
    out = raster.dsr(torch.from_numpy(ls).cuda(), 0.01, 0.001, grad).cpu().numpy()
    assert out[5] == ref["n_big"] and out[6] == ref["n_small"]
    for i, name in enumerate(("L_big", "L_small", "loss", "mu", "sigma")):
        assert out[i] == pytest.approx(ref[name], rel=1e-10, abs=1e-14), name
    assert np.max(np.abs(grad.cpu().numpy() - gref)) <= 1e-6 * max(np.max(np.abs(gref)), 1e-12)
    again = raster.dsr(torch.from_numpy(ls).cuda(), 0.01, 0.001).cpu().numpy()
    assert np.array_equal(out, again)
