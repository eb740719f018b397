"""The BH hash with a token group's coordinates spread over one, two or four waves: codes bit-equal to the oracle
and weights within its tolerance at the edges of the split (one token, a full group of 16, one more; rows that end
inside a tile, a unit of 64 coordinates or a wave's 256; rows of which a whole wave is padding; rows read one
coordinate at a time; tables that cross units and projections)."""
import numpy as np
import pytest

import oracle
from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu

# tau <= 16 fp32 factors and terms, each a few ulp: 16 * 4 * 2^-24 = 4e-6 relative; the library's own bar is 1e-5
TOL_W = 1e-5

CASES = [
    # n, d, k, tau, block, m, x dtype
    (1, 64, 8, 8, 64, 1, "f32"), (17, 100, 9, 7, 16, 2, "f16"), (65, 128, 40, 4, 32, 4, "f32"),      # one wave
    (16, 200, 32, 8, 64, 4, "bf16"), (33, 255, 60, 5, 16, 3, "f32"), (15, 256, 37, 13, 32, 4, "f32"),
    (17, 260, 64, 8, 64, 4, "f32"), (1, 384, 70, 9, 32, 1, "bf16"), (47, 511, 33, 16, 16, 2, "f16"),  # two waves
    (31, 512, 130, 8, 64, 4, "f32"), (16, 509, 57, 9, 64, 5, "bf16"),
    (1, 513, 96, 8, 64, 4, "f32"), (17, 640, 113, 9, 16, 2, "f16"), (15, 766, 170, 9, 64, 4, "f32"),  # four waves
    (48, 768, 96, 8, 16, 1, "bf16"), (33, 769, 256, 4, 32, 3, "f32"), (16, 1023, 64, 16, 64, 4, "bf16"),
    (129, 1024, 171, 12, 32, 4, "f32"),
]


@pytest.mark.parametrize("n,d,k,tau,b,m,xdt", CASES)
def test_bh_split_over_waves(n, d, k, tau, b, m, xdt):
    print(f"bh split n={n} d={d} k={k} tau={tau} block={b} m={m} {xdt}", flush=True)
    w = synth.Workload("t", 7, n, d, m, k, tau, 8, x_dtype=xdt)
    bm = synth.make_bmats(31 * d + b, w.n_proj, m, w.d_pad, b)
    x = synth.make_x(7 * n + d, n, d, xdt)
    want = oracle.bh_hash_codes(x, bm, k, tau)
    xd, bd = B.to_device(x), torch.from_numpy(bm).cuda()
    assert np.array_equal(B.codes_to_numpy(B.lookupffn_hash_bh(xd, bd, k, tau)), want)
    codes, wts = B.lookupffn_hash_bh_weighted(xd, bd, k, tau)
    assert np.array_equal(B.codes_to_numpy(codes), want)
    ref = oracle.weights_from_z(oracle.bh_soft_codes(x, bm, k, tau), k, tau)
    err = np.abs(wts.cpu().numpy().astype(np.float64) - ref) / np.maximum(np.abs(ref), 1e-30)
    assert float(err.max()) <= TOL_W
