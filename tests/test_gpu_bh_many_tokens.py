"""The BH hash of more tokens than one row of a launch grid has work-items for (2^32 along x: 2^30 tokens of d_pad = 64)."""
import numpy as np
import pytest

import oracle
from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu


def test_more_than_two_to_the_thirty_tokens():
    d, k, tau, m, block, period = 33, 1, 5, 2, 16, 4099
    reps = (1 << 30) // period + 1
    n = reps * period                       # just over 2^30; the rows repeat with an odd period
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 90 GiB of free device memory for the rows")
    print(f"bh hash of {n} tokens of {d}", flush=True)
    x = synth.make_x(d, period, d, "bf16")
    bm = synth.make_bmats(d, 1, m, 64, block)
    want = oracle.bh_hash_codes(x, bm, k, tau)
    base = B.to_device(x)
    xd = torch.empty((n, d), dtype=torch.bfloat16, device="cuda")
    xd.view(reps, period, d).copy_(base.expand(reps, period, d))
    bd = torch.from_numpy(bm).cuda()
    codes = B.lookupffn_hash_bh(xd, bd, k, tau)
    rows = codes.view(reps, period, k)
    assert np.array_equal(B.codes_to_numpy(rows[0]), want)
    assert bool((rows == rows[0]).all())
    del rows, codes
    codes, weights = B.lookupffn_hash_bh_weighted(xd, bd, k, tau)
    rows, ws = codes.view(reps, period, k), weights.view(reps, period, k)
    assert np.array_equal(B.codes_to_numpy(rows[-1]), want)
    assert bool((rows == rows[0]).all()) and bool((ws == ws[0]).all()) and bool((ws > 0).all())
    del xd, rows, ws, codes, weights
    torch.cuda.empty_cache()
