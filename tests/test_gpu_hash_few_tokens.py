"""Sign-diagonal hash of few tokens, whose projections are spread over workgroups: codes bit-exact, weights and shares within
1e-5 relative of the oracle's, with tables that run over from one projection into the next and with tables that do not."""
import numpy as np
import pytest
import torch

import oracle
from paper_2403_07221_amd import binding as B
from paper_2403_07221_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k,tau,R", [(64, 40, 9, 2), (33, 17, 16, 4), (119, 170, 8, 4), (256, 170, 9, 3), (500, 200, 11, 1),
                                       (1000, 300, 11, 1), (768, 170, 13, 2), (1024, 256, 9, 3), (1024, 256, 16, 4), (700, 205, 15, 5), (2048, 500, 13, 2)])
@pytest.mark.parametrize("n", [1, 13])
def test_projections_over_workgroups(n, d, k, tau, R):
    print(f"hash few tokens n={n} d={d} k={k} tau={tau} R={R}", flush=True)
    w = synth.Workload("t", 7, n, d, R, k, tau, 8)
    assert w.n_proj >= 3
    signs, x = synth.make_signs(10 * d + tau, w.n_proj, R, w.d_pad), synth.make_x(d + k, n, d, "f32")
    xd, sd = B.to_device(x), B.to_device(signs)
    z = oracle.soft_codes(x, signs, k, tau)
    want, shares = oracle.probe_weights_from_z(z, k, tau)
    assert np.array_equal(B.codes_to_numpy(B.lookupffn_hash(xd, sd, k, tau)), want)
    codes, wt = B.lookupffn_hash_weighted(xd, sd, k, tau)
    assert np.array_equal(B.codes_to_numpy(codes), want)
    np.testing.assert_allclose(wt.cpu().numpy(), oracle.weights_from_z(z, k, tau), rtol=1e-5, atol=1e-30)
    codes, sh = B.lookupffn_hash_probes(xd, sd, k, tau)
    assert np.array_equal(B.codes_to_numpy(codes), want)
    np.testing.assert_allclose(sh.cpu().numpy(), shares, rtol=1e-5, atol=1e-30)
