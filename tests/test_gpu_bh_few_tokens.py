"""BH hash of few tokens, whose projections are spread over workgroups: codes bit-exact and weights within 1e-5 relative of the
oracle's (as for every other batch), with tables that run over from one projection into the next and with tables that do not,
and equal to the same tokens' inside a batch that keeps the projections together."""
import numpy as np
import pytest
import torch

import oracle
from paper_2403_07221_amd import binding as B
from paper_2403_07221_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,k,tau,block", [
    (64, 40, 9, 16), (64, 17, 5, 64), (100, 96, 8, 32), (256, 170, 9, 32), (300, 200, 7, 16), (500, 256, 4, 64),
    (768, 170, 9, 64),  # two projections with a table across them: stay together
    (1024, 256, 16, 16), (1024, 140, 15, 32), (1000, 228, 9, 64), (1024, 256, 16, 64)])
@pytest.mark.parametrize("n", [1, 19])
def test_projections_over_workgroups(n, d, k, tau, block):
    print(f"bh few tokens n={n} d={d} k={k} tau={tau} block={block}", flush=True)
    w = synth.Workload("t", 7, n, d, 4, k, tau, 8)
    bm = synth.make_bmats(100 * d + tau, w.n_proj, 4, w.d_pad, block)
    many = 40000 // w.n_proj                    # workgroups enough that the projections stay together
    x = synth.make_x(d + k, many, d, "f32")
    x[:n] = synth.make_x(d + k + 1, n, d, "f32")
    bd = B.lookupffn_prepare_bh(B.to_device(bm), d, k, tau)
    want, ww = oracle.bh_hash_codes(x[:n], bm, k, tau), oracle.weights_from_z(oracle.bh_soft_codes(x[:n], bm, k, tau), k, tau)
    codes = B.codes_to_numpy(B.lookupffn_hash_bh(B.to_device(x[:n]), bd, k, tau))
    assert np.array_equal(codes, want)
    codes, weights = B.lookupffn_hash_bh_weighted(B.to_device(x[:n]), bd, k, tau)
    assert np.array_equal(B.codes_to_numpy(codes), want)
    np.testing.assert_allclose(weights.cpu().numpy(), ww, rtol=1e-5, atol=1e-30)
    big_codes, big = B.lookupffn_hash_bh_weighted(B.to_device(x), bd, k, tau)
    assert np.array_equal(B.codes_to_numpy(big_codes)[:n], want) and torch.equal(big[:n], weights)
