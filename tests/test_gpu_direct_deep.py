"""The direct gather's form for few wavefronts and many tables (sixteen or thirty-two rows in flight): numbers of tables around its groups
of eight and sixteen and the chunks of eight behind them, one token to the edge of its rule, every row type and slice width.

Bars: plain bit-equal to the sequential fp32 sum; weighted within k * 2^-24 * sum |w row| <= 2e-5 of the output's rms for the
171 terms at most and weights below one."""
import numpy as np
import pytest
import torch

import oracle
from paper_2403_07221_amd import binding as B
from paper_2403_07221_amd import synth

pytestmark = pytest.mark.gpu


KS = [48, 49, 55, 63, 64, 71, 79, 80, 95, 96, 97, 103, 104, 111, 112, 127, 128, 135, 144, 159, 160, 170, 171]
SHAPES = [(1, 4, 40, "f32", False), (9, 9, 264, "f32", True), (300, 6, 128, "f32", False), (67, 5, 136, "bf16", False),
          (130, 4, 648, "f16", False), (1001, 4, 768, "f16", False), (900, 4, 344, "f32", False)]


@pytest.mark.parametrize("k", KS)
@pytest.mark.parametrize("n,tau,d_out,tdt,prep", SHAPES)
def test_deep_direct_gather(n, k, tau, d_out, tdt, prep):
    print(f"deep direct gather n={n} k={k} tau={tau} d_out={d_out} {tdt}", flush=True)
    rng = np.random.default_rng(n + 31 * k)
    tables = synth.make_tables(n + k, k, 1 << tau, d_out, tdt)
    codes = rng.integers(0, 1 << tau, size=(n, k)).astype(np.uint16)
    w = rng.uniform(0.1, 1.0, size=(n, k)).astype(np.float32)
    cd, wd, td = torch.from_numpy(codes.view(np.int16)).cuda(), torch.from_numpy(w).cuda(), B.to_device(tables)
    if prep:
        td = B.lookupffn_prepare_tables(td)
    B.lookupffn_set_option("gather_path", 1)
    try:
        y = B.lookupffn_gather(cd, td).cpu().numpy()
        yw = B.lookupffn_gather_weighted(cd, wd, td).cpu().numpy()
    finally:
        B.lookupffn_set_option("gather_path", 0)
    assert np.array_equal(y, oracle.gather(codes, tables, acc64=False))
    ref = oracle.gather_weighted(codes, w, tables).astype(np.float64)
    assert float(np.max(np.abs(yw - ref)) / np.sqrt(np.mean(ref ** 2))) <= 2e-5
