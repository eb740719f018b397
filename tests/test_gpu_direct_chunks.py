"""The direct gather's chunks of eight codes: numbers of tables around one and two chunks, token rows of codes, weights
and shares that start at every 2- or 4-byte boundary, probe sequences that end inside a group of eight, rows of a whole
number of cache lines and not, one token to more than one full workgroup per column slice."""
import numpy as np
import pytest

import oracle
from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu

CASES = [(n, k, tau, d_out, tdt)
         for k, n, tau in ((1, 1, 4), (2, 33, 1), (7, 70, 3), (8, 9, 5), (9, 40, 4), (15, 5, 2), (16, 64, 6), (17, 129, 11),
                           (23, 8, 5), (24, 31, 16), (25, 1030, 6), (40, 3000, 5))
         for d_out, tdt in ((40, "f32"), (264, "bf16"), (128, "f16")) if (k << tau) * d_out <= 1 << 26]


@pytest.mark.parametrize("n,k,tau,d_out,tdt", CASES)
def test_direct_gather_chunks(n, k, tau, d_out, tdt):
    print(f"direct gather n={n} k={k} tau={tau} d_out={d_out} {tdt}", flush=True)
    rng = np.random.default_rng(n + 31 * k)
    tables = synth.make_tables(n + k, k, 1 << tau, d_out, tdt)
    codes = rng.integers(0, 1 << tau, size=(n, k)).astype(np.uint16)
    w = rng.uniform(0.1, 1.0, size=(n, k)).astype(np.float32)
    p = rng.uniform(0.0, 1.0, size=(n, k, tau + 1)).astype(np.float32)
    cd, wd, pd, td = torch.from_numpy(codes.view(np.int16)).cuda(), torch.from_numpy(w).cuda(), torch.from_numpy(p).cuda(), B.to_device(tables)
    B.lookupffn_set_option("gather_path", 1)
    try:
        y = B.lookupffn_gather(cd, td).cpu().numpy()
        yw = B.lookupffn_gather_weighted(cd, wd, td).cpu().numpy()
        yp = B.lookupffn_gather_probes(cd, pd, td).cpu().numpy()
    finally:
        B.lookupffn_set_option("gather_path", 0)
    assert np.array_equal(y, oracle.gather(codes, tables, acc64=False))
    # a chain of m fused multiply-adds is off by at most m * 2^-24 times the sum of its terms' magnitudes
    mag = np.abs(tables if tdt == "f32" else oracle.gather(np.arange(1 << tau, dtype=np.uint16)[:, None], tables[:1], acc64=True)).max() * 4
    for got, want, m, terms in ((yw, oracle.gather_weighted(codes, w, tables), k, k),
                                (yp, oracle.gather_probes(codes, p, tables), k * (tau + 1), k * (tau + 1))):
        assert np.max(np.abs(got.astype(np.float64) - want)) <= m * 2.0 ** -24 * terms * mag
