"""The staged gather where its stages and lagging groups begin and end: few tables, every table size, small batches (chunks of a
few tokens in the forms of four slots, or six for 64-byte slices, whatever limit is set; the other slot counts:
test_gpu_staged_forms.py).  Multi-probe groups that lag a table behind read zeros in the first and the last step, so an
infinite row of those tables reaches only the tokens that probe it.

Bars: plain bit-equal to the sequential fp32 sum; weighted and multi-probe within 1e-5 of the output's rms (k (1 + tau) <= 88
terms, each with one rounding of 6e-8 of a partial sum of a few rms).
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(autouse=True)
def _staged():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    B.lookupffn_set_option("gather_path", 2)
    yield
    B.lookupffn_set_option("gather_path", 0)
    B.lookupffn_set_option("token_slots", 0)
    B.lookupffn_set_option("slice_lanes", 0)


def make(n, k, tau, d_out):
    g = np.random.default_rng(1000 * n + 10 * k + tau)
    codes = g.integers(0, 1 << tau, (n, k)).astype(np.uint16)
    tables = g.standard_normal((k, 1 << tau, d_out), dtype=np.float32)
    return codes, tables, g


def rms_err(y, ref):
    return float(np.max(np.abs(y.astype(np.float64) - ref)) / np.sqrt(np.mean(np.asarray(ref, np.float64) ** 2)))


@pytest.mark.parametrize("tau,slots", [(7, 0), (7, 3), (8, 0), (8, 5), (9, 0), (9, 8), (10, 0), (10, 13)])
@pytest.mark.parametrize("n,k,d_out", [(1, 2, 96), (1025, 4, 96), (4099, 6, 132), (9000, 8, 32)])
def test_stages_and_slots(n, k, tau, d_out, slots):
    print(f"staged n={n} k={k} tau={tau} d_out={d_out} slots={slots}", flush=True)
    B.lookupffn_set_option("token_slots", slots)
    codes, tables, g = make(n, k, tau, d_out)
    w = g.standard_normal((n, k), dtype=np.float32)
    p = g.random((n, k, 1 + tau), dtype=np.float32)
    cd, td = B.to_device(codes.view(np.int16)), B.to_device(tables)
    for tab in (td, B.lookupffn_prepare_tables(td)):
        y = B.lookupffn_gather(cd, tab).cpu().numpy()
        assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"
        assert np.array_equal(y, oracle.gather(codes, tables, acc64=False))
        y = B.lookupffn_gather_weighted(cd, B.to_device(w), tab).cpu().numpy()
        assert rms_err(y, oracle.gather_weighted(codes, w, tables)) <= TOL
        y = B.lookupffn_gather_probes(cd, B.to_device(p), tab).cpu().numpy()
        assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"
        assert rms_err(y, oracle.gather_probes(codes, p, tables)) <= TOL


@pytest.mark.parametrize("tau", [7, 8, 9, 10])
def test_infinite_rows_reach_only_the_tokens_that_probe_them(tau):
    n, k, d_out = 3000, 4, 64
    print(f"multi-probe infinite rows tau={tau}", flush=True)
    codes, tables, g = make(n, k, tau, d_out)
    hit = np.zeros(n, bool)
    for j in (0, k - 1):
        tables[j, 0] = np.inf
        hit |= (codes[:, j] == 0) | ((codes[:, j] & (codes[:, j] - 1)) == 0)  # row 0 or one flip away from it
    p = g.random((n, k, 1 + tau), dtype=np.float32)
    y = B.lookupffn_gather_probes(B.to_device(codes.view(np.int16)), B.to_device(p), B.to_device(tables)).cpu().numpy()
    assert np.all(np.isinf(y[hit])) and hit.any()
    ref = oracle.gather_probes(codes[~hit], p[~hit], tables)
    assert rms_err(y[~hit], ref) <= TOL


@pytest.mark.parametrize("n", [1, 1025])
def test_one_wide_table_a_stage(n):
    """A stage of one 64 KB table slice and four token slots: the rows read ahead of the sums are the whole stage."""
    k, tau, d_out = 4, 9, 96
    print(f"staged, 128-byte slices of 512-row tables n={n}", flush=True)
    B.lookupffn_set_option("token_slots", 4)
    B.lookupffn_set_option("slice_lanes", 8)
    codes, tables, g = make(n, k, tau, d_out)
    w = g.standard_normal((n, k), dtype=np.float32)
    cd, td = B.to_device(codes.view(np.int16)), B.to_device(tables)
    assert np.array_equal(B.lookupffn_gather(cd, td).cpu().numpy(), oracle.gather(codes, tables, acc64=False))
    y = B.lookupffn_gather_weighted(cd, B.to_device(w), td).cpu().numpy()
    assert rms_err(y, oracle.gather_weighted(codes, w, tables)) <= TOL
    assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"
