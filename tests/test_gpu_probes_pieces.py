"""Multi-probe batches at the limits of the staged gather's 32-bit offsets -- more than 2^25 tokens, which it takes in pieces; two
tables of more than 4 GiB together -- every token against the direct kernel.

Bar: the same bits.  Both kernels add a token's rows table by table and probe by probe with one fused multiply-add each.
"""
import pytest
import torch

from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _path():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    yield
    B.lookupffn_set_option("gather_path", 0)


@pytest.mark.parametrize("tau,k", [(7, 2), (9, 3)])
def test_pieces(tau, k):
    check((1 << 25) + 4097, k, tau, 16)


@pytest.mark.parametrize("tau,d_out", [(8, (1 << 21) + 256), (10, (1 << 19) + 256)])
def test_wide_tables(tau, d_out):
    check(2 << tau, 2, tau, d_out)


def check(n, k, tau, d_out):
    print(f"multi-probe n={n} tau={tau} k={k} d_out={d_out}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(tau)
    codes = torch.randint(0, 1 << tau, (n, k), generator=g, device="cuda", dtype=torch.int16)
    shares = torch.rand(n, k, 1 + tau, generator=g, device="cuda")
    tab = torch.randn(k, 1 << tau, d_out, generator=g, device="cuda")
    y = B.lookupffn_gather_probes(codes, shares, tab)
    assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"
    B.lookupffn_set_option("gather_path", 1)
    ref = B.lookupffn_gather_probes(codes, shares, tab)
    assert B.lookupffn_last_gather_kernel() == "gather_kernel"
    assert torch.equal(y, ref)
    B.lookupffn_release_workspace()
