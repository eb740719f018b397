"""The staged gather in every form it is built with -- token slots, slice width, tables a stage, plain, weighted and multi-probe --
over batches that fill the form's slots but for a few, every token compared.  (That these batches take the forms is checked on
the CPU: test_library_routes.py.)

Bars: plain bit-equal to the sequential fp32 sum; weighted and multi-probe within 1e-5 of the output's rms (8 (1 + tau) <= 88 terms,
each with one rounding of 6e-8 of a partial sum of a few rms).
"""
import pytest
import torch

import staged_forms as forms
from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(autouse=True)
def _staged():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    B.lookupffn_set_option("gather_path", 2)
    yield
    for option in ("gather_path", "token_slots", "slice_lanes"):
        B.lookupffn_set_option(option, 0)


def compare(n, k, tau, d_out, probes, prepared):
    g = torch.Generator(device="cuda").manual_seed(n + tau)
    codes = torch.randint(0, 1 << tau, (n, k), generator=g, device="cuda")
    tab = torch.randn(k, 1 << tau, d_out, generator=g, device="cuda")
    cd = codes.to(torch.int16)
    tables = B.lookupffn_prepare_tables(tab) if prepared else tab

    ref = torch.zeros(n, d_out, device="cuda")
    for j in range(k):
        ref += tab[j][codes[:, j]]
    assert torch.equal(B.lookupffn_gather(cd, tables), ref)
    assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"

    def near(y, terms):
        ref = torch.zeros(n, d_out, device="cuda", dtype=torch.float64)
        for share, j, rows in terms:
            ref += share.double()[:, None] * tab[j][rows].double()
        assert float((y - ref).abs().max() / ref.square().mean().sqrt()) <= TOL
        assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"

    w = torch.randn(n, k, generator=g, device="cuda")
    near(B.lookupffn_gather_weighted(cd, w, tables), ((w[:, j], j, codes[:, j]) for j in range(k)))
    if probes:
        p = torch.rand(n, k, 1 + tau, generator=g, device="cuda")
        near(B.lookupffn_gather_probes(cd, p, tables),
             ((p[:, j, q], j, codes[:, j] ^ (1 << q >> 1)) for j in range(k) for q in range(1 + tau)))


@pytest.mark.parametrize("tau,lanes,slots", forms.RANGES)
def test_token_ranges(tau, lanes, slots):
    print(f"staged form tau={tau} lanes={lanes} slots={slots}", flush=True)
    B.lookupffn_set_option("token_slots", slots)
    B.lookupffn_set_option("slice_lanes", lanes)
    # (128-byte slices of 512 rows are those of row-major tables only: the prepared pieces are 64 bytes)
    compare(forms.tokens(lanes, slots), forms.TABLES, tau, forms.width(lanes), forms.has_probes(tau, lanes), (tau, lanes) != (9, 8))


@pytest.mark.parametrize("d_out,tau,n,allowed,slots", forms.CHUNKS)
def test_whole_chunks(d_out, tau, n, allowed, slots):
    print(f"staged whole chunks tau={tau} d_out={d_out} n={n} slots={slots}", flush=True)
    B.lookupffn_set_option("token_slots", allowed)
    compare(n, 4, tau, d_out, False, True)
