"""The staged gather where the workgroups of an XCD divide whole chunks of its slices instead of token ranges: a workgroup that
changes slice between two chunks, chunks that do not divide evenly, both slice widths.  Every token is compared.

Bars: plain bit-equal to the sequential fp32 sum; weighted within 1e-5 of the output's rms (two terms, each rounded by 6e-8 of at
most some twenty rms).
"""
import pytest
import torch

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


# (32 compute units an XCD) chunks a workgroup with token ranges -> with whole chunks: 3 -> 2, 4 -> 3, 4 -> 3, 4 -> 3, 3 -> 2
@pytest.mark.parametrize("n,d_out,tau,slots", [(25013, 288, 8, 4), (15827, 768, 7, 4), (9703, 1280, 8, 4), (65536, 768, 8, 0),
                                               (61757, 192, 9, 6)])
def test_whole_chunks(n, d_out, tau, slots):
    print(f"whole chunks n={n} d_out={d_out} tau={tau} slots={slots}", flush=True)
    B.lookupffn_set_option("token_slots", slots)
    k = 2
    g = torch.Generator().manual_seed(n + tau)
    codes = torch.randint(0, 1 << tau, (n, k), generator=g)
    cd = codes.to(torch.int16).cuda()
    rows = codes.cuda()
    tab = torch.randn(k, 1 << tau, d_out, generator=g).cuda()
    w = torch.randn(n, k, generator=g).cuda()
    prepared = B.lookupffn_prepare_tables(tab)

    ref = tab[0][rows[:, 0]] + tab[1][rows[:, 1]]
    assert torch.equal(B.lookupffn_gather(cd, prepared), ref)
    assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"

    ref = w[:, 0, None] * tab[0][rows[:, 0]] + w[:, 1, None] * tab[1][rows[:, 1]]
    y = B.lookupffn_gather_weighted(cd, w, prepared)
    assert float((y - ref).abs().max() / ref.square().mean().sqrt()) <= TOL
    assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"
