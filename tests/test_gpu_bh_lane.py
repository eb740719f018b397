"""The BH hash of few tokens with a coordinate to a lane (forward passes): against the oracle's codes, and bit for bit against the
stand-alone hash, which keeps the matrix cores' kernel -- where groups of two and four tokens and rows end, for every width and
block, with tables that run over from one projection into the next, and at both ends of the range of tokens.  Codes and sums
are exact; the weights are formed in the same order by both kernels, so they have the same bits.
"""
import shutil

import numpy as np
import pytest

import recorded as R

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    import oracle
    from paper_2403_07221_amd import binding as B
    from paper_2403_07221_amd import synth

CASES = [  # n, d, k, tau, block, factors, x dtype
    (1, 64, 8, 8, 64, 4, "f32"), (3, 40, 33, 7, 16, 1, "bf16"), (2049, 64, 8, 8, 32, 2, "f32"), (5, 128, 40, 9, 32, 3, "f16"),
    (6, 200, 96, 8, 64, 4, "f32"), (170, 255, 96, 8, 16, 4, "f32"), (171, 256, 96, 8, 32, 4, "bf16"), (7, 300, 33, 16, 16, 2, "f16"),
    (128, 512, 256, 8, 64, 4, "f32"), (129, 500, 57, 13, 32, 4, "f32"), (1, 513, 96, 8, 64, 4, "f32"), (17, 766, 170, 9, 64, 4, "f32"),
    (512, 768, 96, 8, 64, 4, "f32"), (513, 768, 96, 4, 16, 4, "bf16"), (1024, 1024, 128, 8, 64, 4, "f32"), (1025, 768, 96, 8, 64, 1, "f32"),
    (2, 1024, 256, 16, 64, 4, "f32"), (2047, 1000, 64, 15, 32, 2, "f16"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k,tau,b,m,xdt", CASES)
def test_few_tokens(n, d, k, tau, b, m, xdt):
    print(f"bh lane n={n} d={d} k={k} tau={tau} block={b} m={m} {xdt}", flush=True)
    w = synth.Workload("t", 7, n, d, m, k, tau, 8, x_dtype=xdt)
    bm = synth.make_bmats(31 * d + b, w.n_proj, m, w.d_pad, b)
    x = synth.make_x(7 * n + d, n, d, xdt)
    xd, bd = B.to_device(x), B.lookupffn_prepare_bh(torch.from_numpy(bm).cuda(), d, k, tau)
    g = torch.Generator(device="cuda").manual_seed(n)
    tables = torch.randn(k, 1 << tau, 8 if tau > 10 else 32, generator=g, device="cuda")
    want = oracle.bh_hash_codes(x, bm, k, tau)
    for bmats in (bd, torch.from_numpy(bm).cuda()):   # operand order prepared beforehand, and per call
        y = B.lookupffn_forward_bh(xd, bmats, tables)
        assert torch.equal(y, B.lookupffn_gather(torch.from_numpy(want.view(np.int16)).cuda(), tables))
        codes, weights = B.lookupffn_hash_bh_weighted(xd, bd, k, tau)
        y = B.lookupffn_forward_bh_weighted(xd, bmats, tables)
        assert torch.equal(y, B.lookupffn_gather_weighted(codes, weights, tables))


@pytest.mark.gpu
@pytest.mark.parametrize("d,b", [(64, 16), (512, 32), (768, 64)])
def test_infinite_and_nan_entries(d, b):
    n, k, tau = 6, 2 * d // 8, 4
    w = synth.Workload("t", 7, n, d, 2, k, tau, 8)
    bm = synth.make_bmats(d, w.n_proj, 2, w.d_pad, b)
    bm[0, 1, 1, 3, 5], bm[0, 0, 2, 0, 0] = np.inf, np.nan
    x = synth.make_x(d, n, d, "f32")
    x[1, 7], x[3, 0], x[4] = np.inf, np.nan, 0.0
    tables = torch.randn(k, 1 << tau, 16, device="cuda")
    xd, bd = B.to_device(x), torch.from_numpy(bm).cuda()
    assert torch.equal(B.lookupffn_forward_bh(xd, bd, tables), B.lookupffn_gather(B.lookupffn_hash_bh(xd, bd, k, tau), tables))


@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("n,d,k,tau,block,tokens,groups", [
    (1, 768, 96, 8, 64, 2, 1), (512, 768, 96, 8, 64, 2, 1), (513, 768, 96, 8, 64, 4, 1), (1024, 768, 96, 8, 64, 4, 1),
    (1025, 768, 96, 8, 64, 0, 1), (2048, 768, 96, 8, 32, 4, 1), (2049, 768, 96, 8, 32, 0, 1), (19, 1000, 228, 9, 64, 2, 3),
    (17, 768, 170, 9, 64, 2, 1), (128, 512, 256, 8, 64, 2, 4), (4096, 64, 8, 8, 64, 4, 1), (32769, 64, 8, 8, 64, 0, 1)])
def test_route(tmp_path, n, d, k, tau, block, tokens, groups):
    """Tokens of a workgroup and groups of projections; 0: bh_hash_kernel (256 compute units)."""
    calls = [R.option("gather_path", 1)]
    for name in ("lookupffn_forward_bh", "lookupffn_forward_bh_weighted"):
        calls.append([name, R.FAKE, R.FAKE, R.FAKE, R.FAKE, n, d, k, tau, 32, 0x100 | block, 4, 0, 0, R.FAKE, 1 << 40, None])
    for weights, launches in enumerate(R.record(R.build(tmp_path), calls)[1:]):
        hash_ = launches[0]
        assert launches[1].kernel == "gather_kernel" and len(launches) == 2
        if tokens == 0:
            assert hash_.kernel == "bh_hash_kernel"
            continue
        assert hash_.kernel == "bh_lane_kernel" and hash_.params[1:] == (block // 16, tokens, weights)
        assert hash_.grid == (-(-n // tokens), 1, groups) and hash_.block == 1 << hash_.params[0]


# The line of narrow rows in fills of the chip (n * P * d_pad / (256 * 1024)): both sides of it for the widths, bytes of factors and
# projections that it tells apart
@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("weighted,d,k,tau,block,factors,most", [
    (0, 64, 8, 8, 64, 4, 8192), (0, 64, 8, 8, 32, 4, 8192), (0, 64, 8, 8, 16, 4, 11315), (0, 64, 8, 8, 16, 1, 30515), (0, 64, 24, 8, 64, 4, 2730),
    (0, 64, 8, 8, 64, 16, 4496), (0, 128, 8, 8, 64, 4, 5920), (0, 100, 24, 8, 64, 4, 2960), (0, 128, 8, 8, 16, 4, 8320), (0, 128, 8, 8, 16, 1, 16384),
    (0, 128, 8, 8, 32, 4, 8192), (0, 256, 8, 8, 64, 4, 6144), (0, 256, 8, 8, 16, 4, 8192), (0, 256, 96, 8, 32, 4, 2048), (0, 256, 128, 8, 32, 4, 2048),
    (0, 256, 128, 8, 64, 4, 1536), (0, 200, 40, 9, 64, 4, 4096), (1, 64, 7, 9, 16, 4, 19507), (1, 64, 8, 8, 16, 4, 11315), (1, 128, 14, 9, 32, 4, 8768)])
def test_line_of_narrow_rows(tmp_path, weighted, d, k, tau, block, factors, most):
    name = "lookupffn_forward_bh" + ("_weighted" if weighted else "")
    calls = [R.option("gather_path", 1)]
    for n in (most, most + 1):
        calls.append([name, R.FAKE, R.FAKE, R.FAKE, R.FAKE, n, d, k, tau, 32, 0x100 | block, factors, 0, 0, R.FAKE, 1 << 40, None])
    kernels = [launches[0].kernel for launches in R.record(R.build(tmp_path), calls)[1:]]
    assert kernels == ["bh_lane_kernel", "bh_hash_kernel"]
