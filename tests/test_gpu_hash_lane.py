"""The hash of few tokens with a coordinate to a lane (forward passes) against the stand-alone hash, which keeps the kernels that
give a token to a wave and which the other tests hold to the oracle: codes, weights and shares have the same bits, so y has
them too.  Where groups of two and four tokens, rows and projections end, with tables across projections, for every width.
"""
import shutil

import pytest

import recorded as R

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

CASES = [  # n, d, k, tau, rounds, x dtype
    (1, 64, 8, 8, 2, "float32"), (3, 33, 90, 9, 3, "bfloat16"), (2049, 64, 8, 8, 1, "float32"), (5, 100, 33, 7, 3, "float16"),
    (17, 128, 40, 4, 5, "float32"), (16, 200, 96, 8, 3, "float32"), (683, 256, 96, 8, 3, "float32"), (15, 255, 37, 13, 4, "bfloat16"),
    (47, 511, 133, 9, 3, "float16"), (31, 512, 256, 8, 3, "float32"), (1, 513, 96, 8, 3, "float32"), (1001, 700, 97, 7, 3, "float16"),
    (513, 768, 96, 8, 3, "float32"), (512, 768, 170, 9, 2, "float32"), (6, 1024, 171, 12, 1, "float32"), (7, 1000, 300, 11, 3, "float32"),
    (2048, 1023, 64, 16, 3, "float32"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k,tau,rounds,xdt", CASES)
def test_few_tokens(n, d, k, tau, rounds, xdt):
    print(f"hash lane n={n} d={d} k={k} tau={tau} R={rounds} {xdt}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + d + k)
    d_pad = 1 << (d - 1).bit_length()
    x = torch.randn(n, d, generator=g, device="cuda").to(getattr(torch, xdt))
    signs = torch.randint(0, 2, (-(-k * tau // d_pad), rounds, d_pad), generator=g, device="cuda", dtype=torch.int8) * 2 - 1
    if n > 4:  # infinities and zeros stay what they are
        x[1, 7], x[2] = float("inf"), 0.0
    tables = torch.rand(k, 1 << tau, 4 if tau > 11 else 16, generator=g, device="cuda")
    B.lookupffn_set_option("small_tokens", -1)
    try:
        y = B.lookupffn_forward(x, signs, tables)
        assert B.lookupffn_last_hash_kernel() == "hash_lane_kernel"
        assert torch.equal(y, B.lookupffn_gather(B.lookupffn_hash(x, signs, k, tau), tables))
        assert B.lookupffn_last_hash_kernel() != "hash_lane_kernel"
    finally:
        B.lookupffn_set_option("small_tokens", 0)
    for forward, hash_, gather in ((B.lookupffn_forward_weighted, B.lookupffn_hash_weighted, B.lookupffn_gather_weighted),
                                   (B.lookupffn_forward_probes, B.lookupffn_hash_probes, B.lookupffn_gather_probes)):
        y = forward(x, signs, tables)
        assert B.lookupffn_last_hash_kernel() == "hash_lane_kernel"
        assert torch.equal(y.view(torch.int32), gather(*hash_(x, signs, k, tau), tables).view(torch.int32))


@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("n,d,k,tau,tokens,groups", [
    (1, 768, 96, 8, 2, 1), (512, 768, 96, 8, 2, 1), (513, 768, 96, 8, 4, 1), (2048, 768, 96, 8, 4, 1), (2049, 768, 96, 8, 0, 1),
    (1024, 768, 170, 9, 4, 1), (1025, 768, 170, 9, 0, 1), (13, 1000, 300, 11, 2, 4), (64, 512, 256, 8, 2, 4), (600, 512, 256, 8, 4, 2),
    (8192, 64, 8, 8, 2, 1), (8193, 64, 8, 8, 4, 1), (32769, 64, 8, 8, 0, 1), (5, 2048, 96, 8, 0, 1), (5, 32, 8, 8, 0, 1)])
@pytest.mark.parametrize("mode", ["weighted", "probes"])
def test_route(tmp_path, mode, n, d, k, tau, tokens, groups):
    """Tokens of a workgroup and groups of projections; 0: a kernel that gives a token to a wave (256 compute units)."""
    call = ["lookupffn_forward_" + mode, R.FAKE, R.FAKE, R.FAKE, R.FAKE, n, d, k, tau, 32, 3, 0, 0, R.FAKE, 1 << 40, None]
    launch = R.record(R.build(tmp_path), [R.option("gather_path", 1), call])[1][0]
    assert (launch.kernel == "hash_lane_kernel") == (tokens > 0)
    if tokens:
        assert launch.params[1:] == (tokens, R.MODES[mode])
        assert launch.grid == (-(-n // tokens), groups, 1) and launch.block == 1 << launch.params[0]
