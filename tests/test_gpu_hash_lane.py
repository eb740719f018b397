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

CASES = [  # n, d, k, tau, rounds, x dtype, forward passes that take the kernel: plain, weighted, probes
    (1, 64, 8, 8, 2, "float32", "wp"), (3, 33, 90, 9, 3, "bfloat16", "wp"), (2049, 64, 8, 8, 1, "float32", "wp"), (5, 100, 33, 7, 3, "float16", ""),
    (17, 128, 40, 4, 5, "float32", "wp"), (16, 200, 96, 8, 3, "float32", "cwp"), (683, 256, 96, 8, 3, "float32", "cwp"), (15, 255, 37, 13, 4, "bfloat16", "w"),
    (47, 511, 133, 9, 3, "float16", "cwp"), (31, 512, 256, 8, 3, "float32", "cwp"), (1, 513, 96, 8, 3, "float32", "cwp"), (1001, 700, 97, 7, 3, "float16", "cwp"),
    (513, 768, 96, 8, 3, "float32", "cwp"), (512, 768, 170, 9, 2, "float32", "cwp"), (6, 1024, 171, 12, 1, "float32", "cwp"), (7, 1000, 300, 11, 3, "float32", "cwp"),
    (2048, 1023, 64, 16, 3, "float32", "cwp"),
    (259, 61, 96, 8, 3, "float32", "cwp"), (300, 64, 97, 7, 1, "float16", "cwp"), (1025, 127, 64, 8, 3, "float32", "cwp"), (401, 100, 97, 7, 3, "bfloat16", "wp"),
    (4099, 128, 8, 8, 2, "float32", "wp"), (1025, 256, 64, 8, 3, "float32", "cwp"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k,tau,rounds,xdt,takes", CASES)
def test_few_tokens(n, d, k, tau, rounds, xdt, takes):
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
        assert (B.lookupffn_last_hash_kernel() == "hash_lane_kernel") == ("c" in takes)
        assert torch.equal(y, B.lookupffn_gather(B.lookupffn_hash(x, signs, k, tau), tables))
        assert B.lookupffn_last_hash_kernel() != "hash_lane_kernel"
    finally:
        B.lookupffn_set_option("small_tokens", 0)
    for forward, hash_, gather in ((B.lookupffn_forward_weighted, B.lookupffn_hash_weighted, B.lookupffn_gather_weighted),
                                   (B.lookupffn_forward_probes, B.lookupffn_hash_probes, B.lookupffn_gather_probes)):
        y = forward(x, signs, tables)
        assert (B.lookupffn_last_hash_kernel() == "hash_lane_kernel") == (("w" if hash_ is B.lookupffn_hash_weighted else "p") in takes)
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


# Tokens of a workgroup on both sides of the lines that go by width, rounds, projections and what is asked for (256 compute units)
@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("mode,n,d,k,tau,rounds,tokens", [
    ("plain", 255, 64, 96, 8, 3, 0), ("plain", 256, 64, 96, 8, 3, 4), ("plain", 2730, 64, 96, 8, 3, 4), ("plain", 2731, 64, 96, 8, 3, 0),
    ("plain", 4096, 64, 8, 8, 4, 0), ("plain", 2048, 64, 24, 8, 2, 0), ("plain", 2048, 64, 24, 8, 3, 4),
    ("plain", 1024, 128, 64, 8, 3, 0), ("plain", 1025, 128, 64, 8, 3, 4), ("plain", 2560, 128, 64, 8, 3, 4), ("plain", 2561, 128, 64, 8, 3, 0),
    ("plain", 2048, 128, 32, 8, 3, 0), ("plain", 1025, 128, 64, 8, 2, 0), ("plain", 1025, 128, 73, 7, 3, 0),
    ("plain", 1024, 256, 64, 8, 3, 2), ("plain", 1025, 256, 64, 8, 2, 4), ("plain", 64, 256, 32, 8, 3, 0), ("plain", 64, 256, 56, 9, 3, 0), ("plain", 1792, 256, 64, 8, 4, 4), ("plain", 1793, 256, 64, 8, 4, 0),
    ("plain", 1706, 256, 96, 8, 3, 4), ("plain", 1707, 256, 96, 8, 3, 0), ("plain", 2048, 256, 128, 8, 3, 4), ("plain", 2048, 256, 128, 8, 2, 4), ("plain", 300, 256, 96, 8, 2, 0),
    ("plain", 1365, 256, 170, 9, 3, 4), ("plain", 300, 256, 170, 9, 2, 0), ("plain", 896, 256, 112, 9, 3, 4), ("plain", 897, 256, 112, 9, 3, 0), ("plain", 1025, 128, 170, 9, 3, 4), ("plain", 1024, 128, 170, 9, 3, 0),
    ("plain", 4096, 512, 64, 8, 2, 4), ("plain", 2048, 512, 128, 8, 2, 4), ("plain", 2049, 512, 128, 8, 2, 0),
    ("plain", 256, 512, 97, 7, 3, 2), ("plain", 256, 512, 97, 7, 2, 0), ("plain", 513, 512, 128, 9, 2, 4),
    ("plain", 819, 512, 250, 10, 3, 4), ("plain", 1024, 768, 96, 8, 2, 4), ("plain", 1025, 768, 96, 8, 2, 0),
    ("plain", 2047, 768, 96, 8, 3, 4), ("plain", 513, 768, 170, 9, 2, 0), ("plain", 1024, 768, 170, 9, 3, 4), ("plain", 1025, 768, 170, 9, 3, 0),
    ("plain", 513, 768, 250, 8, 4, 0), ("plain", 1024, 767, 250, 8, 2, 4), ("plain", 682, 768, 300, 10, 2, 4), ("plain", 2047, 641, 96, 8, 2, 4), ("plain", 512, 768, 170, 9, 2, 2),
    ("weighted", 512, 768, 170, 9, 2, 2), ("weighted", 513, 768, 170, 9, 2, 4), ("weighted", 512, 768, 256, 8, 2, 4),
    ("weighted", 4095, 128, 8, 8, 3, 0), ("weighted", 4096, 128, 8, 8, 3, 2), ("weighted", 4097, 128, 8, 8, 3, 4), ("probes", 341, 128, 97, 7, 3, 0),
    ("probes", 342, 128, 97, 7, 3, 2), ("weighted", 5119, 128, 24, 9, 2, 0), ("weighted", 5120, 128, 24, 9, 2, 4), ("plain", 4659, 64, 24, 9, 3, 0), ("plain", 1024, 64, 56, 9, 3, 4),
    ("probes", 4095, 64, 8, 10, 3, 0), ("probes", 4096, 64, 8, 10, 3, 2), ("weighted", 512, 64, 8, 10, 3, 2), ("weighted", 513, 64, 8, 10, 3, 0),
    ("probes", 60, 256, 40, 9, 3, 0), ("weighted", 60, 256, 40, 9, 3, 2), ("weighted", 1, 128, 64, 8, 3, 2), ("weighted", 1365, 256, 97, 7, 3, 4), ("weighted", 1366, 256, 97, 7, 3, 0), ("weighted", 1366, 256, 112, 9, 3, 4),
    ("probes", 1366, 256, 96, 8, 3, 4), ("probes", 682, 512, 170, 9, 3, 4), ("probes", 683, 512, 170, 9, 3, 0), ("weighted", 683, 512, 170, 9, 3, 4)])
def test_lines(tmp_path, mode, n, d, k, tau, rounds, tokens, x_dtype=0):
    name = "lookupffn_forward" + ("" if mode == "plain" else "_" + mode)
    call = [name, R.FAKE, R.FAKE, R.FAKE, R.FAKE, n, d, k, tau, 32, rounds, x_dtype, 0, R.FAKE, 1 << 40, None]
    launch = R.record(R.build(tmp_path), [R.option("gather_path", 1), R.option("small_tokens", -1), call])[2][0]
    assert (launch.params[1] if launch.kernel == "hash_lane_kernel" else 0) == tokens


@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("n,d,k,tau,rounds,tokens", [(300, 256, 96, 8, 2, 2), (300, 256, 170, 9, 2, 2), (300, 256, 170, 9, 1, 0), (256, 512, 97, 7, 2, 2), (64, 128, 96, 8, 2, 0)])
def test_lines_of_16_bit_rows(tmp_path, n, d, k, tau, rounds, tokens):
    test_lines(tmp_path, "plain", n, d, k, tau, rounds, tokens, x_dtype=2)
