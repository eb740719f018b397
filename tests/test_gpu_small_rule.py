"""Which batches of narrow inputs lookupffn_forward runs in one launch: both sides of each limit of the rule, with the
oracle's bits on either route; rows and signs that start at any element."""
import numpy as np
import pytest

import oracle
from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu

ONE = "forward_small_kernel"


def layer(n, d, k, tau, d_out, tdt="f32", rounds=2):
    d_pad = 64
    while d_pad < d:
        d_pad *= 2
    return (synth.make_x(n + d, n, d), synth.make_signs(k, -(-k * tau // d_pad), rounds, d_pad),
            synth.make_tables(d_out, k, 1 << tau, d_out, tdt))


# the two columns: tokens that take one launch, tokens that do not (256 compute units)
@pytest.mark.parametrize("d,k,tau,d_out,tdt,one,two", [
    (64, 8, 8, 64, "f32", [1, 300, 512], [513]),          # the option's default batch limit
    (256, 64, 4, 512, "f32", [256, 320], [321]),          # 128 KiB a token: 40 MiB beyond one token a compute unit
    (256, 64, 4, 1024, "f32", [256], [257]),              # 256 KiB a token
    (64, 8, 4, 4096, "f32", [1, 256], [257]),             # rows of four turns
    (64, 8, 4, 1280, "f32", [257], []),                   # of one and a quarter
    (64, 8, 4, 2048, "f32", [256], [257]),                # of two
    (64, 8, 4, 6144, "f32", [], [1, 200]),                # of six, few tables
    (64, 8, 4, 8192, "bf16", [256], [257]),               # 16-bit rows: four turns
    (128, 64, 4, 4096, "f32", [80, 256], [1, 79]),        # eight turns, many tables
    (512, 64, 4, 2048, "f32", [1, 256], [257]),           # 64 tables: two turns of two
    (64, 4, 16, 256, "f32", [1], []),                     # tables of 256 MiB
    (64, 5, 16, 256, "f32", [], [1, 64]),                 # and more
])
def test_both_sides_of_the_rule(d, k, tau, d_out, tdt, one, two):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the sizes are those of 256 compute units")
    n = max(one + two)
    print(f"small rule d={d} k={k} tau={tau} d_out={d_out} {tdt} up to {n}", flush=True)
    x, signs, tables = layer(n, d, k, tau, d_out, tdt)
    want = oracle.forward(x, signs, tables, acc64=False)
    xd, sd, td = B.to_device(x), B.to_device(signs), B.to_device(tables)
    for m in one + two:
        y = B.lookupffn_forward(xd[:m], sd, td)
        assert (B.lookupffn_last_gather_kernel() == ONE) == (m in one), m
        assert np.array_equal(y.cpu().numpy(), want[:m]), m


def test_option_overrides_the_rate_but_not_the_kernel():
    print("small rule: option", flush=True)
    x, signs, tables = layer(600, 64, 8, 4, 6144)
    xd, sd, td = B.to_device(x), B.to_device(signs), B.to_device(tables)
    want = oracle.forward(x, signs, tables, acc64=False)
    try:
        for option, n, kernel in ((600, 600, True), (600, 1, True), (599, 600, False), (-1, 1, False)):
            B.lookupffn_set_option("small_tokens", option)
            y = B.lookupffn_forward(xd[:n], sd, td)
            assert (B.lookupffn_last_gather_kernel() == ONE) == kernel
            assert np.array_equal(y.cpu().numpy(), want[:n])
        # the row offsets of 16400 codes are more than the 64 KB of LDS: the two kernels whatever the option
        x, signs, tables = layer(3, 512, 16400, 1, 8, rounds=1)
        want = oracle.forward(x, signs, tables, acc64=False)
        for option in (0, 512):
            B.lookupffn_set_option("small_tokens", option)
            y = B.lookupffn_forward(B.to_device(x), B.to_device(signs), B.to_device(tables))
            assert B.lookupffn_last_gather_kernel() != ONE
            assert np.array_equal(y.cpu().numpy(), want)
    finally:
        B.lookupffn_set_option("small_tokens", 0)


@pytest.mark.parametrize("xdt", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("d", [33, 100, 512])
def test_rows_and_signs_at_any_element(d, xdt):
    print(f"small launch, unaligned x and signs d={d} {xdt}", flush=True)
    n, k, tau = 37, 9, 7
    d_pad = 64
    while d_pad < d:
        d_pad *= 2
    x = synth.make_x(n + d, n, d, xdt)
    signs, tables = synth.make_signs(k, -(-k * tau // d_pad), 3, d_pad), synth.make_tables(d, k, 1 << tau, 40)
    xd, sd = B.to_device(x), B.to_device(signs)
    xbuf = torch.empty(n * d + 1, dtype=xd.dtype, device="cuda")
    sbuf = torch.empty(signs.size + 1, dtype=torch.int8, device="cuda")
    xs, ss = xbuf[1:].view(n, d).copy_(xd), sbuf[1:].view(sd.shape).copy_(sd)
    y = B.lookupffn_forward(xs, ss, B.to_device(tables))
    assert B.lookupffn_last_gather_kernel() == ONE
    assert np.array_equal(y.cpu().numpy(), oracle.forward(x, signs, tables, acc64=False))
