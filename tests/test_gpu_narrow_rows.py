"""One launch for a batch of one layer of narrow rows at d_pad = 1024 (forward_narrow_kernel): bit-equal to hash and gather as two
launches, which the other tests hold to the oracle -- where rows end in a wave's 64 dwords and in a slice, tables end in a chunk of
fetches, codes cross projections, for every row type and number of rounds; y over x; and both sides of its rule."""
import shutil

import pytest

import recorded as R

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

NAME = "forward_narrow_kernel"
CASES = [  # n, d, k, tau, d_out, rounds, x, tables, y, prepared
    (513, 768, 96, 8, 64, 3, "float32", "float32", "float32", True), (700, 1024, 1, 1, 4, 1, "float32", "float32", "float32", False),
    (1025, 520, 17, 9, 68, 2, "bfloat16", "float32", "float32", True), (600, 900, 33, 7, 252, 4, "float16", "float32", "float16", False),
    (2049, 768, 15, 16, 8, 3, "float32", "bfloat16", "float32", False), (777, 1023, 31, 11, 136, 3, "float32", "float16", "bfloat16", False),
    (514, 768, 250, 8, 512, 3, "float32", "float32", "float32", False), (515, 768, 114, 9, 508, 3, "float32", "float32", "float32", True),
    (519, 800, 64, 10, 1024, 3, "float16", "bfloat16", "bfloat16", False), (530, 640, 300, 13, 16, 2, "float32", "float16", "float32", False),
]


def inputs(n, d, k, tau, d_out, rounds, x, tables):
    g = torch.Generator(device="cuda").manual_seed(n + d + k)
    xd = torch.randn(n, d, generator=g, device="cuda").to(getattr(torch, x))
    xd[2], xd[3, 5] = 0.0, float("inf")
    signs = torch.randint(0, 2, (-(-k * tau // 1024), rounds, 1024), generator=g, device="cuda", dtype=torch.int8) * 2 - 1
    t = torch.randn(k, 1 << tau, d_out, generator=g, device="cuda").to(getattr(torch, tables))
    return xd, signs, t


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k,tau,d_out,rounds,x,tables,y,prepared", CASES)
def test_as_two_launches(n, d, k, tau, d_out, rounds, x, tables, y, prepared):
    print(f"narrow rows n={n} d={d} k={k} tau={tau} d_out={d_out} R={rounds} {x} {tables} {y} prepared={prepared}", flush=True)
    xd, signs, t = inputs(n, d, k, tau, d_out, rounds, x, tables)
    t = B.lookupffn_prepare_tables(t) if prepared else t
    out = torch.empty(n, d_out, device="cuda", dtype=getattr(torch, y))
    B.lookupffn_forward_stack(xd, [signs], [t], y=out)
    assert B.lookupffn_last_gather_kernel() == NAME and B.lookupffn_last_hash_kernel() == NAME
    B.lookupffn_set_option("small_tokens", -1)
    try:
        want = B.lookupffn_forward(xd, signs, t, y=torch.empty_like(out))
        assert B.lookupffn_last_gather_kernel() != NAME
    finally:
        B.lookupffn_set_option("small_tokens", 0)
    bits = torch.int32 if y == "float32" else torch.int16
    assert torch.equal(out.view(bits), want.view(bits))


@pytest.mark.gpu
def test_y_over_x():
    """Rows of one length in bytes (1024 half inputs, 512 fp32 outputs): a workgroup reads its row before it writes it."""
    n, k, tau = 1500, 16, 8
    xd, signs, t = inputs(n, 1024, k, tau, 512, 3, "float16", "float32")
    want = B.lookupffn_forward_stack(xd, [signs], [t], y=torch.empty(n, 512, device="cuda"))
    over = xd.clone()
    B.lookupffn_forward_stack(over, [signs], [t], y=over.view(torch.float32))
    assert B.lookupffn_last_gather_kernel() == NAME
    assert torch.equal(over.view(torch.int32), want.view(torch.int32))


@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("n,d,d_out,dtype,kernel,threads", [
    (512, 768, 64, 0, "forward_stack_kernel", 1024), (513, 768, 64, 0, NAME, 64), (513, 768, 68, 0, NAME, 128), (513, 768, 512, 0, NAME, 512),
    (513, 768, 516, 0, "forward_stack_kernel", 1024), (513, 768, 1024, 1, NAME, 512), (513, 768, 1024, 0x101, "forward_stack_kernel", 1024),
    (513, 768, 512, 0x101, NAME, 512), (1 << 20, 768, 8, 2, NAME, 64)])
def test_route(tmp_path, n, d, d_out, dtype, kernel, threads):
    """256 compute units; the single launch asked for at every batch size."""
    call = ["lookupffn_forward", R.FAKE, R.FAKE, R.FAKE, 1 << 45, n, d, 16, 8, d_out, 3, 0, dtype, R.FAKE, 1 << 40, None]
    (launch,) = R.record(R.build(tmp_path), [R.option("small_tokens", 1 << 20), call])[1]
    assert launch.kernel == kernel and launch.block == threads
