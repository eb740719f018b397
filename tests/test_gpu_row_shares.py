"""Multi-probe forward passes whose hash writes the staged gather's shares itself (hash_row_kernel, tau = 8): held against the
stand-alone hash and gather, which form the shares table by table in the ABI layout.

Both sides take the same z.  A share is 1 / (product of eight factors) times an exponential: three levels of rounding here and
seven there, the reciprocal and the last product 1 ulp each, so two shares differ by no more than 16 * 2^-24 of themselves;
both sums run over the same k * 9 terms in the same order, each adding at most a rounding of its partial sum."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu


def d_pad(d):
    return 1 << max(0, d - 1).bit_length()


@pytest.mark.parametrize("n,d,k,d_out,rounds,x_dtype,y_dtype,kernel", [
    (1536, 768, 96, 128, 3, "float32", "float32", "hash_row_kernel"),     # smallest batch; the form built for 768
    (4097, 1024, 130, 64, 3, "bfloat16", "float32", "hash_row_kernel"),   # two projections, tokens beyond a wave's four
    (5003, 528, 6, 72, 1, "float16", "bfloat16", "hash_row_kernel"),      # a few registers hold coordinates
    (4999, 640, 250, 32, 4, "float32", "float32", "hash_row_kernel"),     # the last register half full
    (1539, 512, 66, 40, 3, "float32", "float32", "hash_row_kernel"),     # eight lanes a token, two projections
    (12293, 272, 64, 128, 2, "bfloat16", "float16", "hash_row_kernel"),
    (1535, 768, 96, 128, 3, "float32", "float32", "hash_lane_kernel"),    # below the line
    (4100, 768, 97, 128, 3, "float32", "float32", "hash1024_kernel"),     # odd k: the last table apart
    (4100, 776, 96, 128, 3, "float32", "float32", "hash1024_kernel"),     # rows no multiple of 16
])
def test_forward_probes_row_shares(n, d, k, d_out, rounds, x_dtype, y_dtype, kernel):
    tau = 8
    x_dtype, y_dtype = getattr(torch, x_dtype), getattr(torch, y_dtype)
    print(f"row shares n={n} d={d} k={k} d_out={d_out} R={rounds}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n + d + k)
    x = torch.randn(n, d, device="cuda", generator=gen).to(x_dtype)
    x[1] *= 40.0       # a hash far from its planes: shares of almost 1 and almost 0
    x[2] = 0.0         # on all of them: equal shares
    P = -(-k * tau // d_pad(d))
    signs = (torch.randint(0, 2, (P, rounds, d_pad(d)), device="cuda", generator=gen) * 2 - 1).to(torch.int8)
    tables = torch.randn(k, 1 << tau, d_out, device="cuda", generator=gen)
    B.lookupffn_set_option("gather_path", 2)
    try:
        y = torch.empty(n, d_out, device="cuda", dtype=y_dtype)
        B.lookupffn_forward_probes(x, signs, tables, y=y)
        assert B.lookupffn_last_hash_kernel() == kernel
        assert B.lookupffn_last_gather_kernel() == "gather_lds_kernel"
    finally:
        B.lookupffn_set_option("gather_path", 0)
    codes, shares = B.lookupffn_hash_probes(x, signs, k, tau)
    ref = B.lookupffn_gather_probes(codes, shares, tables).double()
    size = B.lookupffn_gather_probes(codes, shares, tables.abs()).double()
    bound = (16 + 2 * k * (tau + 1)) * 2.0 ** -24 * size
    bound = bound + {torch.float32: 0.0, torch.bfloat16: 2.0 ** -8, torch.float16: 2.0 ** -11}[y_dtype] * ref.abs()
    if y_dtype is torch.float16:
        bound = bound + 2.0 ** -25  # half the smallest step of the type
    err = (y.double() - ref).abs()
    assert bool((err <= bound + 1e-30).all()), float((err / (bound + 1e-30)).max())
    np.testing.assert_allclose(y[2].float().cpu().numpy(), ref[2].float().cpu().numpy(), rtol=2.0 ** -7, atol=1e-2)
