"""The single launch of a few tokens where its parts begin and end: numbers of tables around the four rows of a fetch and the fetches
in flight, rows that end inside a wave's 64 dwords and rows longer than a workgroup, every number of rounds and several
projections (tables across them), code lengths from 1 to 16, one token and two to a workgroup with one left over.  Against
the two kernels ("small_tokens" -1), which the other tests hold to the oracle: same bits.
"""
import pytest

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu

CASES = [  # n, d, k, tau, d_out, rounds, x dtype, table dtype, prepared
    *[(3, 768, k, 8, 192, 3, "float32", "float32", True) for k in (1, 3, 4, 5, 8, 15, 16, 17, 31, 32, 33, 48, 64, 65)],
    (1, 513, 100, 9, 68, 1, "float32", "float32", True), (2, 1024, 130, 9, 64, 2, "bfloat16", "float32", False),
    (5, 1000, 300, 11, 8, 1, "float16", "float32", False), (4, 640, 97, 7, 648, 4, "float32", "float16", False),
    (1, 900, 40, 16, 8, 2, "float32", "bfloat16", False), (2, 700, 2100, 1, 20, 1, "float32", "float32", False),
    (2, 1024, 128, 10, 1024, 3, "float32", "float32", True), (2, 768, 24, 5, 4352, 3, "float32", "float32", True),
    (3, 768, 24, 5, 4360, 3, "float32", "bfloat16", False), (257, 768, 96, 8, 132, 3, "float32", "float32", True),
    (300, 1024, 17, 8, 1032, 4, "float16", "float16", False), (511, 515, 60, 9, 64, 2, "float32", "float32", True), (555, 768, 33, 8, 520, 3, "float32", "float32", True),
    (16, 100, 33, 9, 200, 3, "float32", "bfloat16", False), (9, 512, 100, 8, 1100, 3, "float32", "float32", True),
]


@pytest.mark.parametrize("n,d,k,tau,d_out,R,xdt,tdt,prepared", CASES)
def test_one_launch_equals_two(n, d, k, tau, d_out, R, xdt, tdt, prepared):
    print(f"stack lanes n={n} d={d} k={k} tau={tau} d_out={d_out} R={R} {xdt} {tdt} {prepared}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + d + k)
    d_pad = 1 << (d - 1).bit_length()
    x = torch.randn(n, d, generator=g, device="cuda").to(getattr(torch, xdt))
    signs = torch.randint(0, 2, (-(-k * tau // d_pad), R, d_pad), generator=g, device="cuda", dtype=torch.int8) * 2 - 1
    tables = torch.randn(k, 1 << tau, d_out, generator=g, device="cuda").to(getattr(torch, tdt))
    tables = B.lookupffn_prepare_tables(tables) if prepared else tables
    out = []
    try:
        for y_dtype in (torch.float32, torch.bfloat16, torch.float16):
            for option in (1024, -1):
                B.lookupffn_set_option("small_tokens", option)
                out.append(B.lookupffn_forward(x, signs, tables, y=torch.empty(n, d_out, dtype=y_dtype, device="cuda")))
                if option == 1024:
                    assert B.lookupffn_last_hash_kernel() == ("forward_stack_kernel" if d > 512 else "forward_small_kernel")
            assert torch.equal(out[-2], out[-1])
    finally:
        B.lookupffn_set_option("small_tokens", 0)


@pytest.mark.parametrize("n", [1, 257, 512, 513, 768, 769])
@pytest.mark.parametrize("d,k,tau,R,tdt", [(768, 33, 8, 3, "float32"), (520, 170, 9, 1, "float16"), (1024, 230, 9, 4, "float32")])
def test_chain_equals_its_layers(n, d, k, tau, R, tdt):
    g = torch.Generator(device="cuda").manual_seed(n + d)
    x = torch.randn(n, d, generator=g, device="cuda")
    signs = [torch.randint(0, 2, (-(-k * tau // 1024), R, 1024), generator=g, device="cuda", dtype=torch.int8) * 2 - 1 for _ in range(3)]
    tables = [(torch.randn(k, 1 << tau, d, generator=g, device="cuda") / k ** 0.5).to(getattr(torch, tdt)) for _ in range(3)]
    y = B.lookupffn_forward_stack(x, signs, tables)
    B.lookupffn_set_option("small_tokens", -1)
    try:
        for s, t in zip(signs, tables):
            x = B.lookupffn_forward(x, s, t)
    finally:
        B.lookupffn_set_option("small_tokens", 0)
    assert torch.equal(x, y)
