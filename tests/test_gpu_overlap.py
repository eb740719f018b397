"""lookupffn_forward with y over x.  Hash and gather as two launches read all of x before y is written; one launch may
only do it in place with rows of the same length, so every other overlap has to be the two-launch route."""
import numpy as np
import pytest

import oracle
from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu

ONE_LAUNCH = ("forward_small_kernel", "forward_stack_kernel")


# first byte of y after the first byte of x; one launch allowed
@pytest.mark.parametrize("n,d,d_out,xdt,ydt,shift,one", [
    (256, 64, 64, "f32", "f32", 0, True),       # in place, rows of one length
    (256, 64, 128, "f16", "f16", 0, False),     # rows of y twice as long: token t's store covers rows 2t, 2t + 1 of x
    (256, 64, 32, "f32", "f32", 0, False),      # half as long
    (200, 512, 512, "f32", "f32", 2048, False),  # rows of one length, one row on
    (200, 512, 512, "f32", "f32", -2048, False),
    (100, 96, 64, "f32", "f32", 100 * 96 * 4 - 16, False),  # the last 16 bytes of x
    (100, 96, 64, "f32", "f32", 100 * 96 * 4, True),        # just past x
    (100, 96, 64, "f32", "f32", -100 * 64 * 4, True),       # ends where x starts
    (128, 64, 64, "bf16", "f32", 0, False),     # same number of columns, other types
    (100, 1024, 1024, "f32", "f32", 0, True),   # the d_pad = 1024 kernel
    (100, 1024, 512, "f32", "f32", 0, False),
    (257, 1024, 1024, "f32", "f32", 0, True),   # two tokens to a workgroup, the last one alone
    (512, 1024, 1024, "f32", "f32", 0, True),
    (511, 1024, 512, "f16", "f32", 0, True),    # rows of one length in bytes
    (257, 1024, 1024, "f32", "f32", 4096, False),
])
def test_forward_over_its_own_input(n, d, d_out, xdt, ydt, shift, one):
    print(f"overlap n={n} d={d} d_out={d_out} {xdt} -> {ydt} y at x{shift:+d}", flush=True)
    k, tau, rounds = 16, 8, 3
    d_pad = 64
    while d_pad < d:
        d_pad *= 2
    x = synth.make_x(n + d, n, d, xdt)
    signs = synth.make_signs(d, -(-k * tau // d_pad), rounds, d_pad)
    tables = synth.make_tables(d_out, k, 1 << tau, d_out)
    xd, sd, td = B.to_device(x), B.to_device(signs), B.to_device(tables)
    ydtype = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[ydt]
    y_bytes = n * d_out * (4 if ydt == "f32" else 2)
    x_bytes = xd.numel() * xd.element_size()
    apart = torch.empty((n, d_out), dtype=ydtype, device="cuda")
    ws = torch.empty(B.lookupffn_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
    B.lookupffn_forward(xd, sd, td, y=apart, workspace=ws)
    if ydt == "f32":
        assert np.array_equal(apart.cpu().numpy(), oracle.forward(x, signs, tables, acc64=False))
    x_at, y_at = max(0, -shift), max(0, shift)
    buf = torch.zeros(max(x_at + x_bytes, y_at + y_bytes), dtype=torch.uint8, device="cuda")
    buf[x_at:x_at + x_bytes] = xd.view(torch.uint8).flatten()
    x_in = buf[x_at:x_at + x_bytes].view(xd.dtype).view(n, d)
    y_out = buf[y_at:y_at + y_bytes].view(ydtype).view(n, d_out)
    B.lookupffn_forward(x_in, sd, td, y=y_out, workspace=ws)
    torch.cuda.synchronize()
    assert (B.lookupffn_last_gather_kernel() in ONE_LAUNCH) == one
    assert torch.equal(y_out.view(torch.uint8), apart.view(torch.uint8))
