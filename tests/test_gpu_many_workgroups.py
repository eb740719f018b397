"""Launches of more work-items than one row of a grid holds (2^32 along x): every token is still computed."""
import numpy as np
import pytest

import oracle
from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu

PERIOD = 4099   # the tokens repeat with an odd period, so a token left out or computed from another one shows


def repeated(base, reps):
    big = torch.empty((reps * base.shape[0],) + tuple(base.shape[1:]), dtype=base.dtype, device="cuda")
    big.view(reps, *base.shape).copy_(base.expand(reps, *base.shape))
    return big


@pytest.mark.parametrize("xcd", [1, -1])
def test_direct_gather(xcd):
    # a token of one 16-byte piece to each wavefront: four tokens a workgroup of 256 work-items
    reps, k, tau = (1 << 26) // PERIOD + 1, 2, 3
    print(f"direct gather of {reps * PERIOD} tokens, xcd order {xcd}", flush=True)
    tables = synth.make_tables(1, k, 1 << tau, 4)
    codes = np.random.default_rng(0).integers(0, 1 << tau, size=(PERIOD, k)).astype(np.uint16)
    cd = repeated(torch.from_numpy(codes.view(np.int16)).cuda(), reps)
    y = torch.full((reps * PERIOD, 4), float("nan"), device="cuda")
    for key, value in (("lanes_per_token", 64), ("xcd_order", xcd), ("gather_path", 1)):
        B.lookupffn_set_option(key, value)
    try:
        B.lookupffn_gather(cd, B.to_device(tables), y=y)
    finally:
        for key in ("lanes_per_token", "xcd_order", "gather_path"):
            B.lookupffn_set_option(key, 0)
    want = torch.from_numpy(oracle.gather(codes, tables, acc64=False)).cuda()
    assert bool((y.view(reps, PERIOD, 4) == want).all())


def test_forward_stack():
    # 1024 work-items to each token
    reps, d, k, tau, d_out = (1 << 22) // PERIOD + 1, 520, 2, 3, 1024
    print(f"forward_stack of {reps * PERIOD} tokens", flush=True)
    x = synth.make_x(d, PERIOD, d, "bf16")
    signs, tables = synth.make_signs(k, 1, 1, 1024), synth.make_tables(2, k, 1 << tau, d_out)
    xd = repeated(B.to_device(x), reps)
    y = torch.full((reps * PERIOD, d_out), float("nan"), dtype=torch.float32, device="cuda")
    B.lookupffn_forward_stack(xd, [B.to_device(signs)], [B.to_device(tables)], y=y)
    want = torch.from_numpy(oracle.forward(x, signs, tables, acc64=False)).cuda()
    ok = y.view(reps, PERIOD, d_out)
    assert all(bool((ok[i:i + 64] == want).all()) for i in range(0, reps, 64))
