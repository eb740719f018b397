"""Plain forward of small batches with rows of d_pad 64 .. 512 in one launch (forward_small_kernel): bit-equal to the
oracle's sequential fp32 sum and to the two-kernel route."""
import numpy as np
import pytest
import torch

import oracle
from paper_2403_07221_amd import binding as B
from paper_2403_07221_amd import synth

pytestmark = pytest.mark.gpu

# n, d, k, tau, d_out, rounds: one register per lane (d_pad 64) to eight (512); one projection, more projections than
# the row's waves, more than sixteen (a wave then takes several); k not a multiple of a fetch chunk and one past it; codes
# across words and projections; ragged last slice, rows wider than 1024 dwords; more rounds than the wider kernel takes
SHAPES = [
    (1, 33, 1, 1, 8, 1),
    (64, 64, 8, 8, 64, 2),
    (5, 64, 33, 16, 8, 3),
    (3, 60, 256, 8, 40, 2),
    (7, 100, 31, 7, 648, 5),
    (9, 256, 97, 9, 1032, 3),
    (2, 300, 64, 11, 264, 4),
    (512, 512, 256, 8, 72, 3),
]


@pytest.mark.parametrize("n,d,k,tau,d_out,rounds", SHAPES)
@pytest.mark.parametrize("xdt,tdt", [("f32", "f32"), ("bf16", "bf16"), ("f16", "f16")])
def test_small_batches_in_one_launch(n, d, k, tau, d_out, rounds, xdt, tdt):
    print(f"small launch n={n} d={d} k={k} tau={tau} d_out={d_out} R={rounds} {xdt} {tdt}", flush=True)
    N = 64
    while N < d:
        N *= 2
    x = synth.make_x(n + d, n, d, xdt)
    signs = synth.make_signs(k, -(-k * tau // N), rounds, N)
    tables = synth.make_tables(n + k, k, 1 << tau, d_out, tdt)
    want = oracle.forward(x, signs, tables, acc64=False)
    xd, sd, td = B.to_device(x), B.to_device(signs), B.to_device(tables)
    for tab in (td, B.lookupffn_prepare_tables(td)):
        y = B.lookupffn_forward(xd, sd, tab)
        torch.cuda.synchronize()
        assert B.lookupffn_last_gather_kernel() == "forward_small_kernel"
        assert np.array_equal(y.cpu().numpy(), want)
    try:
        B.lookupffn_set_option("small_tokens", -1)
        y = B.lookupffn_forward(xd, sd, td)
        assert B.lookupffn_last_gather_kernel() != "forward_small_kernel"
        assert np.array_equal(y.cpu().numpy(), want)
    finally:
        B.lookupffn_set_option("small_tokens", 0)
