"""The kernel counters time the launches a call makes without them: turning them on changes no route."""
import numpy as np
import pytest

from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu


# d, small_tokens, launches counted as (hash, gather) by a call: the narrow and the wide single launch, the two kernels
@pytest.mark.parametrize("d,small,counts", [(64, 0, (1, 1)), (512, 0, (1, 1)), (768, 0, (0, 1)), (64, -1, (1, 1)),
                                            (768, -1, (1, 1))])
def test_timing_keeps_the_route(d, small, counts):
    print(f"timing route d={d} small_tokens={small}", flush=True)
    n, k, tau = 33, 8, 8
    d_pad = 64
    while d_pad < d:
        d_pad *= 2
    xd, td = B.to_device(synth.make_x(d, n, d)), B.to_device(synth.make_tables(d, k, 1 << tau, 64))
    sd = B.to_device(synth.make_signs(d, -(-k * tau // d_pad), 3, d_pad))
    B.lookupffn_set_option("small_tokens", small)
    try:
        want = B.lookupffn_forward(xd, sd, td)
        route = B.lookupffn_last_hash_kernel(), B.lookupffn_last_gather_kernel()
        for mask in (1, 2, 3):
            B.lookupffn_timing_reset()
            B.lookupffn_timing_enable(mask)
            for _ in range(3):
                y = B.lookupffn_forward(xd, sd, td)
            assert (B.lookupffn_last_hash_kernel(), B.lookupffn_last_gather_kernel()) == route
            for which in (0, 1):
                ms, launches = B.lookupffn_timing_read(which)
                assert launches == (3 * counts[which] if mask >> which & 1 else 0)
                assert (ms > 0) == (launches > 0)
            assert np.array_equal(y.cpu().numpy(), want.cpu().numpy())
    finally:
        B.lookupffn_timing_enable(0)
        B.lookupffn_timing_reset()
        B.lookupffn_set_option("small_tokens", 0)
