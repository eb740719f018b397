"""Which kernels the library launches for a call, and with what extents: the dispatch rules and the kernels' 32-bit limits at the
sizes where they change, recorded on the CPU (tests/recorded.py; no GPU and no memory is needed, whatever the batch).
"""
import shutil

import pytest

import recorded as R

pytestmark = pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
PREPARED = 0x100


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    return R.build(tmp_path_factory.mktemp("recorder"))


# Multi-probe: a lane without a table takes its share from byte offset 2^31 of a buffer that must end before it.  The buffer holds
# the (1 + tau) rows of n_pad shares between the two tables a wavefront reads, and a window of up to 16 KB.
WINDOW = 16 * 1024


@pytest.mark.parametrize("tau,n", [(7, 67104513), (7, 67104640), (8, 59648001), (8, 59648128), (9, 53682561), (9, 53682944),
                                   (10, 48800000), (8, 59647500), (8, 59648129), (8, 1 << 27), (7, (1 << 25) + 1), (7, 1 << 25)])
def test_multi_probe_shares_end_before_the_offset_of_a_lane_without_a_table(recorder, tau, n):
    (launches,) = R.record(recorder, [R.gather("probes", n, 2, tau, 64, PREPARED)])
    tokens = 0
    for launch in launches:
        if launch.kernel == "gather_lds_kernel":
            a = launch.args(R.GatherLdsArgs)
            assert (1 + tau) * a.n_pad * 4 + WINDOW <= 1 << 31
            assert a.y == R.FAKE + tokens * 64 * 4
            tokens += a.n
    assert tokens == n and not any(launch.kernel == "gather_kernel" for launch in launches)


def test_multi_probe_batch_in_pieces(recorder):
    """Each piece has its own codes, shares and rows of y, and the scratch of one piece."""
    n, k, tau, d_out = (1 << 26) + 5, 4, 8, 32
    (launches,) = R.record(recorder, [R.gather("probes", n, k, tau, d_out, PREPARED)])
    codes, shares, staged = [[x for x in launches if x.kernel == name]
                             for name in ("repack_codes_kernel", "repack_shares_kernel", "gather_lds_kernel")]
    assert len(codes) == len(shares) == len(staged) == 3 and len(launches) == 9
    start = 0
    for c, w, s in zip(codes, shares, staged):
        a = s.args(R.GatherLdsArgs)
        assert c.pointers(2) == (R.FAKE + start * k * 2, a.packed)
        assert w.pointers(2) == (R.FAKE + start * k * (1 + tau) * 4, a.wpk)
        assert a.packed == staged[0].args(R.GatherLdsArgs).packed and a.wpk == staged[0].args(R.GatherLdsArgs).wpk
        assert a.y == R.FAKE + start * d_out * 4
        start += a.n
    assert start == n


@pytest.mark.parametrize("mode", ["plain", "weighted", "probes"])
@pytest.mark.parametrize("tau,d_out,staged", [(8, 1 << 21, True), (8, (1 << 22) - 4, True), (8, 1 << 22, False), (9, 1 << 20, True),
                                              (10, (1 << 20) - 4, True), (10, 1 << 20, False)])
def test_wide_tables(recorder, mode, tau, d_out, staged):
    """The staged kernel's offsets are 32-bit inside one table; two of them may be larger."""
    launches = R.record(recorder, [R.gather(mode, 4096, 2, tau, d_out)])[0]
    assert launches[-1].kernel == ("gather_lds_kernel" if staged else "gather_kernel")
