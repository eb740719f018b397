"""Which kernels the library launches for a call, and with what extents: the dispatch rules and the kernels' 32-bit limits at the
sizes where they change, recorded on the CPU (tests/recorded.py; no GPU and no memory is needed, whatever the batch).
"""
import shutil

import pytest

import recorded as R
import staged_forms as forms
import test_gpu_direct_deep as deep_tests

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


def hash_call(mode, n, d, k, tau, rounds=3, x_dtype=0):
    name = "lookupffn_hash" + {"plain": "", "weighted": "_weighted", "probes": "_probes"}[mode]
    return [name, *[R.FAKE] * (3 if mode == "plain" else 4), n, d, k, tau, rounds, x_dtype, None]


def hash_bh_call(mode, n, d, k, tau, block, factors=4):
    name = "lookupffn_hash_bh" + ("_weighted" if mode == "weighted" else "")
    return [name, *[R.FAKE] * (4 if mode == "weighted" else 3), n, d, k, tau, PREPARED | block, factors, 0, None, 0, None]


# Projections of few tokens go out over workgroups; every other call takes the form without their bounds, which is the faster one.
# Tables that run over from one projection into the next (their tau does not divide d_pad) take two projections to a workgroup.
@pytest.mark.parametrize("mode", ["plain", "weighted", "probes"])
@pytest.mark.parametrize("n,d,k,tau,groups", [(1, 64, 7, 9, 1), (1, 64, 8, 8, 1), (1, 64, 9, 8, 2), (1, 64, 14, 9, 1), (1, 64, 15, 9, 3),
                                              (200, 512, 60, 8, 1), (200, 512, 170, 8, 3), (700, 512, 170, 8, 2),
                                              (2000, 512, 170, 8, 1), (1, 1024, 128, 8, 1), (1, 768, 170, 9, 1), (3, 1024, 256, 10, 3),
                                              (13, 1000, 300, 11, 4), (13, 2048, 500, 13, 4)])
def test_projections_of_few_tokens(recorder, mode, n, d, k, tau, groups):
    ((launch,),) = R.record(recorder, [hash_call(mode, n, d, k, tau)])
    assert launch.kernel == ("hash1024_kernel" if 512 < d <= 1024 else "hash_kernel")
    assert launch.grid[1] == groups and launch.params[-1] == (groups > 1)


@pytest.mark.parametrize("mode", ["plain", "weighted"])
@pytest.mark.parametrize("n,d,k,tau,block,groups,few", [
    (1, 64, 8, 8, 16, 1, 0), (1, 64, 20, 8, 16, 3, 0), (1, 64, 20, 9, 16, 3, 0), (20, 145, 12, 8, 32, 1, 0),
    (2000, 256, 96, 8, 64, 3, 0), (16384, 256, 96, 8, 64, 1, 0), (1, 768, 170, 9, 64, 1, 1), (19, 1000, 228, 9, 64, 3, 1), (19, 1024, 256, 16, 64, 4, 1), (128, 1024, 256, 16, 64, 4, 1),
    (1000, 1024, 256, 16, 64, 4, 1), (1100, 1024, 256, 16, 64, 2, 1), (4096, 1024, 96, 8, 64, 1, 1), (4097, 1024, 96, 8, 64, 1, 0)])
def test_bh_projections_of_few_tokens(recorder, mode, n, d, k, tau, block, groups, few):
    ((launch,),) = R.record(recorder, [hash_bh_call(mode, n, d, k, tau, block)])
    assert launch.kernel == "bh_hash_kernel" and launch.grid[2] == groups
    assert launch.params[-2:] == (few, groups > 1)


@pytest.mark.parametrize("block,bounds", [(16, 1), (32, 1), (64, 0)])
def test_bh_weights_in_registers_keep_the_form_with_bounds(recorder, block, bounds):
    ((launch,),) = R.record(recorder, [hash_bh_call("weighted", 16384, 1024, 96, 8, block)])
    assert launch.grid[2] == 1 and launch.params[-2:] == (0, bounds)


# The direct gather's deep form: both sides of each line of its rule (256 compute units; row types fp32, bf16, half)
@pytest.mark.parametrize("mode,n,k,d_out,table,deep", [
    ("weighted", 5, 47, 768, 0, 0), ("weighted", 5, 48, 768, 0, 16), ("weighted", 1, 48, 768, 0, 16), ("weighted", 1, 47, 768, 2, 0),
    ("weighted", 1, 48, 768, 2, 16), ("weighted", 1, 48, 768, 1, 16), ("weighted", 424, 48, 768, 0, 16), ("weighted", 425, 48, 768, 0, 8),
    ("weighted", 592, 48, 768, 0, 8), ("weighted", 593, 48, 768, 0, 0), ("weighted", 848, 48, 768, 2, 16), ("weighted", 849, 48, 768, 2, 8),
    ("weighted", 1360, 48, 768, 2, 8), ("weighted", 1361, 48, 768, 2, 0), ("weighted", 64, 48, 8, 2, 0),
    ("plain", 64, 95, 768, 0, 0), ("plain", 64, 96, 768, 0, 16), ("plain", 1, 96, 64, 0, 16), ("plain", 424, 96, 768, 0, 16),
    ("plain", 425, 96, 768, 0, 0), ("plain", 64, 170, 768, 2, 0), ("plain", 64, 170, 768, 1, 0), ("probes", 64, 170, 768, 0, 0)])
def test_deep_direct_gather(recorder, mode, n, k, d_out, table, deep):
    launch = R.record(recorder, [R.option("gather_path", 1), R.gather(mode, n, k, 8, d_out, table)])[1][0]
    assert launch.kernel == "gather_kernel" and launch.params[0] == table and launch.params[3] == deep


MODE = {"plain": 0, "weighted": 1, "probes": 2}


@pytest.mark.parametrize("tau,lanes", forms.WIDTHS)
def test_staged_forms_take_their_slots(recorder, tau, lanes):
    """The batches of the GPU tests of the staged gather's forms (staged_forms.py): slots, copy rounds, mode, lanes."""
    cases = [(mode, slots) for t, w, slots in forms.RANGES if (t, w) == (tau, lanes) for mode in MODE
             if mode != "probes" or forms.has_probes(tau, lanes)]
    calls = [R.option("gather_path", 2), R.option("slice_lanes", lanes)]
    for mode, slots in cases:
        calls += [R.option("token_slots", slots), R.gather(mode, forms.tokens(lanes, slots), forms.TABLES, tau, forms.width(lanes),
                                                           0 if (tau, lanes) == (9, 8) else PREPARED)]
    for (mode, slots), launches in zip(cases, R.record(recorder, calls)[3::2]):
        staged = [x for x in launches if x.kernel == "gather_lds_kernel"]
        assert [x.params for x in staged] == [(slots, (1 << tau) // (1024 // lanes), MODE[mode], lanes)]
        assert staged[0].args(R.GatherLdsArgs).unit_chunks == 0


def test_staged_forms_divide_whole_chunks(recorder):
    for d_out, tau, n, allowed, slots in forms.CHUNKS:
        for mode in ("plain", "weighted"):
            calls = [R.option("gather_path", 2), R.option("token_slots", allowed), R.gather(mode, n, 4, tau, d_out, PREPARED)]
            (launch,) = [x for x in R.record(recorder, calls)[2] if x.kernel == "gather_lds_kernel"]
            assert launch.params[0] == slots and launch.args(R.GatherLdsArgs).unit_chunks > 0, (d_out, tau, n)


def test_deep_direct_gather_tests_take_the_deep_form(recorder):
    kind = {"f32": 0, "bf16": 1, "f16": 2}
    calls = [R.option("gather_path", 1)] + [R.gather("weighted", n, k, tau, d_out, kind[t] | (PREPARED if prep else 0))
                                            for n, tau, d_out, t, prep in deep_tests.SHAPES for k in deep_tests.KS]
    depths = [launches[0].params[3] for launches in R.record(recorder, calls)[1:]]
    assert set(depths) == {8, 16}


# 256 compute units hold a workgroup of two tokens each: what is left over from whole rounds takes a token to a workgroup where one round
# holds them.
@pytest.mark.parametrize("n,tokens,groups", [(256, 1, 256), (257, 2, 129), (512, 2, 256), (513, 2, 257), (558, 2, 302), (768, 2, 512), (769, 2, 385),
                                             (1023, 2, 512), (1024, 2, 512), (1108, 2, 596), (1281, 2, 641)])
def test_groups_of_the_single_launch(recorder, n, tokens, groups):
    call = ["lookupffn_forward", R.FAKE, R.FAKE << 1, R.FAKE << 2, R.FAKE << 3, n, 768, 96, 8, 768, 3, 0, 0, R.FAKE, 1 << 40, None]
    (launch,) = R.record(recorder, [["lookupffn_set_option", "small_tokens", 4096], call])[-1]
    assert (launch.kernel, launch.params[2], launch.grid, launch.block) == ("forward_stack_kernel", tokens, (groups, 1, 1), 1024)
