"""From how many tokens a forward pass stages its tables (256 compute units): a token to either side of each line, where lines
differ -- mode, tau, prepared or row-major tables, few or an odd number of them."""
import shutil

import pytest

import recorded as R

PREPARED = 0x100
CASES = [  # entry, k, tau, d_out, prepared, tokens of the line
    ("lookupffn_forward", 96, 8, 768, True, 4791), ("lookupffn_forward", 96, 8, 768, False, 4791),
    ("lookupffn_forward_weighted", 96, 8, 768, True, 4151), ("lookupffn_forward_probes", 96, 8, 768, True, 2231),
    ("lookupffn_forward", 170, 9, 768, True, 3196), ("lookupffn_forward_weighted", 128, 10, 1024, True, 3325),
    ("lookupffn_forward_probes", 64, 9, 1024, True, 2301), ("lookupffn_forward", 170, 9, 768, False, 5116),
    ("lookupffn_forward", 62, 8, 768, True, 5111), ("lookupffn_forward_weighted", 97, 8, 768, True, 5111),
    ("lookupffn_forward_probes", 24, 8, 768, True, 3191), ("lookupffn_forward_probes", 97, 8, 768, True, 3191),
    # a slice and less to a workgroup of an XCD, and two to one
    ("lookupffn_forward_weighted", 64, 8, 544, True, 4089), ("lookupffn_forward_weighted", 64, 8, 352, True, 6641), ("lookupffn_forward_weighted", 128, 8, 976, True, 3577),
    ("lookupffn_forward", 128, 8, 976, True, 4089), ("lookupffn_forward_probes", 80, 8, 584, True, 2297), ("lookupffn_forward_weighted", 64, 9, 528, True, 8185),
    ("lookupffn_forward_weighted", 64, 9, 496, True, 5113), ("lookupffn_forward_weighted", 146, 9, 592, True, 5113), ("lookupffn_forward_probes", 64, 9, 544, True, 3325),
    ("lookupffn_forward", 96, 10, 528, True, 9721), ("lookupffn_forward", 64, 10, 720, True, 8185), ("lookupffn_forward_weighted", 96, 10, 528, True, 8697),
    ("lookupffn_forward_weighted", 250, 8, 648, True, 3321), ("lookupffn_forward_probes", 96, 8, 920, True, 1785), ("lookupffn_forward", 64, 9, 560, True, 8185),
    ("lookupffn_forward", 170, 9, 296, True, 5113), ("lookupffn_forward", 128, 10, 880, True, 6649),
    ("lookupffn_forward_probes", 96, 7, 768, True, 2551), ("lookupffn_forward_probes", 24, 10, 512, True, 5625),
]


@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("entry,k,tau,d_out,prepared,line", CASES)
def test_line(tmp_path, entry, k, tau, d_out, prepared, line):
    lib = R.build(tmp_path)
    for n in (line - 1, line):
        call = [entry, R.FAKE, R.FAKE, R.FAKE, R.FAKE, n, 768, k, tau, d_out, 3, 0, PREPARED if prepared else 0, R.FAKE, 1 << 40, None]
        kernels = [launch.kernel for launch in R.record(lib, [call])[0]]
        assert ("gather_lds_kernel" in kernels) == (n == line), (n, kernels)


@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("mode,n,staged", [("plain", 5110, False), ("plain", 5111, True), ("weighted", 5110, False),
                                           ("probes", 5110, False), ("probes", 5111, True)])
def test_line_of_a_callers_codes(tmp_path, mode, n, staged):
    """Codes of the caller's: two tokens a row, and no scratch memory below that."""
    launches = R.record(R.build(tmp_path), [R.gather(mode, n, 96, 8, 768, PREPARED)])[0]
    assert [launch.kernel for launch in launches][-1] == ("gather_lds_kernel" if staged else "gather_kernel")


# A BH hash of several projections, which a direct gather's codes have spread over workgroups: as far as that holds its lines are
# others (one projection, rows of 512 and wider, and batches that fill the chip with tokens keep those above)
@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("weighted,d,k,tau,d_out,line", [
    (False, 256, 96, 8, 768, 5111), (True, 64, 96, 8, 768, 5111), (True, 512, 128, 8, 768, 4151), (False, 512, 96, 8, 768, 4791),
    (True, 512, 96, 8, 672, 4089), (True, 512, 96, 8, 704, 4089), (True, 512, 64, 8, 704, 3321),
    (False, 64, 170, 9, 768, 4476), (True, 200, 170, 9, 768, 4476), (True, 512, 170, 9, 768, 3196), (True, 128, 128, 10, 1024, 4605), (True, 512, 128, 10, 768, 4156), (True, 200, 96, 10, 768, 4156), (True, 128, 96, 10, 768, 5756),
    (True, 768, 96, 8, 768, 4151), (False, 64, 64, 8, 128, 30657), (True, 64, 64, 8, 128, 26561)])
def test_line_of_bh_codes(tmp_path, weighted, d, k, tau, d_out, line):
    lib = R.build(tmp_path)
    for n in (line - 1, line):
        call = ["lookupffn_forward_bh" + ("_weighted" if weighted else ""), R.FAKE, R.FAKE, R.FAKE, R.FAKE, n, d, k, tau, d_out, PREPARED | 16, 4, 0,
                PREPARED, R.FAKE, 1 << 40, None]
        kernels = [launch.kernel for launch in R.record(lib, [call])[0]]
        assert ("gather_lds_kernel" in kernels) == (n == line), (n, kernels)
    # the packed layout comes from the matrix cores' kernel alone, also where the batch is few enough tokens for the other
    assert "bh_hash_kernel" in kernels and "bh_lane_kernel" not in kernels


@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("k,hash_kernel", [(8, "bh_hash_kernel"), (9, "bh_lane_kernel")])
def test_hash_of_a_staged_batch_of_few_narrow_tokens(tmp_path, k, hash_kernel):
    """An even number of tables is hashed into the staged gather's layout, an odd one turned around for it."""
    call = ["lookupffn_forward_bh", R.FAKE, R.FAKE, R.FAKE, R.FAKE, 5200, 64, k, 8, 768, PREPARED | 16, 2, 0, PREPARED, R.FAKE, 1 << 40, None]
    kernels = [launch.kernel for launch in R.record(R.build(tmp_path), [call])[0]]
    assert "gather_lds_kernel" in kernels and hash_kernel in kernels


# Multi-probe with a few tables: what is turned around between the kernels (odd numbers, and all but what hash_row_kernel writes) has later lines
@pytest.mark.skipif(not shutil.which("gcc"), reason="gcc not found")
@pytest.mark.parametrize("d,k,tau,d_out,line", [
    (768, 8, 8, 768, 3191), (760, 8, 8, 768, 5111), (256, 8, 8, 768, 5111), (256, 10, 8, 768, 3831), (256, 14, 8, 768, 3831), (256, 16, 8, 768, 3191), (768, 9, 8, 768, 5111), (768, 11, 8, 768, 4471),
    (768, 13, 8, 768, 3831), (768, 17, 8, 768, 3191), (768, 12, 8, 768, 3191), (768, 8, 9, 768, 5116), (768, 10, 9, 768, 3516), (768, 11, 9, 768, 4476), (768, 13, 9, 768, 3516), (768, 4, 10, 512, 9209),
    (768, 6, 10, 512, 5625), (768, 7, 10, 512, 7161), (768, 12, 10, 512, 5625), (768, 13, 10, 512, 5625)])
def test_line_of_few_tables(tmp_path, d, k, tau, d_out, line):
    lib = R.build(tmp_path)
    for n in (line - 1, line):
        call = ["lookupffn_forward_probes", R.FAKE, R.FAKE, R.FAKE, R.FAKE, n, d, k, tau, d_out, 3, 0, PREPARED, R.FAKE, 1 << 40, None]
        kernels = [launch.kernel for launch in R.record(lib, [call])[0]]
        assert ("gather_lds_kernel" in kernels) == (n == line), (n, kernels)
