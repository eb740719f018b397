"""The direct gather bit for bit: each output is one chain of fp32 additions (plain sum) or of fp32 fused multiply-adds
(weighted: tables in order; multi-probe: table by table, the selected row and then its neighbours) from +0."""
import numpy as np
import pytest

import oracle
from paper_2403_07221_amd import synth

torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2403_07221_amd import binding as B

pytestmark = pytest.mark.gpu


def fma32(a, b, c):
    """round(a * b + c) of float32 arrays, rounded once: the float64 sum is rounded to odd (its last bit set when it is
    inexact, after a step towards zero if it was rounded away), so that the rounding to float32 is the only one."""
    p, c = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)      # the product is exact
    s = p + c
    bb = s - p
    err = (p - (s - bb)) + (c - bb)                                                # s + err = p + c exactly
    bits = s.view(np.int64).copy()
    bits -= ((err != 0) & (np.signbit(err) != np.signbit(s)) & (s != 0)).astype(np.int64)
    bits |= (err != 0).astype(np.int64)
    return bits.view(np.float64).astype(np.float32)


def widened(tables, tdt):
    """the rows in float32, [k][rows][d_out]"""
    if tdt == "f32":
        return tables
    if tdt == "f16":
        return tables.astype(np.float32)
    return (tables.astype(np.uint32) << 16).view(np.float32)


def chain(codes, factors, rows32):
    """factors [n][k] or [n][k][1 + tau]"""
    n, k = codes.shape
    acc = np.zeros((n, rows32.shape[2]), np.float32)
    f = factors.reshape(n, k, -1)
    for j in range(k):
        for p in range(f.shape[2]):
            c = codes[:, j] ^ (0 if p == 0 else 1 << (p - 1))
            acc = fma32(f[:, j, p:p + 1], rows32[j][c], acc)
    return acc


def check(n, k, tau, d_out, tdt, prepared=False):
    rng = np.random.default_rng(n + 31 * k)
    tables = synth.make_tables(n + k, k, 1 << tau, d_out, tdt)
    codes = rng.integers(0, 1 << tau, size=(n, k)).astype(np.uint16)
    w = rng.uniform(0.1, 1.0, size=(n, k)).astype(np.float32)
    p = rng.uniform(0.0, 1.0, size=(n, k, tau + 1)).astype(np.float32)
    cd, td = torch.from_numpy(codes.view(np.int16)).cuda(), B.to_device(tables)
    wd, pd = torch.from_numpy(w).cuda(), torch.from_numpy(p).cuda()
    if prepared:
        td = B.lookupffn_prepare_tables(td)
    B.lookupffn_set_option("gather_path", 1)
    try:
        y = B.lookupffn_gather(cd, td).cpu().numpy()
        yw = B.lookupffn_gather_weighted(cd, wd, td).cpu().numpy()
        yp = B.lookupffn_gather_probes(cd, pd, td).cpu().numpy()
        assert B.lookupffn_last_gather_kernel() == "gather_kernel"
    finally:
        B.lookupffn_set_option("gather_path", 0)
    rows32 = widened(tables, tdt)
    assert np.array_equal(y, oracle.gather(codes, tables, acc64=False))
    assert np.array_equal(yw, chain(codes, w, rows32))
    pick = np.unique(np.concatenate([np.arange(0, n, max(1, n // 150)), np.arange(max(0, n - 70), n)]))
    assert np.array_equal(yp[pick], chain(codes[pick], p[pick], rows32))


# every number of tables left over beside no, one, two and three whole chunks of eight
@pytest.mark.parametrize("k", list(range(1, 8)) + list(range(9, 16)) + [18, 19, 21, 23, 25, 28, 30, 31])
@pytest.mark.parametrize("tdt,d_out", [("f32", 36), ("bf16", 40), ("f16", 72)])
def test_left_over_tables(k, tdt, d_out):
    print(f"direct chains k={k} {tdt}", flush=True)
    check(61, k, 4, d_out, tdt)


# the probe sequence: two to seventeen rows a table, one to five tables in eight rows, whole and partial last eights, less
# than eight codes, codes of the last eight reached at every place
@pytest.mark.parametrize("tau", [1, 2, 3, 7, 8, 11, 16])
@pytest.mark.parametrize("k", [1, 7, 8, 9, 12, 15, 16, 17, 23, 41])
def test_probe_sequences(k, tau):
    print(f"direct chains, probes k={k} tau={tau}", flush=True)
    check(21, min(k, 9) if tau == 16 else k, tau, 8, "f32")


# By default a token has eight lanes and a full workgroup 32 tokens; fewer than 512 full workgroups go out as one-wave
# ones, and from 1024 tokens on tables over 4 MiB in the XCD order: one wave, plain and XCD; four waves, plain and XCD
@pytest.mark.parametrize("n,k,tau,d_out,tdt", [(1030, 5, 4, 256, "f32"), (1100, 9, 9, 256, "f32"), (2817, 3, 5, 768, "f32"),
                                               (1100, 5, 9, 768, "f32"), (1100, 9, 9, 520, "bf16"), (2100, 5, 10, 1032, "f16")])
def test_default_launch_forms(n, k, tau, d_out, tdt):
    print(f"direct chains n={n} k={k} tau={tau} d_out={d_out} {tdt}", flush=True)
    check(n, k, tau, d_out, tdt)


# four rows in flight instead of sixteen: 16-bit rows, and fp32 rows of no whole number of lines, when a slice of all the
# tables is over 4 MiB and there are nine wavefronts to a compute unit (below and from there on), every number left over
@pytest.mark.parametrize("tdt,d_out,few,many", [("bf16", 776, 1400, 1500), ("f16", 1024, 1100, 1200), ("f32", 504, 1100, 1300)])
@pytest.mark.parametrize("k", [17, 18, 19, 20])
def test_four_rows_in_flight(tdt, d_out, few, many, k):
    print(f"direct chains, four rows k={k} {tdt} d_out={d_out}", flush=True)
    tables = synth.make_tables(k, k, 2048, d_out, tdt)
    codes = np.random.default_rng(k).integers(0, 2048, size=(many, k)).astype(np.uint16)
    want = oracle.gather(codes, tables, acc64=False)
    cd, td = torch.from_numpy(codes.view(np.int16)).cuda(), B.to_device(tables)
    B.lookupffn_set_option("gather_path", 1)
    try:
        for n in (few, many):
            assert np.array_equal(B.lookupffn_gather(cd[:n], td).cpu().numpy(), want[:n])
    finally:
        B.lookupffn_set_option("gather_path", 0)


# prepared tables of 512 and 1024 rows are read in pieces of four lanes (a full workgroup has 64 tokens): below and from
# 1000 tokens on, the plain and the XCD order
@pytest.mark.parametrize("n", [999, 1000, 1664])
@pytest.mark.parametrize("k,tau,d_out", [(11, 9, 264), (6, 10, 520)])
def test_prepared_pieces_in_both_orders(n, k, tau, d_out):
    print(f"direct chains, prepared n={n} k={k} tau={tau} d_out={d_out}", flush=True)
    check(n, k, tau, d_out, "f32", prepared=True)


# 2817 tokens of 50 pieces of 16 bytes are 575 to 708 full workgroups at every number of lanes: four waves each, the last one's
# tokens ragged
@pytest.mark.parametrize("lpt", [1, 2, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("xcd", [1, -1])
@pytest.mark.parametrize("tdt,d_out", [("f32", 200), ("f16", 400)])
def test_four_wave_workgroups_at_every_lane_count(lpt, xcd, tdt, d_out):
    print(f"direct chains lpt={lpt} xcd={xcd} {tdt}", flush=True)
    B.lookupffn_set_option("lanes_per_token", lpt)
    B.lookupffn_set_option("xcd_order", xcd)
    try:
        check(2817, 5, 3, d_out, tdt)
    finally:
        B.lookupffn_set_option("lanes_per_token", 0)
        B.lookupffn_set_option("xcd_order", 0)
