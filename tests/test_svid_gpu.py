"""GPU parity of the SVID projection (section 3.2; dbf_svid) against the oracle's svid() on the same
seeded matrices: Sign(Z) in the packed tile layout must be bit-exact (including +0.0 and -0.0 -> +1 and
zero padding bits), and the two fp32 factors of the rank-one decomposition of |Z| must agree with the
fp64 power iteration after the same number of rounds.

Tolerance: every entry of a and m is a sum of up to 4096 non-negative fp32 products followed by a
normalisation; sequential fp32 summation of n positive terms has relative error at most n * 2^-24
(2.4e-4 at n = 4096), the tree-shaped parts far less, and the errors of one round enter the next
through well-conditioned positive sums.  The gate is 2e-4 of the largest entry of each vector."""
import ctypes
import time

import numpy as np
import pytest
import torch

import gpu_util as G
from oracle import dbf_oracle as O
from paper_2505_11076_amd import binding as B
from paper_2505_11076_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 2e-4


def _parts(rows, cols):
    """Workgroups of the one launch for all rounds; 0: there is none at this size."""
    wsb = B.dbf_svid_workspace_bytes(rows, cols)
    up256 = lambda n: (n + 255) // 256 * 256   # noqa: E731
    groups = 16 * ((rows + 127) // 128)
    per, cpl = (groups + 255) // 256, (cols + 2047) // 2048
    chunks = max((rows + 63) // 64, (groups + per - 1) // per)
    least = up256(4 * rows) + up256(4 * cols) + up256(4 * chunks * cols) + up256(4 * ((cols + 31) // 32 if cols <= 8192 else (cols + 63) // 64))
    if wsb == least:
        return 0
    assert wsb == least + 2304
    if cpl == 1 and per == 5:
        per = 6
    return (groups + per - 1) // per


def _run(Z, iters, before=None, less=0, **forced):
    """a, m, sign words; with a wait or the door forced, or something to do `before`, also how many workgroups were inside (the second word of what the
    one launch keeps in the workspace's last 2304 bytes)."""
    rows, cols = Z.shape
    z = torch.from_numpy(Z.copy()).cuda()
    a = torch.full((rows,), float("nan"), dtype=torch.float32, device="cuda")
    m = torch.full((cols,), float("nan"), dtype=torch.float32, device="cuda")
    nb = B.dbf_tiled_bytes(rows, cols)
    bits = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    wsb = B.dbf_svid_workspace_bytes(rows, cols) - less
    ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    if before:
        before()
    if forced:
        p = ctypes.c_void_p
        fn = B.lib().dbf_svid_forced
        fn.argtypes = [p, ctypes.c_int, ctypes.c_int, ctypes.c_int, p, p, p, p, ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_int, p]
        assert fn(z.data_ptr(), rows, cols, iters, a.data_ptr(), m.data_ptr(), bits.data_ptr(), ws.data_ptr(), wsb,
                  forced.get("door", 256), forced.get("door_spins", 1 << 21), forced.get("spins", 1 << 21), G.stream_handle()) == 0
    else:
        B.dbf_svid(z.data_ptr(), rows, cols, iters, a.data_ptr(), m.data_ptr(), bits.data_ptr(), ws.data_ptr(), wsb,
                   G.stream_handle())
    torch.cuda.synchronize()
    words = B.dbf_untile_host(rows, cols, bits.cpu().numpy())
    out = a.cpu().numpy().astype(np.float64), m.cpu().numpy().astype(np.float64), words
    return out + (int(ws[-2304:].view(torch.int32)[1]),) if forced or before else out


@pytest.mark.parametrize("shape,iters", [(s, i) for s in [(512, 256), (100, 77), (130, 1000), (1000, 129),
                                                          (4096, 2048), (3, 5),
                                                          (300, 4100), (77, 11008), (24, 24580)]
                          for i in (1, 4)]
                         # matrices large enough for the one-pass round (1, 2, 3 and 6 float4s per thread and row,
                         # ragged last batches of rows; 24580 columns are too many for it)
                         + [((6151, 4096), 3), ((3100, 8196), 2), ((2309, 11008), 2), ((1033, 24576), 2), ((1100, 24580), 2)]
                         + [((4096, 4096), 8), ((11008, 4096), 8)])  # the last two: what bench.py times
def test_svid_matches_the_oracle(shape, iters):
    rows, cols = shape
    G.say("start svid %dx%d iters=%d" % (rows, cols, iters))
    Z = I.make_svid_matrix(rows, cols, I.seed_for(8, rows + cols))
    S, a_ref, m_ref = O.svid(Z.astype(np.float64), iters)
    a, m, words = _run(Z, iters)
    assert np.array_equal(words, O.pack_signs(S)), "sign bits differ"
    ea = np.max(np.abs(a - a_ref)) / np.max(np.abs(a_ref))
    em = np.max(np.abs(m - m_ref)) / np.max(np.abs(m_ref))
    G.say("  rel err a %.2e m %.2e (tol %.0e)" % (ea, em, TOL))
    assert ea <= TOL and em <= TOL
    assert abs(np.linalg.norm(m) - 1.0) <= 1e-5


def test_svid_reproduces_a_matrix_of_its_own_form():
    rng = np.random.default_rng(66)
    p, q = rng.uniform(0.5, 2.0, 300).astype(np.float32), rng.uniform(0.5, 2.0, 520).astype(np.float32)
    S0 = np.where(rng.random((300, 520)) < 0.5, 1.0, -1.0).astype(np.float32)
    Z = (p[:, None] * S0 * q[None, :]).astype(np.float32)
    a, m, words = _run(Z, 2)
    assert np.array_equal(words, O.pack_signs(S0.astype(np.float64)))
    back = a[:, None] * S0.astype(np.float64) * m[None, :]
    assert np.max(np.abs(back - Z.astype(np.float64))) <= 1e-5 * np.max(np.abs(Z))


def test_svid_argument_errors():
    z = torch.zeros((4, 4), dtype=torch.float32, device="cuda")
    a = torch.zeros(4, dtype=torch.float32, device="cuda")
    bits = torch.zeros(B.dbf_tiled_bytes(4, 4), dtype=torch.uint8, device="cuda")
    wsb = B.dbf_svid_workspace_bytes(4, 4)
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    assert B.dbf_svid_workspace_bytes(0, 4) == 0
    ok = (z.data_ptr(), 4, 4, 1, a.data_ptr(), a.data_ptr(), bits.data_ptr(), ws.data_ptr(), wsb, 0)
    for pos, val in ((0, 0), (1, 0), (3, 0), (4, 0), (6, 0), (7, 0), (8, wsb - 1), (7, ws.data_ptr() + 4)):
        bad = list(ok)
        bad[pos] = val
        with pytest.raises(B.DbfError):
            B.dbf_svid(*bad)


@pytest.mark.parametrize("rows,cols", [(5, 7), (17, 1020), (129, 1023), (128, 1028), (255, 2047), (4200, 2052), (2049, 4095), (257, 4097), (130, 8188),
                                       (131, 8194), (70, 12285), (66, 12290), (40, 16380), (33, 20484)])
def test_svid_one_pass_rounds_at_the_edges_of_their_row_lengths(rows, cols):
    """A round in one pass over the matrix: 4, 8 and 16 wavefronts per workgroup, 1 to 6 float4s per thread and row, rows that can be read in
    16-byte pieces and rows that cannot (12285 columns are the last few of those), groups of rows that hang over the end, several
    groups per workgroup.  Tolerance: as above."""
    Z = I.make_svid_matrix(rows, cols, I.seed_for(8, 40 + rows + cols))
    for iters in (1, 3):
        G.say("start svid %dx%d iters=%d" % (rows, cols, iters))
        S, a_ref, m_ref = O.svid(Z.astype(np.float64), iters)
        a, m, words = _run(Z, iters)
        assert np.array_equal(words, O.pack_signs(S)), "sign bits differ"
        assert np.max(np.abs(a - a_ref)) <= TOL * np.max(np.abs(a_ref))
        assert np.max(np.abs(m - m_ref)) <= TOL * np.max(np.abs(m_ref))


@pytest.mark.parametrize("rows,cols", [(1, 31), (1023, 32), (1025, 33), (4097, 8192), (260, 8193), (4100, 95), (2, 1030)])
def test_svid_at_the_edges_of_its_reductions(rows, cols):
    """32 or 64 columns to a workgroup of the column reduction (8192 columns and less, more), 1024 entries of either factor to a workgroup of the last
    kernel, which takes the rows' lengths 4096 at a time.  Tolerance: as above."""
    Z = I.make_svid_matrix(rows, cols, I.seed_for(8, 80 + rows + cols))
    for iters in (1, 2, 5):
        G.say("start svid %dx%d iters=%d" % (rows, cols, iters))
        S, a_ref, m_ref = O.svid(Z.astype(np.float64), iters)
        a, m, words = _run(Z, iters)
        assert np.array_equal(words, O.pack_signs(S)), "sign bits differ"
        assert np.max(np.abs(a - a_ref)) <= TOL * np.max(np.abs(a_ref))
        assert np.max(np.abs(m - m_ref)) <= TOL * np.max(np.abs(m_ref))


@pytest.mark.parametrize("rows,cols", [(128, 512), (2049, 2052), (4096, 2048), (6000, 1000), (8000, 900), (12000, 260), (5000, 4096), (2000, 6140),
                                       (4000, 5000), (1000, 8192), (1500, 10240), (300, 12288)])
def test_svid_rounds_in_one_launch(rows, cols):
    """Six rounds and more: Z in registers, 1 to 5 float4s per thread and row, 8 to 48 rows per workgroup, 16, 32 and 64 columns added up at a time, rows too long for
    it.  With a door that lets only some of the workgroups in, these take over the others' rows: the same bits.  Tolerance: as above."""
    Z = I.make_svid_matrix(rows, cols, I.seed_for(8, 120 + rows + cols))
    for iters in (6, 7):
        G.say("start svid %dx%d iters=%d" % (rows, cols, iters))
        S, a_ref, m_ref = O.svid(Z.astype(np.float64), iters)
        a, m, words = _run(Z, iters)
        assert np.array_equal(words, O.pack_signs(S)), "sign bits differ"
        assert np.max(np.abs(a - a_ref)) <= TOL * np.max(np.abs(a_ref))
        assert np.max(np.abs(m - m_ref)) <= TOL * np.max(np.abs(m_ref))
        parts = _parts(rows, cols)
        assert (parts == 0) == (cols == 12288)
        for door in [n for n in (1, 3, 60, parts - 1) if 0 < n < parts]:
            G.say("  %d of %d workgroups inside" % (door, parts))
            a0, m0, words0, inside = _run(Z, iters, door=door)
            assert inside == door
            assert np.array_equal(a, a0) and np.array_equal(m, m0) and np.array_equal(words, words0)


@pytest.mark.parametrize("rows,cols", [(768, 1024), (4096, 3076)])
@pytest.mark.parametrize("entry", [float("nan"), float("inf"), 0.0, 1e19, 3e-23])
def test_svid_gives_the_same_outside_the_numbers_whatever_the_launches(rows, cols, entry):
    """NaN is not supported, but the factors must not depend on how many rounds there are, or on whether these are one launch or, with the
    workspace's last 2304 bytes left out, a launch each: one entry that is no number or infinite makes a zero and m no numbers; a zero matrix gives zeros; and so on where the
    squares leave the range.  Tolerance for what are numbers: as above."""
    Z = I.make_svid_matrix(rows, cols, I.seed_for(8, 175 + rows))
    if entry == entry and entry < 1e38:
        Z = (Z * entry).astype(np.float32)
    else:
        Z[rows // 2, cols // 3] = entry
    for iters in (2, 3, 6):
        G.say("start svid %dx%d %g iters=%d" % (rows, cols, entry, iters))
        a, m, words = _run(Z, iters)
        a1, m1, words1 = _run(Z, iters, less=2304)
        assert np.array_equal(words, words1)
        for x, y in ((a, a1), (m, m1)):
            G.say("  %d no numbers, %d zeros of %d" % (np.sum(np.isnan(x)), np.sum(x == 0), x.size))
            assert np.allclose(x, y, rtol=TOL, atol=0, equal_nan=True)
        if entry != entry or entry > 1e38:
            assert np.all(a == 0) and np.all(np.isnan(m))


def test_svid_waits_for_workgroups_that_a_busy_device_lets_in_late():
    """248 compute units are busy with another stream's projection, for some 600 us, when a projection of 256 workgroups starts: the eight that find a
    place would take a millisecond for everyone's rows, so they wait for the others, and all are inside in the end.  (Had they gone on alone, the bits would be
    the same.)"""
    rows, cols, iters, busy_rows = 4096, 4096, 8, 3968
    Z = I.make_svid_matrix(rows, cols, I.seed_for(8, 170))
    a_ref, m_ref, words_ref = _run(Z, iters)
    z = torch.from_numpy(Z[:busy_rows].copy()).cuda()
    f = lambda n: torch.empty(n, dtype=torch.float32, device="cuda")   # noqa: E731
    a, m, ws = f(busy_rows), f(cols), torch.empty(B.dbf_svid_workspace_bytes(busy_rows, cols), dtype=torch.uint8, device="cuda")
    bits = torch.empty(B.dbf_tiled_bytes(busy_rows, cols), dtype=torch.uint8, device="cuda")
    assert _parts(busy_rows, cols) == 248 and _parts(rows, cols) == 256
    busy = torch.cuda.Stream()
    G.say("start svid beside a busy device")

    def occupy():
        B.dbf_svid(z.data_ptr(), busy_rows, cols, 80, a.data_ptr(), m.data_ptr(), bits.data_ptr(), ws.data_ptr(), ws.numel(), busy.cuda_stream)
        time.sleep(2e-4)   # (until it has its places)

    a0, m0, words0, inside = _run(Z, iters, before=occupy)
    G.say("  %d of 256 workgroups inside" % inside)
    assert np.array_equal(a_ref, a0) and np.array_equal(m_ref, m0) and np.array_equal(words_ref, words0)
    assert inside == 256


@pytest.mark.parametrize("rows,cols", [(768, 512), (2049, 2052), (1500, 10240)])
def test_svid_waits_that_run_out_leave_no_wrong_numbers(rows, cols):
    """All rounds in one launch with a wait of the workgroups, for all to be in or for each other's sums, cut to a few polls (they are seconds long): what was
    not waited for must not pass for a number.  Every entry of the product of the two factors is right, to the bit, or no number; with no polls at all none is
    right."""
    Z = I.make_svid_matrix(rows, cols, I.seed_for(8, 160 + rows + cols))
    a_ref, m_ref, _ = _run(Z, 6)
    want = a_ref[:, None] * m_ref[None, :]
    for wait in ("door_spins", "spins"):
        for polls in (0, 1, 2, 3, 4, 6, 8, 12, 16, 64):
            G.say("start svid %dx%d, %s %d" % (rows, cols, wait, polls))
            a, m, _, _ = _run(Z, 6, **{wait: polls})
            got = a[:, None] * m[None, :]
            none = np.isnan(got)
            G.say("  %.3f of the entries are no numbers" % np.mean(none))
            assert np.all(none | (got == want))
            assert polls > 0 or np.all(none)
