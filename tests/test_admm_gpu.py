"""GPU parity of one ADMM update (section 3.2; dbf_admm_step) against the oracle's admm_step_from() on
the same seeded operands.  The two constant matrices Minv = (B^T B + rho I)^-1 and C = B^T W are formed
here with numpy in fp64 and rounded to fp32; both sides start from those fp32 values.

What is compared, and why these gates:
  * Z = W_hat + U is not an output, but the outputs determine it: U' + a' . S' . m'^T = Z up to fp32
    rounding of the last subtraction.  That sum is compared with the oracle's Z.  Each entry of Z is an
    fp32 sum of q <= 2048 products on the matrix cores: error bound q * 2^-24 * sum|terms|, typically
    sqrt(q) * 2^-24 of the row's scale, i.e. 1e-6 .. 1e-5 of rms(Z).  Gate: 1e-4 of rms(Z).
  * the signs S' are those of the oracle's Z wherever |Z| exceeds that gate (closer to zero either sign
    is right: the decision is taken on a value that differs by rounding; the first check covers them);
  * a', m' as in the SVID test: 2e-4 of the largest entry, plus the gate on Z;
  * U' against the oracle where the signs are decided: U' = Z - a' m' s, so 5e-4 of max(a') max(m').
"""
import numpy as np
import pytest
import torch

import gpu_util as G
from oracle import dbf_oracle as O
from paper_2505_11076_amd import binding as B
from paper_2505_11076_amd import inputs as I

pytestmark = pytest.mark.gpu

Z_GATE = 1e-4
VEC_TOL = 2e-4 + Z_GATE
U_TOL = 5e-4


def _constants(Bm, W, rho):
    B64, W64 = Bm.astype(np.float64), W.astype(np.float64)
    Minv = np.linalg.inv(B64.T @ B64 + rho * np.eye(B64.shape[1]))
    return Minv.astype(np.float32), (B64.T @ W64).astype(np.float32)


class DeviceState:
    """The iterate (a, m, packed S, U) on the device, plus the constants and the workspace."""

    def __init__(self, Minv, C, S, a, m, U):
        self.q, self.r = C.shape
        # the library applies its first operand transposed (it reads it by rows of the summation index), so it
        # is handed the transpose of what the oracle multiplies from the left
        self.Minv = torch.from_numpy(np.ascontiguousarray(Minv.T)).cuda()
        self.C = torch.from_numpy(C.copy()).cuda()
        self.a = torch.from_numpy(a.copy()).cuda()
        self.m = torch.from_numpy(m.copy()).cuda()
        self.U = torch.from_numpy(U.copy()).cuda()
        tiled = B.dbf_tile_host(self.q, self.r, O.pack_signs(S.astype(np.float64)))
        self.bits = torch.from_numpy(tiled.copy()).cuda()
        self.wsb = B.dbf_admm_workspace_bytes(self.q, self.r)
        self.ws = torch.full((self.wsb,), 0xA5, dtype=torch.uint8, device="cuda")

    def step(self, rho, iters):
        B.dbf_admm_step(self.Minv.data_ptr(), self.C.data_ptr(), self.q, self.r, rho, iters, self.a.data_ptr(),
                        self.m.data_ptr(), self.bits.data_ptr(), self.U.data_ptr(), self.ws.data_ptr(), self.wsb,
                        G.stream_handle())
        torch.cuda.synchronize()

    def host(self):
        words = B.dbf_untile_host(self.q, self.r, self.bits.cpu().numpy())
        S = O.unpack_signs(words, self.q, self.r)
        return S, self.a.cpu().numpy().astype(np.float64), self.m.cpu().numpy().astype(np.float64), \
            self.U.cpu().numpy().astype(np.float64)


def _check_step(what, before, after, Minv, C, rho, iters, z_gate=Z_GATE):
    S0, a0, m0, U0 = before
    S1, a1, m1, U1 = after
    S_ref, a_ref, m_ref, U_ref, W_hat = O.admm_step_from(Minv.astype(np.float64), C.astype(np.float64), rho, S0, a0,
                                                         m0, U0, iters)
    Z_ref = W_hat + U0
    rms = np.sqrt(np.mean(Z_ref ** 2))
    assert np.all(np.isfinite(U1)) and np.all(np.isfinite(a1)) and np.all(np.isfinite(m1)), what
    Z_gpu = U1 + a1[:, None] * S1 * m1[None, :]
    ez = np.max(np.abs(Z_gpu - Z_ref)) / rms
    decided = np.abs(Z_ref) > z_gate * rms
    ea = np.max(np.abs(a1 - a_ref)) / np.max(np.abs(a_ref))
    em = np.max(np.abs(m1 - m_ref)) / np.max(np.abs(m_ref))
    eu = np.max(np.abs(U1 - U_ref)[decided]) / (np.max(a_ref) * np.max(m_ref))
    G.say("  %s: Z err %.2e of rms (gate %.0e), undecided signs %d of %d, a %.2e m %.2e (tol %.1e), U %.2e (tol %.0e)"
          % (what, ez, z_gate, int(np.sum(~decided)), decided.size, ea, em, VEC_TOL, eu, U_TOL))
    assert ez <= z_gate, what
    assert np.array_equal(S1[decided], S_ref[decided]), what + ": sign bits differ"
    assert np.sum(~decided) <= max(4, decided.size // 1000), what
    assert ea <= VEC_TOL and em <= VEC_TOL, what
    assert eu <= U_TOL, what


@pytest.mark.parametrize("shape", [(96, 64, 80), (300, 200, 333), (520, 260, 516), (40, 3, 5), (700, 513, 1030)])
@pytest.mark.parametrize("rho,iters", [(1.0, 1), (0.5, 3)])
def test_admm_step_matches_the_oracle(shape, rho, iters):
    p, q, r = shape
    G.say("start admm p=%d q=%d r=%d rho=%g iters=%d" % (p, q, r, rho, iters))
    Bm, W, S, a, m, U = I.make_admm_problem(p, q, r, I.seed_for(9, p + q + r))
    Minv, C = _constants(Bm, W, rho)
    dev = DeviceState(Minv, C, S, a, m, U)
    state0 = dev.host()
    dev.step(rho, iters)
    state1 = dev.host()
    _check_step("step 1", state0, state1, Minv, C, rho, iters)
    # a second update from the device's own state (each update is checked from the inputs it was given)
    dev.step(rho, iters)
    _check_step("step 2", state1, dev.host(), Minv, C, rho, iters)


@pytest.mark.parametrize("q,r", [(1, 1), (15, 33), (16, 31), (17, 64), (127, 128), (128, 129), (129, 127), (257, 96)])
def test_admm_step_at_the_edges_of_the_contraction_tiles(q, r):
    """The contraction works on fragments of 16 summation indices by 32 outputs and tiles of 128 x 128: one less, equal
    and one more in each.  The gates are those above (what the split operands leave out, at most 2^-21 of a
    product and a quarter of that on average, is a few times fp32's own rounding)."""
    p, rho = 2 * q + 40, 0.7
    Bm, W, S, a, m, U = I.make_admm_problem(p, q, r, I.seed_for(9, 300 + q + r))
    Minv, C = _constants(Bm, W, rho)
    dev = DeviceState(Minv, C, S, a, m, U)
    state0 = dev.host()
    dev.step(rho, 2)
    _check_step("q=%d r=%d" % (q, r), state0, dev.host(), Minv, C, rho, 2)


@pytest.mark.parametrize("q", [2048, 4096])
def test_admm_step_at_full_size(q):
    """The sizes bench.py times: a 4096 x 4096 weight at 1 and 2 bits per weight, i.e. q = k = 2048 or 4096
    middle channels, r = 4096; the oracle still takes only seconds there, so everything is compared."""
    p, r, rho, iters = 4096, 4096, 1.0, 2
    G.say("start admm full size p=%d q=%d r=%d" % (p, q, r))
    Bm, W, S, a, m, U = I.make_admm_problem(p, q, r, I.seed_for(9, 1 + q // 4096))
    Minv, C = _constants(Bm, W, rho)
    G.say("  constants formed")
    dev = DeviceState(Minv, C, S, a, m, U)
    state0 = dev.host()
    dev.step(rho, iters)
    _check_step("full size", state0, dev.host(), Minv, C, rho, iters)


# ---- the constant matrices formed on the device from the packed fixed factor -------------------------
#
# Gates.  C = B^T W is an fp32 matrix-core sum of p products per entry: as for Z, 1e-4 of rms(C).  Minv comes
# from a blocked fp32 Cholesky factorisation of G = B^T B + rho I, the inverse of the factor and one more
# contraction; the backward error of Cholesky is of order q * 2^-24 * ||G|| and the inverse amplifies it by
# the condition number (a few units for these inputs: rows of comparable norm, rho of order one), so entries
# of Minv are good to about q * 2^-24 * cond(G) * max|Minv| ~ 1e-3 at worst for q = 4096, typically a
# hundredth of that.  Gate: 3e-4 of max|Minv| -- and what matters downstream is tested with it: the update
# that starts from the packed factor must pass the same gates as the one that is handed fp64-made constants,
# with the gate on Z doubled (Z inherits the error of Minv times the right-hand side).
C_GATE = 1e-4
MINV_GATE = 3e-4


class PackedProblem:
    def __init__(self, p, q, r, seed):
        self.p, self.q, self.r = p, q, r
        self.S_B, self.m2, self.b, self.W, self.S, self.a, self.m, self.U = I.make_admm_packed_problem(p, q, r, seed)
        self.B_dense = O.fixed_factor_dense(self.S_B, self.b, self.m2)

    def prepare_on_device(self, rho, less=0):
        p, q, r = self.p, self.q, self.r
        tiled = B.dbf_tile_host(q, p, O.pack_signs(self.S_B.astype(np.float64)))
        bits = torch.from_numpy(tiled.copy()).cuda()
        m2, b, W = (torch.from_numpy(x.copy()).cuda() for x in (self.m2, self.b, self.W))
        Minv = torch.full((q, q), float("nan"), dtype=torch.float32, device="cuda")
        Cm = torch.full((q, r), float("nan"), dtype=torch.float32, device="cuda")
        flag = torch.full((1,), 77, dtype=torch.int32, device="cuda")
        wsb = B.dbf_admm_prepare_workspace_bytes(p, q, r) - less
        ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
        B.dbf_admm_prepare(bits.data_ptr(), m2.data_ptr(), b.data_ptr(), W.data_ptr(), p, q, r, rho, Minv.data_ptr(),
                           Cm.data_ptr(), ws.data_ptr(), wsb, flag.data_ptr(), G.stream_handle())
        torch.cuda.synchronize()
        assert int(flag.item()) == 0
        return Minv.cpu().numpy(), Cm.cpu().numpy()


def _check_constants(what, prob, rho, Minv, Cm):
    Minv_ref, C_ref = O.admm_constants(prob.B_dense, prob.W, rho)
    assert np.all(np.isfinite(Minv)) and np.all(np.isfinite(Cm)), what
    ec = np.max(np.abs(Cm - C_ref)) / np.sqrt(np.mean(C_ref ** 2))
    em = np.max(np.abs(Minv - Minv_ref)) / np.max(np.abs(Minv_ref))
    es = np.max(np.abs(Minv - Minv.T)) / np.max(np.abs(Minv_ref))
    G.say("  %s: C err %.2e of rms (gate %.0e), Minv err %.2e of max (gate %.0e), asymmetry %.1e"
          % (what, ec, C_GATE, em, MINV_GATE, es))
    assert ec <= C_GATE and em <= MINV_GATE and es <= MINV_GATE, what


@pytest.mark.parametrize("shape", [(5, 3, 4), (200, 130, 150), (300, 257, 129), (700, 520, 516), (1000, 64, 200),
                                   (128, 128, 128), (77, 300, 50)])
@pytest.mark.parametrize("rho", [1.0, 0.3])
def test_admm_prepare_matches_the_oracle_and_feeds_the_update(shape, rho):
    """From the packed fixed factor, W and rho alone: the constants formed on the device against the oracle's,
    then one update that uses them against the oracle's full update (dense B, fp64)."""
    p, q, r = shape
    G.say("start admm prepare p=%d q=%d r=%d rho=%g" % (p, q, r, rho))
    prob = PackedProblem(p, q, r, I.seed_for(9, 100 + p + q + r))
    Minv, Cm = prob.prepare_on_device(rho)
    _check_constants("constants", prob, rho, Minv, Cm)
    # (DeviceState hands the library the transpose of its first argument: Minv reaches it exactly as it was made)
    dev = DeviceState(np.ascontiguousarray(Minv.T), Cm, prob.S, prob.a, prob.m, prob.U)
    state0 = dev.host()
    dev.step(rho, 2)
    Minv64, C64 = O.admm_constants(prob.B_dense, prob.W, rho)
    _check_step("update from the packed factor", state0, dev.host(), Minv64, C64, rho, 2, z_gate=2 * Z_GATE)


@pytest.mark.parametrize("q", [2048, 4096])
def test_admm_prepare_at_full_size(q):
    p, r, rho = 4096, 4096, 1.0
    G.say("start admm prepare full size p=%d q=%d r=%d" % (p, q, r))
    prob = PackedProblem(p, q, r, I.seed_for(9, 50 + q // 2048))
    Minv, Cm = prob.prepare_on_device(rho)
    _check_constants("constants at full size", prob, rho, Minv, Cm)


def test_admm_prepare_argument_errors_and_the_definiteness_flag():
    p, q, r = 64, 32, 16
    prob = PackedProblem(p, q, r, 3)
    bits = torch.from_numpy(B.dbf_tile_host(q, p, O.pack_signs(prob.S_B.astype(np.float64))).copy()).cuda()
    f = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    m2, b, W = f(prob.m2), f(prob.b), f(prob.W)
    Minv = torch.zeros((q, q), dtype=torch.float32, device="cuda")
    Cm = torch.zeros((q, r), dtype=torch.float32, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    wsb = B.dbf_admm_prepare_workspace_bytes(p, q, r)
    assert wsb >= 4 * q * q and B.dbf_admm_prepare_workspace_bytes(0, q, r) == 0
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    ok = [bits.data_ptr(), m2.data_ptr(), b.data_ptr(), W.data_ptr(), p, q, r, 1.0, Minv.data_ptr(), Cm.data_ptr(),
          ws.data_ptr(), wsb, flag.data_ptr(), 0]
    B.dbf_admm_prepare(*ok)
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    for pos, val in ((0, 0), (1, 0), (2, 0), (3, 0), (4, 0), (5, 0), (6, 0), (7, 0.0), (7, float("nan")), (8, 0), (9, 0),
                     (10, 0), (11, wsb - 1), (10, ws.data_ptr() + 8), (12, flag.data_ptr() + 2)):
        bad = list(ok)
        bad[pos] = val
        with pytest.raises(B.DbfError):
            B.dbf_admm_prepare(*bad)
    # a pivot that is not positive (here: a NaN scale, which the entry point does not support but must survive):
    # the flag is raised, nothing hangs or faults
    nan_m2 = prob.m2.copy()
    nan_m2[0] = np.nan
    m2n = f(nan_m2)
    bad = list(ok)
    bad[1] = m2n.data_ptr()
    B.dbf_admm_prepare(*bad)
    torch.cuda.synchronize()
    assert int(flag.item()) >= 1


@pytest.mark.parametrize("p,q,rho", [(64, 512, 1e-12), (40, 300, 1e20)])
def test_admm_prepare_leaves_numbers_behind_pivots_that_are_not_positive(p, q, rho):
    """G = B^T B + rho I of rank p with rho far below its rounding, or with scales that make it so behind the first block (m2 = 0 in that, 1e18 behind it, rho = 1e20): pivots that are not positive raise the flag, and their rows count as zero.  Minv is not the inverse then, but has no infinities or NaN."""
    rng = np.random.default_rng(I.seed_for(6, 935 + q))
    S = np.where(rng.random((q, p)) < 0.5, -1.0, 1.0)
    m2 = rng.uniform(0.5, 1.5, q).astype(np.float32)
    if rho > 1:
        m2 = np.where(np.arange(q) < 128, 0, 1e18 * m2).astype(np.float32)
    b, W = np.full(p, 0.25, np.float32), rng.standard_normal((p, 16)).astype(np.float32)
    bits = torch.from_numpy(B.dbf_tile_host(q, p, O.pack_signs(S)).copy()).cuda()
    dev = [torch.from_numpy(x.copy()).cuda() for x in (m2, b, W)]
    Minv, Cm = torch.empty((q, q), device="cuda"), torch.empty((q, 16), device="cuda")
    flag = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    wsb = B.dbf_admm_prepare_workspace_bytes(p, q, 16)
    ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
    B.dbf_admm_prepare(bits.data_ptr(), dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(), p, q, 16, rho, Minv.data_ptr(), Cm.data_ptr(),
                       ws.data_ptr(), wsb, flag.data_ptr(), G.stream_handle())
    torch.cuda.synchronize()
    G.say("  p=%d q=%d: %d blocks with such pivots, largest entry %.2g" % (p, q, int(flag.item()), float(Minv.abs().max())))
    assert 1 <= int(flag.item()) <= (q + 127) // 128 and bool(torch.isfinite(Minv).all())


def test_admm_fixed_point_on_an_exactly_factorisable_target():
    """W = B A* with A* of the SVID form and U = 0: the update must give A* back and leave U at zero
    (to fp32 accuracy)."""
    p, q, r = 300, 128, 192
    Bm, _, S, a, m, _ = I.make_admm_problem(p, q, r, 5)
    A_star = a[:, None].astype(np.float64) * S * m[None, :]
    W = (Bm.astype(np.float64) @ A_star).astype(np.float32)
    Minv, C = _constants(Bm, W, 1.0)
    dev = DeviceState(Minv, C, S, a, m, np.zeros((q, r), dtype=np.float32))
    dev.step(1.0, 2)
    S1, a1, m1, U1 = dev.host()
    assert np.array_equal(S1, S.astype(np.float64))
    assert np.max(np.abs(np.outer(a1, m1) - np.outer(a, m))) <= 1e-4 * np.max(np.outer(a, m))
    assert np.max(np.abs(U1)) <= 1e-4 * np.max(np.abs(A_star))


def test_admm_argument_errors():
    q, r = 8, 8
    f = lambda *s: torch.zeros(s, dtype=torch.float32, device="cuda")
    Minv, C, a, m, U = f(q, q), f(q, r), f(q), f(r), f(q, r)
    bits = torch.zeros(B.dbf_tiled_bytes(q, r), dtype=torch.uint8, device="cuda")
    wsb = B.dbf_admm_workspace_bytes(q, r)
    ws = torch.zeros(wsb, dtype=torch.uint8, device="cuda")
    assert B.dbf_admm_workspace_bytes(0, 4) == 0 and wsb >= 2 * 4 * q * r
    ok = (Minv.data_ptr(), C.data_ptr(), q, r, 1.0, 1, a.data_ptr(), m.data_ptr(), bits.data_ptr(), U.data_ptr(),
          ws.data_ptr(), wsb, 0)
    B.dbf_admm_step(*ok)
    torch.cuda.synchronize()
    for pos, val in ((0, 0), (1, 0), (2, 0), (3, 0), (4, 0.0), (4, -1.0), (4, float("inf")), (5, 0), (6, 0), (7, 0),
                     (8, 0), (9, 0), (10, 0), (11, wsb - 1), (10, ws.data_ptr() + 4), (9, U.data_ptr() + 2)):
        bad = list(ok)
        bad[pos] = val
        with pytest.raises(B.DbfError):
            B.dbf_admm_step(*bad)


def test_admm_iterations_on_the_device_approach_a_factorisable_target():
    """Twenty consecutive updates on the device (state kept there, each call the next iteration) on a target
    W = B A* with A* of the SVID form, from a start far away: the residual ||B A - W|| of the projected iterate
    must fall to under a hundredth of the start's, as the fp64 oracle's does (its own pin shows a thousandth
    after 30 updates)."""
    rng = np.random.default_rng(21)
    p, q, r = 300, 96, 160
    Bm = (rng.standard_normal((p, q)) / np.sqrt(p)).astype(np.float32)
    S_star = np.where(rng.random((q, r)) < 0.5, 1.0, -1.0)
    A_star = rng.uniform(0.5, 1.5, q)[:, None] * S_star * rng.uniform(0.5, 1.5, r)[None, :]
    W = (Bm.astype(np.float64) @ A_star).astype(np.float32)
    Minv, C = _constants(Bm, W, 1.0)
    S0 = np.where(rng.random((q, r)) < 0.5, 1, -1).astype(np.int8)
    a0, m0 = np.full(q, 0.1, dtype=np.float32), np.full(r, 0.1, dtype=np.float32)
    dev = DeviceState(Minv, C, S0, a0, m0, np.zeros((q, r), dtype=np.float32))
    B64, W64 = Bm.astype(np.float64), W.astype(np.float64)

    def residual(state):
        S, a, m, _ = state
        return np.linalg.norm(B64 @ (a[:, None] * S * m[None, :]) - W64)

    res0 = residual(dev.host())
    for _ in range(20):
        dev.step(1.0, 3)
    res = residual(dev.host())
    G.say("  residual %.3e -> %.3e" % (res0, res))
    assert res < 1e-2 * res0


@pytest.mark.parametrize("p,q,r", [(33, 1, 1), (48, 17, 130), (300, 129, 64), (64, 191, 257), (900, 193, 1500), (260, 1536, 1400), (100, 2048, 2100)])
def test_admm_contractions_with_their_steps_and_blocks_cut_by_size(p, q, r):
    """The contraction's three forms -- 64 x 128 blocks and 128 x 128 blocks with the steps in two halves (up to 128 and up to 256 blocks of 128 x
    128), 128 x 128 blocks whole -- at ragged sizes, with one step, an odd number and an even number of them; the factorisation with one, two
    and sixteen block rows, the last of them short.  Gates: as above."""
    rho = 0.8
    prob = PackedProblem(p, q, r, I.seed_for(9, 500 + p + q + r))
    Minv, Cm = prob.prepare_on_device(rho)
    _check_constants("constants p=%d q=%d r=%d" % (p, q, r), prob, rho, Minv, Cm)
    dev = DeviceState(np.ascontiguousarray(Minv.T), Cm, prob.S, prob.a, prob.m, prob.U)
    state0 = dev.host()
    dev.step(rho, 1)
    Minv64, C64 = O.admm_constants(prob.B_dense, prob.W, rho)
    _check_step("update q=%d r=%d" % (q, r), state0, dev.host(), Minv64, C64, rho, 1, z_gate=2 * Z_GATE)


@pytest.mark.parametrize("q", [127, 129, 256, 385, 511, 2830])
def test_admm_prepare_at_the_edges_of_the_elimination_blocks(q):
    """Blocks of 128 with one row or column more or less, one to five block rows; 2830: 23 block rows, the first of which have more than 256 blocks below
    them and so are made in a launch of their own.  Gates: as above."""
    prob = PackedProblem(60, q, 33, I.seed_for(9, 700 + q))
    Minv, Cm = prob.prepare_on_device(0.9)
    _check_constants("constants q=%d" % q, prob, 0.9, Minv, Cm)


@pytest.mark.parametrize("p,q,r", [(2100, 300, 1000), (1100, 200, 16600), (700, 520, 516)])
def test_admm_prepare_with_parts_of_C_beside_the_elimination(p, q, r):
    """C in three parts a block, in two with more block columns than there is room for, in one; and with the workspace that a call can do with, without the
    planes that are apart then (two pieces of max(p, q) x q in whole blocks of 128, four bytes a line and block): the same one after the other.  Gates: as above."""
    prob = PackedProblem(p, q, r, I.seed_for(9, 800 + p + q))
    n = (q + 127) // 128 * ((max(p, q) + 127) // 128)
    for less in (0, 256, n * 65536 + 512 * n):
        Minv, Cm = prob.prepare_on_device(0.9, less)
        _check_constants("constants p=%d q=%d r=%d, %d bytes less" % (p, q, r, less), prob, 0.9, Minv, Cm)
    with pytest.raises(B.DbfError):
        prob.prepare_on_device(0.9, less + 256)


@pytest.mark.parametrize("p,q,r", [(100, 70, 90), (520, 300, 260)])
def test_sign_tiles_may_start_at_any_multiple_of_four_bytes(p, q, r):
    """The packed signs of the constants and of an update are documented as 4-byte aligned: the same tiles 4, 8 and 12 bytes further on
    give the same bits."""
    rng = np.random.default_rng(I.seed_for(6, 900 + p))
    S = np.where(rng.random((q, p)) < 0.5, -1.0, 1.0)
    tiles = torch.from_numpy(B.dbf_tile_host(q, p, O.pack_signs(S)).copy()).cuda()
    step = torch.from_numpy(B.dbf_tile_host(q, r, O.pack_signs(np.where(rng.random((q, r)) < 0.5, -1.0, 1.0))).copy()).cuda()
    f = lambda *s: torch.from_numpy(rng.uniform(0.5, 1.5, s).astype(np.float32)).cuda()   # noqa: E731
    m2, b, W, a, m, U = f(q), f(p), f(p, r), f(q), f(r), f(q, r)
    wsb = max(B.dbf_admm_prepare_workspace_bytes(p, q, r), B.dbf_admm_workspace_bytes(q, r))
    want = None
    for off in (0, 4, 8, 12):
        G.say("sign tiles %d bytes on, p=%d q=%d r=%d" % (off, p, q, r))
        ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
        moved = torch.zeros(tiles.numel() + 16, dtype=torch.uint8, device="cuda")
        moved[off:off + tiles.numel()] = tiles
        st = torch.zeros(step.numel() + 16, dtype=torch.uint8, device="cuda")
        st[off:off + step.numel()] = step
        Minv, C = torch.empty((q, q), device="cuda"), torch.empty((q, r), device="cuda")
        a1, m1, U1 = a.clone(), m.clone(), U.clone()
        B.dbf_admm_prepare(moved.data_ptr() + off, m2.data_ptr(), b.data_ptr(), W.data_ptr(), p, q, r, 1.0, Minv.data_ptr(), C.data_ptr(),
                           ws.data_ptr(), wsb, 0, G.stream_handle())
        B.dbf_admm_step(Minv.data_ptr(), C.data_ptr(), q, r, 1.0, 2, a1.data_ptr(), m1.data_ptr(), st.data_ptr() + off, U1.data_ptr(),
                        ws.data_ptr(), wsb, G.stream_handle())
        torch.cuda.synchronize()
        got = [t.cpu().numpy().copy() for t in (Minv, C, a1, m1, U1, st[off:off + step.numel()])]
        if want is None:
            want = got
        for g, w in zip(got, want):
            assert np.array_equal(g.view(np.uint8), w.view(np.uint8)), off


@pytest.mark.parametrize("q,r", [(130, 70), (300, 200), (513, 129)])
def test_admm_contraction_with_operands_of_many_magnitudes(q, r):
    """Minv = D M D and C = C0 / D with D from 2^-12 to 2^12: along a line of either operand entries differ by 2^24 and more, while all terms of
    a sum count alike.  The operands are split relative to the largest of 128 entries of a line, exactly to 2^-23 down to 2^-27 of it, and the product of two rests,
    2^-22, is left out: at worst 2^-21 of the sum of the terms' magnitudes.  As much again is for R's own roundings and the fp32 additions."""
    rng = np.random.default_rng(I.seed_for(6, 970 + q))
    D = np.exp2(rng.uniform(-12, 12, q))
    M = rng.uniform(0.2, 1.0, (q, q)) * np.where(rng.random((q, q)) < 0.5, -1.0, 1.0)
    Minv = ((M + M.T) * D[:, None] * D[None, :]).astype(np.float32)
    C = (rng.standard_normal((q, r)) / D[:, None]).astype(np.float32)
    S = np.where(rng.random((q, r)) < 0.5, 1, -1).astype(np.int8)
    a, m = (0.3 / D).astype(np.float32), rng.uniform(0.5, 1.5, r).astype(np.float32)
    U = (0.1 * rng.standard_normal((q, r)) / D[:, None]).astype(np.float32)
    dev = DeviceState(Minv, C, S, a, m, U)
    dev.step(1.0, 2)
    S1, a1, m1, U1 = dev.host()
    R = C.astype(np.float64) + a.astype(np.float64)[:, None] * S * m - U
    Z = Minv.astype(np.float64) @ R + U
    terms = np.abs(Minv.astype(np.float64)) @ (np.abs(C).astype(np.float64) + np.abs(a.astype(np.float64)[:, None] * m) + np.abs(U)) + np.abs(U)
    got = U1 + a1[:, None] * S1 * m1[None, :]
    err = np.abs(got - Z)
    gate = 2.0 ** -20 * terms + 2.0 ** -23 * np.abs(a1[:, None] * m1[None, :])   # (the latter: U' = Z - a' S' m' on the device)
    G.say("  magnitudes q=%d r=%d: largest error %.2g of the gate" % (q, r, np.max(err / gate)))
    assert np.all(err <= gate)


@pytest.mark.parametrize("below", [20, 27, 32, 40])
@pytest.mark.parametrize("outlier_in", ["Minv", "C"])
def test_admm_contraction_of_entries_far_below_the_largest_of_their_chunk(outlier_in, below):
    """One entry of a chunk of a line is 1.5 and meets a zero of the other operand, the one that counts is 2^-below of it: met to 2^-50 of the
    largest (dbf.h), which is more than its own 2^-23 from 2^-27 on.  Z has one term an entry, so that nothing else is in it but the split
    (2^-21 of the term at worst) and the roundings of Z, U and this test's sum."""
    q, r = 256, 200
    rng = np.random.default_rng(I.seed_for(6, 975 + below))
    v, C = rng.uniform(0.5, 1.0, q), rng.uniform(0.5, 1.0, (q, r)) * np.where(rng.random((q, r)) < 0.5, -1, 1)
    heads = np.arange(0, q, 128)                  # the summation index of a chunk that has the large entry
    if outlier_in == "Minv":
        Minv = np.diag(v * 2.0 ** -below)
        for i in range(q):
            Minv[heads[i // 128], i] = Minv[i, heads[i // 128]] = 1.5
        C[heads] = 0
    else:
        Minv = np.diag(v)
        C *= 2.0 ** -below
        C[heads] = 1.5
    Minv, C = Minv.astype(np.float32), C.astype(np.float32)
    S = np.where(rng.random((q, r)) < 0.5, 1, -1).astype(np.int8)
    dev = DeviceState(Minv, C, S, np.zeros(q, np.float32), np.ones(r, np.float32), np.zeros((q, r), np.float32))
    dev.step(1.0, 1)
    S1, a1, m1, U1 = dev.host()
    rest = np.setdiff1d(np.arange(q), heads)
    Z = (Minv.astype(np.float64) @ C.astype(np.float64))[rest]
    A1 = (a1[:, None] * S1 * m1[None, :])[rest]
    floor = 2.0 ** -50 * 1.5 * (np.abs(C[rest]) if outlier_in == "Minv" else v[rest, None])
    gate = floor + 2.0 ** -21 * np.abs(Z) + 2.0 ** -23 * (np.abs(Z) + np.abs(A1))
    err = np.abs(U1[rest] + A1 - Z)
    G.say("  outlier in %s, 2^-%d below: largest error %.2g of the gate, 2^%.1f of the entry" % (outlier_in, below, np.max(err / gate),
                                                                                                 np.log2(np.max(err / np.abs(Z)))))
    assert np.all(err <= gate)


@pytest.mark.parametrize("q,r", [(130, 70), (300, 200), (2048, 2048), (2304, 2304)])
@pytest.mark.parametrize("exponent", [110, 96, -96])
def test_admm_contraction_between_a_large_and_a_small_operand(q, r, exponent):
    """Minv = 2^e D M D and C = 2^-e C0 / D, D from 2^-14 to 2^14 and the same for 128 rows: the products are of ordinary size, though entries of
    Minv reach 2^124 (or fall to 2^-124, those of C reaching 2^110): no sum may leave the range on its way through the two operands' scales.  D does not vary inside
    a chunk, so that all terms are met to 2^-22 or better, as in the test above; its gate.  (Sizes: every shape of blocks.)"""
    rng = np.random.default_rng(I.seed_for(6, 930 + q + exponent))
    steps = rng.integers(-14, 15, (q + 127) // 128)
    steps[0] = 14 if exponent > 0 else -14
    D = np.exp2(np.repeat(steps - (14 if exponent > 96 else 0), 128)[:q].astype(np.float64))
    M = rng.uniform(0.2, 1.0, (q, q)) * np.where(rng.random((q, q)) < 0.5, -1.0, 1.0)
    Minv = ((M + M.T) * D[:, None] * D[None, :] * 2.0 ** exponent).astype(np.float32)
    small = 2.0 ** -exponent / D[:, None]
    C = (rng.standard_normal((q, r)) * small).astype(np.float32)
    S = np.where(rng.random((q, r)) < 0.5, 1, -1).astype(np.int8)
    a = (0.3 * 2.0 ** -(exponent // 2) / D).astype(np.float32)
    m = (rng.uniform(0.5, 1.5, r) * 2.0 ** -(exponent - exponent // 2)).astype(np.float32)
    U = (0.1 * rng.standard_normal((q, r)) * np.minimum(small, 1.0)).astype(np.float32)   # (Z has it too, and is of ordinary size)
    assert np.all(np.isfinite(Minv)) and np.all(np.isfinite(C)) and np.max(np.abs(Minv if exponent > 0 else C)) > 2.0 ** 106
    dev = DeviceState(Minv, C, S, a, m, U)
    dev.step(1.0, 2)
    S1, a1, m1, U1 = dev.host()
    am = np.abs(a.astype(np.float64)[:, None] * m)
    R = C.astype(np.float64) + a.astype(np.float64)[:, None] * S * m - U
    Z = Minv.astype(np.float64) @ R + U
    terms = np.abs(Minv.astype(np.float64)) @ (np.abs(C).astype(np.float64) + am + np.abs(U)) + np.abs(U)
    got = U1 + a1[:, None] * S1 * m1[None, :]
    gate = 2.0 ** -20 * terms + 2.0 ** -23 * np.abs(a1[:, None] * m1[None, :])   # (the latter: U' = Z - a' S' m' on the device)
    with np.errstate(invalid="ignore"):
        err = np.abs(got - Z)
    G.say("  large and small q=%d r=%d 2^%d: largest error %.2g of the gate" % (q, r, exponent, np.max(err / gate)))
    assert np.all(np.isfinite(got)) and np.all(err <= gate)


def _scaled_error(p, q, m2, rho, seed, b=None):
    """Minv from the device against 64 bits, entries relative to the roots of their diagonal entries: the largest error, its norm over Minv's, the condition
    of B^T B + rho I with its diagonal scaled to one, and the mean error of Minv's diagonal."""
    rng = np.random.default_rng(seed)
    S = np.where(rng.random((q, p)) < 0.5, -1.0, 1.0)
    b = ((rng.uniform(0.5, 1.5, p) if b is None else np.full(p, b)) / np.sqrt(p)).astype(np.float32)
    W = rng.standard_normal((p, 16)).astype(np.float32)
    bits = torch.from_numpy(B.dbf_tile_host(q, p, O.pack_signs(S)).copy()).cuda()
    dev = [torch.from_numpy(x.copy()).cuda() for x in (m2, b, W)]
    Minv, Cm = torch.empty((q, q), device="cuda"), torch.empty((q, 16), device="cuda")
    flag = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    wsb = B.dbf_admm_prepare_workspace_bytes(p, q, 16)
    ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
    B.dbf_admm_prepare(bits.data_ptr(), dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(), p, q, 16, rho, Minv.data_ptr(), Cm.data_ptr(),
                       ws.data_ptr(), wsb, flag.data_ptr(), G.stream_handle())
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    Bt = m2.astype(np.float64)[:, None] * (S * b.astype(np.float64))
    A = Bt @ Bt.T + float(np.float32(rho)) * np.eye(q)
    s = 1 / np.sqrt(np.diag(A))
    A *= s[:, None] * s
    values = np.linalg.eigvalsh(A)
    want = np.linalg.inv(A)
    got = Minv.cpu().numpy().astype(np.float64) / (s[:, None] * s)
    d = 1 / np.sqrt(np.diag(want))
    err = (got - want) * d[:, None] * d
    return np.max(np.abs(err)), np.linalg.norm(err) / np.linalg.norm(want * d[:, None] * d), values[-1] / values[0], np.mean(np.diag(err))


@pytest.mark.parametrize("p,q", [(400, 100), (2000, 500), (5400, 2830)])
@pytest.mark.parametrize("decades", [2, 6, 8])
def test_admm_prepare_with_scales_of_many_magnitudes(p, q, decades):
    """m2 from 10^-d to 10^d and rho far below all of it: an elimination in floating point does not feel the scales of rows and columns, so the error, entries
    relative to the roots of their diagonal entries, stays that of the problem with its diagonal scaled to one: about its condition times the roundings of
    q numbers that add up at random, 2^-24 sqrt(q).  (2830: block rows made first.)"""
    rng = np.random.default_rng(I.seed_for(6, 940 + q + decades))
    m2 = (10 ** rng.uniform(-decades, decades, q)).astype(np.float32)
    worst, norm, cond, _ = _scaled_error(p, q, m2, 10.0 ** (-2 * decades - 9), I.seed_for(6, 941 + q + decades))
    G.say("  scales of %d decades p=%d q=%d: largest error %.2e, of the norm %.2e, condition %.1f" % (2 * decades, p, q, worst, norm, cond))
    assert worst <= 2.0 ** -24 * np.sqrt(q) * cond


@pytest.mark.parametrize("p,q,rho", [(2000, 500, 1.0), (600, 1000, 1.0), (1024, 1024, 0.1), (779, 1728, 1.0), (512, 1024, 1e-3), (300, 700, 1e-3), (64, 512, 1e-2),
                                     (1500, 2830, 1e-2)])
def test_admm_prepare_is_as_exact_as_its_condition_allows(p, q, rho):
    """Ordinary and badly conditioned problems, q > p with a small rho among them: the error of Minv in norm is 2^-24 times the condition to a factor of two
    (2^-25.5 to 2^-23.7 times it with an elimination in fp32)."""
    rng = np.random.default_rng(I.seed_for(6, 945 + p + q))
    m2 = rng.uniform(0.5, 1.5, q).astype(np.float32)
    worst, norm, cond, mean = _scaled_error(p, q, m2, rho, I.seed_for(6, 946 + p + q))
    G.say("  p=%d q=%d rho=%g: error of the norm %.2e = 2^%.2f of the condition, %.0f; largest %.2e, mean of the diagonal %.1e"
          % (p, q, rho, norm, np.log2(norm / cond), cond, worst, mean))
    assert norm <= 2.0 ** -23 * cond


def test_admm_prepare_loses_nothing_of_one_sign():
    """Entries on the diagonal of G - R^T R are sums of squares, of which the products of the operands' low pieces must not be missing: 2^-24.5 of each on
    average, of one sign, which shows in the mean error of Minv's diagonal.  With scales whose products are exact, B^T B is, and the mean over 16 problems is known to
    2e-9: -6.1e-8 without these products, -2.8e-8 with them (what is left comes from elsewhere, from sums that the matrix cores round down for all that is
    known).  The gate is half-way."""
    rng = np.random.default_rng(I.seed_for(6, 948))
    means = [_scaled_error(64, 1000, rng.uniform(0.5, 1.5, 1000).astype(np.float32), 1.0, I.seed_for(6, 960 + n), b=1.0)[3]
             for n in range(16)]
    G.say("  mean error of Minv's diagonal %.2e (16 problems, %.1e each)" % (np.mean(means), np.std(means)))
    assert abs(np.mean(means)) <= 4.4e-8


@pytest.mark.parametrize("q", [40, 200])
def test_admm_prepare_with_subnormal_pivots(q):
    """Pivots below 2^-126, where the reciprocal and root instructions take none: G = B^T B + rho I with rho = 9e-39 and B^T B a
    hundredth of it, so that Minv is near the top of the range (1.1e38).  Against 64 bits; G itself has a spacing of 2^-149, 1.6e-7 of rho."""
    p, r, rho = 64, 16, np.float32(9e-39)
    rng = np.random.default_rng(I.seed_for(6, 950 + q))
    S = np.where(rng.random((q, p)) < 0.5, -1.0, 1.0)
    m2 = np.full(q, 1.2e-21, dtype=np.float32)
    b, W = np.ones(p, dtype=np.float32), rng.standard_normal((p, r)).astype(np.float32)
    bits = torch.from_numpy(B.dbf_tile_host(q, p, O.pack_signs(S)).copy()).cuda()
    dev = [torch.from_numpy(x.copy()).cuda() for x in (m2, b, W)]
    Minv, Cm = torch.empty((q, q), device="cuda"), torch.empty((q, r), device="cuda")
    flag = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    wsb = B.dbf_admm_prepare_workspace_bytes(p, q, r)
    ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
    B.dbf_admm_prepare(bits.data_ptr(), dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(), p, q, r, float(rho), Minv.data_ptr(),
                       Cm.data_ptr(), ws.data_ptr(), wsb, flag.data_ptr(), G.stream_handle())
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    Bt = m2.astype(np.float64)[:, None] * S
    want = np.linalg.inv((Bt @ Bt.T + float(rho) * np.eye(q)) * 1e38) * 1e38
    got = Minv.cpu().numpy().astype(np.float64)
    err = np.max(np.abs(got - want)) / np.max(np.abs(want))
    G.say("  subnormal pivots q=%d: Minv err %.2e of max" % (q, err))
    assert np.all(np.isfinite(got)) and err <= 2e-5


@pytest.mark.parametrize("q", [40, 200])
def test_admm_prepare_with_pivots_at_the_top_of_the_range(q):
    """Diagonal entries of G = B^T B + rho I from 6e37 to 1.6e38, on both sides of 2^126 = 8.5e37, above which the reciprocal of a pivot is subnormal and
    the instruction returns zero.  Against 64 bits; Minv is near the bottom of the range (1e-38), whose spacing 2^-149 is 1.4e-7 of it."""
    p, r, rho = 64, 16, np.float32(6e37)
    rng = np.random.default_rng(I.seed_for(6, 955 + q))
    S = np.where(rng.random((q, p)) < 0.5, -1.0, 1.0)
    m2 = (1.25e18 * rng.uniform(0.1, 1.0, q)).astype(np.float32)
    b, W = np.ones(p, dtype=np.float32), rng.standard_normal((p, r)).astype(np.float32)
    bits = torch.from_numpy(B.dbf_tile_host(q, p, O.pack_signs(S)).copy()).cuda()
    dev = [torch.from_numpy(x.copy()).cuda() for x in (m2, b, W)]
    Minv, Cm = torch.empty((q, q), device="cuda"), torch.empty((q, r), device="cuda")
    flag = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    wsb = B.dbf_admm_prepare_workspace_bytes(p, q, r)
    ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
    B.dbf_admm_prepare(bits.data_ptr(), dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(), p, q, r, float(rho), Minv.data_ptr(),
                       Cm.data_ptr(), ws.data_ptr(), wsb, flag.data_ptr(), G.stream_handle())
    torch.cuda.synchronize()
    assert int(flag.item()) == 0
    Bt = m2.astype(np.float64)[:, None] * S
    want = np.linalg.inv((Bt @ Bt.T + float(rho) * np.eye(q)) * 1e-38) * 1e-38
    got = Minv.cpu().numpy().astype(np.float64)
    err = np.max(np.abs(got - want)) / np.max(np.abs(want))
    G.say("  pivots up to 1.6e38 q=%d: Minv err %.2e of max" % (q, err))
    assert np.all(np.isfinite(got)) and err <= 2e-5


@pytest.mark.parametrize("q,r", [(40, 4096), (300, 4096), (2048, 4096)])
def test_admm_contraction_meets_the_largest_entry_of_a_line_exactly(q, r):
    """Minv = D, of 24 significant bits (and, at the larger sizes, a hundredth of its size beside it).  An error of an entry of the diagonal is common to
    its row of Z, and the row's factor keeps all of it; those of R and of the sums differ from column to column: at most 2^-22 of an entry each, so that their
    mean over r = 4096 columns has a deviation of at most 2^-22 / sqrt(3 r) = 2^-28.8.  Gate: six of these.  (An entry with two bits less: 2^-24.5.)"""
    rng = np.random.default_rng(I.seed_for(6, 990 + q))
    Minv = np.diag(rng.uniform(0.3, 0.7, q))
    if q > 40:
        M = 0.002 / np.sqrt(q) * rng.standard_normal((q, q))
        Minv += M + M.T
    Minv = Minv.astype(np.float32)
    C = (np.where(rng.random((q, r)) < 0.5, 1, -1) * rng.uniform(0.5, 1.5, (q, r))).astype(np.float32)
    S = np.where(rng.random((q, r)) < 0.5, 1, -1).astype(np.int8)
    dev = DeviceState(Minv, C, S, np.zeros(q, np.float32), np.ones(r, np.float32), np.zeros((q, r), np.float32))
    dev.step(1.0, 1)
    S1, a1, m1, U1 = dev.host()
    Z = Minv.astype(np.float64) @ C.astype(np.float64)
    err = np.sum((U1 + a1[:, None] * S1 * m1[None, :] - Z) * np.sign(Z), axis=1) / np.sum(np.abs(Z), axis=1)
    G.say("  rows of Z q=%d r=%d: common error 2^%.2f at most, 2^%.2f on average" % (q, r, np.log2(np.max(np.abs(err))), np.log2(np.mean(np.abs(err)))))
    assert np.max(np.abs(err)) <= 6 * 2.0 ** -22 / np.sqrt(3 * r)


@pytest.mark.parametrize("q,r,iters", [(1, 1, 1), (129, 65, 1), (300, 200, 2), (127, 2052, 8), (300, 2052, 8), (2048, 16388, 1)])
def test_admm_step_ends_as_the_projection_and_the_dual(q, r, iters):
    """The last kernel of an update forms a' and m' beside U', or after dbf_svid's own last kernel where it has too many
    workgroups (2048 x 16388), or after all rounds in one launch (8 rounds of 300 x 2052).  Z lies before the
    projection's part at the end of the workspace: dbf_svid of it gives the same signs and, but for sums of squares in
    64 bits in another order, the same a' and m' (rounded to fp32 once or twice: 4 x 2^-24), and U' = Z - a' S' m'^T to
    its two roundings.  m' may start at any multiple of four bytes.  Where that or the one launch takes the rounds to other
    kernels, their fp32 sums of positive terms, each through at most 128 additions, are in another order: 2 x 128 x 2^-24."""
    G.say("start admm ending q=%d r=%d iters=%d" % (q, r, iters))
    gen = torch.Generator(device="cuda").manual_seed(I.seed_for(31, q + r))
    rand = lambda *n: torch.randn(*n, generator=gen, device="cuda")  # noqa: E731
    Minv = torch.eye(q, device="cuda") + 0.01 * rand(q, q) / q ** 0.5
    C, U0, a0, m0 = rand(q, r), 0.1 * rand(q, r), rand(q).abs(), rand(r).abs()
    svid_bytes = B.dbf_svid_workspace_bytes(q, r)
    wsb = B.dbf_admm_workspace_bytes(q, r)
    end = wsb - svid_bytes
    up256 = lambda n: (n + 255) // 256 * 256  # noqa: E731
    tiles = (q + 127) // 128 * ((r + 63) // 64) * 1024
    results = []
    for shift in (0, 1):
        ws = torch.full((wsb,), 0xA5, dtype=torch.uint8, device="cuda")
        a, U, bits = a0.clone(), U0.clone(), torch.zeros(tiles, dtype=torch.uint8, device="cuda")
        m = torch.full((r + 2,), -7.0, device="cuda")
        m[shift:shift + r] = m0
        B.dbf_admm_step(Minv.data_ptr(), C.data_ptr(), q, r, 1.0, iters, a.data_ptr(), m.data_ptr() + 4 * shift, bits.data_ptr(),
                        U.data_ptr(), ws.data_ptr(), wsb, G.stream_handle())
        torch.cuda.synchronize()
        assert (m[:shift] == -7.0).all() and (m[shift + r:] == -7.0).all()
        results.append((a, m[shift:shift + r].clone(), bits, U))
    Z = ws[end - up256(4 * q * r):][:4 * q * r].view(torch.float32).reshape(q, r).clone()
    a, m, bits, U = results[0]
    tol = (4 if iters < 3 and r < 16384 else 2 * 128) * 2.0 ** -24
    for other in results[1:]:
        assert torch.equal(bits, other[2])
        for x, y in zip((a, m, U), (other[0], other[1], other[3])):
            assert (x - y).abs().max() <= tol * x.abs().max()
    sa, sm, sbits = torch.empty_like(a0), torch.empty_like(m0), torch.zeros_like(bits)
    sws = torch.empty(svid_bytes, dtype=torch.uint8, device="cuda")
    B.dbf_svid(Z.data_ptr(), q, r, iters, sa.data_ptr(), sm.data_ptr(), sbits.data_ptr(), sws.data_ptr(), svid_bytes, G.stream_handle())
    torch.cuda.synchronize()
    assert torch.equal(bits, sbits)
    assert ((a - sa).abs() <= tol * sa.abs()).all() and ((m - sm).abs() <= tol * sm.abs()).all()
    am = a[:, None] * m[None, :]
    assert ((U - (Z - torch.where(Z >= 0, am, -am))).abs() <= 2.0 ** -23 * (Z.abs() + am)).all()
