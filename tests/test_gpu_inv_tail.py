"""The late iterations of the coupled Newton-Schulz inverse (from the 17th on a
launch that scans for the submatrices that still iterate) against the oracle.
S and K are diagonal, S with one entry of 2e-5 in some submatrices (S^-1 stays
inside the FP16 range): there the smallest value of Z Y grows by 9/4 an
iteration from 2e-5, so they take about ln(5e4) / ln(9/4) = 13.3 iterations
and 4 to 6 more. The others (S = I, a residual of exactly zero, which the
stopping rule on its decrease does not end) iterate beside them to the last
slot and are not checked. A_J has the eigenvalues +-1, and D is diagonal:
1 / S at the occupied ones, to the 16-bit error of S^-1: the rounding of the
starting value (in FP16 below the normal range, 2^-25 of 2e-5: 1.5e-3) and of
Y and Z, held to the bounds of the route, 3e-2 in FP16 and 2.5e-1 in BF16."""
import numpy as np
import pytest

from oracle import nolsm as o
from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu

BOUNDS = {"fp16": 3e-2, "bf16": 2.5e-1}


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    return t


def diagonal_system(nmol, cutoff):
    s = synth.water_cube(nmol, cutoff, config_id=131)
    d = np.ones((nmol, s.K.bs))
    d[::3, 2] = 2e-5
    sign = np.where(np.arange(s.K.bs) % 2 == 0, -1.0, 1.0)
    for m, diag in ((s.S, d), (s.K, d * sign)):
        m.val[...] = 0.0
        for J in range(nmol):
            q = m.row_ptr[J] + list(m.col_idx[m.row_ptr[J]:m.row_ptr[J + 1]]).index(J)
            m.val[q] = np.diag(diag[J])
    return s


# isolated molecules (6 rows, 64-row tiles), the whole matrix of 10 molecules
# (one 64-row tile) and of 43 (258 rows: three 128-row tiles, the last with 2)
@pytest.mark.parametrize("nmol,cutoff", [(40, 0.1), (10, 2.2), (43, 2.2)])
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_late_inverse_iterations(torch, nmol, cutoff, prec):
    from paper_2104_08245_amd import Solver
    s = diagonal_system(nmol, cutoff)
    ref = o.nolsm(s)
    sv = Solver(s, prec=prec, device="cuda:0", inverse=L.INV_COUPLED_NS)
    sv.run()
    torch.cuda.synchronize()
    st, dc = sv.host_stats(), sv.host_dcols()
    slow = np.arange(nmol) % 3 == 0 if cutoff < 1 else np.ones(nmol, bool)
    print("[gpu]", nmol, cutoff, prec, "iterations", st["iters_inv"].min(), st["iters_inv"].max(), flush=True)
    assert np.all(st["status"][slow] == 0)
    assert np.all((st["iters_inv"][slow] > 16) & (st["iters_inv"][slow] < 39))
    for J in np.flatnonzero(slow):
        err = np.linalg.norm(dc[J] - ref.Dcols[J]) / np.linalg.norm(ref.Dcols[J])
        assert err <= BOUNDS[prec], (J, err)
