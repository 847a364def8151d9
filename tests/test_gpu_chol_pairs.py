"""The Cholesky factor by pairs of 64-row panels: one to five panels (odd and
even), on the routes that factor in FP64 and in FP32, against the oracle; and
a pivot that fails in the first and in the second panel of a pair."""
import dataclasses

import numpy as np
import pytest

import synth
from oracle import nolsm as o
from paper_2104_08245_amd import _lib as L

pytestmark = pytest.mark.gpu

# FP64 parity bound; 16-bit rounding of the sign iterate on the others
ROUTES = [("fp64", {}, 1e-10),
          ("fp16", dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32), 5e-3),
          ("fp16", dict(sym_sign=1, inverse=L.INV_CHOLESKY_FP32), 5e-3),
          ("bf16", dict(inverse=L.INV_CHOLESKY_FP32), 4e-2)]


def run(s, prec, kw):
    import torch
    from paper_2104_08245_amd import Solver
    sv = Solver(s, prec=prec, **kw)
    sv.run()
    torch.cuda.synchronize()
    return sv


# full cells: 60 (one panel), 126 (two), 180 (three), 252 (four), 318 rows (five)
@pytest.mark.parametrize("nmol", [10, 21, 30, 42, 53])
@pytest.mark.parametrize("prec,kw,tol", ROUTES)
def test_factor_by_panel_pairs(nmol, prec, kw, tol):
    s = synth.water_cube(nmol, 2.2, config_id=123)
    sv = run(s, prec, kw)
    ref = o.nolsm(s, molecules=[0, nmol - 1])
    assert np.all(sv.host_stats()["status"] == L.MOL_OK)
    dc = sv.host_dcols()
    for J in (0, nmol - 1):
        assert np.linalg.norm(dc[J] - ref.Dcols[J]) <= tol * np.linalg.norm(ref.Dcols[J]), J
    # the last rows of S made indefinite: the pivot fails in the last panel,
    # which is the first or the second of its pair
    val = s.S.val.copy()
    last = int(s.S.row_ptr[nmol] - 1)   # block (nmol - 1, nmol - 1) of a full cell
    assert s.S.col_idx[last] == nmol - 1
    val[last] -= 5.0 * np.eye(6)
    bad = dataclasses.replace(s, S=dataclasses.replace(s.S, val=val))
    sv = run(bad, prec, kw)
    assert np.all(sv.host_stats()["status"] == L.MOL_NOT_SPD)
    assert not np.any(sv.host_D())
