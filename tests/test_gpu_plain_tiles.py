"""The general 16-bit tile product at the edges of its tiles, in the iteration
on A_J and in the coupled Newton-Schulz inverse: one, several and half-filled
tiles per side, 64- and 128-row tiles, the scanning and the persistent
launches. Full cells (every submatrix is the whole matrix), against the
oracle."""
import numpy as np
import pytest

import synth
from oracle import nolsm as o
from paper_2104_08245_amd import _lib as L

pytestmark = pytest.mark.gpu

TOL = {"fp16": 5e-3, "bf16": 4e-2}          # 16-bit rounding of the sign iterate
TOL_INV = {"fp16": 3e-2, "bf16": 2.5e-1}    # and of the inverse, as in the coupled route's own tests
ALL64 = (1 << 64) - 1


# molecules -> rows: 60 (one 64-row tile), 126 and 132 (either side of one
# 128-row tile), 192, 258, 318 (two and a half), 390 (three and a half)
@pytest.mark.parametrize("nmol", [10, 21, 22, 32, 43, 53, 65])
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
@pytest.mark.parametrize("inverse", [L.INV_CHOLESKY, L.INV_COUPLED_NS])
def test_general_product_at_tile_edges(nmol, prec, inverse):
    import torch
    from paper_2104_08245_amd import Solver
    s = synth.water_cube(nmol, 2.2, config_id=122)
    mols = [0, nmol - 1]
    ref = o.nolsm(s, molecules=mols)
    tol = TOL_INV if inverse == L.INV_COUPLED_NS else TOL
    first = None
    for kw in ({}, {"ns_small_tile_mask": 0}, {"ns_small_tile_mask": ALL64}, {"sched": L.SCHED_PERSISTENT}):
        sv = Solver(s, prec=prec, inverse=inverse, **kw)
        stream = torch.cuda.Stream()
        sv.run(stream=stream)
        sv.run(stream=stream)
        torch.cuda.synchronize()
        st, dc = sv.host_stats(), sv.host_dcols()
        assert np.all(st["status"] == 0), (kw, st["status"])
        for J in mols:
            err = np.linalg.norm(dc[J] - ref.Dcols[J]) / np.linalg.norm(ref.Dcols[J])
            assert err <= tol[prec], (kw, J, err)
        # the tile size and the launches change neither the products nor
        # their order
        D = sv.host_D()
        if first is None:
            first = D
        else:
            assert np.array_equal(D, first), kw
