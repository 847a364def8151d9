"""The FP64 and FP32 sign iterations at the edges of their tiles: one and
several 64-row tiles, pairs of column tiles with and without a last single
one, chunks on either side of the switch to the wider tasks, the restart, the
scanning and the persistent launches. Full cells (every submatrix is the whole
matrix), against the oracle."""
import numpy as np
import pytest

import synth
from oracle import nolsm as o
from paper_2104_08245_amd import _lib as L

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-10, "fp32": 1e-4}   # the bounds of the parity tests on Dcols


# molecules -> rows (64-row tiles, tasks of two): 60 (1), 126 (2), 192 (3),
# 324 (6; 972 tasks, narrow), 342 (6; 1026, wide), 390 (7; 1820, wide)
@pytest.mark.parametrize("nmol", [10, 21, 32, 54, 57, 65])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_fp64_fp32_iteration_at_tile_edges(nmol, prec):
    import torch
    from paper_2104_08245_amd import Solver
    s = synth.water_cube(nmol, 2.2, config_id=121)
    mols = [0, nmol - 1]
    ref = o.nolsm(s, molecules=mols)
    first = None
    for kw in ({}, {"sched": L.SCHED_PERSISTENT}, {"debug_force_stall": 0}, {"max_iter": 24}):
        sv = Solver(s, prec=prec, **kw)
        stream = torch.cuda.Stream()
        sv.run(stream=stream)
        sv.run(stream=stream)
        torch.cuda.synchronize()
        st, dc = sv.host_stats(), sv.host_dcols()
        assert np.all(st["status"] == 0), (kw, st["status"])
        for J in mols:
            err = np.linalg.norm(dc[J] - ref.Dcols[J]) / np.linalg.norm(ref.Dcols[J])
            assert err <= TOL[prec], (kw, J, err)
        if "debug_force_stall" in kw:
            # the same matrix for every molecule: the restart at iteration 2
            # costs the first one three steps
            assert st["fallback"][0] == 1 and st["iters"][0] == st["iters"][1] + 3
        D = sv.host_D()
        if first is None:
            first = D
        elif "debug_force_stall" not in kw:
            assert np.array_equal(D, first), kw
