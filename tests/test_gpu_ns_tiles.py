"""The symmetric 16-bit sign iteration at the edges of its tiles: one, several
and half-filled tiles per side, 64- and 128-row tiles, the fused and the
separate completion of the iterate below its diagonal tiles, the scanning and
the persistent launches. Full cells (every submatrix is the whole matrix),
against the oracle."""
import numpy as np
import pytest

from oracle import nolsm as o
from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu

# mixed-precision bound on Dcols (16-bit rounding of the iterate)
TOL = {"fp16": 5e-3, "bf16": 4e-2}
ALL64 = (1 << 64) - 1


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    return t


# molecules -> rows: 60 (one 64-row tile), 126 and 132 (either side of one
# 128-row tile), 192, 252 and 258 (either side of two), 318 (two and a half),
# 390 (three and a half), 516 (four and a half)
@pytest.mark.parametrize("nmol", [10, 21, 22, 32, 42, 43, 53, 65, 86])
@pytest.mark.parametrize("prec", ["fp16", "bf16"])
def test_symmetric_iteration_at_tile_edges(torch, nmol, prec):
    from paper_2104_08245_amd import Solver
    s = synth.water_cube(nmol, 2.2, config_id=120)
    assert int(np.diff(s.K.row_ptr).min()) == nmol
    mols = [0, nmol - 1]
    ref = o.nolsm(s, molecules=mols)
    first = None
    for kw in ({}, {"ns_small_tile_mask": 0}, {"ns_small_tile_mask": ALL64}, {"finish_rows": 1},
               {"sched": L.SCHED_PERSISTENT}, {"combine": True}):
        sv = Solver(s, prec=prec, sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32, **kw)
        stream = torch.cuda.Stream()
        sv.run(stream=stream)
        sv.run(stream=stream)
        torch.cuda.synchronize()
        st, dc = sv.host_stats(), sv.host_dcols()
        assert np.all(st["status"] == 0), (kw, st["status"])
        for J in mols:
            err = np.linalg.norm(dc[J] - ref.Dcols[J]) / np.linalg.norm(ref.Dcols[J])
            assert err <= TOL[prec], (kw, J, err)
        # the tile size and the launches change neither the products nor
        # their order
        D = sv.host_D()
        if first is None:
            first = D
        elif "finish_rows" not in kw and "combine" not in kw:
            assert np.array_equal(D, first), kw
