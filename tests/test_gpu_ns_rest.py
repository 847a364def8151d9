"""The late iterations of the sign iteration, which one launch runs to their
end, against the launch-per-half persistent schedule: the same tiles in the
same order of sums, so every output is equal bit for bit. The iteration counts
lie around the first iteration of that launch (16 in 16 bits, 22 in FP64 and
FP32) and at max_iter; the systems give it one tile, a few workgroups per
submatrix, and more tasks than workgroups."""
import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu

# molecules, cutoff (2.2: every submatrix is the whole matrix)
SYSTEMS = [(8, 2.2), (53, 2.2), (64, 0.6), (216, 0.9)]
ROUTES = [("fp16", dict(sym_sign=1)), ("bf16", dict(sym_sign=1)), ("fp16", {}), ("fp64", {}), ("fp32", {})]


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    return t


@pytest.mark.parametrize("nmol,cutoff", SYSTEMS)
@pytest.mark.parametrize("prec,route", ROUTES, ids=lambda v: v if isinstance(v, str) else "sym" if v else "plain")
def test_rest_of_the_iteration_is_the_same(torch, nmol, cutoff, prec, route):
    from paper_2104_08245_amd import Solver
    s = synth.water_cube(nmol, cutoff, config_id=130)
    for kw in (dict(fixed_iters=15), dict(fixed_iters=17), dict(fixed_iters=21), dict(fixed_iters=23),
               dict(fixed_iters=30), dict(max_iter=24, fixed_iters=25), dict(max_iter=17, fixed_iters=17)):
        out = []
        for sched in (L.SCHED_PERSISTENT, L.SCHED_STREAM, L.SCHED_GRAPH):
            print("[gpu]", nmol, cutoff, prec, route, kw, sched, flush=True)
            sv = Solver(s, prec=prec, sched=sched, **route, **kw)
            stream = torch.cuda.Stream()
            for _ in range(2):
                sv.run(stream=stream)
                torch.cuda.synchronize()
                out.append((sv.host_D(), sv.host_stats()))
        assert out[0][1]["iters"].max() == min(kw["fixed_iters"], kw.get("max_iter", 40) - 1)
        for D, st in out[1:]:
            assert np.array_equal(D, out[0][0], equal_nan=True), kw
            for key in ("iters", "status", "fallback", "resid", "trace_SD", "energy_KD"):
                assert np.array_equal(st[key], out[0][1][key], equal_nan=True), (kw, key)
