"""The graph schedule launches small chunks of different submatrix sizes
together, the stream and persistent schedules each by itself: the same results
bit for bit, in fewer launches. The slab mixes tile classes in one launch (64
and 128 rows; FP64 and FP32 tasks of one and of two tiles), the combined
systems submatrices with one and with several molecules."""
import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu

APPLY32 = dict(inverse=L.INV_CHOLESKY_APPLY_FP32)
CASES = [("slab", "fp64", {}), ("slab", "fp32", {}), ("slab", "fp16", {}), ("slab", "bf16", dict(sym_sign=1)),
         ("slab", "fp16", dict(sym_sign=1, **APPLY32)), ("slab", "fp16", dict(inverse=L.INV_COUPLED_NS)),
         ("combine", "fp16", dict(sym_sign=1, **APPLY32)), ("combine", "fp64", {})]


@pytest.fixture(scope="module")
def systems():
    side = 8.0 * (400 / 16384) ** 0.5
    return {"slab": synth.water_slab(config_id=132, r_c=0.6, n_dense=200, n_dilute=200,
                                     box=np.array([side, side, 16.632])),
            "combine": synth.water_cube(200, 0.7, config_id=133)}


@pytest.mark.parametrize("name,prec,route", CASES)
def test_shared_launches_are_the_same(systems, name, prec, route):
    import torch
    from paper_2104_08245_amd import Solver
    out, launches, chunks = [], [], []
    for sched in (L.SCHED_STREAM, L.SCHED_GRAPH, L.SCHED_PERSISTENT):
        sv = Solver(systems[name], prec=prec, combine=name == "combine", sched=sched, **route)
        chunks.append(sv.plan.info()["nchunks"])
        stream = torch.cuda.Stream()
        for mu in (0.0, 0.1, 0.0):
            print("[gpu]", name, prec, route, sched, mu, flush=True)
            sv.run(mu=mu, stream=stream)
            torch.cuda.synchronize()
            out.append((mu, sv.host_D(), sv.host_stats()))
        sv.set_opts(profile=1)
        sv.run(mu=0.0)
        launches.append(sv.profile()["n_ns_launches"])
    assert chunks[0] == chunks[1] == chunks[2] >= 2
    assert launches[1] < launches[0]
    for k, (mu, D, st) in enumerate(out[3:]):
        assert np.array_equal(D, out[k % 3][1])
        for key in ("iters", "status", "resid", "trace_SD", "energy_KD"):
            assert np.array_equal(st[key], out[k % 3][2][key]), key
