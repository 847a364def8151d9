"""The restart from the Gershgorin scale in the late iterations, which scanning
launches run (from 16 on in 16 bits, 18 in FP64 and FP32), or one launch to the
end in a small chunk (from 16 and 22): the restarted molecule's result, and
every output bit for bit against the persistent schedule, which has a launch
for each half. A small first scale keeps the iteration going until then."""
import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu

J = 11
# precision, options, first scale, iterations to restart at, error bound of the
# owned columns (those of the parity tests)
ROUTES = {"fp16-sym": ("fp16", dict(sym_sign=1), 1e-3, (17, 19), 5e-3),
          "fp16-sym-fp32": ("fp16", dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32), 1e-3, (17,), 5e-3),
          "bf16-sym": ("bf16", dict(sym_sign=1), 1e-3, (17,), 4e-2),
          "fp16": ("fp16", {}, 1e-3, (16, 18), 5e-3),
          "fp64": ("fp64", {}, 1e-5, (19, 23), 1e-10),
          "fp32": ("fp32", {}, 1e-5, (19, 23), 1e-4)}


@pytest.fixture(scope="module")
def systems(box64):
    # the first is a small chunk, the second above the limit of the one launch
    return {"box64": box64, "cube216": synth.water_cube(216, 0.9, config_id=134)}


@pytest.fixture(scope="module")
def exact(systems):
    from paper_2104_08245_amd import Solver
    out = {}
    for name, s in systems.items():
        sv = Solver(s, prec="fp64")
        sv.run()
        out[name] = sv.host_dcols()[J]
    return out


@pytest.mark.parametrize("name", ["box64", "cube216"])
@pytest.mark.parametrize("route", list(ROUTES))
def test_restart_in_the_late_launches(systems, exact, name, route):
    import torch
    from paper_2104_08245_amd import Solver
    prec, kw, scale, its, tol = ROUTES[route]
    plain = Solver(systems[name], prec=prec, **kw)
    plain.run()
    need = int(plain.host_stats()["iters"][J])   # iterations from the Gershgorin scale
    for it in its:
        fits = it + 1 + need < plain.opts.max_iter   # else the slots run out
        out = []
        for sched in (L.SCHED_PERSISTENT, L.SCHED_STREAM, L.SCHED_GRAPH):
            sv = Solver(systems[name], prec=prec, sched=sched, debug_scale_mult=scale, debug_force_stall=J,
                        debug_stall_it=it, **kw)
            stream = torch.cuda.Stream()
            for _ in range(2):
                print("[gpu]", name, route, it, sched, flush=True)
                sv.run(stream=stream)
                torch.cuda.synchronize()
                out.append((sv.host_D(), sv.host_stats(), sv.host_dcols()[J]))
        for D, st, dc in out:
            print("[gpu] iterations", st["iters"][J], "after", it, "and", need, flush=True)
            assert st["fallback"][J] == 1
            assert st["status"][J] == (L.MOL_OK if fits else L.MOL_NOCONV)
            if fits:
                assert st["iters"][J] == it + 1 + need
                assert np.linalg.norm(dc - exact[name]) <= tol * np.linalg.norm(exact[name])
            assert np.array_equal(D, out[0][0], equal_nan=True)
            for key in ("iters", "status", "fallback", "scale", "resid", "trace_SD", "energy_KD"):
                assert np.array_equal(st[key], out[0][1][key], equal_nan=True), key
