"""nolsm_sign_batch_noalloc from several streams: the calls share one workspace
array and nothing waits between them, so each has to start after the one
before; every result equals nolsm_sign_batch's bit for bit."""
import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,route", [("fp16", dict(sym_sign=1)), ("bf16", {}), ("fp64", {})],
                         ids=["fp16-sym", "bf16", "fp64"])
def test_calls_from_several_streams_are_ordered(prec, route):
    import torch
    from paper_2104_08245_amd import Solver
    systems = [synth.water_cube(n, 0.45, config_id=140 + n) for n in (96, 64, 40)]
    want = []
    for s in systems:
        sv = Solver(s, prec=prec, **route)
        sv.run()
        torch.cuda.synchronize()
        want.append((sv.host_D(), sv.host_stats()["iters"]))
    svs = [Solver(s, prec=prec, ws_bytes=L.NOALLOC_WS_BYTES, **route) for s in systems]
    streams = [torch.cuda.Stream(), None, torch.cuda.Stream()]
    torch.cuda.synchronize()
    for rep in range(4):
        print("[gpu]", prec, rep, flush=True)
        for sv, st in zip(svs, streams[rep % 2:] + streams[:rep % 2]):
            sv.run_noalloc(stream=st)
    torch.cuda.synchronize()
    for sv, (D, iters) in zip(svs, want):
        assert np.array_equal(sv.host_D(), D) and np.array_equal(sv.host_stats()["iters"], iters)
