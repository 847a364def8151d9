"""A search for the chemical potential and plain solves in turn on one solver
and stream: they replay one captured graph, and every result is the one that a
fresh solver gives, bit for bit."""
import time

import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu

ROUTES = [("fp16", dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32)), ("fp64", {})]


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    return t


@pytest.mark.parametrize("prec,route", ROUTES, ids=["fp16-sym", "fp64"])
def test_alternating(torch, box64, prec, route):
    from paper_2104_08245_amd import Solver

    def search(sv, stream):
        return sv.mu_bisect(-3.0, 1.0, 4.0 * 64, stream=stream, allow_noconv=True)

    def out(sv):
        torch.cuda.synchronize()
        st = sv.host_stats()
        return [sv.host_D()] + [st[k] for k in ("iters", "status", "resid", "trace_SD", "energy_KD")]

    stream = torch.cuda.Stream()
    sv = Solver(box64, prec=prec, **route)
    assert sv.plan.info()["nchunks"] >= 2
    found = search(Solver(box64, prec=prec, **route), stream)
    fresh = Solver(box64, prec=prec, **route)
    fresh.run(mu=found[0], stream=stream)
    want = out(fresh)
    for rep in range(4):
        print("[gpu] search and solve", prec, rep, flush=True)
        assert search(sv, stream) == found
        assert all(np.array_equal(a, b) for a, b in zip(out(sv), want))
        sv.D.fill_(float("nan"))
        torch.cuda.synchronize()
        sv.run(mu=found[0], stream=stream)
        assert all(np.array_equal(a, b) for a, b in zip(out(sv), want))

    # host time of a solve's call: a replay, one after a search, and one where
    # another option has the graph captured anew
    def host(before):
        took = []
        for k in range(20):
            before(k)
            torch.cuda.synchronize()
            t = time.perf_counter()
            sv.run(stream=stream)
            took.append(time.perf_counter() - t)
            torch.cuda.synchronize()
        return min(took)

    replay = host(lambda k: None)
    after_search = host(lambda k: search(sv, stream))
    anew = host(lambda k: sv.set_opts(switch_theta=0.7 - 1e-9 * (k + 1)))
    print(f"[gpu] host time of a call: replay {replay * 1e6:.0f} us, after a search {after_search * 1e6:.0f} us, "
          f"captured {anew * 1e6:.0f} us", flush=True)
    assert after_search < (replay + anew) / 2
