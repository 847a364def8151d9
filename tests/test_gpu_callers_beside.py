"""Searches, waited solves, solves on the default stream and on others, and
allocation-free ones, from a thread each at the same time: the results that each
gives by itself, bit for bit."""
import threading

import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L

pytestmark = pytest.mark.gpu

SYM = dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32)
JOBS = [("search", "fp16", SYM), ("search", "fp64", {}), ("sync", "fp16", SYM), ("default", "bf16", dict(sym_sign=1)),
        ("stream", "fp32", {}), ("noalloc", "fp16", dict(SYM, ws_bytes=L.NOALLOC_WS_BYTES))]
KEYS = ("iters", "status", "resid", "trace_SD", "energy_KD")


def out(sv):
    st = sv.host_stats()
    return [sv.host_D()] + [st[k] for k in KEYS]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def test_beside_other_callers(box64):
    import torch
    from paper_2104_08245_amd import Solver
    jobs = []   # (a caller's step, solver, stream, its result alone)
    for how, prec, kw in JOBS:
        sv = Solver(box64, prec=prec, sync_errors=int(how == "sync"), **kw)
        st = None if how == "default" else torch.cuda.Stream()
        step = {"search": lambda sv=sv, st=st: sv.mu_bisect(-3.0, 1.0, 256.0, stream=st, allow_noconv=True),
                "noalloc": lambda sv=sv, st=st: sv.run_noalloc(stream=st)}.get(
                    how, lambda sv=sv, st=st: sv.run(stream=st))
        step()
        torch.cuda.synchronize()
        jobs.append((step, sv, st, out(sv)))
    good = [False] * len(jobs)

    def work(k):
        step, sv, st, _ = jobs[k]
        for rep in range(10):
            step()
            if rep % 3 == 2:
                (torch.cuda.current_stream() if st is None else st).synchronize()
        (torch.cuda.current_stream() if st is None else st).synchronize()
        good[k] = True

    print("[gpu] six callers", flush=True)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert all(good)
    assert [same(out(sv), want) for _, sv, _, want in jobs] == [True] * len(jobs)
