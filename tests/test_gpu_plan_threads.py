"""Two host threads on one plan, each with a workspace and outputs of its own:
one launches the chunks side by side directly (default stream), the other
captures them side by side, anew for every call. The chunks' streams belong to
one of them until its launches, or its capture, are done."""
import threading

import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,route", [("fp16", dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32)), ("fp64", {})],
                         ids=["fp16-sym", "fp64"])
def test_two_threads(box64, prec, route):
    import torch
    from paper_2104_08245_amd import Solver
    a = Solver(box64, prec=prec, **route)
    b = Solver(box64, prec=prec, sync_errors=1, **route)
    b.plan = a.plan
    assert a.plan.info()["nchunks"] >= 2
    a.run()
    torch.cuda.synchronize()
    want = a.host_D()
    stream, failed = torch.cuda.Stream(), []

    def work(sv, st, n):
        try:
            for k in range(n):
                if st is not None:
                    sv.set_opts(switch_theta=0.7 - 1e-9 * (k + 1))
                sv.run(stream=st)
                if k % 3 == 0:
                    torch.cuda.current_stream().synchronize() if st is None else st.synchronize()
        except Exception as e:   # noqa: BLE001
            failed.append(e)

    print("[gpu] two threads on one plan", prec, flush=True)
    threads = [threading.Thread(target=work, args=(a, None, 30)), threading.Thread(target=work, args=(b, stream, 30))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not failed, failed
    assert np.array_equal(a.host_D(), want) and np.array_equal(b.host_D(), want)
