"""nolsm_sign_batch_noalloc from more streams and threads than the library
has arrays for them: a call does not wait for one on another stream while there
is an array for each, and whichever a call gets, its results are nolsm_sign_batch's
bit for bit."""
import threading

import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu

APPLY32 = dict(sym_sign=1, inverse=L.INV_CHOLESKY_APPLY_FP32)


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    return t


def solver(nmol, prec, r_c=0.45, **kw):
    from paper_2104_08245_amd import Solver
    return Solver(synth.water_cube(nmol, r_c, config_id=150 + nmol), prec=prec, ws_bytes=L.NOALLOC_WS_BYTES, **kw)


def result(sv):
    return sv.host_D(), sv.host_stats()["iters"]


def same(sv, want):
    return all(np.array_equal(a, b) for a, b in zip(result(sv), want))


def reference(torch, sv):
    sv.run()
    torch.cuda.synchronize()
    want = result(sv)
    sv.D.fill_(float("nan"))
    torch.cuda.synchronize()
    return want


def test_a_call_does_not_wait_for_another_stream(torch):
    svs = [solver(n, "fp16", **APPLY32) for n in (40, 32, 25)]
    want = [reference(torch, sv) for sv in svs]
    streams = [torch.cuda.Stream() for _ in svs]
    for sv, st in zip(svs, streams):
        sv.run_noalloc(stream=st)
    torch.cuda.synchronize()
    # about 0.4 s of one spinning wave on the first stream, from a measured rate
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    torch.cuda._sleep(1_000_000)
    e1.record()
    torch.cuda.synchronize()
    cycles = int(1_000_000 * 400.0 / max(e0.elapsed_time(e1), 1e-2))
    print("[gpu] noalloc behind", cycles, "cycles on another stream", flush=True)
    ends = [torch.cuda.Event() for _ in svs]
    with torch.cuda.stream(streams[0]):
        torch.cuda._sleep(cycles)
    for sv, st, end in zip(svs, streams, ends):
        sv.run_noalloc(stream=st)
        end.record(st)
    # (two others: one of them may share the first one's hardware queue)
    while not any(e.query() for e in ends):
        pass
    first = ends[0].query()
    torch.cuda.synchronize()
    assert not first
    assert all(same(sv, w) for sv, w in zip(svs, want))


def test_more_streams_than_arrays(torch):
    # plans of a few and of all bytes of an array, one and several chunks
    svs = [solver(96, "fp16", **APPLY32), solver(20, "fp64"), solver(64, "fp64", 0.6), solver(40, "bf16"),
           solver(25, "fp32"), solver(53, "fp16", inverse=L.INV_COUPLED_NS)]
    want = [reference(torch, sv) for sv in svs]
    streams = [None] + [torch.cuda.Stream() for _ in svs[1:]]
    for rep in range(6):
        print("[gpu] noalloc, six streams", rep, flush=True)
        order = range(len(svs)) if rep % 2 else reversed(range(len(svs)))
        for k in order:
            svs[k].run_noalloc(stream=streams[(k + rep) % len(svs)] if rep < 3 else streams[k])
            if rep < 3:   # the solver's own outputs, from another stream next
                torch.cuda.synchronize()
    torch.cuda.synchronize()
    assert all(same(sv, w) for sv, w in zip(svs, want))


def test_threads(torch):
    svs = [solver(n, prec, **kw) for n, prec, kw in ((64, "fp16", APPLY32), (40, "fp64", {}), (32, "bf16", {}),
                                                     (25, "fp32", {}), (20, "fp16", {}))]
    want = [reference(torch, sv) for sv in svs]
    good = [0] * len(svs)

    def work(k):
        st = torch.cuda.Stream()
        for rep in range(8):
            svs[k].run_noalloc(stream=st)
            if rep % 3 == 2:
                st.synchronize()
        st.synchronize()
        good[k] = same(svs[k], want[k])

    print("[gpu] noalloc, five threads", flush=True)
    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(svs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(good)


def test_replays_of_a_captured_call_between_direct_calls(torch):
    svs = [solver(64, "fp16", **APPLY32), solver(40, "fp64"), solver(32, "bf16"), solver(25, "fp32")]
    want = [reference(torch, sv) for sv in svs]
    streams = [torch.cuda.Stream() for _ in svs]
    svs[0].run_noalloc(stream=streams[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=streams[0]):
        svs[0].run_noalloc(stream=streams[0])
    for rep in range(5):
        print("[gpu] noalloc replay", rep, flush=True)
        svs[0].D.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(streams[0]):
            g.replay()
        torch.cuda.synchronize()
        for sv, st in zip(svs[1:], streams[1:]):
            sv.run_noalloc(stream=st)
        torch.cuda.synchronize()
        assert all(same(sv, w) for sv, w in zip(svs, want)), rep
