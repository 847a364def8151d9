"""A plan's workspace layout belongs to the schedule it was configured for: the
pipeline, which runs the setup of a chunk beside the solve of the one before,
refuses a plan whose chunks share their bytes. Host-side checks, before any
kernel is launched."""
import ctypes as C

import pytest

from paper_2104_08245_amd import _lib as L
import synth


def call(p, opts, stream):
    """(code, message) of a solve on an unbound plan: it never gets to its
    pointers, which stand for device memory"""
    fake = C.c_void_p(1 << 20)
    rc = L.lib().nolsm_sign_batch(p.h, fake, fake, 0.0, C.byref(opts), fake, 1 << 40, fake, None, fake, stream)
    return rc, L.lib().nolsm_strerror(rc).decode()


@pytest.mark.parametrize("sched,ws_bytes", [(L.SCHED_GRAPH, 32 << 20), (L.SCHED_STREAM, 32 << 20),
                                            (L.SCHED_STREAM, 1 << 30), (L.SCHED_PERSISTENT, 1 << 30)])
def test_pipeline_refuses_plans_whose_chunks_share_bytes(box64, sched, ws_bytes):
    from paper_2104_08245_amd import Plan
    s = box64
    p = Plan(s.K.nb, s.K.bs, s.K.row_ptr, s.K.col_idx)
    stream = C.c_void_p(1 << 20)
    opts = L.default_opts("fp16", sched=sched)
    p.configure(opts, ws_bytes)
    assert p.info()["nchunks"] >= 2
    opts.sched = L.SCHED_PIPELINE
    rc, msg = call(p, opts, stream)
    assert rc == L.E_STATE and "pipeline" in msg
    # in turn, as on the null stream and with phase times, they serve any layout
    for o, st in ((L.default_opts("fp16", sched=L.SCHED_PIPELINE), None),
                  (L.default_opts("fp16", sched=L.SCHED_PIPELINE, profile=1), stream),
                  (L.default_opts("fp16", sched=L.SCHED_GRAPH), stream)):
        rc, msg = call(p, o, st)
        assert rc == L.E_STATE and msg.endswith("not bound")


def test_pipeline_takes_chunks_in_regions_of_their_own(box64):
    from paper_2104_08245_amd import Plan
    s = box64
    p = Plan(s.K.nb, s.K.bs, s.K.row_ptr, s.K.col_idx)
    stream = C.c_void_p(1 << 20)
    for sched, ws_bytes in ((L.SCHED_PIPELINE, 32 << 20), (L.SCHED_PIPELINE, 1 << 30)):
        p.configure(L.default_opts("fp16", sched=sched), ws_bytes)
        assert p.info()["nchunks"] >= 2
        rc, msg = call(p, L.default_opts("fp16", sched=L.SCHED_PIPELINE), stream)
        assert rc == L.E_STATE and msg.endswith("not bound")
    # one chunk has nothing to share: 8 molecules within one cutoff
    s = synth.water_cube(8, 2.2, config_id=1)
    p = Plan(s.K.nb, s.K.bs, s.K.row_ptr, s.K.col_idx)
    p.configure(L.default_opts("fp16"), 1 << 30)
    assert p.info()["nchunks"] == 1
    rc, msg = call(p, L.default_opts("fp16", sched=L.SCHED_PIPELINE), stream)
    assert rc == L.E_STATE and msg.endswith("not bound")
