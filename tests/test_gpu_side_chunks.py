"""The chunks of a graph-schedule call side by side (each in a workspace region
of its own, on the call's stream and the library's) against the same chunks in
turn on one stream: bit for bit, over replays with other chemical potentials,
on the default stream and on one of the caller's, with eager work and other
solves between them, and with a workspace that has no room for it."""
import numpy as np
import pytest

from paper_2104_08245_amd import _lib as L
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    t = pytest.importorskip("torch")
    if not t.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    return t


@pytest.fixture(scope="module")
def systems(box64):
    side = 8.0 * (400 / 16384) ** 0.5   # the default slab's box with a smaller lateral area: 4 chunks
    return {"box64": box64, "slab": synth.water_slab(config_id=132, r_c=0.6, n_dense=200, n_dilute=200,
                                                     box=np.array([side, side, 16.632]))}


APPLY32 = dict(inverse=L.INV_CHOLESKY_APPLY_FP32)


@pytest.mark.parametrize("name", ["box64", "slab"])
@pytest.mark.parametrize("prec,route", [("fp16", dict(sym_sign=1, **APPLY32)), ("bf16", dict(sym_sign=1)), ("fp64", {}),
                                        ("fp16", dict(inverse=L.INV_COUPLED_NS))],
                         ids=["fp16-sym", "bf16-sym", "fp64", "fp16-coupled"])
def test_chunks_side_by_side_are_the_same(torch, systems, name, prec, route):
    from paper_2104_08245_amd import Solver
    s = systems[name]
    mus = (0.0, 0.1, -0.05, 0.0)

    def out(sv):
        torch.cuda.synchronize()
        return sv.host_D(), sv.host_stats()

    def in_turn(ws_bytes):
        ref = Solver(s, prec=prec, sched=L.SCHED_STREAM, ws_bytes=ws_bytes, **route)
        assert ref.plan.info()["nchunks"] >= 2
        want = []
        for mu in mus:
            ref.run(mu=mu)
            want.append(out(ref))
        return want, ref.ws_bytes

    want0, full = in_turn(None)
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    other = Solver(s, prec=prec, **route)
    # side by side: on the default stream, and in a graph where the call is waited for
    for ws_bytes, stream, sync in ((None, one, 0), (None, one, 1), (None, None, 0), (full + (1 << 20), one, 1),
                                   (full // 2, one, 1)):
        sv = Solver(s, prec=prec, ws_bytes=ws_bytes, sync_errors=sync, **route)
        want = in_turn(ws_bytes)[0]   # the same chunks
        for k, mu in enumerate(mus):
            print("[gpu]", name, prec, ws_bytes, stream is None, mu, flush=True)
            other.run(mu=mus[-1 - k], stream=two)   # beside it
            sv.run(mu=mu, stream=stream)
            for (D, st), (D0, st0) in ((out(sv), want[k]), (out(other), want0[-1 - k])):
                assert np.array_equal(D, D0)
                for key in ("iters", "status", "resid", "trace_SD", "energy_KD"):
                    assert np.array_equal(st[key], st0[key]), key
