"""Columns with several events -- receivers on many planes, sources among them -- over z
chunks of every kind, against the oracle (needs an MI355X).  Tolerances are those of the
other comparisons with it: FP32 1e-4, FP64 1e-11, gradients 1e-3 and 1e-9."""

import numpy as np
import pytest

import workloads
from gpu_util import rel_l2, run_gpu, say

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "f64": 1e-11}
KINDS = ["every plane", "sparse", "gap", "many at a point"]


def _events(kind, shape):
    """(receivers, source points): columns in the middle of a tile, next to each other, in the
    first and in the last cell of the grid, which the list ends with."""
    nz, base = shape[0], tuple(n // 2 for n in shape[:0:-1])
    last = tuple(n - 1 for n in shape[:0:-1])
    side = (base[0] + 1,) + base[1:]
    if kind == "every plane":
        rec = [c + (z,) for c in (base, last) for z in range(nz)]
    elif kind == "sparse":  # the steps between a column's events differ, their order is mixed
        rec = [c + (z,) for k, c in enumerate((base, side, last)) for z in range(k, nz, 5 + 2 * k)][::-1]
    elif kind == "gap":  # nothing between the first planes and the last two
        rec = [c + (z,) for c in (base, (0,) * len(base)) for z in (0, 1, 2, nz - 2, nz - 1)]
    else:
        rec = [base + (z,) for z in range(2, nz - 3)] + 9 * [base + (nz // 2,)] + 3 * [last + (nz - 1,)]
    sources = [base + (z,) for z in (nz // 2, nz // 2, nz - 1, 1)] + [last + (nz - 2,)]
    return np.array(rec), sources


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape,r,dtype", [((37, 19, 70), 4, "f32"), ((37, 19, 70), 1, "f64"), ((21, 20, 45), 8, "f64"),
                                           ((41, 18, 67), 5, "f32"), ((90, 131), 4, "f32"), ((70, 140), 8, "f64")])
def test_forward(oracle_mod, kind, shape, r, dtype):
    T, ndim = 12, len(shape)
    v = workloads.layered_velocity(shape, seed=r)
    dt = 0.4 * oracle_mod.dt_max(ndim, r, 10.0, v.max())
    rec, at = _events(kind, shape)
    rng = np.random.default_rng(r)
    u0 = rng.standard_normal(shape)
    for nsrc in (1, 5):  # in the shot's descriptor, in the list
        sources = [(p, rng.standard_normal(T) * 1e6) for p in at[:nsrc]]
        ref = oracle_mod.forward(v, 10.0, dt, r, T, sources, rec, u0=u0, um1=u0)
        first = None
        for tuning in (None, (0, 1), (0, 2), (0, 5), (0, 16), (0, shape[0])):
            got = run_gpu(v, r, 10.0, dt, T, dtype, sources=sources, receivers=rec, u0=u0, um1=u0, tuning=tuning,
                          label=f"{kind}, {nsrc} sources:")
            first = got if first is None else first
            eu, et = rel_l2(got["u"], ref["u"]), rel_l2(got["traces"], ref["traces"])
            say(f"u {eu:.2e} traces {et:.2e} [{got['config']}]")
            assert eu <= TOL[dtype] and et <= TOL[dtype]
            assert np.array_equal(got["u"], first["u"]) and np.array_equal(got["traces"], first["traces"])


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-9), ("f32", 1e-3)])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("shape,r", [((37, 19, 70), 4), ((25, 20, 24), 8), ((90, 131), 2)])
def test_gradient(oracle_mod, kind, shape, r, dtype, tol):
    from test_gpu_adjoint import _gpu_gradient, _problem

    v, pb, _ = _problem(oracle_mod, shape, r, 40, 8, dtype, seed=r)
    pb.receivers = _events(kind, shape)[0]
    wav = oracle_mod.ricker(40, pb.dt, pb.f0, pb.t0)
    obs = oracle_mod.forward(1.02 * v, pb.h, pb.dt, r, 40, [(pb.source, wav)], pb.receivers)["traces"]
    say(f"{kind}: gradient {dtype} shape={shape} r={r}")
    J, g = _gpu_gradient(v, pb, obs)
    ref = oracle_mod.gradient(v, pb.h, pb.dt, r, 40, [(pb.source, wav)], pb.receivers, obs)
    say(f"  grad rel L2 {rel_l2(g, ref['grad_v']):.2e}")
    assert np.linalg.norm(ref["grad_v"]) > 0
    assert rel_l2(g, ref["grad_v"]) <= tol and abs(J - ref["J"]) <= max(tol, 1e-6) * ref["J"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("rxy,rz,dtype", [(12, 8, "f32"), (8, 4, "f32"), (4, 4, "f64"), (2, 1, "f64")])
def test_vti(oracle_mod, kind, rxy, rz, dtype):
    from test_gpu_vti import _model, run_vti_gpu

    shape, h, T = (37, 19, 70), 10.0, 10
    vz, eps, delta = _model(shape, seed=rxy)
    zc = workloads.stretched_z(shape[0], rz, h)
    dt = 0.5 * oracle_mod.vti_dt_max(rxy, rz, h, oracle_mod.z_weights(zc, rz), vz, eps, delta)
    rec, at = _events(kind, shape)
    rng = np.random.default_rng(rz)
    for nsrc in (1, 5):
        src = [(at[i], rng.standard_normal(T) * 1e6, 1.0, 0.3 * i) for i in range(nsrc)]
        ref = oracle_mod.vti_forward(vz, eps, delta, h, dt, rxy, rz, T, zc=zc, sources=src, receivers=rec)
        first = None
        for tuning in (None, (0, 1), (0, 5), (0, 37)):
            got = run_vti_gpu(vz, eps, delta, h, zc, dt, rxy, rz, T, dtype, sources=src, receivers=rec, tuning=tuning,
                              label=f"{kind}, {nsrc} sources:")
            first = got if first is None else first
            for f in ("p", "q", "traces_p", "traces_q"):
                assert rel_l2(got[f], ref[f]) <= TOL[dtype], f
                assert np.array_equal(got[f], first[f]), (f, tuning)
