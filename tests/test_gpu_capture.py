"""Calls captured into a graph find the sources, receivers and sponge that are registered when
the graph is replayed (needs an MI355X)."""

import numpy as np
import pytest

import workloads
from gpu_util import say

pytestmark = pytest.mark.gpu

T = 8


def _registrations(shape):
    """(sources, receivers, sponge) that take each other's place: as many sources as travel
    with a launch and more, none, two at one point; more receivers, fewer, none."""
    mid, zero = tuple(n // 2 for n in shape[::-1]), (0,) * len(shape)
    line = [(x,) + mid[1:] for x in range(0, shape[-1], 2)]
    column = [mid[:-1] + (z,) for z in range(shape[0])]
    return [([mid], line, None), ([zero, mid], line + column + [mid, mid], None), ([], column[:3], (3, 0.05)),
            ([mid, zero, mid], [zero] + line, None), ([zero], [], None), ([mid], column, (2, 0.03))]


def _register(p, wav, reg):
    sources, rec, sponge = reg
    p.clear_sources()
    for k, pos in enumerate(sources):
        p.inject(wav[k], pos, 1e3)
    p.set_damping(*(sponge or (0, 0.0)))
    return p.record(np.array(rec).reshape(len(rec), p.ndim), T)


def _setup(oracle_mod, shape, r, dtype, tuning=None):
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    tdt = torch.float32 if dtype == "f32" else torch.float64
    v = torch.tensor(workloads.layered_velocity(shape, seed=r), dtype=tdt, device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(r)
    u0 = torch.randn(shape, generator=gen, dtype=tdt, device="cuda")
    wav = torch.randn((3, T), generator=gen, dtype=tdt, device="cuda")
    dt = 0.4 * oracle_mod.dt_max(len(shape), r, 10.0, float(v.max()))
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    if tuning is not None:
        F.fd_set_tuning(dtype, r, len(shape), tuning)
    try:
        p = Propagator(v, r, 10.0, dt, dtype, max_sources=3, max_receivers=4 * sum(shape), stream=stream)
    finally:
        F.fd_set_tuning(dtype, r, len(shape), -1)
    return p, u0, wav, stream


@pytest.mark.parametrize("shape,r,dtype,tuning", [
    ((21, 19, 70), 4, "f32", None), ((21, 19, 70), 4, "f32", 1), ((21, 19, 70), 4, "f32", 12), ((11, 20, 37), 8, "f64", None),
    ((60, 131), 4, "f32", None), ((33, 70), 8, "f64", 0), ((256, 256, 256), 4, "f32", None)])
def test_replayed_steps_follow_registrations(oracle_mod, shape, r, dtype, tuning):
    # fd_step and fd_step_record captured once, with the library's tile, tiles set by hand and
    # the stand-in build, in 2-D too: a replay does what the eager call does, whatever is
    # registered by then
    import torch

    from paper_1410_1387_amd import fdwave as F

    p, u0, wav, stream = _setup(oracle_mod, shape, r, dtype, tuning)
    say(f"captured steps {shape} {dtype}: {p.kernel_config}")
    with torch.cuda.stream(stream):
        regs = _registrations(shape)
        _register(p, wav, regs[0])
        f = [p.new_field() for _ in range(3)]

        def start(reg):
            p.set_state(u0, 0.5 * u0, 0)
            p.save_padded(f[0], f[1])
            return _register(p, wav, reg)

        def calls(explicit):
            if explicit:
                F.fd_step_record(p.ctx, f[0], f[1], f[2], 0)
                F.fd_step_record(p.ctx, f[2], f[0], f[1], 1)
            else:
                p.step(T)

        for explicit in (False, True):
            start(regs[0])
            p.sync()
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                calls(explicit)
            for reg in regs + regs[:1]:
                got = []
                for replay in (False, True, True):
                    traces = start(reg)
                    g.replay() if replay else calls(explicit)
                    got.append([x.clone() for x in (*(f[1:] if explicit else p.state()[:2]), traces)])
                p.sync()
                for again in got[1:]:
                    assert all(torch.equal(a, b) for a, b in zip(got[0], again)), (explicit, reg[0], reg[2])
                assert not reg[1] or float(got[0][2].abs().max()) > 0


@pytest.mark.parametrize("shape,r,dtype", [((13, 22, 70), 4, "f32"), ((60, 131), 3, "f64")])
def test_replayed_adjoint_follows_receivers(oracle_mod, shape, r, dtype):
    # fd_adjoint_segment captured once: a replay takes the receivers, and the row length of
    # their residual, that are registered by then
    import torch

    from paper_1410_1387_amd import fdwave as F

    p, u0, wav, stream = _setup(oracle_mod, shape, r, dtype)
    say(f"captured adjoint {shape} {dtype}: {p.adjoint_config}")
    with torch.cuda.stream(stream):
        regs = [reg for reg in _registrations(shape) if reg[2] is None]
        n = p.new_field().numel()
        resid = torch.randn(T * 4 * sum(shape), dtype=p.tdtype, device="cuda")
        cur, prev, mu, g, gs = p.new_field(), p.new_field(), torch.zeros(2 * n, dtype=p.tdtype, device="cuda"), \
            p.new_field(), p.new_field()
        ring = torch.zeros((T - 1) * n, dtype=p.tdtype, device="cuda")
        p.set_state(u0, 0.5 * u0, 0)
        p.save_padded(cur, prev)

        def call():
            F.fd_adjoint_segment(p.ctx, cur, prev, 0, T, ring, mu, resid, 0.5, g, gs)

        _register(p, wav, regs[0])
        p.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            call()
        for reg in regs + regs[:1]:
            got = []
            for replay in (False, True, True):
                _register(p, wav, reg)
                mu.zero_()
                g.zero_()
                graph.replay() if replay else call()
                got.append((mu.clone(), g.clone()))
            p.sync()
            assert all(torch.equal(a, b) for again in got[1:] for a, b in zip(got[0], again)), reg[0]
            assert bool(reg[1]) == (float(got[0][1].abs().max()) > 0)


@pytest.mark.parametrize("shape,rxy,rz,dtype", [((19, 22, 70), 4, 2, "f32"), ((21, 17, 40), 12, 8, "f64")])
def test_replayed_vti_steps_follow_registrations(shape, rxy, rz, dtype):
    # fd_vti_step captured once: a replay finds the sources and receivers registered by then
    import torch

    from paper_1410_1387_amd.vti import VtiPropagator

    tdt = torch.float32 if dtype == "f32" else torch.float64
    vz = torch.tensor(workloads.layered_velocity(shape, seed=3), dtype=tdt, device="cuda")
    dt = 0.4 * VtiPropagator.dt_max(rxy, rz, 10.0, shape[0], float(vz.max()), 0.2, 0.1)
    gen = torch.Generator(device="cuda").manual_seed(rz)
    u0 = [torch.randn(shape, generator=gen, dtype=tdt, device="cuda") for _ in range(4)]
    wav = torch.randn((3, T), generator=gen, dtype=tdt, device="cuda")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    regs = [reg for reg in _registrations(shape) if reg[2] is None]
    say(f"captured VTI steps {shape} {dtype}")
    with torch.cuda.stream(stream):
        p = VtiPropagator(vz, 0.2, 0.1, rxy, rz, 10.0, dt, None, dtype, max_sources=3, max_receivers=4 * sum(shape),
                          stream=stream)
        for sources in (1, 2, 3):  # added between replays
            if sources == 1:
                p.inject(wav[0], regs[0][0][0], 1e3, 300.0)
                p.record(np.array(regs[0][1]), T, record_q=True)
                p.sync()
                g = torch.cuda.CUDAGraph()
                with torch.cuda.graph(g, stream=stream):
                    p.step(T)
            else:
                p.inject(wav[sources - 1], (0, 0, 0) if sources == 2 else regs[0][0][0], 1e3, 300.0)
            for rec in (regs[0][1], regs[1][1], [], regs[2][1][:3]):
                got = []
                for replay in (False, True, True):
                    p.set_state(*u0, 0)
                    traces = p.record(np.array(rec).reshape(len(rec), 3), T, record_q=True)
                    g.replay() if replay else p.step(T)
                    got.append([x.clone() for x in (*p.state(), *traces)])
                for again in got[1:]:
                    assert all(torch.equal(a, b) for a, b in zip(got[0], again)), (sources, len(rec))
                assert not rec or float(got[0][4].abs().max()) > 0
