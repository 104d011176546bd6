"""2-D grids, whose steps share launches, against single steps and the oracle (needs an
MI355X)."""

import numpy as np
import pytest

import workloads
from gpu_util import rel_l2, say

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "f64": 1e-11}
T, START = 37, 5


def _run(shape, r, dtype, dt, calls, sources, rec, v, u0, um1, damping):
    """T steps from step START in calls of the given sizes, recorded from the second call on."""
    import torch

    from paper_1410_1387_amd import Propagator

    tdt = torch.float32 if dtype == "f32" else torch.float64

    def dev(a):
        return torch.tensor(np.asarray(a), dtype=tdt, device="cuda")

    p = Propagator(dev(v), r, 10.0, dt, dtype, max_sources=max(1, len(sources)), max_receivers=len(rec))
    if damping:
        p.set_damping(*damping)
    for pos, wav in sources:
        p.inject(dev(wav), pos)
    p.set_state(dev(u0), dev(um1), START)
    p.step(calls[0])
    traces = p.record(rec, T)
    for n in calls[1:]:
        p.step(n)
    u, u_prev, step = p.state()
    p.sync()
    assert step == START + T
    return u.cpu().numpy(), u_prev.cpu().numpy(), traces.cpu().numpy()


def _inputs(oracle_mod, shape, r, nsrc, seed):
    # sources that share a point, lie in corners, end early and (the third) end the sharing;
    # receivers on every point of two lines, on a source and twice at one point
    nz, nx = shape
    rng = np.random.default_rng(seed)
    v = workloads.layered_velocity(shape, seed=seed)
    u0 = rng.standard_normal(shape)
    dt = 0.4 * oracle_mod.dt_max(2, r, 10.0, v.max())
    at = [(nx // 2, nz // 3), (nx // 2, nz // 3), (nx - 1, nz - 1)]
    sources = [(at[i], 100.0 * rng.standard_normal(START + T - 11 * i)) for i in range(nsrc)]
    rec = [(x, nz // 2) for x in range(nx)] + [(nx // 3, z) for z in range(nz)] + [at[0], (0, 0), (0, 0), at[2]]
    return v, u0, 0.5 * u0, dt, sources, np.array(rec)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("r", range(1, 9))
def test_shared_launches_bitwise(oracle_mod, r, dtype):
    # one tile, several with remainders, and (as many tiles as choose the deep, the shallow
    # and no shared launch) larger grids; whole calls and calls of every size
    for shape, nsrc, damping in [((1, 1), 0, None), ((5, 3), 1, None), ((29, 133), 2, (6, 0.05)), ((75, 38), 2, None),
                                 ((33, 66), 3, None), ((521, 545), 1, (9, 0.03)), ((550, 1601), 1, None),
                                 ((1101, 1599), 2, None)]:
        v, u0, um1, dt, sources, rec = _inputs(oracle_mod, shape, r, nsrc, r)
        one = [1] * T
        say(f"2-D shared launches shape={shape} r={r} dtype={dtype} sources={nsrc} damping={damping}")
        want = _run(shape, r, dtype, dt, one, sources, rec, v, u0, um1, damping)
        for calls in ([T], [1, T - 1], [2, 3, 5, 9, 1, 17]):
            got = _run(shape, r, dtype, dt, calls, sources, rec, v, u0, um1, damping)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1]), (shape, calls)
            n = T - calls[0]  # rows recorded by both
            assert np.array_equal(got[2][:n], want[2][T - 1 - n:T - 1]), (shape, calls)
        if shape[0] * shape[1] > 4000:
            continue
        late = [(p, np.concatenate([w[START:], np.zeros(START + T - len(w))])) for p, w in sources]
        ref = oracle_mod.forward(v, 10.0, dt, r, T, late, rec, u0=u0, um1=um1, damping=damping)
        assert rel_l2(want[0], ref["u"]) <= TOL[dtype] and rel_l2(want[2][:T - 1], ref["traces"][1:]) <= TOL[dtype]


def test_shared_launches_under_capture(oracle_mod):
    # a captured call of several steps replays what it did, from the state it is given
    import torch

    from paper_1410_1387_amd import Propagator

    v, u0, um1, dt, sources, rec = _inputs(oracle_mod, (90, 210), 4, 1, 3)
    stream = torch.cuda.Stream()
    vd = torch.tensor(v, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    p = Propagator(vd, 4, 10.0, dt, "f32", max_receivers=len(rec), stream=stream)
    state = [torch.tensor(a, dtype=torch.float32, device="cuda") for a in (u0, um1)]
    wav = torch.tensor(sources[0][1], dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        p.inject(wav, sources[0][0])
        traces = p.record(rec, 2 * T)
        p.set_state(state[0], state[1], 0)
        p.step(20)
        want, want_tr = p.state()[0].clone(), traces.clone()
        p.sync()
        p.set_state(state[0], state[1], 0)
        p.sync()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            p.step(20)
        for _ in range(3):
            p.set_state(state[0], state[1], 20)
            traces.zero_()
            g.replay()
            assert torch.equal(p.state()[0], want)
            assert torch.equal(traces, want_tr)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_own_chunks_bitwise(oracle_mod, dtype):
    # the library's own rows per chunk (few, many short ones, and those of a grid past the
    # last-level cache) give the bits of one chunk of all rows
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    tdt = torch.float32 if dtype == "f32" else torch.float64
    for shape, r in [((3, 2000), 8), ((1203, 801), 5), ((1600, 1601), 8), ((4500, 4300), 6)]:
        say(f"2-D chunks shape={shape} r={r} dtype={dtype}")
        v = torch.full(shape, 2000.0, dtype=tdt, device="cuda")
        gen = torch.Generator(device="cuda").manual_seed(r)
        u0 = torch.randn(shape, generator=gen, dtype=tdt, device="cuda")
        got = []
        for tuning in (None, (0, shape[0])):
            if tuning:
                F.fd_set_tuning(dtype, r, 2, *tuning)
            try:
                p = Propagator(v, r, 10.0, 0.4 * oracle_mod.dt_max(2, r, 10.0, 2000.0), dtype)
            finally:
                F.fd_set_tuning(dtype, r, 2, -1, 0)
            p.set_state(u0, 0.5 * u0, 0)
            for _ in range(3):
                p.step(1)
            got.append(p.state()[0])
            p.sync()
        assert torch.equal(*got)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("shape,r", [((45, 130), 1), ((300, 420), 4), ((700, 900), 4), ((61, 77), 8), ((801, 900), 8),
                                     ((20, 24, 30), 2)])
def test_kept_states_bitwise(oracle_mod, shape, r, dtype):
    # every state kept, in one call and step by step; the adjoint of the kept states and of
    # states recomputed from a checkpoint, all with the bits of single steps
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    tdt = torch.float32 if dtype == "f32" else torch.float64
    nd = len(shape)
    v = torch.tensor(workloads.layered_velocity(shape, seed=r), dtype=tdt, device="cuda")
    dt = 0.4 * oracle_mod.dt_max(nd, r, 10.0, float(v.max()))
    nx, nz = shape[-1], shape[0]
    mid = (shape[1] // 2,) if nd == 3 else ()
    rec = np.array([(x, *mid, nz // 2) for x in range(0, nx, 3)] + [(1, *mid, z) for z in range(nz)])
    for T in (1, 2, 3, 9, 20):
        say(f"kept states shape={shape} r={r} dtype={dtype} T={T}")
        kept = []
        for whole in (True, False):
            p = Propagator(v, r, 10.0, dt, dtype, max_receivers=len(rec))
            p.inject(p.ricker(T, 30.0, 0.0), (nx // 2, *mid, nz // 3))
            traces = p.record(rec, T)
            n = p.new_field().numel()
            fields = torch.zeros((T + 1, n), dtype=tdt, device="cuda")
            gen = torch.Generator(device="cuda").manual_seed(7)
            u0 = torch.randn(shape, generator=gen, dtype=tdt, device="cuda")
            p.set_state(u0, 0.5 * u0, 0)
            p.save_padded(fields[0], fields[T])
            start = [fields[0].clone(), fields[T].clone()]
            if whole:
                F.fd_steps_record(p.ctx, fields, T)
            else:
                prev, cur = fields[T], fields[0]
                for k in range(T):
                    F.fd_step_record(p.ctx, cur, prev, fields[k + 1], k)
                    prev, cur = cur, fields[k + 1]
            resid = traces.clone()
            grads = []
            for stored in (True, False):
                mu = torch.zeros(2 * n, dtype=tdt, device="cuda")
                g = p.new_field()
                if stored:
                    F.fd_adjoint_stored(p.ctx, fields, 0, T, mu, resid, 1.0, g, None)
                else:
                    ring = torch.zeros((T, n), dtype=tdt, device="cuda")
                    F.fd_adjoint_segment(p.ctx, start[0], start[1], 0, T, ring, mu, resid, 1.0, g, None)
                grads.append(g)
            p.sync()
            assert torch.equal(*grads)
            kept.append((fields, traces, grads[0]))
        for a, b in zip(*kept):
            assert torch.equal(a, b)
        assert float(kept[0][1].abs().max()) > 0 and float(kept[0][2].abs().max()) > 0


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5])
def test_adjoint_launches_bitwise(oracle_mod, r, dtype):
    # adjoint steps that share launches against the tile set by hand, which steps alone: one tile and less, remainders, the larger grids' tiles; receivers
    # in corners, on lines and several at one point; segments of every length, their images
    # summed directly and by segment
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    tdt = torch.float32 if dtype == "f32" else torch.float64
    steps = 21
    for shape in [(1, 1), (6, 3), (33, 133), (70, 38), (801, 1203), (270, 265)]:
        nz, nx = shape
        say(f"2-D adjoint launches shape={shape} r={r} dtype={dtype}")
        v = torch.tensor(workloads.layered_velocity(shape, seed=r), dtype=tdt, device="cuda")
        rec = np.array([(x, nz // 2) for x in range(nx)] + [(nx // 3, z) for z in range(nz)] +
                       [(0, 0), (nx - 1, nz - 1), (0, 0)])
        out = []
        for one in (True, False):
            if one:
                F.fd_set_adj_tuning(dtype, r, 2, 0)
            try:
                p = Propagator(v, r, 10.0, 0.4 * oracle_mod.dt_max(2, r, 10.0, float(v.max())), dtype,
                               max_receivers=len(rec))
            finally:
                F.fd_set_adj_tuning(dtype, r, 2, -1)
            p.record(rec, steps)
            n = p.new_field().numel()
            gen = torch.Generator(device="cuda").manual_seed(5)
            states = torch.zeros((steps, n), dtype=tdt, device="cuda")
            for k in range(steps):
                u = torch.randn(shape, generator=gen, dtype=tdt, device="cuda")
                p.set_state(u, u, 0)
                p.save_padded(states[k], p.new_field())
            resid = torch.randn((steps, len(rec)), generator=gen, dtype=tdt, device="cuda")
            for seg in (False, True):
                for cuts in ([0, steps], [0, 1, 3, 6, 20, steps]):
                    mu, g, gs = torch.zeros(2 * n, dtype=tdt, device="cuda"), p.new_field(), p.new_field()
                    for lo, hi in reversed(list(zip(cuts, cuts[1:]))):
                        F.fd_adjoint_stored(p.ctx, states[lo:], lo, hi, mu, resid, 0.5, g, gs if seg else None)
                    p.sync()
                    out.append((mu, g))
        half = len(out) // 2
        for a, b in zip(out[:half], out[half:]):
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        assert float(out[0][1].abs().max()) > 0 or max(shape) == 1


@pytest.mark.parametrize("shape,r,dtype", [((300, 420), 4, "f32"), ((90, 130), 2, "f64"), ((20, 24, 30), 2, "f32")])
def test_ring_over_checkpoint(oracle_mod, shape, r, dtype):
    # u^{k_lo-1} of the checkpoint may lie in the ring, whose first step then writes over it (or
    # a later one); u^{k_lo} may not be the ring's first field
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    tdt, steps = torch.float32 if dtype == "f32" else torch.float64, 9
    v = torch.tensor(workloads.layered_velocity(shape, seed=r), dtype=tdt, device="cuda")
    p = Propagator(v, r, 10.0, 0.4 * oracle_mod.dt_max(len(shape), r, 10.0, float(v.max())), dtype, max_receivers=1)
    p.record([tuple(n // 2 for n in shape[::-1])], steps)
    n = p.new_field().numel()
    u0 = torch.randn(shape, generator=torch.Generator(device="cuda").manual_seed(5), dtype=tdt, device="cuda")
    resid = torch.ones((steps, 1), dtype=tdt, device="cuda")
    got = []
    for place in (None, 0, 2, steps - 2):
        say(f"ring over checkpoint shape={shape} dtype={dtype} place={place}")
        ring = torch.zeros((steps - 1, n), dtype=tdt, device="cuda")
        cur, prev = p.new_field(), p.new_field() if place is None else ring[place]
        p.set_state(u0, 0.5 * u0, 0)
        p.save_padded(cur, prev)
        mu, g = torch.zeros(2 * n, dtype=tdt, device="cuda"), p.new_field()
        F.fd_adjoint_segment(p.ctx, cur, prev, 0, steps, ring, mu, resid, 1.0, g, None)
        p.sync()
        got.append((ring, mu, g))
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
    assert float(got[0][2].abs().max()) > 0
    with pytest.raises(F.FdError) as e:
        F.fd_adjoint_segment(p.ctx, ring[0], cur, 0, steps, ring, mu, resid, 1.0, g, None)
    assert e.value.status == F.FD_E_INVAL


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_two_streams_at_once(oracle_mod, dtype):
    # a context moved to a second stream while a first adjoint run is queued behind other work:
    # the two runs, in fields of their own, end as they do one after the other
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    tdt, steps, shape, r = torch.float32 if dtype == "f32" else torch.float64, 24, (300, 420), 4
    v = torch.tensor(workloads.layered_velocity(shape, seed=r), dtype=tdt, device="cuda")
    p = Propagator(v, r, 10.0, 0.4 * oracle_mod.dt_max(2, r, 10.0, float(v.max())), dtype, max_receivers=400)
    rec = np.array([(x, 5) for x in range(400)])
    p.record(rec, steps)
    n = p.new_field().numel()
    gen = torch.Generator(device="cuda").manual_seed(5)
    states = torch.zeros((steps, n), dtype=tdt, device="cuda")
    for k in range(steps):
        u = torch.randn(shape, generator=gen, dtype=tdt, device="cuda")
        p.set_state(u, u, 0)
        p.save_padded(states[k], p.new_field())
    resid = torch.randn((2, steps, 400), generator=gen, dtype=tdt, device="cuda")
    busy = torch.randn((4096, 4096), generator=gen, dtype=torch.float32, device="cuda")
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    p.sync()
    torch.cuda.synchronize()
    runs = []
    for together in (False, True):
        say(f"two streams {dtype} together={together}")
        out = [(torch.zeros(2 * n, dtype=tdt, device="cuda"), p.new_field()) for _ in streams]
        torch.cuda.synchronize()
        for k, s in enumerate(streams):
            F.fd_set_stream(p.ctx, F.stream_ptr(s))
            with torch.cuda.stream(s):
                if together and k == 0:
                    for _ in range(4):
                        busy @ busy
                F.fd_adjoint_stored(p.ctx, states, 0, steps, out[k][0], resid[k], 1.0, out[k][1], None)
            if not together:
                p.sync()
        torch.cuda.synchronize()
        p.sync()
        runs.append(out)
    for a, b in zip(*runs):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        assert float(a[1].abs().max()) > 0


@pytest.mark.parametrize("shape,r,dtype", [((300, 420), 4, "f32"), ((90, 130), 6, "f64")])
def test_workspace_without_second_pair(oracle_mod, shape, r, dtype):
    # a workspace without the optional part gives the bits of one with it, forward and adjoint;
    # one byte less is refused; a server's budget holds a shot that just fits without it
    import torch

    from paper_1410_1387_amd import fdwave as F
    from paper_1410_1387_amd.serving import ShotRequest, ShotServer, run_sequential, shot_footprint, staging_bytes

    tdt, steps = torch.float32 if dtype == "f32" else torch.float64, 21
    v = torch.tensor(workloads.layered_velocity(shape, seed=r), dtype=tdt, device="cuda")
    dt = 0.4 * oracle_mod.dt_max(2, r, 10.0, float(v.max()))
    src = (25, 9)
    rec = np.array([(x, 9) for x in range(50)])
    whole, opt = F.fd_workspace_bytes(shape, r, dtype, 1, 50), F.fd_workspace_optional_bytes(shape, r, dtype)
    sp = F.stream_ptr(None)
    got = []
    for nbytes in (whole, whole - opt):
        say(f"2-D workspace shape={shape} dtype={dtype} bytes={nbytes}")
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        ctx = F.fd_create(shape, r, 10.0, dt, v, dtype, "zero", ws, 1, 50, sp)
        wav = torch.empty(steps, dtype=tdt, device="cuda")
        F.fd_ricker(wav, dt, 30.0, 0.0, sp)
        F.fd_inject(ctx, wav, src, 1e6)
        traces = torch.zeros((steps, 50), dtype=tdt, device="cuda")
        F.fd_record(ctx, rec, traces, steps)
        F.fd_step(ctx, steps)
        n = F.fd_field_bytes(shape, r, dtype) // v.element_size()
        f = [torch.zeros(k * n, dtype=tdt, device="cuda") for k in (1, 1, steps, 2, 1)]
        F.fd_get_state(ctx, f[0], f[1], F.FD_PADDED)
        F.fd_adjoint_segment(ctx, f[0], f[1], 0, steps, f[2], f[3], traces, 1.0, f[4])
        F.fd_sync(ctx)
        F.fd_destroy(ctx)
        got.append([traces] + f)
    assert all(torch.equal(a, b) for a, b in zip(*got)) and float(got[0][5].abs().max()) > 0
    with pytest.raises(F.FdError) as e:
        F.fd_create(shape, r, 10.0, dt, v, dtype, "zero", ws[:-256], 1, 50, sp)
    assert e.value.status == F.FD_E_NOMEM
    req = ShotRequest(0, workloads.layered_velocity(shape, seed=r), steps, src, rec)
    server = ShotServer(r, dtype, budget_bytes=shot_footprint(shape, steps, 50, r, dtype) + staging_bytes(shape, dtype))
    res, ref = server.serve_trace([req], realtime=False), run_sequential([req], r, dtype, realtime=False)
    assert res[0].status == ref[0].status == "ok", (res[0].error, ref[0].error)
    assert torch.equal(res[0].traces, ref[0].traces)


@pytest.mark.parametrize("shape,r,dtype,fwd,adj", [
    ((256, 256), 1, "f32", (8, 64, 32), (8, 32, 32)), ((90, 210), 4, "f32", (8, 32, 32), (6, 32, 32)),
    ((550, 1601), 4, "f32", (3, 64, 32), (4, 64, 32)), ((1101, 1599), 4, "f32", (2, 64, 32), (4, 64, 32)),
    ((801, 1203), 3, "f32", (4, 64, 32), None), ((521, 545), 2, "f32", (4, 64, 32), (4, 32, 16)),
    ((300, 420), 8, "f32", (3, 32, 32), None), ((801, 1203), 8, "f32", None, None),
    ((256, 256), 4, "f64", (6, 16, 16), (6, 16, 16)), ((270, 265), 4, "f64", (4, 32, 32), (3, 32, 32)),
    ((270, 265), 3, "f64", (6, 32, 32), (3, 32, 32)), ((521, 545), 3, "f64", (4, 32, 32), (3, 32, 32)),
    ((70, 38), 5, "f64", (4, 16, 16), (4, 16, 16)), ((270, 265), 5, "f64", (3, 32, 32), None),
    ((801, 1203), 5, "f64", None, None), ((4500, 4300), 1, "f32", None, None)])
def test_config_names_the_shared_launch(shape, r, dtype, fwd, adj):
    # the configuration strings name the kernel that most steps take: the deep, the shallow or no
    # shared launch by grid and radius; a tile set by hand and the periodic boundary step alone
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    def name(entry):
        if entry is None:
            return "; single steps"
        k, tx, tz = entry
        return f"; up to {k} steps per launch, tile {tx}x{tz}, {-(-shape[1] // tx) * -(-shape[0] // tz)} wg"

    v = torch.full(shape, 2000.0, dtype=torch.float32 if dtype == "f32" else torch.float64, device="cuda")

    def configs(bc="zero"):
        p = Propagator(v, r, 10.0, 1e-4, dtype, bc=bc)
        say(f"{p.kernel_config} | {p.adjoint_config}")
        return [c[c.index(";"):] for c in (p.kernel_config, p.adjoint_config)]

    assert configs() == [name(fwd), name(adj)]
    assert configs("periodic") == [name(None)] * 2
    F.fd_set_tuning(dtype, r, 2, 0)
    F.fd_set_adj_tuning(dtype, r, 2, 0)
    try:
        assert configs() == [name(None)] * 2
    finally:
        F.fd_set_tuning(dtype, r, 2, -1)
        F.fd_set_adj_tuning(dtype, r, 2, -1)
