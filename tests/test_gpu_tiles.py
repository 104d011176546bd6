"""Every registered forward tile, and every way a source or a receiver reaches the kernel,
against the oracle (needs an MI355X)."""

import numpy as np
import pytest

import workloads
from gpu_util import rel_l2, run_gpu, say

pytestmark = pytest.mark.gpu

TOL = {"f32": 1e-4, "f64": 1e-11}


def _case(shape, seed):
    rng = np.random.default_rng(seed)
    u0 = rng.standard_normal(shape)
    return workloads.layered_velocity(shape, seed=seed), u0, 0.5 * u0


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("r", range(1, 9))
def test_registered_tiles_bitwise(oracle_mod, r, dtype):
    # one plane per chunk, chunks with a remainder and one chunk, on a grid that divides no
    # tile, damped and not: every registered tile gives the first one's bits, and the first
    # one the oracle's solution (8 steps: FP32 rounding stays far below the parity bar)
    from paper_1410_1387_amd import fdwave as F

    shape, T = (11, 35, 133), 8
    v, u0, um1 = _case(shape, r)
    dt = 0.5 * oracle_mod.dt_max(3, r, 10.0, v.max())
    rec = workloads.surface_receivers(shape[2], shape[1], 3, 4)
    for damping in (None, (3, 0.05, 63)):
        base = None
        cfg = 0
        while True:
            try:
                F.fd_set_tuning(dtype, r, 3, cfg)
            except F.FdError:
                break
            for zch in (1, 4, 11):
                got = run_gpu(v, r, 10.0, dt, T, dtype, receivers=rec, u0=u0, um1=um1,
                              ricker=((66, 17, 3), 30.0, 0.0), tuning=(cfg, zch), damping=damping, label="tiles")
                base = base or got
                assert np.array_equal(got["u"], base["u"]), (cfg, zch, got["config"])
                assert np.array_equal(got["u_prev"], base["u_prev"]), (cfg, zch)
                assert np.array_equal(got["traces"], base["traces"]), (cfg, zch)
            cfg += 1
        F.fd_set_tuning(dtype, r, 3, -1)
        assert cfg >= 3
        src = [((66, 17, 3), oracle_mod.ricker(T, dt, 30.0, 0.0))]
        ref = oracle_mod.forward(v, 10.0, dt, r, T, src, rec, u0=u0, um1=um1, damping=damping and damping[:2])
        assert rel_l2(base["u"], ref["u"]) <= TOL[dtype] and rel_l2(base["traces"], ref["traces"]) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 6])
def test_own_choice_bitwise(oracle_mod, r, dtype):
    # the library's own tile and chunk gives the bits of the first tile with one chunk: fewer
    # planes than a short chunk has, many short chunks, one round, and (the last shape) fields
    # past the last-level cache, whose loads have another cache policy
    T = 5
    for shape in [(1, 17, 40), (2, 300, 130), (3, 9, 1000), (61, 70, 300), (200, 33, 333), (150, 410, 310)]:
        v, u0, um1 = _case(shape, r)
        dt = 0.5 * oracle_mod.dt_max(3, r, 10.0, v.max())
        rec = workloads.surface_receivers(shape[2], shape[1], shape[0] // 2, 16)
        kw = dict(receivers=rec, u0=u0, um1=um1, ricker=((shape[2] // 2, 8, 0), 30.0, 0.0), label="own choice")
        got = run_gpu(v, r, 10.0, dt, T, dtype, **kw)
        base = run_gpu(v, r, 10.0, dt, T, dtype, tuning=(0, shape[0]), **kw)
        say(got["config"])
        for k in ("u", "u_prev", "traces"):
            assert np.array_equal(got[k], base[k]), (shape, k, got["config"])


@pytest.mark.parametrize("nsrc", [1, 2, 3, 5])
@pytest.mark.parametrize("shape,r", [((13, 20, 70), 4), ((30, 75), 8)])
def test_sources_and_receivers_vs_oracle(oracle_mod, shape, r, nsrc):
    # a few sources travel in the shot descriptor, more of them in the event list; receivers
    # are one per column, several in one column (a vertical line), and on top of a source;
    # two sources share a point, and a wavelet ends before the run does
    T, dtype = 14, "f64"
    v, u0, um1 = _case(shape, nsrc)
    nd = len(shape)
    dt = 0.4 * oracle_mod.dt_max(nd, r, 10.0, v.max())
    ext = shape[::-1]
    at = [(5, 2, 4), (5, 2, 4), (69, 19, 12), (0, 0, 0), (37, 11, 7)]
    at = [tuple(min(a, n - 1) for a, n in zip(p[:nd] if nd == 3 else (p[0], p[2]), ext)) for p in at]
    rng = np.random.default_rng(7)
    sources = [(at[i], rng.standard_normal(T - 3 * i) * 1e6) for i in range(nsrc)]
    if nd == 3:
        rec = [(x, 2, 4) for x in range(0, 70, 3)] + [(5, 2, 4)] + [(37, 11, z) for z in range(13)] + [(69, 19, 12)]
    else:
        rec = [(x, 4) for x in range(75)] + [(5, 4), (37, 7)] + [(40, z) for z in range(30)]
    rec = np.array(rec)
    got = run_gpu(v, r, 10.0, dt, T, dtype, sources=sources, receivers=rec, u0=u0, um1=um1, label="events")
    padded = [(p, np.concatenate([w, np.zeros(T - len(w))])) for p, w in sources]
    ref = oracle_mod.forward(v, 10.0, dt, r, T, padded, rec, u0=u0, um1=um1)
    say(f"u {rel_l2(got['u'], ref['u']):.2e} traces {rel_l2(got['traces'], ref['traces']):.2e}")
    assert rel_l2(got["u"], ref["u"]) <= TOL[dtype]
    assert rel_l2(got["traces"], ref["traces"]) <= TOL[dtype]
    assert np.all(got["traces"][:, -1] != 0.0)


@pytest.mark.parametrize("sides", [(64, 64, 64, 64), (40, 96, 20, 130), (33,), (130, 160, 64, 40, 170, 120),
                                   (50, 272, 60, 280, 281, 30), (170, 160, 130, 280, 40, 150, 165, 30)])
def test_batch_tile_choice_bitwise(oracle_mod, sides):
    # a batch picks one tile for its members, whatever they step with alone: damped and
    # undamped members, with few and many sources, end with the bits they have alone; in one
    # launch per step, in groups, with members too large for the cache that take small ones
    # along, and with such members between groups
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    T, dt = 9, 4e-4
    stream = torch.cuda.Stream()

    def make(i, n):
        v = torch.tensor(workloads.layered_velocity((n, n + 3, n + 1), seed=i), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
        p = Propagator(v, 4, 10.0, dt, "f32", max_sources=4, max_receivers=40, stream=stream)
        if i % 2:
            p.set_damping(5, 0.03)
        with torch.cuda.stream(stream):
            for k in range(1 + i % 4):
                p.inject(p.ricker(T, 30.0, 0.0), (n // 2, n // 2 + k, 2), 1e6)
            tr = p.record([(n // 2 - 10 + x, n // 2, 2) for x in range(20)], T)
        return p, tr

    alone = [make(i, n) for i, n in enumerate(sides)]
    for p, _ in alone:
        p.step(T)
    both = [make(i, n) for i, n in enumerate(sides)]
    ws = torch.empty(F.fd_batch_workspace_bytes(len(sides)), dtype=torch.uint8, device="cuda")
    b = F.fd_batch_create(len(sides), ws, F.stream_ptr(stream))
    F.fd_batch_set(b, [p.ctx for p, _ in both], [T] * len(sides))
    F.fd_batch_step(b, 5)
    F.fd_batch_step(b, 4)
    for (pa, ta), (pb, tb) in zip(alone, both):
        with torch.cuda.stream(stream):
            ua, ub = pa.state(), pb.state()
        stream.synchronize()
        assert torch.equal(ua[0], ub[0]) and torch.equal(ua[1], ub[1]) and torch.equal(ta, tb)
        assert float(ta.abs().max()) > 0
    F.fd_batch_destroy(b)


@pytest.mark.parametrize("dtype,tol", [("f64", 1e-9), ("f32", 1e-3)])
@pytest.mark.parametrize("r", [1, 3, 4, 5, 8])
def test_registered_adjoint_tiles(oracle_mod, r, dtype, tol):
    # chunks of one, two and an odd number of planes, a grid that divides no tile, the image
    # summed straight into g and by segments of one and several steps: every registered tile
    # gives the first one's bits, and that the oracle's gradient (the adjoint's bars)
    from paper_1410_1387_amd import fdwave as F
    from test_gpu_adjoint import _gpu_gradient, _problem

    v, pb, obs = _problem(oracle_mod, (23, 21, 133), r, 40, 7, dtype, seed=20 + r)
    ref = oracle_mod.gradient(v, pb.h, pb.dt, r, pb.nsteps, [(pb.source, oracle_mod.ricker(40, pb.dt, pb.f0, pb.t0))],
                              pb.receivers, obs)
    for blocked, ckpt in ((False, 7), (True, 7), (True, 13)):
        pb.blocked, pb.ckpt = blocked, ckpt
        base, cfg = None, 0
        try:
            while True:
                try:
                    F.fd_set_adj_tuning(dtype, r, 3, cfg)
                except F.FdError:
                    break
                say(f"adjoint tile {cfg} {dtype} r={r} blocked={blocked} segments of {ckpt}")
                g = _gpu_gradient(v, pb, obs)[1]
                base = g if base is None else base
                assert np.array_equal(g, base), (cfg, blocked, ckpt)
                cfg += 1
        finally:
            F.fd_set_adj_tuning(dtype, r, 3, -1)
        assert rel_l2(_gpu_gradient(v, pb, obs)[1], base) == 0.0
        assert rel_l2(base, ref["grad_v"]) <= tol


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-4), ("f64", 1e-11)])
@pytest.mark.parametrize("rxy,rz,nsrc", [(12, 8, 1), (4, 4, 3), (8, 2, 2), (2, 1, 5)])
def test_registered_vti_tiles(oracle_mod, rxy, rz, nsrc, dtype, tol):
    # every registered tile and chunks of one, several and all planes give the bits of the
    # library's own choice, and that the oracle's solution; few and many sources, two of
    # them at one point, and receivers one per column, in a line and on the sources
    from paper_1410_1387_amd import fdwave as F
    from test_gpu_vti import _model, run_vti_gpu

    shape, h, T = (11, 19, 70), 10.0, 8
    vz, eps, delta = _model(shape, seed=rxy)
    zc = workloads.stretched_z(shape[0], rz, h)
    dt = 0.5 * oracle_mod.vti_dt_max(rxy, rz, h, oracle_mod.z_weights(zc, rz), vz, eps, delta)
    rng = np.random.default_rng(rz)
    at = [(5, 2, 4), (5, 2, 4), (69, 18, 10), (0, 0, 0), (37, 11, 7)]
    src = [(at[i], rng.standard_normal(T) * 1e6, 1.0, 0.3 * i) for i in range(nsrc)]
    rec = np.array([(x, 2, 4) for x in range(0, 70, 3)] + [(5, 2, 4)] + [(6, 3, z) for z in range(11)] + [(69, 18, 10)])
    ref = oracle_mod.vti_forward(vz, eps, delta, h, dt, rxy, rz, T, zc=zc, sources=src, receivers=rec)
    base = run_vti_gpu(vz, eps, delta, h, zc, dt, rxy, rz, T, dtype, sources=src, receivers=rec)
    for f in ("p", "q", "traces_p", "traces_q"):
        assert rel_l2(base[f], ref[f]) <= tol, f
    cfg = 0
    while True:
        try:
            F.fd_vti_set_tuning(dtype, rxy, rz, cfg, 1)
        except F.FdError:
            break
        for zch in (1, 3, 11):
            got = run_vti_gpu(vz, eps, delta, h, zc, dt, rxy, rz, T, dtype, sources=src, receivers=rec,
                              tuning=(cfg, zch))
            assert all(np.array_equal(got[f], base[f]) for f in base if isinstance(base[f], np.ndarray)), (cfg, zch)
        cfg += 1
    F.fd_vti_set_tuning(dtype, rxy, rz, 0, 0)
    assert cfg >= 3


@pytest.mark.parametrize("dtype,r,shape", [("f32", 4, (1, 250, 300)), ("f64", 4, (1, 250, 300)), ("f32", 8, (1, 250, 300)),
                                           ("f32", 2, (1, 250, 300))])
def test_batch_takes_the_tile_set_by_hand(oracle_mod, dtype, r, shape):
    # a batch whose members were all created with one tile steps with that tile: the prefix at
    # the end of its table counts the workgroups of that tile (one plane: one chunk), and the
    # bits are those of a member alone; with two tiles among them, too
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    T, tdt = 6, torch.float32 if dtype == "f32" else torch.float64
    v, u0, um1 = (torch.tensor(a, dtype=tdt, device="cuda") for a in _case(shape, r))
    dt = 0.5 * oracle_mod.dt_max(3, r, 10.0, float(v.max()))
    base, counts = [], []

    def member(cfg, damped):
        F.fd_set_tuning(dtype, r, 3, cfg)
        try:
            p = Propagator(v, r, 10.0, dt, dtype)
        finally:
            F.fd_set_tuning(dtype, r, 3, -1)
        if damped:
            p.set_damping(5, 0.03)
        p.set_state(u0, um1, 0)
        return p

    def batch(ps):
        ws = torch.empty(F.fd_batch_workspace_bytes(2), dtype=torch.uint8, device="cuda")
        b = F.fd_batch_create(2, ws, F.stream_ptr(None))
        F.fd_batch_set(b, [p.ctx for p in ps], [T, T])
        prefix = ws[-256:][:12].view(torch.int32).tolist()
        F.fd_batch_step(b, T)
        got = [p.state()[:2] for p in ps]
        torch.cuda.synchronize()
        F.fd_batch_destroy(b)
        assert all(torch.equal(x, y) for one, other in zip(got, base) for x, y in zip(one, other))
        assert prefix[0] == 0 and prefix[2] == 2 * prefix[1]
        return prefix[1]

    for damped in (False, True):
        p = member(-1, damped)
        p.step(T)
        base.append(p.state()[:2])
    own = batch([member(-1, False), member(-1, True)])
    cfg = 0
    while True:
        try:
            ps = [member(cfg, False), member(cfg, True)]
        except F.FdError as e:
            assert e.status == F.FD_E_RANGE
            break
        say(f"batch by hand {ps[0].kernel_config}")
        counts.append(batch(ps))
        assert counts[-1] == int(ps[0].kernel_config.split("grid ")[1].split()[0])
        cfg += 1
    assert len(set(counts)) >= 3
    batch([member(0, False), member(cfg - 1, True)])
    assert own in counts


@pytest.mark.parametrize("dtype,r,shapes", [
    ("f64", 4, [(40, 43, 41), (64, 67, 65), (212, 215, 213), (96, 99, 97)]), ("f32", 2, [(50, 53, 51), (130, 133, 131), (268, 271, 269)]),
    ("f32", 8, [(50, 53, 51), (130, 133, 131), (268, 271, 269)]), ("f64", 1, [(33, 36, 34), (100, 103, 101), (90, 93, 300)]),
    ("f64", 7, [(33, 36, 34), (100, 103, 101)]), ("f32", 4, [(300, 420), (801, 1203), (33, 70), (4300, 4301)]),
    ("f64", 8, [(300, 420), (801, 1203), (3100, 3000), (1, 9)]), ("f32", 2, [(256, 256)] * 5 + [(90, 700)]),
    ("f64", 5, [(40, 40, 32), (64, 64, 64), (33, 30, 96)]), ("f32", 4, [(128, 128, 128)] * 9),
    ("f64", 4, [(2500, 2500)] * 4), ("f64", 3, [(96, 95, 97)] * 5)])
def test_batch_tile_choice_types(oracle_mod, dtype, r, shapes):
    # the tiles, chunks and loads that batches choose in either type, at other radii and in 2-D:
    # members that stay in the last-level cache and ones that do not, whole rows that stream,
    # groups that a member more would overfill; damped and undamped, with few and many sources,
    # all end with the bits they have alone
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    T, tdt = 7, torch.float32 if dtype == "f32" else torch.float64
    dt = 0.4 * oracle_mod.dt_max(len(shapes[0]), r, 10.0, 4500.0)
    stream = torch.cuda.Stream()

    def make(i, shape):
        v = torch.full(shape, 2000.0, dtype=tdt, device="cuda")
        v[shape[0] // 2:] = 2500.0 + 100 * i
        u0 = torch.randn(shape, generator=torch.Generator(device="cuda").manual_seed(i), dtype=tdt, device="cuda")
        torch.cuda.synchronize()
        mid = tuple(n // 2 for n in shape[::-1])
        rec = [(x,) + mid[1:] for x in range(0, shape[-1], 3)] + [mid[:-1] + (z,) for z in range(shape[0])]
        p = Propagator(v, r, 10.0, dt, dtype, max_sources=4, max_receivers=len(rec), stream=stream)
        with torch.cuda.stream(stream):
            if i % 2:
                p.set_damping(3, 0.03)
            for k in range(1 + i % 4):
                p.inject(p.ricker(T, 30.0, 0.0), (mid[0], *mid[1:-1], min(k, shape[0] - 1)), 1e6)
            tr = p.record(rec, T)
            p.set_state(u0, 0.5 * u0, 0)
        stream.synchronize()
        return p, tr

    say(f"batch {dtype} r={r} {shapes}")
    alone = [make(i, s) for i, s in enumerate(shapes)]
    for p, _ in alone:
        p.step(T)
    both = [make(i, s) for i, s in enumerate(shapes)]
    ws = torch.empty(F.fd_batch_workspace_bytes(len(shapes)), dtype=torch.uint8, device="cuda")
    b = F.fd_batch_create(len(shapes), ws, F.stream_ptr(stream))
    F.fd_batch_set(b, [p.ctx for p, _ in both], [T] * len(shapes))
    F.fd_batch_step(b, 4)
    F.fd_batch_step(b, 3)
    for (pa, ta), (pb, tb) in zip(alone, both):
        with torch.cuda.stream(stream):
            ua, ub = pa.state(), pb.state()
        stream.synchronize()
        assert torch.equal(ua[0], ub[0]) and torch.equal(ua[1], ub[1]) and torch.equal(ta, tb), pa.shape
        assert float(ta.abs().max()) > 0
    F.fd_batch_destroy(b)


@pytest.mark.parametrize("leave", [True, False])
def test_tiles_set_by_hand_end_with_their_test(leave):
    # the second run of this test does not find what the first one left set
    import torch

    from paper_1410_1387_amd import Propagator
    from paper_1410_1387_amd import fdwave as F

    v = torch.full((50, 30, 60), 2000.0, dtype=torch.float32, device="cuda")
    assert "zchunk 17," not in Propagator(v, 3, 10.0, 1e-4).kernel_config
    if leave:
        F.fd_set_tuning("f32", 3, 3, 0, 17)
        assert "zchunk 17," in Propagator(v, 3, 10.0, 1e-4).kernel_config
