"""GPU parity of kernel paths chosen by size, at the sizes where each can go wrong."""
import numpy as np
import pytest

from oracle import box

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# Every 3 * 2^m plan, whole half spectrum: one butterfly a thread (12, 24), partial
# rounds of radix-4 (48, 192, twice in 192) and radix-8 butterflies (96).  Bars:
# FP64 1e-13 of the maximum for each 16 points of a line; FP32 1e-6 rel-L2
# (three passes of about log2(N) 2^-24 each).
@pytest.mark.parametrize("n", [12, 24, 48, 96, 192])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_radix_6_plans_transform_both_ways(n, precision):
    from paper_2406_01322_amd.psms import Solver
    rng = np.random.default_rng(n)
    s = Solver(n, 100.0, 1.0, 0.05, 20.0, 1e-3, precision=precision)
    real, cplx = (np.float64, np.complex128) if precision == "fp64" else (np.float32, np.complex64)
    f = rng.standard_normal((n, n, n)).astype(real)
    want = box.transform_forward(f.astype(np.float64))
    got = _host(s.transform(+1, _dev(f), 0)).astype(np.complex128)
    fh = want.astype(cplx)
    back = _host(s.transform(-1, _dev(fh), 0)).astype(np.float64)
    wback = box.transform_inverse(fh.astype(np.complex128))
    for a, b in ((got, want), (back, wback)):
        if precision == "fp64":
            assert np.max(np.abs(a - b)) <= 1e-13 * max(1, n // 16) * np.max(np.abs(b))
        else:
            assert np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b)


# The x and z stages of the smallest boxes: one workgroup or a few, the last one
# partly filled, most of the band's line tiles past its end (n = 8: 15 lines).  An
# AB1 and an AB2 step against the oracle, to the bars of the larger boxes' tests.
@pytest.mark.parametrize("n", [8, 12, 16, 24])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
def test_smallest_box_steps(n, precision, tol):
    from paper_2406_01322_amd.psms import Solver
    prm = box.Params(n=n, re=50.0, we=1.0, ch=0.2, pe=5.0, dt=1e-3)
    rng = np.random.default_rng(n)
    x = 2 * np.pi * np.arange(n) / n
    z, y, x = np.meshgrid(x, x, x, indexing="ij")
    u = np.stack([np.sin(x) * np.cos(y) * np.cos(z), -np.cos(x) * np.sin(y) * np.cos(z), 0.3 * np.cos(x + 2 * y)])
    phi = np.cos(x) * np.sin(y - z) + 0.1 * rng.standard_normal((n, n, n))
    s = Solver(n, prm.re, prm.we, prm.ch, prm.pe, prm.dt, precision=precision)
    s.init_state(_dev(u), _dev(phi))
    st = box.init_state(u, phi, prm)
    for _ in range(2):
        s.step(1)
        st = box.step(st, prm)
        uh, ph = (_host(t) for t in s.get_state())
        for a, b in [(uh[i], st["uh"][i]) for i in range(3)] + [(ph, st["ph"])]:
            assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b)


# A box alone takes the z stage with a group of threads per field, boxes enough of one
# size the one with the fields in registers: the same bits (AB1, then AB2 steps).
@pytest.mark.parametrize("n,boxes", [(12, 92), (16, 63), (24, 35), (32, 18), (48, 9), (64, 5), (96, 2)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_z_stages_give_the_same_bits(n, boxes, precision):
    from paper_2406_01322_amd.psms import Batch, Solver
    p = dict(n=n, re=50.0, we=1.0, ch=0.2, pe=5.0, dt=1e-3)
    rng = np.random.default_rng(n)
    u, phi = rng.standard_normal((3, n, n, n)), rng.standard_normal((n, n, n))
    s = Solver(precision=precision, **p)
    s.init_state(_dev(u), _dev(phi))
    b = Batch([p] * boxes, precision=precision)
    for i in (0, boxes - 1):
        b.init_state(i, _dev(u), _dev(phi))
    for i in range(1, boxes - 1):
        b.init_state(i, _dev(np.zeros_like(u)), _dev(np.zeros_like(phi)))
    s.step(3)
    b.step(3)
    torch.cuda.synchronize()
    want = s.get_state()
    for i in (0, boxes - 1):
        got = b.get_state(i)
        assert all(torch.equal(x, y) for x, y in zip(got, want))


# Fields are transformed several per launch, in chunks that the scratch holds: more
# fields than a chunk give each field what it gives alone, bit for bit, with and
# without the mask pass, and an inverse over its own input the same.
@pytest.mark.parametrize("n", [8, 48])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("flags", [0, 1 | 4])
def test_transform_chunks_of_fields(n, precision, flags):
    from paper_2406_01322_amd import psms
    s = psms.Solver(n, 100.0, 1.0, 0.05, 20.0, 1e-3, precision=precision)
    real = np.float64 if precision == "fp64" else np.float32
    f = _dev(np.random.default_rng(n).standard_normal((9, n, n, n)).astype(real))
    fh = s.transform(+1, f, flags)
    assert all(torch.equal(fh[k], s.transform(+1, f[k], flags)) for k in range(9))
    back = s.transform(-1, fh, flags)
    assert all(torch.equal(back[k], s.transform(-1, fh[k], flags)) for k in range(9))
    psms._check(psms.lib().psms_transform(s.ctx, -1, 9, psms._ptr(fh), psms._ptr(fh), flags))
    inplace = torch.view_as_real(fh).reshape(-1)[: 9 * n ** 3].reshape(9, n, n, n)
    assert torch.equal(inplace, back)


# The pieced wall solves: chains shorter than the 8 pieces (nc = 4 .. 12), with a partly
# filled last piece, line counts around the 64 of a workgroup, and (nc = 20, 33) the
# lengths that keep the one-lane-per-chain solve.  Bar: 1e-11 of each line's largest
# coefficient, as for the other wall-solve tests.
@pytest.mark.parametrize("nc,nl", [(4, 1), (6, 63), (8, 64), (12, 65), (24, 3), (48, 5), (64, 129), (96, 2), (256, 66),
                                   (20, 7), (33, 7)])
def test_pieced_wall_solve_sizes(nc, nl):
    from oracle import channel as ch
    from paper_2406_01322_amd import psms
    rng = np.random.default_rng(nc)
    kx, ky = np.arange(nl) % 7 * 0.5, (np.arange(nl) // 7 - 2) * 1.0      # a mean line from nl = 15 on
    g = [(rng.standard_normal((nc + 1, nl)) + 1j * rng.standard_normal((nc + 1, nl)))
         * np.exp(-0.05 * np.arange(nc + 1))[:, None] for _ in range(3)]
    bn, ba, bb = 3e4, 40.0, 700.0
    k2 = kx ** 2 + ky ** 2
    want = ch.wall_normal_solve_lines(*g, kx, ky, k2 + bn, k2 + ba, k2 + bb)
    got = psms.wall_solve(_dev(kx), _dev(ky), bn, ba, bb, *[_dev(x) for x in g])
    for key in ("omega", "w", "phi", "u", "v"):
        a, b = _host(got[key]), want[key]
        assert np.all(np.max(np.abs(a - b), axis=0) <= 1e-11 * np.max(np.abs(b), axis=0)), key


def _channel_fields(nx, ny, nc, seed):
    from paper_2406_01322_amd import synth
    lx, ly = 4.0 * np.pi, 2.0 * np.pi
    X, Y, Z = synth.channel_grid(nx, ny, nc, lx, ly)
    rng = np.random.default_rng(seed)
    up, vp, wp = synth.channel_perturbation(X, Y, Z, lx, ly, rng, min(4, (nx - 1) // 3, (ny - 1) // 3), 1.0)
    phi = np.tanh(2.0 * np.cos(0.5 * X + rng.uniform(0, 6)) * np.cos(Y) + Z ** 2 * (1.5 - Z ** 2 / 2) - 0.3)
    return 10.0 * (1.0 - Z ** 2) + up, vp, wp, phi


# The wall-normal half of the channel step in one launch: chains shorter than the
# pieces or with a partly filled last piece, band line counts below, at and above the
# 64 of a workgroup, each wall combination (with different walls the workgroup holds
# both parities).  An AB1 and an AB2 step against the oracle: 1e-12 of each field's
# maximum, as for the other step tests.  (At these coarse time steps the rounding of
# the explicit terms, which grows as nc^2, passes that bar from nc = 96 on; the
# longer chains are held to their wall conditions below.)
@pytest.mark.parametrize("nx,ny,nc,walls,single", [
    (8, 8, 4, "nn", False), (12, 8, 6, "ff", False), (16, 12, 8, "fn", False), (24, 24, 12, "nf", False),
    (16, 24, 24, "nn", True), (32, 16, 48, "fn", True), (16, 16, 64, "nf", False)])
def test_channel_step_sizes_and_walls(nx, ny, nc, walls, single):
    from oracle import channel_step as cs
    from paper_2406_01322_amd.psms import Channel
    kinds = tuple({"n": "noslip", "f": "freeslip"}[c] for c in walls)
    prm = cs.ChannelParams(nx=nx, ny=ny, nc=nc, re=20.0, we=1.0, ch=0.2, pe=5.0, dt=1e-3, walls=kinds)
    f = list(_channel_fields(nx, ny, nc, nc))
    if single:
        f[3] = np.zeros_like(f[3])
    c = Channel(nx, ny, nc, prm.re, prm.we, prm.ch, prm.pe, prm.dt, single_phase=single, walls=kinds)
    c.init_state(*[_dev(x) for x in f])
    st = cs.init_state(*f, prm)
    for _ in range(2):
        c.step(1)
        st = cs.step(st, prm)
        got, mean = (_host(x) for x in c.get_state())
        for a, b in ((got[0], st["om"]), (got[1], st["w"]), (got[2], st["phi"]), (mean, st["mean"])):
            assert np.max(np.abs(a - b)) <= 1e-12 * max(np.max(np.abs(b)), 1e-300)


# The single-phase x stage (3 fields in, 6 products out) over line lengths with one
# and with several workgroups, partly filled ones among them, in both field groupings:
# an AB1 and an AB2 step against the oracle, FP64 to 1e-12 and MIXED to 1e-5 of each
# field's maximum, as for the other single-phase step tests.
@pytest.mark.parametrize("nx,ny", [(8, 12), (12, 8), (48, 8), (96, 12), (128, 8), (192, 8), (256, 8)])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
def test_single_phase_x_stage(nx, ny, precision, tol):
    from oracle import channel_step as cs
    from paper_2406_01322_amd.psms import Channel
    prm = cs.ChannelParams(nx=nx, ny=ny, nc=8, re=20.0, we=1.0, ch=0.2, pe=5.0, dt=1e-3)
    f = list(_channel_fields(nx, ny, 8, 7))
    f[3] = np.zeros_like(f[3])
    c = Channel(nx, ny, 8, prm.re, prm.we, prm.ch, prm.pe, prm.dt, precision=precision, single_phase=True)
    c.init_state(*[_dev(x) for x in f])
    st = cs.init_state(*f, prm)
    for _ in range(2):
        c.step(1)
        st = cs.step(st, prm)
        got, mean = (_host(x) for x in c.get_state())
        for a, b in ((got[0], st["om"]), (got[1], st["w"]), (mean, st["mean"])):
            assert np.max(np.abs(a - b)) <= tol * max(np.max(np.abs(b)), 1e-300)


# Grids with enough line tiles for a workgroup to take two of the wall-normal
# transforms (the smaller ones above give each its own): a step against the oracle,
# FP64 to 1e-12 and MIXED to 1e-5 of each field's maximum, as for the other step tests.
@pytest.mark.parametrize("nx,ny,nc,single", [(96, 96, 8, False), (96, 96, 12, True), (96, 64, 48, False)])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-12), ("mixed", 1e-5)])
def test_channel_step_paired_transforms(nx, ny, nc, single, precision, tol):
    from oracle import channel_step as cs
    from paper_2406_01322_amd.psms import Channel
    prm = cs.ChannelParams(nx=nx, ny=ny, nc=nc, re=20.0, we=1.0, ch=0.2, pe=5.0, dt=1e-3)
    f = list(_channel_fields(nx, ny, nc, 9))
    if single:
        f[3] = np.zeros_like(f[3])
    c = Channel(nx, ny, nc, prm.re, prm.we, prm.ch, prm.pe, prm.dt, precision=precision, single_phase=single)
    c.init_state(*[_dev(x) for x in f])
    c.step(1)
    st = cs.step(cs.init_state(*f, prm), prm)
    got, mean = (_host(x) for x in c.get_state())
    for a, b in ((got[0], st["om"]), (got[1], st["w"]), (got[2], st["phi"]), (mean, st["mean"])):
        assert np.max(np.abs(a - b)) <= tol * max(np.max(np.abs(b)), 1e-300)


# The boundary rows of the solutions for the longer chains (17 slots a piece at nc =
# 256), to the bars that the wall-solve tests hold them to: 1e-12 of the field's
# maximum for a value at a wall, 1e-9 for a slope (weights n^2).
@pytest.mark.parametrize("nc", [96, 128, 256])
@pytest.mark.parametrize("walls", ["nn", "fn", "nf", "ff"])
def test_channel_step_wall_conditions(nc, walls):
    from paper_2406_01322_amd.psms import Channel
    kinds = tuple({"n": "noslip", "f": "freeslip"}[c] for c in walls)
    c = Channel(24, 16, nc, 150.0, 3.0, 0.1, 10.0, 1e-4, walls=kinds)
    c.init_state(*[_dev(x) for x in _channel_fields(24, 16, nc, nc)])
    c.step(2)
    (om, w, phi), mean = (_host(x) for x in c.get_state())
    n = np.arange(nc + 1.0)
    sign = (-1.0) ** n
    value = {"t": np.ones(nc + 1), "b": sign}
    slope = {"t": n * n, "b": -sign * n * n}

    def zero(rows, side, a):
        a = a.reshape(nc + 1, -1)
        assert np.all(np.isfinite(a))
        assert np.max(np.abs(rows[side] @ a)) <= (1e-12 if rows is value else 1e-9) * np.max(np.abs(a))

    for j, side in enumerate("tb"):
        for a in (om, mean.T):
            zero(value if walls[j] == "n" else slope, side, a)
        zero(value, side, w)
        if walls[j] == "n":
            zero(slope, side, w)
        zero(slope, side, phi)


# D w and D phi of the state stay in the workspace between steps: a state that is set
# later, or diagnostics in between, must not meet those of another state.
def test_channel_derivatives_follow_the_state():
    from paper_2406_01322_amd.psms import Channel
    args = (16, 12, 16, 20.0, 1.0, 0.2, 5.0, 1e-3)
    a, b, c = (Channel(*args) for _ in range(3))
    f = [[_dev(x) for x in _channel_fields(16, 12, 16, s)] for s in (1, 2)]
    a.init_state(*f[0])
    a.step(2)
    saved = [t.clone() for t in a.get_state(with_history=True)]
    a.step(1)
    want = a.get_state()
    b.init_state(*f[1])
    b.step(3)
    b.set_state(*saved, nstep=2)      # another state over a context that has stepped
    b.step(1)
    c.set_state(*saved, nstep=2)
    c.diagnostics()
    c.step(1)
    for x in (b, c):
        assert all(torch.equal(p, q) for p, q in zip(x.get_state(), want))


# The adjoint's x stage, a wavefront per field: 1 to 32 row pairs a wavefront, a partly
# filled last workgroup (8, 12), padded (8, 12, 24) and swizzled rows.  Against the
# oracle's adjoint to the bar of the adjoint tests.
@pytest.mark.parametrize("n", [8, 12, 32, 48, 64])
def test_adjoint_x_stage(n):
    from oracle import adjoint as oadj
    from paper_2406_01322_amd.psms import Adjoint
    prm = box.Params(n=n, re=50.0, we=1.0, ch=0.2, pe=5.0, dt=1e-3)
    rng = np.random.default_rng(n)
    x = 2 * np.pi * np.arange(n) / n
    z, y, x = np.meshgrid(x, x, x, indexing="ij")
    u = np.stack([np.sin(x) * np.cos(y) * np.cos(z), -np.cos(x) * np.sin(y) * np.cos(z), 0.3 * np.cos(x + 2 * y)])
    phi = np.cos(x) * np.sin(y - z) + 0.1 * rng.standard_normal((n, n, n))
    J0, d0, w0, _ = oadj.gradient(u, phi, prm, 2)
    a = Adjoint(n, prm.re, prm.we, prm.ch, prm.pe, prm.dt, precision="fp64", max_steps=2, seg_len=1)
    J = a.forward(_dev(u), _dev(phi), 2)
    d, w = a.backward()
    assert abs(J - J0) <= 1e-10 * abs(J0)
    assert np.linalg.norm(_host(d) - d0) <= 1e-10 * np.linalg.norm(d0)
    assert abs(w - w0) <= 1e-10 * abs(w0)


# A step that the caller has captured in its own graph, replayed after other states
# were set: what the same step gives when it is launched directly, bit for bit.
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("single", [False, True])
def test_captured_channel_step_follows_the_state(precision, single):
    from paper_2406_01322_amd.psms import Channel
    with torch.cuda.stream(torch.cuda.Stream()):
        stream = torch.cuda.current_stream()
        c, d = (Channel(16, 12, 16, 20.0, 1.0, 0.2, 5.0, 1e-3, precision=precision, single_phase=single, stream=stream)
                for _ in range(2))
        states = []
        for seed in (1, 2, 3):
            f = _channel_fields(16, 12, 16, seed)
            d.init_state(*[_dev(x) for x in (f[:3] + (np.zeros_like(f[3]),) if single else f)])
            d.step(2)
            states.append([t.clone() for t in d.get_state(with_history=True)])
        c.set_state(*states[0], nstep=2)
        c.step(1)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            c.step(1)
        for s in (1, 2, 0, 1):
            c.set_state(*states[s], nstep=2)
            graph.replay()
            d.set_state(*states[s], nstep=2)
            d.step(1)
            torch.cuda.synchronize()
            assert all(torch.equal(x, y) for x, y in zip(c.get_state(), d.get_state())), s
        torch.cuda.synchronize()


# Outputs of the wall solves in the place of arrays that are no longer needed: u or v
# over w or omega, a solution over its own or another equation's right-hand side (nc =
# 20: the solves with one lane per chain, which read them in that order, omega and psi
# in one launch).  What is not overwritten is what separate arrays hold, bit for bit.
_PLACES = ["u=w", "v=w", "u=om", "v=om", "u=om,v=w", "u=w,v=om", "u=g_om,v=g_phi", "w=g_om", "phi=g_om", "phi=g_w",
           "om=g_om,w=g_w,phi=g_phi", "om=g_w,w=g_phi,phi=g_om"]


@pytest.mark.parametrize("nc,nl,place", [(*size, p) for size in ((8, 129), (64, 70), (256, 66)) for p in _PLACES]
                         + [(20, 129, p) for p in _PLACES[:-1]])
def test_wall_solve_in_place(nc, nl, place):
    import ctypes
    from paper_2406_01322_amd import psms
    rng = np.random.default_rng(nc)
    kx, ky = _dev(np.arange(nl) % 7 * 0.5), _dev((np.arange(nl) // 7 - 2) * 1.0)
    g = [_dev(rng.standard_normal((nc + 1, nl)) + 1j * rng.standard_normal((nc + 1, nl))) for _ in range(3)]
    want = psms.wall_solve(kx, ky, 3e4, 40.0, 700.0, *g)
    at = dict(zip(("g_om", "g_w", "g_phi"), (x.clone() for x in g)))
    at.update({k: torch.empty_like(g[0]) for k in ("om", "w", "phi", "u", "v")})
    over = dict(p.split("=") for p in place.split(","))
    for k, v in over.items():
        at[k] = at[v]
    nbytes = ctypes.c_size_t(0)
    psms._check(psms.lib().psms_wall_workspace_bytes(nc, nl, ctypes.byref(nbytes)))
    work = torch.empty(nbytes.value, dtype=torch.uint8, device="cuda")
    a = psms.WallArgs(nc, 0, nl, kx.data_ptr(), ky.data_ptr(), 3e4, 40.0, 700.0,
                      *[at[k].data_ptr() for k in ("g_om", "g_w", "g_phi", "om", "w", "phi", "u", "v")])
    psms._check(psms.lib().psms_wall_solve(ctypes.byref(a), psms._ptr(work), nbytes.value, psms._stream()))
    for k, name in (("om", "omega"), ("w", "w"), ("phi", "phi"), ("u", "u"), ("v", "v")):
        if k not in over.values():
            assert torch.equal(at[k], want[name]), k


# beta far beyond any time step's, where the product of a piece's rows passes the
# largest double: w and phi as the dense oracle has them, to the bar of the other
# wall-solve tests.  (Not omega: its last coefficients are differences of terms of beta
# times their size, here and in the oracle.)
@pytest.mark.parametrize("nc", [16, 32, 64, 96, 128, 256])
@pytest.mark.parametrize("beta", [1e38, 1e60, 1e150])
def test_wall_solve_of_very_large_beta(nc, beta):
    from oracle import channel as ch
    from paper_2406_01322_amd import psms
    rng = np.random.default_rng(nc)
    kx, ky = np.array([0.0, 0.5, 3.0]), np.array([0.0, -1.0, 2.0])
    g = [(rng.standard_normal((nc + 1, 3)) + 1j * rng.standard_normal((nc + 1, 3)))
         * np.exp(-0.05 * np.arange(nc + 1))[:, None] for _ in range(3)]
    k2 = kx ** 2 + ky ** 2
    want = ch.wall_normal_solve_lines(*g, kx, ky, k2 + beta, k2 + beta, k2 + 700.0)
    got = psms.wall_solve(_dev(kx), _dev(ky), beta, beta, 700.0, *[_dev(x) for x in g])
    assert all(np.all(np.isfinite(_host(x))) for x in got.values())
    for key in ("w", "phi"):
        a, b = _host(got[key]), want[key]
        assert np.all(np.max(np.abs(a - b), axis=0) <= 1e-11 * np.max(np.abs(b), axis=0)), key


# Chains longer than the table of the rows' constants (n <= 256), to the bars that the
# shorter ones are held to.
@pytest.mark.parametrize("kind", ["dirichlet", "neumann"])
@pytest.mark.parametrize("nc", [257, 258, 300, 513])
def test_helmholtz_beyond_the_table(kind, nc):
    from oracle import channel as ch
    from paper_2406_01322_amd import psms
    rng = np.random.default_rng(nc)
    g = (rng.standard_normal((nc + 1, 5)) + 1j * rng.standard_normal((nc + 1, 5))) \
        * np.exp(-0.03 * np.arange(nc + 1))[:, None]
    beta = 1e3 * (0.5 + rng.random(5))
    bcv = rng.standard_normal((5, 2)) + 1j * rng.standard_normal((5, 2))
    want = np.stack([ch.helmholtz(g[:, l], beta[l], kind, *bcv[l]) for l in range(5)], axis=1)
    for f in (psms.cheb_helmholtz, psms.cheb_helmholtz_noalloc):
        got = _host(f(_dev(g), _dev(beta), kind, _dev(bcv)))
        assert np.max(np.abs(got - want)) <= 1e-11 * np.max(np.abs(want))


@pytest.mark.parametrize("nc,nl", [(258, 7), (287, 3)])
def test_wall_solve_beyond_the_table(nc, nl):
    test_pieced_wall_solve_sizes(nc, nl)


# A run continued from a saved state takes the bits of the run that saved it: the
# derivatives of a state that is set are those that the step leaves, in every form of
# the step's kernel (longest chains, both parities in a workgroup, single phase).
@pytest.mark.parametrize("nc,walls,single", [(8, "nn", False), (48, "fn", False), (96, "nf", False), (128, "nn", False),
                                             (128, "fn", False), (128, "ff", False), (256, "nn", False),
                                             (256, "fn", False), (256, "nn", True)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_restart_takes_the_same_bits(nc, walls, single, precision):
    from paper_2406_01322_amd.psms import Channel
    kinds = tuple({"n": "noslip", "f": "freeslip"}[c] for c in walls)
    a, b = (Channel(24, 16, nc, 150.0, 3.0, 0.1, 10.0, 1e-4, walls=kinds, single_phase=single, precision=precision)
            for _ in range(2))
    f = list(_channel_fields(24, 16, nc, nc))
    if single:
        f[3] = np.zeros_like(f[3])
    a.init_state(*[_dev(x) for x in f])
    a.step(2)
    b.set_state(*[t.clone() for t in a.get_state(with_history=True)], nstep=2)
    for s in (a, b):
        s.step(2)
    assert all(torch.equal(x, y) for x, y in zip(a.get_state(with_history=True), b.get_state(with_history=True)))


# Chains in one piece (up to nc = 16) and just beyond: line counts around a workgroup's
# 64, alone and in a step whose walls couple the parities.
@pytest.mark.parametrize("nc,nl", [(4, 64), (12, 63), (16, 65), (24, 128), (32, 63), (48, 130), (64, 1)])
def test_wall_solve_piece_counts(nc, nl):
    test_pieced_wall_solve_sizes(nc, nl)


@pytest.mark.parametrize("nc,walls", [(4, "fn"), (12, "fn"), (16, "nf"), (24, "fn"), (32, "nf")])
def test_channel_step_piece_counts(nc, walls):
    test_channel_step_sizes_and_walls(24, 16, nc, walls, False)


# The longest chains against the oracle on every coefficient: two-phase at 17 slots a
# piece, and each pair of walls that is not no-slip at both, an AB1 and an AB2 step
# from the oracle's state.  State to 1e-12 of each field's maximum, the explicit terms
# to 4e-9 (nc / 256)^2, as for the other one-step tests.
@pytest.mark.parametrize("nc,walls", [(256, "nn")] + [(nc, w) for nc in (96, 128, 256) for w in ("fn", "nf", "ff")])
@pytest.mark.parametrize("nprev", [0, 1])
def test_long_chains_one_step_parity(nc, walls, nprev):
    from oracle import channel_step as cs
    from paper_2406_01322_amd.psms import Channel
    kinds = tuple({"n": "noslip", "f": "freeslip"}[c] for c in walls)
    prm = cs.ChannelParams(nx=16, ny=12, nc=nc, re=150.0, we=3.0, ch=0.1, pe=10.0, dt=1e-4, walls=kinds)
    st = cs.run(cs.init_state(*_channel_fields(16, 12, nc, nc), prm), prm, nprev)
    c = Channel(16, 12, nc, prm.re, prm.we, prm.ch, prm.pe, prm.dt, walls=kinds)
    c.set_state(*[_dev(x) for x in (np.stack([st["om"], st["w"], st["phi"]]), st["mean"],
                                    np.stack([st["h_om"], st["h_w"], st["h_phi"]]), st["h_mean"])], nstep=nprev)
    c.step(1)
    want = cs.step(st, prm)
    state, mean, hist, hmean = (_host(x) for x in c.get_state(with_history=True))
    bar, hbar = 1e-12, 4e-9 * (nc / 256.0) ** 2
    for a, b, tol in ((state[0], want["om"], bar), (state[1], want["w"], bar), (state[2], want["phi"], bar),
                      (mean, want["mean"], bar), (hist[0], want["h_om"], hbar), (hist[1], want["h_w"], hbar),
                      (hist[2], want["h_phi"], hbar), (hmean, want["h_mean"], hbar)):
        assert np.max(np.abs(a - b)) <= tol * np.max(np.abs(b))


# The same for the two smallest sizes, with boxes enough (more than 4096 lines of the
# band) to leave the z stage of few lines.
@pytest.mark.parametrize("n,boxes", [(8, 274), (12, 147)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_z_stages_give_the_same_bits_smallest(n, boxes, precision):
    K = (n - 1) // 3
    assert (2 * K + 1) * (K + 1) * boxes > 4096
    test_z_stages_give_the_same_bits(n, boxes, precision)


# Partial radix rounds on swizzled rows: one step against the oracle's adjoint, to the
# same bar.
def test_adjoint_x_stage_96():
    from oracle import adjoint as oadj
    from paper_2406_01322_amd.psms import Adjoint
    n = 96
    prm = box.Params(n=n, re=50.0, we=1.0, ch=0.2, pe=5.0, dt=1e-3)
    x = 2 * np.pi * np.arange(n) / n
    z, y, x = np.meshgrid(x, x, x, indexing="ij")
    u = np.stack([np.sin(x) * np.cos(y) * np.cos(z), -np.cos(x) * np.sin(y) * np.cos(z), 0.3 * np.cos(x + 2 * y)])
    phi = np.cos(x) * np.sin(y - z) + 0.1 * np.random.default_rng(n).standard_normal((n, n, n))
    J0, d0, w0, _ = oadj.gradient(u, phi, prm, 1)
    a = Adjoint(n, prm.re, prm.we, prm.ch, prm.pe, prm.dt, precision="fp64", max_steps=1, seg_len=1)
    J = a.forward(_dev(u), _dev(phi), 1)
    d, w = a.backward()
    assert abs(J - J0) <= 1e-10 * abs(J0)
    assert np.linalg.norm(_host(d) - d0) <= 1e-10 * np.linalg.norm(d0)
    assert abs(w - w0) <= 1e-10 * abs(w0)


# The largest two: the derivatives along one direction of phi0 and in We against
# central differences of J (two step sizes, extrapolated), to the 1e-6 of the adjoint
# tests.
@pytest.mark.parametrize("n", [192, 256])
def test_adjoint_of_the_largest_grids(n):
    from paper_2406_01322_amd.psms import Adjoint
    x = 2 * np.pi * torch.arange(n, dtype=torch.float64, device="cuda") / n
    z, y, x = torch.meshgrid(x, x, x, indexing="ij")
    rng = np.random.default_rng(n)

    def field():
        f = torch.zeros_like(x)
        for _ in range(6):
            k, s = rng.integers(-3, 4, size=3), rng.uniform(0, 6)
            f += float(rng.uniform(0.1, 0.3)) * torch.cos(float(k[0]) * x + float(k[1]) * y + float(k[2]) * z + s)
        return f

    u = torch.stack([torch.sin(x) * torch.cos(y) * torch.cos(z), -torch.cos(x) * torch.sin(y) * torch.cos(z),
                     0.3 * torch.cos(x + 2 * y)])
    phi, e = field(), field()

    def J(s, we=1.0):
        return Adjoint(n, 50.0, we, 0.2, 5.0, 1e-3, precision="fp64", max_steps=2, seg_len=2).forward(u, phi + s * e, 2)

    def slope(f, h):
        d = [(f(s) - f(-s)) / (2 * s) for s in (h, h / 2)]
        return (4 * d[1] - d[0]) / 3

    a = Adjoint(n, 50.0, 1.0, 0.2, 5.0, 1e-3, precision="fp64", max_steps=2, seg_len=2)
    a.forward(u, phi, 2)
    d, dwe = a.backward()
    for got, want in ((float((d * e).sum()), slope(J, 1e-2)), (dwe, slope(lambda s: J(0.0, 1.0 + s), 1e-2))):
        assert abs(got - want) <= 1e-6 * abs(want), (got, want)


# The nc-point route to the DCT-I (FP64, nc >= 96) sums the odd orders from both ends, so
# the rounding error of the upper half of the coefficients is that of the lower half
# (1.25 times at most, over 64 lines), where one sum over all of them leaves it 1.4 to 1.9
# times as large.  Against sums in long double.
@pytest.mark.parametrize("nc", [96, 128, 256])
@pytest.mark.parametrize("kind", ["smooth", "random"])
@pytest.mark.parametrize("direction", [+1, -1])
def test_dct_upper_orders_are_as_accurate_as_the_lower(nc, kind, direction):
    from paper_2406_01322_amd import psms
    rng = np.random.default_rng(nc)
    z = np.cos(np.pi * np.arange(nc + 1) / nc)[:, None]
    if kind == "smooth":
        x = (1 - z * z) ** 2 * (1 + 0.3 * np.sin(3 * z + rng.uniform(0, 6, 64))) * np.exp(1j * rng.uniform(0, 6, 64))
    else:
        x = rng.standard_normal((nc + 1, 64)) + 1j * rng.standard_normal((nc + 1, 64))
    n = np.arange(nc + 1)
    pi = np.longdouble("3.14159265358979323846264338327950288")
    M = np.cos(pi * (np.outer(n, n) % (2 * nc)).astype(np.longdouble) / nc)
    if direction > 0:
        cbar = np.where((n == 0) | (n == nc), 2, 1).astype(np.longdouble)
        M = (2 / np.longdouble(nc)) * M / cbar[:, None] / cbar[None, :]
    want = M @ x.real.astype(np.longdouble) + 1j * (M @ x.imag.astype(np.longdouble))
    e = np.abs(_host(psms.cheb_transform(_dev(x), direction)) - want)
    low, high = (float(np.sqrt(np.sum(e[k] ** 2))) for k in (slice(0, nc // 2), slice(nc // 2, None)))
    assert high <= 1.25 * low
