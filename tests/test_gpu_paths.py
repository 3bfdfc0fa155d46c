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
