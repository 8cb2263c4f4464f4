"""The fused V-cycle legs (one kernel down, one up per level) against the
separate generic kernels (stencil = 1) on grids that end inside, at and just
past their tiles, for every boundary type, both transfers, both smoothers and
both precisions.

Tolerances: both sides run the same V-cycle in the same precision with sums
in another order.  A level's operators amplify a rounding by at most
|M| / |D| <= 3 and a cycle chains fewer than 40 of them, so 1e3 eps of the
precision bounds the relative difference with room for the levels' sum."""
import numpy as np
import pytest

import problems as P

D, N = P.DIRICHLET, P.NATURAL

pytestmark = pytest.mark.gpu

WALLS = (D,) * 6
GRIDS = {
    # 8 x 8 tiles: remainders 4 and 2, one cell row past a tile
    "2d_small": P.Grid(2, (40, 36, 1), 1 / 36, WALLS, 0),
    "2d_rem2": P.Grid(2, (50, 58, 1), 1 / 58, (D, N, D, D, D, D), -1),
    "2d_nat": P.Grid(2, (64, 48, 1), 1 / 48, (N, D, D, N, D, D), 64 * 21 + 33),
    # 32 x 16 tiles: remainder 16, exact
    "2d_large": P.Grid(2, (368, 368, 1), 1 / 368, WALLS, 367),
    "2d_large_nat": P.Grid(2, (512, 272, 1), 1 / 272, (D, N, N, D, D, D), -1),
    # 4^3 tiles, 8 x 8 x 4 tiles, 8^3 tiles
    "3d_small": P.Grid(3, (10, 12, 14), 1 / 12, WALLS, 5 * 120 + 37),
    "3d_small_nat": P.Grid(3, (16, 12, 14), 1 / 12, (D, N, N, D, D, N), -1),
    "3d_medium": P.Grid(3, (20, 20, 18), 1 / 20, WALLS, 0),
    "3d_medium_nat": P.Grid(3, (36, 20, 24), 1 / 20, (N, D, D, N, N, D), -1),
    "3d_large": P.Grid(3, (40, 40, 44), 1 / 40, WALLS, 9 * 1600 + 8 * 40 + 7),
    "3d_large_nat": P.Grid(3, (72, 40, 40), 1 / 40, (D, N, D, D, D, N), -1),
}


def _dev(x, dtype):
    import torch
    return torch.tensor(np.asarray(x), dtype=dtype, device="cuda")


@pytest.mark.parametrize("smoother,transfer,varmu,precision", [
    ("jacobi", "div", False, "fp64"), ("jacobi", "smooth", True, "mixed"),
    ("hybrid", "smooth", False, "mixed"), ("hybrid", "div", True, "fp64")])
@pytest.mark.parametrize("name", list(GRIDS))
def test_fused_legs_match_separate_kernels(name, smoother, transfer, varmu, precision):
    import torch
    import paper_2001_10424_amd as gk
    print("[case] legs", name, smoother, transfer, varmu, precision, flush=True)
    g = GRIDS[name]
    mu = np.exp(np.random.default_rng(5).standard_normal(g.n_cells)) if varmu else None
    nu = 1 if smoother == "hybrid" else 2
    dt = torch.float64 if precision == "fp64" else torch.float32
    # entries at faces that are no unknown must not matter
    r = _dev(np.random.default_rng(11).standard_normal(g.m_full), dt)
    out = []
    for stencil in (0, 1):
        s = gk.Solver(g, mu, 1e2, inner="mg", stencil=stencil, smoother=smoother, nu_pre=nu,
                      nu_post=nu, mg_transfer=transfer, precision=precision)
        z = s.precondition(r, precision)
        out.append(z.double().cpu().numpy())
        # PCG with its scalar steps folded into the product, the update and
        # the way down (stencil = 0) needs the same iterations, and its
        # recursive residual is the true one (FP32 iterates: to their rounding)
        f = _dev(P.random_vector(g, 6), torch.float64)
        x, it = s.inner_solve(f, 1e-4)
        res = f - s.apply("M", x)
        assert float(res.norm() / f.norm()) <= (1.0001e-4 if precision == "fp64" else 1e-2)
        out.append(it)
        s.close()
    a, ia, b, ib = out
    eps = 2.0 ** -52 if precision == "fp64" else 2.0 ** -23
    assert np.linalg.norm(a - b) <= 1e3 * eps * np.linalg.norm(b)
    assert np.all(a[g.face_mask() == 0] == 0)
    assert abs(ia - ib) <= 1 + 0.02 * ib, (ia, ib)


@pytest.mark.parametrize("n", [32, 56])
def test_direction_buffers_alternate_for_any_chunk(n):
    """FP32 PCG alternates between two direction buffers: chunks of an even
    and of an odd number of iterations, and single iterations, are the same
    arithmetic (32^3: folded steps; 56^3: the separate kernels, where an odd
    chunk runs the plain update, whose result is the same bits up to the
    contraction of one multiply-add)."""
    import torch
    import paper_2001_10424_amd as gk
    print("[case] chunks", n, flush=True)
    pr = P.stokes_problem(3, n, seed=6, eta=10.0)
    f = _dev(pr.g, torch.float64)
    out = []
    for chunk in (8, 5, 1):
        s = gk.Solver(pr.grid, None, pr.eta, inner="mg", precision="mixed", check_every=chunk)
        x, it = s.inner_solve(f, 1e-4)
        out.append((x, it))
        s.close()
    for x, it in out[1:]:
        assert it == out[0][1]
        assert float((x - out[0][0]).norm() / x.norm()) <= (0.0 if n == 32 else 1e-5)


@pytest.mark.parametrize("name,smoother,precision", [
    ("2d_nat", "hybrid", "fp64"), ("3d_medium", "hybrid", "mixed"), ("3d_large", "jacobi", "fp64")])
def test_precondition_on_its_input(name, smoother, precision):
    """z on r: the same bits as in a vector of its own."""
    import ctypes as C

    import torch
    import paper_2001_10424_amd as gk
    from paper_2001_10424_amd import _abi
    print("[case] precondition in place", name, smoother, precision, flush=True)
    g = GRIDS[name]
    nu = 1 if smoother == "hybrid" else 2
    for stencil in (0, 1):
        s = gk.Solver(g, None, 1e2, inner="mg", stencil=stencil, smoother=smoother, nu_pre=nu,
                      nu_post=nu, precision=precision)
        r = _dev(np.random.default_rng(8).standard_normal(g.m_full),
                 torch.float64 if precision == "fp64" else torch.float32)
        z = s.precondition(r, precision)
        p = C.c_void_p(r.data_ptr())
        prec = _abi.FP64 if precision == "fp64" else _abi.MIXED
        assert gk.library().gkb_precondition(s._ctx, prec, p, p) == 0
        assert torch.equal(r, z)
        s.close()


@pytest.mark.parametrize("smoother,precision", [("jacobi", "fp64"), ("hybrid", "mixed")])
def test_large_2d_legs_with_separate_scalar_steps(smoother, precision):
    """2D grids with more partials than the folded PCG steps sum (2048): legs
    beside the separate update and scalar kernels, against the generic
    kernels (stencil = 1), in the tolerances of the smaller grids."""
    import torch
    import paper_2001_10424_amd as gk
    print("[case] large 2D legs", smoother, precision, flush=True)
    g = P.Grid(2, (1344, 1088, 1), 1 / 1088, (D, N, D, D, D, D), -1)
    nu = 1 if smoother == "hybrid" else 2
    dt = torch.float64 if precision == "fp64" else torch.float32
    r = _dev(np.random.default_rng(11).standard_normal(g.m_full), dt)
    f = _dev(P.random_vector(g, 6), torch.float64)
    out = []
    for stencil in (0, 1):
        s = gk.Solver(g, None, 10.0, inner="mg", stencil=stencil, smoother=smoother, nu_pre=nu,
                      nu_post=nu, precision=precision)
        x, it = s.inner_solve(f, 1e-4)
        res = f - s.apply("M", x)
        assert float(res.norm() / f.norm()) <= (1.0001e-4 if precision == "fp64" else 1e-2)
        out.append((s.precondition(r, precision).double(), it))
        s.close()
    (a, ia), (b, ib) = out
    eps = 2.0 ** -52 if precision == "fp64" else 2.0 ** -23
    assert float((a - b).norm()) <= 1e3 * eps * float(b.norm())
    assert abs(ia - ib) <= 1 + 0.02 * ib, (ia, ib)


@pytest.mark.parametrize("name,smoother,precision", [
    ("2d_small", "hybrid", "fp64"), ("3d_medium", "jacobi", "fp64"), ("3d_small", "jacobi", "mixed")])
def test_breakdown_keeps_the_iterate(name, smoother, precision):
    """A right-hand side that is not finite ends an inner solve in its first
    update: the error code, and the iterate of that time (0), also where the
    update is folded."""
    import ctypes as C

    import torch
    import paper_2001_10424_amd as gk
    from paper_2001_10424_amd import _abi
    print("[case] breakdown", name, smoother, precision, flush=True)
    g = GRIDS[name]
    nu = 1 if smoother == "hybrid" else 2
    for stencil in (0, 1):
        s = gk.Solver(g, None, 10.0, inner="mg", stencil=stencil, smoother=smoother, nu_pre=nu,
                      nu_post=nu, precision=precision)
        for bad in (float("nan"), float("inf")):
            f = _dev(P.random_vector(g, 6), torch.float64)
            f[int(torch.nonzero(f)[f.count_nonzero() // 2])] = bad
            x, it = torch.ones_like(f), C.c_int(-1)
            rc = gk.library().gkb_inner_solve(s._ctx, C.c_void_p(f.data_ptr()),
                                              C.c_void_p(x.data_ptr()), 1e-4, C.byref(it))
            assert (rc, it.value) == (_abi.GKB_ENAN, 0)
            assert float(x.abs().max()) == 0.0
        s.close()
