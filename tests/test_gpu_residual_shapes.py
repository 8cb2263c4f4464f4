"""The saddle residual kernel against the CPU oracle where its columns, planes
and boundary selects change: extents below, at and past a block's 512 columns
and an odd number of planes, do-nothing sides on every axis, a pinned cell in
the middle, two cells per axis, constant and variable viscosity, with and
without the face residual.

Tolerance: both sides form every entry in FP64 from at most 30 products; the
difference is below 64 eps of the largest entry of |g| + |W||w| + |A||p|,
which the largest residual entry is of (random inputs)."""
import numpy as np
import pytest

import oracle
import problems as P

D, N = P.DIRICHLET, P.NATURAL
pytestmark = pytest.mark.gpu

GRIDS = {
    "3d_two": P.Grid(3, (2, 2, 2), 0.5, (D,) * 6, 0),
    "3d_thin": P.Grid(3, (31, 15, 2), 0.1, (D, N, D, D, N, D), -1),   # 32 x 16 columns = 512
    "3d_odd": P.Grid(3, (23, 37, 19), 1 / 37, (D,) * 6, 23 * 37 * 9 + 23 * 18 + 11),
    "3d_nat": P.Grid(3, (22, 9, 13), 1 / 9, (N, D, D, N, N, N), -1),
    "3d_deep": P.Grid(3, (130, 127, 62), 1 / 127, (D, N, D, D, D, D), 0),
    "2d_small": P.Grid(2, (5, 3, 1), 1 / 3, (N, N, D, D, D, D), -1),
    "2d_odd": P.Grid(2, (73, 34, 1), 1 / 34, (D, D, N, D, D, D), 100),
}


@pytest.mark.parametrize("varmu", [False, True])
@pytest.mark.parametrize("name", list(GRIDS))
def test_residual_matches_oracle(name, varmu):
    import torch
    import paper_2001_10424_amd as gk
    print("[case] residual", name, varmu, flush=True)
    grid = GRIDS[name]
    rng = np.random.default_rng(3)
    mu = np.exp(rng.standard_normal(grid.n_cells)) if varmu else None
    mask = grid.face_mask()
    g, w = rng.standard_normal(grid.m_full) * mask, rng.standard_normal(grid.m_full) * mask
    r, p = rng.standard_normal(grid.n_cells), rng.standard_normal(grid.n_cells)
    ref_w, ref_r, _ = oracle.saddle_residual(grid, g, r, w, p, mu=mu)
    rp = r.copy()
    if grid.pin >= 0:
        rp[grid.pin] = 0.0
    # NumPy sums in pairs: a few eps (the oracle adds its squares one by one,
    # up to an eps per entry)
    sq = [np.sum(a * a) for a in (ref_w, ref_r, g, rp)]
    ref_n = np.sqrt([sq[0] + sq[1], sq[0], sq[1], sq[2] + sq[3]])
    s = gk.Solver(grid, mu, 10.0, inner="jacobi")
    dev = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in (g, r, w, p)]
    norms, rw, rr = s.residual(*dev, want_vectors=True)
    norms2, _, _ = s.residual(*dev)
    s.close()
    eps = 64 * 2.0 ** -52
    for a, b in ((rw, ref_w), (rr, ref_r)):
        assert np.abs(a.cpu().numpy() - b).max() <= eps * max(np.abs(b).max(), 1.0)
    # sums of squares: a few eps per entry and one per addition level
    assert np.allclose(norms, ref_n, rtol=eps, atol=0) and norms2 == norms


@pytest.mark.parametrize("name", ["3d_nat", "3d_deep", "2d_odd"])
def test_results_on_their_inputs(name):
    """res_w on g, and res_r on r, on p or at the start of g: the same norms,
    and the residuals of buffers of their own (up to the contraction of a
    multiply-add: 64 eps of the largest entry)."""
    import ctypes as C

    import torch
    import paper_2001_10424_amd as gk
    print("[case] residual in place", name, flush=True)
    grid = GRIDS[name]
    gen = torch.Generator(device="cuda").manual_seed(4)
    n = {"g": grid.m_full, "r": grid.n_cells, "w": grid.m_full, "p": grid.n_cells}
    v = {k: torch.randn(m, generator=gen, dtype=torch.float64, device="cuda") for k, m in n.items()}
    s = gk.Solver(grid, None, 10.0, inner="jacobi")
    norms, rw, rr = s.residual(*v.values(), want_vectors=True)

    def call(on_w, on_r, alloc):
        c = {k: t.clone() for k, t in v.items()}
        ow = c[on_w] if on_w else None
        if not alloc:
            got, _, _ = gk.residual_noalloc(grid, *c.values(), res_w=ow, res_r=c[on_r][:grid.n_cells])
        else:
            got = (C.c_double * 4)()
            rc = gk.library().gkb_residual(s._ctx, *[gk._ptr(t) for t in c.values()], gk._ptr(ow),
                                           gk._ptr(c[on_r]), got)
            assert rc == 0
        return list(got), ow, c[on_r][:grid.n_cells]

    for alloc in (True, False):
        for on_w, on_r in (("g", "r"), ("g", "p"), (None, "p"), (None, "g")):
            got, ow, orr = call(on_w, on_r, alloc)
            assert got == norms
            assert ow is None or torch.equal(ow, rw)
            assert float((orr - rr).abs().max()) <= 64 * 2.0 ** -52 * float(rr.abs().max())
    s.close()
