"""The marching V-cycle legs of the large 3D levels against the separate
generic kernels (stencil = 1): extents that end inside, at and just past the
tiles (32 x 16 and 16 x 16) and the chunks of planes, every boundary type, the
pinned cell at the edge of a tile and chunk, both transfers, both precisions.

Tolerance: the same V-cycle in the same precision with sums in another order.
A level's operators amplify a rounding by at most |M| / |D| <= 3 and a cycle
chains fewer than 40 of them, so 1e3 eps of the precision bounds the relative
difference."""
import numpy as np
import pytest

import problems as P

D, N = P.DIRICHLET, P.NATURAL
pytestmark = pytest.mark.gpu

WALLS = (D,) * 6
GRIDS = {
    "exact": P.Grid(3, (64, 64, 96), 1 / 64, WALLS, 0),
    "ragged": P.Grid(3, (72, 40, 88), 1 / 40, WALLS, (31 * 40 + 15) * 72 + 32),
    "thin": P.Grid(3, (136, 72, 40), 1 / 72, (D, D, D, D, D, N), -1),
    "nat": P.Grid(3, (48, 72, 88), 1 / 72, (N, D, D, N, N, N), -1),
    "nat_x": P.Grid(3, (80, 48, 72), 1 / 48, (D, N, N, D, D, D), (36 * 48 + 47) * 80 + 79),
}


@pytest.mark.parametrize("transfer,precision", [
    ("smooth", "fp64"), ("smooth", "mixed"), ("div", "fp64")])
@pytest.mark.parametrize("name", list(GRIDS))
def test_marching_legs_match_separate_kernels(name, transfer, precision):
    import torch
    import paper_2001_10424_amd as gk
    print("[case] march", name, transfer, precision, flush=True)
    g = GRIDS[name]
    dt = torch.float64 if precision == "fp64" else torch.float32
    # entries at faces that are no unknown must not matter
    r = torch.tensor(np.random.default_rng(11).standard_normal(g.m_full), dtype=dt, device="cuda")
    out = []
    for stencil in (0, 1):
        s = gk.Solver(g, None, 1e2, inner="mg", stencil=stencil, nu_pre=2, nu_post=2,
                      mg_transfer=transfer, precision=precision)
        z = s.precondition(r, precision)
        assert torch.equal(z, s.precondition(r, precision))
        out.append(z.double().cpu().numpy())
        s.close()
    assert np.all(out[0][g.face_mask() == 0] == 0)
    eps = 2.0 ** -52 if precision == "fp64" else 2.0 ** -23
    err = np.linalg.norm(out[0] - out[1]) / np.linalg.norm(out[1])
    big = np.abs(out[0] - out[1]).max() / np.abs(out[1]).max()
    print("   relative difference", err, big, flush=True)
    assert err <= 1e3 * eps and big <= 1e4 * eps


@pytest.mark.parametrize("n,eta", [((256, 256, 2), 1.0), ((250, 200, 2), 1e3), ((254, 250, 3), 1.0)])
def test_slabs_too_thin_to_march(n, eta):
    """Grids of two and three planes with more cells than the box legs take:
    set up with the Jacobi inner solver, their residual against the oracle
    (entries of at most 30 products: 64 eps), and refused for multigrid,
    whose coarsest level they are."""
    import oracle
    import torch
    import paper_2001_10424_amd as gk
    print("[case] slab", n, eta, flush=True)
    g = P.Grid(3, n, 0.5, WALLS, 0)
    rng = np.random.default_rng(3)
    mask = g.face_mask()
    v = [rng.standard_normal(g.m_full) * mask, rng.standard_normal(g.n_cells),
         rng.standard_normal(g.m_full) * mask, rng.standard_normal(g.n_cells)]
    s = gk.Solver(g, None, eta, inner="jacobi")
    dev = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in v]
    _, rw, rr = s.residual(*dev, want_vectors=True)
    s.close()
    for a, b in zip((rw, rr), oracle.saddle_residual(g, *v)[:2]):
        assert np.abs(a.cpu().numpy() - b).max() <= 64 * 2.0 ** -52 * np.abs(b).max()
    with pytest.raises(RuntimeError, match="invalid argument"):
        gk.Solver(g, None, eta, inner="mg")


@pytest.mark.parametrize("transfer,precision", [
    ("smooth", "fp64"), ("smooth", "mixed"), ("div", "fp64")])
@pytest.mark.parametrize("name", ["ragged", "thin", "nat", "nat_x"])
def test_marching_legs_in_pcg(name, transfer, precision):
    """Inner solves whose r.z comes from the marching legs' partial sums: the
    same iterates as with the separate kernels.  A face missed or counted twice
    changes r.z by 1e-6 of it, a row of faces by 1e-4.

    Tolerance: rounding of up to 40 operators a cycle adds up like a random
    walk, sqrt(40) times 3 eps, and the recurrences carry it along (a factor of
    5): 1e2 eps per iteration.  That holds for the first iterations and without
    a pinned cell, whose single mode CG finds first and then again from
    rounding."""
    import dataclasses

    import torch
    import paper_2001_10424_amd as gk
    print("[case] march in PCG", name, transfer, precision, flush=True)
    g = dataclasses.replace(GRIDS[name], pin=-1)
    f = torch.tensor(P.random_vector(g, 6), dtype=torch.float64, device="cuda")
    out = []
    for stencil in (0, 1):
        s = gk.Solver(g, None, 1e2, inner="mg", stencil=stencil, nu_pre=2, nu_post=2,
                      mg_transfer=transfer, precision=precision)
        out.append(s.inner_solve(f, 0.3))
        s.close()
    (x, its), (xs, its_s) = out
    eps = 2.0 ** -52 if precision == "fp64" else 2.0 ** -23
    err = float((x - xs).norm() / xs.norm())
    print("   iterations", its, its_s, "relative difference", err, flush=True)
    assert its == its_s and its >= 8
    assert err <= 1e2 * eps * its
