"""The separate edge sweep and prolongation of the hybrid V(1,1) cycle
(stencil = 1) against the fused box legs, an implementation of their own
(stencil = 0), on grids that end inside, at and past the edge sweep's 32 x 14
tiles and chunks of planes, for every boundary type and both transfers.

Tolerance: the same cycle in the same precision with sums in another order; a
level's operators amplify a rounding by at most |M| / |D| <= 3 and a cycle
chains fewer than 40 of them: 1e3 eps."""
import numpy as np
import pytest

import problems as P

D, N = P.DIRICHLET, P.NATURAL
pytestmark = pytest.mark.gpu

GRIDS = {
    "past_x": P.Grid(3, (64, 16, 16), 1 / 16, (D,) * 6, 63 + 64 * 7),
    "two_tiles": P.Grid(3, (128, 8, 8), 1 / 8, (N, D, D, N, D, N), -1),
    "ragged": P.Grid(3, (72, 28, 12), 1 / 28, (D, N, N, D, N, D), -1),
    "at_y": P.Grid(3, (12, 56, 20), 1 / 56, (D,) * 6, 0),
}


@pytest.mark.parametrize("transfer,varmu", [("div", True), ("smooth", False)])
@pytest.mark.parametrize("name", list(GRIDS))
def test_separate_hybrid_kernels_match_box_legs(name, transfer, varmu):
    import torch
    import paper_2001_10424_amd as gk
    print("[case] edge tiles", name, transfer, varmu, flush=True)
    g = GRIDS[name]
    mu = np.exp(np.random.default_rng(5).standard_normal(g.n_cells)) if varmu else None
    r = torch.tensor(np.random.default_rng(11).standard_normal(g.m_full), dtype=torch.float32,
                     device="cuda")
    out = []
    for stencil in (0, 1):
        s = gk.Solver(g, mu, 1e2, inner="mg", stencil=stencil, smoother="hybrid", nu_pre=1,
                      nu_post=1, mg_transfer=transfer, precision="mixed")
        out.append(s.precondition(r, "mixed").double().cpu().numpy())
        s.close()
    assert np.linalg.norm(out[0] - out[1]) <= 1e3 * 2.0 ** -23 * np.linalg.norm(out[1])
