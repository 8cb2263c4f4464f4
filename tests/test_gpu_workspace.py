"""max_workspace_bytes: the device footprints of contexts stay within what they
were before the fused kernels took buffers of their own (the bounds below), so
a limit that sufficed goes on sufficing; one byte less than the footprint is
refused."""
import pytest

import problems as P
from csr_cases import random_system

D = P.DIRICHLET
pytestmark = pytest.mark.gpu

LIMITS = [  # grid, options, bytes
    ((2, 2, 1), dict(inner="mg", precision="mixed", krylov="fgmres"), 43080),
    ((2, 2, 2), dict(inner="jacobi", precision="mixed", krylov="fgmres"), 50984),
    ((8, 6, 1), dict(inner="jacobi", precision="fp64", krylov="fgmres"), 111192),
    ((64, 16, 1), dict(inner="mg", precision="fp64"), 2931136),
    ((64, 64, 1), dict(inner="mg", precision="mixed", krylov="fgmres"), 5979960),
    ((512, 512, 1), dict(inner="mg", precision="fp64", smoother="hybrid"), 144280288),
    ((1280, 1024, 1), dict(inner="mg", precision="mixed"), 492153600),
    ((1280, 1024, 1), dict(inner="mg", precision="fp64"), 625112992),
    ((16, 16, 16), dict(inner="mg", precision="fp64", krylov="fgmres"), 33120216),
    ((32, 32, 32), dict(inner="mg", precision="fp64"), 45907952),
    ((48, 40, 40), dict(inner="mg", precision="mixed", krylov="fgmres"), 101065944),
    ((72, 40, 88), dict(inner="mg", precision="fp64"), 190751264),
]
CSR_LIMITS = [  # m, n, density, options, bytes
    (60, 20, 0.02, dict(precision="mixed", krylov="fgmres"), 67984),
    (300, 100, 0.02, dict(precision="fp64"), 170520),
    (3000, 500, 0.02, dict(precision="mixed", krylov="fgmres"), 9672856),
    (20000, 2000, 0.0005, dict(precision="fp64", krylov="fgmres"), 23015888),
]


def _check(make, limit):
    s = make(limit)
    used = s.stats()["workspace_bytes"]
    s.close()
    assert used <= limit
    with pytest.raises(RuntimeError, match="memory|cap|workspace"):
        make(used - 1)


@pytest.mark.parametrize("n,options,limit", LIMITS)
def test_grid_context_fits_its_limit(n, options, limit):
    import paper_2001_10424_amd as gk
    print("[case] workspace", n, options, flush=True)
    dim = 2 if n[2] == 1 else 3
    g = P.Grid(dim, n, 1.0 / min(n[:dim]), (D,) * 6, 0)
    nu = 1 if options.get("smoother") == "hybrid" else 2
    _check(lambda cap: gk.Solver(g, None, 10.0, nu_pre=nu, nu_post=nu, max_workspace_bytes=cap,
                                 **options), limit)


@pytest.mark.parametrize("m,n,density,options,limit", CSR_LIMITS)
def test_assembled_context_fits_its_limit(m, n, density, options, limit):
    import paper_2001_10424_amd as gk
    print("[case] workspace assembled", m, n, options, flush=True)
    W, A = random_system(m, n, 5, density=density)
    _check(lambda cap: gk.CsrSolver(W, A, 1.0, max_workspace_bytes=cap, **options), limit)
