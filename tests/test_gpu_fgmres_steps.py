"""FGMRES steps where their kernels change form: the basis size crosses a
register bucket (8, 16, 32 vectors), the restart cycle ends full or early, rows
fill one block, several, or more than the blocks whose partials the next
kernel sums itself.  The oracle is FGMRES in plain NumPy (modified
Gram-Schmidt), and for the large grid the FP64 residual."""
import numpy as np
import pytest

from csr_cases import random_system

pytestmark = pytest.mark.gpu

D = 0


def _fgmres(M, d, f, tol, restart, maxit):
    """x and the number of steps of restarted, Jacobi right-preconditioned
    GMRES from zero."""
    x, it, r0 = np.zeros_like(f), 0, np.linalg.norm(f)
    while True:
        r = f - M @ x
        beta = np.linalg.norm(r)
        if beta <= tol * r0 or it >= maxit:
            return x, it
        V, Z, H = [r / beta], [], np.zeros((restart + 1, restart))
        for j in range(restart):
            Z.append(V[j] / d)
            w = M @ Z[j]
            for _ in range(2):
                for i in range(j + 1):
                    h = V[i] @ w
                    H[i, j] += h
                    w = w - h * V[i]
            H[j + 1, j] = np.linalg.norm(w)
            V.append(w / H[j + 1, j])
            it += 1
            e = np.zeros(j + 2)
            e[0] = beta
            y = np.linalg.lstsq(H[:j + 2, :j + 1], e, rcond=None)[0]
            if np.linalg.norm(e - H[:j + 2, :j + 1] @ y) <= tol * r0:
                break
        x = x + np.array(Z).T @ y


@pytest.mark.parametrize("m,n,restart,eta", [(200, 40, 8, 2.0), (257, 60, 9, 2.0),
                                             (300, 1, 17, 2.0), (900, 200, 33, 300.0),
                                             (900, 200, 64, 300.0), (1500, 300, 1, 2.0)])
def test_steps_match_numpy(m, n, restart, eta):
    """On the centrally scaled system (condition number below 1e4; the step
    counts of the oracle do not move under relative perturbations of M by
    1e-15): the same step count up to one, and the same solution: both
    residuals are below tol |f|, so the solutions differ by at most
    2 tol cond(M) |x|."""
    import torch
    import paper_2001_10424_amd as gk
    W, A = random_system(m, n, 5)
    tol = 1e-9
    W_, A_ = W.toarray(), A.toarray()
    sw = 1 / np.sqrt(np.diag(W_))
    sp = 1 / np.sqrt((A_ ** 2 * sw[:, None] ** 2).sum(0))
    A_ = sw[:, None] * A_ * sp
    M = sw[:, None] * W_ * sw + eta * A_ @ A_.T
    f = np.random.default_rng(m).standard_normal(m)
    x_ref, it_ref = _fgmres(M, np.diag(M), f, tol, restart, 3000)
    s = gk.CsrSolver(W, A, eta, scaling="central", krylov="fgmres", fgmres_restart=restart,
                     inner_maxit=4000)
    for _ in range(2):  # the second solve replays the captured cycle
        x, its = s.inner_solve(torch.tensor(f, device="cuda"), tol)
        x = x.cpu().numpy()
        print(m, n, restart, "steps", its, it_ref, flush=True)
        assert np.linalg.norm(f - M @ x) <= tol * np.linalg.norm(f) * (1 + 1e-6)
        assert np.linalg.norm(x - x_ref) <= 2 * tol * np.linalg.cond(M) * np.linalg.norm(x_ref)
        assert abs(its - it_ref) <= 1
    s.close()


@pytest.mark.parametrize("n,precision", [((48, 40, 40), "fp64"), ((40, 40, 40), "fp64"),
                                         ((40, 40, 36), "fp64"), ((48, 40, 40), "mixed")])
def test_steps_beside_the_block_limit(n, precision):
    """Grids above, just above and just below 196608 faces, V-cycle preconditioner: the
    solution meets the tolerance (FP32 inner solves stop on their estimate,
    which is good to about eps_32 |M| |x| / |f|, here below 1e-3)."""
    import types

    import torch
    import paper_2001_10424_amd as gk
    g = types.SimpleNamespace(dim=3, n=n, h=1.0 / n[1], bc=(D,) * 6, pin=0)
    tol = 1e-9 if precision == "fp64" else 1e-3
    s = gk.Solver(g, None, 1.0, inner="mg", krylov="fgmres", fgmres_restart=12,
                  precision=precision)
    gen = torch.Generator(device="cuda").manual_seed(3)
    x0 = torch.randn(s.m_full, generator=gen, dtype=torch.float64, device="cuda")
    f = s.apply("M", x0)
    x, its = s.inner_solve(f, tol)
    res = f - s.apply("M", x)
    print(n, precision, "faces", s.m_full, "steps", its, float(res.norm() / f.norm()), flush=True)
    assert float(res.norm()) <= (1 + 1e-6 if precision == "fp64" else 2) * tol * float(f.norm())
    s.close()
