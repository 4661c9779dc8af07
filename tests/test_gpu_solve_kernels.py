"""The solve kernels at the sizes where their work splits change, against dense FP64 algebra.

The problems are chains of 2-DOF elements [[1, -1], [-1, 1]] + 0.05 I: A is tridiagonal with
eigenvalues in [0.05, 4.1], so a PCG solution with relative residual rho has a relative error of at
most 82 rho (2-norm condition number).
"""
import numpy as np
import pytest

from fegen.common import uniform_problem

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

COND = 82.0


def _lsdd():
    import paper_2607_07485_amd as P
    return P


def _chain(n):
    dofs = np.stack([np.arange(n - 1), np.arange(1, n)], axis=1)
    blocks = np.repeat((np.array([[1.0, -1.0], [-1.0, 1.0]]) + 0.05 * np.eye(2))[None], n - 1, axis=0)
    return uniform_problem(n, dofs, blocks, np.arange(n))


def _dense(prob):
    A = np.zeros((prob.n, prob.n))
    for e in range(prob.n_elem):
        d, B = prob.element(e)
        A[np.ix_(d, d)] += B
    return A


@pytest.mark.parametrize("nrhs", [1, 8, 9])
@pytest.mark.parametrize("n", [2, 255, 257, 1024, 1025, 2049])
def test_pcg_reduction_blocks(n, nrhs):
    """Segments of one reduction block, a full one, one entry more, several (1024 entries per block
    of a single vector, 256 DOFs of a block of 8 right-hand sides)."""
    P = _lsdd()
    prob = _chain(n)
    B = np.random.default_rng(n).standard_normal((nrhs, n))
    ref = np.linalg.solve(_dense(prob), B.T).T
    with P.Hierarchy.setup_problem(prob, P.Params.default(rtol=1e-12)) as h:
        X, infos = h.solve(torch.from_numpy(B if nrhs > 1 else B[0]).cuda())
    X = np.atleast_2d(X.cpu().numpy())
    assert all(f.converged == 1 and f.rel_res <= 1e-12 for f in infos)
    for x, r in zip(X, ref):
        assert np.linalg.norm(x - r) <= 2 * COND * 1e-12 * np.linalg.norm(r)


@pytest.mark.parametrize("nrhs", [1, 8, 9])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_non_finite_right_hand_side_leaves_the_output(nrhs, bad):
    P = _lsdd()
    prob = _chain(300)
    B = np.random.default_rng(0).standard_normal((nrhs, prob.n))
    B[-1, -1] = bad
    x = torch.full((nrhs, prob.n) if nrhs > 1 else (prob.n,), 7.0, dtype=torch.float64, device="cuda")
    with P.Hierarchy.setup_problem(prob) as h:
        with pytest.raises(P.LsddError) as e:
            h.solve(torch.from_numpy(B if nrhs > 1 else B[0]).cuda(), x)
        assert e.value.code == 1 and bool((x == 7.0).all())
        y, infos = h.solve(torch.ones(prob.n, dtype=torch.float64, device="cuda"))   # still usable
        assert infos[0].converged == 1
