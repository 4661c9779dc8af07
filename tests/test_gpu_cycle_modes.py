"""Which kernels a cycle runs, for every smoother, precision and tuning."""
import numpy as np
import pytest

import fegen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _lsdd():
    import paper_2607_07485_amd as P
    return P


def _separate(h):
    """Separate launches on every level: shapes that are neither in effect nor the autotuner's."""
    for l in range(h.info()["levels"]):
        t = h.level_tuning(l)
        h.set_level_tuning(l, dict(lanes=t["lanes"], lanes_block=t["lanes_block"], tiles_per_item=t["tiles_per_item"],
                                   finalize_threads=40 - t["finalize_threads"], elem_apply=t["elem_apply"],
                                   shared_cols=t["shared_cols"], fact_stash=t["fact_stash"]))


@pytest.mark.parametrize("tuned", [False, True])
@pytest.mark.parametrize("smoother", [1, 2])
def test_smoothers_without_a_colouring(smoother, tuned):
    """Block Jacobi updates 1,936 aggregates that share elements from one x, restricted Schwarz reads
    all residuals before its updates: the V-cycle repeats bit for bit, is symmetric, and is that of
    separate launches (the same sums in another order, 1e-10), also in the modes the autotuner picks."""
    P = _lsdd()
    prob = fegen.elasticity_q1(129, nu=0.3)
    rng = np.random.default_rng(2)
    r, s = (torch.from_numpy(rng.standard_normal(prob.n)).cuda() for _ in range(2))
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, modes_fixed=4, smoother=smoother)) as h:
        assert len(np.unique(h.export_level(0)["agg_of_dof"])) > 1000
        if tuned:
            h.autotune()
        z = h.vcycle(r)
        for _ in range(5):
            assert torch.equal(h.vcycle(r), z)
        zs = h.vcycle(s)
        # z = M r with a symmetric M: s^T M r = r^T M s up to rounding
        assert abs(float(s @ z - r @ zs)) <= 1e-10 * float(s.norm() * z.norm())
        _separate(h)
        assert float((h.vcycle(r) - z).norm()) <= 1e-10 * float(z.norm())


@pytest.mark.parametrize("nrhs", [1, 8])
@pytest.mark.parametrize("precision", [0, 1])
def test_refused_solve_leaves_its_stream_idle(nrhs, precision):
    """A right-hand side with a NaN is found after the next cycle is queued; the call returns when that
    has ended, so that a solve on another stream has the hierarchy's vectors to itself."""
    P = _lsdd()
    prob = fegen.elasticity_q1(96, nu=0.3)
    rng = np.random.default_rng(3)
    shape = (prob.n,) if nrhs == 1 else (nrhs, prob.n)
    good = torch.from_numpy(rng.standard_normal(shape)).cuda()
    bad = good.clone()
    bad.view(-1)[-1] = float("nan")
    prm = P.Params.default(max_levels=3, tau_const=0.75, precision=precision)
    with P.Hierarchy.setup_problem(prob, prm) as h:
        ref = h.solve(good)[0]
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with P.Hierarchy.setup_problem(prob, prm) as h:
        for _ in range(3):
            with torch.cuda.stream(sa):
                with pytest.raises(P.LsddError):
                    h.solve(bad)
                assert sa.query()
            with torch.cuda.stream(sb):
                x = h.solve(good)[0]
            sb.synchronize()
            assert torch.equal(x, ref)
