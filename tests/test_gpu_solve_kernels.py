"""The solve kernels at the sizes where their work splits change, against dense FP64 algebra.

The problems are chains of 2-DOF elements [[1, -1], [-1, 1]] + 0.05 I: A is tridiagonal with
eigenvalues in [0.05, 4.1], so a PCG solution with relative residual rho has a relative error of at
most 82 rho (2-norm condition number).
"""
import numpy as np
import pytest

from fegen.common import Problem, uniform_problem

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


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("max_iter", [1, 2, 5])
def test_iterations_stop_at_max_iter(max_iter, graph):
    """A solve that is cut off returns the iterate its reported residual belongs to (the cycle
    enqueued behind the last step must not touch it)."""
    import fegen
    P = _lsdd()
    prob, b = fegen.elasticity_small(N=12)
    A = _dense(prob)
    with torch.cuda.stream(torch.cuda.Stream()), \
            P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, modes_fixed=4, max_iter=max_iter)) as h:
        h.set_graph(graph)
        for _ in range(2):
            x, infos = h.solve(torch.from_numpy(b).cuda(), allow_noconv=True)
            r = np.linalg.norm(b - A @ x.cpu().numpy()) / np.linalg.norm(b)
            assert infos[0].iters == max_iter and infos[0].converged == 0
            assert abs(infos[0].rel_res - r) <= 1e-10


def _cycle_problem(kind):
    import fegen
    rng = np.random.default_rng(4)
    if kind.startswith("q1"):      # overlaps of at most 50 DOFs, ragged patches at the edges
        return fegen.elasticity_q1(int(kind[2:])), dict(max_levels=2, modes_fixed=4)
    if kind == "p1":               # overlaps of 65 to 128 DOFs, some smaller at the corners
        return fegen.diffusion_p1_triangles(40), dict(max_levels=3, tau_const=1.0)
    if kind == "bfs":              # overlaps of several hundred DOFs, few of them
        return fegen.hyperdiffusion_h2(24, eps=1.0)[0], dict(max_levels=3, tau_const=1.0)
    return fegen.graddiv_rtcf3(12, kappa=np.exp(rng.standard_normal(144)), beta=1.0), dict(max_levels=3, max_density=1.0)


@pytest.mark.parametrize("kind", ["q14", "q117", "p1", "bfs", "rtcf"])
def test_fused_cycle_matches_separate_launches(kind):
    """The fused colour, transfer and coarsest kernels against the separate launches (which a set
    of launch shapes brings back), before and after an update of the operator: the same sums in
    another order, held to the 1e-10 of the FP64 parity; the FP32 cycle stays as far from the FP64
    cycle as with separate launches (within 4x)."""
    P = _lsdd()
    prob, kw = _cycle_problem(kind)
    rng = np.random.default_rng(1)
    r = torch.from_numpy(rng.standard_normal(prob.n)).cuda()
    blocks = torch.from_numpy(np.ascontiguousarray(prob.blocks)).cuda()
    theta = torch.ones(prob.n_elem, dtype=torch.float64, device="cuda")
    with P.Hierarchy.setup_elements_scaled(prob.n, prob.elem_ptr, prob.elem_dofs, blocks, theta, prob.node_of_dof,
                                           prob.agg_of_dof, P.Params.default(precision=1, **kw)) as h:
        def cycles():
            out = []
            for scale in (1.0, 1.25):
                h.update_theta(theta * scale)
                for prec in (0, 1):
                    h.set_cycle_precision(prec)
                    out.append(h.vcycle(r))
            return out

        fused = cycles()
        for l in range(h.info()["levels"]):
            h.set_level_tuning(l, h.level_tuning(l))
        apart = cycles()
    for i in (0, 2):
        n = float(apart[i].norm())
        assert float((fused[i] - apart[i]).norm()) <= 1e-10 * n
        assert float((fused[i + 1] - fused[i]).norm()) <= 4 * float((apart[i + 1] - apart[i]).norm()) + 1e-12 * n


@pytest.mark.parametrize("n", [2, 15, 16, 17, 63, 64, 65, 129, 200])
def test_direct_solve_tile_edges(n):
    """A one-level hierarchy is a dense Cholesky factorisation and its inverse: tiles of 64 in
    blocks of 16.  An explicit inverse in FP64 is within a few n cond eps of the solution."""
    P = _lsdd()
    prob = _chain(n)
    r = np.random.default_rng(n).standard_normal(n)
    ref = np.linalg.solve(_dense(prob), r)
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=1)) as h:
        z = h.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.linalg.norm(z - ref) <= 4 * n * COND * 2.3e-16 * np.linalg.norm(ref)


@pytest.mark.parametrize("width", [1, 4, 8, 16])
def test_blocked_eigensolver_sizes(width):
    """Local spectral problems of 66 width DOFs (the smallest the blocked reduction takes, then one,
    two and four rows per thread and more threads), whose spectra hold clusters of more than 64
    members, against the reduction in one workgroup: eigenvalues to 1e-10, the V-cycle, which does
    not depend on the basis, to 1e-10."""
    import fegen
    P = _lsdd()
    prob = fegen.elasticity_q1(32, nu=0.3)
    prob.agg_of_dof = (np.arange(prob.n) // (66 * width)).astype(np.int32)
    r = torch.from_numpy(np.random.default_rng(width).standard_normal(prob.n)).cuda()
    out = []
    for blocked in (-1, 66):
        with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, blocked_eig_min=blocked)) as h:
            ex = h.export_level(0)
            out.append((ex["k"], ex["mu"], h.vcycle(r)))
    (k0, mu0, z0), (k1, mu1, z1) = out
    assert np.array_equal(k0, k1) and k0.max() > 64
    assert np.abs(mu0 - mu1).max() <= 1e-10
    assert float((z0 - z1).norm()) <= 1e-10 * float(z0.norm())


def test_element_factors_at_block_sizes():
    """G^T G = A of singular element blocks with a cluster of equal eigenvalues, at the sizes where
    the eigensolver changes (Jacobi up to 48; pairs without a partner; a wave's rows, 64 and 128).
    The Jacobi route is backward stable (50 n eps); in the other, vectors of different clusters are
    orthogonal to eps over the clusters' distance, 1e-4 (1e-11)."""
    P = _lsdd()
    rng = np.random.default_rng(3)
    sizes = [1, 2, 3, 8, 24, 47, 48, 49, 64, 65, 127, 128]
    blocks = []
    for n in sizes:
        w = np.concatenate([np.zeros(n // 3), np.ones(n // 3), rng.uniform(0.1, 10.0, n - 2 * (n // 3))])
        Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
        B = Q @ np.diag(w) @ Q.T
        blocks.append(0.5 * (B + B.T))
    N = sum(sizes)
    ptr = np.concatenate([np.cumsum([0] + sizes), N + np.arange(1, N + 1)])
    prob = Problem(n=N, elem_ptr=ptr.astype(np.int64), elem_dofs=np.tile(np.arange(N, dtype=np.int32), 2),
                   blocks=np.concatenate([b.ravel() for b in blocks] + [np.full(N, 0.1)]),
                   node_of_dof=np.arange(N, dtype=np.int32))
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=1)) as h:
        ranks, G = h.export_gram(ptr)
    off = 0
    for n, r, B in zip(sizes, ranks, blocks):
        g = G[off:off + n * n].reshape(n, n)
        off += n * n
        assert r == n - n // 3 and not g[r:].any()
        assert np.abs(g.T @ g - B).max() <= (50 * n * np.finfo(float).eps if n <= 48 else 1e-11) * 10.0


def test_local_assembly_in_lds_and_memory():
    """Aggregates of 300 DOFs, assembled in LDS, and the same ones in a batch with one of 700 DOFs,
    which is assembled in memory: the same arithmetic, so equal eigenvalues."""
    P = _lsdd()
    a, b = _chain(600), _chain(700)
    both = uniform_problem(1300, np.concatenate([a.elem_dofs.reshape(-1, 2), 600 + b.elem_dofs.reshape(-1, 2)]),
                           np.concatenate([a.blocks, b.blocks]).reshape(-1, 2, 2), np.arange(1300))
    a.agg_of_dof = (np.arange(600) // 300).astype(np.int32)
    both.agg_of_dof = np.minimum(np.arange(1300) // 300, 2).astype(np.int32)
    out = []
    for prob in (a, both):
        with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2)) as h:
            ex = h.export_level(0)
            out.append((ex["k"][:2], ex["mu"][:600]))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


@pytest.mark.parametrize("hook", [False, True])
def test_setup_memory(hook):
    """Set-ups that share nothing, one that fails, calls on other streams that allocate after the
    set-up, and everything given back at the end (up to the 64 MB the runtime may keep)."""
    import fegen
    P = _lsdd()
    prob = fegen.elasticity_q1(24, nu=0.3)
    B = torch.from_numpy(np.random.default_rng(0).standard_normal((3, prob.n))).cuda()
    bad = uniform_problem(4, np.array([[0, 1], [2, 3]]), np.stack([np.eye(2), -np.eye(2)]), np.arange(4))
    P.set_torch_allocator(hook)
    try:
        P.Hierarchy.setup_problem(prob, P.Params.default()).close()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        free = torch.cuda.mem_get_info()[0]
        hs = [P.Hierarchy.setup_problem(prob, P.Params.default(rtol=1e-10)) for _ in range(3)]
        with pytest.raises(P.LsddError):
            P.Hierarchy.setup_problem(bad, P.Params.default())
        hs.pop(1).close()
        X = hs[0].solve(B)[0]
        with torch.cuda.stream(torch.cuda.Stream()):
            torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
            Y = hs[1].solve(B)[0]
            G1 = hs[1].export_gram_level(1)
            Y2 = hs[1].solve(B)[0]
            torch.cuda.current_stream().synchronize()
        G0 = hs[0].export_gram_level(1)
        assert torch.equal(X, Y) and torch.equal(Y, Y2)
        assert np.array_equal(G0["ranks"], G1["ranks"]) and np.array_equal(G0["G"], G1["G"])
        for h in hs:
            h.close()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        assert torch.cuda.mem_get_info()[0] >= free - (64 << 20)
    finally:
        P.set_torch_allocator(False)


@pytest.mark.parametrize("width", [0, 66, 264])
def test_mixed_scale_keeps_its_kernels(width):
    """Unknowns of two dimensions (every second DOF scaled by 2^14, so that an element's diagonal spans
    2^28) take the fixed-order kernels; the local eigenvalues do not depend on the scaling, which is
    exact, so both routes give the same ones (1e-10) and the same modes, for aggregates in each size
    class of the eigensolver, and the solves converge."""
    import fegen
    P = _lsdd()
    out = []
    for scale in (1.0, 2.0 ** 14):
        prob = fegen.elasticity_q1(24, nu=0.3)
        if width:
            prob.agg_of_dof = (np.arange(prob.n) // width).astype(np.int32)
        D = np.where(np.arange(prob.n) % 2, scale, 1.0)
        off = prob.block_offsets()
        for e in range(prob.n_elem):
            d, B = prob.element(e)
            prob.blocks[off[e]:off[e] + len(d) ** 2] = (B * D[d][:, None] * D[d]).ravel()
        b = torch.from_numpy(D * np.random.default_rng(1).standard_normal(prob.n)).cuda()
        with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, rtol=1e-8)) as h:
            ex = h.export_level(0)
            info = h.solve(b)[1]
            info = info[0] if isinstance(info, (list, tuple)) else info
            out.append((ex["k"], ex["mu"], info))
    (k0, mu0, i0), (k1, mu1, i1) = out
    assert np.array_equal(k0, k1)
    assert np.abs(mu0 - mu1).max() <= 1e-10
    assert i0.converged == 1 and i1.converged == 1


@pytest.mark.parametrize("nrhs", [1, 3, 5])
@pytest.mark.parametrize("sizes", [[1], [8] * 70, [32] * 5, [33] * 5, [81] * 9, [256] * 3, [257] * 2, [513] * 2,
                                   [2, 31, 1, 32, 7], [300, 1, 257, 64, 600, 33]])
def test_element_contraction_sizes(sizes, nrhs):
    """Waves and workgroups per element, several elements and partial groups of them, rows in LDS and
    in memory, equal and mixed sizes; a sum of n^2 nrhs terms in any order is within 2 n eps of
    the sum of their magnitudes (n + n partial sums deep at most)."""
    P = _lsdd()
    rng = np.random.default_rng(len(sizes) + nrhs)
    ptr = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    dofs = rng.integers(0, 700, ptr[-1]).astype(np.int32)
    blocks = [rng.standard_normal((n, n)) for n in sizes]
    u, v = rng.standard_normal((2, nrhs, 700))
    out = P.elem_bilinear(ptr, torch.from_numpy(dofs).cuda(), torch.from_numpy(np.concatenate([b.ravel() for b in blocks])).cuda(),
                          torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda(), scale=-2.0).cpu().numpy()
    for e, (n, B) in enumerate(zip(sizes, blocks)):
        d = dofs[ptr[e]:ptr[e + 1]]
        want = -2.0 * sum(u[k, d] @ B @ v[k, d] for k in range(nrhs))
        size = 2.0 * sum(np.abs(u[k, d]) @ np.abs(B) @ np.abs(v[k, d]) for k in range(nrhs))
        assert abs(out[e] - want) <= 2 * (n + nrhs) * np.finfo(float).eps * size


@pytest.mark.parametrize("width", [1, 2, 3, 13, 14, 15, 29, 30, 31, 45, 46, 47, 61, 62])
def test_small_overlaps_fp32_blocks(width):
    """Overlaps of width + 2 DOFs (one less at the ends) around the 4- and 16-wide steps, FP32 cycle, 8
    right-hand sides: the preconditioner is the FP64 one's up to FP32 rounding, so PCG to 1e-6 takes
    as many iterations, give or take one."""
    P = _lsdd()
    prob = _chain(5 * width + max(1, width // 2))
    prob.agg_of_dof = (np.arange(prob.n) // width).astype(np.int32)
    B = torch.from_numpy(np.random.default_rng(width).standard_normal((8, prob.n))).cuda()
    its = []
    for precision in (0, 1):
        with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, min_coarse=1, max_density=1.0, rtol=1e-6,
                                                              precision=precision)) as h:
            assert h.info()["levels"] == 2
            its.append([f.iters for f in h.solve(B)[1]])
            assert all(f.converged == 1 for f in h.solve(B)[1])
    assert max(abs(a - b) for a, b in zip(*its)) <= 1
