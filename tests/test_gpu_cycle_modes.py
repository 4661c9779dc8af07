"""Which kernels a cycle runs, for every smoother, precision and tuning."""
import contextlib
import ctypes as C
import os

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


def _scale_second_dofs(prob, factor):
    D = np.where(np.arange(prob.n) % 2, factor, 1.0)
    off = prob.block_offsets()
    for e in range(prob.n_elem):
        d, B = prob.element(e)
        prob.blocks[off[e]:off[e] + len(d) ** 2] = (B * D[d][:, None] * D[d]).ravel()
    return prob


@pytest.mark.parametrize("kind", ["q1", "q2"])
@pytest.mark.parametrize("first", [True, False])
def test_instances_do_not_depend_on_their_batch(kind, first):
    """An instance's element factors, modes, coarse operators and V-cycle are the same bits beside an
    instance like itself and beside one whose element diagonals span 2^28 (which the set-up treats in
    another order of operations), with element blocks of either eigensolver."""
    P = _lsdd()

    def make(factor):
        prob = fegen.elasticity_q1(16, nu=0.3) if kind == "q1" else fegen.elasticity_q2hex(3, nu=0.3)
        return _scale_second_dofs(prob, factor)

    kw = dict(max_levels=2, modes_fixed=4) if kind == "q1" else dict(max_levels=3, agg_passes=1, tau_const=0.75)
    r = np.random.default_rng(5).standard_normal(make(1.0).n)
    out = []
    for own in (1.0, 2.0 ** 14):
        for mate in (1.0, 2.0 ** 14):
            probs = [make(own), make(mate)] if first else [make(mate), make(own)]
            with P.Hierarchy.setup_batched(probs, P.Params.default(**kw)) as h:
                part = []
                i = 0 if first else 1
                ptr = np.concatenate([probs[0].elem_ptr, probs[0].elem_ptr[-1] + probs[1].elem_ptr[1:]])
                ranks, G = h.export_gram(ptr)
                ne, nb = probs[0].n_elem, len(probs[0].blocks)
                part += [ranks[i * ne:(i + 1) * ne], G[i * nb:(i + 1) * nb]]
                for l in range(h.info()["levels"] - 1):
                    off = h.level_segments(l)[0]
                    ex = h.export_level(l)
                    part.append(ex["mu"][off[i]:off[i + 1]])
                rr = np.zeros(2 * len(r))
                rr[i * len(r):(i + 1) * len(r)] = r
                part.append(h.vcycle(torch.from_numpy(rr).cuda()).cpu().numpy()[i * len(r):(i + 1) * len(r)])
                out.append(part)
    for a, b in ((out[0], out[1]), (out[2], out[3])):
        assert len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


def test_mixed_scale_keeps_its_vcycle_with_large_elements():
    """Element blocks above 48 DOFs of mixed scale: the V-cycle, which the rounding of the set-up moves by
    1e-7 there, is the recorded one (of the library before it had a second eigensolver)."""
    P = _lsdd()
    prob = _scale_second_dofs(fegen.elasticity_q2hex(3, nu=0.3), 2.0 ** 14)
    ref = np.load(os.path.join(os.path.dirname(__file__), "golden", "mixed_scale_q2hex3_vcycle.npz"))["z"]
    r = np.random.default_rng(0).standard_normal(prob.n)
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=3, tau_const=0.75, agg_passes=1)) as h:
        z = h.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.linalg.norm(z - ref) <= 1e-10 * np.linalg.norm(ref)


def test_scaled_hermites_keep_their_vcycle():
    """Hermite bicubics in unknowns scaled by the mesh size (element diagonals span 5e3 instead of 9e10):
    still a V-cycle that the rounding of the set-up moves by 1e-5, so it is the recorded one (every
    16th entry, of the library before it had a second eigensolver)."""
    P = _lsdd()
    prob, _ = fegen.hyperdiffusion_h2(48, eps=1e-4)
    D = np.tile([1.0, 64.0, 64.0, 4096.0], prob.n // 4)
    off = prob.block_offsets()
    for e in range(prob.n_elem):
        d, B = prob.element(e)
        prob.blocks[off[e]:off[e] + len(d) ** 2] = (B * D[d][:, None] * D[d]).ravel()
    ref = np.load(os.path.join(os.path.dirname(__file__), "golden", "scaled_hermite48_vcycle.npz"))["z"]
    r = np.random.default_rng(0).standard_normal(prob.n)
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=4, tau_const=1.0)) as h:
        z = h.vcycle(torch.from_numpy(r).cuda()).cpu().numpy()[::16]
    assert np.linalg.norm(z - ref) <= 1e-10 * np.linalg.norm(ref)


@pytest.mark.parametrize("mate", [1100, 2200])
def test_eigenpairs_do_not_depend_on_larger_aggregates_in_the_batch(mate):
    """Aggregates of 400 and 900 DOFs beside ones like themselves and beside one of 1,100 or 2,200, for
    which the reduction has other workgroups: the same eigenvalues and modes, bit for bit."""
    P = _lsdd()

    def make(*cuts):
        prob = fegen.elasticity_q1(40, nu=0.3)
        prob.agg_of_dof = np.searchsorted(np.array(cuts), np.arange(prob.n), side="right").astype(np.int32)
        return prob

    out = []
    for other in (make(400, 1300, 2200, 2700), make(400, 400 + mate)):
        own = make(400, 1300, 2200, 2700)
        with P.Hierarchy.setup_batched([own, other], P.Params.default(max_levels=2, tau_const=0.75)) as h:
            ex = h.export_level(0)
            nz = sum(int(k) * w for k, w in zip(ex["k"][:5], (400, 900, 900, 500, own.n - 2700)))
            out.append((ex["k"][:5], ex["mu"][:own.n], np.asarray(ex["Z"]).ravel()[:nz]))
    assert all(np.array_equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("nrhs", [1, 3])
@pytest.mark.parametrize("count", [64, 65, 1200])
def test_many_instances(count, nrhs):
    """Instances beyond what one workgroup adds up by itself (64), and more of them than it has threads:
    each converges in the iterations it takes in a batch of two, to the same residual (cycles in
    separate launches, which do not depend on the size of the batch)."""
    P = _lsdd()
    kinds = [fegen.elasticity_q1(4, nu=nu) for nu in (0.3, 0.45)]
    n = kinds[0].n
    rng = np.random.default_rng(8)
    rhs = rng.standard_normal((nrhs, 2, n))
    rhs[0, 1] = 0.0                                     # a pair that never starts
    prm = P.Params.default(max_levels=2, modes_fixed=2, min_coarse=1, max_density=1.0, rtol=1e-10)

    def solve(reps):
        b = np.concatenate([rhs.reshape(nrhs, -1)] * reps, axis=1)
        with P.Hierarchy.setup_batched([kinds[i % 2] for i in range(2 * reps)], prm) as h:
            _separate(h)
            x, infos = h.solve(torch.from_numpy(b if nrhs > 1 else b[0]).cuda())
        return (x.cpu().numpy().reshape(nrhs, reps, 2 * n),
                [[(f.iters, f.rel_res, f.converged) for f in infos[k * 2 * reps:(k + 1) * 2 * reps]] for k in range(nrhs)])

    x2, i2 = solve(1)
    x, infos = solve((count + 1) // 2)
    assert all(i[2] == 1 for row in i2 for i in row) and i2[0][1][0] == 0
    for k in range(nrhs):
        assert infos[k] == i2[k] * ((count + 1) // 2)
        assert np.array_equal(x[k], np.broadcast_to(x2[k], x[k].shape))


def _kernels(h):
    return [h.level_kernels(l) for l in range(h.info()["levels"] - 1)]


def _launched(h, r):
    """Names and counts of the traced launches of one V-cycle."""
    h.trace(True)
    h.vcycle(r)
    h.trace(False)
    return {k: v["launches"] for k, v in h.trace_read().items() if v["launches"]}


def test_tuning_describes_the_tuned_state():
    """Reading the shapes and setting them back changes nothing, tuned or not; the tuning of every
    precision brings its kernels back after the others were tuned, on this hierarchy, on a new one and
    through the seven shapes alone; shapes set by hand run in separate launches."""
    P = _lsdd()
    prob = fegen.elasticity_q1(64, nu=0.3)
    r = torch.from_numpy(np.random.default_rng(9).standard_normal(prob.n)).cuda()
    prm = P.Params.default(max_levels=3, tau_const=0.75, precision=2)
    shapes = ("lanes", "lanes_block", "tiles_per_item", "finalize_threads", "elem_apply", "shared_cols", "fact_stash")
    with P.Hierarchy.setup_problem(prob, prm) as h, P.Hierarchy.setup_problem(prob, prm) as other:
        levels = range(h.info()["levels"])
        h.set_cycle_precision(0)
        rule, ran = _kernels(h), _launched(h, r)
        assert any(k[0] for k in rule) and not any(k[2] for k in rule) and "colour_step" in ran
        h.set_tuning([h.level_tuning(l) for l in levels])
        assert _kernels(h) == rule and _launched(h, r) == ran
        tuned, state, names = {}, {}, {}
        for p in (0, 1, 2):
            h.set_cycle_precision(p)
            tuned[p] = h.autotune()
            state[p], names[p] = _kernels(h), _launched(h, r)
        assert "colour_step" not in names[2] and "sub_rows" not in names[2]
        for p in (0, 2, 1, 0, 1, 2, 0):
            h.set_cycle_precision(p)
            h.set_tuning(tuned[p])
            assert _kernels(h) == state[p] and _launched(h, r) == names[p]
            other.set_cycle_precision(p)
            other.set_tuning(tuned[p])
            assert _kernels(other) == state[p] and _launched(other, r) == names[p]
        h.set_cycle_precision(1)
        h.autotune(block=True)                              # other shapes, the same kernels
        assert [k[:2] for k in _kernels(h)] == [k[:2] for k in state[1]]
        for p in (0, 1):                                    # by the shapes alone
            h.set_cycle_precision(p)
            h.set_tuning([{k: t[k] for k in shapes} for t in tuned[p]])
            assert _kernels(h) == state[p]
        _separate(h)
        for p in (0, 1):
            h.set_cycle_precision(p)
            assert _kernels(h) == [(0, 0, 0)] * (len(levels) - 1)
            assert not {"colour_step", "sub_rows", "resid_restrict", "prolong_agg"} & set(_launched(h, r))
        h.set_cycle_precision(0)
        for bad in ((3, 0), (-1, 0), (0, 4)):
            with pytest.raises(P.LsddError) as e:
                h.set_level_kernels(0, *bad)
            assert e.value.code == 1
        h.set_cycle_precision(2)
        with pytest.raises(P.LsddError) as e:
            h.set_level_kernels(0, 1, 0)
        assert e.value.code == 7
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, modes_fixed=4, smoother=2)) as h:
        with pytest.raises(P.LsddError) as e:               # its one class is no colouring
            h.set_level_kernels(0, 1, 0)
        assert e.value.code == 7


@pytest.mark.parametrize("kind", ["q14", "q117", "p1", "bfs", "rtcf"])
def test_every_kernel_of_the_cycle_matches_separate_launches(kind):
    """All combinations of sweeps and transfers a hierarchy has against separate launches, FP64 and FP32,
    before and after an update of the operator (the same sums in another order: 1e-10; the FP32 cycle
    within 4x of the distance separate launches have from the FP64 cycle)."""
    from test_gpu_solve_kernels import _cycle_problem
    P = _lsdd()
    prob, kw = _cycle_problem(kind)
    r = torch.from_numpy(np.random.default_rng(1).standard_normal(prob.n)).cuda()
    theta = torch.ones(prob.n_elem, dtype=torch.float64, device="cuda")
    blocks = torch.from_numpy(np.ascontiguousarray(prob.blocks)).cuda()
    with P.Hierarchy.setup_elements_scaled(prob.n, prob.elem_ptr, prob.elem_dofs, blocks, theta, prob.node_of_dof,
                                           prob.agg_of_dof, P.Params.default(precision=1, **kw)) as h:
        def cycles(sweeps, transfers):
            out = []
            for scale in (1.0, 1.25):
                h.update_theta(theta * scale)
                for prec in (0, 1):
                    h.set_cycle_precision(prec)
                    for l in range(h.info()["levels"] - 1):
                        h.set_level_kernels(l, sweeps, transfers)
                    out.append(h.vcycle(r))
            return out

        apart, tried = cycles(0, 0), 0
        for sweeps in (0, 1, 2):
            for transfers in (0, 1, 2, 3):
                try:
                    z = cycles(sweeps, transfers)
                except P.LsddError as e:
                    assert e.code == 7 and (sweeps == 1 or transfers)
                    continue
                tried += 1
                for i in (0, 2):
                    n = float(apart[i].norm())
                    assert float((z[i] - apart[i]).norm()) <= 1e-10 * n
                    assert float((z[i + 1] - z[i]).norm()) <= 4 * float((apart[i + 1] - apart[i]).norm()) + 1e-12 * n
        assert tried >= 5


def test_memory_of_the_kernels_is_bounded_and_reused():
    """The tables of kernels that no precision runs go back to the hierarchy's memory, which going to and
    fro between the kernels and tuning do not grow; a level whose padded row tables would take gigabytes does
    without them, and solves all the same."""
    P = _lsdd()

    def used(fn):
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        out = fn()
        torch.cuda.synchronize()
        return free - torch.cuda.mem_get_info()[0], out

    prob = fegen.elasticity_q2hex(5, nu=0.3)
    r = torch.from_numpy(np.random.default_rng(10).standard_normal(prob.n)).cuda()
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, agg_passes=1, tau_const=0.75, precision=1)) as h:
        def to_and_fro():
            out = []
            for k in ((0, 0), (2, 2), (0, 3), (2, 0)):
                for prec in (0, 1):
                    h.set_cycle_precision(prec)
                    h.set_level_kernels(0, *k)
                h.set_cycle_precision(0)
                out.append(h.vcycle(r))
            for prec in (1, 0):
                h.set_cycle_precision(prec)
                h.autotune()
            return out

        z = to_and_fro()
        for _ in range(3):
            taken, again = used(to_and_fro)
            assert taken <= 0
            z += again                                      # in other orders: the tuning picks the shapes
        assert all(float((a - z[0]).norm()) <= 1e-10 * float(z[0].norm()) for a in z)
    # 20,000 aggregates of 2 DOFs beside one of 3,000: 20,001 x 3,008 rows of 16 bytes would be 0.96 GB
    # beside the coarsest level's 1.61 (20,001 unknowns in packed tiles)
    n = 43000
    dofs = np.stack([np.arange(n - 1), np.arange(1, n)], axis=1)
    B = np.repeat((np.array([[1.0, -1.0], [-1.0, 1.0]]) + 0.05 * np.eye(2))[None], n - 1, axis=0)
    from fegen.common import uniform_problem
    chain = uniform_problem(n, dofs, B, np.arange(n))
    chain.agg_of_dof = np.where(np.arange(n) < 3000, 0, 1 + (np.arange(n) - 3000) // 2).astype(np.int32)
    b = torch.from_numpy(np.random.default_rng(11).standard_normal(n)).cuda()
    took, h = used(lambda: P.Hierarchy.setup_problem(chain, P.Params.default(max_levels=2, modes_fixed=1, min_coarse=1,
                                                                             max_density=1.0, rtol=1e-8)))
    with h:
        assert took < 2.1e9 and h.level_kernels(0)[1] == 0
        with pytest.raises(P.LsddError) as e:
            h.set_level_kernels(0, 0, 3)
        assert e.value.code == 7
        x, info = h.solve(b)
        A = torch.zeros(n, dtype=torch.float64, device="cuda")
        A[:] = 2.1 * x
        A[0] -= 1.05 * x[0]
        A[-1] -= 1.05 * x[-1]
        A[1:] -= x[:-1]
        A[:-1] -= x[1:]
        assert info[0].converged == 1 and float((A - b).norm()) <= 1.1e-8 * float(b.norm())


@contextlib.contextmanager
def _allocator(alloc, free):
    """alloc(bytes) and free(pointer) behind lsdd_set_allocator."""
    from paper_2607_07485_amd import lsdd as binding
    fa = C.CFUNCTYPE(C.c_void_p, C.c_uint64, C.c_void_p)(lambda nbytes, ctx: alloc(nbytes))
    ff = C.CFUNCTYPE(None, C.c_void_p, C.c_void_p)(lambda ptr, ctx: free(ptr))
    binding.lib().lsdd_set_allocator(C.cast(fa, C.c_void_p), C.cast(ff, C.c_void_p), None)
    try:
        yield
    finally:
        binding.lib().lsdd_set_allocator(None, None, None)


def test_kernels_without_room_for_their_tables():
    """With an allocator that refuses what the tables need, asking for the kernels is refused and changes
    nothing, and the autotuner does without them."""
    P = _lsdd()
    limit = [1 << 60]

    def alloc(nbytes):
        return torch.cuda.caching_allocator_alloc(int(nbytes)) if nbytes <= limit[0] else 0

    prob = fegen.elasticity_q2hex(4, nu=0.3)
    r = torch.from_numpy(np.random.default_rng(12).standard_normal(prob.n)).cuda()
    with _allocator(alloc, torch.cuda.caching_allocator_delete):
        with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, agg_passes=1, tau_const=0.75)) as h:
            z = h.vcycle(r)
            assert h.level_kernels(0)[0] == 2
            h.set_level_kernels(0, 0, 0)
            apart = h.vcycle(r)
            limit[0] = 16 << 20                         # the unpacked inverses are some 60 MB
            with pytest.raises(P.LsddError) as e:
                h.set_level_kernels(0, 2, 0)
            assert e.value.code == 3 and h.level_kernels(0)[:2] == (0, 0)
            assert torch.equal(h.vcycle(r), apart)
            h.autotune()
            assert h.level_kernels(0)[0] == 0
            assert float((h.vcycle(r) - z).norm()) <= 1e-10 * float(z.norm())
            limit[0] = 1 << 60
            h.autotune()
            assert float((h.vcycle(r) - z).norm()) <= 1e-10 * float(z.norm())
            torch.cuda.synchronize()


@pytest.mark.parametrize("precision", [0, 1])
def test_allocator_with_8_byte_alignment(precision):
    """Memory aligned to 8 bytes only: no kernel that reads 16 at a time runs on it (rows of the fused
    kernels, blocks of right-hand sides), and the results are those of aligned memory."""
    P = _lsdd()
    prob = fegen.elasticity_q1(24, nu=0.3)
    B = torch.from_numpy(np.random.default_rng(13).standard_normal((8, prob.n))).cuda()
    prm = P.Params.default(max_levels=3, tau_const=0.75, rtol=1e-10, precision=precision)

    def run():
        with P.Hierarchy.setup_problem(prob, prm) as h:
            out = [h.solve(B)[0], h.solve(B[0].clone())[0]]
            kernels = _kernels(h)
            h.autotune()
            kernels += _kernels(h)
            out.append(h.solve(B[0].clone())[0])
            torch.cuda.synchronize()
            return out, kernels

    ref, kernels = run()
    assert any(k[0] == 1 and k[1] for k in kernels)
    with _allocator(lambda n: torch.cuda.caching_allocator_alloc(int(n) + 8) + 8,
                    lambda p: torch.cuda.caching_allocator_delete(p - 8)):
        out, kernels = run()
    assert not any(k[0] == 1 or k[1] for k in kernels)
    for a, b in zip(ref, out):
        assert float((a - b).norm()) <= 1e-8 * float(a.norm())


@pytest.mark.parametrize("n", [64, 81, 128])
def test_element_factors_of_large_clusters(n):
    """Element blocks that are projectors (three quarters of the eigenvalues equal): G^T G = A to
    128 eps, the bound of n rounded terms; the members of so large a cluster come out nearly dependent
    from their solves."""
    from fegen.common import Problem
    P = _lsdd()
    rng = np.random.default_rng(0)
    blocks = []
    for _ in range(40):
        Q = np.linalg.qr(rng.standard_normal((n, n)))[0][:, n // 4:]
        B = Q @ Q.T
        blocks.append(0.5 * (B + B.T))
    N = n * len(blocks)
    ptr = np.concatenate([n * np.arange(len(blocks) + 1), N + np.arange(1, N + 1)]).astype(np.int64)
    prob = Problem(n=N, elem_ptr=ptr, elem_dofs=np.tile(np.arange(N, dtype=np.int32), 2),
                   blocks=np.concatenate([b.ravel() for b in blocks] + [np.full(N, 0.1)]),
                   node_of_dof=np.arange(N, dtype=np.int32))
    with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=1)) as h:
        ranks, G = h.export_gram(ptr)
    for k, B in enumerate(blocks):
        g = G[k * n * n:(k + 1) * n * n].reshape(n, n)
        assert ranks[k] == n - n // 4
        assert np.abs(g.T @ g - B).max() <= 128 * np.finfo(float).eps * np.abs(B).max()


def test_modes_of_large_aggregates_stay_orthogonal():
    """Aggregates of 450 to 825 DOFs that keep all their modes, in clusters of hundreds: Z^T A_ww Z = I to
    n eps over the clusters' distance of 1e-4 (geometric mean over the aggregates, 2e-9)."""
    import scipy.sparse as sp
    P = _lsdd()
    off_by = []
    for width in range(450, 900, 75):
        prob = fegen.elasticity_q1(32, nu=0.3)
        prob.agg_of_dof = (np.arange(prob.n) // width).astype(np.int32)
        with P.Hierarchy.setup_problem(prob, P.Params.default(max_levels=2, tau_const=0.3)) as h:
            ex = h.export_level(0)
        A = sp.csr_matrix((ex["val"], ex["col"], ex["rowptr"]), shape=(prob.n, prob.n))
        at = 0
        for i in range(-(-prob.n // width)):
            d = np.arange(i * width, min((i + 1) * width, prob.n))
            k = int(ex["k"][i])
            Z = ex["Z"][at:at + len(d) * k].reshape(len(d), k)
            at += len(d) * k
            off_by.append(np.abs(Z.T @ (A[d][:, d] @ Z) - np.eye(k)).max())
    assert np.exp(np.mean(np.log(off_by))) <= 900 * np.finfo(float).eps / 1e-4


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("smoother", [0, 2])
def test_unpacked_inverses_of_the_setup_and_unpacked_again(precision, smoother):
    """A level that starts out with rows of the unpacked inverses runs on those of its set-up; given back and
    unpacked again they are the same, bit for bit, in either precision."""
    P = _lsdd()
    prob = fegen.elasticity_q2hex(4, nu=0.3)
    prm = P.Params.default(max_levels=2, agg_passes=1, tau_const=0.75, precision=precision, smoother=smoother)
    r = torch.from_numpy(np.random.default_rng(14).standard_normal(prob.n)).cuda()
    with P.Hierarchy.setup_problem(prob, prm) as h:
        for p in range(precision + 1):
            h.set_cycle_precision(p)
            h.set_level_kernels(0, 2, 0)
        for p in range(precision + 1):
            h.set_cycle_precision(p)
            first = h.vcycle(r)
            h.set_level_kernels(0, 0, 0)
            h.set_level_kernels(0, 2, 0)
            assert torch.equal(h.vcycle(r), first)
