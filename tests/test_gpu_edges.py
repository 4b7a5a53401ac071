"""GPU kernels at the sizes where their tiles, lane groups and dispatch rules
change, against the oracle or the plain definition of each result."""
import numpy as np
import pytest

from oracle import gomea_ref as G
from oracle import ref
from oracle import surrogate_ref as R
from paper_2202_11001_amd import workloads as W
from tests._common import assert_delta_close, assert_objectives_close, feasible_population, oracle_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2202_11001_amd import dsm  # noqa: E402

DEV = "cuda:0"


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.fixture(scope="module")
def tiny_problem():
    w = W.tiny()
    return w, dsm.Problem.from_workload(w, max_solutions=512, max_fos_points=4)


def _random_population(w, S, seed):
    """Lattice coordinates with full-rank spread; feasibility plays no part."""
    rng = np.random.default_rng(seed)
    base = W.regular_grid(w.dims, w.mesh).astype(np.float64)
    d = rng.normal(0, 2.0, (S, 2, w.P, 3)) * W.free_mask(w.mesh)[None, None]
    return W.snap(np.clip(base[None, None] + d, -0.5, np.array(w.dims) - 0.5))


# one staging tile of 192 selected solutions: below, exactly one, one more, three with skipped indices among them
@pytest.mark.parametrize("n_sel", [30, 192, 193, 500])
def test_estimate_tiles(tiny_problem, n_sel):
    w, gp = tiny_problem
    X = _random_population(w, 512, n_sel)
    sel = np.random.default_rng(n_sel).permutation(512)[:n_sel].astype(np.int32)
    if n_sel == 500:
        sel[[0, 191, 192, 499]] = [-1, 512, 600, -7]
    tets = gp.topology()["tets"]
    off = np.array([0, 4, 7, 9, 10, 14], dtype=np.int32)  # 4, 3, 2, 1 points and 4 again
    pts = np.concatenate([tets[0], tets[20][:3], tets[30][:2], [13], tets[47]]).astype(np.int32)
    mean, chol = gp.estimate_elements(_t(X), _t(sel), _t(off), _t(pts))
    rmean, _, rchol = G.estimate_elements(X, sel, off, pts, w.mesh)
    np.testing.assert_allclose(mean.cpu().numpy(), rmean, rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(chol.cpu().numpy(), np.array([G.packed_lower(L) for L in rchol]), rtol=1e-8, atol=1e-10)
    p1 = np.arange(w.P, dtype=np.int32)
    mean, chol = gp.estimate_distributions(_t(X), _t(sel), _t(p1))
    rmean, _, rchol = G.estimate(X, sel, p1, w.mesh)
    np.testing.assert_allclose(mean.cpu().numpy(), rmean, rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(chol.cpu().numpy(), np.array([G.packed_lower(L) for L in rchol]), rtol=1e-9, atol=1e-12)


# rows that end inside a wave's lane groups; elements of every number of points, an invalid one, K candidates a point
@pytest.mark.parametrize("S,K", [(1, 1), (7, 3), (33, 2)])
def test_sampled_variables_follow_their_factor(tiny_problem, S, K):
    """With one factor column set at a time to 1, the candidates of variable v
    and of the column's own variable take the same draw; so L z is checked
    against the draws themselves (a diagonal factor), variable by variable."""
    w, gp = tiny_problem
    X = _random_population(w, S, S + K)
    tets = gp.topology()["tets"]
    inner = 13  # the only point of the 3^3 mesh with 6 free coordinates
    off = np.array([0, 1, 5, 10, 12], dtype=np.int32)  # 1 point, 4 points, 5 points (rejected), 2 points
    pts = np.concatenate([[inner], tets[3], [0, 1, 2, 3, 4], [inner, inner]]).astype(np.int32)
    F = len(off) - 1
    rng = np.random.default_rng(3 * S + K)
    mean = rng.uniform(8, 20, (1, F, 24))
    low = np.tril(rng.uniform(0.2, 1.0, (F, 24, 24)))
    mult = rng.uniform(0.5, 2.0, (1, F)).astype(np.float32)

    def sample(Ls, mu):
        packed = np.array([[G.packed_lower(L) for L in Ls]])
        return gp.sample_elements(_t(X), _t(off), _t(pts), _t(mu), _t(packed), _t(mult), 5, 9).cpu().numpy()

    # each draw at 1/1024 of a voxel a unit would round away; spread it over 256 lattice steps instead
    eye = np.repeat(2.0 * np.eye(24)[None], F, axis=0)
    zero = np.full((1, F, 24), 15.5)
    draws = (sample(eye, zero).astype(np.float64) - 15.5) / 2.0
    cand = sample(low, mean).astype(np.float64)
    free = W.free_mask(w.mesh)
    for f in (0, 1, 3):
        n = 6 * (off[f + 1] - off[f])
        fr = np.concatenate([np.tile(free[p], 2) for p in pts[off[f]:off[f + 1]]])
        cur = np.concatenate([X[:, :, p].reshape(S, 6) for p in pts[off[f]:off[f + 1]]], axis=1).astype(np.float64)
        z = draws[:, off[f]:off[f + 1]].reshape(S, n) / np.sqrt(mult[0, f])
        z[:, ~fr] = 0.0  # pinned variables' draws do not show: leave them out of the factor
        L = low[f][:n, :n] * fr[None, :]
        got = cand[:, off[f]:off[f + 1]].reshape(S, n)
        if fr.all():
            want = mean[0, f, :n] + np.sqrt(mult[0, f]) * z @ L.T
            # a draw is known to half a lattice step (1/256) over 2 sqrt(mult); L's rows sum to at most n
            tol = 1 / 256 + n / 2 / 256
            inside = (want > 0) & (want < 31)
            assert np.all(np.abs(got - want)[inside] <= tol)
        assert np.all(got[:, ~fr] == cur[:, ~fr])
        assert np.all(np.rint((got + 0.5) * 128) == (got + 0.5) * 128)
    assert np.all(np.isnan(cand[:, off[2]:off[3]]))
    # single points: candidate k of point f of solution s takes draws 6 ((s F + f) K + k) ...; one call of K
    # candidates equals the K-fold repetition of the points in a call of one
    p1 = np.array([inner, 4, -1, 22], dtype=np.int32)
    m1, l1 = rng.uniform(8, 20, (1, 4, 6)), np.tril(rng.uniform(0.2, 1.0, (4, 6, 6)))
    pk1 = np.array([[G.packed_lower(L) for L in l1]])
    mu1 = rng.uniform(0.5, 2, (1, 4)).astype(np.float32)
    a = gp.sample_estimated(_t(X), _t(p1), K, _t(m1), _t(pk1), _t(mu1), 5, 9).cpu().numpy().reshape(S, 4, K, 6)
    r = np.repeat(np.arange(4), K)
    b = gp.sample_estimated(_t(X), _t(p1[r]), 1, _t(m1[:, r]), _t(pk1[:, r]), _t(mu1[:, r]), 5, 9)
    np.testing.assert_array_equal(a, b.cpu().numpy().reshape(S, 4, K, 6))
    assert np.all(np.isnan(a[:, 2])) and not np.any(np.isnan(a[:, [0, 1, 3]]))


# archives that end inside, at and after a wave's 64 rows, with and without padding
@pytest.mark.parametrize("n_arch,pad", [(0, 0), (1, 70), (63, 1), (64, 0), (64, 64), (65, 200), (130, 0)])
def test_acceptance_against_archives(tiny_problem, n_arch, pad):
    w, gp = tiny_problem
    S, pts = 24, np.array([0, 2, 13, 26], dtype=np.int32)
    F = len(pts)
    rng = np.random.default_rng(n_arch + pad)
    X = _random_population(w, S, 5)
    cand = W.candidates(X, np.arange(F + 1), pts, w.mesh, w.dims, 1.0, 6).astype(np.float32)
    obj = rng.uniform(1, 2, (S, 3))
    old = rng.uniform(0, 1, (S, F, 3))
    new = old + rng.choice([-0.2, 0.0, 0.2], (S, F, 3))
    flags = rng.choice([0, 0, 0, 1], (S, F)).astype(np.int32)
    arch = rng.uniform(0.9, 2.2, (n_arch, 3))
    behind = np.concatenate([np.full((min(pad, 1), 3), np.inf), np.zeros((max(pad - 1, 0), 3))])  # not looked at
    arch_all = np.concatenate([arch, behind])
    tc, cache = rng.uniform(0, 1, (2, S, gp.T, 3))
    d = new - old
    dX, dcache, dobj = _t(X.copy()), _t(cache.copy()), _t(obj.copy())
    acc = torch.empty((S, F), dtype=torch.uint8, device=DEV)
    gp.accept(dX, _t(pts), _t(cand), _t(old), _t(new), _t(flags), _t(tc), dcache, dobj,
              archive=_t(arch_all) if len(arch_all) else None, accepted=acc)
    nv = obj[:, None] + d
    want = (d <= 0).all(2) & (d < 0).any(2)
    if len(arch_all):
        dom = ((arch[None, None] <= nv[:, :, None]).all(3) & (arch[None, None] < nv[:, :, None]).any(3)).any(2)
        want |= (d < 0).any(2) & ~dom
    want &= flags == 0
    np.testing.assert_array_equal(acc.cpu().numpy() != 0, want)
    eX, ecache = X.copy(), cache.copy()
    topo = gp.topology()
    for s in range(S):
        for f in np.nonzero(want[s])[0]:
            p = pts[f]
            eX[s, :, p] = cand[s, f]
            star = topo["star"][topo["star_off"][p]:topo["star_off"][p + 1]]
            ecache[s, star] = tc[s, star]
    # stars of the four points overlap on this small mesh, but every element copies the same terms_cand rows
    np.testing.assert_array_equal(dX.cpu().numpy(), eX)
    np.testing.assert_array_equal(dcache.cpu().numpy(), ecache)


# solutions that fill a tile of 256, spill over it by one, and take two; all, some and none accepted
@pytest.mark.parametrize("S,share", [(1, 1.0), (64, 0.5), (256, 1.0), (257, 0.3), (520, 1.0), (520, 0.0)])
def test_improvement_ratio_tiles(S, share):
    rng = np.random.default_rng(S)
    F, C = 3, 2
    off = np.array([0, 4, 5, 10], dtype=np.int32)  # 4 points, 1 point, 5 points (rejected)
    cand = rng.normal(30, 3, (S, 10, 2, 3)).astype(np.float32)
    acc = (rng.uniform(0, 1, (S, F)) < share).astype(np.uint8)
    cl = rng.integers(0, C, S).astype(np.int32)
    mean = rng.normal(30, 1, (C, F, 24))
    Ls = np.tril(rng.uniform(0.5, 1.5, (C, F, 24, 24)))
    packed = np.array([[G.packed_lower(Ls[j, f]) for f in range(F)] for j in range(C)])
    got = dsm.improvement_ratio(_t(off), _t(cand), _t(acc), _t(mean), _t(packed), cluster=_t(cl)).cpu().numpy()
    for j in range(C):
        for f in range(2):
            n = 6 * (off[f + 1] - off[f])
            rows = [cand[s, off[f]:off[f + 1]].reshape(-1) for s in range(S) if cl[s] == j and acc[s, f]]
            L = Ls[j, f][:n, :n]
            want = G.standard_deviation_ratio(np.array(rows).reshape(-1, n), mean[j, f, :n], L @ L.T)
            np.testing.assert_allclose(got[j, f], want, rtol=1e-9, atol=1e-12)
    assert np.all(got[:, 2] == -1.0)


# batch sizes around the 16-row blocks and the 16 steps of 32 rows that are kept in flight
@pytest.mark.parametrize("N", [1, 17, 480, 512, 513, 1024, 4096, 6000])
def test_gradient_batches(N):
    rng = np.random.default_rng(N)
    p = rng.normal(0, 0.15, R.NPARAMS).astype(np.float32)
    p[R.W3 + R.OUT * R.HID:R.B3] = 0.0
    p[R.B3 + R.OUT:] = 0.0
    x = torch.from_numpy(rng.normal(size=(N, R.IN)).astype(np.float32)).to(torch.bfloat16)
    t = rng.normal(size=(N, R.OUT)).astype(np.float32)
    sur = dsm.Surrogate(seed=1, max_rows=64, max_batch=6016)
    sur.params(p)
    g, loss = sur.gradient(x.view(torch.int16).to(DEV), _t(t))
    want_loss, want = R.loss_and_grad(p.astype(np.float64), x.double().numpy(), t.astype(np.float64), bf16_round=True)
    # FP32 sums of the same BF16 operands: a hidden value can round to the neighbouring BF16 number, which moves a
    # row's share of a gradient by 2^-8; per parameter block the largest entry bounds it
    assert float(loss.item()) == pytest.approx(want_loss, rel=1e-3)
    g = g.cpu().numpy().astype(np.float64)
    for a, b in ((R.W1, R.B1), (R.B1, R.W2), (R.W2, R.B2), (R.B2, R.W3), (R.W3, R.B3), (R.B3, R.NPARAMS)):
        tol = 1e-3 * np.abs(want[a:b]) + 5e-4 * np.abs(want[a:b]).max()
        assert np.all(np.abs(g[a:b] - want[a:b]) <= tol)


# capacities around the 64-row words; more points than a staging tile (512); payload rows of even and odd length,
# aligned to 8 bytes and not; a NaN vector, which has no place in the order, does no harm
@pytest.mark.parametrize("capacity,m,row_floats,offset", [(63, 9, 1, 0), (64, 1, 6, 0), (65, 30, 6, 1), (200, 61, 7, 0),
                                                          (4097, 513, 0, 0), (3000, 700, 514, 0)])
def test_archive_merge_shapes(capacity, m, row_floats, offset):
    rng = np.random.default_rng(capacity)
    A = dsm.Archive(capacity=capacity, m_max=m, row_floats=row_floats)
    vec, rows = np.zeros((0, 3)), np.zeros((0, max(row_floats, 1)), np.float32)
    overflowed = 0
    for r in range(6):
        pts = rng.integers(0, 60, (m, 3)) / 4.0
        pts[: m // 2, 2] = 40 - pts[: m // 2, :2].sum(1) - 0.25 * r  # a front that improves, so rows are dropped
        new = rng.normal(size=(m, max(row_floats, 1))).astype(np.float32)
        buf = torch.empty(m * row_floats + offset, dtype=torch.float32, device=DEV)
        d = buf[offset:].view(m, row_floats) if row_floats else None
        if row_floats:
            d.copy_(_t(new))
        A.merge(_t(pts), d)
        want, want_rows = G.archive_merge(vec, pts, rows, new)
        if len(want) > capacity:  # unchanged
            overflowed += 1
            assert int(A.overflow.item()) == 1
        else:
            vec, rows = want, want_rows
            assert int(A.overflow.item()) == 0
        assert A.n == len(vec)
        v = A.vec.cpu().numpy()
        np.testing.assert_array_equal(v[:len(vec)], vec)
        assert np.all(v[len(vec):] == np.inf)
        if row_floats:
            np.testing.assert_array_equal(A.rows[:len(vec)].cpu().numpy(), rows)
    A.merge(_t(np.full((1, 3), np.nan)), torch.zeros((1, row_floats), device=DEV) if row_floats else None)
    assert A.n in (len(vec), len(vec) + 1)


# guidance points: none, fewer and more than the lanes that share them (8 and 16), several points of one correspondence;
# with and without cached terms, chunks that divide the stars and chunks that do not
@pytest.mark.parametrize("n_guid,cached,chunk", [(0, True, 8), (1, True, 5), (7, False, 8), (40, True, 4), (40, False, 7)])
def test_terms_of_a_chunk(n_guid, cached, chunk):
    rng = np.random.default_rng(n_guid + chunk)
    shape, mesh, S = (18, 22, 26), (3, 4, 3), 5
    mov, fix = rng.uniform(0, 1, (2,) + shape).astype(np.float32)
    dims = (shape[2], shape[1], shape[0])
    hi = np.array(dims) - 1.0
    gm, gf = W.snap(rng.uniform(0, 1, (2, n_guid, 3)) * hi) if n_guid else np.zeros((2, 0, 3), np.float32)
    corr = np.arange(n_guid, dtype=np.int32) // (3 if n_guid == 40 else 1)  # threes share a correspondence
    spacing = (0.9, 1.1, 2.5)
    held = tuple(float(np.float32(v)) for v in spacing)  # the library holds the spacing in FP32
    rp = ref.Problem(mov, fix, mesh, held, 0.1, guid_moving=gm, corr_moving=corr, guid_fixed=gf, corr_fixed=corr)
    P = int(np.prod(mesh))
    gp = dsm.Problem(mov, fix, mesh, spacing, 0.1, gm, corr, gf, corr, max_solutions=S, max_fos=P + 1, max_fos_points=3)
    gp.set_part_chunk(chunk)
    X = W.population(dims, mesh, S, 1.0, 7, reject=lambda x: rp.fold_check(x)[0] != 0)
    off = np.concatenate([np.arange(P), [P, P + 3]]).astype(np.int32)  # every point, then one element of three
    pts = np.concatenate([np.arange(P), [0, 16, 17]]).astype(np.int32)
    cand = W.candidates(X, off, pts, mesh, dims, 1.0, 8)
    cand[0, 3, 0, 1] += 1 / 512.0   # off the lattice
    cand[1, 5, 1, 2] = np.nan
    cand[2, 16] = cand[2, 16] + 20.0  # folds
    F = len(off) - 1
    Xd = _t(X)
    cache = torch.empty((S, gp.T, 3), dtype=torch.float64, device=DEV)
    obj, flags = gp.eval_full(Xd, tet_terms=cache)
    robj, rflags, rterms, _ = rp.eval_full(X, want_terms=True)
    assert np.all(flags.cpu().numpy() == 0) and np.all(rflags == 0)
    assert_objectives_close(obj.cpu().numpy(), robj)
    # deformation and guidance are FP64 on both sides: a few hundred roundings of terms up to 1e3
    np.testing.assert_allclose(cache.cpu().numpy()[..., 1:], rterms[..., 1:], rtol=1e-10, atol=1e-10)
    old, new, fl, vc = gp.eval_partial(Xd, _t(off), _t(pts), _t(cand), tet_terms_in=cache if cached else None,
                                       voxel_count=True)
    rold, rnew, rfl, rnv = rp.eval_partial(X, off, pts, cand, tet_terms=rterms if cached else None)
    np.testing.assert_array_equal(fl.cpu().numpy().astype(np.uint32), rfl)
    np.testing.assert_array_equal(vc.cpu().numpy()[rfl == 0], rnv[rfl == 0])
    assert (rfl == 0).sum() > S * F // 2 and (rfl[[0, 1, 2], [3, 5, 16]] != 0).all()
    assert_objectives_close(old.cpu().numpy(), rold, what="current sums")
    assert_delta_close(old.cpu().numpy(), new.cpu().numpy(), rold, rnew, rfl)


# faces through voxel centres (whole-voxel and half-voxel vertices, undeformed cubes of equal sides), where a span's end
# is an integer and has to be decided exactly; many short slices (marks) and few long ones (walk) per unit
@pytest.mark.parametrize("dims,mesh,step", [((17, 17, 17), (3, 3, 3), 0.0), ((17, 17, 17), (3, 3, 3), 1.0),
                                            ((24, 24, 24), (7, 7, 7), 0.5), ((40, 9, 33), (3, 3, 9), 1.0),
                                            ((64, 120, 10), (3, 3, 3), 1.0), ((30, 30, 30), (6, 6, 6), 1 / 128)])
def test_owner_map_with_faces_through_centres(dims, mesh, step):
    rng = np.random.default_rng(int(sum(dims) + 1000 * step))
    shape = (dims[2], dims[1], dims[0])
    img = np.zeros(shape, np.float32)
    rp = ref.Problem(img, img, mesh, (1.0, 1.0, 1.0), 0.1)
    gp = dsm.Problem(img, img, mesh, max_solutions=1)
    base = W.regular_grid(dims, mesh).astype(np.float64)
    free = W.free_mask(mesh)
    for _ in range(6):
        x = base.copy()
        if step:
            h = np.array(dims) / (np.array(mesh) - 1)
            moved = np.rint((base + rng.uniform(-0.2, 0.2, base.shape) * h) / step) * step
            x = np.where(free, np.clip(moved, -0.5, np.array(dims) - 0.5), base)
        x = W.snap(x)
        if rp.fold_check(np.stack([x, x])[None])[0][0]:
            continue
        owner, overlap = gp.rasterize_owner(_t(x))
        want, count = rp.owner_bruteforce(x)
        assert int(overlap.item()) == 0 and np.all(count == 1)
        np.testing.assert_array_equal(owner.cpu().numpy(), want)


# as many elements as the slot table takes (4096), and more, which go without; malformed and empty elements among them
# (and nothing else); chunks that divide the stars and chunks that do not
@pytest.mark.parametrize("F,chunk", [(1, 8), (9, 4), (1025, 7), (4096, 8), (4097, 5)])
def test_slot_table_covers_every_chunk(F, chunk):
    w = W.tiny()
    gp = dsm.Problem.from_workload(w, max_solutions=2, max_fos=5000, max_fos_points=2)
    gp.set_part_chunk(chunk)
    rng = np.random.default_rng(F)
    X = w.population(S=2)
    size = rng.integers(0, 4, F)  # 0 to 3 points: 3 is malformed
    if F == 9:
        size = np.array([0, 3] * 4 + [3])
    off = np.concatenate([[0], np.cumsum(size)]).astype(np.int32)
    pts = rng.integers(0, w.P, off[-1]).astype(np.int32)
    cand = W.candidates(X, off, pts, w.mesh, w.dims, 1.0, 3) if off[-1] else np.zeros((2, 0, 2, 3), np.float32)
    Xd = _t(X)
    cache = torch.empty((2, gp.T, 3), dtype=torch.float64, device=DEV)
    gp.eval_full(Xd, tet_terms=cache)

    def run(f0, f1, method):
        o = off[f0:f1 + 1]
        return method(Xd, _t(o - o[0]), _t(np.append(pts[o[0]:o[-1]], 0).astype(np.int32)),
                      _t(np.concatenate([cand[:, o[0]:o[-1]]], axis=1)), tet_terms_in=cache, voxel_count=True)

    whole = [t.cpu().numpy() for t in run(0, F, gp.eval_partial)]
    parts = [run(a, min(a + 300, F), gp.eval_partial_noalloc) for a in range(0, F, 300)]
    for k in range(4):
        np.testing.assert_array_equal(whole[k], np.concatenate([p[k].cpu().numpy() for p in parts], axis=1))
    assert np.all((whole[2] == 64) == (size == 3)[None])
    assert np.all(whole[3][:, size == 0] == 0) and np.all(whole[1][:, size == 0] == 0)


# rows that end inside a 64-row tile, fill it, and leave an XCD or all but one without a tile
@pytest.mark.parametrize("S,F,K", [(1, 1, 1), (3, 7, 3), (16, 1, 4), (5, 13, 1), (33, 9, 2)])
def test_feature_tiles(tiny_problem, S, F, K):
    w, gp = tiny_problem
    rp = ref.Problem(w.moving, w.fixed, w.mesh, w.spacing, w.tau)
    rng = np.random.default_rng(S * F * K)
    X = _random_population(w, S, S + F)
    pts = rng.integers(0, w.P, F).astype(np.int32)
    cand = np.stack([W.candidates(X, np.arange(F + 1), pts, w.mesh, w.dims, 2.0, k) for k in range(K)], axis=2)
    cand = np.ascontiguousarray(cand)  # [S][F][K][2][3]
    got = dsm.Surrogate.features(gp, _t(X), _t(pts), _t(cand)).cpu().numpy()
    want = R.features(rp, X, pts, cand).reshape(-1, 192)
    # FP32 differences of coordinates up to 32 and of interpolated values up to about 1.1
    np.testing.assert_allclose(got, want, rtol=0, atol=1e-4)
    sur = dsm.Surrogate(seed=2, max_rows=S * F * K, max_batch=32)
    sur.set_scaling(rng.normal(0, 0.2, 192).astype(np.float32), rng.uniform(0.5, 2, 192).astype(np.float32),
                    np.zeros(3, np.float32), np.ones(3, np.float32))
    packed = sur.features_packed(gp, _t(X), _t(pts), _t(cand))
    np.testing.assert_array_equal(packed.cpu().numpy(), sur.pack(_t(got))[0].cpu().numpy())
    # the screening kernel computes the same rows in LDS: its predictions are the network's on the packed rows
    pred = sur.screen(gp, _t(X), _t(pts), _t(cand))[2]
    np.testing.assert_array_equal(pred.cpu().numpy().reshape(-1, 3), sur.forward(packed).cpu().numpy())


# one tile more than the persistent grid of 768 takes at once, and tiles that are not full: a row's outputs do not
# depend on its place, so the rows of a call equal those of calls of one tile (which are checked against the reference)
@pytest.mark.parametrize("N", [63, 64, 65, 513, 768 * 64, 768 * 64 + 1])
def test_forward_tiles(N):
    rng = np.random.default_rng(N)
    p = rng.normal(0, 0.15, R.NPARAMS).astype(np.float32)
    x = torch.from_numpy(rng.normal(size=(N, R.IN)).astype(np.float32)).to(torch.bfloat16).view(torch.int16).to(DEV)
    sur = dsm.Surrogate(seed=1, max_rows=64, max_batch=32)
    sur.params(p)
    y = sur.forward(x)
    for a in (0, 64 * (N // 128), max(0, N - 64), max(0, N - 1)):
        part = x[a:a + 64].contiguous()
        assert torch.equal(y[a:a + 64], sur.forward(part))
    order = torch.from_numpy(rng.permutation(N)).to(DEV)
    assert torch.equal(sur.forward(x[order].contiguous()), y[order])


# archives around the 512-row staging tile and its 32-row steps, ended by padding or not; pairs that end inside a workgroup
@pytest.mark.parametrize("n_arch,pad", [(1, 0), (31, 3), (511, 1), (512, 0), (512, 600), (513, 0), (1100, 0)])
def test_screening_against_archives(tiny_problem, n_arch, pad):
    w, gp = tiny_problem
    rng = np.random.default_rng(n_arch + pad)
    S, K = 21, 2
    pts = np.arange(w.P, dtype=np.int32)
    X = _random_population(w, S, 3)
    cand = np.stack([W.candidates(X, np.arange(w.P + 1), pts, w.mesh, w.dims, 1.0, k) for k in range(K)], axis=2)
    sur = dsm.Surrogate(seed=5, max_rows=S * w.P * K, max_batch=32)
    sur.set_scaling(np.zeros(192, np.float32), np.ones(192, np.float32), np.zeros(3, np.float32),
                    np.full(3, 20.0, np.float32))
    obj = rng.uniform(0.5, 1.5, (S, 3))
    arch = rng.uniform(0.4, 1.6, (n_arch, 3))
    if n_arch > 1:
        arch[:-1] += 1.0  # the last row decides for most
    behind = np.concatenate([np.full((min(pad, 1), 3), np.inf), np.zeros((max(pad - 1, 0), 3))])  # not looked at
    pick, run, pred, cp = sur.screen(gp, _t(X), _t(pts), _t(np.ascontiguousarray(cand)), obj=_t(obj),
                                     archive=_t(np.concatenate([arch, behind])))
    pick, run, pred = pick.cpu().numpy(), run.cpu().numpy(), pred.cpu().numpy().astype(np.float64)
    d = np.take_along_axis(pred, pick[..., None, None].astype(np.int64), axis=2)[:, :, 0]
    nv = obj[:, None] + d
    dom = ((arch[None, None] <= nv[:, :, None]).all(3) & (arch[None, None] < nv[:, :, None]).any(3)).any(2)
    want = ((d <= 0).all(2) & (d < 0).any(2)) | ((d < 0).any(2) & ~dom)
    np.testing.assert_array_equal(run != 0, want)
    np.testing.assert_array_equal(cp.cpu().numpy(), np.take_along_axis(cand, pick[..., None, None, None].astype(np.int64), axis=2)[:, :, 0])


# a volume whose outputs are cleared only if a voxel can stay uncovered, in tetrahedra split over workgroups and taller
# than the slice table; each way in which a voxel can: a border point off the box, points off the lattice in either grid,
# a grid that covers a part of the box, flat tetrahedra
@pytest.mark.parametrize("what", ["covered", "border", "off-lattice", "other-off-lattice", "shrunk", "flat"])
def test_transform_of_uncovered_voxels(what):
    w = W.batched(shape=(200, 80, 112), mesh=(3, 3, 3))
    rp = oracle_problem(w)
    I = W.regular_grid(w.dims, w.mesh)
    rng = np.random.default_rng(8)
    X = np.stack([W.snap(np.clip(I + rng.normal(0, 2, I.shape) * W.free_mask(w.mesh), -0.5, np.array(w.dims) - 0.5))] * 2)
    X[1] = W.snap(np.clip(I + rng.normal(0, 2, I.shape) * W.free_mask(w.mesh), -0.5, np.array(w.dims) - 0.5))
    own = 1
    if what == "border":
        X[own, 12, 0] += 5.0  # the middle of the face x = -0.5
    elif what == "off-lattice":
        X[own, 12, 1] += 1.0 / 512
    elif what == "other-off-lattice":
        X[1 - own, 0, 2] = np.nan
    elif what == "shrunk":
        X[own] = W.snap(0.75 * X[own] + 0.125 * np.array(w.dims))
    elif what == "flat":
        X[own, 13, 0] = -0.5  # onto the face of the point next to it
        X[own, 13, 1:] = X[own, 12, 1:]
    rd, rm = rp.transform(own, X)
    assert np.isnan(rm).any() == (what not in ("covered", "flat"))
    gp = dsm.Problem.from_workload(w)
    d, m = gp.transform(_t(X), own=own)
    # displacements below 64 voxels rounded to FP32, and values up to 1
    np.testing.assert_allclose(d.cpu().numpy(), rd, rtol=0, atol=4e-6)
    np.testing.assert_allclose(m.cpu().numpy(), rm, rtol=0, atol=1e-6)
    only = gp.transform(_t(X), own=own, dvf=False)[1]
    np.testing.assert_array_equal(only.cpu().numpy(), m.cpu().numpy())


# numbers of pairs on both sides of 4096 and 65536, where the lanes of a pair change: a pair's results do not depend on
# the others, so they are those of calls of 2700 pairs
@pytest.mark.parametrize("S", [151, 152, 2427, 2428])
def test_screening_of_many_pairs(tiny_problem, S):
    w, gp = tiny_problem
    rng = np.random.default_rng(S)
    K = 2
    pts = _t(np.arange(w.P, dtype=np.int32))
    base = _random_population(w, 100, 3)
    X = np.ascontiguousarray(base[np.arange(S) % 100])
    cand = np.ascontiguousarray(rng.normal(0, 1, (S, w.P, K, 2, 3)).astype(np.float32) +
                                X.transpose(0, 2, 1, 3)[:, :, None])
    obj, arch = rng.uniform(0.5, 1.5, (S, 3)), rng.uniform(0.8, 1.6, (700, 3))
    sur = dsm.Surrogate(seed=5, max_rows=S * w.P * K, max_batch=32)
    sur.set_scaling(np.zeros(192, np.float32), np.ones(192, np.float32), np.zeros(3, np.float32),
                    np.full(3, 20.0, np.float32))
    got = sur.screen(gp, _t(X), pts, _t(cand), obj=_t(obj), archive=_t(arch))
    for a in range(0, S, 100):
        part = sur.screen(gp, _t(X[a:a + 100]), pts, _t(cand[a:a + 100]), obj=_t(obj[a:a + 100]), archive=_t(arch))
        for g, p in zip(got, part):
            assert torch.equal(g[a:a + 100], p)


# affected sets from a bitmap (one word a lane, two, the most that fit in LDS) and sorted on larger meshes; elements of
# one point, a repeated one, more than a wave has lanes, and more star entries than the sort takes; an invalid point
@pytest.mark.parametrize("mesh,dims", [((3, 3, 3), (16, 16, 16)), ((8, 8, 8), (24, 24, 24)), ((19, 19, 17), (40, 40, 36)),
                                       ((21, 19, 17), (44, 40, 36))])
def test_affected_sets(mesh, dims):
    rng = np.random.default_rng(mesh[0])
    img = [rng.uniform(0, 1, dims[::-1]).astype(np.float32) for _ in range(2)]
    w = W.Workload("affected", img[0], img[1], mesh, (1.0, 1.0, 1.0), 0.2, 1, 1.0, 1.0, 7, 8)
    rp = oracle_problem(w)
    P = w.P
    many = rng.permutation(P)[:min(70, P)]
    groups = [[P // 2], [0, 1, mesh[0], mesh[0] * mesh[1]], [5, 5], list(range(min(P, 40))), list(many), [P], [P // 2, -1]]
    off = np.cumsum([0] + [len(g) for g in groups]).astype(np.int32)
    pts = np.concatenate(groups).astype(np.int32)
    gp = dsm.Problem.from_workload(w, max_solutions=1, max_fos_points=70)
    X = np.stack([W.regular_grid(dims, mesh)] * 2)[None]
    Xd = _t(X)
    cand = X[:, :, np.clip(pts, 0, P - 1)].transpose(0, 2, 1, 3).copy()
    old, new, fl, vc = gp.eval_partial(Xd, _t(off), _t(pts), _t(cand), voxel_count=True)
    n = off[5]  # the oracle takes valid points only
    rold, rnew, rfl, rnv = rp.eval_partial(X, off[:6], pts[:n], np.ascontiguousarray(cand[:, :n]))
    assert not rfl.any()
    np.testing.assert_array_equal(fl.cpu().numpy(), [[0] * 5 + [dsm.FLAG_BAD_FOS] * 2])
    np.testing.assert_array_equal(vc.cpu().numpy()[:, :5], rnv)
    # the parts are sums over the affected tetrahedra: a missing or repeated one shows in each
    assert_objectives_close(old.cpu().numpy()[:, :5], rold)
    assert_objectives_close(new.cpu().numpy()[:, :5], rnew)


# numbers of elements on both sides of 256, where the slot table's order is found in another way, and of its 1024 threads
@pytest.mark.parametrize("F", [1, 16, 255, 256, 257, 1025])
def test_slot_table_orders(tiny_problem, F):
    w, gp0 = tiny_problem
    rng = np.random.default_rng(F)
    gp = dsm.Problem.from_workload(w, max_solutions=2, max_fos=F, max_fos_points=2)
    sizes = rng.integers(1, 3, F)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    pts = rng.integers(0, w.P, off[-1]).astype(np.int32)
    X = _random_population(w, 2, F)
    cand = X[:, :, pts].transpose(0, 2, 1, 3).copy()
    got = gp.eval_partial(_t(X), _t(off), _t(pts), _t(cand))
    one = dsm.Problem.from_workload(w, max_solutions=2, max_fos=1, max_fos_points=2)
    for f in rng.permutation(F)[:12]:  # an element's results do not depend on the others
        o = np.array([0, sizes[f]], np.int32)
        sl = slice(off[f], off[f + 1])
        part = one.eval_partial(_t(X), _t(o), _t(pts[sl]), _t(cand[:, sl]))
        for g, q in zip(got[:3], part[:3]):
            assert torch.equal(g[:, f], q[:, 0])


@pytest.mark.parametrize("n_clusters,n_sel", [(1, 5), (3, 193), (16, 40)])
def test_estimates_of_clusters(tiny_problem, n_clusters, n_sel):
    w, gp = tiny_problem
    rng = np.random.default_rng(n_sel)
    X = _t(_random_population(w, 512, n_clusters))
    members = _t(rng.integers(-1, 513, (n_clusters, n_sel)).astype(np.int32))
    off, pts = _t(np.array([0, 4, 5, 7], np.int32)), _t(rng.integers(0, w.P, 7).astype(np.int32))
    for o, single in ((off, lambda m: gp.estimate_elements(X, m, off, pts)),
                      (None, lambda m: gp.estimate_distributions(X, m, pts))):
        mean, chol = gp.estimate_clusters(X, members, pts, o)
        for c in range(n_clusters):
            m1, c1 = single(members[c])
            assert torch.equal(mean[c], m1) and torch.equal(chol[c], c1)
    for bad in (0, 17):
        with pytest.raises(dsm.DsmError):
            gp.estimate_clusters(X, members.new_zeros((bad, 4)), pts)


# (2048 workgroups that exist keep every SIMD at 8 waves; the switch is at 8192 launched ones, which have room for the
# largest element everywhere, and only where one version is swept: 30 solutions lie above it with cached terms)
# launches on both sides of the 2048 workgroups from which the sweep's other instruction order is used, in both row
# orders, with the current terms cached or recomputed: a solution's results do not depend on the others
@pytest.mark.parametrize("rows", [0, 1])
@pytest.mark.parametrize("cached", [True, False])
def test_sweep_orders_agree(rows, cached):
    w = W.batched(shape=(24, 24, 24), mesh=(4, 4, 4))
    rp = oracle_problem(w)
    S = 30
    X = feasible_population(w, rp, S=S)
    pts = np.arange(w.P, dtype=np.int32)
    off = np.arange(w.P + 1, dtype=np.int32)
    cand = W.candidates(X, off, pts, w.mesh, w.dims, 1.0, 3)
    gp = dsm.Problem.from_workload(w, max_solutions=S)
    gp.set_row_order(rows)

    def run(s):
        terms = torch.empty((len(s), gp.T, 3), dtype=torch.float64, device=DEV)
        obj, _ = gp.eval_full(_t(X[s]), tet_terms=terms)
        old, new, fl, vc = gp.eval_partial(_t(X[s]), _t(off), _t(pts), _t(cand[s]), tet_terms_in=terms if cached else None,
                                           voxel_count=True)
        return obj, terms, old, new, fl, vc

    many = run(np.arange(S))  # 30 x 64 elements of up to 6 chunks
    for s in (0, 7, S - 1):
        for m, o in zip(many, run(np.array([s]))):
            assert torch.equal(m[s:s + 1], o)
    rold, rnew, rfl, rnv = rp.eval_partial(X, off, pts, cand)
    np.testing.assert_array_equal(many[4].cpu().numpy().astype(np.uint32), rfl)
    ok = rfl == 0
    np.testing.assert_array_equal(many[5].cpu().numpy()[ok], rnv[ok])
    assert_objectives_close(many[3].cpu().numpy()[ok], rnew[ok])
    assert_objectives_close(many[2].cpu().numpy(), rold)


# the sweep sets the constraint bits of a full evaluation: one bad coordinate or fold at a time, in either grid, in the
# first, a middle and the last group of 8 tetrahedra, against the fold check
@pytest.mark.parametrize("grid", [0, 1])
def test_full_evaluation_flags(grid):
    w = W.batched(shape=(24, 24, 24), mesh=(4, 4, 4))
    rp = oracle_problem(w)
    gp = dsm.Problem.from_workload(w, max_solutions=40)
    X = np.repeat(np.stack([W.regular_grid(w.dims, w.mesh)] * 2)[None], 40, axis=0)
    P = w.P
    for i, p in enumerate((0, 21, 42, P - 1)):
        for j, (c, by) in enumerate(((0, 1 / 512), (1, np.nan), (2, 1.0), (0, 100.0), (1, -1.0), (2, np.inf), (0, 9.0), (1, -9.0))):
            X[8 * i + j, grid, p, c] += by
    X[36, grid, [21, 22]] = X[36, grid, [22, 21]]
    X[37, :, 42] -= 8.0
    rfl = rp.fold_check(X)[0]
    fl = gp.eval_full(_t(X))[1].cpu().numpy().astype(np.uint32)
    np.testing.assert_array_equal(fl, rfl)
    np.testing.assert_array_equal(gp.fold_check(_t(X)).cpu().numpy().astype(np.uint32), rfl)
    assert (rfl != 0).sum() > 25 and not rfl[38:].any()


# a layer of tetrahedra between two voxel slices: none of them has a candidate row, all of them hold guidance points
@pytest.mark.parametrize("rows", [0, 1])
def test_guidance_without_candidate_rows(rows):
    dims, mesh, S = (16, 16, 16), (3, 3, 4), 24
    rng = np.random.default_rng(rows)
    img = [rng.uniform(0, 1, dims[::-1]).astype(np.float32) for _ in range(2)]
    n = 40
    guid = [np.concatenate([W.snap(rng.uniform(0.5, 14.5, (n, 2))), np.full((n, 1), z, np.float32)], 1) for z in (5.5, 5.53125)]
    corr = np.arange(n, dtype=np.int32)
    w = W.Workload("thin layer", img[0], img[1], mesh, (1.0, 1.0, 1.0), 0.2, S, 1.0, 1.0, 7, 8, guid_moving=guid[0],
                   corr_moving=corr, guid_fixed=guid[1], corr_fixed=corr)
    rp = oracle_problem(w)
    X = np.repeat(np.stack([W.regular_grid(dims, mesh)] * 2)[None], S, axis=0)
    X[:, :, 9:18, 2], X[:, :, 18:27, 2] = 5.25, 5.75  # the second and third layer of points
    X[:, :, [13, 22], :2] += W.snap(rng.uniform(-2, 2, (S, 2, 2, 2)))  # their inner points, in x and y
    rfl = rp.fold_check(X)[0]
    assert not rfl.any()
    robj, _, rterms, _ = rp.eval_full(X, want_terms=True)
    layer = np.array([set(t) <= set(range(9, 27)) for t in rp.tets().tolist()])
    assert (rterms[:, layer, 2] > 0).any(1).all() and (rterms[:, ~layer, 2] == 0).all()
    gp = dsm.Problem.from_workload(w, max_solutions=S)
    gp.set_row_order(rows)
    terms = torch.empty((S, gp.T, 3), dtype=torch.float64, device=DEV)
    obj, fl = gp.eval_full(_t(X), tet_terms=terms)
    assert not fl.any()
    np.testing.assert_allclose(terms.cpu().numpy()[:, :, 2], rterms[:, :, 2], rtol=1e-9, atol=1e-9)
    assert_objectives_close(obj.cpu().numpy(), robj)
    off, pts = w.fos()
    cand = X[:, :, pts].transpose(0, 2, 1, 3).copy()
    rold, _, _, _ = rp.eval_partial(X, off, pts, cand)
    for cache in (None, terms):
        old, new, fl, _ = gp.eval_partial(_t(X), _t(off), _t(pts), _t(cand), tet_terms_in=cache)
        assert not fl.any()
        for part in (old, new):
            np.testing.assert_allclose(part.cpu().numpy()[..., 2], rold[..., 2], rtol=1e-9, atol=1e-9)


def _guided(shape, mesh, n, seed):
    """A batched workload with n guidance pairs at random lattice positions."""
    w = W.batched(shape=shape, mesh=mesh)
    rng = np.random.default_rng(seed)
    w.guid_moving, w.guid_fixed = (W.snap(rng.uniform(1, min(shape) - 2, (n, 3))) for _ in range(2))
    w.corr_moving = w.corr_fixed = np.arange(n, dtype=np.int32)
    return w


# every chunk; elements of 1 point and of 4, whose last chunk is full or not; current terms cached or recomputed
@pytest.mark.parametrize("chunk", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("cached", [True, False])
def test_unchanged_candidates_have_no_delta(chunk, cached):
    w = _guided((24, 24, 24), (4, 4, 4), 150, 5)
    X = _t(feasible_population(w, oracle_problem(w), S=6))
    gp = dsm.Problem.from_workload(w, max_solutions=6, max_fos=500, max_fos_points=4)
    gp.set_part_chunk(chunk)
    tets = gp.topology()["tets"]
    off = np.concatenate([np.arange(w.P), w.P + 4 * np.arange(len(tets) + 1)]).astype(np.int32)
    pts = np.concatenate([np.arange(w.P), tets.reshape(-1)]).astype(np.int32)
    terms = torch.empty((6, gp.T, 3), dtype=torch.float64, device=DEV)
    gp.eval_full(X, tet_terms=terms)
    assert (terms[..., 2] > 0).sum() > 200
    old, new, fl, _ = gp.eval_partial(X, _t(off), _t(pts), X[:, :, _t(pts).long()].transpose(1, 2).contiguous(),
                                      tet_terms_in=terms if cached else None)
    assert not fl.any()
    assert torch.equal(old[..., 1:], new[..., 1:])


# several guidance points in most tetrahedra: one version swept (cached terms, full evaluation) or two (recomputed)
@pytest.mark.parametrize("chunk", [4, 8])
def test_guidance_terms_do_not_depend_on_the_cache(chunk):
    w = _guided((24, 24, 24), (5, 5, 5), 1500, 6)
    X = _t(feasible_population(w, oracle_problem(w), S=4))
    gp = dsm.Problem.from_workload(w, max_solutions=4)
    gp.set_part_chunk(chunk)
    pts = np.array([i + 5 * j + 25 * k for k in (1, 3) for j in (1, 3) for i in (1, 3)], np.int32)  # disjoint stars
    off = np.arange(len(pts) + 1, dtype=np.int32)
    cand = _t(W.candidates(X.cpu().numpy(), off, pts, w.mesh, w.dims, 0.5, 3))
    full, one, two = (torch.zeros((4, gp.T, 3), dtype=torch.float64, device=DEV) for _ in range(3))
    gp.eval_full(X, tet_terms=full)
    gp.eval_partial(X, _t(off), _t(pts), cand, tet_terms_in=full, tet_terms_new=one)
    gp.eval_partial(X, _t(off), _t(pts), cand, tet_terms_new=two)
    assert (one[..., 2] > 0).sum() > 300
    assert torch.equal(one[..., 1:], two[..., 1:])
    moved = X.clone()
    moved[:, :, _t(pts).long()] = cand.transpose(1, 2)
    gp.eval_full(moved, tet_terms=full)
    assert torch.equal(full[..., 1:], one[..., 1:])  # every tetrahedron of this mesh is in the star of one of them


# coordinates about 0, on both sides of what vanishes next to 0.5 in FP64: 2^-54 above, 2^-55 below
def test_flags_of_coordinates_about_zero():
    w = W.batched(shape=(24, 24, 24), mesh=(4, 4, 4))
    rp = oracle_problem(w)
    f = np.float32
    tiny = [f(2.0 ** -53), np.nextafter(f(2.0 ** -54), f(1)), f(2.0 ** -54), f(0.75 * 2.0 ** -54),
            np.nextafter(f(2.0 ** -55), f(1)), f(2.0 ** -55), f(2.0 ** -60), f(1e-40), f(0)]
    vals = np.array(tiny + [-v for v in tiny], f)
    S, p = 3 * len(vals), 21  # the first inner point
    X = np.repeat(np.stack([W.regular_grid(w.dims, w.mesh)] * 2)[None], S, axis=0)
    cand = np.repeat(X[:, :, p][:, None], 1, axis=1).copy()
    for c in range(3):
        for i, v in enumerate(vals):
            cand[3 * i + c, 0, c % 2, c] = v
    moved = X.copy()
    moved[:, :, p] = cand[:, 0]
    rfl = rp.fold_check(moved)[0]
    lat = (rfl & dsm.FLAG_LATTICE) != 0
    assert lat.reshape(-1, 3).all(1).sum() == 2 + 5 and lat.reshape(-1, 3).any(1).sum() == 2 + 5
    gp = dsm.Problem.from_workload(w, max_solutions=S)
    np.testing.assert_array_equal(gp.eval_full(_t(moved))[1].cpu().numpy().astype(np.uint32), rfl)
    np.testing.assert_array_equal(gp.fold_check(_t(moved)).cpu().numpy().astype(np.uint32), rfl)
    off, pts = np.array([0, 1], np.int32), np.array([p], np.int32)
    _, _, pfl, _ = rp.eval_partial(X, off, pts, cand)
    fl = gp.eval_partial(_t(X), _t(off), _t(pts), _t(cand))[2]
    np.testing.assert_array_equal(fl.cpu().numpy().astype(np.uint32), pfl)
    for i in np.flatnonzero(lat)[:4]:  # a tetrahedron with such a vertex is not mapped
        assert torch.isnan(gp.transform(_t(moved[i]), 1)[0]).any()


# the points' rows in the archive's own buffer: its free rows, its first rows, some of both; a result moves nearly every row
@pytest.mark.parametrize("first", [40, 0, 30])
def test_archive_rows_merged_in_place(first):
    rng = np.random.default_rng(first)
    m, row = 40, 33000
    u = rng.uniform(0, 1, (2 * m, 2))
    front = np.concatenate([u, 2.0 - u.sum(1, keepdims=True)], 1)  # a plane: no vector dominates another
    rows = _t(rng.normal(size=(2 * m, row)).astype(np.float32))
    both = []
    for own in (False, True):
        A = dsm.Archive(capacity=100, m_max=m, row_floats=row)
        A.rows.zero_()
        A.merge(_t(front[:m]), rows[:m].contiguous())
        assert A.n == m
        A.rows[m:2 * m] = rows[m:]
        src = A.rows[first:first + m]
        A.merge(_t(front[m:]), src if own else src.clone())
        assert A.n == 2 * m
        both.append((A.vec.clone(), A.rows[:2 * m].clone()))
    for a, b in zip(*both):
        assert torch.equal(a, b)


# rows of one part (8192 floats), one part and a bit, several, in pairs of floats and alone, against the merge on the host
@pytest.mark.parametrize("capacity,row", [(7, 8192), (7, 8193), (5, 40000), (64, 16386)])
def test_archive_rows_in_parts(capacity, row):
    rng = np.random.default_rng(row)
    A = dsm.Archive(capacity=capacity, m_max=3, row_floats=row)
    vec, rows = np.zeros((0, 3)), np.zeros((0, row), np.float32)
    for _ in range(4):
        pts = rng.integers(0, 12, (3, 3)) / 4.0
        new = rng.normal(size=(3, row)).astype(np.float32)
        A.merge(_t(pts), _t(new))
        want, want_rows = G.archive_merge(vec, pts, rows, new)
        if len(want) <= capacity:
            vec, rows = want, want_rows
        assert A.n == len(vec) and int(A.overflow.item()) == (len(want) > capacity)
        np.testing.assert_array_equal(A.vec[:len(vec)].cpu().numpy(), vec)
        np.testing.assert_array_equal(A.rows[:len(vec)].cpu().numpy(), rows)


# the last and first sizes of the acceptance rule's three ranges (49,152 and 196,608 pairs), points and elements of 4
# points, an archive of more rows than a group's lanes that ends inside a round, some solutions with one objective only
@pytest.mark.parametrize("S", [1820, 1821, 7281, 7282])
@pytest.mark.parametrize("elements", [False, True])
def test_acceptance_of_many_pairs(tiny_problem, S, elements):
    w, _ = tiny_problem
    gp = dsm.Problem.from_workload(w, max_solutions=S)
    topo = gp.topology()
    F = 27
    groups = [t.tolist() for t in topo["tets"][:F]] if elements else [[p] for p in range(F)]
    rng = np.random.default_rng(S)
    X, moved = (rng.uniform(0, 31, (S, 2, w.P, 3)).astype(np.float32) for _ in range(2))
    pts = np.concatenate(groups).astype(np.int32)
    off = np.cumsum([0] + [len(g) for g in groups]).astype(np.int32)
    cand = moved[:, :, pts].transpose(0, 2, 1, 3).copy()  # a point moves to the same place in every element
    obj, old = rng.uniform(1, 2, (S, 3)), rng.uniform(0, 1, (S, F, 3))
    new = old + rng.choice([-0.2, 0.0, 0.2], (S, F, 3))
    flags = rng.choice([0, 0, 0, 1], (S, F)).astype(np.int32)
    arch = rng.uniform(0.9, 2.2, (70, 3))
    single = rng.integers(-1, 9, S).astype(np.int32)
    tc, cache = (torch.rand((S, gp.T, 3), dtype=torch.float64, device=DEV) for _ in range(2))
    dX, dcache, dobj = _t(X), cache.clone(), _t(obj)
    acc = torch.empty((S, F), dtype=torch.uint8, device=DEV)
    args = (_t(cand), _t(old), _t(new), _t(flags), tc, dcache, dobj)
    kw = dict(archive=_t(np.concatenate([arch, np.full((9, 3), np.inf), np.zeros((5, 3))])), accepted=acc,
              single_objective=_t(single))
    if elements:
        gp.accept_elements(dX, _t(off), _t(pts), *args, **kw)
    else:
        gp.accept(dX, _t(pts), *args, **kw)
    d = new - old
    nv = obj[:, None] + d
    dom = np.zeros((S, F), bool)
    for a in arch:
        dom |= (a <= nv).all(2) & (a < nv).any(2)
    want = (d <= 0).all(2) & (d < 0).any(2) | (d < 0).any(2) & ~dom
    one = (single >= 0) & (single < 3)
    want[one] = np.take_along_axis(d[one], single[one][:, None, None].repeat(F, 1), 2)[..., 0] < 0
    want &= flags == 0
    np.testing.assert_array_equal(acc.cpu().numpy() != 0, want)
    hit_p, hit_t = np.zeros((S, w.P), bool), np.zeros((S, gp.T), bool)
    for f, g in enumerate(groups):
        hit_p[:, g] |= want[:, f][:, None]
        for p in g:
            hit_t[:, topo["star"][topo["star_off"][p]:topo["star_off"][p + 1]]] |= want[:, f][:, None]
    assert torch.equal(dX, torch.where(_t(hit_p)[:, None, :, None], _t(moved), _t(X)))
    assert torch.equal(dcache, torch.where(_t(hit_t)[..., None], tc, cache))


# the last number of candidates with a lane per variable (40,960) and the first with a thread each; clusters, shifts,
# points that do not exist: a candidate does not depend on the others of its call
@pytest.mark.parametrize("S", [512, 513])
def test_candidates_of_many_points(tiny_problem, S):
    w, gp = tiny_problem
    F, K, C = 20, 4, 3
    rng = np.random.default_rng(S)
    X = _random_population(w, S, 8)
    pts = np.array([13, 4, -1, 22, 27, 0] + rng.integers(0, w.P, 14).tolist(), np.int32)
    mean = _t(rng.uniform(8, 20, (C, F, 6)))
    chol = _t(np.array([[G.packed_lower(np.tril(rng.uniform(0.2, 1.0, (6, 6)))) for _ in range(F)] for _ in range(C)]))
    mult = _t(rng.uniform(0.5, 2, (C, F)).astype(np.float32))
    cluster = rng.integers(0, C, S).astype(np.int32)
    cluster[7] = C  # no such cluster
    shift, ams = _t(rng.uniform(-1, 1, (w.P, 6))), rng.integers(0, 2, S).astype(np.uint8)

    def sample(n):
        return gp.sample_estimated(_t(X[:n]), _t(pts), K, mean, chol, mult, 5, 9, cluster=_t(cluster[:n]), shift=shift,
                                   ams=_t(ams[:n])).cpu().numpy()

    got, few = sample(S), sample(200)  # counters follow (s, f, k), so the first solutions draw the same
    np.testing.assert_array_equal(got[:200], few)
    assert np.isnan(got[7]).all() and np.isnan(got[:, [2, 4]]).all()
    rest = np.delete(np.delete(got, 7, 0), [2, 4], 1)
    assert not np.isnan(rest).any() and np.all(np.rint((rest + 0.5) * 128) == (rest + 0.5) * 128)


# more threads than a dimension of a grid holds (2^32): 32 to a candidate of an element, 320 to an element's factor, 256 to
# a standard-deviation ratio
def test_more_elements_than_a_grid_dimension():
    img = [np.random.default_rng(3).uniform(0, 1, (4, 4, 4)).astype(np.float32) for _ in range(2)]
    w = W.Workload("cube", img[0], img[1], (2, 2, 2), (1.0, 1.0, 1.0), 0.2, 1, 1.0, 1.0, 7, 8)
    gp = dsm.Problem.from_workload(w, max_solutions=1, max_fos=1, max_fos_points=1)
    F, S = 4, (1 << 25) + 3
    X = torch.randint(0, 512, (S, 2, 8, 3), dtype=torch.int32, device=DEV).float().div_(128).sub_(0.5)
    pts, off = _t(np.array([0, 5, 2, 7], np.int32)), _t(np.arange(F + 1, dtype=np.int32))
    mean, chol = (torch.ones((1, F, n), dtype=torch.float64, device=DEV) for n in (24, 300))
    out = torch.full((S, F, 2, 3), -7.0, device=DEV)
    gp.sample_elements(X, off, pts, mean, chol, torch.ones((1, F), device=DEV), 1, 1, out=out)
    for i, p in enumerate((0, 5, 2, 7)):  # corners: every coordinate is pinned and stays the solution's
        assert torch.equal(out[:, i], X[:, :, p])
    F = (1 << 32) // 320 + 5
    X = X[:3].contiguous()
    del out
    torch.cuda.empty_cache()
    off, pts = torch.arange(F + 1, dtype=torch.int32, device=DEV), torch.arange(F, dtype=torch.int32, device=DEV) % 8
    mean, chol = gp.estimate_elements(X, _t(np.arange(3, dtype=np.int32)), off, pts)
    want = X.double().mean(0).transpose(0, 1).reshape(8, 6)
    for a in (0, F // 16 * 8, F // 8 * 8 - 8):
        torch.testing.assert_close(mean[a:a + 8, :6], want, rtol=1e-14, atol=0)
    assert (mean[:, 0] != 0).all() and not chol[F - 1].any()
    del mean, chol
    torch.cuda.empty_cache()
    C, F = 16, (1 << 20) + 1
    off, acc = torch.arange(F + 1, dtype=torch.int32, device=DEV), torch.ones((1, F), dtype=torch.uint8, device=DEV)
    mean, chol = torch.zeros((C, F, 6), dtype=torch.float64, device=DEV), torch.zeros((C, F, 21), dtype=torch.float64, device=DEV)
    chol[..., 0] = 2.0  # the first variable alone varies
    sdr = dsm.improvement_ratio(off, torch.full((1, F, 2, 3), 3.0, device=DEV), acc, mean, chol,
                                cluster=torch.full((1,), C - 1, dtype=torch.int32, device=DEV))
    assert (sdr[:C - 1] == -1).all() and (sdr[C - 1] == 1.5).all()


# two workgroups of 256 threads an element: nearly as many as a dimension of a grid holds (2^24), and more
@pytest.mark.parametrize("F", [(1 << 23) - 3, (1 << 23) + 6])
def test_more_chunks_than_a_grid_dimension(F):
    rng = np.random.default_rng(F)
    img = [rng.uniform(0, 1, (4, 4, 4)).astype(np.float32) for _ in range(2)]
    w = W.Workload("cube", img[0], img[1], (3, 2, 2), (1.0, 1.0, 1.0), 0.2, 1, 1.0, 1.0, 7, 8)
    gp = dsm.Problem.from_workload(w, max_solutions=1, max_fos=F, max_fos_points=1)
    assert gp.max_affected == 12  # two chunks of 8 an element
    gp.set_part_chunk(8)
    X = np.stack([W.regular_grid(w.dims, w.mesh)] * 2)[None]
    one = X[:, :, np.arange(F, F + 12) % 12].transpose(0, 2, 1, 3).copy()
    one[..., 0] += rng.integers(-20, 21, one.shape[:3]) / 128
    pts = torch.arange(F, F + F, dtype=torch.int32, device=DEV) % 12
    cand = _t(one).repeat(1, F // 12 + 1, 1, 1)[:, :F].contiguous()
    off = torch.arange(F + 1, dtype=torch.int32, device=DEV)
    out = tuple(torch.full((1, F, 3), -7.0, dtype=torch.float64, device=DEV) for _ in range(2)) + (
        torch.full((1, F), -7, dtype=torch.int32, device=DEV), None)
    old, new, fl = gp.eval_partial(_t(X), off, pts, cand, out=out)[:3]
    small = dsm.Problem.from_workload(w, max_solutions=1, max_fos=12, max_fos_points=1)
    small.set_part_chunk(8)
    want = small.eval_partial(_t(X), off[:13].contiguous(), pts[:12].contiguous(), cand[:, :12].contiguous())
    for got, ref_ in zip((old, new, fl), want):
        assert torch.equal(got[:, :F // 12 * 12].reshape(F // 12, 12, -1), ref_.reshape(1, 12, -1).expand(F // 12, -1, -1))


# full evaluations on both sides of the 8,192 workgroups (21 a solution here) from which the sweep's other instruction
# order is used, in both row orders: a solution's results do not depend on the others
@pytest.mark.parametrize("rows", [0, 1])
def test_full_evaluation_orders_agree(rows):
    w = W.batched(shape=(24, 24, 24), mesh=(4, 4, 4))
    rp = oracle_problem(w)
    S = 391
    X = feasible_population(w, rp, S=S)
    gp = dsm.Problem.from_workload(w, max_solutions=S)
    gp.set_row_order(rows)
    assert S * 21 > 8192 >= (S - 1) * 21 and -(-gp.T // 8) == 21

    def run(x):
        terms = torch.empty((len(x), gp.T, 3), dtype=torch.float64, device=DEV)
        return gp.eval_full(_t(x), tet_terms=terms) + (terms,)

    many, fewer = run(X), run(X[1:])
    for m, o in zip(many, fewer):
        assert torch.equal(m[1:], o)
    for s in (0, 195, S - 1):
        for m, o in zip(many, run(X[s:s + 1])):
            assert torch.equal(m[s:s + 1], o)
    robj, rfl, _, _ = rp.eval_full(X[::30], want_terms=True)
    np.testing.assert_array_equal(many[1].cpu().numpy()[::30].astype(np.uint32), rfl)
    assert_objectives_close(many[0].cpu().numpy()[::30], robj)


# the last and first sizes on either side of the rules for few rows: network outputs (768 tiles of 64 rows), features in
# FP32 (8,192 rows) and BF16 (16,384): a row's values do not depend on the others of its call
@pytest.mark.parametrize("N", [49152, 49153])
def test_forward_of_few_tiles(N):
    rng = np.random.default_rng(5)
    x = _t(rng.integers(-(1 << 14), 1 << 14, (49153, R.IN)).astype(np.int16) & np.int16(~0x4000))  # |x| < 2
    sur = dsm.Surrogate(seed=3, max_rows=64, max_batch=32)
    got, first, last = sur.forward(x[:N]), sur.forward(x[:640].contiguous()), sur.forward(x[N - 641:N].contiguous())
    assert not torch.isnan(got).any()
    assert torch.equal(got[:640], first) and torch.equal(got[N - 641:], last)


@pytest.mark.parametrize("packed,rows", [(False, 8192), (True, 16384)])
@pytest.mark.parametrize("K", [1, 3])
def test_features_of_few_rows(tiny_problem, packed, rows, K):
    w, gp = tiny_problem
    pts = np.array([13, 0, 5, 22, -1, 26, 4, 14], np.int32)
    F = len(pts)
    S = rows // (F * K) + 1
    rng = np.random.default_rng(K)
    X = _t(rng.uniform(0, 31, (S, 2, w.P, 3)).astype(np.float32))
    cand = _t(rng.uniform(0, 31, (S, F, K, 2, 3)).astype(np.float32))
    sur = dsm.Surrogate(seed=3, max_rows=64, max_batch=32)
    sur.set_scaling(rng.normal(size=R.IN), rng.uniform(0.5, 2, R.IN), np.zeros(3), np.ones(3))

    def run(a, b):
        args = (X[a:b].contiguous(), _t(pts), cand[a:b].contiguous())
        return sur.features_packed(gp, *args) if packed else dsm.Surrogate.features(gp, *args)

    many = run(0, S)  # more rows than the rule's line
    n = rows // (F * K)
    assert (S * F * K > rows) and n * F * K <= rows
    assert torch.equal(many[:n * F * K], run(0, n))
    assert torch.equal(many[F * K:], run(1, S))
    assert torch.equal(many[-F * K:], run(S - 1, S))
