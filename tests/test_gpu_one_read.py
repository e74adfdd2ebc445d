"""The one-read pass (the quad form of D: four rows share a list of columns)
against float64 and against the two separate passes, where it can go wrong:
rows that do not fill a quad, quads without nonzeros, quads that span several
blocks, idle lanes, the largest beamlet counts, non-finite and huge vectors."""
import numpy as np
import pytest
import scipy.sparse as sp

from gpu_util import banner, rel_normwise, to_dev, to_host

pytestmark = pytest.mark.gpu

TABLE = [(2.0, 3.0, 1.0, 0.5), (0.0, 1.5, 0.0, 0.3)]


def _matrix(nv, nb, longest, seed, empty=0.2):
    """Ragged rows of up to `longest` nonzeros, dyadic 8-bit values (exact in
    every storage, a column's largest being 1), some rows empty."""
    rng = np.random.default_rng(seed)
    lens = np.minimum(rng.integers(0, longest + 1, nv), nb)
    lens[rng.random(nv) < empty] = 0
    lens[nv // 2:nv // 2 + 40] = 0
    lens[-1] = min(nb, longest)
    rows = np.repeat(np.arange(nv), lens)
    cols = np.concatenate([np.sort(rng.choice(nb, n, replace=False)) for n in lens]) if lens.sum() else np.zeros(0, int)
    vals = (rng.integers(1, 129, len(rows)) / 128.0).astype(np.float32)
    D = sp.csr_matrix((vals, (rows, cols)), shape=(nv, nb))
    top = np.asarray(D.argmax(axis=0)).ravel()
    for c in range(nb):
        if D[:, c].nnz:
            D[top[c], c] = 1.0
    D.sort_indices()
    return D, rng.integers(0, 2, nv).astype(np.uint8)


def _plan(D, sid, storage, one_read):
    from paper_0908_4421_amd.imrt import Context, Dose, Plan
    ctx = Context(0, one_read=one_read)
    lib = Dose.from_csr(ctx, D.shape[0], D.shape[1], D.indptr.astype(np.int32), D.indices.astype(np.int32), D.data,
                        storage=storage)
    plan = Plan(ctx, lib)
    plan.set_structures(sid, len(TABLE))
    plan.set_penalties(TABLE)
    return ctx, lib, plan


def _reference(D, sid, x):
    z = D.astype(np.float64) @ x.astype(np.float64)
    t = np.array(TABLE)[sid]
    u, o = np.minimum(z - t[:, 0], 0.0), np.maximum(z - t[:, 1], 0.0)
    G = float((t[:, 2] * u * u + t[:, 3] * o * o).sum())
    return z, G, 2.0 * (D.T.astype(np.float64) @ (t[:, 2] * u + t[:, 3] * o))


# (rows, beamlets, longest row): quad remainders, one row, one column, idle
# lanes, quads of 4, 16, 64 lanes, quads beyond one block (256 entries in
# float32, 384 in 16 bits) and beyond two, the largest staged vector
SHAPES = [(1, 1, 1), (3, 5, 5), (130, 7, 7), (203, 40, 33), (1001, 300, 64), (402, 700, 280), (150, 1400, 900),
          (300, 8191, 60)]


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("nv,nb,longest", SHAPES)
def test_products_against_float64_and_two_passes(nv, nb, longest, storage):
    import torch
    banner(f"one-read pass {nv} x {nb}, rows up to {longest}, {storage}")
    D, sid = _matrix(nv, nb, longest, seed=nv + nb)
    rng = np.random.default_rng(1)
    x = (rng.uniform(0.0, 1.0, nb) * (8.0 / max(1.0, longest / 4))).astype(np.float32)
    z, G, g = _reference(D, sid, x)
    got = {}
    for mode in (2, 0):
        ctx, lib, plan = _plan(D, sid, storage, mode)
        dose = torch.full((nv,), float("nan"), device="cuda")
        Gm = plan.objective(to_dev(x), dose)
        gm, G2 = plan.gradient(to_dev(x))
        gn = torch.empty_like(gm)
        assert plan.gradient_noalloc(to_dev(x), gn) == G2 == Gm
        assert torch.equal(gn, gm) and torch.equal(lib.apply(to_dev(x)), dose)
        lam, sigma = plan.lambda0(torch.ones(nb, device="cuda"), 5)
        got[mode] = (to_host(dose), Gm, to_host(gm), lam, sigma)
        # a row of n products: n roundings of at most 2^-24 each way
        eps = (longest + 4) * 2.0 ** -24
        assert np.max(np.abs(got[mode][0] - z)) <= eps * np.max(np.abs(z), initial=1e-30)
        assert abs(Gm - G) <= 4 * eps * max(G, 1e-30) + 1e-12
        assert rel_normwise(got[mode][2], g) <= 8 * eps
    assert got[2][3] == got[0][3] and abs(got[2][4] - got[0][4]) <= 1e-5 * got[0][4]


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_quads_of_exact_sizes(storage):
    """Quads one entry around the sizes that fill one, two, three and four
    blocks (256 entries in float32, 384 in 16 bits), every row full."""
    sizes = [n for full in (256, 384) for k in (1, 2, 3, 4) for n in (k * full - 1, k * full, k * full + 1)]
    nb = max(sizes)
    rng = np.random.default_rng(11)
    rows = [r for q, n in enumerate(sizes) for r in 4 * q + np.repeat(np.arange(4), n)]
    cols = np.concatenate([np.tile(np.sort(rng.choice(nb, n, replace=False)), 4) for n in sizes])
    vals = (rng.integers(64, 128, len(cols)) / 128.0).astype(np.float32)
    D = sp.csr_matrix((vals, (rows, cols)), shape=(4 * len(sizes), nb))
    for c in range(nb):   # a largest value of 1 in every column: exact in 16 bits
        D[int(D[:, c].argmax()), c] = 1.0
    D.sort_indices()
    sid = rng.integers(0, 2, D.shape[0]).astype(np.uint8)
    x = rng.uniform(0.0, 0.02, nb).astype(np.float32)
    z, G, g = _reference(D, sid, x)
    ctx, lib, plan = _plan(D, sid, storage, 2)
    eps = (nb + 4) * 2.0 ** -24
    assert np.max(np.abs(to_host(lib.apply(to_dev(x))) - z)) <= eps * np.max(np.abs(z))
    got, Gm = plan.gradient(to_dev(x))
    assert abs(Gm - G) <= 4 * eps * G and rel_normwise(to_host(got), g) <= 8 * eps


@pytest.mark.parametrize("nt", [1, 2, 4])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_solve_equals_two_pass_steps(storage, nt):
    """The same steps, backtracks and objectives (to float32 rounding of the
    iterates) as the two separate passes; repeated bit for bit; per-voxel
    targets included."""
    banner(f"one-read solve {storage} nt={nt}")
    D, sid = _matrix(1501, 211, 40, seed=7)
    x1 = np.ones(211, np.float32)
    tr = {}
    for mode in (2, 0):
        ctx, lib, plan = _plan(D, sid, storage, mode)
        for targets in (False, True):
            if targets:
                T = np.random.default_rng(5).uniform(1.0, 3.0, 1501).astype(np.float32)
                plan.set_voxel_targets(T, T)
            lam, _ = plan.lambda0(to_dev(x1), 20)
            runs = []
            for _ in range(2):
                x = to_dev(x1)
                res, t = plan.solve(x, eps=1e-4, alpha=2.0, lambda0=4 * lam, max_iter=25, fixed_iters=True,
                                    trials_per_pass=nt, trace=True, warm_start=True)
                runs.append((t, to_host(x).tobytes(), res.G_final, res.forward_passes, res.adjoint_passes))
            assert runs[0] == runs[1]
            assert plan.objective(x) == res.G_final
            tr[mode, targets] = runs[0]
    for targets in (False, True):
        a, b = tr[2, targets], tr[0, targets]
        assert a[3:] == b[3:] and len(a[0]) == len(b[0])
        for (k, m, lam, s, G), (k2, m2, lam2, s2, G2) in zip(a[0], b[0]):
            assert (k, m, lam) == (k2, m2, lam2) and abs(G - G2) <= 1e-5 * G2


def test_non_finite_and_huge_vectors():
    """A column of infinity or NaN reaches the rows that hold it and no other;
    residuals near float32's limit come out as the two passes give them."""
    import torch
    D, sid = _matrix(403, 60, 9, seed=3)
    for value in (np.inf, -np.inf, np.nan, 3e37, -2e36):
        x = np.random.default_rng(2).uniform(0.0, 2.0, 60).astype(np.float32)
        x[17] = value
        out = {}
        for mode in (2, 0):
            ctx, lib, plan = _plan(D, sid, "f32", mode)
            dose = torch.empty(403, device="cuda")
            G = plan.objective(to_dev(x), dose)
            g, _ = plan.gradient(to_dev(x))
            out[mode] = (to_host(dose), G, to_host(g))
        for a, b in zip(out[2], out[0]):
            a, b = np.atleast_1d(np.asarray(a, np.float64)), np.atleast_1d(np.asarray(b, np.float64))
            fin = np.isfinite(b)
            assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[~fin & ~np.isnan(b)], b[~fin & ~np.isnan(b)])
            assert np.allclose(a[fin], b[fin], rtol=1e-5, atol=1e-5 * np.max(np.abs(b[fin]), initial=0.0))


def test_beamlets_beyond_the_staged_vector():
    """8,192 beamlets keep the two separate passes."""
    D, sid = _matrix(64, 8192, 20, seed=9)
    a = _plan(D, sid, "f32", 2)[2].gradient(to_dev(np.ones(8192, np.float32)))
    b = _plan(D, sid, "f32", 0)[2].gradient(to_dev(np.ones(8192, np.float32)))
    assert a[1] == b[1] and np.array_equal(to_host(a[0]), to_host(b[0]))


def test_row_blocks_made_when_first_needed():
    """The workgroup-wide forward is never a one-read pass: it makes the
    matrix's row blocks on first use and gives the one-read pass's steps."""
    D, sid = _matrix(703, 4001, 50, seed=13)
    ctx, lib, plan = _plan(D, sid, "f32", 2)
    x1 = np.full(4001, 0.5, np.float32)
    lam, _ = plan.lambda0(to_dev(x1), 20)
    z, G64, g64 = _reference(D, sid, x1)
    eps = 54 * 2.0 ** -24
    tr = []
    for wave in (1, 0):
        ctx.set_option("fwd_wave", wave)
        x = to_dev(x1)
        res, t = plan.solve(x, eps=1e-4, alpha=2.0, lambda0=2 * lam, max_iter=8, fixed_iters=True, trace=True)
        tr.append(t)
        g, G = plan.gradient(to_dev(x1))
        assert plan.objective(to_dev(x1)) == G and abs(G - G64) <= 4 * eps * G64
        assert rel_normwise(to_host(g), g64) <= 8 * eps
        assert np.max(np.abs(to_host(lib.apply(to_dev(x1))) - z)) <= eps * np.max(np.abs(z))
    for (k, m, s, _, Ga), (k2, m2, s2, _, Gb) in zip(*tr):
        assert (k, m, s) == (k2, m2, s2) and abs(Ga - Gb) <= 1e-5 * Gb


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("nv,nb,longest", [(9, 2, 2), (403, 17, 9), (1501, 211, 40), (2003, 1024, 25), (20003, 130, 25)])
def test_one_launch_per_iteration_equals_two(nv, nb, longest, storage):
    """A small plan's launch that decides, steps and passes in one gives the
    bits of the two launches that a profiled solve keeps; with the stopping
    rule, backtracks and resumption too.  (1,024 beamlets: one per thread;
    20,003 rows: several rounds of column sums.)"""
    D, sid = _matrix(nv, nb, longest, seed=nv)
    ctx, lib, plan = _plan(D, sid, storage, 2)
    x1 = np.ones(nb, np.float32)
    lam, _ = plan.lambda0(to_dev(x1), 20)
    for kw in (dict(max_iter=30, fixed_iters=True), dict(max_iter=400, delta=1e-4, warm_start=True),
               dict(max_iter=5, fixed_iters=True, warm_start=True), dict(max_iter=0)):
        out = []
        for profile in (0, 3):
            x = to_dev(x1)
            res, t = plan.solve(x, eps=1e-4, alpha=2.0, lambda0=4 * lam, trace=True, profile=profile, **kw)
            out.append((t, to_host(x).tobytes(), res.G_initial, res.G_final, res.iterations, res.status,
                        res.forward_passes, res.adjoint_passes))
        assert out[0] == out[1], kw
