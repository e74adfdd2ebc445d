"""Each column of a gradient on its own against float64: columns far smaller
than the largest (a vector with one huge entry, columns scaled down, weights
decades apart, residuals that nearly vanish), and vectors with infinities or
residuals beyond float32's range, which repeat bit for bit."""
import numpy as np
import pytest
import scipy.sparse as sp

from gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu

BLOCKS, ROWS, COLS = 12, 101, 9     # a block-diagonal matrix: blocks share no row
NV, NB = BLOCKS * ROWS, BLOCKS * COLS
TABLE = [(2.0, 3.0, 1.0, 0.5), (0.0, 1.5, 0.0, 0.3)]


def _blocks(seed, scale=None):
    rng = np.random.default_rng(seed)
    D = np.zeros((NV, NB), np.float32)
    for b in range(BLOCKS):
        D[b * ROWS:(b + 1) * ROWS, b * COLS:(b + 1) * COLS] = \
            rng.integers(1, 129, (ROWS, COLS)) / 128.0 * (rng.random((ROWS, COLS)) < 0.7)
    if scale is not None:
        D *= np.asarray(scale, np.float32)
    return sp.csr_matrix(D)


def _plan(D, table, sid, one_read, storage="f32"):
    from paper_0908_4421_amd.imrt import Context, Dose, Plan
    lib = Dose.from_csr(Context(0, one_read=one_read), D.shape[0], D.shape[1], D.indptr.astype(np.int32),
                        D.indices.astype(np.int32), D.data, storage=storage)
    plan = Plan(lib.ctx, lib)
    plan.set_structures(sid, len(table))
    plan.set_penalties(table)
    return lib, plan


def _check(D, table, sid, x, solve_steps=0):
    """Every column within 1e-6 of sum_j |D_jc| (2 |r_j| + what a dose's
    rounding moves it: at most COLS + 4 roundings of 2^-24)."""
    t = np.array(table, np.float64)[sid]
    D64 = D.astype(np.float64)
    z = D64 @ x.astype(np.float64)
    r = t[:, 2] * np.minimum(z - t[:, 0], 0.0) + t[:, 3] * np.maximum(z - t[:, 1], 0.0)
    want = 2.0 * (D64.T @ r)
    zabs = D64 @ np.abs(x.astype(np.float64))
    active = (r != 0.0) | (np.abs(z - t[:, 0]) < 1e-5 * np.abs(z)) | (np.abs(z - t[:, 1]) < 1e-5 * np.abs(z))
    slack = D64.T @ (1e-6 * 2.0 * np.abs(r) + active * (t[:, 2] + t[:, 3]) * 2 * (COLS + 4) * 2.0 ** -24 * zabs)
    out = []
    for mode in (0, 2):
        lib, plan = _plan(D, table, sid, mode)
        g, G = plan.gradient(to_dev(x))
        g2, G2 = plan.gradient(to_dev(x))
        gn = to_dev(np.full(NB, np.nan, np.float32))
        assert plan.gradient_noalloc(to_dev(x), gn) == G == G2
        g = to_host(g)
        assert np.array_equal(g, to_host(g2)) and np.array_equal(g, to_host(gn))
        err = np.abs(g - want)
        assert np.all(err <= slack), (mode, np.max(err / np.maximum(slack, 1e-300)), int(np.argmax(err / np.maximum(slack, 1e-300))))
        out.append(g)
    return out


@pytest.mark.parametrize("spike", [1e4, 1e6, 1e10, 1e14, 1e18, 1e24, 1e30])
def test_one_huge_entry(spike):
    banner(f"one entry of {spike:g}")
    rng = np.random.default_rng(1)
    x = rng.uniform(0.0, 1.0, NB).astype(np.float32)
    x[4] = spike
    _check(_blocks(0), TABLE, rng.integers(0, 2, NV).astype(np.uint8), x)


@pytest.mark.parametrize("small", [1e-4, 1e-6, 1e-10, 1e-12, 1e-14, 1e-20])
def test_columns_decades_apart(small):
    banner(f"columns scaled by {small:g}")
    rng = np.random.default_rng(2)
    x = rng.uniform(0.0, 1.0, NB).astype(np.float32)
    scale = np.where(np.arange(NB) % 3 == 1, small, 1.0)
    _check(_blocks(1, scale), TABLE, rng.integers(0, 2, NV).astype(np.uint8), x)


@pytest.mark.parametrize("weight", [1e4, 1e8, 1e12, 1e20])
def test_weights_decades_apart(weight):
    """Heavy voxels in the first blocks only."""
    banner(f"weights {weight:g} apart")
    rng = np.random.default_rng(3)
    x = rng.uniform(0.0, 1.0, NB).astype(np.float32)
    sid = np.where(np.arange(NV) < 3 * ROWS, 2, rng.integers(0, 2, NV)).astype(np.uint8)
    _check(_blocks(2), TABLE + [(2.0, 2.0, weight, weight)], sid, x)


@pytest.mark.parametrize("gap", [1e-3, 1e-6, 1e-9, 1e-12])
def test_residuals_that_nearly_vanish(gap):
    """Doses all but at their thresholds (D and x exact in float32, so that the
    residuals are), of one sign and of both in a column."""
    banner(f"residuals of {gap:g}")
    rng = np.random.default_rng(4)
    D = _blocks(3)
    x = (rng.integers(1, 9, NB) / 8.0).astype(np.float32)
    z = D.astype(np.float64) @ x.astype(np.float64)
    for both in (False, True):
        sid = np.zeros(NV, np.uint8)
        values = np.unique(z)
        assert len(values) <= 4 * NV
        T = np.sort(rng.choice(values, 255, replace=False))
        # a voxel's structure: the threshold nearest its dose; the others satisfied
        near = np.searchsorted(T, z).clip(0, 254)
        hit = T[near] == z
        sid = np.where(hit, near, 255).astype(np.uint8)
        sign = np.where(rng.random(255) < 0.5, 1.0, -1.0) if both else np.ones(255)
        table = [(t * (1.0 + gap) if s > 0 else 0.0, t * (1.0 - gap) if s < 0 else 1e3, 1.0, 1.0)
                 for t, s in zip(T, sign)] + [(0.0, 1e3, 1.0, 1.0)]
        t = np.array(table)[sid]
        r = np.minimum(z - t[:, 0], 0.0) + np.maximum(z - t[:, 1], 0.0)
        want = 2.0 * (D.astype(np.float64).T @ r)
        size = 2.0 * (D.astype(np.float64).T @ np.abs(r))
        for mode in (0, 2):
            g, G = _plan(D, table, sid, mode)[1].gradient(to_dev(x))
            # residuals and the result each rounded once to float32
            assert np.all(np.abs(to_host(g) - want) <= 2.0 ** -22 * size), (mode, both)


@pytest.mark.parametrize("nt", [1, 2, 4])
def test_solves_of_such_plans(nt):
    """Solves step as the two separate passes do, and repeat bit for bit:
    small plans in one launch an iteration (nt 1, and in two when profiled),
    several trials a pass, a batch."""
    from paper_0908_4421_amd.imrt import Plan
    rng = np.random.default_rng(5)
    scale = np.where(np.arange(NB) % 3 == 1, 1e-10, 1.0)
    sid = np.where(np.arange(NV) < 3 * ROWS, 2, rng.integers(0, 2, NV)).astype(np.uint8)
    for D, table in ((_blocks(5, scale), TABLE + [(2.0, 2.0, 1.0, 1.0)]),
                     (_blocks(6), TABLE + [(2.0, 2.0, 1e8, 1e8)])):
        out = {}
        for mode in (0, 2):
            lib, plan = _plan(D, table, sid, mode)
            lam, _ = plan.lambda0(to_dev(np.ones(NB, np.float32)), 20)
            args = dict(eps=1e-4, alpha=2.0, max_iter=12, fixed_iters=True, trials_per_pass=nt)
            runs = []
            for profile in (0, 0, 2):
                x = to_dev(np.full(NB, 0.4, np.float32))
                res, tr = plan.solve(x, lambda0=4 * lam, trace=True, profile=profile, **args)
                runs.append((tr, to_host(x).tobytes(), res.G_final))
            assert runs[0] == runs[1] == runs[2]
            xs = [to_dev(np.full(NB, 0.4, np.float32))]
            Plan.solve_batch([plan], xs, lambda0s=[4 * lam], **args)
            assert to_host(xs[0]).tobytes() == runs[0][1]
            out[mode] = runs[0]
        for (k, m, s, _, G), (k2, m2, s2, _, G2) in zip(out[0][0], out[2][0]):
            assert (k, m, s) == (k2, m2, s2) and abs(G - G2) <= 1e-5 * G2
        a, b = (np.frombuffer(out[m][1], np.float32) for m in (0, 2))
        assert np.allclose(a, b, rtol=1e-4, atol=1e-6)


@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e37, -2e36, 3e38])
def test_wild_vectors_repeat_and_equal_two_passes(value, storage):
    """Infinity, NaN and values whose residuals leave float32: each column as
    the two separate passes give it, the same on every run."""
    rng = np.random.default_rng(7)
    D = _blocks(8)
    top = np.asarray(D.argmax(axis=0)).ravel()
    D = D.tolil()
    for c in range(NB):
        D[top[c], c] = 1.0      # exact in 16 bits
    D = D.tocsr()
    D.sort_indices()
    sid = rng.integers(0, 2, NV).astype(np.uint8)
    x = rng.uniform(0.0, 1.0, NB).astype(np.float32)
    x[4] = value
    got = {}
    for mode in (0, 2):
        lib, plan = _plan(D, TABLE, sid, mode, storage)
        runs = [to_host(plan.gradient(to_dev(x))[0]) for _ in range(4)]
        assert all(r.tobytes() == runs[0].tobytes() for r in runs)
        got[mode] = runs[0].astype(np.float64)
    a, b = got[2], got[0]
    fin = np.isfinite(b)
    assert np.array_equal(np.isnan(a), np.isnan(b))
    assert np.array_equal(a[~fin & ~np.isnan(b)], b[~fin & ~np.isnan(b)])
    z = D.astype(np.float64) @ np.abs(np.nan_to_num(x.astype(np.float64), nan=0.0, posinf=0.0, neginf=0.0))
    size = D.astype(np.float64).T @ (z + 3.0)
    assert np.all(np.abs(a - b)[fin] <= 2 * (COLS + 4) * 2.0 ** -23 * size[fin] + 2.0 ** -23 * np.abs(b[fin]))


@pytest.mark.parametrize("spike", [1e6, 1e14, 1e25])
def test_power_iteration_of_a_spiked_vector(spike):
    """One power iteration from a vector with one huge entry: the step size
    and sigma of the two separate passes (the block of the entry decides)."""
    rng = np.random.default_rng(9)
    D = _blocks(10)
    v = rng.uniform(0.5, 1.0, NB).astype(np.float32)
    v[4] = spike
    sid = np.zeros(NV, np.uint8)
    got = [_plan(D, TABLE[:1], sid, mode)[1].lambda0(to_dev(v), it) for mode in (0, 2) for it in (1, 3)]
    for a, b in zip(got[:2], got[2:]):
        assert a[0] == b[0] and abs(a[1] - b[1]) <= 1e-6 * a[1]


def test_wild_vectors_repeat_over_many_workgroups():
    """Column sums of a wild vector that many waves add to: one order."""
    rng = np.random.default_rng(11)
    nv, nb = 40003, 60
    cols = np.concatenate([np.sort(rng.choice(nb, 20, replace=False)) for _ in range(nv)])
    D = sp.csr_matrix((rng.uniform(0.1, 1.0, 20 * nv).astype(np.float32), (np.repeat(np.arange(nv), 20), cols)),
                      shape=(nv, nb))
    x = rng.uniform(0.0, 1.0, nb).astype(np.float32)
    x[17] = 2e37
    lib, plan = _plan(D, TABLE, rng.integers(0, 2, nv).astype(np.uint8), 2)
    runs = {to_host(plan.gradient(to_dev(x))[0]).tobytes() for _ in range(12)}
    assert len(runs) == 1


def test_a_solve_whose_residuals_vanish():
    """A plan that its beamlets can meet exactly: G falls by decades and the
    columns' sums with it, whose integers stop being precise on the way.  The
    same bits in one launch an iteration, in two, and in a batch; the steps of
    the two separate passes while G is above rounding."""
    from paper_0908_4421_amd.imrt import Plan
    rng = np.random.default_rng(12)
    nv, nb = 900, 300
    D = sp.random(nv, nb, density=0.02, random_state=np.random.RandomState(3), format="csr", dtype=np.float32)
    D.data[:] = rng.integers(32, 129, D.nnz) / 128.0
    D.sort_indices()
    goal = rng.uniform(0.5, 1.5, nb)
    z = D.astype(np.float64) @ goal
    T = z.astype(np.float32)
    sid = np.zeros(nv, np.uint8)
    tr = {}
    for mode in (0, 2):
        lib, plan = _plan(D, [(0.0, 0.0, 1.0, 1.0)], sid, mode)
        plan.set_voxel_targets(T, T)
        lam, _ = plan.lambda0(to_dev(np.ones(nb, np.float32)), 20)
        args = dict(eps=1e-4, alpha=2.0, max_iter=1500, fixed_iters=True)
        runs = []
        for profile in (0, 4):
            x = to_dev(np.ones(nb, np.float32))
            res, t = plan.solve(x, lambda0=lam, trace=True, profile=profile, **args)
            runs.append((t, to_host(x).tobytes(), res.status))
        assert runs[0] == runs[1]
        xs = [to_dev(np.ones(nb, np.float32))]
        Plan.solve_batch([plan], xs, lambda0s=[lam], **args)
        assert to_host(xs[0]).tobytes() == runs[0][1]
        tr[mode] = runs[0][0]
    G0 = tr[0][0][4]
    assert min(e[4] for e in tr[2]) < 1e-9 * G0      # it did fall that far
    for (k, m, s, _, G), (k2, m2, s2, _, G2) in zip(tr[0], tr[2]):
        if G < 1e-6 * G0:
            break
        assert (k, m, s) == (k2, m2, s2) and abs(G - G2) <= 1e-3 * G2, k


def test_served_plans_with_weights_apart():
    """Re-plans of one patient that share the matrix's pass, with a target
    weighted a hundred million times: as served alone and as solved alone."""
    from paper_0908_4421_amd.imrt import Context, Dose, Plan, Server
    from workloads import SMALL, penalty_table
    base = np.array(penalty_table(SMALL), np.float64)
    tables = []
    for w in (1.0, 1e8, 1e10, 1e8):
        t = base.copy()
        t[1, 2:] *= w
        tables.append(t)
    out = {}
    for share in (1, 0):
        srv = Server(Context(0, serve_shared_adjoint=share), budget_bytes=8 << 30, max_live=16)
        tickets = [srv.submit(5, SMALL, t, max_iter=60, fixed_iters=True) for t in tables]
        nb = None
        got = []
        for tk in tickets:
            res, times, x = srv.wait(tk, nb or 0) if nb else (None, None, None)
            if nb is None:
                ctx = Context(0)
                dose = Dose.from_geometry(ctx, SMALL)
                nb = dose.nb
                res, times, x = srv.wait(tk, nb)
            got.append((res.iterations, res.status, res.G_final, np.asarray(x).tobytes(), times.lambda0))
        stats = srv.stats()
        srv.close()
        assert (stats["adjoint_groups_shared"] > 0) == bool(share)
        out[share] = got
    assert out[1] == out[0]
    dose.repartition_targets(ctx.get_option("serve_adjoint_workgroups"), ctx.get_option("serve_forward_workgroups"))
    for t, (it, status, G, xb, lam) in zip(tables, out[1]):
        plan = Plan(ctx, dose)
        plan.set_structures(None, len(t))
        plan.set_penalties(t)
        x = to_dev(np.ones(nb, np.float32))
        res, _ = plan.solve(x, eps=1e-4, alpha=2.0, lambda0=lam, max_iter=60, fixed_iters=True)
        assert (res.iterations, res.status, res.G_final, to_host(x).tobytes()) == (it, status, G, xb)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_stored_negative_zeros(storage):
    """A stored -0 is a nonzero place like a stored 0: times infinity it is
    NaN, as in the two separate passes, and with finite vectors it adds
    nothing."""
    import torch
    rng = np.random.default_rng(13)
    D = _blocks(14).tocsr()
    D.data[:] = 1.0
    zero = rng.random(D.nnz) < 0.2
    D.data[zero] = np.where(rng.random(zero.sum()) < 0.5, -0.0, 0.0)
    sid = rng.integers(0, 2, NV).astype(np.uint8)
    for spike in (0.5, np.inf):
        x = rng.uniform(0.0, 1.0, NB).astype(np.float32)
        x[4] = x[22] = spike
        out = {}
        for mode in (0, 2):
            lib, plan = _plan(D, TABLE, sid, mode, storage)
            dose = torch.empty(NV, device="cuda")
            G = plan.objective(to_dev(x), dose)
            out[mode] = (to_host(dose), to_host(lib.apply(to_dev(x))), to_host(plan.gradient(to_dev(x))[0]))
        assert np.isinf(spike) == bool(np.isnan(out[0][0]).any())
        for a, b in zip(out[2], out[0]):
            assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
            fin = np.isfinite(b)
            assert np.allclose(a[fin], b[fin], rtol=1e-5, atol=1e-5 * np.max(np.abs(b[fin]), initial=0.0))


@pytest.mark.parametrize("nt", [1, 2])
@pytest.mark.parametrize("storage", ["f32", "bf16", "f16"])
def test_solves_with_targets_and_weights_apart(storage, nt):
    """Columns summed again in every storage, with per-voxel targets: stored
    residuals and those made from the rows."""
    from paper_0908_4421_amd.imrt import Plan
    rng = np.random.default_rng(15)
    D = _blocks(16)
    top = np.asarray(D.argmax(axis=0)).ravel()
    D = D.tolil()
    for c in range(NB):
        D[top[c], c] = 1.0      # exact in 16 bits
    D = D.tocsr()
    D.sort_indices()
    sid = np.where(np.arange(NV) < 3 * ROWS, 2, rng.integers(0, 2, NV)).astype(np.uint8)
    table = TABLE + [(2.0, 2.0, 1e9, 1e9)]
    T = rng.uniform(1.0, 3.0, NV).astype(np.float32)
    out = {}
    for mode in (0, 2):
        lib, plan = _plan(D, table, sid, mode, storage)
        plan.set_voxel_targets(T, T + 0.25)
        lam, _ = plan.lambda0(to_dev(np.ones(NB, np.float32)), 20)
        args = dict(eps=1e-4, alpha=2.0, max_iter=40, fixed_iters=True, trials_per_pass=nt)
        runs = []
        for profile in (0, 3):
            x = to_dev(np.full(NB, 0.4, np.float32))
            res, tr = plan.solve(x, lambda0=4 * lam, trace=True, profile=profile, **args)
            runs.append((tr, to_host(x).tobytes(), res.G_final))
        assert runs[0] == runs[1]
        xs = [to_dev(np.full(NB, 0.4, np.float32))]
        Plan.solve_batch([plan], xs, lambda0s=[4 * lam], **args)
        assert to_host(xs[0]).tobytes() == runs[0][1]
        out[mode] = runs[0]
    for (k, m, s, _, G), (k2, m2, s2, _, G2) in zip(out[0][0], out[2][0]):
        assert (k, m, s) == (k2, m2, s2) and abs(G - G2) <= 1e-5 * G2
    a, b = (np.frombuffer(out[m][1], np.float32) for m in (0, 2))
    assert np.allclose(a, b, rtol=1e-4, atol=1e-6)
