"""Finite thresholds far beyond any dose ("no limit"): of a side without
weight, of a structure without voxels, of a side that no dose reaches, per
structure and per voxel.  They never enter a residual, so objective, gradient
and steps are those of the same plan with ordinary thresholds there."""
import numpy as np
import pytest
import scipy.sparse as sp

from gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu

NV, NB, LONGEST = 1203, 97, 40
# (the usual table: structures 0 and 1; structure 2 has no voxels)
TABLE = [(2.0, 3.0, 1.0, 0.5), (0.0, 1.5, 0.0, 0.3), (0.0, 0.0, 0.0, 0.0)]
TOP = 1.7e308


def _table(where, T):
    t = [list(row) for row in TABLE]
    if where == "no weight":        # upper limit of the target without weight
        t[0] = [2.0, T, 1.0, 0.0]
    elif where == "no weight below":
        t[1] = [T, 1.5, 0.0, 0.3]
    elif where == "absent":         # a structure without voxels, both sides weighted
        t[2] = [T, -T, 1.0, 1.0]
    elif where == "unreachable":    # weighted, but above every dose
        t[0] = [2.0, T, 1.0, 0.5]
    elif where == "unreachable below":
        t[1] = [-T, 1.5, 0.7, 0.3]
    return t


def _problem():
    rng = np.random.default_rng(5)
    lens = rng.integers(1, LONGEST + 1, NV)
    rows = np.repeat(np.arange(NV), lens)
    cols = np.concatenate([np.sort(rng.choice(NB, n, replace=False)) for n in lens])
    vals = (rng.integers(1, 129, len(rows)) / 128.0).astype(np.float32)
    D = sp.csr_matrix((vals, (rows, cols)), shape=(NV, NB))
    return D, rng.integers(0, 2, NV).astype(np.uint8), rng.uniform(0.0, 0.5, NB).astype(np.float32)


def _reference(D, t, x):
    """G, gradient, and a bound on each column's rounding: a dose of n products
    carries n + 4 roundings of 2^-24, its residual one more, the result one."""
    D = D.astype(np.float64)
    z = D @ x.astype(np.float64)
    u, o = np.minimum(z - t[:, 0], 0.0), np.maximum(z - t[:, 1], 0.0)
    r = t[:, 2] * u + t[:, 3] * o
    dr = (t[:, 2] + t[:, 3]) * (LONGEST + 4) * 2.0 ** -24 * z + 2.0 ** -24 * np.abs(r)
    g = 2.0 * (D.T @ r)
    slack = 2.0 * (D.T @ dr) + 2.0 ** -23 * (D.T @ np.abs(r))
    return float((t[:, 2] * u * u + t[:, 3] * o * o).sum()), g, slack + 2.0 ** -24 * np.abs(g)


def _run(D, sid, table, targets, x, one_read):
    from paper_0908_4421_amd.imrt import Context, Dose, Plan
    lib = Dose.from_csr(Context(0, one_read=one_read), NV, NB, D.indptr.astype(np.int32), D.indices.astype(np.int32),
                        D.data)
    plan = Plan(lib.ctx, lib)
    plan.set_structures(sid, 3)
    plan.set_penalties(table)
    if targets is not None:
        plan.set_voxel_targets(*targets)
    g, G = plan.gradient(to_dev(x))
    again, G2 = plan.gradient(to_dev(x))
    assert G == G2 and np.array_equal(to_host(g), to_host(again))
    lam, _ = plan.lambda0(to_dev(np.ones(NB, np.float32)), 20)
    out = [to_host(g), G]
    for nt in (1, 2):
        xs = to_dev(x)
        res, tr = plan.solve(xs, eps=1e-4, alpha=2.0, lambda0=lam, max_iter=15, fixed_iters=True, trace=True,
                             trials_per_pass=nt)
        out += [tr, to_host(xs)]
    return out


def _check(D, sid, table, targets, x):
    t = np.array(table, np.float64)[sid]
    if targets is not None:
        t[:, 0], t[:, 1] = targets[0], targets[1]
    G64, g64, slack = _reference(D, t, x)
    one, two = _run(D, sid, table, targets, x, 2), _run(D, sid, table, targets, x, 0)
    for g, G, *_ in (one, two):
        assert abs(G - G64) <= 4 * (LONGEST + 4) * 2.0 ** -24 * G64
        assert np.all(np.abs(g - g64) <= slack), np.max(np.abs(g - g64) / slack)
    for k in (2, 4):   # the same steps, and iterates that agree
        assert len(one[k]) == len(two[k]) == 15
        for (i, m, lam, _, G), (i2, m2, lam2, _, G2) in zip(one[k], two[k]):
            assert (i, m, lam) == (i2, m2, lam2) and abs(G - G2) <= 1e-5 * G2
        assert np.allclose(one[k + 1], two[k + 1], rtol=1e-4, atol=1e-5)


@pytest.mark.parametrize("T", [1e10, 1e14, 1e18, 1e30, TOP])
@pytest.mark.parametrize("where", ["no weight", "no weight below", "absent", "unreachable", "unreachable below"])
def test_structure_thresholds(where, T):
    banner(f"threshold {T:g}: {where}")
    D, sid, x = _problem()
    _check(D, sid, _table(where, T), None, x)


@pytest.mark.parametrize("replaced", [False, True])
@pytest.mark.parametrize("T", [1e10, 1e18, 3e38])
def test_voxel_targets(T, replaced):
    """Per-voxel targets without an upper limit, those of sides without weight
    out of any range, and (replaced) structure thresholds that they replace."""
    D, sid, x = _problem()
    table = [(TOP, -TOP, 1.0, 0.5), (TOP, 1.5, 0.0, 0.3), (TOP, -TOP, 1.0, 1.0)] if replaced else TABLE
    rng = np.random.default_rng(6)
    Tu = np.where(sid == 0, rng.uniform(1.0, 3.0, NV), T).astype(np.float32)
    To = np.where(rng.random(NV) < 0.5, rng.uniform(1.0, 3.0, NV), T).astype(np.float32)
    banner(f"voxel targets {T:g}")
    _check(D, sid, table, (Tu, To), x)


def test_targets_before_structures_and_new_tables():
    """The bound follows structures, penalties and targets set in any order."""
    from paper_0908_4421_amd.imrt import Context, Dose, Plan
    D, sid, x = _problem()
    lib = Dose.from_csr(Context(0, one_read=2), NV, NB, D.indptr.astype(np.int32), D.indices.astype(np.int32), D.data)
    plan = Plan(lib.ctx, lib)
    To = np.full(NV, 2.0, np.float32)
    Tu = np.where(sid == 1, 1e20, 1.0).astype(np.float32)
    plan.set_voxel_targets(Tu, To)
    for flip in (0, 1):
        ids = (sid ^ flip).astype(np.uint8)
        plan.set_structures(ids, 2)
        for w in (0.0, 0.25):   # the huge targets without and with weight
            table = [(0.0, 0.0, 1.0, 0.5), (0.0, 0.0, w, 0.3)]
            plan.set_penalties(table)
            t = np.array(table, np.float64)[ids]
            t[:, 0], t[:, 1] = Tu, To
            G64, g64, slack = _reference(D, t, x)
            g, G = plan.gradient(to_dev(x))
            assert abs(G - G64) <= 4 * (LONGEST + 4) * 2.0 ** -24 * G64
            assert np.all(np.abs(to_host(g) - g64) <= slack), np.max(np.abs(to_host(g) - g64) / slack)
    plan.set_voxel_targets(None, None)
    plan.set_penalties(TABLE[:2])
    G64, g64, slack = _reference(D, np.array(TABLE, np.float64)[ids], x)
    g, G = plan.gradient(to_dev(x))
    assert np.all(np.abs(to_host(g) - g64) <= slack)
