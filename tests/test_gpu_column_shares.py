"""The adjoint partition with bounds at column starts (columns short against a
workgroup's share) and with equal shares, around the line between them:
columns of equal, ragged and no nonzeros against float64."""
import numpy as np
import pytest
import scipy.sparse as sp

from gpu_util import banner, rel_normwise, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("lengths", [
    [512] * 40,                                  # a share of 1,024 holds two columns exactly
    [513] * 40,                                  # one nonzero over the line: equal shares
    [0] * 7 + [300, 0, 0, 511, 1] * 30 + [0] * 9,  # empty columns at, before and after bounds
    [2] * 4096,                                  # many columns a workgroup
    [512],                                       # fewer nonzeros than a share
], ids=["at", "over", "ragged", "short", "one"])
def test_transpose_and_solve(lengths, storage):
    from paper_0908_4421_amd.imrt import Context, Dose, Plan
    nv, nb = 1200, len(lengths)
    banner(f"column shares: {nb} columns of up to {max(lengths)}, {storage}")
    rng = np.random.default_rng(nb)
    cols = np.repeat(np.arange(nb), lengths)
    rows = np.concatenate([rng.choice(nv, n, replace=False) for n in lengths])
    vals = np.ones(len(rows), np.float32)   # (exact in every storage)
    D = sp.csr_matrix((vals, (rows, cols)), shape=(nv, nb))
    D.sort_indices()
    ctx = Context(0, one_read=0)
    lib = Dose.from_csr(ctx, nv, nb, D.indptr.astype(np.int32), D.indices.astype(np.int32), D.data, storage=storage)
    r = rng.normal(0.0, 1.0, nv).astype(np.float32)
    want = D.T.astype(np.float64) @ r.astype(np.float64)
    # float64 sums, rounded once to float32
    for share in (1024, 16, 4096, 1024):
        lib.repartition(share, 1)
        y = to_host(lib.apply_transpose(to_dev(r)))
        assert np.max(np.abs(y - want)) <= 2.0 ** -23 * np.max(np.abs(want))
        assert np.array_equal(y, to_host(lib.apply_transpose(to_dev(r))))
        assert np.all(y[np.array(lengths) == 0] == 0.0)
    plan = Plan(ctx, lib)
    plan.set_structures(np.zeros(nv, np.uint8), 1)
    plan.set_penalties([(3.0, 3.0, 1.0, 1.0)])
    x = to_dev(np.ones(nb, np.float32))
    lam, _ = plan.lambda0(x, 20)
    res, tr = plan.solve(x, eps=1e-4, alpha=2.0, lambda0=lam, max_iter=20, fixed_iters=True, trace=True)
    g, _ = plan.gradient(to_dev(np.ones(nb, np.float32)))
    z = D.astype(np.float64) @ np.ones(nb)
    assert rel_normwise(to_host(g), 2.0 * (D.T.astype(np.float64) @ (z - 3.0))) <= 1e-6
    assert all(b[4] < a[4] for a, b in zip(tr, tr[1:])) and res.G_final < res.G_initial
