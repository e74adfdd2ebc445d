"""Solves with several trial steps per pass around the beamlet counts where
the one-read pass's vectors and column sums reach a workgroup's LDS: the same
steps as the two separate passes on either side of the line."""
import numpy as np
import pytest
import scipy.sparse as sp

from gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu


# (16-bit matrices of so many beamlets solve with two trials only once they are
# partitioned for shared dispatches; four trials are refused before the line)
@pytest.mark.parametrize("nt,nb,storage", [(2, nb, st) for nb in (6527, 6528, 6799, 6804, 6811, 6823, 6824)
                                           for st in ("f32", "bf16")] +
                         [(4, nb, "f32") for nb in (3001, 3399, 3404, 3411)])
def test_solve_at_the_edge(nt, nb, storage):
    from paper_0908_4421_amd.imrt import IMRT_EUNSUPPORTED, Context, Dose, ImrtError, Plan
    banner(f"{nt} trials of {nb} beamlets, {storage}")
    nv, row = 601, 60
    rng = np.random.default_rng(nb)
    cols = np.concatenate([np.sort(rng.choice(nb, row, replace=False)) for _ in range(nv)])
    D = sp.csr_matrix((np.full(nv * row, 0.5, np.float32), (np.repeat(np.arange(nv), row), cols)), shape=(nv, nb))
    sid = rng.integers(0, 2, nv).astype(np.uint8)
    out, refused = {}, []
    for mode in (2, 0):
        lib = Dose.from_csr(Context(0, one_read=mode), nv, nb, D.indptr.astype(np.int32), D.indices.astype(np.int32),
                            D.data, storage=storage)
        if storage == "bf16":
            lib.repartition_targets(128, 32)
        plan = Plan(lib.ctx, lib)
        plan.set_structures(sid, 2)
        plan.set_penalties([(2.0, 3.0, 1.0, 0.5), (0.0, 1.5, 0.0, 0.3)])
        x = to_dev(np.full(nb, 0.5, np.float32))
        lam, _ = plan.lambda0(x, 10)
        try:
            res, tr = plan.solve(x, eps=1e-4, alpha=2.0, lambda0=4 * lam, max_iter=6, fixed_iters=True, trace=True,
                                 trials_per_pass=nt)
        except ImrtError as e:
            assert e.code == IMRT_EUNSUPPORTED
            refused.append(mode)
            continue
        out[mode] = (tr, to_host(x), res.forward_passes)
    if nt == 4 and nb >= 3399:
        assert refused == [2, 0]
        return
    assert out[2][2] == out[0][2] and len(out[2][0]) == len(out[0][0])
    for (k, m, s, _, G), (k2, m2, s2, _, G2) in zip(out[2][0], out[0][0]):
        assert (k, m, s) == (k2, m2, s2) and abs(G - G2) <= 1e-5 * G2
    assert np.allclose(out[2][1], out[0][1], rtol=1e-4, atol=1e-5)
