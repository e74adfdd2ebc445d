"""What a matrix with the quad form gets on first use (the row blocks of the
two separate passes, after fwd_wave was set to 0), while plans of several
contexts and threads share it."""
import threading

import numpy as np
import pytest
import scipy.sparse as sp

from gpu_util import banner, to_dev, to_host

pytestmark = pytest.mark.gpu

TABLE = [(2.0, 3.0, 1.0, 0.5), (0.0, 1.5, 0.0, 0.3)]


def _problem(nv=3003, nb=120, row=24, seed=3):
    rng = np.random.default_rng(seed)
    cols = np.concatenate([np.sort(rng.choice(nb, row, replace=False)) for _ in range(nv)])
    vals = (rng.integers(1, 129, nv * row) / 128.0).astype(np.float32)
    D = sp.csr_matrix((vals, (np.repeat(np.arange(nv), row), cols)), shape=(nv, nb))
    return D, rng.integers(0, 2, nv).astype(np.uint8), rng.uniform(0.0, 0.4, nb).astype(np.float32)


def _dose(ctx, D, storage="f32"):
    from paper_0908_4421_amd.imrt import Dose
    return Dose.from_csr(ctx, D.shape[0], D.shape[1], D.indptr.astype(np.int32), D.indices.astype(np.int32), D.data,
                         storage=storage)


def _plan(ctx, dose, sid):
    from paper_0908_4421_amd.imrt import Plan
    plan = Plan(ctx, dose)
    plan.set_structures(sid, 2)
    plan.set_penalties(TABLE)
    return plan


def test_contexts_and_threads_share_a_matrix():
    """One thread solves on the context that built the matrix while another,
    with a context of its own, makes the matrix's row blocks on first use."""
    import torch
    from paper_0908_4421_amd.imrt import Context
    D, sid, x0 = _problem(nv=20003)
    want = None
    for rep in range(6):
        banner(f"shared matrix {rep}")
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        c1 = Context(0, stream=s1.cuda_stream, one_read=2)
        dose = _dose(c1, D)
        c2 = Context(0, stream=s2.cuda_stream)
        c2.set_option("fwd_wave", 0)
        p1, p2 = _plan(c1, dose, sid), _plan(c2, dose, sid)
        torch.cuda.synchronize()
        x1, x2 = to_dev(x0), to_dev(x0)
        torch.cuda.synchronize()
        out, errors = {}, []

        def first():
            try:
                for _ in range(4):
                    x = x1.clone()
                    torch.cuda.synchronize()
                    res, tr = p1.solve(x, eps=1e-4, alpha=2.0, lambda0=2.0 ** -9, max_iter=40, fixed_iters=True,
                                       trace=True)
                    out.setdefault("solve", []).append((tr, to_host(x).tobytes()))
            except Exception as e:   # noqa: BLE001 (reported below)
                errors.append(e)

        def second():
            try:
                out["objective"] = p2.objective(x2)
                g, G = p2.gradient(x2)
                out["gradient"] = to_host(g).tobytes()
            except Exception as e:   # noqa: BLE001
                errors.append(e)

        threads = [threading.Thread(target=f) for f in (first, second)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not errors, errors
        assert all(r == out["solve"][0] for r in out["solve"])
        got = (out["solve"][0], out["objective"], out["gradient"])
        want = want or got
        assert got == want
