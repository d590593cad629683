"""Upload staging of the server: more requests in flight than it keeps uploads, small and large
ones mixed so that its ring wraps at different places (the largest that is staged, the smallest
that is not), and packed launches that gather many requests.  Every result is that of the same
steps made alone, bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def test_many_requests_equal_plain_steps():
    import torch

    from paper_1403_6126_amd import rt
    from paper_1403_6126_amd.serve import Server
    from paper_1403_6126_amd.solver import Solver, quadrature_for
    kinds = [(64, 8, 20), (1, 16, 5), (500, 30, 10), (18000, 8, 2), (19000, 8, 2), (6000, 24, 3)]
    wls = [W.request_workload(dict(id=i, seed=77_000 + i, ndim=1, shape=(n,), quad=("gl", na),
                                   nsteps=st), precision="mixed")
           for i, (n, na, st) in enumerate(kinds)]
    g = np.random.Generator(np.random.PCG64(5))
    order = [int(k) for k in g.choice(len(kinds), size=400, p=[.4, .2, .2, .08, .04, .08])]
    with Server(pool_bytes=2 << 30, max_active=512) as s:
        hs = [s.submit(wls[k]) for k in order]
        got = [s.wait(h) for h in hs]
    ref = []
    for wl in wls:
        mu, w = quadrature_for(wl.quad)
        sv = Solver(wl, mu=mu, w=w, I0=torch.zeros((len(w), wl.ncell), dtype=torch.float64,
                                                   device="cuda"))
        rt.rt_equilibrium_intensity(sv.ctx, sv.T, sv.I[0], torch.cuda.current_stream().cuda_stream)
        sv.step(wl.nsteps)
        ref.append(sv.state())
        sv.close()
    for i, (k, r) in enumerate(zip(order, got)):
        assert r["status"] == 0, (i, k, r["status"])
        for f in ("T", "E", "F", "totals"):
            assert np.array_equal(np.asarray(r[f]), ref[k][f]), (i, kinds[k], f)
