"""FP32-mixed steps with ghosts on every axis: angle tables and position-dependent tables on all
six faces, vacuum and copy faces, one to four angle groups a wave and more waves than four, rows
that start anywhere in a tile, axes of one and two cells (both faces in one stencil), fused,
second order, and feedback.  Against the FP64 oracle within the bound of the mixed form (1e-5)."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

F, V, C = W.BC_FIXED, W.BC_VACUUM, W.BC_COPY
P = (W.BC_PERIODIC, W.BC_PERIODIC)
CASES = [
    (1, (67,), ("gl", 8), ((F, V), P, P), {}),
    (1, (1,), ("gl", 12), ((F, F), P, P), {}),
    (2, (2, 70), ("ls", 6), ((F, C), (V, F), P), {}),
    (3, (13, 9, 7), ("ls", 8), ((F, F),) * 3, {}),
    (3, (13, 9, 7), ("ls", 8), ((V, V), (C, V), (V, F)), dict(second_order=True)),
    (3, (9, 1, 11), ("ls", 10), ((V, F), (F, V), (F, F)), {}),
    (3, (7, 11, 5), ("ls", 10), ((F, V), P, (C, F)), dict(feedback=True)),
    (3, (66, 5, 4), ("ls", 12), ((F, F), (F, V), (V, F)), {}),
    (2, (21, 13), ("ls", 16), ((V, F), (F, F), P), dict(second_order=True)),
]


def _nerr(a, b):
    den = np.abs(b).max()
    return float(np.abs(a - b).max() / den) if den > 0 else float(np.abs(a - b).max())


@pytest.mark.parametrize("tables", ["angle", "place"])
@pytest.mark.parametrize("ndim,shape,quad,bc,opt", CASES)
def test_ghosts_of_every_kind(ndim, shape, quad, bc, opt, tables):
    import oracle

    from paper_1403_6126_amd.solver import Solver
    wl = W.small_case(ndim, shape, quad, seed=91 + ndim, nsteps=3, kappa_a=3.0, kappa_s=2.0,
                      vscale=0.03, bc=bc, ghost_seed=8, rho_s=0.5, T_s=0.2, courant=0.3)
    if tables == "place":
        n = tuple(wl.n)

        def ghost_face(mu):
            g = np.random.Generator(np.random.PCG64(9))
            return {(d, s): g.uniform(0.0, 0.2, (np.asarray(mu).shape[0], wl.ncell // n[d]))
                    for d in range(ndim) for s in range(2) if bc[d][s] == F}
        wl.ghost_face = ghost_face
    ref = oracle.run(wl, nsteps=3, **opt)
    s = Solver(wl, precision="mixed", **opt)
    print(f"case {wl.name} nang={s.nang} {opt} {tables}", flush=True)
    s.step(3)
    st = s.state()
    status = s.status()
    s.close()
    assert status == 0
    errs = {k: _nerr(st[k], r) for k, r in (("I", ref.I), ("T", ref.T), ("E", ref.E),
                                            ("F", ref.F), ("P", ref.Pr))}
    print("   errors", errs, flush=True)
    assert max(errs.values()) <= 1e-5, errs
