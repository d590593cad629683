"""Rays through a vacuum with empty cells: the slope of an interface value is exactly zero beside
an empty cell, so such a cell sends nothing out.  After n steps every intensity is non-negative
(dt holds the outflow of a cell below its content, sum_d nu_d (2 - nu_d) < 1) and exactly zero in
every cell that no lit cell reaches in n upwind moves, whichever launch shape forms the faces:
alone in each cell or shared along x, periodic or beyond vacuum faces."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

V = (W.BC_VACUUM, W.BC_VACUUM)
P = (W.BC_PERIODIC, W.BC_PERIODIC)
CASES = [
    (3, (50, 23, 17), ("ls", 8), (P, P, P)),    # shared x faces, rows anywhere in a tile
    (3, (64, 17, 16), ("ls", 8), (V, P, V)),    # shared, every tile starts a row
    (3, (41, 21, 20), ("ls", 10), (V, V, V)),
    (2, (130, 128), ("ls", 12), (V, V, P)),     # twelve waves
    (3, (6, 55, 52), ("ls", 8), (V, V, V)),     # rows too short to share
    (3, (16, 16, 16), ("ls", 8), (P, V, V)),    # five angles a wave
    (3, (12, 11, 9), ("ls", 4), (V, P, P)),     # two angles a wave
    (1, (500,), ("gl", 400), (V, P, P)),        # in chunks
]


def _reach(lit, mu, bc, steps):
    """lit (nang, nz, ny, nx) grown by one upwind cell an axis and step."""
    for _ in range(steps):
        out = lit.copy()
        for m in range(len(mu)):
            for d in range(3):
                n = lit.shape[3 - d]
                if mu[m, d] == 0.0 or n == 1:
                    continue
                s = 1 if mu[m, d] > 0 else -1
                moved = np.roll(lit[m], s, axis=2 - d)
                if bc[d] is V:
                    edge = [slice(None)] * 3
                    edge[2 - d] = 0 if s > 0 else n - 1
                    moved[tuple(edge)] = False
                out[m] |= moved
        lit = out
    return lit


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("ndim,shape,quad,bc", CASES)
def test_empty_cells_stay_empty(ndim, shape, quad, bc, precision):
    from paper_1403_6126_amd.solver import Solver
    wl = W.small_case(ndim, shape, quad, seed=31, kappa_a=0.0, kappa_s=0.0, vscale=0.0, bc=bc,
                      courant=0.3)
    n = tuple(wl.n)
    g = np.random.Generator(np.random.PCG64(32))

    def init(mu):
        I = np.zeros((len(mu),) + n[::-1])
        for m in range(len(mu)):
            c = [g.integers(0, x) for x in n]
            box = tuple(slice(c[d], c[d] + max(1, n[d] // 3)) for d in (2, 1, 0))
            I[m][box] = g.uniform(0.5, 1.0, I[m][box].shape)
        return I.reshape(len(mu), -1)
    wl.init = init
    s = Solver(wl, precision=precision)
    print(f"case {wl.name} nang={s.nang} {precision}", flush=True)
    lit = s.current().cpu().numpy().reshape((s.nang,) + n[::-1]) != 0.0
    s.step(3)
    st = s.state()
    assert s.status() == 0
    mu = s.mu
    s.close()
    I = st["I"].reshape(lit.shape)
    assert I.min() >= 0.0, I.min()
    dark = ~_reach(lit, mu, bc, 3)
    assert dark.any() and not I[dark].any(), np.abs(I[dark]).max()
