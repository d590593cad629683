"""The FP64 step in two calls, transport and source from its increment, at every launch shape of
the fused step: one to thirty angles per wave, one wave to twelve, chunks (more than 360
directions, staged in the output buffer), shared x faces or not.  Both paths run the same
arithmetic on the same increment, in instances of their own: the state agrees normwise to 1e-13
(a hundred roundings), the gas changes to 1e-13 of the sums that they are differences of, the
radiation's energy and momentum and the gas's own.  Without an increment (NULL) the source step
of a uniform static medium equals the fused one, whose increment is zero."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

FV = ((W.BC_FIXED, W.BC_VACUUM), (W.BC_COPY, W.BC_FIXED), (W.BC_VACUUM, W.BC_COPY))
CASES = [
    (1, (65,), ("gl", 2), None), (1, (500,), ("gl", 34), FV), (1, (16500,), ("gl", 6), None),
    (1, (500,), ("gl", 338), FV), (1, (16600,), ("gl", 340), None), (1, (500,), ("gl", 362), FV),
    (1, (16600,), ("gl", 400), FV), (2, (129, 131), ("ls", 12), FV), (2, (70, 30), ("ls", 16), FV),
    (3, (50, 23, 17), ("ls", 8), None), (3, (33, 26, 21), ("ls", 10), FV),
    (3, (41, 29, 30), ("ls", 14), FV), (3, (12, 11, 9), ("ls", 8), FV),
]


def _solver(ndim, shape, quad, bc, **kw):
    from paper_1403_6126_amd.solver import Solver
    wl = W.small_case(ndim, shape, quad, seed=17, kappa_a=3.0, kappa_s=2.0, vscale=0.03, bc=bc,
                      ghost_seed=6 if bc else None, rho_s=0.5, T_s=0.2, courant=0.3, **kw)
    wl.sigma_s[::3] *= 5.0              # both routings of the increment
    return wl, Solver(wl)


@pytest.mark.parametrize("ndim,shape,quad,bc", CASES)
def test_split_step_equals_fused(ndim, shape, quad, bc):
    wl, a = _solver(ndim, shape, quad, bc)
    print(f"case {wl.name} nang={a.nang}", flush=True)
    a.step(1)
    f = a.state()
    assert a.status() == 0
    a.close()
    wl, b = _solver(ndim, shape, quad, bc)
    b.source(b.transport())
    s = b.state()
    assert b.status() == 0
    b.close()
    scale = {k: np.abs(f[k]).max() for k in ("I", "T", "E", "F", "P")}
    gas = (wl.rho * wl.R / (wl.gamma - 1.0) * f["T"]).max()
    scale["dEgas"] = gas + wl.P * scale["E"]
    scale["dMom"] = (wl.rho * np.abs(wl.v)).max() + wl.P / wl.C * scale["E"]
    for k, den in scale.items():
        assert np.abs(s[k] - f[k]).max() <= 1e-13 * den, (k, np.abs(s[k] - f[k]).max() / den)
    assert np.allclose(s["totals"][[0, 1]], f["totals"][[0, 1]], rtol=1e-12)


@pytest.mark.parametrize("shape,quad", [((500,), ("gl", 400)), ((500,), ("gl", 34)),
                                        ((16600,), ("gl", 80))])
def test_source_without_an_increment(shape, quad):
    res = []
    for split in (False, True):
        wl, s = _solver(1, shape, quad, None)
        for x in (s.sa, s.ss, s.rho, s.T):
            x.fill_(1.25)
        s.v.zero_()
        s.I[0].fill_(0.3)               # uniform, out of equilibrium with T
        if split:
            s.source(None)
        else:
            s.step(1)
        res.append(s.state())
        assert s.status() == 0
        s.close()
    for k in ("I", "T", "E", "P"):
        assert np.abs(res[1][k] - res[0][k]).max() <= 1e-13 * np.abs(res[0][k]).max(), k
