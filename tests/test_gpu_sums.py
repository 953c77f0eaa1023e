"""Nusselt numbers and diagnostics of more contexts than have a slot of pinned
memory for their sums (64): those with and without one, and those that take
over a slot given back, must agree to the last bit, and with the sums over the
fields to rounding."""
import numpy as np
import pytest

from paper_2211_03160_amd import lbm, workloads as W

pytestmark = pytest.mark.gpu


def _values(c):
    d = c.diagnostics()
    return (*c.nusselt(), *(d[k] for k in ("mass", "energy", "umax", "nu_vol", "re", "nonfinite")))


@pytest.mark.parametrize("dim,shape", [(2, (65, 33)), (2, (700, 600)), (3, (17, 9, 5))])
def test_slots(dim, shape):
    cfg = W.rayleigh_benard(dim, shape, ra=1e5, pr=0.71, storage="fp32")

    def make():
        c = lbm.Cavity(cfg)
        c.init(3, 1e-2)
        c.step(7)
        return c

    many = [make() for _ in range(66)]
    want = _values(many[0])
    assert all(_values(c) == want for c in many)
    for c in many[10:20]:
        c.close()
    assert all(_values(make()) == want for _ in range(3))
    rho, u, T = many[0].fields()
    n = rho.size
    # n additions of values of one sign, in FP64, in any order
    assert want[2] == pytest.approx(rho.sum(), rel=n * 2.0 ** -53)
    assert want[4] == pytest.approx(np.sqrt((u * u).sum(axis=0)).max(), rel=1e-15 * 4)
