"""The library's parameter map over the whole temperature range: the search
for the spinodal densities takes a coarse grid, and a fine one where the dip
of the pressure slope is narrower than that (T_r close to 1)."""
import pytest

import paper_1809_02390_amd as pkg
from oracle import hostmap as hm
from paper_1809_02390_amd import lbm as L


# dips of 60 % of the density range down to 0.3 % (0.99999: coarse step 0.5 %)
@pytest.mark.parametrize("tr", [0.3, 0.6, 0.8, 0.95, 0.999, 0.9999, 0.99999])
def test_coexistence_against_oracle(tr):
    """rho_g, rho_l to 1e-8: double rounding (1e-16) over the relative slope
    of the pressure at the coexistence densities (1 - T_r >= 1e-5), with a
    margin of 1e3."""
    d = L.lbm_derive(pkg.make_params(64, 64, tr=tr))
    rg, rl, _ = hm.maxwell(tr)
    assert d.rho_g == pytest.approx(rg, rel=1e-8) and d.rho_l == pytest.approx(rl, rel=1e-8)


def test_sigma_and_jacobian_follow_from_one_map():
    """lbm_sigma_paper and the default sigma of lbm_derive agree to the bit;
    the Jacobian's closed-form entries follow from the derived coefficients."""
    p = pkg.make_params(64, 64, tr=0.7, width=12.0)
    d = L.lbm_derive(p)
    assert d.sigma == L.lbm_sigma_paper(12.0, 0.7)
    jac = L.lbm_param_jacobian(p)
    assert jac[0][0] == d.g2 / d.sigma and jac[1][1] == -d.kp / d.width and jac[2][2] == d.tc
