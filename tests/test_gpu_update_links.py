"""Above 65536 sites a parity the FP64 residuals of a mixed solve's reliable
updates read two-row links if the links are SU(3): links that are, and links
that are not, whose solution the rebuilt third row would miss by 1e-3.  The
residual |phi - D^dag D X| is formed here from the operator on its own: below
the solve's 1e-11 and its own rounding, some 1e-15."""
import pytest

import lgt_inputs as li
from gpu_common import to_dev

pytestmark = pytest.mark.gpu
DIMS, KAPPA, TOL = (16, 16, 16, 36), 0.1, 1e-11


@pytest.mark.parametrize("precision", ["mixed_fp32", "mixed_bf16"])
@pytest.mark.parametrize("scale", [1.0, 1.001])
def test_solution_satisfies_the_operator(precision, scale, margin):
    import paper_2602_20516_amd as lgt
    lat = lgt.Lattice(DIMS)
    U, phi = to_dev(scale * li.random_links(DIMS, 0.3, 95)), to_dev(li.gaussian_spinor(DIMS, 96))
    X, Y, st = lat.cg_solve(U, phi, KAPPA, lgt.Params(tol=TOL, precision=precision))
    assert st["reliable_updates"] > 0
    r = phi - lat.dslash(U, lat.dslash(U, X, KAPPA), KAPPA, dagger=True)
    margin(f"residual {precision} links x {scale}", float(r.norm() / phi.norm()), 1.01 * TOL)
