"""Small lattices run a CG iteration as two launches of two hops each (blocks
of 2x2x2x2 boxes with their halo), larger ones, and a context that has chosen
its hop blocks, hop by hop: extents of 2 (a box that is its own neighbour), of
different sizes, the largest lattices of the rule and those past it, both
boundary signs, links that are and are not SU(3), solves and forces.  At kappa
= 0.05 the singular values of D lie in [0.59, 1.41], so X is off by at most
(1.41 / 0.59)^2 < 6 times a residual, 1e-13 each; the force is bilinear in two
such fields."""
import numpy as np
import pytest

import lgt_inputs as li
from gpu_common import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
KAPPA, TOL = 0.05, 1e-13


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp32"])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 4, 6, 2), (4, 2, 2, 10), (6, 10, 4, 12), (8, 8, 8, 8),
                                  (8, 8, 8, 10), (8, 8, 8, 12), (8, 8, 8, 14)])
def test_matches_single_hops(dims, precision, margin):
    import paper_2602_20516_amd as lgt
    U, phi = li.random_links(dims, 0.4, 91), to_dev(li.gaussian_spinor(dims, 92))
    for scale in (1.0, 1.001):  # 1.001: not SU(3), all nine components of a link are read
        Ud = to_dev(scale * U)
        for bc in (1, -1):
            lat = lgt.Lattice(dims, bc)
            prm = lgt.Params(tol=TOL, precision=precision)
            X, Y, st = lat.cg_solve(Ud, phi, KAPPA, prm)
            F = lat.fermion_force(Ud, phi, KAPPA, prm)[0]
            lat.set_hop_block_sites(64)
            Xr, Yr, ref = lat.cg_solve(Ud, phi, KAPPA, prm)
            Fr = lat.fermion_force(Ud, phi, KAPPA, prm)[0]
            name = f"{dims} {precision} bc {bc} links x {scale}"
            assert 0 < st["true_rel_residual"] <= TOL and abs(st["iters"] - ref["iters"]) <= 4 + ref["iters"] // 4, name
            margin(f"X {name}", rel_err(to_host(X), to_host(Xr)), 12 * TOL)
            margin(f"Y {name}", rel_err(to_host(Y), to_host(Yr)), 12 * TOL)
            margin(f"F {name}", rel_err(to_host(F), to_host(Fr)), 100 * TOL)
