"""The shifts' vectors are carried through up to eight iterations at a time,
and a rational force takes its terms in groups whose size depends on their
number (fields in scratch below three terms): solves that stop at and beside
the ends of a group, and forces of 1 to 25 terms against the sum of one-term
forces.  Solves to 1e-13: X and the forces agree to 1e-11."""
import numpy as np
import pytest

import lgt_inputs as li
from gpu_common import rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu
DIMS = (4, 4, 4, 6)
KAPPA = 0.12


@pytest.fixture(scope="module")
def f():
    import paper_2602_20516_amd as lgt
    lat = lgt.Lattice(DIMS)
    return lgt, lat, to_dev(li.random_links(DIMS, 0.4, 81)), to_dev(li.gaussian_spinor(DIMS, 82))


@pytest.mark.parametrize("tol", [1e-1, 1e-2, 1e-3, 1e-4, 1e-5, 1e-6, 1e-7, 1e-8, 1e-9, 1e-13])
def test_every_stopping_place(f, margin, tol):
    lgt, lat, U, phi = f
    shifts = [0.0, 0.03, 0.7, 5.0, 40.0]
    X, st = lat.cg_solve_multishift(U, phi, KAPPA, shifts, lgt.Params(tol=tol))
    assert 0 < st["true_rel_residual"] <= tol
    ref, _ = lat.cg_solve_multishift(U, phi, KAPPA, shifts, lgt.Params(tol=1e-14))
    for x, r, s in zip(X, ref, shifts):
        # the residual bounds the error through the operator's smallest eigenvalue, above 0.05 here
        margin(f"X at tol {tol} shift {s}", rel_err(to_host(x), to_host(r)), 50 * tol + 1e-12)


@pytest.mark.parametrize("n", [1, 2, 3, 5, 6, 9, 24, 25])
@pytest.mark.parametrize("mode", ["force", "grad", "momentum"])
def test_force_of_n_terms_is_the_sum_of_its_terms(f, margin, n, mode):
    lgt, lat, U, phi = f
    shifts = [0.01 * 1.5 ** k for k in range(n)]
    res = [(-1.0) ** k * (1.0 + 0.1 * k) for k in range(n)]
    prm = lgt.Params(tol=1e-13)
    start = to_dev(li.random_momenta(DIMS, 83))
    got, S, _ = lat.rational_force_eo(U, phi, KAPPA, shifts, res, 0.3, prm, mode=mode, dt=0.1, out=start.clone())
    ref, s_ref = 0, 0.0
    for k in range(n):
        t, s, _ = lat.rational_force_eo(U, phi, KAPPA, [shifts[k]], [res[k]], 0.0, prm,
                                        mode="grad" if mode == "grad" else "force")
        ref, s_ref = ref + t, s_ref + s
    odd = (np.indices(tuple(reversed(DIMS))).sum(0) % 2 == 1)[..., None, None]
    s_ref += 0.3 * float((np.abs(to_host(phi) * odd) ** 2).sum())
    if mode == "momentum":
        ref = start - 0.1 * ref
    margin(f"{n} terms {mode}", rel_err(to_host(got), to_host(ref)), 1e-11)
    margin(f"{n} terms action", abs(S - s_ref) / abs(s_ref), 1e-11)
