"""Mixed solves whose FP32 recursion breaks down at once, again after every
restart: 1 - kappa^2 H_oe H_eo overflows FP32 (kappa^2 = 1e40), or its square
does (kappa^2 = 1e20).  They end in an error, at the latest at the iteration
cap, and leave nothing behind: the context's next solve has the bits of a new
context's.  Lattices of each form of the iteration: two launches (4^4), four
with 32-site and with 64-site blocks (10x8^3), and the separate step
kernel (BF16)."""
import numpy as np
import pytest

import lgt_inputs as li
from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["mixed_fp32", "mixed_bf16"])
@pytest.mark.parametrize("dims,sites", [((4, 4, 4, 4), 0), ((10, 8, 8, 8), 0), ((10, 8, 8, 8), 64)])
def test_breakdown_ends_and_leaves_nothing(dims, sites, precision):
    import paper_2602_20516_amd as lgt
    U, phi = to_dev(li.random_links(dims, 0.4, 21)), to_dev(li.gaussian_spinor(dims, 22))
    lat, new = lgt.Lattice(dims), lgt.Lattice(dims)
    for x in (lat, new):
        x.set_hop_block_sites(sites)
    with pytest.raises(lgt.LGTNonFinite):
        lat.cg_solve(U, phi, 1e20, lgt.Params(precision=precision, tol=1e-10))
    with pytest.raises(lgt.LGTError):
        lat.cg_solve(U, phi, 1e10, lgt.Params(precision=precision, tol=1e-10, max_iter=20))
    prm = lgt.Params(precision=precision, tol=1e-10)
    X, Y, _ = lat.cg_solve(U, phi, 0.12, prm)
    Xn, Yn, _ = new.cg_solve(U, phi, 0.12, prm)
    assert np.array_equal(to_host(X), to_host(Xn)) and np.array_equal(to_host(Y), to_host(Yn))
