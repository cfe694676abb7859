"""lgt_dslash reads the caller's fields in one launch, in blocks of 64
consecutive sites: lattices of less than one block, whole blocks, a ragged
last block, an extent of 2 (both neighbours the same site) and t-fastest
block groups, against the oracle; and a call whose output lies over its input
(through packed copies), against a separate output.  The two sides differ in
summation order only: 1e-13, as for the other deterministic FP64 maps."""
import numpy as np
import pytest

import lgt_inputs as li
from gpu_common import rel_err, to_dev, to_host
from oracle import dirac

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lgt():
    import paper_2602_20516_amd as m
    return m


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 2, 2, 4), (4, 4, 4, 4), (6, 2, 10, 4), (6, 6, 6, 6)])
@pytest.mark.parametrize("bc", [-1, 1])
@pytest.mark.parametrize("dagger", [False, True])
def test_against_the_oracle(lgt, margin, dims, bc, dagger):
    u, psi = li.random_links(dims, 0.6, 71), li.gaussian_spinor(dims, 72)
    lat = lgt.Lattice(dims, bc)
    U, P = to_dev(u), to_dev(psi)
    got = to_host(lat.dslash(U, P, 0.13, dagger))
    ref = (dirac.dslash_dag if dagger else dirac.dslash)(u, psi, 0.13, bc=bc)
    margin(f"D {dims} bc {bc} dagger {dagger}", rel_err(got, ref), 1e-13)
    over = P.clone()
    lat.dslash(U, over, 0.13, dagger, out=over)
    margin(f"D in place {dims} bc {bc} dagger {dagger}", rel_err(to_host(over), ref), 1e-13)
    if not dagger:
        over = P.clone()
        lgt.lgt_dslash_noalloc(dims, U, over, over, 0.13, fermion_bc=bc)
        margin(f"noalloc D in place {dims} bc {bc}", rel_err(to_host(over), ref), 1e-13)


def test_t_fastest_blocks_cover_every_site(lgt):
    """16x16x32x64 (t-fastest groups) repeats the 4^4 result at every site."""
    cell, dims = (4, 4, 4, 4), (16, 16, 32, 64)
    U, P = to_dev(li.random_links(cell, 0.5, 73)), to_dev(li.gaussian_spinor(cell, 74))
    small = lgt.Lattice(cell, 1).dslash(U, P, 0.12)
    rep = (16, 8, 4, 4)
    big = lgt.Lattice(dims, 1).dslash(U.repeat(rep + (1, 1, 1)), P.repeat(rep + (1, 1)), 0.12)
    assert np.array_equal(to_host(big), to_host(small.repeat(rep + (1, 1))))
