"""The operator through packed copies, the route of a call whose output lies
over its input: both block shapes and both block orders of the hop kernel on
their own (lgt_dslash with a separate output has a kernel without them),
against the oracle; and lgt_dslash_noalloc's scratch at its largest lattice,
then on a smaller one that finds it filled, against lgt_dslash bit for bit.
The sides differ from the oracle in summation order only: 1e-13, as for the
other deterministic FP64 maps."""
import numpy as np
import pytest

import lgt_inputs as li
from gpu_common import max_rel_err, rel_err, to_dev, to_host
from oracle import dirac, eo

pytestmark = pytest.mark.gpu

# (sites per block, order of the 64-site blocks) and lattices: below one block,
# ragged last blocks, whole blocks, an extent of 2, t-fastest groups of 2, 8 and 4
SHAPES = [(32, 0), (64, 1), (64, 2)]
DIMS = [(2, 2, 2, 4), (6, 2, 10, 4), (6, 6, 6, 4), (10, 6, 6, 6), (8, 4, 6, 4), (8, 4, 8, 6), (16, 4, 4, 8),
        (8, 8, 8, 12)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dims", DIMS)
def test_both_shapes_in_place_and_schur(dims, shape, margin):
    import paper_2602_20516_amd as lgt
    u, psi = li.random_links(dims, 0.5, 501), li.gaussian_spinor(dims, 502)
    U, P = to_dev(u), to_dev(psi)
    lat = lgt.Lattice(dims)
    lat.set_hop_block_sites(shape[0])
    lat.set_hop_block_order(shape[1])
    for dag in (False, True):
        over = P.clone()
        got = to_host(lat.dslash(U, over, 0.13, dag, out=over))
        ref = (dirac.dslash_dag if dag else dirac.dslash)(u, psi, 0.13)
        margin("in place rel_err", rel_err(got, ref), 1e-13)
        margin("in place max_rel_err", max_rel_err(got, ref), 1e-13)
        odd = eo.parity_mask(dims, 1)
        ref = odd * (eo.schur_dag if dag else eo.schur)(u, odd * psi, 0.13)
        margin("Schur rel_err", rel_err(odd * to_host(lat.schur_dslash(U, P, 0.13, dag)), ref), 1e-13)


@pytest.mark.parametrize("dagger", [False, True])
def test_noalloc_scratch_large_then_small(dagger, margin):
    import paper_2602_20516_amd as lgt
    for dims, eps, kappa, bc in [((16, 16, 16, 16), 0.3, 0.125, -1), ((6, 4, 4, 8), 0.5, 0.13, +1)]:
        u, psi = li.random_links(dims, eps, 611), li.gaussian_spinor(dims, 612)
        U, P = to_dev(u), to_dev(psi)
        over, ctx = P.clone(), P.clone()
        lgt.lgt_dslash_noalloc(dims, U, over, over, kappa, dagger, fermion_bc=bc)
        lgt.Lattice(dims, fermion_bc=bc).dslash(U, ctx, kappa, dagger, out=ctx)
        assert np.array_equal(to_host(over), to_host(ctx)), f"{dims}: differs from lgt_dslash"
        ref = (dirac.dslash_dag if dagger else dirac.dslash)(u, psi, kappa, bc=bc)
        margin(f"noalloc D in place {dims}", rel_err(to_host(over), ref), 1e-13)
