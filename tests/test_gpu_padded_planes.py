"""Lattices whose packed planes are padded apart (more than 16384 sites per
parity, a multiple of 16384): what sums whole fields must not see the padding,
in particular that of a batched field, which moves with the number of
right-hand sides."""
import pytest

import lgt_inputs as li
from gpu_common import to_dev

pytestmark = pytest.mark.gpu
DIMS = (16, 16, 32, 64)  # 262144 sites per parity
CELL = (4, 4, 4, 4)


@pytest.fixture(scope="module")
def lgt():
    import paper_2602_20516_amd as m
    return m


def tiled(a):
    """A 4^4 field repeated over DIMS: exact copies of the small lattice's result."""
    lx, ly, lz, lt = (d // c for d, c in zip(DIMS, CELL))
    return a.repeat((lt, lz, ly, lx) + (1,) * (a.dim() - 4)).contiguous()


@pytest.mark.parametrize("sizes", [(3, 2, 1)])
def test_batches_of_falling_size_repeat_the_small_lattice(lgt, margin, sizes):
    """X of the repeated field is the repeated X: both solved to a true residual
    of 1e-12 (X within 1e-10 of each other at this kappa)."""
    small, big = lgt.Lattice(CELL, 1), lgt.Lattice(DIMS, 1)  # periodic: the repetition is a solution
    U = to_dev(li.random_links(CELL, 0.3, 901))
    prm = lgt.Params(precision="mixed_fp32", tol=1e-12)
    for n in sizes:
        kappas = [0.10 + 0.01 * k for k in range(n)]
        phis = [to_dev(li.gaussian_spinor(CELL, 910 + k)) for k in range(n)]
        xs, _, _ = small.cg_solve_batch(U, phis, kappas, prm)
        xb, _, st = big.cg_solve_batch(tiled(U), [tiled(p) for p in phis], kappas, prm)
        for k in range(n):
            assert st[k]["true_rel_residual"] <= 1e-12
            ref = tiled(xs[k])
            margin(f"padded batch of {n}, X {k}", float((xb[k] - ref).norm() / ref.norm()), 1e-10)


def test_multishift_after_another_number_of_shifts(lgt, margin):
    big, small = lgt.Lattice(DIMS, 1), lgt.Lattice(CELL, 1)
    U, phi = to_dev(li.random_links(CELL, 0.3, 901)), to_dev(li.gaussian_spinor(CELL, 921))
    prm = lgt.Params(tol=1e-12)
    for shifts in ([0.1, 1.0], [0.5]):
        xs, _ = small.cg_solve_multishift(U, phi, 0.12, shifts, prm)
        xb, st = big.cg_solve_multishift(tiled(U), tiled(phi), 0.12, shifts, prm)
        assert st["true_rel_residual"] <= 1e-12
        for a, b in zip(xb, xs):
            margin("padded multi-shift X", float((a - tiled(b)).norm() / tiled(b).norm()), 1e-10)
