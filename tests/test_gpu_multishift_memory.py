"""Multi-shift solves and rational forces with little device memory left: the
ring of residuals, which only saves traffic, must not take what the rest of
the call needs.  32^3x32 with one shift needs 16 half spinors beside the
caller's fields (4 of the solve, 8 in four full fields, 4 of two-row links),
the force 6 more (a gauge field), and the whole ring 7 more than either.  The
results are those of a run with all the memory, bit for bit."""
import gc

import pytest

import lgt_inputs as li
from gpu_common import to_dev

pytestmark = pytest.mark.gpu
CELL, REP, DIMS = (4, 4, 4, 4), (8, 8, 8, 8), (32, 32, 32, 32)


def _fields():
    U, phi = to_dev(li.random_links(CELL, 0.3, 41)), to_dev(li.gaussian_spinor(CELL, 42))
    return U.repeat(REP + (1, 1, 1)).contiguous(), phi.repeat(REP + (1, 1)).contiguous()


def _leave(free):
    """Tensors that take all device memory but `free` bytes."""
    import torch
    torch.cuda.empty_cache()
    held, chunk = [], 8 << 30
    while (left := torch.cuda.mem_get_info()[0] - free) > (16 << 20):
        held.append(torch.empty(min(left, chunk), dtype=torch.uint8, device="cuda"))
    return held


@pytest.mark.parametrize("force", [False, True])
def test_fits_with_little_memory(force):
    import torch
    import paper_2602_20516_amd as lgt
    half = 12 * 16 * (32 ** 4 // 2)
    U, phi = _fields()
    out = torch.empty_like(U) if force else None

    def run(lat):
        prm = lgt.Params(tol=1e-6, max_iter=60)
        if force:
            F, S, st = lat.rational_force_eo(U, phi, 0.1, [0.5], [1.0], 0.2, prm, out=out)
            return F, S, st["true_rel_residual"]
        (X,), st = lat.cg_solve_multishift(U, phi, 0.1, [0.5], prm)
        return X, st["true_rel_residual"]

    lat = lgt.Lattice(DIMS)
    ref = run(lat)
    ref = (ref[0].clone(),) + ref[1:]
    lat.close()
    gc.collect()
    lat = lgt.Lattice(DIMS)
    # 3 to spare; the solve's output is a torch tensor of two halves
    held = _leave((16 + 3 + (6 if force else 2)) * half)
    try:
        got = run(lat)
    finally:
        del held
        torch.cuda.empty_cache()
    assert torch.equal(got[0], ref[0]) and got[1:] == ref[1:]
    lat.close()
