"""A mixed solve has the same bits whatever else holds device memory: 16^3x48,
past the volume where the CG step is a launch of its own, with all of it and
with less than a quarter of it free."""
import numpy as np
import pytest

import lgt_inputs as li
from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


def test_same_bits_with_little_memory_free():
    import torch
    import paper_2602_20516_amd as lgt
    cell, rep, dims = (4, 4, 4, 6), (8, 4, 4, 4), (16, 16, 16, 48)
    U = to_dev(li.random_links(cell, 0.3, 51)).repeat(rep + (1, 1, 1)).contiguous()
    phi = to_dev(np.tile(li.gaussian_spinor(cell, 52), rep + (1, 1)) + 0.1 * li.gaussian_spinor(dims, 53))
    prm = lgt.Params(precision="mixed_fp32", tol=1e-9)

    def run():
        lat = lgt.Lattice(dims)
        X, _, st = lat.cg_solve(U, phi, 0.1, prm)
        lat.close()
        return to_host(X), st["iters"]

    X, n = run()
    torch.cuda.empty_cache()
    free, total = torch.cuda.mem_get_info()
    held = [torch.empty(8 << 30, dtype=torch.uint8, device="cuda") for _ in range((free - total // 5) >> 33)]
    try:
        Xh, nh = run()
    finally:
        del held
        torch.cuda.empty_cache()
    assert n == nh and np.array_equal(X, Xh)
