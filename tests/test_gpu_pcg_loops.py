"""The conjugate-gradient loop's own control: iterations run in batches on the device, and the passes
launched behind the iteration that converges do nothing.

A solve to a tolerance that took k iterations, with passes launched past the k-th, has the iterate of
the solve of k iterations bit for bit (the same kernels on the same data), in 3D, where a z pass
counts the iterations and raises the stop flag, and in 2D, where the preconditioner's x pass does.
Grids on both sides of the launch rules (a wavefront a block, 256 threads)."""
import numpy as np
import pytest

from paper_2211_08263_amd import newmark as nmb
from paper_2211_08263_amd import workloads as W

from gpu_common import dev, field3, random_problem

pytestmark = pytest.mark.gpu

GRIDS = [(3, (8, 8, 8)), (3, (32, 16, 64)), (3, (128, 64, 128)), (2, (8, 8)), (2, (64, 128)), (2, (512, 512))]


@pytest.mark.parametrize("dim,n", GRIDS, ids=["x".join(map(str, n)) for _, n in GRIDS])
def test_passes_behind_the_last_iteration_do_nothing(dim, n):
    import torch
    pb = random_problem(dim, n, seed=31 + sum(n), aniso=False)
    nn = tuple(n) + (1,) * (3 - len(n))
    shape = (dim, nn[2], nn[1], nn[0])
    b = dev(field3(W.random_field(shape, seed=3), dim)).reshape(-1)
    x0 = dev(field3(W.random_field(shape, seed=4), dim)).reshape(-1)
    with nmb.newmark_init_problem(pb, nmb.Options()) as ctx:
        for tol in (1e-3, 1e-6, 1e-9, 1e-10):
            x = x0.clone()
            k, rel = nmb.pcg_solve(ctx, b, x, tol=tol)
            y = x0.clone()
            kf, relf = nmb.pcg_solve(ctx, b, y, tol=tol, fixed_iters=k)
            print(f"{n} tol {tol}: {k} iterations, {rel:.2e}", flush=True)
            assert kf == k and relf == rel <= tol
            assert torch.equal(x, y) and np.isfinite(rel)
