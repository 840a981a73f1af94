"""A change of units by powers of two leaves a mixed-precision step's solution as it is.

Lengths and times 2^28 times and displacements 2^-34 times as large: the operator, its fields and the
residuals keep their exponents apart from the common 2^-34, and every FP32 number of the step stays
normal (the smallest, the divergence of the stresses, is of order 2^-90 before convergence takes 2^-17
off it).  The elastic energy of a direction alone, strain times stress = 2^-124, leaves FP32's range:
its products belong in FP64, like every other product that a step length is made of.

Bar: both steps end at a residual of 1e-9, so they differ by 1e-9 times the condition number (below
1e3): 1e-6; the same iteration to rounding, so the FP32 iterations differ by one a sweep at most."""
import dataclasses

import numpy as np
import pytest

from paper_2211_08263_amd import newmark as nmb

from gpu_common import random_problem, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,n", [(3, (16, 16, 16)), (3, (64, 32, 128)), (2, (64, 64))],
                         ids=["16x16x16", "64x32x128", "64x64"])
def test_mixed_step_in_other_units(dim, n):
    pb = random_problem(dim, n, seed=5, aniso=False)
    N = int(np.prod(n))
    g = np.sort(np.random.default_rng(6).choice(N, size=N // 20, replace=False)).astype(np.int64)
    rng = np.random.default_rng(7)
    U, u0, v0 = rng.standard_normal((g.size, dim)), rng.standard_normal((dim, N)), rng.standard_normal((dim, N))
    got = []
    for length, amp in ((1.0, 1.0), (2.0 ** 28, 2.0 ** -34)):
        q = dataclasses.replace(pb, gamma_idx=g, L=tuple(length * x for x in pb.L), dt=length * pb.dt)
        opts = nmb.Options(precision=nmb.PREC_MIXED, tol=1e-9, true_residual=1, max_iter=300)
        with nmb.newmark_init_problem(q, opts, u0=amp * u0, v0=amp / length * v0) as ctx:
            st = nmb.newmark_step(ctx, amp * U, per_point=True)
            got.append((nmb.get_state(ctx)["u"] / amp, st))
    (u, a), (w, b) = got
    err = rel_l2(w, u)
    print(f"units {n}: {a['inner_iters']} and {b['inner_iters']} FP32 iterations, difference {err:.2e}", flush=True)
    assert b["relres"] <= 1e-9 and err <= 1e-6
    assert abs(a["inner_iters"] - b["inner_iters"]) <= max(a["sweeps"], b["sweeps"])
