"""The operator's and the preconditioner's passes at the edges of their launch shapes, against the
FP64 oracle.

The column passes hold tiles of columns (fewer columns than a tile on the smallest grids), the stress
pass pairs of x rows (one wavefront per pair up to 256 voxels, two at 512), the preconditioner's x
pass pairs of mirrored rows (own mirrors at ky, kz = 0 and n/2; butterflies from one to sixty-four
threads per row); in 3D the z passes carry the reductions of the passes before, in 2D there are no z
passes.  The grids put the shortest and the longest axis in every place.

Bars: FP64 1e-12 and FP32 1e-5 of the largest entry (a few hundred roundings of eps), as for the
other operator checks; the conjugate-gradient solve replayed for the same number of iterations
1e-10 in the 2-norm (rounding differences grow with the condition number, below 1e3 here)."""
import numpy as np
import pytest

import oracle
from paper_2211_08263_amd import newmark as nmb
from paper_2211_08263_amd import workloads as W

from gpu_common import dev, field3, random_problem, rel_l2, rel_max

pytestmark = pytest.mark.gpu

CASES = [(3, (8, 8, 8)), (3, (16, 8, 16)), (3, (512, 8, 8)), (3, (8, 512, 8)), (3, (8, 8, 512)), (3, (256, 8, 16)),
         (3, (128, 16, 8)), (2, (8, 8)), (2, (8, 512)), (2, (512, 8))]


@pytest.mark.parametrize("dim,n", CASES, ids=["x".join(map(str, n)) for _, n in CASES])
def test_passes_at_the_edges_of_their_shapes(dim, n):
    import torch
    pb = random_problem(dim, n, seed=11 + sum(n))
    op = oracle.OracleProblem.from_problem(pb)
    u = W.random_field(op.field_shape, seed=5)
    b = W.random_field(op.field_shape, seed=6)
    want = {"operator": field3(op.apply(u), dim), "precond": field3(op.precond(u), dim)}
    with nmb.newmark_init_problem(pb, nmb.Options(tol=1e-10)) as ctx:
        for dtype, bar in ((torch.float64, 1e-12), (torch.float32, 1e-5)):
            ud = dev(field3(u, dim), dtype)
            for name, fn in (("operator", nmb.apply_operator), ("precond", nmb.precond_apply)):
                out = torch.full_like(ud, 7.0)
                fn(ctx, ud, out)
                torch.cuda.synchronize()
                err = rel_max(out.double().cpu().numpy(), want[name])
                print(f"{name} {n} {dtype}: {err:.2e}", flush=True)
                assert err <= bar
        x = torch.zeros(3 * ctx.N, dtype=torch.float64, device="cuda")
        it, rel = nmb.pcg_solve(ctx, dev(field3(b, dim)).reshape(-1), x, tol=1e-10)
        assert 1 < it < 300 and rel <= 1e-10
        got = x.cpu().numpy().reshape(3, -1)
    ref, _, _ = op.pcg(b, fixed_iters=it)
    err = rel_l2(got, field3(ref, dim))
    print(f"pcg {n}: {it} iterations, {err:.2e}", flush=True)
    assert err <= 1e-10


@pytest.mark.parametrize("dim,n", CASES[:3] + CASES[5:8], ids=["x".join(map(str, n)) for _, n in CASES[:3] + CASES[5:8]])
def test_residual_from_the_last_pass(dim, n):
    """The operator's last pass forms b - A x and its norm: a solve of no iterations reports
    |P (b - A x)| over its reference norm, |b| or, with the Gamma voxels masked, |P (b - A x_Gamma)|.
    Norms of sums of some ten FP64 roundings an entry: 1e-12."""
    import dataclasses
    pb = random_problem(dim, n, seed=2 + sum(n))
    N = int(np.prod(n))
    g = np.sort(np.random.default_rng(5).choice(N, size=N // 5, replace=False)).astype(np.int64)
    pb = dataclasses.replace(pb, gamma_idx=g)
    op = oracle.OracleProblem.from_problem(pb)
    x, b = W.random_field(op.field_shape, seed=8), W.random_field(op.field_shape, seed=9)
    free = np.ones(N, bool)
    free[g] = False
    norm = lambda f, keep: np.linalg.norm(np.where(keep, f.reshape(f.shape[0], -1), 0.0))
    xg = np.where(free, 0.0, x.reshape(x.shape[0], -1)).reshape(x.shape)
    r = b - op.apply(x)
    want = {False: norm(r, True) / norm(b, True), True: norm(r, free) / norm(b - op.apply(xg), free)}
    with nmb.newmark_init_problem(pb, nmb.Options()) as ctx:
        for masked, ref in want.items():
            xd = dev(field3(x, dim)).reshape(-1)
            it, rel = nmb.pcg_solve(ctx, dev(field3(b, dim)).reshape(-1), xd, masked=masked, fixed_iters=0)
            print(f"residual {n} masked {masked}: {rel:.15e} want {ref:.15e}", flush=True)
            assert it == 0 and abs(rel - ref) <= 1e-12 * ref


EXPLICIT_CASES = [(3, (8, 8, 8), False), (3, (16, 128, 8), True), (3, (8, 256, 16), False), (3, (8, 512, 8), True),
                  (2, (8, 64), False), (2, (64, 16), True)]


@pytest.mark.parametrize("dim,n,per_point", EXPLICIT_CASES, ids=["x".join(map(str, n)) for _, n, _ in EXPLICIT_CASES])
def test_explicit_batch_is_its_steps_one_by_one(dim, n, per_point):
    """Within a batch of explicit steps the y passes of a step's end and of the next one's start are one
    pass that keeps the half step's velocity instead of the acceleration; a batch of one has them
    apart.  Five steps, both ways: the same sums in another order, a few roundings a step (1e-13 of
    the largest entry), grown by a stable scheme at most linearly."""
    import dataclasses
    pb = random_problem(dim, n, seed=3 + sum(n))
    N = int(np.prod(n))
    g = np.sort(np.random.default_rng(7).choice(N, size=min(37, N // 4), replace=False)).astype(np.int64)
    xi = [np.pi * (m - 2) / l for m, l in zip(pb.n, pb.L) if m > 1]
    dt = 0.3 * 2.0 / np.sqrt(6 * np.abs(pb.C21).max() * sum(x * x for x in xi) / np.min(pb.rho))
    pb = dataclasses.replace(pb, gamma_idx=g, dt=dt, beta=0.0, gamma_nm=0.5)
    rows = np.random.default_rng(8).standard_normal((5, dim * (g.size if per_point else 1)))
    got = []
    for batches in ([5], [1] * 5):
        with nmb.newmark_init_problem(pb, nmb.Options()) as ctx:
            u0 = np.random.default_rng(9).standard_normal((3, 3 * ctx.N))
            u0[:, dim * ctx.N:] = 0.0
            nmb.set_state(ctx, *u0, 0)
            k = 0
            for nb in batches:
                nmb.explicit_step(ctx, rows[k:k + nb], per_point=per_point, n_steps=nb)
                k += nb
            st = nmb.get_state(ctx)
            got.append([st[q].copy() for q in ("u", "v", "a", "F")])
    for q, x, y in zip("uvaF", *got):
        err = rel_max(x, y)
        print(f"explicit {n} {q}: {err:.2e}", flush=True)
        assert np.isfinite(x).all() and err <= 1e-12


@pytest.mark.parametrize("which", [0, 1])
def test_profile_fills_every_entry(which):
    """The nine durations that nm_profile_passes asks room for: its passes', then zeros, so that a sum
    over them is the chain whatever its number of passes."""
    import ctypes as C
    import torch
    pb = random_problem(3, (16, 16, 16))
    with nmb.newmark_init_problem(pb, nmb.Options()) as ctx:
        u = torch.zeros(3 * ctx.N, dtype=torch.float64, device="cuda")
        out = torch.zeros_like(u)
        ms = (C.c_double * 9)(*[float("nan")] * 9)
        ctx.check(nmb.load_library().nm_profile_passes(ctx.handle, which, u.data_ptr(), out.data_ptr(), nmb.NM_FP64, 3, ms))
    n = len(nmb.OPERATOR_PASSES if which == 0 else nmb.PRECOND_PASSES)
    assert all(0 < t < 1e3 for t in ms[:n]) and all(t == 0 for t in ms[n:])


@pytest.mark.parametrize("dim,n", [(3, (16, 16, 16)), (3, (32, 8, 8)), (3, (128, 64, 128)), (2, (64, 32))],
                         ids=["16x16x16", "32x8x8", "128x64x128", "64x32"])
def test_fp32_preconditioner_on_a_nearly_incompressible_medium(dim, n):
    """The multiplier's inverse is formed in FP64 for FP32 fields too.  At a Poisson ratio of 0.49999 its
    cofactors cancel by the ratio of the moduli, 5e4: in FP32 that would leave 5e4 eps = 3e-3 of
    them.  Bar: 1e-5 of the largest entry, as for the other FP32 checks here."""
    import dataclasses
    import torch
    pb = random_problem(dim, n, seed=8, dt=2.0)
    C21 = np.stack([W.voigt_to21(W.isotropic_voigt66(1.0, 0.49999))] * 3)
    pb = dataclasses.replace(pb, C21=C21)
    N = int(np.prod(n))
    nn = tuple(n) + (1,) * (3 - len(n))
    r = W.random_field((dim, nn[2], nn[1], nn[0]), seed=3).astype(np.float32).astype(np.float64)
    with nmb.newmark_init_problem(pb, nmb.Options()) as ctx:
        got = {}
        for dtype in (torch.float64, torch.float32):
            z = torch.empty(3, N, dtype=dtype, device="cuda")
            rd = dev(field3(r, dim), dtype)
            torch.cuda.synchronize()
            nmb.precond_apply(ctx, rd, z)
            torch.cuda.synchronize()
            got[dtype] = z.double().cpu().numpy()
    want = got[torch.float64]
    if N <= 1 << 12:
        want = field3(oracle.OracleProblem.from_problem(pb).precond(r), dim)
    err = rel_max(got[torch.float32], want)
    print(f"precond nu 0.49999 {n}: {err:.2e}", flush=True)
    assert err <= 1e-5
