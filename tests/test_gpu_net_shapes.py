"""The convolution's block depth and the weight gradient's reduction at the edges of their rules.

Blocks cover 16 planes on large grids and fewer, down to 2, on small ones; the reduction sums up to
1024 partial slots in sixteen interleaved groups (fewer slots than groups on the smallest grid, a
number that the groups do not divide, and all 1024 on the largest here).  Against the FP64 oracle on
BF16-valued inputs; bars as for the other checks of these kernels (1e-5 forward and backward-data,
1e-4 weight gradient: FP32 accumulation of up to 27 * 32 and of N products)."""
import numpy as np
import pytest

import oracle
from paper_2211_08263_amd import newmark as nmb

from test_gpu_net import bf16_bits, bf16_val, cf_to_cl, cl_to_cf, dev_u16

pytestmark = pytest.mark.gpu


# voxels / 16 = 4, 32, 160 and 2048 tiles; block depths 2 and 4
@pytest.mark.parametrize("n", [(16, 2, 2), (16, 8, 4), (16, 16, 8), (64, 64, 8)])
def test_layer_kernels_at_the_edges_of_their_launches(n):
    import torch
    rng = np.random.default_rng(sum(n))
    N = n[0] * n[1] * n[2]
    for cinp, cin, cout in ((32, 31, 16), (16, 16, 3)):
        x = bf16_val(rng.standard_normal((N, cinp)))
        dy = np.zeros((N, 16))
        dy[:, :cout] = bf16_val(rng.standard_normal((N, cout)))
        w = rng.standard_normal((cout, cin, 27)).astype(np.float32) * 0.3
        wv = bf16_val(w).reshape(cout, cin, 3, 3, 3)
        out = torch.zeros(N * 16, dtype=torch.float32, device="cuda")
        nmb.conv3d_bf16(0, n, cinp, cin, cout, x=dev_u16(bf16_bits(x)), w=w, out=out)
        got = out.cpu().numpy().reshape(N, 16)[:, :cout]
        want = cf_to_cl(oracle.conv3d_fwd(cl_to_cf(x, n, cin), wv, np.zeros(cout), n))
        assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()
        if cinp == 16:
            nmb.conv3d_bf16(1, n, 16, cin, cout, w=w, dy=dev_u16(bf16_bits(dy)), out=out)
            got = out.cpu().numpy().reshape(N, 16)[:, :cin]
            want = cf_to_cl(oracle.conv3d_bwd_data(cl_to_cf(dy, n, cout), wv, n))
            assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()
        dw, db = nmb.conv3d_bf16(2, n, cinp, cin, cout, x=dev_u16(bf16_bits(x)), dy=dev_u16(bf16_bits(dy)))
        wdw, wdb = oracle.conv3d_bwd_weight(cl_to_cf(x, n, cin), cl_to_cf(dy, n, cout), cin, cout, n)
        assert np.abs(dw - wdw.reshape(cout, cin, 27)).max() <= 1e-4 * np.abs(wdw).max()
        assert np.abs(db - wdb).max() <= 1e-4 * np.abs(wdb).max()


# one voxel along y, along z, along both: a neighbour across the wrap is the voxel itself
@pytest.mark.parametrize("n", [(32, 1, 4), (64, 1, 8), (32, 1, 2), (16, 1, 2), (32, 4, 1), (32, 1, 1), (16, 1, 1)])
def test_layer_kernels_on_axes_of_one_voxel(n):
    test_layer_kernels_at_the_edges_of_their_launches(n)
