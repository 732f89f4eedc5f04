"""RMS norm and the chain's two residual steps at the edges of their kernels'
ranges: row lengths around the register tiles, rows that are not whole 16-byte
pieces, one row and more rows than the small-batch rule takes, and magnitudes
whose mean square leaves the fp32 range."""

import numpy as np
import pytest

from oracle import routing as o_routing

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    from paper_2609_18063_amd import binding
    binding.lib()
    return torch


@pytest.mark.parametrize("T", [1, 513])
@pytest.mark.parametrize("d", [1, 3, 4, 250, 252, 1024, 4096, 4100, 8192, 8196])
def test_rmsnorm_bit_exact(torch_cuda, T, d):
    from paper_2609_18063_amd import binding as B
    torch = torch_cuda
    xi = np.random.default_rng(d + T).standard_normal((T, d)).astype(np.float32)
    if T > 1:
        xi[1] *= 1e25                            # the mean square is past the largest fp32
        xi[2] *= 1e-25
        xi[3] = 0.0
    x = torch.empty(T, d, dtype=torch.float16, device="cuda")
    B.rmsnorm_f16(torch.from_numpy(xi).cuda(), x)
    got = x.cpu().numpy()
    for t in ({0, 1, 2, 3, T - 1} if T > 1 else {0}):
        assert np.array_equal(got[t].view(np.uint16), o_routing.rms_norm_f16(xi[t]).view(np.uint16)), (t, d)


@pytest.mark.parametrize("d", [1, 100, 1025, 2048, 2049, 4097, 8192])
def test_chain_steps(torch_cuda, d):
    from paper_2609_18063_amd import binding as B
    torch = torch_cuda
    g = np.random.default_rng(d)
    xi, r0 = (g.standard_normal(d).astype(np.float32) for _ in range(2))
    mix, perm = (g.standard_normal(d) * 0.5).astype(np.float16), g.permutation(d).astype(np.int32)
    r = torch.from_numpy(r0.copy()).cuda()
    B.chain_token_start(torch.from_numpy(xi).cuda(), r)
    v = r0.astype(np.float64)
    ref = (xi + v / np.sqrt(np.mean(v * v) + 1e-6)).astype(np.float32)
    r1 = r.cpu().numpy()
    # one rounding to fp32; the float64 norm agrees to a few of its ulps, so a
    # rounding tie may fall the other way
    assert np.all(np.abs(r1.view(np.int32) - ref.view(np.int32)) <= 1)
    x = torch.empty(d, dtype=torch.float16, device="cuda")
    B.chain_mix_rmsnorm(torch.from_numpy(mix).cuda(), torch.from_numpy(perm).cuda(), r, x)
    # the fused multiply-add rounds once: mix * r is exact in float64
    ref2 = (r1.astype(np.float64) + mix.astype(np.float64) * r1[perm]).astype(np.float32)
    r2 = r.cpu().numpy()
    assert np.array_equal(r2, ref2)
    assert np.array_equal(x.cpu().numpy().view(np.uint16), o_routing.rms_norm_f16(r2).view(np.uint16))
