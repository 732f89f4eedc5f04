"""Router logits and top-k at the edges of their kernels' ranges: the row kernel
and the matrix-core kernels (16, 32 and 64 rows a block) with ragged T and E,
and the wave top-k with up to 1024 experts, ties, NaN and infinities."""

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


def _route(torch, T, d, E, K, x, W):
    from paper_2609_18063_amd import binding as B
    spec = B.make_spec(d, E, K, 0, 256, 0, 0.0)
    xt, Wt = torch.from_numpy(x).cuda(), torch.from_numpy(W).cuda()
    # every output byte is written, whatever the buffers held
    lg = torch.full((T, E), float("nan"), device="cuda")
    idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, K), float("nan"), device="cuda")
    ws = torch.full((B.workspace_bytes(spec, T),), 255, dtype=torch.uint8, device="cuda")
    B.route(spec, xt, Wt, idx, w, ws, logits=lg)
    torch.cuda.synchronize()
    return lg.cpu().numpy(), idx.cpu().numpy(), w.cpu().numpy()


# (T, d, E, K): one token; the last sizes of the row kernel and the first of
# the 16-row blocks; ragged 16-, 32- and 64-row blocks; E past a multiple of 16
@pytest.mark.parametrize("T,d,E,K", [
    (1, 512, 16, 2), (1, 2048, 256, 8), (3, 8192, 7, 7), (32, 2048, 256, 8), (33, 2048, 256, 8), (128, 512, 5, 2),
    (129, 512, 5, 2), (65, 4096, 65, 4), (513, 2048, 250, 8), (641, 2048, 256, 8), (1025, 1024, 1000, 8),
    (3073, 512, 241, 3)])
def test_route_logits_and_selection(torch_cuda, T, d, E, K):
    g = np.random.default_rng(T * 7 + E)
    x = g.standard_normal((T, d)).astype(np.float16)
    W = (g.standard_normal((E, d)) * 0.02).astype(np.float16)
    W[0] = (W[0].astype(np.float32) * 2.0 ** -12).astype(np.float16)   # subnormal weights count
    lg, idx, w = _route(torch_cuda, T, d, E, K, x, W)
    x64, W64 = x.astype(np.float64), W.astype(np.float64)
    ref = x64 @ W64.T
    # exact products, at most d/8 + 16 sequential fp32 roundings on any path
    bound = (d / 8 + 16) * 2.0 ** -24 * (np.abs(x64) @ np.abs(W64).T)
    assert np.all(np.abs(lg - ref) <= bound)
    for t in {0, T // 2, T - 1}:
        ri, rw = o_routing.softmax_topk(lg[t], K)   # the selection of the device's own logits is exact
        assert idx[t].tolist() == list(ri)
        np.testing.assert_allclose(w[t], rw, rtol=2e-6)


@pytest.mark.parametrize("E,K", [(1, 1), (64, 32), (255, 8), (256, 32), (257, 32), (1000, 8), (1024, 32)])
def test_topk_ties_and_special_values(torch_cuda, E, K):
    from paper_2609_18063_amd import binding as B
    torch = torch_cuda
    T = 5
    g = np.random.default_rng(E + K)
    lg = g.standard_normal((T, E)).astype(np.float32)
    lg[1] = np.round(lg[1])                     # heavy ties: the lower id wins
    lg[2] = -0.0
    lg[2, ::2] = 0.0                            # -0 and +0 tie
    lg[3, : E - K] = -np.inf                    # the set is the K finite logits
    if E > K:
        lg[4, 0] = np.nan                       # NaN ranks with -inf, never selected here
        lg[4, 1:] = np.abs(lg[4, 1:])
    spec = B.make_spec(512, E, K, 0, 256, 0, 0.0)
    idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, K), float("nan"), device="cuda")
    B.topk(spec, torch.from_numpy(lg).cuda(), idx, w)
    torch.cuda.synchronize()
    idx, w = idx.cpu().numpy(), w.cpu().numpy()
    ref = np.where(np.isnan(lg), -np.inf, lg) + 0.0
    for t in range(T):
        order = np.lexsort((np.arange(E), -ref[t]))[:K]
        assert idx[t].tolist() == order.tolist(), t
        ex = np.exp(ref[t][order].astype(np.float64) - ref[t][order[0]])
        np.testing.assert_allclose(w[t], ex / ex.sum(), rtol=2e-6)


@pytest.mark.parametrize("E,K,T", [(7, 7, 1), (7, 7, 280), (7, 7, 281), (16, 5, 1), (16, 6, 1), (16, 6, 240), (16, 6, 241), (60, 32, 1280), (60, 32, 1281),
                                   (255, 8, 320), (256, 8, 321), (256, 32, 64), (257, 8, 3)])
def test_topk_by_wave_or_workgroup(torch_cuda, E, K, T):
    """Both selections around the rule that chooses between them, on random logits and
    on heavy ties (the lower id first)."""
    from paper_2609_18063_amd import binding as B
    torch = torch_cuda
    g = np.random.default_rng(E + K + T)
    lg = g.standard_normal((T, E)).astype(np.float32)
    lg[T // 2] = np.round(lg[T // 2])
    spec = B.make_spec(512, E, K, 0, 256, 0, 0.0)
    idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
    w = torch.full((T, K), float("nan"), device="cuda")
    B.topk(spec, torch.from_numpy(lg).cuda(), idx, w)
    torch.cuda.synchronize()
    order = np.argsort(-lg, axis=1, kind="stable")[:, :K]
    assert np.array_equal(idx.cpu().numpy(), order)
    top = np.take_along_axis(lg, order, 1).astype(np.float64)
    ex = np.exp(top - top[:, :1])
    np.testing.assert_allclose(w.cpu().numpy(), ex / ex.sum(1, keepdims=True), rtol=2e-6)
