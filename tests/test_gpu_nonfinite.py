"""Infinities and NaN in a token's input: they reach that token's outputs and no
other token's, in the router (row products and matrix-core blocks), the per-token
experts and the grouped experts (both gate/up shapes)."""

import numpy as np
import pytest

from tests.test_gpu_grouped_shapes import _bundle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    from paper_2609_18063_amd import binding
    binding.lib()
    return torch


def _poison(x, rows):
    y = x.copy()
    for q, t in enumerate(rows):
        y[t, 3 + q] = (np.inf, -np.inf, np.nan)[q % 3]
    return y


@pytest.mark.parametrize("T,d,E,K", [(5, 512, 16, 8), (40, 2048, 256, 8), (200, 512, 65, 3), (700, 2048, 256, 8),
                                     (1300, 1024, 1000, 4)])
def test_route(torch_cuda, T, d, E, K):
    from paper_2609_18063_amd import binding as B
    torch = torch_cuda
    g = np.random.default_rng(T + E)
    x = g.standard_normal((T, d)).astype(np.float16)
    W = torch.from_numpy((g.standard_normal((E, d)) * 0.02).astype(np.float16)).cuda()
    bad = sorted({0, 1, T // 2, T - 1})
    spec = B.make_spec(d, E, K, 0, 256, 0, 0.0)
    out = []
    for v in (x, _poison(x, bad)):
        lg = torch.full((T, E), 7.0, device="cuda")
        idx = torch.full((T, K), -1, dtype=torch.int32, device="cuda")
        w = torch.full((T, K), 7.0, device="cuda")
        ws = torch.full((B.workspace_bytes(spec, T),), 255, dtype=torch.uint8, device="cuda")
        B.route(spec, torch.from_numpy(v).cuda(), W, idx, w, ws, logits=lg)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (lg, idx, w)])
    good = np.setdiff1d(np.arange(T), bad)
    for a, b in zip(*out):
        assert np.array_equal(a[good], b[good])
    lg, idx, _ = out[1]
    for t in bad:
        assert not np.isfinite(lg[t]).any(), t
        assert len(set(idx[t].tolist())) == K and idx[t].min() >= 0 and idx[t].max() < E, t
        order = np.lexsort((np.arange(E), -np.where(np.isnan(lg[t]), -np.inf, lg[t])))[:K]
        assert idx[t].tolist() == order.tolist(), t


@pytest.mark.parametrize("path,T,d,I,E,K,S,r", [
    ("rows", 1, 512, 256, 4, 2, 1, 8), ("rows", 9, 2048, 512, 6, 2, 1, 16), ("rows", 30, 1024, 1024, 6, 3, 0, 5),
    ("rows", 3, 512, 2048, 4, 2, 0, 16), ("grouped", 33, 512, 256, 4, 2, 1, 8), ("grouped", 70, 2048, 1024, 6, 2, 0, 16),
    ("grouped", 200, 512, 512, 4, 1, 1, 3), ("grouped", 1040, 1024, 512, 8, 8, 1, 16)])
def test_experts(torch_cuda, path, T, d, I, E, K, S, r):
    from paper_2609_18063_amd import binding as B, weights as W
    torch = torch_cuda
    g = np.random.default_rng(T + d + I)
    buf, offs, _ = W.pack_host([_bundle(g, d, I, r) for _ in range(E + S)])
    dev = W.upload(buf)
    spec = B.make_spec(d, E, K, S, I, r, 2.0)
    table = B.SlotTable(1, E + S, E + S)
    W.bind_layer(table, 0, dev, offs)
    table.sync()
    x = g.standard_normal((T, d)).astype(np.float16)
    idx = torch.from_numpy(np.stack([g.permutation(E)[:K] for _ in range(T)]).astype(np.int32)).cuda()
    bad = sorted({T // 3, T // 2, T - 1})
    ffn = B.expert_ffn if path == "rows" else B.expert_ffn_grouped
    out = []
    for v in (x, _poison(x, bad)):
        ye = torch.full((T, K + S, d), 7.0, device="cuda")
        status = torch.zeros(1, dtype=torch.int32, device="cuda")
        ws = torch.full((B.workspace_bytes(spec, T),), 255, dtype=torch.uint8, device="cuda")
        ffn(spec, table, 0, torch.from_numpy(v).cuda(), idx, ye, status, ws)
        torch.cuda.synchronize()
        assert status.item() == 0
        out.append(ye.cpu().numpy())
    good = np.setdiff1d(np.arange(T), bad)
    assert np.isfinite(out[0]).all()
    assert np.array_equal(out[0][good], out[1][good])
    assert not np.isfinite(out[1][bad]).any()
    table.close()
