"""The grouped expert call at the edges of its shapes: group sizes around the row
blocks, tiles and size classes of both gate/up shapes, more routing ids than the
permutation holds at once, ranks 0 to 16, shared experts, and pairs without an
expert."""

import numpy as np
import pytest

from oracle import expert as o_expert
from tests.gpu_harness import TOL_REL_INF, rel_inf

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible GPU")
    from paper_2609_18063_amd import binding
    binding.lib()
    return torch


def _bundle(g, d, I, r):
    b = {"lora": {}}
    for p, (o, i) in (("gate", (I, d)), ("up", (I, d)), ("down", (d, I))):
        s = (g.uniform(0.9, 1.1, (o, i // 64)) * 0.02 / np.sqrt(255 / 12)).astype(np.float16)
        z = (-7.5 * s.astype(np.float64) + 0.005 * g.uniform(-1, 1, s.shape)).astype(np.float16)
        b[p] = (g.integers(0, 256, (o, i // 2), dtype=np.uint8), s, z)
        b["lora"][p] = ((g.standard_normal((r, i)) / r).astype(np.float16),
                        (g.standard_normal((o, r)) * 0.1).astype(np.float16)) if r else None
    return b


# group sizes per routed expert (K = 1: a token per row), the last expert's group
# absent or without a slot; rows 64 a group and 256 wide workgroups choose the wide
# gate/up shape (d_expert 8192 brings 64 column slabs to a small batch)
NARROW = (1, 15, 16, 17, 32, 33, 48, 63, 64, 65, 127, 128, 129)
WIDE = (1, 16, 17, 33, 64, 65, 96, 97, 127, 128, 129, 400)


@pytest.mark.parametrize("counts,d,I,r,S,bad", [
    (NARROW, 512, 256, 8, 1, False), (NARROW, 1024, 512, 0, 0, True), (NARROW, 4096, 256, 16, 2, False),
    (WIDE, 512, 8192, 16, 0, False), (WIDE, 1024, 4096, 5, 2, True), ((9000, 20), 512, 256, 3, 1, False)])
def test_group_sizes(torch_cuda, counts, d, I, r, S, bad):
    from paper_2609_18063_amd import binding as B, weights as W
    torch = torch_cuda
    g = np.random.default_rng(len(counts) * 1000 + d + I + r)
    E = len(counts) + 1                      # the last id has no slot
    bundles = [_bundle(g, d, I, r) for _ in range(E + S)]
    buf, offs, _ = W.pack_host(bundles)
    dev = W.upload(buf)
    spec = B.make_spec(d, E, 1, S, I, r, 2.0 if r else 0.0)
    table = B.SlotTable(1, E + S, E + S)
    W.bind_layer(table, 0, dev, offs, np.arange(E + S)[::-1])
    table.unbind(0, E - 1)
    table.sync()
    idx = np.repeat(np.arange(len(counts)), counts)
    if bad:
        idx = np.concatenate([idx, [E - 1] * 3, [E, -1, E + 100]])
    idx = g.permutation(idx).astype(np.int32)
    T = len(idx)
    x = g.standard_normal((T, d)).astype(np.float16)
    ws = torch.full((B.workspace_bytes(spec, T),), 255, dtype=torch.uint8, device="cuda")
    ye = torch.full((T, 1 + S, d), float("nan"), device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.expert_ffn_grouped(spec, table, 0, torch.from_numpy(x).cuda(), torch.from_numpy(idx[:, None].copy()).cuda(), ye,
                         status, ws)
    torch.cuda.synchronize()
    got = ye.cpu().numpy()
    assert np.isfinite(got).all()
    assert status.item() == (B.MOE_STATUS_SLOT_MISS | B.MOE_STATUS_BAD_INDEX if bad else 0)
    for e in range(len(counts)):
        rows = np.flatnonzero(idx == e)
        for t in {rows[0], rows[len(rows) // 2], rows[-1]}:
            ref, _ = o_expert.expert_forward(bundles[e], x[t], 2.0 if r else 0.0)
            assert rel_inf(got[t, 0], ref) <= TOL_REL_INF, (e, t)
    for t in np.flatnonzero((idx < 0) | (idx >= len(counts))):
        assert not got[t, 0].any(), t
    for s in range(S):
        for t in {0, T // 2, T - 1}:
            ref, _ = o_expert.expert_forward(bundles[E + s], x[t], 2.0 if r else 0.0)
            assert rel_inf(got[t, 1 + s], ref) <= TOL_REL_INF, (s, t)
    # every row of a group: a batch of its own through the per-token call
    rows = torch.full((T, 1 + S, d), float("nan"), device="cuda")
    for a in range(0, T, 512):
        n = min(512, T - a)
        B.expert_ffn(spec, table, 0, torch.from_numpy(x[a:a + n]).cuda(), torch.from_numpy(idx[a:a + n, None].copy()).cuda(),
                     rows[a:a + n], status, torch.empty(B.workspace_bytes(spec, n), dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    # the fp16 roundings (weights, h, lora_scale A v: 2^-11 each) scale with the terms
    # of a row's sums, not with what is left of them where LoRA and base cancel: the
    # error is taken against no less than the median row's largest output
    size = rows.abs().amax(-1)
    diff = (ye - rows).abs().amax(-1) / torch.maximum(size, size[size > 0].median())
    assert float(diff.max()) <= TOL_REL_INF
    table.close()


@pytest.mark.parametrize("E,S,K,T", [(7, 0, 7, 1), (124, 4, 1, 3), (125, 4, 8, 9), (300, 1, 4, 64), (1024, 4, 32, 2),
                                     (1024, 4, 32, 33), (1024, 4, 32, 300)])
def test_many_groups(torch_cuda, E, S, K, T):
    """The permutation's waves own 128 groups each and take 64 of 1024 ids a step:
    group counts around whole waves, fewer and more ids than one pass of them."""
    from paper_2609_18063_amd import binding as B, weights as W
    torch = torch_cuda
    g = np.random.default_rng(E + K + T)
    d, I, r = 512, 256, 8
    bundles = [_bundle(g, d, I, r) for _ in range(8)]
    buf, offs, _ = W.pack_host(bundles)
    dev = W.upload(buf)
    spec = B.make_spec(d, E, K, S, I, r, 2.0)
    table = B.SlotTable(1, E + S, E + S)
    W.bind_layer(table, 0, dev, [offs[e % 8] for e in range(E + S)], g.permutation(E + S))
    table.sync()
    x = torch.from_numpy(g.standard_normal((T, d)).astype(np.float16)).cuda()
    idx = torch.from_numpy(np.stack([g.permutation(E)[:K] for _ in range(T)]).astype(np.int32)).cuda()
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = []
    for ffn in (B.expert_ffn_grouped, B.expert_ffn):
        ws = torch.full((B.workspace_bytes(spec, T),), 255, dtype=torch.uint8, device="cuda")
        out.append(torch.full((T, K + S, d), float("nan"), device="cuda"))
        ffn(spec, table, 0, x, idx, out[-1], status, ws)
    torch.cuda.synchronize()
    ye, rows = out
    assert status.item() == 0
    size = rows.abs().amax(-1)
    # (the bound of test_group_sizes)
    diff = (ye - rows).abs().amax(-1) / torch.maximum(size, size.median())
    assert float(diff.max()) <= TOL_REL_INF
    table.close()


@pytest.mark.parametrize("counts,d,I,r,S,bad", [
    (NARROW, 512, 1024, 5, 1, True), (NARROW, 2048, 1024, 16, 1, False), ((1, 2), 4096, 1024, 16, 0, False),
    (NARROW, 512, 2048, 3, 0, True)])
def test_down_shapes(torch_cuda, counts, d, I, r, S, bad):
    """d_expert 1024 takes 128 or 256 output columns by the number of workgroups, with
    more slab partials of A_d h than are fetched before the k loop."""
    test_group_sizes(torch_cuda, counts, d, I, r, S, bad)


@pytest.mark.parametrize("d,I,E,K,S,r,T", [(2048, 512, 16, 8, 1, 16, 1037), (4096, 1024, 16, 4, 0, 16, 1026),
                                           (4096, 512, 12, 8, 2, 7, 900)])
def test_wide_shape_of_long_rows(torch_cuda, d, I, E, K, S, r, T):
    """The wide gate/up shape with 16 and 32 chunks a row, up to 64 KB of (s, z) rows and
    several experts a token: every row against the per-token call, some against the
    oracle."""
    from paper_2609_18063_amd import binding as B, weights as W
    torch = torch_cuda
    assert T * K >= 64 * E and T * (K + S) // 128 * (I // 128) >= 256   # the wide plan's rule
    g = np.random.default_rng(d + I + T)
    bundles = [_bundle(g, d, I, r) for _ in range(E + S)]
    buf, offs, _ = W.pack_host(bundles)
    dev = W.upload(buf)
    spec = B.make_spec(d, E, K, S, I, r, 2.0)
    table = B.SlotTable(1, E + S, E + S)
    W.bind_layer(table, 0, dev, offs, np.arange(E + S)[::-1])
    table.sync()
    x = g.standard_normal((T, d)).astype(np.float16)
    # expert 0 in every token (the largest group), the rest at random
    idx = np.stack([np.concatenate([[0], 1 + g.permutation(E - 1)[:K - 1]]) for _ in range(T)]).astype(np.int32)
    xd, idxd = torch.from_numpy(x).cuda(), torch.from_numpy(idx).cuda()
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    ye = torch.full((T, K + S, d), float("nan"), device="cuda")
    ws = torch.full((B.workspace_bytes(spec, T),), 255, dtype=torch.uint8, device="cuda")
    B.expert_ffn_grouped(spec, table, 0, xd, idxd, ye, status, ws)
    rows = torch.full((T, K + S, d), float("nan"), device="cuda")
    for a in range(0, T, 512):
        n = min(512, T - a)
        B.expert_ffn(spec, table, 0, xd[a:a + n], idxd[a:a + n], rows[a:a + n], status, ws)
    torch.cuda.synchronize()
    assert status.item() == 0
    size = rows.abs().amax(-1)
    # (the bound of test_group_sizes)
    diff = (ye - rows).abs().amax(-1) / torch.maximum(size, size.median())
    assert float(diff.max()) <= TOL_REL_INF
    for t in (0, T // 2, T - 1):
        for k, e in enumerate(list(idx[t]) + list(range(E, E + S))):
            ref, _ = o_expert.expert_forward(bundles[e], x[t], 2.0)
            assert rel_inf(ye[t, k].cpu().numpy(), ref) <= TOL_REL_INF, (t, k)
    table.close()
