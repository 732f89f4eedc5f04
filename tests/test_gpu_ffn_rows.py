"""The per-token expert call over the shapes its launches branch on: every d_expert
(h in the down launch up to 1024, a launch of its own beyond), ranks that are and
are not whole 16-byte pieces, token counts from one row run per workgroup to all
of them, and experts without a slot or with an id out of range."""

import numpy as np
import pytest

from oracle import expert as o_expert
from tests.gpu_harness import rel_inf

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


@pytest.mark.parametrize("d,I,r,T", [
    (512, 256, 8, 1), (512, 256, 0, 3), (512, 512, 16, 40), (1024, 512, 5, 2), (2048, 512, 33, 70), (4096, 1024, 64, 9),
    (512, 1024, 24, 1), (8192, 256, 4, 5), (512, 2048, 16, 2), (1024, 4096, 7, 1)])
def test_rows_against_oracle(torch_cuda, d, I, r, T):
    from paper_2609_18063_amd import binding as B, weights as W
    torch = torch_cuda
    E, K, S = 5, 2, 1
    g = np.random.default_rng(d + I + r)
    bundles = [_bundle(g, d, I, r) for _ in range(E + S)]
    buf, offs, _ = W.pack_host(bundles)
    dev = W.upload(buf)
    spec = B.make_spec(d, E, K, S, I, r, 2.0 if r else 0.0)
    table = B.SlotTable(1, E + S, E + S)
    W.bind_layer(table, 0, dev, offs)
    table.unbind(0, 3)
    table.sync()
    x = g.standard_normal((T, d)).astype(np.float16)
    idx = np.stack([g.permutation(3)[:K] for _ in range(T)]).astype(np.int32)
    idx[T - 1] = (3, 7) if T > 1 else (3, 0)      # not resident; out of range
    ws = torch.full((B.workspace_bytes(spec, T),), 255, dtype=torch.uint8, device="cuda")
    ye = torch.full((T, K + S, d), float("nan"), device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.expert_ffn(spec, table, 0, torch.from_numpy(x).cuda(), torch.from_numpy(idx).cuda(), ye, status, ws)
    torch.cuda.synchronize()
    got = ye.cpu().numpy()
    assert status.item() == B.MOE_STATUS_SLOT_MISS | (B.MOE_STATUS_BAD_INDEX if T > 1 else 0)
    for t in sorted({0, T // 2, T - 1}):
        for k, e in enumerate(list(idx[t]) + [E]):
            if e in (3, 7):
                assert not got[t, k].any()
                continue
            ref, _ = o_expert.expert_forward(bundles[e], x[t], 2.0 if r else 0.0)
            # fp32 throughout: the products' roundings and the sums' over d and I terms
            # stay far below 2^-24 sqrt(d + I) of the largest output
            assert rel_inf(got[t, k], ref) <= 4 * 2.0 ** -24 * np.sqrt(d + I), (t, k)
    table.close()


@pytest.mark.parametrize("d,I,r,T", [
    (512, 1024, 5, 9), (2048, 1024, 16, 4), (2048, 1024, 64, 4), (512, 1024, 40, 30), (4096, 1024, 33, 2),
    (8192, 1024, 32, 3), (1024, 1024, 0, 30), (4096, 1024, 0, 24)])
def test_runs_per_workgroup(torch_cuda, d, I, r, T):
    """The runs of rows a down workgroup takes at d_expert 1024: by the workgroups that
    fit at once, up to four, up to eight beyond rank 32, and half as many at rank 0 where
    the last round would be short."""
    test_rows_against_oracle(torch_cuda, d, I, r, T)
