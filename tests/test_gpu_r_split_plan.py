"""Which decode calls plan one split per sequence to save the merge launch: those that save it. With the fp16
residual the merge launch runs whatever the plan (it attends the tail), so windows beyond what one round of a
work-group's waves covers (16) are split, as under a forced number of groups. Seen from the records that the
split launch leaves in the caller's workspace (4224 bytes per split of a sequence and KV head; none where the
only split writes the outputs itself)."""

import math

import pytest

pytestmark = pytest.mark.gpu
RECORD = 4224 // 4


@pytest.mark.parametrize("residual,tokens,groups,splits", [
    (0, 1024, None, 0), (0, 1056, None, 3), (0, 1024, "256", 2),
    (128, 640, None, 1), (128, 672, None, 2), (128, 1152, None, 2), (128, 1184, None, 3)])
def test_records_of_the_split_launch(residual, tokens, groups, splits, monkeypatch):
    import torch

    import paper_2609_11582_amd as okvq
    B, H, Hq = 2, 2, 14
    g = torch.Generator(device="cuda").manual_seed(tokens)
    cache = okvq.KVCache(B, H, Hq, -(-tokens // 32) * 32, torch.ones(128), torch.eye(128).repeat(3, 1, 1), residual=residual)
    k, v = (torch.randn(B, H, tokens, 128, generator=g, device="cuda").half() for _ in range(2))
    q = torch.randn(B, Hq, 128, generator=g, device="cuda").half()
    n = torch.tensor([tokens] * B, dtype=torch.int32, device="cuda")
    print(f"[gpu-case] split plan residual={residual} tokens={tokens} groups={groups}", flush=True)
    okvq.okvq_append(cache, [0] * B, k, v, torch.ones(B, tokens, dtype=torch.uint8, device="cuda"), [tokens] * B, n, tokens)
    if groups:
        monkeypatch.setenv("OKVQ_DECODE_GROUPS", groups)
    ws = okvq.decode_workspace(cache.dims, tokens).view(torch.float32)
    ws.fill_(float("nan"))
    out = torch.full((B, Hq, 128), float("nan"), device="cuda")
    okvq.okvq_decode_attention(cache, [tokens] * B, q, 1 / math.sqrt(128), out, ws)
    torch.cuda.synchronize()
    assert torch.isfinite(out).all()
    written = torch.isfinite(ws[: ws.numel() // RECORD * RECORD].view(-1, RECORD)).any(1)
    assert int(written.sum()) == B * H * splits
