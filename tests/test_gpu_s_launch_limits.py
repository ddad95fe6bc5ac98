"""Codec calls whose sequences and heads need 2^32 threads or more, which no launch takes: they are cut into launches
by sequence. At one token each, against the bytes of the same rows in a small call."""

import pytest

pytestmark = pytest.mark.gpu


def _codec_inputs(B, H):
    import torch
    g = torch.Generator(device="cuda").manual_seed(B)
    x = torch.randn(B, H, 1, 128, generator=g, device="cuda", dtype=torch.float16)
    return x, torch.randint(0, 3, (B, 1), generator=g, device="cuda", dtype=torch.uint8)


def test_ladder_append_of_many_heads():
    import torch

    import paper_2609_11582_amd as okvq
    B, H, seqs, heads = 256, 32769, [0, 127, 128, 255], [0, 32768]
    print(f"[gpu-case] ladder append B={B} H={H}", flush=True)
    x, mod = _codec_inputs(B, H)

    def append(x, mod):
        b, h = x.shape[:2]
        c = okvq.KVCache(b, h, h, 32, torch.ones(128), torch.eye(128).repeat(3, 1, 1), key_meta="turboquant", key_bits=2,
                         value_bits=2)
        okvq.okvq_append(c, [0] * b, x, x, mod, [1] * b, torch.ones(b, dtype=torch.int32, device="cuda"), 1)
        return c.views()
    got = append(x, mod)
    want = append(x[seqs][:, heads].contiguous(), mod[seqs].contiguous())
    for name in ("k_codes", "v_codes", "k_norm", "v_norm"):
        assert torch.equal(got[name][seqs][:, heads], want[name]), name
    assert bool((got["seq_lens"] == 1).all()) and torch.equal(got["modality"][:, :1], mod)


def test_stateless_values_of_many_heads():
    import torch

    import paper_2609_11582_amd as okvq
    B, H, seqs, heads = 129, 65535, [0, 63, 64, 128], [0, 65534]
    print(f"[gpu-case] stateless values B={B} H={H}", flush=True)
    x, mod = _codec_inputs(B, H)
    rot = torch.eye(128, device="cuda").repeat(3, 1, 1).contiguous()

    def values(x, mod):
        b, h = x.shape[:2]
        codes = torch.empty(b, h, 1024, dtype=torch.uint8, device="cuda")
        norms = torch.empty(b, h, 32, dtype=torch.float16, device="cuda")
        okvq.okvq_quantize_values(okvq.make_dims(b, h, h, 32), x, mod, 1, [1] * b, rot, 0, codes, norms)
        return codes, norms
    got = values(x, mod)
    for a, b in zip(got, values(x[seqs][:, heads].contiguous(), mod[seqs].contiguous())):
        assert torch.equal(a[seqs][:, heads], b)

