"""The block codec and the window-parallel append (forced) against the tile codec (forced): every buffer of the cache byte for byte, for each
key metadata format, over plans that end units of 64 and 128 tokens inside, at and just past their edges,
start inside a window, leave a sequence empty, and use the residual rings and the single global rotation; one
case has enough value units (at least 512 of 128 tokens) for the whole-size variant, the others take the
half-size one. Both write the documented order's bytes, so nothing may differ."""

import numpy as np
import pytest

from synth import gen_layer, workload

pytestmark = pytest.mark.gpu


def _fill(path, monkeypatch, meta, lens, plan, heads, residual, flags):
    import torch

    import gpu_helpers as gh
    import paper_2609_11582_amd as okvq
    wl = workload("omni3b_b4_64k_stream")
    lay = gen_layer(wl, 1, lengths=np.asarray(lens, np.int32), n_tokens=max(lens))
    k, v = (np.concatenate([lay[f]] * heads, 1)[:, :heads].copy() for f in ("k", "v"))
    monkeypatch.setenv("OKVQ_APPEND_PATH", path)
    cap = (max(lens) + 31) // 32 * 32
    cache = okvq.KVCache(len(lens), heads, heads, cap, torch.from_numpy(lay["signs"]), torch.from_numpy(lay["rot"]),
                         key_meta=meta, residual=residual)
    gh.append_chunks(cache, k, v, lay["modality"], lens, plan, flags=flags)
    assert okvq.okvq_cache_status(cache) == 0
    return {n: t.cpu().numpy() for n, t in cache.buffers.items()}


@pytest.mark.parametrize("meta,residual,flags", [("fp16", 128, 0), ("fp16", 0, 2), ("mxfp4", 128, 0), ("turboquant", 0, 2)])
@pytest.mark.parametrize("lens,plan,heads", [([1, 0, 33], [[1, 0, 33]], 1), ([64, 65, 127], [[64, 65, 127]], 2),
                                             ([128, 129, 257], [[31, 1, 200], [97, 128, 57]], 1),
                                             ([8300, 8129], [[8200, 8129], [100, 0]], 4)])
def test_block_and_window_codecs_write_the_tile_codecs_bytes(meta, residual, flags, lens, plan, heads, monkeypatch):
    print(f"[gpu-case] block codec {meta} residual={residual} flags={flags} lens={lens} plan={plan}", flush=True)
    want = _fill("tile", monkeypatch, meta, lens, plan, heads, residual, flags)
    for path in ("block", "window"):
        got = _fill(path, monkeypatch, meta, lens, plan, heads, residual, flags)
        for name in want:
            a, b = got[name].view(np.uint8), want[name].view(np.uint8)
            assert np.array_equal(a, b), f"{path}, {name}: {int((a != b).sum())} bytes differ"


@pytest.mark.parametrize("lens,heads,flags", [([33000], 1, 0), ([256, 255, 0], 64, 2), ([257, 1, 300], 33, 0),
                                              ([1024, 993], 17, 0), ([256, 200], 64, 0)])
def test_stateless_values_write_the_appended_bytes(lens, heads, flags):
    """okvq_quantize_values from the fp32 matrix against the block codec's append from the prepared fragments: the
    same split of R_m and the same order of products, so the same bytes. More than 128 units of 256 tokens take the
    wide kernel (all but the last case, at 128), with lengths at, inside and past a unit's and a window's edge."""
    import torch

    import gpu_helpers as gh
    import paper_2609_11582_amd as okvq
    rng = np.random.default_rng(sum(lens) + heads)
    wl = workload("omni3b_b4_64k_stream")
    n, B = max(lens), len(lens)
    lay = gen_layer(wl, 1, lengths=np.asarray([32], np.int32), n_tokens=32)
    v = rng.standard_normal((B, heads, n, 128)).astype(np.float16)
    v[:, :, :: 57] = 0
    mod = rng.integers(0, 3, (B, n)).astype(np.uint8)
    mod[:, n // 2:] = 1
    cap = (n + 31) // 32 * 32
    print(f"[gpu-case] stateless values lens={lens} heads={heads} flags={flags}", flush=True)
    cache = okvq.KVCache(B, heads, heads, cap, torch.from_numpy(lay["signs"]), torch.from_numpy(lay["rot"]))
    vd, md = gh.f16dev(v), gh.dev(mod)
    nd = torch.tensor(lens, dtype=torch.int32, device="cuda")
    okvq.okvq_append(cache, [0] * B, vd, vd, md, lens, nd, n, flags)
    codes, norms = torch.zeros_like(cache["v_codes"]), torch.zeros_like(cache["v_norm"])
    okvq.okvq_quantize_values(cache.dims, vd, md, n, lens, cache.v_rot, flags, codes, norms)
    torch.cuda.synchronize()
    assert torch.equal(norms.view(torch.int16), cache["v_norm"].view(torch.int16))
    assert torch.equal(codes, cache["v_codes"])


@pytest.mark.parametrize("meta,kb,vb", [("fp16", 3, 3), ("turboquant", 3, 2), ("fp16", 4, 4), ("turboquant", 2, 4)])
def test_ladder_append_of_a_long_prompt_writes_the_stateless_bytes(meta, kb, vb):
    """The ladder's append as a long prompt takes it: keys and values in one launch, at least 256 units of each in
    alternation, value units of 128 tokens and prepared fragments. Against the stateless calls of the same rows (one
    role a launch, the fp32 matrix), whose codes the ladder tests compare with the oracle."""
    import torch

    import paper_2609_11582_amd as okvq
    B, H, n = 1, 4, 16501
    g = torch.Generator(device="cuda").manual_seed(10 * kb + vb)
    k, v = (torch.randn(B, H, n, 128, generator=g, device="cuda").half() for _ in range(2))
    k[:, :, 77], v[:, :, 33] = 0, 0
    mod = torch.randint(0, 3, (B, n), generator=g, device="cuda", dtype=torch.uint8)
    rot = torch.linalg.qr(torch.randn(3, 128, 128, generator=g, device="cuda"))[0].contiguous()
    print(f"[gpu-case] ladder prompt {meta} K{kb}V{vb}", flush=True)
    caches = [okvq.KVCache(B, H, H, -(-n // 32) * 32, torch.where(torch.arange(128) % 3 == 0, -1, 1), rot.cpu(),
                           key_meta=meta, key_bits=kb, value_bits=vb) for _ in range(2)]
    okvq.okvq_append(caches[0], [0], k, v, mod, [n], torch.tensor([n], dtype=torch.int32, device="cuda"), n)
    c = caches[1]
    if meta == "fp16":
        okvq.okvq_quantize_keys(c.dims, k, n, [n], c.key_signs, c["k_codes"], c["k_min"], c["k_step"], c["k_norm"])
    else:
        okvq.okvq_quantize_keys_tq(c.dims, k, n, [n], c.key_signs, c["k_codes"], c["k_norm"])
    okvq.okvq_quantize_values(c.dims, v, mod, n, [n], c.v_rot, 0, c["v_codes"], c["v_norm"])
    torch.cuda.synchronize()
    for name in ("k_codes", "k_norm", "v_codes", "v_norm") + (("k_min", "k_step") if meta == "fp16" else ()):
        a, b = (x[name].view(torch.uint8) for x in caches)
        assert torch.equal(a, b), f"{name}: {int((a != b).sum())} bytes differ"
