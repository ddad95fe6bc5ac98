"""Decode plans of one split per sequence write the output rows without a merge launch. Against the same plan
with its merge launch (the timed entry points), at lengths around the largest such plan, with an empty
sequence and 7 of 8 head slots in use: the merge multiplies the split's output by its sum L and by 1 / L, three
fp32 roundings, so rows agree within 4 * 2^-24 of each value; and beyond that plan the two are bit-identical."""

import math

import numpy as np
import pytest

from synth import gen_layer, gen_queries, workload

pytestmark = pytest.mark.gpu
FORMATS = [("fp16", 0, 0, 0), ("mxfp4", 0, 0, 0), ("turboquant", 0, 0, 2), ("fp16", 3, 4, 0)]


@pytest.mark.parametrize("lens", [[1, 0, 33], [511, 512, 1], [513, 0, 700], [1024, 1000, 0], [1025, 64, 1056]])
@pytest.mark.parametrize("meta,kb,vb,flags", FORMATS + [("dense", 0, 0, 0)])
def test_one_split_equals_its_merge(meta, kb, vb, flags, lens):
    import torch

    import gpu_helpers as gh
    import paper_2609_11582_amd as okvq
    B, H, Hq, n = len(lens), 2, 14, max(lens)
    wl = workload("omni3b_b4_64k_stream")
    lay = gen_layer(wl, 1, lengths=np.asarray(lens, np.int32), n_tokens=n)
    k, v = (lay[f][:, :H].copy() for f in ("k", "v"))
    q = gh.f16dev(gen_queries(wl.wid, 1, B, Hq))
    cap = (n + 31) // 32 * 32
    print(f"[gpu-case] one split {meta} K{kb}V{vb} lens={lens}", flush=True)
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
    for e in ev:
        e.record()
    out = torch.full((2, B, Hq, 128), float("nan"), device="cuda")
    sm = 1 / math.sqrt(128)
    if meta == "dense":
        dims = okvq.make_dims(B, H, Hq, cap)
        kd, vd = (torch.zeros(B, H, cap, 128, dtype=torch.float16, device="cuda") for _ in range(2))
        kd[:, :, :n], vd[:, :, :n] = gh.f16dev(k), gh.f16dev(v)
        sl, ws = torch.tensor(lens, dtype=torch.int32, device="cuda"), okvq.dense_workspace(dims, n)
        okvq.okvq_decode_attention_dense(dims, kd, vd, sl, lens, q, sm, out[0], ws)
        okvq.okvq_decode_attention_dense(dims, kd, vd, sl, lens, q, sm, out[1], ws, events=ev)
    else:
        cache = okvq.KVCache(B, H, Hq, cap, torch.from_numpy(lay["signs"]), torch.from_numpy(lay["rot"]), key_meta=meta,
                             key_bits=kb, value_bits=vb)
        gh.append_chunks(cache, k, v, lay["modality"], lens, [lens], flags=flags)
        ws = okvq.decode_workspace(cache.dims, n)
        okvq.okvq_decode_attention(cache, lens, q, sm, out[0], ws, flags=flags)
        okvq.okvq_decode_attention_timed(cache, lens, q, sm, out[1], ws, ev, flags=flags)
    torch.cuda.synchronize()
    got, want = out.cpu().numpy()
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - want) <= 4 * 2.0 ** -24 * np.abs(want))
    if n > (1024 if meta != "dense" and not kb else 512):
        assert np.array_equal(got, want)
    for b, L in enumerate(lens):
        assert L > 0 or not got[b].any()
