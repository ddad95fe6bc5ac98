"""The residual tail of the merge launch by itself: with at most 128 tokens no split holds any, so the outputs are the
tail's fp32 attention over raw keys (below 128 tokens) or dequantized ones (at 128), at slot counts around a wave's 32.

Bound: a base-2 score is a sum of 128 products (256 with the window's q'.m for quantized keys) in fp32, at most 260
roundings of partial sums below S, the largest sum of the products' magnitudes: as independent errors of at most
2^-25 S each, six standard deviations are 6 sqrt(260) 2^-25 S. Weights and outputs are off by 2 ln 2 times that and by
140 more roundings, relative to the largest value. (A token left out moves an output by about 1 / 128 of a value.)"""

import math

import numpy as np
import pytest

from oracle.residual import decode_layer_residual
from synth import gen_layer, gen_queries, workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [[1, 31, 32, 0], [33, 64, 65, 128], [96, 97, 127, 128]])
@pytest.mark.parametrize("meta", ["fp16", "mxfp4"])
def test_residual_tail_alone(meta, lens):
    import torch

    import gpu_helpers as gh
    import paper_2609_11582_amd as okvq
    B, H, Hq = len(lens), 2, 14
    wl = workload("omni3b_b4_64k_stream")
    lay = gen_layer(wl, 1, lengths=np.asarray(lens, np.int32), n_tokens=128)
    k, v = (lay[f][:, :H].copy() for f in ("k", "v"))
    q = gen_queries(wl.wid, 1, B, Hq)
    print(f"[gpu-case] residual tail {meta} lens={lens}", flush=True)
    cache = okvq.KVCache(B, H, Hq, 128, torch.from_numpy(lay["signs"]), torch.from_numpy(lay["rot"]), key_meta=meta,
                         residual=128)
    gh.append_chunks(cache, k, v, lay["modality"], lens, [lens])
    got = gh.decode(cache, q, lens)
    sm = 1 / math.sqrt(128)
    want = decode_layer_residual(gh.cache_to_numpy(cache), k, v, q, lens, lay["signs"], lay["rot"], sm)
    # |q'.m| + |q' step|.code <= |q| (|m| + |3 step|) <= 4 |q| |k| per unit norm (m and m + 3 step span the window)
    s = 4 * sm * math.log2(math.e) * np.linalg.norm(q.astype(np.float64), axis=-1).max() \
        * np.linalg.norm(k.astype(np.float64), axis=-1).max()
    tol = (2 * math.log(2) * 6 * math.sqrt(260) * s + 280) * 2.0 ** -25 * np.abs(v.astype(np.float64)).max()
    err = np.abs(got - want).max()
    print(f"  max error {err:.2e}, bound {tol:.2e}", flush=True)
    assert err <= tol
    assert not got[[b for b, L in enumerate(lens) if L == 0]].any()
