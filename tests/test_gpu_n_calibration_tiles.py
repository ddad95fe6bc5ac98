"""Calibration kernels at the edges of their tiles: 128 queries or keys per work-group, 64 rows per
staged tile, 32 per wave, runs of two 64-token covariance chunks, and a negative softmax scale (carried
by the held operand). Against the float64 oracle at the bounds of test_gpu_g_calibration.py: weights
within 3e-4 of each weight plus 1e-7 of the largest (fp32 scores, hardware exp2 and fp32 sums), the
covariance within 1e-5 of sum_t w_t |v_t| |v_t|^T per element (fp16 hi + lo products, fp32 sums)."""

import math

import numpy as np
import pytest

from oracle.calibration import attention_weights, value_covariance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,H,Hq,sign", [([1, 31, 32, 33], 1, 1, 1), ([63, 64, 65, 0], 2, 6, -1),
                                            ([127, 128, 129], 1, 8, 1), ([255, 257, 320, 385], 1, 2, -1)])
def test_weights_and_covariance_at_tile_edges(lens, H, Hq, sign):
    import torch

    import gpu_helpers as gh
    import paper_2609_11582_amd as okvq
    rng = np.random.default_rng(sum(lens) + Hq)
    B, N, sm = len(lens), max(lens), sign / math.sqrt(128)
    q = rng.standard_normal((B, Hq, N, 128)).astype(np.float16)
    k = (2 * rng.standard_normal((B, H, N, 128))).astype(np.float16)
    v = rng.standard_normal((B, H, N, 128)).astype(np.float16)
    mod = rng.integers(0, 3, (B, N)).astype(np.uint8)
    print(f"[gpu-case] calibration tiles lens={lens} H={H} Hq={Hq} scale={sm:.4f}", flush=True)
    dims = okvq.make_dims(B, H, Hq, 32)
    ws = okvq.calibration_workspace(dims, N)
    w = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    cov = torch.full((3, 128, 128), float("nan"), dtype=torch.float32, device="cuda")
    okvq.okvq_calibration_weights(dims, gh.f16dev(q), gh.f16dev(k), N, lens, sm, w, ws)
    okvq.okvq_value_covariance(dims, gh.f16dev(v), gh.dev(mod), w, N, lens, cov, ws)
    torch.cuda.synchronize()
    got, ref = w.cpu().numpy().astype(np.float64), attention_weights(q, k, lens, sm)
    assert np.all(np.abs(got - ref) <= 3e-4 * ref + 1e-7 * ref.max())
    want = value_covariance(v, mod, got, lens)
    scale = value_covariance(np.abs(v.astype(np.float64)), mod, got, lens)
    assert np.all(np.abs(cov.cpu().numpy() - want) <= 1e-5 * scale + 1e-30)


@pytest.mark.parametrize("sm", [0.0, -0.0, 1e-45, -1e-39])
def test_weights_at_scale_zero(sm):
    """A zero scale (and one that underflows) attends every earlier key alike: w_t is the sum over the group's
    heads and the positions i >= t of 1 / (i + 1)^2. The same bounds."""
    import torch

    import gpu_helpers as gh
    import paper_2609_11582_amd as okvq
    rng = np.random.default_rng(5)
    lens, H, Hq = [1, 33, 130, 0, 200], 2, 6
    B, N = len(lens), max(lens)
    q = rng.standard_normal((B, Hq, N, 128)).astype(np.float16)
    k = rng.standard_normal((B, H, N, 128)).astype(np.float16)
    q[4], k[4] = 60000 * np.sign(q[4]), 60000 * np.sign(k[4])  # the largest scores
    print(f"[gpu-case] calibration weights scale={sm}", flush=True)
    dims = okvq.make_dims(B, H, Hq, 32)
    w = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    okvq.okvq_calibration_weights(dims, gh.f16dev(q), gh.f16dev(k), N, lens, sm, w, okvq.calibration_workspace(dims, N))
    torch.cuda.synchronize()
    got, ref = w.cpu().numpy().astype(np.float64), attention_weights(q, k, lens, 0.0)
    assert np.all(np.abs(got - ref) <= 3e-4 * ref + 1e-7 * ref.max())


@pytest.mark.parametrize("lens,H", [([64, 65, 0], 1), ([4031], 1), ([4033], 1), ([129, 2000], 2)])
def test_covariance_runs_of_one_and_two_chunks(lens, H):
    """Fewer than 64 chunks of 64 tokens (over sequences and heads) take one chunk a partial, more take two; the
    first and last of each kind, with odd chunk counts. The same bound as above."""
    import torch

    import gpu_helpers as gh
    import paper_2609_11582_amd as okvq
    rng = np.random.default_rng(sum(lens))
    B, N = len(lens), max(lens)
    v = rng.standard_normal((B, H, N, 128)).astype(np.float16)
    w = rng.random((B, H, N)).astype(np.float32)
    mod = rng.integers(0, 3, (B, N)).astype(np.uint8)
    print(f"[gpu-case] covariance runs lens={lens} H={H}", flush=True)
    dims = okvq.make_dims(B, H, H, 32)
    cov = torch.full((3, 128, 128), float("nan"), dtype=torch.float32, device="cuda")
    okvq.okvq_value_covariance(dims, gh.f16dev(v), gh.dev(mod), gh.dev(w), N, lens, cov, okvq.calibration_workspace(dims, N))
    torch.cuda.synchronize()
    want = value_covariance(v, mod, w.astype(np.float64), lens)
    scale = value_covariance(np.abs(v.astype(np.float64)), mod, w.astype(np.float64), lens)
    assert np.all(np.abs(cov.cpu().numpy() - want) <= 1e-5 * scale + 1e-30)
