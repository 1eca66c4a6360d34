"""The top-K selection of the group masks on keys that stress its digits: one value, few values, the whole range of
float32 magnitudes, ties across waves.  With T = 1 and unit norms the score of a neuron is |h| itself, so the expected
mask is a stable sort of the inputs: exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_19104_amd as rm  # noqa: E402


def _keys(kind, n):
    r = np.random.default_rng(n)
    if kind == "equal":
        return np.full(n, 0.375, np.float32)
    if kind == "two":
        return np.where(r.random(n) < 0.5, np.float32(1.0), np.nextafter(np.float32(1.0), np.float32(2.0)))
    if kind == "range":  # zeros, subnormals, every exponent, infinity
        v = r.integers(0, 0x7f800001, n, dtype=np.uint32).view(np.float32).copy()
        v[r.random(n) < 0.05] = 0.0
        return v
    if kind == "dense":  # neighbouring bit patterns: the last digits decide
        return (np.uint32(0x3f800000) + r.permutation(n).astype(np.uint32)).view(np.float32)
    return np.round(np.abs(r.standard_normal(n)) * 8).astype(np.float32)  # "ties"


@pytest.mark.parametrize("kind", ["equal", "two", "range", "dense", "ties"])
@pytest.mark.parametrize("d_ff", [1, 64, 255, 257, 4096, 4097, 16384])
def test_top_k_is_a_stable_sort(kind, d_ff):
    v = _keys(kind, d_ff)
    order = np.argsort(-v.view(np.int32).astype(np.int64), kind="stable")
    h = torch.from_numpy(v).cuda().view(1, 1, d_ff, 1)
    norms = torch.ones(1, d_ff, device="cuda")
    scores = torch.empty(1, 1, d_ff, device="cuda")
    mask = torch.full((1, d_ff), 7, dtype=torch.uint8, device="cuda")
    for k in sorted({0, 1, d_ff // 3, d_ff - 1, d_ff}):
        rm.rm_group_masks(h, norms, k, scores, mask)
        assert np.array_equal(scores.cpu().numpy().ravel(), v)
        want = np.zeros(d_ff, np.uint8)
        want[order[:k]] = 1
        assert np.array_equal(mask.cpu().numpy().ravel(), want), f"k={k}"
