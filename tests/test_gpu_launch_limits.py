"""Calls whose rows come near what one launch can hold (a grid dimension takes fewer than 2^32 threads).  They need some
tens of GB of device memory and well under a second."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_19104_amd as rm  # noqa: E402
from gpu_helpers import TOL_BF16  # noqa: E402


def _weights(seed, *shapes):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return [(torch.randn(s, generator=g, device="cuda") * 0.1).bfloat16() for s in shapes]


def _glu(x, wg, wu):
    a, b = x.double() @ wg.double().t(), x.double() @ wu.double().t()
    return a * torch.sigmoid(a) * b


def _close(got, want):
    assert float((got.double() - want).abs().max() / want.abs().max()) <= TOL_BF16


def test_context_ffn_with_more_rows_than_workgroups_of_a_launch():
    # 2^24 rows of one 256-thread workgroup each are one thread too many (the launch then runs the rest of 2^32 only).
    n, d, d_ff, cnt = (1 << 24) + 1, 64, 128, 300
    if torch.cuda.mem_get_info()[0] < 24e9:
        pytest.skip("needs 24 GB")
    wg, wu, wd = _weights(1, (d_ff, d), (d_ff, d), (d, d_ff))
    x, y = torch.zeros(n, d, device="cuda"), torch.zeros(n, d, device="cuda")
    listed = torch.from_numpy(np.sort(np.random.default_rng(1).choice(n, cnt, replace=False))).cuda()
    listed[-1] = n - 1
    x[listed] = torch.randn(cnt, d, device="cuda", generator=torch.Generator(device="cuda").manual_seed(2))
    rows = listed.int()
    count = torch.tensor([cnt], dtype=torch.int32, device="cuda")
    rm.rm_context_ffn(x, y, wg, wu, wd, rows, count, n, rm.context_workspace(d, d_ff, n, n, "silu"), "silu")
    _close(y[listed], _glu(x[listed], wg, wu) @ wd.double().t())
    y[listed] = 0.0
    assert not bool(y.any())


def test_dense_layer_with_as_many_rows_as_the_prologue_takes():
    # The prologue's 64 threads per token just fit a launch; beside the identity lists' workgroups they would not.
    T, d, d_ff = 67108860, 32, 32
    if torch.cuda.mem_get_info()[0] < 48e9:
        pytest.skip("needs 48 GB")
    wg, wu, wd = _weights(3, (d_ff, d), (d_ff, d), (d_ff, d))
    x = torch.randn(1, T, d, device="cuda", generator=torch.Generator(device="cuda").manual_seed(4))
    at = torch.cat([torch.arange(100), torch.arange(T // 2, T // 2 + 100), torch.arange(T - 100, T)]).cuda()
    xs = x[0, at].clone()
    rm.rm_dense_ffn_ref(x, x, (wg, wu, wd, None), rm.workspace(d, d_ff, rm.RM_BF16, 1, T, d_ff))
    _close(x[0, at] - xs, _glu(xs, wg, wu) @ wd.double())
