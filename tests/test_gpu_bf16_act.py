"""The bf16 kernels' activations over the range of their argument, extremes included: one neuron
with w_up = w_down = 1 gives h * 1, so y - x is the activation times the up sum, rounded to bf16 once.  Bar: 2^-8 relative
(bf16's half ulp 2^-9 of h, doubled) plus |z| 2^-126 (smaller values than 1 / (1 + e^-z) = 2^-126 gives are not asked for).

The anchor step keeps the same h in float32: there the activation itself is measured."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2609_19104_amd as rm  # noqa: E402


@pytest.mark.parametrize("act", ["silu", "gelu_tanh"])
def test_activation_range(act):
    d = 256
    z = np.concatenate([np.linspace(-12, 12, 49), [-1e4, -200.0, -104.0, -88.0, -64.0, 40.0, 90.0, 3e4]])
    z = torch.from_numpy(z.astype(np.float32)).bfloat16().float()
    T = z.numel()
    x = torch.zeros(1, T, d)
    x[0, :, 0] = z      # the gate sum
    x[0, :, 1] = 1.0    # the up sum
    w = torch.zeros(3, 8, d)
    w[0, 0, 0] = w[1, 0, 1] = w[2, 0, 5] = 1.0
    layer = tuple(m.cuda().bfloat16() for m in w) + (None,)
    idx = torch.full((1, 8), -1, dtype=torch.int32, device="cuda")
    idx[0, 0] = 0
    cnt = torch.ones(1, dtype=torch.int32, device="cuda")
    xt = x.cuda()
    y = torch.empty_like(xt)
    rm.rm_sparse_ffn_layer(xt, y, layer, idx, cnt, 1, rm.workspace(d, 8, rm.RM_BF16, 1, T, 1), act=act)
    got = y[0, :, 5].cpu().double()
    zd = z.double()
    u = zd if act == "silu" else 2 * 0.7978845608028654 * (zd + 0.044715 * zd ** 3)
    want = zd * torch.sigmoid(u)
    err = (got - want).abs()
    assert bool((err <= want.abs() * 2.0 ** -8 + zd.abs() * 2.0 ** -126).all()), (zd, got, want)


@pytest.mark.parametrize("act", ["silu", "gelu_tanh"])
def test_activation_is_float32(act):
    # h of one neuron with up sum 1, as the anchor keeps it, against 64 bits.  Bar in units of 2^-24: 2 for e^-w, 1 each
    # for 1 + e^-w and the division; GELU's w is rounded 6 times before e^-w multiplies that error by |w|.  Below
    # 1 / (1 + e^-w) = 2^-128 the exponential overflows.
    d = 256
    z = np.concatenate([np.linspace(-88, 40, 2000), np.linspace(-6, 6, 2000), [-1e4, -200.0, -104.0, -88.0, 90.0, 3e4]])
    z = torch.from_numpy(z.astype(np.float32)).bfloat16().float()
    T = z.numel()
    x = torch.zeros(1, T, d)
    x[0, :, 0] = z
    x[0, :, 1] = 1.0
    w = torch.zeros(3, 8, d)
    w[0, 0, 0] = w[1, 0, 1] = 1.0
    layer = tuple(m.cuda().bfloat16() for m in w) + (None,)
    idx = torch.full((1, 1, 8), -1, dtype=torch.int32, device="cuda")
    idx[0, 0, 0] = 0
    cnt = torch.ones(1, 1, dtype=torch.int32, device="cuda")
    xt = x.cuda()
    y, ya = torch.empty_like(xt), torch.empty(1, 1, T, d, device="cuda")
    h = torch.zeros(1, 1, 1, T, device="cuda")
    rm.rm_anchor_ffn_stack(xt, y, [layer], idx, cnt, 1, ya, h, rm.workspace(d, 8, rm.RM_BF16, 1, T, 8), 1e-6, act)
    got = h[0, 0, 0].cpu().double()
    zd = z.double()
    u = zd if act == "silu" else 2 * 0.7978845608028654 * (zd + 0.044715 * zd ** 3)
    want = zd * torch.sigmoid(u)
    units = 4.0 + (6.0 * u.abs() if act == "gelu_tanh" else 0.0)
    bar = want.abs() * units * 2.0 ** -24 + zd.abs() * 2.0 ** -128
    worst = ((got - want).abs() / bar).argmax()
    assert bool(((got - want).abs() <= bar).all()), (zd[worst], got[worst], want[worst])
