"""The tiled gate/up kernel (most calls with at least 1024 groups of 8 listed neurons over samples and token blocks) at the
edges of its tiles and stages, and the calls of that size that the other kernels take, against the float64 oracle within the bf16 bar, and Eq. 4 through it."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gpu_helpers import TOL_BF16, compact, dev_weights, errors, run_anchor, run_delta, run_layer  # noqa: E402

# d, d_ff, T, B, longest list, norm
CASES = [
    (96, 300, 3, 70, 131, "random"),    # a last stage of 32 columns; one token tile
    (32, 300, 17, 40, 250, "none"),     # one half stage only; two token tiles
    (160, 400, 130, 8, 380, "ones"),    # three token blocks of 48 rows
    (512, 700, 64, 16, 600, "random"),  # full token block, whole stages
    (2080, 800, 20, 12, 700, "random"), # more than 64 norm partials per row
    (64, 2600, 51, 8, 2561, "none"),    # one stage; lists of 81 chunks, 12 groups per workgroup
    (320, 9000, 5, 1, 8201, "ones"),    # one sample
    # Calls of the same size on either side of the rule that chooses between the tiled kernel and the others.
    (256, 8300, 5, 1, 8192, "random"),    # pipelined, 256 workgroups of 4 groups
    (256, 8300, 5, 1, 8193, "random"),    # tiled (514 workgroups of 2)
    (256, 4200, 20, 8, 4096, "none"),     # pipelined, 512 workgroups of 8, two per compute unit
    (512, 8300, 33, 3, 8192, "random"),   # pipelined, 768 workgroups of 4, two per compute unit
    (512, 8300, 32, 3, 8192, "random"),   # tiled: half of the pipelined kernel's 64 tokens
    (512, 16400, 3, 1, 16384, "none"),    # tiled
    (96, 4200, 130, 8, 4096, "ones"),     # staged, three token blocks
]


@pytest.mark.parametrize("d,d_ff,T,B,k,norm", CASES)
def test_tiled_gateup_edges(d, d_ff, T, B, k, norm):
    layer = wl.make_layer(92, d, d, d_ff, "bf16", norm=norm)
    x = wl.make_x(92, (B, T, d), d_ff, T)
    counts = [k] if B == 1 else [(k, 0, 1, k - 7, k // 2, 33, k - 1, 8)[b % 8] for b in range(B)]
    masks = wl.ragged_masks(92, d_ff, counts, d, T)
    idx, cnt = compact(masks)
    y = run_layer(dev_weights(layer), x, idx, cnt, k)
    wg, wu, wd, g = layer.f64()
    refs = np.stack([oracle.masked_ffn(x[b], wg, wu, wd, masks[b].astype(np.float64), g) for b in range(B)])
    for b, c in enumerate(counts):
        if c == 0:
            assert np.array_equal(y[b].view(np.uint32), x[b].view(np.uint32))
        elif b < 16:
            ey, ed = errors(y[b], refs[b], x[b])
            assert ey <= TOL_BF16 and ed <= TOL_BF16, f"sample {b} count {c}: rel err y {ey:.3e}, delta {ed:.3e}"
    # Every sample, those of one count together: the input's rounding is relative to the products, not to their sum, so one
    # neuron whose up sum cancels (-0.009 out of products of 0.1 in sample 66 of the first case) is 5 % off by itself.
    for c in sorted(set(counts) - {0}):
        same = [b for b in range(B) if counts[b] == c]
        ey, ed = errors(y[same], refs[same], x[same])
        assert ey <= TOL_BF16 and ed <= TOL_BF16, f"samples of count {c}: rel err y {ey:.3e}, delta {ed:.3e}"
    assert np.isfinite(y).all()


def test_tiled_gateup_anchor_and_delta():
    # At the anchor's own input h - h_a is exactly zero, so the delta step returns the anchor's y bit for bit; at another
    # input it follows Eq. 4 in float64.
    d, d_ff, T, B, L, k = 160, 500, 9, 20, 2, 420
    layers = [wl.make_layer(93, l, d, d_ff, "bf16", norm="random") for l in range(L)]
    x = wl.make_x(93, (B, T, d), 0)
    masks = np.stack([wl.ragged_masks(93, d_ff, [k - 11 * b for b in range(B)], l) for l in range(L)])
    idx, cnt = compact(masks.reshape(L * B, d_ff))
    dev = [dev_weights(l) for l in layers]
    y_a, ya, ha = run_anchor(dev, x, idx, cnt, k)
    assert np.array_equal(run_delta(dev, x, idx, cnt, k, ya, ha).view(np.uint32), y_a.cpu().numpy().view(np.uint32))
    x2 = wl.perturb(x, wl.make_noise(93, x.shape, 1, scale=0.1))
    y = run_delta(dev, x2, idx, cnt, k, ya, ha)
    for b in (0, 7, B - 1):
        ref, at = x2[b].astype(np.float64), x[b].astype(np.float64)
        for l in range(L):
            w = layers[l].f64()
            m = masks[l, b].astype(np.float64)
            f_a = oracle.dense_ffn(at, *w) - at
            delta = (oracle.masked_ffn(ref, *w[:3], m, w[3]) - ref) - (oracle.masked_ffn(at, *w[:3], m, w[3]) - at)
            ref, at = ref + f_a + delta, at + f_a
        ey, ed = errors(y[b], ref, x2[b])
        assert ey <= TOL_BF16 and ed <= TOL_BF16, f"sample {b}: rel err y {ey:.3e}, delta {ed:.3e}"
