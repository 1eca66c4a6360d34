"""The float32 FFN kernels at the edges of their tiles, rounds and launch rules, against the float64 oracle.

Bar: TOL_F32 on y and on the FFN delta (the float32 parity bar).  A neuron no list holds has infinite weights: slots
past a list's end are computed from some neuron's rows, and nothing of them may reach a result."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from gpu_helpers import TOL_F32, compact, dev_weights, errors, run_layer  # noqa: E402

# d, d_ff, T, counts, max_count, norm
CASES = [
    (32, 40, 1, [15], 15, "random"),               # one unit of columns, one token, a partial chunk of 16 slots
    (32, 40, 16, [16], 39, "none"),                # whole token tile and chunk; max_count past the count
    (96, 300, 17, [17, 0, 250], 250, "ones"),      # three units for 8 waves; two token tiles; an empty list
    (288, 300, 32, [129], 129, "random"),          # nine units: waves with one and two
    (64, 1200, 3, [1100], 1100, "none"),           # few workgroups, over 64 chunks: two slices and the epilogue
    (64, 2300, 5, [1025, 2200], 2200, "random"),   # slices past the first sample's list
    (2048, 2304, 33, [2100], 2100, "none"),        # one slice longer than the 2048 staged indices
    (1024, 4096, 51, [1229], 1229, "random"),      # 16 neurons per gate/up workgroup
    (512, 700, 40, [300, 299, 1, 64, 65, 500, 0, 128], 500, "ones"),  # 64-column x 32-token down tiles
    (544, 700, 65, [201, 333], 340, "random"),     # three token blocks; a column tile past d
    (1056, 520, 64, [500, 513, 7, 130], 520, "none"),  # the same with 64-column tiles
]


@pytest.mark.parametrize("d,d_ff,T,counts,max_count,norm", CASES)
def test_f32_layer_edges(d, d_ff, T, counts, max_count, norm):
    layer = wl.make_layer(91, d, d, d_ff, "f32", norm=norm)
    x = wl.make_x(91, (len(counts), T, d), d_ff, T)
    masks = np.zeros((len(counts), d_ff), np.uint8)
    masks[:, 1:] = wl.ragged_masks(91, d_ff - 1, counts, d, T)  # neuron 0 is in no list
    idx, cnt = compact(masks)
    dev = dev_weights(layer)
    for w in dev[:3]:
        w[0] = float("inf")
    y = run_layer(dev, x, idx, cnt, max_count)
    wg, wu, wd, g = layer.f64()
    for b, c in enumerate(counts):
        if c == 0:
            assert np.array_equal(y[b].view(np.uint32), x[b].view(np.uint32))
            continue
        ref = oracle.masked_ffn(x[b], wg, wu, wd, masks[b].astype(np.float64), g)
        ey, ed = errors(y[b], ref, x[b])
        assert ey <= TOL_F32 and ed <= TOL_F32, f"sample {b} count {c}: rel err y {ey:.3e}, delta {ed:.3e}"
