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

import paper_2609_19104_amd as rm  # noqa: E402
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
    (544, 700, 65, [201, 333], 340, "random"),     # three token blocks
    (1056, 520, 64, [500, 513, 7, 130], 520, "none"),  # 64-column tiles, the last one half past d
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


# The bars are the errors of plain 8-lane dot products and short slices, each rounded once per term, on these inputs.  One
# chain of sums per wave over d / 8 columns and a list's eighth of the slots is above them (h 2.9, 5.5, 5.6; FFN 3.5, 6.8,
# 8.8), chains of 8 columns and 16 slots that are then added up are below (2.3, 3.4, 3.4; 2.8, 3.9, 4.1).
@pytest.mark.parametrize("d,d_ff,T,norm,bar_h,bar_f", [(256, 256, 8, False, 2.54, 3.02), (1024, 1229, 51, True, 5.41, 6.16),
                                                       (1024, 4096, 51, True, 5.46, 6.43)])
def test_f32_rounding_error(d, d_ff, T, norm, bar_h, bar_f):
    # Through an anchor step, which keeps h and the FFN output without the residual.  2-norm error in units of 2^-24.
    g = torch.Generator(device="cuda").manual_seed(d + d_ff + T + 1)
    draw = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
    w = [draw(d_ff, d) * 0.02 for _ in range(3)]
    gain = 1 + 0.1 * draw(d) if norm else None
    x = draw(1, T, d)
    idx = torch.arange(d_ff, dtype=torch.int32, device="cuda").view(1, 1, d_ff)
    cnt = torch.full((1, 1), d_ff, dtype=torch.int32, device="cuda")
    ya, ha = torch.empty(1, 1, T, d, device="cuda"), torch.empty(1, 1, d_ff, T, device="cuda")
    rm.rm_anchor_ffn_stack(x, torch.empty_like(x), [(*w, gain)], idx, cnt, d_ff, ya, ha,
                           rm.workspace(d, d_ff, rm.RM_F32, 1, T, d_ff))
    xd = x[0].double()
    if norm:
        xd = xd / torch.sqrt((xd * xd).mean(-1, keepdim=True) + 1e-6) * gain.double()
    a, b = xd @ w[0].double().t(), xd @ w[1].double().t()
    h = a * torch.sigmoid(a) * b
    f = h @ w[2].double()
    units = lambda got, ref: float((got.double() - ref).norm() / ref.norm()) * 2 ** 24  # noqa: E731
    eh, ef = units(ha[0, 0].t(), h), units(ya[0, 0], f)
    print(f"rounding error: h {eh:.2f}, FFN {ef:.2f} units of 2^-24")
    assert eh <= bar_h and ef <= bar_f


# d, d_ff, L, B, T, longest list.  The down kernel's forms: 64 columns x 32 tokens with the last column tile half past d; the
# list in slices with the epilogue (two for the lists, three for the dense anchor); 32 x 16 in one slice.
EQ4_CASES = [(544, 300, 2, 5, 70, 200), (64, 2300, 3, 1, 3, 1500), (96, 150, 2, 2, 17, 65)]


@pytest.mark.parametrize("d,d_ff,L,B,T,k", EQ4_CASES)
def test_f32_eq4_gates_and_stacks(d, d_ff, L, B, T, k):
    # Anchor, delta and plain stacks with output gates, y in place of x as well; a delta step at the anchor's own input is
    # the anchor bit for bit.
    layers = [wl.make_layer(94, l, d, d_ff, "f32", norm="random") for l in range(L)]
    r = np.random.default_rng(95)
    gates = [(1.0 + 0.3 * r.standard_normal((B, d))).astype(np.float32) for _ in range(L)]
    dev = [dev_weights(l) + (torch.from_numpy(g).cuda(),) for l, g in zip(layers, gates)]
    xa = wl.make_x(94, (B, T, d), d_ff, T)
    xt = (xa + 0.05 * r.standard_normal(xa.shape)).astype(np.float32)
    masks = np.stack([wl.ragged_masks(94, d_ff, [k - 7 * b for b in range(B)], l) for l in range(L)])
    idx, cnt = compact(masks.reshape(L * B, d_ff))
    to = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    ya, ha = torch.empty(L, B, T, d, device="cuda"), torch.empty(L, B, k, T, device="cuda")
    ws_d = rm.workspace(d, d_ff, rm.RM_F32, B, T, d_ff)
    ws = rm.workspace(d, d_ff, rm.RM_F32, B, T, k)
    y_a = to(xa)
    rm.rm_anchor_ffn_stack(y_a, y_a, dev, idx, cnt, k, ya, ha, ws_d, act="gelu_tanh")
    y_t, y_same, y_s, y_in = to(xt), torch.empty_like(y_a), torch.empty_like(y_a), to(xt)
    rm.rm_delta_ffn_stack(y_t, y_t, dev, idx, cnt, k, ya, ha, ws, act="gelu_tanh")
    rm.rm_delta_ffn_stack(to(xa), y_same, dev, idx, cnt, k, ya, ha, ws, act="gelu_tanh")
    rm.rm_sparse_ffn_stack(to(xt), y_s, dev, idx, cnt, k, ws, act="gelu_tanh")
    rm.rm_sparse_ffn_stack(y_in, y_in, dev, idx, cnt, k, ws, act="gelu_tanh")
    assert torch.equal(y_same, y_a) and torch.equal(y_in, y_s)
    lay = [l.f64() for l in layers]
    for b in range(B):
        g = [q[b] for q in gates]
        m = [masks[l, b].astype(np.float64) for l in range(L)]
        ra, rya, rha = oracle.anchor_stack(xa[b], lay, act="gelu_tanh", gates=g)
        rt = oracle.delta_stack(xt[b], lay, m, rya, rha, act="gelu_tanh", gates=g)
        rs = oracle.ffn_stack(xt[b], lay, m, act="gelu_tanh", gates=g)
        assert oracle.rel_err(ya[:, b].cpu().numpy().astype(np.float64), rya) <= TOL_F32
        for name, got, ref, x in (("anchor", y_a, ra, xa), ("delta", y_t, rt, xt), ("stack", y_s, rs, xt)):
            ey, ed = errors(got[b].cpu().numpy(), ref, x[b])
            assert ey <= TOL_F32 and ed <= TOL_F32, f"{name} sample {b}: rel err y {ey:.3e}, delta {ed:.3e}"
