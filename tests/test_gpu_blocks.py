"""The fp32 MLP building blocks (MFMA kernels) against the same network in
float64 torch: every compiled shape, input widths that fill a 4-wide step and
that do not, and sample counts at the edges of a 16-sample group, of a
workgroup's pass and of the rule that chooses groups per wave.

Tolerance: each value is a chain of at most 64-term fp32 sums through at most
four layers, a normwise error of a few 1e-6 at most; the bar is the 1e-5 that
the other fp32 results are held to.  A unit within fp32 rounding of its ReLU
kink may fall on either side, so dL/do is zero for samples that have one.
"""
import numpy as np
import pytest
import torch

from tests.test_gpu_parity import dev, make, normwise
from oracle import dvnr_oracle as o

pytestmark = pytest.mark.gpu


def reference(ws, x):
    h, acts, kink = x, [], torch.zeros(x.shape[0], dtype=torch.bool, device=x.device)
    for w in ws[:-1]:
        z = h @ w.t()
        kink |= (z.abs() < 1e-5 * z.abs().max()).any(dim=1)
        h = torch.relu(z)
        acts.append(h)
    return (h @ ws[-1].t())[:, 0], kink


@pytest.mark.parametrize("levels,features", [(16, 2), (3, 2), (5, 1)])
@pytest.mark.parametrize("hidden,width", [(1, 16), (2, 16), (3, 16), (1, 32), (2, 32), (3, 32), (1, 64), (2, 64), (3, 64)])
def test_mlp_blocks_fp32(levels, features, hidden, width):
    model = make((o.Encoding(levels, features, 8, 4, 1.2), o.MLP(hidden, width)), [((8, 8, 8), 0)])
    n_in = levels * features
    shapes = [(width, n_in)] + [(width, width)] * (hidden - 1) + [(1, width)]
    gen = torch.Generator(device="cuda").manual_seed(hidden * 100 + width + n_in)
    flat = torch.cat([(torch.rand(a * b, device="cuda", generator=gen) * 2 - 1) * (6.0 / (a + b)) ** 0.5 for a, b in shapes])
    for n in (1, 17, 64, 65, 32767, 32768, 40001):
        print(f"[blocks] {levels}x{features} {hidden}x{width} n={n}", flush=True)
        x = torch.rand((n, n_in), device="cuda", generator=gen) * 2 - 1
        dout = torch.rand(n, device="cuda", generator=gen) * 2 - 1
        ws, at = [], 0
        for a, b in shapes:
            ws.append(flat[at:at + a * b].double().reshape(a, b).requires_grad_())
            at += a * b
        xd = x.double().requires_grad_()
        ref, kink = reference(ws, xd)
        dout[kink] = 0.0
        grads = torch.autograd.grad(ref, [xd] + ws, dout.double())
        out = model.mlp_forward(x, flat)
        dw = torch.full_like(flat, 0.5)  # added to
        dx = model.mlp_backward(x, flat, dout, dw)
        ref_dw = torch.cat([g.reshape(-1) for g in grads[1:]])
        assert normwise(out.cpu(), ref.detach().cpu()) < 1e-5
        assert normwise(dx.cpu(), grads[0].cpu()) < 1e-5
        assert normwise((dw.double() - 0.5).cpu(), ref_dw.cpu()) < 1e-5 + 2e-7 / float(ref_dw.abs().max())


@pytest.mark.parametrize("levels,features", [(16, 2), (9, 1), (8, 4), (4, 8), (3, 1)])
def test_encode_blocks_fp32(levels, features):
    """Encoding forward and backward over sample counts at the edges of a
    256-sample tile, for both level mappings (more than 8 levels, and fewer)."""
    enc = o.Encoding(levels, features, 10, 4, 1.25)
    lay = o.layout(enc, o.MLP(1, 16))
    model = make((enc, o.MLP(1, 16)), [((8, 8, 8), 0)])
    rng = np.random.default_rng(levels)
    for n in (1, 255, 257, 1000):
        print(f"[blocks] encode {levels}x{features} n={n}", flush=True)
        x = rng.random((n, 3)).astype(np.float32)
        table = rng.uniform(-1, 1, lay.n_table_params).astype(np.float32)
        dy = rng.uniform(-1, 1, (n, levels * features)).astype(np.float32)
        g = torch.zeros(lay.n_table_params, device="cuda")
        feats = model.encode_forward(dev(x), dev(table))
        model.encode_backward(dev(x), dev(dy), g)
        assert normwise(feats.cpu(), o.encode(lay, table.astype(np.float64), x)) < 1e-5
        assert normwise(g.cpu(), o.encode_backward(lay, x, dy.astype(np.float64))) < 1e-5
