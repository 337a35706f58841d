"""The fused decode, and queries at coordinates, against the float64 oracle's
inference, at the sizes its choices turn on: input widths of one, two and four
lane groups (up to 8, 16 and 32 features), every feature count, grids with
ragged and thin sides around the 16 x 4 x 4 brick, one brick and runs of them,
and levels so fine that a brick's vertex box is gathered instead of staged.

Tolerances are the repository's: fp32 1e-5 and bf16 1e-2 of the largest
magnitude.
"""
import numpy as np
import pytest
import torch

from oracle import dvnr_oracle as o
from tests.test_gpu_parity import make, normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("levels,features,hidden,width", [
    (4, 2, 1, 16), (5, 1, 2, 32), (2, 4, 3, 64), (1, 8, 1, 16),       # one lane group
    (8, 2, 2, 16), (16, 1, 3, 32), (3, 4, 2, 64), (2, 8, 1, 64),      # two
    (16, 2, 2, 64), (9, 2, 3, 64), (8, 4, 3, 16), (4, 8, 1, 32)])     # four
@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_decode_shapes(levels, features, hidden, width, precision):
    enc = o.Encoding(levels, features, 12, 4, 1.5 if levels > 8 else 2.2)  # finest far above the voxel grids
    mlp = o.MLP(hidden, width)
    lay = o.layout(enc, mlp)
    sizes = [(1, 1, 2), (16, 4, 4), (17, 5, 3), (33, 9, 6), (70, 41, 40)]
    rng = np.random.default_rng(levels * 10 + features)
    model = make((enc, mlp), [(d, 1) for d in sizes], precision=precision)
    model.bind_volumes([torch.rand((d[2] + 2, d[1] + 2, d[0] + 2), device="cuda") for d in sizes])
    p = rng.uniform(-0.5, 0.5, lay.n_params).astype(np.float32)
    model.load_params([p] * len(sizes))
    lo, hi = model.ranges()
    p64 = p.astype(np.float64)
    if precision == "mixed":  # the oracle evaluates the rounded working copy
        tab = p[:lay.n_table_params].astype(np.float16).astype(np.float64)
        p64 = np.concatenate([tab, torch.tensor(p[lay.n_table_params:]).to(torch.bfloat16).double().numpy()])
    for b, dims in enumerate(sizes):
        print(f"[decode] {levels}x{features} {hidden}x{width} {precision} {dims}", flush=True)
        ref = o.decode(lay, p64, dims, lo[b], hi[b]) - lo[b]
        got = model.decode(b).cpu().numpy().astype(np.float64) - lo[b]
        # the value range's offset rounds the fp32 output once more
        tol = 1e-5 + 2e-7 / np.abs(ref).max() if precision == "fp32" else 1e-2
        assert normwise(got, ref) < tol, (dims, normwise(got, ref))


@pytest.mark.parametrize("levels,features,hidden,width", [
    (4, 2, 1, 16), (2, 4, 3, 64), (1, 8, 2, 32), (16, 1, 3, 32), (2, 8, 1, 64), (16, 2, 2, 64), (9, 2, 1, 16),
    (8, 4, 3, 16), (3, 8, 2, 64)])
@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_sample_routes(levels, features, hidden, width, precision):
    """Sample counts at the edges of a wave's and a workgroup's share and on
    both sides of the one-kernel / two-pass choice; a point has the same value
    whatever the route and whatever else is asked with it."""
    enc = o.Encoding(levels, features, 12, 4, 1.4 if levels > 8 else 2.0)
    mlp = o.MLP(hidden, width)
    lay = o.layout(enc, mlp)
    rng = np.random.default_rng(levels * 10 + features)
    model = make((enc, mlp), [((6, 5, 4), 1)] * 2, precision=precision, max_batch=1 << 17)
    model.bind_volumes([torch.rand((6, 7, 8), device="cuda") for _ in range(2)])
    p = rng.uniform(-0.5, 0.5, lay.n_params).astype(np.float32)
    model.load_params([rng.uniform(-0.5, 0.5, lay.n_params).astype(np.float32), p])
    lo, hi = model.ranges()
    p64 = p.astype(np.float64)
    if precision == "mixed":
        tab = p[:lay.n_table_params].astype(np.float16).astype(np.float64)
        p64 = np.concatenate([tab, torch.tensor(p[lay.n_table_params:]).to(torch.bfloat16).double().numpy()])
    x = rng.random((140001, 3)).astype(np.float32)
    x[:6] = [[0, 0, 0], [1, 1, 1], [0, 1, 0.5], [-0.5, 0.5, 2.0], [1, 0, 0], [0.999999, 0.5, 1]]
    ref = o.infer(lay, p64, np.clip(x[:9000], 0, 1)) * (hi[1] - lo[1])
    xd = torch.as_tensor(x, device="cuda")
    whole = model.sample(1, xd)
    tol = 1e-5 + 2e-7 / np.abs(ref).max() if precision == "fp32" else 1e-2
    assert normwise(whole[:9000].cpu().numpy().astype(np.float64) - lo[1], ref.reshape(-1)) < tol
    for n in (1, 16, 17, 63, 65, 257, 1000, 8192, 8193, 32768, 32769, 131072, 131073):
        assert torch.equal(model.sample(1, xd[:n]), whole[:n]), n
