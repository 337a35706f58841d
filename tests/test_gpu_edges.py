"""The records of the destination-partitioned encoding backward, which hold the
two corners of a cell edge along x, where they can go wrong: edges that cross
slices (dense, and hashed beyond a slice's entries), points whose x weight the
packed record cannot hold (inside the first cell's first quarter), points on
the last plane, tiles with more single corners than one round stages and
buckets that overflow.

Bar: 1e-5 as for every fp32 gradient, and what the fp32 position x (R - 1) is
off: R 2^-24 an axis against weights of 0.58 rms, three axes, so 6 R 2^-24.
Entries that no contribution reaches stay exactly zero."""
import numpy as np
import pytest
import torch

from fixtures import gaussian_sum_field, init_param_draws
from oracle import dvnr_oracle as o
from tests.test_gpu_parity import dev, make, normwise

pytestmark = pytest.mark.gpu

# (features, part_slice, samples, points)
CASES = [(2, 4096, 65536, "uniform"), (2, 8192, 4096, "first"), (2, 16384, 4099, "last"), (2, 4096, 5000, "mixed"),
         (1, 4096, 65536, "uniform"), (4, 4096, 5000, "mixed"), (8, 4096, 4099, "last"), (8, 4096, 65536, "uniform")]


@pytest.mark.parametrize("F,slice_floats,n,points", CASES)
def test_edge_records(F, slice_floats, n, points):
    print(f"[edges] F={F} slice {slice_floats} n={n} {points}", flush=True)
    cfg = (o.Encoding(3, F, 13, 18, 4.0), o.MLP(1, 16))  # 18^3 dense, 72^3 and 288^3 hashed to 2^13
    lay = o.layout(*cfg)
    dims = (32, 30, 28)
    vol = gaussian_sum_field(32, seed=3)[:dims[2], :dims[1], :dims[0]].copy()
    model = make(cfg, [(dims, 0)], precision="fp32", max_batch=1 << 16, seed=1)
    model.bind_volumes([dev(vol)])
    p = np.abs(init_param_draws(lay.n_table_params, lay.mlp_shapes, seed=2).astype(np.float64))
    p[:lay.n_table_params] *= 1e3
    model.load_params([p])
    for k, v in (("apply_update", 0), ("use_graph", 0), ("scatter_part", 0), ("part_slice", slice_floats)):
        model.set_option(k, v)
    r = np.random.RandomState(9)
    x = r.rand(n, 3).astype(np.float32)
    some = r.rand(n) < (0.5 if points == "mixed" else 1.0)
    if points in ("first", "mixed"):  # any binary exponent down to 2^-40
        x[some, 0] = np.ldexp(r.rand(n), -r.randint(6, 40, n)).astype(np.float32)[some]
    if points == "last":
        x[:, r.randint(3)] = 1.0
        x[: n // 2, 0] = 1.0
    loss = model.train_step_coords(dev(x), [n])
    assert model.partitioned_levels() == 0
    pref = model.block_params(0).cpu().numpy().astype(np.float64)
    tgt = o.normalized_targets(vol, dims, 0, x)
    want, g, _ = o.loss_and_grad(lay, pref, x, tgt)
    got = model.block_grads(0).cpu().numpy()
    assert abs(loss[0].item() - want) <= 1e-5 * want
    for l, lv in enumerate(lay.levels):
        a, b = lv.off * F, (lv.off + lv.E) * F
        assert normwise(got[a:b], g[a:b]) <= 1e-5 + 6 * lv.R * 2.0 ** -24, f"level {l}"
        assert (got[a:b][g[a:b] == 0] == 0).all(), f"level {l}"
