"""The whole-table encoding backward (levels whose gradient table fits LDS)
against the float64 oracle: tables at and below both LDS sizes (8192 and 16384
accumulators), dense and hashed, every feature count, one chunk and many,
ragged sample counts and several blocks.  The bar is the fp32 gradients' 1e-5
of the largest magnitude; all parameters are positive, so that no hidden unit
lies at its ReLU kink."""
import numpy as np
import pytest
import torch

from fixtures import gaussian_sum_field, init_param_draws
from oracle import dvnr_oracle as o
from tests.test_gpu_parity import dev, make, normwise

pytestmark = pytest.mark.gpu


def _model(cfg, dims, seed=31, max_batch=1 << 15):
    lay = o.layout(*cfg)
    vols = [gaussian_sum_field(32, seed=3 + b)[:d[2], :d[1], :d[0]].copy() for b, d in enumerate(dims)]
    model = make(cfg, [(d, 0) for d in dims], precision="fp32", max_batch=max_batch, seed=seed)
    model.bind_volumes([dev(v) for v in vols])
    ps = []
    for b in range(len(dims)):
        p = np.abs(init_param_draws(lay.n_table_params, lay.mlp_shapes, seed=2 + b).astype(np.float64))
        p[:lay.n_table_params] *= 1e3
        ps.append(p)
    model.load_params(ps)
    model.set_option("spatial_sort", 1)
    model.set_option("apply_update", 0)
    return lay, vols, model


# (levels, features, log2 T, base, scale, samples)
CASES = [(4, 2, 12, 4, 2.0, 4096), (4, 4, 11, 8, 2.0, 20000), (8, 1, 13, 4, 1.5, 257), (4, 8, 10, 4, 1.8, 1000),
         (4, 8, 11, 8, 2.0, 5001), (6, 1, 14, 8, 1.6, 300), (4, 2, 13, 20, 1.1, 9999), (3, 4, 12, 2, 3.0, 1)]


@pytest.mark.parametrize("L,F,T,base,scale,n", CASES)
def test_whole_table_gradient(L, F, T, base, scale, n):
    cfg = (o.Encoding(L, F, T, base, scale), o.MLP(2, 32))
    print(f"[table] {L}x{F} T=2^{T} n={n}", flush=True)
    dims = (32, 30, 28)
    lay, (vol,), model = _model(cfg, [dims])
    loss = model.train(1, n, want_loss=True)
    assert model.partitioned_levels() == L
    x = o.training_coords(31, 0, 0, n)
    tgt = o.normalized_targets(vol, dims, 0, x)
    p = model.block_params(0).cpu().numpy().astype(np.float64)
    want, g, _ = o.loss_and_grad(lay, p, x, tgt)
    got = model.block_grads(0).cpu().numpy()
    assert abs(loss[0, 0].item() - want) <= 1e-5 * want
    for l, lv in enumerate(lay.levels):
        a, b = lv.off * F, (lv.off + lv.E) * F
        assert normwise(got[a:b], g[a:b]) <= 1e-5, f"level {l}"


def test_whole_table_gradient_of_blocks():
    """Several blocks, one of them too small to draw a sample: its gradient stays zero."""
    cfg = (o.Encoding(4, 2, 12, 4, 2.0), o.MLP(1, 16))
    dims = [(32, 30, 28), (2, 2, 2), (17, 32, 9)]
    lay, vols, model = _model(cfg, dims)
    total = 4096
    n = o.apportion([int(np.prod(d)) for d in dims], total)
    assert n[1] == 0
    model.train(1, total)
    for b in range(3):
        got = model.block_grads(b).cpu().numpy()[:lay.n_table_params]
        if n[b] == 0:
            assert not got.any()
            continue
        x = o.training_coords(31, b, 0, int(n[b]))
        p = model.block_params(b).cpu().numpy().astype(np.float64)
        _, g, _ = o.loss_and_grad(lay, p, x, o.normalized_targets(vols[b], dims[b], 0, x))
        assert normwise(got, g[:lay.n_table_params]) <= 1e-5, b


def test_whole_table_keeps_nonfinite_gradients():
    """An infinite weight makes dL/dy infinite or NaN: the entries that the
    direct backward leaves non-finite are non-finite here too."""
    cfg = (o.Encoding(4, 2, 12, 4, 2.0), o.MLP(1, 16))
    masks = []
    for priv in (-1, 0):
        lay, _, model = _model(cfg, [(32, 30, 28)])
        model.set_option("priv_levels", priv)
        with torch.no_grad():
            model.block_params(0)[-1] = float("inf")
        model.train(1, 2000)
        masks.append(torch.isfinite(model.block_grads(0)[:lay.n_table_params]))
    assert torch.equal(*masks) and not masks[0].all()
