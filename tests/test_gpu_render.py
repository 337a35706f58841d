"""GPU parity of the sample-streaming volume renderer (Sec. IV) against the oracle.

Ray setup and sample positions are float32 round-to-nearest in the same
operation order on both sides, so every ray has the same samples; what
differs is the INR evaluation (fp32 within 1e-5, the bf16 MLP within 1e-2)
and the compositing arithmetic.  Bars: fp32 images within 5e-5 per channel;
mixed precision (oracle on the fp16 / bf16 working copy) within 2e-2; with
early termination, a pixel whose stopping sample differs may move by at most
the opacity left at the limit.
"""
import sys

import numpy as np
import pytest
import torch

from fixtures import gaussian_sum_field, init_param_draws
from oracle import dvnr_oracle as o

pytestmark = pytest.mark.gpu

ENC, MLP = o.Encoding(5, 2, 12, 4, 2.0), o.MLP(2, 32)


def say(msg):
    print(f"[gpu-render] {msg}", flush=True)
    sys.stdout.flush()


def _model(precision, samples_cap=1 << 13):
    from paper_2304_10516_amd.dvnr import DVNR, EncodingCfg, MlpCfg, OptimCfg
    e = EncodingCfg(ENC.n_levels, ENC.n_features, ENC.log2_table_size, ENC.base_resolution,
                    ENC.per_level_scale, ENC.finest_resolution)
    vol = gaussian_sum_field(24, seed=8)
    model = DVNR(e, MlpCfg(MLP.n_hidden_layers, MLP.width), [((24, 24, 24), 0)], OptimCfg(lr=1e-2),
                 precision=precision, max_batch=samples_cap, seed=1)
    model.bind_volumes([torch.as_tensor(vol, device="cuda")])
    lay = o.layout(ENC, MLP)
    p = init_param_draws(lay.n_table_params, lay.mlp_shapes, seed=6).astype(np.float64)
    p[:lay.n_table_params] = np.random.default_rng(6).normal(size=lay.n_table_params) * 0.4
    model.load_params([p])
    if precision == "mixed":
        nt = lay.n_table_params
        w = torch.tensor(p[nt:]).to(torch.bfloat16).to(torch.float64).numpy()
        pe = np.concatenate([p[:nt].astype(np.float16).astype(np.float64), w])
    else:
        pe = model.block_params(0).cpu().numpy().astype(np.float64)
    return model, lay, pe, float(vol.min()), float(vol.max())


TF = np.array([[0.1, 0.2, 0.9, 0.0], [0.2, 0.8, 0.3, 0.2], [0.9, 0.7, 0.1, 0.5], [1.0, 0.2, 0.1, 0.9]])


@pytest.mark.parametrize("precision,eye,spr", [("fp32", (1.9, 1.4, 2.3), 64), ("fp32", (0.6, 0.5, 0.4), 7),
                                               ("mixed", (-0.9, 1.6, 1.7), 32)])
def test_render_matches_oracle(precision, eye, spr):
    say(f"render {precision} eye={eye} samples_per_round={spr}")
    model, lay, pe, vmin, vmax = _model(precision)
    cam = o.Camera(eye=eye, center=(0.5, 0.5, 0.5), up=(0.0, 1.0, 0.0), fovy_deg=50.0, width=40, height=30)
    lo, hi = vmin - 0.1 * (vmax - vmin), vmax
    dt, ref = 1.0 / 40, 1.0 / 64
    img = model.render(0, cam.eye, cam.center, cam.up, cam.fovy_deg, cam.width, cam.height,
                       torch.tensor(TF, dtype=torch.float32), (lo, hi), dt, ref, samples_per_round=spr)
    torch.cuda.synchronize()
    ref_img = o.render(lay, pe, vmin, vmax, cam, TF, lo, hi, dt, ref)
    err = np.abs(img.cpu().numpy() - ref_img)
    say(f"max abs diff {err.max():.3e}, covered pixels {(ref_img[..., 3] > 0).mean():.2f}")
    assert (ref_img[..., 3] > 0).mean() > 0.2
    assert err.max() <= (5e-5 if precision == "fp32" else 2e-2)


def test_render_early_termination():
    say("render fp32 with early termination at A >= 0.8")
    model, lay, pe, vmin, vmax = _model("fp32")
    cam = o.Camera(eye=(1.9, 1.4, 2.3), center=(0.5, 0.5, 0.5), up=(0.0, 1.0, 0.0), fovy_deg=50.0, width=40,
                   height=30)
    tf = TF.copy()
    tf[:, 3] = np.minimum(1.0, tf[:, 3] * 3)
    lo, hi = vmin, vmax
    dt, ref = 1.0 / 40, 1.0 / 64
    img = model.render(0, cam.eye, cam.center, cam.up, cam.fovy_deg, cam.width, cam.height,
                       torch.tensor(tf, dtype=torch.float32), (lo, hi), dt, ref, alpha_stop=0.8,
                       samples_per_round=16).cpu().numpy()
    ref_img = o.render(lay, pe, vmin, vmax, cam, tf, lo, hi, dt, ref, alpha_stop=0.8)
    err = np.abs(img - ref_img)
    stopped = ref_img[..., 3] >= 0.8
    covered = ref_img[..., 3] > 0
    say(f"covered pixels {covered.mean():.2f}, stopped {stopped.mean():.2f}, max abs diff {err.max():.3e}")
    assert stopped.sum() > 0.5 * covered.sum() > 0
    assert np.all(img[..., 3][stopped] >= 0.8)
    assert np.mean(err.max(axis=-1) <= 5e-5) >= 0.99
    assert err.max() <= 0.2 + 5e-5  # the opacity left at the limit bounds a shifted stopping sample


def test_render_long_rays_over_several_launches():
    """A step so small that a ray's samples take two launches (4096 samples
    each): image and sample count as if they were one march.  Each of the n
    compositing steps rounds (C, A) once more than the oracle's."""
    say("render fp32, thousands of samples per ray")
    model, lay, pe, vmin, vmax = _model("fp32")
    cam = o.Camera(eye=(1.9, 1.4, 2.3), center=(0.5, 0.5, 0.5), up=(0.0, 1.0, 0.0), fovy_deg=40.0, width=9, height=7)
    lo, hi = vmin - 0.1 * (vmax - vmin), vmax
    dt, ref = 1.0 / 6000, 1.0 / 8
    for stop in (1.0, 0.7):
        img = model.render(0, cam.eye, cam.center, cam.up, cam.fovy_deg, cam.width, cam.height,
                           torch.tensor(TF, dtype=torch.float32), (lo, hi), dt, ref, alpha_stop=stop,
                           samples_per_round=50).cpu().numpy()
        ref_img = o.render(lay, pe, vmin, vmax, cam, TF, lo, hi, dt, ref, alpha_stop=stop)
        org, d = o.camera_rays(cam)
        t0, t1 = o.ray_box(org, d)
        n = max(int((t1 - t0).max() / dt), 1)
        assert n > 4096
        err = np.abs(img - ref_img).max()
        # the sample that reaches the limit may shift by a few, each of opacity 1 - (1 - 0.9)^(dt / ref) at most
        slack = 5e-5 + n * 2.0 ** -24 + (0.0 if stop == 1.0 else 4 * (1 - 0.1 ** (dt / ref)))
        say(f"alpha_stop {stop}: max abs diff {err:.2e} (bar {slack:.2e}), {model.last_render_samples} samples")
        assert err <= slack
        if stop == 1.0 and ref_img[..., 3].max() < 1.0:
            rounds = 0
            for a, b in zip(t0[t1 > t0], t1[t1 > t0]):
                k = np.arange(int((b - a) / dt) + 3)
                rounds += int((~o.sample_params(a, b, dt, k)[1]).argmax()) // 50 + 1
            assert model.last_render_samples == rounds * 50
