"""Performance cases of the framework: the calls a program makes through the
Python entry points, over the sizes it makes them at.

`listed()` names the cases, `draw(rng)` gives further ones of the same ranges,
`prepare(case, seed)` builds what a program holds before the call, `run(state)`
is one pass, `work(case)` the bytes and operations a pass cannot do without,
and `exact(case, seed)` the same results in 64 bits, in plain torch.

Kinds of case:
  train   n optimizer steps of a batch of INRs (sampling, forward, loss, backward, Adam)
  until   the same under the training-length policy (per-block budget, loss checks)
  decode  every block back to its voxel grid
  sample  one block's INR at given coordinates
  render  direct volume rendering of one block's INR
  grad    the differentiable INR: forward, and backward to table and weights
"""
import math
import random

import torch

from paper_2304_10516_amd import DVNR, EncodingCfg, MlpCfg, OptimCfg
from paper_2304_10516_amd.autograd import inr

# Grids and networks of the presets: the small 64^3 block, the 256^3 block, the
# many-block workload, and a small wide-feature grid as in situ runs use.
C1 = dict(levels=4, features=2, log2_table=12, base=4, scale=2.0, finest=0, hidden=1, width=16)
C2 = dict(levels=16, features=2, log2_table=19, base=16, scale=0.0, finest=256, hidden=2, width=64)
C3 = dict(levels=16, features=2, log2_table=17, base=16, scale=0.0, finest=160, hidden=2, width=64)
INSITU = dict(levels=4, features=4, log2_table=11, base=8, scale=2.0, finest=0, hidden=2, width=16)

# A block grid: axis^3 blocks, extents lo..hi per axis (uneven cut of one field).
ONE = dict(axis=1, ghost=0, cut=0)


def _one(nx, ny, nz, ghost=0):
    return dict(ONE, nx=nx, ny=ny, nz=nz, lo=0, hi=0, ghost=ghost)


def _cut(axis, lo, hi, cut):
    return dict(axis=axis, nx=0, ny=0, nz=0, lo=lo, hi=hi, ghost=1, cut=cut)


def listed():
    train = dict(loss="l2", boundary=0.0)
    return [
        # a small model trained step after step: launches and latency count
        dict(C1, **_one(64, 64, 64), **train, name="train 64^3 small", kind="train", precision="mixed",
             samples=4096, steps=16),
        # one simulation block at full size: the time-series workload's inner loop
        dict(C2, **_one(256, 256, 256), **train, name="train 256^3", kind="train", precision="mixed",
             samples=1 << 18, steps=8),
        # many uneven partitions trained at once: the benchmark's headline step
        dict(C3, **_cut(4, 96, 160, 3), **train, name="train 64 blocks", kind="train", precision="mixed",
             samples=1 << 20, steps=4),
        # full precision on the ordered, partitioned plan
        dict(C2, **_one(128, 128, 128), **train, name="train 128^3 fp32", kind="train", precision="fp32",
             samples=1 << 17, steps=4),
        # an in situ rank: ragged block with ghosts, boundary loss, bounded training length
        dict(INSITU, **_one(216, 160, 161, 1), name="until 216x160x161 in situ", kind="until", precision="mixed",
             loss="l1", boundary=0.15, samples=1 << 16, steps=16),
        # reconstruction of one block, of every partition, and of a small fp32 model with ragged sides
        dict(C2, **_one(256, 256, 256), name="decode 256^3", kind="decode", precision="mixed"),
        dict(C3, **_cut(4, 96, 160, 3), name="decode 64 blocks", kind="decode", precision="mixed"),
        dict(C1, **_one(67, 61, 50), name="decode 67x61x50 small fp32", kind="decode", precision="fp32"),
        # queries: a probe line of few points, and a large set of scattered points
        dict(C2, **_one(64, 64, 64), name="sample 1000 points", kind="sample", precision="mixed", points=1000),
        dict(C2, **_one(64, 64, 64), name="sample 2^20 points", kind="sample", precision="mixed", points=1 << 20),
        # a picture of one block's model
        dict(C2, **_one(128, 128, 128), name="render 512x512", kind="render", precision="mixed", pixels_x=512,
             pixels_y=512, step=1.0 / 256),
        # a custom loss trained through the differentiable INR
        dict(C3, **_one(64, 64, 64), name="grad 2^16 points", kind="grad", precision="fp32", points=1 << 16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, sizes over the ranges the listed cases span."""
    kind = rng.choice(["train", "train", "until", "decode", "decode", "sample", "sample", "render", "grad"])
    features = rng.choice([1, 2, 2, 2, 4, 8])
    levels = rng.choice([v for v in (4, 5, 8, 12, 16) if v * features <= 32])
    finest = _log_int(rng, 32, 256)
    c = dict(kind=kind, levels=levels, features=features, log2_table=rng.randint(11, 19), base=rng.choice([4, 8, 16]),
             scale=0.0, finest=finest, hidden=rng.choice([1, 2, 2, 3]), width=rng.choice([16, 32, 64, 64]),
             precision=rng.choice(["mixed", "mixed", "fp32"]))
    if kind in ("train", "decode") and rng.random() < 0.4:
        lo = rng.randint(24, 64)
        c.update(_cut(2, lo, lo + rng.randint(1, 48), rng.randint(1, 1000)))
    else:
        c.update(_one(rng.randint(32, 200), rng.randint(32, 200), rng.randint(32, 200), rng.randint(0, 1)))
    if kind in ("train", "until"):
        if rng.random() < 0.3:
            c.update(loss="l1", boundary=0.15)
        else:
            c.update(loss="l2", boundary=0.0)
        n = _log_int(rng, 4096, 1 << 18)
        c.update(samples=max(8, n // 256) * 256 if c["axis"] > 1 else n, steps=rng.choice([4, 8]))
    elif kind == "sample":
        c.update(points=_log_int(rng, 200, 1 << 20))
    elif kind == "render":
        c.update(pixels_x=_log_int(rng, 64, 512), pixels_y=_log_int(rng, 64, 512),
                 step=1.0 / rng.choice([100, 128, 200, 256]))
    elif kind == "grad":
        c.update(points=_log_int(rng, 500, 1 << 17), precision="fp32")
    return c


# ---------------------------------------------------------------------------
# Geometry and inputs (made from the seed alone, on the GPU)
# ---------------------------------------------------------------------------
def _blocks(c):
    """[(dims, ghost)] and each block's first voxel in the whole field."""
    if c["axis"] == 1:
        return [((c["nx"], c["ny"], c["nz"]), c["ghost"])], [(0, 0, 0)]
    r = random.Random(c["cut"])
    ext = [[r.randint(c["lo"], c["hi"]) for _ in range(c["axis"])] for _ in range(3)]
    blocks, first = [], []
    for k in range(c["axis"]):
        for j in range(c["axis"]):
            for i in range(c["axis"]):
                blocks.append(((ext[0][i], ext[1][j], ext[2][k]), c["ghost"]))
                first.append((sum(ext[0][:i]), sum(ext[1][:j]), sum(ext[2][:k])))
    return blocks, first


def _resolutions(c):
    if c["scale"] > 0:
        b = c["scale"]
    else:
        b = math.exp(math.log(c["finest"] / c["base"]) / (c["levels"] - 1))
    return [int(math.floor(c["base"] * b ** k + 1e-6)) for k in range(c["levels"])]


def _entries(c):
    return [min(r ** 3, 1 << c["log2_table"]) for r in _resolutions(c)]


def _shapes(c):
    d = c["levels"] * c["features"]
    return [(c["width"], d)] + [(c["width"], c["width"])] * (c["hidden"] - 1) + [(1, c["width"])]


def _counts(c):
    """(table parameters, network parameters, elements per block)."""
    nt = sum(_entries(c)) * c["features"]
    nm = sum(a * b for a, b in _shapes(c))
    return nt, nm, (nt + nm + 63) // 64 * 64


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _volumes(c, seed):
    """Each block's stored voxels: a random-phase field with k^(-11/6) modes, ghosts from the field itself."""
    blocks, first = _blocks(c)
    n = max(max(f[a] + d[a] for (d, _), f in zip(blocks, first)) for a in range(3))
    r = random.Random(int(seed))
    modes = [(r.randint(-20, 20), r.randint(-20, 20), r.randint(-20, 20)) for _ in range(48)]
    modes = [m for m in modes if any(m)]
    amp = torch.tensor([sum(v * v for v in m) ** (-11.0 / 12.0) for m in modes], device="cuda")
    phase = torch.tensor([r.uniform(0, 2 * math.pi) for _ in modes], device="cuda")
    k = torch.tensor(modes, dtype=torch.float32, device="cuda") * (2 * math.pi / n)
    out = []
    for (d, g), f in zip(blocks, first):
        ax = [torch.arange(-g, d[a] + g, device="cuda", dtype=torch.float32) + (f[a] + 0.5) for a in range(3)]
        x, y, z = (torch.polar(torch.ones((), device="cuda"), ax[a][:, None] * k[None, :, a]) for a in range(3))
        z = z * torch.polar(amp, phase)
        zy = (z[:, None, :] * y[None, :, :]).reshape(-1, len(modes))
        v = zy.real.contiguous() @ x.real.t().contiguous() - zy.imag.contiguous() @ x.imag.t().contiguous()
        out.append(v.reshape(d[2] + 2 * g, d[1] + 2 * g, d[0] + 2 * g))
    return out


def _parameters(c, seed):
    """A trained model's parameters, block after block: tables U(-0.1, 0.1), Glorot-uniform weights."""
    nt, nm, stride = _counts(c)
    nb = len(_blocks(c)[0])
    p = torch.empty((nb, stride), device="cuda").uniform_(-0.1, 0.1, generator=_generator(seed))
    at = nt
    for a, b in _shapes(c):
        p[:, at:at + a * b] *= 10.0 * math.sqrt(6.0 / (a + b))
        at += a * b
    p[:, nt + nm:] = 0.0
    return p


def _moments(c, seed):
    """Adam's moments of a run under way, at the size its gradients have."""
    nt, nm, stride = _counts(c)
    nb = len(_blocks(c)[0])
    g = _generator(seed)
    size = torch.full((stride,), 0.3 * nb / c["samples"], device="cuda")
    size[nt:] = 0.03
    size[nt + nm:] = 0.0
    m = torch.empty((nb, stride), device="cuda").uniform_(-1, 1, generator=g) * size
    v = torch.empty((nb, stride), device="cuda").uniform_(0.5, 1.5, generator=g) * size * size
    return m, v


def _points(c, seed):
    return torch.rand((c["points"], 3), device="cuda", generator=_generator(seed + 7))


def _upstream(c, seed):
    return torch.randn(c["points"], device="cuda", generator=_generator(seed + 9)) / c["points"]


CAMERA = dict(eye=(1.6, 1.3, 2.1), center=(0.5, 0.5, 0.5), up=(0.0, 1.0, 0.0), fovy_deg=45.0)
TRANSFER = [[0.05, 0.1, 0.6, 0.0], [0.1, 0.6, 0.7, 0.05], [0.9, 0.8, 0.2, 0.3], [1.0, 0.3, 0.1, 0.8]]
REF_STEP = 1.0 / 256

OPTIM = dict(lr=1e-2, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=1e-9)


def _model(c, seed, max_batch):
    blocks, _ = _blocks(c)
    enc = EncodingCfg(c["levels"], c["features"], c["log2_table"], c["base"], c["scale"], c["finest"])
    m = DVNR(enc, MlpCfg(c["hidden"], c["width"]), blocks, OptimCfg(**OPTIM), precision=c["precision"],
             max_batch=max_batch, seed=int(seed))
    m.bind_volumes(_volumes(c, seed))
    nt, nm, _ = _counts(c)
    m.load_params([p[:nt + nm] for p in _parameters(c, seed)])
    return m


_STREAM = []


def _stream():
    """The program's stream (step graphs are replayed on a stream of one's own)."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def prepare(case, seed):
    c = case
    s = {"case": c, "stream": _stream()}
    if c["kind"] in ("train", "until"):
        m = s["model"] = _model(c, seed, max(256, c["samples"]))
        mom, vel = _moments(c, seed + 1)
        m.adam_m.copy_(mom.reshape(-1))
        m.adam_v.copy_(vel.reshape(-1))
        m.set_loss(c["loss"], c["boundary"])
        if c["precision"] == "fp32":  # the plan that mixed precision has by default
            big = m.enc.n_levels
            while big > 0 and m.level_info()[3][big - 1] >= 1 << 15:
                big -= 1
            m.set_option("spatial_sort", 1)
            m.set_option("scatter_grouped", 1)
            m.set_option("scatter_part", big)
    elif c["kind"] == "decode":
        s["model"] = _model(c, seed, 1 << 18)
        s["grids"] = [torch.empty((d[2], d[1], d[0]), device="cuda") for d, _ in s["model"].blocks]
    elif c["kind"] == "sample":
        s["model"] = _model(c, seed, 1 << 18)
        s["points"] = _points(c, seed)
    elif c["kind"] == "render":
        m = s["model"] = _model(c, seed, 1 << 18)
        lo, hi = m.ranges()
        s["range"] = (lo[0], hi[0])
        s["tf"] = torch.tensor(TRANSFER, device="cuda")
    else:
        m = s["model"] = _model(c, seed, 1 << 18)
        nt, nm, _ = _counts(c)
        s["points"], s["dout"] = _points(c, seed), _upstream(c, seed)
        s["table"] = m.block_params(0)[:nt].clone().requires_grad_()
        s["weights"] = m.block_params(0)[nt:].clone().requires_grad_()
    torch.cuda.synchronize()
    return s


def run(state):
    s, c = state, state["case"]
    m = s["model"]
    with torch.cuda.stream(s["stream"]):
        if c["kind"] == "train":
            loss = m.train(c["steps"], c["samples"], want_loss=True)
            return {"loss": loss, "params": m.params, "m": m.adam_m, "v": m.adam_v}
        if c["kind"] == "until":
            steps, avg = m.train_until(c["samples"], min_steps=c["steps"], epochs=0, loss_threshold=1e-6,
                                       window=4, check_every=4)
            return {"steps": steps, "avg": avg, "params": m.params, "m": m.adam_m, "v": m.adam_v}
        if c["kind"] == "decode":
            return [m.decode(b, out=g) for b, g in enumerate(s["grids"])]
        if c["kind"] == "sample":
            return m.sample(0, s["points"])
        if c["kind"] == "render":
            return m.render(0, width=c["pixels_x"], height=c["pixels_y"], tf=s["tf"], tf_range=s["range"],
                            step=c["step"], ref_step=REF_STEP, samples_per_round=64, **CAMERA)
        out = inr(s["points"], s["table"], s["weights"], m)
        dtable, dweights = torch.autograd.grad(out, (s["table"], s["weights"]), s["dout"])
        return {"out": out.detach(), "dtable": dtable, "dweights": dweights}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    c = case
    blocks, _ = _blocks(c)
    nt, nm, _ = _counts(c)
    macs = sum(a * b for a, b in _shapes(c))
    lookup = c["levels"] * 8 * c["features"]
    te = 2 if c["precision"] == "mixed" else 4
    point = 2 * macs + 3 * lookup  # network, and weighted sums of the corners
    voxels = [d[0] * d[1] * d[2] for d, _ in blocks]
    model = lambda n: min(nt * te, n * lookup * te) + nm * te  # noqa: E731
    if c["kind"] in ("train", "until"):
        n, p = c["samples"], len(blocks) * (nt + nm)
        # parameters and moments read and written, the 16-bit copy written, the voxels that the samples meet
        by = p * (24 + (2 if te == 2 else 0)) + min(4 * sum(voxels), 32 * n) + min(p * te, n * lookup * te)
        return {"bytes": c["steps"] * by, "flops": c["steps"] * n * 3 * point}
    if c["kind"] == "decode":
        return {"bytes": sum(4 * v + model(v) for v in voxels), "flops": sum(voxels) * point}
    if c["kind"] == "sample":
        return {"bytes": 16 * c["points"] + model(c["points"]), "flops": c["points"] * point}
    if c["kind"] == "render":
        t0, t1, _ = _rays(dict(c, pixels_x=64, pixels_y=64), c["pixels_x"] / c["pixels_y"], "cpu")
        n = float((t1 - t0).clamp(min=0).sum()) / c["step"] * c["pixels_x"] * c["pixels_y"] / 4096
        return {"bytes": 16 * c["pixels_x"] * c["pixels_y"] + model(n), "flops": n * (point + 20)}
    n = c["points"]
    # coordinates, outputs and upstream gradient, the table read, its gradient cleared and written
    return {"bytes": 20 * n + model(n) + 4 * nt + min(4 * nt, 8 * n * lookup), "flops": n * 3 * point}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------
def _split(c, flat):
    """Table [entries][features] per block and its weight matrices, from one block's parameters."""
    nt = _counts(c)[0]
    ws, at = [], nt
    for a, b in _shapes(c):
        ws.append(flat[at:at + a * b].reshape(a, b))
        at += a * b
    return flat[:nt].reshape(-1, c["features"]), ws


def _corners(c, x):
    """(level, corner) -> entry indices and weights of the points x, one pair at a time."""
    off = 0
    for R, E in zip(_resolutions(c), _entries(c)):
        p = x.clamp(0, 1) * (R - 1)
        i = p.floor().clamp(max=R - 2)
        t = p - i
        i = i.long()
        for k in range(8):
            bit = (k & 1, (k >> 1) & 1, k >> 2)
            v = [i[:, a] + bit[a] for a in range(3)]
            w = math.prod(t[:, a] if bit[a] else 1 - t[:, a] for a in range(3))
            if E == R ** 3:
                e = v[0] + R * (v[1] + R * v[2])
            else:
                e = (v[0] ^ (v[1] * 2654435761) ^ (v[2] * 805459861)) & (E - 1)
            yield (off + e), w, k
        off += E


def _encode(c, table, x):
    cols, acc = [], None
    for e, w, k in _corners(c, x):
        part = w[:, None] * table[e]
        acc = part if k == 0 else acc + part
        if k == 7:
            cols.append(acc)
    return torch.cat(cols, dim=1)


def _encode_grad(c, x, dfeat, rows):
    g = torch.zeros((rows, c["features"]), dtype=torch.float64, device=x.device)
    F = c["features"]
    for n, (e, w, _) in enumerate(_corners(c, x)):
        level = n // 8
        g.index_add_(0, e, w[:, None] * dfeat[:, level * F:(level + 1) * F])
    return g


def _mlp(ws, h):
    for w in ws[:-1]:
        h = torch.relu(h @ w.t())
    return (h @ ws[-1].t())[:, 0]


def _infer(c, flat, x):
    table, ws = _split(c, flat)
    return torch.cat([_mlp(ws, _encode(c, table, q.double())) for q in x.split(1 << 20)])


def _philox(n, step, block, tag, seed):
    """Philox4x32-10 (Salmon et al., SC'11) of the counters (i, step, block, tag), i < n."""
    low = 0xFFFFFFFF

    def mul(a, b):  # 32 x 32 -> (high, low)
        p0, p1 = (a & 0xFFFF) * b, (a >> 16) * b
        return (p1 + (p0 >> 16)) >> 16, (a * b) & low

    i = torch.arange(n, dtype=torch.int64, device="cuda")
    w = [i, torch.full_like(i, step), torch.full_like(i, block), torch.full_like(i, tag)]
    k0, k1 = seed & low, (seed >> 32) & low
    for _ in range(10):
        h0, l0 = mul(0xD2511F53, w[0])
        h1, l1 = mul(0xCD9E8D57, w[2])
        w = [h1 ^ w[1] ^ k0, l1, h0 ^ w[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return w


def _draws(c, n, step, block, seed):
    """The step's sample coordinates of one block: uniform, the last ones near the faces."""
    near = int(math.floor(c["boundary"] * n + 0.5))
    u24 = lambda v: (v >> 8).double() * 2.0 ** -24  # noqa: E731
    x = torch.stack([u24(v) for v in _philox(n, step, block, 0x44564E52, seed)[:3]], dim=1)
    if near:
        u = _philox(n, step, block, 0x44564E42, seed)
        face = (u[3] * 6) >> 32
        d = (0.005 * math.sqrt(2) * torch.erfinv(u24(u[2]))).clamp(max=1)
        d = torch.where(face % 2 == 1, 1 - d, d)
        a, b = u24(u[0]), u24(u[1])
        y = torch.stack([torch.where(face < 2, d, a), torch.where(face // 2 == 1, d, torch.where(face < 2, a, b)),
                         torch.where(face // 2 == 2, d, b)], dim=1)
        x[n - near:] = y[n - near:]
    return x


def _truth(vol, dims, ghost, x):
    """Trilinear, cell-centered values of the block at x, normalized by its stored range."""
    v = vol.double()
    N = [d + 2 * ghost for d in dims]
    i, t = [], []
    for a in range(3):
        p = x[:, a] * dims[a] - 0.5 + ghost
        q = p.floor().clamp(0, N[a] - 2)
        i.append(q.long())
        t.append((p - q).clamp(0, 1))
    val = 0
    for k in range(8):
        b = (k & 1, (k >> 1) & 1, k >> 2)
        w = math.prod(t[a] if b[a] else 1 - t[a] for a in range(3))
        val = val + w * v[i[2] + b[2], i[1] + b[1], i[0] + b[0]]
    lo, hi = v.min(), v.max()
    return (val - lo) / (hi - lo)


def _apportion(c):
    voxels = [d[0] * d[1] * d[2] for d, _ in _blocks(c)[0]]
    if len(voxels) == 1:
        return [c["samples"]]
    units = c["samples"] // 256
    quota = [units * v / sum(voxels) for v in voxels]
    n = [int(q) for q in quota]
    for b in sorted(range(len(n)), key=lambda b: -(quota[b] - n[b]))[:units - sum(n)]:
        n[b] += 1
    return [256 * v for v in n]


def _exact_train(c, seed):
    blocks, _ = _blocks(c)
    vols = _volumes(c, seed)
    p = _parameters(c, seed).double()
    m, v = (t.double() for t in _moments(c, seed + 1))
    counts = _apportion(c)
    nt, nm, _ = _counts(c)
    losses = torch.zeros((c["steps"], len(blocks)), dtype=torch.float64, device="cuda")
    b1, b2 = OPTIM["beta1"], OPTIM["beta2"]
    for b, n in enumerate(counts):
        for step in range(c["steps"] if n else 0):
            x = _draws(c, n, step, b, seed)
            y = _truth(vols[b], blocks[b][0], blocks[b][1], x)
            table, ws = _split(c, p[b])
            feat = _encode(c, table, x).requires_grad_()
            ws = [w.clone().requires_grad_() for w in ws]
            r = _mlp(ws, feat) - y
            loss = r.abs().mean() if c["loss"] == "l1" else r.square().mean()
            loss.backward()
            losses[step, b] = loss.detach()
            g = torch.cat([_encode_grad(c, x, feat.grad, table.shape[0]).reshape(-1)] +
                          [w.grad.reshape(-1) for w in ws])
            t = step + 1
            q, mb, vb = p[b, :nt + nm], m[b, :nt + nm], v[b, :nt + nm]
            g += OPTIM["weight_decay"] * q
            mb.mul_(b1).add_(g, alpha=1 - b1)
            vb.mul_(b2).addcmul_(g, g, value=1 - b2)
            q.sub_(OPTIM["lr"] * (mb / (1 - b1 ** t)) / ((vb / (1 - b2 ** t)).sqrt() + OPTIM["eps"]))
    return losses, {"params": p.reshape(-1), "m": m.reshape(-1), "v": v.reshape(-1)}


def _rays(c, aspect, device):
    """Entry and exit parameter of every pixel's ray with the unit cube, and its direction."""
    f64 = dict(dtype=torch.float64, device=device)
    eye, center, up = (torch.tensor(CAMERA[k], **f64) for k in ("eye", "center", "up"))
    f = torch.nn.functional.normalize(center - eye, dim=0)
    r = torch.nn.functional.normalize(torch.linalg.cross(f, up), dim=0)
    u = torch.linalg.cross(r, f)
    tan = math.tan(math.radians(CAMERA["fovy_deg"]) / 2)
    px = (2 * (torch.arange(c["pixels_x"], **f64) + 0.5) / c["pixels_x"] - 1) * tan * aspect
    py = (1 - 2 * (torch.arange(c["pixels_y"], **f64) + 0.5) / c["pixels_y"]) * tan
    d = f + px[None, :, None] * r + py[:, None, None] * u
    d = (d / d.norm(dim=2, keepdim=True)).reshape(-1, 3)
    a, b = (0 - eye) / d, (1 - eye) / d
    t0 = torch.minimum(a, b).max(dim=1).values.clamp(min=0)
    t1 = torch.maximum(a, b).min(dim=1).values
    return t0, t1, d


def _exact_render(c, seed):
    t0, t1, d = _rays(c, c["pixels_x"] / c["pixels_y"], "cuda")
    eye = torch.tensor(CAMERA["eye"], dtype=torch.float64, device="cuda")
    vol = _volumes(c, seed)[0].double()
    lo, hi = vol.min(), vol.max()
    flat = _parameters(c, seed)[0].double()
    tf = torch.tensor(TRANSFER, dtype=torch.float64, device="cuda")
    rgba = torch.zeros((t0.numel(), 4), dtype=torch.float64, device="cuda")
    k, live = 0, (t1 > t0).nonzero()[:, 0]
    while live.numel():
        t = t0[live] + (k + 0.5) * c["step"]
        live, t = live[t < t1[live]], t[t < t1[live]]
        if not live.numel():
            break
        s = _infer(c, flat, eye + t[:, None] * d[live]).clamp(0, 1) * (len(TRANSFER) - 1)
        i = s.floor().long().clamp(max=len(TRANSFER) - 2)
        col = tf[i] + (s - i)[:, None] * (tf[i + 1] - tf[i])
        alpha = 1 - (1 - col[:, 3].clamp(0, 1)) ** (c["step"] / REF_STEP)
        w = (1 - rgba[live, 3]) * alpha
        rgba[live] += w[:, None] * torch.cat([col[:, :3], torch.ones_like(w)[:, None]], dim=1)
        k += 1
    return rgba.reshape(c["pixels_y"], c["pixels_x"], 4)


def exact(case, seed):
    c = case
    if c["kind"] == "train":
        losses, state = _exact_train(c, int(seed))
        return dict(state, loss=losses)
    if c["kind"] == "until":
        losses, state = _exact_train(c, int(seed))
        return dict(state, steps=[None], avg=[float(losses[-4:, 0].mean())])
    if c["kind"] == "render":
        return _exact_render(c, seed)
    params = _parameters(c, seed)
    if c["kind"] in ("decode", "sample"):
        grids = []
        for b, ((d, _), vol) in enumerate(zip(_blocks(c)[0], _volumes(c, seed))):
            lo, hi = vol.double().min(), vol.double().max()
            if c["kind"] == "sample":
                return _infer(c, params[b].double(), _points(c, seed)) * (hi - lo) + lo
            z, y, x = (((torch.arange(n, device="cuda") + 0.5) / n).double() for n in (d[2], d[1], d[0]))
            out = []
            for zz in z.split(max(1, (1 << 20) // (d[0] * d[1]))):
                q = torch.stack(torch.meshgrid(zz, y, x, indexing="ij"), dim=3).reshape(-1, 3).flip(1)
                out.append(_infer(c, params[b].double(), q))
            grids.append((torch.cat(out) * (hi - lo) + lo).reshape(d[2], d[1], d[0]))
        return grids
    x, dout = _points(c, seed).double(), _upstream(c, seed).double()
    nt, nm, _ = _counts(c)
    table, ws = _split(c, params[0, :nt + nm].double())
    feat = _encode(c, table, x).requires_grad_()
    ws = [w.clone().requires_grad_() for w in ws]
    out = _mlp(ws, feat)
    out.backward(dout)
    return {"out": out.detach(), "dtable": _encode_grad(c, x, feat.grad, table.shape[0]).reshape(-1),
            "dweights": torch.cat([w.grad.reshape(-1) for w in ws])}
