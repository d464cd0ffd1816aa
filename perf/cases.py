"""The performance cases of the framework: what its users have it do, over the range of sizes.

A case is one pass through the public entry points of `paper_2308_02494_amd`, on inputs made
from a seed alone.  Six kinds of call:

* forward -- `apmg_forward`: field values at points (probing, resampling, rendering);
* dd      -- `apmg_dd_forward`: global queries over all brick models of a domain decomposition;
* autograd -- `APMGFunction` inside a torch program: forward, loss, backward, all gradients;
* adjoint -- `apmg_backward` with caller-held outputs, for programs with their own loss;
* variant -- the hash-grid and 4-D encoders: forward, dL/df, adjoint;
* step    -- `Trainer.step`: the whole training iteration of one model or of a set of bricks.

`exact` gives the same outputs in float64 with plain torch and numpy: the integer decisions of
the encoder (which cell, inside or not) are taken in float32 with the fused multiply-adds the
paper's float32 encoder implies, the values that follow them in float64.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2308_02494_amd as A

DEV = "cuda"


# --------------------------------------------------------------------------- the cases
def listed():
    """Twelve cases from a latency-bound probe to an 80-model training step."""
    return [
        # an interactive probe: a few hundred sample positions (a line or a cursor) of a small
        # float32 model, where launches and host work are all there is
        dict(name="probe_257", kind="forward", M=16, C=2, R=16, H=64, n=257, mlp="f32", grids="f32",
             layout="paper", points="uniform"),
        # resampling the single-model network at a million scattered positions in float32
        dict(name="query_f32_1m", kind="forward", M=32, C=2, R=32, H=64, n=1000003, mlp="f32", grids="f32",
             layout="paper", points="uniform"),
        # a 1920 x 1080 frame, eight samples a ray, of the large BF16 model: the renderer's call
        dict(name="render_bf16_frame", kind="forward", M=64, C=4, R=64, H=128, n=1920 * 1080 * 8, mlp="bf16",
             grids="f32", layout="paper", points="rays"),
        # global queries over the 80 brick models of a 1000 x 1200 x 900 volume
        dict(name="dd_query_80_bricks", kind="dd", nx=1000, ny=1200, nz=900, B=256, ghost=1, M=16, C=2, R=32, H=64,
             n=4000037, mlp="bf16", grids="f32"),
        # the paper's batch of about 100,000 points through torch autograd (forward and backward)
        dict(name="autograd_f32_100k", kind="autograd", M=32, C=2, R=32, H=64, n=100003, mlp="f32", grids="f32"),
        # adjoint of the large BF16 model (64 grids at 64^3 x 4, MLP 256-128-128-1)
        dict(name="adjoint_wide_bf16", kind="adjoint", M=64, C=4, R=64, H=128, n=1 << 19, mlp="bf16", grids="f32",
             layout="paper"),
        # fine-tuning a hash grid inside each adaptive grid: forward and adjoint of one batch
        dict(name="hash_train_f32", kind="variant", enc="hash", M=8, L=4, T=1 << 16, res0=16, growth=2.0, n=1 << 20,
             mlp="f32"),
        # a time-varying field on 4-D grids: forward and adjoint of one batch
        dict(name="time_train_f32", kind="variant", enc="time", M=32, R=32, Rt=8, n=1 << 20, mlp="f32"),
        # one training step of a small model on a 64^3 volume
        dict(name="step_tiny_f32", kind="step", nx=64, ny=64, nz=64, B=64, ghost=0, M=16, C=2, R=16, H=64, n=65536,
             mlp="f32", grids="f32", density=True),
        # the benchmark's training step: 256^3 volume, 32 grids at 32^3 x 2, 2^20 points
        dict(name="step_f32_1m", kind="step", nx=256, ny=256, nz=256, B=256, ghost=0, M=32, C=2, R=32, H=64,
             n=1 << 20, mlp="f32", grids="f32", density=True),
        # mixed precision on a 1024^3 volume: BF16 MLP, FP16 gathers, 2^21 points
        dict(name="step_mixed_2m", kind="step", nx=1024, ny=1024, nz=1024, B=1024, ghost=0, M=32, C=2, R=32, H=64,
             n=1 << 21, mlp="bf16", grids="f16", density=True),
        # domain-decomposed training: 80 brick models a step, 2^17 points each
        dict(name="step_80_bricks_bf16", kind="step", nx=1000, ny=1200, nz=900, B=256, ghost=1, M=16, C=2, R=32,
             H=64, n=1 << 17, mlp="bf16", grids="f32", density=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges (kind, shape, size, dtype and option all vary)."""
    kind = rng.choice(["forward", "forward", "dd", "autograd", "adjoint", "variant", "step", "step"])
    mlp = rng.choice(["f32", "bf16"])
    grids = rng.choice(["f32", "f32", "f16"])
    if kind == "variant":
        n = _log_int(rng, 1 << 12, 1 << 20)
        if rng.random() < 0.5:
            M, L = rng.randint(2, 8), rng.randint(2, 4)
            return dict(kind=kind, enc="hash", M=M, L=L, T=1 << rng.randint(12, 17), res0=rng.randint(8, 20),
                        growth=round(rng.uniform(1.4, 2.0), 2), n=n, mlp=mlp)
        return dict(kind=kind, enc="time", M=rng.randint(4, 32), R=rng.randint(9, 32), Rt=rng.randint(2, 9), n=n,
                    mlp=mlp)
    # model shapes: the small-MLP shapes of training, or up to the wide decoder
    wide = kind in ("forward", "adjoint") and rng.random() < 0.35
    C = rng.choice([1, 2, 2, 4])
    if wide:
        M, R, H = rng.randint(17, 64), _log_int(rng, 16, 64), 128
    else:
        M, R, H = rng.randint(4, 64 // C if C > 1 else 40), _log_int(rng, 8, 40), 64
    if kind == "forward":
        return dict(kind=kind, M=M, C=C, R=R, H=H, n=_log_int(rng, 32, 1 << 21), mlp=mlp, grids=grids,
                    layout=rng.choice(["paper", "last"]), points=rng.choice(["uniform", "rays"]))
    if kind == "adjoint":
        return dict(kind=kind, M=M, C=C, R=R, H=H, n=_log_int(rng, 1 << 10, 1 << 19), mlp=mlp, grids=grids,
                    layout=rng.choice(["paper", "last"]))
    if kind == "autograd":
        return dict(kind=kind, M=M, C=C, R=R, H=H, n=_log_int(rng, 1 << 10, 1 << 18), mlp=mlp, grids="f32")
    nx, ny, nz = (rng.randint(48, 300) for _ in range(3))
    B = rng.randint(max(48, max(nx, ny, nz) // 3), 300)
    out = dict(kind=kind, nx=nx, ny=ny, nz=nz, B=B, ghost=rng.choice([1, 1, 8]), M=min(M, 24), C=C, R=min(R, 33),
               H=64, mlp=mlp, grids=grids)
    bricks = -(-nx // B) * -(-ny // B) * -(-nz // B)
    if kind == "dd":
        out["n"] = _log_int(rng, 1 << 10, 1 << 21)
    else:
        out["n"] = _log_int(rng, 1 << 11, (1 << 20) // bricks)
        out["density"] = rng.random() < 0.75
    return out


# --------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _uniform(g, shape, lo, hi):
    return torch.rand(shape, generator=g, device=DEV) * (hi - lo) + lo


def _transforms(g, M, spread=0.0):
    """The paper's initial transforms: N(1, 0.05) diagonal, N(0, 0.05) elsewhere; `spread` adds a
    translation, as trained grids that have moved over the features have."""
    G = torch.randn((M, 3, 4), generator=g, device=DEV) * 0.05
    for d in range(3):
        G[:, d, d] += 1.0
    if spread:
        G[:, :, 3] += _uniform(g, (M, 3), -spread, spread)
    return G


def _weights(g, widths):
    """Glorot-uniform weights [out][in]."""
    out = []
    for i, o in zip(widths[:-1], widths[1:]):
        lim = math.sqrt(6.0 / (i + o))
        out.append(_uniform(g, (o, i), -lim, lim))
    return out


def _points(g, n, kind="uniform"):
    """[3][n]: uniform in the cube, or the ray layout of a frame of about n samples (pixels in
    rows, eight samples a ray), moved by the seed."""
    if kind == "uniform":
        return _uniform(g, (3, n), -1.0, 1.0)
    rays = -(-n // 8)
    width = max(1, int(round(math.sqrt(rays * 16 / 9))))
    height = -(-rays // width)
    px = (torch.arange(width, device=DEV) * 2.0 + 1.0) / width - 1.0
    py = ((torch.arange(height, device=DEV) * 2.0 + 1.0) / height - 1.0) * 0.5625
    pz = (torch.arange(8, device=DEV) * 2.0 + 1.0) / 8 - 1.0
    Y, X, Z = torch.meshgrid(py, px, pz, indexing="ij")
    pts = torch.stack([X.reshape(-1), Y.reshape(-1), Z.reshape(-1)])[:, :n]
    return (pts + _uniform(g, (3, 1), -0.01, 0.01)).contiguous()


def _volume(g, nz, ny, nx):
    """A smooth field in [0, 1]: four products of one-dimensional waves."""
    vol = torch.full((nz, ny, nx), 0.5, device=DEV)
    for _ in range(4):
        ax = []
        for m in (nz, ny, nx):
            k, ph = _uniform(g, (2,), 1.0, 12.0).tolist()
            ax.append(torch.sin(torch.linspace(-1, 1, m, device=DEV) * k + ph))
        vol.addcmul_((ax[0] * 0.125)[:, None, None] * ax[1][None, :, None], ax[2][None, None, :])
    return vol


def _dtype(c):
    return A.BF16 if c["mlp"] == "bf16" else A.F32


def _grid_dtype(c):
    return torch.float16 if c.get("grids") == "f16" else torch.float32


def _levels(c):
    return [int(c["res0"] * c["growth"] ** k) for k in range(c["L"])]


def _params(c, g, spread=0.0):
    """Host-program parameters of a dense model, as trained grids hold them (U(-0.3, 0.3))."""
    M, C, R, H = c["M"], c["C"], c["R"], c["H"]
    F = _uniform(g, (M, C, R, R, R), -0.3, 0.3).to(_grid_dtype(c))
    return _transforms(g, M, spread), F, _weights(g, [M * C, H, H, 1])


def _bricks(c):
    return A.apmg_make_bricks(c["nx"], c["ny"], c["nz"], c["B"], c["ghost"])


def prepare(case, seed):
    """What a program holds before the call: parameters, points, workspaces, the trainer."""
    c, g = case, _gen(seed)
    kind = c["kind"]
    if kind in ("forward", "adjoint"):
        G, F, W = _params(c, g, 0.3 if c["H"] == 128 else 0.0)
        layout = A.GRIDS_MCRRR
        if c["layout"] == "last":
            F, layout = F.permute(0, 2, 3, 4, 1).contiguous(), A.GRIDS_MRRRC
        model = A.Model(G, F, W, 0.0, 1.0, _dtype(c), layout)
        n = c["n"]
        s = dict(c=c, model=model, pts=_points(g, n, c.get("points", "uniform")))
        op = A.OP_FORWARD if kind == "forward" else A.OP_BACKWARD
        s["ws"] = torch.empty(A._lib.apmg_workspace_bytes(op, ctypes.byref(model.struct()), n), dtype=torch.uint8,
                              device=DEV)
        if kind == "forward":
            s["out"] = torch.empty(n, device=DEV)
        else:
            s["df"] = torch.randn(n, generator=g, device=DEV) / n
            s["dF"] = torch.empty(model.F.shape, device=DEV)
            s["dG"] = torch.empty(G.shape, dtype=torch.float64, device=DEV)
            s["dW"] = [torch.empty_like(w) for w in W]
        return s
    if kind == "autograd":
        G, F, W = _params(c, g)
        pts = _points(g, c["n"]).t().contiguous()
        v = _uniform(g, (c["n"],), 0.0, 1.0)
        return dict(c=c, pts=pts, v=v, p=[t.requires_grad_(True) for t in [G, F] + W])
    if kind == "variant":
        M, n = c["M"], c["n"]
        G = _transforms(g, M)
        if c["enc"] == "hash":
            F = _uniform(g, (M, c["L"], c["T"], 2), -0.3, 0.3)
            W = _weights(g, [M * c["L"] * 2, 64, 64, 1])
            model = A.VariantModel(A.ENC_HASH, G, F, W, 0.0, 1.0, _dtype(c), level_res=_levels(c))
            pts = _points(g, n)
        else:
            F = _uniform(g, (M, 2, c["Rt"], c["R"], c["R"], c["R"]), -0.3, 0.3)
            W = _weights(g, [M * 2, 64, 64, 1])
            model = A.VariantModel(A.ENC_TIME, G, F, W, 0.0, 1.0, _dtype(c))
            pts = _uniform(g, (4, n), -1.0, 1.0)
        m, e = model.structs()
        ws = [torch.empty(A._lib.apmg_variant_workspace_bytes(op, ctypes.byref(m), ctypes.byref(e), n),
                          dtype=torch.uint8, device=DEV) for op in (A.OP_FORWARD, A.OP_BACKWARD)]
        return dict(c=c, model=model, pts=pts, v=_uniform(g, (n,), 0.0, 1.0), ws=ws,
                    out=torch.empty(n, device=DEV))
    table, bricks = _bricks(c)
    nb = len(bricks)
    M, C, R, H = c["M"], c["C"], c["R"], c["H"]
    widths = [M * C, H, H, 1]
    if kind == "dd":
        G = torch.stack([_transforms(g, M) for _ in range(nb)])
        F = _uniform(g, (nb, M, C, R, R, R), -0.3, 0.3).to(_grid_dtype(c))
        W = torch.stack([torch.cat([w.reshape(-1) for w in _weights(g, widths)]) for _ in range(nb)])
        dd = A.DDModels(G, F, W, widths, table, bricks, _dtype(c))
        n = c["n"]
        ws = torch.empty(A._lib.apmg_workspace_bytes(A.OP_DD_FORWARD, ctypes.byref(dd.struct), n), dtype=torch.uint8,
                         device=DEV)
        return dict(c=c, dd=dd, F=dd.F, pts=_points(g, n), ws=ws, out=torch.empty(n, device=DEV))
    return dict(c=c, tr=_trainer(c, g, seed, bricks, widths))


def _trainer(c, g, seed, bricks, widths):
    """A trainer in the middle of a run: moments of the size the gradients have, counters past
    the start, rates reduced as late in a run (the transforms' far enough that thousands of
    steps leave them where they are).  |det| is the density reading for long runs."""
    nb, M, C, R = len(bricks), c["M"], c["C"], c["R"]
    vol = _volume(g, c["nz"], c["ny"], c["nx"])
    hosts = [dict(G=_transforms(g, M), F=_uniform(g, (M, C, R, R, R), -0.1, 0.1), W=_weights(g, widths))
             for _ in range(nb)]
    tr = A.Trainer(hosts, vol, bricks, c["n"], seed=7 + int(seed) % 1000, mlp_dtype=_dtype(c),
                   grid_dtype=_grid_dtype(c), lr=1e-3, lr_G=1e-6, flags=A.DENSITY_ABS_DET)
    del hosts
    for m, v, size in ((tr.mF, tr.vF, 0.15 / R ** 3), (tr.mW, tr.vW, 1e-2), (tr.mG, tr.vG, 1e-4)):
        m.copy_(torch.randn(m.shape, generator=g, device=DEV) * size)
        v.copy_(_uniform(g, v.shape, 0.5, 2.0) * size ** 2)
    tr.t.fill_(200)
    tr.tG.fill_(100)
    tr.step_ctr.fill_(200 + int(seed) % 977)
    tr.density_active.fill_(1 if c["density"] else 0)
    return tr


def run(s):
    """One pass; outputs whole."""
    kind = s["c"]["kind"]
    if kind == "forward":
        return A.apmg_forward(s["model"], s["pts"], out=s["out"], ws=s["ws"])
    if kind == "dd":
        return A.apmg_dd_forward(s["dd"], s["pts"], out=s["out"], ws=s["ws"])
    if kind == "adjoint":
        dF, dG, dW = A.apmg_backward(s["model"], s["pts"], s["df"], dF=s["dF"], dG=s["dG"], dW=s["dW"], ws=s["ws"])
        return dict(dF=dF, dG=dG.to(torch.float32), dW=dW)      # the parameters' dtype, for the optimiser
    if kind == "autograd":
        G, F, W1, W2, W3 = s["p"]
        for t in s["p"]:
            t.grad = None
        f = A.APMGFunction.apply(s["pts"], G, F, W1, W2, W3, 0.0, 1.0, _dtype(s["c"]))
        ((f - s["v"]) ** 2).mean().backward()
        return dict(f=f, grads=[t.grad for t in s["p"]])
    if kind == "variant":
        f = A.apmg_variant_forward(s["model"], s["pts"], out=s["out"], ws=s["ws"][0])
        df = (f - s["v"]) * (2.0 / f.numel())
        dF, dG, dW = A.apmg_variant_backward(s["model"], s["pts"], df, ws=s["ws"][1])
        return dict(f=f, dF=dF, dG=dG.to(torch.float32), dW=dW)
    tr = s["tr"]
    tr.step()
    return dict(losses=tr.losses.to(torch.float32), F=tr.F, G=tr.G, W=tr.W, mF=tr.mF, vF=tr.vF, mG=tr.mG, vG=tr.vG,
                mW=tr.mW, vW=tr.vW)


# --------------------------------------------------------------------------- work
def work(case):
    """Bytes (each input read once, each output written once) and operations of one pass."""
    c = case
    kind, n = c["kind"], c["n"]
    H = c.get("H", 64)
    C = c.get("C", 2)
    grids = c["M"] * c.get("L", 1)
    K = grids * C
    gsz = 2 if c.get("grids") == "f16" else 4
    taps = 16 if c.get("enc") == "time" else 8
    nb = 1
    if kind in ("dd", "step"):
        nb = -(-c["nx"] // c["B"]) * -(-c["ny"] // c["B"]) * -(-c["nz"] // c["B"])
    if kind == "variant":
        values = c["M"] * c["L"] * c["T"] * 2 if c["enc"] == "hash" else c["M"] * 2 * c["Rt"] * c["R"] ** 3
    else:
        values = c["M"] * C * c["R"] ** 3
    mlp = K * H + H * H + H
    enc = grids * (24 + 2 * taps * C)
    fwd = 2 * mlp + enc
    both = fwd + 4 * mlp + grids * (2 * taps * C)           # + dL/dW, dL/dy, and the grid gradient
    if kind == "forward":
        return dict(bytes=n * 16 + values * gsz + mlp * 4, flops=n * fwd)
    if kind == "dd":
        return dict(bytes=n * 16 + nb * (values * gsz + mlp * 4), flops=n * fwd)
    if kind == "step":
        # the volume samples (8 voxels share a line pair), parameters and moments read and written
        dens = 120 * c["M"] if c["density"] else 0
        return dict(bytes=nb * (n * 8 * 4 + (values + mlp) * 4 * 6), flops=nb * n * (both + dens))
    trans = grids * (60 + 6 * taps * C)                      # the transform gradient
    return dict(bytes=n * 20 + values * (gsz + 4) + mlp * 8, flops=n * (both + trans))


# --------------------------------------------------------------------------- float64 reference
CHUNK = 1 << 17


def _fma32(a, b, c):
    return (a.double() * b.double() + c.double()).float()


def _local(G32, G64, x):
    """Local coordinates of one grid: float32 (fused, for the decisions) and float64."""
    l32, l64 = [], []
    for r in range(3):
        a = G32[r]
        l32.append(_fma32(a[2], x[2], _fma32(a[1], x[1], _fma32(a[0], x[0], a[3].expand_as(x[0])))))
        b, xd = G64[r], x.double()
        l64.append(b[0] * xd[0] + b[1] * xd[1] + b[2] * xd[2] + b[3])
    return l32, l64


def _cell(l32, l64, cells):
    """(inside, lower vertex, weights) at `cells` cells per axis."""
    h = torch.tensor(0.5 * cells, device=DEV)
    inside = torch.ones_like(l32[0], dtype=torch.bool)
    i0, w = [], []
    for a, b in zip(l32, l64):
        inside &= (a >= -1) & (a <= 1)
        u = _fma32(a, h, h.expand_as(a))
        k = torch.nan_to_num(torch.floor(u)).clamp(0, cells - 1).long()
        i0.append(torch.where(inside, k, torch.zeros_like(k)))
        w.append((b + 1) * (0.5 * cells) - k)
    i0 = [torch.where(inside, k, torch.zeros_like(k)) for k in i0]
    return inside, i0, w


def _trilinear(rows, inside, i0, w, index):
    out = 0.0
    for q in range(8):
        k = [i0[d] + ((q >> d) & 1) for d in range(3)]
        wq = 1.0
        for d in range(3):
            wq = wq * (w[d] if (q >> d) & 1 else 1.0 - w[d])
        out = out + wq[:, None] * torch.index_select(rows, 0, index(*k))
    return torch.where(inside[:, None], out, torch.zeros_like(out))


def _features(c, G64, F64, x):
    """[n][K] features of the points x [3 or 4][n] float32; F64: rows per feature grid."""
    G32 = G64.detach().float()
    feats = []
    for g in range(c["M"]):
        l32, l64 = _local(G32[g], G64[g], x[:3])
        if c.get("enc") == "hash":
            for k, N in enumerate(_levels(c)):
                inside, i0, w = _cell(l32, l64, N)
                T = c["T"]

                def index(vx, vy, vz, N=N, T=T):
                    if (N + 1) ** 3 <= T:
                        return vx + (N + 1) * (vy + (N + 1) * vz)
                    m = 0xFFFFFFFF
                    return (vx ^ ((vy * 2654435761) & m) ^ ((vz * 805459861) & m)) % T

                feats.append(_trilinear(F64[g * c["L"] + k], inside, i0, w, index))
            continue
        R = c["R"]
        inside, i0, w = _cell(l32, l64, R - 1)
        if c.get("enc") == "time":
            tau, ht = x[3], torch.tensor(0.5 * (c["Rt"] - 1), device=DEV)
            ut = _fma32(tau, ht, ht.expand_as(tau))
            t0 = torch.floor(ut).clamp(0, c["Rt"] - 2).long()
            wt = (tau.double() + 1) * (0.5 * (c["Rt"] - 1)) - t0
            inside = inside & (tau >= -1) & (tau <= 1)
            two = [_trilinear(F64[g], inside, i0, w,
                              lambda vx, vy, vz, s=s: (((t0 + s) * R + vz) * R + vy) * R + vx) for s in (0, 1)]
            feats.append((1 - wt)[:, None] * two[0] + wt[:, None] * two[1])
        else:
            feats.append(_trilinear(F64[g], inside, i0, w, lambda vx, vy, vz: (vz * R + vy) * R + vx))
    return torch.cat(feats, 1)


def _field(c, G64, F64, W64, x):
    h = _features(c, G64, F64, x)
    for w in W64[:-1]:
        h = torch.relu(h @ w.t())
    return (h @ W64[-1].t())[:, 0]


def _rows(F, layout="paper"):
    """Grids [M][C][...] (paper order) or [M][...][C] as float64 rows [M][V][C]."""
    F = F.detach().double()
    if layout == "paper":
        return F.reshape(F.shape[0], F.shape[1], -1).transpose(1, 2).contiguous()
    return F.reshape(F.shape[0], -1, F.shape[-1]).contiguous()


def _unrows(rows, shape, layout="paper"):
    return (rows.transpose(1, 2) if layout == "paper" else rows).reshape(shape)


def _forward64(c, G, rows, W, x):
    G, W = G.double(), [w.double() for w in W]
    with torch.no_grad():
        return torch.cat([_field(c, G, rows, W, x[:, i:i + CHUNK]) for i in range(0, x.shape[1], CHUNK)])


def _grads64(c, G, rows, W, x, df_of):
    """f and the gradients of sum df f, df = df_of(f, positions), chunk by chunk."""
    p = [t.detach().double().requires_grad_(True) for t in [G, rows] + list(W)]
    fs = []
    for i in range(0, x.shape[1], CHUNK):
        f = _field(c, p[0], p[1], p[2:], x[:, i:i + CHUNK])
        (f * df_of(f.detach(), i)).sum().backward()
        fs.append(f.detach())
    return torch.cat(fs), [t.grad for t in p]


def _density_rho(G, x):
    """sum_i |det A_i| exp(-sum_d l^20) at points x [3][n] float32."""
    rho = 0.0
    xd = x.double()
    for g in range(G.shape[0]):
        l = G[g, :, :3] @ xd + G[g, :, 3:]
        rho = rho + torch.linalg.det(G[g, :, :3]).abs() * torch.exp(-(l ** 20).sum(0))
    return rho


def _density64(G, x, err, eps=1e-12):
    """(loss, dL/dG) of the feature-density loss with the target held constant."""
    n = x.shape[1]
    G = G.detach().double().requires_grad_(True)
    with torch.no_grad():
        rho = torch.cat([_density_rho(G, x[:, i:i + CHUNK]) for i in range(0, n, CHUNK)])
        S = rho.sum()
        rs = rho / S
        lg = torch.log(rs + eps)
        lt = err.mean() / (err + eps) * lg
        t = torch.exp(lt)
        loss = torch.where(t > 0, t * (lt - lg), torch.zeros_like(t)).sum() / n
        a = -t / (n * (rs + eps))
        coef = (a - (a * rs).sum()) / S
    for i in range(0, n, CHUNK):
        (_density_rho(G, x[:, i:i + CHUNK]) * coef[i:i + CHUNK]).sum().backward()
    return loss, G.grad


def _batch_points(seed, step, stream, n):
    """The step's points: Philox4x64-10, counter (j, step, stream, 0), on a 24-bit lattice."""
    bg = np.random.Philox(key=np.array([seed, 0x41504D47], dtype=np.uint64),
                          counter=np.array([2 ** 64 - 1, step - 1, stream, 0], dtype=np.uint64))
    w = bg.random_raw(4 * n).reshape(n, 4)[:, :3]
    x = (w >> np.uint64(40)).astype(np.float64) * 2.0 ** -23 - 1.0
    return torch.from_numpy(np.ascontiguousarray(x.T).astype(np.float32)).to(DEV)


def _sample(vol, brick, x):
    """Trilinear samples of the brick's extent at x [3][n]; the voxel in float32."""
    i0, w, st = [], [], (1, vol.shape[2], vol.shape[2] * vol.shape[1])
    base = 0
    for d in range(3):
        m = brick.e1[d] - brick.e0[d] + 1
        h = torch.tensor(0.5 * (m - 1), device=DEV)
        k = torch.floor(_fma32(x[d], h, h.expand_as(x[d]))).clamp(0, m - 2).long()
        base = base + (k + brick.e0[d]) * st[d]
        w.append((x[d].double() + 1) * (0.5 * (m - 1)) - k)
    flat, out = vol.reshape(-1), 0.0
    for q in range(8):
        wq, off = 1.0, base
        for d in range(3):
            wq = wq * (w[d] if (q >> d) & 1 else 1.0 - w[d])
            off = off + ((q >> d) & 1) * st[d]
        out = out + wq * flat[off].double()
    return out


def _adam64(theta, m, v, g, t, lr, out):
    """Adam on one model's slice, float64, from the float32 rates the trainer holds."""
    b1, b2 = float(np.float32(0.9)), float(np.float32(0.99))
    m, v = m.double(), v.double()
    m = b1 * m + (1 - b1) * g
    v = b2 * v + (1 - b2) * g * g
    step = lr / (1 - b1 ** t)
    out[0].append(theta.double() - step * m / (torch.sqrt(v / (1 - b2 ** t)) + float(np.float32(1e-8))))
    out[1].append(m)
    out[2].append(v)


def _step64(c, tr, bricks):
    n, H, K = c["n"], c["H"], c["M"] * c["C"]
    seed, step = int(tr.batch.seed), int(tr.step_ctr.item())
    F, G, W = [([], [], []) for _ in range(3)]
    losses = []
    lr, lr_G = float(np.float32(1e-3)), float(np.float32(1e-6))
    for b, br in enumerate(bricks):
        x = _batch_points(seed, step, b, n)
        v = torch.cat([_sample(tr.volume, br, x[:, i:i + CHUNK]) for i in range(0, n, CHUNK)])
        Wl = [tr.W[b][:H * K].view(H, K), tr.W[b][H * K:H * K + H * H].view(H, H), tr.W[b][H * K + H * H:].view(1, H)]
        Fb = tr.F[b].to(_grid_dtype(c))
        f, gr = _grads64(c, tr.G[b], _rows(Fb), Wl, x, lambda f, i: 2 * (f - v[i:i + f.numel()]) / n)
        err = (f - v) ** 2
        ld, dG = torch.zeros((), device=DEV, dtype=torch.float64), None
        if c["density"]:
            ld, dG = _density64(tr.G[b], x, err)
        losses.append(torch.stack([err.mean(), ld]))
        _adam64(tr.F[b], tr.mF[b], tr.vF[b], _unrows(gr[1], tr.F[b].shape), 201, lr, F)
        _adam64(tr.W[b], tr.mW[b], tr.vW[b], torch.cat([t.reshape(-1) for t in gr[2:]]), 201, lr, W)
        if c["density"]:
            _adam64(tr.G[b], tr.mG[b], tr.vG[b], dG, 101, lr_G, G)
        else:
            for o, t in zip(G, (tr.G[b], tr.mG[b], tr.vG[b])):
                o.append(t.double())
    s = torch.stack
    return dict(losses=s(losses), F=s(F[0]), G=s(G[0]), W=s(W[0]), mF=s(F[1]), vF=s(F[2]), mG=s(G[1]), vG=s(G[2]),
                mW=s(W[1]), vW=s(W[2]))


def _dd64(c, dd, F, pts, bricks, table):
    """Each point by the model of the brick that holds its voxel, in that brick's frame."""
    dims = [table.dims[d] for d in range(3)]
    bid, u32 = 0, []
    for d in range(3):
        m = (c["nx"], c["ny"], c["nz"])[d]
        h = torch.tensor(0.5 * (m - 1), device=DEV)
        u32.append(_fma32(pts[d], h, h.expand_as(pts[d])))
        k = torch.div(torch.floor(u32[d]).clamp(min=0).long(), c["B"], rounding_mode="floor").clamp(max=dims[d] - 1)
        bid = bid + k * (1, dims[0], dims[0] * dims[1])[d]
    out = torch.empty(pts.shape[1], dtype=torch.float64, device=DEV)
    H, K = c["H"], c["M"] * c["C"]
    for b, br in enumerate(bricks):
        idx = torch.nonzero(bid == b)[:, 0]
        if not idx.numel():
            continue
        x = []
        for d in range(3):
            span = torch.tensor(float(br.e1[d] - br.e0[d]), device=DEV)
            sc = 2.0 / span if br.e1[d] > br.e0[d] else torch.zeros((), device=DEV)
            a = u32[d][idx] - float(br.e0[d])
            x.append(_fma32(a, sc, torch.full_like(a, -1.0)))
        w = dd.W[b]
        Wl = [w[:H * K].view(H, K), w[H * K:H * K + H * H].view(H, H), w[H * K + H * H:].view(1, H)]
        out[idx] = _forward64(c, dd.G[b], _rows(F[b]), Wl, torch.stack(x))
    return out


def exact(case, seed):
    """What run returns on prepare(case, seed), in float64 (the BF16 and FP16 roundings of the
    MLP products are not imitated; FP16 grids are)."""
    c, s = case, prepare(case, seed)
    kind = c["kind"]
    if kind == "forward":
        m = s["model"]
        return _forward64(c, m.G, _rows(m.F, c["layout"]), m.W, s["pts"])
    if kind == "adjoint":
        m = s["model"]
        _, gr = _grads64(c, m.G, _rows(m.F, c["layout"]), m.W, s["pts"],
                         lambda f, i: s["df"][i:i + f.numel()].double())
        return dict(dF=_unrows(gr[1], m.F.shape, c["layout"]), dG=gr[0], dW=gr[2:])
    if kind == "autograd":
        G, F = s["p"][:2]
        n = c["n"]
        f, gr = _grads64(c, G, _rows(F), s["p"][2:], s["pts"].t().contiguous(),
                         lambda f, i: 2 * (f - s["v"][i:i + f.numel()].double()) / n)
        return dict(f=f, grads=[gr[0], _unrows(gr[1], F.shape)] + gr[2:])
    if kind == "variant":
        m, n = s["model"], c["n"]
        lay = "last" if c["enc"] == "hash" else "paper"
        rows = m.F.double().reshape(-1, c["T"], 2) if lay == "last" else _rows(m.F)
        f, gr = _grads64(c, m.G, rows, m.W, s["pts"], lambda f, i: 2 * (f - s["v"][i:i + f.numel()].double()) / n)
        dF = gr[1].reshape(m.F.shape) if lay == "last" else _unrows(gr[1], m.F.shape)
        return dict(f=f, dF=dF, dG=gr[0], dW=gr[2:])
    table, bricks = _bricks(c)
    if kind == "dd":
        return _dd64(c, s["dd"], s["F"], s["pts"], bricks, table)
    return _step64(c, s["tr"], bricks)
