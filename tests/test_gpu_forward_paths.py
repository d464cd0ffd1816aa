"""Forward paths that only order or lay out the work differently give the same bits."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_parity import A, DEV, make_points, soa

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("dims,B", [((96, 64, 80), 48), ((40, 40, 40), 40), ((70, 70, 70), 8)])
@pytest.mark.parametrize("bf16", [False, True])
def test_dd_spatial_order_is_bitwise_the_plain_one(dims, B, bf16):
    # from 2^15 points on, a brick's points are also ordered by bins inside the brick (a 40^3
    # volume: one brick; 70^3 in 8^3 bricks: 729 models)
    table, bricks = A().apmg_make_bricks(*dims, B, 1)
    nb = len(bricks)
    hosts = [synth.init_model(3, 2, 6, [6, 64, 64, 1], seed=b, grid_range=0.4) for b in range(nb)]
    G = torch.stack([torch.from_numpy(h["G"]) for h in hosts]).to(DEV)
    F = torch.stack([torch.from_numpy(h["F"]) for h in hosts]).to(DEV)
    W = torch.stack([torch.cat([torch.from_numpy(w).reshape(-1) for w in h["W"]]) for h in hosts]).to(DEV)
    dd = A().DDModels(G, F, W, [6, 64, 64, 1], table, bricks, A().BF16 if bf16 else A().F32)
    pts = soa(make_points(40001))                    # among them corners, outside and NaN points
    whole = A().apmg_dd_forward(dd, pts)
    parts = [A().apmg_dd_forward(dd, pts[:, i:i + 13334].contiguous()) for i in range(0, 40001, 13334)]
    assert torch.equal(whole, torch.cat(parts))


@pytest.mark.parametrize("M,C,R", [(1, 1, 2), (5, 1, 7), (16, 2, 16), (7, 2, 9), (31, 2, 5), (3, 4, 6), (16, 4, 8)])
@pytest.mark.parametrize("grids", [torch.float32, torch.float16])
@pytest.mark.parametrize("bf16", [False, True])
def test_small_batches_give_the_bits_of_large_ones(M, C, R, grids, bf16):
    # up to 2^14 points one launch reads the caller's grids, transforms and weights as they are;
    # above, the tiles walk a sorted order of copies
    host = synth.init_model(M, C, R, [M * C, 64, 64, 1], seed=M, grid_range=0.5, extra_translation=0.2, vmin=-1.0,
                            vmax=2.0)
    mlp = A().BF16 if bf16 else A().F32
    model = A().Model.from_host(host, DEV, grid_dtype=grids, mlp_dtype=mlp)
    pts = soa(make_points(40000))
    large = A().apmg_forward(model, pts)
    G4 = torch.zeros((M, 4, 4), device=DEV)
    G4[:, :3] = model.G
    G4[:, 3] = float("nan")                          # row 3 is never read
    last = A().Model(G4, model.F.permute(0, 2, 3, 4, 1).contiguous(), model.W, -1.0, 2.0, mlp, A().GRIDS_MRRRC)
    for n in (1, 31, 33, 16384):
        for m in (model, last):
            assert torch.equal(A().apmg_forward(m, pts, n=n), large[:n]), n          # (rows ld = 40000 apart)
        assert torch.equal(A().apmg_forward_noalloc(model, pts, n=n), large[:n])


def test_small_batch_weights_at_any_alignment():
    # weight rows that are not 16-byte aligned take the scalar loads
    host = synth.init_model(8, 2, 5, [16, 64, 64, 1], seed=3, grid_range=0.5)
    model = A().Model.from_host(host, DEV)
    flat = torch.zeros(1 + sum(w.numel() for w in model.W), device=DEV)
    shifted, o = [], 1
    for w in model.W:
        v = flat[o:o + w.numel()].view(w.shape)
        v.copy_(w)
        shifted.append(v)
        o += w.numel()
    pts = soa(make_points(1000))
    other = A().Model(model.G, model.F, shifted, model.vmin, model.vmax)
    assert torch.equal(A().apmg_forward(model, pts), A().apmg_forward(other, pts))


@pytest.mark.parametrize("n", [1023, 1025, 131071, 131072, 131073])
def test_sort_tiles_and_modes(n):
    # tiles of 1024 keys up to 2^17 keys, of 4096 above: the sorted forward gives the direct bits, and
    # the gradients gathered from the sorted points add up to those of two parts sorted apart
    # (float32 sums in another order: 1e-5 normwise)
    host = synth.init_model(4, 2, 9, [8, 64, 64, 1], seed=5, grid_range=0.5)
    model = A().Model.from_host(host, DEV)
    x = make_points(n)
    pts = soa(x)
    assert torch.equal(A().apmg_forward(model, pts), A().apmg_forward_noalloc(model, pts))
    df = torch.from_numpy(np.random.default_rng(n).normal(size=n).astype(np.float32)).to(DEV)
    h = n // 3
    whole = A().apmg_backward(model, pts, df)
    again = A().apmg_backward(model, pts, df)
    a = A().apmg_backward(model, pts[:, :h].contiguous(), df[:h])
    b = A().apmg_backward(model, pts[:, h:].contiguous(), df[h:].contiguous())
    assert torch.equal(whole[0], again[0]) and torch.equal(whole[1], again[1])
    for g, ga, gb in zip([whole[0], whole[1], *whole[2]], [a[0], a[1], *a[2]], [b[0], b[1], *b[2]]):
        want = (ga.double() + gb.double())
        assert (g.double() - want).norm() <= 1e-5 * want.norm()


def test_batched_sort_modes_give_the_same_brick():
    # a brick sorts alone in small tiles, or with enough others in large ones: the same points in the
    # same order, so with fixed launch shapes the same step, bit for bit
    vol = synth.make_volume("blobs_sine", (24, 24, 24 * 12)).to(DEV)
    _, bricks = A().apmg_make_bricks(24 * 12, 24, 24, 24, 0)
    hosts = [synth.init_model(4, 2, 6, [8, 64, 64, 1], seed=b, grid_range=0.3) for b in range(12)]
    out = []
    for k in (1, 12):
        tr = A().Trainer(hosts[:k], vol, bricks[:k], 20000, tuning={"tile_blocks": 4})
        tr.density_active.fill_(1)
        tr.step()
        torch.cuda.synchronize()
        out.append([t[0].clone() for t in (tr.losses, tr.F, tr.G, tr.W, tr.mF, tr.mG, tr.mW)])
    for a, b in zip(*out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("M,C,R,dtype", [(2, 4, 511, torch.float32), (2, 4, 512, torch.float32),
                                         (3, 4, 512, torch.float16)])
def test_grids_of_four_gib(M, C, R, dtype):
    # grids below 4 GiB are read through 32-bit offsets of a buffer resource (above 2 GiB here, so the
    # upper half of the offsets is used), grids from 4 GiB on with 64-bit addresses; small batches
    # read the caller's grids another way.  The forward pass gives the same bits, and the adjoint's
    # weight gradients are those of a float64 interpolation and MLP, 1e-3 normwise
    g = torch.Generator(device=DEV).manual_seed(R + M)
    F = torch.empty((M, R, R, R, C), dtype=dtype, device=DEV).normal_(generator=g)
    G = torch.zeros((M, 3, 4), device=DEV)
    for m in range(M):
        G[m, :, :3] = torch.eye(3, device=DEV) * (0.97 - 0.1 * m)
        G[m, :, 3] = 0.01
    W = [torch.randn(s, generator=g, device=DEV) / s[1] ** 0.5 for s in ((64, M * C), (64, 64), (1, 64))]
    model = A().Model(G, F, W, -1.0, 2.0, A().F32, A().GRIDS_MRRRC)
    n = 20000
    x = torch.rand((3, n), generator=g, device=DEV) * 2 - 1
    large = A().apmg_forward(model, x)
    assert torch.equal(large, torch.cat([A().apmg_forward(model, x[:, :9000].contiguous()),
                                         A().apmg_forward(model, x[:, 9000:].contiguous())]))
    df = torch.randn(n, generator=g, device=DEV)
    dW = A().apmg_backward(model, x, df, want_dF=False, want_dG=False)[2]
    feats = []
    for m in range(M):
        # Eqs. (1) and (2) in the float32 steps that define the cell decision (fused multiply-adds, z
        # first): a float64 cell would turn ReLUs by itself
        fma = lambda a, b, c: (a.double() * b.double() + c.double()).float()
        g4 = G[m]
        loc = torch.stack([fma(g4[d, 2], x[2], fma(g4[d, 1], x[1], fma(g4[d, 0], x[0], g4[d, 3]))) for d in range(3)])
        inside = ((loc >= -1) & (loc <= 1)).all(0)
        hr = torch.tensor(0.5 * (R - 1), device=DEV)
        u = fma(loc, hr, hr)
        i0 = u.floor().clamp(0, R - 2)
        w, i0 = (u - i0).double(), i0.long()
        e = torch.zeros((C, n), dtype=torch.float64, device=DEV)
        for q in range(8):
            b = [(q >> d) & 1 for d in range(3)]
            wq = torch.stack([w[d] if b[d] else 1 - w[d] for d in range(3)]).prod(0)
            e += wq * F[m, i0[2] + b[2], i0[1] + b[1], i0[0] + b[0]].double().T
        feats.append(e * inside)
    Wd = [w.double().requires_grad_() for w in W]
    h = torch.relu(Wd[1] @ torch.relu(Wd[0] @ torch.cat(feats)))
    ((Wd[2] @ h)[0] * 3.0 * df.double()).sum().backward()     # the output's scale: vmax - vmin
    for got, want in zip(dW, Wd):
        assert (got.double() - want.grad).norm() <= 1e-3 * want.grad.norm()


@pytest.mark.parametrize("R,H", [(511, 64), (512, 64), (511, 128), (512, 128)])
def test_gradients_of_four_gib_grids(R, H):
    # 2 grids of R^3 x 4 in float32, below and at 4 GiB, with the narrow and the wide (activation path)
    # decoder: every gradient against float64 from the float32 cell decision and offsets.  Points whose
    # hidden units lie within 1e-4 of a kink have dL/df = 0, so no ReLU turns; the rest are the float32
    # bars, 1e-5 normwise
    M, C, n = 2, 4, 20000
    g = torch.Generator(device=DEV).manual_seed(R + H)
    F = torch.empty((M, R, R, R, C), device=DEV).normal_(generator=g)
    G = torch.zeros((M, 3, 4), device=DEV)
    for m in range(M):
        G[m, :, :3] = torch.eye(3, device=DEV) * (0.97 - 0.1 * m)
        G[m, :, 3] = 0.01
    W = [torch.randn(s, generator=g, device=DEV) / s[1] ** 0.5 for s in ((H, M * C), (H, H), (1, H))]
    model = A().Model(G, F, W, -1.0, 2.0, A().F32, A().GRIDS_MRRRC)
    x = torch.rand((3, n), generator=g, device=DEV) * 2 - 1
    fma = lambda a, b, c: (a.double() * b.double() + c.double()).float()
    G64, W64 = G.double().requires_grad_(), [w.double().requires_grad_() for w in W]
    feats, corners, weights = [], [], []
    for m in range(M):
        g4, hr = G[m], torch.tensor(0.5 * (R - 1), device=DEV)
        loc = torch.stack([fma(g4[d, 2], x[2], fma(g4[d, 1], x[1], fma(g4[d, 0], x[0], g4[d, 3]))) for d in range(3)])
        inside = ((loc >= -1) & (loc <= 1)).all(0)
        u = fma(loc, hr, hr)
        i0 = u.floor().clamp(0, R - 2)
        u64 = (G64[m, :, :3] @ x.double() + G64[m, :, 3:] + 1) * (0.5 * (R - 1))
        w, i0 = (u - i0).double() + (u64 - u64.detach()), i0.long()     # the float32 offsets, with a gradient
        e = 0.0
        for q in range(8):
            b = [(q >> d) & 1 for d in range(3)]
            wq = torch.stack([w[d] if b[d] else 1 - w[d] for d in range(3)]).prod(0) * inside
            v = ((i0[2] + b[2]) * R + i0[1] + b[1]) * R + i0[0] + b[0]
            e = e + wq * F[m].view(-1, C)[v].double().T
            corners.append(v)
            weights.append(wq.detach())
        feats.append(e)
    y = torch.cat(feats)
    y.retain_grad()
    z1 = W64[0] @ y
    z2 = W64[1] @ torch.relu(z1)
    near = torch.minimum(z1.abs().min(0).values, z2.abs().min(0).values) < 1e-4
    df = torch.where(near, 0.0, torch.randn(n, generator=g, device=DEV))
    ((W64[2] @ torch.relu(z2))[0] * 3.0 * df.double()).sum().backward()
    dF, dG, dW = A().apmg_backward(model, x, df)
    for got, want in zip(dW, W64):
        assert (got.double() - want.grad).norm() <= 1e-5 * want.grad.norm()
    assert (dG - G64.grad).norm() <= 1e-5 * G64.grad.norm()
    for m in range(M):
        want = torch.zeros((R ** 3, C), dtype=torch.float64, device=DEV)
        for v, wq in zip(corners[8 * m:8 * m + 8], weights[8 * m:8 * m + 8]):
            want.index_add_(0, v, (wq * y.grad[4 * m:4 * m + 4]).T.contiguous())
        assert (dF[m].view(-1, C).double() - want).norm() <= 1e-5 * want.norm()
