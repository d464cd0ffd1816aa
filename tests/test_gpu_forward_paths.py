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
