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
