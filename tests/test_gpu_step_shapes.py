"""Launch shapes of the training step and the density passes at their edges.

The density sums are float64 over float32 per-point terms: bars as the other density tests
(1e-5).  A step with another number of tile blocks adds the same float32 terms in another order:
1e-5 normwise on the first moments.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import apmg_oracle as O
from test_gpu_parity import A, DEV, assert_close, f64, host_model, make_points, soa

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("n", [64, 511, 513, 131071, 131073, 262145])
def test_density_chunks(n, norm):
    # points per chunk of the gradient pass: 512 below 2^17 points, 2048 below 2^18, then 4096
    host = host_model(5, 1, 4, 64, seed=2, extra_t=0.2)
    x = make_points(n, special=False)
    err = np.random.default_rng(n).uniform(0.01, 1.0, size=n).astype(np.float32)
    model = A().Model.from_host(host, DEV)
    loss, dG, _ = A().apmg_density_loss(model, soa(x), torch.from_numpy(err).to(DEV),
                                        flags=A().DENSITY_NORM_TARGET if norm else 0)
    r = O.density_loss(f64(host)["G"], x.astype(np.float64), err.astype(np.float64), norm_target=norm)
    assert_close("loss", loss.cpu().numpy(), [r["loss"]])
    assert_close("dG", dG.cpu().numpy(), r["dG"])


@pytest.mark.parametrize("nb", [1, 3, 7])
@pytest.mark.parametrize("bf16", [False, True])
def test_default_tile_blocks_match_one_block(nb, bf16):
    vol = synth.make_volume("blobs_sine", (32, 32, 32 * nb)).to(DEV)
    _, bricks = A().apmg_make_bricks(32 * nb, 32, 32, 32, 0)
    hosts = [synth.init_model(6, 2, 9, [12, 64, 64, 1], seed=b, grid_range=0.3) for b in range(nb)]
    out = []
    for tuning in (None, {"tile_blocks": 1}):
        tr = A().Trainer(hosts, vol, bricks, 3000, mlp_dtype=A().BF16 if bf16 else A().F32, tuning=tuning)
        tr.density_active.fill_(1)
        tr.step()
        torch.cuda.synchronize()
        assert tr.t.tolist() == [1] * nb and tr.tG.tolist() == [1] * nb and tr.step_ctr.item() == 1
        out.append([t.cpu().numpy() for t in (tr.losses, tr.mF, tr.mW, tr.mG)])
    for name, a, b in zip(("losses", "mF", "mW", "mG"), *out):
        assert_close(name, a, b)


# 4 blocks of cells a grid: one wave a block below 256 points per block, four from there on
@pytest.mark.parametrize("C", [1, 2, 4])
@pytest.mark.parametrize("n", [1023, 1024, 20001])
def test_step_gathers_agree_on_both_sides_of_the_split(C, n):
    vol = synth.make_volume("blobs_sine", (24, 24, 48)).to(DEV)
    _, bricks = A().apmg_make_bricks(48, 24, 24, 24, 0)
    hosts = [synth.init_model(3, C, 6, [3 * C, 64, 64, 1], seed=b, grid_range=0.3) for b in range(2)]
    out = []
    for tuning in ({"cell_kernel": 2}, {"cell_kernel": 1}, {"cell_kernel": 1, "cell_group": 8}):
        tr = A().Trainer(hosts, vol, bricks, n, tuning=tuning, flags=A().ADD_REC_DG)
        tr.density_active.fill_(1)
        tr.step()
        torch.cuda.synchronize()
        out.append([t.clone() for t in (tr.mF, tr.mG, tr.mW, tr.losses)])
    cells, blocks, group = out
    assert all(torch.equal(a, b) for a, b in zip(blocks, group))   # the lanes per run have no effect
    assert torch.equal(cells[2], blocks[2]) and torch.equal(cells[3], blocks[3])
    for a, b in zip(cells[:2], blocks[:2]):
        assert (a - b).norm() <= 1e-5 * b.norm()
