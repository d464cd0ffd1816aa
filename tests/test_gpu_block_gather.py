"""The matrix-product grid-gradient gather at the edges of its blocks (3 x 3 cells in z and y, 7 or
15 in x), with one wave and with four waves per block, against the FP64 oracle.

Bars: the offsets carry the float32 rounding of u = fma(l, h, h), (R - 1) / 2 * 2^-24 absolute
(1e-6 at R = 17), the sums a few roundings of 6e-8 each: 1e-5 normwise and of the largest entry,
the bars of the other float32 gradients.
"""
import numpy as np
import pytest
import torch

from oracle import apmg_oracle as O
from oracle import apmg_variants as V
from test_gpu_parity import A, DEV, assert_close, f64, host_model, kink_free, make_points, soa
from test_gpu_variants import f64 as vf64
from test_gpu_variants import kink_free as v_kink_free
from test_gpu_variants import hash_host, hash_model
from test_gpu_variants import points as v_points
from test_gpu_variants import time_host, time_model

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# n below 256 points per block: one wave per block; above: four
@pytest.mark.parametrize("C", [1, 2, 4])
@pytest.mark.parametrize("R,n", [(2, 200), (4, 3000), (5, 900), (8, 9000), (9, 1500), (16, 4000), (17, 30000)])
def test_block_gather_edges(R, n, C):
    host = host_model(3, C, R, 64, seed=R, extra_t=0.2)
    x = kink_free(host, make_points(n))
    df = np.random.default_rng(n).normal(size=x.shape[0]).astype(np.float32)
    model = A().Model.from_host(host, DEV)
    dfd = torch.from_numpy(df).to(DEV)
    dF, dG, _ = A().apmg_backward(model, soa(x), dfd)
    alone, _, _ = A().apmg_backward(model, soa(x), dfd, want_dG=False, want_dW=False)
    assert torch.equal(dF, alone)                  # with and without the transform gradient: the same bits
    go = O.backward(f64(host), x.astype(np.float64), df.astype(np.float64))
    assert_close("dF", dF.cpu().numpy(), go["dF"])
    assert_close("dG", dG.cpu().numpy(), go["dG"])


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("C,n", [(1, 5000), (2, 60), (2, 5000), (4, 60)])
def test_block_gather_keeps_nonfinite_gradients_in_their_cells(C, n, bad):
    # one point with a non-finite dL/df: exactly the 8 corners of its cell in every grid that holds
    # it are non-finite (a zero weight of another vertex of the block does not spread it)
    R = 8
    host = host_model(3, C, R, 64, seed=5)
    x = make_points(n, special=False)
    x[7] = [0.11, -0.23, 0.37]
    df = np.random.default_rng(3).normal(size=n).astype(np.float32)
    df[7] = bad
    model = A().Model.from_host(host, DEV)
    dF, _, _ = A().apmg_backward(model, soa(x), torch.from_numpy(df).to(DEV), want_dG=False, want_dW=False)
    want = np.zeros((3, R, R, R), bool)
    cell, inside = A().apmg_cells(model, soa(x[7:8]))
    for g in range(3):
        assert inside[0, g]
        cx, cy, cz = cell[0, g].tolist()
        want[g, cz:cz + 2, cy:cy + 2, cx:cx + 2] = True
    got = ~torch.isfinite(dF).cpu().numpy()
    for c in range(C):
        assert np.array_equal(got[:, c], want)


@pytest.mark.parametrize("Rt", [2, 3])
@pytest.mark.parametrize("R,n", [(4, 3000), (9, 2000)])
def test_time_block_gather_edges(R, n, Rt):
    h = time_host(M=4, R=R, Rt=Rt, seed=R)
    x = v_points(n, seed=n, time=True)
    _, cache = V.time_forward(vf64(h), x[:, :3].astype(np.float64), x[:, 3].astype(np.float64))
    x = x[v_kink_free(cache)]
    df = np.random.default_rng(17).normal(size=x.shape[0]).astype(np.float32)
    go = V.time_backward(vf64(h), x[:, :3].astype(np.float64), x[:, 3].astype(np.float64), df.astype(np.float64))
    dfd = torch.from_numpy(df).to(DEV)
    for cl in (False, True):
        dF, dG, _ = A().apmg_variant_backward(time_model(h, channel_last=cl), soa(x), dfd)
        again, _, _ = A().apmg_variant_backward(time_model(h, channel_last=cl), soa(x), dfd)
        assert torch.equal(dF, again)
        dFn = dF.cpu().numpy()
        assert_close(f"dF4 (channel-last {cl})", dFn.transpose(0, 5, 1, 2, 3, 4) if cl else dFn, go["dF4"])
        assert_close("dG", dG.cpu().numpy(), go["dG"])


# levels of one entry per vertex, hashed levels whose rows of N + 1 vertices fill runs of 64, 128 and
# 256 entries (exactly, and one past), and levels left to the atomics: more than four vertices a
# point, or a table smaller than a run
@pytest.mark.parametrize("res,T,M,n,fixed_order", [
    ((1, 7, 20, 31), 1 << 12, 3, 40000, True),
    ((63, 64), 1 << 12, 2, 80000, True),
    ((127, 128), 1 << 14, 1, 545000, True),
    ((3, 100), 1 << 6, 4, 3000, False),
    ((15, 40), 1 << 6, 2, 20000, False),
])
def test_hash_table_gradient_levels(res, T, M, n, fixed_order):
    h = hash_host(M=M, L=len(res), T=T, res=res, seed=n)
    x = v_points(n, seed=n + 1)
    _, cache = V.hash_forward(vf64(h), x.astype(np.float64))
    # points at a ReLU kink stay in the batch (its size picks the path) with dL/df = 0
    df = np.where(v_kink_free(cache), np.random.default_rng(8).normal(size=n), 0.0).astype(np.float32)
    dfd, xd = torch.from_numpy(df).to(DEV), soa(x)
    model = hash_model(h)
    dF, dG, _ = A().apmg_variant_backward(model, xd, dfd)
    again, _, _ = A().apmg_variant_backward(model, xd, dfd, want_dG=False, want_dW=False)
    if fixed_order:
        assert torch.equal(dF, again)
    go = V.hash_backward(vf64(h), x.astype(np.float64), df.astype(np.float64))
    for k in range(len(res)):
        assert_close(f"dTheta level {k}", dF[:, k].cpu().numpy(), go["dTheta"][:, k])
    assert_close("dG", dG.cpu().numpy(), go["dG"])
