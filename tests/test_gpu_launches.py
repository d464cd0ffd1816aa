"""Launches per call: the kernel nodes of a graph captured around one call.

Small calls are bound by their launches (about 5 us each), so rules that choose a path by size are
checked by what they launch.
"""
import ctypes

import pytest
import torch

import synth
from test_gpu_parity import A, DEV

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


class KernelNode(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("args", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


def kernel_grids(fn):
    """The launch grids of the kernels that one call of fn records."""
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        out = fn()
    hip = ctypes.CDLL(next(ln.split()[-1] for ln in open("/proc/self/maps") if "libamdhip64" in ln))
    g, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(g, None, ctypes.byref(n)) == 0
    nodes = (ctypes.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(g, nodes, ctypes.byref(n)) == 0
    grids, p = [], KernelNode()
    for node in nodes:
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        grids.append(tuple(p.grid))
    del out
    return grids


def launches(fn):
    return len(kernel_grids(fn))


def brick_models(R, M, bf16, half=True):
    table, bricks = A().apmg_make_bricks(60, 60, 60, 20, 1)
    nb = len(bricks)
    g = torch.Generator(device=DEV).manual_seed(R)
    F = torch.rand((nb, M, 2, R, R, R), generator=g, device=DEV) - 0.5
    hosts = [synth.init_model(M, 2, 4, [2 * M, 64, 64, 1], seed=b) for b in range(nb)]
    G = torch.stack([torch.from_numpy(h["G"]) for h in hosts]).to(DEV)
    W = torch.stack([torch.cat([torch.from_numpy(w).reshape(-1) for w in h["W"]]) for h in hosts]).to(DEV)
    return A().DDModels(G, F.half() if half else F, W, [2 * M, 64, 64, 1], table, bricks,
                        A().BF16 if bf16 else A().F32)


# bins inside the bricks are ordered (a second radix pass: three launches more) where the lookups'
# cache misses cost more than that: by points, grids and bytes of grids, and the MLP that hides them
@pytest.mark.parametrize("R,M,bf16,half,n,order", [
    (16, 8, True, True, 1 << 18, False), (16, 8, False, False, 1 << 18, False), (16, 16, False, True, 1 << 18, False),
    (32, 16, True, False, 1 << 18, True), (32, 16, False, False, 1 << 18, True), (32, 16, False, True, 1 << 14, False),
])
def test_brick_queries_order_bins_where_it_pays(R, M, bf16, half, n, order):
    dd = brick_models(R, M, bf16, half)
    pts = torch.rand((3, n), device=DEV) * 2 - 1
    out = torch.empty(n, device=DEV)
    start = pts[:, :1000].contiguous()
    few = launches(lambda: A().apmg_dd_forward(dd, start, out=out[:1000]))
    got = launches(lambda: A().apmg_dd_forward(dd, pts, out=out))
    scan = 1 if n > 1 << 17 else 0          # (of more than 2^17 points, a pass has a row scan of its own)
    assert got == few + scan + (2 + scan if order else 0)
    # ordered or not, the same bits as queries of fewer points, which are not ordered
    parts = [A().apmg_dd_forward(dd, p.contiguous()) for p in pts.split(30000, dim=1)]
    assert torch.equal(A().apmg_dd_forward(dd, pts), torch.cat(parts))


# one launch up to 2^13 points, and beyond while the blocks that queue stay cheap: few features and channels,
# channel-last grids where they have four channels, large ones where they have two
@pytest.mark.parametrize("M,C,R,last,n,small", [
    (40, 4, 5, False, 8192, True), (40, 4, 5, True, 8193, False), (24, 4, 5, True, 10000, False),
    (96, 2, 5, False, 12288, False), (16, 4, 5, False, 12288, True), (16, 4, 5, False, 12289, False),
    (16, 4, 5, True, 16384, True), (64, 2, 5, True, 12288, True), (64, 2, 23, False, 16384, False),
    (64, 2, 24, False, 16384, True), (32, 2, 5, False, 16384, True), (128, 1, 5, False, 16384, True),
    (8, 4, 5, False, 16384, True), (32, 2, 5, False, 16385, False),
])
def test_small_forward_sizes(M, C, R, last, n, small):
    host = synth.init_model(M, C, R, [M * C, 64, 64, 1], seed=M, grid_range=0.5)
    model = A().Model.from_host(host, DEV)
    if last:
        model = A().Model(model.G, model.F.permute(0, 2, 3, 4, 1).contiguous(), model.W, layout=A().GRIDS_MRRRC)
    pts = torch.rand((3, n), device=DEV) * 2 - 1
    out = torch.empty(n, device=DEV)
    ws = torch.empty(A()._lib.apmg_workspace_bytes(A().OP_FORWARD, ctypes.byref(model.struct()), n),
                     dtype=torch.uint8, device=DEV)
    assert (launches(lambda: A().apmg_forward(model, pts, out=out, ws=ws)) == 1) == small
    parts = [A().apmg_forward(model, p.contiguous()) for p in pts.split(5000, dim=1)]
    assert torch.equal(out, torch.cat(parts))


def test_one_time_cell_is_not_sorted_by_time():
    # with two time vertices the spatial order is the (time cell, bin) order: no pass by time cell
    # (keys and scatter) and no starts of its own
    g = torch.Generator(device=DEV).manual_seed(2)
    n, counts = 3000, []
    pts = torch.rand((4, n), generator=g, device=DEV) * 2.2 - 1.1     # among them times outside
    df = torch.randn(n, generator=g, device=DEV)
    for Rt in (2, 3):
        host = synth.init_model(4, 2, 4, [8, 64, 64, 1], seed=Rt, grid_range=0.3)
        F = torch.rand((4, 2, Rt, 6, 6, 6), generator=g, device=DEV) - 0.5
        model = A().VariantModel(A().ENC_TIME, torch.from_numpy(host["G"]).to(DEV), F,
                                 [torch.from_numpy(w).to(DEV) for w in host["W"]])
        counts.append(launches(lambda: A().apmg_variant_backward(model, pts, df)))
    assert counts[0] == counts[1] - 3


# one to sixteen points a thread: four blocks per compute unit (256) over the feature grids where there
# are points enough for them
@pytest.mark.parametrize("n,points", [(257, 1), (5000, 1), (149797, 4), (1 << 20, 16)])
def test_transform_gradient_blocks(n, points):
    M, R, Rt = 7, 6, 2
    host = synth.init_model(M, 2, 4, [2 * M, 64, 64, 1], seed=1, grid_range=0.3)
    g = torch.Generator(device=DEV).manual_seed(n)
    F = torch.rand((M, 2, Rt, R, R, R), generator=g, device=DEV) - 0.5
    model = A().VariantModel(A().ENC_TIME, torch.from_numpy(host["G"]).to(DEV), F,
                             [torch.from_numpy(w).to(DEV) for w in host["W"]])
    pts = torch.rand((4, n), generator=g, device=DEV) * 2 - 1
    df = torch.randn(n, generator=g, device=DEV)
    grad = lambda x, d: A().apmg_variant_backward(model, x, d, want_dF=False, want_dW=False)[1]
    assert (-(-n // (256 * points)), M, 1) in kernel_grids(lambda: grad(pts, df))
    # the float64 sums of the same float32 terms: those of the two halves add up to the whole
    h = n // 2
    parts = grad(pts[:, :h].contiguous(), df[:h].contiguous()) + grad(pts[:, h:].contiguous(), df[h:].contiguous())
    whole = grad(pts, df)
    assert (whole - parts).norm() <= 1e-10 * whole.norm()


# 3 levels (of 9^3 and 13^3 entries, and one hashed): the atomics take one launch for all the levels
# that are left to them, the gather two per level from 4096 points on
@pytest.mark.parametrize("n,res,gathered", [(100, (8, 12, 40), 0), (4095, (8, 12, 40), 0), (4096, (8, 12, 40), 2),
                                            (4096, (30, 40, 50), 0), (20000, (8, 12, 40), 3)])
def test_hash_levels_share_the_scatter(n, res, gathered):
    host = synth.init_model(2, 2, 4, [12, 64, 64, 1], seed=1, grid_range=0.3)
    g = torch.Generator(device=DEV).manual_seed(n)
    F = torch.rand((2, 3, 1 << 12, 2), generator=g, device=DEV) - 0.5
    model = A().VariantModel(A().ENC_HASH, torch.from_numpy(host["G"]).to(DEV)[:2], F,
                             [torch.from_numpy(w).to(DEV) for w in host["W"]], level_res=res)
    pts = torch.rand((3, n), generator=g, device=DEV) * 2 - 1
    df = torch.randn(n, generator=g, device=DEV)
    none = launches(lambda: A().apmg_variant_backward(model, pts, df, want_dF=False, want_dG=False))
    grad = lambda: A().apmg_variant_backward(model, pts, df, want_dG=False)
    # (the table gradient is cleared first)
    assert launches(grad) == none + 1 + 2 * gathered + (1 if gathered < 3 else 0)
    # the scatter adds a float32 term per corner: 1e-6 normwise between two orders
    a, b = grad()[0].double(), grad()[0].double()
    assert (a - b).norm() <= 1e-6 * a.norm()


# four waves share a block of cells (a workgroup per block instead of per four) where the points per
# block pay for the set-up of each: the more the more blocks, and from twice as many in a step
@pytest.mark.parametrize("M,C,R,n,step,groups", [
    (16, 2, 16, 75 * 512 - 1, False, 19), (16, 2, 16, 75 * 512, False, 75),
    (16, 2, 16, 75 * 1024 - 1, True, 19), (16, 2, 16, 75 * 1024, True, 75),
    (16, 2, 30, 1 << 17, False, 125), (16, 2, 30, 666667, False, 500), (16, 2, 30, 1 << 17, True, 125),
    (7, 4, 10, 18 * 256 - 1, True, 5), (7, 4, 10, 18 * 256, True, 18), (3, 2, 24, (1 << 16) - 1, False, 64),
    (3, 2, 24, 1 << 16, False, 256),
    (32, 1, 32, 1 << 18, False, 91), (32, 1, 32, 1 << 20, False, 363), (32, 2, 32, 1 << 21, False, 152),
])
def test_gather_waves_per_block(M, C, R, n, step, groups):
    host = synth.init_model(M, C, R, [M * C, 64, 64, 1], seed=M, grid_range=0.3)
    if step:
        vol = synth.make_volume("blobs_sine", (24, 24, 24)).to(DEV)
        tr = A().Trainer([host], vol, A().apmg_make_bricks(24, 24, 24, 24, 0)[1], n)
        call = tr.step
    else:
        model = A().Model.from_host(host, DEV)
        pts = torch.rand((3, n), device=DEV) * 2 - 1
        df = torch.full((n,), 1.0 / n, device=DEV)
        call = lambda: A().apmg_backward(model, pts, df, want_dG=False, want_dW=False)
    assert (groups * M, 1, 1) in kernel_grids(call)


@pytest.mark.parametrize("bf16", [False, True])
def test_activation_path_runs_two_blocks_per_compute_unit(bf16):
    # H = 128: blocks of four waves, two on each of the 256 compute units (512 blocks of 4 tiles here)
    n, mlp = 1 << 16, A().BF16 if bf16 else A().F32
    host = synth.init_model(9, 2, 6, [18, 128, 128, 1], seed=1, grid_range=0.3)
    model = A().Model.from_host(host, DEV, mlp_dtype=mlp)
    pts = torch.rand((3, n), device=DEV) * 2 - 1
    df = torch.full((n,), 1.0 / n, device=DEV)
    assert (512, 1, 1) in kernel_grids(lambda: A().apmg_backward(model, pts, df))
    vol = synth.make_volume("blobs_sine", (24, 24, 24)).to(DEV)
    tr = A().Trainer([host], vol, A().apmg_make_bricks(24, 24, 24, 24, 0)[1], n, mlp_dtype=mlp)
    assert (512, 1, 1) in kernel_grids(tr.step)
