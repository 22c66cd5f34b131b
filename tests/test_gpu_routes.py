"""Which launches a call makes, read from a captured graph that is never replayed, where that is what a rule decides:
the results are the same either way."""
import ctypes as C

import pytest
import torch

from paper_2502_00340_amd import binding as Bn
from paper_2502_00340_amd import workloads as WL
from tests.test_gpu_parity import LORA_SHAPES, _random_layer, say

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class _KernelNode(C.Structure):     # hipKernelNodeParams
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3), ("params", C.c_void_p),
                ("shared", C.c_uint32)]


def _hip():
    """The HIP runtime that this process has loaded."""
    with open("/proc/self/maps") as f:
        return C.CDLL(next(line.split()[-1] for line in f if "libamdhip64.so" in line))


def launches(call):
    """Grid of every kernel that `call` launches on the current stream, in order."""
    call()                                  # first use sets kernel attributes
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    hip, raw, n = _hip(), C.c_void_p(graph.raw_cuda_graph()), C.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(raw, nodes, C.byref(n)) == 0
    grids = []
    for node in nodes[:n.value]:
        kind, p = C.c_int(-1), _KernelNode()
        assert hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)) == 0
        if kind.value == 0:                 # hipGraphNodeTypeKernel
            assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
            grids.append((p.grid.x, p.grid.y, p.grid.z))
    return grids


def _compact_case(S, kept, main_grad=False):
    shape = WL.LayerShape("routes", B=1, S=S, H=512, Hq=8, Hkv=2, d=64, F=256, dtype="bf16")
    sv, W, dy = _random_layer(shape, S)
    mask = torch.zeros((1, S), dtype=torch.uint8, device=DEV)
    mask[0, torch.randperm(S, generator=torch.Generator().manual_seed(kept))[:kept].to(DEV)] = 1
    idx, cu, n_dev, n = Bn.build_keep_index(mask)
    plan = lambda: Bn.LayerBackward(Bn.make_desc(1, S, 512, 8, 2, 64, 256, "bf16"), device=DEV, main_grad=main_grad)
    return sv, W, Bn.gather_rows(dy, idx, n), idx, cu, n_dev, plan


@pytest.mark.parametrize("main_grad", [False, True])
def test_layer_output_behind_the_upstream_gradient(main_grad):
    """A count on the device leaves open where the caller's upstream gradient ends: a parameter gradient that lies right behind its
    rows, within the bound, and dx over them, give the bits and the number of launches of outputs elsewhere."""
    sv, W, dyk, idx, cu, n_dev, plan = _compact_case(400, 100, main_grad)
    roomy = torch.empty(400, 512, dtype=torch.bfloat16, device=DEV)         # rows up to the bound: nothing else lies there
    roomy[:100] = dyk
    dyk = roomy[:100]
    ref = plan()
    ref_launches = launches(lambda: ref.compact_dev(sv, W, dyk, idx, cu, n_dev))
    for g in ref.grads.values():
        g.zero_()
    ref.compact_dev(sv, W, dyk, idx, cu, n_dev)
    for where in ("dwd behind dy", "dx over dy", "dx one row into dy"):
        say("layer, " + where)
        p = plan()
        buf = torch.zeros(400 * 512 * 4 + p.grads["dwd"].numel() * 4, dtype=torch.uint8, device=DEV)
        dy2 = buf[:dyk.numel() * 2].view(torch.bfloat16).view(dyk.shape)
        if where == "dwd behind dy":
            g = p.grads["dwd"]
            at = dyk.numel() * 2
            p.grads["dwd"] = buf[at:at + g.numel() * g.element_size()].view(g.dtype).view(g.shape)
            p._g.dwd = p.grads["dwd"].data_ptr()
        else:
            at = 0 if where == "dx over dy" else 512 * 2
            p.grads["dx"] = buf[at:at + 400 * 512 * 2].view(torch.bfloat16).view(400, 512)
            p._g.dx = p.grads["dx"].data_ptr()
        call = lambda: p.compact_dev(sv, W, dy2, idx, cu, n_dev)
        assert len(launches(call)) == len(ref_launches)
        for g in p.grads.values():
            g.zero_()
        dy2.copy_(dyk)
        call()
        torch.cuda.synchronize()
        for k in ref.grads:
            a, b = (t[:100] if k == "dx" else t for t in (p.grads[k], ref.grads[k]))
            assert torch.equal(a, b), (where, k)


@pytest.mark.parametrize("main_grad", [False, True])
@pytest.mark.parametrize("which", ["dg1", "dg2"])
def test_layer_gain_gradient_over_an_operand_of_the_products_beside_it(which, main_grad):
    """More than one round of parameter-gradient tiles, so that the gain gradients are summed up while the products run: one that lies
    over the caller's upstream gradient (an operand of dWd) or attention output (of dWo, dense) gives the bits of outputs elsewhere."""
    shape = WL.LayerShape("gain_overlap", B=1, S=400, H=2056, Hq=4, Hkv=2, d=64, F=4864, dtype="bf16")
    sv, W, dy = _random_layer(shape, 5)
    mask = torch.zeros((1, 400), dtype=torch.uint8, device=DEV)
    mask[0, torch.randperm(400, generator=torch.Generator().manual_seed(6))[:300].to(DEV)] = 1
    idx, cu, n_dev, n = Bn.build_keep_index(mask)
    dyk = Bn.gather_rows(dy, idx, n)
    plan = lambda: Bn.LayerBackward(Bn.make_desc(1, 400, 2056, 4, 2, 64, 4864, "bf16"), device=DEV, main_grad=main_grad)
    size = 2056 * (4 if main_grad else 2)
    for src, call in (("dy", lambda p, dy, a: p.compact_dev(sv, W, dy, idx, cu, n_dev)),
                      ("attn_out", lambda p, dy, a: p.dense(dict(sv, attn_out=a), W, dy))):
        say("layer, %s over %s" % (which, src))
        kept = dyk if src == "dy" else dy
        ref, p = plan(), plan()
        call(ref, kept, sv["attn_out"])
        under = (kept if src == "dy" else sv["attn_out"]).clone()
        first = 16000                                                       # inside both, on a 16-byte boundary
        bytes_ = under.view(torch.uint8).view(-1)
        p.grads[which] = bytes_[first:first + size].view(p.grads[which].dtype)
        setattr(p._g, which, p.grads[which].data_ptr())
        if main_grad:       # what is added to: the operand's own bytes, so the expected sum starts from them
            ref.grads[which].copy_(ref.grads[which] + p.grads[which])
        call(p, under if src == "dy" else kept, under if src != "dy" else sv["attn_out"])
        torch.cuda.synchronize()
        for k in ref.grads:
            a, b = (t[:n] if k == "dx" and src == "dy" else t for t in (p.grads[k], ref.grads[k]))
            assert torch.equal(a, b), (src, k)


def _attn_call(B, S, Hq, Hkv, d, n):
    """cf_attn_bwd_filtered of n rows, the first n / B of every sequence."""
    bf = lambda *s: torch.randn(s, device=DEV).to(torch.bfloat16)
    idx = (torch.arange(B, device=DEV)[:, None] * S + torch.arange(n // B, device=DEV)).reshape(-1).int()
    cu = torch.arange(B + 1, device=DEV, dtype=torch.int32) * (n // B)
    q, o, do, k, v = bf(n, Hq * d), bf(n, Hq * d), bf(n, Hq * d), bf(B * S, Hkv * d), bf(B * S, Hkv * d)
    lse = torch.full((B, Hq, S), 8.0, device=DEV)
    desc = Bn.make_desc(B, S, 8, Hq, Hkv, d, 8, "bf16")
    return lambda: Bn.attn_bwd_filtered(desc, q, k, v, o, lse, do, idx, cu, n)


@pytest.mark.parametrize("S,Hq,Hkv,d,n", [(4200, 12, 4, 64, 4200), (4096, 16, 16, 64, 3481), (4500, 8, 8, 128, 4300)])
def test_attn_key_ranges_of_coarse_tiles(S, Hq, Hkv, d, n):
    """A chain on tiles of 128 queries takes longer than one on 64: on 256 CUs these calls take two ranges."""
    say("attn routes S=%d Hq=%d d=%d" % (S, Hq, d))
    assert launches(_attn_call(1, S, Hq, Hkv, d, n))[0][2] == 2


@pytest.mark.parametrize("B,S,Hq,Hkv,d,n", [(8, 933, 32, 4, 64, 3352), (8, 516, 64, 8, 64, 1856), (3, 700, 24, 8, 128, 1800)])
def test_attn_grid_has_no_fine_tiles_that_cannot_be_taken(B, S, Hq, Hkv, d, n):
    """The host knows the rows: with more of them than take fine tiles, dQ and dK/dV have a block for every tile of 128 that a
    sequence may fill, and no more."""
    say("attn routes B=%d S=%d Hq=%d d=%d rows=%d" % (B, S, Hq, d, n))
    grids = launches(_attn_call(B, S, Hq, Hkv, d, n))
    tiles = -(-S // 128)
    assert grids[0][:2] == (Hq * B, tiles) and grids[1] == (Hq * B * tiles, 1, 1)


@pytest.mark.parametrize("B,S,Hq,Hkv,d,n,fine", [
    (1, 600, 64, 8, 128, 512, True), (8, 300, 24, 8, 128, 1200, False), (4, 600, 24, 8, 128, 1200, True), (8, 768, 24, 8, 128, 1024, True),
    (8, 768, 24, 8, 128, 1032, False), (8, 776, 24, 8, 128, 1280, True), (4, 192, 32, 32, 128, 768, False), (4, 256, 32, 32, 128, 512, True),
    (4, 256, 32, 32, 128, 516, False), (8, 256, 32, 8, 128, 288, True), (8, 256, 32, 8, 128, 296, False), (4, 257, 32, 32, 128, 880, True), (4, 257, 32, 32, 128, 884, False),
    (2, 128, 24, 8, 128, 128, False), (2, 128, 24, 8, 128, 130, True), (2, 129, 24, 8, 128, 128, True), (1, 300, 64, 8, 64, 300, True),
    (8, 300, 32, 4, 64, 1200, True), (8, 300, 32, 4, 64, 1208, False), (8, 800, 32, 4, 64, 1536, True), (4, 256, 64, 8, 64, 288, True),
    (4, 256, 64, 8, 64, 292, False), (1, 64, 8, 8, 64, 64, False), (1, 70, 8, 8, 64, 65, True),
    # at most 128 rows in a sequence: two fine blocks for every coarse one, up to 448 (d = 128) or 768
    (7, 800, 32, 8, 128, 700, True), (30, 800, 8, 8, 128, 1950, False), (30, 800, 8, 8, 128, 3840, False), (30, 800, 8, 8, 128, 3870, True),
    (12, 800, 32, 8, 128, 768, True), (12, 800, 32, 8, 128, 780, False), (12, 800, 32, 4, 64, 1536, True), (13, 800, 32, 4, 64, 832, True),
    (13, 800, 32, 4, 64, 845, False),
    # 33 to 64: as many, which either leave slots free (416 and 624) or save a second round (from 513 and 769)
    (13, 800, 32, 8, 128, 520, True), (14, 800, 32, 8, 128, 448, True), (14, 800, 32, 8, 128, 462, False), (14, 800, 32, 8, 128, 896, False), (17, 800, 32, 8, 128, 680, True),
    (24, 800, 32, 4, 64, 840, False), (25, 800, 32, 4, 64, 875, True),
])
def test_attn_rows_that_take_fine_query_tiles(B, S, Hq, Hkv, d, n, fine):
    """Lines for 256 CUs.  A grid for fine tiles has a row of blocks for every 64 rows that a sequence may hold, one for coarse tiles for
    every 128."""
    say("attn routes B=%d S=%d Hq=%d d=%d rows=%d" % (B, S, Hq, d, n))
    assert launches(_attn_call(B, S, Hq, Hkv, d, n))[0][1] == -(-min(S, n) // (64 if fine else 128))


@pytest.mark.parametrize("B,S,Hq,Hkv,n,fine", [
    (1, 700, 64, 8, 640, True), (1, 700, 64, 8, 641, False), (2, 1500, 64, 8, 384, True), (2, 1500, 64, 8, 386, False),
    (2, 1500, 32, 4, 1280, True), (2, 1500, 32, 4, 1282, False), (3, 400, 64, 8, 255, True), (3, 400, 64, 8, 258, False),
    (8, 1500, 32, 4, 256, True), (8, 1500, 32, 4, 264, False), (9, 800, 8, 8, 3960, True), (9, 800, 8, 8, 3969, False),
    (9, 800, 8, 8, 4608, False), (9, 800, 8, 8, 4617, True), (9, 800, 8, 8, 5121, False),
    (1, 300, 8, 8, 130, True), (8, 320, 64, 8, 80, False),
])
def test_attn_rows_that_take_fine_key_tiles(B, S, Hq, Hkv, n, fine):
    """Lines for 256 CUs at d = 64; the grid as for the queries."""
    say("attn routes B=%d S=%d Hq=%d d=64 rows=%d" % (B, S, Hq, n))
    assert launches(_attn_call(B, S, Hq, Hkv, 64, n))[1][0] == Hq * B * -(-min(S, n) // (64 if fine else 128))


@pytest.mark.parametrize("B,S,Hq,Hkv,d,each", [(14, 776, 32, 8, 128, 32), (14, 776, 32, 8, 128, 33), (8, 776, 32, 8, 128, 64), (8, 776, 32, 8, 128, 65),
                                               (13, 776, 32, 4, 64, 64), (13, 776, 32, 4, 64, 65),
                                               (9, 2500, 8, 8, 64, 441), (9, 2500, 8, 8, 64, 513)])
def test_layer_of_sequences_with_few_rows_each(B, S, Hq, Hkv, d, each):
    """Tiles follow the live rows: the default bound, the tight one and a host count give the same bits on both sides of a line."""
    say("layer routes B=%d S=%d Hq=%d d=%d each=%d" % (B, S, Hq, d, each))
    shape = WL.LayerShape("few_each", B=B, S=S, H=64, Hq=Hq, Hkv=Hkv, d=d, F=64, dtype="bf16")
    sv, W, dy = _random_layer(shape, S + each)
    gen = torch.Generator().manual_seed(each)
    mask = torch.zeros(B, S, dtype=torch.uint8).scatter_(1, torch.rand(B, S, generator=gen).topk(each, 1).indices, 1).to(DEV)
    desc, rows = Bn.make_desc(B, S, 64, Hq, Hkv, d, 64, "bf16"), B * each
    full, tight, host = (Bn.LayerBackward(desc, device=DEV, max_kept=m) for m in (None, rows, None))
    assert full.filtered(sv, W, dy, mask) == rows
    tight.filtered(sv, W, dy, mask)
    host.compact(sv, W, Bn.gather_rows(dy, full.idx, rows), full.idx, full.cu_kept, rows)
    torch.cuda.synchronize()
    for other in (tight, host):
        for k, v in full.grads.items():
            assert torch.equal(v[:rows] if k == "dx" else v, other.grads[k][:rows] if k == "dx" else other.grads[k]), k


@pytest.mark.parametrize("S,Hq,max_kept,kernels", [(4224, 12, None, 2), (2560, 16, None, 1), (2688, 16, None, 2), (2688, 16, 2560, 1),
                                                   (2048, 32, None, 1), (8448, 8, None, 1)])
def test_layer_dkv_launches_with_a_count_on_the_device(S, Hq, max_kept, kernels):
    """Grouped heads of 64 on 256 CUs: one launch, the plain kernel, where the pipelined one gains no more than a launch (2048 rows),
    where the rows up to the bound take fine tiles (2560) and where chains do not decide (528 tiles); both in between."""
    say("layer routes S=%d Hq=%d max_kept=%s" % (S, Hq, max_kept))
    shape = WL.LayerShape("dkv_routes", B=1, S=S, H=64, Hq=Hq, Hkv=4, d=64, F=64, dtype="bf16")
    sv, W, dy = _random_layer(shape, S)
    idx, cu, n_dev, n = Bn.build_keep_index(torch.ones((1, S), dtype=torch.uint8, device=DEV))
    plan = Bn.LayerBackward(Bn.make_desc(1, S, 64, Hq, 4, 64, 64, "bf16"), device=DEV, max_kept=max_kept)
    assert len(launches(lambda: plan.compact_dev(sv, W, dy, idx, cu, n_dev))) == 12 + kernels


def test_lora_grouped_products_in_parts():
    """A dense adapter call of 320 rows, contractions of 64 and 65 steps: t_o, the four products t_q, t_k, t_v and u_o, and the three
    of the other orientation u_q, u_k, u_v are each summed up by a launch of 16 blocks for every tile (3, 12 and 9)."""
    say("lora routes")
    shape = WL.LayerShape("lora_routes", dtype="bf16", **LORA_SHAPES["splitk"])
    sv, W, dy = _random_layer(shape, 3)
    bf = lambda *s: torch.randn(s, device=DEV).mul_(0.02).to(torch.bfloat16)
    lo = {"scale": 2.0}
    for p, (i, o) in dict(q=(shape.H, shape.Nq), k=(shape.H, shape.Nkv), v=(shape.H, shape.Nkv), o=(shape.Nq, shape.H)).items():
        lo["a" + p], lo["b" + p] = bf(i, 64), bf(64, o)
    plan = Bn.LoraBackward(Bn.make_desc(1, shape.S, shape.H, shape.Hq, shape.Hkv, shape.d, shape.F, "bf16"), 64, device=DEV)
    grids = [g[0] for g in launches(lambda: plan.run_async(sv, W, lo, dy, None))]
    cut = [b for a, b in zip(grids, grids[1:]) if a == 256 and b in (16 * 3, 16 * 12, 16 * 9)]     # behind a launch of a block per CU
    assert cut == [16 * 3, 16 * 12, 16 * 9], grids
