"""GPU parity tests: every entry point of the C-ABI library against the CPU
oracle on identical seeded inputs.  Integer/byte results must be bit-exact;
floating-point results must stay within the relative Frobenius tolerance of
the benchmark contract (2e-2 in bf16, 1e-4 in the fp32 check mode)."""
import math

import numpy as np
import pytest
import torch

from oracle import layer_oracle as O
from paper_2502_00340_amd import binding as Bn
from paper_2502_00340_amd import workloads as WL
from tests import harness as Hn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def say(msg):
    print("[case] " + msg, flush=True)


# ---------------------------------------------------------------------------
# A1 keep index
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("B,S,p", [
    (1, 1, 1.0), (1, 7, 0.5), (3, 17, 0.5), (2, 128, 0.5), (4, 2048, 0.5), (2, 4096, 0.3),
    (5, 1000, 0.7), (2, 333, 0.0), (2, 333, 1.0), (1, 8192, 0.5),
    (3, 40961, 0.5),          # above 8 blocks: two-kernel path, ragged tail
    (1, (1 << 20) + 17, 0.5),
    (8, 1 << 21, 0.5),        # 4096 blocks: every thread of the block-count scan owns several entries
])
def test_keep_index_bit_exact(B, S, p):
    say("keep_index B=%d S=%d p=%g" % (B, S, p))
    rng = np.random.default_rng(B * 7919 + S)
    mask = (rng.random((B, S)) < p).astype(np.uint8)
    if B * S > 64:
        mask.reshape(-1)[rng.integers(0, B * S, 5)] *= 255     # any non-zero byte counts as kept
    if B * S <= 200000:
        ridx, rcu, rn = O.keep_index(mask)
    else:   # the oracle's double loop is too slow here; its pins show it equals these library routines
        ridx = np.flatnonzero(mask.reshape(-1)).astype(np.int32)
        rcu = np.concatenate([[0], np.cumsum((mask != 0).sum(axis=1))]).astype(np.int32)
        rn = len(ridx)
    idx, cu, n_dev, n = Bn.build_keep_index(torch.from_numpy(mask).to(DEV))
    assert n == rn and int(n_dev.item()) == rn
    assert np.array_equal(cu.cpu().numpy(), rcu)
    assert np.array_equal(idx[:n].cpu().numpy(), ridx)


def test_keep_index_unaligned_mask_pointer():
    say("keep_index unaligned")
    rng = np.random.default_rng(5)
    raw = (rng.random(3 + 6 * 1001) < 0.5).astype(np.uint8)
    t = torch.from_numpy(raw).to(DEV)
    view = t[3:].view(6, 1001)
    ridx, rcu, rn = O.keep_index(raw[3:].reshape(6, 1001))
    idx, cu, _, n = Bn.build_keep_index(view)
    assert n == rn and np.array_equal(cu.cpu().numpy(), rcu) and np.array_equal(idx[:n].cpu().numpy(), ridx)


@pytest.mark.parametrize("off", [0, 3])
@pytest.mark.parametrize("B,S", [(1, 32768), (1, 32769), (2, 65536), (1, 131073), (131089, 1), (4097, 33), (7, 8192 * 9 + 1)])
def test_keep_index_on_both_sides_of_the_second_launch(B, S, off):
    """One launch up to 32 chunks of 4096 tokens (8 where the mask does not lie on a 16-byte boundary), two beyond; sequences that
    start inside a thread's 16 tokens, at every one of them, and at a chunk's and a span's first."""
    say("keep_index B=%d S=%d off=%d" % (B, S, off))
    for p in (0.02, 0.5, 1.0):
        mask = (np.random.default_rng(B + S).random(B * S) < p).astype(np.uint8) * 128
        t = torch.zeros(off + B * S, dtype=torch.uint8, device=DEV)
        t[off:] = torch.from_numpy(mask).to(DEV)
        idx, cu, n_dev, n = Bn.build_keep_index(t[off:].view(B, S))
        rcu = np.concatenate([[0], np.cumsum((mask.reshape(B, S) != 0).sum(axis=1))])
        assert n == rcu[-1] and int(n_dev.item()) == n
        assert np.array_equal(cu.cpu().numpy(), rcu) and np.array_equal(idx[:n].cpu().numpy(), np.flatnonzero(mask))


@pytest.mark.parametrize("off", [0, 3])
@pytest.mark.parametrize("B,S", [(1, 1), (8, 4096), (1, 32769)])
def test_keep_index_without_a_host_count(B, S, off):
    """sync=False: up to 32768 tokens without a workspace, one more token with one."""
    say("keep_index, no sync B=%d S=%d off=%d" % (B, S, off))
    mask = (np.random.default_rng(S + off).random(B * S) < 0.6).astype(np.uint8)
    t = torch.zeros(off + B * S, dtype=torch.uint8, device=DEV)
    t[off:] = torch.from_numpy(mask).to(DEV)
    idx, cu, n_dev, n = Bn.build_keep_index(t[off:].view(B, S), sync=False)
    rcu = np.concatenate([[0], np.cumsum(mask.reshape(B, S).sum(axis=1, dtype=np.int64))])
    assert n is None and int(n_dev.item()) == rcu[-1] and np.array_equal(cu.cpu().numpy(), rcu)
    assert np.array_equal(idx[:rcu[-1]].cpu().numpy(), np.flatnonzero(mask))


# ---------------------------------------------------------------------------
# A2 gather
# ---------------------------------------------------------------------------

@pytest.mark.parametrize("rows,cols,dtype,frac", [
    (256, 256, torch.float32, 0.5), (1000, 688, torch.float32, 0.5), (513, 6, torch.bfloat16, 0.5),
    (4096, 2048, torch.bfloat16, 0.5), (2048, 5632, torch.bfloat16, 0.3), (300, 8, torch.bfloat16, 1.0),
    (64, 14336, torch.bfloat16, 0.5), (100, 4, torch.float32, 0.0),
])
def test_gather_rows_bit_exact(rows, cols, dtype, frac):
    say("gather rows=%d cols=%d %s" % (rows, cols, dtype))
    rng = np.random.default_rng(rows + cols)
    src = torch.from_numpy(rng.standard_normal((rows, cols)).astype(np.float32)).to(DEV).to(dtype)
    keep = np.flatnonzero(rng.random(rows) < frac).astype(np.int32)
    idx = torch.from_numpy(keep).to(DEV)
    if len(keep) == 0:
        idx = torch.zeros(1, dtype=torch.int32, device=DEV)
    out = Bn.gather_rows(src, idx, len(keep))
    raw = src.view(torch.int16 if dtype == torch.bfloat16 else torch.int32).cpu().numpy()
    ref = O.gather_rows(raw, keep)
    got = out.view(torch.int16 if dtype == torch.bfloat16 else torch.int32).cpu().numpy()
    assert got.shape == ref.shape and np.array_equal(got, ref)


@pytest.mark.parametrize("rows,cols", [(33000, 4096), (33000, 4098)])
def test_gather_rows_beyond_the_cache(rows, cols):
    """More than 256 MB of gathered rows go past the caches, as 16-byte words and (rows of 4098 elements) as 4-byte words.
    The live rows decide: with a device-side count just above, below and far below that amount under the same bound the rows
    are the same, and those past the count are left alone."""
    src = torch.randint(-2 ** 15, 2 ** 15, (rows, cols), dtype=torch.int16, device=DEV).view(torch.bfloat16)
    idx = torch.randperm(rows, device=DEV).to(torch.int32)
    ref = src.view(torch.int16)[idx.long()]
    assert torch.equal(Bn.gather_rows(src, idx, rows).view(torch.int16), ref)
    edge = -(-(256 << 20) // (2 * cols))        # the first count whose rows are 256 MB
    for n in (rows - 100, edge, edge - 1, rows - 777, 1000, 0):
        out = torch.zeros_like(src)
        Bn.gather_rows(src, idx, rows, out=out, n_kept_dev=torch.tensor([n], dtype=torch.int32, device=DEV))
        assert torch.equal(out.view(torch.int16)[:n], ref[:n])
        assert not bool(out.view(torch.int16)[n:].any())


# ---------------------------------------------------------------------------
# A3 reduced linear backward
# ---------------------------------------------------------------------------

LINEAR_CASES = [
    # n_kept, in, out
    (128, 256, 688), (1, 8, 8), (77, 264, 200), (333, 64, 1024), (1000, 2048, 512),
    (257, 688, 256), (2867, 512, 1536),
    (4000, 4096, 1024),      # enough 256x256 tiles for the large-tile kernels (dX and dW)
    (2049, 3584, 4096),
    # more output tiles than CUs with ragged edges in both directions: blocks walk through several
    # tiles, the last round is cut into sub-tiles, some of which lie outside the matrix
    (520, 4232, 4360),
    # dX outputs that fill 256 CUs better as 256x192 tiles: one round with a ragged last tile column
    # (10 x 19 tiles), and two tiles per block (23 x 22 tiles)
    (2500, 3600, 264), (5700, 4200, 136),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_kept,fin,fout", LINEAR_CASES)
def test_linear_bwd_reduced(dtype, n_kept, fin, fout):
    say("linear %s n=%d in=%d out=%d" % (dtype, n_kept, fin, fout))
    rng = np.random.default_rng(n_kept + fin + fout)
    x = Hn.quantize(rng.standard_normal((n_kept, fin)), dtype)
    dy = Hn.quantize(rng.standard_normal((n_kept, fout)), dtype)
    w = Hn.quantize(rng.standard_normal((fin, fout)) * 0.02, dtype)
    rdx, rdw = O.linear_bwd(x.astype(np.float64), dy.astype(np.float64), w.astype(np.float64))
    dx, dw = Bn.linear_bwd_reduced(Hn.to_dev(x, dtype), Hn.to_dev(dy, dtype), Hn.to_dev(w, dtype))
    torch.cuda.synchronize()
    e1, e2 = Hn.rel_fro(Hn.to_np(dx), rdx), Hn.rel_fro(Hn.to_np(dw), rdw)
    say("  rel err dx %.3e dw %.3e" % (e1, e2))
    assert e1 <= Hn.TOL[dtype] and e2 <= Hn.TOL[dtype]
    # element-wise as well: no misplaced tile can hide inside a Frobenius norm
    tol_abs = (3e-2 if dtype == "bf16" else 1e-4)
    assert np.max(np.abs(Hn.to_np(dx) - rdx)) <= tol_abs * max(1.0, np.max(np.abs(rdx)))
    assert np.max(np.abs(Hn.to_np(dw) - rdw)) <= tol_abs * max(1.0, np.max(np.abs(rdw)))


@pytest.mark.parametrize("k", [8, 64, 72, 128, 136, 192, 200, 256, 264, 320, 440, 520, 584])
def test_linear_small_tiles_short_contraction(k):
    """Outputs of a few 128x128 tiles with contractions of one to ten 64-wide steps, whole and ragged: every position of
    the ring of four steps as the last one.  Reference in fp64 on the GPU; one rounding to bf16 and fp32 sums of k terms
    give 2^-9 relative to the value plus about k * 2^-24 * |terms|, far below the bounds used."""
    gen = torch.Generator(device=DEV).manual_seed(k)
    rn = lambda *s: torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16)
    for n, fin, fout in ((k, 264, 136), (200, 136, k)):         # dW contracts over n, dX over out
        x, dy, w = rn(n, fin), rn(n, fout), rn(fin, fout)
        dx, dw = Bn.linear_bwd_reduced(x, dy, w)
        rdx, rdw = dy.double() @ w.double().T, x.double().T @ dy.double()
        for got, ref in ((dx, rdx), (dw, rdw)):
            err = (got.double() - ref).abs()
            assert bool((err <= ref.abs() * 2.0 ** -8 + 1e-4 * math.sqrt(k)).all()), (n, fin, fout, err.max().item())


@pytest.mark.parametrize("k", [8, 56, 72, 104, 128, 136, 200])
@pytest.mark.parametrize("n,fin", [(2048, 8192), (2500, 3600), (1024, 8192)])
def test_linear_large_tiles_ragged_contraction(n, fin, k):
    """dX outputs on 256x256, 256x192 and 256x128 tiles whose contraction ends inside a 64-wide step, in its first or its
    second half.  Bounds as above."""
    gen = torch.Generator(device=DEV).manual_seed(k + n)
    rn = lambda *s: torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16)
    dy, w, dx = rn(n, k), rn(fin, k), torch.empty(n, fin, dtype=torch.bfloat16, device=DEV)
    Bn._check(Bn.lib().cf_linear_bwd_reduced(None, Bn._ptr(dy), Bn._ptr(w), n, fin, k, Bn.CF_BF16, Bn._ptr(dx), None, 0.0,
                                             Bn._stream()), "cf_linear_bwd_reduced")
    ref = dy.double() @ w.double().T
    err = (dx.double() - ref).abs()
    assert bool((err <= ref.abs() * 2.0 ** -8 + 1e-4 * math.sqrt(k)).all()), err.max().item()


@pytest.mark.parametrize("n,fin,fout", [(38, 256, 4096), (97, 512, 4096), (129, 512, 8200), (31, 1024, 4104), (257, 840, 8192), (445, 4096, 4096),
                                        (16, 8, 4104), (1, 2048, 3072)])
def test_linear_in_parts(n, fin, fout):
    """dX of few tiles and a long contraction with scratch: its parts summed up in a launch of their own or, where both products share a
    launch (the first two sizes and the seventh), by the grouped launch's; without scratch, and with dW over W.  Bounds as above."""
    gen = torch.Generator(device=DEV).manual_seed(n)
    rn = lambda *s: torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16)
    x, dy, w = rn(n, fin), rn(n, fout), rn(fin, fout)
    need = Bn.lib().cf_linear_workspace_bytes(n, fin, fout, Bn.CF_BF16)
    assert need > 0
    rdx, rdw = dy.double() @ w.double().T, x.double().T @ dy.double()
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    for scratch, over in ((ws, False), (None, False), (ws, True)):
        w2 = w.clone()
        dx, dw = torch.empty(n, fin, dtype=torch.bfloat16, device=DEV), w2 if over else torch.empty_like(w)
        Bn._check(Bn.lib().cf_linear_bwd_reduced_ws(Bn._ptr(x), Bn._ptr(dy), Bn._ptr(w2), n, fin, fout, Bn.CF_BF16, Bn._ptr(dx),
                                                    Bn._ptr(dw), 0.0, Bn._ptr(scratch), need, Bn._stream()), "cf_linear_bwd_reduced_ws")
        for got, ref, k in ((dx, rdx, fout), (dw, rdw, n)):
            err = (got.double() - ref).abs()
            assert bool((err <= ref.abs() * 2.0 ** -8 + 1e-4 * math.sqrt(k)).all()), (scratch is None, over, err.max().item())
    got = Bn.linear_bwd_reduced(x, dy, w)
    assert bool(((got[0].double() - rdx).abs() <= rdx.abs() * 2.0 ** -8 + 1e-4 * math.sqrt(fout)).all())


@pytest.mark.parametrize("fin,fout", [(0, 64), (64, 0)])
def test_linear_without_features_is_a_shape_error(fin, fout):
    """Refused before any launch, for its shape, not for the empty tensors' missing addresses."""
    t = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(Bn.CfError) as e:
        Bn.linear_bwd_reduced(t(16, fin), t(16, fout), t(fin, fout))
    assert e.value.code == 2


@pytest.mark.parametrize("n,fin,fout", [(128, 2048, 256), (300, 1032, 520), (2048, 2048, 2048)])
def test_linear_dw_over_w(n, fin, fout):
    """dW written over W: dX still comes from the weights that were there, whether the two products would share a launch
    (the first two sizes) or not."""
    gen = torch.Generator(device=DEV).manual_seed(n)
    rn = lambda *s: torch.randn(s, generator=gen, device=DEV).to(torch.bfloat16)
    x, dy, w = rn(n, fin), rn(n, fout), rn(fin, fout)
    rdx, rdw = Bn.linear_bwd_reduced(x, dy, w)
    for _ in range(5):
        dx, wdw = torch.empty_like(rdx), w.clone()
        Bn._check(Bn.lib().cf_linear_bwd_reduced(Bn._ptr(x), Bn._ptr(dy), Bn._ptr(wdw), n, fin, fout, Bn.CF_BF16, Bn._ptr(dx),
                                                 Bn._ptr(wdw), 0.0, Bn._stream()), "cf_linear_bwd_reduced")
        assert torch.equal(dx, rdx) and torch.equal(wdw, rdw)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_linear_dw_accumulate_and_empty(dtype):
    say("linear accumulate/empty %s" % dtype)
    rng = np.random.default_rng(3)
    n, fin, fout = 100, 72, 136
    x = Hn.quantize(rng.standard_normal((n, fin)), dtype)
    dy = Hn.quantize(rng.standard_normal((n, fout)), dtype)
    w = Hn.quantize(rng.standard_normal((fin, fout)), dtype)
    prev = Hn.quantize(rng.standard_normal((fin, fout)), dtype)
    acc = Hn.to_dev(prev, dtype)
    Bn.linear_bwd_reduced(Hn.to_dev(x, dtype), Hn.to_dev(dy, dtype), None, need_dx=False,
                          dw_accumulate_into=acc)
    ref = prev.astype(np.float64) + x.astype(np.float64).T @ dy.astype(np.float64)
    assert Hn.rel_fro(Hn.to_np(acc), ref) <= Hn.TOL[dtype]
    # dw only / dx only
    dx, dw = Bn.linear_bwd_reduced(None, Hn.to_dev(dy, dtype), Hn.to_dev(w, dtype), need_dw=False)
    assert dw is None and Hn.rel_fro(Hn.to_np(dx), dy.astype(np.float64) @ w.astype(np.float64).T) <= Hn.TOL[dtype]
    # no kept rows: dw = 0, dx has no rows
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    e = lambda c: torch.empty((0, c), dtype=tdt, device=DEV)
    dx0, dw0 = Bn.linear_bwd_reduced(e(fin), e(fout), Hn.to_dev(w, dtype))
    assert dx0.shape == (0, fin) and torch.count_nonzero(dw0).item() == 0
    keepacc = acc.clone()
    Bn.linear_bwd_reduced(e(fin), e(fout), None, need_dx=False, dw_accumulate_into=acc)
    assert torch.equal(acc, keepacc)


# ---------------------------------------------------------------------------
# A5 filtered attention backward
# ---------------------------------------------------------------------------

def _attn_case(dtype, B, S, Hq, Hkv, d, mask, seed, f8=np.float64):
    rng = np.random.default_rng(seed)
    T = B * S
    q = Hn.quantize(rng.standard_normal((T, Hq * d)), dtype)
    k = Hn.quantize(rng.standard_normal((T, Hkv * d)), dtype)
    v = Hn.quantize(rng.standard_normal((T, Hkv * d)), dtype)
    da = Hn.quantize(rng.standard_normal((T, Hq * d)), dtype)
    kw = dict(B=B, S=S, Hq=Hq, Hkv=Hkv, d=d)
    a, lse = O.attn_fwd(q.astype(f8), k.astype(f8), v.astype(f8), scale=1 / math.sqrt(d), **kw)
    a = Hn.quantize(a, dtype)
    lse = lse.astype(np.float32)
    rdq, rdk, rdv = O.attn_bwd_filtered(q.astype(f8), k.astype(f8), v.astype(f8), a.astype(f8),
                                        lse.astype(f8), da.astype(f8), mask, **kw)
    ridx, rcu, n = O.keep_index(mask)
    desc = Bn.make_desc(B, S, 8 * Hq, Hq, Hkv, d, 8, dtype)
    tidx = torch.from_numpy(ridx if n else np.zeros(1, np.int32)).to(DEV)
    sel = lambda arr: Hn.to_dev(arr[ridx], dtype)
    dq, dk, dv = Bn.attn_bwd_filtered(desc, sel(q), Hn.to_dev(k, dtype), Hn.to_dev(v, dtype), sel(a),
                                      torch.from_numpy(lse).to(DEV), sel(da), tidx,
                                      torch.from_numpy(rcu).to(DEV), n)
    torch.cuda.synchronize()
    errs = (Hn.rel_fro(Hn.to_np(dq), rdq[ridx]), Hn.rel_fro(Hn.to_np(dk), rdk[ridx]),
            Hn.rel_fro(Hn.to_np(dv), rdv[ridx]))
    say("  rel err dq %.3e dk %.3e dv %.3e (n_kept %d)" % (errs + (n,)))
    assert max(errs) <= Hn.TOL[dtype]
    # row by row and column by column: a wrong tail row or tile edge cannot hide in the norm of the tensor
    lines = (Hn.line_err(Hn.to_np(dq), rdq[ridx]), Hn.line_err(Hn.to_np(dk), rdk[ridx]),
             Hn.line_err(Hn.to_np(dv), rdv[ridx]))
    say("  worst row/column dq %.3e dk %.3e dv %.3e" % lines)
    assert max(lines) <= Hn.TOL_LINE[dtype]
    return errs


ATTN_SHAPES = [
    # B, S, Hq, Hkv, d
    (2, 128, 4, 4, 64),        # config 0 (MHA)
    (3, 200, 8, 2, 64),        # GQA, S not a tile multiple, ragged
    (2, 300, 4, 2, 128),
    (1, 1024, 4, 1, 128),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("B,S,Hq,Hkv,d", ATTN_SHAPES)
def test_attn_bwd_filtered_random_mask(dtype, B, S, Hq, Hkv, d):
    say("attn %s B=%d S=%d Hq=%d Hkv=%d d=%d" % (dtype, B, S, Hq, Hkv, d))
    rng = np.random.default_rng(S + d)
    mask = (rng.random((B, S)) < rng.uniform(0.2, 0.8, size=(B, 1))).astype(np.uint8)
    _attn_case(dtype, B, S, Hq, Hkv, d, mask, seed=S * 3 + d)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attn_bwd_filtered_degenerate_masks(dtype):
    B, S, Hq, Hkv, d = 3, 160, 4, 2, 64
    say("attn degenerate %s" % dtype)
    m = np.zeros((B, S), np.uint8)
    m[0, -1] = 1                       # only the last token of sequence 0; sequences 1, 2 empty
    _attn_case(dtype, B, S, Hq, Hkv, d, m, seed=1)
    m = np.ones((B, S), np.uint8)      # everything kept == dense attention backward
    _attn_case(dtype, B, S, Hq, Hkv, d, m, seed=2)
    m = np.zeros((B, S), np.uint8)
    m[1, 0] = 1                        # only the first token of the middle sequence
    m[2, 5:70] = 1                     # one contiguous span
    _attn_case(dtype, B, S, Hq, Hkv, d, m, seed=3)


LONG_ATTN_CASES = [
    # S, Hq, Hkv, d, mask kind: long sequences reach the unmasked steady-state steps of both kernels,
    # the span and ragged masks their tile edges; few heads keep the oracle's S x S matrices affordable
    (4096, 4, 2, 128, "spans"), (4096, 4, 1, 64, "ragged"), (8192, 2, 1, 128, "ragged"),
    (8192, 2, 2, 64, "spans"), (16384, 2, 1, 128, "topk"),
]


@pytest.mark.parametrize("S,Hq,Hkv,d,kind", LONG_ATTN_CASES)
def test_attn_bwd_filtered_long_context(S, Hq, Hkv, d, kind):
    say("attn long bf16 S=%d Hq=%d Hkv=%d d=%d %s" % (S, Hq, Hkv, d, kind))
    rng = np.random.default_rng(S + d + Hq)
    shape = WL.LayerShape("attn_long", B=1, S=S, H=8, Hq=Hq, Hkv=Hkv, d=d, F=8, dtype="bf16", rho=0.5,
                          mask_kind=kind)
    mask = WL.make_mask(shape, rng)
    _attn_case("bf16", 1, S, Hq, Hkv, d, mask, seed=S + 7 * d, f8=np.float32 if S > 4096 else np.float64)


@pytest.mark.parametrize("B,S,Hq,Hkv,d,kind,rho", [
    # enough key tiles that a dK/dV block takes several query heads of its KV group in a row
    # (the launcher wants about two blocks per CU of a 256-CU chip):
    (8, 2048, 8, 4, 128, "spans", 1.0),     # 128 key tiles x 8 heads: the whole group of two in one block, no partials
    (12, 2048, 16, 2, 128, "ragged", 0.8),  # half of every sequence, 96 x 16: two heads of a group of eight, four partials
    (12, 2047, 16, 2, 128, "topk", 0.8),    # 154 x 16, ragged tiles: four heads of a group of eight, two partials
    # at d = 64 a CU holds two blocks and the launcher wants twice as many
    (4, 2048, 16, 4, 64, "topk", 1.0),      # 64 x 16: one head per block, four partials
    (8, 2048, 8, 4, 64, "topk", 1.0),       # 128 x 8: one head per block, two partials
    (12, 2048, 16, 2, 64, "ragged", 0.8),   # 96 x 16: one head per block, eight partials
    (12, 2047, 16, 2, 64, "topk", 0.8),     # 154 x 16, ragged tiles: two heads of a group of eight, four partials
    (16, 1024, 16, 8, 64, "topk", 1.0),     # 128 x 16: the whole group of two in one block, no partials
    (16, 1024, 16, 2, 64, "topk", 1.0),     # two heads of a group of eight per block, four partials
    (3, 1531, 32, 4, 64, "topk", 0.3),      # 11 x 32, ragged tiles, one head per block
])
def test_attn_bwd_filtered_heads_sharing_a_block(B, S, Hq, Hkv, d, kind, rho):
    say("attn bf16 heads per block B=%d S=%d Hq=%d Hkv=%d d=%d %s rho=%.1f" % (B, S, Hq, Hkv, d, kind, rho))
    rng = np.random.default_rng(B * S + Hq)
    shape = WL.LayerShape("attn_hp", B=B, S=S, H=8, Hq=Hq, Hkv=Hkv, d=d, F=8, dtype="bf16", rho=rho, mask_kind=kind)
    mask = np.ones((B, S), np.uint8) if rho >= 1.0 else WL.make_mask(shape, rng)
    _attn_case("bf16", B, S, Hq, Hkv, d, mask, seed=S + Hq + d, f8=np.float32)


@pytest.mark.parametrize("B,S,Hq,Hkv,d", [(2, 400, 4, 2, 128), (1, 1601, 3, 3, 64), (3, 701, 4, 1, 128), (1, 3100, 16, 16, 64)])
def test_attn_bwd_filtered_split_keys(B, S, Hq, Hkv, d):
    """Few query tiles: dQ is summed from several key ranges.  The last sequence keeps only tokens near its start and
    one at its end, so that most of its tiles leave ranges empty and the last one is ragged; with and without KV groups."""
    say("attn bf16 split keys B=%d S=%d Hq=%d Hkv=%d d=%d" % (B, S, Hq, Hkv, d))
    mask = (np.random.default_rng(S).random((B, S)) < 0.6).astype(np.uint8)
    if B > 1:
        mask[-1, 70:-1] = 0
        mask[-1, -1] = 1
    _attn_case("bf16", B, S, Hq, Hkv, d, mask, seed=S + d)


@pytest.mark.parametrize("S,rows", [(800, 640), (800, 641), (1200, 640)])
def test_layer_fine_key_tiles_follow_the_live_rows(S, rows):
    """64 heads of 64: on 256 CUs 640 rows are the last that take tiles of 64 keys in the dK/dV kernel.  The kernel that has them runs
    wherever rows may be so few: the default bound, the tight one and a host count give the same bits on both sides of the line."""
    shape = WL.LayerShape("fine_keys", B=1, S=S, H=128, Hq=64, Hkv=8, d=64, F=128, dtype="bf16")
    sv, W, dy = _random_layer(shape, S + rows)
    mask = torch.zeros((1, S), dtype=torch.uint8, device=DEV)
    mask[0, torch.randperm(S, generator=torch.Generator().manual_seed(rows))[:rows].to(DEV)] = 1
    desc = Bn.make_desc(1, S, 128, 64, 8, 64, 128, "bf16")
    full, tight, host = (Bn.LayerBackward(desc, device=DEV, max_kept=m) for m in (None, rows, None))
    assert full.filtered(sv, W, dy, mask) == rows
    tight.filtered(sv, W, dy, mask)
    host.compact(sv, W, Bn.gather_rows(dy, full.idx, rows), full.idx, full.cu_kept, rows)
    torch.cuda.synchronize()
    for other in (tight, host):
        for k in full.grads:
            assert torch.equal(full.grads[k][:rows] if k == "dx" else full.grads[k],
                               other.grads[k][:rows] if k == "dx" else other.grads[k]), k


@pytest.mark.parametrize("B,S,Hq,Hkv,d,n", [
    (1, 600, 64, 8, 128, 512), (1, 600, 64, 8, 128, 513),       # 256 CUs: 4 tiles of 64 heads are the last fine ones at d = 128
    (1, 800, 64, 64, 64, 768), (1, 800, 64, 64, 64, 769),       # 6 at d = 64
    (1, 700, 64, 8, 64, 640), (1, 700, 64, 8, 64, 641),         # 5 tiles of keys at d = 64
    (3, 130, 4, 1, 128, 99), (2, 97, 4, 4, 64, 66),             # a second tile of a few rows, a wave without rows
])
def test_attn_bwd_filtered_fine_query_tiles(B, S, Hq, Hkv, d, n):
    """Tiles of 64 queries whose keys two waves share out, up to the row count where tiles of 128 take over, and one row more."""
    say("attn bf16 fine tiles B=%d S=%d Hq=%d Hkv=%d d=%d rows=%d" % (B, S, Hq, Hkv, d, n))
    mask = np.zeros(B * S, np.uint8)
    mask[np.random.default_rng(n).permutation(B * S)[:n]] = 1
    _attn_case("bf16", B, S, Hq, Hkv, d, mask.reshape(B, S), seed=n)


@pytest.mark.parametrize("Hq,Hkv,d", [(4, 1, 128), (2, 2, 128), (8, 1, 64), (2, 2, 64)])
def test_attn_bwd_filtered_rows_around_groups_of_16(Hq, Hkv, d):
    """A lane holds two rows 16 apart, a wave 32: kept rows per sequence around these, a tile of 64 and one of 128, and none."""
    counts = (0, 1, 15, 16, 17, 31, 32, 33, 47, 49, 64, 65, 129)
    say("attn bf16 rows around groups of 16 Hq=%d Hkv=%d d=%d" % (Hq, Hkv, d))
    rng = np.random.default_rng(d + Hq)
    mask = np.zeros((len(counts), 140), np.uint8)
    for b, c in enumerate(counts):
        mask[b, rng.permutation(140)[:c]] = 1
    _attn_case("bf16", len(counts), 140, Hq, Hkv, d, mask, seed=Hq + d)


@pytest.mark.parametrize("S,Hq,Hkv,d,n", [(2700, 16, 4, 64, 2673), (2700, 16, 4, 64, 2692), (1500, 4, 1, 128, 1377), (400, 8, 2, 128, 258)])
def test_attn_bwd_partials_of_ragged_key_tiles(S, Hq, Hkv, d, n):
    """dK/dV partials leave by way of LDS, two (d = 128) or four rows to a store: last tiles of 2 to 113 keys, behind long chains at d = 64,
    which the pipelined kernel takes there."""
    say("attn bf16 ragged partials S=%d Hq=%d Hkv=%d d=%d rows=%d" % (S, Hq, Hkv, d, n))
    mask = np.zeros((1, S), np.uint8)
    mask[0, np.random.default_rng(n).permutation(S)[:n]] = 1
    _attn_case("bf16", 1, S, Hq, Hkv, d, mask, seed=n, f8=np.float32)


@pytest.mark.parametrize("Hq,d,counts", [(2, 128, (300, 128, 127, 97, 96, 95, 64, 63, 33, 32, 31)), (16, 64, (2692,)), (16, 64, (2689,))])
def test_attn_bwd_whole_and_ragged_rows_of_a_wave_without_groups(Hq, d, counts):
    """Without KV groups dK and dV leave as bf16: 32 rows of a wave by way of LDS, four (d = 128) or eight to a store, fewer straight."""
    S = max(counts) + 30
    say("attn bf16 rows of a wave Hq=%d d=%d rows=%s" % (Hq, d, counts))
    rng = np.random.default_rng(d + len(counts))
    mask = np.zeros((len(counts), S), np.uint8)
    for b, c in enumerate(counts):
        mask[b, rng.permutation(S)[:c]] = 1
    _attn_case("bf16", len(counts), S, Hq, Hq, d, mask, seed=Hq + counts[0], f8=np.float32)


def test_attn_fp32_small_head_dims():
    for d in (8, 32):
        say("attn f32 d=%d" % d)
        rng = np.random.default_rng(d)
        mask = (rng.random((2, 50)) < 0.5).astype(np.uint8)
        _attn_case("f32", 2, 50, 4, 2, d, mask, seed=d)


# ---------------------------------------------------------------------------
# whole layer
# ---------------------------------------------------------------------------

SMALL_BF16 = WL.LayerShape("small_bf16", B=2, S=320, H=256, Hq=4, Hkv=2, d=64, F=704, dtype="bf16")
SMALL_BF16_D128 = WL.LayerShape("small_bf16_d128", B=3, S=200, H=384, Hq=4, Hkv=1, d=128, F=520, dtype="bf16")


def _run_layer(problem, dense=False):
    sv, W, dy, mask = problem.device_tensors(DEV)
    desc = problem.desc()
    if dense:
        got = Bn.layer_bwd_dense(desc, sv, W, dy)
        torch.cuda.synchronize()
        return got, None, None
    got, idx, cu, n = Bn.layer_bwd_filtered(desc, sv, W, dy, mask)
    torch.cuda.synchronize()
    ridx, rcu, rn = O.keep_index(problem.mask)
    assert n == rn
    assert np.array_equal(idx.cpu().numpy(), ridx) and np.array_equal(cu.cpu().numpy(), rcu)
    return got, ridx, n


@pytest.mark.parametrize("mode", ["consistent", "independent"])
def test_layer_config0_tiny_fp32(mode):
    shape = WL.CONFIGS[0]
    say("layer %s %s" % (shape.name, mode))
    p = Hn.Problem(shape, WL.config_seed(0), mode)
    got, ridx, n = _run_layer(p)
    errs = Hn.check_layer(p, got, p.oracle(), ridx, Hn.TOL["f32"])
    say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))
    gotd, _, _ = _run_layer(p, dense=True)
    Hn.check_layer(p, gotd, p.oracle(dense=True), None, Hn.TOL["f32"])


# Hq*d and Hkv*d multiples of 256: the three projection dW run as one grouped launch
SMALL_BF16_GROUPED = WL.LayerShape("small_bf16_grouped", B=2, S=192, H=320, Hq=8, Hkv=4, d=64, F=384, dtype="bf16")


@pytest.mark.parametrize("shape", [SMALL_BF16, SMALL_BF16_D128, SMALL_BF16_GROUPED], ids=lambda s: s.name)
@pytest.mark.parametrize("rho", [0.5, 0.3])
def test_layer_small_bf16(shape, rho):
    say("layer %s rho=%g" % (shape.name, rho))
    p = Hn.Problem(shape, 77, "independent", rho=rho)
    got, ridx, n = _run_layer(p)
    errs = Hn.check_layer(p, got, p.oracle(), ridx, Hn.TOL["bf16"])
    say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))
    gotd, _, _ = _run_layer(p, dense=True)
    Hn.check_layer(p, gotd, p.oracle(dense=True), None, Hn.TOL["bf16"])


def _random_layer_cases(seed, n):
    """Seeded random layer shapes: every size a multiple of 8 only, all head-group ratios, both head
    dims, every mask kind and keep ratio, with and without rotary tables."""
    rng = np.random.default_rng(seed)
    out = []
    for it in range(n):
        d = int(rng.choice([64, 128]))
        Hkv = int(rng.choice([1, 2, 4]))
        Hq = Hkv * int(rng.choice([1, 2, 4]))
        out.append(dict(
            shape=WL.LayerShape("rand%d" % it, B=int(rng.integers(1, 4)), S=int(rng.choice([64, 128, 200, 256, 320, 512])),
                                H=8 * int(rng.integers(8, 96)), Hq=Hq, Hkv=Hkv, d=d, F=8 * int(rng.integers(8, 160)),
                                dtype="bf16" if rng.random() < 0.7 else "f32",
                                rho=float(rng.choice([0.1, 0.3, 0.5, 0.7, 0.9, 1.0])),
                                mask_kind=str(rng.choice(["topk", "spans", "ragged"]))),
            rope=bool(rng.random() < 0.3), seed=7000 + it))
    return out


@pytest.mark.parametrize("case", _random_layer_cases(2024, 14), ids=lambda c: c["shape"].name)
def test_layer_random_shapes(case):
    shape = case["shape"]
    say("layer random %s: B=%d S=%d H=%d Hq=%d Hkv=%d d=%d F=%d %s rho=%.1f %s rope=%s" % (
        shape.name, shape.B, shape.S, shape.H, shape.Hq, shape.Hkv, shape.d, shape.F, shape.dtype, shape.rho,
        shape.mask_kind, case["rope"]))
    p = Hn.Problem(shape, case["seed"], "independent",
                   oracle_dtype=np.float64 if shape.dtype == "f32" else np.float32, rope=case["rope"])
    sv, W, dy, mask = p.device_tensors(DEV)
    got, idx, cu, n = Bn.layer_bwd_filtered(p.desc(), sv, W, dy, mask)
    torch.cuda.synchronize()
    ridx = np.flatnonzero(p.mask.reshape(-1))
    assert n == len(ridx) and np.array_equal(idx.cpu().numpy()[:n], ridx)
    if n == 0:
        return
    errs = Hn.check_layer(p, got, p.oracle(), ridx, Hn.TOL[shape.dtype])
    say("  n_kept=%d max rel err %.2e worst line %.2e" % (n, max(v for k, v in errs.items() if k != "worst_line"), errs["worst_line"]))


def test_layer_with_a_count_known_beforehand_never_synchronises():
    """Top-k filtering keeps a known number of tokens: index build without the host copy, gather and
    the compact entry point give bit for bit what cf_layer_bwd_filtered gives."""
    shape = SMALL_BF16
    say("layer known count %s" % shape.name)
    p = Hn.Problem(shape, 61, "independent", rho=0.5)
    sv, W, dy, mask = p.device_tensors(DEV)
    ref = Bn.LayerBackward(p.desc(), device=DEV)
    n = ref.filtered(sv, W, dy, mask)
    assert n == int(p.mask.sum())
    plan = Bn.LayerBackward(p.desc(), device=DEV)
    plan.filtered_known(sv, W, dy, mask, n)
    torch.cuda.synchronize()
    assert torch.equal(plan.idx[:n], ref.idx[:n]) and torch.equal(plan.cu_kept, ref.cu_kept)
    assert int(plan.n_kept_dev.item()) == n
    for name in Hn.GRADS:
        assert torch.equal(plan.grads[name], ref.grads[name]), name
    assert torch.equal(plan.grads["dx"][:n], ref.grads["dx"][:n])


def test_layer_filtered_call_replays_from_a_captured_graph_with_other_masks():
    """The filtered call allocates nothing, never synchronises and sizes nothing on the host by the kept
    count, so it can be captured once into a HIP graph and replayed for ANY mask: every replay (with
    eager work and synchronisations between them, a different mask, kept count and upstream gradient
    each time) must give bit for bit what the eager call gives for the same inputs."""
    shape = SMALL_BF16_GROUPED
    say("layer graph capture %s" % shape.name)
    p = Hn.Problem(shape, 71, "independent", rho=0.5)
    sv, W, dy, mask = p.device_tensors(DEV)
    ref = Bn.LayerBackward(p.desc(), device=DEV)
    plan = Bn.LayerBackward(p.desc(), device=DEV)
    plan.filtered_async(sv, W, dy, mask)        # outside the capture: one-time function attributes
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.filtered_async(sv, W, dy, mask)
    rng = np.random.default_rng(72)
    for rep, rho in enumerate((0.5, 0.2, 0.9, 0.0)):
        new_mask = (rng.random((shape.B, shape.S)) < rho).astype(np.uint8)
        mask.copy_(torch.from_numpy(new_mask).to(DEV))
        dy.copy_(Hn.to_dev(Hn.quantize(rng.standard_normal((shape.T, shape.H)), "bf16"), "bf16", DEV))
        n = ref.filtered(sv, W, dy, mask)       # eager, synchronises
        assert n == int(new_mask.sum())
        for t in list(plan.grads.values()) + [plan.idx, plan.cu_kept, plan.n_kept_dev]:
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        say("  replay %d: n_kept %d" % (rep, n))
        assert int(plan.n_kept_dev.item()) == n and int(plan._n_host[0]) == n
        assert torch.equal(plan.idx[:n], ref.idx[:n]) and torch.equal(plan.cu_kept, ref.cu_kept)
        for name in Hn.GRADS:
            assert torch.equal(plan.grads[name], ref.grads[name]), (rep, name)
        assert torch.equal(plan.grads["dx"][:n], ref.grads["dx"][:n]), rep


def test_layer_device_side_count_with_a_tight_bound_and_a_stack_without_any_host_read():
    """The filtered call reads N_k on the device.  (1) A workspace and launch bound of exactly N_k
    (max_kept = N_k, the smallest legal one) gives bit for bit what the default bound T gives.
    (2) A layer below takes the count from the device as well (cf_layer_bwd_compact_dev): the same
    bits as cf_layer_bwd_compact with the host count.  Nothing is synchronised until the end."""
    shape = SMALL_BF16_D128
    say("layer device-side count %s" % shape.name)
    p = Hn.Problem(shape, 62, "independent", rho=0.4)
    low = Hn.Problem(shape, 63, "independent", mask=p.mask)
    sv, W, dy, mask = p.device_tensors(DEV)
    sv1, W1, _, _ = low.device_tensors(DEV)
    n_true = int(p.mask.sum())
    full = Bn.LayerBackward(p.desc(), device=DEV)                       # max_kept = T
    tight = Bn.LayerBackward(p.desc(), device=DEV, max_kept=n_true)
    assert tight.ws_bytes < full.ws_bytes
    full.filtered_async(sv, W, dy, mask)
    tight.filtered_async(sv, W, dy, mask)
    lo_dev = Bn.LayerBackward(p.desc(), device=DEV)
    lo_dev.compact_dev(sv1, W1, full.grads["dx"], full.idx, full.cu_kept, full.n_kept_dev)
    n = full.n_kept()                                                   # the first synchronisation
    assert n == n_true == tight.n_kept()
    for name in Hn.GRADS:
        assert torch.equal(full.grads[name], tight.grads[name]), name
    assert torch.equal(full.grads["dx"][:n], tight.grads["dx"][:n])
    assert torch.equal(full.idx[:n], tight.idx[:n])
    lo_host = Bn.LayerBackward(p.desc(), device=DEV)
    lo_host.compact(sv1, W1, full.grads["dx"][:n], full.idx, full.cu_kept, n)
    torch.cuda.synchronize()
    for name in Hn.GRADS:
        assert torch.equal(lo_dev.grads[name], lo_host.grads[name]), name
    assert torch.equal(lo_dev.grads["dx"][:n], lo_host.grads["dx"][:n])
    # and the result is right
    errs = Hn.check_layer(p, dict(full.grads, dx=full.grads["dx"][:n]), p.oracle(), np.flatnonzero(p.mask.reshape(-1)),
                          Hn.TOL["bf16"])
    say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))


@pytest.mark.parametrize("S,Hq,Hkv,d,kept", [
    (1024, 16, 16, 64, 1024), (1024, 16, 16, 64, 300), (1024, 16, 16, 64, 1),   # of up to five key ranges: none, some, all
    (1024, 32, 8, 128, 1024), (1024, 32, 8, 128, 400), (1024, 4, 1, 128, 1024),
    # dK/dV blocks by the bound T: 576, two of them per CU; by the true count fewer, one per CU
    (2304, 32, 4, 64, 400), (2304, 32, 32, 64, 1500),
    # more rows than take fine query tiles, in two key ranges
    (4200, 12, 4, 64, 4200), (4500, 8, 8, 128, 4300),
    # two dK/dV launches with a count on the device, at the line between them and well to either side
    (2688, 16, 16, 64, 2560), (2688, 16, 16, 64, 2561), (2688, 16, 4, 64, 500), (2688, 16, 4, 64, 40),
])
def test_layer_key_ranges_follow_the_live_rows(S, Hq, Hkv, d, kept):
    """How far the dQ kernel splits the keys is decided from the live rows, by the host where it knows them and by every
    block where the device has the count; which dK/dV kernel runs at d = 64 goes by the bound.  The same bits for a host count,
    a device count under the bound T and one under a tight bound.  dQ, seen through dWq and dx, is that of the same rows without any split (the fp32 library call) up to
    the rounding of bf16."""
    say("layer key ranges S=%d Hq=%d Hkv=%d d=%d kept=%d" % (S, Hq, Hkv, d, kept))
    shape = WL.LayerShape("ranges", B=1, S=S, H=256, Hq=Hq, Hkv=Hkv, d=d, F=256, dtype="bf16")
    sv, W, dy = _random_layer(shape, kept + Hq)
    mask = torch.zeros((1, shape.S), dtype=torch.uint8, device=DEV)
    mask[0, torch.randperm(shape.S, device=DEV)[:kept]] = 1
    desc = lambda dt: Bn.make_desc(1, shape.S, shape.H, Hq, Hkv, d, shape.F, dt)
    idx, cu, n_dev, n = Bn.build_keep_index(mask)
    dyk = Bn.gather_rows(dy, idx, n)
    host, full, tight = (Bn.LayerBackward(desc("bf16"), device=DEV, max_kept=m) for m in (kept, None, kept))
    host.compact(sv, W, dyk, idx, cu, n)
    full.compact_dev(sv, W, dyk, idx, cu, n_dev)
    tight.compact_dev(sv, W, dyk, idx, cu, n_dev)
    f32 = Bn.LayerBackward(desc("f32"), device=DEV, max_kept=kept)
    up = lambda ts: {k: v.float().contiguous() for k, v in ts.items()}
    f32.compact(up(sv), up(W), dyk.float(), idx, cu, n)
    for name in Bn.GRAD_NAMES:
        cut = (lambda t: t[:n]) if name == "dx" else (lambda t: t)
        assert torch.equal(cut(host.grads[name]), cut(full.grads[name])), name
        assert torch.equal(cut(host.grads[name]), cut(tight.grads[name])), name
        assert Hn.rel_fro(Hn.to_np(cut(host.grads[name])), Hn.to_np(cut(f32.grads[name]))) <= Hn.TOL["bf16"], name


def test_layer_mask_that_keeps_more_than_max_kept_stays_inside_its_buffers():
    """A caller's bound that the mask exceeds: the call processes the first max_kept kept tokens, writes
    nothing outside buffers sized for max_kept, and reports the true count, which exposes the mistake."""
    shape = WL.LayerShape("overflow", B=2, S=256, H=256, Hq=4, Hkv=2, d=64, F=384, dtype="bf16")
    say("layer max_kept exceeded")
    p = Hn.Problem(shape, 64, "independent", rho=0.5)
    sv, W, dy, mask = p.device_tensors(DEV)
    n_true = int(p.mask.sum())
    bound = n_true - 37
    plan = Bn.LayerBackward(p.desc(), device=DEV, max_kept=bound)
    PAD = 4096
    nbytes = plan.ws.numel()
    buf = torch.full((nbytes + 2 * PAD,), 0xA5, dtype=torch.uint8, device=DEV)
    plan.ws = buf[PAD:PAD + nbytes]
    dxb = torch.full((bound * shape.H * 2 + 2 * PAD,), 0xA5, dtype=torch.uint8, device=DEV)
    plan.grads["dx"] = dxb[PAD:PAD + bound * shape.H * 2].view(torch.bfloat16).view(bound, shape.H)
    plan._g = Bn.Grads(*([plan.grads[n].data_ptr() for n in Bn.GRAD_NAMES] + [0]))
    n = plan.filtered(sv, W, dy, mask)
    assert n == n_true > bound
    for b in (buf, dxb):
        assert bool((b[:PAD] == 0xA5).all()) and bool((b[-PAD:] == 0xA5).all())
    # the first `bound` kept tokens of a single sequence mask would be a legal problem of its own: here we only
    # require finite outputs
    assert bool(torch.isfinite(plan.grads["dx"].float()).all())
    assert bool(torch.isfinite(plan.grads["dwd"].float()).all())


MAIN_GRAD_SHAPES = [
    SMALL_BF16, SMALL_BF16_D128, SMALL_BF16_GROUPED,
    WL.LayerShape("main_grad_f32", B=2, S=96, H=128, Hq=2, Hkv=1, d=64, F=256, dtype="f32"),
]


@pytest.mark.parametrize("shape", MAIN_GRAD_SHAPES, ids=lambda s: s.name)
def test_layer_main_grad_accumulation(shape):
    """main_grad = 1: the parameter gradients are fp32 buffers the calls add to.  Start from random
    buffers G0, run the filtered backward twice and the dense one once: the buffers must hold
    G0 + 2*filtered + dense gradients of the oracle; dx is the last call's, as without the flag."""
    say("layer main-grad %s" % shape.name)
    p = Hn.Problem(shape, 91, "independent", rho=0.5)
    ref, refd = p.oracle(), p.oracle(dense=True)
    sv, W, dy, mask = p.device_tensors(DEV)
    plan = Bn.LayerBackward(p.desc(), device=DEV, main_grad=True)
    rng = np.random.default_rng(92)
    g0 = {}
    for name in Hn.GRADS:
        assert plan.grads[name].dtype == torch.float32
        g0[name] = (rng.standard_normal(ref[name].shape) * ref[name].std()).astype(np.float32)
        plan.grads[name].copy_(torch.from_numpy(g0[name]))
    n = plan.filtered(sv, W, dy, mask)
    plan.filtered(sv, W, dy, mask)
    torch.cuda.synchronize()
    ridx = np.flatnonzero(p.mask.reshape(-1))
    assert n == len(ridx)
    assert Hn.rel_fro(Hn.to_np(plan.grads["dx"][:n]), ref["dx"][ridx]) <= Hn.TOL[shape.dtype]
    plan.dense(sv, W, dy)
    torch.cuda.synchronize()
    assert Hn.rel_fro(Hn.to_np(plan.grads["dx"]), refd["dx"]) <= Hn.TOL[shape.dtype]
    errs = {}
    for name in Hn.GRADS:
        added = Hn.to_np(plan.grads[name]).astype(np.float64) - g0[name]
        errs[name] = Hn.rel_fro(added, 2.0 * ref[name] + refd[name])
    say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))
    bad = {k: v for k, v in errs.items() if not (v <= Hn.TOL[shape.dtype])}
    assert not bad, bad


def _random_layer(shape, seed):
    """Saved activations, weights, upstream gradient of a bf16 layer, drawn on the GPU (lse: a constant near that of N(0,1) scores)."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rn = lambda *s, std=1.0: (torch.randn(s, generator=gen, device=DEV) * std).to(torch.bfloat16)
    T, H, F, Nq, Nkv = shape.T, shape.H, shape.F, shape.Nq, shape.Nkv
    sv = dict(x=rn(T, H), r=rn(T, H), q=rn(T, Nq), k=rn(T, Nkv), v=rn(T, Nkv), attn_out=rn(T, Nq), gate=rn(T, F), up=rn(T, F),
              lse=torch.full((shape.B, shape.Hq, shape.S), 6.0, device=DEV))
    W = {n: rn(i, o, std=0.02) for n, (i, o) in dict(wq=(H, Nq), wk=(H, Nkv), wv=(H, Nkv), wo=(Nq, H), wg=(H, F), wu=(H, F),
                                                    wd=(F, H)).items()}
    W.update(g1=rn(H) * 0.02 + 1.0, g2=rn(H) * 0.02 + 1.0)
    return sv, W, rn(T, H)


@pytest.mark.parametrize("F", [4352, 5632, 6656])
@pytest.mark.parametrize("kept", [96, 700])
def test_layer_main_grad_full_round_and_a_remainder(F, kept):
    """dWg and dWu of a 2048-wide layer are 16 * F/256 tiles of 256x256 in one launch: one round of 256 CUs and 16, 96 or 160
    tiles more, which go out in quarters, halves or whole.  The blocks with a part of the remainder start its loads right
    behind the write-out of a whole tile, into the LDS that the fp32 write-out stages its rows in.  Both outputs are made from
    the same fp32 accumulators, so the fp32 buffers rounded to bf16 have the bits of the bf16 call; added to itself once
    more every element doubles exactly."""
    say("layer main-grad remainder F=%d kept=%d" % (F, kept))
    shape = WL.LayerShape("main_grad_rounds", B=1, S=1024, H=2048, Hq=4, Hkv=2, d=64, F=F, dtype="bf16")
    sv, W, dy = _random_layer(shape, F + kept)
    mask = torch.zeros((1, shape.S), dtype=torch.uint8, device=DEV)
    mask[:, shape.S - kept:] = 1
    desc = Bn.make_desc(shape.B, shape.S, shape.H, shape.Hq, shape.Hkv, shape.d, F, "bf16")
    ref = Bn.LayerBackward(desc, device=DEV)
    plan = Bn.LayerBackward(desc, device=DEV, main_grad=True)
    assert ref.filtered(sv, W, dy, mask) == kept
    for rep in (1, 2):
        plan.filtered(sv, W, dy, mask)
        for name in ("dwq", "dwk", "dwv", "dwo", "dwg", "dwu", "dwd"):
            got = plan.grads[name] / rep
            bad = (got.to(torch.bfloat16) != ref.grads[name]).nonzero()
            assert bad.numel() == 0, (name, rep, bad.shape[0], bad[0].tolist())


@pytest.mark.parametrize("F", [1792, 4864])
def test_layer_gain_gradients_beside_the_products(F):
    """The column sums of the gain gradients go out with the parameter-gradient products where these have more than one round of
    tiles (F = 4864: 513 and more tiles on 256 CUs), before them otherwise; H is no multiple of a block's 32 columns.  The fp32
    buffers come from the same sums, so rounded they have the bits of the bf16 call, and doubled by a second call they double exactly."""
    shape = WL.LayerShape("gain_grads", B=2, S=40, H=2056, Hq=4, Hkv=2, d=64, F=F, dtype="bf16")
    say("layer gain gradients F=%d" % F)
    p = Hn.Problem(shape, F, "independent", rho=0.5)
    got, ridx, n = _run_layer(p)
    Hn.check_layer(p, got, p.oracle(), ridx, Hn.TOL["bf16"])
    sv, W, dy, mask = p.device_tensors(DEV)
    plan = Bn.LayerBackward(p.desc(), device=DEV, main_grad=True)
    ref = Bn.LayerBackward(p.desc(), device=DEV)
    ref.filtered(sv, W, dy, mask)
    for rep in (1, 2):
        plan.filtered(sv, W, dy, mask)
        for name in ("dg1", "dg2"):
            assert torch.equal((plan.grads[name] / rep).to(torch.bfloat16), ref.grads[name]), (name, rep)


@pytest.mark.parametrize("main_grad", [False, True])
@pytest.mark.parametrize("H,Hq,Hkv,d,F", [(512, 8, 2, 64, 256), (840, 12, 4, 64, 2312), (2048, 32, 4, 64, 4864), (2048, 32, 4, 64, 5632)])
def test_layer_parameter_gradients_in_one_launch_or_one_by_one(H, Hq, Hkv, d, F, main_grad):
    """The seven dW products share a launch, also where an output lies over an operand that the caller owns (dx over dy in a dense
    call, here: they read a copy of it).  The list's remainder of tiles is cut
    into quarters (first size), stays whole at the end of ragged matrices (second), is cut into halves (600 tiles) and stays whole
    behind two full rounds (672).  Both calls give the same bits."""
    shape = WL.LayerShape("one_launch", B=1, S=328, H=H, Hq=Hq, Hkv=Hkv, d=d, F=F, dtype="bf16")
    sv, W, dy = _random_layer(shape, F)
    desc = Bn.make_desc(shape.B, shape.S, H, Hq, Hkv, d, F, "bf16")
    ref, over = (Bn.LayerBackward(desc, device=DEV, main_grad=main_grad) for _ in range(2))
    ref.dense(sv, W, dy)
    dy2 = dy.clone()
    over._g.dx = dy2.data_ptr()
    over.dense(sv, W, dy2)
    torch.cuda.synchronize()
    for k in ref.grads:
        assert torch.equal(dy2 if k == "dx" else over.grads[k], ref.grads[k]), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_layer_invariants_on_gpu_outputs(dtype):
    """Keep ratio 1 reproduces the dense call bit for bit (same kernels, same
    shapes); an empty mask gives zero parameter gradients; garbage in the
    filtered rows of dy does not leak."""
    shape = WL.LayerShape("inv", B=2, S=192, H=256, Hq=4, Hkv=2, d=64, F=512, dtype=dtype)
    say("layer invariants %s" % dtype)
    ones = np.ones((shape.B, shape.S), np.uint8)
    p = Hn.Problem(shape, 5, "independent", mask=ones)
    got, ridx, n = _run_layer(p)
    gotd, _, _ = _run_layer(p, dense=True)
    assert n == shape.T
    for name in Hn.GRADS + ("dx",):
        assert torch.equal(got[name], gotd[name]), name
    # empty mask
    p0 = Hn.Problem(shape, 5, "independent", mask=np.zeros_like(ones))
    got0, _, n0 = _run_layer(p0)
    assert n0 == 0 and got0["dx"].shape[0] == 0
    for name in Hn.GRADS:
        assert torch.count_nonzero(got0[name]).item() == 0, name
    # garbage in filtered rows of dy
    ph = Hn.Problem(shape, 6, "independent", rho=0.5)
    got1, ridx1, _ = _run_layer(ph)
    dead = ph.mask.reshape(-1) == 0
    ph.dy[dead] = Hn.quantize(1e4 * np.ones_like(ph.dy[dead]), dtype)
    got2, _, _ = _run_layer(ph)
    for name in Hn.GRADS + ("dx",):
        assert torch.equal(got1[name], got2[name]), name


def test_layer_ragged_batch_with_empty_sequence():
    shape = WL.LayerShape("ragged", B=4, S=96, H=128, Hq=2, Hkv=1, d=64, F=256, dtype="bf16")
    say("layer ragged")
    rng = np.random.default_rng(9)
    mask = np.zeros((4, 96), np.uint8)
    mask[0] = rng.random(96) < 0.8
    mask[1] = 0
    mask[2] = rng.random(96) < 0.2
    mask[3, -1] = 1
    p = Hn.Problem(shape, 9, "independent", mask=mask)
    got, ridx, n = _run_layer(p)
    Hn.check_layer(p, got, p.oracle(), ridx, Hn.TOL["bf16"])


def test_layer_stack_of_two_shares_one_index():
    """Two layers chained: the compact dx of the upper layer is the compact upstream
    gradient of the lower one, which reuses the index and is not synchronised.  The
    oracle runs the same chain on full-length tensors (its dx is zero on filtered rows)."""
    shape = WL.LayerShape("stack", B=2, S=288, H=256, Hq=4, Hkv=2, d=64, F=640, dtype="bf16")
    say("layer stack of two")
    top = Hn.Problem(shape, 21, "independent", rho=0.5)
    low = Hn.Problem(shape, 22, "independent", mask=top.mask)
    sv2, W2, dy, mask = top.device_tensors(DEV)
    sv1, W1, _, _ = low.device_tensors(DEV)
    plan2 = Bn.LayerBackward(top.desc(), device=DEV)
    plan1 = Bn.LayerBackward(low.desc(), device=DEV)
    n = plan2.filtered(sv2, W2, dy, mask)
    plan1.compact(sv1, W1, plan2.grads["dx"][:n], plan2.idx, plan2.cu_kept, n)
    torch.cuda.synchronize()
    ref2 = top.oracle()
    low.dy = np.asarray(ref2["dx"], dtype=np.float64)      # full length, zero on filtered rows
    ref1 = low.oracle()
    ridx = np.flatnonzero(top.mask.reshape(-1))
    got = dict(plan1.grads)
    got["dx"] = got["dx"][:n]
    errs = Hn.check_layer(low, got, ref1, ridx, Hn.TOL["bf16"])
    say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))
    # the compact call on the upper layer's own inputs reproduces the filtered call bit for bit
    keep = {k: v.clone() for k, v in plan2.grads.items()}
    dyk = Bn.gather_rows(dy, plan2.idx, n)
    plan2.compact(sv2, W2, dyk, plan2.idx, plan2.cu_kept, n)
    torch.cuda.synchronize()
    for k in keep:
        a, b = (plan2.grads[k][:n], keep[k][:n]) if k == "dx" else (plan2.grads[k], keep[k])
        assert torch.equal(a, b), k


def test_layer_stack_of_eight_error_growth_over_depth():
    """Eight different layers chained through the compact entry point: the top layer builds the index,
    every layer below takes the compact dx of the layer above (the library's own, with its rounding)
    as upstream gradient.  The oracle runs the same chain in float64 on full-length tensors.  The
    relative error of every layer's outputs against the chained oracle is printed and must stay
    within the single-layer tolerance: rounding errors handed down the stack do not blow up."""
    depth = 8
    shape = WL.LayerShape("stack8", B=2, S=288, H=256, Hq=4, Hkv=2, d=64, F=640, dtype="bf16")
    say("layer stack of eight")
    probs = [Hn.Problem(shape, 300 + l, "independent", rho=0.5) for l in range(depth)]
    mask_np = probs[0].mask
    ridx = np.flatnonzero(mask_np.reshape(-1))
    plans = [Bn.LayerBackward(shape_p.desc(), device=DEV) for shape_p in probs[:2]]
    dev = [p.device_tensors(DEV) for p in probs]
    worst = []
    ref_dy = probs[0].dy.astype(np.float64)
    n = None
    for l in range(depth):
        sv, W, dy, mask = dev[l]
        plan = plans[l & 1]
        if l == 0:
            n = plan.filtered(sv, W, dy, mask)
        else:
            plan.compact(sv, W, plans[(l - 1) & 1].grads["dx"][:n], plans[0].idx, plans[0].cu_kept, n)
        torch.cuda.synchronize()
        probs[l].mask = mask_np
        probs[l].dy = ref_dy
        ref = probs[l].oracle()
        got = dict(plan.grads)
        got["dx"] = got["dx"][:n]
        errs = Hn.check_layer(probs[l], got, ref, ridx, Hn.TOL["bf16"])
        worst.append(max(v for k, v in errs.items() if k != "worst_line"))
        say("  layer %d below the top: dx %.2e worst tensor %.2e" % (l, errs["dx"], worst[-1]))
        ref_dy = np.asarray(ref["dx"], dtype=np.float64)       # full length, zero on filtered rows
    assert max(worst) <= Hn.TOL["bf16"]
    # no blow-up: the deepest layer is within a small factor of the top one
    assert worst[-1] <= 4.0 * worst[0] + 1e-3


@pytest.mark.parametrize("dtype,mode", [("f32", "consistent"), ("bf16", "independent")])
def test_layer_with_rotary_embedding(dtype, mode):
    """q and k are rotated tensors: the layer applies the transposed rotation to dq and dk at
    the original positions of the kept rows (filtered and dense calls)."""
    shape = WL.LayerShape("rope", B=2, S=160, H=256, Hq=4, Hkv=2, d=64, F=384, dtype=dtype)
    say("layer rotary %s" % dtype)
    p = Hn.Problem(shape, 31, mode, rho=0.5, rope=True)
    got, ridx, n = _run_layer(p)
    ref = p.oracle()
    errs = Hn.check_layer(p, got, ref, ridx, Hn.TOL[dtype])
    say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))
    gotd, _, _ = _run_layer(p, dense=True)
    Hn.check_layer(p, gotd, p.oracle(dense=True), None, Hn.TOL[dtype])
    # the rotation matters: without it dWq is far from the reference
    p.rope, keep = None, p.rope
    got0, _, _ = _run_layer(p)
    p.rope = keep
    assert Hn.rel_fro(Hn.to_np(got0["dwq"]), ref["dwq"]) > 10 * Hn.TOL[dtype]


@pytest.mark.parametrize("Hq,Hkv,d,S,rho", [
    (4, 4, 64, 100, 0.5),       # one key tile, dQ and dK written by their own kernels
    (3, 3, 128, 301, 0.7),      # the same at d = 128, several tiles, ragged
    (4, 1, 128, 170, 0.6),      # dK from partials
    (2, 2, 64, 401, 0.6),       # dQ from key ranges, dK whole
    (4, 2, 128, 401, 0.4),      # both from partials
    # more rows than take fine tiles: dQ from coarse ones; dK at d = 64 whole from the plain kernel and, dense, the pipelined one
    (32, 32, 64, 800, 0.98), (32, 4, 64, 800, 0.98), (32, 32, 128, 600, 0.9), (32, 8, 128, 600, 0.9),
])
def test_layer_rotary_embedding_wherever_dq_and_dk_are_written(Hq, Hkv, d, S, rho):
    """Lines for 256 CUs."""
    shape = WL.LayerShape("rope_routes", B=2, S=S, H=256, Hq=Hq, Hkv=Hkv, d=d, F=128, dtype="bf16")
    say("layer rotary %d/%d d=%d S=%d" % (Hq, Hkv, d, S))
    p = Hn.Problem(shape, S + d, "independent", rho=rho, rope=True)
    got, ridx, n = _run_layer(p)
    Hn.check_layer(p, got, p.oracle(), ridx, Hn.TOL["bf16"])
    gotd, _, _ = _run_layer(p, dense=True)
    Hn.check_layer(p, gotd, p.oracle(dense=True), None, Hn.TOL["bf16"])


def test_no_write_outside_the_outputs_and_the_workspace():
    """Every output tensor and the workspace sit inside a larger allocation filled with a
    sentinel; after filtered, compact and dense calls on a ragged shape (no dimension a tile
    multiple) the guard bands are untouched."""
    shape = WL.LayerShape("guard", B=3, S=200, H=264, Hq=6, Hkv=2, d=64, F=520, dtype="bf16")
    say("guard bands")
    p = Hn.Problem(shape, 41, "independent", rho=0.37)
    sv, W, dy, mask = p.device_tensors(DEV)
    desc = p.desc()
    plan = Bn.LayerBackward(desc, device=DEV)
    PAD = 4096                                      # bytes on each side
    raw = {}

    def guarded(t):
        nbytes = t.numel() * t.element_size()
        buf = torch.full((nbytes + 2 * PAD,), 0xA5, dtype=torch.uint8, device=DEV)
        view = buf[PAD:PAD + nbytes].view(t.dtype).view(t.shape)
        return buf, view

    for name in list(plan.grads):
        raw[name], plan.grads[name] = guarded(plan.grads[name])
    raw["idx"], plan.idx = guarded(plan.idx)
    raw["cu"], plan.cu_kept = guarded(plan.cu_kept)
    raw["ws"], plan.ws = guarded(plan.ws)
    plan._g = Bn.Grads(*[plan.grads[n].data_ptr() for n in Bn.GRAD_NAMES])
    n = plan.filtered(sv, W, dy, mask)
    dyk = Bn.gather_rows(dy, plan.idx, n)
    plan.compact(sv, W, dyk, plan.idx, plan.cu_kept, n)
    plan.dense(sv, W, dy)
    torch.cuda.synchronize()
    for name, buf in raw.items():
        assert bool((buf[:PAD] == 0xA5).all()) and bool((buf[-PAD:] == 0xA5).all()), name


LORA_NAMES = ("daq", "dbq", "dak", "dbk", "dav", "dbv", "dao", "dbo")


def _run_lora(p, lora_np, rank, mask_on=True):
    sv, W, dy, mask = p.device_tensors(DEV)
    lo = {k: (Hn.to_dev(v, p.dtype, DEV) if isinstance(v, np.ndarray) else v) for k, v in lora_np.items()}
    plan = Bn.LoraBackward(p.desc(), rank, device=DEV)
    n = plan.run(sv, W, lo, dy, mask if mask_on else None)
    torch.cuda.synchronize()
    return plan, n


LORA_SHAPES = {
    "small": dict(B=2, S=224, H=256, Hq=4, Hkv=2, d=64, F=384),
    # few tiles and contractions of 64 and 65 steps: the grouped launches cut them into several parts, the last one ragged (H = 4104)
    "splitk": dict(B=1, S=320, H=4104, Hq=64, Hkv=16, d=64, F=512),
    # d_act, dh2, da and dh1 in parts (five and six segments with the rank-16 products), the grouped launches whole
    "parts": dict(B=2, S=129, H=2048, Hq=16, Hkv=4, d=64, F=4104),
    # with every token kept 4 x 65 row tiles in one grouped launch: nothing is split and blocks take a second item
    "rows": dict(B=5, S=1664, H=128, Hq=2, Hkv=1, d=64, F=128),
}


@pytest.mark.parametrize("dtype,mode,rank,which", [("f32", "consistent", 8, "small"),
                                                   ("bf16", "independent", 16, "small"),
                                                   ("bf16", "independent", 64, "small"),
                                                   ("bf16", "independent", 64, "splitk"),
                                                   ("bf16", "independent", 24, "splitk"),
                                                   ("bf16", "independent", 136, "splitk"),
                                                   ("bf16", "independent", 8, "rows")])
def test_layer_lora(dtype, mode, rank, which):
    """Adapters on q, k, v, o with frozen base weights: adapter gradients and compact dx against
    the oracle, filtered and with every token kept."""
    shape = WL.LayerShape("lora", dtype=dtype, **LORA_SHAPES[which])
    say("layer lora %s rank %d %s" % (dtype, rank, which))
    rng = np.random.default_rng(51)
    lora_np = {k: (Hn.quantize(v, dtype) if isinstance(v, np.ndarray) else v)
               for k, v in WL.make_lora(shape, rng, rank=rank, alpha=2.0 * rank).items()}
    p = Hn.Problem(shape, 52, mode, rho=0.9 if which == "splitk" else 0.5)
    if mode == "consistent":    # saved tensors of the adapted forward
        lo64 = {k: (v.astype(np.float64) if isinstance(v, np.ndarray) else v) for k, v in lora_np.items()}
        _, sv = O.layer_fwd(p.saved["x"].astype(np.float64), {k: v.astype(np.float64) for k, v in p.W.items()},
                            lora=lo64, **p.kw)
        p.saved = {k: (np.asarray(v, dtype=np.float32) if k == "lse" else Hn.quantize(v, dtype)) for k, v in sv.items()}
    lo = {k: (v.astype(p.oracle_dtype) if isinstance(v, np.ndarray) else v) for k, v in lora_np.items()}
    svo = {k: v.astype(p.oracle_dtype) for k, v in p.saved.items()}
    Wo = {k: v.astype(p.oracle_dtype) for k, v in p.W.items()}
    for mask_on in (True, False):
        plan, n = _run_lora(p, lora_np, rank, mask_on)
        ref = O.layer_bwd(svo, Wo, p.dy.astype(p.oracle_dtype), p.mask if mask_on else None, lora=lo, **p.kw)
        ridx = np.flatnonzero(p.mask.reshape(-1)) if mask_on else np.arange(shape.T)
        assert n == len(ridx)
        errs = {k: Hn.rel_fro(Hn.to_np(plan.grads[k]), ref[k]) for k in LORA_NAMES}
        errs["dx"] = Hn.rel_fro(Hn.to_np(plan.grads["dx"][:n]), ref["dx"][ridx])
        say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))
        bad = {k: v for k, v in errs.items() if not (v <= Hn.TOL[dtype])}
        assert not bad, bad
        if mask_on:
            # the same call with the tightest bound (max_kept = N_k): launches and split-K plans are sized
            # for it instead of for T, the result must meet the same tolerance
            sv_d, W_d, dy_d, mask_d = p.device_tensors(DEV)
            lo_d = {k: (Hn.to_dev(v, p.dtype, DEV) if isinstance(v, np.ndarray) else v) for k, v in lora_np.items()}
            plan.max_kept = n
            assert plan.run(sv_d, W_d, lo_d, dy_d, mask_d) == n
            errs = {k: Hn.rel_fro(Hn.to_np(plan.grads[k]), ref[k]) for k in LORA_NAMES}
            errs["dx"] = Hn.rel_fro(Hn.to_np(plan.grads["dx"][:n]), ref["dx"][ridx])
            bad = {k: v for k, v in errs.items() if not (v <= Hn.TOL[dtype])}
            assert not bad, ("tight bound", bad)


def test_layer_lora_nothing_kept():
    """A mask that keeps no token: the count is only known on the device, every adapter gradient must
    come out zero (the kernels run on empty row and contraction ranges)."""
    shape = WL.LayerShape("lora0", dtype="bf16", **LORA_SHAPES["splitk"])
    say("layer lora, empty mask")
    rng = np.random.default_rng(53)
    lora_np = {k: (Hn.quantize(v, "bf16") if isinstance(v, np.ndarray) else v)
               for k, v in WL.make_lora(shape, rng, rank=64, alpha=128.0).items()}
    p = Hn.Problem(shape, 54, "independent", mask=np.zeros((shape.B, shape.S), np.uint8))
    plan, n = _run_lora(p, lora_np, 64, True)
    assert n == 0
    for k in LORA_NAMES:
        assert not bool(plan.grads[k].float().abs().max() > 0), k


def test_layer_lora_same_result_twice():
    """2572 kept rows of a 4096-wide layer: the dh2 and dh1 products run on 242 tiles of 256x192.  With a device-side count
    there are as many blocks as CUs, more than tiles, and the spare ones leave.  The adapter call gives the same bits
    every time and under the true count as its bound; the call without adapters gives those of a host count, whose launches
    have a block per tile and none to spare."""
    shape = WL.LayerShape("lora_spare_blocks", B=4, S=732, H=4096, Hq=4, Hkv=1, d=128, F=256, dtype="bf16")
    say("layer lora, fewer tiles than blocks")
    sv, W, dy = _random_layer(shape, 61)
    gen = torch.Generator(device=DEV).manual_seed(62)
    rn = lambda *s: (torch.randn(s, generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
    H, Nq, Nkv, R = shape.H, shape.Nq, shape.Nkv, 16
    lo = {"scale": 2.0}
    for p, (i, o) in dict(q=(H, Nq), k=(H, Nkv), v=(H, Nkv), o=(Nq, H)).items():
        lo["a" + p], lo["b" + p] = rn(i, R), rn(R, o)
    mask = torch.zeros((shape.B, shape.S), dtype=torch.uint8, device=DEV)
    mask[:, :643] = 1
    n = 4 * 643
    desc = Bn.make_desc(shape.B, shape.S, H, shape.Hq, shape.Hkv, shape.d, shape.F, "bf16")
    plan, tight = Bn.LoraBackward(desc, R, device=DEV), Bn.LoraBackward(desc, R, device=DEV)
    tight.max_kept = n
    first = None
    for it, pl in enumerate([plan] * 5 + [tight]):
        assert pl.run(sv, W, lo, dy, mask) == n
        got = {k: v.clone() for k, v in pl.grads.items()}
        got["dx"] = got["dx"][:n]
        first = first or got
        for k in got:
            assert torch.equal(got[k], first[k]), (it, k)
    idx, cu, n_dev, _ = Bn.build_keep_index(mask)
    dyk = Bn.gather_rows(dy, idx, n)
    dev, host = Bn.LayerBackward(desc, device=DEV), Bn.LayerBackward(desc, device=DEV)
    dev.compact_dev(sv, W, dyk, idx, cu, n_dev)
    host.compact(sv, W, dyk, idx, cu, n)
    for k in Bn.GRAD_NAMES:
        cut = n if k == "dx" else None
        assert torch.equal(dev.grads[k][:cut], host.grads[k][:cut]), k


def test_layer_dense_dx_over_attn_out():
    """The attention output is dead when a dense call writes dx: a caller may let dx lie over it, with and without adapters."""
    say("dx over attn_out")
    shape = WL.LayerShape("dx_over_attn_out", B=2, S=512, H=512, Hq=8, Hkv=2, d=64, F=256, dtype="bf16")
    sv, W, dy = _random_layer(shape, 71)
    gen = torch.Generator(device=DEV).manual_seed(72)
    rn = lambda *s: (torch.randn(s, generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
    H, Nq, Nkv, R = shape.H, shape.Nq, shape.Nkv, 16
    lo = {"scale": 2.0}
    for p, (i, o) in dict(q=(H, Nq), k=(H, Nkv), v=(H, Nkv), o=(Nq, H)).items():
        lo["a" + p], lo["b" + p] = rn(i, R), rn(R, o)
    desc = Bn.make_desc(shape.B, shape.S, H, shape.Hq, shape.Hkv, shape.d, shape.F, "bf16")
    for make, call in ((lambda: Bn.LoraBackward(desc, R, device=DEV), lambda pl, s: pl.run(s, W, lo, dy, None)),
                       (lambda: Bn.LayerBackward(desc, device=DEV), lambda pl, s: pl.dense(s, W, dy))):
        ref, over = make(), make()
        call(ref, sv)
        for _ in range(5):
            s2 = dict(sv, attn_out=sv["attn_out"].clone())
            over._g.dx = s2["attn_out"].data_ptr()
            call(over, s2)
            torch.cuda.synchronize()
            for k in ref.grads:
                assert torch.equal(s2["attn_out"] if k == "dx" else over.grads[k], ref.grads[k]), k


PARTS_SHAPE = dict(B=2, H=2048, Hq=16, Hkv=4, d=64, F=4104)


@pytest.mark.parametrize("S,rho", [(45, 0.7), (129, 0.6), (250, 0.9)])
def test_layer_products_in_parts(S, rho):
    """A few rows against long contractions: d_act, dh2, da and dh1 are left in up to sixteen fp32 parts that the next pass adds up.
    62 (one tile row), 154 and 450 rows; a contraction that ends inside a step (F = 4104), a part that spans two segments.  The
    parts follow the live count: the default bound, the tight one and a host count give the same bits."""
    shape = WL.LayerShape("parts", S=S, dtype="bf16", **PARTS_SHAPE)
    say("layer in parts S=%d" % S)
    p = Hn.Problem(shape, S, "independent", rho=rho, rope=True, oracle_dtype=np.float32)
    sv, W, dy, mask = p.device_tensors(DEV)
    ridx = np.flatnonzero(p.mask.reshape(-1))
    n = len(ridx)
    full = Bn.LayerBackward(p.desc(), device=DEV)
    assert full.filtered(sv, W, dy, mask) == n
    errs = Hn.check_layer(p, dict(full.grads, dx=full.grads["dx"][:n]), p.oracle(), ridx, Hn.TOL["bf16"])
    say("  " + " ".join("%s=%.1e" % kv for kv in errs.items()))
    tight, host = Bn.LayerBackward(p.desc(), device=DEV, max_kept=n), Bn.LayerBackward(p.desc(), device=DEV)
    tight.filtered(sv, W, dy, mask)
    host.compact(sv, W, Bn.gather_rows(dy, full.idx, n), full.idx, full.cu_kept, n)
    torch.cuda.synchronize()
    for other in (tight, host):
        for k in full.grads:
            assert torch.equal(full.grads[k][:n] if k == "dx" else full.grads[k], other.grads[k][:n] if k == "dx" else other.grads[k]), k
    gotd, _, _ = _run_layer(p, dense=True)
    Hn.check_layer(p, gotd, p.oracle(dense=True), None, Hn.TOL["bf16"])


def test_layer_lora_products_in_parts():
    """The same products of an adapter call (five and six segments with the rank-16 ones), filtered and dense."""
    test_layer_lora("bf16", "independent", 16, "parts")
