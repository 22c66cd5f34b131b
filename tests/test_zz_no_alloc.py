"""The index build that allocates nothing (cf_build_keep_index_static) against the ordinary entry
point: bit-exact idx, cu_kept and N_k on two calls in a row, the second on a smaller input, through
the C ABI with caller-owned buffers only."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2502_00340_amd import binding as Bn

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _both(mask_np, idx, cu, n_dev, off=0):
    """off: bytes between the mask and an aligned address"""
    B, S = mask_np.shape
    mask = torch.zeros(off + B * S, dtype=torch.uint8, device=DEV)[off:].view(B, S)
    mask.copy_(torch.from_numpy(mask_np))
    ridx, rcu, rn_dev, rn = Bn.build_keep_index(mask)          # the existing entry point (workspace argument)
    idx.fill_(-7)
    cu.fill_(-7)
    n_dev.fill_(-7)
    lib = Bn.lib()
    vp = lambda t: C.c_void_p(t.data_ptr())
    rc = lib.cf_build_keep_index_static(vp(mask), B, S, vp(idx), vp(cu), vp(n_dev),
                                        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, rc
    torch.cuda.synchronize()
    n = int(n_dev.item())
    assert n == rn == int(mask_np.astype(bool).sum())
    assert torch.equal(cu[:B + 1], rcu)
    assert torch.equal(idx[:n], ridx[:n])
    assert np.array_equal(idx[:n].cpu().numpy(), np.flatnonzero(mask_np.reshape(-1)).astype(np.int32))
    return n


def test_static_scratch_index_build_matches_the_workspace_one_on_two_calls_in_a_row():
    print("[case] no-alloc keep index, two calls", flush=True)
    rng = np.random.default_rng(11)
    # caller-owned buffers, sized once for the larger call
    idx = torch.empty(3 * 200001, dtype=torch.int32, device=DEV)
    cu = torch.empty(8, dtype=torch.int32, device=DEV)
    n_dev = torch.empty(1, dtype=torch.int32, device=DEV)
    big = (rng.random((3, 200001)) < 0.5).astype(np.uint8)      # 74 spans: counts and flag bits go through the scratch
    small = (rng.random((2, 70001)) < 0.3).astype(np.uint8)     # 18 spans: fewer counts, and the bits elsewhere in the same scratch
    n1 = _both(big, idx, cu, n_dev)
    n2 = _both(small, idx, cu, n_dev)
    assert n1 > n2 > 0
    odd = (rng.random((3, 20001)) < 0.5).astype(np.uint8)       # 8 spans, not on a 16-byte boundary: two launches from 32769 tokens on
    _both(odd, idx, cu, n_dev, off=5)
    for B, S in ((3, 40961), (2, 20000), (2, 300)):             # 31, 10 and one chunk: one launch, no scratch
        _both((rng.random((B, S)) < 0.5).astype(np.uint8), idx, cu, n_dev)


def test_static_scratch_index_build_at_its_maximum_size():
    print("[case] no-alloc keep index, 2^24 tokens", flush=True)
    rng = np.random.default_rng(12)
    mask = (rng.random((4, 1 << 22)) < 0.5).astype(np.uint8)
    idx = torch.empty(1 << 24, dtype=torch.int32, device=DEV)
    cu = torch.empty(5, dtype=torch.int32, device=DEV)
    n_dev = torch.empty(1, dtype=torch.int32, device=DEV)
    _both(mask, idx, cu, n_dev)
