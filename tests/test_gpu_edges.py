"""Tile and wave edges of the attention kernels against the fp64 oracle: row counts around a
wave (32), a workgroup (256 queries, 128 keys) and a key or query tile (64, 96), documents that
start inside a wave's 32 rows, tiles over more documents than the kernels look up by scalar
loads, and ring segments of 32 rows.  Before each case the kernels run on NaN inputs of a full
tile, so that rows which a short tile leaves as they were in LDS hold NaN."""
import numpy as np
import pytest
import torch

import oracle
from paper_2609_34318_amd import inputs, ring

from gpu_util import assert_grad_close, assert_lse_close, assert_o_close, dev_bf16, f32

pytestmark = pytest.mark.gpu
D_QK, D_V = 192, 128


def _run(cu, H, q_segs, steps, q, kv, do, Hkv, ds):
    sh = ring.make_share(cu, H, q_segs, steps, n_kv_heads=Hkv, ds_kv_heads=1 if ds else 0)
    o, lse, _ = ring.forward(sh, q, kv)
    dq = torch.zeros((sh.nq, H, D_QK), device="cuda")
    dkv = [(torch.zeros((k.shape[0], Hkv, D_QK), device="cuda"), torch.zeros((k.shape[0], Hkv, D_V), device="cuda"))
           for k, _ in kv]
    ring.backward(sh, q, kv, do, dq, dkv)
    torch.cuda.synchronize()
    return o.cpu().numpy(), lse.cpu().numpy(), dq.cpu().numpy(), [(a.cpu().numpy(), b.cpu().numpy()) for a, b in dkv]


def _poison(H, Hkv, ds):
    """A full-tile problem on NaN: every kernel leaves NaN in the LDS it used."""
    nan = lambda *shape: torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    n = 512
    _run([0, n], H, [(0, n)], [[(0, n)]], nan(n, H, D_QK), [(nan(n, Hkv, D_QK), nan(n, Hkv, D_V))], nan(n, H, D_V),
         Hkv, ds)


def _check(cu, H, q_segs, steps, Hkv, ds, seed):
    q = inputs.rows("q", q_segs, H, D_QK, seed, "sharp")
    do = inputs.rows("do", q_segs, H, D_V, seed, "sharp")
    kv = [(inputs.rows("k", s, Hkv, D_QK, seed, "sharp"), inputs.rows("v", s, Hkv, D_V, seed, "sharp")) for s in steps]
    _poison(H, Hkv, ds)
    o, lse, dq, dkv = _run(cu, H, q_segs, steps, dev_bf16(q), [(dev_bf16(k), dev_bf16(v)) for k, v in kv], dev_bf16(do),
                           Hkv, ds)
    union = [s for st in steps for s in st]
    O, L = oracle.attn_fwd(f32(q), np.concatenate([f32(k) for k, _ in kv]), np.concatenate([f32(v) for _, v in kv]), cu,
                           q_segs, union)
    assert_o_close(o, O)
    assert_lse_close(lse, L)
    ref_dq = np.zeros(q.shape)
    for i, (st, (k, v)) in enumerate(zip(steps, kv)):
        a, b, c = oracle.attn_bwd(f32(q), f32(k), f32(v), O, L, f32(do), cu, q_segs, st)
        ref_dq += a
        assert_grad_close(dkv[i][0], b, what=f"dK step {i}")
        assert_grad_close(dkv[i][1], c, what=f"dV step {i}")
    assert_grad_close(dq, ref_dq, what="dQ")


@pytest.mark.parametrize("n", [1, 31, 33, 64, 95, 97, 129, 255, 257, 353])
def test_row_counts_around_the_tiles(n):
    _check([0, n], 2, [(0, n)], [[(0, n)]], 2, False, 40)


@pytest.mark.parametrize("lens,ds", [
    ([40, 9, 70, 1, 8, 200, 24], False),       # starts inside a wave's rows, the last inside the last wave
    ([3, 5, 0, 7, 11, 2, 13, 1, 17, 4, 9, 6, 100, 3, 2, 1, 60, 90, 10], False),  # > 9 documents in a tile
    ([40, 9, 70, 1, 8, 200, 24], True),
    ([3, 5, 0, 7, 11, 2, 13, 1, 17, 4, 9, 6, 100, 3, 2, 1, 60, 96, 12], True),
])
def test_documents_inside_waves_and_tiles(lens, ds):
    cu = [0] + [int(x) for x in np.cumsum(lens)]
    n = cu[-1]
    assert not ds or n % 32 == 0
    _check(cu, 8, [(0, n)], [[(0, n)]], 2, ds, 41)


@pytest.mark.parametrize("ds", [False, True])
def test_segments_of_one_wave(ds):
    """K/V segments of 32 and 96 rows side by side: a 64-key step of the dQ kernel ends past its
    segment, at or beyond the end of the next one."""
    segs = [(0, 32), (64, 32), (160, 96), (288, 32)]
    _check([0, 352], 2, [(32, 64), (256, 96)], [segs, [(96, 64), (256, 32)]], 2, ds, 42)
