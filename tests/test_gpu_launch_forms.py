"""Forms of one launch against each other: a ring step merged by its own kernel against the partial
and the merge call; split work items against whole ones; the
split dK/dV of the stored-dS passes against the recompute path's; recorded calls before and after an
upload for the same problem; calls on one plan that overlap."""
import math

import pytest
import torch

from paper_2609_34318_amd import hydra

pytestmark = pytest.mark.gpu
D_QK, D_V = 192, 128
BF16, F32 = torch.bfloat16, torch.float32


def _randn(g, shape, dtype=BF16, scale=1.0):
    return (torch.randn(shape, generator=g, device="cuda") * scale).to(dtype)


def _inputs(p, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return (_randn(g, (p.nq, p.n_heads, D_QK)), _randn(g, (p.nk, p.n_kv_heads, D_QK)),
            _randn(g, (p.nk, p.n_kv_heads, D_V), scale=0.1), g)


def _ws(p):
    return torch.empty(hydra.workspace_size(p), dtype=torch.uint8, device="cuda")


def _scratch(p):
    n = hydra.split_scratch_size(p)
    return torch.empty(n, dtype=torch.uint8, device="cuda") if n else None


CASES = [
    # cu, heads, K/V heads, q segments, K/V segments
    ([0, 353], 2, 2, [(0, 353)], [(0, 100)]),                       # rows of several waves, odd ends
    ([0, 40, 49, 300], 8, 2, [(0, 300)], [(60, 200)]),              # rows that see no key of the step
    ([0, 4001], 1, 1, [(2001, 1999)], [(0, 2001)]),                 # items that a scratch splits
    ([0, 4001], 1, 1, [(1000, 1001), (3000, 97)], [(0, 3000)]),     # some of them, a short tile
    ([0, 1024], 3, 3, [(0, 512)], [(512, 512)]),                    # no tile at all
    ([0, 64], 4, 1, [(0, 64)], []),                                 # no key
]


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("bf16,planned", [(False, False), (True, False), (True, True)])
@pytest.mark.parametrize("split", [False, True])
def test_merged_step(case, bf16, planned, split):
    cu, H, Hkv, q_segs, k_segs = CASES[case]
    p = hydra.Problem(cu, H, q_segs, k_segs, n_kv_heads=Hkv)
    q, k, v, g = _inputs(p, 50 + case)
    o = _randn(g, (p.nq, H, D_V), F32, 0.1)
    lse = _randn(g, (H, p.nq), F32, 2.0) + 5
    lse[:, ::7] = -math.inf  # nothing seen so far
    o[::7] = 0
    o_ref, lse_ref, part, part_lse = o.clone(), lse.clone(), torch.empty_like(o), torch.empty_like(lse)
    b = torch.full(o.shape, 7.0, dtype=BF16, device="cuda") if bf16 else None
    b_ref = torch.empty_like(b) if bf16 else None
    ws, scratch = _ws(p), _scratch(p) if split else None
    assert not split or case not in (2, 3) or scratch is not None
    hydra.attn_fwd(p, q, k, v, part, part_lse, ws, scratch=scratch)
    hydra.lse_merge(o_ref, lse_ref, part, part_lse, o_bf16=b_ref)
    if planned:
        hydra.attn_plan(p, ws)
    hydra.attn_fwd_merge(p, q, k, v, o, lse, ws, o_bf16=b, planned=planned, scratch=scratch)
    torch.cuda.synchronize()
    # the same operations in 32 bits; a product fused into the sum moves it by one rounding of it
    assert torch.equal(torch.isinf(lse), torch.isinf(lse_ref))
    torch.testing.assert_close(lse, lse_ref, rtol=2 ** -22, atol=2 ** -22)
    torch.testing.assert_close(o, o_ref, rtol=0, atol=2 ** -22 * max(o.abs().max().item(), 1.0))
    if bf16:
        assert torch.equal(b, o.to(BF16))


def test_merged_step_of_weight_zero_is_dropped():
    """A partial whose weight underflows to 0 leaves the merge as it was, whatever it holds."""
    p = hydra.Problem([0, 256], 2, [(128, 128)], [(0, 128)])
    q, k, v, g = _inputs(p, 60)
    v.fill_(math.inf)
    o, lse = _randn(g, (p.nq, 2, D_V), F32), torch.full((2, p.nq), 300.0, device="cuda")
    want = o.clone()
    hydra.attn_fwd_merge(p, q, k, v, o, lse, _ws(p))
    torch.cuda.synchronize()
    assert torch.equal(o, want) and bool((lse == 300.0).all())


def _backward(call, p, t, ds=None, **kw):
    q, k, v, o, lse, d_o, ws = t
    out = [torch.zeros((p.nq, p.n_heads, D_QK), device="cuda"), torch.zeros((p.nk, p.n_kv_heads, D_QK), device="cuda"),
           torch.zeros((p.nk, p.n_kv_heads, D_V), device="cuda")]
    if call is hydra.attn_bwd_noalloc:
        call(p, q, k, v, o, lse, d_o, *out)
    elif ds is not None:
        call(p, q, k, v, o, lse, d_o, *out, ds, ws, **kw)
    else:
        call(p, q, k, v, o, lse, d_o, *out, ws, **kw)
    torch.cuda.synchronize()
    return out


def _tensors(p, seed):
    q, k, v, g = _inputs(p, seed)
    o = torch.empty((p.nq, p.n_heads, D_V), device="cuda")
    lse = torch.empty((p.n_heads, p.nq), device="cuda")
    b = torch.empty(o.shape, dtype=BF16, device="cuda")
    ws = _ws(p)
    hydra.attn_fwd(p, q, k, v, o, lse, ws, o_bf16=b)
    return q, k, v, b, lse, _randn(g, o.shape), ws


@pytest.mark.parametrize("cu,H,Hkv", [([0, 4000], 1, 1), ([0, 1900, 4096], 4, 1), ([0, 2048], 2, 2)])
def test_split_and_whole_items(cu, H, Hkv):
    """The same sums in another order: dK, dV and dQ of the parts are 32-bit partial sums of the same
    products, so that they differ by 32-bit rounding.  A scratch that holds dK/dV's parts alone
    leaves dQ whole; one too small for anything, and the no-allocation call, all items."""
    p = hydra.Problem(cu, H, [(0, cu[-1])], [(0, cu[-1])], n_kv_heads=Hkv)
    t = _tensors(p, 61)
    scratch = _scratch(p)
    whole = _backward(hydra.attn_bwd, p, t)
    split = _backward(hydra.attn_bwd, p, t, scratch=scratch)
    assert any(not torch.equal(a, b) for a, b in zip(whole, split))
    for a, b in zip(whole, split):
        # sums of up to 4096 terms of either sign, in 32 bits: a few roundings of the largest partial sum
        assert (a - b).norm() <= 2 ** -20 * a.norm()
    for a, b in zip(whole, _backward(hydra.attn_bwd, p, t, scratch=scratch[:1024])):
        assert torch.equal(a, b)
    for a, b in zip(whole, _backward(hydra.attn_bwd_noalloc, p, t)):
        assert torch.equal(a, b)
    some = _backward(hydra.attn_bwd, p, t, scratch=scratch[:scratch.numel() - 16])
    assert all(torch.equal(x, a) or torch.equal(x, b) for x, a, b in zip(some, whole, split))


@pytest.mark.parametrize("kv_heads", [1, 2])
@pytest.mark.parametrize("split", [False, True])
def test_stored_ds_passes_sum_dk_dv_alike(kv_heads, split):
    p = hydra.Problem([0, 1920, 4096], 4, [(0, 4096)], [(0, 4096)], n_kv_heads=2)
    t = _tensors(p, 62)
    ds = torch.empty(hydra.bwd_ds_bytes(p, kv_heads), dtype=torch.uint8, device="cuda")
    scratch = _scratch(p) if split else None
    a, b = _backward(hydra.attn_bwd, p, t, scratch=scratch), _backward(hydra.attn_bwd_ds, p, t, ds, scratch=scratch)
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])


@pytest.mark.parametrize("split", [False, True])
def test_recorded_calls_survive_a_forward_of_the_same_problem(split):
    """A forward that uploads its own plan into the workspace of a recorded forward and backward of
    the same problem writes the bytes that are there: the replays read the same plan."""
    for cu, H in (([0, 3000, 4096], 2), ([0, 300], 3)):  # split and whole items
        p = hydra.Problem(cu, H, [(0, cu[-1])], [(0, cu[-1])])
        q, k, v, b, lse, d_o, ws = _tensors(p, 63)
        scratch, other = (_scratch(p), _scratch(p)) if split else (None, None)
        hydra.attn_plan(p, ws)
        o = torch.empty((p.nq, H, D_V), device="cuda")
        grads = [torch.empty((p.nq, H, D_QK), device="cuda"), torch.empty((p.nk, H, D_QK), device="cuda"),
                 torch.empty((p.nk, H, D_V), device="cuda")]
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for t in grads:
                t.fill_(0.0)
            hydra.attn_fwd(p, q, k, v, o, lse, ws, o_bf16=b, planned=True, scratch=scratch)
            hydra.attn_bwd(p, q, k, v, b, lse, d_o, *grads, ws, planned=True, scratch=scratch)
        want = None
        for rep in range(3):
            graph.replay()
            torch.cuda.synchronize()
            got = [t.clone() for t in grads + [o, lse]]
            want = want or got
            for x, y in zip(got, want):
                assert torch.equal(x, y), rep
            assert all(bool(t.abs().max() > 0) for t in got)
            hydra.attn_fwd(p, q, k, v, torch.empty_like(o), torch.empty_like(lse), ws, scratch=other)
            torch.cuda.synchronize()


@pytest.mark.parametrize("split", [False, True])
def test_planned_forwards_of_one_plan_overlap(split):
    """A planned forward only reads the workspace: forwards of one plan on two streams, beside a
    backward of it on a third, give what they give one after another."""
    p = hydra.Problem([0, 3000, 4096], 2, [(0, 4096)], [(0, 4096)])
    q, k, v, b, lse, d_o, ws = _tensors(p, 64)
    hydra.attn_plan(p, ws)
    torch.cuda.synchronize()
    before = ws.clone()
    qs = [q, q * 2]
    scratch = [_scratch(p) if split else None for _ in range(3)]
    out = lambda: [(torch.empty((p.nq, 2, D_V), device="cuda"), torch.empty((2, p.nq), device="cuda")) for _ in qs]  # noqa: E731
    want, got = out(), out()
    for x, (o, l), s in zip(qs, want, scratch):
        hydra.attn_fwd(p, x, k, v, o, l, ws, planned=True, scratch=s)
        torch.cuda.synchronize()
        assert torch.equal(ws, before)
    grads = [[torch.zeros((p.nq, 2, d), device="cuda") for d in (D_QK, D_QK, D_V)] for _ in range(2)]
    hydra.attn_bwd(p, q, k, v, b, lse, d_o, *grads[0], ws, planned=True, scratch=scratch[2])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(3)]
    for _ in range(5):
        for x, (o, l), s, st in zip(qs, got, scratch, streams):
            hydra.attn_fwd(p, x, k, v, o, l, ws, planned=True, scratch=s, stream=st)
    hydra.attn_bwd(p, q, k, v, b, lse, d_o, *grads[1], ws, planned=True, scratch=scratch[2], stream=streams[2])
    torch.cuda.synchronize()
    for (o, l), (o2, l2) in zip(want, got):
        assert torch.equal(o, o2) and torch.equal(l, l2)
    for x, y in zip(*grads):
        assert torch.equal(x, y)
