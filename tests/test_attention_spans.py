"""How an attention call is split: the columns (workgroup spans) of sequences whose contexts are
device data, by a model of the rule on the CPU, and on the GPU at the contexts where it can go
wrong, against fp64 attention over the decoded cache."""
import math

import numpy as np
import pytest

import workloads
from parity import Setup, bf16_bits_to_torch
from test_gpu_parity import LayerCfg, _draw


def _plan(d, B, H, n_pass, max_ctx, block, slots=4096):
    """The plan of a paged call: (tiles per context, n_part, spare, max_span, chunk columns)."""
    vpw = 64 // (d // 32)
    max_chunk = min(4096, 63 * block)
    step = 2 * vpw
    per_row = max(1, slots // (B * H * n_pass))
    ch = max(-(-(-(-max_ctx // per_row)) // step) * step, 4 * vpw)
    ch = min(ch, max_chunk // step * step)
    n_chunks = -(-max_ctx // ch)
    tiles = -(-max_ctx // vpw)
    max_span = 4 * (max_chunk // vpw)
    need = -(-tiles // max_span)
    most = min(-(-tiles // 4), n_chunks)
    n_part = max(B * need, min(slots // 4 // (H * n_pass), B * most))
    return n_part, n_part - B * need, max_span, n_chunks


def _counts(T, spare, max_span):
    total = max(int(T.sum()), 1)
    c = np.maximum(1, -(-T // max_span))
    more = (T.astype(np.float64) * np.float64(spare) / np.float64(total)).astype(np.int64)
    return np.maximum(c, np.minimum(c + more, -(-T // 4)))


def test_span_counts_fit_the_columns():
    """Random batches, heads, passes, block sizes and contexts (zero, equal, one long among
    short, up to the bound): the counts never exceed the columns, nor the columns the workspace
    rule's partials; every wave's share is within what it can address; equal contexts share the
    columns evenly."""
    rng = np.random.default_rng(1)
    for case in range(4000):
        d = (64, 128)[case % 2]
        vpw = 64 // (d // 32)
        B = int(math.exp(rng.uniform(0, math.log(300))))
        H, n_pass = int(rng.choice([1, 2, 4, 8, 32])), int(rng.integers(1, 17))
        block = 32 << int(rng.integers(0, 12))
        max_ctx = int(math.exp(rng.uniform(0, math.log(300000))))
        n_part, spare, max_span, n_chunks = _plan(d, B, H, n_pass, max_ctx, block)
        assert B <= n_part <= B * n_chunks and spare >= 0
        kind = case % 4
        lens = rng.integers(0, max_ctx + 1, B)
        if kind == 1:
            lens[:] = max_ctx
        elif kind == 2:
            lens[:] = rng.integers(0, min(max_ctx, 40) + 1, B)
            lens[rng.integers(0, B)] = max_ctx
        elif kind == 3:
            lens[:] = 0
        T = -(-lens // vpw)
        n = _counts(T, spare, max_span)
        assert n.min() >= 1 and n.sum() <= n_part
        share = -(-(-(-T // n)) // 4)                   # most tiles of a wave
        assert (share * vpw <= min(4096, 63 * block)).all()
        if kind == 1 and T[0] // 4 >= n_part // B:
            assert (n == n_part // B).all()


@pytest.mark.gpu
@pytest.mark.parametrize("d,H,G,max_ctx,block,lens", [
    # more sequences than a wave has lanes (two, five a lane); empty, one-token and tile-edge
    # contexts
    (128, 1, 4, 300, 32, [0, 1, 15, 16, 17, 300, 63, 64, 65] + [33] * 70),
    (128, 2, 4, 600, 32, [600, 0, 17, 64] * 72 + [1, 600, 599]),
    (64, 2, 3, 300, 64, [0, 1, 31, 32, 33, 300, 127, 128, 129] + [5] * 62),
    # every context one span: the workgroups store the outputs themselves
    (128, 2, 8, 64, 32, [64, 0, 1, 40]),
    (64, 2, 4, 128, 32, [128, 100, 3]),
    # one long context among short ones; contexts longer than a span can be at this block size
    (128, 1, 6, 9000, 32, [9000, 20, 8065, 0]),
    (64, 1, 4, 9000, 32, [8064, 8999, 1]),
])
def test_attention_spans(gpu, d, H, G, max_ctx, block, lens):
    """fp32 outputs within 1e-5 of fp64 attention over the decoded pool (the bound the entry
    point states), zeros for an empty context, and the contiguous entry point within the same
    bound where every context is the full one."""
    import torch
    B = len(lens)
    s = Setup(1, H, d, [LayerCfg(64, 64)], workloads.sign_table(23, 1, d)).build()
    k, v = _draw(workloads.get("C2"), 1, B, H, max_ctx, d, "bf16", 24)
    per = -(-max_ctx // block)
    lay = s.gpu.pool_layout(B * per, block)
    pool = torch.zeros((lay.total_bytes,), dtype=torch.uint8, device="cuda")
    tab = torch.from_numpy(np.random.default_rng(5).permutation(B * per).astype(np.int32)
                           .reshape(B, per)).cuda()
    kd, vd = bf16_bits_to_torch(k).cuda(), bf16_bits_to_torch(v).cuda()
    s.gpu.encode_paged(kd, vd, torch.zeros(B, dtype=torch.int32, device="cuda"), tab, pool, lay)
    ko = torch.empty((1, B, H, max_ctx, d), dtype=torch.float32, device="cuda")
    vo = torch.empty_like(ko)
    s.gpu.decode_paged(pool, lay, tab, 0, max_ctx, ko, vo)
    q = torch.randn((B, H * G, d), generator=torch.Generator("cuda").manual_seed(6), device="cuda")
    ctx = torch.tensor(lens, dtype=torch.int32, device="cuda")
    out = torch.full_like(q, float("nan"))
    scale = d ** -0.5
    s.gpu.attention_paged(pool, lay, tab, ctx, max_ctx, 0, q, out, scale)
    flat = s.gpu.layout(B, max_ctx)
    cache = torch.zeros((flat.total_bytes,), dtype=torch.uint8, device="cuda")
    s.gpu.encode(kd, vd, cache, flat)
    full = torch.full_like(q, float("nan"))
    s.gpu.attention(cache, flat, 0, max_ctx, q, full, scale)
    torch.cuda.synchronize()
    qc, kc, vc = q.cpu().double(), ko[0].cpu().double(), vo[0].cpu().double()

    def check(got, n, b):
        for h in range(H):
            qs = qc[b, h * G:(h + 1) * G]
            w = torch.softmax(qs @ kc[b, h, :n].T * scale, -1)
            ref = w @ vc[b, h, :n]
            err = (got[b, h * G:(h + 1) * G].double() - ref).norm(dim=-1) / ref.norm(dim=-1)
            assert err.max() < 1e-5, (b, h, n, float(err.max()))
    got, got_full = out.cpu(), full.cpu()
    for b, n in enumerate(lens):
        if n == 0:
            assert not got[b].any()
        else:
            check(got, n, b)
        if b < 6:
            check(got_full, max_ctx, b)


@pytest.mark.gpu
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [40, 3000])
def test_query_head_of_nan(gpu, d, T):
    """A query head of NaN has no score above -inf and gives zeros, like an empty context, with one
    span per sequence (T = 40: the workgroups store the outputs) as with several (the merge does);
    the other heads of its pass are what they are without it."""
    import torch
    B, H, G = 2, 2, 4
    s = Setup(1, H, d, [LayerCfg(64, 64)], workloads.sign_table(31, 1, d)).build()
    k, v = _draw(workloads.get("C2"), 1, B, H, T, d, "bf16", 32)
    lay = s.gpu.layout(B, T)
    cache = torch.zeros((lay.total_bytes,), dtype=torch.uint8, device="cuda")
    s.gpu.encode(bf16_bits_to_torch(k).cuda(), bf16_bits_to_torch(v).cuda(), cache, lay)
    q = torch.randn((B, H * G, d), generator=torch.Generator("cuda").manual_seed(7), device="cuda")
    want, got = torch.empty_like(q), torch.empty_like(q)
    s.gpu.attention(cache, lay, 0, T, q, want, d ** -0.5)
    q[1, 5] = float("nan")
    s.gpu.attention(cache, lay, 0, T, q, got, d ** -0.5)
    want[1, 5] = 0
    assert torch.isfinite(want).all() and torch.equal(got, want)
