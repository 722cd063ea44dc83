"""How an attention call is split into columns (workgroup spans): the shipped arithmetic compiled
for the CPU over random calls, and on the GPU the contexts where it can go wrong, against fp64
attention over the decoded cache."""
import ctypes
import math
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads
from parity import Setup, bf16_bits_to_torch
from test_gpu_parity import LayerCfg, _draw

NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "attn_spans.cpp")


class Split:
    FIELDS = ("chunk", "n_chunks", "n_part", "per_seq", "spare", "max_span", "min_log2")

    def __init__(self, so):
        self.lib = ctypes.CDLL(so)
        self.lib.split.argtypes = [ctypes.c_int64] * 7 + [ctypes.c_void_p]
        self.lib.unit.argtypes = [ctypes.c_uint32] * 3 + [ctypes.c_int, ctypes.c_void_p]
        self.lib.counts.argtypes = [ctypes.c_void_p, ctypes.c_int64] + [ctypes.c_uint32] * 3 + \
            [ctypes.c_void_p]

    def plan(self, *args):
        out = np.zeros(7, np.int64)
        self.lib.split(*args, out.ctypes.data)
        return dict(zip(self.FIELDS, (int(x) for x in out)))

    def unit(self, u, heads, n_part, columns_first):
        out = np.zeros(2, np.uint32)
        self.lib.unit(u, heads, n_part, columns_first, out.ctypes.data)
        return int(out[0]), int(out[1])

    def counts(self, tiles, p):
        tiles, out = np.ascontiguousarray(tiles, np.uint32), np.zeros(len(tiles), np.uint32)
        self.lib.counts(tiles.ctypes.data, len(tiles), p["spare"], p["max_span"], p["min_log2"],
                        out.ctypes.data)
        return out.astype(np.int64)


@pytest.fixture(scope="module")
def spans(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not found")
    so = str(tmp_path_factory.mktemp("spans") / "spans.so")
    subprocess.run([cxx, "-O2", "-std=c++17", "-shared", "-fPIC", "-o", so, NATIVE], check=True)
    return Split(so)


def test_columns_fit(spans):
    """Random batches, heads, passes, block sizes, contexts (zero, equal, one long among short,
    up to the bound) and devices: every sequence has a column, the counts never exceed the columns
    nor the columns the workspace's partials, no sequence holds more columns than it has tiles,
    every wave's share is within what it can address, and spans are as even as tvq_spans.h
    states."""
    rng = np.random.default_rng(1)
    for case in range(6000):
        vpw = (32, 16)[case % 2]
        B = int(math.exp(rng.uniform(0, math.log(6000))))
        H, n_pass = int(rng.choice([1, 2, 4, 8, 32])), int(rng.integers(1, 17))
        block = 0 if case % 5 == 0 else 32 << int(rng.integers(0, 12))
        max_ctx = int(math.exp(rng.uniform(0, math.log(300000))))
        slots = int(rng.choice([256, 3072, 4096, 4864]))
        p = spans.plan(B, H, n_pass, max_ctx, block, vpw, slots)
        if p["n_part"] == 0:                            # a wave per row: its tokens and blocks
            assert 2 * B * H * n_pass >= slots and max_ctx <= 32 * vpw <= 63 * 32
            continue
        assert B <= p["n_part"] <= B * p["n_chunks"] and p["spare"] >= 0
        kind = 1 if block == 0 else case % 4
        lens = rng.integers(0, max_ctx + 1, B)
        if kind == 1:
            lens[:] = max_ctx
        elif kind == 2:
            lens[:] = rng.integers(0, min(max_ctx, 40) + 1, B)
            lens[rng.integers(0, B)] = max_ctx
        elif kind == 3:
            lens[:] = 0
        T = -(-lens // vpw)
        if block == 0:
            assert p["spare"] == 0 and p["n_part"] == B * p["per_seq"]
            n = np.full(B, p["per_seq"])
        else:
            n = spans.counts(T, p)
            if p["spare"] == 0:
                assert p["n_part"] == B * p["per_seq"] and n.max() <= p["per_seq"]
            else:
                assert B <= 4096
        assert n.min() >= 1 and n.sum() <= p["n_part"] and (n <= np.maximum(T, 1)).all()
        span = -(-T // n)
        assert (-(-span // 4) * vpw <= min(4096, 63 * block or 4096)).all()
        if p["spare"]:
            total = int(T.sum())
            assert (span <= max(1 << p["min_log2"], -(-total // p["spare"]))).all()


@pytest.mark.parametrize("B,H,n_pass", [(33, 8, 1), (49, 8, 1), (65, 8, 1), (72, 8, 1), (98, 8, 1),
                                        (129, 8, 1), (160, 8, 1), (33, 8, 2), (13, 8, 2),
                                        (17, 32, 1), (3, 8, 1), (16, 8, 1)])
@pytest.mark.parametrize("block", [0, 256])
def test_rows_that_do_not_divide_the_device(spans, B, H, n_pass, block):
    """4,096-token contexts on a device of 1,024 workgroups: a compute unit's share of the work,
    placed four workgroups at a time as places fall free, is never 1.15 times that of a wave per
    chunk of the workspace rule (four waves on the fullest of its SIMDs, in whole chunks): what
    that split spends on waves of its own for the tables and the partials."""
    p = spans.plan(B, H, n_pass, 4096, block, 16, 4096)
    T = 256
    c = int(spans.counts(np.full(B, T), p)[0]) if block else p["per_seq"]
    rows, units = B * H * n_pass, 256
    span = -(-T // c)
    groups = rows * c
    # at most one go: the fullest unit's whole spans; more: an even share and a last span alone
    load = -(-groups // units) * span if groups <= 1024 else groups / units * span + span
    chunks = -(-rows * p["n_chunks"] // 1024) * (p["chunk"] // 16) * 4
    assert load <= 1.15 * chunks, (p, load, chunks)


def test_wave_per_row(spans):
    """The calls of test_attention_spans that name it take a wave per row on a device of 4,096 wave
    slots, and their neighbours do not: a longer context, fewer rows."""
    for args, rows in (((32, 8, 16, 128, 32, 16), True), ((32, 8, 16, 129, 32, 16), False),
                       ((64, 8, 16, 512, 32, 16), True), ((64, 8, 16, 513, 0, 16), False),
                       ((31, 8, 16, 128, 0, 16), False), ((45, 7, 13, 100, 32, 32), True),
                       ((45, 7, 13, 129, 32, 32), False), ((16, 8, 15, 100, 0, 32), False)):
        assert (spans.plan(*args, 4096)["n_part"] == 0) == rows, args


@pytest.mark.parametrize("H", [1, 2, 8, 32])
def test_units_of_a_sequence_are_neighbours(spans, H):
    """Every (column, head) has one unit in either order, and where the contexts differ the units
    of a column are consecutive, so that one long sequence's workgroups go round the XCDs and
    their compute units."""
    n_part = 129
    every = [(c, h) for c in range(n_part) for h in range(H)]
    assert sorted(spans.unit(u, H, n_part, 0) for u in range(n_part * H)) == every
    assert [spans.unit(u, H, n_part, 1) for u in range(n_part * H)] == every


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
    # a wave per row: as many rows as wave slots, contexts up to the longest of them; a last
    # workgroup of three rows and a last pass of two heads
    (128, 8, 64, 512, 32, [512, 0, 1, 15, 16, 17, 511, 500] * 8),
    (128, 8, 64, 128, 32, [128, 0, 1, 15, 16, 17, 127, 113] * 4),
    (64, 7, 50, 100, 32, [100, 0, 1, 31, 32, 33, 99, 64, 65] * 5),
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
    # of thousands of heads some have scores of 400, whose own rounding moves the weights by 1.7e-5
    # in any split: a quarter of it keeps them to the bound
    q *= 0.25 if G > 8 else 1.0
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
    the other heads of its pass are within rounding of what they are without it."""
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
    assert torch.isfinite(want).all() and torch.equal(got[1, 5], want[1, 5])
    # the heads of a wave share the moment at which their reference points are raised, so the
    # others' weights may be rounded at another point: the bound the entry point states
    err = (got - want).norm(dim=-1) / want.norm(dim=-1).clamp(min=1e-30)
    assert err.max() < 1e-5
