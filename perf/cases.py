"""Cases whose speed is measured: the calls that a serving program makes of the codec.

A case is one pass through `Codec`'s entry points:

  encode     tokens of every (layer, sequence, head) into a cache or a paged pool (prefill, append)
  decode     a range of cached tokens back to bf16 or fp32
  roundtrip  encode, then decode of what was encoded
  attention  one query token per sequence over the cached tokens of each layer
  step       one decode step of a served batch over a paged pool: append a token per sequence,
             then attention of every layer over the sequences' own lengths

Fields: d (head dimension), layers, batch, heads (KV heads), tokens (encoded or decoded by the
call, or attended to), start (first token position, or the cached tokens before the call),
formats (a key of FORMATS), dtype (of the inputs and outputs), paged (bool), group (query heads
per KV head).  Inputs follow the distributions of the codec's workloads: K with log-normal
channel scales and four outlier channels, V normal.  Caches that a case only reads are drawn as
codes directly: uniform angle codes, and norm codes of Rayleigh-distributed pair norms.
"""
import math

import numpy as np
import torch

import paper_2603_27467_amd as tvq

F32, LIN, LOG = tvq.TVQ_NORM_F32, tvq.TVQ_NORM_LINEAR, tvq.TVQ_NORM_LOG
BLOCK = 256          # tokens per block of a paged pool

# (n_K, n_V) of the first four layers and of the others; (bits, mode) of the K and V norms
_K8V4 = ((8, LIN), (4, LOG))
FORMATS = {
    "n64": ((64, 64), (64, 64), _K8V4),                # one codebook for every layer
    "boost": ((256, 256), (64, 64), _K8V4),            # early-boost of K and V
    "kboost": ((256, 64), (64, 64), _K8V4),            # early-boost of K only
    "preset": ((256, 128), (128, 64), _K8V4),          # Table 3 presets, K128/V64 baseline
    "preset8": ((256, 128), (128, 64), ((8, LIN), (8, LIN))),   # the same, 8-bit linear norms
    "f32norms": ((64, 64), (64, 64), ((32, F32), (32, F32))),   # angle-only quantization
}


def listed():
    return [
        # the per-step append of a long-context server: one token of 16 sequences, 32 layers
        dict(name="append", op="encode", d=128, layers=32, batch=16, heads=8, tokens=1, start=31,
             formats="boost", dtype="bf16", paged=False, group=1),
        # prefill of a Mistral-7B-shaped cache, the benchmark's shape
        dict(name="prefill", op="encode", d=128, layers=32, batch=1, heads=8, tokens=4096, start=0,
             formats="n64", dtype="bf16", paged=False, group=1),
        # prefill of a prompt of odd length with the published Mistral-7B configuration
        dict(name="prefill-preset", op="encode", d=128, layers=32, batch=1, heads=8, tokens=1999,
             start=0, formats="preset", dtype="bf16", paged=False, group=1),
        # batched prefill of a 1B-class model into a paged pool, sequences at different positions
        dict(name="prefill-paged", op="encode", d=64, layers=16, batch=8, heads=8, tokens=777,
             start=300, formats="kboost", dtype="bf16", paged=True, group=1),
        # the smallest use: one layer in fp32 with fp32 norms, encoded and decoded (an evaluation
        # that measures the angle quantization alone)
        dict(name="roundtrip-f32", op="roundtrip", d=64, layers=1, batch=1, heads=4, tokens=256,
             start=0, formats="f32norms", dtype="f32", paged=False, group=1),
        # the whole Mistral-7B-shaped cache back to bf16, the benchmark's shape
        dict(name="decode", op="decode", d=128, layers=32, batch=1, heads=8, tokens=4096, start=0,
             formats="n64", dtype="bf16", paged=False, group=1),
        # a TinyLlama-shaped batch (22 layers, 4 KV heads) of odd length in its published
        # configuration, back to bf16 for an ordinary attention
        dict(name="decode-preset", op="decode", d=64, layers=22, batch=4, heads=4, tokens=4097,
             start=0, formats="preset", dtype="bf16", paged=False, group=1),
        # a window of a paged pool, from a position inside a block, to fp32
        dict(name="decode-window", op="decode", d=128, layers=8, batch=4, heads=8, tokens=700,
             start=333, formats="boost", dtype="f32", paged=True, group=1),
        # attention of one layer of the long-context server, 32 query heads
        dict(name="attention-long", op="attention", d=128, layers=1, batch=16, heads=8,
             tokens=32770, start=0, formats="n64", dtype="bf16", paged=False, group=4),
        # attention of a 1B-class batch, 32 query heads, four boosted layers and two others
        dict(name="attention-d64", op="attention", d=64, layers=6, batch=8, heads=8, tokens=8195,
             start=0, formats="kboost", dtype="bf16", paged=False, group=4),
        # one sequence of a short conversation, eight layers
        dict(name="attention-short", op="attention", d=128, layers=8, batch=1, heads=8,
             tokens=1000, start=0, formats="n64", dtype="bf16", paged=False, group=4),
        # a decode step of eight sequences of 1 to 4 thousand tokens over a paged pool
        dict(name="step-paged", op="step", d=128, layers=16, batch=8, heads=8, tokens=4100,
             start=0, formats="boost", dtype="bf16", paged=True, group=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: KV tensors up to 256 MB, attended caches up to 400 MB."""
    op = rng.choice(("encode", "encode", "decode", "decode", "roundtrip", "attention", "attention",
                     "step"))
    attends = op in ("attention", "step")
    c = dict(op=op, d=rng.choice((64, 128)), layers=_log_int(rng, 1, 32),
             batch=_log_int(rng, 1, 16), heads=rng.choice((2, 4, 8)),
             tokens=_log_int(rng, 64, 32770) if attends else _log_int(rng, 1, 8192),
             start=0 if attends else rng.choice((0, 0, rng.randrange(1, 500))),
             formats=rng.choice(("n64", "boost", "kboost") if attends else sorted(FORMATS)),
             dtype=rng.choice(("bf16", "bf16", "bf16", "f32")),
             paged=op == "step" or rng.random() < 0.35,
             group=rng.choice((1, 2, 4, 4, 6, 8)) if attends else 1)
    if op == "roundtrip":
        c["layers"], c["tokens"] = min(c["layers"], 4), min(c["tokens"], 1024)
        c["paged"] = False
    if attends:
        c["layers"] = min(c["layers"], 16)

    def size():
        rows = c["layers"] * c["batch"] * c["heads"]
        if attends:
            return rows * c["tokens"] * 240 * c["d"] / 128 / 400e6
        return 2 * rows * (c["tokens"] + c["start"]) * c["d"] * _elem(c) / 256e6
    while size() > 1:
        k = "layers" if c["layers"] > 1 and rng.random() < 0.5 else "tokens"
        k = "batch" if c["batch"] > 1 and rng.random() < 0.3 else k
        c[k] = max(1, c[k] * 2 // 3)
    return c


# ------------------------------------------------------------------------------ shapes
def _elem(c):
    return 2 if c["dtype"] == "bf16" else 4


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _table(c):
    """(n, bits, mode) of K and of V, layer by layer."""
    early, base, norms = FORMATS[c["formats"]]
    return [tuple((n,) + norms[kind] for kind, n in enumerate(early if l < 4 else base))
            for l in range(c["layers"])]


def _records(d, fmt):
    """Bytes per vector of the angle, norm and header planes."""
    n, bits, mode = fmt
    w = (n - 1).bit_length()
    return (d // 2 * w // 8, 2 * d if mode == F32 else d // 2 * bits // 8, 0 if mode == F32 else 8)


def _lens(c):
    """Context lengths of the sequences: from the full length down to a quarter of it."""
    b = c["batch"]
    if not c["paged"]:
        return [c["tokens"]] * b
    return [max(1, c["tokens"] - 3 * c["tokens"] // 4 * i // max(b - 1, 1)) for i in range(b)]


def _positions(c):
    """First positions that a paged encode writes."""
    return [c["start"] * i // c["batch"] for i in range(c["batch"])]


def _capacity(c):
    """Slots per sequence: of the contiguous cache, or of the blocks that a sequence holds."""
    n = c["start"] + c["tokens"] + (1 if c["op"] == "step" else 0)
    return -(-n // BLOCK) * BLOCK if c["paged"] else n


def work(case):
    c = case
    d, rows = c["d"], c["batch"] * c["heads"]
    rec = sum(sum(sum(_records(d, f)) for f in kv) for kv in _table(c))   # K + V, all layers
    kv = 2 * c["layers"] * d * _elem(c)                                   # per (row, token)
    hadamard = 2 * c["layers"] * d * int(math.log2(d))
    if c["op"] in ("attention", "step"):
        tokens = sum(_lens(c)) * c["heads"]
        qo = 2 * c["layers"] * rows * c["group"] * d * _elem(c)
        step = c["op"] == "step"
        return {"bytes": tokens * rec + qo + (rows * (kv + rec) if step else 0),
                "flops": 4 * tokens * c["layers"] * c["group"] * d + (rows * hadamard if step else 0)}
    once = rows * c["tokens"]
    twice = 2 if c["op"] == "roundtrip" else 1
    return {"bytes": twice * once * (kv + rec), "flops": twice * once * hadamard}


def tolerance(case):
    """Codes: about 1e-7 of a turn separates two correct evaluations of an angle in fp32, which
    moves 4e-5 of the codes of n = 256 over a bin boundary (measured: the library's angle bins
    against its polynomial), plus a tie or two in the smallest outputs.  Headers and fp32 norms:
    another order of the transform's sums (measured: 5e-8, 5e-7 at most).  Decoded values follow
    from the codes; in bf16 one in 3e4 falls on the other side of a rounding boundary (2e-5, one
    unit of the last place).  Attention: 5e-7 to 8e-7 in fp32; in bf16 a single large value rounded the
    other way is 6e-4 of one layer's output.  A round trip and a step also carry a code that fell
    on the other side of a boundary to the outputs: one pair of one vector turned by 2 pi / n."""
    c = case
    smallest = min((c["d"] // 2) * bits // 8 if mode != F32 else c["d"] // 2 * 6 // 8
                   for kv in _table(c) for _, bits, mode in kv)
    vectors = c["batch"] * c["heads"] * (1 if c["op"] == "step" else c["tokens"])
    codes = min(1.6e-4 + 2.0 / (smallest * vectors), 0.01)
    if c["op"] == "encode":
        return {"rel": 2e-7, "max": 2e-6, "differ": codes}
    if c["op"] == "roundtrip":
        return {"rel": 2e-3, "max": 0.1, "differ": codes}
    if c["op"] == "step":
        return {"rel": 2.5e-3, "max": 1e-2, "differ": 1.6e-4}
    if c["op"] == "attention":
        return {"rel": 2.5e-3, "max": 1e-2} if c["dtype"] == "bf16" else {"rel": 4e-6}
    return {"rel": 1e-4, "max": 1e-2} if c["dtype"] == "bf16" else {"rel": 4e-7}


# ------------------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed * 7919 + 17)


def _signs(c, seed):
    rng = np.random.default_rng([seed, 99])
    return np.where(rng.integers(0, 2, (c["layers"], c["d"])) == 1, 1, -1).astype(np.int8)


def _codec(c, seed):
    layers = [tvq.LayerCfg(k[0], v[0], k[1], v[1], k[2], v[2]) for k, v in _table(c)]
    return tvq.Codec(c["layers"], c["heads"], c["d"], layers, signs=_signs(c, seed))


def _kv(c, seed, tokens):
    """K and V of `tokens` tokens, [L, B, H, T, d]."""
    g, out = _gen(seed), []
    for kind in range(2):
        x = torch.empty((c["layers"], c["batch"], c["heads"], tokens, c["d"]), dtype=_dtype(c),
                        device="cuda")
        for l in range(c["layers"]):
            y = torch.randn(x.shape[1:], generator=g, device="cuda")
            if kind == 0:
                scale = torch.randn((c["heads"], c["d"]), generator=g, device="cuda").exp()
                at = torch.rand((c["heads"], c["d"]), generator=g, device="cuda").argsort(1)
                y *= torch.where(at < 4, 30.0 * scale, scale)[None, :, None, :]
            x[l] = y
        out.append(x)
    return out


def _block_table(c, seed):
    """Pool blocks of the sequences in a shuffled order, [B, blocks] int32."""
    per = _capacity(c) // BLOCK
    order = torch.from_numpy(np.random.default_rng([seed, 5]).permutation(c["batch"] * per))
    return order.to(torch.int32).reshape(c["batch"], per).cuda()


def _slots(c):
    return c["batch"] * c["heads"] * _capacity(c)


def _cache_bytes(c):
    return _slots(c) * sum(sum(sum(_records(c["d"], f)) for f in kv) for kv in _table(c))


def _fill_codes(c, seed, cache):
    """Codes of a whole cache, as an earlier encode left them."""
    g, off, slots, pairs = _gen(seed + 1), 0, _slots(c), c["d"] // 2
    for kv in _table(c):
        for kind, fmt in enumerate(kv):
            n, bits, mode = fmt
            ra, rn, rh = _records(c["d"], fmt)
            planes = [cache[off:off + slots * ra].view(slots, ra)]
            planes.append(cache[off + slots * ra:off + slots * (ra + rn)].view(slots, rn))
            planes.append(cache[off + slots * (ra + rn):off + slots * (ra + rn + rh)])
            off += slots * (ra + rn + rh)
            planes[0].random_(0, 256, generator=g)      # n a power of two: any bits are codes
            for s in range(0, slots, 1 << 20):
                e = min(s + (1 << 20), slots)
                r = torch.rand((e - s, pairs), generator=g, device="cuda").clamp_(min=1e-7)
                r = r.log_().mul_(-2).sqrt_().mul_(2.0 if kind == 0 else 1.0)
                if mode == F32:
                    planes[1][s:e] = r.view(torch.uint8)
                    continue
                lo, hi = r.min(1, keepdim=True)[0], r.max(1, keepdim=True)[0]
                t = (r - lo) / (hi - lo) if mode == LIN else (r / lo).log() / (hi / lo).log()
                q = (t * (2 ** bits - 1) + 0.5).clamp_(0, 2 ** bits - 1).to(torch.uint8)
                planes[1][s:e] = q if bits == 8 else q[:, 0::2] | (q[:, 1::2] << 4)
                planes[2].view(slots, 8)[s:e] = torch.cat((lo, hi), 1).view(torch.uint8)


def _plane_views(c, cache):
    """The cache as its planes, one view per kind and plane over each run of equal layers: codes
    as bytes, headers and fp32 norms as floats."""
    table, slots, off, out, first = _table(c), _slots(c), 0, [], 0
    words = cache[:cache.numel() // 4 * 4].view(torch.float32)
    while first < len(table):
        run = 1
        while first + run < len(table) and table[first + run] == table[first]:
            run += 1
        layer = slots * sum(sum(_records(c["d"], f)) for f in table[first])
        at = off
        for fmt in table[first]:
            for plane, rec in enumerate(_records(c["d"], fmt)):
                if rec == 0:
                    continue
                if plane == 2 or (plane == 1 and fmt[2] == F32):
                    out.append(words.as_strided((run, slots, rec // 4), (layer // 4, rec // 4, 1),
                                                at // 4))
                else:
                    out.append(cache.as_strided((run, slots, rec), (layer, rec, 1), at))
                at += slots * rec
        off += run * layer
        first += run
    return out


def prepare(case, seed):
    c = case
    s = {"case": c, "codec": _codec(c, seed), "start": c["start"], "tokens": c["tokens"]}
    if c["paged"]:
        s["lay"] = s["codec"].pool_layout(c["batch"] * _capacity(c) // BLOCK, BLOCK)
        s["table"] = _block_table(c, seed)
    else:
        s["lay"] = s["codec"].layout(c["batch"], _capacity(c))
    s["cache"] = torch.zeros(s["lay"].total_bytes, dtype=torch.uint8, device="cuda")
    if c["op"] in ("encode", "roundtrip"):
        s["k"], s["v"] = _kv(c, seed, c["tokens"])
        s["planes"] = _plane_views(c, s["cache"])
        s["positions"] = torch.tensor(_positions(c), dtype=torch.int32, device="cuda")
    else:
        _fill_codes(c, seed, s["cache"])
    if c["op"] in ("decode", "roundtrip"):
        shape = (c["layers"], c["batch"], c["heads"], c["tokens"], c["d"])
        s["ko"] = torch.empty(shape, dtype=_dtype(c), device="cuda")
        s["vo"] = torch.empty(shape, dtype=_dtype(c), device="cuda")
    if c["op"] in ("attention", "step"):
        hq = c["heads"] * c["group"]
        s["q"] = [torch.randn((c["batch"], hq, c["d"]), generator=_gen(seed + 2 + l),
                              device="cuda").to(_dtype(c)) for l in range(c["layers"])]
        s["o"] = [torch.empty_like(q) for q in s["q"]]
        s["scale"] = c["d"] ** -0.5
        s["max_ctx"] = c["tokens"] + (1 if c["op"] == "step" else 0)
        if c["paged"]:
            need = s["codec"].attention_paged_workspace_bytes(c["batch"], hq, s["max_ctx"], BLOCK)
            extra = 1 if c["op"] == "step" else 0
            s["lens"] = torch.tensor([n + extra for n in _lens(c)], dtype=torch.int32,
                                     device="cuda")
        else:
            need = s["codec"].attention_workspace_bytes(c["batch"], hq, s["max_ctx"])
        s["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    if c["op"] == "step":
        s["k"], s["v"] = _kv(c, seed, 1)
        s["positions"] = torch.tensor(_lens(c), dtype=torch.int32, device="cuda")
    return s


# ------------------------------------------------------------------------------ the calls
def _encode(s):
    if s["case"]["paged"]:
        s["codec"].encode_paged(s["k"], s["v"], s["positions"], s["table"], s["cache"], s["lay"])
    else:
        s["codec"].encode(s["k"], s["v"], s["cache"], s["lay"], s["start"])


def _decode(s):
    lo, hi = s["start"], s["start"] + s["tokens"]
    if s["case"]["paged"]:
        s["codec"].decode_paged(s["cache"], s["lay"], s["table"], lo, hi, s["ko"], s["vo"])
    else:
        s["codec"].decode(s["cache"], s["lay"], lo, hi, s["ko"], s["vo"])


def _attend(s):
    codec, lay = s["codec"], s["lay"]
    for l, (q, o) in enumerate(zip(s["q"], s["o"])):
        if s["case"]["paged"]:
            codec.attention_paged(s["cache"], lay, s["table"], s["lens"], s["max_ctx"], l, q, o,
                                  s["scale"], s["workspace"])
        else:
            codec.attention(s["cache"], lay, l, s["max_ctx"], q, o, s["scale"], s["workspace"])


def run(state):
    op = state["case"]["op"]
    if op == "encode":
        _encode(state)
        return {"planes": state["planes"]}
    if op == "decode":
        _decode(state)
        return {"k": state["ko"], "v": state["vo"]}
    if op == "roundtrip":
        _encode(state)
        _decode(state)
        return {"planes": state["planes"], "k": state["ko"], "v": state["vo"]}
    if op == "step":
        _encode(state)
    _attend(state)
    return {"o": state["o"], "cache": state["cache"]} if op == "step" else {"o": state["o"]}


# ------------------------------------------------------------------------------ in 64 bits
def _fwht(x):
    """Unnormalized Sylvester-ordered Walsh-Hadamard transform of the last dimension."""
    n, h = x.shape[-1], 1
    while h < n:
        y = x.reshape(x.shape[:-1] + (n // (2 * h), 2, h))
        x = torch.stack((y[..., 0, :] + y[..., 1, :], y[..., 0, :] - y[..., 1, :]), -2)
        x = x.reshape(x.shape[:-3] + (n,))
        h *= 2
    return x


def _slot_map(c, seed, starts, tokens):
    """Slot of token starts[b] + t of (b, h), [B, H, T] (int64, on the GPU)."""
    cap, H = _capacity(c), c["heads"]
    pos = torch.tensor(starts, device="cuda")[:, None] + torch.arange(tokens, device="cuda")
    b = torch.arange(c["batch"], device="cuda")[:, None, None]
    h = torch.arange(H, device="cuda")[None, :, None]
    if not c["paged"]:
        return (b * H + h) * cap + pos[:, None, :]
    blk = torch.gather(_block_table(c, seed).long(), 1, pos // BLOCK)
    return (blk[:, None, :] * H + h) * BLOCK + pos[:, None, :] % BLOCK


def _unpack(rows, w, count):
    """`count` codes of w bits from each row of bytes (least significant bit first)."""
    if w == 8:
        return rows.long()
    x = rows.reshape(rows.shape[0], count // 8, w).long()
    word = sum(x[..., i] << (8 * i) for i in range(w))
    return torch.stack([(word >> (w * i)) & ((1 << w) - 1) for i in range(8)], -1).reshape(-1, count)


class _Segment:
    """The planes of one (layer, kind) of a cache, and y' = y^ / sqrt(d) of some of its slots."""

    def __init__(self, c, cache, layer, kind):
        self.c, self.fmt, slots, off = c, _table(c)[layer][kind], _slots(c), 0
        for l, kv in enumerate(_table(c)):
            for k, fmt in enumerate(kv):
                if (l, k) == (layer, kind):
                    self.off = off
                off += slots * sum(_records(c["d"], fmt))
        self.cache, self.slots = cache, slots

    def rotated(self, slots):
        """y^ of the slots (a flat index tensor), [len, d]."""
        n, bits, mode = self.fmt
        pairs, at, got = self.c["d"] // 2, self.off, []
        for rec in _records(self.c["d"], self.fmt):
            got.append(self.cache[at:at + self.slots * rec].view(self.slots, rec)[slots]
                       if rec else None)
            at += self.slots * rec
        th = _unpack(got[0], (n - 1).bit_length(), pairs).double() * (2 * math.pi / n)
        if mode == F32:
            r = got[1].contiguous().view(torch.float32).double()
        else:
            q = _unpack(got[1], bits, pairs).double() / (2 ** bits - 1)
            lo, hi = got[2].contiguous().view(torch.float32).double().split(1, 1)
            r = lo + q * (hi - lo) if mode == LIN else torch.exp(lo.log() + q * (hi / lo).log())
        return torch.stack((r * th.cos(), r * th.sin()), -1).reshape(-1, 2 * pairs)


def _exact_planes(c, seed, k, v):
    """Headers (and fp32 norms) of the encoded vectors as _plane_views lays them out."""
    views = _plane_views(c, torch.zeros(_cache_bytes(c), dtype=torch.uint8, device="cuda"))
    starts = _positions(c) if c["paged"] else [c["start"]] * c["batch"]
    slots = _slot_map(c, seed, starts, c["tokens"])
    signs = torch.from_numpy(_signs(c, seed)).cuda().double()
    out, at, first, table = [None] * len(views), 0, 0, _table(c)
    while first < len(table):
        run = 1
        while first + run < len(table) and table[first + run] == table[first]:
            run += 1
        for kind, fmt in enumerate(table[first]):
            planes = [p for p, rec in enumerate(_records(c["d"], fmt)) if rec]
            where = at + planes.index(1 if fmt[2] == F32 else 2)
            val = torch.zeros(views[where].shape, dtype=torch.float64, device="cuda")
            for l in range(run):
                x = (k, v)[kind][first + l].double() * signs[first + l]
                z = _fwht(x) / math.sqrt(c["d"])
                r = (z[..., 0::2] ** 2 + z[..., 1::2] ** 2).sqrt()
                if fmt[2] != F32:
                    r = torch.stack((r.min(-1)[0], r.max(-1)[0]), -1)
                val[l][slots.reshape(-1)] = r.reshape(-1, r.shape[-1])
            out[where] = val
            at += len(planes)
        first += run
    return out


def exact(case, seed):
    c = case
    if c["op"] == "encode":
        return {"planes": _exact_planes(c, seed, *_kv(c, seed, c["tokens"]))}
    if c["op"] == "roundtrip":
        planes = _exact_planes(c, seed, *_kv(c, seed, c["tokens"]))
        return {"planes": planes, "k": None, "v": None}     # the codes decide k and v
    cache = torch.zeros(_cache_bytes(c), dtype=torch.uint8, device="cuda")
    _fill_codes(c, seed, cache)
    signs = torch.from_numpy(_signs(c, seed)).cuda().double()
    if c["op"] == "decode":
        slots = _slot_map(c, seed, [c["start"]] * c["batch"], c["tokens"])
        out = []
        for kind in range(2):
            x = torch.empty((c["layers"],) + slots.shape + (c["d"],), dtype=torch.float64,
                            device="cuda")
            for l in range(c["layers"]):
                y = _Segment(c, cache, l, kind).rotated(slots.reshape(-1))
                x[l] = (_fwht(y) / math.sqrt(c["d"]) * signs[l]).reshape(x.shape[1:])
            out.append(x)
        return {"k": out[0], "v": out[1]}
    if c["op"] == "step":
        return None             # the appended token's codes are the library's own
    lens, hq, out = _lens(c), c["heads"] * c["group"], []
    slots = _slot_map(c, seed, [0] * c["batch"], c["tokens"])
    for l in range(c["layers"]):
        q = torch.randn((c["batch"], hq, c["d"]), generator=_gen(seed + 2 + l), device="cuda")
        q = q.to(_dtype(c)).double() * signs[l]
        qr = _fwht(q) / math.sqrt(c["d"])
        kseg, vseg = _Segment(c, cache, l, 0), _Segment(c, cache, l, 1)
        o = torch.empty_like(q)
        for b in range(c["batch"]):
            for h in range(c["heads"]):
                at = slots[b, h, :lens[b]]
                own = slice(h * c["group"], (h + 1) * c["group"])
                sc = qr[b, own] @ kseg.rotated(at).T * c["d"] ** -0.5
                o[b, own] = torch.softmax(sc, -1) @ vseg.rotated(at)
        out.append(_fwht(o) / math.sqrt(c["d"]) * signs[l])
    return {"o": out}
