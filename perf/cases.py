"""Performance cases: what a serving engine has the library do for one layer of its KV cache.

Every case goes through the Python binding's public calls with inputs made on the GPU from a
seed.  A case is a plain dict; `kind` says which of the engine's steps it is:

  step    kv_quant_write of every sequence's newest q_len tokens, then paged_decode_attn over
          everything stored: a decode step (q_len 1), the verification of a few speculated tokens
          (with `prefix`: over a prompt prefix whose blocks the batch shares), or a chunk of a
          prompt over what is already cached (q_len in the hundreds)
  write   kv_quant_write of whole prompts
  move    kvq_blocks_export of some blocks and kvq_blocks_import of others (tiered cache)

The values follow the benchmark's recipe: K, V and q are N(0, 1) in bf16, one K channel in a
hundred is 20 times as large; block tables are a random permutation of a pool with room to spare.
Sequence lengths are spread evenly (or evenly in their logarithm) over [lo, hi]; the seed decides
which sequence has which, so that the work of a case does not depend on it.
"""
import math

import numpy as np
import torch

from paper_2605_29639_amd import kvq
from paper_2605_29639_amd.workloads import STATIC_SCALES

MODES = {"int8": kvq.MODE_INT8, "fp8": kvq.MODE_FP8, "bf16": kvq.MODE_BF16,
         "fp8_tensor": kvq.MODE_FP8_TENSOR, "int4": kvq.MODE_INT4, "int4_group": kvq.MODE_INT4_GROUP}
FILL_TOKENS = 65536   # tokens per call when a pool is filled


def _case(name, kind, mode, batch, lo, hi, q_len=1, hq=32, hkv=8, d=128, bs=16, log=False, prefix=0,
          blocks=0, host=False):
    c = {"name": name, "kind": kind, "mode": mode, "batch": batch, "lo": lo, "hi": hi, "q_len": q_len,
         "hq": hq, "hkv": hkv, "d": d, "bs": bs, "log": log, "prefix": prefix, "blocks": blocks,
         "host": host}
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # one user, a short conversation: latency and launches
        _case("decode_1_int8", "step", "int8", 1, 600, 600),
        # a small model's layer (head_dim 64) under static scales, odd batch, short ragged contexts
        _case("decode_17_d64_fp8_tensor", "step", "fp8_tensor", 17, 33, 1500, hq=16, hkv=4, d=64),
        # the benchmark's headline: an 8B-class layer, 64 sequences
        _case("decode_64_int8", "step", "int8", 64, 512, 4096),
        # the same layer with the smallest cache that keeps outlier channels apart
        _case("decode_64_int4_group", "step", "int4_group", 64, 512, 4096),
        # a large batch appending to per-block scales (blocks may have to be re-encoded)
        _case("decode_128_fp8", "step", "fp8", 128, 1024, 8192),
        # long contexts, 16 query heads per kv head, 64-token blocks
        _case("decode_32_long_int8", "step", "int8", 32, 16384, 65536, hq=64, hkv=4, bs=64, log=True),
        # verification of 4 speculated tokens over a shared 1024-token prompt prefix
        _case("verify_64_prefix_int8", "step", "int8", 64, 2048, 16384, q_len=4, hq=64, prefix=1024),
        # chunked prefill: eight prompts advance by 512 tokens over 4096 cached ones
        _case("chunk_8x512_int8", "step", "int8", 8, 4608, 4608, q_len=512),
        # chunked prefill of one long prompt
        _case("chunk_1x512_fp8", "step", "fp8", 1, 16896, 16896, q_len=512),
        # prompts written at once
        _case("prompt_write_int8", "write", "int8", 13, 512, 4096),
        _case("prompt_write_bf16", "write", "bf16", 13, 512, 4096),
        # eviction of 256 blocks to pinned host memory, and 256 loaded back
        _case("evict_load_host_int8", "move", "int8", 0, 0, 0, blocks=256, host=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another case of the same ranges; none costs more than the largest listed one."""
    kind = rng.choice(("decode", "decode", "verify", "chunk", "write", "move"))
    mode = rng.choice(tuple(MODES))
    d = 128 if mode.startswith("int4") or rng.random() < 0.75 else 64
    hq, hkv = rng.choice(((32, 8), (64, 8), (64, 4), (16, 4), (28, 4), (12, 2), (8, 8)))
    bs = rng.choice((16, 16, 32, 64, 128))
    token_bytes = 2 * hkv * d * {"bf16": 2.0, "int4": 0.53, "int4_group": 0.63}.get(mode, 1.03)
    if kind == "move":
        blocks, host = _log_int(rng, 8, 4096), rng.random() < 0.5
        blocks = max(1, min(blocks, int((16e6 if host else 128e6) / (token_bytes * bs))))
        return _case(None, "move", mode, 0, 0, 0, hq=hq, hkv=hkv, d=d, bs=bs, blocks=blocks, host=host)
    if kind == "write":
        total, batch = _log_int(rng, 48, 32768), _log_int(rng, 1, 32)
        hi = max(2, int(1.6 * total / batch))
        return _case(None, "write", mode, batch, max(1, hi // 4), hi, hq=hq, hkv=hkv, d=d, bs=bs)
    prefix = 0
    if kind == "chunk":
        q_len, batch, cached = _log_int(rng, 17, 1024), rng.randint(1, 8), _log_int(rng, 16, 32768)
        # (4 d operations per query row and position, in the listed chunk's range)
        while batch * q_len * hq * (cached + q_len) * 4.0 * d > 2.5e11:
            cached, q_len = max(16, cached * 3 // 4), max(17, q_len * 3 // 4)
        lo, hi = q_len + cached // 2, q_len + cached
    else:
        q_len = 1 if kind == "decode" else rng.randint(2, 16)
        batch, hi = _log_int(rng, 1, 256), _log_int(rng, 32, 32768)
        if kind == "verify" and batch > 1 and rng.random() < 0.5:
            prefix = 256 * rng.randint(1, 8)
            hi += prefix
        rows = q_len * hq // hkv
        while batch > 1 and batch * hi * token_bytes * max(1, rows // 32) > 9e8:
            batch = max(1, batch * 3 // 4)
        while hi - prefix > 64 and batch * hi * token_bytes * max(1, rows // 32) > 9e8:
            hi = prefix + (hi - prefix) * 3 // 4
        lo = max(prefix + q_len, hi // rng.randint(1, 8), q_len)
        hi = max(hi, lo)
        prefix = prefix if batch > 1 else 0
    return _case(None, "step", mode, batch, lo, hi, q_len=q_len, hq=hq, hkv=hkv, d=d, bs=bs,
                 log=hi > 10 * lo, prefix=prefix)


# ------------------------------------------------------------------------------- inputs

def _lengths(case):
    """The case's sequence lengths, in rising order."""
    n, lo, hi = case["batch"], case["lo"], case["hi"]
    at = (np.arange(n) + 0.5) / max(n, 1)
    x = np.exp(np.log(lo) + at * (np.log(hi) - np.log(lo))) if case["log"] else lo + at * (hi - lo)
    return np.floor(x).astype(np.int64)


def _layout(case, seed):
    """(lengths in the batch's order, block tables, pool size): a shared prefix has the same
    blocks in every table."""
    rng = np.random.default_rng([seed, 1])
    lens, bs, prefix = rng.permutation(_lengths(case)), case["bs"], case["prefix"]
    shared = prefix // bs
    own = (lens + bs - 1) // bs - shared
    pool = shared + int(own.sum())
    pool += pool // 4 + 1
    perm = rng.permutation(pool).astype(np.int32)
    tables = np.full((len(lens), shared + int(own.max())), -1, dtype=np.int32)
    at = shared
    for b, n in enumerate(own):
        tables[b, :shared] = perm[:shared]
        tables[b, shared:shared + n] = perm[at:at + n]
        at += n
    return lens, tables, pool


def _rows(case, seed, b, n, device="cuda"):
    """K and V of positions 0 .. n - 1 of sequence b (bf16 [n, hkv, d]).  Positions inside a shared
    prefix are the same for every sequence."""
    h, d, prefix = case["hkv"], case["d"], case["prefix"]
    gain = torch.ones(h * d, device=device)
    picked = np.random.default_rng([seed, 2]).choice(h * d, size=max(1, h * d // 100), replace=False)
    gain[torch.from_numpy(picked).to(device)] = 20.0

    def part(owner, count):
        g = torch.Generator(device=device)
        g.manual_seed((seed * 1000003 + owner) % (1 << 62))
        x = torch.randn((2, count, h * d), generator=g, device=device)
        x[0] *= gain
        return x.to(torch.bfloat16).view(2, count, h, d)

    if not prefix:
        return tuple(part(b + 1, n))
    both = torch.cat((part(0, prefix), part(b + 1, n - prefix)), dim=1)
    return both[0].contiguous(), both[1].contiguous()


def _slots(case, tables, b, start, stop):
    p = np.arange(start, stop, dtype=np.int64)
    return tables[b, p // case["bs"]].astype(np.int64) * case["bs"] + p % case["bs"]


def _queries(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1000003 + 999983) % (1 << 62))
    shape = (case["batch"] * case["q_len"], case["hq"], case["d"])
    return torch.randn(shape, generator=g, device="cuda").to(torch.bfloat16)


def _pool(case, blocks):
    desc = kvq.make_desc(MODES[case["mode"]], blocks, case["bs"], case["hkv"], case["d"])
    cache, scales = kvq.alloc_cache(desc)
    if case["mode"] == "fp8_tensor":
        scales.copy_(torch.tensor(STATIC_SCALES))
    return desc, cache, scales


class _Writer:
    """Collects rows and writes them in calls of FILL_TOKENS tokens or one sequence."""

    def __init__(self, desc, cache, scales):
        self.to, self.k, self.v, self.s, self.n = (cache, scales, desc), [], [], [], 0

    def add(self, k, v, slots):
        self.k.append(k), self.v.append(v), self.s.append(slots)
        self.n += len(slots)
        if self.n >= FILL_TOKENS:
            self.flush()

    def flush(self):
        if self.n:
            kvq.kv_quant_write(torch.cat(self.k), torch.cat(self.v),
                               torch.from_numpy(np.concatenate(self.s)).cuda(), *self.to)
        self.k, self.v, self.s, self.n = [], [], [], 0


def prepare(case, seed):
    if case["kind"] == "move":
        return _prepare_move(case, seed)
    lens, tables, blocks = _layout(case, seed)
    desc, cache, scales = _pool(case, blocks)
    state = {"kind": case["kind"], "desc": desc, "cache": cache, "scales": scales}
    if case["kind"] == "write":
        rows = [_rows(case, seed, b, int(n)) for b, n in enumerate(lens)]
        slots = [_slots(case, tables, b, 0, int(n)) for b, n in enumerate(lens)]
        return dict(state, k=torch.cat([r[0] for r in rows]), v=torch.cat([r[1] for r in rows]),
                    slots=torch.from_numpy(np.concatenate(slots)).cuda())
    q_len, prefix = case["q_len"], case["prefix"]
    fill, k_new, v_new, s_new = _Writer(desc, cache, scales), [], [], []
    for b, n in enumerate(int(n) for n in lens):
        k, v = _rows(case, seed, b, n)
        first, old = (0 if b == 0 else prefix), n - q_len   # the first sequence writes the shared prefix
        if old > first:
            fill.add(k[first:old], v[first:old], _slots(case, tables, b, first, old))
        k_new.append(k[old:].clone()), v_new.append(v[old:].clone())
        s_new.append(_slots(case, tables, b, old, n))
    fill.flush()
    q = _queries(case, seed)
    longest = int(lens.max())
    return dict(state, k=torch.cat(k_new), v=torch.cat(v_new),
                slots=torch.from_numpy(np.concatenate(s_new)).cuda(), q=q, q_len=q_len, prefix=prefix,
                tables=torch.from_numpy(tables).cuda(),
                lens=torch.from_numpy(lens.astype(np.int32)).cuda(), longest=longest,
                sm_scale=1.0 / math.sqrt(case["d"]), out=torch.empty(q.shape, device="cuda"),
                workspace=kvq.alloc_workspace(desc, case["batch"], q_len, case["hq"], longest,
                                              shared_prefix_tokens=prefix))


def _prepare_move(case, seed):
    n = case["blocks"]
    pool = 4 * n
    desc, cache, scales = _pool(case, pool)
    rng = np.random.default_rng([seed, 3])
    k, v = _rows(case, seed, 0, pool * case["bs"])
    kvq.kv_quant_write(k, v, torch.arange(pool * case["bs"], device="cuda"), cache, scales, desc)
    ids = torch.from_numpy(rng.permutation(pool).astype(np.int32)).cuda()
    nbytes, nscales = kvq.packed_sizes(desc, n)
    where = {"pin_memory": True} if case["host"] else {"device": "cuda"}
    area = [(torch.zeros(nbytes, dtype=torch.uint8, **where), torch.zeros(nscales, **where))
            for _ in range(2)]
    # what is to be loaded: other blocks of the same pool, evicted earlier
    kvq.blocks_export(cache, scales, desc, ids[n:2 * n].contiguous(), *area[1])
    return {"kind": "move", "desc": desc, "cache": cache, "scales": scales, "evict": ids[:n].contiguous(),
            "load": ids[2 * n:3 * n].contiguous(), "evicted": area[0], "loaded": area[1]}


# ------------------------------------------------------------------------------- the passes

def run(s):
    desc, cache, scales = s["desc"], s["cache"], s["scales"]
    if s["kind"] == "move":
        kvq.blocks_export(cache, scales, desc, s["evict"], *s["evicted"])
        kvq.blocks_import(*s["loaded"], desc, s["load"], cache, scales)
        return {"packed": s["evicted"][0], "packed_scales": s["evicted"][1], "cache": cache,
                "scales": scales}
    kvq.kv_quant_write(s["k"], s["v"], s["slots"], cache, scales, desc)
    if s["kind"] == "write":
        return {"cache": cache, "scales": scales}
    kvq.paged_decode_attn(s["q"], cache, scales, desc, s["tables"], s["lens"], s["q_len"], s["longest"],
                          s["sm_scale"], s["out"], s["workspace"], shared_prefix_tokens=s["prefix"])
    return {"out": s["out"], "cache": cache, "scales": scales}


def _stored_bytes(case):
    """Bytes one token takes in the cache: codes and scales of K and V, all heads."""
    mode, h, d = case["mode"], case["hkv"], case["d"]
    row = {"int8": d + 4.0, "int4": d / 2 + 4.0, "int4_group": d / 2 + 4.0 * d / 32, "bf16": 2.0 * d,
           "fp8": d + 4.0 / case["bs"], "fp8_tensor": float(d)}[mode]
    return 2 * h * row


def work(case):
    token, row = _stored_bytes(case), case["hkv"] * case["d"] * 2.0 * 2   # bf16 K and V in
    if case["kind"] == "move":
        return {"bytes": 2 * 2 * case["blocks"] * (case["bs"] * token + 4.0), "flops": 0.0}
    lens, q_len = _lengths(case), case["q_len"]
    if case["kind"] == "write":
        return {"bytes": float(lens.sum()) * (row + token + 8), "flops": 0.0}
    new = case["batch"] * q_len
    positions = float(lens.sum()) - (case["batch"] - 1) * case["prefix"]
    tables = 4.0 * float(((lens + case["bs"] - 1) // case["bs"]).sum()) + 4.0 * case["batch"]
    q_out = new * case["hq"] * case["d"] * (2.0 + 4.0)
    seen = float(sum(q_len * n - q_len * (q_len - 1) / 2 for n in lens))   # (query token, position) pairs
    return {"bytes": new * (row + token + 8) + positions * token + tables + q_out,
            "flops": seen * case["hq"] * case["d"] * 4.0}


def tolerance(case):
    # codes and scales are defined to the bit, whatever the order of the work
    if case["kind"] != "step":
        return "exact"
    # exact codes, sums in fp32, probabilities in f16 (11 bits; an unquantized cache: 16 bits).
    # Measured against 64 bits: 3e-5 .. 9e-5, with scales per group of channels 1.6e-4, bf16 4e-6.
    rel = {"bf16": 5e-5, "int4_group": 8e-4}.get(case["mode"], 4e-4)
    return {"rel": rel, "differ": 0.0}


# ------------------------------------------------------------------------------- 64 bits

def _e4m3(y):
    """Nearest E4M3 value of y (ties to even, saturating at 448), in float64."""
    a = y.abs().clamp(max=448.0)
    step = torch.exp2((torch.frexp(a).exponent.double() - 1).clamp(min=-6.0) - 3)
    return (torch.round(a / step) * step).clamp(max=448.0) * torch.sign(y)


def _over(x, s):
    """x / s where s > 0, else 0."""
    return torch.where(s > 0, x / torch.where(s > 0, s, torch.ones_like(s)), torch.zeros_like(x))


def _quantized(case, x, old, kv):
    """What the cache holds of the rows x [n, h, d] (float64) after the first `old` were written by
    one call and the rest by another: (values, scales per token or per block, or None)."""
    mode, bs = case["mode"], case["bs"]
    n, h, d = x.shape
    if mode == "bf16":
        return x, None
    if mode in ("int8", "int4", "int4_group"):
        top = 127.0 if mode == "int8" else 7.0
        groups = x.reshape(n, h, d // 32, 32) if mode == "int4_group" else x
        exact = groups.abs().amax(-1, keepdim=True) / top
        s = exact.float().double()
        codes = torch.round(_over(groups, s)).clamp(-top, top)
        return (codes * s).reshape(n, h, d), exact.squeeze(-1)
    if mode == "fp8_tensor":
        s = torch.tensor(STATIC_SCALES[kv], dtype=torch.float32).double().item()
        return _e4m3(x / s) * s, None
    nb = (n + bs - 1) // bs
    blocks = torch.zeros((nb * bs, h, d), dtype=torch.float64, device=x.device)
    blocks[:n] = x
    blocks = blocks.view(nb, bs, h, d)
    is_old = (torch.arange(nb * bs, device=x.device) < old).view(nb, bs, 1, 1)
    before = (blocks * is_old).abs().amax((1, 3), keepdim=True) / 448.0
    after = (blocks * ~is_old).abs().amax((1, 3), keepdim=True) / 448.0
    s_prev, s_run = before.float().double(), after.float().double()
    s = torch.maximum(s_prev, s_run)
    codes = _e4m3(_over(blocks, s_prev))
    codes = torch.where(s > s_prev, _e4m3(_over(codes * s_prev, s)), codes)
    codes = torch.where(is_old, codes, _e4m3(_over(blocks, s)))
    return (codes * s).reshape(nb * bs, h, d)[:n], torch.maximum(before, after).view(nb, h)


def exact(case, seed):
    if case["kind"] == "move" or (case["kind"] == "write" and case["mode"] in ("bf16", "fp8_tensor")):
        return None   # bytes only
    lens, tables, blocks = _layout(case, seed)
    h, d, bs, q_len, hq = case["hkv"], case["d"], case["bs"], case["q_len"], case["hq"]
    step = case["kind"] == "step"
    shape = {"int8": (blocks, 2, h, bs), "int4": (blocks, 2, h, bs), "fp8": (blocks, 2, h),
             "int4_group": (blocks, 2, h, bs, d // 32)}.get(case["mode"])
    scales = torch.zeros(shape, dtype=torch.float64, device="cuda") if shape else None
    out = torch.empty((case["batch"], q_len, hq, d), dtype=torch.float64, device="cuda")
    q = _queries(case, seed).double().view(case["batch"], q_len, h, hq // h, d) if step else None
    for b, n in enumerate(int(n) for n in lens):
        held = []
        slots = torch.from_numpy(_slots(case, tables, b, 0, n)).cuda()
        for kv, rows in enumerate(_rows(case, seed, b, n)):
            x, s = _quantized(case, rows.double(), n - q_len if step else 0, kv)
            held.append(x)
            if s is not None and case["mode"] == "fp8":
                scales[slots[::bs] // bs, kv] = s
            elif s is not None:
                scales[slots // bs, kv, :, slots % bs] = s
        if not step:
            continue
        seen = torch.arange(n, device="cuda") <= n - q_len + torch.arange(q_len, device="cuda")[:, None]
        for i in range(h):
            k, v = held[0][:, i].t().contiguous(), held[1][:, i].contiguous()
            logits = torch.mm(q[b, :, i].reshape(-1, d), k) / math.sqrt(d)
            logits = logits.view(q_len, hq // h, n).masked_fill(~seen[:, None], -math.inf)
            p = torch.softmax(logits, dim=-1).view(-1, n)
            out[b, :, i * (hq // h):(i + 1) * (hq // h)] = torch.mm(p, v).view(q_len, hq // h, d)
    if case["mode"] == "fp8_tensor":
        scales = torch.tensor(STATIC_SCALES, dtype=torch.float64)
    found = {"cache": None, "scales": scales}
    return dict(found, out=out.view(-1, hq, d)) if step else found
