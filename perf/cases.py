"""The work that a serving program has this library do, as cases that can be timed: decode steps over a ragged
KV cache (one s3_decode_step per layer, or s3_kv_append + s3_decode_attention), and the row traffic between the
steps (prompt rows of newcomers, doublings, evictions to and re-admissions from device staging memory).

A case is a dict of plain values:
  op        "step": s3_decode_step per layer; "attend": s3_kv_append and s3_decode_attention per layer;
            "move": admit `batch` newcomers (rows of every layer), double one, gather and scatter one, free them all
  heads, kv_heads, dim    query heads, cached heads, head dimension
  cache, act, out         types of the cached rows, of queries and new rows, of the outputs
  layers, batch, max_len  layers one pass runs over, sequences, longest reservation
  shortest, longest, lengths, length_seed   context lengths before the step: "uniform" or "lognormal" between the two

Lengths belong to the case; the values of every tensor come from the seed: N(0,1) queries, keys and values rounded
once to their type, as the library's own workloads draw them.
"""
import math
import random

import numpy as np
import torch

from paper_2306_06000_amd import binding as s3

DEV = "cuda:0"
_CODE = {"f16": s3.S3_F16, "bf16": s3.S3_BF16, "f32": s3.S3_F32, "e4m3": s3.S3_E4M3}
_TORCH = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32, "e4m3": torch.uint8}
_BYTES = {"f16": 2, "bf16": 2, "f32": 4, "e4m3": 1}
GRANULE = 64


def _case(name, op, shape, types, layers, batch, lens, max_len=2048, length_seed=1):
    heads, kv_heads, dim = shape
    cache, act, out = types
    shortest, longest, lengths = lens
    case = dict(op=op, heads=heads, kv_heads=kv_heads, dim=dim, cache=cache, act=act, out=out, layers=layers, batch=batch,
                shortest=shortest, longest=longest, lengths=lengths, max_len=max_len, length_seed=length_seed)
    return dict(case, name=name) if name else case


def listed():
    return [
        # four short prompts of a model with sixteen heads of 256 (the smallest batch the tests serve): latency of one call
        _case("few_short_f16", "step", (16, 16, 256), ("f16", "f16", "f32"), 1, 4, (17, 128, "uniform")),
        # one user with a long conversation, a whole token through the 28 layers of that model
        _case("one_user_28_layers_f16", "step", (16, 16, 256), ("f16", "f16", "f32"), 28, 1, (1400, 1500, "uniform")),
        # an ordinary serving batch: 64 requests at any point of prompt and answer
        _case("serving_b64_f16", "step", (16, 16, 256), ("f16", "f16", "f32"), 4, 64, (32, 1000, "uniform")),
        # a large batch with a long tail of lengths
        _case("ragged_b512_f16", "step", (16, 16, 256), ("f16", "f16", "f32"), 1, 512, (40, 1600, "lognormal")),
        # one GPU's twelve heads of a 96-head model under tensor parallelism, long contexts
        _case("long_b128_bf16", "step", (12, 12, 128), ("bf16", "bf16", "f32"), 2, 128, (512, 2048, "uniform")),
        # grouped-query attention, ordinary batch
        _case("grouped_b256_bf16", "step", (32, 8, 128), ("bf16", "bf16", "f32"), 2, 256, (32, 1000, "uniform")),
        # grouped-query attention, three users with long documents, outputs in the type of the next layer
        _case("grouped_few_long_bf16", "step", (32, 8, 128), ("bf16", "bf16", "bf16"), 8, 3, (512, 8192, "uniform"),
              max_len=16384, length_seed=4),
        # multi-query attention: sixteen query heads on one cached head
        _case("multi_query_b256_f16", "step", (16, 1, 256), ("f16", "f16", "f32"), 4, 256, (32, 1000, "uniform")),
        # 8-bit cache rows
        _case("rows8_b128_f16", "step", (16, 16, 256), ("e4m3", "f16", "f32"), 2, 128, (32, 1000, "uniform")),
        # 8-bit rows of shared heads: the batch that two footprint savings together admit
        _case("grouped_rows8_b1024_bf16", "step", (32, 8, 128), ("e4m3", "bf16", "f32"), 1, 1024, (32, 1000, "uniform")),
        # append and attention as separate calls, 64 heads of 96 (44-layer model of the paper's worked example)
        _case("append_attend_d96_bf16", "attend", (64, 64, 96), ("bf16", "bf16", "bf16"), 2, 24, (64, 1500, "uniform")),
        # between the steps: newcomers' prompt rows in every layer, one doubling, one eviction and its return
        _case("admit_and_move_bf16", "move", (16, 16, 256), ("bf16", "bf16", "f32"), 28, 4, (64, 512, "uniform")),
    ]


_SHAPES = [(16, 16, 256), (16, 16, 256), (12, 12, 128), (16, 16, 64), (64, 64, 96), (32, 32, 128), (3, 3, 128), (32, 8, 128), (32, 8, 128),
           (16, 1, 256), (8, 1, 64), (12, 4, 128), (24, 8, 64), (64, 8, 128), (40, 5, 128), (16, 8, 128), (6, 3, 256), (12, 2, 128)]
_MOST_BYTES = 1.7e9  # below the largest listed case


def draw(rng):
    op = rng.choice(["step"] * 7 + ["attend", "attend", "move"])
    shape = rng.choice(_SHAPES)
    act = rng.choice(["f16", "bf16"])
    cache = act if shape[2] == 96 or rng.random() < 0.75 else "e4m3"
    out = rng.choice(["f32", "f32", act])
    max_len = 16384 if rng.random() < 0.2 else 2048
    longest = int(round(math.exp(rng.uniform(math.log(24), math.log(max_len - 1)))))
    shortest = max(1, int(longest * rng.uniform(0.02, 0.9)))
    batch = int(round(math.exp(rng.uniform(0.0, math.log(1024 if op != "move" else 16)))))
    layers = int(round(math.exp(rng.uniform(0.0, math.log(28)))))
    c = _case(None, op, shape, (cache, act, out), layers, batch, (shortest, longest, rng.choice(["uniform", "lognormal"])),
              max_len, rng.randrange(1 << 30))
    while work(c)["bytes"] > _MOST_BYTES:  # fewer layers first, then fewer sequences, then shorter ones
        if c["layers"] > 1:
            c["layers"] = (c["layers"] + 1) // 2
        elif c["batch"] > 1:
            c["batch"] = c["batch"] * 3 // 4
        else:
            c["longest"] = c["longest"] * 3 // 4
            c["shortest"] = min(c["shortest"], c["longest"])
    return c


def _lens(case):
    """Rows each sequence holds before the step."""
    r = random.Random(case["length_seed"])
    lo, hi = case["shortest"], case["longest"]
    if case["lengths"] == "uniform":
        return [r.randint(lo, hi) for _ in range(case["batch"])]
    mid, sigma = math.sqrt(lo * hi), math.log(hi / lo) / 4 if hi > lo else 0.0
    return [max(lo, min(hi, int(round(mid * math.exp(r.gauss(0.0, sigma)))))) for _ in range(case["batch"])]


def _values(case, seed):
    """Generator of the case's tensors in a fixed order: per layer (K rows, V rows of all sequences one after the
    other, q, k_new, v_new)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    total, n = sum(_lens(case)), case["batch"]
    act = _TORCH[case["act"]]

    def rows(count):
        x = torch.empty((count, case["kv_heads"], case["dim"]), dtype=act, device=DEV).normal_(generator=g)
        return x.to(torch.float8_e4m3fn).view(torch.uint8) if case["cache"] == "e4m3" else x

    for _ in range(case["layers"]):
        k, v = rows(total), rows(total)
        q = torch.empty((n, case["heads"], case["dim"]), dtype=act, device=DEV).normal_(generator=g)
        k_new = torch.empty((n, case["kv_heads"], case["dim"]), dtype=act, device=DEV).normal_(generator=g)
        v_new = torch.empty((n, case["kv_heads"], case["dim"]), dtype=act, device=DEV).normal_(generator=g)
        yield k, v, q, k_new, v_new


class _State:
    """What a serving program holds between two calls."""

    def __del__(self):
        if getattr(self, "arena", None) is not None:
            torch.cuda.synchronize()
            s3.s3_kv_arena_destroy(self.arena)
            self.arena = None


def prepare(case, seed):
    s = _State()
    s.case = case
    lens, n, layers = _lens(case), case["batch"], case["layers"]
    cfg = s3.make_config(layers, case["heads"], case["dim"], _CODE[case["cache"]], GRANULE, case["max_len"],
                         0 if case["kv_heads"] == case["heads"] else case["kv_heads"], _CODE[case["act"]])
    bpt = s3.s3_kv_bytes_per_token(cfg)
    # reservations: room for the prompt and a few more tokens; "move" keeps free room for the doubled slot
    preds = [min(case["max_len"], length + 1 + (length * 7) % 50) for length in lens]
    if case["op"] == "move":
        preds = lens
    caps = [s3.s3_kv_capacity_for(cfg, p) for p in preds]
    spare = 2 * max(caps) + GRANULE if case["op"] == "move" else 0
    s.memory = torch.zeros((sum(caps) + spare) * bpt, dtype=torch.uint8, device=DEV)
    s.cache = s.memory if case["cache"] == "e4m3" else s.memory.view(torch.int16)  # outputs: the cached bits
    st, s.arena = s3.s3_kv_arena_init(cfg, s.memory, s.memory.numel())
    s3.check(st, "s3_kv_arena_init")
    s.lens, s.preds = np.array(lens, np.int32), preds
    stream = torch.cuda.current_stream().cuda_stream
    starts = np.concatenate([[0], np.cumsum(lens)])
    if case["op"] == "move":
        s.rows = []
        for k, v, _q, _k, _v in _values(case, seed):
            s.rows.append(([k[starts[i]:starts[i + 1]] for i in range(n)], [v[starts[i]:starts[i + 1]] for i in range(n)]))
        s.stage = torch.zeros(s3.s3_kv_evict_bytes(s.arena, max(lens)), dtype=torch.uint8, device=DEV)
        s.most = int(np.argmax(s.lens))
        return s
    admitted, ids, offs, _caps = s3.s3_kv_alloc(s.arena, preds)
    if admitted != n:
        raise RuntimeError("the arena does not hold the batch")
    s.slot_off = torch.tensor(offs.tolist(), dtype=torch.int64, device=DEV)
    s.pos = torch.tensor(lens, dtype=torch.int32, device=DEV)
    s.len = torch.zeros_like(s.pos)
    s.inputs = []
    for layer, (k, v, q, k_new, v_new) in enumerate(_values(case, seed)):
        s3.check(s3.s3_kv_fill_batch(s.arena, layer, ids, s.lens, [k[starts[i]:starts[i + 1]] for i in range(n)],
                                     [v[starts[i]:starts[i + 1]] for i in range(n)], stream), "s3_kv_fill_batch")
        s.inputs.append((q, k_new, v_new))
    s.out = torch.zeros((layers, n, case["heads"], case["dim"]), dtype=_TORCH[case["out"]], device=DEV)
    s.outs = list(s.out)
    s3.check(s3.s3_kv_reserve_scratch(s.arena, n), "s3_kv_reserve_scratch")
    torch.cuda.synchronize()
    return s


def run(s):
    case = s.case
    stream = torch.cuda.current_stream().cuda_stream
    if case["op"] == "move":
        return _run_move(s, stream)
    n, out_dtype = case["batch"], _CODE[case["out"]]
    if case["op"] == "step":
        for layer, (q, k_new, v_new) in enumerate(s.inputs):
            s3.check(s3.s3_decode_step(s.arena, layer, n, s.slot_off, s.pos, q, k_new, v_new, s.outs[layer], out_dtype, 0.0,
                                       s.len, stream), "s3_decode_step")
    else:
        torch.add(s.pos, 1, out=s.len)
        for layer, (q, k_new, v_new) in enumerate(s.inputs):
            s3.check(s3.s3_kv_append(s.arena, layer, n, s.slot_off, s.pos, k_new, v_new, stream), "s3_kv_append")
            s3.check(s3.s3_decode_attention(s.arena, layer, n, q, s.slot_off, s.len, s.outs[layer], out_dtype, 0.0, stream),
                     "s3_decode_attention")
    return {"out": s.out, "len": s.len, "cache": s.cache}


def _run_move(s, stream):
    """One scheduling step's row traffic; the slots are free again at its end, so a pass can follow a pass."""
    n = s.case["batch"]
    admitted, ids, _offs, _caps = s3.s3_kv_alloc(s.arena, s.preds)
    if admitted != n:
        raise RuntimeError("the arena does not hold the newcomers")
    for layer, (k, v) in enumerate(s.rows):
        s3.check(s3.s3_kv_fill_batch(s.arena, layer, ids, s.lens, k, v, stream), "s3_kv_fill_batch")
    most, length = int(ids[s.most]), int(s.lens[s.most])
    cap = s3.s3_kv_slot_info(s.arena, most)[2]
    if cap < s.case["max_len"]:
        s3.check(s3.s3_kv_grow(s.arena, most, length, stream)[0], "s3_kv_grow")
    s3.check(s3.s3_kv_gather_rows(s.arena, most, length, s.stage, stream), "s3_kv_gather_rows")
    s3.check(s3.s3_kv_free(s.arena, most), "s3_kv_free")
    admitted, back, _offs, _caps = s3.s3_kv_alloc(s.arena, [s.preds[s.most]])
    if admitted != 1:
        raise RuntimeError("the arena does not hold the returning sequence")
    s3.check(s3.s3_kv_scatter_rows(s.arena, int(back[0]), length, s.stage, stream), "s3_kv_scatter_rows")
    for i, sid in enumerate(ids.tolist()):
        s3.check(s3.s3_kv_free(s.arena, int(back[0]) if i == s.most else sid), "s3_kv_free")
    return {"stage": s.stage, "cache": s.cache}


def work(case):
    lens, n = _lens(case), case["batch"]
    row = case["kv_heads"] * case["dim"]
    cached, act, out = _BYTES[case["cache"]], _BYTES[case["act"]], _BYTES[case["out"]]
    if case["op"] == "move":
        # rows read and written: all newcomers' (fill), the longest one's for the doubling, the gather and the scatter
        grown = -(-max(lens) // GRANULE) * GRANULE < case["max_len"]
        return {"bytes": 2.0 * case["layers"] * 2 * row * cached * (sum(lens) + max(lens) * (2 + grown)), "flops": 0.0}
    heads = case["heads"] * case["dim"]
    # cached rows once, queries and outputs once, new rows read once and written once
    per_layer = 2 * row * cached * sum(lens) + n * heads * (act + out) + 2 * n * row * (act + cached)
    flops = 4.0 * heads * (sum(lens) + n)
    return {"bytes": float(case["layers"] * per_layer), "flops": case["layers"] * flops}


def tolerance(case):
    # About four times the distance to 64 bits that was measured: 2.3e-7 (weights in fp32) to 2.3e-6 (weights as two
    # bfloat16 parts) with 32-bit outputs, 2.1e-4 with fp16 and 1.7e-3 with bfloat16 outputs (one rounding).
    if case["op"] == "move":
        return "exact"
    return {"rel": {"f32": 1e-5, "f16": 1e-3, "bf16": 8e-3}[case["out"]]}


def exact(case, seed):
    """The attention of every layer in 64 bits over the stored values (the appended row included)."""
    if case["op"] == "move":
        return None
    lens, n = _lens(case), case["batch"]
    heads, kv, dim = case["heads"], case["kv_heads"], case["dim"]

    def wide(x):
        return (x.view(torch.float8_e4m3fn) if x.dtype == torch.uint8 else x).to(torch.float64)

    def stored(x):  # a new row as the cache holds it
        return x.to(torch.float8_e4m3fn) if case["cache"] == "e4m3" else x

    layers = []
    for k, v, q, k_new, v_new in _values(case, seed):
        out = torch.empty((n, heads, dim), dtype=torch.float64, device=DEV)
        at = 0
        for b, length in enumerate(lens):
            kb = torch.cat([wide(k[at:at + length]), wide(stored(k_new[b:b + 1]))]).permute(1, 0, 2).contiguous()
            vb = torch.cat([wide(v[at:at + length]), wide(stored(v_new[b:b + 1]))]).permute(1, 0, 2).contiguous()
            qb = q[b].to(torch.float64).view(kv, heads // kv, dim)
            scores = torch.matmul(qb, kb.transpose(1, 2).contiguous()) / math.sqrt(dim)
            out[b] = torch.matmul(torch.softmax(scores, dim=-1), vb).view(heads, dim)
            at += length
        layers.append(out)
    return {"out": torch.stack(layers), "len": None, "cache": None}
