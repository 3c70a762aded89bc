"""The work that a program built on this library has it do, as cases that can be timed and checked.

A case names one path of a weight update through the public binding:

  encode   the sender compares its previous and its new weights and fills every destination's bucket
           (bf16 or fp32-master input, default or arithmetic payload, a whole model or one sender's share)
  refresh  the same, and the sender's previous weights become the new ones
  update   a whole update of a co-located program: encode, the overflow check of every bucket, apply of every bucket
  apply    a receiver applies the bucket of its shard
  pack     a sender cuts a bucket into transport objects
  objects  a receiver applies the objects of its shard
  dense    a sender copies whole shards, the path above the density where the sparse form pays

and the model it works on: a decoder (embedding, layers of norm / QKV / o / norm / gate-up / down, norm, head)
or a single matrix, with sizes of bench.py's workloads and of the tests, or generic ones.  All of a side's
tensors lie in one flat buffer, as parameter buffers do: each at a multiple of 256 elements, or (packed) one
right behind the other from an odd element on, so that odd sizes leave the ones behind them unaligned.

Every output is a bit pattern or a whole number, so every tolerance is "exact".
"""
import torch

import paper_2605_06534_amd as R

REPLICATED, SPLIT_ROWS, SPLIT_COLS, FUSED_ROWS = 0, 1, 2, 3
OBJECT_ENTRIES = (64 << 20) // 6        # a 64 MB object, the push size of the paper


# ---------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------
def _decoder(layers, hidden, q_heads, kv_heads, head_dim, inter, vocab):
    return {"model": "decoder", "layers": layers, "hidden": hidden, "q_heads": q_heads, "kv_heads": kv_heads,
            "head_dim": head_dim, "inter": inter, "vocab": vocab}


def _7b(layers=32):
    return _decoder(layers, 4096, 32, 32, 128, 11008, 32000)


def _8b(layers=36):
    return _decoder(layers, 4096, 32, 8, 128, 12288, 151936)


def _32b(layers=64):
    return _decoder(layers, 5120, 40, 8, 128, 27648, 152064)


def _case(path, model, tp, density, dtype="bf16", payload="new", packed=False, scratch="own", tp_src=1, src_rank=0,
          pp_src=1, stage_src=0, pp_dst=1):
    return dict(model, path=path, tp=tp, density=density, dtype=dtype, payload=payload, packed=packed,
                scratch=scratch, tp_src=tp_src, src_rank=src_rank, pp_src=pp_src, stage_src=stage_src, pp_dst=pp_dst)


def listed():
    def named(name, c):
        return dict(c, name=name)

    return [
        # the smallest real update: a draft or reward model's few million weights, synchronised inside one
        # process after every optimizer step; launches and latency are all there is
        named("update_small_tp4", _case("update", _decoder(2, 512, 8, 4, 64, 1408, 4096), 4, 0.05)),
        # one weight matrix synchronised by itself (a tuned projection, an adapter merged into it)
        named("encode_matrix4096", _case("encode", {"model": "matrix", "rows": 4096, "cols": 4096}, 1, 0.01)),
        # the ordinary sender: a whole 7B-style model re-sharded to four receivers after an RL step
        named("encode_7b_tp4", _case("encode", _7b(), 4, 0.05)),
        # a trainer with fp32 masters and a GQA model of the 32B style (two of its layers) for eight receivers
        named("encode_f32_32b_tp8", _case("encode", _32b(2), 8, 0.016, dtype="f32")),
        # one of sixteen trainer ranks: TP8 x PP2 feeding TP4, the paper's example, a rank's share of the 32B style
        named("encode_sender_32b", _case("encode", _32b(), 4, 0.02, tp_src=8, src_rank=3, pp_src=2, stage_src=1)),
        # a model whose widths are no multiple of eight, its tensors packed in one flat parameter buffer
        named("encode_ragged_packed", _case("encode", _decoder(4, 1530, 10, 2, 153, 4094, 10006), 2, 0.02, packed=True)),
        # the sender keeps its previous weights current for the next step (twelve layers of the 8B style)
        named("refresh_8b_tp4", _case("refresh", _8b(12), 4, 0.02)),
        # payloads that the receiver adds (eight layers of the 7B style)
        named("encode_arith_7b_tp4", _case("encode", _7b(8), 4, 0.05, payload="arith")),
        # a receiver of the 7B style at TP4 applies its bucket
        named("apply_7b_tp4", _case("apply", _7b(), 4, 0.05)),
        # the same bucket as 64 MB objects, on the sending and on the receiving side
        named("pack_7b_tp4", _case("pack", _7b(), 4, 0.05)),
        named("objects_7b_tp4", _case("objects", _7b(), 4, 0.05)),
        # dense synchronisation of every shard (eight layers of the 7B style)
        named("dense_7b_tp4", _case("dense", _7b(8), 4, 1.0)),
    ]


def _log_uniform(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def draw(rng):
    """One more case: any path, a model of a million to two billion weights, odd widths, any option."""
    path = rng.choice(["encode", "encode", "encode", "refresh", "update", "apply", "apply", "pack", "objects", "dense"])
    tp = rng.choice([1, 2, 4, 8])
    tp_src = rng.choice([1, 1, 1, 2, 4, 8]) if path in ("encode", "refresh") else 1
    big = max(tp, tp_src)                              # powers of two: the larger one is a multiple of the other
    target = _log_uniform(rng, 1e6, 2e9) * (1 if tp_src == 1 else tp_src ** 0.5)
    if tp_src == 1 and rng.random() < 0.2:
        rows = big * max(1, int(_log_uniform(rng, 64, 16384)) // big)
        cols = big * max(1, int(target / rows) // big)
        model = {"model": "matrix", "rows": rows, "cols": cols}
    else:
        odd = rng.random() < 0.35                      # widths that are no multiple of eight on a shard
        step = 1 if odd else rng.choice([8, 64])
        kv = big * rng.choice([1, 1, 2])
        q = kv * rng.choice([1, 2, 4, 5])
        head_dim = max(8, int(_log_uniform(rng, 512, 6144) * (target / 2e9) ** 0.25) // q)
        head_dim = head_dim + 1 - head_dim % 2 if odd else -(-head_dim // 8) * 8
        hidden = q * head_dim
        inter = big * step * max(1, int(hidden * rng.uniform(2.0, 5.4) / (big * step)))
        vocab = big * max(8, int(_log_uniform(rng, 1000, 160000) * min(1.0, target / 1e9) / big))
        per_layer = hidden * (2 * q * head_dim + 2 * kv * head_dim + 3 * inter)
        layers = max(1, min(64, int((target - 2 * vocab * hidden) / per_layer)))
        model = _decoder(layers, hidden, q, kv, head_dim, inter, vocab)
    dtype = rng.choice(["bf16", "bf16", "f32"]) if path in ("encode", "refresh", "update", "dense") else "bf16"
    payload = "arith" if path in ("encode", "refresh") and rng.random() < 0.25 else "new"
    density = 1.0 if path == "dense" else round(_log_uniform(rng, 0.0005, 0.5 if rng.random() < 0.25 else 0.15), 5)
    pp_src = rng.choice([1, 2]) if tp_src > 1 and model["layers"] % 2 == 0 else 1
    return _case(path, model, tp, density, dtype=dtype, payload=payload, packed=rng.random() < 0.4,
                 scratch=rng.choice(["own", "own", "built-in"]), tp_src=tp_src, src_rank=rng.randrange(tp_src),
                 pp_src=pp_src, stage_src=rng.randrange(pp_src))


# ---------------------------------------------------------------------------------------------------
# models, buffers, inputs
# ---------------------------------------------------------------------------------------------------
def _tensors(c):
    if c["model"] == "matrix":
        return [{"rows": c["rows"], "cols": c["cols"], "rule": SPLIT_ROWS}]
    h, q, kv, inter, v = c["hidden"], c["q_heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"], c["inter"], c["vocab"]
    ts = [{"rows": v, "cols": h, "rule": SPLIT_ROWS, "layer": R.LAYER_FIRST}]
    for i in range(c["layers"]):
        ts += [{"rows": 1, "cols": h, "rule": REPLICATED, "layer": i},
               {"rows": q + 2 * kv, "cols": h, "rule": FUSED_ROWS, "sections": [q, kv, kv], "layer": i},
               {"rows": h, "cols": q, "rule": SPLIT_COLS, "layer": i},
               {"rows": 1, "cols": h, "rule": REPLICATED, "layer": i},
               {"rows": 2 * inter, "cols": h, "rule": FUSED_ROWS, "sections": [inter, inter], "layer": i},
               {"rows": h, "cols": inter, "rule": SPLIT_COLS, "layer": i}]
    return ts + [{"rows": 1, "cols": h, "rule": REPLICATED, "layer": R.LAYER_LAST},
                 {"rows": v, "cols": h, "rule": SPLIT_ROWS, "layer": R.LAYER_LAST}]


def _plan(c, ts):
    if c["pp_src"] > 1 or c["pp_dst"] > 1:
        return R.shard_plan(ts, c["tp"], c["tp_src"], c["src_rank"], c["layers"], c["pp_src"], c["stage_src"], c["pp_dst"])
    return R.shard_plan(ts, c["tp"], c["tp_src"], c["src_rank"])


def _layout(numels, packed):
    """Offset of each tensor in a flat buffer, and the buffer's length."""
    offs, at = [], 1 if packed else 0
    for n in numels:
        offs.append(at)
        at += n if packed else -(-n // 256) * 256
    return offs, max(at, 1)


def _views(flat, numels, packed):
    return [flat[o:o + n] for o, n in zip(_layout(numels, packed)[0], numels)]


def _gen(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + what * 7919 + 12345) & 0x7FFFFFFF)
    return g


_CHUNK = 1 << 27


def _weights(n, g):
    """bf16 patterns of weights, N(0, 0.02^2), as int16."""
    out = torch.empty(n, dtype=torch.int16, device="cuda")
    for a in range(0, n, _CHUNK):
        m = min(_CHUNK, n - a)
        out[a:a + m] = torch.randn(m, generator=g, device="cuda").mul_(0.02).to(torch.bfloat16).view(torch.int16)
    return out


def _changed(old, density, g, rows_of=None):
    """A copy of the patterns in which a share `density` has moved by a few units in the last place (1 to 7: the
    three low bits differ).  rows_of: the change rate differs from one stretch of this length to the next (as it
    does between rows of a matrix in training) and is `density` on average."""
    new = old.clone()
    for a in range(0, old.numel(), _CHUNK):
        m = min(_CHUNK, old.numel() - a)
        rate = density
        if rows_of:
            u = torch.rand(-(-m // rows_of), generator=g, device="cuda")
            rate = (u * u * (3 * density)).clamp_(max=1.0).repeat_interleave(rows_of)[:m]
        hit = torch.rand(m, generator=g, device="cuda") < rate
        by = torch.randint(1, 8, (m,), generator=g, device="cuda", dtype=torch.int16)
        new[a:a + m] ^= torch.where(hit, by, torch.zeros_like(by))
    return new


def _masters(bits, g):
    """fp32 masters that round to these bf16 patterns: each lies less than half a unit in the last place away."""
    out = torch.empty(bits.numel(), dtype=torch.int32, device="cuda")
    for a in range(0, bits.numel(), _CHUNK):
        b = bits[a:a + _CHUNK].to(torch.int32) << 16
        out[a:a + b.numel()] = b + torch.randint(-0x7FFF, 0x8000, b.shape, generator=g, device="cuda", dtype=torch.int32)
    return out.view(torch.float32)


def _bucket(capacity, n_tensors):
    b = R.Bucket(capacity, n_tensors)
    b.idx.zero_()
    b.val.zero_()
    return b


def _sized(capacity, density):
    """Entries a program provides for: a quarter more than it expects, never more than can come."""
    return min(capacity, int(1.25 * density * capacity) + 16384)


def _send_state(c, seed):
    ts = _tensors(c)
    plan = _plan(c, ts)
    plan.upload()
    numels = [plan.src_numel(t) for t in range(len(ts))]
    _, total = _layout(numels, c["packed"])
    rows_of = 4096 if c["dtype"] == "f32" else None
    s = {"case": c, "plan": plan, "tensors": ts, "numels": numels, "turn": 0}
    s["old"] = _weights(total, _gen(seed, 1))
    new = _changed(s["old"], c["density"], _gen(seed, 2), rows_of)
    if c["path"] == "refresh":
        # two sets of new weights taken in turn: after a pass the previous weights are the one, the next is the other
        s["news"] = [new, s["old"].clone()]
    else:
        s["news"] = [new]
    if c["dtype"] == "f32":
        s["news"] = [_masters(x, _gen(seed, 3 + i)) for i, x in enumerate(s["news"])]
    s["old_tab"] = R.ptr_table(_views(s["old"], numels, c["packed"]))
    s["new_tabs"] = [R.ptr_table(_views(x, numels, c["packed"])) for x in s["news"]]
    s["new_dtype"] = R.FP32_RNE if c["dtype"] == "f32" else R.BF16
    s["flags"] = (R.ENCODE_REFRESH if c["path"] == "refresh" else 0) | (R.ENCODE_ARITH if c["payload"] == "arith" else 0)
    if c["path"] != "dense":
        s["buckets"] = [_bucket(_sized(plan.bucket_capacity(d), c["density"]), len(ts)) for d in range(plan.n_buckets)]
        s["ws"] = R.workspace(plan) if c["scratch"] == "own" else None
    if c["path"] in ("update", "dense"):
        s["dst"], s["dst_tabs"] = [], []
        for d in range(plan.n_buckets):
            ln = [plan.local_numel(t, d) for t in range(len(ts))]
            flat = torch.zeros(_layout(ln, c["packed"])[1], dtype=torch.int16, device="cuda")
            if c["path"] == "update":                  # the receiver holds its shard of the previous weights
                for dst, w in zip(_views(flat, ln, c["packed"]), _shard(s, s["old"], d)):
                    dst.copy_(w)
            s["dst"].append(flat)
            s["dst_tabs"].append(R.ptr_table(_views(flat, ln, c["packed"])))
    return s


def _receive_state(c, seed):
    """Shard 0 of a receiver and the bucket that has come for it."""
    ts = _tensors(c)
    plan = _plan(c, ts)
    plan.upload()
    ln = [plan.local_numel(t, 0) for t in range(len(ts))]
    s = {"case": c, "plan": plan, "tensors": ts, "numels": ln}
    g = _gen(seed, 5)
    parts, seg = [], [0]
    for n in ln:
        got = 0
        for a in range(0, n, _CHUNK):
            m = min(_CHUNK, n - a)
            hit = (torch.rand(m, generator=g, device="cuda") < c["density"]).nonzero().view(-1)
            parts.append((hit + a).to(torch.int32))
            got += hit.numel()
        seg.append(seg[-1] + got)
    b = s["bucket"] = _bucket(_sized(plan.bucket_capacity(0), c["density"]), len(ts))
    s["total"] = seg[-1]
    b.idx[:seg[-1]] = torch.cat(parts)
    b.val[:seg[-1]] = _weights(seg[-1], _gen(seed, 6))
    b.seg_off.copy_(torch.tensor(seg, dtype=torch.int64))
    del parts
    if c["path"] != "pack":
        s["dst"] = _weights(_layout(ln, c["packed"])[1], _gen(seed, 7))
        s["dst_tab"] = R.ptr_table(_views(s["dst"], ln, c["packed"]))
    if c["path"] != "apply":
        # fixed-size places for the objects, as many as the bucket's capacity could need, side by side
        per = min(max(OBJECT_ENTRIES, -(-b.capacity // 32)), b.capacity)
        size = R.object_bytes(plan, per)
        s["store"] = torch.zeros(size * -(-b.capacity // per), dtype=torch.uint8, device="cuda")
        s["ranges"] = [(a, min(per, seg[-1] - a)) for a in range(0, max(seg[-1], 1), per)]
        s["objects"] = [s["store"][i * size:i * size + R.object_bytes(plan, n)] for i, (_, n) in enumerate(s["ranges"])]
    if c["path"] == "objects":
        for (a, n), o in zip(s["ranges"], s["objects"]):
            R.bucket_pack(plan, 0, b, a, n, o)
        del s["bucket"]
    return s


def prepare(case, seed):
    return (_receive_state if case["path"] in ("apply", "pack", "objects") else _send_state)(case, seed)


# ---------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------
def _encode(s, new_tab):
    if s["ws"] is None:
        R.delta_encode_static(s["plan"], s["old_tab"], new_tab, s["new_dtype"], s["flags"], s["buckets"])
    elif s["flags"]:
        R.delta_encode_ex(s["plan"], s["old_tab"], new_tab, s["new_dtype"], s["flags"], s["buckets"], s["ws"])
    else:
        R.delta_encode(s["plan"], s["old_tab"], new_tab, s["new_dtype"], s["buckets"], s["ws"])


def _bucket_outputs(s):
    return [{"idx": b.idx, "val": b.val, "seg_off": b.seg_off} for b in s["buckets"]]


def run(state):
    s, path = state, state["case"]["path"]
    if path == "encode":
        _encode(s, s["new_tabs"][0])
        return {"buckets": _bucket_outputs(s)}
    if path == "refresh":
        _encode(s, s["new_tabs"][s["turn"]])
        s["turn"] ^= 1
        return {"buckets": _bucket_outputs(s), "old": s["old"]}
    if path == "update":
        _encode(s, s["new_tabs"][0])
        counts = [R.bucket_check(s["plan"], b) for b in s["buckets"]]
        for d, b in enumerate(s["buckets"]):
            R.delta_apply(s["plan"], d, b, s["dst_tabs"][d])
        return {"buckets": _bucket_outputs(s), "counts": counts, "shards": s["dst"]}
    if path == "apply":
        R.delta_apply(s["plan"], 0, s["bucket"], s["dst_tab"])
        return {"shard": s["dst"]}
    if path == "pack":
        for (a, n), o in zip(s["ranges"], s["objects"]):
            R.bucket_pack(s["plan"], 0, s["bucket"], a, n, o)
        return {"objects": s["store"]}
    if path == "objects":
        for o in s["objects"]:
            R.object_apply(s["plan"], o, s["dst_tab"])
        return {"shard": s["dst"]}
    for d in range(s["plan"].n_buckets):
        R.dense_copy(s["plan"], d, s["new_tabs"][0], s["new_dtype"], s["dst_tabs"][d])
    return {"shards": s["dst"]}


# ---------------------------------------------------------------------------------------------------
# what a pass cannot do without, and what it must give
# ---------------------------------------------------------------------------------------------------
def work(case):
    """Bytes: weights read once, entries (4 bytes of index, 2 of value) read or written once, changed weights
    written once.  Nothing is computed that counts as an operation beside the comparison of each element."""
    c, ts = case, _tensors(case)
    stage = (lambda t: (0 if t["layer"] == R.LAYER_FIRST else c["pp_src"] - 1 if t["layer"] == R.LAYER_LAST
                        else t["layer"] // (c["layers"] // c["pp_src"])) if c["pp_src"] > 1 else 0)
    held = sent = to_shard = 0
    for i, t in enumerate(ts):
        n = t["rows"] * t["cols"]
        to_shard += n // (1 if t["rule"] == REPLICATED else c["tp"])
        if stage(t) != c["stage_src"]:
            continue
        if t["rule"] == REPLICATED:
            held += n
            sent += n * c["tp"] if i % c["tp_src"] == c["src_rank"] else 0
        else:
            held += n // c["tp_src"]
            sent += n // c["tp_src"]
    wide = 4 if c["dtype"] == "f32" else 2
    path, p = c["path"], c["density"]
    if path in ("apply", "objects"):
        return {"bytes": 8 * p * to_shard, "flops": 0}
    if path == "pack":
        return {"bytes": 12 * p * to_shard, "flops": 0}
    if path == "dense":
        return {"bytes": wide * held + 2 * sent, "flops": 0}
    nbytes = (2 + wide) * held + 6 * p * sent
    if path == "refresh":
        nbytes += 2 * p * held
    if path == "update":
        nbytes += 8 * p * sent
    return {"bytes": nbytes, "flops": held}


def tolerance(case):
    return "exact"          # patterns, indices and counts: one right answer


def _shard(s, flat, d):
    """Shard d of every tensor in the flat buffer, by plain slicing (a sender that holds the whole model)."""
    c, out = s["case"], []
    for t, w in zip(s["tensors"], _views(flat, s["numels"], c["packed"])):
        m, tp = w.view(t["rows"], t["cols"]), c["tp"]
        if t["rule"] == SPLIT_ROWS:
            m = m[d * (t["rows"] // tp):(d + 1) * (t["rows"] // tp)]
        elif t["rule"] == SPLIT_COLS:
            m = m[:, d * (t["cols"] // tp):(d + 1) * (t["cols"] // tp)]
        elif t["rule"] == FUSED_ROWS:
            parts, at = [], 0
            for rows in t["sections"]:
                parts.append(m[at + d * (rows // tp):at + (d + 1) * (rows // tp)])
                at += rows
            m = torch.cat(parts)
        out.append(m.reshape(-1))
    return out


def _value(bits):
    return bits.contiguous().view(torch.bfloat16).to(torch.float64)


def _rounded(x):
    """The nearest bf16 pattern (ties to even) of a value that 64 bits hold exactly: 32 bits hold the sums and
    differences met here exactly too."""
    return x.to(torch.float32).to(torch.bfloat16).view(torch.int16)


def exact(case, seed):
    """The same outputs by plain slicing, comparison and assignment in torch."""
    c = case
    if c["tp_src"] > 1 or c["pp_src"] > 1 or c["pp_dst"] > 1:
        return None
    s = prepare(case, seed)
    if c["path"] == "pack":
        return None                                    # a format, not numbers
    if c["path"] in ("apply", "objects"):
        b = s.get("bucket")
        if b is None:
            b = _receive_state(dict(case, path="apply"), seed)["bucket"]
        seg = b.seg_off.tolist()
        for t, w in enumerate(_views(s["dst"], s["numels"], c["packed"])):
            w[b.idx[seg[t]:seg[t + 1]].long()] = b.val[seg[t]:seg[t + 1]]
        return {"shard": s["dst"]}
    new = s["news"][0]
    if c["dtype"] == "f32":
        new = torch.cat([x.to(torch.bfloat16).view(torch.int16) for x in new.split(_CHUNK)])
    shards = []
    for d in range(c["tp"]):
        parts = list(zip(_shard(s, s["old"], d), _shard(s, new, d)))
        if c["path"] in ("dense", "update"):
            ln = [x.numel() for _, x in parts]
            flat = s["dst"][d]
            for v, (_, n) in zip(_views(flat, ln, c["packed"]), parts):
                v.copy_(n)
            shards.append(flat)
        if c["path"] == "dense":
            continue
        b, at, seg = s["buckets"][d], 0, [0]
        for o, n in parts:
            where = (o != n).nonzero().view(-1)
            idx, val = where.to(torch.int32), n[where]
            if c["payload"] == "arith":
                was, now = _value(o[where]), _value(val)
                step = _rounded(now - was)
                lost = (_rounded(was + _value(step)) != val) | _value(step).isnan()
                val = torch.where(lost, val, step)
                idx = torch.where(lost, idx | -0x80000000, idx)
            b.idx[at:at + idx.numel()], b.val[at:at + idx.numel()] = idx, val
            at += idx.numel()
            seg.append(at)
        b.seg_off.copy_(torch.tensor(seg, dtype=torch.int64))
    if c["path"] == "dense":
        return {"shards": shards}
    got = {"buckets": _bucket_outputs(s)}
    if c["path"] == "refresh":
        held = s["old"].clone()
        for v, n in zip(_views(held, s["numels"], c["packed"]), _views(new, s["numels"], c["packed"])):
            v.copy_(n)
        got["old"] = held
    if c["path"] == "update":
        got["counts"] = [int(b.seg_off[-1]) for b in s["buckets"]]
        got["shards"] = shards
    return got
