"""The work a training program has this library do each step, as cases that can be timed and compared.

A case names a model's shape (dense transformer, mixture of experts, or ragged tensor lists), the sharding
(alignment, Z3, Z1, rank), and one of the operations:

  update        hzp_adamw_shard over all layers, one call per dtype class: sums R gradient contributions, AdamW on
                master / m / v, cast parameters.  reduced=True: from one fp32 gradient that is already summed (R == 0)
  reduce        hzp_reduce_shard per layer, as a backward pass produces gradients (issue="thread": through the
                scheduler's background thread)
  post_gather   after the step: each ZeRO-3 shard rebuilt from its ZeRO-1 owners (hzp_gather_layers; hzp_gather_shard
                where Z3 does not divide Z1)
  layer_gather  before a layer is used: its ZeRO-3 shards gathered into the bucket, into its tensors, or both
  param_gather  the same at parameter granularity (hzp_gather_tensor)
  step          update, post_gather and layer_gather into tensors, as one training step runs them

What a program keeps from step to step (plan, device tables, buffers, pointer arrays, scheduler) is made by prepare().
"""
import math
import random

import torch

import paper_2510_20111_amd as hzp

DEV = "cuda:0"
ADAMW = dict(lr=1e-4, beta1=0.9, beta2=0.95, eps=1e-8, weight_decay=0.1)
STEP = 100              # well into training: momentum and variance are not zero
SIGMA = 1e-3            # of one gradient contribution
BF16, F32 = 0, 1
FIRST = dict(cls="bf16", decay="uniform", rank=0, align=128)

DENSE7B = dict(shape="dense", layers=32, hidden=4096, kv=4096, ffn=11008, vocab=32000, z3=8, z1=64, R=8)
MOE = dict(shape="moe", hidden=4096, ffn=1408, experts=66, z3=4, z1=16, R=16)


def listed():
    cases = [
        # A unit-test sized model: one small launch, all latency.
        dict(name="update_tiny", op="update", shape="dense", layers=2, hidden=256, kv=256, ffn=1024, vocab=1024, z3=2, z1=4,
             rank=2, R=4),
        # 4096 tensors of 1 to 65536 elements in 64 groups, every fourth one fp32 without decay: the whole step, launch bound.
        dict(name="step_ragged", op="step", shape="ragged", layers=64, tensors=64, largest=65536, shape_seed=0, align=256,
             z3=2, z1=32, rank=5, R=16, cls="mixed", decay="norms_off"),
        # One rank's share of a 7B-class dense model, the ordinary optimizer step.
        dict(name="update_dense7b", op="update", rank=9, **DENSE7B),
        # The same where norm weights take no decay, as most training recipes have it.
        dict(name="update_dense7b_norms_undecayed", op="update", rank=9, decay="norms_off", **DENSE7B),
        # Eight layers of a mixture of experts with 16 contributions: the largest update.
        dict(name="update_moe", op="update", layers=8, rank=5, **MOE),
        # Six data-parallel replicas, grouped queries, norms kept in fp32: not a power of two anywhere.
        dict(name="update_six_replicas", op="update", shape="dense", layers=24, hidden=2560, kv=640, ffn=6912, vocab=0, z3=8,
             z1=48, rank=13, R=6, cls="mixed", decay="norms_off"),
        # 70B-class layers, gradients accumulated in fp32 over the micro-batches beforehand.
        dict(name="update_reduced_dense70b", op="update", shape="dense", layers=16, hidden=8192, kv=1024, ffn=28672, vocab=0,
             z3=8, z1=128, rank=9, R=1, reduced=True),
        # Backward pass: every layer's ZeRO-3 gradient shard summed as soon as it is there, from the background thread.
        dict(name="reduce_backward_dense7b", op="reduce", level=3, grads="bf16", accumulate=False, issue="thread", rank=9,
             **dict(DENSE7B, layers=16, vocab=0)),
        # fp32 contributions of one micro-batch added to the resident fp32 shard.
        dict(name="accumulate_fp32", op="reduce", shape="dense", layers=12, hidden=2048, kv=2048, ffn=5504, vocab=0, z3=8,
             z1=32, rank=3, R=4, level=2, grads="f32", accumulate=True, issue="call"),
        # After the step: all layers' parameter shards from their optimizer shards, the rank's own piece in place.
        dict(name="post_gather_dense7b", op="post_gather", rank=9, **DENSE7B),
        # Forward pass on flat layer buckets.
        dict(name="layer_gather_dense7b", op="layer_gather", out="bucket", rank=9, **dict(DENSE7B, layers=12, vocab=0)),
        # Forward pass on separate expert tensors, 199 to a layer.
        dict(name="layer_gather_moe_tensors", op="layer_gather", out="tensors", layers=2, rank=5, **MOE),
    ]
    return [dict(FIRST, **c) for c in cases]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of these ranges; sizes over their logarithm, odd ones among them."""
    while True:
        op = rng.choice(["update"] * 6 + ["reduce"] * 3 + ["post_gather"] * 2 + ["layer_gather"] * 3 + ["param_gather", "step"])
        c = dict(FIRST, op=op, shape=rng.choice(["dense", "dense", "moe", "ragged"]), layers=_log(rng, 1, 48))
        if c["shape"] == "ragged":
            c.update(tensors=_log(rng, 2, 96), largest=_log(rng, 512, 1 << 21), shape_seed=rng.randrange(1 << 20))
        else:
            hidden = _log(rng, 64, 8192)
            if rng.random() < 0.7:
                hidden = -(-hidden // 64) * 64
            c.update(hidden=hidden, kv=max(1, hidden // rng.choice([1, 1, 4, 8])), ffn=int(hidden * rng.choice([0.35, 1.0, 2.6875, 3.5, 4])))
            if c["shape"] == "moe":
                c.update(experts=_log(rng, 4, 72), ffn=max(8, c["ffn"] // 4))
            else:
                c.update(vocab=rng.choice([0, 0, 32000, 50257]))
        c.update(align=rng.choice([8, 64, 128, 128, 256]), z3=rng.choice([1, 2, 4, 8, 8]))
        c["z1"] = c["z3"] * rng.choice([1, 2, 3, 4, 8, 16])
        if op == "post_gather" and rng.random() < 0.4:
            c["z1"] = rng.choice([6, 12, 20, 36])       # group sizes that may not nest
        c.update(rank=rng.randrange(c["z1"]), R=rng.choice([1, 2, 3, 4, 4, 5, 6, 8, 8, 8, 12, 16, 16, 24, 32]),
                 cls=rng.choice(["bf16", "bf16", "bf16", "mixed", "f32"]), decay=rng.choice(["uniform", "norms_off"]))
        if op in ("update", "step"):
            c["reduced"] = rng.random() < 0.2
            c["calls"] = rng.choice(["range", "range", "range", "layer"])
            if c["reduced"]:
                c["R"] = 1
        if op == "reduce":
            c.update(level=rng.choice([1, 2, 3]), grads=rng.choice(["bf16", "bf16", "f32"]), accumulate=rng.random() < 0.4,
                     issue=rng.choice(["call", "call", "thread"]))
        if op in ("layer_gather", "step"):
            c["out"] = rng.choice(["bucket", "tensors", "both"]) if op == "layer_gather" else "tensors"
        got = work(c)["bytes"]
        if 2e5 <= got <= 3e10 and _resident(c) <= 4e10:
            return c


# ------------------------------------------------------------------------------------------------ shapes and layout

def tensors_of(case):
    """Per layer a list of (numel, class, decay multiplier)."""
    big = F32 if case["cls"] == "f32" else BF16
    small = BF16 if case["cls"] == "bf16" else F32
    off = 0.0 if case["decay"] == "norms_off" else 1.0
    if case["shape"] == "ragged":
        r = random.Random(case["shape_seed"])
        sizes = [max(1, int(math.exp(r.uniform(0.0, math.log(case["largest"]))))) for _ in range(case["layers"] * case["tensors"])]
        flat = [(n, small, off) if i % 4 == 3 else (n, big, 1.0) for i, n in enumerate(sizes)]
        return [flat[i:i + case["tensors"]] for i in range(0, len(flat), case["tensors"])]
    h, f = case["hidden"], case["ffn"]
    if case["shape"] == "moe":
        layer = [(64 * h, small, off)] + [(f * h, big, 1.0)] * (3 * case["experts"])
        return [layer] * case["layers"]
    norm = (h, small, off)
    mats = [(n, big, 1.0) for n in (h * h, case["kv"] * h, case["kv"] * h, h * h, f * h, f * h, f * h)]
    layers = [[norm] + mats[:4] + [norm] + mats[4:]] * case["layers"]
    if case["vocab"]:
        layers = layers + [[(case["vocab"] * h, big, 1.0)], [(case["vocab"] * h, big, 1.0), norm]]
    return layers


def layout(case):
    """Per class the buckets of the layers that have one: layer, tensors (offset, numel), padded length P, shard lengths."""
    z1, z3, A = case["z1"], case["z3"], case["align"]
    unit = A * (z1 * z3 // math.gcd(z1, z3))
    out = {}
    for layer, ts in enumerate(tensors_of(case)):
        for cls in (BF16, F32):
            at, end, rows = 0, 0, []
            for n, c, wd in ts:
                if c == cls:
                    rows.append((at, n, wd))
                    end = at + n
                    at = -(-end // A) * A
            if rows:
                P = -(-end // unit) * unit
                out.setdefault(cls, []).append(dict(layer=layer, rows=rows, P=P, S1=P // z1, S3=P // z3))
    return out


def shard_of(case, level):
    """Index of the shard the rank owns (Z2 = Z3)."""
    z1, z3, r = case["z1"], case["z3"], case["rank"]
    if level != 1:
        return r % z3
    return (r % z3) * (z1 // z3) + (r // z3) % (z1 // z3) if z1 % z3 == 0 else r % z1


def _gather_bytes(case, b, es, out):
    payload = sum(n for _, n, _ in b["rows"])
    return {"bucket": 2 * b["P"], "tensors": 2 * payload, "both": 2 * b["P"] + payload}[out] * es


def work(case):
    nbytes = flops = 0
    for cls, buckets in layout(case).items():
        es = 4 if cls == F32 else 2
        for b in buckets:
            if case["op"] in ("update", "step"):
                grads = 4 if case.get("reduced") else case["R"] * es
                nbytes += b["S1"] * (grads + 24 + es)
                flops += b["S1"] * (case["R"] + 18)
            if case["op"] == "reduce":
                n = b["P"] // (case["z1"] if case["level"] == 1 else case["z3"])
                nbytes += n * (case["R"] * (4 if case["grads"] == "f32" else 2) + (8 if case["accumulate"] else 4))
                flops += n * (case["R"] + 1)
            if case["op"] in ("post_gather", "step"):
                own = b["S1"] if case["z1"] % case["z3"] == 0 else 0
                nbytes += 2 * (b["S3"] - own) * es
            if case["op"] in ("layer_gather", "step"):
                nbytes += _gather_bytes(case, b, es, case.get("out", "tensors"))
            if case["op"] == "param_gather":
                nbytes += _gather_bytes(case, b, es, "tensors")
    return {"bytes": nbytes, "flops": flops}


def _resident(case):
    """Bytes of one state, roughly."""
    total = 0
    for cls, buckets in layout(case).items():
        es = 4 if cls == F32 else 2
        for b in buckets:
            total += 3 * b["P"] * es + b["S1"] * (4 * case["R"] + 16)
    return total + work(case)["bytes"]


def tolerance(case):
    """Reductions are documented as bit exact and gathers are copies.  For the update, master, m and v stay within 5e-8 of a
    64-bit evaluation (1e-6 of the rms at the worst element); a master weight that an fp32 ulp moves across the middle between
    two bf16 values moves its cast parameter by a bf16 ulp (up to 2^-7 of its value), which in the smallest arrays (1e4 values)
    is 4e-5 of the norm."""
    if case["op"] not in ("update", "step"):
        return "exact"
    if case["cls"] == "f32":
        return {"rel": 2e-7, "max": 4e-6}
    return {"rel": 4e-5, "max": 1e-2}


# ------------------------------------------------------------------------------------------------ inputs

def _normal(t, gen, std):
    t.normal_(0.0, std, generator=gen)


def _padding(case, buckets, begin_of, len_of):
    """Positions of the padding in a stream that holds [begin_of(b), begin_of(b) + len_of(b)) of each bucket, back to back."""
    parts, at = [], 0
    for b in buckets:
        lo, hi = begin_of(b), begin_of(b) + len_of(b)
        ends = [o + n for o, n, _ in b["rows"]]
        starts = [o for o, _, _ in b["rows"][1:]] + [b["P"]]
        for e, s in zip(ends, starts):
            x, y = max(e, lo), min(s, hi)
            if x < y:
                parts.append(torch.arange(at + x - lo, at + y - lo))
        at += len_of(b)
    return torch.cat(parts).to(DEV) if parts else None


def fill_update(case, cls, buckets, gen, streams):
    """Gradients, master, m, v of one class: normal values, zeros in the padding.  streams: [gradients..., master, m, v]."""
    i = shard_of(case, 1)
    pad = _padding(case, buckets, lambda b: i * b["S1"], lambda b: b["S1"])
    n = len(streams) - 3
    mean_std = SIGMA / math.sqrt(case["R"])
    for k, t in enumerate(streams):
        _normal(t, gen, SIGMA if k < n else (0.02, 0.3 * mean_std, mean_std)[k - n])
        if k == n + 2:
            t.square_()
        if pad is not None:
            t.index_fill_(0, pad, 0.0)


def fill_parameters(gen, t):
    _normal(t, gen, 0.02)


def _split(t, lengths):
    return list(torch.split(t, lengths))


# ------------------------------------------------------------------------------------------------ prepare and run

def _plan(case):
    layers = tensors_of(case)
    flat = [t for layer in layers for t in layer]
    plan = hzp.hzp_plan([len(layer) for layer in layers], [t[0] for t in flat], case["align"], case["z3"], case["z1"],
                        tensor_class=[t[1] for t in flat], tensor_wd_mult=[t[2] for t in flat])
    plan.prepare()
    return plan, len(layers)


def _dtype(cls):
    return torch.float32 if cls == F32 else torch.bfloat16


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _arena(plan, cls, R, grad_dtype):
    """The rank's buffers of one class in one allocation: a function that gives a stream's slices of all buckets as one tensor."""
    size, unit = plan.arena(cls, R, grad_dtype), hzp.HZP_ARENA_ALIGN
    raw = torch.empty(size + unit, dtype=torch.uint8, device=DEV)
    start = -raw.data_ptr() % unit

    def stream(kind, index, buckets, dtype):
        spans = [plan.arena_slice(cls, R, kind, index, b["layer"], grad_dtype) for b in buckets]
        lo, hi = start + spans[0][0], start + spans[-1][0] + spans[-1][1]
        return raw[lo:hi].view(dtype)
    return stream


def _by_layer(n_layers, buckets, tensors):
    """Pointer list over all layers (NULL where a layer has no bucket of the class)."""
    at = {b["layer"]: t for b, t in zip(buckets, tensors)}
    return [at.get(layer) for layer in range(n_layers)]


def _update_calls(case, plan, n_layers, cls, buckets, grads, master, m, v, out):
    """Arguments of the update's calls: one for the layer range, or one per layer."""
    R = len(grads)
    lens = [b["S1"] for b in buckets]
    per = [_by_layer(n_layers, buckets, _split(t, lens)) for t in grads]
    g = [per[r][layer] for layer in range(n_layers) for r in range(R)]
    state = [_by_layer(n_layers, buckets, _split(t, lens)) for t in (master, m, v)] + [_by_layer(n_layers, buckets, out)]
    Rarg = 0 if case.get("reduced") else R
    if case.get("calls") == "layer":
        spans = [(b["layer"], b["layer"] + 1) for b in buckets]
    else:
        spans = [(0, n_layers)]
    return [(lo, hi, cls, Rarg, hzp.ptr_array(g[lo * R:hi * R]), [hzp.ptr_array(x[lo:hi]) for x in state]) for lo, hi in spans]


def _prepare_update(case, st, gen, in_place):
    plan, n_layers = st["plan"], st["n_layers"]
    for cls, buckets in layout(case).items():
        reduced = bool(case.get("reduced"))
        gdt = hzp.HZP_GRAD_F32 if reduced else hzp.HZP_GRAD_DEFAULT
        R = 1 if reduced else case["R"]
        stream = _arena(plan, cls, R, gdt)
        dt = _dtype(cls)
        gtype = torch.float32 if reduced else dt
        grads = [stream(hzp.HZP_STREAM_GRAD, r, buckets, gtype) for r in range(R)]
        master, m, v = (stream(k, 0, buckets, torch.float32) for k in (hzp.HZP_STREAM_MASTER, hzp.HZP_STREAM_M, hzp.HZP_STREAM_V))
        fill_update(case, cls, buckets, gen, grads + [master, m, v])
        outs = {"master": master, "m": m, "v": v}
        if in_place:
            shard3 = stream(hzp.HZP_STREAM_SHARD3, 0, buckets, dt)
            k = shard_of(case, 1) % (case["z1"] // case["z3"])
            whole = _split(shard3, [b["S3"] for b in buckets])
            own = [s[k * b["S1"]:(k + 1) * b["S1"]] for s, b in zip(whole, buckets)]
            st["shard3"][cls] = whole
            outs["shard3"] = shard3
            st["stream"][cls] = stream
        else:
            param = stream(hzp.HZP_STREAM_PARAM_OUT, 0, buckets, dt)
            own = _split(param, [b["S1"] for b in buckets])
            outs["param"] = param
        st["updates"] += _update_calls(case, plan, n_layers, cls, buckets, grads, master, m, v, own)
        st["out"]["class%d" % cls] = outs


def _prepare_post_gather(case, st, gen):
    plan, n_layers = st["plan"], st["n_layers"]
    z1, z3 = case["z1"], case["z3"]
    j = shard_of(case, 3)
    for cls, buckets in layout(case).items():
        dt = _dtype(cls)
        if z1 % z3:
            owners, jobs = [], []
            flat = torch.zeros(sum(b["S3"] for b in buckets), dtype=dt, device=DEV)
            for b, dst in zip(buckets, _split(flat, [b["S3"] for b in buckets])):
                first, n = plan.cover(b["layer"], cls, j)
                src = torch.empty(n * b["S1"], dtype=dt, device=DEV)
                fill_parameters(gen, src)
                owners.append(src)
                jobs.append((b["layer"], cls, j, hzp.ptr_array(_split(src, [b["S1"]] * n)), dst))
            st["shard_jobs"] += jobs
            st["keep"].append(owners)
            st["out"]["shard3_%d" % cls] = flat
            continue
        K = z1 // z3
        own = shard_of(case, 1) % K
        if cls in st["shard3"]:                     # the update of the same step wrote the rank's own piece
            whole, stream = st["shard3"][cls], st["stream"][cls]
            recv = [stream(hzp.HZP_STREAM_RECV1, k, buckets, dt) for k in range(K - 1)]
        else:
            flat = torch.zeros(sum(b["S3"] for b in buckets), dtype=dt, device=DEV)
            whole = _split(flat, [b["S3"] for b in buckets])
            recv = [torch.empty(sum(b["S1"] for b in buckets), dtype=dt, device=DEV) for _ in range(K - 1)]
            st["out"]["shard3_%d" % cls] = flat
            mine = torch.empty(sum(b["S1"] for b in buckets), dtype=dt, device=DEV)
            fill_parameters(gen, mine)
            for s, b, x in zip(whole, buckets, _split(mine, [b["S1"] for b in buckets])):
                s[own * b["S1"]:(own + 1) * b["S1"]] = x
        for t in recv:
            fill_parameters(gen, t)
        parts = [_split(t, [b["S1"] for b in buckets]) for t in recv]
        srcs = [None] * (n_layers * K)
        for n, b in enumerate(buckets):
            pieces = [p[n] for p in parts]
            pieces.insert(own, whole[n][own * b["S1"]:(own + 1) * b["S1"]])
            srcs[b["layer"] * K:(b["layer"] + 1) * K] = pieces
        st["keep"].append(recv)
        st["post"].append((cls, hzp.ptr_array(srcs), K, hzp.ptr_array(_by_layer(n_layers, buckets, whole))))


def tensor_places(buckets):
    """Where the tensors of all buckets lie in one flat buffer, each on a multiple of 256 elements, and its length."""
    places, at = [], 0
    for b in buckets:
        row = []
        for _, n, _ in b["rows"]:
            row.append(at)
            at += -(-n // 256) * 256
        places.append(row)
    return places, at


def _prepare_layer_gather(case, st, gen):
    z3, out = case["z3"], case.get("out", "tensors")
    j = shard_of(case, 3)
    ids = {}
    for layer, ts in enumerate(tensors_of(case)):
        for n, c, _ in ts:
            ids.setdefault((layer, c), []).append(len(ids.setdefault("all", [])))
            ids["all"].append(n)
    for cls, buckets in layout(case).items():
        dt = _dtype(cls)
        recv = [None if cls in st["shard3"] and s == j else torch.empty(sum(b["S3"] for b in buckets), dtype=dt, device=DEV)
                for s in range(z3)]
        for t in recv:
            if t is not None:
                fill_parameters(gen, t)
        parts = [st["shard3"][cls] if t is None else _split(t, [b["S3"] for b in buckets]) for t in recv]
        st["keep"].append(recv)
        flat_bucket = flat_tensors = None
        places, total = tensor_places(buckets)
        if out in ("bucket", "both"):
            flat_bucket = torch.zeros(sum(b["P"] for b in buckets), dtype=dt, device=DEV)
            whole = _split(flat_bucket, [b["P"] for b in buckets])
            st["out"]["bucket_%d" % cls] = flat_bucket
        if out in ("tensors", "both") or case["op"] == "param_gather":
            flat_tensors = torch.zeros(total, dtype=dt, device=DEV)
            st["out"]["tensors_%d" % cls] = flat_tensors
        for n, b in enumerate(buckets):
            shards = hzp.ptr_array([p[n] for p in parts])
            views = None
            if flat_tensors is not None:
                views = [flat_tensors[at:at + r[1]] for at, r in zip(places[n], b["rows"])]
            if case["op"] == "param_gather":
                st["params"] += [(t, shards, view.data_ptr()) for t, view in zip(ids[(b["layer"], cls)], views)]
            else:
                st["layers"].append((b["layer"], cls, shards, whole[n].data_ptr() if flat_bucket is not None else None,
                                     hzp.ptr_array(views) if views is not None else None))


def _prepare_reduce(case, st, gen):
    plan = st["plan"]
    gtype = torch.float32 if case["grads"] == "f32" else torch.bfloat16
    div = case["z1"] if case["level"] == 1 else case["z3"]
    i = shard_of(case, case["level"])
    for cls, buckets in layout(case).items():
        lens = [b["P"] // div for b in buckets]
        pad = _padding(case, buckets, lambda b: i * (b["P"] // div), lambda b: b["P"] // div)
        grads = [torch.empty(sum(lens), dtype=gtype, device=DEV) for _ in range(case["R"])]
        acc = torch.empty(sum(lens), dtype=torch.float32, device=DEV)
        for t in grads + [acc]:
            _normal(t, gen, SIGMA)
            if pad is not None:
                t.index_fill_(0, pad, 0.0)
        parts = [_split(t, lens) for t in grads]
        dsts = _split(acc, lens)
        sched = None
        if case["issue"] == "thread":
            sched = hzp.Sched(plan, cls, gather_slots=1, queue_capacity=64, pool_bytes=-(-max(b["P"] for b in buckets) * 4 // 256) * 256)
            st["scheds"].append(sched)
        for n in reversed(range(len(buckets))):     # the backward pass goes from the last layer to the first
            st["reduces"].append((sched, buckets[n]["layer"], cls, hzp.ptr_array([p[n] for p in parts]), dsts[n].data_ptr()))
        st["keep"].append(grads)
        st["out"]["reduced_%d" % cls] = acc


def prepare(case, seed):
    case = dict(case)
    plan, n_layers = _plan(case)
    gen = _gen(seed)
    st = dict(case=case, plan=plan, n_layers=n_layers, out={}, keep=[], updates=[], post=[], shard_jobs=[], layers=[], params=[],
              reduces=[], scheds=[], shard3={}, stream={}, hyper=hzp.adamw_hyper(grad_scale=1.0 / case["R"], step=STEP, **ADAMW),
              s=torch.cuda.current_stream().cuda_stream)
    op = case["op"]
    if op in ("update", "step"):
        _prepare_update(case, st, gen, in_place=op == "step")
    if op in ("post_gather", "step"):
        _prepare_post_gather(case, st, gen)
    if op in ("layer_gather", "param_gather", "step"):
        _prepare_layer_gather(case, st, gen)
    if op == "reduce":
        _prepare_reduce(case, st, gen)
    torch.cuda.synchronize()
    return st


def run(st):
    case, plan, s = st["case"], st["plan"], st["s"]
    rank = case["rank"]
    for sched, layer, cls, grads, dst in st["reduces"]:
        gdt = hzp.HZP_GRAD_F32 if case["grads"] == "f32" else hzp.HZP_GRAD_BF16
        if sched is None:
            hzp.hzp_reduce_shard(plan, layer, cls, case["level"], rank, grads, 1.0 / case["R"], case["accumulate"], dst, stream=s,
                                 grad_dtype=gdt)
        else:
            sched.reduce(layer, case["level"], rank, grads, 1.0 / case["R"], case["accumulate"], dst, producer=s, grad_dtype=gdt)
    for sched in st["scheds"]:
        sched.join(s)
    for lo, hi, cls, R, grads, (master, m, v, out) in st["updates"]:
        hzp.hzp_adamw_shard(plan, lo, hi, cls, rank, st["hyper"], grads, R, master, m, v, out, stream=s)
    for cls, srcs, K, dsts in st["post"]:
        hzp.hzp_gather_layers(plan, 0, st["n_layers"], cls, 1, srcs, K, dsts, stream=s)
    for layer, cls, j, owners, dst in st["shard_jobs"]:
        hzp.hzp_gather_shard(plan, layer, cls, j, owners, dst, stream=s)
    for layer, cls, shards, bucket, tensors in st["layers"]:
        hzp.hzp_gather_layer(plan, layer, cls, 3, shards, bucket, tensors, stream=s)
    for t, shards, dst in st["params"]:
        hzp.hzp_gather_tensor(plan, t, shards, dst, stream=s)
    return st["out"]


# ------------------------------------------------------------------------------------------------ in 64 bits

def _exact_update(case, cls, buckets, gen):
    reduced = bool(case.get("reduced"))
    gtype = torch.float32 if reduced else _dtype(cls)
    n = sum(b["S1"] for b in buckets)
    R = 1 if reduced else case["R"]
    streams = [torch.empty(n, dtype=gtype, device=DEV) for _ in range(R)] + [torch.empty(n, dtype=torch.float32, device=DEV) for _ in range(3)]
    fill_update(case, cls, buckets, gen, streams)
    wd = torch.ones(n, device=DEV)
    at, i = 0, shard_of(case, 1)
    for b in buckets:
        lo, hi = i * b["S1"], (i + 1) * b["S1"]
        for o, k, mult in b["rows"]:
            if mult != 1.0 and max(o, lo) < min(o + k, hi):
                wd[at + max(o, lo) - lo:at + min(o + k, hi) - lo] = mult
        at += b["S1"]
    lr, b1, b2, eps, decay = (float(torch.tensor(ADAMW[k])) for k in ("lr", "beta1", "beta2", "eps", "weight_decay"))
    scale = float(torch.tensor(1.0 / case["R"]))
    outs = [torch.empty(n, dtype=torch.float64, device=DEV) for _ in range(3)]
    for lo in range(0, n, 1 << 26):
        hi = min(n, lo + (1 << 26))
        g = streams[0][lo:hi].double()
        for t in streams[1:R]:
            g += t[lo:hi].double()
        g *= scale
        p, m, v = (t[lo:hi].double() for t in streams[R:])
        m = b1 * m + (1 - b1) * g
        v = b2 * v + (1 - b2) * g * g
        u = (m / (1 - b1 ** STEP)) / ((v / (1 - b2 ** STEP)).sqrt() + eps)
        p = p - lr * (u + decay * wd[lo:hi].double() * p)
        for dst, x in zip(outs, (p, m, v)):
            dst[lo:hi] = x
    return outs


def exact(case, seed):
    case, gen, got = dict(case), _gen(seed), {}
    op, z1, z3 = case["op"], case["z1"], case["z3"]
    shard3 = {}
    if op in ("update", "step"):
        for cls, buckets in layout(case).items():
            p, m, v = _exact_update(case, cls, buckets, gen)
            got["class%d" % cls] = dict(master=p, m=m, v=v)
            if op == "update":
                got["class%d" % cls]["param"] = p
            else:
                got["class%d" % cls]["shard3"] = None       # filled by the gather below
                shard3[cls] = p
    if op in ("post_gather", "step"):
        j = shard_of(case, 3)
        for cls, buckets in layout(case).items():
            dt, rows = _dtype(cls), []
            if z1 % z3:
                for b in buckets:
                    first, last = j * b["S3"] // b["S1"], -(-(j + 1) * b["S3"] // b["S1"])
                    src = torch.empty((last - first) * b["S1"], dtype=dt, device=DEV)
                    fill_parameters(gen, src)
                    rows.append(src[j * b["S3"] - first * b["S1"]:][:b["S3"]])
                got["shard3_%d" % cls] = torch.cat(rows)
                continue
            K, n = z1 // z3, sum(b["S1"] for b in buckets)
            own = shard_of(case, 1) % K
            mine = shard3.get(cls)
            if mine is None:
                mine = torch.empty(n, dtype=dt, device=DEV)
                fill_parameters(gen, mine)
            recv = [torch.empty(n, dtype=dt, device=DEV) for _ in range(K - 1)]
            for t in recv:
                fill_parameters(gen, t)
            recv.insert(own, mine)
            parts = [_split(t.to(mine.dtype), [b["S1"] for b in buckets]) for t in recv]
            whole = [torch.cat([p[i] for p in parts]) for i in range(len(buckets))]
            if cls in shard3:
                shard3[cls] = whole
                got["class%d" % cls]["shard3"] = torch.cat(whole)
            else:
                got["shard3_%d" % cls] = torch.cat(whole)
    if op in ("layer_gather", "param_gather", "step"):
        j, out = shard_of(case, 3), case.get("out", "tensors")
        for cls, buckets in layout(case).items():
            n = sum(b["S3"] for b in buckets)
            parts = []
            for s in range(z3):
                if cls in shard3 and s == j:
                    parts.append(shard3[cls])
                    continue
                t = torch.empty(n, dtype=_dtype(cls), device=DEV)
                fill_parameters(gen, t)
                parts.append(_split(t, [b["S3"] for b in buckets]))
            kind = torch.float64 if cls in shard3 else _dtype(cls)
            whole = [torch.cat([p[i].to(kind) for p in parts]) for i in range(len(buckets))]
            if op != "param_gather" and out in ("bucket", "both"):
                got["bucket_%d" % cls] = torch.cat(whole)
            if op == "param_gather" or out in ("tensors", "both"):
                places, total = tensor_places(buckets)
                flat = torch.zeros(total, dtype=kind, device=DEV)
                for i, b in enumerate(buckets):
                    for at, (o, k, _) in zip(places[i], b["rows"]):
                        flat[at:at + k] = whole[i][o:o + k]
                got["tensors_%d" % cls] = flat
    if op == "reduce":
        gtype = torch.float32 if case["grads"] == "f32" else torch.bfloat16
        div = z1 if case["level"] == 1 else z3
        i = shard_of(case, case["level"])
        scale = float(torch.tensor(1.0 / case["R"]))
        for cls, buckets in layout(case).items():
            n = sum(b["P"] // div for b in buckets)
            pad = _padding(case, buckets, lambda b: i * (b["P"] // div), lambda b: b["P"] // div)
            total = torch.zeros(n, dtype=torch.float64, device=DEV)
            for r in range(case["R"] + 1):
                t = torch.empty(n, dtype=gtype if r < case["R"] else torch.float32, device=DEV)
                _normal(t, gen, SIGMA)
                if pad is not None:
                    t.index_fill_(0, pad, 0.0)
                if r < case["R"]:
                    total += t.double()
            total *= scale
            if case["accumulate"]:
                total += t.double()
            got["reduced_%d" % cls] = total
    return got
