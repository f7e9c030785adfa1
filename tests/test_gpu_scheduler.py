"""The asynchronous scheduler (background thread, dedicated streams, cyclic persistent pool):
results must equal the synchronous entry points' and the oracle's, bit for bit, whatever the
interleaving with a busy compute stream."""
import numpy as np
import pytest
import torch

import hzp_inputs
import paper_2510_20111_amd as hzp
from oracle import numeric as on
from oracle import planner as op

from gpu_util import DEV, assert_bf16_within_one_ulp, oracle_plan, to_dev, to_host
from test_gpu_parity import lib_plan, say

pytestmark = pytest.mark.gpu


class _DevView:
    """Zero-copy torch view of `n` int16 elements at a raw device address."""

    def __init__(self, ptr, n):
        self.__cuda_array_interface__ = {"shape": (n,), "typestr": "<i2", "data": (ptr, False), "version": 3}


def view16(ptr, n):
    return torch.as_tensor(_DevView(ptr, n), device=DEV)


def _layers(n_layers, seed):
    rng = np.random.default_rng(seed)
    numel = [int(x) for x in rng.integers(20000, 90000, size=n_layers)]
    desc = dict(tensors_per_layer=[1] * n_layers, tensor_numel=numel)
    oplan, plan = oracle_plan(desc, 8, 4, 8), lib_plan(desc, 8, 4, 8)
    shards = []
    for b in oplan["buckets"]:
        bucket = rng.integers(0, 1 << 16, size=b["P"], dtype=np.uint64).astype(np.uint16)
        shards.append([np.ascontiguousarray(bucket[j * b["S3"]:(j + 1) * b["S3"]]) for j in range(4)])
    return oplan, plan, shards


def test_prefetch_pipeline_through_a_two_slot_pool():
    say("scheduler: prefetch pipeline")
    n_layers = 9
    oplan, plan, shards = _layers(n_layers, 50)
    dshards = [[to_dev(s) for s in layer] for layer in shards]
    sched = hzp.Sched(plan, gather_slots=2, queue_capacity=4)
    consumer = torch.cuda.Stream()
    busy = torch.randn(2048, 2048, device=DEV)
    outs = [torch.zeros(oplan["buckets"][l]["P"], dtype=torch.int16, device=DEV) for l in range(n_layers)]
    torch.cuda.synchronize()
    sched.prefetch(0, dshards[0])
    sched.prefetch(1, dshards[1])
    for l in range(n_layers):
        with torch.cuda.stream(consumer):
            busy = busy @ busy * 1e-3                 # keeps the compute stream behind the gathers
        ptr = sched.acquire(l, consumer)
        with torch.cuda.stream(consumer):
            outs[l].copy_(view16(ptr, outs[l].numel()))
        sched.release(l, consumer)
        if l + 2 < n_layers:
            sched.prefetch(l + 2, dshards[l + 2])
    consumer.synchronize()
    sched.drain()
    for l in range(n_layers):
        want = on.gather_concat(shards[l])
        assert np.array_equal(to_host(outs[l], np.uint16), want), l
    st = sched.stats()
    assert st.gathers_issued == n_layers and st.peak_live_slots == 2
    assert st.pool_bytes == 2 * st.slot_bytes
    assert st.slot_bytes >= 2 * max(b["P"] for b in oplan["buckets"])
    assert st.peak_live_bytes <= st.pool_bytes
    sched.destroy()


def test_protocol_errors_and_back_pressure():
    say("scheduler: protocol errors")
    oplan, plan, shards = _layers(4, 51)
    dshards = [[to_dev(s) for s in layer] for layer in shards]
    sched = hzp.Sched(plan, gather_slots=2, queue_capacity=8)

    def status(fn, *a):
        with pytest.raises(hzp.HzpError) as e:
            fn(*a)
        return e.value.status

    assert status(sched.acquire, 0) == hzp.HZP_ERR_INVALID_ARG          # never prefetched
    assert status(sched.prefetch, 9, dshards[0]) == hzp.HZP_ERR_RANGE
    assert status(sched.prefetch, 0, dshards[0][:3]) == hzp.HZP_ERR_INVALID_ARG
    sched.prefetch(0, dshards[0])
    assert status(sched.prefetch, 0, dshards[0]) == hzp.HZP_ERR_INVALID_ARG   # already in the pool
    sched.prefetch(1, dshards[1])
    assert status(sched.prefetch, 2, dshards[2]) == hzp.HZP_ERR_NOMEM         # pool full: back pressure
    assert status(sched.release, 0) == hzp.HZP_ERR_INVALID_ARG                # not acquired yet
    sched.acquire(0)
    assert status(sched.acquire, 0) == hzp.HZP_ERR_INVALID_ARG
    sched.acquire(1)
    sched.release(1)                                                          # out of order ...
    assert status(sched.prefetch, 2, dshards[2]) == hzp.HZP_ERR_NOMEM         # ... the cycle's next slot is layer 0's
    sched.release(0)
    sched.prefetch(2, dshards[2])
    ptr = sched.acquire(2)
    torch.cuda.synchronize()
    sched.drain()
    got = to_host(view16(ptr, oplan["buckets"][2]["P"]).clone(), np.uint16)
    assert np.array_equal(got, on.gather_concat(shards[2]))
    sched.release(2)
    # a refused reduction leaves the scheduler usable (it is refused at submission, not on the thread)
    g = [torch.zeros(64, dtype=torch.int16, device=DEV)]
    out = torch.zeros(64, device=DEV)
    assert status(sched.reduce, 0, 4, 0, g, 1.0, False, out) == hzp.HZP_ERR_RANGE            # level
    assert status(sched.reduce, 0, 3, 99, g, 1.0, False, out) == hzp.HZP_ERR_RANGE           # rank
    assert status(sched.reduce, 0, 3, 0, [g[0][1:]], 1.0, False, out) == hzp.HZP_ERR_ALIGN
    assert status(sched.reduce, 0, 3, 0, g, 1.0, False, out[1:]) == hzp.HZP_ERR_ALIGN
    sched.prefetch(3, dshards[3])
    ptr = sched.acquire(3)
    sched.drain()
    assert np.array_equal(to_host(view16(ptr, oplan["buckets"][3]["P"]).clone(), np.uint16), on.gather_concat(shards[3]))
    sched.release(3)
    assert sched.stats().reduces_issued == 0
    sched.destroy()
    with pytest.raises(hzp.HzpError):
        hzp.Sched(plan, gather_slots=0)


def test_hungry_reduce_after_the_producer_and_join():
    say("scheduler: hungry reduce")
    oplan, plan, _ = _layers(3, 52)
    R, rank = 4, 5
    rng = np.random.default_rng(53)
    sched = hzp.Sched(plan, gather_slots=1, queue_capacity=16)
    producer, consumer = torch.cuda.Stream(), torch.cuda.Stream()
    host, dev, outs = [], [], []
    busy = torch.randn(2048, 2048, device=DEV)
    for layer, b in enumerate(oplan["buckets"]):
        _, n = op.shard_range(oplan, b, 3, rank)
        g = [hzp_inputs.to_bf16_bits((rng.standard_normal(n) * 1e-3).astype(np.float32)) for _ in range(R)]
        host.append(g)
        staged = [to_dev(x) for x in g]
        slices = [torch.zeros(n, dtype=torch.int16, device=DEV) for _ in range(R)]
        out = torch.full((n,), 3.0, device=DEV)
        dev.append((staged, slices))
        outs.append(out)
    torch.cuda.synchronize()
    want = [on.reduce(host[layer], scale=0.25) for layer in range(3)]
    rounds = 12     # the reductions run beside a busy compute stream; repeat to vary the interleaving
    for rnd in range(rounds):
        for layer in range(3):
            staged, slices = dev[layer]
            with torch.cuda.stream(producer):
                busy = busy @ busy * 1e-3             # the "backward pass" that produces the gradients
                for dst, src in zip(slices, staged):
                    dst.zero_()
                    dst.copy_(src)
            sched.reduce(layer, 3, rank, slices, 0.25, False, outs[layer], producer)
        sched.join(consumer)
        with torch.cuda.stream(consumer):
            copies = [o.clone() for o in outs]
            for o in outs:
                o.fill_(3.0)
        consumer.synchronize()
        producer.wait_stream(consumer)
        for layer in range(3):
            got = to_host(copies[layer], np.float32)
            bad = np.nonzero(got.view(np.uint32) != want[layer].view(np.uint32))[0]
            assert bad.size == 0, (rnd, layer, bad.size, bad[:8].tolist(), got[bad[:8]].tolist(),
                                   want[layer][bad[:8]].tolist())
    assert sched.stats().reduces_issued == 3 * rounds
    sched.destroy()


def test_ring_pool_with_layers_of_different_sizes():
    """Buckets of very different sizes move through a ring that is smaller than three of the largest.
    Checked without a model of the ring's arithmetic: every bucket arrives intact; regions that are
    live at the same time never overlap; all regions lie inside one window of pool_bytes; the live
    bytes never exceed the pool; a full pool refuses with NOMEM and an empty one always accepts."""
    say("scheduler: ring pool, ragged layers")
    rng = np.random.default_rng(60)
    n_layers = 14
    numel = [int(x) for x in rng.choice([3000, 20000, 90000, 150000], size=n_layers)]
    numel[0], numel[5] = 150000, 150000
    desc = dict(tensors_per_layer=[1] * n_layers, tensor_numel=numel)
    oplan, plan = oracle_plan(desc, 8, 4, 8), lib_plan(desc, 8, 4, 8)
    shards, dshards = [], []
    for b in oplan["buckets"]:
        bucket = rng.integers(0, 1 << 16, size=b["P"], dtype=np.uint64).astype(np.uint16)
        shards.append([np.ascontiguousarray(bucket[j * b["S3"]:(j + 1) * b["S3"]]) for j in range(4)])
        dshards.append([to_dev(s) for s in shards[-1]])
    sizes = [2 * b["P"] for b in oplan["buckets"]]
    cap = 2 * ((max(sizes) + 255) // 256 * 256) + 4096
    slots = 4
    sched = hzp.Sched(plan, gather_slots=slots, queue_capacity=8, pool_bytes=cap)
    consumer = torch.cuda.Stream()
    outs = [torch.zeros(b["P"], dtype=torch.int16, device=DEV) for b in oplan["buckets"]]
    torch.cuda.synchronize()
    pending, held = [], []          # prefetched but not acquired; acquired: (layer, address, bytes)
    seen, nxt, refusals = [], 0, 0

    def prefetch_all_it_takes():
        nonlocal nxt, refusals
        while nxt < n_layers:
            try:
                sched.prefetch(nxt, dshards[nxt], consumer)
            except hzp.HzpError as e:
                assert e.status == hzp.HZP_ERR_NOMEM
                assert pending or held, "an empty pool refused a region that fits"
                refusals += 1
                return
            pending.append(nxt)
            nxt += 1
            assert len(pending) + len(held) <= slots

    prefetch_all_it_takes()
    while pending or held:
        # acquire everything that is prefetched: all of these regions are live at the same time
        while pending:
            l = pending.pop(0)
            ptr = sched.acquire(l, consumer)
            held.append((l, ptr, sizes[l]))
            seen.append((ptr, sizes[l]))
        for i, (la, pa, na) in enumerate(held):
            for lb, pb, nb in held[i + 1:]:
                assert pa + na <= pb or pb + nb <= pa, "regions of layers %d and %d overlap" % (la, lb)
        assert sum(n for _, _, n in held) <= cap
        lo, hi = min(p for p, _ in seen), max(p + n for p, n in seen)
        assert hi - lo <= cap, "regions span more than the pool"
        # use and give back the oldest one (two at times, so that the number of live regions varies)
        for _ in range(2 if len(held) > 2 and held[0][0] % 3 == 0 else 1):
            l, ptr, _ = held.pop(0)
            with torch.cuda.stream(consumer):
                outs[l].copy_(view16(ptr, outs[l].numel()))
            sched.release(l, consumer)
        prefetch_all_it_takes()
    consumer.synchronize()
    sched.drain()
    for l in range(n_layers):
        assert np.array_equal(to_host(outs[l], np.uint16), on.gather_concat(shards[l])), l
    st = sched.stats()
    assert st.pool_bytes == cap and st.gathers_issued == n_layers
    assert st.peak_live_bytes <= cap and 2 <= st.peak_live_slots <= slots
    assert refusals > 0                                     # the pool did fill up
    # space is lost only where a region does not fit before the end of the buffer: less than one
    # region each time, and not more often than regions were placed
    assert 0 < st.wrap_skipped_bytes < n_layers * max(sizes)
    sched.destroy()


def test_prefetch_right_behind_the_update_without_a_host_wait():
    """Section 4.1.2: the optimizer step writes the new bf16 parameters into the rank's piece of the
    ZeRO-3 shard and the next step's prefetch is issued at once.  The update sits behind a long
    kernel on the compute stream when the prefetch is queued; the gather must wait for it through the
    producer's event alone (no host synchronisation anywhere)."""
    say("scheduler: prefetch ordered behind the producer stream")
    desc = dict(tensors_per_layer=[2, 2], tensor_numel=[50000, 30000, 70000, 10000])
    z3, z1, R = 2, 4, 2
    oplan, plan = oracle_plan(desc, 8, z3, z1), lib_plan(desc, 8, z3, z1)
    rank = 3                                    # j = 1, k = 1
    j, k, i = plan.rank(rank)
    hp = hzp_inputs.ADAMW
    hy = hzp.adamw_hyper(hp["lr"], hp["beta1"], hp["beta2"], hp["eps"], hp["weight_decay"], 1.0 / R, 1)
    rng = np.random.default_rng(70)
    compute = torch.cuda.Stream()
    sched = hzp.Sched(plan, gather_slots=2, queue_capacity=8)
    busy = torch.randn(4096, 4096, device=DEV)
    host, dev = [], []
    for layer, b in enumerate(oplan["buckets"]):
        beg, n = op.shard_range(oplan, b, 1, rank)
        g = [hzp_inputs.to_bf16_bits((rng.standard_normal(n) * 1e-3).astype(np.float32)) for _ in range(R)]
        p = (rng.standard_normal(n) * 0.02).astype(np.float32)
        other = [rng.integers(0, 1 << 16, size=b["S3"], dtype=np.uint64).astype(np.uint16) for _ in range(z3)]
        dsh = [to_dev(o) for o in other]            # shard j holds stale values where the update will write
        host.append(dict(g=g, p=p, other=other, S1=b["S1"], S3=b["S3"], P=b["P"]))
        dev.append(dict(g=[to_dev(x) for x in g], p=to_dev(p), m=torch.zeros(n, device=DEV), v=torch.zeros(n, device=DEV),
                        shards=dsh, out=dsh[j][k * b["S1"]:(k + 1) * b["S1"]]))
    torch.cuda.synchronize()
    with torch.cuda.stream(compute):
        for _ in range(30):
            busy = busy @ busy * 1e-3           # the update below is queued behind this
    hzp.hzp_adamw_shard(plan, 0, 2, 0, rank, hy, [x for d in dev for x in d["g"]], R, [d["p"] for d in dev],
                        [d["m"] for d in dev], [d["v"] for d in dev], [d["out"] for d in dev], stream=compute)
    ptrs = [x for d in dev for x in d["shards"]]
    assert sched.prefetch_ahead(0, 2, ptrs, z3, compute) == 2       # queued at once, ordered by the event
    got = []
    for layer in range(2):
        ptr = sched.acquire(layer, compute)
        with torch.cuda.stream(compute):
            got.append(view16(ptr, host[layer]["P"]).clone())
        sched.release(layer, compute)
    compute.synchronize()
    sched.drain()
    for layer, h in enumerate(host):
        want16 = on.adamw(on.reduce(h["g"], scale=1.0 / R), h["p"].copy(), np.zeros_like(h["p"]), np.zeros_like(h["p"]),
                          step=1, **hp)
        shards = [o.copy() for o in h["other"]]
        bucket = to_host(got[layer], np.uint16)
        mine = bucket[j * h["S3"] + k * h["S1"]:j * h["S3"] + (k + 1) * h["S1"]]
        # the piece written by the update: the oracle's cast parameters within one bf16 ulp
        big = np.abs(h["p"]) > 1e-4         # away from zero one bf16 ulp is far wider than the fp32 tolerance
        assert_bf16_within_one_ulp(mine[big], want16[big], "layer %d: piece written by the update" % layer)
        assert not np.array_equal(mine, shards[j][k * h["S1"]:(k + 1) * h["S1"]])   # not the stale values
        shards[j][k * h["S1"]:(k + 1) * h["S1"]] = mine
        assert np.array_equal(bucket, on.gather_concat(shards)), layer
    sched.destroy()


def test_prefetch_ahead_fills_the_pool_and_the_turn_from_forward_to_backward():
    """Section 4.1.2: prefetch as far ahead as the memory allows; at the end of the forward pass the
    last layer's parameters, released after their use, are gathered again for the backward pass."""
    say("scheduler: prefetch ahead and the forward/backward turn")
    n_layers = 6
    oplan, plan, shards = _layers(n_layers, 54)
    dshards = [[to_dev(s) for s in layer] for layer in shards]
    flat = [x for layer in dshards for x in layer]
    slots = 3
    sched = hzp.Sched(plan, gather_slots=slots, queue_capacity=8)
    consumer = torch.cuda.Stream()
    torch.cuda.synchronize()
    seen = []

    def use(l):
        ptr = sched.acquire(l, consumer)
        with torch.cuda.stream(consumer):
            seen.append((l, view16(ptr, oplan["buckets"][l]["P"]).clone()))
        sched.release(l, consumer)

    # forward: layers 0..5, the pool holds three
    nxt = sched.prefetch_ahead(0, n_layers, flat, 4, consumer)
    assert nxt == slots
    assert sched.prefetch_ahead(nxt, n_layers - nxt, flat[4 * nxt:], 4, consumer) == 0      # full: nothing more, no error
    for l in range(n_layers):
        use(l)
        if nxt < n_layers:
            nxt += sched.prefetch_ahead(nxt, 1, flat[4 * nxt:], 4, consumer)
    assert nxt == n_layers
    # the turn: layer 5 was released; backward needs 5, 4, 3, ... again
    order = list(range(n_layers - 1, -1, -1))
    issued = 0
    for l in order[:slots]:
        sched.prefetch(l, dshards[l], consumer)
        issued += 1
    for idx, l in enumerate(order):
        use(l)
        if issued < n_layers:
            sched.prefetch(order[issued], dshards[order[issued]], consumer)
            issued += 1
    consumer.synchronize()
    sched.drain()
    assert [l for l, _ in seen] == list(range(n_layers)) + order
    for l, t in seen:
        assert np.array_equal(to_host(t, np.uint16), on.gather_concat(shards[l])), l
    st = sched.stats()
    assert st.gathers_issued == 2 * n_layers and st.peak_live_slots == slots
    with pytest.raises(hzp.HzpError) as e:
        sched.prefetch_ahead(4, 5, flat, 4, consumer)
    assert e.value.status == hzp.HZP_ERR_RANGE
    sched.destroy()


def test_prefetch_one_parameter_at_a_time():
    """The paper's granularity: every tensor of a plan prefetched, acquired and released on its own,
    three ahead, through a ring much smaller than a layer."""
    say("scheduler: per-parameter prefetch")
    desc = hzp_inputs.irregular_desc(30, seed=61, max_numel=40000, tensors_per_layer=6, f32_every=0)
    desc = dict(desc, tensor_class=None, tensor_wd_mult=None)
    z3 = 4
    oplan, plan = oracle_plan(desc, 8, z3, 8), lib_plan(desc, 8, z3, 8)
    rng = np.random.default_rng(62)
    shards, dshards = {}, {}
    for bi, b in enumerate(oplan["buckets"]):
        bucket = rng.integers(0, 1 << 16, size=b["P"], dtype=np.uint64).astype(np.uint16)
        shards[bi] = [np.ascontiguousarray(bucket[j * b["S3"]:(j + 1) * b["S3"]]) for j in range(z3)]
        dshards[bi] = [to_dev(s) for s in shards[bi]]
    n_t = len(oplan["tensors"])
    biggest = max(t["numel"] for t in oplan["tensors"])
    sched = hzp.Sched(plan, gather_slots=3, queue_capacity=8, pool_bytes=(3 * 2 * biggest + 255) // 256 * 256 + 512)
    consumer = torch.cuda.Stream()
    outs = [torch.zeros(t["numel"], dtype=torch.int16, device=DEV) for t in oplan["tensors"]]
    torch.cuda.synchronize()

    def ptrs_of(t):
        rec = oplan["tensors"][t]
        b = oplan["buckets"][rec["bucket"]]
        j0, j1 = rec["offset"] // b["S3"], (rec["offset"] + rec["numel"] - 1) // b["S3"]
        return [dshards[rec["bucket"]][j] if j0 <= j <= j1 else None for j in range(z3)]

    for t in range(3):
        sched.prefetch_tensor(t, ptrs_of(t))
    with pytest.raises(hzp.HzpError) as e:
        sched.prefetch_tensor(3, ptrs_of(3))
    assert e.value.status == hzp.HZP_ERR_NOMEM                      # three regions are live
    with pytest.raises(hzp.HzpError) as e:
        sched.acquire(0)                                            # layer 0 was never prefetched, tensor 0 was
    assert e.value.status == hzp.HZP_ERR_INVALID_ARG
    for t in range(n_t):
        ptr = sched.acquire_tensor(t, consumer)
        with torch.cuda.stream(consumer):
            outs[t].copy_(view16(ptr, outs[t].numel()))
        sched.release_tensor(t, consumer)
        if t + 3 < n_t:
            sched.prefetch_tensor(t + 3, ptrs_of(t + 3))
    consumer.synchronize()
    sched.drain()
    for t in range(n_t):
        rec = oplan["tensors"][t]
        want = on.unpack_tensor(shards[rec["bucket"]], rec["offset"], rec["numel"])
        assert np.array_equal(to_host(outs[t], np.uint16), want), t
    st = sched.stats()
    assert st.gathers_issued == n_t and st.peak_live_slots == 3
    sched.destroy()


def test_a_layers_parameters_with_one_call_each():
    """Parameter granularity (one gather and one pool region per tensor) driven with one prefetch, one
    acquire and one release per layer, two layers ahead, through a ring that wraps inside layers; mixed
    with the one-tensor calls on one layer; all-or-nothing back-pressure."""
    say("scheduler: a layer's parameters with one call each")
    desc = hzp_inputs.irregular_desc(42, seed=71, max_numel=60000, tensors_per_layer=6, f32_every=0)
    desc = dict(desc, tensor_class=None, tensor_wd_mult=None)
    z3 = 4
    oplan, plan = oracle_plan(desc, 8, z3, 8), lib_plan(desc, 8, z3, 8)
    rng = np.random.default_rng(72)
    shards, dshards = {}, {}
    for bi, b in enumerate(oplan["buckets"]):
        bucket = rng.integers(0, 1 << 16, size=b["P"], dtype=np.uint64).astype(np.uint16)
        shards[bi] = [np.ascontiguousarray(bucket[j * b["S3"]:(j + 1) * b["S3"]]) for j in range(z3)]
        dshards[bi] = [to_dev(s) for s in shards[bi]]
    n_layers = oplan["n_layers"]
    ids = [op.find_bucket(oplan, l, 0)["tensor_ids"] for l in range(n_layers)]
    layer_bytes = [sum((2 * oplan["tensors"][t]["numel"] + 255) // 256 * 256 for t in ids[l]) for l in range(n_layers)]
    # room for two and a half of the largest layers: the ring wraps in the middle of layers
    pool = (5 * max(layer_bytes) // 2 + 255) // 256 * 256
    sched = hzp.Sched(plan, gather_slots=12, queue_capacity=16, pool_bytes=pool)
    consumer = torch.cuda.Stream()
    outs = [torch.zeros(t["numel"], dtype=torch.int16, device=DEV) for t in oplan["tensors"]]
    torch.cuda.synchronize()
    sched.prefetch_params(0, dshards[0])
    sched.prefetch_params(1, dshards[1])
    with pytest.raises(hzp.HzpError) as e:
        sched.prefetch_params(2, dshards[2])                        # 12 regions are live: nothing of layer 2 is taken
    assert e.value.status == hzp.HZP_ERR_NOMEM
    assert sched.stats().peak_live_slots == 12
    with pytest.raises(hzp.HzpError) as e:
        sched.prefetch_params(1, dshards[1])                        # already in the pool
    assert e.value.status == hzp.HZP_ERR_INVALID_ARG
    with pytest.raises(hzp.HzpError) as e:
        sched.release_params(0, consumer)                           # not acquired yet
    assert e.value.status == hzp.HZP_ERR_INVALID_ARG
    for l in range(n_layers):
        if l == 3:                                                  # this layer one tensor at a time
            ptrs = [sched.acquire_tensor(t, consumer) for t in ids[l]]
        else:
            ptrs = sched.acquire_params(l, len(ids[l]), consumer)
        with torch.cuda.stream(consumer):
            for t, ptr in zip(ids[l], ptrs):
                outs[t].copy_(view16(ptr, outs[t].numel()))
        if l == 4:
            for t in ids[l]:
                sched.release_tensor(t, consumer)
        else:
            sched.release_params(l, consumer)
        if l + 2 == 5:                                              # one by one and backwards: acquired together all the same
            for t in reversed(ids[5]):
                sched.prefetch_tensor(t, dshards[5])
        elif l + 2 < n_layers:
            sched.prefetch_params(l + 2, dshards[l + 2])
    consumer.synchronize()
    sched.drain()
    for t, rec in enumerate(oplan["tensors"]):
        want = on.unpack_tensor(shards[rec["bucket"]], rec["offset"], rec["numel"])
        assert np.array_equal(to_host(outs[t], np.uint16), want), t
    st = sched.stats()
    assert st.gathers_issued == len(oplan["tensors"]) and st.peak_live_slots == 12
    assert st.wrap_skipped_bytes > 0                                # the ring did wrap
    sched.destroy()


@pytest.mark.parametrize("order", ["grgr", "rrgn", "nrng", "gnrb", "bnnb"])
def test_join_after_gathers_reductions_or_neither(order):
    """Joins after a gather (g), a reduction (r), both (b) or nothing new (n): what ran before each, on either stream, is there for the
    consumer, which copies it without any other wait; several consumers in turn."""
    say("scheduler: join after " + order)
    oplan, plan, shards = _layers(2, 53)
    dshards = [[to_dev(s) for s in layer] for layer in shards]
    lens = [b["P"] for b in oplan["buckets"]]
    sched = hzp.Sched(plan, gather_slots=2, queue_capacity=8)
    producer, consumers = torch.cuda.Stream(), [torch.cuda.Stream(), torch.cuda.Stream()]
    busy = torch.randn(2048, 2048, device=DEV)
    n = oplan["buckets"][0]["S3"]
    grads = [torch.full((n,), float(k + 1), device=DEV) for k in range(2)]
    acc = torch.zeros(n, device=DEV)
    torch.cuda.synchronize()
    reduced = 0
    for i, what in enumerate(order):
        consumer, layer = consumers[i % 2], i % 2
        with torch.cuda.stream(producer):
            busy = busy @ busy * 1e-3                 # keeps what follows pending
        if what in "gb":
            sched.prefetch(layer, dshards[layer], producer)
        if what in "rb":
            sched.reduce(0, 3, 0, grads, 1.0, True, acc, producer, grad_dtype=hzp.HZP_GRAD_F32)
            reduced += 1
        sched.join(consumer)
        with torch.cuda.stream(consumer):
            seen = acc.clone()
        if what in "gb":
            ptr = sched.acquire(layer, consumer)
            with torch.cuda.stream(consumer):
                got = view16(ptr, lens[layer]).clone()
            sched.release(layer, consumer)
        consumer.synchronize()
        assert torch.equal(seen, torch.full_like(seen, 3.0 * reduced)), i
        if what in "gb":
            assert np.array_equal(to_host(got, np.uint16), on.gather_concat(shards[layer])), i
        producer.wait_stream(consumer)                # the next reduction writes what this consumer has read
    sched.drain()
    sched.destroy()
