"""The forms one update, reduction or post-step gather can be launched in, against the CPU oracle: segments merged, listed
with pointers of their own or sharing one set, found by a 2-D grid or by search, decay constant or looked up; every
number of contributions; sizes at the edges of a group of 256 elements and of a block of 16 groups."""
import numpy as np
import pytest
import torch

import hzp_inputs
import paper_2510_20111_amd as hzp
from oracle import numeric as on
from oracle import planner as op

from gpu_util import DEV, REL_TOL, RMS_FLOOR, U_ERR, assert_cast_of, assert_close_f32, launches_of, oracle_plan, to_dev, to_host, wd_mult_array

pytestmark = pytest.mark.gpu

HP = hzp_inputs.ADAMW
EDGES = [8, 248, 256, 264, 15 * 256 + 8, 16 * 256, 16 * 256 + 8, 33 * 256 - 8]


def carve(sizes, dtype, place):
    """Buffers of the given lengths: each alone ("own"), back to back in one allocation ("packed"), or at equal
    distances in one allocation, in ascending ("spread") or descending ("down") order of address."""
    if place == "own":
        return [torch.zeros(n, dtype=dtype, device=DEV) for n in sizes]
    if place == "packed":
        return list(torch.split(torch.zeros(sum(sizes), dtype=dtype, device=DEV), sizes))
    step = max(sizes) + 264
    whole = torch.zeros(step * len(sizes), dtype=dtype, device=DEV)
    at = [k * step for k in range(len(sizes))]
    return [whole[a:a + n] for a, n in zip(at if place == "spread" else at[::-1], sizes)]


def update_against_oracle(desc, align, z1, R, rank, cls, place, out_place=None, split=False, seed=3):
    """One update of class `cls` over all layers (or call by call) from random states, compared with the oracle."""
    oplan = oracle_plan(desc, align, 1, z1)
    plan = hzp.hzp_plan(desc["tensors_per_layer"], desc["tensor_numel"], align, 1, z1,
                        tensor_class=desc.get("tensor_class"), tensor_wd_mult=desc.get("tensor_wd_mult"))
    buckets = [b for b in oplan["buckets"] if b["cls"] == cls]
    sizes = [b["S1"] for b in buckets]
    rng = np.random.default_rng(seed)
    g16 = cls == 0
    grads = [[rng.standard_normal(n, dtype=np.float32) * np.float32(1e-3) for _ in range(R)] for n in sizes]
    if g16:
        grads = [[hzp_inputs.to_bf16_bits(g) for g in per] for per in grads]
    p, m = ([rng.standard_normal(n, dtype=np.float32) * np.float32(s) for n in sizes] for s in (0.02, 1e-4))
    v = [np.square(rng.standard_normal(n, dtype=np.float32)) * np.float32(1e-7) for n in sizes]
    dev_g = [carve(sizes, torch.int16 if g16 else torch.float32, place) for _ in range(R)]
    dev = [carve(sizes, torch.float32, place) for _ in range(3)]
    out = carve(sizes, torch.int16 if g16 else torch.float32, out_place or place)
    for i in range(len(sizes)):
        for r in range(R):
            dev_g[r][i].copy_(to_dev(grads[i][r]))
        for d, h in zip(dev, (p, m, v)):
            d[i].copy_(to_dev(h[i]))
    hy = hzp.adamw_hyper(HP["lr"], HP["beta1"], HP["beta2"], HP["eps"], HP["weight_decay"], 1.0 / R, 3)
    at = {b["layer"]: i for i, b in enumerate(buckets)}
    flat = lambda lists, lo, hi: [lists[at[layer]] if layer in at else 0 for layer in range(lo, hi)]  # noqa: E731
    spans = [(0, oplan["n_layers"])] if not split else [(k, k + 1) for k in sorted(at)]
    for lo, hi in spans:
        gl = [dev_g[r][at[layer]] if layer in at else 0 for layer in range(lo, hi) for r in range(R)]
        hzp.hzp_adamw_shard(plan, lo, hi, cls, rank, hy, gl, R, *(flat(d, lo, hi) for d in dev), flat(out, lo, hi))
    torch.cuda.synchronize()
    got = [[to_host(d[i], np.float32) for i in range(len(sizes))] for d in dev]
    for i, b in enumerate(buckets):
        beg, n = op.shard_range(oplan, b, 1, rank)
        wd = wd_mult_array(oplan, b, beg, n) if desc.get("tensor_wd_mult") else None
        on.adamw(on.reduce(grads[i], scale=1.0 / R), p[i], m[i], v[i], step=3, wd_mult=wd, out_bf16=g16, **HP)
        tag = "%s R=%d layer %d n=%d" % (place, R, b["layer"], n)
        for key, have, want in zip("pmv", got, (p[i], m[i], v[i])):
            assert_close_f32(have[i], want, tag + " " + key, key)
        if g16:
            assert_cast_of(to_host(out[i], np.uint16), got[0][i], tag + " out")
        else:
            assert np.array_equal(to_host(out[i], np.uint32), got[0][i].view(np.uint32)), tag + " out"
    return got


@pytest.mark.parametrize("R", range(1, 33))
@pytest.mark.parametrize("cls", [0, 1])
def test_every_number_of_contributions_at_group_edges(R, cls):
    """Segments of unlike length in one call (found by search) and call by call (one segment each): the same bits."""
    print("R=%d class %d" % (R, cls), flush=True)
    desc = dict(tensors_per_layer=[1] * len(EDGES), tensor_numel=EDGES, tensor_class=[cls] * len(EDGES))
    a = update_against_oracle(desc, 8, 1, R, 0, cls, "own")
    b = update_against_oracle(desc, 8, 1, R, 0, cls, "own", split=True)
    for x, y in zip(a, b):
        assert all(np.array_equal(s.view(np.uint32), t.view(np.uint32)) for s, t in zip(x, y))


@pytest.mark.parametrize("cls,R,groups", [(0, R, g) for R in (6, 7, 8) for g in ((32769,), (65536,), (32768, 32768), (60000, 5536), (10241, 10240), (18000, 2481))] +
                         [(0, R, g) for R in (6, 7, 8) for g in ((65537,), (32769, 32768), (60000, 6000))] +
                         [(0, R, g) for R in (5, 8, 9, 16, 28, 29) for g in ((20481,), (10241, 10240), (18000, 2481))] +
                         [(0, R, (g,)) for R, g in ((5, 20481), (6, 20481), (9, 24577), (12, 24577), (13, 20481), (28, 20481))] +
                         [(1, R, g) for R in (4, 7, 16, 17) for g in ((10241,), (5121, 5120), (9000, 1241))] +
                         [(1, R, (g,)) for R, g in ((4, 24577), (7, 16385), (8, 16385), (10, 10241), (16, 10241))])
def test_long_launches_and_their_quarters(cls, R, groups):
    """Launches at the lengths where the number of contributions at a time changes, and the same elements in calls of a quarter of each
    segment: the same bits (one segment, segments of like length, and found by search; the last group is not full)."""
    sizes = [g * 256 - 8 for g in groups]
    total = sum(sizes)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(R)
    dtype, bits = (torch.float32, torch.int32) if cls else (torch.bfloat16, torch.int16)
    grads = [torch.empty(total, device=DEV).normal_(0, 1e-3, generator=gen).to(dtype) for _ in range(R)]
    start = [torch.empty(total, device=DEV).normal_(0, s, generator=gen) for s in (0.02, 1e-4, 1e-4)]
    start[2].square_()
    hy = hzp.adamw_hyper(HP["lr"], HP["beta1"], HP["beta2"], HP["eps"], HP["weight_decay"], 1.0 / R, 3)
    results = []
    for parts in (1, 4):            # one call over the segments; a call for each quarter of each
        at, spans = 0, []
        for n in sizes:
            q = n // parts // 8 * 8
            spans += [(at + k * q, q if k + 1 < parts else n - k * q) for k in range(parts)]
            at += n
        plan = hzp.hzp_plan([1] * len(spans), [n for _, n in spans], 8, 1, 1, tensor_class=[cls] * len(spans))
        apart = parts == 1 and len(spans) > 1       # copies that do not follow each other, so that they stay segments
        def views(t):
            return [t[a:a + n].clone() if apart else t[a:a + n] for a, n in spans]
        g = [views(t) for t in grads]
        s = [views(t.clone()) for t in start]
        o = views(torch.zeros(total, dtype=dtype, device=DEV))
        calls = [(0, len(spans))] if parts == 1 else [(k, k + 1) for k in range(len(spans))]
        for lo, hi in calls:
            hzp.hzp_adamw_shard(plan, lo, hi, cls, 0, hy, [g[r][k] for k in range(lo, hi) for r in range(R)], R, *(x[lo:hi] for x in s), o[lo:hi])
        torch.cuda.synchronize()
        results.append([torch.cat(x) for x in s] + [torch.cat(o)])
    for a, b in zip(*results):
        assert torch.equal(a.view(bits if a.dtype == dtype else torch.int32), b.view(bits if b.dtype == dtype else torch.int32))
    assert not torch.equal(results[0][0], start[0])


def larger_chunks_from(cls, R, one):
    """Longest launch, in groups, in small chunks (one segment, or several), or None where a longer one has the same."""
    if cls:
        return None if R <= 3 or R in (5, 6, 9) or R > 16 else 24576 if one and R == 4 else 16384 if one and R <= 9 else 10240
    return None if R <= 4 else 32768 if one and R in (7, 8) else 24576 if one and 9 <= R <= 12 else 20480


@pytest.mark.parametrize("cls,R", [(0, R) for R in range(1, 33)] + [(1, R) for R in range(1, 33)])
def test_the_number_of_contributions_at_a_time_follows_the_length(cls, R):
    """One segment: the launches on the two sides of each limit have different kernels, and those within it the same."""
    limit = larger_chunks_from(cls, R, True)
    kernel = [update_launches(groups, cls, R)[0][2] for groups in (2049, limit or 24577, (limit or 24577) + 1)]
    assert kernel[0] == kernel[1] and (kernel[1] != kernel[2]) == (limit is not None)
    if not cls and 5 < R <= 8:          # in one chunk between the limits
        assert update_launches(65536, cls, R)[0][2] == kernel[2] and update_launches(65537, cls, R)[0][2] == kernel[1]


@pytest.mark.parametrize("cls,R", [(0, 1), (0, 2), (1, 1), (0, 0)])
@pytest.mark.parametrize("groups", [3073, 4000, 5120])
def test_updates_with_a_pause_between_their_requests(cls, R, groups):
    """One segment whose wavefronts are 12 to 20 to a CU has a kernel of its own; the bits are those of its two halves, which have not
    (R = 0: from an already reduced fp32 shard)."""
    n = groups * 256 - 8
    half = n // 16 * 8
    gen = torch.Generator(device=DEV)
    gen.manual_seed(groups)
    g32, dtype = cls or R == 0, torch.float32 if cls else torch.bfloat16
    g = [torch.empty(n, device=DEV).normal_(0, 1e-3, generator=gen).to(torch.float32 if g32 else dtype) for _ in range(max(R, 1))]
    start = [torch.empty(n, device=DEV).normal_(0, s, generator=gen) for s in (0.02, 1e-4, 1e-4)]
    start[2].square_()
    hy = hzp.adamw_hyper(HP["lr"], HP["beta1"], HP["beta2"], HP["eps"], HP["weight_decay"], 1.0, 3)
    results, kernels = [], []
    for spans in ([(0, n)], [(0, half), (half, n)]):
        plan = hzp.hzp_plan([1] * len(spans), [b - a for a, b in spans], 8, 1, 1, tensor_class=[cls] * len(spans))
        plan.prepare()
        s, out = [x.clone() for x in start], torch.full((n + 64,), 0.5, dtype=dtype, device=DEV)

        def call(k, a, b):
            hzp.hzp_adamw_shard(plan, k, k + 1, cls, 0, hy, [x[a:b] for x in g], R, *([x[a:b]] for x in s), [out[a:b]])
        kernels += [launches_of(lambda: call(0, *spans[0]))[0][2]]
        for k, (a, b) in enumerate(spans):
            call(k, a, b)
        torch.cuda.synchronize()
        results.append([*s, out])
        assert bool((out[n:] == 0.5).all())
    assert kernels[0] != kernels[1]
    for a, b in zip(*results):
        assert torch.equal(a.view(torch.int32 if a.dtype == torch.float32 else torch.int16), b.view(torch.int32 if a.dtype == torch.float32 else torch.int16))
    assert not torch.equal(results[0][0], start[0])


@pytest.mark.parametrize("cls,R", [(0, R) for R in range(1, 33)] + [(1, R) for R in range(1, 33)])
def test_update_of_every_number_of_contributions_in_longer_launches(cls, R):
    """Small and large chunks of every R in the three forms of a launch (one segment, two of a length, two of very different ones that are
    found by search), against the fp32 sum in order and an update in 64 bits."""
    dtype = torch.float32 if cls else torch.bfloat16
    one, several = (larger_chunks_from(cls, R, True) or 20480) + 1, (larger_chunks_from(cls, R, False) or 10240) + 2
    forms = ((3000,), (one,), (several // 2, several // 2), (several - several // 8, several // 8))
    longest = max(map(sum, forms)) * 256
    gen = torch.Generator(device=DEV)
    gen.manual_seed(R)
    grads = [torch.empty(longest, device=DEV).normal_(0, 1e-3, generator=gen).to(dtype) for _ in range(R)]
    start = [torch.empty(longest, device=DEV).normal_(0, s, generator=gen) for s in (0.02, 1e-4, 1e-4)]
    start[2].square_()
    total = grads[0].to(torch.float32, copy=True)
    for x in grads[1:]:
        total += x
    total *= torch.tensor(1.0 / R, dtype=torch.float32, device=DEV)
    # (the hyper-parameters as the fp32 numbers that the entry point takes; bias corrections in 64 bits)
    lr, b1, b2, eps, wd = (float(np.float32(HP[k])) for k in ("lr", "beta1", "beta2", "eps", "weight_decay"))
    ge, p, m, v = total.double(), *(x.double() for x in start)
    terms = b1 * m.abs() + (1 - b1) * ge.abs()
    m = b1 * m + (1 - b1) * ge
    v = b2 * v + (1 - b2) * ge * ge
    denom = (v / (1 - b2 ** 3)).sqrt() + eps
    u = (m / (1 - b1 ** 3)) / denom
    p = p - lr * (u + wd * p)
    want = (p, m, v)
    # u is good to half of U_ERR relative (where |u| stays below 2; here it does not, as v comes close to 0), and to the two roundings of m, a
    # 2^-24 of its terms each, over the denominator
    step_error = lr * (U_ERR / 2 * u.abs() + 2 ** -23 * terms / (1 - b1 ** 3) / denom)
    hy = hzp.adamw_hyper(HP["lr"], HP["beta1"], HP["beta2"], HP["eps"], HP["weight_decay"], 1.0 / R, 3)
    for groups in forms:
        sizes = [g * 256 for g in groups]
        sizes[-1] -= 8
        print("class %d R=%d groups %s" % (cls, R, groups), flush=True)
        spans = [(sum(sizes[:k]), sum(sizes[:k + 1])) for k in range(len(sizes))]
        assert spans[-1][1] <= longest
        def views(t):           # (copies, so that segments do not follow each other)
            return [torch.cat([t[a:b], torch.full((64,), 0.5, dtype=t.dtype, device=DEV)]) for a, b in spans]
        g, s, o = [views(t) for t in grads], [views(t) for t in start], views(torch.zeros(longest, dtype=dtype, device=DEV))
        plan = hzp.hzp_plan([1] * len(sizes), sizes, 8, 1, 1, tensor_class=[cls] * len(sizes))
        hzp.hzp_adamw_shard(plan, 0, len(sizes), cls, 0, hy, [g[r][k] for k in range(len(sizes)) for r in range(R)], R, *s, o)
        torch.cuda.synchronize()
        for k, (a, b) in enumerate(spans):
            for key, have, ref in zip("pmv", s, want):
                w = ref[a:b].float().double()
                got = have[k][:b - a].double()
                bound = REL_TOL * torch.maximum(got.abs(), w.abs()) + RMS_FLOOR[key] * float(w.square().mean().sqrt()) + 1e-37
                if key == "p":
                    bound += step_error[a:b]
                assert bool(((got - w).abs() <= bound).all()), key
            assert torch.equal(o[k][:b - a], s[0][k][:b - a].to(dtype))
            assert all(bool((x[k][b - a:] == 0.5).all()) for x in (*s, o))


@pytest.mark.parametrize("place,out_place", [("packed", None), ("spread", None), ("down", None), ("packed", "spread"),
                                             ("spread", "down"), ("own", None), ("spread", "own"), ("own", "packed")])
@pytest.mark.parametrize("R,layers,ragged", [(8, 50, False), (8, 50, True), (32, 30, True), (3, 200, True)])
def test_many_segments_in_every_placement(place, out_place, R, layers, ragged):
    """More buckets than one launch lists with pointers of their own (34 at R = 8, 12 at R = 32, 53 at R = 3)."""
    print(place, out_place, R, layers, ragged, flush=True)
    rng = np.random.default_rng(layers)
    numel = [int(x) for x in rng.integers(1, 3000, layers)] if ragged else [1000] * layers
    wd = [float(k % 5 == 4) for k in range(layers)] if ragged else None        # equal inside a bucket
    desc = dict(tensors_per_layer=[1] * layers, tensor_numel=numel, tensor_wd_mult=wd)
    update_against_oracle(desc, 8, 1, R, 0, 0, place, out_place)


@pytest.mark.parametrize("z1,rank", [(1, 0), (3, 1)])
@pytest.mark.parametrize("place", ["packed", "own", "spread"])
def test_decay_looked_up_in_long_and_short_tables(z1, rank, place):
    """Up to 400 changes of the multiplier in a bucket, several inside one group, beside buckets without any."""
    rng = np.random.default_rng(8)
    layers = [[8] * 400, [3000], [int(x) for x in rng.integers(1, 30, 300)], [5000, 64, 5000], [70000, 8, 8, 70000],
              [int(x) for x in rng.integers(200, 600, 70)]] * 8
    numel = [n for layer in layers for n in layer]
    wd = [float(w) for w in rng.choice([0.0, 1.0, 0.5], len(numel))]
    desc = dict(tensors_per_layer=[len(x) for x in layers], tensor_numel=numel, tensor_wd_mult=wd)
    update_against_oracle(desc, 8, z1, 8, rank, 0, place)


@pytest.mark.parametrize("R", range(1, 33))
@pytest.mark.parametrize("g32", [False, True])
def test_reduction_of_every_number_of_contributions_at_group_edges(R, g32):
    print("reduce R=%d %s" % (R, "fp32" if g32 else "bf16"), flush=True)
    plan = hzp.hzp_plan([1] * len(EDGES), EDGES, align=8, z3=1, z1=1)
    rng = np.random.default_rng(R)
    for layer, n in enumerate(EDGES):
        g = [rng.standard_normal(n, dtype=np.float32) for _ in range(R)]
        if not g32:
            g = [hzp_inputs.to_bf16_bits(x) for x in g]
        for acc in (False, True):
            want = on.reduce(g, scale=0.3, accumulate=acc, out=np.full(n, 0.5, np.float32) if acc else None)
            whole = torch.full((n + 64,), 0.5, device=DEV)
            hzp.hzp_reduce_shard(plan, layer, 0, 1, 0, [to_dev(x) for x in g], 0.3, acc, whole[:n],
                                 grad_dtype=hzp.HZP_GRAD_F32 if g32 else hzp.HZP_GRAD_BF16)
            torch.cuda.synchronize()
            assert np.array_equal(to_host(whole[:n], np.uint32), want.view(np.uint32)), (n, acc)
            assert bool((whole[n:] == 0.5).all())


@pytest.mark.parametrize("g32", [False, True])
def test_reduction_cut_into_launches(g32):
    """A slice of more than 3 GB of nine contributions and the sum: two launches, the second one shorter."""
    R, es = 9, 4 if g32 else 2
    n = 3_100_000_000 // (R * es + 8) // 8 * 8 + 8
    print(n, R, g32, flush=True)
    plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1)
    torch.manual_seed(1)
    g = [torch.empty(n, dtype=torch.float32 if g32 else torch.bfloat16, device=DEV).normal_() for _ in range(R)]
    out = torch.full((n + 64,), 0.5, device=DEV)
    want = g[0].to(torch.float32, copy=True)
    for x in g[1:]:
        want += x
    want *= 0.3
    want += 0.5
    hzp.hzp_reduce_shard(plan, 0, 0, 1, 0, g, 0.3, True, out[:n], grad_dtype=hzp.HZP_GRAD_F32 if g32 else hzp.HZP_GRAD_BF16)
    torch.cuda.synchronize()
    assert torch.equal(out[:n], want)
    assert bool((out[n:] == 0.5).all())


@pytest.mark.parametrize("R", [17, 32])
@pytest.mark.parametrize("groups", [5120, 5121, 8192, 8193, 10240, 10241])
def test_reduction_that_just_fits_the_chip(R, groups):
    n = groups * 256 - 8
    print(n, R, flush=True)
    plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1)
    torch.manual_seed(groups)
    g = [torch.empty(n, dtype=torch.bfloat16, device=DEV).normal_() for _ in range(R)]
    want = g[0].to(torch.float32, copy=True)
    for x in g[1:]:
        want += x
    want *= 0.3
    for acc in (False, True):
        out = torch.full((n + 64,), 0.5, device=DEV)
        hzp.hzp_reduce_shard(plan, 0, 0, 1, 0, g, 0.3, acc, out[:n], grad_dtype=hzp.HZP_GRAD_BF16)
        torch.cuda.synchronize()
        assert torch.equal(out[:n], want + 0.5 if acc else want), acc
        assert bool((out[n:] == 0.5).all())


@pytest.mark.parametrize("place", ["own", "packed"])
@pytest.mark.parametrize("layers,K", [(24, 16), (40, 4)])
def test_post_step_gather_of_uneven_layers(place, layers, K):
    """Two layers a thousand times the others: more launches than one, longest pieces first, in one list or with shared distances."""
    print(place, layers, K, flush=True)
    rng = np.random.default_rng(K)
    numel = [2_000_000 if layer in (3, layers - 1) else int(rng.integers(1, 4000)) for layer in range(layers)]
    plan = hzp.hzp_plan([1] * layers, numel, align=8, z3=1, z1=K)
    sizes = [plan.bucket(layer).s1 for layer in range(layers)]
    whole = [torch.full((n * K + 8,), -1, dtype=torch.int16, device=DEV) for n in sizes]
    sources = [carve(sizes, torch.int16, place) for _ in range(K)]
    want = [rng.integers(-30000, 30000, (K, n)).astype(np.int16) for n in sizes]
    for i in range(layers):
        for k in range(K):
            sources[k][i].copy_(torch.from_numpy(want[i][k]))
    hzp.hzp_gather_layers(plan, 0, layers, 0, 1, [sources[k][i] for i in range(layers) for k in range(K)], K,
                          [w[:-8] for w in whole])
    torch.cuda.synchronize()
    for i in range(layers):
        got = whole[i].cpu().numpy()
        assert np.array_equal(got[:-8], want[i].reshape(-1)), i
        assert (got[-8:] == -1).all()


@pytest.mark.parametrize("place", ["own", "packed", "spread", "down"])
@pytest.mark.parametrize("layers,K,own,ragged", [(30, 8, None, True), (30, 8, 3, True), (210, 4, 0, True), (250, 1, None, False),
                                                 (5, 64, 63, False), (3, 2, 1, True)])
def test_post_step_gather_of_many_layers_in_every_placement(place, layers, K, own, ragged):
    """More pieces than one list holds (192) and fewer; layers at equal distances in every source or not; one piece of
    each layer already in place or none."""
    print(place, layers, K, own, flush=True)
    rng = np.random.default_rng(layers + K)
    numel = [int(x) for x in rng.integers(1, 40000, layers)] if ragged else [2500] * layers
    plan = hzp.hzp_plan([1] * layers, numel, align=8, z3=1, z1=K)
    sizes = [plan.bucket(layer).s1 for layer in range(layers)]
    whole = [torch.full((n * K,), -1, dtype=torch.int16, device=DEV) for n in sizes]
    sources = [carve(sizes, torch.int16, place) for _ in range(K)]
    want = []
    for i, n in enumerate(sizes):
        host = rng.integers(-30000, 30000, (K, n)).astype(np.int16)
        want.append(host.reshape(-1))
        for k in range(K):
            if k == own:
                sources[k][i] = whole[i][k * n:(k + 1) * n]
            sources[k][i].copy_(torch.from_numpy(host[k]))
    hzp.hzp_gather_layers(plan, 0, layers, 0, 1, [sources[k][i] for i in range(layers) for k in range(K)], K, whole)
    torch.cuda.synchronize()
    for i in range(layers):
        assert np.array_equal(whole[i].cpu().numpy(), want[i]), i


@pytest.mark.parametrize("cls", [0, 1])
@pytest.mark.parametrize("shift", [0, 1, 4])
@pytest.mark.parametrize("name,numel,z3", [("few", [5000, 64, 5000], 1), ("edges", [1, 7, 8, 9, 511, 512, 513, 4096, 70001], 3),
                                           ("lopsided", [3000001] + [40] * 60, 4), ("many", [9000] * 260, 2), ("tiny", [3] * 450, 2),
                                           ("one", [1234567], 8), ("cut", [1, 7, 8, 9, 511, 512, 513, 4096, 4000001], 3),
                                           ("uneven", [300007, 5, 70001, 513] * 30, 2), ("even", [30011] * 150, 2),
                                           ("even launches", [70011] * 260, 2), ("uneven launches", [1300003, 400007] * 160, 2),
                                           ("tiny and one", [100] * 700 + [3000001] + [100] * 500, 4)])
def test_tensors_and_bucket_in_one_pass_or_two(name, numel, z3, shift, cls):
    """The unpacking gather alone, with the bucket beside it and for one tensor at a time; tensors that start on a 16-byte
    boundary (one pass serves both outputs), an element and half a vector behind one."""
    print(name, z3, shift, cls, flush=True)
    plan = hzp.hzp_plan([len(numel)], numel, align=8, z3=z3, z1=z3, tensor_class=[cls] * len(numel))
    info = plan.bucket(0, cls)
    dt = torch.int32 if cls else torch.int16
    gen = torch.Generator(device=DEV).manual_seed(len(numel) + shift)
    bucket = torch.randint(-30000, 30000, (info.padded,), dtype=dt, device=DEV, generator=gen)
    shards = [bucket[j * info.s3:(j + 1) * info.s3].clone() for j in range(z3)]
    places, at = [], 16
    for n in numel:
        places.append(at + shift)
        at += -(-(n + 24) // 16) * 16
    want = torch.full((at,), 77, dtype=dt, device=DEV)
    for t, (n, place) in enumerate(zip(numel, places)):
        off = plan.tensor(t).offset
        want[place:place + n] = bucket[off:off + n]

    def views(flat):
        return [flat[place:place + n] for n, place in zip(numel, places)]
    alone, beside, single = (torch.full((at,), 77, dtype=dt, device=DEV) for _ in range(3))
    whole = torch.full((info.padded + 32,), 77, dtype=dt, device=DEV)
    hzp.hzp_gather_layer(plan, 0, cls, 3, shards, None, views(alone))
    hzp.hzp_gather_layer(plan, 0, cls, 3, shards, whole[16:16 + info.padded], views(beside))
    for t in range(0, len(numel), max(1, len(numel) // 40)):
        hzp.hzp_gather_tensor(plan, t, shards, views(single)[t])
        views(want)[t].eq(views(single)[t]).all().item() or pytest.fail("tensor %d" % t)
    torch.cuda.synchronize()
    assert torch.equal(alone, want)
    assert torch.equal(beside, want)
    assert torch.equal(whole[16:16 + info.padded], bucket)
    assert bool((whole[:16] == 77).all()) and bool((whole[16 + info.padded:] == 77).all())


@pytest.mark.parametrize("numel,most", [([5000] * 199, 1), ([100, 20000] * 80, 1), ([5000, 5000, 20000] * 100, 1), ([16384] * 800, 2),
                                        ([100] * 5000 + [50000000] + [100] * 5000, 26), ([1000000] * 150, 1)])
def test_unpacking_takes_no_more_launches_than_the_tensors_need(numel, most):
    """Short copies of many tensors: a launch for every 400 tensors, whatever their sizes."""
    print(len(numel), flush=True)
    plan = hzp.hzp_plan([len(numel)], numel, align=8, z3=2, z1=2)
    plan.prepare()
    info = plan.bucket(0)
    shards = [torch.empty(info.s3, dtype=torch.int16, device=DEV) for _ in range(2)]
    views = list(torch.split(torch.empty(sum(numel), dtype=torch.int16, device=DEV), numel))
    got = launches_of(lambda: hzp.hzp_gather_layer(plan, 0, 0, 3, shards, None, views))
    assert len(got) <= most, len(got)


def test_a_copy_of_few_pieces_travels_in_a_small_block():
    """1 to 8, 9 to 64 and more pieces have a kernel with an argument block each."""
    kernel = {}
    for k in (1, 8, 9, 16, 64):
        plan = hzp.hzp_plan([1], [8 * k], align=8, z3=k, z1=k)
        plan.prepare()
        shards = [torch.empty(8, dtype=torch.int16, device=DEV) for _ in range(k)]
        out = torch.empty(8 * k, dtype=torch.int16, device=DEV)
        got = launches_of(lambda: hzp.hzp_gather_layer(plan, 0, 0, 3, shards, out, None))
        assert [g[:2] for g in got] == [((1, k, 1), 0)]
        kernel[k] = got[0][2]
    plan = hzp.hzp_plan([1] * 10, [80] * 10, align=8, z3=1, z1=10)
    plan.prepare()
    own = [torch.empty(8, dtype=torch.int16, device=DEV) for _ in range(100)]
    out = [torch.empty(80, dtype=torch.int16, device=DEV) for _ in range(10)]
    got = launches_of(lambda: hzp.hzp_gather_layers(plan, 0, 10, 0, 1, own, 10, out))
    assert [g[:2] for g in got] == [((1, 100, 1), 0)]
    assert kernel[1] == kernel[8] and kernel[9] == kernel[16] == kernel[64] and len({kernel[8], kernel[64], got[0][2]}) == 3


@pytest.mark.parametrize("k", [9, 16, 64])
def test_bucket_of_many_shards(k):
    n = 8 * 64 * 3 + 8
    plan = hzp.hzp_plan([1], [n * k], align=8, z3=k, z1=k)
    want = torch.randint(-30000, 30000, (n * k,), dtype=torch.int16, device=DEV)
    shards = [x.clone() for x in torch.split(want, n)]
    out = torch.full((n * k + 8,), 77, dtype=torch.int16, device=DEV)
    hzp.hzp_gather_layer(plan, 0, 0, 3, shards, out[:n * k], None)
    torch.cuda.synchronize()
    assert torch.equal(out[:n * k], want) and bool((out[n * k:] == 77).all())


def update_launches(groups, cls, R, layers=1, split=None):
    """The launches of one update call over `layers` buckets of separate buffers that hold `groups` groups of 256 elements together;
    split: a second tensor of so many elements without decay in each bucket."""
    n = groups * 256 // layers
    numel = [n] if split is None else [n - split, split]
    wd = None if split is None else [1.0, 0.0] * layers
    plan = hzp.hzp_plan([len(numel)] * layers, numel * layers, align=8, z3=1, z1=1, tensor_class=[cls] * (len(numel) * layers),
                        tensor_wd_mult=wd)
    plan.prepare()
    grad, out = (torch.float32, torch.float32) if cls else (torch.bfloat16, torch.bfloat16)

    def buffers(dtype, count=layers):
        return [torch.empty(n + 64, dtype=dtype, device=DEV) for _ in range(count)]
    hy = hzp.adamw_hyper(HP["lr"], HP["beta1"], HP["beta2"], HP["eps"], HP["weight_decay"], 1.0 / R, 3)
    g, p, m, v, o = buffers(grad, layers * R), *(buffers(torch.float32) for _ in range(3)), buffers(out)
    return launches_of(lambda: hzp.hzp_adamw_shard(plan, 0, layers, cls, 0, hy, g, R, p, m, v, o))


@pytest.mark.parametrize("layers,split", [(1, None), (4, None), (4, 128)])
@pytest.mark.parametrize("cls,R", [(0, 4), (0, 32), (1, 1), (1, 4)])
def test_short_updates_are_not_capped(cls, R, layers, split):
    """All wavefronts of a launch of up to 5120 groups are resident; longer ones are capped by unused LDS."""
    for groups in (2060, 3600, 4096, 5120):
        assert [lds for _, lds, _ in update_launches(groups, cls, R, layers, split)] == [0], groups
    assert update_launches(5124, cls, R, layers, split)[0][1] > 0


@pytest.mark.parametrize("layers,split", [(1, None), (4, None), (4, 128)])
@pytest.mark.parametrize("cls,R", [(0, 16), (1, 16)])
def test_many_contributions_of_few_groups_have_a_kernel_of_their_own(cls, R, layers, split):
    """One segment, several, and several whose decay is looked up."""
    few, more = (update_launches(groups, cls, R, layers, split) for groups in (600, 3000))
    assert len(few) == len(more) == 1 and few[0][2] != more[0][2]


def reduce_plan(n):
    plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1)
    plan.prepare()
    return plan


# edges of the forms, in groups of 256 elements: many at a time, chunks of 4, chunks of 2 on two quads per lane, capped
@pytest.mark.parametrize("R,g32,few,fours,twos", [(16, False, 2048, 5120, 10240), (32, False, 2048, 5120, 10240), (9, False, 2048, 6826, 10240),
                                                  (16, True, 2048, 3072, 8192), (32, True, 2048, 3072, 8192), (9, True, 2048, 4096, 8192)])
@pytest.mark.parametrize("acc", [False, True])
def test_reduction_forms_at_their_edges(R, g32, few, fours, twos, acc):
    """The grid and the LDS say which form a launch has; the results are those of the sum in order, bit for bit."""
    dt, gd = (torch.float32, hzp.HZP_GRAD_F32) if g32 else (torch.bfloat16, hzp.HZP_GRAD_BF16)
    torch.manual_seed(R)
    most = (twos + 3) * 256
    g = [torch.empty(most, dtype=dt, device=DEV).normal_() for _ in range(R)]
    want = g[0].to(torch.float32, copy=True)
    for x in g[1:]:
        want += x
    want *= 0.3
    if acc:
        want += 0.5
    for groups, per_lane in ((few, 1), (few + 1, 1), (fours, 1), (fours + 1, 2), (twos, 2), (twos + 1, 1)):
        for n in (groups * 256, groups * 256 - 248):
            print(R, g32, acc, n, flush=True)
            plan, out = reduce_plan(n), torch.full((most + 64,), 0.5, device=DEV)
            slices = [x[:n] for x in g]

            def call():
                hzp.hzp_reduce_shard(plan, 0, 0, 1, 0, slices, 0.3, acc, out[:n], grad_dtype=gd)
            (grid, lds, _), = launches_of(call)
            assert grid == (-(-groups // per_lane), 1, 1) and (lds > 0) == (groups > twos)
            call()
            torch.cuda.synchronize()
            assert torch.equal(out[:n], want[:n]) and bool((out[n:] == 0.5).all())


def in_order_sum(g, acc):
    """0.3 times the left-to-right fp32 sum, added to 0.5 where `acc`."""
    want = g[0].to(torch.float32, copy=True)
    for x in g[1:]:
        want += x
    want *= 0.3
    return want + 0.5 if acc else want


# The longest launches, in bytes of contributions, whose arguments are all read from the block; longer ones, and accumulating ones of
# any length, have other kernels.
@pytest.mark.parametrize("R,g32", [(1, False), (2, False), (3, False), (4, False), (8, False), (9, False), (13, False), (32, False),
                                   (1, True), (2, True), (5, True), (8, True), (11, True), (32, True)])
def test_short_reductions_read_their_arguments_from_the_block(R, g32):
    dt, gd, es = (torch.float32, hzp.HZP_GRAD_F32, 4) if g32 else (torch.bfloat16, hzp.HZP_GRAD_BF16, 2)
    longest = (2 << 20 if R * es <= 4 else 1250000) // (R * es) // 8 * 8
    torch.manual_seed(R)
    g = [torch.empty(longest + 8, dtype=dt, device=DEV).normal_() for _ in range(R)]
    kernels = []
    for n in (8, 256, longest, longest + 8):
        for acc in (False, True):
            print(R, g32, n, acc, flush=True)
            plan, out = reduce_plan(n), torch.full((n + 64,), 0.5, device=DEV)

            def call():
                hzp.hzp_reduce_shard(plan, 0, 0, 1, 0, [x[:n] for x in g], 0.3, acc, out[:n], grad_dtype=gd)
            (_, _, kernel), = launches_of(call, replay=True)
            kernels.append(kernel)
            for how in ("replayed", "eager"):           # (from 13 contributions on two forms)
                if how == "eager":
                    out.fill_(0.5)
                    call()
                    torch.cuda.synchronize()
                assert torch.equal(out[:n], in_order_sum([x[:n] for x in g], acc)) and bool((out[n:] == 0.5).all()), how
    block, registers, accumulating = kernels[0], kernels[6], kernels[1]
    assert kernels == [block, accumulating] * 3 + [registers, accumulating] and len({block, registers, accumulating}) == 3


@pytest.mark.parametrize("R", [5, 7, 10, 11, 13, 14, 19, 23, 29, 31])
@pytest.mark.parametrize("g32", [False, True])
def test_reduction_in_chunks_of_different_sizes(R, g32):
    """Numbers of contributions that are no multiple of a chunk, in each form of a launch (up to 2048 groups, all resident, chunks of 2,
    capped): the sum in order, bit for bit."""
    dt, gd = (torch.float32, hzp.HZP_GRAD_F32) if g32 else (torch.bfloat16, hzp.HZP_GRAD_BF16)
    torch.manual_seed(R)
    g = [torch.empty(12000 * 256, dtype=dt, device=DEV).normal_() for _ in range(R)]
    for groups in (2048, 2900, 7500, 10000, 12000):
        n = groups * 256 - 8
        for acc in (False, True):
            print(R, g32, n, acc, flush=True)
            plan, out = reduce_plan(n), torch.full((n + 64,), 0.5, device=DEV)
            hzp.hzp_reduce_shard(plan, 0, 0, 1, 0, [x[:n] for x in g], 0.3, acc, out[:n], grad_dtype=gd)
            torch.cuda.synchronize()
            assert torch.equal(out[:n], in_order_sum([x[:n] for x in g], acc)) and bool((out[n:] == 0.5).all())


def guarded(n, shift=0):
    """n elements of -1 at `shift` elements behind a 16-byte boundary, with eight more on both sides."""
    whole = torch.full((n + 24,), -1, dtype=torch.int16, device=DEV)
    return whole, whole[8 + shift:8 + shift + n]


def assert_only(whole, view, want):
    torch.cuda.synchronize()
    at = (view.data_ptr() - whole.data_ptr()) // 2
    got = whole.cpu().numpy()
    assert np.array_equal(got[at:at + len(want)], want)
    assert (got[:at] == -1).all() and (got[at + len(want):] == -1).all()


@pytest.mark.parametrize("numel", [5, 1023, 70001])
@pytest.mark.parametrize("k", [1, 2, 4, 5, 6, 7, 8, 9, 10])
def test_calls_of_few_pieces(k, numel):
    """Numbers of pieces around those whose argument blocks are the smallest: buckets (a shard in place or none), several layers' shards,
    one tensor and several tensors, all to the bit and nothing beside them."""
    print(k, numel, flush=True)
    rng = np.random.default_rng(k + numel)
    # one bucket of k shards, which holds one tensor
    plan = hzp.hzp_plan([1], [numel * k], align=8, z3=k, z1=k)
    s3 = plan.bucket(0).s3
    host = rng.integers(0, 30000, (k, s3)).astype(np.int16)
    shards = [to_dev(h) for h in host]
    for own in {None, 0, k - 1}:
        whole, out = guarded(k * s3)
        given = [out[j * s3:(j + 1) * s3] if j == own else s for j, s in enumerate(shards)]
        if own is not None:
            given[own].copy_(shards[own])
        hzp.hzp_gather_layer(plan, 0, 0, 3, given, out, None)
        assert_only(whole, out, host.reshape(-1))
    for shift in (0, 1, 5):
        whole, out = guarded(numel * k, shift)
        hzp.hzp_gather_tensor(plan, 0, shards, out)
        assert_only(whole, out, host.reshape(-1)[:numel * k])
    # the middle one of three tensors, whose first and last parts are short
    plan = hzp.hzp_plan([3], [numel, numel * k, 3], align=8, z3=k + 1, z1=k + 1)
    info, s3 = plan.tensor(1), plan.bucket(0).s3
    host = rng.integers(0, 30000, (k + 1, s3)).astype(np.int16)
    for shift in (0, 3):
        whole, out = guarded(numel * k, shift)
        hzp.hzp_gather_tensor(plan, 1, [to_dev(h) for h in host], out)
        assert_only(whole, out, host.reshape(-1)[info.offset:info.offset + numel * k])
    # k tensors of one shard
    plan = hzp.hzp_plan([k], [numel + t for t in range(k)], align=8, z3=1, z1=1)
    host = rng.integers(0, 30000, plan.bucket(0).s3).astype(np.int16)
    outs = [guarded(numel + t, t % 8) for t in range(k)]
    hzp.hzp_gather_layer(plan, 0, 0, 3, [to_dev(host)], None, [o for _, o in outs])
    for t, (whole, out) in enumerate(outs):
        at = plan.tensor(t).offset
        assert_only(whole, out, host[at:at + numel + t])
    # several layers' shards, k pieces in all
    for layers in {n for n in (1, 2, 3, k) if k % n == 0}:
        plan = hzp.hzp_plan([1] * layers, [numel * (n + 1) for n in range(layers)], align=8, z3=1, z1=k // layers)
        sizes = [plan.bucket(n).s1 for n in range(layers)]
        host = [rng.integers(0, 30000, (k // layers, n)).astype(np.int16) for n in sizes]
        outs = [guarded(h.size) for h in host]
        hzp.hzp_gather_layers(plan, 0, layers, 0, 1, [to_dev(x) for h in host for x in h], k // layers, [o for _, o in outs])
        for h, (whole, out) in zip(host, outs):
            assert_only(whole, out, h.reshape(-1))


@pytest.mark.parametrize("z1,z3", [(3, 2), (7, 2), (9, 2), (11, 2), (13, 2), (15, 2), (17, 2), (31, 2), (64, 3)])
def test_shard_from_few_and_many_owners(z1, z3):
    """2 to 9 and more whole and partial pieces: those that the smallest argument block holds, one more, one list of eight and longer."""
    print(z1, z3, flush=True)
    rng = np.random.default_rng(z1)
    plan = hzp.hzp_plan([1], [90001], align=8, z3=z3, z1=z1)
    b = plan.bucket(0)
    bucket = rng.integers(0, 30000, b.padded).astype(np.int16)
    for j in range(z3):
        first, n = plan.cover(0, 0, j)
        whole, out = guarded(b.s3)
        hzp.hzp_gather_shard(plan, 0, 0, j, [to_dev(bucket[(first + q) * b.s1:(first + q + 1) * b.s1]) for q in range(n)], out)
        assert_only(whole, out, bucket[j * b.s3:(j + 1) * b.s3])


def lengths(kind, n, rng):
    """n tensor lengths: of 1 to 8 elements (a tile of 512 meets 65 of them at an alignment of 8), alike, or very different."""
    return [int(x) for x in {"tiny": lambda: rng.integers(1, 9, n), "even": lambda: np.full(n, 1003),
                             "spread": lambda: np.maximum(1, np.exp(rng.normal(6.5, 1.5, n)))}[kind]()]


@pytest.mark.parametrize("cls", [0, 1])
@pytest.mark.parametrize("z3", [1, 3, 8, 9])
@pytest.mark.parametrize("kind,n", [("tiny", 6), ("tiny", 64), ("tiny", 65), ("tiny", 700), ("even", 7), ("even", 64), ("even", 300),
                                    ("spread", 3), ("spread", 40), ("spread", 64), ("spread", 65), ("spread", 129), ("spread", 500)])
def test_tensors_that_lie_as_in_the_bucket(kind, n, z3, cls):
    """Views of one flat buffer at the bucket's own offsets (one pass over the bucket, each vector's tensor looked up), and the same with one
    tensor elsewhere (lists): tensors, gaps between them untouched, with and without the bucket, a shard in place or none, in or beside the bucket."""
    print(kind, n, z3, cls, flush=True)
    rng = np.random.default_rng(n * 31 + z3)
    numel = lengths(kind, n, rng)
    plan = hzp.hzp_plan([n], numel, align=8, z3=z3, z1=z3, tensor_class=[cls] * n)
    b = plan.bucket(0, cls)
    dtype = torch.int32 if cls else torch.int16
    host = rng.integers(0, 30000, b.padded).astype(np.int32 if cls else np.int16)
    at = [plan.tensor(t).offset for t in range(n)]
    inside = np.zeros(b.padded, dtype=bool)
    for a, k in zip(at, numel):
        inside[a:a + k] = True
    whole = to_dev(host)
    shards = [whole[j * b.s3:(j + 1) * b.s3].clone() for j in range(z3)]
    for moved in (None, n // 2):
        for own in (False, None, 0, z3 - 1):                # False: no bucket
            flat = torch.full((b.padded + 16,), -1, dtype=dtype, device=DEV)
            views = [flat[8 + a:8 + a + k] for a, k in zip(at, numel)]
            apart = torch.full((numel[n // 2] + 1,), -1, dtype=dtype, device=DEV)
            if moved is not None:
                views[moved] = apart[1:]
            bucket = None if own is False else torch.full((b.padded,), -1, dtype=dtype, device=DEV)
            given = list(shards)
            if own is not None and own is not False:
                given[own] = bucket[own * b.s3:(own + 1) * b.s3]
                given[own].copy_(shards[own])
            hzp.hzp_gather_layer(plan, 0, cls, 3, given, bucket, views)
            torch.cuda.synchronize()
            want = np.where(inside, host, -1)
            if moved is not None:
                want[at[moved]:at[moved] + numel[moved]] = -1
                assert np.array_equal(apart.cpu().numpy()[1:], host[at[moved]:at[moved] + numel[moved]]) and int(apart[0]) == -1
            got = flat.cpu().numpy()
            assert np.array_equal(got[8:-8], want) and (got[:8] == -1).all() and (got[-8:] == -1).all()
            if bucket is not None:
                assert np.array_equal(bucket.cpu().numpy(), host)
    bucket = torch.full((b.padded,), -1, dtype=dtype, device=DEV)          # the tensors are views of the bucket
    hzp.hzp_gather_layer(plan, 0, cls, 3, shards, bucket, [bucket[a:a + k] for a, k in zip(at, numel)])
    torch.cuda.synchronize()
    assert np.array_equal(bucket.cpu().numpy(), host)


@pytest.mark.parametrize("numel,both,launches", [([1000] * 9, False, 1), ([300000] * 9, False, 1), ([200, 90000] * 5, False, 1), ([3000] * 100, False, 1),
                                                 ([100, 9000] * 50, False, 1), ([100, 90000] * 50, False, 1), ([100, 9000] * 300, False, 1),
                                                 ([9000] * 200, True, 1), ([1000] * 9, True, 1), ([300000] * 9, True, 1)])
def test_every_choice_between_lists_and_the_bucket_s_own_layout(numel, both, launches):
    """Sizes on both sides of each line of the choice, from 3 shards, to the bit: the captured call, in one launch, and the eager one, whose form
    may be another (test_launch_choice.py asserts both)."""
    n = len(numel)
    plan = hzp.hzp_plan([n], numel, align=64, z3=3, z1=3)
    plan.prepare()
    b = plan.bucket(0)
    whole = torch.randint(0, 30000, (b.padded,), dtype=torch.int16, device=DEV)
    shards = [whole[j * b.s3:(j + 1) * b.s3].clone() for j in range(3)]
    flat = torch.full((b.padded,), -1, dtype=torch.int16, device=DEV)
    views = [flat[plan.tensor(t).offset:plan.tensor(t).offset + numel[t]] for t in range(n)]
    bucket = torch.empty_like(whole) if both else None
    got = launches_of(lambda: hzp.hzp_gather_layer(plan, 0, 0, 3, shards, bucket, views), replay=True)
    assert len(got) == launches
    for how in ("replayed", "eager"):
        if how == "eager":
            flat.fill_(-1)
            if both:
                bucket.fill_(-1)
            hzp.hzp_gather_layer(plan, 0, 0, 3, shards, bucket, views)
            torch.cuda.synchronize()
        for t, v in enumerate(views):
            assert torch.equal(v, whole[plan.tensor(t).offset:plan.tensor(t).offset + numel[t]]), (how, t)
        assert not both or torch.equal(bucket, whole), how


@pytest.fixture(scope="module")
def wide_room():
    """An allocation whose ends lie further apart than 32 bits of 16-byte units reach."""
    room = torch.empty((33 << 30) + (16 << 20), dtype=torch.uint8, device=DEV)
    yield room
    room.untyped_storage().resize_(0)                       # given back with the module
    torch.cuda.empty_cache()


@pytest.mark.parametrize("cls,R", [(0, R) for R in range(1, 10)] + [(1, R) for R in range(1, 10)] + [(0, 0)])
@pytest.mark.parametrize("n", [8, 248, 256, 504, 10248])
def test_short_updates_with_streams_near_and_far(cls, R, n, wide_room):
    """Streams in any order, near each other and with one of them 33 GiB away (up to two contributions are always equally distant and go by their
    distance, more by pointers): the same bits, with scalars from the call and from device memory, with an output and without."""
    print(cls, R, n, flush=True)
    rng = np.random.default_rng(R * 7 + n)
    k, wide = max(R, 1), cls == 1 or R == 0
    types = [torch.float32 if wide else torch.bfloat16] * k + [torch.float32] * 3 + [torch.float32 if cls else torch.bfloat16]
    room = 4 * n + 256
    start = [torch.from_numpy(rng.standard_normal(n, dtype=np.float32) * np.float32(s)).to(DEV).to(t)
             for s, t in zip([1e-3] * k + [0.02, 1e-4, 1e-4], types)]
    start[-1].square_()
    plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1, tensor_class=[cls])
    hy = hzp.adamw_hyper(HP["lr"], HP["beta1"], HP["beta2"], HP["eps"], HP["weight_decay"], 1.0 / k, 3)
    scalars = torch.tensor(hzp.hzp_adamw_scalars(hy), dtype=torch.float32, device=DEV)
    first = None
    for far in (None, k - 1, k, k + 2, k + 3):              # the last contribution, master weights, variance, output
        at = [int(p) * room + ((33 << 30) if i == far else 0) for i, p in enumerate(rng.permutation(k + 4))]
        streams = [wide_room[a:a + n * t.itemsize].view(t) for a, t in zip(at, types)]
        for call, scal in ((hzp.hzp_adamw_shard, hy), (hzp.hzp_adamw_shard_dev, scalars)):
            for given in (True, False):
                for t, s in zip(streams, start):
                    t.copy_(s)
                streams[-1].fill_(7)
                call(plan, 0, 1, cls, 0, scal, streams[:k], R, [streams[k]], [streams[k + 1]], [streams[k + 2]], [streams[k + 3]] if given else None)
                torch.cuda.synchronize()
                got = [t.clone() for t in streams[k:k + 3]]
                first = first or got
                assert all(torch.equal(a, b) for a, b in zip(got, first)), (far, call, given)
                want = got[0].to(types[-1]) if given else torch.full_like(streams[-1], 7)
                assert torch.equal(streams[-1], want), (far, call, given)
    for t, s in zip(streams, start):                        # the form of a captured call
        t.copy_(s)
    launches_of(lambda: hzp.hzp_adamw_shard(plan, 0, 1, cls, 0, hy, streams[:k], R, *[[t] for t in streams[k:]]), replay=True)
    assert all(torch.equal(a, b) for a, b in zip(streams[k:], first + [first[0].to(types[-1])]))


@pytest.mark.parametrize("accumulate", [0, 1])
@pytest.mark.parametrize("g32", [0, 1])
@pytest.mark.parametrize("R", [12, 13, 16, 17, 23, 24, 31, 32])
@pytest.mark.parametrize("n", [8, 264, 384 * 256, 384 * 256 + 8, 768 * 256, 768 * 256 + 8])
def test_short_reductions_by_distance(n, R, g32, accumulate, wide_room):
    """Contributions at equal distances, upwards and downwards, in any order, and one of them 33 GiB away: the sum in order, bit for bit."""
    print(n, R, g32, accumulate, flush=True)
    rng = np.random.default_rng(R + n)
    gt = torch.float32 if g32 else torch.bfloat16
    grads = [torch.from_numpy(rng.standard_normal(n, dtype=np.float32)).to(DEV).to(gt) for _ in range(R)]
    before = torch.from_numpy(rng.standard_normal(n, dtype=np.float32)).to(DEV)
    want = grads[0].float()
    for t in grads[1:]:
        want = want + t.float()
    want = want * 0.5
    want = before + want if accumulate else want
    plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1)
    size = n * grads[0].itemsize
    step = size + 16
    raw = torch.empty(step * R, dtype=torch.uint8, device=DEV)
    mixed = [int(r) * step for r in rng.permutation(R)]
    for placed, far in (([step * r for r in range(R)], False), ([step * (R - 1 - r) for r in range(R)], False), (mixed, False), (mixed, True)):
        g = [raw[a:a + size].view(gt) for a in placed]
        if far:
            g[R // 2] = wide_room[33 << 30:(33 << 30) + size].view(gt)
        for t, x in zip(g, grads):
            t.copy_(x)
        out = before.clone()
        hzp.hzp_reduce_shard(plan, 0, 0, 3, 0, g, 0.5, accumulate, out, grad_dtype=hzp.HZP_GRAD_F32 if g32 else hzp.HZP_GRAD_BF16)
        torch.cuda.synchronize()
        assert torch.equal(out, want), (placed[:3], far)
    out = before.clone()                                    # the form of a captured call
    launches_of(lambda: hzp.hzp_reduce_shard(plan, 0, 0, 3, 0, g, 0.5, accumulate, out, grad_dtype=hzp.HZP_GRAD_F32 if g32 else hzp.HZP_GRAD_BF16), replay=True)
    assert torch.equal(out, want)


@pytest.mark.parametrize("cls,R", [(c, R) for c in (0, 1) for R in (2, 3, 4, 5, 8, 9, 16, 17, 31, 32)])
@pytest.mark.parametrize("n", [8, 264, 640 * 256, 640 * 256 + 8, 1024 * 256, 1024 * 256 + 8, 1536 * 256, 1536 * 256 + 8, 2048 * 256 + 8])
def test_short_updates_with_equally_distant_contributions(cls, R, n):
    """Contributions at equal distances, upwards and downwards, and with the last one 16 bytes off: the same bits on both sides of each limit, and
    close to the sum and step in float64."""
    print(cls, R, n, flush=True)
    gen = torch.Generator(device=DEV).manual_seed(R + n)
    gt = torch.float32 if cls else torch.bfloat16
    grads = [(torch.randn(n, device=DEV, generator=gen) * 1e-3).to(gt) for _ in range(R)]
    state = [torch.randn(n, device=DEV, generator=gen) * s for s in (0.02, 1e-4, 1e-4)]
    state[2].square_()
    plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1, tensor_class=[cls])
    hy = hzp.adamw_hyper(HP["lr"], HP["beta1"], HP["beta2"], HP["eps"], HP["weight_decay"], 1.0 / R, 3)
    size = n * grads[0].itemsize
    step = size + 272
    raw = torch.empty(step * R + 64, dtype=torch.uint8, device=DEV)
    first = None
    for placed in ([step * r for r in range(R)], [step * (R - 1 - r) for r in range(R)], [step * r + 16 * (r == R - 1) for r in range(R)]):
        g = [raw[a:a + size].view(gt) for a in placed]
        for t, x in zip(g, grads):
            t.copy_(x)
        got = [t.clone() for t in state] + [torch.zeros(n, dtype=gt, device=DEV)]
        hzp.hzp_adamw_shard(plan, 0, 1, cls, 0, hy, g, R, *[[t] for t in got])
        torch.cuda.synchronize()
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(got, first))
    mean = sum(t.double() for t in grads) / R
    m = HP["beta1"] * state[1].double() + (1 - HP["beta1"]) * mean
    # (each of at most 31 sums rounds by 2^-24 of what is summed so far, the scaling and the step by four times as much)
    bound = 2.0 ** -24 * ((R + 4) * sum(t.double().abs() for t in grads) / R + 4 * state[1].double().abs())
    assert ((first[1].double() - m).abs() <= bound).all()
    assert torch.equal(first[3], first[0].to(gt))


@pytest.mark.parametrize("cls", [0, 1])
@pytest.mark.parametrize("kind,n,z3", [("tiny", 6, 1), ("tiny", 12, 3), ("spread", 6, 8), ("spread", 12, 8), ("spread", 13, 8), ("even", 12, 2), ("long", 6, 3),
                                       ("long", 12, 8), ("long", 13, 8), ("long", 64, 8), ("long", 64, 9), ("long", 65, 2)])
def test_tensors_that_lie_near_each_other_and_far(kind, n, z3, cls, wide_room):
    """Tensors and shards in any order, on 16 bytes (distances in the argument block), one of them 33 GiB away or off 16 bytes (lists): to the
    bit, and nothing beside them written."""
    print(kind, n, z3, cls, flush=True)
    rng = np.random.default_rng(n * 31 + z3 + cls)
    numel = [700000 // n * (1 + 5 * (t % 7 == 3)) + t for t in range(n)] if kind == "long" else lengths(kind, n, rng)
    plan = hzp.hzp_plan([n], numel, align=8, z3=z3, z1=z3, tensor_class=[cls] * n)
    b, es = plan.bucket(0, cls), 4 if cls else 2
    dtype = torch.int32 if cls else torch.int16
    host = torch.from_numpy(rng.integers(0, 30000, b.padded).astype(np.int32 if cls else np.int16)).to(DEV)
    sizes = [b.s3] * z3 + numel
    room = [-(-k * es // 16) * 16 + 48 for k in sizes]
    assert sum(room) < 16 << 20
    for odd, far in ((None, None), (None, 0), (None, z3 - 1), (None, z3), (None, z3 + n - 1), (z3 + n // 2, None), (z3, None)):
        raw = wide_room[:sum(room)].view(dtype)
        raw.fill_(-1)
        wide_room[33 << 30:].fill_(255)
        at, places = 0, [0] * len(sizes)
        for i in rng.permutation(len(sizes)):
            places[i], at = at, at + room[i]
        parts = []
        for i, k in enumerate(sizes):
            start = (places[i] % (1 << 20) // 16 * 16 + (33 << 30) if i == far else places[i]) + 16 + (es if i == odd else 0)
            parts.append(wide_room[start:start + k * es].view(dtype))
        for j in range(z3):
            parts[j].copy_(host[j * b.s3:(j + 1) * b.s3])
        before = wide_room[:sum(room)].clone()
        hzp.hzp_gather_layer(plan, 0, cls, 3, parts[:z3], None, parts[z3:])
        torch.cuda.synchronize()
        for t, v in enumerate(parts[z3:]):
            first = plan.tensor(t).offset
            assert torch.equal(v, host[first:first + numel[t]]), (odd, far, t)
            v.fill_(-1)
        assert torch.equal(wide_room[:sum(room)], before), (odd, far)       # nothing else changed


@pytest.mark.parametrize("cls", [0, 1])
@pytest.mark.parametrize("K,s1", [(1, 8), (2, 520), (8, 64), (9, 128), (10, 8)])
@pytest.mark.parametrize("layers", [2, 7, 33, 210])
def test_layers_of_one_length_at_equal_distances(layers, K, s1, cls):
    """All layers of a post-step gather, upwards and downwards, with the rank's own piece in place, with one layer elsewhere, one source's layers at
    another distance, one piece of one layer in place and the last layer longer: to the bit, and nothing beside the outputs written."""
    print(layers, K, s1, cls, flush=True)
    rng = np.random.default_rng(layers * 11 + K + s1)
    es, dtype = 4 if cls else 2, torch.int32 if cls else torch.int16
    for form in ("up", "down", "own", "layer", "source", "piece", "longer"):
        own = K // 2
        lens = [s1] * layers
        if form == "longer":
            lens[-1] = s1 + 8
        plan = hzp.hzp_plan([1] * layers, [n * K for n in lens], align=8, z3=1, z1=K, tensor_class=[cls] * layers)
        assert [plan.bucket(l, cls).s1 for l in range(layers)] == lens
        step = s1 + 16
        room = step * (layers + 3)
        src = torch.from_numpy(rng.integers(0, 30000, (K, room)).astype(np.int32 if cls else np.int16)).to(DEV)
        out = torch.full((layers + 3, (s1 + 8) * K + 32), -1, dtype=dtype, device=DEV)
        order = list(range(layers))[::-1] if form == "down" else list(range(layers))
        if form == "layer":
            order[layers // 2] = layers + 1
        dsts = [out[order[l], 16:16 + lens[l] * K] for l in range(layers)]
        parts, expect = [], torch.full_like(out, -1)
        for l in range(layers):
            for k in range(K):
                at = order[l] * (step + (8 if form == "source" and k == 0 and 8 * layers <= 3 * step else 0))
                piece = src[k, at:at + lens[l]]
                if (form == "own" and k == own) or (form == "piece" and k == 0 and l == layers - 1):
                    place = dsts[l][k * lens[l]:(k + 1) * lens[l]]
                    place.copy_(piece)
                    parts.append(place)
                else:
                    parts.append(piece)
                expect[order[l], 16 + k * lens[l]:16 + (k + 1) * lens[l]] = piece
        before = src.clone()
        hzp.hzp_gather_layers(plan, 0, layers, cls, 1, parts, K, dsts)
        torch.cuda.synchronize()
        assert torch.equal(out, expect), form
        assert torch.equal(src, before), form
