"""What the entry points launch, without a GPU: libhzp's host code with a stand-in for the HIP runtime that records launches
(tests/dispatch).  Calls that are captured and calls that are not are told apart by the stand-in's capture status; nothing runs."""
import ctypes
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
STREAM = 0x1000         # (any but the null stream, which cannot be captured)


def load(name, *path):
    spec = importlib.util.spec_from_file_location(name, os.path.join(ROOT, *path))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


class Recorder:
    """The binding over the recording build, and what that recorded."""

    def __init__(self):
        before = os.environ.get("HZP_LIBRARY")
        os.environ["HZP_LIBRARY"] = load("dispatch_build", "tests", "dispatch", "build.py").build()
        try:
            self.hzp = load("hzp_recorded", "paper_2510_20111_amd", "binding.py")
        finally:
            if before is None:
                del os.environ["HZP_LIBRARY"]
            else:
                os.environ["HZP_LIBRARY"] = before
        self.lib = self.hzp._L
        self.lib.recorded_kernel.restype = ctypes.c_char_p

    def launches(self, call, captured=False):
        """(kernel's name with its template arguments, grid, dynamic LDS) of each launch of `call`."""
        self.lib.forget()
        self.lib.set_capture(1 if captured else 0)
        try:
            call()
        finally:
            self.lib.set_capture(0)
        out = []
        for i in range(self.lib.recorded()):
            shape = (ctypes.c_uint * 4)()
            self.lib.recorded_shape(i, shape)
            name = self.lib.recorded_kernel(i).decode().replace("hzp::", "").replace("(anonymous namespace)::", "")
            out.append((name[:name.index("(")].removeprefix("void "), tuple(shape[:3]), shape[3]))
        return out


@pytest.fixture(scope="module")
def rec():
    return Recorder()


def test_tables_whose_copies_were_not_waited_for_are_not_used(rec):
    """The wait behind the tables' copies fails: so does the call that makes them, nothing is launched and nothing kept, and the next call
    makes them anew."""
    hzp = rec.hzp
    numel = [100] * 9
    plan = hzp.hzp_plan([9], numel, align=64, z3=1, z1=1)
    shard, tensors = 0x7000000000, [0x7100000000 + 4096 * t for t in range(9)]
    rec.lib.set_wait_status(719)
    try:
        for call in (lambda: plan.prepare(stream=STREAM), lambda: hzp.hzp_gather_layer(plan, 0, 0, 3, [shard], None, tensors, stream=STREAM)):
            with pytest.raises(hzp.HzpError) as caught:
                rec.launches(call)
            assert caught.value.status == hzp.HZP_ERR_HIP
            assert rec.lib.recorded() == 0 and rec.lib.live_allocations() == 0
    finally:
        rec.lib.set_wait_status(0)
    assert len(rec.launches(lambda: hzp.hzp_gather_layer(plan, 0, 0, 3, [shard], None, tensors, stream=STREAM))) == 1
    assert rec.lib.live_allocations() == 4
    del plan
    assert rec.lib.live_allocations() == 0


def test_calls_that_run_out_of_host_memory_end_with_a_status(rec):
    """Each host allocation of a call fails in turn: the call returns HZP_ERR_NOMEM (nothing is thrown through the C boundary), holds no
    device memory that it had not before, and works afterwards."""
    hzp = rec.hzp
    n = 300
    plan = hzp.hzp_plan([n, n], [700 + t % 5 for t in range(2 * n)], align=8, z3=2, z1=4)
    hy = hzp.adamw_hyper(1e-4, .9, .95, 1e-8, .1, 1.0, 1)
    at = lambda k: 0x7000000000 + k * 0x10000000
    tensors = [at(8) + 4096 * t + 2 for t in range(n)]
    calls = [lambda: plan.prepare(stream=STREAM),
             lambda: hzp.hzp_gather_layer(plan, 0, 0, 3, [at(0), at(1)], None, tensors, stream=STREAM),
             lambda: hzp.hzp_gather_layer(plan, 0, 0, 3, [at(0), at(1)], at(2), [t - 2 for t in tensors], stream=STREAM),
             lambda: hzp.hzp_gather_layers(plan, 0, 2, 0, 1, [at(0), at(1), at(2), at(3)], 2, [at(4), at(5)], stream=STREAM),
             lambda: hzp.hzp_adamw_shard(plan, 0, 2, 0, 0, hy, [at(0), at(1)], 1, *[[at(2 * i), at(2 * i + 1)] for i in range(1, 5)], stream=STREAM),
             lambda: hzp.hzp_reduce_shard(plan, 0, 0, 1, 0, [at(0), at(1)], 1.0, 0, at(2), stream=STREAM)]
    for call in calls:
        for which in range(1000):
            held = rec.lib.live_allocations()
            rec.lib.fail_host_allocation(which)
            try:
                call()
                failed = None
            except hzp.HzpError as error:
                failed = error
            if not rec.lib.host_allocation_failed():
                assert failed is None
                break
            assert failed is not None and failed.status == hzp.HZP_ERR_NOMEM and rec.lib.live_allocations() == held
        call()


def unpacking(rec, numel, both, place, z3=3, align=64, cls=0):
    """A plan of one bucket and the call that unpacks it: tensors as in the bucket ("placed"), at distances of their own ("near") or one of them
    off 16 bytes ("off")."""
    hzp, n, es = rec.hzp, len(numel), 4 if cls else 2
    plan = hzp.hzp_plan([n], numel, align=align, z3=z3, z1=z3, tensor_class=[cls] * n)
    plan.prepare(stream=STREAM)
    shards = [0x7000000000 + j * 0x40000000 for j in range(z3)]
    at = [plan.tensor(t).offset * es for t in range(n)]
    if place != "placed":
        at = [a + 4096 * t for t, a in enumerate(at)]
    if place == "off":
        at[n // 2] += es
    tensors = [0x7800000000 + a for a in at]
    return plan, lambda: hzp.hzp_gather_layer(plan, 0, cls, 3, shards, 0x7900000000 if both else None, tensors, stream=STREAM)


@pytest.mark.parametrize("place", ["placed", "near"])
@pytest.mark.parametrize("both", [False, True])
@pytest.mark.parametrize("numel", [[30000] * 9, [100, 90000] * 5, [600, 30000] * 30, [9000, 100] * 50, [300000] * 100, [400000] * 300])
def test_captured_unpacking_that_lists_serve_reads_nothing_of_the_plan(rec, numel, both, place):
    """What a graph of such a call reads is in its launches' arguments, so that it outlives the plan: no kernel that reads the spans.  (Where lists
    do not serve the plan's tables are read in any case.)"""
    plan, call = unpacking(rec, numel, both, place)
    names = [k for k, _, _ in rec.launches(call, captured=True)]
    assert names and all(k.startswith(("unpack_list_kernel", "copy_")) for k in names), names
    plan, call = unpacking(rec, [3000, 200] * 200, both, "placed")
    assert [k.split("<")[0] for k, _, _ in rec.launches(call, captured=True)] == ["unpack_placed_kernel"]


def name_of(kernel):
    return kernel.split("<")[0]


def streams_at(k, distance, odd=None):
    """k addresses at equal distances (contribution `odd` 16 bytes off)."""
    return [0x7000000000 + r * distance + (16 if r == odd else 0) for r in range(k)]


@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("g32", [0, 1])
@pytest.mark.parametrize("R", [1, 4, 8, 9, 12, 13, 16, 23, 24, 32])
def test_form_of_a_reduction(rec, R, g32, captured):
    """By size, type, number and distances of the contributions: from 13 equally distant ones their distance, up to 768 groups of 256 elements (fp32
    384); all pointers where the call is captured."""
    hzp, limit = rec.hzp, 384 if g32 else 768
    for groups in (1, limit, limit + 1):
        n = groups * 256 - 8
        plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1)
        for odd in (None, 1, R - 1):
            for distance in (n * 4, -n * 4, 1 << 40):
                def call():
                    hzp.hzp_reduce_shard(plan, 0, 0, 3, 0, streams_at(R, distance, odd), 0.5, 0, 0x6000000000, stream=STREAM,
                                         grad_dtype=hzp.HZP_GRAD_F32 if g32 else hzp.HZP_GRAD_BF16)
                (kernel, grid, _), = rec.launches(call, captured)
                even = R >= 13 and groups <= limit and odd is None and not captured
                assert (name_of(kernel) == "reduce_even_kernel") == even, (kernel, groups, odd, distance)
                assert even or name_of(kernel) in ("reduce_kernel", "reduce_block_kernel")
                assert grid[1:] == (1, 1) and ("<%du, %s, false" % (R, "true" if g32 else "false")) in kernel


@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("cls", [0, 1])
@pytest.mark.parametrize("R", [0, 1, 2, 3, 4, 5, 8, 9, 16, 32])
def test_form_of_an_update_of_one_segment(rec, R, cls, captured):
    """Equally distant contributions (up to two always are) by their distance: up to 2048 groups of 256 elements, 3 contributions and 4 bf16 ones up to
    1024, more than 8 up to 640; all pointers where the call is captured; with the scalars from the call and from device memory, with an output and
    without."""
    hzp, k = rec.hzp, max(R, 1)
    limit = 640 if R > 8 else 1024 if R == 3 or (R == 4 and not cls) else 2048
    hy = hzp.adamw_hyper(1e-4, .9, .95, 1e-8, .1, 1.0, 1)
    for groups in (1, limit, limit + 1):
        n = groups * 256 - 8
        plan = hzp.hzp_plan([1], [n], align=8, z3=1, z1=1, tensor_class=[cls])
        for odd in (None, R - 1):
            for distance in (n * 4, -n * 4, 1 << 40):
                for call, scal in ((hzp.hzp_adamw_shard, hy), (hzp.hzp_adamw_shard_dev, 0x5000000000)):
                    for out in ([0x6300000000], None):
                        (kernel, grid, _), = rec.launches(lambda: call(plan, 0, 1, cls, 0, scal, streams_at(k, distance, odd), R, [0x6000000000], [0x6100000000],
                                                                       [0x6200000000], out, stream=STREAM), captured)
                        even = groups <= limit and (odd is None or R < 3) and not captured
                        assert name_of(kernel) == ("fused_even_kernel" if even else "fused_one_kernel"), (kernel, groups, odd, distance)
                        assert grid == (groups, 1, 1) and kernel.split("<")[1].startswith("%du, " % k)


def spread(n, total):
    """n lengths of about `total` in all, every ninth 61 times the others."""
    weights = [61 if t % 9 == 3 else 1 for t in range(n)]
    return [max(1, total * w // sum(weights)) for w in weights]


# tensors' lengths, how they lie, with the bucket, shards: the kernel of an eager call (bf16; sizes are the bucket's)
UNPACKINGS = [
    ([200] * 5, "placed", False, 1, "unpack_list_kernel"),                  # 5 parts: the smallest list
    ([200] * 6, "placed", False, 1, "unpack_placed_kernel"),
    (spread(9, 60000), "placed", False, 3, "unpack_placed_kernel"),
    (spread(6, 4000), "near", False, 3, "unpack_near_kernel"),
    (spread(9, 140000), "near", False, 3, "unpack_near_kernel"),
    (spread(9, 280000), "off", False, 3, "unpack_list_kernel"),
    (spread(12, 140000), "near", False, 3, "unpack_near_kernel"),
    (spread(13, 280000), "near", False, 3, "unpack_list_kernel"),           # (from 1 MiB)
    (spread(13, 560000), "near", False, 3, "unpack_near_kernel"),
    (spread(64, 560000), "near", False, 8, "unpack_near_kernel"),
    (spread(65, 560000), "near", False, 8, "unpack_list_kernel"),
    (spread(9, 280000), "near", False, 9, "unpack_list_kernel"),            # more shards than an argument block holds
    (spread(9, 280000), "placed", False, 9, "unpack_list_kernel"),
    ([170000] * 12, "placed", False, 1, "unpack_placed_kernel"),            # even parts: 4.1 MB,
    ([180000] * 12, "placed", False, 1, "unpack_list_kernel"),              # 4.3 MB,
    ([2000] * 12, "near", False, 1, "unpack_near_kernel"),
    ([170000] * 12, "near", False, 1, "unpack_near_kernel"),
    ([180000] * 12, "near", False, 1, "unpack_list_kernel"),
    ([60000] * 13, "near", False, 1, "unpack_list_kernel"),
    ([3000] * 100, "placed", False, 1, "unpack_list_kernel"),
    (spread(100, 250000), "placed", False, 3, "unpack_list_kernel"),        # one launch of uneven parts: 0.5 MB,
    (spread(100, 280000), "placed", False, 3, "unpack_placed_kernel"),
    (spread(100, 2000000), "placed", False, 3, "unpack_placed_kernel"),     # 4 MB,
    (spread(100, 2200000), "placed", False, 3, "unpack_list_kernel"),
    (spread(400, 12000000), "placed", False, 3, "unpack_placed_kernel"),    # lists of three launches: 24 MB,
    (spread(400, 14000000), "placed", False, 3, "unpack_kernel"),           # 28 MB, by the tables
    ([200] * 2, "placed", True, 1, "unpack_placed_kernel"),                 # with the bucket, one pass of lists: any up to 4 MiB
    (spread(9, 2000000), "placed", True, 3, "unpack_placed_kernel"),
    (spread(9, 2200000), "placed", True, 3, "unpack_list_kernel"),
    (spread(80, 250000), "placed", True, 3, "unpack_list_kernel"),          # more than 64 tensors: 0.5 MB,
    (spread(80, 280000), "placed", True, 3, "unpack_placed_kernel"),
    (spread(9, 280000), "near", True, 3, "unpack_list_kernel"),
    ([100] * 200, "placed", True, 3, "unpack_placed_kernel"),               # (else two passes)
]


@pytest.mark.parametrize("numel,place,both,z3,kernel", UNPACKINGS)
def test_form_of_an_unpacking(rec, numel, place, both, z3, kernel):
    """Both sides of each line of the choice, eager and captured (lists where they serve); a grid is (tiles of a shard, shards) where the bucket
    is passed over, and (tiles, parts) or flat where lists are."""
    plan, call = unpacking(rec, numel, both, place, z3)
    (got, grid, _), = rec.launches(call)
    assert name_of(got) == kernel
    if kernel in ("unpack_placed_kernel", "unpack_near_kernel"):
        assert grid == (-(-plan.bucket(0).s3 // 512), z3, 1)
        few = len(numel) <= 64
        assert kernel == "unpack_near_kernel" or got == "unpack_placed_kernel<2, %s, %s>" % (str(both).lower(), str(few).lower())
    captured = rec.launches(call, captured=True)
    if kernel == "unpack_list_kernel":
        assert captured == [(got, grid, 0)]


def test_form_of_a_gather_of_equal_layers(rec):
    """Layers at equal distances in every source and in the outputs go by the first one's pieces, captured or not; else by lists."""
    hzp, layers, K, s1 = rec.hzp, 33, 4, 520
    plan = hzp.hzp_plan([1] * layers, [s1 * K] * layers, align=8, z3=1, z1=K)
    src = [0x7000000000 + k * 0x10000000 for k in range(K)]
    for captured in (False, True):
        for odd, stack in ((None, True), ("layer", False), ("source", False), ("piece", False), ("own", True)):
            dsts = [0x7800000000 + l * 8192 + (4096 if odd == "layer" and l == 9 else 0) for l in range(layers)]
            parts = [src[k] + l * (1072 if odd == "source" and k == 1 else 1056) for l in range(layers) for k in range(K)]
            for l in range(layers):
                if odd == "own" or (odd == "piece" and l == 9):
                    parts[l * K + 2] = dsts[l] + 2 * s1 * 2
            got = rec.launches(lambda: hzp.hzp_gather_layers(plan, 0, layers, 0, 1, parts, K, dsts, stream=STREAM), captured)
            names = {name_of(k) for k, _, _ in got}
            if stack:
                assert names == {"copy_stack_kernel"} and [g for _, g, _ in got] == [(-(-s1 // 512), K - (odd == "own"), layers)]
            else:
                assert names and "copy_stack_kernel" not in names
