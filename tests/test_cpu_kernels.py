"""The kernels' own sources on the CPU (tests/cpu_device): synchronisation, by schedules that let
one wave run as far ahead of the others as the barriers allow, and forms of calls compared with the
oracle. Every access is bounds checked. One or two workgroups stand for the device, so a few dozen
tasks reach what takes thousands on 256 compute units."""
import numpy as np
import pytest

from oracle import ref_decode
from paper_2606_26666_amd import costmodel
from tests import cpu_cases
from tests.cpu_cases import ASCENDING, DESCENDING, Call

HEADS = [(2, 2), (4, 2), (8, 2), (16, 2)]  # G = 1, 2, 4, 8
SCHEDULES = [ASCENDING, DESCENDING, 12345]
PAGE_ID, TASK = 2, 4  # device error bits

pytestmark = pytest.mark.skipif(cpu_cases.compiler() is None, reason="needs clang")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return cpu_cases.Program(cpu_cases.build(str(tmp_path_factory.mktemp("cpu_device"))))


def params(hkv, split_max=4, target=64, split_min=1, policy=1, tile=32):
    return (16, tile, hkv, split_min, split_max, target, policy)


def reference(c, call=0):
    return ref_decode(c.q, c.k, c.v, c.bt, c.lens[call])


def close(out, ref, what=""):
    """fp16 outputs of fp32 sums: half an fp16 unit of the value, and 2^-20 of the largest."""
    err = np.abs(out.astype(np.float64) - ref)
    assert np.all(err <= np.abs(ref) * 2.0 ** -11 + np.abs(ref).max() * 2.0 ** -20 + 2.0 ** -25), (what, err.max())


def kernels(launched):
    return [k for k, _ in launched]


@pytest.mark.parametrize("order", SCHEDULES)
@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("route", ["separate", "fused", "plan_decode"])
def test_more_units_than_one_stream_holds(program, route, hq, hkv, order):
    """One workgroup, 70 units, 32 to a stream: the records of the next stream go where the
    last one's lie, so no wave may still be reading those."""
    c = Call([1 + (7 * i) % 32 for i in range(70)], hq=hq, hkv=hkv, seed=3)
    (a,), launched = c.run(program, route, params(hkv, target=700), order=order, compute_units=1)
    assert any(k.startswith("stream_kernel") for k in kernels(launched)), launched
    assert a.status == 0 and a.error_bits == 0 and a.counters_left == 0 and a.num_tasks == 70 * hkv
    close(a.out, reference(c), f"{route} G={hq // hkv}")


@pytest.mark.parametrize("order", SCHEDULES)
@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("page", [0, 3, 7])
def test_bad_page_of_a_hinted_unit_is_kept(program, hq, hkv, page, order):
    """The second call starts from the first one's list, so each wave reads its first page of unit 0
    while the plan is formed: a page id outside the pool is flagged then, and the row is zero.
    With wave 0 last, the waves that set the flag are past it when wave 0 begins."""
    lens = [128] * 6 + [40]
    c = Call([lens, lens], hq=hq, hkv=hkv, seed=4)
    c.bt[0, page] = c.num_pages + 3
    answers, launched = c.run(program, "plan_decode", params(hkv, split_max=1), order=order, compute_units=2)
    assert kernels(launched)[0].startswith("stream_kernel"), launched
    bt = c.bt.copy()
    bt[0, page] = 0
    ref = ref_decode(c.q, c.k, c.v, bt, c.lens[0])
    for n, a in enumerate(answers):
        assert a.error_bits == PAGE_ID and a.counters_left == 0, (n, a.error_bits)
        assert np.all(a.out[0] == 0), n
        close(a.out[1:], ref[1:], n)


def route_args(route, hkv):
    return dict(S=3) if route == "rect" else dict(bucket_tokens=32) if route == "buckets" else {}


@pytest.mark.parametrize("route", ["plan_decode", "fused", "separate", "rect"])
@pytest.mark.parametrize("hq,hkv", [(2, 2), (4, 2), (3, 3), (6, 3)])
def test_infinite_values_stay_infinite(program, hq, hkv, route):
    """One query head per KV head, or two: an infinite V with a positive weight is an infinite output,
    whatever the weight's bits, and no other dimension sees it."""
    c = Call([70, 33], hq=hq, hkv=hkv, seed=5)
    at = {(0, 0, 3): np.inf, (0, 37, 64): -np.inf, (1, 32, 127): np.inf}  # row, token, dim
    for (row, tok, dim), x in at.items():
        c.v[c.bt[row, tok // 16], tok % 16, :, dim] = x
    (a,), _ = c.run(program, route, params(hkv, split_max=3), **route_args(route, hkv))
    seen = np.zeros(a.out.shape, dtype=bool)
    for (row, _, dim), x in at.items():
        assert np.all(a.out[row, :, dim] == x), (row, dim, a.out[row, :, dim])
        seen[row, :, dim] = True
    v, c.v = c.v, np.where(np.isinf(c.v), np.float16(0), c.v)
    ref = reference(c)
    assert np.all(np.isfinite(a.out[~seen]))
    close(np.where(seen, ref, a.out), ref)


@pytest.mark.parametrize("route", ["plan_decode", "separate", "rect"])
@pytest.mark.parametrize("hq,hkv", HEADS)
def test_small_weights(program, hq, hkv, route):
    """One token has the largest weight and V = 0, 62 others about 2^-30 of it and V = 65504: the
    output is their share, 3.4e-3. With one or two query heads the weights are fp32 throughout. With
    more they enter the product as fp16 halves of 2^14 times the weight, with an error of at most
    2^-39 of the largest weight each."""
    n = 63
    c = Call([n], hq=hq, hkv=hkv, seed=6)
    c.k[:], c.q[:] = 0, 0
    c.q[:, :, 0] = 1
    pages = c.bt[0, : (n + 15) // 16]
    c.k[pages, :, :, 0] = np.float16(-20.95)
    c.v[pages] = 65504
    c.k[pages[0], 0, :, 0] = 0
    c.v[pages[0], 0] = 0
    (a,), _ = c.run(program, route, params(hkv, split_max=2), **route_args(route, hkv))
    w = np.exp(np.float64(np.float16(-20.95)))
    ref = 62 * w * 65504 / (1 + 62 * w)
    bound = ref * (2.0 ** -11 + 2.0 ** -20) + (0 if hq // hkv <= 2 else 62 * 65504 * 2.0 ** -39)
    assert np.abs(a.out.astype(np.float64) - ref).max() <= bound


@pytest.mark.parametrize("route", ["fused", "separate"])
@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("lens", [[0, 0, 0, 0, 70, 0], [90, 0, 0, 1, 0, 0], [70, 400, 0, 0, 0, 0], [33] * 5 + [0]])
def test_short_lists_where_long_ones_stream(program, route, hq, hkv, lens):
    """Six rows are expected to have 48 tasks or more, so the stream kernel is launched; empty and
    short rows leave one to six rounds of them on two workgroups, which run one by one where a stream
    would leave a workgroup idle. The same bits as from the one-task kernels (many workgroups)."""
    c = Call([lens, lens], hq=hq, hkv=hkv, seed=7)
    p = params(hkv, split_max=3, target=12)
    for order in SCHEDULES:
        answers, launched = c.run(program, route, p, order=order, compute_units=2)
        assert any(k.startswith("stream_kernel") for k in kernels(launched)), launched
        one, launched = c.run(program, route, p, compute_units=64)
        assert any(k.startswith("split_kernel") for k in kernels(launched)), launched
        for a, b in zip(answers, one):
            assert a.error_bits == 0 and a.counters_left == 0
            assert np.array_equal(a.out.view(np.uint16), b.out.view(np.uint16))
        close(answers[0].out, reference(c))


def own_list(lens, hkv, splits, apart, rng):
    """A task list in a plan's order (row, split, KV head) with the caller's own ranges: rows named in
    `apart` are cut at other tokens for every KV head, the others alike."""
    tasks, offsets = [], [0]
    for row, n in enumerate(lens):
        ns = min(splits, n)
        cuts = []
        for h in range(hkv):
            if h == 0 or row in apart:
                c = sorted(rng.choice(np.arange(1, n), size=ns - 1, replace=False).tolist()) if ns > 1 else []
                c = [x // 16 * 16 for x in c] if len({x // 16 for x in c} - {0}) == len(c) else [16 * (i + 1) for i in range(ns - 1)]
            cuts.append([0] + c + [n])
        for s in range(ns):
            tasks += [(row, h, s, cuts[h][s], cuts[h][s + 1]) for h in range(hkv)]
        offsets.append(offsets[-1] + ns)
    return np.array(tasks, dtype=np.int32), np.array(offsets, dtype=np.int32)


@pytest.mark.parametrize("order", [ASCENDING, DESCENDING])
@pytest.mark.parametrize("route", ["fused", "separate"])
@pytest.mark.parametrize("hq,hkv,splits", [(2, 2, 3), (4, 2, 1), (16, 4, 3), (16, 2, 2), (8, 2, 70)])
def test_lists_of_the_callers_own(program, route, hq, hkv, splits, order):
    """Task lists whose neighbours are not KV heads g and g + 1 of one range, in some rows or in all:
    the stream runs those tasks one head at a time, with the bits of the one-task kernels."""
    long = splits > 64
    lens = [1200, 1300] if long else [100 + (13 * i) % 60 for i in range(40 if splits == 1 else 14)]
    c = Call(lens, hq=hq, hkv=hkv, seed=8)
    rng = np.random.Generator(np.random.PCG64(8))
    for apart in ([1], range(len(lens)), [0, 2, 13, 33]):
        given = own_list(lens, hkv, splits, set(apart), rng)
        p = params(hkv, split_max=max(splits, 4))
        (a,), launched = c.run(program, route, p, given=given, order=order, compute_units=2)
        assert any(k.startswith("stream_kernel") for k in kernels(launched)), launched
        (b,), launched = c.run(program, route, p, given=given, compute_units=512)
        assert any(k.startswith("split_kernel") for k in kernels(launched)), launched
        assert a.error_bits == b.error_bits == 0 and a.counters_left == 0
        assert np.array_equal(a.out.view(np.uint16), b.out.view(np.uint16))
        close(a.out, reference(c), route)


@pytest.mark.parametrize("cut", [1, 2, 3])
def test_a_list_cut_short(program, cut):
    """The two-kernel route stores the state of every task that is listed, an odd last one too."""
    lens = [120] * 12
    c = Call(lens, hq=8, hkv=2, seed=9)
    tasks, offsets = own_list(lens, 2, 2, set(), np.random.Generator(np.random.PCG64(9)))
    keep = len(tasks) - cut
    (a,), launched = c.run(program, "separate", params(2), given=(tasks, offsets), num_tasks=keep, compute_units=2)
    assert any(k.startswith("stream_kernel") for k in kernels(launched)), launched
    missing = {(r, h) for r, h, *_ in tasks[keep:].tolist()}
    ref = reference(c).reshape(12, 2, 4, 128)
    out = a.out.reshape(12, 2, 4, 128)
    for row in range(12):
        for h in range(2):
            if (row, h) not in missing:
                close(out[row, h], ref[row, h], (row, h))


@pytest.mark.parametrize("compute_units", [2, 64])
@pytest.mark.parametrize("route", ["fused", "separate"])
def test_records_that_are_no_tasks_are_flagged(program, route, compute_units):
    """Rows, heads and ranges outside the batch, as one record of a pair and as both; split_offsets
    past the capacity: flagged, nothing outside the buffers touched, and the rows without one right."""
    lens = [120] * 12
    c = Call(lens, hq=8, hkv=2, seed=10)
    tasks, offsets = own_list(lens, 2, 2, set(), np.random.Generator(np.random.PCG64(9)))
    ref = reference(c)
    for at, word, value in [(4, 0, 99), (5, 0, -1), (9, 1, 2), (8, 1, -3), (12, 3, -16), (13, 4, 1 << 20), (20, 4, 0)]:
        for both in (False, True):
            bad = tasks.copy()
            bad[at, word] = value
            if both:
                bad[at ^ 1, word] = value + (word == 1)
            (a,), _ = c.run(program, route, params(2), given=(bad, offsets), compute_units=compute_units)
            assert a.error_bits & TASK, (at, word)
            ok = [r for r in range(12) if r != tasks[at, 0]]
            close(a.out[ok], ref[ok], (at, word, both))
    wrong = offsets.copy()
    wrong[6:] += 1 << 24
    (a,), _ = c.run(program, route, params(2), given=(tasks, wrong), compute_units=compute_units)
    assert a.error_bits & TASK
    close(a.out[:5], ref[:5])


@pytest.mark.parametrize("hq,hkv", HEADS + [(3, 3), (12, 3)])
@pytest.mark.parametrize("S,longest", [(2, 600), (4, 300), (9, 300)])
def test_rectangular_kernels(program, hq, hkv, S, longest):
    """Pairs of heads, the dense kernel and both together are chosen by slots per compute unit of the
    device, and give the bits of one slot per workgroup; empty splits and rows, named rows."""
    lens = [longest, 1, 0, 33, 17, 200]
    c = Call(lens, hq=hq, hkv=hkv, seed=11)
    seen = set()
    base = None
    for compute_units in (256, 16, 8, 3, 1):
        (a,), launched = c.run(program, "rect", params(hkv), S=S, order=DESCENDING, compute_units=compute_units)
        seen.add(kernels(launched)[0].split("<")[0] + kernels(launched)[0][-3:])
        base = a.out if base is None else base
        assert a.status == 0 and a.error_bits == 0
        assert np.array_equal(a.out.view(np.uint16), base.view(np.uint16)), (compute_units, launched)
        (b,), _ = c.run(program, "rect", params(hkv), S=S, row_ids=[5, 0, 2], compute_units=compute_units)
        assert np.array_equal(b.out[[5, 0, 2]].view(np.uint16), base[[5, 0, 2]].view(np.uint16))
    close(base, reference(c))
    assert len(seen) >= 2 or (hkv % 2 and hq // hkv <= 2 and longest > 256 * S), seen  # long slots, odd head: one by one


@pytest.mark.parametrize("route,name", [("plan_decode", "one-launch"), ("fused", "plan+fused"), ("separate", "two-kernel")])
@pytest.mark.parametrize("hq,hkv,B", [(2, 2, 9), (4, 4, 17), (8, 2, 33), (32, 4, 20), (32, 4, 49), (3, 3, 70), (16, 2, 97)])
def test_reported_heads_per_workgroup(program, route, name, hq, hkv, B):
    """What the benchmark reports of a launch on 256 compute units, against the kernel that is launched
    there (pairs and streams read two heads)."""
    c = Call([1] * B, hq=hq, hkv=hkv, seed=12)
    for target in (256, 511, 512, 768, 769, 2047, 2048):
        _, launched = c.run(program, route, params(hkv, split_max=1, target=target, policy=0), compute_units=256)
        kernel = [k for k in kernels(launched) if k.startswith(("split_kernel", "stream_kernel"))][0]
        two = kernel.startswith("stream") or kernel.endswith(" 2>")
        tasks = 10 ** 6  # the launch: the host's part of the rule
        assert costmodel.heads_per_workgroup(name, hq, hkv, B, target, tasks) == 1 + two, (target, kernel)
        if name != "one-launch":
            break
    assert costmodel.heads_per_workgroup("rect", hq, hkv, B, 4096, 0) == 1
    assert costmodel.heads_per_workgroup("plan+fused", 32, 8, 64, 2048, 256) == 1  # a short list runs task by task
