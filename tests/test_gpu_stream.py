"""The kernels for launches of many tasks: the stream of KV-head pairs (one-launch, fused and
two-kernel routes) and the dense rectangular grid. The one-launch route streams from 2048 tasks
on (G = 8: from 769), the routes behind pkv_plan where 4 * B * Hkv is more than 768, or more
than 256 and up to 512 (G < 8), and the list itself is no shorter, so a small batch with a large task target is planned and
streamed in one launch and run task by task behind pkv_plan; both must agree bitwise.
Rectangular grids change kernels at 1536 and 6144 slots, and between 257 and 1535 at slots of
more than 16 pages."""
import numpy as np
import pytest
import torch

import paper_2606_26666_amd as pkv
from oracle import PlanParams, ref_decode, ref_plan
from tests.gpu_cases import Case, assert_close, plan_params, read_plan, run_decode, run_plan, run_rect

pytestmark = pytest.mark.gpu

HEADS = [(8, 8), (16, 8), (32, 8), (32, 4)]  # G = 1, 2, 4, 8


def bufs_for(case, split_max, rect_splits=0):
    return pkv.DecodeBuffers(case.B, case.hq, case.hkv, case.d, split_max, "cuda", rect_splits=rect_splits)


def one_launch(case, bufs, p, lens=None, bt=None):
    bufs.partial_region().fill_(0xFF)
    out = torch.full((case.B, case.hq, case.d), float("nan"), dtype=torch.float16, device="cuda")
    pkv.pkv_plan_decode(case.q_dev, case.k_dev, case.v_dev, case.bt_dev if bt is None else bt,
                        case.lens_dev if lens is None else lens, p, bufs.tasks, bufs.split_offsets, bufs.num_tasks, 1.0,
                        out, bufs.ws)
    return out


def planned(case, split_max, p, fused=True):
    bufs = bufs_for(case, split_max)
    run_plan(case, bufs, p)
    out = run_decode(case, bufs, fused=fused)
    tasks, offs = read_plan(bufs)
    assert pkv.pkv_check_device_status(bufs.ws) == 0
    return out, tasks, offs


def lengths(kind, rng):
    if kind == "edges":        # one token, one page, one tile, and one more or less of each; empty rows
        return [1, 16, 17, 0, 33, 127, 257, 128]
    if kind == "ragged":
        return rng.integers(0, 3000, size=8)
    return [40000, 13, 20001, 0, 5000]   # "long": several blocks of 64 page ids per wave


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("kind,split_max,target", [("edges", 64, 4096), ("ragged", 64, 2048), ("ragged", 64, 6000),
                                                   ("ragged", 1, 2048), ("long", 1, 2048), ("long", 200, 6400)])
def test_stream_matches_one_task_kernels(hq, hkv, kind, split_max, target):
    """Few and many rounds of units (strided and weighted ranges), single-page units, waves
    without pages, rows with one split (written at once) and with more than 64; the second and third call start from the first's task list."""
    case = Case(lengths(kind, np.random.Generator(np.random.PCG64(71))), hq=hq, hkv=hkv, seed=71)
    assert 4 * case.B * hkv <= 256  # behind pkv_plan these run task by task
    p = plan_params(hkv, 1, split_max, target, policy=1)
    expect, tasks_ref, offs_ref = planned(case, split_max, p)
    bufs = bufs_for(case, split_max)
    for rep in range(3):
        out = one_launch(case, bufs, p)
        tasks, offs = read_plan(bufs)
        assert np.array_equal(tasks, tasks_ref) and np.array_equal(offs, offs_ref), rep
        assert torch.equal(out, expect), rep
    assert_close(out, ref_decode(case.q, case.k, case.v, case.bt, case.lens), f"{kind} G={hq // hkv}")
    assert pkv.pkv_check_device_status(bufs.ws) == 0


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("B,target", [(64, 2100), (64, 9000), (65, 9000), (400, 40000)])
def test_stream_of_large_batches(hq, hkv, B, target):
    """Both planners (64 rows and more), fused and two-kernel merges over streamed states, more
    units per workgroup than one stream holds (32; the 400 rows), and batches whose lengths change between calls on one workspace (stale hints)."""
    rng = np.random.Generator(np.random.PCG64(72))
    lens = rng.integers(0, 500, size=B).astype(np.int32)
    lens[::7] = 0
    case = Case(lens + 40, hq=hq, hkv=hkv, seed=72)
    p = plan_params(hkv, 1, 16, target, policy=1)
    bufs = bufs_for(case, 16)
    for step in range(3):
        case.lens = np.maximum(lens + 17 * step, 0).astype(np.int32)
        case.lens[step::5] = 0
        case.lens_dev = torch.from_numpy(case.lens).cuda()
        out = one_launch(case, bufs, p)
        tasks, offs = read_plan(bufs)
        ref = ref_plan(case.lens, PlanParams(p.page_size, p.tile_tokens, hkv, 1, 16, target, 1),
                       max_pages_per_row=case.bt.shape[1])
        assert np.array_equal(tasks, ref[0]) and np.array_equal(offs, ref[1]), step
        fused, _, _ = planned(case, 16, p)
        two, _, _ = planned(case, 16, p, fused=False)
        assert torch.equal(out, fused) and torch.equal(out, two), step
    assert_close(out, ref_decode(case.q, case.k, case.v, case.bt, case.lens), f"B={B} G={hq // hkv}")
    assert pkv.pkv_check_device_status(bufs.ws) == 0


def own_list(lens, hkv, splits, apart):
    """A task list in a plan's order with the caller's own ranges: rows where `apart` are cut at other
    tokens for every second KV head."""
    tasks, offsets = [], [0]
    for row, n in enumerate(lens.tolist()):
        ns = min(splits, -(-n // 16))
        for s in range(ns):
            for h in range(hkv):
                shift = 16 if apart[row] and h % 2 else 0
                cut = [min(n, (i * n // ns) // 16 * 16 + shift * (0 < i < ns)) if i < ns else n for i in (s, s + 1)]
                tasks.append((row, h, s, cut[0], cut[1]))
        offsets.append(offsets[-1] + ns)
    return np.array(tasks, dtype=np.int32), np.array(offsets, dtype=np.int32)


def put_list(bufs, tasks, offsets):
    bufs.tasks[: len(tasks)] = torch.from_numpy(tasks).cuda()
    bufs.split_offsets.copy_(torch.from_numpy(offsets))
    bufs.num_tasks.fill_(len(tasks))


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("kind", ["plan", "some", "all", "short"])
def test_lists_of_the_callers_own(hq, hkv, kind):
    """Behind pkv_plan, lists in a plan's order whose neighbours are not always KV heads g and g + 1 of
    one range (none, some rows, all), and a list far shorter than the batch lets expect: against the
    oracle, fused and two-kernel bitwise alike."""
    rng = np.random.Generator(np.random.PCG64(77))
    B = 120
    lens = rng.integers(300, 900, size=B).astype(np.int32)
    if kind == "short":
        lens[5:] = 0
    case = Case(lens, hq=hq, hkv=hkv, seed=77)
    apart = {"plan": np.zeros(B), "some": rng.random(B) < 0.2, "all": np.ones(B), "short": np.ones(B)}[kind]
    tasks, offsets = own_list(case.lens, hkv, 4, apart)
    assert 4 * B * hkv > 768 and (len(tasks) > 768) == (kind != "short")
    bufs = bufs_for(case, 4)
    put_list(bufs, tasks, offsets)
    fused, two = run_decode(case, bufs), run_decode(case, bufs, fused=False)
    assert torch.equal(fused, two)
    assert_close(fused, ref_decode(case.q, case.k, case.v, case.bt, case.lens), f"{kind} G={hq // hkv}")
    assert torch.equal(run_decode(case, bufs), fused)
    assert pkv.pkv_check_device_status(bufs.ws) == 0


@pytest.mark.parametrize("fused", [True, False])
def test_records_that_are_no_tasks_are_flagged(fused):
    """Records outside the batch in a list long enough to stream: flagged, the other rows unchanged, and
    the workspace usable again once the status has been read."""
    case = Case(np.full(60, 500, dtype=np.int32), seed=78)
    tasks, offsets = own_list(case.lens, 8, 4, np.zeros(60))
    assert len(tasks) > 768
    bufs = bufs_for(case, 4)
    put_list(bufs, tasks, offsets)
    clean = run_decode(case, bufs, fused=fused)
    for at, word, value in [(100, 0, 60), (101, 0, -1), (333, 1, 8), (800, 3, -16), (900, 4, 1 << 20), (901, 4, 0)]:
        bad = tasks.copy()
        bad[at, word] = value
        put_list(bufs, bad, offsets)
        out = run_decode(case, bufs, fused=fused)
        assert pkv.pkv_check_device_status(bufs.ws) & pkv.PKV_DEVERR_TASK
        ok = [r for r in range(60) if r != tasks[at, 0]]
        assert torch.equal(out[ok], clean[ok]), (at, word)
    put_list(bufs, tasks, offsets)
    assert torch.equal(run_decode(case, bufs, fused=fused), clean)
    assert pkv.pkv_check_device_status(bufs.ws) == 0


def test_stream_flags_a_bad_page_of_one_row():
    """A page id outside the pool, in the hinted first units and elsewhere: flagged, that row's
    output zero, every other row bitwise the clean call's."""
    lens = np.full(20, 700, dtype=np.int32)
    case = Case(lens, seed=73)
    p = plan_params(8, 1, 16, 2048, policy=1)
    bufs = bufs_for(case, 16)
    clean = one_launch(case, bufs, p)
    for row in (0, 11, 19):
        bt = case.bt_dev.clone()
        bt[row, 13] = case.num_pages + 5
        out = one_launch(case, bufs, p, bt=bt)
        assert pkv.pkv_check_device_status(bufs.ws) & pkv.PKV_DEVERR_PAGE_ID
        assert torch.all(out[row] == 0)
        keep = [i for i in range(case.B) if i != row]
        assert torch.equal(out[keep], clean[keep]), row
    assert torch.equal(one_launch(case, bufs, p), clean)
    assert pkv.pkv_check_device_status(bufs.ws) == 0


@pytest.mark.parametrize("hq,hkv,B,S", [(8, 8, 12, 16), (32, 8, 12, 16), (32, 4, 26, 15), (16, 8, 48, 16),
                                        (32, 8, 48, 16), (64, 8, 48, 16), (12, 3, 40, 13), (12, 3, 64, 33)])
def test_dense_rectangular_grid(hq, hkv, B, S):
    """1536 slots and more (one per workgroup), 6144 and more (two, for an even number of KV
    heads), empty splits and rows: bitwise the workqueue at the same split count."""
    rng = np.random.Generator(np.random.PCG64(74))
    lens = rng.integers(0, 1200, size=B).astype(np.int32)
    lens[1::6] = 0
    lens[0] = 9000
    case = Case(lens, hq=hq, hkv=hkv, seed=74)
    assert B * hkv * S >= 1536
    bufs = bufs_for(case, S, rect_splits=S)
    run_plan(case, bufs, plan_params(hkv, S, S, 1))
    expect = run_decode(case, bufs)
    rect = run_rect(case, bufs, S)
    assert torch.equal(rect, expect)
    assert_close(rect, ref_decode(case.q, case.k, case.v, case.bt, case.lens), f"rect B={B} S={S}")
    assert pkv.pkv_check_device_status(bufs.ws) == 0


@pytest.mark.parametrize("extra", [-1, 0, 1])
@pytest.mark.parametrize("hq,hkv,B,S", [(8, 8, 5, 16), (16, 8, 3, 11), (32, 8, 3, 11), (32, 8, 11, 17), (64, 8, 5, 16),
                                        (12, 3, 9, 12)])
def test_short_rectangular_slots_in_pairs(hq, hkv, B, S, extra):
    """257 to 1535 slots of at most 16 pages (32-token tiles: rows of 256 S tokens) run as pairs
    of KV heads (G <= 4, even Hkv); one token more and they run one by one. Empty rows and
    splits, whole batch and length buckets: bitwise the workqueue at the same split count."""
    rng = np.random.Generator(np.random.PCG64(76))
    lens = rng.integers(0, 700, size=B).astype(np.int32)
    lens[0] = 256 * S + extra
    lens[1] = 0
    lens[2] = 17
    case = Case(lens, hq=hq, hkv=hkv, seed=76)
    assert 256 < B * hkv * S < 1536
    bufs = bufs_for(case, S, rect_splits=S)
    p = plan_params(hkv, S, S, 1)
    run_plan(case, bufs, p)
    expect = run_decode(case, bufs)
    assert torch.equal(run_rect(case, bufs, S), expect)
    out = torch.full_like(expect, float("nan"))
    pkv.pkv_decode_buckets(case.q_dev, case.k_dev, case.v_dev, case.bt_dev, case.lens_dev, case.lens, 8192, p, 1.0, out,
                           bufs.ws)
    assert torch.equal(out, expect)
    assert_close(expect, ref_decode(case.q, case.k, case.v, case.bt, case.lens), f"rect B={B} S={S}")
    assert pkv.pkv_check_device_status(bufs.ws) == 0


@pytest.mark.parametrize("hq,hkv", HEADS)
@pytest.mark.parametrize("target", [256, 2048])
def test_many_small_weights_add_up(hq, hkv, target):
    """One token holds the maximum and 40000 others have 2^-26 of its weight each, all with
    V = 1 where the first has 0: the output is their share, 6.0e-4. At G = 4 and 8 weights enter
    the product in fp16, which ends at 2^-24, so they are only seen if they are scaled. Bound: the
    output's own fp16 rounding (2^-11) and 2^-13 (a weight's error is 2^-39 of the largest one,
    2^-13 of itself); at G = 1 and 2, fp32 weights, the first alone would do."""
    n = 40001
    case = Case([n], hq=hq, hkv=hkv, seed=75)
    k = torch.zeros_like(case.k_dev)
    v = torch.zeros_like(case.v_dev)
    pages = case.bt_dev[0].long()
    k[pages, :, :, 0] = -26.0 * float(np.log(2.0))
    v[pages] = 1.0
    k[pages[0], 0, :, 0] = 0.0
    v[pages[0], 0] = 0.0
    q = torch.zeros_like(case.q_dev)
    q[:, :, 0] = 1.0
    case.k_dev, case.v_dev, case.q_dev = k, v, q
    p = plan_params(hkv, 1, 64, target, policy=1)
    out = one_launch(case, bufs_for(case, 64), p).double()
    w = float(np.exp(np.float64(k[pages[1], 0, 0, 0].item())))
    ref = 40000 * w / (1 + 40000 * w)
    assert float((out - ref).abs().max()) <= ref * (2.0 ** -11 + 2.0 ** -13)


@pytest.mark.parametrize("side", [False, True])
def test_calls_go_to_the_current_stream(side):
    """The stream a call uses when none is given is torch's current one."""
    from paper_2606_26666_amd import _binding

    s = torch.cuda.Stream() if side else torch.cuda.current_stream()
    with torch.cuda.stream(s):
        assert _binding._stream(None) == s.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert _binding._stream(s) == s.cuda_stream
