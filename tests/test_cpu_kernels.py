"""The kernels' own sources on the CPU (tests/cpu_device): synchronisation, by schedules that let
one wave run as far ahead of the others as the barriers allow, and forms of calls compared with the
oracle. Every access is bounds checked. One or two workgroups stand for the device, so a few dozen
tasks reach what takes thousands on 256 compute units."""
import numpy as np
import pytest

from oracle import ref_decode
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
