"""The host-side plan of the streaming window kernels (kv::stream_plan): where segments outnumber the
chip's 256 CUs, one launch of longer segments or of workgroups of several is taken only if no CU then
streams more than two segments' keys.  The schedule is followed here on its own: workgroup i of a grid
goes to XCD i mod 8 (empty workgroups of short units counted), one workgroup to a CU, the CU that is
free first next."""
import ctypes
import heapq

import numpy as np
import pytest

from paper_2609_30738_amd import _lib

EVEN, ANY, WHOLE = 0, 1, 2  # kv::WgRule


class Shape(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("dtype", "n_prob", "h_q", "h_kv", "d", "w", "max_len")] + [
        ("lens", ctypes.c_void_p), ("tok_off", ctypes.c_void_p)]


class Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("seg_keys", "max_segs", "per_wg", "max_wgs")] + [
        ("n_wgs", ctypes.c_int64), ("ragged", ctypes.c_bool)]


def plan(lens, w, rule=EVEN, h_kv=8):
    f = _lib.lib()._ZN2kv11stream_planERKNS_5ShapeEPKiNS_6WgRuleE
    f.restype, f.argtypes = Plan, [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int]
    a = np.asarray(lens, dtype=np.int32)
    s = Shape(1, len(lens), 4 * h_kv, h_kv, 128, w, max(lens), None, None)
    return f(ctypes.addressof(s), a.ctypes.data, rule)


def even_segment(lens, w, h_kv=8):
    """One segment to a CU, in whole 256-key steps, at least 1024 keys at w = 32."""
    seg = -(-(-(-h_kv * sum(lens) // 256)) // 256) * 256
    least = 1024 if w == 32 or max(lens) <= 1024 else 256
    return min(max(least, seg), -(-max(lens) // 256) * 256)


def busiest_cu(lens, keys, seg, h_kv=8):
    ragged = len({-(-L // seg) for L in lens}) > 1  # then the grid's columns are odd
    wgs = -(-max(lens) // keys) | ragged
    xcds = [[] for _ in range(8)]
    for u in range(len(lens) * h_kv):
        left = lens[u // h_kv]
        for i in range(-(-left // keys)):
            xcds[(u * wgs + i) % 8].append(min(keys, left - i * keys))
    most = 0
    for queue in xcds:
        cus = [0] * 32
        for n in queue:
            most = max(most, heapq.heapreplace(cus, cus[0] + n) + n)
    return most


RAGGED = [(100001,) + (1000,) * 30, (60000,) + (2000,) * 3, (60000,) * 7 + (2000,) * 21, (30000,) * 14 + (3000,) * 14,
          (32000,) * 8 + (3000,) * 24, tuple(range(2000, 31000, 1200)), (5000, 3000, 700) * 9,
          (30000,) * 4 + (8000,) * 32, (4000,) * 10 + (600,) * 12, (60000,) + (700,) * 40]


@pytest.mark.parametrize("w", [8, 16, 32])
@pytest.mark.parametrize("lens", RAGGED, ids=lambda l: f"{len(l)}x{max(l)}")
def test_one_launch_leaves_no_cu_more_than_two_segments(lens, w):
    p, seg = plan(lens, w), even_segment(lens, w)
    n_even = sum(8 * -(-L // seg) for L in lens)
    keys = p.seg_keys * p.per_wg
    assert p.max_segs == -(-max(lens) // p.seg_keys) and p.max_wgs == -(-p.max_segs // p.per_wg)
    assert p.n_wgs == sum(8 * -(-L // keys) for L in lens)
    assert p.ragged == (len({-(-L // p.seg_keys) for L in lens}) > 1)
    if keys > seg and n_even > 256:  # a lengthened or several-segment plan
        assert busiest_cu(lens, keys, p.seg_keys) <= 2 * seg
    else:  # the even plan: fits the chip, or two launches
        assert (p.seg_keys, p.per_wg) == (seg, 1)


@pytest.mark.parametrize("w,layers,L,segs", [(32, 20, 14000, 2), (32, 10, 30000, 4), (32, 24, 5000, 2),
                                             (8, 20, 14000, 1), (16, 20, 2500, 1)])
def test_even_lengths_over_the_chip_take_one_launch(w, layers, L, segs):
    p = plan((L,) * layers, w)
    assert p.max_segs == segs and p.n_wgs <= 256
    assert p.per_wg == (2 if w == 32 else 1)


def test_rules_of_the_pruned_second_passes():
    """The candidate kernel takes whole units of up to three segments; a second pass that revisits few
    tiles takes as many segments to a workgroup as it takes to fit the chip."""
    assert plan((30000,) * 16, 32, WHOLE).max_wgs == 1
    lens = (100001,) + (1000,) * 30
    assert plan(lens, 32, ANY).n_wgs <= 256 and plan(lens, 32, ANY).per_wg > 2
    assert plan(lens, 32).per_wg == 1
