"""How a restore is launched (restore_launch in plan.cpp): which rows are stored at device scope, in which start order and
at what residency, by the plan's sizes and the caches' addresses."""
import ctypes
import dataclasses

import numpy as np
import pytest

from paper_2609_26219_amd import binding as pb
from paper_2609_26219_amd import workloads as wl

MIXED, K8V4, K4V4 = (1, 2, 7, 0), (0, 0, 1, 0), (0, 0, 0, 1)


def restore_launch(case, layers=0, k=0, v=0):
    fn = pb.load().pkv_internal_restore_launch
    fn.argtypes = [ctypes.POINTER(pb.PkvModel), ctypes.POINTER(pb.PkvRequest), ctypes.c_int32, ctypes.c_int64,
                   ctypes.c_uint64, ctypes.c_uint64, ctypes.c_void_p]
    fn.restype = ctypes.c_int32
    m, reqs, out = pb.make_model(case.shape), pb._Requests(case.requests), np.zeros(5, np.int64)
    assert fn(ctypes.byref(m), reqs.array, reqs.count, layers, k, v, out.ctypes.data) == 0
    return dict(zip(("per_cu", "late", "one_round", "device", "single"), out.tolist()))


def make(H, D, B=32, P=16, tokens=4096, L=1, mix=MIXED, delta=-700, paired=False, style=wl.ROPE_HALF, rotary=0):
    case = wl.make_custom(5, L=L, H=H, D=D, B=B, P=P, n_tokens=(tokens,), deltas=(delta,), rho0s=(max(0, 2000 - delta),),
                          tag_set=(0, 1, 2, 3), mix=mix, repair_frac=0.1, out_dtype=wl.OUT_BF16)
    case.shape = dataclasses.replace(case.shape, rope_style=style, rotary_dim=rotary,
                                     kv_layout=wl.KV_PAIRED if paired else wl.KV_SEPARATE)
    return case


@pytest.mark.parametrize("offset,device", [(0, 1), (16, 0), (32, 0), (48, 0), (64, 1)])
def test_device_scope_by_address(offset, device):
    """Either cache inside a 64-byte sector would be written through in parts of sectors."""
    case = make(8, 128)
    assert restore_launch(case, k=1 << 20, v=(1 << 21) + offset)["device"] == device
    assert restore_launch(case, k=(1 << 20) + offset, v=1 << 21)["device"] == device


@pytest.mark.parametrize("args,device", [
    (dict(H=8, D=96), 0), (dict(H=8, D=80), 0), (dict(H=1, D=256), 1),
    # one-row units, below 2 KB and from there on
    (dict(H=7, D=128, P=1), 0), (dict(H=7, D=128, P=2), 1), (dict(H=7, D=128, B=1, tokens=256), 0), (dict(H=8, D=128, P=1), 1),
    (dict(H=2, D=128, rotary=32), 0), (dict(H=2, D=128, rotary=32, style=wl.ROPE_INTERLEAVED), 1),
    # pieces of half a line: 8 x 64, 26 layers of 4096 tokens write 196 MB
    (dict(H=8, D=64, L=26), 0), (dict(H=8, D=64, L=26, mix=K8V4), 1), (dict(H=8, D=64, L=26, mix=K4V4), 1),
    (dict(H=8, D=64, L=26, delta=0), 1), (dict(H=8, D=64, L=8), 1), (dict(H=8, D=64, L=26, paired=True), 0),
    (dict(H=4, D=128, rotary=64, L=26), 0), (dict(H=4, D=128, rotary=64, L=26, style=wl.ROPE_INTERLEAVED), 1),
])
def test_device_scope_by_rows(args, device):
    assert restore_launch(make(**args))["device"] == device


def test_device_scope_by_launch_size():
    """The streamed restore launches a layer at a time: what counts is the launch."""
    case = make(8, 64, L=26)
    assert restore_launch(case)["device"] == 0 and restore_launch(case, layers=1)["device"] == 1


@pytest.mark.parametrize("args,single", [(dict(H=8, D=128, P=1), 1), (dict(H=8, D=128, B=1, tokens=64), 1),
                                         (dict(H=8, D=128, P=2), 0), (dict(H=32, D=128, B=64, P=1), 1)])
def test_single_rows(args, single):
    """Work items of one row, which load their launch arguments piece by piece."""
    assert restore_launch(make(**args))["single"] == single


def _units(case):
    lib, n = pb.load(), ctypes.c_int64()
    m, reqs = pb.make_model(case.shape), pb._Requests(case.requests)
    lib.pkv_internal_host_units.argtypes = [ctypes.POINTER(pb.PkvModel), ctypes.POINTER(pb.PkvRequest), ctypes.c_int32,
                                            ctypes.c_void_p, ctypes.c_int64, ctypes.POINTER(ctypes.c_int64)]
    assert lib.pkv_internal_host_units(ctypes.byref(m), reqs.array, reqs.count, None, 0, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("dim,paired,rounds", [(128, False, 12), (128, True, 6), (96, False, 6), (96, True, 6), (80, False, 6)])
def test_late_order_by_rounds(dim, paired, rounds):
    """The late start order up to `rounds` rounds of resident workgroups on 256 compute units."""
    for tokens in (20000, 60000, 90000, 130000, 260000):
        case = make(8, dim, B=64, P=64, tokens=tokens, paired=paired)
        got, units = restore_launch(case), _units(case)
        assert got["late"] == (units <= rounds * 256 * got["per_cu"]), (tokens, units, got)


@pytest.mark.parametrize("dim", [128, 96])
def test_one_round_for_whole_sectors(dim):
    """Launches of up to three workgroups to a compute unit run in one round where rows are whole sectors."""
    for tokens in (4000, 7000, 9000, 12000, 20000):
        case = make(8, dim, B=64, P=64, tokens=tokens)
        got, units = restore_launch(case), _units(case)
        assert got["one_round"] == (dim == 128 and got["per_cu"] < 3 and units <= 768), (tokens, units, got)


@pytest.mark.parametrize("args,per_cu", [
    # 2 heads of 128: one wave, 2731 elements on average; 0.61 bytes read per byte written: 10 * sqrt(1.5) waves,
    # and where 755 MB are written 8.5 * sqrt(1.5)
    (dict(H=2, D=128, mix=(37, 25, 14, 24)), 12), (dict(H=2, D=128, mix=(37, 25, 14, 24), L=200), 10),
    (dict(H=2, D=128), 13),          # 0.47: 10.5 * sqrt(1.5)
    (dict(H=2, D=128, L=200), 9),    # the same, 755 MB: 23592 / 2731
    (dict(H=2, D=128, mix=K4V4), 10), (dict(H=2, D=128, mix=(1, 0, 0, 0)), 6), (dict(H=2, D=128, delta=0), 6),
    (dict(H=2, D=64), 16), (dict(H=2, D=64, mix=(37, 25, 14, 24)), 12),  # half lines: 23592 / 1365, 15729 / 1365
    (dict(H=4, D=128, mix=(37, 25, 14, 24)), 4),  # two waves, 5461 elements: 10 * sqrt(0.75) / 2
    (dict(H=4, D=128, P=1, mix=(37, 25, 14, 24)), 16),  # one-token pages
])
def test_residency_of_narrow_rows(args, per_cu):
    """Destination rows start twelve slots into a 16-token page, so a block's units are 4, 16 and 12 tokens."""
    assert restore_launch(make(**args))["per_cu"] == per_cu


def link_groups(case, units=0):
    fn = pb.load().pkv_internal_link_groups
    fn.argtypes = [ctypes.POINTER(pb.PkvModel), ctypes.POINTER(pb.PkvRequest), ctypes.c_int32, ctypes.c_int64,
                   ctypes.POINTER(ctypes.c_int64)]
    fn.restype = ctypes.c_int32
    m, reqs, out = pb.make_model(case.shape), pb._Requests(case.requests), ctypes.c_int64()
    assert fn(ctypes.byref(m), reqs.array, reqs.count, units, ctypes.byref(out)) == 0
    return out.value


@pytest.mark.parametrize("args,groups", [
    (dict(H=8, D=128, mix=K8V4, L=8), 16), (dict(H=32, D=128, mix=(1, 0, 0, 0), L=8), 16), (dict(H=2, D=128, L=8), 48),
    (dict(H=1, D=128, mix=K4V4, L=32), 176), (dict(H=8, D=128, P=1, mix=K8V4, L=4), 160), (dict(H=2, D=128, P=1), 0),
    (dict(H=8, D=128, mix=K8V4), 64), (dict(H=8, D=128, tokens=100), 7),  # 6 MB in all; never more than work items
])
def test_link_groups(args, groups):
    """Workgroups of a restore over the host link: as many as keep some 256 KB of reads in flight; 0 is one per item."""
    assert link_groups(make(**args)) == groups


def test_link_launches_of_any_size():
    """Narrow one-token pages take an ordinary launch while its threads are fewer than 2^32, a loop beyond."""
    case = make(1, 16, B=2, P=1, tokens=512)
    assert link_groups(case, (1 << 26) - 1) == 0 and link_groups(case, 1 << 26) == 4096
