"""The allocation-free streamed restore (pkv_restore_from_host_noalloc)
against pkv_restore_from_host, through the C ABI: identical caches, bit for
bit, on two calls in a row (the second with a smaller plan), and the oracle's
restore on both.  Host buffers that a kernel can address in whole loads are
read in place by one looping launch; buffers four bytes into an allocation
cannot be, so they go through the stage, the first case's request-layers, which
span more than its 64 MiB, in several payload windows."""
import ctypes

import numpy as np
import pytest

from paper_2609_26219_amd import binding as pb
from paper_2609_26219_amd import workloads as wl

from parity import check_full, log, oracle_checkpoint

pytestmark = pytest.mark.gpu

FILL = 0x5A


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    pb.load()
    return _t


def _paired(case):
    import dataclasses
    case.shape = dataclasses.replace(case.shape, kv_layout=wl.KV_PAIRED)
    return case


def _big():
    # 32768 tokens x 8 heads x 128, mostly FP16: about 98 MiB per request-layer
    # (two windows), plus a short second request; two layers.
    return _paired(wl.make_custom(31, L=2, H=8, D=128, B=32, P=16, n_tokens=(32768, 900), deltas=(-1500, 37),
                                  rho0s=(5007, 40000), tag_set=(0, 1, 2, 3), mix=(0.6, 0.2, 0.1, 0.1),
                                  repair_frac=0.15, out_dtype=wl.OUT_BF16, theta=5e5, outlier_pairs=1))


def _pinned(torch, array, offset):
    """The bytes of a host array, `offset` bytes into a pinned allocation: (tensor, address)."""
    raw = array.view(np.uint8)
    t = torch.zeros(raw.size + 64, dtype=torch.uint8).pin_memory()
    t[offset:offset + raw.size] = torch.from_numpy(raw)
    return t, t.data_ptr() + offset


def _both(case, torch, offset):
    from paper_2609_26219_amd.device import DeviceRestore

    ckpt = oracle_checkpoint(case)
    hp = torch.from_numpy(ckpt[0]).pin_memory()
    hs = torch.from_numpy(ckpt[1].view(np.int16)).pin_memory()
    blank = (np.full(ckpt[0].shape, FILL, np.uint8), np.full(ckpt[1].shape, FILL * 0x101, np.uint16))
    dr = DeviceRestore(case, checkpoint=blank)
    pb.restore_from_host_tensors(dr.plan, hp, hs, dr.payload, dr.scales, dr.k_cache, dr.v_cache)
    torch.cuda.synchronize()
    ref = dr.host_caches()
    dr.prefill()
    (keep_p, p), (keep_s, s) = _pinned(torch, ckpt[0], offset), _pinned(torch, ckpt[1], offset)
    assert p % 16 == offset and s % 8 == offset % 8
    st = pb.pkv_restore_from_host_noalloc_status(dr.plan, p, ckpt[0].nbytes, s, ckpt[1].nbytes,
                                                 dr.k_cache.data_ptr(), dr.v_cache.data_ptr(),
                                                 pb.cache_nbytes(dr.k_cache, dr.v_cache),
                                                 torch.cuda.current_stream().cuda_stream)
    assert st == pb.PKV_OK, pb.pkv_status_string(st)
    torch.cuda.synchronize()
    got = dr.host_caches()
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    stats = check_full(dr, ckpt)
    log(f"  {case.name}: identical to pkv_restore_from_host; oracle: {stats.n} elements, "
        f"{stats.n_near_tie} near-tie neighbours, 0 wrong")


@pytest.mark.parametrize("offset", [0, 4], ids=["in_place", "staged"])
def test_noalloc_matches_streamed_restore_two_calls(offset, torch):
    from test_stage_schedule import stage_schedule

    big, tiny = _big(), wl.make_case("tiny")
    steps = stage_schedule(big.shape, big.requests)[0]
    assert len(steps) == 2 * (2 + 1)  # two layers: two windows of the long request, one of the short
    log("[gpu] allocation-free streamed restore, %s: a case of two windows, then tiny" % ("staged" if offset else "in place"))
    _both(big, torch, offset)
    _both(tiny, torch, offset)


def _groups(case):
    fn = pb.load().pkv_internal_link_groups
    fn.argtypes = [ctypes.POINTER(pb.PkvModel), ctypes.POINTER(pb.PkvRequest), ctypes.c_int32, ctypes.c_int64,
                   ctypes.POINTER(ctypes.c_int64)]
    m, reqs, out = pb.make_model(case.shape), pb._Requests(case.requests), ctypes.c_int64()
    assert fn(ctypes.byref(m), reqs.array, reqs.count, 0, ctypes.byref(out)) == 0
    return out.value


@pytest.mark.parametrize("params,groups", [
    # 16 and 64 workgroups and hundreds of items: requests with and without rotation follow each other in one workgroup
    (dict(L=4, H=16, D=128, B=32, P=16, n_tokens=(600, 400, 33), deltas=(-3, 0, 70), rho0s=(7, 11, 90)), 16),
    (dict(L=3, H=3, D=96, B=32, P=16, n_tokens=(700, 390), deltas=(5, 0), rho0s=(7, 11)), 64),
    (dict(L=2, H=2, D=128, B=16, P=1, n_tokens=(40, 3), deltas=(5, 0), rho0s=(7, 1)), 0),  # an ordinary launch
    (dict(L=1, H=32, D=128, B=16, P=16, n_tokens=(20,), deltas=(5,), rho0s=(0,)), 5),  # fewer items than workgroups
])
@pytest.mark.parametrize("style", [wl.ROPE_HALF, wl.ROPE_INTERLEAVED], ids=["half", "interleaved"])
@pytest.mark.parametrize("dtype", [wl.OUT_BF16, wl.OUT_FP16], ids=["bf16", "fp16"])
def test_noalloc_looping_launch(params, groups, style, dtype, torch):
    import dataclasses
    case = wl.make_custom(34, tag_set=(0, 1, 2, 3), mix=(1, 1, 1, 1), repair_frac=0.0, out_dtype=dtype, **params)
    case.shape = dataclasses.replace(case.shape, rope_style=style)
    assert _groups(case) == groups
    _both(case, torch, 0)


def test_noalloc_rejects_pageable_and_oversized(torch):
    """Pageable host memory, and a request-layer whose scales exceed the 4 MiB
    stage, are refused before anything is enqueued."""
    from paper_2609_26219_amd.device import DeviceRestore

    case = wl.make_case("tiny")
    ckpt = oracle_checkpoint(case)
    dr = DeviceRestore(case, checkpoint=ckpt)
    before = dr.host_caches()
    p, s = np.ascontiguousarray(ckpt[0]), np.ascontiguousarray(ckpt[1])
    cb = pb.cache_nbytes(dr.k_cache, dr.v_cache)
    st = pb.pkv_restore_from_host_noalloc_status(dr.plan, p.ctypes.data, p.nbytes, s.ctypes.data, s.nbytes,
                                                 dr.k_cache.data_ptr(), dr.v_cache.data_ptr(), cb)
    assert st == pb.PKV_ERR_INVALID_ARGUMENT
    # 1 KV head x 32 channels, blocks of 1 token: ceil(N / B) * H * 8 bytes of scales per layer, 8 bytes over
    big = wl.make_custom(3, L=1, H=1, D=32, B=1, P=1024, n_tokens=(524289,), deltas=(1,), rho0s=(0,),
                         tag_set=(1,), mix=(1.0,), repair_frac=0.0, out_dtype=wl.OUT_FP16)
    plan = pb.pkv_restore_plan(big.shape, big.requests)
    hp = torch.zeros(big.payload_nbytes, dtype=torch.uint8).pin_memory()
    hs = torch.zeros(big.scale_elems, dtype=torch.int16).pin_memory()
    k = torch.zeros(pb.pkv_plan_query(plan)["cache_bytes"] // 2, dtype=torch.int16, device="cuda")
    v = torch.zeros_like(k)
    st = pb.pkv_restore_from_host_noalloc_status(plan, hp.data_ptr(), big.payload_nbytes, hs.data_ptr(),
                                                 2 * big.scale_elems, k.data_ptr(), v.data_ptr(), 2 * k.numel())
    assert st == pb.PKV_ERR_INVALID_ARGUMENT
    torch.cuda.synchronize()
    after = dr.host_caches()
    assert np.array_equal(before[0], after[0]) and np.array_equal(before[1], after[1])
    assert int(k.abs().sum()) == 0 and int(v.abs().sum()) == 0


@pytest.mark.parametrize("offset", [0, 16, 4], ids=["base", "inside", "unaligned"])
def test_noalloc_host_buffer_placement(offset, torch):
    """A checkpoint at the start of a pinned allocation or 16 bytes into it is read in place; one that a kernel
    cannot address in whole loads is staged.  Both restore what the oracle does."""
    from paper_2609_26219_amd.device import DeviceRestore

    case = wl.make_custom(33, L=3, H=2, D=64, B=16, P=16, n_tokens=(137, 16, 50), deltas=(3, 0, -7), rho0s=(3, 6, 13),
                          tag_set=(0, 1, 2, 3), mix=(1, 1, 1, 1), repair_frac=0.3, out_dtype=wl.OUT_BF16)
    ckpt = oracle_checkpoint(case)
    raw_p, raw_s = ckpt[0].view(np.uint8), ckpt[1].view(np.uint8)
    hp = torch.zeros(raw_p.size + 64, dtype=torch.uint8).pin_memory()
    hs = torch.zeros(raw_s.size + 64, dtype=torch.uint8).pin_memory()
    hp[offset:offset + raw_p.size] = torch.from_numpy(raw_p)
    hs[offset:offset + raw_s.size] = torch.from_numpy(raw_s)
    blank = (np.full(ckpt[0].shape, FILL, np.uint8), np.full(ckpt[1].shape, FILL * 0x101, np.uint16))
    dr = DeviceRestore(case, checkpoint=blank)
    st = pb.pkv_restore_from_host_noalloc_status(
        dr.plan, hp.data_ptr() + offset, raw_p.size, hs.data_ptr() + offset, raw_s.size, dr.k_cache.data_ptr(),
        dr.v_cache.data_ptr(), pb.cache_nbytes(dr.k_cache, dr.v_cache), torch.cuda.current_stream().cuda_stream)
    assert st == pb.PKV_OK, pb.pkv_status_string(st)
    torch.cuda.synchronize()
    check_full(dr, ckpt)
