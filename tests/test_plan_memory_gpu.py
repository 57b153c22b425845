"""Plans share slabs of device memory: work lists of many plans alive at once,
freed in any order and made again keep their contents, from several threads
too, and a plan freed right behind its launch stays readable until the launch
is done, also where a slab is filled again."""
import threading

import numpy as np
import pytest

from paper_2609_26219_amd import binding as pb
from paper_2609_26219_amd import workloads as wl

from parity import check_full, oracle_checkpoint

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    pb.load()
    return _t


def _case(seed, tokens):
    return wl.make_custom(seed, L=2, H=2, D=64, B=16, P=16, n_tokens=(tokens, 16), deltas=(37, 0), rho0s=(40, 6),
                          tag_set=(0, 1, 2, 3), mix=(1, 1, 1, 1), repair_frac=0.2, out_dtype=wl.OUT_BF16)


def _restore(dr, ckpt, plan):
    dr.prefill()
    pb.restore_tensors(plan, dr.payload, dr.scales, dr.k_cache, dr.v_cache)


def test_plans_freed_in_any_order(torch):
    from paper_2609_26219_amd.device import DeviceRestore

    rng = np.random.default_rng(8)
    cases = [_case(60 + i, n) for i, n in enumerate((100, 531, 17))]
    ckpts = [oracle_checkpoint(c) for c in cases]
    drs = [DeviceRestore(c, checkpoint=k) for c, k in zip(cases, ckpts)]
    plans = []
    for step in range(300):  # some hundred work lists, several slabs' worth with the long ones below
        i = int(rng.integers(3))
        plans.append((i, pb.pkv_restore_plan(cases[i].shape, cases[i].requests)))
        if len(plans) > 40:
            pb.pkv_free(plans.pop(int(rng.integers(len(plans))))[1])
    # Work lists of 250 KB fill a slab with 16 plans; one of 4 MB takes an allocation of its own.
    shape = wl.make_custom(70, L=1, H=1, D=16, B=2, P=2, n_tokens=(8000,), deltas=(1,), rho0s=(0,), repair_frac=0.0)
    wide = wl.make_custom(71, L=1, H=1, D=16, B=2, P=2, n_tokens=(140000,), deltas=(1,), rho0s=(0,), repair_frac=0.0)
    fill = [pb.pkv_restore_plan(shape.shape, shape.requests) for _ in range(50)]
    big = pb.pkv_restore_plan(wide.shape, wide.requests)
    for p in fill[::2]:
        pb.pkv_free(p)
    for i, plan in (plans[0], plans[len(plans) // 2], plans[-1]):
        _restore(drs[i], ckpts[i], plan)
        torch.cuda.synchronize()
        check_full(drs[i], ckpts[i])
    for p in fill[1::2] + [big] + [p for _, p in plans]:
        pb.pkv_free(p)


def test_plan_freed_behind_its_launch(torch):
    """Freed while its launch waits on the stream, with new plans made right behind it."""
    from paper_2609_26219_amd.device import DeviceRestore

    case = _case(80, 531)
    ckpt = oracle_checkpoint(case)
    dr = DeviceRestore(case, checkpoint=ckpt)
    other = _case(81, 900)
    dr.prefill()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        busy = torch.randn(4096, 4096, device="cuda")
        for _ in range(20):
            busy = torch.tanh(busy @ busy)
        plan = pb.pkv_restore_plan(case.shape, case.requests)
        pb.restore_tensors(plan, dr.payload, dr.scales, dr.k_cache, dr.v_cache)
        pb.pkv_free(plan)
        new = [pb.pkv_restore_plan(other.shape, other.requests) for _ in range(20)]
    torch.cuda.synchronize()
    check_full(dr, ckpt)
    del new


def test_slab_is_reused_behind_launches(torch):
    """Work lists of 250 KB, each freed right behind a launch that still waits on its stream: 40 of them use a 4 MiB slab
    more than twice, and every launch finds its own list."""
    from paper_2609_26219_amd.device import DeviceRestore

    keep = wl.make_custom(100, L=1, H=1, D=16, B=2, P=2, n_tokens=(60000,), deltas=(1,), rho0s=(0,), repair_frac=0.0)
    kept = pb.pkv_restore_plan(keep.shape, keep.requests)  # an allocation of its own; with it the slab outlives the others
    cases = [wl.make_custom(101 + i, L=1, H=1, D=16, B=2, P=2, n_tokens=(7000 + 100 * (i % 7),), deltas=(5 - 3 * i,), rho0s=(i,),
                            tag_set=(0, 1, 2, 3), mix=(1, 1, 1, 1), repair_frac=0.1, out_dtype=wl.OUT_BF16) for i in range(10)]
    ckpts = [oracle_checkpoint(c) for c in cases]
    drs = [DeviceRestore(c, checkpoint=k) for c, k in zip(cases, ckpts)]
    side = torch.cuda.Stream()
    for turn in range(4):
        for dr in drs:
            dr.prefill()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            busy = torch.randn(4096, 4096, device="cuda")
            for _ in range(20):
                busy = torch.tanh(busy @ busy)
            for dr, case in zip(drs, cases):
                plan = pb.pkv_restore_plan(case.shape, case.requests)
                pb.restore_tensors(plan, dr.payload, dr.scales, dr.k_cache, dr.v_cache)
                pb.pkv_free(plan)
        torch.cuda.synchronize()
        for dr, ckpt in zip(drs, ckpts):
            check_full(dr, ckpt)
    pb.pkv_free(kept)


def test_plans_from_several_threads(torch):
    from paper_2609_26219_amd.device import DeviceRestore

    case = _case(90, 300)
    ckpt = oracle_checkpoint(case)
    drs = [DeviceRestore(case, checkpoint=ckpt) for _ in range(4)]
    errors = []

    def work(dr):
        try:
            stream = torch.cuda.Stream()
            stream.wait_stream(torch.cuda.default_stream())
            with torch.cuda.stream(stream):
                for _ in range(50):
                    plan = pb.pkv_restore_plan(case.shape, case.requests)
                    pb.restore_tensors(plan, dr.payload, dr.scales, dr.k_cache, dr.v_cache)
                    stream.synchronize()
                    pb.pkv_free(plan)
        except Exception as e:  # reported by the main thread
            errors.append(e)

    for dr in drs:
        dr.prefill()
    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(dr,)) for dr in drs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors
    torch.cuda.synchronize()
    for dr in drs:
        check_full(dr, ckpt)
