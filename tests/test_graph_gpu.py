"""Both device entry points enqueue one kernel on the caller's stream and
allocate nothing, so a caller can capture them in a HIP graph; so can a plan's
first streamed restore, whose copies a kernel makes.  Each test
captures one call, then replays the graph several times with eager work in
between (the outputs are overwritten before every replay) and checks every
replay against the eager result."""
import pytest

from paper_2609_26219_amd import binding as pb
from paper_2609_26219_amd import workloads as wl
from parity import log, oracle_checkpoint

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    pb.load()
    return _t


def test_restore_replays_from_a_graph(torch):
    from paper_2609_26219_amd.device import DeviceRestore
    log("[gpu] graph capture: pkv_restore on llama8b_1l, 4 replays")
    case = wl.make_case("llama8b_1l")
    dr = DeviceRestore(case, checkpoint=oracle_checkpoint(case))
    dr.run()
    torch.cuda.synchronize()
    want_k, want_v = dr.k_cache.clone(), dr.v_cache.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        pb.restore_tensors(dr.plan, dr.payload, dr.scales, dr.k_cache, dr.v_cache)
    for _ in range(4):
        dr.prefill()
        torch.cuda.synchronize()
        assert not torch.equal(dr.k_cache, want_k)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dr.k_cache, want_k) and torch.equal(dr.v_cache, want_v)


def test_checkpoint_write_replays_from_a_graph(torch):
    from paper_2609_26219_amd.device import DeviceCheckpoint, OldCaches
    log("[gpu] graph capture: pkv_quantize_gather on llama8b_1l, 4 replays")
    case = wl.make_case("llama8b_1l")
    ck = DeviceCheckpoint(case, OldCaches(case))
    ck.write()
    torch.cuda.synchronize()
    want_p, want_s = ck.payload.clone(), ck.scales.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        pb.quantize_gather_tensors(ck.plan, ck.old.k, ck.old.v, ck.payload, ck.scales)
    for i in range(4):
        ck.payload.fill_(0xA0 + i)
        ck.scales.fill_(0x1234 + i)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(ck.payload, want_p) and torch.equal(ck.scales, want_s)


def test_first_streamed_restore_replays_from_a_graph(torch):
    """The first call on a plan, captured: its copies and restores are in the graph, and neither it nor an eager first
    call takes device memory."""
    from paper_2609_26219_amd.device import DeviceRestore
    case = wl.make_custom(51, L=5, H=8, D=128, B=32, P=16, n_tokens=(2300, 40), deltas=(-3, 0), rho0s=(7, 11),
                          tag_set=(0, 1, 2, 3), mix=(1, 1, 1, 1), repair_frac=0.2, out_dtype=wl.OUT_BF16)
    ckpt = oracle_checkpoint(case)
    dr = DeviceRestore(case, checkpoint=ckpt)
    dr.run()
    torch.cuda.synchronize()
    want_k, want_v = dr.k_cache.clone(), dr.v_cache.clone()
    hp = torch.from_numpy(ckpt[0]).pin_memory()
    hs = torch.from_numpy(ckpt[1].view("int16")).pin_memory()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        pb.restore_from_host_tensors(dr.plan, hp, hs, dr.payload, dr.scales, dr.k_cache, dr.v_cache)
    for i in range(4):
        dr.prefill()
        dr.payload.fill_(0x5A + i)
        dr.scales.fill_(0x1234 + i)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dr.k_cache, want_k) and torch.equal(dr.v_cache, want_v)


def test_first_streamed_restore_allocates_no_device_memory(torch):
    import gc

    case = wl.make_custom(52, L=2, H=1, D=16, B=2, P=2, n_tokens=(60000,), deltas=(1,), rho0s=(0,), repair_frac=0.0,
                          tag_set=(1,), mix=(1,))
    nb = case.payload_nbytes
    hp, hs = torch.zeros(nb, dtype=torch.uint8).pin_memory(), torch.zeros(case.scale_elems, dtype=torch.int16).pin_memory()
    payload, scales = torch.zeros(nb, dtype=torch.uint8, device="cuda"), torch.zeros(case.scale_elems, dtype=torch.int16, device="cuda")
    gc.collect()  # plans of earlier tests hold the slabs that small allocations are cut from
    plan = pb.pkv_restore_plan(case.shape, case.requests)  # 1.9 MB: an allocation of its own
    k = torch.zeros(pb.pkv_plan_query(plan)["cache_bytes"] // 2, dtype=torch.int16, device="cuda")
    v = torch.zeros_like(k)
    torch.cuda.synchronize()
    call = lambda p: pb.restore_from_host_tensors(p, hp, hs, payload, scales, k, v)
    call(plan)  # streams and events, the kernels' code
    torch.cuda.synchronize()
    pb.pkv_free(plan)
    plan = pb.pkv_restore_plan(case.shape, case.requests)
    free = torch.cuda.mem_get_info()[0]
    call(plan)
    torch.cuda.synchronize()
    # The call's new streams take some (2 MB); an allocation of the library's would be a 4 MiB slab more.
    assert free - torch.cuda.mem_get_info()[0] < 4 << 20
