"""One layer whose experts all fit, called with one to four tokens by turns before and after the host knows that all of them
are there: the calls change between the single launch (which reads one copy of the layer's table, writes the other and counts
on the device) and the routing launch (which updates the current copy in place and is counted on the host).  Outputs, the
whole trace and the counters against the oracle, across a reset."""
import numpy as np
import pytest

import oracle
from tests.helpers import TOL, OracleStack, compare_traces_and_stats, rel_err
from workload import Workload, get_config, widen

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def oracle_threads():
    oracle.set_threads(16)
    yield
    oracle.set_threads(1)


@pytest.mark.parametrize("int4", [False, True])
def test_interleaved_small_batches(int4):
    import torch
    from paper_2602_11192_amd import pool as P
    cfg = get_config("olmoe_like")
    E, K, d = cfg.n_experts, cfg.top_k, cfg.d_model
    wl = Workload(cfg)
    cache = P.make_cache(wl, capacity=E, max_batch=16, trace_capacity=1 << 14, fetch_mode=P.B.MOE_FETCH_IN_KERNEL, int4=int4)
    ost = OracleStack(wl, capacity=E, keep=E, int4=int4)
    cache.moe_cache_set_profiling(True)
    trace, step = [], 0

    def call(batch, single):
        nonlocal step
        print("interleaved", int4, step, batch, flush=True)
        xs = np.stack([wl.tokens(s)[step % cfg.n_steps] for s in range(batch)])
        bias = np.stack([wl.bias(0, s) for s in range(batch)])
        y = torch.empty((batch, d), dtype=torch.bfloat16, device="cuda:0")
        idx = torch.empty((batch, K), dtype=torch.int32, device="cuda:0")
        w = torch.empty((batch, K), dtype=torch.float32, device="cuda:0")
        cache.moe_cache_timing(clear=True)
        cache.moe_layer_decode(0, P.to_device(xs), y, torch.from_numpy(bias).cuda(), idx, w)
        tm = cache.moe_cache_timing(clear=True)
        res = ost.decode(0, widen(xs), bias)
        torch.cuda.synchronize()
        assert idx.cpu().numpy().tolist() == res.idx.tolist()
        np.testing.assert_allclose(w.cpu().numpy(), res.w, rtol=0, atol=2e-5)
        assert rel_err(P.to_numpy(y), res.y).max() <= TOL["bf16"]
        assert (tm["route_launches"] == 0) == single, (batch, tm)
        trace.extend(res.trace)
        step += 1
        return all(r[2] for r in res.trace)

    def preload():
        ids = list(range(E))
        cache.moe_cache_prefill_pins(0, ids)
        ost.caches[0].pin(ids)

    call(1, True), call(4, True), call(2, True)               # filled by their own misses, no answer is waited for
    preload()
    for batch in (1, 2, 3, 4, 1, 16, 4, 1, 1, 3):             # known to be resident
        assert call(batch, batch == 1)
    cache.moe_cache_reset(0)
    ost.caches[0].reset()
    assert not call(4, True)                                  # empty again: misses, and back in the single launch
    assert not call(2, True)
    call(1, True)
    preload()
    assert call(4, False) and call(1, True) and call(2, False)
    compare_traces_and_stats(cache, ost, [trace], P.int4_block_bytes(cfg) if int4 else cfg.expert_bytes)
    cache.close()
