"""fp32 layers whose experts are all in memory, the whole call in one launch: at both ends of its limits (64 tokens, 64 experts, one expert),
on odd widths and several steps of a workgroup, under LRU and discounted counts.  Outputs, selections, trace, counters and resident sets
against the oracle; recency against the kernels with a routing launch; in place; and replayed from a graph."""
import ctypes as C

import numpy as np
import pytest

import oracle
from tests.helpers import TOL, OracleStack, compare_traces_and_stats, rel_err
from workload import MoEConfig, Workload, widen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,K,ns,d,f", [(8, 2, 0, 64, 128), (64, 8, 1, 36, 20), (1, 1, 0, 260, 8), (63, 3, 2, 100, 60), (64, 1, 0, 1024, 8)])
@pytest.mark.parametrize("policy,gamma", [(oracle.POLICY_LRU, 1.0), (oracle.POLICY_GAMMA, 0.9)])
def test_whole_layer(E, K, ns, d, f, policy, gamma):
    import torch
    from paper_2602_11192_amd import pool as P
    cfg = MoEConfig("token_layer", 61, "fp32", 1, d, f, E, ns, K, E, 66, 5, 0, 1.5, min(K, 3), min(K, 3), 1e-5)
    wl = Workload(cfg)
    cache = P.make_cache(wl, max_batch=66, trace_capacity=4096, policy=P.B.MOE_POLICY_LRU if policy == oracle.POLICY_LRU else P.B.MOE_POLICY_GAMMA,
                         gamma=gamma)
    ost = OracleStack(wl, policy=policy, gamma=gamma, keep=E)
    ids = list(range(E))[::-1]
    cache.moe_cache_prefill_pins(0, ids)
    ost.caches[0].pin(ids)
    trace = []
    for step, batch in enumerate((1, 64, 2, 65, 7)):             # (65: routed by a launch of its own)
        print("token layer", E, K, policy, batch, flush=True)
        xs = np.stack([wl.tokens(s)[step] for s in range(batch)])
        bias = np.stack([wl.bias(0, s) for s in range(batch)])
        idx = torch.empty((batch, K), dtype=torch.int32, device="cuda:0")
        w = torch.empty((batch, K), dtype=torch.float32, device="cuda:0")
        y = P.to_device(xs)                                      # in place
        cache.moe_layer_decode(0, y, y, torch.from_numpy(bias).cuda(), idx, w)
        res = ost.decode(0, widen(xs), bias)
        torch.cuda.synchronize()
        assert idx.cpu().numpy().tolist() == res.idx.tolist()
        np.testing.assert_allclose(w.cpu().numpy(), res.w, rtol=0, atol=2e-5)
        assert rel_err(P.to_numpy(y), res.y).max() <= TOL["fp32"]
        trace.extend(res.trace)
    compare_traces_and_stats(cache, ost, [trace], cfg.expert_bytes)
    cache.close()


@pytest.mark.parametrize("E,K,ns,d,f", [(8, 2, 0, 64, 128), (64, 8, 1, 36, 20), (1, 1, 0, 260, 8), (63, 3, 2, 100, 60), (64, 1, 0, 1024, 8)])
@pytest.mark.parametrize("policy,gamma", [(oracle.POLICY_LRU, 1.0), (oracle.POLICY_GAMMA, 0.9)])
def test_recency_is_that_of_a_launch_for_the_routing(E, K, ns, d, f, policy, gamma):
    """Last lookups, discounted counts and clock after every call, against a layer of the same router and tokens whose experts are too
    large for the one launch (nothing is evicted from a full layer, so no trace would tell)."""
    import torch
    from paper_2602_11192_amd import binding as B
    gen = torch.Generator().manual_seed(E * d)
    router = (torch.randn(1, E, d, generator=gen) * d ** -0.5).cuda()
    caches = []
    for width in (f, ((1 << 20) // (12 * (K + ns) * d) // 4 + 1) * 4):
        pool = torch.zeros(E * 3 * d * width, pin_memory=True)
        cache = B.MoECache(n_layers=1, n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=width, capacity=E, dtype=B.MOE_DTYPE_FP32, router_w=router,
                           expert_pool=pool, shared_w=torch.zeros(ns * 3 * d * width, device="cuda:0") if ns else None, max_batch=64, trace_capacity=4096,
                           policy=B.MOE_POLICY_LRU if policy == oracle.POLICY_LRU else B.MOE_POLICY_GAMMA, gamma=gamma)
        cache.moe_cache_prefill_pins(0, list(range(E))[::-1])
        cache.moe_cache_set_profiling(True)
        caches.append(cache)
    for batch in (1, 64, 2, 7):
        print("recency", E, K, policy, batch, flush=True)
        x, bias = torch.randn(batch, d, generator=gen).cuda(), torch.randn(batch, E, generator=gen).cuda()
        seen = []
        for cache in caches:
            idx = torch.empty((batch, K), dtype=torch.int32, device="cuda:0")
            cache.moe_layer_decode(0, x, torch.empty_like(x), bias, idx)
            tick, score, clock = np.zeros(E, np.uint64), np.zeros(E, np.float64), np.zeros(1, np.int64)
            assert B.lib.moe_test_recency(cache._h, 0, *(v.ctypes.data_as(C.c_void_p) for v in (tick, score, clock))) == 0
            seen.append((idx.cpu().tolist(), tick.tolist(), score.tolist(), clock.tolist(), cache.moe_cache_read_trace(0)[0].tolist()))
        assert seen[0] == seen[1]
        assert len(set(seen[0][1])) == E and (policy == oracle.POLICY_LRU or max(seen[0][2]) > 0)
    launches = [cache.moe_cache_timing() for cache in caches]
    assert launches[0]["decode_single_launches"] >= 1 and launches[1]["decode_single_launches"] == 0      # (1024 x 8: 64 tokens only)
    for cache in caches:
        cache.close()


# (either side of the line between the one launch and the kernels per expert)
@pytest.mark.parametrize("E,K,ns,d,f,batch,one", [(24, 2, 0, 140, 244, 64, 0), (8, 1, 0, 180, 196, 8, 0), (16, 4, 0, 192, 112, 64, 0),
                                                  (4, 2, 1, 80, 236, 32, 1), (8, 2, 0, 64, 128, 64, 1), (8, 2, 0, 64, 128, 65, 0)])
def test_calls_that_take_the_one_launch(E, K, ns, d, f, batch, one):
    import torch
    from paper_2602_11192_amd import pool as P
    print("one launch", E, K, ns, d, f, batch, flush=True)
    cfg = MoEConfig("token_layer", 63, "fp32", 1, d, f, E, ns, K, E, batch, 1, 0, 1.5, min(K, 3), min(K, 3), 1e-5)
    wl = Workload(cfg)
    cache = P.make_cache(wl, max_batch=batch)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    ost = OracleStack(wl, keep=E)
    ost.caches[0].pin(list(range(E)))
    xs = np.stack([wl.tokens(s)[0] for s in range(batch)])
    x = P.to_device(xs)
    y = torch.empty_like(x)
    cache.moe_cache_set_profiling(True)
    cache.moe_layer_decode(0, x, y)
    assert cache.moe_cache_timing()["decode_single_launches"] == one
    assert rel_err(P.to_numpy(y), ost.decode(0, widen(xs), None).y).max() <= TOL["fp32"]
    cache.close()


# (few pairs on wide rows, 14 to 27 % slower in the one launch; and calls that it makes 1.4 and 1.5 times as fast)
@pytest.mark.parametrize("E,K,ns,d,f,batch,one", [(8, 1, 0, 240, 164, 7, 0), (16, 2, 0, 88, 172, 3, 0), (32, 1, 0, 228, 244, 12, 0),
                                                  (48, 6, 0, 56, 92, 6, 1), (64, 8, 2, 100, 24, 4, 1)])
def test_calls_of_six_and_more_steps(E, K, ns, d, f, batch, one):
    test_calls_that_take_the_one_launch(E, K, ns, d, f, batch, one)


def test_replays_of_a_captured_call():
    import torch
    from paper_2602_11192_amd import pool as P
    E, K, d, f, batch = 16, 2, 64, 128, 5
    cfg = MoEConfig("token_layer", 62, "fp32", 1, d, f, E, 0, K, E, 30, 2, 0, 1.5, 2, 2, 1e-5)
    wl = Workload(cfg)
    cache = P.make_cache(wl, max_batch=batch)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    x = P.to_device(np.stack([wl.tokens(s)[0] for s in range(batch)]))
    y, eager = torch.empty_like(x), torch.empty_like(x)
    cache.moe_layer_decode(0, x, y)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cache.moe_layer_decode(0, x, y)
    for i in range(5):
        x.copy_(P.to_device(np.stack([wl.tokens((i * batch + s) % 30)[1] for s in range(batch)])))
        graph.replay()
        cache.moe_layer_decode(0, x, eager)
        torch.cuda.synchronize()
        assert torch.equal(y, eager), i
    cache.close()
