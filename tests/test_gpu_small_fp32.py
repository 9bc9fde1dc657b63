"""fp32 calls of 2 to 8 tokens that one workgroup routes: at both ends of the limits of that path (128 products of token
and expert, 128 KiB of router rows), with more products than the waves take in a round and rows longer than a
wave reads at once, against the layer in 64 bits; and through a cache - resident, constrained with few spare buffers, LRU
and discounted counts - against the oracle."""
import numpy as np
import pytest

import oracle
from tests.helpers import TOL, OracleStack, compare_traces_and_stats, rel_err
import tests.test_gpu_rowmajor as rowmajor
from workload import MoEConfig, Workload, widen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,E,K,ns,d,f", [(8, 16, 4, 0, 256, 20), (8, 16, 4, 0, 260, 20), (8, 9, 2, 1, 64, 12),
                                              (7, 10, 3, 0, 300, 8), (2, 8, 2, 0, 2048, 16), (2, 8, 2, 0, 2052, 16),
                                              (2, 64, 8, 0, 256, 8), (3, 43, 5, 0, 64, 8), (4, 1, 1, 0, 512, 8)])
def test_layer_at_the_limits(batch, E, K, ns, d, f):
    rowmajor.test_rowmajor_layer("fp32", batch, E, K, ns, d, f)


@pytest.mark.parametrize("policy,gamma", [(oracle.POLICY_LRU, 1.0), (oracle.POLICY_GAMMA, 0.9), (oracle.POLICY_GAMMA, 1.0)])
@pytest.mark.parametrize("capacity,staging", [(12, 0), (5, 16), (4, 1)])
def test_cache_of_small_batches(policy, gamma, capacity, staging):
    import torch
    from paper_2602_11192_amd import pool as P
    K = 3
    cfg = MoEConfig("small_fp32", 41, "fp32", 1, 96, 40, 12, 1, K, capacity, 8, 12, 0, 1.5, 3, 3, 1e-5)
    wl = Workload(cfg)
    cache = P.make_cache(wl, max_batch=8, staging_buffers=staging, trace_capacity=4096,
                         policy=P.B.MOE_POLICY_LRU if policy == oracle.POLICY_LRU else P.B.MOE_POLICY_GAMMA, gamma=gamma)
    ost = OracleStack(wl, policy=policy, gamma=gamma)
    trace = []
    for step, batch in enumerate((2, 8, 3, 1, 5, 8, 4, 7, 2, 6, 8, 8)):
        print("small fp32", policy, gamma, capacity, step, batch, flush=True)
        xs = np.stack([wl.tokens(s)[step] for s in range(batch)])
        bias = np.stack([wl.bias(0, s) for s in range(batch)])
        y = torch.empty((batch, cfg.d_model), dtype=torch.float32, device="cuda:0")
        idx = torch.empty((batch, K), dtype=torch.int32, device="cuda:0")
        cache.moe_layer_decode(0, P.to_device(xs), y, torch.from_numpy(bias).cuda(), idx)
        res = ost.decode(0, widen(xs), bias)
        torch.cuda.synchronize()
        assert idx.cpu().numpy().tolist() == res.idx.tolist()
        assert rel_err(P.to_numpy(y), res.y).max() <= TOL["fp32"]
        trace.extend(res.trace)
    compare_traces_and_stats(cache, ost, [trace], cfg.expert_bytes)
    st = cache.moe_cache_stats()
    assert st["misses"] > 0 and (st["evictions"] > 0) == (capacity < cfg.n_experts)
    cache.close()
