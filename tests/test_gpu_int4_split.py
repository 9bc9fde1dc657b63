"""The 4-bit grouped GEMM where groups of waves split the contraction: contractions that do not divide among two or four groups, in both
passes and both tile sizes, and grids just too large to be split."""
import pytest

from tests.helpers import OracleStack, compare_traces_and_stats
from tests.test_gpu_int4 import q4_bytes
from tests.test_gpu_parity import batched_step, small_cfg
from workload import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,d_ff,n_experts,batch", [
    (2304, 1056, 2, 17), (2048, 1024, 3, 33), (2304, 1120, 2, 90),          # four groups; two groups of the larger tile
    (1792, 480, 4, 20), (256, 32, 8, 40),                                   # two groups, the second one with nothing to add
    (256, 8192, 4, 24), (4096, 32, 32, 40), (256, 8192, 2, 129), (4096, 32, 12, 400)])      # one group, in the first or the second pass
def test_groups_that_split_the_contraction(d_model, d_ff, n_experts, batch):
    import torch
    from paper_2602_11192_amd import pool as P
    cfg = small_cfg(d_model=d_model, d_ff=d_ff, n_experts=n_experts, top_k=2, n_seqs=batch, n_steps=1, n_layers=1,
                    capacity=n_experts, n_shared=1, beta=1.0, pref_lo=1, pref_hi=1)
    wl = Workload(cfg)
    cache = P.make_cache(wl, int4=True, max_batch=batch, trace_capacity=4096)
    ost = OracleStack(wl, int4=True, capacity=n_experts, keep=33)
    traces = [[]]
    traces[0].extend(batched_step(torch, P, wl, cache, ost, 0, list(range(batch)), 0))
    compare_traces_and_stats(cache, ost, traces, q4_bytes(cfg))
    cache.close()


# (either side of the line from which fewer than 17 tokens take the GEMM: 85 and 113 MB of experts over all pairs)
@pytest.mark.parametrize("batch", [6, 8])
def test_few_tokens_on_a_large_layer(batch):
    import torch
    from paper_2602_11192_amd import pool as P
    cfg = small_cfg(d_model=4096, d_ff=512, n_experts=8, top_k=4, n_seqs=batch, n_steps=1, n_layers=1, capacity=8, n_shared=0,
                    beta=1.0, pref_lo=1, pref_hi=1)
    wl = Workload(cfg)
    cache = P.make_cache(wl, int4=True, max_batch=batch, trace_capacity=4096)
    cache.moe_cache_prefill_pins(0, list(range(8)))
    ost = OracleStack(wl, int4=True, capacity=8, keep=9)
    ost.caches[0].pin(list(range(8)))
    traces = [batched_step(torch, P, wl, cache, ost, 0, list(range(batch)), 0)]
    compare_traces_and_stats(cache, ost, traces, q4_bytes(cfg))
    cache.close()
