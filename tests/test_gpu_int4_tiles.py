"""The 4-bit grouped GEMM at the edges of its tiles: both tile sizes, a tile exactly full and one token over, a single k-block
in the down pass, an odd number of k-blocks and of row blocks."""
import pytest

from tests.helpers import OracleStack, compare_traces_and_stats
from tests.test_gpu_int4 import q4_bytes
from tests.test_gpu_parity import batched_step, small_cfg
from workload import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_model,d_ff,n_experts,batch", [
    (256, 32, 8, 17), (256, 64, 2, 32), (256, 96, 2, 33), (768, 224, 4, 129), (256, 160, 2, 64), (512, 32, 2, 65)])
def test_tiles_of_the_int4_gemm(d_model, d_ff, n_experts, batch):
    import torch
    from paper_2602_11192_amd import pool as P
    cfg = small_cfg(d_model=d_model, d_ff=d_ff, n_experts=n_experts, top_k=2, n_seqs=batch, n_steps=2, n_layers=1,
                    capacity=n_experts, n_shared=1, beta=1.0, pref_lo=1, pref_hi=1)
    wl = Workload(cfg)
    cache = P.make_cache(wl, int4=True, max_batch=batch, trace_capacity=4096)
    ost = OracleStack(wl, int4=True, capacity=n_experts, keep=16)
    traces = [[]]
    for step in range(cfg.n_steps):
        traces[0].extend(batched_step(torch, P, wl, cache, ost, 0, list(range(batch)), step))
    compare_traces_and_stats(cache, ost, traces, q4_bytes(cfg))
    cache.close()
