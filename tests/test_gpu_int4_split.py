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


# Every token of part p of the call prefers the experts of set p, so that the parts take turns in the slots.  Where the split of a part by itself would be
# another than that of the whole call: (4096 x 512, 256) down pass, 1024 and 512 workgroups, and gate/up, 512 and 256; (1024 x 256, 1400) 64-token tiles;
# (512 x 1024, 1000) one set: 32-token tiles by the experts, 64-token ones by the slots.
@pytest.mark.parametrize("d,f,E,C,batch,parts", [(4096, 512, 48, 24, 256, 2), (1024, 256, 48, 24, 1400, 2), (512, 1024, 64, 16, 1000, 1)])
def test_a_call_run_as_waves_has_the_bits_of_the_unsplit_one(d, f, E, C, batch, parts):
    import torch
    from paper_2602_11192_amd import binding as B
    K = 2
    gen = torch.Generator().manual_seed(3)
    gate_up = torch.randint(0, 256, (E, f // 16 * (d // 128), 2304), generator=gen, dtype=torch.uint8)       # 2048 bytes of codes, 256 of scales
    down = torch.randint(0, 256, (E, f // 32 * (d // 64), 1152), generator=gen, dtype=torch.uint8)           # 1024 and 128
    for records, codes in ((gate_up, 2048), (down, 1024)):
        scales = torch.rand(*records.shape[:2], (records.shape[2] - codes) // 2, generator=gen) * 0.02 + 0.005
        records[..., codes:] = scales.bfloat16().view(torch.uint8)
    pool = torch.cat([gate_up.reshape(E, -1), down.reshape(E, -1)], dim=1).reshape(-1).pin_memory()
    router = (torch.randn(1, E, d, generator=gen) * d ** -0.5).bfloat16().cuda()
    x = torch.randn(batch, d, generator=gen).bfloat16().cuda()
    bias = torch.zeros(batch, E)
    for p in range(parts):
        bias[p * batch // parts:(p + 1) * batch // parts, p * C:(p + 1) * C] = 60.0
    bias = bias.cuda()
    out = []
    for staging in (0, E):
        print("waves", d, f, batch, staging, flush=True)
        cache = B.MoECache(n_layers=1, n_experts=E, top_k=K, d_model=d, d_ff=f, capacity=C, dtype=B.MOE_DTYPE_BF16, router_w=router, expert_pool=pool,
                           max_batch=batch, staging_buffers=staging, pool_layout=B.MOE_LAYOUT_TILED_INT4)
        y = torch.empty(batch, d, dtype=torch.bfloat16, device="cuda:0")
        idx = torch.empty(batch, K, dtype=torch.int32, device="cuda:0")
        w = torch.empty(batch, K, device="cuda:0")
        cache.moe_layer_decode(0, x, y, bias, idx, w)
        torch.cuda.synchronize()
        out.append((y.cpu().view(torch.int16), idx.cpu(), w.cpu(), cache.moe_cache_stats(0)))
        cache.close()
    assert out[0][3] == out[1][3] and out[0][3]["misses"] >= parts * (C - 1)
    assert torch.isfinite(out[0][0].view(torch.bfloat16).float()).all()
    for a, b in zip(out[0][:3], out[1][:3]):
        assert torch.equal(a, b)
