"""Prompts through a layer whose experts are all resident, before and after the host knows it (the GEMM then takes the tiles of
resident calls instead of those for experts that cross the link), against the oracle; nothing is streamed, inserted or
counted."""
import numpy as np
import pytest

from tests.helpers import TOL, OracleStack, rel_err
from workload import MoEConfig, Workload, widen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("int4", [False, True])
@pytest.mark.parametrize("n", [1, 7, 40, 300])
def test_prompt_through_a_resident_layer(int4, n):
    import torch
    from paper_2602_11192_amd import pool as P
    cfg = MoEConfig("prefill_resident", 43, "bf16", 1, 256, 160, 12, 1, 3, 12, 8, 40, 0, 1.0, 3, 3, 1e-3)
    wl = Workload(cfg)
    cache = P.make_cache(wl, capacity=12, max_batch=n, trace_capacity=4096, fetch_mode=P.B.MOE_FETCH_IN_KERNEL, int4=int4)
    ost = OracleStack(wl, capacity=12, keep=12, int4=int4)
    toks = np.concatenate([wl.tokens(s) for s in range(8)])[:n]
    bias = np.stack([wl.bias(0, i // 40) for i in range(n)])
    x, b = P.to_device(toks), torch.from_numpy(bias).cuda()
    for e in range(12):                       # one-token calls fill the layer; none of them is waited for
        one = np.full((1, 12), -50.0, np.float32)
        one[0, [e, (e + 1) % 12, (e + 2) % 12]] = 0.0
        cache.moe_layer_decode(0, x[:1], torch.empty_like(x[:1]), torch.from_numpy(one).cuda())
        ost.decode(0, widen(toks[:1]), one, compute_y=False)
    before = cache.moe_cache_stats(0)
    assert cache.moe_cache_resident(0) == list(range(12))
    res = ost.prefill(0, widen(toks), bias)
    for _ in range(3):
        print("prompt through a resident layer", int4, n, flush=True)
        y = torch.full((n, 256), 7.0, dtype=torch.bfloat16, device="cuda:0")
        idx = torch.full((n, 3), -1, dtype=torch.int32, device="cuda:0")
        cache.moe_layer_prefill(0, x, y, b, idx, None)
        torch.cuda.synchronize()
        assert idx.cpu().numpy().tolist() == res.idx.tolist()
        assert rel_err(P.to_numpy(y), res.y).max() <= TOL["bf16"]
    assert cache.moe_cache_stats(0) == before and before["stream_loads"] == 0
    cache.close()
