"""One-token calls whose workgroups form the router logits together: every workgroup brings a unit of 16 experts x a slice of the
contraction and takes the others' from its die's L2.  Shapes with several units per workgroup, one, and fewer units than
workgroups, ragged last tiles and slices, all three expert kernels; and the words of one call must not reach the next."""
import numpy as np
import pytest

from tests.helpers import TOL, OracleStack, compare_traces_and_stats, rel_err, run_sequence_serial
from tests.test_gpu_parity import small_cfg
from workload import Workload, widen

pytestmark = pytest.mark.gpu

# experts, top-k, capacity, shared experts, d_model, d_ff
CHUNK = [(256, 8, 20, 0, 512, 64),       # 16 units for two workgroups of a die
         (100, 5, 24, 1, 1024, 96),      # seven tiles, the last of four experts
         (48, 4, 10, 0, 1536, 160),      # four waves; 48 k-blocks in one slice
         (64, 8, 16, 0, 2048, 128),      # four units for four workgroups
         (60, 6, 12, 0, 4096, 352)]      # two slices of 64 k-blocks
TILES = [(72, 8, 16, 1, 1024, 1152), (64, 6, 8, 2, 2048, 1408)]
INT4 = [(256, 8, 20, 0, 512, 64), (48, 4, 10, 0, 1536, 160), (100, 5, 24, 1, 1280, 96), (64, 8, 16, 0, 2048, 256)]


@pytest.mark.parametrize("int4,shape", [(False, s) for s in CHUNK + TILES] + [(True, s) for s in INT4])
def test_one_token_calls(int4, shape):
    import torch
    from paper_2602_11192_amd import pool as P
    E, K, cap, ns, d, f = shape
    print("shared logits", int4, shape, flush=True)
    cfg = small_cfg(n_experts=E, top_k=K, capacity=cap, n_shared=ns, d_model=d, d_ff=f, n_layers=2, n_seqs=2, n_steps=6, pref_lo=min(K, 4),
                    pref_hi=K + 1, beta=2.0, cfg_id=71)
    wl = Workload(cfg)
    cache = P.make_cache(wl, tiled=not int4, int4=int4, trace_capacity=4096, fetch_mode=P.B.MOE_FETCH_IN_KERNEL)
    ost = OracleStack(wl, keep=24, int4=int4)
    _, _, traces = run_sequence_serial(wl, cache, ost, torch=torch, y_every=2)
    compare_traces_and_stats(cache, ost, traces, P.int4_block_bytes(cfg) if int4 else cfg.expert_bytes)
    cache.close()


@pytest.mark.parametrize("int4", [False, True])
def test_replays_of_a_captured_call(int4):
    """A recorded call carries the same number in every replay: its words would pass for the next one's if they were left standing."""
    import torch
    from paper_2602_11192_amd import pool as P
    E, K, d, f = 64, 8, 2048, 128 if not int4 else 256
    cfg = small_cfg(n_experts=E, top_k=K, capacity=E, d_model=d, d_ff=f, n_layers=1, n_seqs=4, n_steps=8, pref_lo=4, pref_hi=9, cfg_id=72)
    wl = Workload(cfg)
    cache = P.make_cache(wl, tiled=not int4, int4=int4, fetch_mode=P.B.MOE_FETCH_IN_KERNEL)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    ost = OracleStack(wl, capacity=E, keep=E, int4=int4)
    tokens = [wl.tokens(s)[t] for s in range(4) for t in range(4)]
    x = P.to_device(np.stack(tokens[:1]))
    y = torch.empty((1, d), dtype=torch.bfloat16, device="cuda:0")
    idx = torch.empty((1, K), dtype=torch.int32, device="cuda:0")
    eager = torch.empty_like(y)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        cache.moe_layer_decode(0, x, y, None, idx)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        cache.moe_layer_decode(0, x, y, None, idx)
    for i, tok in enumerate(tokens):
        x.copy_(P.to_device(tok[None]))
        graph.replay()
        if i % 3 == 2:
            cache.moe_layer_decode(0, x, eager)
        torch.cuda.synchronize()
        res = ost.decode(0, widen(tok[None]), None)
        assert idx.cpu().numpy().tolist() == res.idx.tolist(), i
        assert float(rel_err(P.to_numpy(y), res.y)[0]) <= TOL["bf16"], i
        if i % 3 == 2:
            assert torch.equal(y.view(torch.int16), eager.view(torch.int16)), i
    cache.close()


@pytest.mark.parametrize("int4,shape", [(False, CHUNK[0]), (False, CHUNK[1]), (False, CHUNK[3]), (False, TILES[0]), (True, INT4[0]), (True, INT4[3])])
def test_logits_that_do_not_arrive_in_time(int4, shape):
    """A workgroup whose looks for the others' logits were in vain forms all of them by itself.  Here all workgroups do without looking, or every other
    one of a die while the rest take what arrives (the bookkeeping one is among the odd): selections, weights, outputs, trace and counters keep their bits."""
    import torch
    from paper_2602_11192_amd import pool as P
    E, K, cap, ns, d, f = shape
    cfg = small_cfg(n_experts=E, top_k=K, capacity=cap, n_shared=ns, d_model=d, d_ff=f, n_layers=1, n_seqs=1, n_steps=5, pref_lo=min(K, 4),
                    pref_hi=K + 1, beta=2.0, cfg_id=73)
    wl = Workload(cfg)
    x = P.to_device(wl.tokens(0))
    bias = torch.from_numpy(wl.bias(0, 0)[None, :]).cuda()
    runs = []
    for blind in (0, 3, 2, 1):
        print("blind", blind, int4, shape, flush=True)
        cache = P.make_cache(wl, tiled=not int4, int4=int4, trace_capacity=256, fetch_mode=P.B.MOE_FETCH_IN_KERNEL)
        assert P.B.lib.moe_test_share_blind(cache._h, blind) == 0
        out = []
        for t in range(cfg.n_steps):
            y = torch.empty((1, d), dtype=torch.bfloat16, device="cuda:0")
            idx = torch.empty((1, K), dtype=torch.int32, device="cuda:0")
            w = torch.empty((1, K), dtype=torch.float32, device="cuda:0")
            cache.moe_layer_decode(0, x[t:t + 1], y, bias, idx, w)
            out += [y.view(torch.int16), idx, w.view(torch.int32)]
        torch.cuda.synchronize()
        trace, total = cache.moe_cache_read_trace(0)
        runs.append([o.cpu().tolist() for o in out] + [trace.tolist(), total, cache.moe_cache_stats(0)])
        cache.close()
    assert runs[0][-1]["misses"] > 0 and runs[0][-2] == cfg.n_steps * K
    for other in runs[1:]:
        assert other == runs[0]
