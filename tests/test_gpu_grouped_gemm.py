"""The grouped bf16 GEMM at the edges of its tiles: token counts around the column blocks and both tile sizes, more than one
tile per expert, contractions shorter than the ring and of odd length, row counts below a workgroup's block, experts
streamed from the host; against the layer in 64 bits."""
import numpy as np
import pytest

from tests.helpers import TOL
from tests.test_gpu_route_tile import layer64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "these tests need the MI355X"
    return t


@pytest.fixture(scope="module")
def B():
    from paper_2602_11192_amd import binding
    return binding


@pytest.mark.parametrize("batch,E,K,ns,d,f", [
    (7, 8, 2, 0, 32, 32),          # one k-block in either pass, two row tiles
    (9, 8, 2, 1, 96, 160),         # three and five k-blocks, odd numbers of row tiles per workgroup
    (16, 8, 2, 0, 2048, 96), (40, 4, 4, 1, 256, 128),
    (64, 2, 1, 0, 160, 1024), (65, 4, 1, 2, 160, 96),
    (80, 64, 2, 0, 64, 96),        # by-die order of the work list
    (257, 4, 4, 0, 288, 352),      # every expert one row more than the large tile
    (300, 2, 1, 1, 64, 64), (512, 3, 3, 0, 128, 32)])
def test_grouped_gemm(torch, B, batch, E, K, ns, d, f):
    gen = torch.Generator().manual_seed(batch * 100 + d)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, d) * d ** -0.5).bfloat16(), rnd(batch, d).bfloat16(), rnd(batch, E)
    blocks = (rnd(E + ns, 3 * d * f) * 0.1).bfloat16()
    idx, _, y, gap = layer64(torch, x, router, bias, blocks[:E], blocks[E:], K, d, f)
    sure = gap > 1e-5
    packed = torch.empty_like(blocks)
    for src, dst in zip(blocks, packed):
        B.moe_pack_expert(src.view(torch.int16).numpy().view(np.uint16), dst.view(torch.int16).numpy().view(np.uint16), d, f)
    pool = packed[:E].reshape(-1).pin_memory()
    shared = packed[E:].reshape(-1).cuda() if ns else None
    xd, bd, rd = x.cuda(), bias.cuda(), router.cuda()

    def check(run):
        yd = torch.full((batch, d), 7.0, dtype=torch.bfloat16, device="cuda:0")
        i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        run(yd, i)
        torch.cuda.synchronize()
        assert torch.equal(i.cpu().long()[sure], idx[sure])
        err = (yd.cpu().double() - y).abs().max(-1).values / y.abs().max(-1).values
        assert float(err[sure].max()) <= TOL["bf16"]
        return yd

    experts = pool.cuda()
    first = check(lambda yd, i: B.moe_layer_decode_resident_noalloc(
        n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16, pool_layout=B.MOE_LAYOUT_TILED,
        router_w=rd, experts=experts, shared_w=shared, x=xd, y=yd, logit_bias=bd, topk_idx=i))
    cap = max(K, E // 2)
    cache = B.MoECache(n_layers=1, n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, capacity=cap,
                       staging_buffers=E - cap, dtype=B.MOE_DTYPE_BF16, router_w=rd, expert_pool=pool, shared_w=shared,
                       max_batch=batch, pool_layout=B.MOE_LAYOUT_TILED, fetch_mode=B.MOE_FETCH_IN_KERNEL)
    cache.moe_cache_prefill_pins(0, list(range(cap)))
    check(lambda yd, i: cache.moe_layer_prefill(0, xd, yd, bd, i))        # half of the experts stream
    check(lambda yd, i: cache.moe_layer_decode(0, xd, yd, bd, i))         # ... and are fetched
    again = check(lambda yd, i: B.moe_layer_decode_resident_noalloc(
        n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16, pool_layout=B.MOE_LAYOUT_TILED,
        router_w=rd, experts=experts, shared_w=shared, x=xd, y=yd, logit_bias=bd, topk_idx=i))
    assert torch.equal(first.view(torch.int16), again.view(torch.int16))
    cache.close()
