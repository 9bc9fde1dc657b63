"""Which router matrix a call reads: a batched decode call, a prompt, or a call on a constrained cache follows the caller's
router_w as it is at the call, also with in-kernel fetch (where create makes a copy for the smallest calls); and such a
call routes bit for bit as the allocation-free entry point does on the same tokens."""
import numpy as np
import pytest

from tests.helpers import TOL
from tests.test_gpu_route_tile import layer64

pytestmark = pytest.mark.gpu

E, K, D, F = 64, 4, 256, 32


@pytest.fixture(scope="module")
def torch():
    import torch as t
    assert t.cuda.is_available(), "these tests need the MI355X"
    return t


def inputs(torch, B, batch):
    gen = torch.Generator().manual_seed(batch)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, D) * 0.3).bfloat16(), rnd(batch, D).bfloat16(), rnd(batch, E)
    blocks = (rnd(E, 3 * D * F) * 0.1).bfloat16()
    pool = blocks.reshape(-1).clone()
    for src, dst in zip(blocks, pool.view(E, -1)):
        B.moe_pack_expert(src.view(torch.int16).numpy().view(np.uint16), dst.view(torch.int16).numpy().view(np.uint16), D, F)
    return router, x, bias, blocks, pool


def make(B, router, pool, capacity, batch, **kw):
    return B.MoECache(n_layers=1, n_experts=E, top_k=K, d_model=D, d_ff=F, capacity=capacity, dtype=B.MOE_DTYPE_BF16,
                      router_w=router, expert_pool=pool.pin_memory(), max_batch=batch, pool_layout=B.MOE_LAYOUT_TILED,
                      fetch_mode=B.MOE_FETCH_IN_KERNEL, **kw)


@pytest.mark.parametrize("call,capacity,batch", [("decode", 64, 5), ("decode", 64, 16), ("decode", 64, 40), ("decode", 16, 2),
                                                 ("decode", 16, 17), ("prefill", 16, 33), ("prefill", 64, 4)])
def test_a_router_changed_in_place_is_followed(torch, call, capacity, batch):
    from paper_2602_11192_amd import binding as B
    router, x, bias, blocks, pool = inputs(torch, B, batch)
    rd, xd, bd = router.cuda(), x.cuda(), bias.cuda()
    cache = make(B, rd, pool, capacity, batch)
    cache.moe_cache_prefill_pins(0, list(range(capacity)))
    for matrix in (router, router.flip(0).contiguous()):
        print("router matrix test", call, capacity, batch, flush=True)
        rd.copy_(matrix)
        idx, w, y, gap = layer64(torch, x, matrix, bias, blocks, [], K, D, F)
        sure = gap > 1e-5                     # fp32 logits of a few units are off by under 1e-5
        yd = torch.full((batch, D), 7.0, dtype=torch.bfloat16, device="cuda:0")
        i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        wd = torch.full((batch, K), -1.0, device="cuda:0")
        (cache.moe_layer_decode if call == "decode" else cache.moe_layer_prefill)(0, xd, yd, bd, i, wd)
        torch.cuda.synchronize()
        assert torch.equal(i.cpu().long()[sure], idx[sure])
        assert float((wd.cpu().double() - w)[sure].abs().max()) < 1e-5
        err = (yd.cpu().double() - y).abs().max(-1).values / y.abs().max(-1).values
        assert float(err[sure].max()) <= TOL["bf16"]
    cache.close()


@pytest.mark.parametrize("batch", [5, 16, 31, 40, 130])
def test_batched_calls_route_as_the_allocation_free_entry_point(torch, batch):
    same_as_allocation_free(torch, batch)


# caches whose tables are not the register table (neither takes the single launch, so two tokens are a batched call, too)
@pytest.mark.parametrize("policy,staging", [("gamma", 0), ("lru", 16)])
@pytest.mark.parametrize("batch", [2, 16, 40, 111, 130])
def test_full_caches_of_any_policy_and_spare_buffers_do(torch, policy, staging, batch):
    from paper_2602_11192_amd import binding as B
    same_as_allocation_free(torch, batch, staging_buffers=staging, **(dict(policy=B.MOE_POLICY_GAMMA, gamma=0.9) if policy == "gamma" else {}))


def same_as_allocation_free(torch, batch, **kw):
    from paper_2602_11192_amd import binding as B
    router, x, bias, blocks, pool = inputs(torch, B, batch)
    rd, xd, bd = router.cuda(), x.cuda(), bias.cuda()
    cache = make(B, rd, pool, E, batch, **kw)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    print("same routing, batch", batch, flush=True)
    out = []
    for run in (lambda y, i, w: cache.moe_layer_decode(0, xd, y, bd, i, w),
                lambda y, i, w: B.moe_layer_decode_resident_noalloc(
                    n_experts=E, top_k=K, d_model=D, d_ff=F, dtype=B.MOE_DTYPE_BF16, pool_layout=B.MOE_LAYOUT_TILED,
                    router_w=rd, experts=pool.cuda(), x=xd, y=y, logit_bias=bd, topk_idx=i, topk_w=w)):
        y = torch.full((batch, D), 7.0, dtype=torch.bfloat16, device="cuda:0")
        i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        w = torch.full((batch, K), -1.0, device="cuda:0")
        run(y, i, w)
        torch.cuda.synchronize()
        out.append((i.cpu(), w.cpu(), y.cpu().view(torch.int16)))
    for a, b in zip(*out):
        assert torch.equal(a, b)
    cache.close()


def test_spare_buffers_choose_no_other_expert_kernel(torch):
    # 6 tokens x 2 of 8 experts of 29 MB: the one-launch FFN; were every pair to have a buffer of its own, the grouped GEMM
    from paper_2602_11192_amd import binding as B
    n, k, d, f, batch = 8, 2, 2048, 2400, 6
    gen = torch.Generator(device="cuda:0").manual_seed(1)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda:0")
    router, x, bias = (rnd(n, d) * d ** -0.5).bfloat16(), rnd(batch, d).bfloat16(), rnd(batch, n)
    blocks = (rnd(n * 3 * d * f) * d ** -0.5).bfloat16()         # (any values in tiled order are an expert)
    y = [torch.full((batch, d), 7.0, dtype=torch.bfloat16, device="cuda:0") for _ in range(2)]
    shape = dict(n_experts=n, top_k=k, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16, pool_layout=B.MOE_LAYOUT_TILED, router_w=router)
    B.moe_layer_decode_resident_noalloc(experts=blocks, x=x, y=y[0], logit_bias=bias, **shape)
    cache = B.MoECache(n_layers=1, n_shared=0, capacity=n, expert_pool=blocks.cpu().pin_memory(), max_batch=batch, staging_buffers=8,
                       fetch_mode=B.MOE_FETCH_IN_KERNEL, **shape)
    cache.moe_cache_prefill_pins(0, list(range(n)))
    cache.moe_layer_decode(0, x, y[1], bias)
    torch.cuda.synchronize()
    assert torch.equal(y[0], y[1])
    cache.close()
