"""Row-major experts that are all in memory, a workgroup per token: rows of fewer pieces than sixteen lanes, of odd piece counts around
32 and 64 lanes and of several rounds, row counts that are no multiple of what a workgroup holds, more pairs than waves, shared
experts, more groups than lanes; fp32 and bf16, through both entry points and in place, against the layer in 64 bits."""
import pytest

from tests.helpers import TOL
from tests.test_gpu_route_tile import layer64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("batch,E,K,ns,d,f", [
    (1, 8, 2, 0, 64, 128), (4, 8, 2, 0, 64, 128), (3, 4, 1, 1, 8, 8), (5, 3, 3, 0, 72, 40),
    (2, 24, 17, 1, 24, 16),        # more pairs than waves
    (70, 80, 2, 0, 136, 24),       # more groups than lanes
    (1, 4, 1, 0, 520, 24), (2, 4, 1, 0, 24, 520),       # rows of more than 64 pieces
    (300, 8, 2, 0, 64, 64), (128, 4, 2, 1, 128, 136),   # two rounds of workgroups; many pairs per expert
    # the same with so many tokens that both types run it: more pairs than waves, more groups than lanes, rows of more than 64 pieces
    (24, 4, 1, 1, 8, 8), (60, 24, 17, 1, 24, 16), (130, 80, 2, 0, 24, 16), (300, 80, 2, 0, 136, 24), (90, 4, 1, 0, 520, 24), (90, 4, 1, 0, 24, 520)])
def test_token_ffn(dtype, batch, E, K, ns, d, f):
    import torch
    from paper_2602_11192_amd import binding as B
    tdt = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator().manual_seed(batch * 1000 + d)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, d) * d ** -0.5).to(tdt), rnd(batch, d).to(tdt), rnd(batch, E)
    blocks = (rnd(E + ns, 3 * d * f) * 0.1).to(tdt)
    idx, w, y, gap = layer64(torch, x, router, bias, blocks[:E], blocks[E:], K, d, f)
    sure = gap > 1e-5
    dt = B.MOE_DTYPE_FP32 if dtype == "fp32" else B.MOE_DTYPE_BF16
    rd, bd = router.cuda(), bias.cuda()
    shared = blocks[E:].reshape(-1).cuda() if ns else None

    def check(run, in_place=False):
        xd = x.cuda()
        yd = xd if in_place else torch.full((batch, d), 7.0, dtype=tdt, device="cuda:0")
        i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        run(xd, yd, i)
        torch.cuda.synchronize()
        assert torch.equal(i.cpu().long()[sure], idx[sure])
        err = (yd.cpu().double() - y).abs().max(-1).values / y.abs().max(-1).values
        assert float(err[sure].max()) <= TOL[dtype]
        return yd

    experts = blocks[:E].reshape(-1).cuda()
    noalloc = lambda xd, yd, i: B.moe_layer_decode_resident_noalloc(
        n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, dtype=dt, pool_layout=B.MOE_LAYOUT_ROWMAJOR, router_w=rd,
        experts=experts, shared_w=shared, x=xd, y=yd, logit_bias=bd, topk_idx=i)
    first = check(noalloc)
    assert torch.equal(check(noalloc, in_place=True), first)
    cache = B.MoECache(n_layers=1, n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, capacity=E, dtype=dt, router_w=rd,
                       expert_pool=blocks[:E].reshape(-1).pin_memory(), shared_w=shared, max_batch=batch,
                       pool_layout=B.MOE_LAYOUT_ROWMAJOR, fetch_mode=B.MOE_FETCH_COPY_ENGINE)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    decode = lambda xd, yd, i: cache.moe_layer_decode(0, xd, yd, bd, i)
    assert torch.equal(check(decode), first)
    cache.close()


# spare buffers are beside the point where every expert is resident: the same kernels with and without, and through both entry points
@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_spare_buffers_of_a_full_layer(dtype):
    import torch
    from paper_2602_11192_amd import binding as B
    batch, E, K, d, f = 40, 8, 2, 128, 128
    tdt, dt = (torch.float32, B.MOE_DTYPE_FP32) if dtype == "fp32" else (torch.bfloat16, B.MOE_DTYPE_BF16)
    gen = torch.Generator().manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias, blocks = (rnd(E, d) * d ** -0.5).to(tdt).cuda(), rnd(batch, d).to(tdt).cuda(), rnd(batch, E).cuda(), (rnd(E * 3 * d * f) * 0.1).to(tdt)
    y = [torch.full((batch, d), 7.0, dtype=tdt, device="cuda:0") for _ in range(3)]
    shape = dict(n_experts=E, top_k=K, d_model=d, d_ff=f, dtype=dt, pool_layout=B.MOE_LAYOUT_ROWMAJOR, router_w=router)
    B.moe_layer_decode_resident_noalloc(experts=blocks.cuda(), x=x, y=y[0], logit_bias=bias, **shape)
    for i, spare in enumerate((0, 24)):
        cache = B.MoECache(n_layers=1, n_shared=0, capacity=E, expert_pool=blocks.pin_memory(), max_batch=batch, staging_buffers=spare,
                           fetch_mode=B.MOE_FETCH_COPY_ENGINE, **shape)
        cache.moe_cache_prefill_pins(0, list(range(E)))
        cache.moe_layer_decode(0, x, y[1 + i], bias)
        torch.cuda.synchronize()
        cache.close()
    assert torch.equal(y[1], y[0]) and torch.equal(y[2], y[0])
