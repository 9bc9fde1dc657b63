"""Routing of a batch in units of 16 tokens x 16 experts x a slice of the contraction: every lookup hits on a cache that does not hold
every expert, pairs put in order in LDS at the limits of that, calls of more than 1024 tokens, contractions that the slices do
not divide, more experts than slots; against a stable sort of the selected experts and the layer in 64 bits."""
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


# (1024 / 12288 pairs are the limits of the ordering in LDS, 1024 tokens a pass of the grouping)
@pytest.mark.parametrize("batch,E,K,ns,d,held", [(2, 24, 3, 0, 2080, 24), (17, 64, 8, 1, 64, 40), (127, 60, 8, 0, 64, 60),
                                                 (128, 64, 8, 0, 64, 30), (120, 8, 2, 1, 96, 6), (1024, 64, 8, 0, 32, 50),
                                                 (1025, 32, 7, 1, 32, 32), (2100, 24, 3, 0, 32, 20), (16, 33, 4, 64, 1056, 30),
                                                 # more experts than slots of the register table
                                                 (112, 65, 2, 0, 64, 64), (130, 100, 5, 1, 2080, 60), (1030, 256, 3, 0, 32, 40),
                                                 # pairs in LDS that are no multiple of four; a wave's second round over its chain;
                                                 # units of several expert tiles (above, too), of all of them
                                                 (147, 64, 7, 0, 64, 64), (1024, 64, 4, 0, 4128, 64), (4100, 20, 2, 0, 32, 20),
                                                 (1365, 64, 8, 1, 64, 50), (1366, 64, 8, 1, 64, 64)])
def test_batch_that_hits(torch, B, batch, E, K, ns, d, held):
    f = 32
    gen = torch.Generator().manual_seed(batch * 1000 + E)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, d) * 0.3 / (d / 64) ** 0.5).bfloat16(), rnd(batch, d).bfloat16(), rnd(batch, E)
    lost = torch.randperm(E, generator=gen)[held:]
    bias[:, lost] -= 1e4                                   # nobody selects the experts that the cache does not hold
    blocks, shared = (rnd(E, 3 * d * f) * 0.1).bfloat16(), (rnd(ns, 3 * d * f) * 0.1).bfloat16()
    idx, w, y, gap = layer64(torch, x, router, bias, blocks, shared, K, d, f)
    # fp32 logits of a few units are off by under 1e-5: tokens whose rank K is closer than that have no fixed set
    sure = gap > 1e-5
    assert sure.float().mean() > 0.9
    cache = B.MoECache(n_layers=1, n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, capacity=held, dtype=B.MOE_DTYPE_BF16,
                       router_w=router.cuda(), expert_pool=blocks.reshape(-1).pin_memory(), max_batch=batch,
                       shared_w=shared.reshape(-1).cuda() if ns else None, trace_capacity=2 * batch * K,
                       pool_layout=B.MOE_LAYOUT_ROWMAJOR, fetch_mode=B.MOE_FETCH_COPY_ENGINE)
    order = [e for e in torch.randperm(E, generator=gen).tolist() if e not in set(lost.tolist())]
    cache.moe_cache_prefill_pins(0, order)
    xd, bd = x.cuda(), bias.cuda()
    seen = []
    for _ in range(2):
        yd = torch.full((batch, d), 7.0, dtype=torch.bfloat16, device="cuda:0")
        i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        wd = torch.full((batch, K), -1.0, device="cuda:0")
        cache.moe_layer_decode(0, xd, yd, bd, i, wd)
        torch.cuda.synchronize()
        i, wd, yd = i.cpu().long(), wd.cpu().double(), yd.cpu().double()
        assert torch.equal(i[sure], idx[sure])
        assert float((wd - w)[sure].abs().max()) < 1e-5
        err = (yd - y).abs().max(-1).values / y.abs().max(-1).values
        assert float(err[sure].max()) <= TOL["bf16"]
        seen.append(i.reshape(-1).numpy())
    rec, total = cache.moe_cache_read_trace(0)
    assert total == 2 * batch * K
    assert rec[:, 1].tolist() == np.concatenate(seen).tolist()
    assert rec[:, 0].tolist() == 2 * np.repeat(np.arange(batch), K).tolist()
    assert rec[:, 2].tolist() == [1] * total and rec[:, 3].tolist() == [-1] * total
    st = cache.moe_cache_stats(0)
    assert st["hits"] == total and st["misses"] == 0 and st["evictions"] == 0
    if held < E:
        # recency: whoever was looked up last the longest ago goes first when the lost experts are asked for
        last = {e: n for n, e in enumerate(order)}
        last.update({int(e): len(order) + n for n, e in enumerate(np.concatenate(seen))})
        want = sorted(order, key=lambda e: last[e])
        n_new = min(K, len(lost))
        b2 = torch.full((1, E), -1e4)
        b2[0, lost[:n_new]] = 1e4
        kept = [e for e in reversed(want)][:K - n_new]
        if kept:
            b2[0, kept] = 5e3
        cache.moe_layer_decode(0, xd[:1], torch.empty(1, d, dtype=torch.bfloat16, device="cuda:0"), b2.cuda(), None, None)
        assert sorted(cache.moe_cache_resident(0)) == sorted(set(order) - set(want[:n_new]) | set(lost[:n_new].tolist()))
    cache.close()


# (slices by batch: 64 x 2048 and 64 x 4128 one at 960 tokens, two at 512, four below; 32 x 4128 and 17 x 2080 two and four; 16 x 1056 two.
# 4128, 2080 and 1056 columns are not divided by them)
@pytest.mark.parametrize("E,d", [(64, 2048), (64, 4128), (32, 4128), (17, 2080), (16, 1056)])
def test_logits_do_not_depend_on_the_batch(torch, B, E, d):
    K, f = 2, 32
    gen = torch.Generator().manual_seed(E + d)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, d) * 2 / d ** 0.5).bfloat16(), rnd(960, d).bfloat16(), rnd(960, E)
    z = x.double() @ router.double().t() + bias.double()
    top = torch.topk(z, K + 1, dim=-1)
    sure = top.values[:, K - 1] - top.values[:, K] > 1e-5        # fp32 logits of a few units are off by under 1e-5
    want = top.indices[:, :K].sort(-1).values
    rd, xd, bd = router.cuda(), x.cuda(), bias.cuda()
    blocks = (rnd(E * 3 * d * f) * 0.1).bfloat16().cuda()

    def run(rows):
        n = rows.stop - rows.start
        i, w = torch.empty(n, K, dtype=torch.int32, device="cuda:0"), torch.empty(n, K, device="cuda:0")
        # (weights that are not normalised over the two show every bit of the logits)
        B.moe_layer_decode_resident_noalloc(n_experts=E, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16, norm_topk=0,
                                            pool_layout=B.MOE_LAYOUT_ROWMAJOR, router_w=rd, experts=blocks, x=xd[rows],
                                            y=torch.empty(n, d, dtype=torch.bfloat16, device="cuda:0"), logit_bias=bd[rows], topk_idx=i, topk_w=w)
        torch.cuda.synchronize()
        return i.cpu(), w.cpu()
    i, w = run(slice(0, 960))
    assert torch.equal(i.long()[sure], want[sure])
    assert float((w.double() - torch.softmax(z, -1).gather(1, i.long())).abs().max()) < 1e-5
    for rows in (slice(0, 512), slice(100, 356), slice(500, 533), slice(900, 916), slice(7, 9)):
        ri, rw = run(rows)
        assert torch.equal(ri, i[rows]) and torch.equal(rw, w[rows])
