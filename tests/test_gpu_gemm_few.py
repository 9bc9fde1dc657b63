"""Grouped bf16 GEMM for calls of up to 16 tokens: contractions shorter than the ring is deep, and of every remainder, row tiles that
the last workgroup lacks, one and two row tiles per wave; against the layer in 64 bits.  A token's result does not depend on how many others share the call."""
import numpy as np
import pytest

from tests.helpers import TOL
from tests.test_gpu_route_tile import layer64

pytestmark = pytest.mark.gpu


# (E copies of few experts' shapes: more tokens than the one-launch kernel takes; d a multiple of 128, f of 32)
@pytest.mark.parametrize("batch,E,K,ns,d,f", [(7, 8, 2, 0, 128, 32), (9, 4, 2, 1, 256, 96), (16, 16, 4, 0, 384, 160), (16, 2, 2, 0, 512, 224),
                                              (12, 64, 8, 2, 640, 480), (10, 8, 1, 0, 2176, 512), (16, 24, 8, 1, 2560, 64)])
def test_few_tokens(batch, E, K, ns, d, f):
    import torch
    from paper_2602_11192_amd import binding as B
    gen = torch.Generator().manual_seed(batch * 1000 + f)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    scale = 0.8 / d ** 0.5
    router, x, bias = (rnd(E, d) * scale).bfloat16(), rnd(batch, d).bfloat16(), rnd(batch, E)
    blocks, shared = (rnd(E, 3 * d * f) * scale).bfloat16(), (rnd(ns, 3 * d * f) * scale).bfloat16()
    idx, w, y, gap = layer64(torch, x, router, bias, blocks, shared, K, d, f)
    sure = gap > 1e-5                       # (fp32 logits of a few units are off by under 1e-5)

    def pack(b):
        out = b.clone()
        for src, dst in zip(b, out):
            B.moe_pack_expert(src.view(torch.int16).numpy().view(np.uint16), dst.view(torch.int16).numpy().view(np.uint16), d, f)
        return out.reshape(-1).cuda()
    yd = torch.full((batch, d), 7.0, dtype=torch.bfloat16, device="cuda:0")
    i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
    for _ in range(2):
        B.moe_layer_decode_resident_noalloc(n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16,
                                            pool_layout=B.MOE_LAYOUT_TILED, router_w=router.cuda(), experts=pack(blocks),
                                            shared_w=pack(shared) if ns else None, x=x.cuda(), y=yd, logit_bias=bias.cuda(), topk_idx=i,
                                            topk_w=None)
        torch.cuda.synchronize()
        assert torch.equal(i.cpu().long()[sure], idx[sure])
        err = (yd.cpu().double() - y).abs().max(-1).values / y.abs().max(-1).values
        assert float(err[sure].max()) <= TOL["bf16"]


# (17 tokens: the staged kernel, 9 to 16: the one without staging; fewer than 64 groups and more.  Rows enough that sums in another order
# would round some to another bf16 number)
@pytest.mark.parametrize("E,K,ns,d,f", [(4, 4, 0, 1024, 4096), (64, 8, 2, 512, 1024)])
def test_the_same_bits_beside_more_tokens(E, K, ns, d, f):
    import torch
    from paper_2602_11192_amd import binding as B
    gen = torch.Generator().manual_seed(d)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, d) * d ** -0.5).bfloat16().cuda(), rnd(17, d).bfloat16().cuda(), rnd(17, E).cuda()
    # (any values in tiled order are an expert: nothing is compared with another layout)
    blocks, shared = (rnd(E * 3 * d * f) * d ** -0.5).bfloat16().cuda(), (rnd(ns * 3 * d * f) * d ** -0.5).bfloat16().cuda()

    def run(n):
        y, w = torch.empty(n, d, dtype=torch.bfloat16, device="cuda:0"), torch.empty(n, K, device="cuda:0")
        B.moe_layer_decode_resident_noalloc(n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16,
                                            pool_layout=B.MOE_LAYOUT_TILED, router_w=router, experts=blocks,
                                            shared_w=shared if ns else None, x=x[:n], y=y, logit_bias=bias[:n], topk_idx=None, topk_w=w)
        torch.cuda.synchronize()
        return y, w
    y, w = run(17)
    for n in (9, 13, 16):
        yn, wn = run(n)
        assert torch.equal(wn, w[:n]) and torch.equal(yn, y[:n])
