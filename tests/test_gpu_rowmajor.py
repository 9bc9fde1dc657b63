"""Row-major experts: widths that are and are not whole 16-byte pieces of a W_d row and token counts around the four that a
wave takes at a time; fp32 and bf16, against the layer in 64 bits.  (Calls that one workgroup routes, at their limits:
test_gpu_small_fp32.py.)"""
import pytest

from tests.helpers import TOL
from tests.test_gpu_route_tile import layer64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("batch,E,K,ns,d,f", [(1, 8, 2, 0, 64, 128), (2, 4, 1, 1, 8, 4), (4, 8, 2, 0, 64, 128), (5, 3, 3, 0, 72, 37),
                                              (8, 16, 4, 0, 264, 250), (8, 17, 2, 0, 136, 8), (9, 2, 2, 1, 520, 258),
                                              (30, 4, 1, 0, 16, 1)])
def test_rowmajor_layer(dtype, batch, E, K, ns, d, f):
    import torch
    from paper_2602_11192_amd import binding as B
    tdt = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator().manual_seed(batch * 1000 + d)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, d) * d ** -0.5).to(tdt), rnd(batch, d).to(tdt), rnd(batch, E)
    blocks = (rnd(E + ns, 3 * d * f) * 0.1).to(tdt)
    idx, w, y, gap = layer64(torch, x, router, bias, blocks[:E], blocks[E:], K, d, f)
    sure = gap > 1e-5
    xd, yd = x.cuda(), torch.full((batch, d), 7.0, dtype=tdt, device="cuda:0")
    i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
    B.moe_layer_decode_resident_noalloc(
        n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_FP32 if dtype == "fp32" else B.MOE_DTYPE_BF16,
        pool_layout=B.MOE_LAYOUT_ROWMAJOR, router_w=router.cuda(), experts=blocks[:E].reshape(-1).cuda(),
        shared_w=blocks[E:].reshape(-1).cuda() if ns else None, x=xd, y=yd, logit_bias=bias.cuda(), topk_idx=i)
    torch.cuda.synchronize()
    assert torch.equal(i.cpu().long()[sure], idx[sure])
    err = (yd.cpu().double() - y).abs().max(-1).values / y.abs().max(-1).values
    assert float(err[sure].max()) <= TOL[dtype]
