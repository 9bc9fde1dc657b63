"""Batches at the limit of the allocation-free entry point's device array.  Beyond the tables, an accepted batch needs
4 NP (d_ff + d_model) bytes for its NP = batch (top_k + n_shared) pairs where the grouped GEMM runs it; that GEMM's work
list must not take more.  The refusals are made on the host, before the GPU is touched."""
import ctypes as C

import pytest


def scratch_refused(B, batch, **kw):
    f = dict(n_shared=0, dtype=B.MOE_DTYPE_BF16, norm_topk=1, pool_layout=B.MOE_LAYOUT_TILED, router_w=0x3000,
             experts=0x4000, shared_w=None)
    f.update(kw)
    f["shared_w"] = 0x5000 if f["n_shared"] else None
    layer = B.moe_resident_layer_t(**f)
    rc = B.lib.moe_layer_decode_resident_noalloc(C.byref(layer), 0x1000, None, batch, 0x2000, None, None, None)
    assert rc in (B.MOE_ERR_UNSUPPORTED, B.MOE_ERR_HIP), B.moe_last_error()
    return rc == B.MOE_ERR_UNSUPPORTED


@pytest.mark.parametrize("int4,batch,E,K,ns,d,f", [
    (0, 101, 256, 8, 1, 4096, 5120), (0, 88, 160, 8, 0, 4096, 7808), (0, 21, 200, 29, 0, 3360, 10400),
    (0, 1321, 512, 1, 0, 5696, 640), (1, 157, 200, 3, 1, 768, 12576), (1, 739, 400, 1, 1, 5632, 32),
    (0, 127, 256, 8, 1, 32, 7296)])
def test_a_batch_at_the_limit_is_accepted(int4, batch, E, K, ns, d, f):
    import torch
    from paper_2602_11192_amd import binding as B
    if torch.cuda.is_available():
        pytest.skip("an accepted call would run on these addresses")
    kw = dict(n_experts=E, top_k=K, n_shared=ns, d_model=d, d_ff=f,
              pool_layout=B.MOE_LAYOUT_TILED_INT4 if int4 else B.MOE_LAYOUT_TILED)
    assert not scratch_refused(B, batch, **kw), B.moe_last_error()
    assert scratch_refused(B, batch + batch // 8 + 1, **kw) and "scratch" in B.moe_last_error()


@pytest.mark.gpu
def test_results_at_the_limit():
    import numpy as np
    import torch
    from paper_2602_11192_amd import binding as B
    from tests.helpers import TOL
    from tests.test_gpu_route_tile import layer64
    batch, E, K, ns, d, f = 127, 256, 8, 1, 32, 7296
    gen = torch.Generator().manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=gen)
    router, x, bias = (rnd(E, d) * 0.3).bfloat16(), rnd(batch, d).bfloat16(), rnd(batch, E)
    blocks = torch.stack([(rnd(3 * d * f) * 0.1).bfloat16() for _ in range(E + ns)])
    idx, w, y, gap = layer64(torch, x, router, bias, blocks[:E], blocks[E:], K, d, f)
    sure = gap > 1e-5                     # fp32 logits of a few units are off by under 1e-5
    packed = torch.empty_like(blocks)
    for src, dst in zip(blocks, packed):
        B.moe_pack_expert(src.view(torch.int16).numpy().view(np.uint16), dst.view(torch.int16).numpy().view(np.uint16), d, f)
    packed = packed.cuda()
    for _ in range(2):
        print("allocation-free call at its limit", flush=True)
        yd = torch.full((batch, d), 7.0, dtype=torch.bfloat16, device="cuda:0")
        i = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        wd = torch.full((batch, K), -1.0, device="cuda:0")
        B.moe_layer_decode_resident_noalloc(
            n_experts=E, n_shared=ns, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16, pool_layout=B.MOE_LAYOUT_TILED,
            router_w=router.cuda(), experts=packed[:E], shared_w=packed[E:], x=x.cuda(), y=yd, logit_bias=bias.cuda(),
            topk_idx=i, topk_w=wd)
        torch.cuda.synchronize()
        assert torch.equal(i.cpu().long()[sure], idx[sure])
        assert float((wd.cpu().double() - w)[sure].abs().max()) < 1e-5
        err = (yd.cpu().double() - y).abs().max(-1).values / y.abs().max(-1).values
        assert float(err[sure].max()) <= TOL["bf16"]


@pytest.mark.parametrize("int4,batch,E,K,ns,d,f", [(1, 15, 400, 35, 64, 5632, 32), (0, 4, 128, 62, 0, 33792, 32)])
def test_a_batch_that_fits_the_one_launch_kernel_alone_is_accepted(int4, batch, E, K, ns, d, f):
    """Heavy layers take the GEMM from a few tokens on; where only the one-launch kernel's partial sums,
    NP (d_ff / 32) d_model floats, fit the array, that kernel runs."""
    import torch
    from paper_2602_11192_amd import binding as B
    if torch.cuda.is_available():
        pytest.skip("an accepted call would run on these addresses")
    kw = dict(n_experts=E, top_k=K, n_shared=ns, d_model=d, d_ff=f,
              pool_layout=B.MOE_LAYOUT_TILED_INT4 if int4 else B.MOE_LAYOUT_TILED)
    assert not scratch_refused(B, batch, **kw), B.moe_last_error()
