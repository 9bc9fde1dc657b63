"""Calls of a few tokens on a layer that is known to be resident: which of them stay with the single launch."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("int4", [False, True])
def test_int4_leaves_the_single_launch_beyond_two_workgroups_a_unit(int4):
    """8 experts of 1024 x 4096, top-2: 128 workgroups per pair, 512 at two tokens and 768 at three; workgroups x E x d stays
    under 10 M, far below the line at which bf16 experts leave it."""
    import torch
    from paper_2602_11192_amd import binding as B
    d, f, E, K = 1024, 4096, 8, 2
    layout = B.MOE_LAYOUT_TILED_INT4 if int4 else B.MOE_LAYOUT_TILED
    pool = torch.zeros(E * B.moe_expert_block_bytes(d, f, B.MOE_DTYPE_BF16, layout), dtype=torch.uint8).pin_memory()
    cache = B.MoECache(n_layers=1, n_experts=E, top_k=K, d_model=d, d_ff=f, capacity=E, dtype=B.MOE_DTYPE_BF16,
                       router_w=torch.zeros(1, E, d, dtype=torch.bfloat16, device="cuda:0"), expert_pool=pool, max_batch=4,
                       pool_layout=layout, fetch_mode=B.MOE_FETCH_IN_KERNEL)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    cache.moe_cache_set_profiling(True)
    for batch, single in ((1, True), (2, True), (3, not int4), (4, not int4)):
        print("small batch", int4, batch, flush=True)
        cache.moe_cache_timing(clear=True)
        x = torch.zeros(batch, d, dtype=torch.bfloat16, device="cuda:0")
        cache.moe_layer_decode(0, x, torch.empty_like(x))
        tm = cache.moe_cache_timing(clear=True)
        assert tm["decode_single_launches"] == int(single) and tm["route_launches"] == int(not single)
    cache.close()


@pytest.mark.parametrize("int4,d,f,E,K,batch,gemm", [
    (True, 512, 12288, 16, 4, 10, False), (True, 2048, 8192, 8, 2, 16, False), (True, 2048, 1024, 64, 8, 6, True),
    (True, 2048, 1024, 64, 8, 4, False), (False, 1536, 6144, 8, 2, 4, False), (False, 1536, 6144, 8, 2, 8, False),
    (False, 2048, 2048, 16, 4, 6, True), (False, 2048, 2048, 16, 4, 3, False)])
def test_where_the_grouped_gemm_takes_over(int4, d, f, E, K, batch, gemm):
    """Resident layers that read 120 MB (bf16 350 MB) and more a call: the GEMM from 5 (4) tokens on, unless d_model is so
    narrow that its down pass has fewer workgroups than the units need."""
    import torch
    from paper_2602_11192_amd import binding as B
    layout = B.MOE_LAYOUT_TILED_INT4 if int4 else B.MOE_LAYOUT_TILED
    pool = torch.zeros(E * B.moe_expert_block_bytes(d, f, B.MOE_DTYPE_BF16, layout), dtype=torch.uint8).pin_memory()
    cache = B.MoECache(n_layers=1, n_experts=E, top_k=K, d_model=d, d_ff=f, capacity=E, dtype=B.MOE_DTYPE_BF16,
                       router_w=torch.zeros(1, E, d, dtype=torch.bfloat16, device="cuda:0"), expert_pool=pool,
                       max_batch=batch, pool_layout=layout)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    cache.moe_cache_set_profiling(True)
    cache.moe_cache_timing(clear=True)
    print("GEMM or one launch", int4, d, f, batch, flush=True)
    x = torch.zeros(batch, d, dtype=torch.bfloat16, device="cuda:0")
    cache.moe_layer_decode(0, x, torch.empty_like(x))
    tm = cache.moe_cache_timing(clear=True)
    assert (tm["ffn_launches"], tm["ffn_fused_launches"]) == ((1, 0) if gemm else (0, 1))
    cache.close()
