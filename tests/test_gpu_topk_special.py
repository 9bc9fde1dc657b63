"""Top-K selection on logits with NaN (below everything, whatever its sign) and with infinities, through each kernel that
routes.  Zero hidden states make the logits equal to the bias; the expected set is a stable descending sort (ties to the
lower id), returned in ascending id order."""
import numpy as np
import pytest

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


def rows_of(E, K, rng):
    nan = np.float32(np.nan)
    one = rng.standard_normal(E).astype(np.float32)
    one[E // 2] = nan
    signs = rng.standard_normal(E).astype(np.float32)
    signs[::3], signs[1::3] = nan, np.copysign(nan, np.float32(-1.0))
    few = np.full(E, nan, np.float32)                                    # fewer values than are to be selected
    few[rng.permutation(E)[:K // 2]] = 1.0
    low = np.where(rng.random(E) < 0.5, -np.inf, nan).astype(np.float32)
    return np.stack([one, signs, few, low, np.full(E, nan, np.float32), np.full(E, -np.inf, np.float32),
                     np.where(rng.random(E) < 0.7, -np.inf, 1.0).astype(np.float32),
                     np.where(rng.random(E) < 0.3, np.inf, 1.0).astype(np.float32)])


def expected(bias, K):
    order = [sorted(range(len(r)), key=lambda e: (np.isnan(r[e]), -float(r[e]) if not np.isnan(r[e]) else 0.0, e)) for r in bias]
    return [sorted(o[:K]) for o in order]


# one wave per token in fp32; sixteen tokens a workgroup in bf16 (32 tokens and more on over 32 experts, 112 on fewer)
@pytest.mark.parametrize("dtype,E,K,batch", [("fp32", 8, 2, 16), ("fp32", 8, 2, 8), ("fp32", 64, 8, 8), ("fp32", 256, 17, 8),
                                             ("fp32", 1024, 8, 8), ("fp32", 100, 3, 8), ("fp32", 1024, 2, 8),
                                             ("bf16", 63, 7, 40), ("bf16", 200, 20, 120), ("bf16", 200, 4, 120),
                                             ("bf16", 16, 4, 120)])
def test_special_values_in_the_router_kernels(torch, B, dtype, E, K, batch):
    d, f = 64, 32
    bias = np.resize(rows_of(E, K, np.random.default_rng(E + K)), (batch, E))
    tdt = torch.float32 if dtype == "fp32" else torch.bfloat16
    x = torch.zeros(batch, d, dtype=tdt, device="cuda:0")
    idx = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
    print("special logits", dtype, E, K, batch, flush=True)
    B.moe_layer_decode_resident_noalloc(
        n_experts=E, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_FP32 if dtype == "fp32" else B.MOE_DTYPE_BF16,
        pool_layout=B.MOE_LAYOUT_ROWMAJOR, router_w=torch.zeros(E, d, dtype=tdt, device="cuda:0"),
        experts=torch.zeros(E * 3 * d * f, dtype=tdt, device="cuda:0"), x=x, y=torch.empty_like(x),
        logit_bias=torch.from_numpy(bias).cuda(), topk_idx=idx)
    torch.cuda.synchronize()
    assert idx.cpu().numpy().tolist() == expected(bias, K)


@pytest.mark.parametrize("E,K", [(8, 2), (63, 7), (64, 32)])
@pytest.mark.parametrize("batch", [1, 2])
@pytest.mark.parametrize("preloaded", [True, False])
def test_special_values_in_the_single_launch_call(torch, B, E, K, batch, preloaded):
    d, f = 256, 32
    bias = rows_of(E, K, np.random.default_rng(E * K))
    cache = B.MoECache(n_layers=1, n_experts=E, top_k=K, d_model=d, d_ff=f, capacity=E, dtype=B.MOE_DTYPE_BF16,
                       router_w=torch.zeros(1, E, d, dtype=torch.bfloat16, device="cuda:0"),
                       expert_pool=torch.zeros(E * 3 * d * f, dtype=torch.bfloat16).pin_memory(), max_batch=batch,
                       trace_capacity=4096, pool_layout=B.MOE_LAYOUT_TILED, fetch_mode=B.MOE_FETCH_IN_KERNEL)
    if preloaded:
        cache.moe_cache_prefill_pins(0, list(range(E)))
    requested = []
    for r in range(0, len(bias) - batch + 1):
        print("special logits, single launch", E, K, batch, r, flush=True)
        idx = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        x = torch.zeros(batch, d, dtype=torch.bfloat16, device="cuda:0")
        cache.moe_layer_decode(0, x, torch.empty_like(x), torch.from_numpy(bias[r:r + batch].copy()).cuda(), idx)
        torch.cuda.synchronize()
        want = expected(bias[r:r + batch], K)
        assert idx.cpu().numpy().tolist() == want
        requested += sum(want, [])
    rec, total = cache.moe_cache_read_trace(0)
    assert total == len(requested) and rec[:, 1].tolist() == requested
    cache.close()
