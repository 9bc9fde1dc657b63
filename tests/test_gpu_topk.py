"""Top-K selection on logits that a random router hardly produces: ties, both zeros, infinities, one value repeated.
Zero hidden states make the logits equal to the bias; the expected set is a stable descending sort (ties to the lower
id), returned in ascending id order."""
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


def rows_of(E, rng):
    ties = rng.integers(-2, 3, E).astype(np.float32)
    return np.stack([np.zeros(E, np.float32),
                     np.where(np.arange(E) % 2, 0.0, -0.0).astype(np.float32),
                     ties, -ties - 100.0,
                     rng.standard_normal(E).astype(np.float32) * 1e30,
                     np.where(rng.random(E) < 0.5, -np.inf, 1.0).astype(np.float32),
                     np.arange(E, dtype=np.float32), -np.arange(E, dtype=np.float32),
                     (1.0 + np.arange(E) * 2.0 ** -23).astype(np.float32)])      # neighbouring floats


def expected(bias, K):
    return np.sort(np.argsort(-bias.astype(np.float64), axis=1, kind="stable")[:, :K], axis=1)


@pytest.mark.parametrize("E,K", [(2, 1), (8, 8), (63, 7), (64, 8), (64, 64), (65, 2), (256, 8), (1024, 17)])
def test_topk_of_the_router_kernel(torch, B, E, K):
    d, f = 64, 32
    bias = rows_of(E, np.random.default_rng(E + K))
    n = len(bias)
    x = torch.zeros(n, d, device="cuda:0")
    y = torch.empty_like(x)
    idx = torch.full((n, K), -1, dtype=torch.int32, device="cuda:0")
    B.moe_layer_decode_resident_noalloc(
        n_experts=E, top_k=K, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_FP32, pool_layout=B.MOE_LAYOUT_ROWMAJOR,
        router_w=torch.zeros(E, d, device="cuda:0"), experts=torch.zeros(E * 3 * d * f, device="cuda:0"), x=x, y=y,
        logit_bias=torch.from_numpy(bias).cuda(), topk_idx=idx)
    torch.cuda.synchronize()
    assert idx.cpu().numpy().tolist() == expected(bias, K).tolist()


@pytest.mark.parametrize("E,K", [(8, 2), (63, 7), (64, 8), (64, 32)])
@pytest.mark.parametrize("batch", [1, 2])
def test_topk_of_the_single_launch_call(torch, B, E, K, batch):
    d, f = 256, 32
    rng = np.random.default_rng(E * K)
    bias = rows_of(E, rng)
    bias[~np.isfinite(bias)] = -50.0
    pool = torch.zeros(E * 3 * d * f, dtype=torch.bfloat16).pin_memory()
    cache = B.MoECache(n_layers=1, n_experts=E, top_k=K, d_model=d, d_ff=f, capacity=E, dtype=B.MOE_DTYPE_BF16,
                       router_w=torch.zeros(1, E, d, dtype=torch.bfloat16, device="cuda:0"), expert_pool=pool,
                       max_batch=batch, trace_capacity=4096, pool_layout=B.MOE_LAYOUT_TILED,
                       fetch_mode=B.MOE_FETCH_IN_KERNEL)
    cache.moe_cache_prefill_pins(0, list(range(E)))
    for r in range(len(bias) - batch + 1):
        b = torch.from_numpy(bias[r:r + batch].copy()).cuda()
        x = torch.zeros(batch, d, dtype=torch.bfloat16, device="cuda:0")
        y = torch.empty_like(x)
        idx = torch.full((batch, K), -1, dtype=torch.int32, device="cuda:0")
        cache.moe_layer_decode(0, x, y, b, idx)
        torch.cuda.synchronize()
        assert idx.cpu().numpy().tolist() == expected(bias[r:r + batch], K).tolist()
        assert torch.equal(y.float(), torch.zeros_like(y, dtype=torch.float32))
    rec, total = cache.moe_cache_read_trace(0)
    assert total == (len(bias) - batch + 1) * batch * K and int(rec[:, 2].min()) == 1
    cache.close()
