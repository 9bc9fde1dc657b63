"""The grouped bf16 GEMM where it takes its larger token tiles on resident experts: the middle tile (128 tokens) and the large
one (256), with rows and contractions that are no multiple of a workgroup's block, groups of one token more than a tile, and
the same call on a constrained cache, against the layer in 64 bits."""
import pytest

from tests.test_gpu_grouped_gemm import B, torch  # noqa: F401  (fixtures)
import tests.test_gpu_grouped_gemm as grouped

pytestmark = pytest.mark.gpu


def tile(batch, K, ns, E, d, f):
    """The rule of the host (plan_ffn_gemm), restated."""
    load, g = batch * (K + ns), min(batch * K, E) + ns
    tiles = lambda t: max(g, load / t + 0.5 * g)
    blocks = lambda rows, per: -(-rows // per)
    if load <= 40 * g or tiles(64) * (d * blocks(f, 64) + f * blocks(d, 128)) / (d + f) < 1.35 * 256:
        return 64
    fills = tiles(128) * blocks(f, 128) >= 192 and tiles(256) * blocks(d, 256) >= (96 if load > 112 * g else 192)
    return 256 if fills else 128


@pytest.mark.parametrize("want,batch,E,K,ns,d,f", [
    (128, 129, 12, 12, 0, 928, 928),     # every expert one token more than the tile; 29 k-blocks
    (128, 129, 8, 8, 1, 1216, 1312), (128, 340, 40, 6, 1, 416, 544), (128, 700, 9, 2, 0, 928, 1248),
    (256, 257, 16, 16, 0, 800, 544),     # every expert one token more than the tile; 25 and 17 k-blocks
    (256, 700, 32, 8, 1, 544, 288)])
def test_larger_tiles(torch, B, want, batch, E, K, ns, d, f):  # noqa: F811
    assert tile(batch, K, ns, E, d, f) == want
    grouped.test_grouped_gemm(torch, B, batch, E, K, ns, d, f)
