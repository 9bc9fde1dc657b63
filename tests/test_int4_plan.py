"""CPU: which kernels an INT4 layer in memory takes, on either side of the lines between them (the slower side was measured at every row)."""
import pytest

from paper_2602_11192_amd import binding as B


@pytest.mark.parametrize("d,f,E,K,ns,batch,plan", [
    (4096, 14336, 8, 2, 0, 20, 14), (1024, 512, 16, 2, 0, 20, 22),            # four groups need four steps each
    (256, 128, 8, 2, 0, 385, 11), (256, 64, 60, 2, 0, 79, 11),                # two need two
    (768, 288, 64, 8, 0, 63, 12), (512, 288, 48, 2, 0, 99, 22),               # ... and beyond 320 workgroups four
    (2560, 448, 40, 2, 0, 62, 21), (4096, 1024, 16, 2, 0, 20, 44),            # four: 280 and 256 workgroups with a tile
    (2560, 224, 60, 2, 2, 111, 21), (2560, 224, 58, 2, 2, 32, 41),            # a shared expert of 111 tokens has four tiles
])
def test_groups_that_split_the_contraction(d, f, E, K, ns, batch, plan):
    assert B.lib.moe_test_int4_plan(d, f, E, K, ns, batch) == plan


@pytest.mark.parametrize("d,f,E,K,ns,batch,gemm", [
    (4096, 14336, 8, 2, 0, 8, True), (4096, 14336, 8, 2, 0, 7, False),        # workgroups of the down pass x tokens
    (3072, 1024, 12, 2, 0, 10, True), (3072, 1536, 8, 1, 0, 12, False), (2560, 544, 60, 6, 0, 7, False),      # 106, 96 and 99 MB
    (3072, 2016, 16, 1, 0, 10, False), (4096, 3104, 8, 1, 0, 10, True),       # one expert a token: 105 and 215 MB
    (768, 1696, 64, 8, 2, 15, True), (1024, 4736, 64, 4, 0, 13, False), (1024, 7136, 64, 8, 0, 8, True),      # many experts of few columns
])
def test_few_tokens(d, f, E, K, ns, batch, gemm):
    assert (B.lib.moe_test_int4_plan(d, f, E, K, ns, batch) > 0) == gemm
