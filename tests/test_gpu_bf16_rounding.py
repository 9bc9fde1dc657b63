"""How results become bf16: random bit patterns, halfway cases, denormals, the largest numbers, infinities and NaN leave a layer as the rounding
to nearest even of the integer form gives them.  The experts are made so that an output is one chosen fp32 number: W_d holds it
in pieces of eight bits, which h of 1 or 2^-16 adds up without rounding.  32 and 36 columns of d_ff: a workgroup per token, and the kernels per
expert with their combine."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def rounded(bits):
    up = ((bits.astype(np.uint64) + 0x7fff + ((bits >> 16) & 1)) >> 16).astype(np.uint16)
    nan = (bits & 0x7fffffff) > 0x7f800000
    return np.where(nan, ((bits >> 16) | 0x40).astype(np.uint16), up), nan


def pieces(bits):
    """three bf16 bit patterns that add up to each number (times 2^16 where it is small) and whether it is"""
    with np.errstate(invalid="ignore"):
        v = bits.view(np.float32).astype(np.float64)
    small = np.abs(v) < 2.0 ** -100
    rest, out = np.where(small, v * 2.0 ** 16, v), []
    for _ in range(3):
        top = rest.astype(np.float32).view(np.uint32) & 0xffff0000
        out.append((top >> 16).astype(np.uint16))
        with np.errstate(invalid="ignore"):
            rest = np.where(np.isfinite(rest), rest - top.view(np.float32), 0.0)
    assert not rest.any()
    nan = np.isnan(v)
    out[0] = np.where(nan, (bits >> 16) | 0x40, out[0]).astype(np.uint16)
    return out, small


@pytest.mark.parametrize("f", [32, 36])
def test_results_round_to_nearest_even(f):
    import torch
    from paper_2602_11192_amd import binding as B
    E, d = 64, 256
    rng = np.random.default_rng(1)
    bits = rng.integers(0, 1 << 32, E * d, dtype=np.uint64).astype(np.uint32)
    half = bits[: 4 * d] & 0xffff0000                     # halfway and its neighbours; every kind of exponent
    bits[: 4 * d] = half | np.tile(np.array([0x7fff, 0x8000, 0x8001, 0], dtype=np.uint32), d)
    bits[4 * d: 6 * d] &= 0x807fffff                      # denormal
    bits[6 * d: 6 * d + 8] = [0x7f7fffff, 0x7f7f8000, 0x7f7f7fff, 0xff7fffff, 0x7f800000, 0xff800000, 0x7fc00001, 0x7f800001]
    bits = np.where(bits & 0x7fffffff == 0, 1, bits).astype(np.uint32)       # (a sum of zeros has no sign to keep)
    parts, small = pieces(bits)
    bf = lambda v: np.array(v, dtype=np.float32).view(np.uint32) >> 16
    blocks = np.zeros((E, 3 * d * f), dtype=np.uint16)
    wg, wu, wd = blocks[:, : f * d].reshape(E, f, d), blocks[:, f * d: 2 * f * d].reshape(E, f, d), blocks[:, 2 * f * d:].reshape(E, d, f)
    wg[:, :6, 0] = bf(64.0)                               # silu(64) = 64
    wu[:, :3, 0], wu[:, 3:6, 0] = bf(2.0 ** -6), bf(2.0 ** -22)
    for i, p in enumerate(parts):
        p, s = p.reshape(E, d), small.reshape(E, d)
        wd[:, :, i], wd[:, :, 3 + i] = np.where(s, 0, p), np.where(s, p, 0)
    dev = lambda a: torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).cuda()
    x = torch.zeros(E, d, dtype=torch.bfloat16, device="cuda:0")
    x[:, 0] = 1
    y, w = torch.full_like(x, 7.0), torch.empty(E, 1, device="cuda:0")
    B.moe_layer_decode_resident_noalloc(n_experts=E, top_k=1, d_model=d, d_ff=f, dtype=B.MOE_DTYPE_BF16, norm_topk=1,
                                        pool_layout=B.MOE_LAYOUT_ROWMAJOR, router_w=torch.zeros_like(x), experts=dev(blocks.reshape(-1)), x=x, y=y,
                                        logit_bias=(8 * torch.eye(E)).cuda(), topk_idx=None, topk_w=w)       # token e: expert e
    torch.cuda.synchronize()
    assert bool((w == 1).all())
    got, (want, nan) = y.cpu().view(torch.int16).numpy().view(np.uint16).reshape(-1), rounded(bits)
    assert (got == want)[~nan].all()
    assert ((got[nan] & 0x7fff) > 0x7f80).all()
