// Expert SwiGLU FFN (paper section 2, Eq. 3) on INT4 group-quantised experts
// (section 3.2) as a grouped GEMM, for calls in which an expert sees many
// tokens: batched decode and prompt processing.
//
// One workgroup = 1, 2 or 4 groups of 4 waves x a tile of up to TOK of one expert's tokens.  Tokens
// are the A operand of v_mfma_f32_16x16x32_bf16, staged through LDS in fragment
// order, four k-blocks (128 columns) per step of the gate/up pass and two per step of the down pass, double buffered; weights are the
// B operand, unpacked from 4-bit codes in registers (see ffn_fused_q4.hip for
// the 128 + q mantissa trick and the -136 correction fed through the C input).
// A lane holds one weight row for four tokens, so the per-group scale is one
// multiplier per k-block.
//   gate/up pass: wave w owns row tile 4 bx + w; one 16-byte load per lane
//     brings the codes of four k-blocks of W_g, another those of W_u, a third
//     the eight scales.  h = silu(g) * u is written as bf16, rows in group order.
//   down pass: wave w owns the block of 64 rows 4 bx + w of W_d; per k-block one
//     16-byte load per lane brings the codes of its four row tiles.
//   The groups share the rows and split the contraction, a step each in turn; their sums meet in LDS.
// Codes and tokens are requested R - 1 steps ahead of their use into a ring of fixed register slots.
// Every weight byte is read by exactly one wave of a token tile, so a group whose expert is not
// resident can stream it from the pinned host pool (prompt streaming).
#include <type_traits>

#include "device_utils.hpp"
#include "moe_internal.hpp"
#include "q4_layout.hpp"

namespace moe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWaves = 4;

template <typename V>
__device__ __forceinline__ V ldnt(const void* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const V*>(p));
}

__device__ __forceinline__ bf16x8 codes_to_bf16(uint32_t w) {
  u32x4 r;
  r[0] = (w & 0x000F000Fu) | 0x43004300u;
  r[1] = ((w >> 4) & 0x000F000Fu) | 0x43004300u;
  r[2] = ((w >> 8) & 0x000F000Fu) | 0x43004300u;
  r[3] = ((w >> 12) & 0x000F000Fu) | 0x43004300u;
  return __builtin_bit_cast(bf16x8, r);
}

template <typename V>
__device__ __forceinline__ float scale_at(V v, int e) {
  const uint32_t dw = v[e >> 1];
  return __uint_as_float((e & 1) ? (dw & 0xFFFF0000u) : (dw << 16));
}

__device__ __forceinline__ const char* group_weights(const FfnArgs& a, int id) {
  return id < a.P ? a.buffers + (size_t)id * a.expert_bytes
                  : a.shared + (size_t)(id - a.P) * a.expert_bytes;
}

// TOK: tokens per workgroup.  R: steps in flight.  MINW: waves per SIMD the registers have to leave room for.
// STREAM: experts may have to be read over the link: nothing is requested beyond the contraction (a branch around the
// loads; without it the last requests of a wave repeat its last step).
// KG: groups of kWaves waves that share the rows and split the contraction; group 0 adds up their sums.
template <int NMAT, int TOK, int R, int MINW, bool STREAM, int KG>
__global__ void __launch_bounds__(64 * kWaves * KG, MINW) ffn_gemm_q4_kernel(FfnArgs a) {
  constexpr int CB = TOK / 16;        // column blocks of 16 tokens
  constexpr int kSkb = NMAT == 2 ? 4 : 2;                   // k-blocks per step of a group
  constexpr int NA = NMAT == 2 ? 2 : 4;                     // accumulators per column block
  constexpr int PIECES = TOK * kSkb * 4 / (64 * kWaves);    // 16-byte pieces of the token tile each thread stages per step
  // [buffer][k-block of the step][column block][lane] x 16 bytes; after the loop the sums of the groups behind the first
  constexpr int kStage = 2 * kSkb * KG * CB, kSums = (KG - 1) * kWaves * CB * NA;
  __shared__ u32x4 lds[(kStage > kSums ? kStage : kSums)][64];
  auto& xs = reinterpret_cast<u32x4(&)[2][kSkb * KG][CB][64]>(lds);
  const int d = a.d, f = a.f;
  const int n_units = NMAT == 2 ? (f >> 4) : (d >> 6);         // row tiles of 16 / row blocks of 64
  const int n_rb = (n_units + kWaves - 1) / kWaves;
  const int item_id = blockIdx.x / n_rb, rb = blockIdx.x % n_rb;
  const int n_items = a.t.work[0].x;
  const int4 item = a.t.work[1 + min(item_id, a.work.cap - 1)];
  if (item_id >= n_items) return;
  const int tok0 = item.x, begin = item.z, cnt = item.w & 0x3fffffff, miss = (item.w >> 30) & 1;
  if (a.pass != 2 && miss != a.pass) return;
  const int n_tok = min(TOK, cnt - tok0);
  const int n_cb = (n_tok + 15) >> 4;

  const int lane = threadIdx.x & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = KG > 1 ? wave_id % kWaves : wave_id, group = KG > 1 ? wave_id / kWaves : 0;
  const int n = lane & 15, q = lane >> 4;
  const int nkb = (NMAT == 2 ? d : f) >> 5;                    // k-blocks of the contraction
  const int n_steps = (nkb + kSkb * KG - 1) / (kSkb * KG);
  const int unit = rb * kWaves + wave;                         // this wave's row tile / row block
  const bool has_rows = unit < n_units;
  const int uc = has_rows ? unit : n_units - 1;                // clamped: loads stay in bounds, results are dropped

  const char* wsrc = (a.fetch != 0 && miss != 0) ? a.pool + (size_t)item.y * a.expert_bytes : group_weights(a, item.y);
  // gate/up: records [row tile][super-block of 4 k-blocks]; down: records [k-block][row block]
  const int nsb = d >> 7, n_dq = d >> 6;
  const char* wrec = NMAT == 2 ? wsrc + (size_t)uc * nsb * q4::kGateUpRecord
                               : wsrc + q4::gate_up_bytes(d, f) + (size_t)uc * q4::kDownRecord;
  // weights of one step: gate/up = codes of W_g, W_u and 8 scales of one super-block;
  //                      down    = codes of 4 row tiles and 4 scales for each of 2 k-blocks
  constexpr int NW = 3;
  u32x4 wr[R][NW];
  auto req_w = [&](int slot, int step) {
    if (NMAT == 2) {
      const char* rec = wrec + (size_t)(KG > 1 ? min(step * KG + group, nsb - 1) : step) * q4::kGateUpRecord;
      wr[slot][0] = ldnt<u32x4>(rec + lane * 16);
      wr[slot][1] = ldnt<u32x4>(rec + 1024 + lane * 16);
      wr[slot][2] = ldnt<u32x4>(rec + 2048 + n * 16);
    } else {
#pragma unroll
      for (int j = 0; j < kSkb; ++j) {
        const int kb = min((step * KG + group) * kSkb + j, nkb - 1);          // clamped; the surplus k-blocks are skipped below
        const char* rec = wrec + (size_t)kb * n_dq * q4::kDownRecord;
        wr[slot][j] = ldnt<u32x4>(rec + lane * 16);
        const u32x2 s2 = ldnt<u32x2>(rec + 1024 + n * 8);
        wr[slot][2][j * 2] = s2[0];
        wr[slot][2][j * 2 + 1] = s2[1];
      }
    }
  };
#pragma unroll
  for (int u = 0; u < R - 1; ++u) req_w(u, min(u, n_steps - 1));

  // ---- token staging: 256 threads x PIECES pieces of 16 bytes = TOK rows x kSkb k-blocks of 64 bytes; rows beyond the
  //      tile repeat its last token, their results are dropped at the end ----
  const uint16_t* src[PIECES];
  int dst[PIECES];
  constexpr int SEGS = 4 * kSkb * KG;                                 // 16-byte segments of a row's step
  const int sg = threadIdx.x % SEGS, kbl = sg >> 2, qq = sg & 3;
  // the lanes that write together hold the (k-block, slice) pieces of one or two rows: the XOR spreads them over the
  // banks, and keeps the rows of neighbouring slices of a k-block apart for the reader
  const auto swz = [](int kb, int slice) { return (slice + 4 * (kb % kSkb)) * (kSkb == 4 ? 1 : 2); };
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int r = threadIdx.x / SEGS + 64 * kWaves * KG / SEGS * i;   // token row of the tile
    dst[i] = (kbl * CB + (r >> 4)) * 64 + qq * 16 + ((r & 15) ^ swz(kbl, qq));
    const int pos = begin + tok0 + min(r, n_tok - 1);
    src[i] = NMAT == 2 ? reinterpret_cast<const uint16_t*>(a.x) + (size_t)(a.t.sorted_pair[pos] / a.KS) * d + qq * 8
                       : reinterpret_cast<const uint16_t*>(a.h) + (size_t)pos * f + qq * 8;
  }
  u32x4 xq[R][PIECES];
  auto req_x = [&](int slot, int step) {
    const int kb = min(step * kSkb * KG + kbl, nkb - 1);
#pragma unroll
    for (int i = 0; i < PIECES; ++i) xq[slot][i] = *reinterpret_cast<const u32x4*>(src[i] + (size_t)kb * 32);
  };
  auto put_x = [&](int b, int slot) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) (&xs[b][0][0][0])[dst[i]] = xq[slot][i];
  };

  const bf16x8 minus136 = __builtin_bit_cast(bf16x8, u32x4{0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u});
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  // gate/up: acc[cb][0] gate, acc[cb][1] up; down: acc[cb][j] row tile j of the block
  f32x4 acc[CB][NA];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int m = 0; m < NA; ++m) acc[cb][m] = zero;

#pragma unroll
  for (int u = 0; u < R - 1; ++u) req_x(u, min(u, n_steps - 1));
  put_x(0, 0);
  __syncthreads();
  // the column blocks in use, rounded up to a quarter or half of the tile, as a compile-time count
  auto run = [&](auto ncb_tag) {
    constexpr int NCB = decltype(ncb_tag)::value;
    auto multiply = [&](int u, int b, int n_kb) {
      u32x4 fr[2][NCB];               // token fragments of a k-block, those of the next one on their way
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) fr[0][cb] = xs[b][group * kSkb][cb][lane ^ swz(0, q)];
#pragma unroll
      for (int j = 0; j < kSkb; ++j) {
        if (j + 1 < kSkb) {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) fr[(j + 1) & 1][cb] = xs[b][group * kSkb + j + 1][cb][lane ^ swz(j + 1, q)];
        }
        __builtin_amdgcn_sched_barrier(0);
        if (j < n_kb) {      // uniform
          bf16x8 wb[NA];
          float sc[NA];
#pragma unroll
          for (int m = 0; m < NA; ++m) {
            wb[m] = codes_to_bf16(NMAT == 2 ? wr[u][m][j] : wr[u][j][m]);
            sc[m] = scale_at(wr[u][2], NMAT == 2 ? 4 * m + j : 4 * j + m);
          }
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            const bf16x8 xa = __builtin_bit_cast(bf16x8, fr[j & 1][cb]);
            const f32x4 off = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, minus136, zero, 0, 0, 0);
#pragma unroll
            for (int m = 0; m < NA; ++m)
              acc[cb][m] += sc[m] * __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa, wb[m], off, 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // (as in ffn_gemm.hip: no branch around a load, tokens requested ahead of the weights of the same step)
#pragma unroll 1
    for (int s0 = 0; s0 < n_steps; s0 += R) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        const int ahead = s0 + u + R - 1;
        if (!STREAM || ahead < n_steps) {
          req_x((u + R - 1) % R, min(ahead, n_steps - 1));
          req_w((u + R - 1) % R, min(ahead, n_steps - 1));
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s0 + u < n_steps) multiply(u, (s0 + u) & 1, nkb - ((s0 + u) * KG + group) * kSkb);
        put_x((s0 + u + 1) & 1, (u + 1) % R);
        __syncthreads();
      }
    }
  };
  if (CB >= 4 && n_cb <= CB / 4) run(std::integral_constant<int, CB / 4 ? CB / 4 : 1>{});
  else if (n_cb <= CB / 2) run(std::integral_constant<int, CB / 2>{});
  else run(std::integral_constant<int, CB>{});

  // ---- epilogue: lane holds weight row n of its tile(s) for tokens 16 cb + 4 q + i ----
  if constexpr (KG > 1) {        // (the loop ended with a barrier)
    auto& sums = reinterpret_cast<f32x4(&)[KG - 1][kWaves][CB][NA][64]>(lds);
    if (group > 0) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        if (cb < n_cb)
#pragma unroll
          for (int m = 0; m < NA; ++m) sums[group - 1][wave][cb][m][lane] = acc[cb][m];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int g = 0; g < KG - 1; ++g)
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        if (cb < n_cb)
#pragma unroll
          for (int m = 0; m < NA; ++m) acc[cb][m] += sums[g][wave][cb][m][lane];
  }
  if (!has_rows) return;
#pragma unroll
  for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tk = cb * 16 + q * 4 + i;
      if (tk < n_tok) {
        const size_t pos = (size_t)(begin + tok0 + tk);
        if (NMAT == 2) {
          reinterpret_cast<uint16_t*>(a.h)[pos * f + unit * 16 + n] =
              f32_to_bf16(silu(acc[cb][0][i]) * acc[cb][NA - 1][i]);
        } else {
          // rows 64 unit + 4 n + m, m = 0..3: one 16-byte store
          *reinterpret_cast<f32x4*>(a.o + pos * d + (size_t)unit * 64 + n * 4) =
              f32x4{acc[cb][0][i], acc[cb][1][i], acc[cb][NA > 2 ? 2 : 0][i], acc[cb][NA > 3 ? 3 : 0][i]};
        }
      }
    }
  }
}

// A wave takes ~0.5 us per step, however far ahead it asks (three and five steps ahead: -2 .. 0 %), for the chain of LDS, products, scaling and
// barrier; where the workgroups leave a SIMD fewer than four waves, groups of waves that split the contraction fill it (us per
// call, one / two / four groups; workgroups of each pass in brackets; at most two pairs of 40 tokens):
//   tiles of 32: 8 experts of 4096 x 14336 (2016 + 144) 239 / 205 / 189, 16 of 4096 x 1024 (288 + 288) 49 / 42.5 / 41, 24 of 2048 x 768 (348
//     + 232) 37.4 / 35.9 / 37.5, 32 of 2048 x 512 (456 + 456; 200 tokens) 46.5 / 45.4 / 57, 64 of 2048 x 1024 (1280 + 640; 64 tokens)
//     59 / 60.5 / 62.
//   Four need four steps each: 16 of 1024 x 512 (144 + 72) 27.6 / 26.1 / 27; and, as they fill a unit, a unit for every workgroup that finds a tile:
//     40 of 2560 x 448, 62 tokens (280 + 400) 39.9 / 38.2 / 45.1.  Two need two each, and beyond 320 workgroups four: 64 of 768 x 288, 63 tokens (395
//     with 6 steps, 237 with 4.5) 27.9 / 28.9, 60 of 1280 x 288, 241 tokens (450 with 10, 450 with 4.5) 35.9 / 37.9, tiles of 64, 8 of 256 x 128, 385 tokens
//     (2 steps) 23.1 / 24.6.
//   tiles of 64: 8 of 4096 x 14336, 400 tokens (4480 + 320) 571 / 534, 8 of 2048 x 1024, 300 (272 + 136) 58.3 / 52, 600 (416 + 208) 66.8 / 68.3.
constexpr int kUnits = 256, kSplit4 = 320, kSplitSteps = 4, kSplitFew = 2, kSplit2 = 512, kSplitLarge = 352;
constexpr int kSmallTile = 5, kLargeTile = 6, kStreamedTile = 7;     // log2 of the tokens per tile
bool small_tile(int64_t load, int groups) { return load <= (int64_t)56 * groups; }

}  // namespace

Q4Split split_ffn_gemm_q4(int batch, int KS, int n_shared, int groups, int d, int f) {
  const int64_t load = (int64_t)batch * KS, routed = groups - n_shared, tile = 1 << kSmallTile;
  const bool small = small_tile(load, groups);
  const int64_t items = groups + (load >> (small ? kSmallTile : kLargeTile));     // upper bound
  // (even loads)
  const int64_t tiles = routed * ((load - (int64_t)batch * n_shared + routed * tile - 1) / (routed * tile)) + n_shared * ((batch + tile - 1) / tile);
  const auto pass = [&](int units, int kblocks, int step) {
    const int64_t blocks = (units + kWaves - 1) / kWaves, wgs = items * blocks;
    if (small && wgs <= kSplit4 && tiles * blocks <= kUnits && kblocks >= 4 * kSplitSteps * step) return 4;
    return wgs <= (small ? kSplit2 : kSplitLarge) && kblocks >= 2 * (wgs <= kSplit4 ? kSplitFew : kSplitSteps) * step ? 2 : 1;
  };
  return {pass(f / 16, d / 32, 4), pass(d / 64, f / 32, 2)};
}

// What bounds it: the vector arithmetic of unpacking and scaling and the exchange through LDS as much as the codes, so
// occupancy beats depth: one step ahead at four waves per SIMD takes 61.6 us per layer call of 64 OLMoE-like tokens, two
// steps ahead at three waves 68.3, three at two 67.1; the former loop on 64-token tiles 83 (gate/up 43.5 us for 151 MB, down
// 27 us for 75 MB).  Tiles of 32 tokens win up to a mean of ~64 pairs per expert: 57 / 61.6 / 74 / 95.5 / 145 / 237 us at 17 /
// 64 / 128 / 256 / 512 / 1024 tokens against 65 / 70 / 79 / 104 / 142 / 229 with tiles of 64.  Experts streamed from the host
// cross the link once per tile: 128 tokens.
// (Four groups exist for tiles of 32 only: they go with them where the buffers of a constrained cache, fewer than the experts, would ask for 64.)
WorkPlan plan_ffn_gemm_q4(int batch, int KS, int g_max, bool streamed, const Q4Split& split) {
  const int64_t load = (int64_t)batch * KS;
  const bool four = split.gate_up == 4 || split.down == 4;
  WorkPlan w{};
  w.shift = streamed ? kStreamedTile : four || small_tile(load, g_max) ? kSmallTile : kLargeTile;
  w.cap = (int)work_capacity(g_max, load);
  return w;
}

hipError_t launch_ffn_gemm_q4(hipStream_t s, const FfnArgs& a, const Q4Split& split, KernelEvents e1, KernelEvents e2) {
  if (a.g_max <= 0) return hipSuccess;
  const int items = a.g_max + (int)(((int64_t)a.max_count * a.KS) >> a.work.shift);     // upper bound
  const auto run = [&](auto kernel, int units, int groups, KernelEvents e) {
    launch_timed(kernel, dim3(items * ((units + kWaves - 1) / kWaves)), dim3(64 * kWaves * groups), 0, s, e, a);
  };
  const int s1 = split.gate_up, s2 = split.down;
  if (a.work.shift == kStreamedTile) {
    run(ffn_gemm_q4_kernel<2, 128, 2, 1, true, 1>, a.f / 16, 1, e1);
    run(ffn_gemm_q4_kernel<1, 128, 2, 1, true, 1>, a.d / 64, 1, e2);
  } else if (a.work.shift == kSmallTile) {
    if (s1 == 4) run(ffn_gemm_q4_kernel<2, 32, 2, 4, false, 4>, a.f / 16, 4, e1);
    else if (s1 == 2) run(ffn_gemm_q4_kernel<2, 32, 2, 4, false, 2>, a.f / 16, 2, e1);
    else run(ffn_gemm_q4_kernel<2, 32, 2, 4, false, 1>, a.f / 16, 1, e1);
    if (s2 == 4) run(ffn_gemm_q4_kernel<1, 32, 2, 4, false, 4>, a.d / 64, 4, e2);
    else if (s2 == 2) run(ffn_gemm_q4_kernel<1, 32, 2, 4, false, 2>, a.d / 64, 2, e2);
    else run(ffn_gemm_q4_kernel<1, 32, 2, 4, false, 1>, a.d / 64, 1, e2);
  } else {
    if (s1 == 2) run(ffn_gemm_q4_kernel<2, 64, 2, 2, false, 2>, a.f / 16, 2, e1);
    else run(ffn_gemm_q4_kernel<2, 64, 2, 3, false, 1>, a.f / 16, 1, e1);
    if (s2 == 2) run(ffn_gemm_q4_kernel<1, 64, 2, 2, false, 2>, a.d / 64, 2, e2);
    else run(ffn_gemm_q4_kernel<1, 64, 2, 2, false, 1>, a.d / 64, 1, e2);
  }
  return hipGetLastError();
}

}  // namespace moe
