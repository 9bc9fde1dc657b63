// Expert SwiGLU FFN (paper section 2, Eq. 3) as a grouped bf16 GEMM for calls
// in which an expert sees several tokens (batched decode, prompt processing).
//
// One workgroup = a block of output rows of one expert (WAVES waves x RT row tiles of 16) x a tile of up to TOK of that
// expert's tokens.
//   * weights: A operand of v_mfma_f32_16x16x32_bf16, read by each wave straight
//     from global memory in the tiled layout (one coalesced KiB per fragment,
//     nontemporal: each fragment is used by exactly one wave of one token tile),
//     R - 1 k-blocks ahead of their use in a ring of fixed register slots;
//   * tokens: B operand, shared by the waves, requested as early and staged through LDS in
//     fragment order, double buffered, one k-block per step.
// Column blocks beyond the tile's token count are skipped, so a large batch
// spread thinly over many experts degrades into weight streaming rather than
// wasted matrix work.  NMAT = 2 computes h = silu(X W_g^T) * (X W_u^T) (bf16,
// rows in group order); NMAT = 1 computes o = h W_d^T (fp32).
//
// What bounds it: HBM while an expert sees few tokens (64 DeepSeekMoE-like tokens, 66 experts: gate/up 122 us for 761 MB
// and down 64 us for 381 MB, i.e. 6.2 and 6.0 TB/s, against 153 and 84 us with a loop that drained its loads at the end of
// every step).  With hundreds of tokens per expert neither HBM (1024 OLMoE-like tokens: 618 MB in 153 us) nor the matrix
// cores: with the weights served from cache the gate/up loop takes 2/3 of the time, with an eighth of the matrix work
// nearly all of it.  What the code leaves there: one workgroup of the large tile per compute unit at a time, so that its ~530
// workgroups make 2.07 rounds, and every tile requests and stages all of its 256 token rows however few it has.
#include <algorithm>
#include <type_traits>

#include "device_utils.hpp"
#include "moe_internal.hpp"

namespace moe {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ const char* group_weights(const FfnArgs& a, int id) {
  return id < a.P ? a.buffers + (size_t)id * a.expert_bytes
                  : a.shared + (size_t)(id - a.P) * a.expert_bytes;
}

// Where a token's row sits inside its 16-row block of the staged tile, for the 8-wide slice q of the k-block.  Sixteen
// lanes write four rows x four slices: the four multiples of 4 put them on different banks.  Reading, the LDS serves
// the lanes of slices 0 and 1 (2 and 3) together, rows 0-3 and 12-15 of the one with rows 4-11 of the other: the
// multiples of such a pair differ in both bits, which keeps these apart too (with 4 q every read took twice as long).
__device__ __forceinline__ int swz(int q) { return (-q & 3) * 4; }

// MINW: waves per SIMD the registers have to leave room for.
template <int NMAT, int RT, int TOK, int WAVES, int R, int MINW>
__global__ void __launch_bounds__(64 * WAVES, MINW) ffn_gemm_kernel(FfnArgs a) {
  constexpr int THREADS = 64 * WAVES;
  constexpr int CB = TOK / 16;                    // column blocks of 16 tokens
  constexpr int PIECES = TOK * 4 / THREADS;       // 16-byte pieces of a staged k-block per thread
  static_assert(TOK * 4 % THREADS == 0 && CB % 4 == 0, "");
  __shared__ u32x4 xs[2][CB][64];                 // [buffer][column block][lane]
  const int n_rb = ((NMAT == 2 ? a.f : a.d) / 16 + RT * WAVES - 1) / (RT * WAVES);
  // Consecutive workgroups go to the eight dies in turn.  by_die: all row blocks of a token tile on one die, whose L2
  // then holds the tile's tokens.
  int item_id = blockIdx.x / n_rb, rb = blockIdx.x % n_rb;
  if (a.by_die) {
    const int j = blockIdx.x >> 3;
    item_id = j / n_rb * 8 + (blockIdx.x & 7);
    rb = j % n_rb;
  }
  // (both loads are issued before the first branch; the index stays inside the list)
  const int n_items = a.t.work[0].x;
  const int4 item = a.t.work[1 + min(item_id, a.work.cap - 1)];
  if (item_id >= n_items) return;
  const int tok0 = item.x, begin = item.z, cnt = item.w & 0x3fffffff, miss = (item.w >> 30) & 1;
  if (a.pass != 2 && miss != a.pass) return;
  const int n_tok = min(TOK, cnt - tok0);         // tokens of this tile
  const int n_cb = (n_tok + 15) >> 4;             // column blocks in use

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nkb = (NMAT == 2 ? a.d : a.f) >> 5;
  const int n_rt = (NMAT == 2 ? a.f : a.d) >> 4;
  const int rt0 = (rb * WAVES + wave) * RT;       // this wave's row tiles

  // a group whose expert is not resident streams it from the pinned host pool (prompt streaming)
  const char* wsrc = (a.fetch != 0 && miss != 0) ? a.pool + (size_t)item.y * a.expert_bytes : group_weights(a, item.y);
  const char* wp[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int rt = min(rt0 + i, n_rt - 1);        // clamped: loads stay in bounds, results are dropped
    wp[i] = NMAT == 2 ? wsrc + (size_t)rt * nkb * 2048 : wsrc + (size_t)4 * a.f * a.d + (size_t)rt * 1024;
  }
  const size_t kb_bytes = NMAT == 2 ? 2048 : (size_t)(a.d >> 4) * 1024;
  u32x4 wr[R][RT][NMAT];
  auto req_w = [&](int slot, int kb) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int m = 0; m < NMAT; ++m)
        wr[slot][i][m] = __builtin_nontemporal_load(
            reinterpret_cast<const u32x4*>(wp[i] + (size_t)kb * kb_bytes + (uint32_t)(lane * 16 + m * 1024)));
  };
  // (requested before the token addresses are looked up)
#pragma unroll
  for (int u = 0; u < R - 1; ++u) req_w(u, min(u, nkb - 1));

  // ---- token staging: a k-block of TOK rows in pieces of 16 bytes; rows beyond the tile repeat its last token, their
  //      columns are dropped at the end ----
  const uint16_t* src[PIECES];
  int dst[PIECES];
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int idx = threadIdx.x + THREADS * i;
    const int r = idx >> 2, q = idx & 3;
    dst[i] = (r >> 4) * 64 + q * 16 + ((r & 15) ^ swz(q));
    const int pos = begin + tok0 + min(r, n_tok - 1);
    src[i] = NMAT == 2 ? reinterpret_cast<const uint16_t*>(a.x) + (size_t)(a.t.sorted_pair[pos] / a.KS) * a.d + q * 8
                       : reinterpret_cast<const uint16_t*>(a.h) + (size_t)pos * a.f + q * 8;
  }
  u32x4 xq[R][PIECES];
  auto req_x = [&](int slot, int kb) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) xq[slot][i] = *reinterpret_cast<const u32x4*>(src[i] + (size_t)kb * 32);
  };
  auto put_x = [&](int b, int slot) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) (&xs[b][0][0])[dst[i]] = xq[slot][i];
  };

  f32x4 acc[CB][RT][NMAT];
#pragma unroll
  for (int cb = 0; cb < CB; ++cb)
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int m = 0; m < NMAT; ++m) acc[cb][i][m] = f32x4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int u = 0; u < R - 1; ++u) req_x(u, min(u, nkb - 1));
  put_x(0, 0);
  __syncthreads();
  const int xlane = lane ^ swz(lane >> 4);
  // the column blocks in use, rounded up to a quarter of the tile, as a compile-time count: no branch in the loop
  auto run = [&](auto ncb_tag) {
    constexpr int NCB = decltype(ncb_tag)::value;
    // the token fragments come from LDS G at a time, two groups in flight (left to itself the compiler waits for
    // every second one: the loop alone took 118 instead of 102 us at 1024 OLMoE-like tokens)
    constexpr int G = TOK > 64 ? 2 : NCB;
    static_assert(NCB % G == 0, "");
    auto multiply = [&](int u, int b) {
      u32x4 fr[2][G];
#pragma unroll
      for (int c = 0; c < (NCB > G ? 2 : 1); ++c)
#pragma unroll
        for (int k = 0; k < G; ++k) fr[c][k] = xs[b][c * G + k][xlane];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < NCB / G; ++c) {
#pragma unroll
        for (int k = 0; k < G; ++k)
#pragma unroll
          for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int m = 0; m < NMAT; ++m)
              acc[c * G + k][i][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, wr[u][i][m]), __builtin_bit_cast(bf16x8, fr[c & 1][k]), acc[c * G + k][i][m], 0, 0, 0);
        if (c + 2 < NCB / G) {
#pragma unroll
          for (int k = 0; k < G; ++k) fr[c & 1][k] = xs[b][(c + 2) * G + k][xlane];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // Between request and use there is no branch around a load and the tokens of a step are requested ahead of its
    // weights, so the compiler waits for exactly what the step needs: weights needed R - 1 steps later stay in flight.
    int s0 = 0;
#pragma unroll 1
    for (; s0 + 2 * R - 1 <= nkb; s0 += R) {
#pragma unroll
      for (int u = 0; u < R; ++u) {
        req_x((u + R - 1) % R, s0 + u + R - 1);
        req_w((u + R - 1) % R, s0 + u + R - 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(u, (s0 + u) & 1);
        put_x((s0 + u + 1) & 1, (u + 1) % R);       // k-block s0 + u + 1, requested R - 2 steps ago
        __syncthreads();
      }
    }
    // the last R - 1 to 2 R - 2 k-blocks: nothing is requested beyond the contraction (a streamed expert would read it
    // over the link)
#pragma unroll
    for (int u = 0; u < 2 * R - 2; ++u) {
      if (s0 + u < nkb) {
        if (s0 + u + R - 1 < nkb) {
          req_x((u + R - 1) % R, s0 + u + R - 1);
          req_w((u + R - 1) % R, s0 + u + R - 1);
        }
        multiply(u % R, (s0 + u) & 1);
        if (s0 + u + 1 < nkb) put_x((s0 + u + 1) & 1, (u + 1) % R);
        __syncthreads();
      }
    }
  };
  constexpr int Q = CB / 4;
  if (n_cb <= Q) run(std::integral_constant<int, Q>{});
  else if (n_cb <= 2 * Q) run(std::integral_constant<int, 2 * Q>{});
  else if (n_cb <= 3 * Q) run(std::integral_constant<int, 3 * Q>{});
  else run(std::integral_constant<int, CB>{});

  // ---- epilogue: lane holds rows (lane/16)*4 .. +3 of a row tile for token column lane%16 ----
  const int n = lane & 15, r4 = (lane >> 4) * 4;
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int rt = rt0 + i;
    if (rt >= n_rt) break;
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
      const int tk = cb * 16 + n;
      if (tk < n_tok) {
        const size_t pos = (size_t)(begin + tok0 + tk);
        if (NMAT == 2) {
          uint16_t hv[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) hv[k] = f32_to_bf16(silu(acc[cb][i][0][k]) * acc[cb][i][NMAT - 1][k]);
          uint2 pk;
          pk.x = (uint32_t)hv[0] | ((uint32_t)hv[1] << 16);
          pk.y = (uint32_t)hv[2] | ((uint32_t)hv[3] << 16);
          *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.h) + pos * a.f + rt * 16 + r4) = pk;
        } else {
          *reinterpret_cast<f32x4*>(a.o + pos * a.d + rt * 16 + r4) = acc[cb][i][0];
        }
      }
    }
  }
}

// Calls of up to 16 tokens: a group has one column block, so nothing is staged and nobody waits for anyone.  Every wave streams
// its own RT row tiles and takes the token fragment of a k-block straight from memory (a few rows that stay in the first cache
// level), all of it R - 1 k-blocks ahead.  The contraction is walked from its start, as in ffn_gemm_kernel: a token's bits do
// not depend on how many share the call.
// The row tiles of a workgroup lie a multiple of d x 64 bytes apart, so waves in lockstep meet in the same memory channels:
// each sends its first requests kFewSkew x 64 clocks after its neighbour (the queues of the memory are full by then, nothing idles).
// What bounds it: HBM, and with one round of workgroups the units that hold one more than the others.  4 Phi-3.5-MoE-like tokens (734 MB,
// 368 MB): gate/up 115.7 -> 107.9 us (6.8 TB/s), down 57.3 -> 55.6; 16 OLMoE-like gate/up 74.7 -> 72.0, down 38.3 / 38.4.  76 points of 4
// to 16 tokens 1.043x in the mean against the staged kernel, the slowest .99; without the wait 1.035x.  With more than one column
// block its L1 traffic overtakes the staging: 64 tokens on 24 experts of 2560 x 2048 135 -> 162 us.
constexpr int kFewTokens = 16;
constexpr int kFewSkew = 4;
template <int NMAT, int RT, int R, int MINW>
__global__ void __launch_bounds__(256, MINW) ffn_few_kernel(FfnArgs a) {
  constexpr int WAVES = 4;
  const int n_rb = ((NMAT == 2 ? a.f : a.d) / 16 + RT * WAVES - 1) / (RT * WAVES);
  int item_id = blockIdx.x / n_rb, rb = blockIdx.x % n_rb;
  if (a.by_die) {                                 // as in ffn_gemm_kernel
    const int j = blockIdx.x >> 3;
    item_id = j / n_rb * 8 + (blockIdx.x & 7);
    rb = j % n_rb;
  }
  const int n_items = a.t.work[0].x;
  const int4 item = a.t.work[1 + min(item_id, a.work.cap - 1)];
  if (item_id >= n_items) return;
  const int begin = item.z, n_tok = item.w & 0x3fffffff, miss = (item.w >> 30) & 1;
  if (a.pass != 2 && miss != a.pass) return;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int nkb = (NMAT == 2 ? a.d : a.f) >> 5, n_rt = (NMAT == 2 ? a.f : a.d) >> 4;
  const int rt0 = (rb * WAVES + wave) * RT;
  if (rt0 >= n_rt) return;
  const char* wsrc = group_weights(a, item.y);    // (experts streamed from the host take the large tile)
  const char* wp[RT];
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int rt = min(rt0 + i, n_rt - 1);        // clamped: loads stay in bounds, results are dropped
    wp[i] = NMAT == 2 ? wsrc + (size_t)rt * nkb * 2048 : wsrc + (size_t)4 * a.f * a.d + (size_t)rt * 1024;
  }
  const size_t kb_bytes = NMAT == 2 ? 2048 : (size_t)(a.d >> 4) * 1024;
  int next = 0;                                   // k-block of the next request
  if (NMAT == 2)
    for (int i = 0; i < wave; ++i) __builtin_amdgcn_s_sleep(kFewSkew);
  const int pos = begin + min(n, n_tok - 1);      // columns beyond the group repeat its last token and are dropped
  const uint16_t* src = NMAT == 2 ? reinterpret_cast<const uint16_t*>(a.x) + (size_t)(a.t.sorted_pair[pos] / a.KS) * a.d + q * 8
                                  : reinterpret_cast<const uint16_t*>(a.h) + (size_t)pos * a.f + q * 8;
  u32x4 wr[R][RT][NMAT], xr[R];
  auto req = [&](int slot) {
    xr[slot] = *reinterpret_cast<const u32x4*>(src + (size_t)next * 32);
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int m = 0; m < NMAT; ++m)
        wr[slot][i][m] = __builtin_nontemporal_load(
            reinterpret_cast<const u32x4*>(wp[i] + (size_t)next * kb_bytes + (uint32_t)(lane * 16 + m * 1024)));
    next = next + 1 == nkb ? 0 : next + 1;
  };
  f32x4 acc[RT][NMAT];
#pragma unroll
  for (int i = 0; i < RT; ++i)
#pragma unroll
    for (int m = 0; m < NMAT; ++m) acc[i][m] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto multiply = [&](int u) {
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int m = 0; m < NMAT; ++m)
        acc[i][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wr[u][i][m]), __builtin_bit_cast(bf16x8, xr[u]),
                                                            acc[i][m], 0, 0, 0);
  };
#pragma unroll
  for (int u = 0; u < R - 1; ++u) req(u);         // (of a contraction that is shorter some k-blocks once more, not used)
  int s0 = 0;
#pragma unroll 1
  for (; s0 + 2 * R - 1 <= nkb; s0 += R) {
#pragma unroll
    for (int u = 0; u < R; ++u) {
      req((u + R - 1) % R);
      __builtin_amdgcn_sched_barrier(0);
      multiply(u);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < 2 * R - 2; ++u) {
    if (s0 + u < nkb) {
      if (s0 + u + R - 1 < nkb) req((u + R - 1) % R);
      multiply(u % R);
    }
  }
  if (n >= n_tok) return;
  const size_t row = (size_t)(begin + n);
#pragma unroll
  for (int i = 0; i < RT; ++i) {
    const int rt = rt0 + i;
    if (rt >= n_rt) break;
    if (NMAT == 2) {
      uint16_t hv[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) hv[k] = f32_to_bf16(silu(acc[i][0][k]) * acc[i][NMAT - 1][k]);
      uint2 pk;
      pk.x = (uint32_t)hv[0] | ((uint32_t)hv[1] << 16);
      pk.y = (uint32_t)hv[2] | ((uint32_t)hv[3] << 16);
      *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.h) + row * a.f + rt * 16 + q * 4) = pk;
    } else {
      *reinterpret_cast<f32x4*>(a.o + row * a.d + rt * 16 + q * 4) = acc[i][0];
    }
  }
}

constexpr int kSmallTile = 6, kMidTile = 7, kLargeTile = 8;     // log2 of the tokens per tile
constexpr int kUnits = 256;                                     // compute units

}  // namespace

// The group sizes are not known on the host; the mean load m = pairs / groups and the workgroups it makes decide the token
// tile.  Tiles of 64 tokens on four waves stream best (three workgroups per compute unit); tiles of 256 on eight waves read a
// busy expert's weights once where the small ones read them per 64 tokens, but they leave the chip idle where they are few; tiles
// of 128 on eight waves lie between.  Up to m = 40 the small one (OLMoE-like, small / large: at m = 24 155 / 170 us per layer
// call, at 40 173 / 179; Phi-3.5-MoE-like at 32 423 / 452).  Beyond, the small one while it needs less than 1.35 workgroups per
// compute unit, the two passes weighted by their length (8 experts of 1024 x 512, small / middle / large: m = 64 39 / 46 / 53 us,
// m = 256 52 / 59 / 84; one of 2048 x 2048, m = 256: 55 / 78 / 132); then the large one where its workgroups, too, fill the units -
// three quarters of them in the gate/up pass, as many in the down pass, or half that from m = 112 on (OLMoE-like, m = 128 390 /
// 302 / 230; 24 of 2560 x 2048, m = 171, 444 / 340 / 242; at m = 64 OLMoE-like 258 / 188 / 190, and with a few experts preferred 10 %
// more with the middle than with the large one) - and the middle one where not (4 of 3072 x 3072, m = 200, 171 / 125 / 179;
// 8 of 1024 x 4096, m = 256, 179 / 143 / 187).  Of 262 points (25 shapes, m = 30 to 1024) with evenly spread experts none is slower
// than with the kernels before the ring, with preferred experts three are, by 5 %; 1.22x and 1.25x in the mean against two tiles
// split at m = 40.  Experts streamed from the host cross the link once per tile: the large one.
WorkPlan plan_ffn_gemm(int batch, int KS, int g_max, int d, int f, bool streamed) {
  const int64_t load = (int64_t)batch * KS;
  WorkPlan w{};
  w.cap = (int)work_capacity(g_max, load);
  w.shift = streamed ? kLargeTile : kSmallTile;
  if (streamed || load <= (int64_t)40 * g_max) return w;
  // tiles to expect: half a tile per group is lost to its last one
  const auto tiles = [&](int shift) { return std::max((double)g_max, (double)load / (1 << shift) + 0.5 * g_max); };
  const auto blocks = [](int rows, int per_wg) { return (rows + per_wg - 1) / per_wg; };
  // workgroups of either pass; its length goes with the contraction (gate/up: d, two matrices of half the rows)
  const double small = tiles(kSmallTile) * ((double)d * blocks(f, 64) + (double)f * blocks(d, 128)) / (d + f);
  if (small < 1.35 * kUnits) return w;
  const double gate = tiles(kMidTile) * blocks(f, 128), down = tiles(kLargeTile) * blocks(d, 256);
  const bool fills = gate >= 0.75 * kUnits && down >= (load > (int64_t)112 * g_max ? 0.375 : 0.75) * kUnits;
  w.shift = fills ? kLargeTile : kMidTile;
  return w;
}

hipError_t launch_ffn_gemm(hipStream_t s, const FfnArgs& args, KernelEvents e1, KernelEvents e2) {
  if (args.g_max <= 0) return hipSuccess;
  FfnArgs a = args;
  const int64_t load = (int64_t)a.max_count * a.KS;     // (token, expert) pairs of the call, all groups together
  const int items = a.g_max + (int)(load >> a.work.shift);
  const auto blocks = [&](int rows, int tiles_per_wg) { return dim3((items + 7) / 8 * 8 * ((rows / 16 + tiles_per_wg - 1) / tiles_per_wg)); };
  if (a.work.shift == kSmallTile && a.max_count <= kFewTokens) {
    // (a group is one item of the list.)  One row tile of W_d per wave where two leave units idle: 8 to 16 tokens on 8 + 1 experts of
    // 2048 x 8192, 144 workgroups of eight tiles, 53 / 39 us; on 16 of 1536 x 4096, 192 of them, 26.5 / 31, on 8 of 3072 x 3072 23.5 / 25.5.
    // Row blocks of an item on one die from eight items per die on: OLMoE-like, 8 / 12 / 16 tokens, 97.8 / 125.5 / 127.8 -> 95.6 /
    // 122.4 / 123.3 us per layer call; with six (12 tokens, 4 each of 60 experts of 2048 x 1408) 107.9 -> 114.2.
    a.by_die = a.g_max >= 64;
    const auto grid = [&](int rows, int tiles_per_wg) { return dim3((a.g_max + 7) / 8 * 8 * ((rows / 16 + tiles_per_wg - 1) / tiles_per_wg)); };
    launch_timed(ffn_few_kernel<2, 1, 8, 3>, grid(a.f, 4), dim3(256), 0, s, e1, a);
    if ((int64_t)a.g_max * ((a.d + 127) / 128) < 160) launch_timed(ffn_few_kernel<1, 1, 8, 5>, grid(a.d, 4), dim3(256), 0, s, e2, a);
    else launch_timed(ffn_few_kernel<1, 2, 8, 3>, grid(a.d, 8), dim3(256), 0, s, e2, a);
  } else if (a.work.shift == kSmallTile) {
    // Row blocks of a tile on one die pay where many experts see few tokens each (OLMoE-like, 16 / 64 / 192 tokens: 126 / 139
    // / 158 against 130 / 145 / 163 us); with fewer than four items per die, or busier experts, they leave dies unevenly
    // loaded (Mixtral-like, 12 / 128 tokens: 388 / 525 against 350 / 472 us; OLMoE-like, 256 tokens: 175 against 172).
    a.by_die = a.g_max >= 32 && load <= (int64_t)24 * a.g_max;
    launch_timed(ffn_gemm_kernel<2, 1, 64, 4, 4, 3>, blocks(a.f, 4), dim3(256), 0, s, e1, a);
    launch_timed(ffn_gemm_kernel<1, 2, 64, 4, 4, 3>, blocks(a.d, 8), dim3(256), 0, s, e2, a);
  } else if (a.work.shift == kMidTile) {
    launch_timed(ffn_gemm_kernel<2, 1, 128, 8, 4, 2>, blocks(a.f, 8), dim3(512), 0, s, e1, a);
    launch_timed(ffn_gemm_kernel<1, 1, 128, 8, 4, 4>, blocks(a.d, 8), dim3(512), 0, s, e2, a);
  } else {
    launch_timed(ffn_gemm_kernel<2, 1, 256, 8, 3, 2>, blocks(a.f, 8), dim3(512), 0, s, e1, a);
    launch_timed(ffn_gemm_kernel<1, 2, 256, 8, 3, 2>, blocks(a.d, 16), dim3(512), 0, s, e2, a);
  }
  return hipGetLastError();
}

}  // namespace moe
