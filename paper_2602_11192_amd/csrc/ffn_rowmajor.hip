// Expert SwiGLU FFN (paper section 2, Eq. 3) and the weighted sum of Eq. 2 for
// expert blocks kept in the plain row-major layout W_g | W_u | W_d, fp32 or
// bf16.  This is the layout-agnostic path (one wavefront per output row, four tokens at a time, DPP
// reduction over the contraction); the bf16 production path is ffn_tiled.hip.
#include <algorithm>
#include <type_traits>

#include "device_utils.hpp"
#include "moe_internal.hpp"

namespace moe {

namespace {

constexpr int kRowsPerBlock = 4;

__device__ __forceinline__ const char* group_weights(const FfnArgs& a, int id) {
  return id < a.P ? a.buffers + (size_t)id * a.expert_bytes
                  : a.shared + (size_t)(id - a.P) * a.expert_bytes;
}

// Sixteen bytes of a row, widened (V elements); the caller guarantees that rows are whole multiples of 16 bytes.
template <typename T> constexpr int kVec = 16 / (int)sizeof(T);
__device__ __forceinline__ void load_vec(const float* p, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
}
__device__ __forceinline__ void load_vec(const uint16_t* p, float (&v)[8]) {
  const uint4 t = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) { v[2 * i] = bf16_to_f32((uint16_t)w[i]); v[2 * i + 1] = bf16_to_f32((uint16_t)(w[i] >> 16)); }
}

// Tokens whose products with a row run side by side: a group's tokens one after the other each pay the memory round trip
// and the reduction of a row in full.  What bounds these launches is that chain, not bytes: layer calls in fp32 of 16
// tokens on 8 experts of 256 x 384 36.2 -> 22.1 us, on 64 of 512 x 256 37.5 -> 27.8, of 8 tokens on 16 of 256 x 256 24.3 -> 19.6
// with four tokens side by side and 16-byte loads.  (A workgroup per (token, expert) pair doing both projections in one
// launch saved 2 us on the smallest experts with 16 tokens and lost 3 to 20 elsewhere.)
constexpr int kTok = 4;

// Calls f with the number of tokens a wave takes at a time: no more than the group has.
template <typename F>
__device__ __forceinline__ void by_count(int cnt, F f) {
  if (cnt == 1) f(std::integral_constant<int, 1>{});
  else if (cnt == 2) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, kTok>{});
}

// h[pos][j] = silu(W_g[j,:].x) * (W_u[j,:].x)
template <typename T>
__global__ void __launch_bounds__(64 * kRowsPerBlock) gate_up_rowmajor(FfnArgs a) {
  constexpr int V = kVec<T>;
  const int g = blockIdx.y;
  const int ng = *a.t.n_groups;
  const GroupDesc gd = a.t.grp[g];
  if (g >= ng || (a.pass != 2 && gd.miss != a.pass)) return;
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  if (j >= a.f) return;
  const T* w = reinterpret_cast<const T*>(group_weights(a, gd.buf));
  const T* wg = w + (size_t)j * a.d;
  const T* wu = w + (size_t)a.f * a.d + (size_t)j * a.d;
  const int begin = gd.begin, cnt = gd.count;
  float* h = reinterpret_cast<float*>(a.h);
  by_count(cnt, [&](auto n_tok) {
  constexpr int N = decltype(n_tok)::value;
  for (int t0 = 0; t0 < cnt; t0 += N) {
    const T* xr[N];
    float sg[N], su[N];
#pragma unroll
    for (int t = 0; t < N; ++t) {
      const int p = a.t.sorted_pair[begin + min(t0 + t, cnt - 1)];       // clamped: formed again, dropped below
      xr[t] = reinterpret_cast<const T*>(a.x) + (size_t)(p / a.KS) * a.d;
      sg[t] = su[t] = 0.f;
    }
    for (int i = lane * V; i < a.d; i += kWave * V) {        // host guarantees d % V == 0
      float vg[V], vu[V];
      load_vec(wg + i, vg);
      load_vec(wu + i, vu);
#pragma unroll
      for (int t = 0; t < N; ++t) {
        float x[V];
        load_vec(xr[t] + i, x);
#pragma unroll
        for (int e = 0; e < V; ++e) { sg[t] = fmaf(vg[e], x[e], sg[t]); su[t] = fmaf(vu[e], x[e], su[t]); }
      }
    }
#pragma unroll
    for (int t = 0; t < N; ++t) {
      const float vg = wave_sum(sg[t]), vu = wave_sum(su[t]);
      if (lane == 0 && t0 + t < cnt) h[(size_t)(begin + t0 + t) * a.f + j] = silu(vg) * vu;
    }
  }
  });
}

// o[pos][i] = W_d[i,:].h[pos,:].  VEC: rows of W_d are whole multiples of 16 bytes (f % V == 0).
template <typename T, bool VEC>
__global__ void __launch_bounds__(64 * kRowsPerBlock) down_rowmajor(FfnArgs a) {
  constexpr int V = VEC ? kVec<T> : 1;
  const int g = blockIdx.y;
  const int ng = *a.t.n_groups;
  const GroupDesc gd = a.t.grp[g];
  if (g >= ng || (a.pass != 2 && gd.miss != a.pass)) return;
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * kRowsPerBlock + (threadIdx.x >> 6);
  if (i >= a.d) return;
  const T* wd = reinterpret_cast<const T*>(group_weights(a, gd.buf)) + (size_t)2 * a.f * a.d + (size_t)i * a.f;
  const int begin = gd.begin, cnt = gd.count;
  by_count(cnt, [&](auto n_tok) {
  constexpr int N = decltype(n_tok)::value;
  for (int t0 = 0; t0 < cnt; t0 += N) {
    const float* hr[N];
    float s[N];
#pragma unroll
    for (int t = 0; t < N; ++t) {
      hr[t] = reinterpret_cast<const float*>(a.h) + (size_t)(begin + min(t0 + t, cnt - 1)) * a.f;
      s[t] = 0.f;
    }
    for (int j = lane * V; j < a.f; j += kWave * V) {
      float w[V];
      if constexpr (VEC) load_vec(wd + j, w);
      else w[0] = Elem<T>::load(wd + j);
#pragma unroll
      for (int t = 0; t < N; ++t) {
        float x[V];
        if constexpr (VEC) {
#pragma unroll
          for (int e = 0; e < V; e += 4) {
            float q[4];
            load_vec(hr[t] + j + e, q);
#pragma unroll
            for (int k = 0; k < 4; ++k) x[e + k] = q[k];
          }
        } else {
          x[0] = hr[t][j];
        }
#pragma unroll
        for (int e = 0; e < V; ++e) s[t] = fmaf(w[e], x[e], s[t]);
      }
    }
#pragma unroll
    for (int t = 0; t < N; ++t) {
      const float v = wave_sum(s[t]);
      if (lane == 0 && t0 + t < cnt) a.o[(size_t)(begin + t0 + t) * a.d + i] = v;
    }
  }
  });
}

// Small experts, all of them resident: one workgroup takes a token through its KS experts - both projections of every pair, W_d,
// the weighted sum - with what lies between in LDS.  What bounds such a call is its launches and the memory round trips of
// each, not bytes.  A row of d or f elements belongs to 16, 32 or 64 lanes, as many as it has 16-byte pieces, and a group of lanes has four rows in
// flight: at d = 64 a wave holds four rows at a time where the kernels above keep three quarters of it idle.
constexpr int kTokenThreads = 1024, kTokenRows = 4;
constexpr size_t kTokenLds = 60 << 10;
constexpr int64_t kTokenMost = 1 << 20;
inline int token_lanes(int pieces) { return pieces > 32 ? 64 : pieces > 16 ? 32 : 16; }       // ... of a row of so many
// steps of a workgroup over `rows` rows: as many rows at a time as its groups of lanes have in flight, 16 bytes a lane at a time
inline int64_t token_steps(int64_t rows, int pieces) {
  const int lanes = token_lanes(pieces), at_once = kTokenRows * kTokenThreads / lanes;
  return (rows + at_once - 1) / at_once * ((pieces + lanes - 1) / lanes);
}
inline size_t token_lds(int KS, int d, int f) { return ((size_t)d + (size_t)KS * (f + d) + 2 * KS) * 4; }

// the sum over each group of 16, 32 or 64 lanes
__device__ __forceinline__ float lanes_sum(float v, int lanes) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  v += dpp_mov<0x140>(v);
  if (lanes > 16) v += __shfl_xor(v, 16);
  if (lanes > 32) v += __shfl_xor(v, 32);
  return v;
}

template <typename T>
__global__ void __launch_bounds__(kTokenThreads) ffn_token_rowmajor(FfnArgs a, T* __restrict__ y, int lanes_d, int lanes_f) {
  constexpr int V = kVec<T>;
  extern __shared__ __align__(16) float token_mem[];
  const int KS = a.KS, d = a.d, f = a.f, b = blockIdx.x;
  float* xs = token_mem;                          // [d]; d, f: multiples of V
  float* h = xs + d;                              // [KS][f]
  float* o = h + KS * f;                          // [KS][d]
  float* ws = o + KS * d;                         // [KS] gate weights
  int* ids = reinterpret_cast<int*>(ws + KS);     // [KS] expert buffers
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if ((int)threadIdx.x < KS) ws[threadIdx.x] = a.t.wpair[(size_t)b * KS + threadIdx.x];
  for (int i = threadIdx.x * V; i < d; i += kTokenThreads * V) {
    float v[V];
    load_vec(reinterpret_cast<const T*>(a.x) + (size_t)b * d + i, v);
#pragma unroll
    for (int e = 0; e < V; ++e) xs[i + e] = v[e];
  }
  const int ng = *a.t.n_groups;
  for (int j = wave; j < KS; j += kTokenThreads / 64) {       // the group that holds the pair
    const int pos = a.t.pos_of[(size_t)b * KS + j];
    if (lane == 0) ids[j] = 0;                                // (a call without groups has no expert to name: stay in bounds)
    for (int g = lane; g < a.g_max; g += 64) {                // (g_max descriptors exist: requested beside the count)
      const GroupDesc gd = a.t.grp[g];
      if (g < ng && pos >= gd.begin && pos < gd.begin + gd.count) ids[j] = gd.buf;
    }
  }
  __syncthreads();
  // rows: per group of lanes, four at a time; pair and row of a flat index
  const auto each = [&](int lanes, int per_pair, auto&& rows4) {
    const int n = KS * per_pair, groups = kTokenThreads / lanes, grp = threadIdx.x / lanes, at = threadIdx.x % lanes;
    for (int r0 = grp; r0 < n; r0 += kTokenRows * groups) {
      int r[kTokenRows], j[kTokenRows];
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u) {
        r[u] = min(r0 + u * groups, n - 1);       // clamped: formed again by its owner, with the same result
        j[u] = r[u] / per_pair;
      }
      rows4(r, j, at);
    }
  };
  each(lanes_d, f, [&](const int (&r)[kTokenRows], const int (&j)[kTokenRows], int at) {
    const T* w[kTokenRows];
    float sg[kTokenRows], su[kTokenRows];
#pragma unroll
    for (int u = 0; u < kTokenRows; ++u) {
      w[u] = reinterpret_cast<const T*>(group_weights(a, ids[j[u]])) + (size_t)(r[u] - j[u] * f) * d;
      sg[u] = su[u] = 0.f;
    }
    for (int i = at * V; i < d; i += lanes_d * V) {
      float vg[kTokenRows][V], vu[kTokenRows][V];
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u) {
        load_vec(w[u] + i, vg[u]);
        load_vec(w[u] + (size_t)f * d + i, vu[u]);
      }
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) { sg[u] = fmaf(vg[u][e], xs[i + e], sg[u]); su[u] = fmaf(vu[u][e], xs[i + e], su[u]); }
    }
#pragma unroll
    for (int u = 0; u < kTokenRows; ++u) {
      const float vg = lanes_sum(sg[u], lanes_d), vu = lanes_sum(su[u], lanes_d);
      if (at == 0) h[r[u]] = silu(vg) * vu;
    }
  });
  __syncthreads();
  each(lanes_f, d, [&](const int (&r)[kTokenRows], const int (&j)[kTokenRows], int at) {
    const T* w[kTokenRows];
    float s[kTokenRows];
#pragma unroll
    for (int u = 0; u < kTokenRows; ++u) {
      w[u] = reinterpret_cast<const T*>(group_weights(a, ids[j[u]])) + (size_t)2 * f * d + (size_t)(r[u] - j[u] * d) * f;
      s[u] = 0.f;
    }
    for (int i = at * V; i < f; i += lanes_f * V) {
      float v[kTokenRows][V];
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u) load_vec(w[u] + i, v[u]);
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) s[u] = fmaf(v[u][e], h[j[u] * f + i + e], s[u]);
    }
#pragma unroll
    for (int u = 0; u < kTokenRows; ++u) {
      const float v = lanes_sum(s[u], lanes_f);
      if (at == 0) o[r[u]] = v;
    }
  });
  __syncthreads();
  for (int i = threadIdx.x; i < d; i += kTokenThreads) {
    float acc = 0.f;
    for (int j = 0; j < KS; ++j) acc = fmaf(ws[j], o[j * d + i], acc);
    Elem<T>::store(y + (size_t)b * d + i, acc);
  }
}

// y[b][i] = sum_j wpair[b][j] * o[pos_of[b][j]][i], j over the K selected then the shared experts.
// A thread owns four consecutive columns (16-byte loads); the rows of a batch of pairs are all requested before
// the first is used; the pairs are added in index order, so the result does not depend on the batch size.
typedef float f32x4_c __attribute__((ext_vector_type(4)));
constexpr int kCombinePairs = 8;

template <typename T>
__global__ void __launch_bounds__(256)
combine_kernel(const float* __restrict__ o, const float* __restrict__ wpair, const int32_t* __restrict__ pos_of,
               int KS, int d, T* __restrict__ y) {
  const int b = blockIdx.x;
  const int i = (blockIdx.y * blockDim.x + threadIdx.x) * 4;      // host guarantees d % 4 == 0
  if (i >= d) return;
  const float* wrow = wpair + (size_t)b * KS;
  const int32_t* prow = pos_of + (size_t)b * KS;
  f32x4_c acc = {0.f, 0.f, 0.f, 0.f};
  for (int j0 = 0; j0 < KS; j0 += kCombinePairs) {
    f32x4_c v[kCombinePairs];
    float w[kCombinePairs];
#pragma unroll
    for (int u = 0; u < kCombinePairs; ++u) {
      const int j = j0 + u < KS ? j0 + u : KS - 1;          // clamped: in bounds, weight zeroed below
      w[u] = j0 + u < KS ? wrow[j] : 0.f;
      v[u] = *reinterpret_cast<const f32x4_c*>(o + (size_t)prow[j] * d + i);
    }
#pragma unroll
    for (int u = 0; u < kCombinePairs; ++u) {
      if (j0 + u < KS) {      // uniform
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = fmaf(w[u], v[u][c], acc[c]);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) Elem<T>::store(y + (size_t)b * d + i + c, acc[c]);
}

}  // namespace

hipError_t launch_ffn_rowmajor(hipStream_t s, int dtype, const FfnArgs& a, KernelEvents e1, KernelEvents e2) {
  if (a.g_max <= 0) return hipSuccess;
  dim3 block(64 * kRowsPerBlock);
  dim3 g1((a.f + kRowsPerBlock - 1) / kRowsPerBlock, a.g_max);
  dim3 g2((a.d + kRowsPerBlock - 1) / kRowsPerBlock, a.g_max);
  const auto run = [&](auto t, int vec) {
    using T = decltype(t);
    launch_timed(gate_up_rowmajor<T>, g1, block, 0, s, e1, a);
    if (a.f % vec == 0) launch_timed(down_rowmajor<T, true>, g2, block, 0, s, e2, a);
    else launch_timed(down_rowmajor<T, false>, g2, block, 0, s, e2, a);
  };
  if (dtype == MOE_DTYPE_FP32) run(float{}, 4);
  else run(uint16_t{}, 8);
  return hipGetLastError();
}

// A workgroup's time follows its steps, ~3 us each in fp32 and ~4 in bf16 beside 7 fixed, not its bytes: fp32, 2 of 8 experts, 1 token, 64 x 128
// (192 KB, 1 + 1 steps) 12.9 us per call, 64 x 144 (216 KB, 2 + 2) 16.4, 96 x 128 (288 KB, 2 + 2) 19.2, 128 x 128 (384 KB, 2 + 2) 19.1; bf16, 2 of 8 of
// 64 x 256 (192 KB, 2 + 1) 19.3.  The kernels per expert take 16.4 us, the rate at which four launches are issued, until the
// tokens of their largest group and all pairs together cost more.  Counted in thirds of an fp32 step (a
// bf16 step has four), against the kernels per expert, us per call, here / there:
//   two steps in all, the least there is, in fp32; in bf16 only for one token:        fp32 64 x 128, 2 of 8, 1 / 16 tokens 12.9 / 16.3, 17.6 /
//     19.7, bf16 128 x 256, 1 of 8, 1 / 8 tokens 15.7 / 16.2, 17.3 / 16.2
//   a third more for every 32 pairs, and for every 4 tokens of the largest group that have 64 pieces of a row of W_g or W_d to add
//     up: fp32 128 x 128, 2 of 8, 16 / 64 tokens 24.1 / 19.6, 25.1 / 26.0; 64 x 80, 4 of 16, 25.6 / 22.7, 25.9 / 32.6
// 1430 points (130 shapes of 4 to 64 experts, up to 1024 tokens): 1.36x in the mean against the kernels per expert, 24 of
// them more than 2 % slower (the worst 1.14x); the better of the two at every point would be 1.37x.
bool ffn_token_supported(int pool_layout, int dtype, int batch, int K, int n_shared, int E, int d, int f) {
  if (pool_layout != MOE_LAYOUT_ROWMAJOR) return false;
  const int KS = K + n_shared, elem = dtype == MOE_DTYPE_FP32 ? 4 : 2, V = 16 / elem;
  if (f % V != 0 || KS > kTokenThreads || token_lds(KS, d, f) > kTokenLds || (int64_t)KS * 3 * d * f * elem > kTokenMost) return false;
  const int64_t steps = token_steps((int64_t)KS * f, d / V) + token_steps((int64_t)KS * d, f / V), rounds = ((int64_t)batch + 255) / 256;
  const int64_t pairs = (int64_t)batch * K, largest8 = n_shared > 0 ? 8 * (int64_t)batch : 8 * pairs / std::min<int64_t>(pairs, E);     // (in the mean)
  const int64_t pieces64 = (d / V + 63) / 64 + (f / V + 63) / 64;
  return 32 * steps * rounds * (dtype == MOE_DTYPE_FP32 ? 3 : 4) <= 32 * (batch == 1 ? 8 : 6) + (int64_t)batch * KS + largest8 * pieces64;
}

hipError_t launch_ffn_token(hipStream_t s, int dtype, const FfnArgs& a, int batch, void* y, KernelEvents ev) {
  const size_t lds = token_lds(a.KS, a.d, a.f);
  if (dtype == MOE_DTYPE_FP32)
    launch_timed(ffn_token_rowmajor<float>, dim3(batch), dim3(kTokenThreads), lds, s, ev, a, (float*)y, token_lanes(a.d / 4), token_lanes(a.f / 4));
  else
    launch_timed(ffn_token_rowmajor<uint16_t>, dim3(batch), dim3(kTokenThreads), lds, s, ev, a, (uint16_t*)y, token_lanes(a.d / 8), token_lanes(a.f / 8));
  return hipGetLastError();
}

hipError_t launch_combine(hipStream_t s, int dtype, const float* o, const float* wpair, const int32_t* pos_of,
                          int B, int KS, int d, void* y) {
  dim3 grid(B, (d / 4 + 255) / 256), block(256);
  if (dtype == MOE_DTYPE_FP32)
    hipLaunchKernelGGL(combine_kernel<float>, grid, block, 0, s, o, wpair, pos_of, KS, d, (float*)y);
  else
    hipLaunchKernelGGL(combine_kernel<uint16_t>, grid, block, 0, s, o, wpair, pos_of, KS, d, (uint16_t*)y);
  return hipGetLastError();
}

}  // namespace moe
