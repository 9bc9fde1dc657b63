// Expert SwiGLU FFN (paper section 2, Eq. 3) and the weighted sum of Eq. 2 for
// expert blocks kept in the plain row-major layout W_g | W_u | W_d, fp32 or
// bf16.  This is the layout-agnostic path (one wavefront per output row, four tokens at a time, DPP
// reduction over the contraction); the bf16 production path is ffn_tiled.hip.
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
