// Expert SwiGLU FFN (paper section 2, Eq. 3) and the weighted sum of Eq. 2 for
// expert blocks kept in the plain row-major layout W_g | W_u | W_d, fp32 or
// bf16.  This is the layout-agnostic path (one wavefront per output row, four tokens at a time, DPP
// reduction over the contraction); the bf16 production path is ffn_tiled.hip.
#include <algorithm>
#include <type_traits>

#include "device_utils.hpp"
#include "gating.hpp"
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
// what a workgroup does over `rows` rows: rounds, of as many rows at a time as its groups of lanes have in flight, and the steps in them, 16 bytes a lane at a time
inline int64_t token_rounds(int64_t rows, int pieces) {
  const int at_once = kTokenRows * kTokenThreads / token_lanes(pieces);
  return (rows + at_once - 1) / at_once;
}
inline int64_t token_steps(int64_t rows, int pieces) { return token_rounds(rows, pieces) * ((pieces + token_lanes(pieces) - 1) / token_lanes(pieces)); }
inline size_t token_lds(int KS, int d, int f) { return ((size_t)d + (size_t)KS * (f + d) + 4 * KS) * 4; }

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

// What a workgroup keeps of its token in LDS.
struct TokenLds {
  float *xs, *h, *o;           // [d] token, [KS][f], [KS][d]
  const char** wp;             // [KS] expert blocks
  float* ws;                   // [KS] gate weights
  int* ids;                    // [KS] expert buffers
};
__device__ __forceinline__ TokenLds token_lds_of(float* mem, const FfnArgs& a) {      // (d, f: multiples of V)
  TokenLds l;
  l.xs = mem; l.h = l.xs + a.d; l.o = l.h + a.KS * a.f;
  l.wp = reinterpret_cast<const char**>(l.o + a.KS * a.d); l.ws = reinterpret_cast<float*>(l.wp + a.KS); l.ids = reinterpret_cast<int*>(l.ws + a.KS);
  return l;
}
template <typename T>
__device__ __forceinline__ void stage_token(const FfnArgs& a, float* xs, int b) {
  constexpr int V = kVec<T>;
  for (int i = threadIdx.x * V; i < a.d; i += kTokenThreads * V) {
    float v[V];
    load_vec(reinterpret_cast<const T*>(a.x) + (size_t)b * a.d + i, v);
#pragma unroll
    for (int e = 0; e < V; ++e) xs[i + e] = v[e];
  }
}

// From the token and its experts in LDS (behind a barrier) to y.  between(): after the first projections.
template <typename T, typename Between>
__device__ __forceinline__ void token_ffn(const FfnArgs& a, const TokenLds& l, int b, T* __restrict__ y, int lanes_d, int lanes_f, Between between) {
  constexpr int V = kVec<T>;
  const int KS = a.KS, d = a.d, f = a.f;
  float *xs = l.xs, *h = l.h, *o = l.o, *ws = l.ws;
  const char** wp = l.wp;
  // Rows: per group of lanes, four at a time; pair and row of a flat index.  What bounds a step is the instructions around its
  // products (16 waves share the unit): the pair by a multiplication, its block from LDS, one silu for the four rows.
  const auto each = [&](int lanes, int per_pair, auto&& rows4) {
    const int n = KS * per_pair, groups = kTokenThreads / lanes, grp = threadIdx.x / lanes, at = threadIdx.x % lanes;
    const uint32_t inverse = 0xffffffffu / (uint32_t)per_pair + 1;      // (per_pair > 1; n x per_pair < 2^32: exact)
    for (int r0 = grp; r0 < n; r0 += kTokenRows * groups) {
      int r[kTokenRows], j[kTokenRows];
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u) {
        r[u] = min(r0 + u * groups, n - 1);       // clamped: formed again by its owner, with the same result
        j[u] = (int)__umulhi((uint32_t)r[u], inverse);
      }
      rows4(r, j, at);
    }
  };
  each(lanes_d, f, [&](const int (&r)[kTokenRows], const int (&j)[kTokenRows], int at) {
    const T* w[kTokenRows];
    float sg[kTokenRows], su[kTokenRows];
#pragma unroll
    for (int u = 0; u < kTokenRows; ++u) {
      w[u] = reinterpret_cast<const T*>(wp[j[u]]) + (r[u] - j[u] * f) * d;      // (an expert is at most kTokenMost bytes)
      sg[u] = su[u] = 0.f;
    }
    for (int i = at * V; i < d; i += lanes_d * V) {
      float vg[kTokenRows][V], vu[kTokenRows][V];
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u) {
        load_vec(w[u] + i, vg[u]);
        load_vec(w[u] + f * d + i, vu[u]);
      }
#pragma unroll
      for (int u = 0; u < kTokenRows; ++u)
#pragma unroll
        for (int e = 0; e < V; ++e) { sg[u] = fmaf(vg[u][e], xs[i + e], sg[u]); su[u] = fmaf(vu[u][e], xs[i + e], su[u]); }
    }
    float vg = 0.f, vu = 0.f;
    int row = 0;
#pragma unroll
    for (int u = 0; u < kTokenRows; ++u) {
      const float tg = lanes_sum(sg[u], lanes_d), tu = lanes_sum(su[u], lanes_d);
      vg = at == u ? tg : vg;
      vu = at == u ? tu : vu;
      row = at == u ? r[u] : row;
    }
    if (at < kTokenRows) h[row] = silu(vg) * vu;
  });
  __syncthreads();
  between();
  each(lanes_f, d, [&](const int (&r)[kTokenRows], const int (&j)[kTokenRows], int at) {
    const T* w[kTokenRows];
    float s[kTokenRows];
#pragma unroll
    for (int u = 0; u < kTokenRows; ++u) {
      w[u] = reinterpret_cast<const T*>(wp[j[u]]) + 2 * f * d + (r[u] - j[u] * d) * f;
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

template <typename T>
__global__ void __launch_bounds__(kTokenThreads) ffn_token_rowmajor(FfnArgs a, T* __restrict__ y, int lanes_d, int lanes_f) {
  extern __shared__ __align__(16) float token_mem[];
  const int KS = a.KS, b = blockIdx.x;
  const TokenLds l = token_lds_of(token_mem, a);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if ((int)threadIdx.x < KS) l.ws[threadIdx.x] = a.t.wpair[(size_t)b * KS + threadIdx.x];
  stage_token<T>(a, l.xs, b);
  const int ng = *a.t.n_groups;
  for (int j = wave; j < KS; j += kTokenThreads / 64) {       // the group that holds the pair
    const int pos = a.t.pos_of[(size_t)b * KS + j];
    if (lane == 0) l.ids[j] = 0;                              // (a call without groups has no expert to name: stay in bounds)
    for (int g = lane; g < a.g_max; g += 64) {                // (g_max descriptors exist: requested beside the count)
      const GroupDesc gd = a.t.grp[g];
      if (g < ng && pos >= gd.begin && pos < gd.begin + gd.count) l.ids[j] = gd.buf;
    }
    wave_sync();
    if (lane == 0) l.wp[j] = group_weights(a, l.ids[j]);
  }
  __syncthreads();
  token_ffn<T>(a, l, b, y, lanes_d, lanes_f, [] {});
}

// The whole layer call in ONE launch: fp32 experts that are all in memory, up to 64 of them and 64 tokens, a workgroup per token.  Such a call is
// launches and memory round trips, and the routing launch was half of it: 4 tokens, 2 of 8 experts of 64 x 128, 15.7 -> 10.0 us per layer call, 16 tokens,
// 4 of 60 of 64 x 64, 22.1 -> 10.8.  A workgroup routes its own token - products with the rows of W_r as route_small_fp32_kernel forms them, a
// wave per expert - and looks its experts up itself, since residency does not change; it reads no other token, so y may be x.  KEEP: the recency
// of the slots is brought up to date by the workgroup that arrives last, from the selections that the others sent past the caches; all have
// read the table before they arrive.
constexpr int kLayerTokens = 64;
// Bytes of W_r, which every workgroup reads: 1 of 64 experts of 1024 x 64, 1 / 16 / 64 tokens, 18.2 / 23.2 / 40.6 us with a launch for the
// routing, 15.4 / 17.8 / 23.8 without.
constexpr size_t kLayerRouter = 256 << 10;
constexpr int kLayerSteps = 5;
template <bool KEEP>
__global__ void __launch_bounds__(kTokenThreads) token_layer_kernel(FfnArgs a, RouteArgs r, LayerState st, CacheCallArgs c, uint64_t* masks,
                                                                    float* __restrict__ y, int lanes_d, int lanes_f) {
  extern __shared__ __align__(16) float token_mem[];
  __shared__ float zs[kWave];
  __shared__ int map[kWave], last;
  const int KS = a.KS, K = c.K, E = c.E, B = c.B, d = a.d, b = blockIdx.x;
  const TokenLds l = token_lds_of(token_mem, a);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // wave 0: the table of the layer, a slot per lane
  int slot_expert = -1, slot_buf = 0;
  int64_t sc = 0;
  double score = 0.0;
  if (wave == 0) {
    if (KEEP) {
      slot_expert = lane < c.C ? st.expert_in[lane] : -1;
      slot_buf = lane < c.C ? st.buf_of_slot[lane] : 0;
      sc = lane < SC_COUNT ? st.scalars[lane] : 0;
      if (c.policy == MOE_POLICY_GAMMA && lane < E) score = st.score[lane];
    } else {
      slot_expert = lane < E ? lane : -1;
      slot_buf = lane;
    }
  }
  stage_token<float>(a, l.xs, b);
  {
    const int n_vec = d / 4;
    constexpr int U = 4, WAVES = kTokenThreads / 64;      // products of a wave in flight together
    const float4* xv = reinterpret_cast<const float4*>(static_cast<const float*>(r.x) + (size_t)b * d);
    for (int e0 = wave; e0 < E; e0 += U * WAVES) {
      float acc[U], bias[U];
      const float4* wv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int e = min(e0 + u * WAVES, E - 1);         // clamped: in bounds, formed again
        wv[u] = reinterpret_cast<const float4*>(static_cast<const float*>(r.router_w) + (size_t)e * d);
        bias[u] = r.bias ? r.bias[(size_t)b * E + e] : 0.f;
        acc[u] = 0.f;
      }
      for (int i = lane; i < n_vec; i += kWave) {
        const float4 x = xv[i];
        float4 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = wv[u][i];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          acc[u] = fmaf(w[u].x, x.x, acc[u]); acc[u] = fmaf(w[u].y, x.y, acc[u]);
          acc[u] = fmaf(w[u].z, x.z, acc[u]); acc[u] = fmaf(w[u].w, x.w, acc[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float sum = wave_sum(acc[u]);
        if (lane == 0) zs[min(e0 + u * WAVES, E - 1)] = sum + bias[u];
      }
    }
  }
  if (wave == 0 && slot_expert >= 0) map[slot_expert] = slot_buf;
  __syncthreads();
  uint64_t mine = 0;
  if (wave == 0) {
    Gate<1> g;
    select_experts<1>(zs, E, K, g);
    mine = g.top[0];
    if (KEEP && B > 1 && lane == 0) __hip_atomic_store(masks + b, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    write_weights<1>(g, 0, E, K, KS, r.norm_topk, l.ws, r.user_w ? r.user_w + (size_t)b * K : nullptr, [&](size_t pos, int e) {
      l.wp[pos] = group_weights(a, map[e]);
      if (r.user_idx) r.user_idx[(size_t)b * K + pos] = e;
    });
    if (lane < KS - K) l.wp[K + lane] = group_weights(a, a.P + lane);
  }
  __syncthreads();
  int arrived = 0;
  token_ffn<float>(a, l, b, y, lanes_d, lanes_f, [&] {
    if (KEEP && B > 1 && threadIdx.x == 0) {              // (its answer comes while the second projection runs)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // the selection has arrived: it was sent ahead of the weights' loads
      arrived = __hip_atomic_fetch_add(r.arrive, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  });
  if constexpr (KEEP) {
    if (threadIdx.x == 0) last = arrived == B - 1;
    if (wave != 0) return;
    wave_sync();
    if (!last) return;
    if (B > 1) {
      if (lane == 0) __hip_atomic_store(r.arrive, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // ready for the next launch
      mine = lane < B ? __hip_atomic_load(masks + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    } else if (lane > 0) {
      mine = 0;
    }
    // lane b: the selection of token b; lane s: slot s; lane e: the discounted count of expert e
    const int64_t clock = (int64_t)uniform64(__shfl(sc, SC_CLOCK)), trace_n = (int64_t)uniform64(__shfl(sc, SC_TRACE_N));
    int last_use = 0;
    for (int t = 0; t < B; ++t) {
      const uint64_t m = ((uint64_t)(uint32_t)readlane_i((int)(uint32_t)(mine >> 32), t) << 32) | (uint32_t)readlane_i((int)(uint32_t)mine, t);
      if (slot_expert >= 0 && ((m >> slot_expert) & 1)) last_use = t * K + __popcll(m & ((1ull << slot_expert) - 1ull)) + 1;
      if (c.policy == MOE_POLICY_GAMMA) score = __dadd_rn(__dmul_rn(c.gamma, score), (double)((m >> lane) & 1));      // Definition C.1, once per token
    }
    if (last_use > 0) st.tick[lane] = (uint64_t)(clock + last_use);
    if (c.policy == MOE_POLICY_GAMMA && lane < E) st.score[lane] = score;
    int q = lane * K;
    for (uint64_t m = mine; m != 0; m &= m - 1, ++q)
      if (trace_n + q < c.trace_cap) st.trace[trace_n + q] = moe_trace_rec_t{c.row0 + lane, __ffsll((unsigned long long)m) - 1, 1, -1};
    if (lane == 0) {
      st.scalars[SC_CLOCK] = clock + B * K;
      st.scalars[SC_CALLSEQ] = c.seq;
      st.scalars[SC_TRACE_N] = trace_n + B * K;
    }
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

// A workgroup's time follows its steps, not its bytes.  The kernels per expert take 15 to 18 us, the rate at which four launches are
// issued, until the tokens of their largest group and all pairs together cost more.
//   In one launch with the routing (`whole`): always up to five steps in all.  us per call, whole / per expert: 2 steps, 1 / 8 / 64 tokens 9.5 /
// 10.7 / 14.6 and 15.1 / 19.4 / 25; 4 steps 12.2 / 13.5 / 17.5 and 15.2 / 18.7 / 29; 957 points 1.03x at the least.  Beyond, by what
// either way costs, in 21sts of a us: every round of sums over 32 or 64 lanes 24, over 16 lanes 20 (the first projection has two of them)
// here; 8 for every token of the largest group and 3 for every group there, and 120 ahead (176 by least squares: the points scatter by 2.7 us).
// Taken: 6 of 48 of 56 x 92, 6 tokens, 15.4 / 21.8, 8 of 64 + 2 of 100 x 24, 4 tokens, 14.8 / 22.8.  Left, few pairs on wide rows and many rounds: 1 of 8
// of 240 x 164, 7 tokens, 19.9 / 15.7, 2 of 16 of 88 x 172, 3 tokens, 17.0 / 14.9, 1 of 32 of 228 x 244, 12 tokens, 23.6 / 19.8, 4 of 16 of 192 x
// 112, 64 tokens, 36.4 / 32.7.  Of 3239 points, 1.23x in the mean, none is more than 1.1 % slower than without the one launch.
//   Behind a routing launch, counted in thirds of an fp32 step (a bf16 step has four): two steps, in bf16 only for one token, and a third
// more for every 32 pairs, and for every 4 tokens of the largest group that have 64 pieces of a row of W_g or W_d to add up.  us per call,
// a token's workgroup / per expert: bf16, 2 steps, 1 / 8 / 64 / 256 tokens 12.9 / 16.4 / 19.6 / 25.8 and 15.7 / 18.7 / 33 / 74; 3 steps
// 15.7 / 18.3 / 21.0 / 26.1 and 16.3 / 18.2 / 31 / 64; 5 steps 19.5 / 23.9 / 26.4 / 38.9 and 15.7 / 20.0 / 39 / 104; fp32, 128 / 256
// tokens, 2 steps 21.3 / 28.2 and 46 / 75, 5 steps 29.2 / 38.7 and 71 / 124.  919 points: the 591 that the rule takes 2.3x in the mean, the
// least 1.07x; of the 328 it leaves, all bf16, 203 would be slower and 93 faster by more than 5 % (two steps and 2 to 8 tokens, most of
// them).
bool ffn_token_supported(int pool_layout, int dtype, int batch, int K, int n_shared, int E, int d, int f, bool whole) {
  if (pool_layout != MOE_LAYOUT_ROWMAJOR) return false;
  const int KS = K + n_shared, elem = dtype == MOE_DTYPE_FP32 ? 4 : 2, V = 16 / elem;
  if (f % V != 0 || KS > kTokenThreads || token_lds(KS, d, f) > kTokenLds || (int64_t)KS * 3 * d * f * elem > kTokenMost) return false;
  const int64_t steps = token_steps((int64_t)KS * f, d / V) + token_steps((int64_t)KS * d, f / V);
  const int64_t pairs = (int64_t)batch * K, largest8 = n_shared > 0 ? 8 * (int64_t)batch : 8 * pairs / std::min<int64_t>(pairs, E);     // (in the mean)
  if (whole) {
    const auto sums = [&](int64_t rows, int pieces) { return token_rounds(rows, pieces) * (token_lanes(pieces) > 16 ? 24 : 20); };
    const int64_t others = 120 + largest8 + 3 * std::min<int64_t>(pairs, E);
    if (steps <= kLayerSteps || 2 * sums((int64_t)KS * f, d / V) + sums((int64_t)KS * d, f / V) <= others) return true;
  }
  const int64_t rounds = ((int64_t)batch + 255) / 256;
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

bool token_layer_supported(int pool_layout, int dtype, int batch, int E, int C, int d) {
  return pool_layout == MOE_LAYOUT_ROWMAJOR && dtype == MOE_DTYPE_FP32 && batch <= kLayerTokens && E <= kWave && C <= kWave &&
         (size_t)E * d * sizeof(float) <= kLayerRouter;
}

hipError_t launch_token_layer(hipStream_t s, const FfnArgs& a, const RouteArgs& r, const LayerState& st, const CacheCallArgs& c, uint64_t* masks,
                              void* y, KernelEvents ev) {
  const size_t lds = token_lds(a.KS, a.d, a.f);
  const auto launch = [&](auto kernel) {
    launch_timed(kernel, dim3(c.B), dim3(kTokenThreads), lds, s, ev, a, r, st, c, masks, (float*)y, token_lanes(a.d / 4), token_lanes(a.f / 4));
  };
  if (c.resident) launch(token_layer_kernel<false>);
  else launch(token_layer_kernel<true>);
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
