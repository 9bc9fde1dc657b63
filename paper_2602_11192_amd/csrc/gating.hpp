// Pieces of the routing and cache-lookup phases that more than one kernel uses: the gating of one token by one
// wave (paper Eq. 1 and the gate weights of Eq. 2) and the register-resident LRU table of a layer.
#pragma once
#include "device_utils.hpp"
#include "moe_internal.hpp"

namespace moe {

// ordering point between the lanes of ONE wave (LDS and global), no s_barrier
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ int readlane_i(int v, int lane) { return __builtin_amdgcn_readlane(v, lane); }

__device__ __forceinline__ int64_t uniform64(int64_t v) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)((uint64_t)v >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The call record for the host, written by one lane.  The host polls `seq` in pinned memory instead of waiting for an
// event behind the kernel: an event record between two kernels of a stream costs the GPU 5.6 us of idle time, the
// system-scope release in front of `seq` costs the writing lane under one.  (The miss list is written by the same lane.)
__device__ __forceinline__ void publish_record(Mailbox* mb, int status, int n_miss, int n_evict, int n_groups, int n_hits,
                                               int n_res, uint32_t seq) {
  if (mb == nullptr) return;
  mb->status = status;
  mb->n_miss = n_miss;
  mb->n_evict = n_evict;
  mb->n_groups = n_groups;
  mb->n_hits = n_hits;
  mb->n_res = n_res;
  __hip_atomic_store(&mb->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The register-resident table: LRU, at most 64 slots and 64 buffers, and at most 128 buffer ids in all.
__host__ __device__ inline bool fast_table(int policy, int C, int P, int n_shared) {
  return policy == MOE_POLICY_LRU && C <= kWave && P <= kWave && P + n_shared <= 2 * kWave;
}

// ---------------------------------------------------------------- phase 2
// The K largest of E values held by one wave (value e in z[e / 64] of lane e % 64), as one lane mask per register;
// equal values go to the lower id, NaN counts as less than everything.  Exactly K bits are set whatever the values are
// (K <= E).
// The K-th largest is found bit by bit from the top of its order-preserving integer key: one compare, one ballot and
// a scalar population count per bit, and it ends as soon as a threshold separates exactly K values - after the sign,
// the exponent and a few mantissa bits on router logits.  K rounds of wave-wide arg-max instead take ~250
// cycles each: 1.2 us of a one-token call at K = 8 against 0.3 us.  Beyond 64 values a bit costs as many compares as there
// are registers, and up to kFewRounds rounds are the faster way (one-token call, rounds / bits: 1000 experts, K = 1 67.1 / 70.4
// us, K = 4 71.4 / 72.8, K = 8 76.5 / 75.9; 200 experts, K = 1 27.1 / 28.2, K = 4 28.3 / 29.2, K = 8 31.6 / 31.3).
// kRounds: the kernel has these rounds as well (code that a launch only jumps over costs it 0.2-0.5 us).
constexpr int kFewRounds = 4;
template <int EPL, bool kRounds = false>
__device__ __forceinline__ void top_select(const float (&z)[EPL], int E, int K, uint64_t (&mask)[EPL]) {
  const int lane = threadIdx.x & 63;
  uint32_t key[EPL];
  uint64_t valid[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const uint32_t u = __builtin_bit_cast(uint32_t, z[i] + 0.0f);      // -0 counts as +0
    key[i] = z[i] != z[i] ? 0u : u ^ ((u >> 31) ? 0xffffffffu : 0x80000000u);
    valid[i] = __ballot(lane + i * kWave < E);
  }
  if constexpr (kRounds) {
    if (K <= kFewRounds) {       // K rounds of arg-max
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        mask[i] = 0;
        if (lane + i * kWave >= E) key[i] = 0;
      }
#pragma unroll 1
      for (int k = 0; k < K; ++k) {
        uint32_t m = key[0];
#pragma unroll
        for (int i = 1; i < EPL; ++i) m = max(m, key[i]);
        m = wave_max_u32(m);
        bool done = false;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          const uint64_t at = __ballot(key[i] == m) & valid[i] & ~mask[i];
          if (!done && at != 0) {          // uniform
            const int first = __ffsll((unsigned long long)at) - 1;
            mask[i] |= 1ull << first;
            if (lane == first) key[i] = 0;
            done = true;
          }
        }
      }
      return;
    }
  }
  uint32_t t = 0;          // largest threshold so far that at least K keys reach
#pragma unroll 1
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = t | (1u << bit);
    int n = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) n += __popcll(__ballot(key[i] >= cand) & valid[i]);
    if (n >= K) t = cand;
    if (n == K) break;
  }
  int ties = K;            // entries equal to the threshold that still belong to the K
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    mask[i] = __ballot(key[i] > t) & valid[i];
    ties -= __popcll(mask[i]);
  }
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const uint64_t eq = __ballot(key[i] == t) & valid[i];
    const int before = __popcll(eq & ((1ull << lane) - 1ull));
    mask[i] |= __ballot(((eq >> lane) & 1) != 0 && before < ties);
    ties -= __popcll(eq);
  }
}

// One wave gates one token from the logits in LDS (zs[E]).  kWeights = false: only the selected set (idx_g) is
// formed - same selection, no softmax - for callers that need to know which experts run, not their weights.
template <int EPL, bool kWeights = true, bool kRounds = false>
__device__ __forceinline__ void gate_token(const float* zs, int b, int E, int K, int KS, int norm_topk,
                                           int32_t* idx_g, float* wpair_g, int32_t* user_idx, float* user_w,
                                           int32_t* idx_stage) {
  const int lane = threadIdx.x & 63;
  float z[EPL];
  bool sel[EPL];
  float zmax = -INFINITY;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane + i * kWave;
    z[i] = e < E ? zs[e] : -INFINITY;
    sel[i] = false;
    zmax = fmaxf(zmax, z[i]);
  }
  zmax = wave_max(zmax);
  uint64_t top[EPL];
  top_select<EPL, kRounds>(z, E, K, top);
#pragma unroll
  for (int i = 0; i < EPL; ++i) sel[i] = (top[i] >> lane) & 1;
  if constexpr (!kWeights) {
    int base = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const uint64_t m = __ballot(sel[i]);
      if (sel[i]) idx_g[(size_t)b * K + base + __popcll(m & ((1ull << lane) - 1ull))] = lane + i * kWave;
      base += __popcll(m);
    }
    return;
  }
  float p[EPL];
  float psum = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    p[i] = (lane + i * kWave) < E ? expf(z[i] - zmax) : 0.f;
    psum += p[i];
  }
  psum = wave_sum(psum);
  float selsum = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    p[i] = p[i] / psum;
    selsum += sel[i] ? p[i] : 0.f;
  }
  selsum = wave_sum(selsum);
  int base = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane + i * kWave;
    const uint64_t m = __ballot(sel[i]);
    if (sel[i]) {
      const int pos = base + __popcll(m & ((1ull << lane) - 1ull));   // ascending expert id
      const float w = norm_topk ? p[i] / selsum : p[i];
      idx_g[(size_t)b * K + pos] = e;
      wpair_g[(size_t)b * KS + pos] = w;
      if (idx_stage) idx_stage[(size_t)b * K + pos] = e;
      if (user_idx) user_idx[(size_t)b * K + pos] = e;
      if (user_w) user_w[(size_t)b * K + pos] = w;
    }
    base += __popcll(m);
  }
  if (lane < KS - K) wpair_g[(size_t)b * KS + K + lane] = 1.0f;  // shared experts: weight 1
}

// The same in steps, for a kernel that sets them apart: which experts run (select_experts), their ids in ascending order
// (write_selected), their weights (write_weights).  (gate_token made of these gives the kernels around it other code: 64 tokens on
// 200 experts, looked up in order, 172 -> 175 to 178 us per layer call, one token on 16 18.2 -> 18.4 to 19.4.)
template <int EPL> struct Gate {
  float z[EPL];
  uint64_t top[EPL];       // selected set, one mask per 64 experts
};

template <int EPL, bool kRounds = false>
__device__ __forceinline__ void select_experts(const float* zs, int E, int K, Gate<EPL>& g) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane + i * kWave;
    g.z[i] = e < E ? zs[e] : -INFINITY;
  }
  top_select<EPL, kRounds>(g.z, E, K, g.top);
}

// (idx_g is written at device scope, for another workgroup of the same launch to read)
template <int EPL>
__device__ __forceinline__ void write_selected(const Gate<EPL>& g, int b, int K, int32_t* idx_g, int32_t* idx_stage) {
  const int lane = threadIdx.x & 63;
  int base = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    if ((g.top[i] >> lane) & 1) {
      const size_t pos = (size_t)b * K + base + __popcll(g.top[i] & ((1ull << lane) - 1ull));
      const int e = lane + i * kWave;
      __hip_atomic_store(&idx_g[pos], e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (idx_stage) idx_stage[pos] = e;
    }
    base += __popcll(g.top[i]);
  }
}

// ids(pos, e): expert e is at `pos` of idx; what a caller has to write of that beside the weight
template <int EPL, typename Ids>
__device__ __forceinline__ void write_weights(const Gate<EPL>& g, int b, int E, int K, int KS, int norm_topk, float* wpair_g, float* user_w, Ids ids) {
  const int lane = threadIdx.x & 63;
  float zmax = -INFINITY;
#pragma unroll
  for (int i = 0; i < EPL; ++i) zmax = fmaxf(zmax, g.z[i]);
  zmax = wave_max(zmax);
  float p[EPL];
  float psum = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    p[i] = (lane + i * kWave) < E ? expf(g.z[i] - zmax) : 0.f;
    psum += p[i];
  }
  psum = wave_sum(psum);
  float selsum = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    p[i] = p[i] / psum;
    selsum += ((g.top[i] >> lane) & 1) ? p[i] : 0.f;
  }
  selsum = wave_sum(selsum);
  int base = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    if ((g.top[i] >> lane) & 1) {
      const int pos = base + __popcll(g.top[i] & ((1ull << lane) - 1ull));   // ascending expert id
      const float w = norm_topk ? p[i] / selsum : p[i];
      ids((size_t)b * K + pos, lane + i * kWave);
      wpair_g[(size_t)b * KS + pos] = w;
      if (user_w) user_w[(size_t)b * K + pos] = w;
    }
    base += __popcll(g.top[i]);
  }
  if (lane < KS - K) wpair_g[(size_t)b * KS + K + lane] = 1.0f;  // shared experts: weight 1
}

// ---------------------------------------------------------------- phase 3, register path
// LRU with at most 64 slots, 64 buffers and 64 (token, expert) pairs: lane s holds
// slot s (expert, last-use tick, buffer), lane p holds buffer p's use stamp, lane i
// holds entry i of the free and released-buffer stacks, lane q holds pair q.
struct FastTable {
  int exp, buf, free_b, zomb;
  uint64_t tick;
  uint32_t used;
  int64_t clock, trace_n;
  int n_res, n_free, n_zombie;
};

__device__ __forceinline__ FastTable fast_load(const LayerState& st, int C, int P) {
  const int lane = threadIdx.x & 63;
  FastTable f;
  // the scalars are the same in every lane; telling the compiler so keeps the loops over them and the
  // cross-lane reads indexed by them on the scalar unit
  f.clock = uniform64(st.scalars[SC_CLOCK]);
  f.n_res = __builtin_amdgcn_readfirstlane((int)st.scalars[SC_NRES]);
  f.n_free = __builtin_amdgcn_readfirstlane((int)st.scalars[SC_NFREE]);
  f.n_zombie = __builtin_amdgcn_readfirstlane((int)st.scalars[SC_NZOMBIE]);
  f.trace_n = uniform64(st.scalars[SC_TRACE_N]);
  f.exp = lane < C ? st.expert_in[lane] : -2;
  f.tick = lane < C ? st.tick[lane] : ~0ull;
  f.buf = lane < C ? st.buf_of_slot[lane] : -1;
  f.used = lane < P ? st.used_stamp[lane] : 0u;
  f.free_b = lane < P ? st.free_buf[lane] : -1;
  f.zomb = lane < P ? st.zombie[lane] : -1;
  return f;
}

// index of the lane (< C) holding the smallest tick; ticks of valid lanes are unique
__device__ __forceinline__ int wave_argmin_tick(uint64_t tick) {
  uint32_t hi = (uint32_t)(tick >> 32), lo = (uint32_t)tick;
#define MOE_MIN_STEP(CTRL)                                                                              \
  {                                                                                                     \
    const uint32_t ohi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, 0xf, 0xf, true);       \
    const uint32_t olo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, CTRL, 0xf, 0xf, true);       \
    const bool less = ohi < hi || (ohi == hi && olo < lo);                                              \
    hi = less ? ohi : hi;                                                                               \
    lo = less ? olo : lo;                                                                               \
  }
  MOE_MIN_STEP(0xB1) MOE_MIN_STEP(0x4E) MOE_MIN_STEP(0x141) MOE_MIN_STEP(0x140)
#undef MOE_MIN_STEP
  uint64_t best = ~0ull;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint64_t v = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)hi, r * 16) << 32) |
                       (uint32_t)__builtin_amdgcn_readlane((int)lo, r * 16);
    best = v < best ? v : best;
  }
  return __ffsll((unsigned long long)__ballot(tick == best)) - 1;
}

}  // namespace moe
