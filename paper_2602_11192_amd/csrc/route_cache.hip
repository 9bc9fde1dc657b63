// Router GEMV + softmax/Top-K gating + expert-cache lookup in ONE launch.
//
// Paper section 2: Eq. 1 (p = softmax(W_r x), r = Top-K(p)) and the gate
// weights of Eq. 2; then the offloading runtime of section 2 ("Expert
// Offloading Systems") and section 3.2: a selected expert that is not resident
// is fetched on demand and a cached expert is evicted as the policy dictates.
// LRU is the gamma -> 0+ member and LFU the gamma = 1 member of the
// discounted-count family of Definition C.1; contents change lazily, only by
// inserting the requested expert (Remark after Definition C.1).
//
// Two shapes of the launch, chosen by launch_route_cache:
//   route_cache_kernel: one workgroup per token.  The waves split the E router
//     rows; each forms whole dot products W_r[e,:].x for up to four rows at a time
//     with every 16-byte load issued up front, then DPP reductions; wave 0 gates
//     the token.  Of a batch the workgroup that arrives last at a device-scope
//     counter goes on to the lookups (nobody waits).
//   route_units_kernel: 16 tokens x 16 experts (or several times that) x a slice of
//     the contraction per workgroup, logits on the matrix cores; the last unit of a
//     tile of 16 tokens gates them, a wave per token (route_small_fp32_kernel: a
//     small fp32 call in one workgroup).
// Gating (gate_token, gating.hpp): Top-K of the logits by bisection of their
//   integer keys, ties to the lower id - the same set as Top-K of p - softmax
//   with wave reductions, gate weights, outputs in ascending expert id.
// Lookups, in three forms: all of a call's lookups at once on every wave of the
//   workgroup when every one hits (group_hits: at most 64 slots); one wave in order on
//   the table in registers, one slot per lane, a lookup being a ballot plus a
//   DPP arg-min (cache_phase_fast: LRU, at most 64 slots and buffers); one wave in
//   order on the table in LDS otherwise (cache_phase_general).  In order, because
//   each lookup that misses changes the state the next one sees.  The pairs
//   (token, expert) are grouped by expert buffer for the FFN kernels, the work list
//   of the grouped GEMM is written, and the miss list goes to pinned host memory
//   for the copy scheduler.
// Nothing is committed when the call runs out of spare buffers, so a failed call
// leaves the cache unchanged.
#include <algorithm>
#include <type_traits>

#include "device_utils.hpp"
#include "gating.hpp"
#include "moe_internal.hpp"

namespace moe {


namespace {

// ---------------------------------------------------------------- dot products
template <typename T> struct Vec;
template <> struct Vec<float> {
  static constexpr int N = 4;
  using type = float4;
  static __device__ __forceinline__ float dot(const float4& a, const float4& b, float acc) {
    acc = fmaf(a.x, b.x, acc); acc = fmaf(a.y, b.y, acc);
    acc = fmaf(a.z, b.z, acc); acc = fmaf(a.w, b.w, acc);
    return acc;
  }
};
template <> struct Vec<uint16_t> {
  static constexpr int N = 8;
  using type = uint4;
  static __device__ __forceinline__ float dot(const uint4& a, const uint4& b, float acc) {
    const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc = fmaf(__builtin_bit_cast(float, av[i] << 16), __builtin_bit_cast(float, bv[i] << 16), acc);
      acc = fmaf(__builtin_bit_cast(float, av[i] & 0xffff0000u),
                 __builtin_bit_cast(float, bv[i] & 0xffff0000u), acc);
    }
    return acc;
  }
};

constexpr int kTileMaxE = 256;   // most experts the 16-token tile kernels keep logits for
constexpr int kRouteSliceKb = 16; // fewest k-blocks of the contraction worth a slice of their own
constexpr int kRouteMaxUnits = 256;   // ... and most workgroups that slicing may make: one per compute unit.  (From twice as many
                                      // expert tiles on a unit takes several of them.)

// ---------------------------------------------------------------- LDS layout
struct LdsLayout {
  size_t tick, score, expert_in, buf_of_slot, slot_of, free_buf, zombie, used, filled, pending, count, start,
      logit, idx_stage, pair_stage, total;
};

__host__ __device__ inline bool stage_in_lds(int B, int KS) { return (size_t)B * KS <= kStageMaxPairs; }

__host__ __device__ inline LdsLayout lds_layout(int E, int C, int P, int n_shared, int B, int K, int KS) {
  LdsLayout l;
  size_t o = 0;
  l.tick = o; o += (size_t)C * 8;
  l.score = o; o += (size_t)E * 8;
  l.expert_in = o; o += (size_t)C * 4;
  l.buf_of_slot = o; o += (size_t)C * 4;
  l.slot_of = o; o += (size_t)E * 4;
  l.free_buf = o; o += (size_t)P * 4;
  l.zombie = o; o += (size_t)P * 4;
  l.used = o; o += (size_t)P * 4;
  l.filled = o; o += (size_t)P * 4;
  l.pending = o; o += (size_t)E * 4;
  const int n_keys = (P > E ? P : E) + n_shared;     // grouping keys: buffer ids, or expert ids when streaming a prompt
  l.count = o; o += (size_t)n_keys * 4;
  l.start = o; o += (size_t)n_keys * 4;
  l.logit = o; o += (size_t)E * 4;
  const bool stage = stage_in_lds(B, KS);
  l.idx_stage = o; o += stage ? (size_t)B * K * 4 : 0;
  l.pair_stage = o; o += stage ? (size_t)B * KS * 4 : 0;
  l.total = o;
  return l;
}

// ---------------------------------------------------------------- grouping (any number of pairs)
// Counting sort of the (token, expert) pairs by the buffer they read, run by ONE wave with counters in LDS.
// pair_buf[B*KS] must hold the buffer of every routed pair; shared-expert pairs are filled in here.
// The order of the pairs inside a group is whatever order the LDS atomics resolve in; every pair's arithmetic is
// independent of its position, so the layer output does not depend on it.
__device__ __forceinline__ int group_pairs_lds(int32_t* count, int32_t* cursor, const int32_t* filled, int32_t* pair_buf,
                               const CallTables& t, const CacheCallArgs& a) {
  const int lane = threadIdx.x & 63;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const int K = a.K, KS = a.KS, P = a.P;
  const int NP = a.B * KS, NB = P + a.n_shared;
  for (int p = lane; p < a.B * a.n_shared; p += kWave) {
    const int b = p / a.n_shared, sidx = p - b * a.n_shared;
    pair_buf[(size_t)b * KS + K + sidx] = P + sidx;
  }
  for (int i = lane; i < NB; i += kWave) count[i] = 0;
  wave_sync();
  for (int p = lane; p < NP; p += kWave) atomicAdd(&count[pair_buf[p]], 1);
  wave_sync();
  int n_groups = 0, offset = 0;
  for (int base = 0; base < NB; base += kWave) {        // ids in ascending order, 64 at a time
    const int id = base + lane;
    const int c = id < NB ? count[id] : 0;
    int incl = c;                                       // inclusive prefix sum over the lanes
#pragma unroll
    for (int dlt = 1; dlt < kWave; dlt <<= 1) {
      const int v = __shfl_up(incl, dlt);
      if (lane >= dlt) incl += v;
    }
    const int begin = offset + incl - c;
    const uint64_t gm = __ballot(c > 0);
    if (c > 0) {
      GroupDesc gd;
      const int fe = id < P ? filled[id] : 0;        // expert + 1 of a buffer being filled by this call
      gd.buf = id; gd.begin = begin; gd.count = c; gd.miss = fe != 0;
      gd.pair0 = 0; gd.expert = fe - 1; gd.pad[0] = gd.pad[1] = 0;
      t.grp[n_groups + __popcll(gm & lt_mask)] = gd;
    }
    if (id < NB) cursor[id] = begin;
    n_groups += __popcll(gm);
    offset += __shfl(incl, kWave - 1);
  }
  wave_sync();
  for (int p = lane; p < NP; p += kWave) {
    const int pos = atomicAdd(&cursor[pair_buf[p]], 1);
    t.sorted_pair[pos] = p;
    t.pos_of[p] = pos;
  }
  wave_sync();
  for (int gi = lane; gi < n_groups; gi += kWave) t.grp[gi].pair0 = t.sorted_pair[t.grp[gi].begin];
  return n_groups;
}

// ---------------------------------------------------------------- work list of the grouped GEMM
__device__ __forceinline__ int4 work_item(int tok0, int buf, int begin, int count, int miss) {
  return int4{tok0, buf, begin, count | (miss ? 1 << 30 : 0)};
}

__device__ __forceinline__ int tiles_of(int count, const WorkPlan& w) { return (count + (1 << w.shift) - 1) >> w.shift; }

// The list in the order of the groups, from the descriptors just written; ONE wave.
__device__ __forceinline__ void write_work_list(const CallTables& t, const CacheCallArgs& a, int n_groups) {
  if (a.work.cap == 0) return;
  const int lane = threadIdx.x & 63;
  wave_sync();
  int base = 0;
  for (int g0 = 0; g0 < n_groups; g0 += kWave) {
    GroupDesc gd{};
    if (g0 + lane < n_groups) gd = t.grp[g0 + lane];
    const int buf = a.mode == 2 && gd.miss ? gd.expert : gd.buf;
    const int n = tiles_of(gd.count, a.work);
    int incl = n;
#pragma unroll
    for (int dlt = 1; dlt < kWave; dlt <<= 1) {
      const int v = __shfl_up(incl, dlt);
      if (lane >= dlt) incl += v;
    }
    int4* items = t.work + 1 + base + incl - n;
    for (int i = 0; i < n; ++i) items[i] = work_item(i << a.work.shift, buf, gd.begin, gd.count, gd.miss);
    base += __shfl(incl, kWave - 1);
  }
  if (lane == 0) t.work[0] = int4{base, 0, 0, 0};
}

// ---------------------------------------------------------------- prompt streaming
// Phase 3 of a prefill call: the cache is only READ.  Pairs are grouped by expert; a group whose expert is
// resident reads its buffer, any other group streams its expert from the pinned host pool (miss = 1) and
// nothing is inserted or refreshed, so a one-off scan over a long prompt leaves the cache as the prefetch set
// it.  Runs in ONE wave; idx [B][K] routed experts (LDS or global), keys [B*KS] scratch.
__device__ __forceinline__ void prefill_phase(unsigned char* smem, const LdsLayout& L, const int32_t* idx, int32_t* keys,
                              const LayerState& st, const CallTables& t, const CacheCallArgs& a) {
  int32_t* slot_of = reinterpret_cast<int32_t*>(smem + L.slot_of);
  int32_t* count = reinterpret_cast<int32_t*>(smem + L.count);
  int32_t* cursor = reinterpret_cast<int32_t*>(smem + L.start);
  const int lane = threadIdx.x & 63;
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  const int E = a.E, C = a.C, K = a.K, KS = a.KS, P = a.P;
  const int NP = a.B * KS, NB = E + a.n_shared;
  for (int e = lane; e < E; e += kWave) slot_of[e] = -1;
  for (int i = lane; i < NB; i += kWave) count[i] = 0;
  wave_sync();
  for (int s = lane; s < C; s += kWave) {
    const int ex = st.expert_in[s];
    if (ex >= 0) slot_of[ex] = st.buf_of_slot[s];          // expert -> the buffer that holds it
  }
  for (int p = lane; p < NP; p += kWave) {
    const int b = p / KS, k = p - b * KS;
    keys[p] = k < K ? idx[(size_t)b * K + k] : E + (k - K);
  }
  wave_sync();
  for (int p = lane; p < NP; p += kWave) atomicAdd(&count[keys[p]], 1);
  wave_sync();
  int n_groups = 0, offset = 0, n_stream = 0;
  for (int base = 0; base < NB; base += kWave) {
    const int id = base + lane;
    const int c = id < NB ? count[id] : 0;
    int incl = c;
#pragma unroll
    for (int dlt = 1; dlt < kWave; dlt <<= 1) {
      const int v = __shfl_up(incl, dlt);
      if (lane >= dlt) incl += v;
    }
    const int begin = offset + incl - c;
    const uint64_t gm = __ballot(c > 0);
    const int buf = id < E ? slot_of[id < E ? id : 0] : P + (id - E);
    const bool streamed = c > 0 && id < E && buf < 0;
    if (c > 0) {
      GroupDesc gd;
      gd.buf = streamed ? 0 : buf; gd.begin = begin; gd.count = c; gd.miss = streamed ? 1 : 0;
      gd.pair0 = 0; gd.expert = streamed ? id : -1; gd.pad[0] = gd.pad[1] = 0;
      t.grp[n_groups + __popcll(gm & lt_mask)] = gd;
    }
    if (id < NB) cursor[id] = begin;
    n_groups += __popcll(gm);
    n_stream += __popcll(__ballot(streamed));
    offset += __shfl(incl, kWave - 1);
  }
  wave_sync();
  for (int p = lane; p < NP; p += kWave) {
    const int pos = atomicAdd(&cursor[keys[p]], 1);
    t.sorted_pair[pos] = p;
    t.pos_of[p] = pos;
  }
  wave_sync();
  for (int gi = lane; gi < n_groups; gi += kWave) t.grp[gi].pair0 = t.sorted_pair[t.grp[gi].begin];
  write_work_list(t, a, n_groups);
  if (lane == 0) {
    *t.n_groups = n_groups;
    publish_record(a.mailbox, MOE_OK, n_stream, 0, n_groups, 0, (int)st.scalars[SC_NRES], a.seq);
  }
}

// ---------------------------------------------------------------- phase 3
// General path (any C, P, batch; both policies): the table lives in LDS.
// Runs in ONE wave.  idx: selected experts [B][K] (LDS or global); pair_buf: scratch [B*KS].
__device__ __forceinline__ void cache_phase_general(unsigned char* smem, const LdsLayout& L, const int32_t* idx, int32_t* pair_buf,
                            const LayerState& st, const CallTables& t, const CacheCallArgs& a) {
  uint64_t* tick = reinterpret_cast<uint64_t*>(smem + L.tick);
  double* score = reinterpret_cast<double*>(smem + L.score);
  int32_t* expert_in = reinterpret_cast<int32_t*>(smem + L.expert_in);
  int32_t* buf_of_slot = reinterpret_cast<int32_t*>(smem + L.buf_of_slot);
  int32_t* slot_of = reinterpret_cast<int32_t*>(smem + L.slot_of);
  int32_t* free_buf = reinterpret_cast<int32_t*>(smem + L.free_buf);
  int32_t* zombie = reinterpret_cast<int32_t*>(smem + L.zombie);
  uint32_t* used = reinterpret_cast<uint32_t*>(smem + L.used);
  int32_t* filled = reinterpret_cast<int32_t*>(smem + L.filled);
  int32_t* pending = reinterpret_cast<int32_t*>(smem + L.pending);
  int32_t* count = reinterpret_cast<int32_t*>(smem + L.count);
  int32_t* start = reinterpret_cast<int32_t*>(smem + L.start);

  const int lane = threadIdx.x & 63;
  const int E = a.E, C = a.C, P = a.P, K = a.K, KS = a.KS;
  const bool gamma_policy = a.policy == MOE_POLICY_GAMMA;

  // ---- load the table (independent loads, one round trip) ----
  int64_t clock = st.scalars[SC_CLOCK];
  int n_res = (int)st.scalars[SC_NRES];
  int n_free = (int)st.scalars[SC_NFREE];
  int n_zombie = (int)st.scalars[SC_NZOMBIE];
  const int64_t trace_n = st.scalars[SC_TRACE_N];
  for (int s = lane; s < C; s += kWave) {
    tick[s] = st.tick[s]; expert_in[s] = st.expert_in[s]; buf_of_slot[s] = st.buf_of_slot[s];
  }
  for (int e = lane; e < E; e += kWave) {
    slot_of[e] = -1; pending[e] = 0;
    if (gamma_policy) score[e] = st.score[e];
  }
  for (int i = lane; i < P; i += kWave) {
    used[i] = st.used_stamp[i]; filled[i] = 0;
    // free stack, then the buffers the previous call released (all its kernels have finished)
    if (i < n_free) free_buf[i] = st.free_buf[i];
    else if (i < n_free + n_zombie) free_buf[i] = st.zombie[i - n_free];
  }
  n_free += n_zombie;
  n_zombie = 0;
  wave_sync();
  for (int s = lane; s < C; s += kWave)       // expert -> slot index, rebuilt from the slots
    if (expert_in[s] >= 0) slot_of[expert_in[s]] = s;
  wave_sync();

  const uint32_t seq = a.seq;
  const int n_lookups = a.mode == 0 ? a.B * K : K;
  int status = MOE_OK, n_miss = 0, n_evict = 0, n_hits = 0;
  int64_t trace_added = 0;

  for (int q = 0; q < n_lookups; ++q) {
    const int b = a.mode == 0 ? q / K : 0;
    const int k = a.mode == 0 ? q % K : q;
    const int e = a.mode == 0 ? idx[q] : a.pin_ids[q];
    int s = slot_of[e];
    int evicted = -1, buf;
    const bool hit = s >= 0;
    if (hit) {
      buf = buf_of_slot[s];
      ++n_hits;
    } else {
      if (n_res < C) {            // slots fill in index order, so the lowest empty slot is n_res
        s = n_res;
        buf = free_buf[n_free - 1];
        --n_free;
        ++n_res;
      } else {
        int vs = -1;
        uint64_t vt = ~0ull;
        double vsc = 0.0;
        for (int c = lane; c < C; c += kWave) {
          const uint64_t tc = tick[c];
          if (!gamma_policy) {
            if (tc < vt) { vt = tc; vs = c; }
          } else {
            const int ex = expert_in[c];
            if (pending[ex]) continue;     // wanted by the current token: never a victim
            const double sc = score[ex];
            if (vs < 0 || sc < vsc || (sc == vsc && tc < vt)) { vsc = sc; vt = tc; vs = c; }
          }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
          const int os = __shfl_xor(vs, off);
          const uint64_t ot = __shfl_xor((unsigned long long)vt, off);
          const double osc = __shfl_xor(vsc, off);
          bool take;
          if (os < 0) take = false;
          else if (vs < 0) take = true;
          else if (!gamma_policy) take = ot < vt;
          else take = osc < vsc || (osc == vsc && ot < vt);
          if (take) { vs = os; vt = ot; vsc = osc; }
        }
        s = vs;
        evicted = expert_in[s];
        const int vb = buf_of_slot[s];
        if (used[vb] == seq) {    // an earlier token of this call reads that buffer: leave it intact
          if (n_free == 0) { status = MOE_ERR_STAGING_EXHAUSTED; break; }
          buf = free_buf[n_free - 1];
          --n_free;
          if (lane == 0) zombie[n_zombie] = vb;
          ++n_zombie;
        } else {
          buf = vb;
        }
        ++n_evict;
      }
      if (lane == 0) {
        if (evicted >= 0) slot_of[evicted] = -1;
        expert_in[s] = e;
        slot_of[e] = s;
        buf_of_slot[s] = buf;
        filled[buf] = e + 1;
        if (n_miss < a.max_miss) a.miss_list[n_miss] = MissEntry{e, buf};
      }
      ++n_miss;
    }
    ++clock;
    if (lane == 0) {
      tick[s] = (uint64_t)clock;
      used[buf] = seq;
      pending[e] = 1;
      if (a.mode == 0) {
        pair_buf[(size_t)b * KS + k] = buf;
        if (trace_n + trace_added < a.trace_cap)
          st.trace[trace_n + trace_added] = moe_trace_rec_t{a.row0 + b, e, hit ? 1 : 0, evicted};
      }
    }
    if (a.mode == 0) ++trace_added;
    wave_sync();
    // Definition C.1: the discounted counts advance once per token (each pinned expert is a token)
    if (gamma_policy && (a.mode == 1 || k == K - 1)) {
      for (int x = lane; x < E; x += kWave) {
        score[x] = __dadd_rn(__dmul_rn(a.gamma, score[x]), (double)pending[x]);
        pending[x] = 0;
      }
      wave_sync();
    }
  }
  int n_groups = 0;
  if (status == MOE_OK && a.mode == 0) {
    n_groups = group_pairs_lds(count, start, filled, pair_buf, t, a);
  }
  if (a.mode == 0) {
    if (lane == 0) *t.n_groups = n_groups;
    write_work_list(t, a, n_groups);
  }

  if (status == MOE_OK) {
    // ---- commit ----
    wave_sync();
    for (int s = lane; s < C; s += kWave) {
      st.tick[s] = tick[s]; st.expert_in[s] = expert_in[s]; st.buf_of_slot[s] = buf_of_slot[s];
    }
    if (gamma_policy)
      for (int e = lane; e < E; e += kWave) st.score[e] = score[e];
    for (int i = lane; i < n_free; i += kWave) st.free_buf[i] = free_buf[i];
    for (int i = lane; i < n_zombie; i += kWave) st.zombie[i] = zombie[i];
    for (int i = lane; i < P; i += kWave) st.used_stamp[i] = used[i];
    if (lane == 0) {
      st.scalars[SC_CLOCK] = clock;
      st.scalars[SC_NRES] = n_res;
      st.scalars[SC_NFREE] = n_free;
      st.scalars[SC_NZOMBIE] = n_zombie;
      st.scalars[SC_CALLSEQ] = seq;
      st.scalars[SC_TRACE_N] = trace_n + trace_added;
    }
  }
  if (lane == 0) publish_record(a.mailbox, status, n_miss, n_evict, n_groups, n_hits, n_res, seq);
}

// Runs in ONE wave.  idx_src: the experts to look up, in order (decode: [B][K]; pin: the list);
// pair_buf: scratch [B*KS] (LDS or global), used when the call has more than 64 pairs.
__device__ __forceinline__ void cache_phase_fast(FastTable f, unsigned char* smem, const LdsLayout& L, const int32_t* idx_src,
                                 int32_t* pair_buf, const LayerState& st, const CallTables& t,
                                 const CacheCallArgs& a) {
  const int lane = threadIdx.x & 63;
  const int C = a.C, P = a.P, K = a.K, KS = a.KS;
  // LDS scratch (the table itself lives in registers on this path)
  int32_t* lds_slot_of = reinterpret_cast<int32_t*>(smem + L.slot_of);     // [E] expert -> slot
  int32_t* lds_last = reinterpret_cast<int32_t*>(smem + L.free_buf);       // [P >= C] last lookup of a slot, +1
  int32_t* lds_touch = reinterpret_cast<int32_t*>(smem + L.zombie);        // [P] buffer read by the chunk
  int32_t* lds_filled = reinterpret_cast<int32_t*>(smem + L.filled);       // [P]
  int32_t* lds_count = reinterpret_cast<int32_t*>(smem + L.count);         // [P + n_shared]
  int32_t* lds_cursor = reinterpret_cast<int32_t*>(smem + L.start);        // [P + n_shared]
  // buffers released by the previous call: all its kernels have finished, reuse them
  {
    const int src = lane - f.n_free;
    const int z = __shfl(f.zomb, src < 0 ? 0 : src);
    if (src >= 0 && src < f.n_zombie) f.free_b = z;
    f.n_free += f.n_zombie;
    f.n_zombie = 0;
  }
  const uint32_t seq = a.seq;
  const int n_lookups = a.mode == 0 ? a.B * K : K;
  const int NP = a.B * KS;
  const bool small = NP <= kWave;     // all pairs fit one per lane
  int status = MOE_OK, n_miss = 0, n_evict = 0, n_hits = 0;
  int my_pair = -1;       // small calls: lane p = b*KS + k holds the buffer the pair reads
  int filled = 0;         // lane p: expert + 1 that this call brings into buffer p, 0 if none

  // ---- shortcut for a call whose lookups all hit (the resident regime): residency does not change, and the
  //      recency updates commute - the last lookup of a slot decides its tick.  Lookups run 64 per step. ----
  bool all_hit = false;
  if (a.mode == 0 && f.n_res > 0 && n_lookups >= 16) {     // a handful of lookups takes the register variant below
    for (int e = lane; e < a.E; e += kWave) lds_slot_of[e] = -1;
    if (lane < P) { lds_last[lane] = 0; lds_touch[lane] = 0; }
    wave_sync();
    if (lane < C && f.exp >= 0) lds_slot_of[f.exp] = lane;
    wave_sync();
    uint64_t any_miss = 0;
    for (int chunk0 = 0; chunk0 < n_lookups; chunk0 += kWave) {
      const bool valid = chunk0 + lane < n_lookups;
      any_miss |= __ballot(valid && lds_slot_of[idx_src[chunk0 + lane]] < 0);
    }
    all_hit = any_miss == 0;
  }
  // the same shortcut for a handful of lookups (one per lane), entirely in registers: nothing is changed
  // unless every lookup hits
  if (a.mode == 0 && f.n_res > 0 && n_lookups < 16 && small) {
    const int my_e = lane < n_lookups ? idx_src[lane] : -3;
    int my_slot = 0;
    uint64_t new_tick = f.tick;
    bool ok = true;
    for (int q = 0; q < n_lookups; ++q) {       // uniform
      const uint64_t hm = __ballot(f.exp == readlane_i(my_e, q));
      if (hm == 0) { ok = false; break; }
      const int s = __ffsll((unsigned long long)hm) - 1;
      if (lane == q) my_slot = s;
      if (lane == s) new_tick = (uint64_t)(f.clock + q + 1);    // the last lookup of a slot decides its tick
    }
    if (ok) {
      f.tick = new_tick;
      const int my_buf = __shfl(f.buf, my_slot);                // lane q: buffer that lookup q reads
      for (int q = 0; q < n_lookups; ++q)
        if (lane == readlane_i(my_buf, q)) f.used = seq;
      if (lane < n_lookups && f.trace_n + lane < a.trace_cap)
        st.trace[f.trace_n + lane] = moe_trace_rec_t{a.row0 + lane / K, my_e, 1, -1};
      const int b = lane / KS, k = lane - b * KS;
      const int v = __shfl(my_buf, k < K ? b * K + k : 0);
      if (lane < NP && k < K) my_pair = v;
      f.clock += n_lookups;
      n_hits = n_lookups;
      all_hit = true;
    }
  } else if (all_hit) {
    for (int chunk0 = 0; chunk0 < n_lookups; chunk0 += kWave) {
      const int l = chunk0 + lane;
      const bool valid = l < n_lookups;
      const int my_e = valid ? idx_src[l] : 0;
      const int my_slot = valid ? lds_slot_of[my_e] : 0;
      if (valid) atomicMax(&lds_last[my_slot], l + 1);
      const int my_buf = __shfl(f.buf, my_slot);
      if (valid && f.trace_n + l < a.trace_cap) st.trace[f.trace_n + l] = moe_trace_rec_t{a.row0 + l / K, my_e, 1, -1};
      if (small) {
        // lane p = b*KS + k takes the buffer of lookup b*K + k (a single step)
        const int b = lane / KS, k = lane - b * KS;
        const int v = __shfl(my_buf, k < K ? b * K + k : 0);
        if (lane < NP && k < K) my_pair = v;
      } else if (valid) {
        const int b = l / K;
        pair_buf[(size_t)b * KS + (l - b * K)] = my_buf;
      }
    }
    wave_sync();
    const int last = lane < C ? lds_last[lane] : 0;
    if (last > 0) {
      f.tick = (uint64_t)(f.clock + last);
      lds_touch[f.buf] = 1;
    }
    wave_sync();
    if (lane < P && lds_touch[lane]) f.used = seq;
    f.clock += n_lookups;
    n_hits = n_lookups;
  }

  for (int chunk0 = 0; chunk0 < n_lookups && status == MOE_OK && !all_hit; chunk0 += kWave) {
    const int nl = min(kWave, n_lookups - chunk0);
    const int my_e = lane < nl ? idx_src[chunk0 + lane] : -3;
    int my_buf = -1;      // lane q: buffer that lookup chunk0 + q reads
    {
      for (int q = 0; q < nl; ++q) {
        const int e = readlane_i(my_e, q);
        const uint64_t hm = __ballot(f.exp == e);
        int s, buf, evicted = -1;
        const bool hit = hm != 0;
        if (hit) {
          s = __ffsll((unsigned long long)hm) - 1;
          buf = readlane_i(f.buf, s);
          ++n_hits;
        } else {
          if (f.n_res < C) {          // slots fill in index order, so the lowest empty slot is n_res
            s = f.n_res++;
            buf = readlane_i(f.free_b, --f.n_free);
          } else {
            s = wave_argmin_tick(f.tick);
            evicted = readlane_i(f.exp, s);
            const int vb = readlane_i(f.buf, s);
            if ((uint32_t)readlane_i((int)f.used, vb) == seq) {   // an earlier token of this call reads it
              if (f.n_free == 0) { status = MOE_ERR_STAGING_EXHAUSTED; break; }
              buf = readlane_i(f.free_b, --f.n_free);
              if (lane == f.n_zombie) f.zomb = vb;
              ++f.n_zombie;
            } else {
              buf = vb;
            }
            ++n_evict;
          }
          if (lane == s) { f.exp = e; f.buf = buf; }
          if (lane == buf) filled = e + 1;
          if (lane == 0 && n_miss < a.max_miss) a.miss_list[n_miss] = MissEntry{e, buf};
          ++n_miss;
        }
        ++f.clock;
        if (lane == s) f.tick = (uint64_t)f.clock;
        if (lane == buf) f.used = seq;
        if (lane == q) my_buf = buf;
        if (a.mode == 0 && lane == 0 && f.trace_n + chunk0 + q < a.trace_cap)
          st.trace[f.trace_n + chunk0 + q] = moe_trace_rec_t{a.row0 + (chunk0 + q) / K, e, hit ? 1 : 0, evicted};
      }
    }
    if (a.mode == 0 && status == MOE_OK) {
      if (small) {
        // lane p = b*KS + k takes the buffer of lookup b*K + k (a single chunk)
        const int b = lane / KS, k = lane - b * KS;
        const int v = __shfl(my_buf, k < K ? b * K + k : 0);
        if (lane < NP && k < K) my_pair = v;
      } else if (lane < nl) {
        const int l = chunk0 + lane, b = l / K;
        pair_buf[(size_t)b * KS + (l - b * K)] = my_buf;
      }
    }
  }

  int n_groups = 0;
  if (status == MOE_OK && a.mode == 0) {
    if (small) {
      // ---- group the pairs by buffer: rank every pair against all others (stable) ----
      {
        const int b = lane / KS, k = lane - b * KS;
        if (lane < NP && k >= K) my_pair = P + (k - K);     // shared experts
      }
      int rank = 0, same_before = 0, cnt = 0;
      for (int q = 0; q < NP; ++q) {
        const int bq = readlane_i(my_pair, q);
        rank += (bq < my_pair || (bq == my_pair && q < lane)) ? 1 : 0;
        cnt += bq == my_pair ? 1 : 0;
        same_before += (bq == my_pair && q < lane) ? 1 : 0;
      }
      const bool is_first = lane < NP && same_before == 0;
      const uint64_t fm = __ballot(is_first);
      int gidx = 0;
      for (uint64_t m = fm; m != 0; m &= m - 1) {
        const int q = __ffsll((unsigned long long)m) - 1;
        gidx += readlane_i(my_pair, q) < my_pair ? 1 : 0;
      }
      const int was_filled = __shfl(filled, my_pair < P && my_pair >= 0 ? my_pair : 0);
      if (lane < NP) {
        t.sorted_pair[rank] = lane;
        t.pos_of[lane] = rank;
        if (is_first) {
          GroupDesc gd;
          const int fe = my_pair < P ? was_filled : 0;
          gd.buf = my_pair; gd.begin = rank; gd.count = cnt; gd.miss = fe != 0;
          gd.pair0 = lane;      // stable order: the group's first pair is its lowest pair id
          gd.expert = fe - 1; gd.pad[0] = gd.pad[1] = 0;
          t.grp[gidx] = gd;
        }
      }
      n_groups = __popcll(fm);
    } else {
      // ---- more than 64 pairs: counting sort with the counters in LDS ----
      if (lane < P) lds_filled[lane] = filled;
      wave_sync();
      n_groups = group_pairs_lds(lds_count, lds_cursor, lds_filled, pair_buf, t, a);
    }
  }
  if (a.mode == 0) {
    if (lane == 0) *t.n_groups = n_groups;
    write_work_list(t, a, n_groups);
  }

  if (status == MOE_OK) {
    // ---- commit ----
    if (lane < C) { st.tick[lane] = f.tick; st.expert_in[lane] = f.exp; st.buf_of_slot[lane] = f.buf; }
    if (lane < P) { st.used_stamp[lane] = f.used; st.free_buf[lane] = f.free_b; st.zombie[lane] = f.zomb; }
    if (lane == 0) {
      st.scalars[SC_CLOCK] = f.clock;
      st.scalars[SC_NRES] = f.n_res;
      st.scalars[SC_NFREE] = f.n_free;
      st.scalars[SC_NZOMBIE] = f.n_zombie;
      st.scalars[SC_CALLSEQ] = seq;
      st.scalars[SC_TRACE_N] = f.trace_n + (a.mode == 0 ? n_lookups : 0);
    }
  }
  if (lane == 0) publish_record(a.mailbox, status, n_miss, n_evict, n_groups, n_hits, f.n_res, seq);
}

// One layer's table as loaded: lane i < SC_COUNT holds scalar i (turned into the uniform values of FastTable by
// `table_of`, once they are needed: the loads stay in flight while the logits are formed).
struct RawTable { int64_t sc; int exp, buf, free_b, zomb; uint64_t tick; uint32_t used; };

__device__ __forceinline__ RawTable raw_load(const LayerState& st, const CacheCallArgs& a) {
  const int lane = threadIdx.x & 63;
  RawTable f;
  if (a.resident) {       // a layer all of whose experts are in memory in the order of their ids: nothing to read
    f.sc = lane == SC_NRES ? a.E : 0;
    f.exp = f.buf = lane < a.E ? lane : -2;
    f.tick = 0; f.used = 0; f.free_b = f.zomb = -1;
    return f;
  }
  f.sc = lane < SC_COUNT ? st.scalars[lane] : 0;
  f.exp = lane < a.C ? st.expert_in[lane] : -2;
  f.tick = lane < a.C ? st.tick[lane] : ~0ull;
  f.buf = lane < a.C ? st.buf_of_slot[lane] : -1;
  f.used = lane < a.P ? st.used_stamp[lane] : 0u;
  f.free_b = lane < a.P ? st.free_buf[lane] : -1;
  f.zomb = lane < a.P ? st.zombie[lane] : -1;
  return f;
}

__device__ __forceinline__ FastTable table_of(const RawTable& r) {
  const auto scalar = [&](int i) {
    const uint32_t lo = (uint32_t)readlane_i((int)(uint32_t)r.sc, i);
    const uint32_t hi = (uint32_t)readlane_i((int)(uint32_t)((uint64_t)r.sc >> 32), i);
    return (int64_t)(((uint64_t)hi << 32) | lo);
  };
  FastTable f;
  f.clock = scalar(SC_CLOCK); f.trace_n = scalar(SC_TRACE_N);
  f.n_res = (int)scalar(SC_NRES); f.n_free = (int)scalar(SC_NFREE); f.n_zombie = (int)scalar(SC_NZOMBIE);
  f.exp = r.exp; f.buf = r.buf; f.free_b = r.free_b; f.zomb = r.zomb; f.tick = r.tick; f.used = r.used;
  return f;
}

// ---------------------------------------------------------------- the decode launch
// EB: router rows a wave handles at a time (1 when there are at least as many waves as experts: no spare loads).
// EPL: logits a lane holds while it gates (a kernel of its own for each: code that a launch jumps over costs it as well, 0.5 us
// with the selection for many experts beside the one for up to 64).
// MODES: the calls a kernel has code for.  What else is in it changes the scalar registers and the placement of the lookups' loop, so
// each form is the faster one of the two, us per call with lookups in order / prompt: 64 tokens on 64 experts (discounted counts)
// 295 with both, 282 apart, on 300 experts 165 / 159, 16 prompt tokens on 60 experts 21.9 / 20.9; but 1 token on 16 experts 17.9 / 18.7, 64 on
// 200 experts 171 / 175.
enum RouteModes { kDecodes, kPrompts, kBoth };
template <typename T, int EB, int EPL, RouteModes MODES>
__global__ void __launch_bounds__(1024) route_cache_kernel(RouteArgs r, LayerState st, CallTables t, CacheCallArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_last;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int n_waves = blockDim.x >> 6;
  const int b = blockIdx.x;
  const int E = a.E, K = a.K, KS = a.KS, d = r.d;
  const bool single = gridDim.x == 1;
  const bool prompt = MODES == kPrompts || (MODES == kBoth && a.mode == 2);
  const bool fast = !prompt && fast_table(a.policy, a.C, a.P, a.n_shared);

  // With one workgroup the cache table can be fetched while the router GEMV runs.
  RawTable raw{};
  if (single && fast && wave == 0) raw = raw_load(st, a);

  const LdsLayout L = lds_layout(E, a.C, a.P, a.n_shared, a.B, K, KS);
  float* zs = reinterpret_cast<float*>(smem + L.logit);
  const bool stage = stage_in_lds(a.B, KS);
  int32_t* idx_stage = stage ? reinterpret_cast<int32_t*>(smem + L.idx_stage) : nullptr;
  int32_t* pair_stage = stage ? reinterpret_cast<int32_t*>(smem + L.pair_stage) : t.pair_buf;

  // ---- phase 1: router rows of token b, EB rows per wave at a time ----
  {
    using V = Vec<T>;
    const int n_vec = d / V::N;  // host guarantees d % V::N == 0
    const typename V::type* xv = reinterpret_cast<const typename V::type*>(static_cast<const T*>(r.x) + (size_t)b * d);
    const typename V::type* wbase = reinterpret_cast<const typename V::type*>(r.router_w);
    for (int e0 = wave; e0 < E; e0 += n_waves * EB) {
      const typename V::type* wv[EB];
#pragma unroll
      for (int j = 0; j < EB; ++j) {
        const int e = e0 + j * n_waves;
        wv[j] = wbase + (size_t)(e < E ? e : E - 1) * n_vec;   // clamped: loads stay unconditional
      }
      float acc[EB];
#pragma unroll
      for (int j = 0; j < EB; ++j) acc[j] = 0.f;
      constexpr int CB = 4;   // chunks per lane fetched together: (1 + EB) * CB loads in flight
      for (int c0 = lane; c0 < n_vec; c0 += kWave * CB) {
        typename V::type xc[CB], wc[EB][CB];
#pragma unroll
        for (int i = 0; i < CB; ++i) {
          const int c = c0 + i * kWave;
          const int cc = c < n_vec ? c : n_vec - 1;     // clamped: in bounds, masked below
          xc[i] = xv[cc];
#pragma unroll
          for (int j = 0; j < EB; ++j) wc[j][i] = wv[j][cc];
        }
#pragma unroll
        for (int i = 0; i < CB; ++i) {
          if (c0 + i * kWave < n_vec) {
#pragma unroll
            for (int j = 0; j < EB; ++j) acc[j] = V::dot(wc[j][i], xc[i], acc[j]);
          }
        }
      }
#pragma unroll
      for (int j = 0; j < EB; ++j) {
        const int e = e0 + j * n_waves;
        const float s = wave_sum(acc[j]);
        if (lane == 0 && e < E) zs[e] = s + (r.bias ? r.bias[(size_t)b * E + e] : 0.f);
      }
    }
  }
  __syncthreads();

  // ---- phase 2: gating of token b by wave 0 ----
  if (wave != 0) return;
  gate_token<EPL, true, (EPL > 1)>(zs, b, E, K, KS, r.norm_topk, t.idx, t.wpair, r.user_idx, r.user_w, idx_stage);

  if (!single) {
    // ---- the last workgroup to arrive carries on (no waiting anywhere) ----
    // every lane publishes its own stores (routing results) before lane 0 announces the workgroup
    __threadfence();
    if (lane == 0) s_last = atomicAdd(r.arrive, 1) == (int)gridDim.x - 1;
    wave_sync();
    if (!s_last) return;
    if (lane == 0) __hip_atomic_store(r.arrive, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch on this stream
    __threadfence();
    // routing results of the other workgroups: read at device scope
    if (stage)
      for (int i = lane; i < a.B * K; i += kWave)
        idx_stage[i] = __hip_atomic_load(&t.idx[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (fast) raw = raw_load(st, a);
  }
  wave_sync();

  // ---- phase 3: cache lookups, one wave ----
  if (prompt) {
    if constexpr (MODES != kDecodes) prefill_phase(smem, L, stage ? idx_stage : t.idx, pair_stage, st, t, a);
  } else if constexpr (MODES != kPrompts) {
    if (fast) cache_phase_fast(table_of(raw), smem, L, stage ? idx_stage : t.idx, pair_stage, st, t, a);
    else cache_phase_general(smem, L, stage ? idx_stage : t.idx, pair_stage, st, t, a);
  }
}


// ---------------------------------------------------------------- several tokens per call
constexpr int kTileWaves = 16, kTileThreads = 64 * kTileWaves, kTileTokens = 16;
// Router products and bytes of an fp32 call of 2 to 8 tokens up to which one workgroup routes them all, instead of one per
// token that then meet (layer calls, 4 tokens: 8 experts of 64 columns 18.2 -> 16.9 us, 16 of 128 20.0 -> 18.6, 32 of 256
// 20.4 -> 19.8; 16 tokens x 8 experts 25.2 -> 26.7, 8 tokens x 64 experts of 512 columns 24.8 -> 28.0: not taken).
constexpr int kSmallRouterItems = 128;
constexpr size_t kSmallRouterBytes = 128 << 10;
constexpr int kRouteChains = 16;      // partial sums of a logit (route_units_kernel)
constexpr int kChunk = kTileThreads;  // tokens whose pairs are placed at a time, one per thread

// What the phases behind the logits keep in LDS.
struct TileLds {
  float zs[kTileTokens][kTileMaxE + 4];           // logits (+ 4: the 16 tokens of a column fall on different banks)
  uint64_t sel[kTileTokens];                      // experts each token of the tile selects (up to 64 experts)
  int map[kTileMaxE];                             // expert -> buffer << 8 | slot, -1 when it is not resident
  // A column of the grouping is an expert; of more than 64 experts the resident ones in ascending order have them (kWide)
  int col_expert[kWave], col_map[kWave];          // kWide: the column's expert and its entry of `map`
  // per wave of 64 tokens and column: the tokens that select it, how many, and the position of the first of them
  uint64_t col[kTileWaves][kWave];
  int cnt[kTileWaves][kWave], base[kTileWaves][kWave];
  int first_pair[kWave], last_lookup[kWave];      // ... column: its first pair, its last lookup + 1
  int first[kWave], touched[kWave], slot_last[kWave];
  int last_arrived, any_miss;
};

__device__ __forceinline__ void clear_tile_lds(TileLds& tl, int E) {
  const int tid = threadIdx.x;
  for (int e = tid; e < E; e += kTileThreads) tl.map[e] = -1;
  if (tid == 0) tl.any_miss = 0;
  if (tid < kWave) { tl.first[tid] = tl.last_lookup[tid] = tl.touched[tid] = 0; tl.first_pair[tid] = 1 << 30; }
}

__device__ __forceinline__ uint32_t load_published(const void* p) {
  return __hip_atomic_load(static_cast<const uint32_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Announce this workgroup at a counter once every wave's device-scope stores have arrived; true in the workgroup that
// comes last (nobody waits), which leaves the counter at zero for the next launch.
__device__ __forceinline__ bool arrive_last(int32_t* counter, int n, int& flag) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    const int last = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    if (last) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    flag = last;
  }
  __syncthreads();
  return flag != 0;
}

// Inclusive sum over the lanes of a wave, on the vector unit's own lane shifts (a scan through LDS takes ten times as long).
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
#define MOE_SCAN_STEP(CTRL, ROWS) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false)
  MOE_SCAN_STEP(0x111, 0xf);      // row_shr 1, 2, 4, 8: sums inside a row of 16 lanes
  MOE_SCAN_STEP(0x112, 0xf);
  MOE_SCAN_STEP(0x114, 0xf);
  MOE_SCAN_STEP(0x118, 0xf);
  MOE_SCAN_STEP(0x142, 0xa);      // lane 15 of a row into the next, rows 1 and 3
  MOE_SCAN_STEP(0x143, 0xc);      // lane 31 into rows 2 and 3
#undef MOE_SCAN_STEP
  return v;
}

// Pairs of a call that are put in order in LDS before they are written out.  At the least of them that is neither here nor there, with few
// pairs per token it never pays; the most are what a unit's 160 KB hold beside the kernel's own.  Layer calls, in LDS / scattered:
// 8 each of 64 experts, 256 / 1024 / 2048 / 8192 pairs 20.6 / 23.2 / 25.6 / 39.3 and 20.3 / 23.1 / 26.1 / 42.6 us, with a shared expert, 9216 /
// 12285 pairs, 41.8 / 53.5 and 43.7 / 55.7; 4 each 1024 / 4096 pairs 23.2 / 32.6 and 23.1 / 33.2; 2 each of 16 2048 pairs 25.9 and 25.7.
constexpr int kStagedLeast = 1024, kStagedMost = 12288;
__host__ __device__ inline bool stage_pairs(int B, int KS) { return B * KS >= kStagedLeast && B * KS <= kStagedMost; }

// The 64 x 64 bit matrix whose row r lane r holds, transposed: lane c gets column c.
__device__ __forceinline__ uint64_t transpose_bits(uint64_t x) {
  const int lane = threadIdx.x & 63;
  constexpr uint64_t kLow[6] = {0x5555555555555555ull, 0x3333333333333333ull, 0x0f0f0f0f0f0f0f0full, 0x00ff00ff00ff00ffull,
                                0x0000ffff0000ffffull, 0x00000000ffffffffull};
#pragma unroll
  for (int i = 5; i >= 0; --i) {
    const int j = 1 << i;
    const uint64_t y = __shfl_xor((unsigned long long)x, j);
    x = (lane & j) ? (x & ~kLow[i]) | ((y >> j) & kLow[i]) : (x & kLow[i]) | ((y & kLow[i]) << j);
  }
  return x;
}

// One kernel per kind of call: code that a launch only jumps over is fetched cold with the rest, and its registers spill the others'.
//   kFull    mode 0, at most 64 experts and slots, every expert known to be resident: no lookup can miss, so no buffer is taken or
//            released and the size of the buffer tables (spare ones) does not matter
//   kScored  the same under the discounted-count policy
//   kTable   mode 0 on the register table, up to 64 experts
//   kWide    mode 0 on the register table, 65 to 256 experts
//   kOther   mode 0 on other tables: one wave looks up in order
//   kPrompt  mode 2: prompt streaming
enum RouteKind { kFull, kScored, kTable, kWide, kOther, kPrompt };
template <RouteKind KIND> constexpr bool kHits = KIND == kFull || KIND == kScored;      // no lookup can miss
template <RouteKind KIND> constexpr bool kColumns = KIND < kOther;       // selections travel as masks of columns
template <RouteKind KIND> constexpr bool kMany = KIND >= kWide;          // more than 64 logits of a token

// Phase 3 of kFull to kWide, run by ALL waves of the last workgroup.  The common case -
// every lookup hits - is embarrassingly parallel: residency does not change, and the place of a pair in its group is the number
// of earlier tokens that select the same expert.  A wave holds the selections of 64 tokens as one mask per lane; transposed, lane
// e has the tokens of column e, and counts, prefix sums and the order of the groups are a few instructions in every wave alike.
// Nothing is drawn from a shared counter: with 8192 ranks from LDS atomics this phase took 12 us of a launch.
// False, with nothing changed, when a lookup misses.  kWide: there are at most 64 slots, so the resident experts have a column each,
// and a token whose mask holds fewer than K of them misses.  (Calls that hit, 112 /
// 1024 tokens with 6 each of 128 experts on 60 slots, grouped by one wave 94.7 / 657 us, here 89.0 / 550.)
// masks: the published selections, null: tl.sel.  behind: work of the caller that the first loads leave time for.
template <RouteKind KIND, typename Behind>
__device__ __forceinline__ bool group_hits(unsigned char* smem, TileLds& tl, const RawTable& raw, const uint64_t* masks,
                                           const LayerState& st, const CallTables& t, const CacheCallArgs& a, Behind behind) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int E = a.E, C = a.C, P = a.P, K = a.K, KS = a.KS, ns = a.n_shared, B = a.B;
  const auto mask_of = [&](int b) -> uint64_t {
    if (b >= B) return 0;
    return masks ? __hip_atomic_load(masks + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : tl.sel[b];
  };
  uint64_t mine = mask_of(tid), ahead = mask_of(kChunk + tid);       // (of the next chunk: requested a chunk before its use)
  const uint64_t mine0 = mine;
  behind();
  if constexpr (!kHits<KIND>) {
    if constexpr (KIND == kWide) {
      bool misses = tid < B && __popcll(mine) != K;
      for (int b = kChunk + tid; b < B; b += kChunk) misses |= __popcll(mask_of(b)) != K;
      if (misses) tl.any_miss = 1;
    } else {
      const uint64_t resident = __ballot(lane < E && tl.map[lane] >= 0);
      uint64_t wanted = mine;
      for (int b = kChunk + tid; b < B; b += kChunk) wanted |= mask_of(b);
      if ((wanted & ~resident) != 0) tl.any_miss = 1;
    }
    __syncthreads();
    if (tl.any_miss) return false;
  }
  // lane e of every wave: the tokens of column e in a chunk of 1024, in all of its waves and in those before this one
  const bool ends = !a.resident || a.work.cap == 0;
  int in_chunk, before;
  const auto count_chunk = [&](int c0) {
    if (c0 + wave * kWave < B) {
      const uint64_t col = transpose_bits(mine);
      tl.col[wave][lane] = col;
      tl.cnt[wave][lane] = __popcll(col);
      // the column's first pair (for the kernels that go by groups) and last lookup (recency)
      const uint64_t lower = (1ull << lane) - 1ull;
      if (ends) {
        const int b0 = __ffsll((unsigned long long)col) - 1, b1 = 63 - __clzll(col | 1);
        const int k0 = __popcll(__shfl((unsigned long long)mine, b0 & 63) & lower), k1 = __popcll(__shfl((unsigned long long)mine, b1) & lower);
        if (col != 0) {
          atomicMin(&tl.first_pair[lane], (c0 + wave * kWave + b0) * KS + k0);
          atomicMax(&tl.last_lookup[lane], (c0 + wave * kWave + b1) * K + k1 + 1);
        }
      }
    }
    __syncthreads();
    in_chunk = before = 0;
    const int n = min(kTileWaves, (B - c0 + kWave - 1) / kWave);
    for (int w = 0; w < n; ++w) {
      const int c = tl.cnt[w][lane];
      in_chunk += c;
      before += w < wave ? c : 0;
    }
  };
  count_chunk(0);
  int total = in_chunk;
  for (int c0 = kChunk; c0 < B; c0 += kChunk) {
    mine = ahead;
    ahead = mask_of(c0 + kChunk + tid);
    __syncthreads();
    count_chunk(c0);
    total += in_chunk;
  }
  const int v = KIND == kWide ? tl.col_map[lane] : lane < E ? tl.map[lane] : -1;
  const int begin = (int)wave_scan((uint32_t)total) - total;
  const uint64_t used = __ballot(total > 0);
  const int group = __popcll(used & ((1ull << lane) - 1ull)), n_routed = __popcll(used);
  const int tiles = a.work.cap > 0 ? tiles_of(total, a.work) : 0;
  const int shared_tiles = a.work.cap > 0 ? tiles_of(B, a.work) : 0;
  if (a.work.cap > 0) {
    // work list, groups with the most tokens first (the shared experts': every token), ties by id: a wave compares with four experts
    int larger = 0;
#pragma unroll
    for (int i = 0; i < kWave / kTileWaves; ++i) {
      const int j = wave * (kWave / kTileWaves) + i, cj = readlane_i(total, j);
      larger += cj > total || (cj == total && j < lane) ? tiles_of(cj, a.work) : 0;
    }
    atomicAdd(&tl.first[lane], larger);
  }
  __syncthreads();
  if (wave == kTileWaves - 1) {
    if (total > 0) {
      GroupDesc* gd = &t.grp[group];
      *reinterpret_cast<int4*>(gd) = int4{v >> 8, begin, total, 0};
      *reinterpret_cast<int2*>(&gd->pair0) = int2{tl.first_pair[lane], -1};
      int4* items = t.work + 1 + ns * shared_tiles + tl.first[lane];
      for (int i = 0; i < tiles; ++i) items[i] = work_item(i << a.work.shift, v >> 8, begin, total, 0);
    }
    if (lane < ns) {
      const int first = B * K + lane * B;
      t.grp[n_routed + lane] = GroupDesc{P + lane, first, B, 0, K + lane, -1, {0, 0}};
      for (int i = 0; i < shared_tiles; ++i) t.work[1 + lane * shared_tiles + i] = work_item(i << a.work.shift, P + lane, first, B, 0);
    }
    const int n_items = readlane_i((int)wave_scan((uint32_t)tiles), kWave - 1) + ns * shared_tiles;
    if (lane == 0) {
      *t.n_groups = n_routed + ns;
      if (a.work.cap > 0) t.work[0] = int4{n_items, 0, 0, 0};
    }
  }
  const auto place = [&](int32_t* sorted, int32_t* pos_of) {
    int run = 0;               // the column's pairs in the chunks before
    for (int c0 = 0; c0 < B; c0 += kChunk) {
      if (B > kChunk) {        // more than 1024 tokens: chunk by chunk once more
        __syncthreads();
        mine = c0 == 0 ? mine0 : ahead;
        ahead = mask_of(c0 + kChunk + tid);
        count_chunk(c0);
      }
      if (c0 + wave * kWave < B) {
        tl.base[wave][lane] = begin + before + run;
        wave_sync();
        const int b = c0 + tid;
        const uint64_t lt_mask = (1ull << lane) - 1ull;
        uint64_t m = mine;                             // (K bits; none beyond the call's tokens)
        int p = b * KS;
        constexpr int U = 4;                           // pairs whose reads are in flight together
        for (int k0 = 0; k0 < K; k0 += U) {
          int e[U], pos[U];
          uint64_t col[U];
          bool there[U];
  #pragma unroll
          for (int u = 0; u < U; ++u) {
            there[u] = m != 0;
            e[u] = (__ffsll((unsigned long long)m) - 1) & 63;
            m &= m - 1;
            col[u] = tl.col[wave][e[u]];
            pos[u] = tl.base[wave][e[u]];
          }
  #pragma unroll
          for (int u = 0; u < U; ++u) {
            if (there[u]) {
              pos[u] += __popcll(col[u] & lt_mask);
              sorted[pos[u]] = p + u;
              pos_of[p + u] = pos[u];
            }
          }
          p += U;
        }
      }
      run += in_chunk;
    }
    for (int i = tid; i < B * ns; i += kTileThreads) {
      const int b = i / ns, sidx = i - b * ns, p = b * KS + K + sidx, pos = B * K + sidx * B + b;
      sorted[pos] = p;
      pos_of[p] = pos;
    }
  };
  if (a.trace_cap > 0) {
    const int64_t trace_n = st.scalars[SC_TRACE_N];
    for (int b = tid; b < B; b += kTileThreads) {
      uint64_t m = mask_of(b);
      for (int l = b * K; m != 0; ++l, m &= m - 1) {
        const int c = __ffsll((unsigned long long)m) - 1;
        if (trace_n + l < a.trace_cap) st.trace[trace_n + l] = moe_trace_rec_t{a.row0 + b, KIND == kWide ? tl.col_expert[c] : c, 1, -1};
      }
    }
  }
  // a scattered store takes the address unit a cycle per lane: many pairs are put in order in LDS
  const bool staged = stage_pairs(B, KS);
  if (!staged) {
    place(t.sorted_pair, t.pos_of);
    if (a.resident) return true;
    __syncthreads();
  } else {
    const int n = B * KS;
    int32_t *sorted = reinterpret_cast<int32_t*>(smem), *pos_of = sorted + (n + 3) / 4 * 4;
    place(sorted, pos_of);
    __syncthreads();
    for (int i = tid * 4; i < n; i += kTileThreads * 4) {        // (the tables are whole multiples of 16 bytes long)
      *reinterpret_cast<int4*>(t.sorted_pair + i) = *reinterpret_cast<const int4*>(sorted + i);
      *reinterpret_cast<int4*>(t.pos_of + i) = *reinterpret_cast<const int4*>(pos_of + i);
    }
  }
  if (a.resident || wave != 0) return true;
  // ---- the table after the call: recency of the slots, buffers in use, released buffers free again ----
  FastTable f = table_of(raw);
  if constexpr (KIND == kWide) {
    if (v >= 0) tl.slot_last[v & 255] = tl.last_lookup[lane];
    wave_sync();
  }
  const int last = lane < C && f.exp >= 0 ? (KIND == kWide ? tl.slot_last[lane] : tl.last_lookup[f.exp]) : 0;
  if (last > 0) {
    f.tick = (uint64_t)(f.clock + last);
    if constexpr (!kHits<KIND>) tl.touched[f.buf] = 1;
  }
  if (lane < C) { st.tick[lane] = f.tick; st.expert_in[lane] = f.exp; st.buf_of_slot[lane] = f.buf; }
  if constexpr (!kHits<KIND>) {     // (where no lookup can miss, no buffer was ever released and nobody asks for the use stamps)
    wave_sync();
    if (lane < P && tl.touched[lane]) f.used = a.seq;
    const int src = lane - f.n_free;
    const int z = __shfl(f.zomb, src < 0 ? 0 : src);
    if (src >= 0 && src < f.n_zombie) f.free_b = z;
    if (lane < P) { st.used_stamp[lane] = f.used; st.free_buf[lane] = f.free_b; st.zombie[lane] = f.zomb; }
    if (lane == 0) {
      st.scalars[SC_NFREE] = f.n_free + f.n_zombie;
      st.scalars[SC_NZOMBIE] = 0;
    }
  }
  if constexpr (KIND == kScored) {       // Definition C.1: the discounted counts advance once per token
    double score = lane < E ? st.score[lane] : 0.0;
    for (int b0 = 0; b0 < B; b0 += kWave) {
      const uint64_t m = mask_of(b0 + lane);
      const int n = min(kWave, B - b0);
      for (int j = 0; j < n; ++j) {
        const uint32_t lo = (uint32_t)readlane_i((int)(uint32_t)m, j), hi = (uint32_t)readlane_i((int)(uint32_t)(m >> 32), j);
        const uint32_t wanted = (lane < 32 ? lo >> lane : hi >> (lane - 32)) & 1u;
        score = __dadd_rn(__dmul_rn(a.gamma, score), (double)wanted);
      }
    }
    if (lane < E) st.score[lane] = score;
  }
  if (lane == 0) {
    st.scalars[SC_CLOCK] = f.clock + B * K;
    st.scalars[SC_NRES] = f.n_res;
    st.scalars[SC_CALLSEQ] = a.seq;
    st.scalars[SC_TRACE_N] = f.trace_n + B * K;
    publish_record(a.mailbox, MOE_OK, 0, 0, n_routed + ns, B * K, f.n_res, a.seq);
  }
  return true;
}

// Phases 2 and 3 from the logits of a tile of 16 tokens (tl.zs), by the sixteen waves of one workgroup per tile: a wave selects a
// token's experts, and the last workgroup of the launch goes on to the lookups.  What the others must see of a workgroup - its
// selections - goes past the caches with device-scope stores, so the arrival needs no cache write-back; the gate weights, which
// no one in this launch reads, are formed behind it.
template <RouteKind KIND>
__device__ __forceinline__ void gate_and_group(unsigned char* smem, TileLds& tl, const RawTable& raw, int tile, int n_tiles,
                                               const RouteArgs& r, uint64_t* masks, const LayerState& st, const CallTables& t, const CacheCallArgs& a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int E = a.E, K = a.K, KS = a.KS, b = tile * kTileTokens + wave;
  const bool single = n_tiles == 1, mine = b < a.B;
  if (kColumns<KIND> && wave == 0 && lane < a.C && raw.exp >= 0) tl.map[raw.exp] = raw.buf << 8 | lane;
  if constexpr (KIND == kWide) {
    if (wave == 0) {
      wave_sync();
      int n_cols = 0;
#pragma unroll
      for (int i = 0; i < kTileMaxE / kWave; ++i) {
        const int e = lane + i * kWave, m = e < E ? tl.map[e] : -1;
        const uint64_t there = __ballot(m >= 0);
        const int c = n_cols + __popcll(there & ((1ull << lane) - 1ull));
        if (m >= 0) { tl.col_expert[c] = e; tl.col_map[c] = m; }      // (no more than there are slots)
        n_cols += __popcll(there);
      }
      if (lane >= n_cols) { tl.col_expert[lane] = 0; tl.col_map[lane] = -1; }
    }
    __syncthreads();
  }
  const LdsLayout L = lds_layout(E, a.C, a.P, a.n_shared, a.B, K, KS);
  int32_t* idx_stage = !kHits<KIND> && stage_in_lds(a.B, KS) ? reinterpret_cast<int32_t*>(smem + L.idx_stage) : nullptr;
  constexpr int EPL = kMany<KIND> ? kTileMaxE / kWave : 1;
  Gate<1> g1;
  Gate<EPL> g4;
  const bool few = !kMany<KIND> || (!kColumns<KIND> && E <= kWave);
  const auto publish = [&](uint64_t columns) {
    if (lane != 0) return;
    if (single) tl.sel[wave] = columns;
    else __hip_atomic_store(masks + b, columns, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if (mine) {
    if (few) {
      select_experts<1>(tl.zs[wave], E, K, g1);
      if constexpr (kColumns<KIND>) publish(g1.top[0]);
      if constexpr (!kHits<KIND>) write_selected<1>(g1, b, K, t.idx, single ? idx_stage : nullptr);
    } else {
      select_experts<EPL>(tl.zs[wave], E, K, g4);
      if constexpr (KIND == kWide) {
        const int e = tl.col_expert[lane];
        uint64_t word = g4.top[0];
#pragma unroll
        for (int i = 1; i < EPL; ++i) word = e >> 6 == i ? g4.top[i] : word;
        publish(__ballot(tl.col_map[lane] >= 0 && ((word >> (e & 63)) & 1) != 0));
      }
      write_selected<EPL>(g4, b, K, t.idx, single ? idx_stage : nullptr);
    }
  }
  const auto weights = [&] {
    if (!mine) return;
    const auto ids = [&](size_t pos, int e) { if (r.user_idx) r.user_idx[pos] = e; };
    if (few) write_weights<1>(g1, b, E, K, KS, r.norm_topk, t.wpair, r.user_w, ids);
    else write_weights<EPL>(g4, b, E, K, KS, r.norm_topk, t.wpair, r.user_w, ids);
  };
  if (single) {
    __syncthreads();
  } else if (!arrive_last(r.arrive, n_tiles, tl.last_arrived)) {
    weights();
    return;
  }
  if constexpr (kColumns<KIND>) {
    // the weights fill the time that the others' selections take to arrive; with nothing to wait for they come last
    const bool hits = group_hits<KIND>(smem, tl, raw, single ? nullptr : masks, st, t, a, [&] { if (!single) weights(); });
    if (hits) {
      if (single) weights();
      return;
    }
  }
  if constexpr (!kHits<KIND>) {
    // in order, one wave; the others have the weights of their tokens to form where that is not done
    if (!single && idx_stage)
      for (int i = tid; i < a.B * K; i += kTileThreads) idx_stage[i] = (int)load_published(t.idx + i);
    __syncthreads();
    if (single || !kColumns<KIND>) weights();
    if (wave != 0) return;
    if (!idx_stage) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");     // reads the other workgroups' results directly
    const int32_t* in_order = idx_stage ? idx_stage : t.idx;
    int32_t* pair_stage = idx_stage ? reinterpret_cast<int32_t*>(smem + L.pair_stage) : t.pair_buf;
    if constexpr (kColumns<KIND>) cache_phase_fast(table_of(raw), smem, L, in_order, pair_stage, st, t, a);
    else if constexpr (KIND == kPrompt) prefill_phase(smem, L, in_order, pair_stage, st, t, a);
    else cache_phase_general(smem, L, in_order, pair_stage, st, t, a);
  }
}

// Calls of two and more bf16 tokens.  The router logits are a matrix product (experts x tokens) on the matrix cores: rows of W_r
// are the A operand, the tokens the B operand of v_mfma_f32_16x16x32_bf16.  A workgroup forms 16 experts x 16 tokens over one
// slice of the contraction (a unit), every load of a wave in flight at once; its waves' partial tiles meet in LDS, units publish
// theirs past the caches, and the one that arrives last of its token tile gates (gate_and_group).
// A logit is the sum of sixteen chains: chain c takes the pairs of k-blocks c, c + 16, c + 32 ..., and the sums of chains c and c + 8
// are added up from c = 0.  One wave forms a chain, in whichever slice it lies, so neither the batch nor the number of slices
// that it calls for changes a bit of a token's logits.
// What bounds it is the chain of round trips - first touch after the launch, publication, arrival, gating, arrival, grouping -
// and, with whole tiles of 64 experts in one workgroup, the 320 KB that one compute unit had to pull in: row-major
// fragments are 16 pieces of 64 bytes each, and the address unit sets the pace.
// PACKED: W_r comes from the library's copy in operand order (pack_router_kernel), for the calls of 2 to 4 tokens that may
// read it.  PAIRS: pairs of k-blocks a wave requests at a time.  SLICED: several slices, one expert tile per unit; else the whole
// contraction and one tile or several (a kernel for each: with both in one a call of one unit takes 0.5 us more).
template <int PAIRS, bool PACKED, RouteKind KIND, bool SLICED>
__global__ void __launch_bounds__(kTileThreads) route_units_kernel(RouteArgs r, RouteWork rw, LayerState st, CallTables t, CacheCallArgs a) {
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  extern __shared__ __align__(16) unsigned char smem[];     // partial tiles of the logits, then phase 3's scratch
  __shared__ TileLds tl;
  float* pz = reinterpret_cast<float*>(smem);               // [2 half][256]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, q = lane >> 4;
  const int E = a.E, d = r.d;
  const int n_et = (E + 15) >> 4, n_eu = SLICED ? n_et : (n_et + rw.et_per - 1) / rw.et_per;
  const int slices = SLICED ? rw.slices : 1, units = n_eu * slices;
  const int n_tiles = (a.B + kTileTokens - 1) / kTileTokens;
  const int tile = blockIdx.x / units, u = blockIdx.x - tile * units;
  const int sl = SLICED ? u / n_eu : 0;
  const int et0 = SLICED ? u - sl * n_eu : u * rw.et_per, et1 = SLICED ? et0 + 1 : min(et0 + rw.et_per, n_et);      // expert tiles et0 to et1 - 1
  const int t0 = tile * kTileTokens;
  const int nkb = d >> 5;
  const int tok = t0 + n < a.B ? t0 + n : a.B - 1;          // clamped: in bounds, the column is dropped below
  const u32x4* xrow = reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(r.x) + (size_t)tok * d) + q;
  constexpr int w_step = PACKED ? 64 : 4;                   // (16-byte pieces between k-blocks)
  // the slice's chains: sl * half ... and the same + 8
  const int half = kRouteChains / 2 / slices;
  const int chain = sl * half + (wave < half ? wave : wave - half + kRouteChains / 2);
  const auto form_chain = [&](int et) {
    if (SLICED && wave >= 2 * half) return;
    const u32x4* wrow = PACKED ? static_cast<const u32x4*>(r.router_packed) + (size_t)et * nkb * 64 + lane
                               : reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(r.router_w) + (size_t)min(et * 16 + n, E - 1) * d) + q;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int kb0 = 2 * chain; kb0 < nkb; kb0 += 2 * PAIRS * kRouteChains) {
      u32x4 xb[2 * PAIRS], wa[2 * PAIRS];
#pragma unroll
      for (int i = 0; i < 2 * PAIRS; ++i) {
        const int kb = min(kb0 + (i >> 1) * 2 * kRouteChains + (i & 1), nkb - 1);
        xb[i] = xrow[(size_t)kb * 4];
        wa[i] = wrow[(size_t)kb * w_step];
      }
#pragma unroll
      for (int i = 0; i < 2 * PAIRS; ++i)
        if (kb0 + (i >> 1) * 2 * kRouteChains + (i & 1) < nkb)      // uniform
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa[i]), __builtin_bit_cast(bf16x8, xb[i]), acc, 0, 0, 0);
    }
    *reinterpret_cast<f32x4*>(pz + wave * 256 + lane * 4) = acc;
  };
  form_chain(et0);
  // nobody changes the table before the last workgroup of this launch does: every workgroup may fetch it now
  RawTable raw{};
  if (kColumns<KIND> && wave == 0) raw = raw_load(st, a);
  // element el = tid % 256 of expert tile tid / 256 + 4 j: the MFMA leaves rows 4 (ln / 16) + el % 4, token ln % 16 with ln = el / 4
  const int el = tid & 255, el_tok = (el >> 2) & 15, el_row = (el >> 6) * 4 + (el & 3);
  constexpr int NJ = kMany<KIND> ? kTileMaxE / 16 / (kTileThreads / 256) : 1;
  float bias[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int e = ((tid >> 8) + j * (kTileThreads / 256)) * 16 + el_row;
    bias[j] = (r.bias && e < E && t0 + el_tok < a.B) ? r.bias[(size_t)(t0 + el_tok) * E + e] : 0.f;
  }
  clear_tile_lds(tl, E);
  __syncthreads();
  const auto pair_sum = [&](int c) { return pz[c * 256 + el] + pz[(c + half) * 256 + el]; };
  // published: a unit's logits, or its pair sums [expert tile][8][256] where other units have the others
  constexpr int parts = SLICED ? kRouteChains / 2 : 1;
  float* zt = rw.logits + (size_t)tile * n_et * parts * 256;
  const auto store = [&](int row, float z) {
    __hip_atomic_store(zt + (size_t)row * 256 + tid, z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  if constexpr (SLICED) {
    if (tid < half * 256) store(et0 * parts + sl * half, pair_sum(tid >> 8));
  } else {
    for (int et = et0;; ++et) {
      if (tid < 256) {
        float z = pair_sum(0);
#pragma unroll
        for (int c = 1; c < kRouteChains / 2; ++c) z += pair_sum(c);
        const int e = et * 16 + el_row;
        if (units > 1) store(et, z);
        else if (e < E) tl.zs[el_tok][e] = n_et == 1 ? z + bias[0] : z;
      }
      if (et + 1 == et1) break;
      __syncthreads();
      form_chain(et + 1);
      __syncthreads();
    }
  }
  if (!SLICED && units == 1) {
    if (n_et > 1) {
      __syncthreads();
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int e = ((tid >> 8) + j * (kTileThreads / 256)) * 16 + el_row;
        if (e < E) tl.zs[el_tok][e] += bias[j];
      }
    }
  } else {
    if (!arrive_last(r.arrive + 1 + tile, units, tl.last_arrived)) return;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int t16 = (tid >> 8) + j * (kTileThreads / 256), e = t16 * 16 + el_row;
      if (t16 < n_et) {
        const float* zp = zt + (size_t)t16 * parts * 256 + el;
        float v[parts];
#pragma unroll
        for (int c = 0; c < parts; ++c) v[c] = __builtin_bit_cast(float, load_published(zp + c * 256));
        float z = v[0];
#pragma unroll
        for (int c = 1; c < parts; ++c) z += v[c];
        if (e < E) tl.zs[el_tok][e] = z + bias[j];
      }
    }
  }
  __syncthreads();
  gate_and_group<KIND>(smem, tl, raw, tile, n_tiles, r, rw.masks, st, t, a);
}

// A small fp32 call (kSmallRouterBytes): one workgroup forms the router rows as dot products, one wave per (token, expert),
// sooner than several meet.
template <RouteKind KIND>
__global__ void __launch_bounds__(kTileThreads) route_small_fp32_kernel(RouteArgs r, LayerState st, CallTables t, CacheCallArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ TileLds tl;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int E = a.E, d = r.d;
  RawTable raw{};
  if (kColumns<KIND> && wave == 0) raw = raw_load(st, a);
  clear_tile_lds(tl, E);
  const int n_vec = d / 4, n_items = a.B * E;
  constexpr int U = 4;                                    // products of a wave in flight together
  for (int it0 = wave; it0 < n_items; it0 += U * kTileWaves) {
    float acc[U], bias[U];
    const float4 *xv[U], *wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int it = min(it0 + u * kTileWaves, n_items - 1);       // clamped: in bounds, formed again
      const int b = it / E, e = it - b * E;
      xv[u] = reinterpret_cast<const float4*>(static_cast<const float*>(r.x) + (size_t)b * d);
      wv[u] = reinterpret_cast<const float4*>(static_cast<const float*>(r.router_w) + (size_t)e * d);
      bias[u] = r.bias ? r.bias[(size_t)b * E + e] : 0.f;
      acc[u] = 0.f;
    }
    for (int c = lane; c < n_vec; c += kWave) {
      float4 xc[U], wc[U];
#pragma unroll
      for (int u = 0; u < U; ++u) { xc[u] = xv[u][c]; wc[u] = wv[u][c]; }
#pragma unroll
      for (int u = 0; u < U; ++u) acc[u] = Vec<float>::dot(wc[u], xc[u], acc[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int it = min(it0 + u * kTileWaves, n_items - 1);
      const float sum = wave_sum(acc[u]);
      if (lane == 0) tl.zs[it / E][it % E] = sum + bias[u];
    }
  }
  __syncthreads();
  gate_and_group<KIND>(smem, tl, raw, 0, 1, r, nullptr, st, t, a);
}

__global__ void __launch_bounds__(64) pin_kernel(LayerState st, CallTables t, CacheCallArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  if (fast_table(a.policy, a.C, a.P, a.n_shared)) {
    const LdsLayout L = lds_layout(a.E, a.C, a.P, a.n_shared, 1, a.K, a.KS);
    cache_phase_fast(fast_load(st, a.C, a.P), smem, L, a.pin_ids, nullptr, st, t, a);
  } else {
    const LdsLayout L = lds_layout(a.E, a.C, a.P, a.n_shared, 1, a.K, a.KS);
    cache_phase_general(smem, L, nullptr, nullptr, st, t, a);
  }
}

__global__ void reset_kernel(LayerState st, int E, int C, int P, int clear_trace, unsigned long long* dev_stats) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < C) { st.expert_in[i] = -1; st.tick[i] = 0; st.buf_of_slot[i] = -1; }
  if (i < E) st.score[i] = 0.0;
  if (i < P) { st.free_buf[i] = P - 1 - i; st.zombie[i] = -1; st.used_stamp[i] = 0; }  // buffer 0 is popped first
  if (i == 0) {
    st.scalars[SC_CLOCK] = 0;
    st.scalars[SC_NRES] = 0;
    st.scalars[SC_NFREE] = P;
    st.scalars[SC_NZOMBIE] = 0;
    if (clear_trace) st.scalars[SC_TRACE_N] = 0;
    if (dev_stats) dev_stats[0] = dev_stats[1] = dev_stats[2] = 0;
  }
}

}  // namespace

// Slices pay although they make units meet where one would do: 16 experts of 4096 columns, 8 / 64 tokens, one slice 12.7 / 15.3 us per
// launch, four 9.0 / 11.0; 64 of 2048 columns, 16 / 64 tokens, two 11.0 / 12.2, four 10.2 / 11.8; layer calls on 32 of 1024 columns, 16 /
// 64 tokens, one 21.1 / 25.7, two 20.8 / 25.0.  A unit that is alone in its tile publishes nothing: it is sliced from 2048 columns on
// (4 / 64 tokens on 16 experts of 1024 columns 17.0 / 22.2 us per layer call, in two 18.6 / 22.5).
// Several expert tiles per unit where the tiles alone make 512 units: 1024 tokens on 256 experts of 512 columns 111 us per
// prompt call with a tile each, 94 with two, 83 with four; 2048 on 64 of 2048 144 and 139 with two.
RouteUnits route_units(int B, int E, int d, bool sliced) {
  RouteUnits u{};
  u.tiles = (B + kTileTokens - 1) / kTileTokens;
  const int n_et = (E + 15) / 16, nkb = d / 32;
  u.et_per = (int)std::max<int64_t>(1, std::min<int64_t>(n_et, (int64_t)u.tiles * n_et / kRouteMaxUnits));
  u.slices = 1;
  while (sliced && u.slices < 4 && nkb / (2 * u.slices) >= (n_et * u.slices == 1 ? 2 : 1) * kRouteSliceKb && u.tiles * n_et * u.slices * 2 <= kRouteMaxUnits) u.slices *= 2;
  u.units = u.tiles * ((n_et + u.et_per - 1) / u.et_per) * u.slices;
  u.n_arrive = 1 + u.tiles;
  // (one slice: the logits; several: the eight pair sums of every logit)
  u.logit_bytes = (size_t)u.tiles * n_et * (u.slices > 1 ? kRouteChains / 2 : 1) * 256 * sizeof(float);
  u.scratch_bytes = u.logit_bytes + (size_t)u.tiles * kTileTokens * sizeof(uint64_t);
  return u;
}

size_t route_scratch_bytes(int max_batch, int E, int d) {
  const RouteUnits u = route_units(max_batch, E, d, true);     // (a smaller call may be sliced further, while its units are few enough)
  const size_t sliced = (size_t)std::min(u.tiles * ((E + 15) / 16), kRouteMaxUnits / 2) * (kRouteChains / 2) * 256 * sizeof(float);
  return std::max(u.logit_bytes, sliced) + (size_t)u.tiles * kTileTokens * sizeof(uint64_t);
}

size_t route_cache_lds_bytes(int E, int C, int P, int n_shared, int B, int K, int KS) {
  return lds_layout(E, C, P, n_shared, B, K, KS).total;
}

hipError_t launch_route_cache(hipStream_t s, int dtype, const RouteArgs& r, const LayerState& st, const CallTables& t,
                              const CacheCallArgs& a, const RouteScratch& scratch, KernelEvents ev) {
  // Few tokens: 16 waves per token so that the router rows stream with many loads
  // in flight.  Many tokens: the grid supplies the parallelism.
  int waves = a.B <= 16 ? 16 : 4;
  if (waves > a.E) waves = a.E;
  dim3 grid(a.B), block(64 * waves);
  const size_t lds = route_cache_lds_bytes(a.E, a.C, a.P, a.n_shared, a.B, a.K, a.KS);
  const RouteKind kind = a.mode == 0 && a.full && a.E <= kWave && a.C <= kWave ? (a.policy == MOE_POLICY_LRU ? kFull : kScored)
                         : a.mode == 2 ? kPrompt
                         : a.E > kTileMaxE || !fast_table(a.policy, a.C, a.P, a.n_shared) ? kOther
                         : a.E > kWave ? kWide : kTable;
  const bool hits = kind == kFull || kind == kScored, columns = kind < kOther;
  // Units from two tokens on where every lookup is known to hit, whatever the policy and the spare buffers, so that a full cache routes a
  // batch bit for bit as the allocation-free entry point does (30 points of 8 to 64 experts of 1024 to 4096 columns, 4 to 1024 tokens: 1.19x
  // in the mean against the kernels before, none slower; discounted counts, 64 tokens on 64 / 16 experts, looked up in order by one wave
  // 338 / 94.5 us per layer call, here 118 / 37) and on the register table (16 tokens on 64 experts, half of them resident, 144
  // against 153 us) from 17 experts on: with fewer, and a wave that looks up in order, a workgroup per token keeps up to 112 tokens
  // (16 tokens, 8 experts, misses 21.7 against 22.7 us).  From 112 tokens, too, where one wave looks up in order whatever routes (64
  // tokens on 16 experts under discounted counts 115.8 against 121.1 us), and with more than 64 experts (112 tokens that hit on 128
  // 89 against 108 us); prompts on more than 32 experts from 32.
  const int least = hits ? 2 : kind == kTable ? (a.E > 16 ? 2 : 112) : kind == kPrompt && a.E > 32 ? 32 : 112;
  if (dtype == MOE_DTYPE_BF16 && a.B >= least && a.E <= kTileMaxE && r.d % 32 == 0) {
    // (Lookups in order take far longer than a slice saves.  Prompts whose pairs do not fit the LDS run the code that the kernel without
    // slices has for them faster: 400 / 512 tokens on 64 experts of 2048 columns 95 / 115 us per layer call in slices, 86 / 102 without, 200 / 256
    // tokens, which fit, 57 / 63 and 58 / 64.)
    const RouteUnits ru = route_units(a.B, a.E, r.d, kind == kPrompt ? stage_in_lds(a.B, a.KS) : kind != kOther);
    if (ru.n_arrive <= scratch.n_arrive && ru.scratch_bytes <= scratch.bytes) {
      const RouteWork w{ru.slices, ru.et_per, static_cast<float*>(scratch.ptr),
                        reinterpret_cast<uint64_t*>(static_cast<char*>(scratch.ptr) + ru.logit_bytes)};
      const size_t bytes = std::max({hits ? 0 : lds, (size_t)kTileWaves * 256 * sizeof(float), columns && stage_pairs(a.B, a.KS) ? (size_t)(a.B * a.KS + 3) / 4 * 32 : 0});
      static_assert(sizeof(TileLds) + kStagedMost * 2 * sizeof(int32_t) <= 160 << 10, "a unit's LDS");
      const dim3 units(ru.units), threads(kTileThreads);
      const auto launch = [&](auto kernel) { launch_timed(kernel, units, threads, bytes, s, ev, r, w, st, t, a); };
      const int pairs = (r.d / 32 + 2 * kRouteChains - 1) / (2 * kRouteChains);      // of k-blocks in a chain
      const auto of = [&](auto packed, auto k, auto sliced) {
        constexpr bool P = decltype(packed)::value, S = decltype(sliced)::value;
        constexpr RouteKind Q = decltype(k)::value;
        launch(pairs > 2 ? route_units_kernel<4, P, Q, S> : pairs > 1 ? route_units_kernel<2, P, Q, S> : route_units_kernel<1, P, Q, S>);
      };
      const auto with = [&](auto packed, auto k) {
        if constexpr (decltype(k)::value != kOther)
          if (ru.slices > 1) return of(packed, k, std::true_type{});
        of(packed, k, std::false_type{});
      };
#define MOE_KIND(K) std::integral_constant<RouteKind, K>{}
      if (kind == kFull && r.router_packed) with(std::true_type{}, MOE_KIND(kFull));
      else if (kind == kFull) with(std::false_type{}, MOE_KIND(kFull));
      else if (kind == kScored) with(std::false_type{}, MOE_KIND(kScored));
      else if (kind == kTable) with(std::false_type{}, MOE_KIND(kTable));
      else if (kind == kWide) with(std::false_type{}, MOE_KIND(kWide));
      else if (kind == kPrompt) with(std::false_type{}, MOE_KIND(kPrompt));
      else with(std::false_type{}, MOE_KIND(kOther));
#undef MOE_KIND
      return hipGetLastError();
    }
  }
  if (dtype == MOE_DTYPE_FP32 && a.B >= 2 && a.B <= 8 && a.B * a.E <= kSmallRouterItems &&
      (size_t)a.B * a.E * r.d * sizeof(float) <= kSmallRouterBytes) {
    const auto small = kind == kFull ? route_small_fp32_kernel<kFull> : kind == kScored ? route_small_fp32_kernel<kScored> : kind == kTable ? route_small_fp32_kernel<kTable> : route_small_fp32_kernel<kOther>;
    launch_timed(small, dim3(1), dim3(kTileThreads), hits ? 0 : lds, s, ev, r, st, t, a);
    return hipGetLastError();
  }
  const auto launch = [&](auto type) {
    using T = decltype(type);
    const bool prompt = a.mode == 2;
    const auto of = [&](auto kernel) { launch_timed(kernel, grid, block, lds, s, ev, r, st, t, a); };
    if (a.E <= waves) of(prompt ? route_cache_kernel<T, 1, 1, kPrompts> : route_cache_kernel<T, 1, 1, kBoth>);
    else if (a.E <= 64) of(prompt ? route_cache_kernel<T, 4, 1, kPrompts> : route_cache_kernel<T, 4, 1, kDecodes>);
    else if (a.E <= 256) of(route_cache_kernel<T, 4, 4, kBoth>);
    else of(prompt ? route_cache_kernel<T, 4, 16, kPrompts> : route_cache_kernel<T, 4, 16, kDecodes>);
  };
  if (dtype == MOE_DTYPE_FP32) launch(float{});
  else launch(uint16_t{});
  return hipGetLastError();
}

hipError_t launch_pin(hipStream_t s, const LayerState& st, const CallTables& t, const CacheCallArgs& a) {
  const size_t lds = route_cache_lds_bytes(a.E, a.C, a.P, a.n_shared, 1, a.K, a.KS);
  hipLaunchKernelGGL(pin_kernel, dim3(1), dim3(64), lds, s, st, t, a);
  return hipGetLastError();
}

hipError_t launch_reset(hipStream_t s, const LayerState& st, int E, int C, int P, int clear_trace,
                        unsigned long long* dev_stats) {
  int n = E > C ? E : C;
  n = n > P ? n : P;
  hipLaunchKernelGGL(reset_kernel, dim3((n + 255) / 256), dim3(256), 0, s, st, E, C, P, clear_trace, dev_stats);
  return hipGetLastError();
}

}  // namespace moe
