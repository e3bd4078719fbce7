// moe_build_dispatch: per-expert counts and offsets (the nactive[expert] of Sec. III-E), the stable
// algebraic<->layout row maps (AL Table of Sec. III-D; token id list per tile of Sec. IV-B) and the table of
// distinct (token, rank) pairs (the redundancy of Sec. II-B; rank(e) = e / experts_per_rank, Sec. III-D).
//
// Two small kernels, no atomics on device memory, so the result does not depend on scheduling:
//   1. hist : the token range is cut into <= 64 chunks, one block per chunk counts its pairs per expert and
//             its first-of-rank pairs per rank (LDS counters);
//   2. place: every block first sums the chunk histograms (all chunks -> counts, earlier chunks -> its own
//             starting cursors) and scans the counts across experts into offsets (block 0 writes them out).
//             The chunk is cut once more into one contiguous token range per wave; a count of those ranges
//             (LDS) turns the chunk cursors into per-wave cursors, and every wave then walks its range in pair
//             order: lanes holding the same expert are found with one ballot per bit of the expert id, the
//             popcount of the lower lanes is the rank inside the group, and the highest lane of the group
//             advances the wave's LDS cursor.
#include <algorithm>

#include "route_pick.h"

namespace moe355 {

constexpr int kMaxChunks = 64;

struct PairLane {
  int t, j, e, r;
  bool active, valid;
};

// Lane -> pair assignment of one iteration: floor(64 / k) whole tokens, slot-major inside a token.
__device__ __forceinline__ int ceil_div_dev(int a, int b) { return (a + b - 1) / b; }

__device__ __forceinline__ int load_expert(const int32_t *__restrict__ topk_idx, int t0, int t_end, int k, int tpi) {
  const int lane = lane_id();
  const int tl = lane / k;
  const int t = t0 + tl;
  return (tl < tpi && t < t_end) ? topk_idx[(size_t)t * k + (lane - tl * k)] : -1;
}

// `e` is this lane's expert id as returned by load_expert for the same t0 (fetched one iteration ahead so that
// the walk does not wait on global memory every 64 pairs).
__device__ __forceinline__ PairLane make_pair(int e, int t0, int t_end, int k, int tpi, int E, int epr) {
  PairLane p;
  const int lane = lane_id();
  const int tl = lane / k;
  p.j = lane - tl * k;
  p.t = t0 + tl;
  p.active = tl < tpi && p.t < t_end;
  p.e = p.active ? e : -1;
  p.valid = p.active && p.e >= 0 && p.e < E;
  p.r = p.valid ? p.e / epr : -1;
  return p;
}

// Slots of the same token that lie on the same rank as this lane's slot (bit jj per slot).
__device__ __forceinline__ uint32_t same_rank_slots(const PairLane &p, int k) {
  const int lane = lane_id();
  uint32_t m = 0;
  for (int jj = 0; jj < k; ++jj) {
    const int rr = __shfl(p.r, (lane - p.j + jj) & 63, 64);
    if (p.valid && rr == p.r) m |= 1u << jj;
  }
  return m;
}

// Lanes among `pred` lanes whose `key` equals this lane's key (bits = number of significant key bits).
__device__ __forceinline__ unsigned long long match_lanes(bool pred, int key, int bits) {
  unsigned long long m = __ballot(pred);
  for (int b = 0; b < bits; ++b) {
    const bool bit = (key >> b) & 1;
    const unsigned long long bal = __ballot(pred && bit);
    m &= bit ? bal : ~bal;
  }
  return m;
}

// Adds the pairs of tokens [t_begin, t_end) to the LDS counters cnt[E] / rcnt[R] (one wave; the counters may
// be shared with other waves).
__device__ __forceinline__ void count_range(const int32_t *__restrict__ topk_idx, int t_begin, int t_end, int k,
                                            int E, int epr, int *cnt, int *rcnt) {
  const int tpi = kWave / k;
  int e_next = load_expert(topk_idx, t_begin, t_end, k, tpi);
  for (int t0 = t_begin; t0 < t_end; t0 += tpi) {
    const PairLane p = make_pair(e_next, t0, t_end, k, tpi, E, epr);
    e_next = load_expert(topk_idx, t0 + tpi, t_end, k, tpi);
    const uint32_t slots = same_rank_slots(p, k);
    if (p.valid) {
      atomicAdd(&cnt[p.e], 1);
      if ((slots & ((1u << p.j) - 1u)) == 0) atomicAdd(&rcnt[p.r], 1);  // first slot of its (token, rank)
    }
  }
}

constexpr int kTableThreads = 512;  // block size of both kernels

__global__ __launch_bounds__(kTableThreads) void dispatch_hist_kernel(const int32_t *__restrict__ topk_idx, int T,
                                                                      int E, int k, int R, int tpc,
                                                                      int32_t *__restrict__ chunk_cnt,
                                                                      int32_t *__restrict__ chunk_rcnt) {
  extern __shared__ int sm[];
  int *cnt = sm;
  int *rcnt = sm + E;
  const int c = blockIdx.x;
  const int wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
  for (int i = threadIdx.x; i < E + R; i += blockDim.x) sm[i] = 0;
  __syncthreads();
  const int t_begin = c * tpc;
  const int t_end = min(T, t_begin + tpc);
  const int tpw = ceil_div_dev(tpc, nwaves);
  count_range(topk_idx, min(t_end, t_begin + wave * tpw), min(t_end, t_begin + (wave + 1) * tpw), k, E, E / R, cnt,
              rcnt);
  __syncthreads();
  // histograms are stored expert-major ([expert][chunk]) so that the placement kernel reads one expert's 64
  // chunk counts as one contiguous 256-byte run
  for (int i = threadIdx.x; i < E; i += blockDim.x) chunk_cnt[(size_t)i * kMaxChunks + c] = cnt[i];
  for (int i = threadIdx.x; i < R; i += blockDim.x) chunk_rcnt[(size_t)i * kMaxChunks + c] = rcnt[i];
}

__global__ __launch_bounds__(kTableThreads) void dispatch_place_kernel(
    const int32_t *__restrict__ topk_idx, int T, int E, int k, int R, int tpc, int nch, int ebits, int rbits, int nwalk,
    const int32_t *__restrict__ chunk_cnt, const int32_t *__restrict__ chunk_rcnt, int32_t *__restrict__ counts,
    int32_t *__restrict__ offsets, int32_t *__restrict__ rank_counts, int32_t *__restrict__ rank_offsets,
    int32_t *__restrict__ perm, int32_t *__restrict__ inv_perm, int32_t *__restrict__ dedup_tok,
    uint32_t *__restrict__ dedup_mask, int32_t *__restrict__ pair_to_dedup) {
  extern __shared__ int sm[];
  int *cursor = sm;            // [E] next free layout row of each expert for this chunk
  int *rcursor = sm + E;       // [R] next free dedup entry of each rank for this chunk
  int *tot = rcursor + R;      // [E + R] totals over all chunks
  int *scratch = tot + E + R;  // [17]
  int *sub = scratch + 17;     // [nwalk][E + R] per walking wave: pair counts of its token range, then its cursors
  const int lane = lane_id();
  const int wave = threadIdx.x >> 6;
  const int c = blockIdx.x;
  const int epr = E / R;
  // token range of this wave inside the chunk (waves >= nwalk only help with the tables)
  const int chunk_begin = c * tpc;
  const int chunk_end = min(T, chunk_begin + tpc);
  const int tpw = ceil_div_dev(tpc, nwalk);
  const int t_begin = min(chunk_end, chunk_begin + min(wave, nwalk) * tpw);
  const int t_end = wave < nwalk ? min(chunk_end, t_begin + tpw) : t_begin;
  for (int i = threadIdx.x; i < nwalk * (E + R); i += blockDim.x) sub[i] = 0;
  __syncthreads();
  if (wave < nwalk) count_range(topk_idx, t_begin, t_end, k, E, epr, sub + wave * (E + R), sub + wave * (E + R) + E);
  // per expert / rank: total over all chunks and the part that belongs to earlier chunks
  for (int i = threadIdx.x; i < E + R; i += blockDim.x) {
    const int4 *row = reinterpret_cast<const int4 *>(i < E ? chunk_cnt + (size_t)i * kMaxChunks
                                                           : chunk_rcnt + (size_t)(i - E) * kMaxChunks);
    int4 v[kMaxChunks / 4];
#pragma unroll
    for (int q = 0; q < kMaxChunks / 4; ++q) v[q] = row[q];  // 16 independent 16-byte loads
    int total = 0, before = 0;
#pragma unroll
    for (int q = 0; q < kMaxChunks / 4; ++q) {
      const int vals[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int cc = q * 4 + u;
        const int val = cc < nch ? vals[u] : 0;  // slots of chunks that do not exist hold stale workspace bytes
        total += val;
        before += cc < c ? val : 0;
      }
    }
    tot[i] = total;
    sm[i] = before;
  }
  __syncthreads();
  // exclusive scan of the totals across experts, then across ranks: each thread owns a run of consecutive items
  for (int pass = 0; pass < 2; ++pass) {
    const int n = pass == 0 ? E : R;
    const int *src = pass == 0 ? tot : tot + E;
    int *cur = pass == 0 ? cursor : rcursor;
    int32_t *cnt_out = pass == 0 ? counts : rank_counts;
    int32_t *off_out = pass == 0 ? offsets : rank_offsets;
    const int ipt = (n + blockDim.x - 1) / blockDim.x;
    const int lo = min(n, (int)threadIdx.x * ipt);
    const int hi = min(n, lo + ipt);
    int local = 0;
    for (int i = lo; i < hi; ++i) local += src[i];
    int total;
    int run = block_exclusive_scan(local, scratch, &total);
    for (int i = lo; i < hi; ++i) {
      const int v = src[i];
      if (c == 0) {
        cnt_out[i] = v;
        off_out[i] = run;
      }
      cur[i] += run;
      run += v;
    }
    if (c == 0 && threadIdx.x == 0) off_out[n] = total;
    __syncthreads();
  }
  // chunk cursors -> per-wave cursors: wave w starts where the waves before it end
  for (int i = threadIdx.x; i < E + R; i += blockDim.x) {
    int run = sm[i];
    for (int w = 0; w < nwalk; ++w) {
      const int v = sub[w * (E + R) + i];
      sub[w * (E + R) + i] = run;
      run += v;
    }
  }
  __syncthreads();
  if (wave >= nwalk) return;  // each walk is a single-wave job; no block barrier below
  cursor = sub + wave * (E + R);
  rcursor = cursor + E;
  const int tpi = kWave / k;
  const unsigned long long lower = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const long long npairs = (long long)T * k;
  const long long ndedup = (long long)T * min(k, R);
  int e_next = load_expert(topk_idx, t_begin, t_end, k, tpi);
  for (int t0 = t_begin; t0 < t_end; t0 += tpi) {
    const PairLane p = make_pair(e_next, t0, t_end, k, tpi, E, epr);
    e_next = load_expert(topk_idx, t0 + tpi, t_end, k, tpi);
    const size_t pid = (size_t)p.t * k + p.j;

    // ---- layout row of every pair (stable: lower lanes are earlier pairs) ----
    const unsigned long long grp = match_lanes(p.valid, p.e, ebits);
    int row = -1;
    if (p.valid) row = cursor[p.e] + __popcll(grp & lower);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (p.valid && (lane == 63 || (grp >> (lane + 1)) == 0)) cursor[p.e] = row + 1;
    if (p.active) inv_perm[pid] = row;
    if (p.valid && row >= 0 && row < npairs) perm[row] = (int32_t)pid;

    // ---- distinct (token, rank) entries ----
    const uint32_t slots = same_rank_slots(p, k);
    const bool first = p.valid && (slots & ((1u << p.j) - 1u)) == 0;
    const unsigned long long rgrp = match_lanes(first, p.r, rbits);
    int pos = -1;
    if (first) pos = rcursor[p.r] + __popcll(rgrp & lower);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (first && (lane == 63 || (rgrp >> (lane + 1)) == 0)) rcursor[p.r] = pos + 1;
    if (first && pos >= 0 && pos < ndedup) {
      dedup_tok[pos] = p.t;
      dedup_mask[pos] = slots;
    }
    const int first_slot = slots ? __builtin_ctz(slots) : 0;
    const int pos_of_first = __shfl(pos, (lane - p.j + first_slot) & 63, 64);
    if (p.active) pair_to_dedup[pid] = p.valid ? pos_of_first : -1;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------------------------------------------
// One thread per pair: the form used where a workgroup's share of the pairs and its counters fit the LDS.  Pair it * 1024 +
// thread of the workgroup; the pairs of one wave in one iteration form a "virtual wave" v.  Lanes with the same expert are
// found with one ballot per bit of the expert id, the group's first lane writes its size to sub[v][expert] (no atomics),
// an exclusive sum over v and a scan over the experts turn the sizes into first rows, and the rank of a lane in its group
// does the rest; the same for (token, rank) entries over the lanes that hold the first slot of their token on a rank.
// What bounds it is latency: one read of topk_idx and six barriers, where the walk above makes a serial pass per wave.
//   CHUNKED = false: small batches, all tables in ONE launch of one workgroup (96 tokens, k = 8: 5.5 us against 4.7 + 10.5 us
//   for the two kernels above, which pay a second launch and a round trip of the histograms through memory);
//   CHUNKED = true: one workgroup per chunk of whole tokens, on the chunk histograms of dispatch_hist_pairs_kernel (8192
//   tokens, k = 8, 128 experts: 5.1 + 11.4 us against 5.2 + 14.8 us; 5003 tokens, k = 4: 5.1 + 9.1 against 5.1 + 11.3 us).
// ------------------------------------------------------------------------------------------------
constexpr int kSmallThreads = 1024;
constexpr int kSmallPairs = 4096;         // most pairs of the one-launch form
constexpr size_t kSmallLds = 128 * 1024;  // most LDS

// [ITERS][1024] expert ids | [virtual waves][E + R] counts, then first rows | [E + R] totals | [18] scan scratch
constexpr size_t small_lds_bytes(int iters, int E, int R) {
  return ((size_t)iters * (kSmallThreads + (kSmallThreads / kWave) * (E + R)) + (E + R) + 18) * sizeof(int);
}

// Slots of this pair's token that lie on rank r, among the first n ones; s_e holds the expert ids of the token at p0.
__device__ __forceinline__ uint32_t slots_on_rank(const int *s_e, int p0, int n, int r, int epr) {
  uint32_t m = 0;
  for (int jj = 0; jj < n; ++jj) {
    const int e = s_e[p0 + jj];
    if (e >= r * epr && e < (r + 1) * epr) m |= 1u << jj;
  }
  return m;
}

// Chunk histograms, one thread per pair (LDS counters); layout of dispatch_hist_kernel's.
template <int ITERS>
__global__ __launch_bounds__(kSmallThreads) void dispatch_hist_pairs_kernel(const int32_t *__restrict__ topk_idx, int T,
                                                                            int E, int k, int R, int tpc,
                                                                            int32_t *__restrict__ chunk_cnt,
                                                                            int32_t *__restrict__ chunk_rcnt) {
  extern __shared__ int sm[];
  int *cnt = sm, *s_e = sm + E + R;  // [E + R] | [ITERS * 1024]
  const int tid = threadIdx.x, c = blockIdx.x, epr = E / R;
  const int n = min(T - c * tpc, tpc) * k;
  const int32_t *src = topk_idx + (size_t)c * tpc * k;
  int e[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int p = it * kSmallThreads + tid;
    e[it] = p < n ? src[p] : -1;
  }
  for (int i = tid; i < E + R; i += kSmallThreads) cnt[i] = 0;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) s_e[it * kSmallThreads + tid] = e[it];
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    if (e[it] < 0 || e[it] >= E) continue;
    const int p = it * kSmallThreads + tid, j = p % k, r = e[it] / epr;
    atomicAdd(&cnt[e[it]], 1);
    if (slots_on_rank(s_e, p - j, j, r, epr) == 0) atomicAdd(&cnt[E + r], 1);  // first slot of its (token, rank)
  }
  __syncthreads();
  for (int i = tid; i < E; i += kSmallThreads) chunk_cnt[(size_t)i * kMaxChunks + c] = cnt[i];
  for (int i = tid; i < R; i += kSmallThreads) chunk_rcnt[(size_t)i * kMaxChunks + c] = cnt[E + i];
}

// PER > 0 (one workgroup; E <= 64 PER): the routing as well.  Its waves route the tokens first, one after the other each, and
// hand the picks over in the LDS (16 tokens of 64 experts, k = 8: 3.0 + 5.3 us as two launches).
template <int ITERS, bool CHUNKED, int PER = 0>
__global__ __launch_bounds__(kSmallThreads) void dispatch_pairs_kernel(
    const float *__restrict__ logits, float *__restrict__ topk_w, int32_t *__restrict__ topk_idx, int T, int E, int k, int R,
    int tpc, int nch, int ebits, int rbits, const int32_t *__restrict__ chunk_cnt, const int32_t *__restrict__ chunk_rcnt,
    int32_t *__restrict__ counts, int32_t *__restrict__ offsets, int32_t *__restrict__ rank_counts,
    int32_t *__restrict__ rank_offsets, int32_t *__restrict__ perm, int32_t *__restrict__ inv_perm,
    int32_t *__restrict__ dedup_tok, uint32_t *__restrict__ dedup_mask, int32_t *__restrict__ pair_to_dedup) {
  extern __shared__ int sm[];
  constexpr int kWaves = kSmallThreads / kWave, NV = ITERS * kWaves;
  int *s_e = sm;                           // expert of every pair of this workgroup
  int *sub = s_e + ITERS * kSmallThreads;  // [NV][E + R]
  int *tot = sub + NV * (E + R);           // totals over all pairs
  int *scratch = tot + E + R;
  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int epr = E / R, C = E + R, c = CHUNKED ? blockIdx.x : 0;
  const int base = CHUNKED ? c * tpc * k : 0;  // first pair of this workgroup: whole tokens
  const int n = CHUNKED ? min(T - c * tpc, tpc) * k : T * k;
  int e[ITERS];
  if constexpr (PER > 0) {
    for (int t = wave; t < T; t += kWaves) {
      RowPicker<PER> pick;
      route_load_row(pick, logits + (size_t)t * E, E);
      route_pick_registers<PER>(pick, E, k, t, topk_idx, topk_w, s_e);
    }
    __syncthreads();
  }
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int p = it * kSmallThreads + tid;
    if constexpr (PER > 0) e[it] = p < n ? s_e[p] : -1;
    else e[it] = p < n ? topk_idx[base + p] : -1;
    if (e[it] >= E) e[it] = -1;
  }
  int before = 0;  // pairs of column tid in earlier chunks
  if constexpr (CHUNKED) {
    if (tid < C) {  // (C <= 1024)
      const int4 *row = reinterpret_cast<const int4 *>(tid < E ? chunk_cnt + (size_t)tid * kMaxChunks
                                                               : chunk_rcnt + (size_t)(tid - E) * kMaxChunks);
      int4 v[kMaxChunks / 4];
#pragma unroll
      for (int q = 0; q < kMaxChunks / 4; ++q)
        if (q * 4 < nch) v[q] = row[q];
      int total = 0;
#pragma unroll
      for (int q = 0; q < kMaxChunks / 4; ++q) {
        if (q * 4 >= nch) continue;
        const int vals[4] = {v[q].x, v[q].y, v[q].z, v[q].w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int val = q * 4 + u < nch ? vals[u] : 0;  // slots of chunks that do not exist hold stale workspace bytes
          total += val;
          before += q * 4 + u < c ? val : 0;
        }
      }
      tot[tid] = total;
    }
  }
  for (int i = tid; i < NV * C; i += kSmallThreads) sub[i] = 0;
#pragma unroll
  for (int it = 0; it < ITERS; ++it) s_e[it * kSmallThreads + tid] = e[it];
  __syncthreads();
  const unsigned long long lower = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  int in_grp[ITERS], r_of[ITERS], r_in_grp[ITERS];
  uint32_t slots[ITERS];
  bool first[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int p = it * kSmallThreads + tid, v = it * kWaves + wave;
    const bool valid = e[it] >= 0;
    const unsigned long long grp = match_lanes(valid, e[it], ebits);
    in_grp[it] = __popcll(grp & lower);
    if (valid && in_grp[it] == 0) sub[v * C + e[it]] = __popcll(grp);
    const int j = p % k, r = valid ? e[it] / epr : -1;
    const uint32_t m = valid ? slots_on_rank(s_e, p - j, k, r, epr) : 0;
    r_of[it] = r;
    slots[it] = m;
    first[it] = valid && (m & ((1u << j) - 1u)) == 0;
    const unsigned long long rgrp = match_lanes(first[it], r, rbits);
    r_in_grp[it] = __popcll(rgrp & lower);
    if (first[it] && r_in_grp[it] == 0) sub[v * C + E + r] = __popcll(rgrp);
  }
  __syncthreads();
  // columns (experts, then ranks): thread i owns columns i * ipt ..; exclusive sums over the virtual waves
  const int ipt = (C + kSmallThreads - 1) / kSmallThreads;
  const int lo = min(C, tid * ipt), hi = min(C, lo + ipt);
  int local = 0;
  for (int i = lo; i < hi; ++i) {
    int run = 0;
#pragma unroll 16
    for (int v = 0; v < NV; ++v) {
      const int x = sub[v * C + i];
      sub[v * C + i] = run;
      run += x;
    }
    if (!CHUNKED) tot[i] = run;
    local += CHUNKED ? tot[i] : run;
  }
  // one scan over all columns; the ranks' part starts from zero again
  int total;
  int off = block_exclusive_scan(local, scratch, &total);
  if (lo <= E && E < hi) {  // pairs with a valid expert = the part of the scan that belongs to the experts
    int o = off;
    for (int i = lo; i < E; ++i) o += tot[i];
    scratch[17] = o;
  }
  __syncthreads();
  const int n_valid = scratch[17];
  for (int i = lo; i < hi; ++i) {
    const int mine = tot[i];
    const int first_row = i < E ? off : off - n_valid;
    if (c == 0) {
      if (i < E) {
        counts[i] = mine;
        offsets[i] = first_row;
      } else {
        rank_counts[i - E] = mine;
        rank_offsets[i - E] = first_row;
      }
    }
#pragma unroll 16
    for (int v = 0; v < NV; ++v) sub[v * C + i] += first_row + before;
    off += mine;
  }
  if (c == 0 && tid == 0) {
    offsets[E] = n_valid;
    rank_offsets[R] = total - n_valid;
  }
  __syncthreads();
  const int npairs = T * k, ndedup = T * min(k, R);
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int p = it * kSmallThreads + tid, v = it * kWaves + wave;
    if (e[it] >= 0) {
      const int row = sub[v * C + e[it]] + in_grp[it];
      inv_perm[base + p] = row;
      if (row >= 0 && row < npairs) perm[row] = base + p;
    } else if (p < n) {
      inv_perm[base + p] = -1;
      pair_to_dedup[base + p] = -1;
    }
    int pos = -1;
    if (first[it]) {
      pos = sub[v * C + E + r_of[it]] + r_in_grp[it];
      if (pos >= 0 && pos < ndedup) {
        dedup_tok[pos] = (base + p) / k;
        dedup_mask[pos] = slots[it];
      }
    }
    s_e[p] = pos;  // (the expert ids are not needed any more)
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    const int p = it * kSmallThreads + tid;
    if (e[it] >= 0) pair_to_dedup[base + p] = s_e[p - p % k + __builtin_ctz(slots[it])];
  }
}

}  // namespace moe355

using namespace moe355;

static int chunking(int T, int *tpc) {
  if (T <= 0) {
    *tpc = 1;
    return 0;
  }
  *tpc = ceil_div(T, kMaxChunks);
  return ceil_div(T, *tpc);
}

extern "C" size_t moe_dispatch_workspace_bytes(const moe_shape *shape) {
  Derived dv;
  if (check_shape(shape, &dv) != MOE_OK) return 0;
  return align_up((size_t)kMaxChunks * (shape->E + shape->R) * sizeof(int32_t), 256);
}

// Both forms of the call: the chunk histograms live in `chunk_ws` (kMaxChunks * (E + R) int32).
static int build_dispatch_launches(const moe_shape *shape, const int32_t *topk_idx, const moe_dispatch *out,
                                   int32_t *chunk_ws, hipStream_t st) {
  const int T = shape->T, E = shape->E, k = shape->k, R = shape->R;
  int tpc;
  int ebits = 0, rbits = 0;
  while ((1 << ebits) < E) ++ebits;
  while ((1 << rbits) < R) ++rbits;
#define MOE355_PAIRS(ITERS_, CHUNKED_, GRID_, TPC_, NCH_, CNT_, RCNT_)                                              \
  do {                                                                                                              \
    static std::atomic<uint64_t> done{0};                                                                           \
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&dispatch_pairs_kernel<ITERS_, CHUNKED_>), (int)kSmallLds, \
                           done))                                                                                   \
      return MOE_ERR_HIP;                                                                                           \
    hipLaunchKernelGGL((dispatch_pairs_kernel<ITERS_, CHUNKED_>), dim3(GRID_), dim3(kSmallThreads),                 \
                       small_lds_bytes(ITERS_, E, R), st, nullptr, nullptr, const_cast<int32_t *>(topk_idx), T, E,  \
                       k, R, TPC_, NCH_, ebits, rbits, CNT_, RCNT_, out->counts, out->offsets, out->rank_counts,    \
                       out->rank_offsets, out->perm, out->inv_perm, out->dedup_tok, out->dedup_mask,                \
                       out->pair_to_dedup);                                                                         \
  } while (0)
  // Small batches (up to kSmallPairs pairs whose counters fit the LDS): one launch of one workgroup.
  const auto iters_of = [](int64_t pairs) { return pairs <= 1024 ? 1 : pairs <= 2048 ? 2 : pairs <= 4096 ? 4 : 8; };
  if (T > 0 && (int64_t)T * k <= kSmallPairs && small_lds_bytes(iters_of(T * k), E, R) <= kSmallLds) {
    begin_launches();
    const int iters = iters_of(T * k);
    const int32_t *none = nullptr;
    if (iters == 1) MOE355_PAIRS(1, false, 1, T, 1, none, none);
    else if (iters == 2) MOE355_PAIRS(2, false, 1, T, 1, none, none);
    else MOE355_PAIRS(4, false, 1, T, 1, none, none);
    return launch_status();
  }
  // One thread per pair, as few chunks as keep a workgroup's share at 1024 pairs, up to the chunk limit; beyond eight
  // pairs per thread, or with more counters than fit, the kernels that walk (below).
  if (T > 0 && E + R <= kSmallThreads) {
    const int tpc_p = std::max(ceil_div(T, kMaxChunks), std::max(1, kSmallThreads / k)), nch_p = ceil_div(T, tpc_p);
    const int64_t pairs = (int64_t)tpc_p * k;
    const int iters = iters_of(pairs);
    if (pairs <= 8 * kSmallThreads && small_lds_bytes(iters, E, R) <= kSmallLds) {
      begin_launches();
      int32_t *cnt = chunk_ws, *rcnt = chunk_ws + (size_t)kMaxChunks * E;
      const size_t lds_hist = (size_t)(E + R + iters * kSmallThreads) * sizeof(int);
#define MOE355_CHUNKED(ITERS_)                                                                                     \
  do {                                                                                                             \
    hipLaunchKernelGGL(dispatch_hist_pairs_kernel<ITERS_>, dim3(nch_p), dim3(kSmallThreads), lds_hist, st, topk_idx, \
                       T, E, k, R, tpc_p, cnt, rcnt);                                                              \
    int rc_;                                                                                                       \
    if ((rc_ = launch_status()) != MOE_OK) return rc_;                                                             \
    MOE355_PAIRS(ITERS_, true, nch_p, tpc_p, nch_p, cnt, rcnt);                                                    \
  } while (0)
      if (iters == 1) MOE355_CHUNKED(1); else if (iters == 2) MOE355_CHUNKED(2); else if (iters == 4) MOE355_CHUNKED(4);
      else MOE355_CHUNKED(8);
#undef MOE355_CHUNKED
      return launch_status();
    }
  }
#undef MOE355_PAIRS
  const int nch = chunking(T, &tpc);
  int32_t *chunk_cnt = chunk_ws;
  int32_t *chunk_rcnt = chunk_cnt + (size_t)kMaxChunks * E;
  int rc;
  begin_launches();
  const size_t sm_wave = (size_t)(E + R) * sizeof(int);
  if (nch > 0) {
    hipLaunchKernelGGL(dispatch_hist_kernel, dim3(nch), dim3(kTableThreads), sm_wave, st, topk_idx, T, E, k, R, tpc,
                       chunk_cnt, chunk_rcnt);
    if ((rc = launch_status()) != MOE_OK) return rc;
  }
  // The placement kernel keeps (2 + walking waves) arrays of E + R counters in LDS; with the largest E and R even
  // one walking wave needs more than the default 64 KiB of dynamic LDS, so the limit is raised (once per device).
  constexpr size_t kPlaceLds = 144 * 1024;
  static std::atomic<uint64_t> done{0};
  if (!allow_dynamic_lds(reinterpret_cast<const void *>(&dispatch_place_kernel), (int)kPlaceLds, done))
    return MOE_ERR_HIP;
  const size_t fit = (kPlaceLds - 1024) / sm_wave;  // arrays that fit; at least 3 for E + R <= 8192
  const int nwalk = (int)std::max<size_t>(1, std::min<size_t>(kTableThreads / kWave, fit > 2 ? fit - 2 : 1));
  // with T == 0 a single block still writes the all-zero counts and offsets
  hipLaunchKernelGGL(dispatch_place_kernel, dim3(nch > 0 ? nch : 1), dim3(kTableThreads),
                     (size_t)((2 + nwalk) * (E + R) + 17) * sizeof(int), st, topk_idx, T, E, k, R, tpc, nch, ebits, rbits,
                     nwalk, chunk_cnt,
                     chunk_rcnt, out->counts, out->offsets, out->rank_counts, out->rank_offsets, out->perm,
                     out->inv_perm, out->dedup_tok, out->dedup_mask, out->pair_to_dedup);
  return launch_status();
}

// Routing and tables of a small batch in one launch, where its one workgroup routes the tokens in less time than the launch it
// saves.  A wave's tokens come one after the other and the waves of a SIMD share it: time in proportion to the tokens, to the
// picks plus what loading and sorting a row take (about eight picks) and, more slowly, to the experts per lane.  Gain over two
// launches, microseconds of a step:
//   tokens               8      16      24      32    |  64 experts, k = 2:   1.6   1.3   1.1   0.6
//   64 experts, k = 8    1.5    1.0     0.2    -0.8   |  64 experts, k = 32:  0.9  -1.2  -3.6  -7.2
//   128 experts, k = 8   1.3    0.6    -0.2    -1.4   |  128 experts, k = 4:  1.5   1.1   0.3  -0.4
//   256 experts, k = 8   1.1    0.2    -0.6    -2.3   |  256 experts, k = 2:  1.2   1.0   0.5  -0.2
//   512 experts, k = 8   0.7   -0.9    -2.5    -5.0   |  512 experts, k = 1:  0.8   0.3  -0.5  -1.4
constexpr int kRoutedTokens = 32;
static bool routed_form(const moe_shape *s) {
  const int most = s->E <= 64 ? 384 : s->E <= 128 ? 320 : s->E <= 256 ? 264 : 160;
  return s->T > 0 && s->T <= kRoutedTokens && s->E <= 512 && s->T * (s->k + 8) <= most &&
         small_lds_bytes(1, s->E, s->R) <= kSmallLds;
}
static int launch_routed(const moe_shape *s, const float *logits, int32_t *topk_idx, float *topk_w, const moe_dispatch *out,
                         hipStream_t st) {
  int ebits = 0, rbits = 0;
  while ((1 << ebits) < s->E) ++ebits;
  while ((1 << rbits) < s->R) ++rbits;
  const int32_t *none = nullptr;
  begin_launches();
#define MOE355_ROUTED(PER_)                                                                                         \
  do {                                                                                                              \
    static std::atomic<uint64_t> done{0};                                                                           \
    if (!allow_dynamic_lds(reinterpret_cast<const void *>(&dispatch_pairs_kernel<1, false, PER_>), (int)kSmallLds,  \
                           done))                                                                                   \
      return MOE_ERR_HIP;                                                                                           \
    hipLaunchKernelGGL((dispatch_pairs_kernel<1, false, PER_>), dim3(1), dim3(kSmallThreads),                       \
                       small_lds_bytes(1, s->E, s->R), st, logits, topk_w, topk_idx, s->T, s->E, s->k, s->R, s->T, 1, \
                       ebits, rbits, none, none, out->counts, out->offsets, out->rank_counts, out->rank_offsets,    \
                       out->perm, out->inv_perm, out->dedup_tok, out->dedup_mask, out->pair_to_dedup);              \
  } while (0)
  if (s->E <= 64) MOE355_ROUTED(1);
  else if (s->E <= 128) MOE355_ROUTED(2);
  else if (s->E <= 256) MOE355_ROUTED(4);
  else MOE355_ROUTED(8);
#undef MOE355_ROUTED
  return launch_status();
}

static bool dispatch_outputs_ok(const moe_dispatch *out) {
  return out && out->counts && out->offsets && out->perm && out->inv_perm && out->rank_counts && out->rank_offsets &&
         out->dedup_tok && out->dedup_mask && out->pair_to_dedup;
}

extern "C" int moe_build_dispatch(const moe_shape *shape, const int32_t *topk_idx, const moe_dispatch *out,
                                  void *workspace, size_t workspace_bytes, void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!topk_idx || !dispatch_outputs_ok(out)) return MOE_ERR_INVALID_ARG;
  if (!workspace || workspace_bytes < moe_dispatch_workspace_bytes(shape)) return MOE_ERR_WORKSPACE;
  return build_dispatch_launches(shape, topk_idx, out, static_cast<int32_t *>(workspace), (hipStream_t)stream);
}

// ------------------------------------------------------------------------------------------------
// The same call for callers that cannot allocate device memory (code under HIP graph capture, serving loops,
// harnesses that forbid hipMalloc): the chunk histograms live in a file-scope device array instead of a caller
// workspace.  Every GPU holds its own copy of the array at its own address; the address is looked up once per device
// (hipGetSymbolAddress with that device current) and kept.  In host code the array's name is only a handle for that
// lookup: kernels and copies always get the looked-up pointer.
// ------------------------------------------------------------------------------------------------
namespace moe355 {
constexpr int kStaticMaxCounters = MOE_NOALLOC_MAX_COUNTERS;  // limit on E + R
static __device__ __align__(256) unsigned char scratch[(size_t)kMaxChunks * kStaticMaxCounters * sizeof(int32_t)];
constexpr int kMaxDevices = 64;
static std::atomic<void *> g_scratch_ptr[kMaxDevices];  // zero-initialised: not looked up yet

// Device address of `scratch` on the current device (nullptr on failure).  Allocates nothing.
static void *scratch_on_current_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  void *p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (p) return p;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
    (void)hipGetLastError();
    return nullptr;
  }
  g_scratch_ptr[dev].store(p, std::memory_order_release);  // every thread looks up the same address
  return p;
}
}  // namespace moe355

extern "C" int moe_build_dispatch_noalloc(const moe_shape *shape, const int32_t *topk_idx, const moe_dispatch *out,
                                          void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (!topk_idx || !dispatch_outputs_ok(out)) return MOE_ERR_INVALID_ARG;
  if (shape->E + shape->R > kStaticMaxCounters) return MOE_ERR_UNSUPPORTED;  // beyond the static scratch
  void *ws = scratch_on_current_device();
  if (!ws) return MOE_ERR_HIP;
  // Nothing has to start at zero: the histogram kernel overwrites the rows of every chunk that exists and the
  // placement kernel ignores the others.
  return build_dispatch_launches(shape, topk_idx, out, static_cast<int32_t *>(ws), (hipStream_t)stream);
}

extern "C" int moe_step(const moe_shape *shape, const float *logits, const void *x, int32_t *topk_idx, float *topk_w,
                        const moe_dispatch *tables, void *dispatch_workspace, size_t dispatch_workspace_bytes,
                        const void *packed_gate_up, const void *packed_down, void *y, void *workspace,
                        size_t workspace_bytes, void *stream) {
  Derived dv;
  int rc = check_shape(shape, &dv);
  if (rc != MOE_OK) return rc;
  if (logits && topk_idx && topk_w && dispatch_outputs_ok(tables) && dispatch_workspace &&
      dispatch_workspace_bytes >= moe_dispatch_workspace_bytes(shape) && routed_form(shape)) {
    rc = launch_routed(shape, logits, topk_idx, topk_w, tables, (hipStream_t)stream);
  } else if ((rc = moe_route_topk(shape, logits, topk_idx, topk_w, stream)) == MOE_OK) {
    rc = moe_build_dispatch(shape, topk_idx, tables, dispatch_workspace, dispatch_workspace_bytes, stream);
  }
  if (rc != MOE_OK) return rc;
  return moe_fused_forward(shape, x, topk_idx, topk_w, tables, packed_gate_up, packed_down, y, workspace, workspace_bytes,
                           stream);
}
