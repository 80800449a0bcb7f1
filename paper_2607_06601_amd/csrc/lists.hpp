// Blocks of the routing lists and of the append's bookkeeping, shared by the
// kernels that run them: alone in the stage calls, and in a layer beside the
// blocks of another kernel that does not depend on them (each is a short chain
// in a few blocks, and a launch of its own for each would leave the chip idle
// for its length: of these 2.5 to 5 us each, 16 at 16384 tokens).  A layer
// measured with the launches of its own and with the shared ones: 160M decode
// of one row 70.9 -> 67.6 us, 410M decode of 64 rows 130 -> 127.7, 410M prefill
// of 333 tokens 163.5 -> 152.2, a 1.3B prefill chunk of 2000 736 -> 727.
#pragma once

#include "kernels.hpp"

namespace tr {

constexpr int CHUNK = 1024;  // assignments per expert block

// Per batch row: the slot of each new token in its width pool (its rank
// among the row's earlier tokens of that width, after the pool's current
// length), its position in the pool's position array, the new lengths, and
// the pool lengths before the append.  One block of 16 waves per row walks
// the row's tokens 1024 at a time (ballot counts per wave, then per block).
__device__ __forceinline__ void kv_slots_rows(const CacheView &cv, int T, const int32_t *seq_ids,
                                              const uint8_t *bit, int32_t *old_len, int b) {
  constexpr int NW = 16;
  __shared__ int wc[4][NW];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int s = seq_ids ? seq_ids[b] : b;
  if (s < 0 || s >= cv.n_seq) {
    if (tid == 0) atomicOr(cv.status, int(TRIROUTE_CACHE_BAD_SEQ));
    if (tid < 4) old_len[b * 4 + tid] = -1;
    return;
  }
  const int len0 = cv.seq_len[s];
  if (len0 + T > cv.capacity) {
    if (tid == 0) atomicOr(cv.status, int(TRIROUTE_CACHE_OVERFLOW));
    if (tid < 4) old_len[b * 4 + tid] = -1;
    return;
  }
  int run[4];
#pragma unroll
  for (int bi = 0; bi < 4; ++bi) run[bi] = cv.pool_len[s * 4 + bi];
  if (cv.PT) {
    // paged: count the row's tokens per width, then take the pages the
    // pools grow into from the free stacks (thread bi for width bi)
    __shared__ int cnt_s[4], fail_s;
    if (tid < 4) cnt_s[tid] = 0;
    if (tid == 0) fail_s = 0;
    __syncthreads();
    for (int t0 = 0; t0 < T; t0 += 64 * NW) {
      const int t = t0 + tid;
      const int bi = t < T ? int(bit[int64_t(b) * T + t]) : -1;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint64_t bq = __ballot(bi == q);
        if (lane == 0 && bq) atomicAdd(&cnt_s[q], __popcll(bq));  // a count: order does not matter
      }
    }
    __syncthreads();
    if (tid < 4) {
      const int bi = tid, per = cv.PT * cv.TS;
      const int need = (run[bi] + cnt_s[bi] + per - 1) / per;
      int32_t *held = cv.alloc + s * 4 + bi;
      const int have = *held;
      if (need > have) {
        const int k = need - have;
        const int top = atomicSub(cv.free_top + bi, k);
        if (need > cv.max_pages || top - k < 0) {
          atomicAdd(cv.free_top + bi, k);  // give the claim back
          atomicOr(&fail_s, 1);
        } else {
          for (int q = 0; q < k; ++q)
            cv.page_table[(int64_t(s) * 4 + bi) * cv.max_pages + have + q] = cv.free_list[bi][top - k + q];
          *held = need;
        }
      }
    }
    __syncthreads();
    if (fail_s) {
      if (tid == 0) atomicOr(cv.status, int(TRIROUTE_CACHE_OVERFLOW));
      if (tid < 4) old_len[b * 4 + tid] = -1;
      return;
    }
  }
  if (tid < 4) old_len[b * 4 + tid] = run[tid];
  for (int t0 = 0; t0 < T; t0 += 64 * NW) {
    const int t = t0 + tid;
    const int bi = t < T ? int(bit[int64_t(b) * T + t]) : -1;
    uint64_t bal[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bal[q] = __ballot(bi == q);
    if (lane < 4) wc[lane][w] = __popcll(bal[lane]);
    __syncthreads();
    if (bi >= 0) {
      int slot = run[bi] + __popcll(bal[bi] & lanemask_lt());
      for (int ww = 0; ww < w; ++ww) slot += wc[bi][ww];
      cv.pos_at(s, bi, slot) = len0 + t;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) run[q] += wc[q][ww];
    __syncthreads();
  }
  if (tid == 0) {
#pragma unroll
    for (int bi = 0; bi < 4; ++bi) cv.pool_len[s * 4 + bi] = run[bi];
    cv.seq_len[s] = len0 + T;
  }
}

// Stable scatter of assignment ids into per-expert lists.  Block j first
// forms each expert's first output position for its chunk from the chunk
// histograms (all chunks' totals give the expert offsets; block 0 also
// writes the counts and offsets).
__device__ __forceinline__ void scatter_chunk(const ScatterJob &J, int j) {
  const int32_t *eidx = J.eidx, *hist = J.hist;
  const int nbe = J.nbe, E1 = J.E1, Nk = J.Nk;
  int32_t *rows = J.rows, *exp_cnt = J.exp_cnt, *exp_off = J.exp_off;
  __shared__ int wc[4][64];
  __shared__ int run[64], tot[64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid < E1) {
    int before = 0, all = 0;
    for (int j0 = 0; j0 < nbe; j0 += 16) {  // 16 loads in flight
      int v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = hist[min(j0 + i, nbe - 1) * E1 + tid];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        before += j0 + i < j ? v[i] : 0;
        all += j0 + i < nbe ? v[i] : 0;
      }
    }
    run[tid] = before;
    tot[tid] = all;
  }
  __syncthreads();
  if (tid < E1) {
    int start = 0;  // lists of experts 1 .. tid - 1 come first
    for (int ee = 1; ee < tid; ++ee) start += tot[ee];
    if (tid >= 1) run[tid] += start;
    if (j == 0) {
      exp_cnt[tid] = tot[tid];
      exp_off[tid] = tid == 0 ? 0 : start + tot[tid];
    }
  }
  __syncthreads();
  // (sub rounds past the last assignment are skipped: the bound is uniform
  // over the block, so every barrier below is still reached by all threads)
  for (int sub = 0; sub < CHUNK && j * CHUNK + sub < Nk; sub += 256) {
    const int a = j * CHUNK + sub + tid;
    const int e = a < Nk ? eidx[a] : -1;
    int rank = 0;
    for (int ee = 1; ee < E1; ++ee) {
      uint64_t bal = __ballot(e == ee);
      if (e == ee) rank = __popcll(bal & lanemask_lt());
      if (lane == 0) wc[w][ee] = __popcll(bal);
    }
    __syncthreads();
    if (e >= 1) {
      int pos = run[e] + rank;
      for (int ww = 0; ww < w; ++ww) pos += wc[ww][e];
      rows[pos] = a;
    }
    __syncthreads();
    for (int ee = tid; ee < E1; ee += 256)
      if (ee >= 1) run[ee] += wc[0][ee] + wc[1][ee] + wc[2][ee] + wc[3][ee];
    __syncthreads();
  }
}

// Few assignments (one chunk) and no attention lists (decode): the expert
// lists by one block of 256 threads, histogram, offsets and the same stable
// scatter as above (so the same lists).
__device__ __forceinline__ void experts_one(const ScatterJob &J) {
  const int32_t *eidx = J.eidx;
  const int E1 = J.E1, Nk = J.Nk;
  int32_t *rows = J.rows, *exp_cnt = J.exp_cnt, *exp_off = J.exp_off;
  __shared__ int lh[64], run[64];
  __shared__ int wc[4][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid < E1) lh[tid] = 0;  // E1 <= 64
  __syncthreads();
  for (int a = tid; a < Nk; a += 256) atomicAdd(&lh[eidx[a]], 1);
  __syncthreads();
  if (tid < E1) {
    int start = 0;  // lists of experts 1 .. tid - 1 come first
    for (int ee = 1; ee < tid; ++ee) start += lh[ee];
    run[tid] = start;
    exp_cnt[tid] = lh[tid];
    exp_off[tid] = tid == 0 ? 0 : start + lh[tid];
  }
  __syncthreads();
  for (int sub = 0; sub < Nk; sub += 256) {  // block-uniform bound: every barrier is reached
    const int a = sub + tid;
    const int e = a < Nk ? eidx[a] : -1;
    int rank = 0;
    for (int ee = 1; ee < E1; ++ee) {
      const uint64_t bal = __ballot(e == ee);
      if (e == ee) rank = __popcll(bal & lanemask_lt());
      if (lane == 0) wc[w][ee] = __popcll(bal);
    }
    __syncthreads();
    if (e >= 1) {
      int pos = run[e] + rank;
      for (int ww = 0; ww < w; ++ww) pos += wc[ww][e];
      rows[pos] = a;
    }
    __syncthreads();
    if (tid >= 1 && tid < E1) run[tid] += wc[0][tid] + wc[1][tid] + wc[2][tid] + wc[3][tid];
    __syncthreads();
  }
}

}  // namespace tr
