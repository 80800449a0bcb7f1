// Token compaction by routing decision: deterministic stable partitions by
// prefix sums (no atomics decide any order).
//
//   attention: per (b, h), the ascending t of local and of full queries
//   experts  : per expert 1..E, the ascending assignment ids a = i*k + slot
#include "lists.hpp"

namespace tr {

// Blocks [0, nattn): attention lists of one (b, h), 1024 tokens a round; then
// nbe blocks: expert histograms of a chunk of assignments; then nslot blocks:
// a batch row's slots (kv_slots_rows); the rest: the attention output rows that
// no attention block writes, zeroed (skipped heads, i.e. any mode but local or
// full, and every head of a row whose sequence id lies outside the cache), a
// thread per (token, head) row.  All read the decisions alone.  (As launches
// of their own: 1.3B, 16384 tokens, lists 16 us in 256-token rounds, slots
// 12, zeroing 8; 410M, 333 tokens, 4.4 + 4 + 3.2.)
struct ListsArgs {
  const uint8_t *mode;
  const int32_t *eidx;
  int B, T, H, E1, Nk, nattn, nbe, nslot;
  int32_t *attn_cnt, *attn_idx, *hist;
  CacheView cv;
  const int32_t *seq_ids;
  const uint8_t *bit;
  int32_t *old_len;
  uint4 *o;  // rows of `chunks` 16-byte pieces
  int chunks;
  uint32_t pairs;
};
__global__ __launch_bounds__(1024) void lists_kernel(ListsArgs a) {
  __shared__ int wcnt[2][16];
  __shared__ int lh[64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int bid = blockIdx.x;
  const int T = a.T, H = a.H;
  if (bid < a.nattn) {
    const int b = bid / H, h = bid % H;
    int base[2] = {0, 0};
    for (int t0 = 0; t0 < T; t0 += 1024) {
      const int t = t0 + tid;
      const int m = t < T ? a.mode[(int64_t(b) * T + t) * H + h] : 0;
      uint64_t bal[2];
      bal[0] = __ballot(m == 1);
      bal[1] = __ballot(m == 2);
      if (lane < 2) wcnt[lane][w] = __popcll(bal[lane]);
      __syncthreads();
      int before[2] = {0, 0}, all[2] = {0, 0};
#pragma unroll
      for (int ww = 0; ww < 16; ++ww)
#pragma unroll
        for (int mm = 0; mm < 2; ++mm) {
          const int n = wcnt[mm][ww];
          before[mm] += ww < w ? n : 0;
          all[mm] += n;
        }
#pragma unroll
      for (int mm = 0; mm < 2; ++mm) {
        if (m == mm + 1)
          a.attn_idx[(int64_t(bid) * 2 + mm) * T + base[mm] + before[mm] +
                     __popcll(bal[mm] & lanemask_lt())] = t;
        base[mm] += all[mm];
      }
      __syncthreads();
    }
    if (tid < 2) a.attn_cnt[bid * 2 + tid] = tid ? base[1] : base[0];
    return;
  }
  bid -= a.nattn;
  if (bid < a.nbe) {
    static_assert(CHUNK == 1024, "one assignment a thread");
    if (tid < a.E1) lh[tid] = 0;  // E1 <= 64
    __syncthreads();
    const int i = bid * CHUNK + tid;
    if (i < a.Nk) atomicAdd(&lh[a.eidx[i]], 1);
    __syncthreads();
    if (tid < a.E1) a.hist[bid * a.E1 + tid] = lh[tid];
    return;
  }
  bid -= a.nbe;
  if (bid < a.nslot) {
    kv_slots_rows(a.cv, T, a.seq_ids, a.bit, a.old_len, bid);
    return;
  }
  bid -= a.nslot;
  const uint32_t pair = uint32_t(bid) * 1024u + uint32_t(tid);  // token * H + head
  if (pair >= a.pairs) return;
  const int b = int(pair / (uint32_t(H) * uint32_t(T)));
  const int s = a.seq_ids ? a.seq_ids[b] : b;
  const int m = a.mode[pair];
  if ((m != TRIROUTE_LOCAL && m != TRIROUTE_FULL) || s < 0 || s >= a.cv.n_seq) {
    uint4 *row = a.o + size_t(pair) * a.chunks;
    for (int c = 0; c < a.chunks; ++c) row[c] = make_uint4(0u, 0u, 0u, 0u);
  }
}

__global__ __launch_bounds__(256) void compact_scatter_kernel(ScatterJob J) {
  scatter_chunk(J, blockIdx.x);
}

int compact_hist_ints(int N, int k, int E1) { return ((N * k + CHUNK - 1) / CHUNK) * E1; }

ScatterJob make_scatter_job(const triroute_cfg &cfg, int N, const int32_t *eidx,
                            const triroute_compaction &c, const int32_t *hist) {
  ScatterJob j;
  j.eidx = eidx;
  j.hist = hist;
  j.E1 = cfg.n_experts + 1;
  j.Nk = N * cfg.top_k;
  j.nbe = (j.Nk + CHUNK - 1) / CHUNK;
  j.rows = c.exp_rows;
  j.exp_cnt = c.exp_cnt;
  j.exp_off = c.exp_off;
  return j;
}

hipError_t launch_lists(const triroute_cfg &cfg, int B, int T, const uint8_t *mode,
                        const int32_t *eidx, const triroute_compaction &c, int32_t *hist,
                        bool attn_lists, const AppendJob *app, void *o, hipStream_t st) {
  ListsArgs a{};
  a.mode = mode;
  a.eidx = eidx;
  a.B = B;
  a.T = T;
  a.H = cfg.n_heads;
  a.E1 = cfg.n_experts + 1;
  a.Nk = B * T * cfg.top_k;
  a.nattn = attn_lists ? B * a.H : 0;
  a.nbe = (a.Nk + CHUNK - 1) / CHUNK;
  a.attn_cnt = c.attn_cnt;
  a.attn_idx = c.attn_idx;
  a.hist = hist;
  int zero_blocks = 0;
  if (app) {
    a.cv = app->cv;
    a.seq_ids = app->seq_ids;
    a.bit = app->bit;
    a.old_len = app->ws.old_len;
    a.nslot = app->slots ? B : 0;
    if (o) {
      const int64_t pairs = int64_t(B) * T * a.H;
      a.chunks = cfg.head_dim * (cfg.act == TRIROUTE_BF16 ? 2 : 4) / 16;
      if (pairs >= (int64_t(1) << 31)) {
        const hipError_t e = launch_fill_u32(o, pairs * a.chunks * 4, 0u, st);  // every row
        if (e != hipSuccess) return e;
      } else {
        a.o = (uint4 *)o;
        a.pairs = uint32_t(pairs);
        zero_blocks = int((pairs + 1023) / 1024);
      }
    }
  }
  lists_kernel<<<dim3(unsigned(a.nattn + a.nbe + a.nslot + zero_blocks)), 1024, 0, st>>>(a);
  return hipGetLastError();
}

hipError_t launch_scatter(const ScatterJob &j, hipStream_t st) {
  compact_scatter_kernel<<<j.nbe, 256, 0, st>>>(j);
  return hipGetLastError();
}

hipError_t launch_compact(const triroute_cfg &cfg, int B, int T, const uint8_t *mode,
                          const int32_t *eidx, const triroute_compaction &c, int32_t *hist,
                          hipStream_t st) {
  const hipError_t e = launch_lists(cfg, B, T, mode, eidx, c, hist, true, nullptr, nullptr, st);
  if (e != hipSuccess) return e;
  return launch_scatter(make_scatter_job(cfg, B * T, eidx, c, hist), st);
}

}  // namespace tr
