// Dense and grouped GEMMs of the layer for the fp32 activation dtype (the bf16
// path is gemm_mfma.hip), C = A B^T with both operands K-contiguous, and
// their fused epilogues:
//   QKV   : [n1] x [Wq;Wk;Wv]^T, rotate-half RoPE on q and k
//   O-proj: xt = x + o Wo^T
//   MoE-1 : H = silu(n2 Wgate_e^T) * (n2 Wup_e^T) per expert e (paper Sec.
//           3.2 (B), SwiGLU); n2, H and Y hold one row per entry of the
//           expert lists, in list order (the lists lie back to back)
//   MoE-2 : Y = H Wdown_e^T
// The QKV products are sums of fused multiply-adds in the order of k (the
// cache stores fp32 keys and values verbatim, so their bits do not depend on
// a tile choice); the others run on fp32 MFMA (16x16x4), operands straight
// from global memory to registers.  Grouped problems map block -> (expert, row tile) from the device-side
// expert counts, so no host synchronisation is needed.
#include "kernels.hpp"

namespace tr {

namespace {

// Columns are taken in units of 32: a unit's first and second 16 columns are
// partners (the halves of 16 rotation pairs, gate and up of 16 expert units,
// or plainly the next 16 columns), so that a lane holds both of a pair.
struct Tile {
  int m0, u0, mvalid, e, p0;  // p0: first row of the operand, m0: of the tile within it
};

// ------------------------------------------------------------------ problems
struct QkvProb {
  const float *n1, *Wq, *Wk, *Wv;
  float *q, *k, *v;
  const float2 *rope;  // (cos, sin) of token row, pair j at row * dh / 2 + j
  int N, d, H, Hkv, dh, K;
  __device__ bool map(int bx, int BM, Tile &t) const {
    t.m0 = bx * BM;
    t.mvalid = min(BM, N - t.m0);
    t.e = t.p0 = 0;
    return t.mvalid > 0;
  }
  __device__ const float *a_row(const Tile &t, int r) const { return n1 + int64_t(t.m0 + r) * d; }
  __device__ int head_col(int u, int c) const {  // first-half column of pair 16 u + c
    const int hd = dh >> 1, P = 16 * u + c;
    return P / hd * dh + P % hd;
  }
  __device__ const float *b_row(const Tile &, int u, int c, int half) const {
    int gc = head_col(u, c) + half * (dh >> 1);
    const int Hd = H * dh, Kd = Hkv * dh;
    if (gc < Hd) return Wq + int64_t(gc) * d;
    gc -= Hd;
    if (gc < Kd) return Wk + int64_t(gc) * d;
    return Wv + int64_t(gc - Kd) * d;
  }
  __device__ void store(const Tile &t, int r, int u, int c, float x1, float x2) const {
    const int Hd = H * dh, Kd = Hkv * dh, hd = dh >> 1, gc = head_col(u, c), row = t.m0 + r;
    float *out = q;
    int ld = Hd, col = gc;
    float y1 = x1, y2 = x2;
    if (gc >= Hd + Kd) {
      out = v; ld = Kd; col = gc - Hd - Kd;
    } else {
      if (gc >= Hd) { out = k; ld = Kd; col = gc - Hd; }
      const float2 cs = rope[int64_t(row) * hd + col % dh];
      y1 = x1 * cs.x - x2 * cs.y;
      y2 = x1 * cs.y + x2 * cs.x;
    }
    float *o = out + int64_t(row) * ld + col;
    o[0] = y1;
    o[hd] = y2;
  }
};

struct OprojProb {
  const float *o, *Wo, *x;
  float *xt;
  int N, d, K;
  __device__ bool map(int bx, int BM, Tile &t) const {
    t.m0 = bx * BM;
    t.mvalid = min(BM, N - t.m0);
    t.e = t.p0 = 0;
    return t.mvalid > 0;
  }
  __device__ const float *a_row(const Tile &t, int r) const { return o + int64_t(t.m0 + r) * K; }
  __device__ const float *b_row(const Tile &, int u, int c, int half) const {
    return Wo + int64_t(32 * u + 16 * half + c) * K;
  }
  __device__ void store(const Tile &t, int r, int u, int c, float y1, float y2) const {
    const int64_t at = int64_t(t.m0 + r) * d + 32 * u + c;
    xt[at] = x[at] + y1;
    xt[at + 16] = x[at + 16] + y2;
  }
};

// Map a linear row-tile index to (expert e >= 1, tile within e).
__device__ __forceinline__ bool map_grouped(int bx, int BM, const int32_t *cnt,
                                            const int32_t *off, int E, Tile &t) {
  int rem = bx;
  for (int e = 1; e <= E; ++e) {
    const int c = cnt[e];
    const int nt = (c + BM - 1) / BM;
    if (rem < nt) {
      t.e = e;
      t.p0 = off[e - 1] + rem * BM;
      t.mvalid = min(BM, c - rem * BM);
      t.m0 = 0;
      return true;
    }
    rem -= nt;
  }
  return false;
}

struct Moe1Prob {
  const float *n2, *Wg, *Wu;
  float *Hm;
  const int32_t *cnt, *off;
  int E, d, dff, K;
  __device__ bool map(int bx, int BM, Tile &t) const { return map_grouped(bx, BM, cnt, off, E, t); }
  __device__ const float *a_row(const Tile &t, int r) const { return n2 + int64_t(t.p0 + r) * d; }
  __device__ const float *b_row(const Tile &t, int u, int c, int half) const {
    return (half ? Wu : Wg) + (int64_t(t.e - 1) * dff + 16 * u + c) * d;
  }
  __device__ void store(const Tile &t, int r, int u, int c, float g, float up) const {
    Hm[int64_t(t.p0 + r) * dff + 16 * u + c] = g / (1.0f + expf(-g)) * up;
  }
};

struct Moe2Prob {
  const float *Hm, *Wd;
  float *Y;
  const int32_t *cnt, *off;
  int E, d, dff, K;
  __device__ bool map(int bx, int BM, Tile &t) const { return map_grouped(bx, BM, cnt, off, E, t); }
  __device__ const float *a_row(const Tile &t, int r) const { return Hm + int64_t(t.p0 + r) * dff; }
  __device__ const float *b_row(const Tile &t, int u, int c, int half) const {
    return Wd + (int64_t(t.e - 1) * d + 32 * u + 16 * half + c) * dff;
  }
  __device__ void store(const Tile &t, int r, int u, int c, float y1, float y2) const {
    float *y = Y + int64_t(t.p0 + r) * d + 32 * u + c;
    y[0] = y1;
    y[16] = y2;
  }
};

// -------------------------------------------------------------- fp32 kernel
typedef float f32x4g __attribute__((ext_vector_type(4)));

// A wave makes a 32 x 32 tile: two row blocks by the two halves of a unit.
// Lane l holds, of row l % 16 of a block, k 4 (l / 16) .. + 3 of each 16-wide
// step as one 16-byte load; component i of both operands feeds MFMA i, so
// the products of a step cover its 16 k in an order that both sides share.
// DEPTH steps of loads are in flight: with few blocks the kernel waits on
// nothing else.
//   KS 4: a block is one such tile, its four waves a quarter of K each, added
//         in wave order through LDS: problems that would leave CUs idle.
//   KS 1: a block is 2 x 2 tiles over all of K: the waves share operand rows
//         through the vector cache.
// (64 x 128 tiles of vector FMAs from LDS gave the small fp32 layer's
// products, 128 tokens, 4 to 48 blocks: O-projection 38, gate/up 34, down
// 66 us; now 5, 6 and 7 us.)
template <class P, int KS>
__global__ __launch_bounds__(256) void gemm_f32_kernel(P p, int units) {
  constexpr int BM = KS == 1 ? 64 : 32, DEPTH = 4;
  __shared__ float red[KS == 1 ? 1 : 4][16][64];
  Tile t;
  if (!p.map(blockIdx.x, BM, t)) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, kq = 4 * (lane >> 4);
  const int r0 = KS == 1 ? 32 * (wave >> 1) : 0;
  const int u = KS == 1 ? 2 * blockIdx.y + (wave & 1) : int(blockIdx.y);
  if (KS == 1 && (u >= units || r0 >= t.mvalid)) return;
  const int kn = p.K / KS, kb = KS == 1 ? 0 : wave * kn;
  const float *src[4];  // rows past the tile's read its first one: never stored
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = r0 + 16 * h + c;
    src[h] = p.a_row(t, r < t.mvalid ? r : 0) + kb + kq;
    src[2 + h] = p.b_row(t, u, c, h) + kb + kq;
  }
  f32x4g acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4g{0.f, 0.f, 0.f, 0.f};
  f32x4g buf[DEPTH][4];
  auto load = [&](int s, int k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) buf[s][i] = *(const f32x4g *)(src[i] + k);
  };
#pragma unroll
  for (int s = 0; s < DEPTH; ++s)
    if (16 * s < kn) load(s, 16 * s);
  for (int k = 0; k < kn; k += 16 * DEPTH) {
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
      if (k + 16 * s >= kn) break;
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(buf[s][i][x], buf[s][2 + j][x],
                                                             acc[i][j], 0, 0, 0);
      if (k + 16 * (s + DEPTH) < kn) load(s, k + 16 * (s + DEPTH));
    }
  }
  if constexpr (KS == 1) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int r = r0 + 16 * i + kq + x;
        if (r < t.mvalid) p.store(t, r, u, c, acc[i][0][x], acc[i][1][x]);
      }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int x = 0; x < 4; ++x) red[wave][8 * i + 4 * j + x][lane] = acc[i][j][x];
    __syncthreads();
    // wave w finishes accumulator rows x = w
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float y[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int at = 8 * i + 4 * j + wave;
        y[j] = ((red[0][at][lane] + red[1][at][lane]) + red[2][at][lane]) + red[3][at][lane];
      }
      const int r = 16 * i + kq + wave;
      if (r < t.mvalid) p.store(t, r, u, c, y[0], y[1]);
    }
  }
}

// C tile of 16 TM x 16 TM (TM / 2 units of columns), TM x TM outputs a thread
// (rows and columns 16 apart), each one chain of fused multiply-adds in the
// order of k: 32-wide K steps through two LDS buffers, the next step's loads
// in registers meanwhile.  Rows of 36 floats put the 16 columns that a
// quarter wave reads at once in different banks.  TM 4 balances LDS reads
// and FMAs; TM 2 gives small problems four times the blocks (the small fp32
// layer, 128 tokens: QKV 48 us on 64 x 128 tiles, now 9).
template <class P, int TM>
__global__ __launch_bounds__(256) void gemm_f32_chain_kernel(P p, int units) {
  constexpr int BM = 16 * TM, BK = 32, LD = BK + 4, LPT = TM / 2;  // 16-byte loads a thread and operand
  __shared__ __align__(16) float As[2][BM][LD], Bs[2][BM][LD];
  Tile t;
  if (!p.map(blockIdx.x, BM, t)) return;
  const int tid = threadIdx.x, tr = tid >> 4, tc = tid & 15;
  const int u0 = blockIdx.y * (TM / 2);
  const float *asrc[LPT], *bsrc[LPT];
  const int lr = tid >> 3, lk = 4 * (tid & 7);  // staged row (of 32) and k
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int r = lr + 32 * i;  // row of A; column of B: unit r / 32, half r / 16 % 2
    asrc[i] = p.a_row(t, r < t.mvalid ? r : 0) + lk;
    bsrc[i] = p.b_row(t, min(u0 + (r >> 5), units - 1), r & 15, (r >> 4) & 1) + lk;
  }
  float4 ra[LPT], rb[LPT];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      ra[i] = *(const float4 *)(asrc[i] + k0);
      rb[i] = *(const float4 *)(bsrc[i] + k0);
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      *(float4 *)&As[buf][lr + 32 * i][lk] = ra[i];
      *(float4 *)&Bs[buf][lr + 32 * i][lk] = rb[i];
    }
  };
  float acc[TM][TM];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = 0.f;
  fetch(0);
  put(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < p.K; k0 += BK) {
    const bool more = k0 + BK < p.K;
    if (more) fetch(k0 + BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      float a[TM][4], b[TM][4];
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        *(float4 *)a[i] = *(const float4 *)&As[buf][tr + 16 * i][kk];
        *(float4 *)b[i] = *(const float4 *)&Bs[buf][tc + 16 * i][kk];
      }
#pragma unroll
      for (int x = 0; x < 4; ++x)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TM; ++j) acc[i][j] = fmaf(a[i][x], b[j][x], acc[i][j]);
    }
    if (more) put(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TM / 2; ++j)
      if (tr + 16 * i < t.mvalid && u0 + j < units)
        p.store(t, tr + 16 * i, u0 + j, tc, acc[i][2 * j], acc[i][2 * j + 1]);
}

// ------------------------------------------------------------------ launchers
// m32, m64: row tiles of 32 / 64 rows (bounds, for grouped problems); units
// of 32 columns.  Below 512 tiles of 64 x 64 (two blocks a CU) K is split
// over the block's waves.
template <class P>
hipError_t run_gemm(const P &p, int m32, int m64, int units, hipStream_t st) {
  if (m32 <= 0 || units <= 0) return hipGetLastError();
  const int u2 = (units + 1) / 2;
  if (int64_t(m64) * u2 >= 512)
    gemm_f32_kernel<P, 1><<<dim3(m64, u2), 256, 0, st>>>(p, units);
  else
    gemm_f32_kernel<P, 4><<<dim3(m32, units), 256, 0, st>>>(p, units);
  return hipGetLastError();
}

}  // namespace

// The rotation table (one entry per token and pair serves every q and k
// head of the token), when the first RMSNorm did not already write it.
__global__ __launch_bounds__(256) void rope_table_kernel(int N, const RopeJob r) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (i >= int64_t(N) * r.hd) return;
  r.tab[i] = rope_entry(r, int(i / r.hd), int(i % r.hd));
}

RopeJob make_rope_job(const triroute_cfg &cfg, int Tq, const int32_t *pos_base,
                      const int32_t *pos_idx, int n_base, float *tab) {
  RopeJob r;
  r.pos_base = pos_base;
  r.pos_idx = pos_idx;
  r.n_base = n_base;
  r.Tq = Tq;
  r.hd = cfg.head_dim / 2;
  r.tab = (float2 *)tab;
  for (int j = 0; j < 64; ++j)
    r.inv_freq[j] = j < r.hd ? pow(double(cfg.rope_theta), -2.0 * j / double(cfg.head_dim)) : 0.0;
  return r;
}

size_t qkv_rope_floats(const triroute_cfg &cfg, int N) { return size_t(N) * cfg.head_dim; }

static hipError_t qkv_f32(const triroute_cfg &cfg, int B, int Tq, const void *n1,
                          const triroute_dense_w &w, const float *rope, void *q, void *k, void *v,
                          hipStream_t st) {
  QkvProb p;
  p.n1 = (const float *)n1;
  p.Wq = (const float *)w.Wq;
  p.Wk = (const float *)w.Wk;
  p.Wv = (const float *)w.Wv;
  p.q = (float *)q;
  p.k = (float *)k;
  p.v = (float *)v;
  p.rope = (const float2 *)rope;
  p.N = B * Tq;
  p.d = cfg.d_model;
  p.H = cfg.n_heads;
  p.Hkv = cfg.n_kv_heads;
  p.dh = cfg.head_dim;
  p.K = cfg.d_model;
  const int units = (cfg.n_heads + 2 * cfg.n_kv_heads) * cfg.head_dim / 32;
  const int m64 = (p.N + 63) / 64, u2 = (units + 1) / 2;
  if (int64_t(m64) * u2 >= 512)  // two 64 x 64 tiles a CU
    gemm_f32_chain_kernel<QkvProb, 4><<<dim3(m64, u2), 256, 0, st>>>(p, units);
  else
    gemm_f32_chain_kernel<QkvProb, 2><<<dim3((p.N + 31) / 32, units), 256, 0, st>>>(p, units);
  return hipGetLastError();
}

hipError_t launch_qkv(const triroute_cfg &cfg, int B, int Tq, const void *n1,
                      const triroute_dense_w &w, const int32_t *pos_base, const int32_t *pos_idx,
                      int n_base, void *q, void *k, void *v, float *rope, bool rope_ready,
                      hipStream_t st) {
  const int N = B * Tq;
  if (!rope_ready) {
    const RopeJob r = make_rope_job(cfg, Tq, pos_base, pos_idx, n_base, rope);
    const int64_t n = int64_t(N) * r.hd;
    rope_table_kernel<<<dim3(unsigned((n + 255) / 256)), 256, 0, st>>>(N, r);
  }
  return cfg.act == TRIROUTE_BF16 ? mfma_qkv(cfg, B, Tq, n1, w, rope, q, k, v, st)
                                  : qkv_f32(cfg, B, Tq, n1, w, rope, q, k, v, st);
}

static hipError_t oproj_f32(const triroute_cfg &cfg, int N, const void *x, const void *o,
                            const triroute_dense_w &w, void *xt, hipStream_t st) {
  OprojProb p;
  p.o = (const float *)o;
  p.Wo = (const float *)w.Wo;
  p.x = (const float *)x;
  p.xt = (float *)xt;
  p.N = N;
  p.d = cfg.d_model;
  p.K = cfg.n_heads * cfg.head_dim;
  return run_gemm(p, (N + 31) / 32, (N + 63) / 64, p.d / 32, st);
}

hipError_t launch_oproj(const triroute_cfg &cfg, int N, const void *x, const void *o,
                        const triroute_dense_w &w, void *xt, hipStream_t st) {
  return cfg.act == TRIROUTE_BF16 ? mfma_oproj(cfg, N, x, o, w, xt, st)
                                  : oproj_f32(cfg, N, x, o, w, xt, st);
}

static hipError_t moe_gemms_f32(const triroute_cfg &cfg, int N, const void *n2,
                                const triroute_moe_w &w, const triroute_compaction &c, void *Hm,
                                float *Y, hipStream_t st) {
  const int E = cfg.n_experts, k = cfg.top_k, d = cfg.d_model, dff = cfg.d_ff;
  const int Nk = N * k;
  Moe1Prob p1;
  p1.n2 = (const float *)n2;
  p1.Wg = (const float *)w.Wgate;
  p1.Wu = (const float *)w.Wup;
  p1.Hm = (float *)Hm;
  p1.cnt = c.exp_cnt;
  p1.off = c.exp_off;
  p1.E = E;
  p1.d = d;
  p1.dff = dff;
  p1.K = d;
  hipError_t err = run_gemm(p1, Nk / 32 + E, Nk / 64 + E, dff / 16, st);
  if (err != hipSuccess) return err;
  Moe2Prob p2;
  p2.Hm = (const float *)Hm;
  p2.Wd = (const float *)w.Wdown;
  p2.Y = Y;
  p2.cnt = c.exp_cnt;
  p2.off = c.exp_off;
  p2.E = E;
  p2.d = d;
  p2.dff = dff;
  p2.K = dff;
  return run_gemm(p2, Nk / 32 + E, Nk / 64 + E, d / 32, st);
}

hipError_t launch_moe_gemms(const triroute_cfg &cfg, int N, const void *n2,
                            const triroute_moe_w &w, const triroute_compaction &c, void *Hm,
                            float *Y, hipStream_t st) {
  return cfg.act == TRIROUTE_BF16 ? mfma_moe(cfg, N, n2, w, c, Hm, Y, st)
                                  : moe_gemms_f32(cfg, N, n2, w, c, Hm, Y, st);
}

}  // namespace tr
