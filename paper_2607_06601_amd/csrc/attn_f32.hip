// Routed attention over the mixed-width cache for the fp32 activation dtype
// (the bf16 path is attn_mfma.hip), one wave per query.  Paper Sec. 3.2 (A):
// query head h of a token at position P reads kv head h / (H / Hkv); skip -> 0,
// local -> keys [P - w + 1, P], full -> [0, P]; softmax(q k^T / sqrt(dh)) v over
// the dequantized cache, the token's own key included, in fp32 throughout.
//
// Few queries over short ranges: the launch is bound by the latency of one
// wave's chain, so a wave takes a whole tile (4096 / dh slots) per step: for
// the scores a lane owns a slot (dh 128: half of its channels), for P V a
// channel, and each side's codes are loaded together.  (A key at a time, with
// a wave-wide sum per key and a binary search per pool, took 149 us for 128
// tokens of 4 heads over up to 128 keys; this takes 19 us.)
#include <type_traits>

#include "kernels.hpp"

namespace tr {

namespace {

struct AttnQuery {
  int row;  // token row in q / o / mode
  int s;    // cache sequence
  int P;    // query position
  int h, m;
};

// A wave's LDS: the scaled query, the weights of the tile's slots and the
// scale and zero of their V groups.  (Values are dequantised one by one:
// summing codes and zeros apart would leave a difference of two large sums.)
struct WaveMem {
  float q[128];
  float p[64];
  float s[4][64], z[4][64];
};

// Field f (8 elements) of the lane record at rec, bp bits an element.
template <int BP>
__device__ __forceinline__ void field8(const uint8_t *rec, int f, float (&v)[8]) {
  const uint32_t *w = (const uint32_t *)rec;
  if constexpr (BP == 2) {
    const uint32_t x = w[f >> 1] >> (2 * (f & 1));
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = float((x >> (4 * j)) & 3u);
  } else if constexpr (BP == 4) {
    const uint32_t x = w[f];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = float((x >> (8 * (j & 3) + 4 * (j >> 2))) & 15u);
  } else if constexpr (BP == 8) {
    const uint2 x = *(const uint2 *)(w + 2 * f);
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = float(((j < 4 ? x.x : x.y) >> (8 * (j & 3))) & 255u);
  } else {
    load8((const float *)rec + 8 * f, v);
  }
}

__device__ __forceinline__ float2 scale_zero(const uint8_t *p) {
  const uint32_t w = *(const uint32_t *)p;
  const uint16_t sb = uint16_t(w), zb = uint16_t(w >> 16);
  return make_float2(float(*(const _Float16 *)&sb), float(*(const _Float16 *)&zb));
}

template <int DH>
struct AttnState {
  float m = -INFINITY, l = 0.f;  // l: this lane's slots
  float acc[DH / 64];            // channels lane, lane + 64
};

// One tile of pool width index BI: slots of [0, n) with a position in [lo, hi].
template <int DH, int BI>
__device__ __forceinline__ void attend_tile(AttnState<DH> &st, WaveMem &mem, const CacheView &cv,
                                            const uint8_t *tp, const int32_t *pos, int n, int lo,
                                            int hi) {
  constexpr int BP = BI < 3 ? 2 << BI : 32, TS = 4096 / DH, KS = DH / 32, CB = DH / 16;
  constexpr bool Q = BI < 3;
  const int lane = threadIdx.x & 63, slot = lane & (TS - 1), c0 = TS == 64 ? 0 : 64 * (lane >> 5);
  const int G = cv.G, NG = DH / G;
  // ---- scores: slot's channels c0 .. c0 + 63, in runs of 8
  const int ps = slot < n ? pos[slot] : -1;
  const bool in = ps >= lo && ps <= hi;  // lo >= 0
  float kv[8][8];
  float2 ksz[2];
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    const int c = c0 + 8 * r;
    field8<BP>(tp + (((c >> 3) & 3) * 16 + (slot & 15)) * 8 * BP, (slot >> 4) * KS + (c >> 5), kv[r]);
  }
  if constexpr (Q) {  // G is 32 or 64: at most two groups in the lane's 64 channels
    ksz[0] = scale_zero(tp + cv.k_sz_off(BI) + (slot * NG + c0 / G) * 4);
    ksz[1] = scale_zero(tp + cv.k_sz_off(BI) + (slot * NG + (c0 + 32) / G) * 4);
  }
  float sc = 0.f;
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    float q[8];
    load8(mem.q + c0 + 8 * r, q);
#pragma unroll
    for (int j = 0; j < 8; ++j)
      sc = fmaf(q[j], Q ? fmaf(kv[r][j], ksz[r >> 2].x, ksz[r >> 2].y) : kv[r][j], sc);
  }
  if constexpr (TS == 32) sc += __shfl_xor(sc, 32, 64);
  if (!in) sc = -INFINITY;
  const uint64_t live = __ballot(in);
  if (!live) return;
  const float mn = fmaxf(st.m, wave_max(sc));
  const float corr = expf(st.m - mn), p = in ? expf(sc - mn) : 0.f;
  st.m = mn;
  st.l = st.l * corr + p;
  if (lane < TS) {
    mem.p[slot] = p;
    if constexpr (Q) {
      for (int g = 0; g < NG; ++g) {  // (a slot out of range may hold anything)
        const float2 sz = scale_zero(tp + cv.v_sz_off(BI) + (slot * NG + g) * 4);
        mem.s[g][slot] = in ? sz.x : 0.f;
        mem.z[g][slot] = in ? sz.y : 0.f;
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int r = 0; r < DH / 64; ++r) {
    const int c = lane + 64 * r;
    float a = st.acc[r] * corr;
    const int g = c / G;
#pragma unroll
    for (int f = 0; f < TS / 8; ++f) {  // 32-slot step f / 4, lane group f % 4 of the record
      float v[8];
      field8<BP>(tp + cv.v_codes_off(BI) + ((f & 3) * 16 + (c & 15)) * 8 * BP, (f >> 2) * CB + (c >> 4),
                 v);
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {  // the field's elements: slots s0 .. s0 + 3, twice
        const int s0 = 32 * (f >> 2) + 16 * hb + 4 * (f & 3);
        float pw[4], sw[4], zw[4];
        *(float4 *)pw = *(const float4 *)(mem.p + s0);
        if constexpr (Q) {
          *(float4 *)sw = *(const float4 *)(mem.s[g] + s0);
          *(float4 *)zw = *(const float4 *)(mem.z[g] + s0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float x = v[4 * hb + j];
          if constexpr (Q)
            x = fmaf(x, sw[j], zw[j]);
          else
            x = live >> (s0 + j) & 1 ? x : 0.f;
          a = fmaf(pw[j], x, a);
        }
      }
    }
    st.acc[r] = a;
  }
  __builtin_amdgcn_wave_barrier();
}

template <int DH>
__device__ void attend_one(const CacheView &cv, const float *__restrict__ q, float *__restrict__ o,
                           const AttnQuery &aq, int H, int w, WaveMem &mem) {
  constexpr int TS = 4096 / DH;
  const int lane = threadIdx.x & 63;
  const int g = aq.h / (H / cv.Hkv);
  const int64_t at = (int64_t(aq.row) * H + aq.h) * DH;
  const float scale = 1.0f / sqrtf(float(DH));
#pragma unroll
  for (int r = 0; r < DH / 64; ++r) mem.q[lane + 64 * r] = q[at + lane + 64 * r] * scale;
  const int lo = aq.m == TRIROUTE_LOCAL ? max(0, aq.P - w + 1) : 0;
  int len[4], key[8], res[8];
#pragma unroll
  for (int bi = 0; bi < 4; ++bi) {
    len[bi] = cv.pool_len[aq.s * 4 + bi];
    key[bi] = lo;
    key[4 + bi] = aq.P + 1;
  }
  lower_bounds8(cv, aq.s, len, key, res);
  AttnState<DH> st;
#pragma unroll
  for (int r = 0; r < DH / 64; ++r) st.acc[r] = 0.f;
  auto pool = [&](auto BI) {
    constexpr int bi = decltype(BI)::value;
    if (res[bi] >= res[4 + bi]) return;
    for (int t = res[bi] / TS; t * TS < res[4 + bi]; ++t)
      attend_tile<DH, bi>(st, mem, cv, cv.tile(aq.s, bi, g, t), cv.pos_tile(aq.s, bi, t),
                          len[bi] - t * TS, lo, aq.P);
  };
  pool(std::integral_constant<int, 0>{});
  pool(std::integral_constant<int, 1>{});
  pool(std::integral_constant<int, 2>{});
  pool(std::integral_constant<int, 3>{});
  const float l = wave_sum(lane < TS ? st.l : 0.f);
  const float inv = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
  for (int r = 0; r < DH / 64; ++r) o[at + lane + 64 * r] = st.acc[r] * inv;
}

// Prefill: wave item -> (segment, index in segment).
template <int DH>
__global__ __launch_bounds__(256) void attn_f32_prefill_kernel(
    CacheView cv, int B, int Tq, int H, int w, const int32_t *__restrict__ seq_ids,
    const float *__restrict__ q, const int32_t *__restrict__ cnt, const int32_t *__restrict__ idx,
    float *__restrict__ o) {
  __shared__ __align__(16) WaveMem mem[4];
  const int64_t item = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int nseg = B * H * 2;
  if (item >= int64_t(nseg) * Tq) return;
  const int seg = int(item / Tq), j = int(item % Tq);
  if (j >= cnt[seg]) return;
  AttnQuery aq;
  const int b = seg / (2 * H);
  aq.h = (seg >> 1) % H;
  aq.m = (seg & 1) + 1;
  const int t = idx[int64_t(seg) * Tq + j];
  aq.row = b * Tq + t;
  aq.s = seq_ids ? seq_ids[b] : b;
  if (aq.s < 0 || aq.s >= cv.n_seq) return;
  aq.P = cv.seq_len[aq.s] - Tq + t;
  attend_one<DH>(cv, q, o, aq, H, w, mem[threadIdx.x >> 6]);
}

// Decode: wave item -> (b, h); skip heads write zeros.
template <int DH>
__global__ __launch_bounds__(256) void attn_f32_decode_kernel(CacheView cv, int B, int H, int w,
                                                              const int32_t *__restrict__ seq_ids,
                                                              const float *__restrict__ q,
                                                              const uint8_t *__restrict__ mode,
                                                              float *__restrict__ o) {
  __shared__ __align__(16) WaveMem mem[4];
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= B * H) return;
  AttnQuery aq;
  const int b = item / H;
  aq.h = item % H;
  aq.m = mode[item];
  aq.row = b;
  aq.s = seq_ids ? seq_ids[b] : b;
  const bool bad = aq.s < 0 || aq.s >= cv.n_seq;
  aq.P = bad ? 0 : cv.seq_len[aq.s] - 1;
  if (aq.m == TRIROUTE_SKIP || bad) {
    for (int c = threadIdx.x & 63; c < DH; c += 64) o[int64_t(item) * DH + c] = 0.f;
    return;
  }
  attend_one<DH>(cv, q, o, aq, H, w, mem[threadIdx.x >> 6]);
}

}  // namespace

hipError_t launch_attn_f32_prefill(const triroute_cfg &cfg, const CacheView &cv, int B, int Tq,
                                   const int32_t *seq_ids, const void *q,
                                   const triroute_compaction &c, void *o, hipStream_t st) {
  const int64_t items = int64_t(B) * cfg.n_heads * 2 * Tq;
  dim3 grid(unsigned((items + 3) / 4));
  auto kernel = cfg.head_dim == 64 ? attn_f32_prefill_kernel<64> : attn_f32_prefill_kernel<128>;
  kernel<<<grid, 256, 0, st>>>(cv, B, Tq, cfg.n_heads, cfg.window, seq_ids, (const float *)q,
                               c.attn_cnt, c.attn_idx, (float *)o);
  return hipGetLastError();
}

hipError_t launch_attn_f32_decode(const triroute_cfg &cfg, const CacheView &cv, int B,
                                  const int32_t *seq_ids, const void *q, const uint8_t *mode,
                                  void *o, hipStream_t st) {
  dim3 grid(unsigned((B * cfg.n_heads + 3) / 4));
  auto kernel = cfg.head_dim == 64 ? attn_f32_decode_kernel<64> : attn_f32_decode_kernel<128>;
  kernel<<<grid, 256, 0, st>>>(cv, B, cfg.n_heads, cfg.window, seq_ids, (const float *)q, mode,
                               (float *)o);
  return hipGetLastError();
}

}  // namespace tr
