// Controller (paper Sec. 3.3 controller equation) and hard inference
// decisions (Sec. 3.8), fp32 end to end.
//
//   rms_norm1   : r_i = 1/sqrt(mean(x_i^2) + eps); n1 = x r g1 (act out, for QKV; fp64)
//   trunk1      : partial W1 [x r g1 ; psi] over K chunks    fp32 MFMA, N x 128
//   tail        : u = GELU(sum + b1), h = W2 u + b2, h^ = RMSNorm(h) gr,
//                 z = W_{a,e,b} h^ + c, argmax / top-k decisions and gates
#include "kernels.hpp"

namespace tr {

// One wave per token row, 8 consecutive elements per lane access.
template <typename T>
__global__ __launch_bounds__(256) void rms_norm1_kernel(const T *__restrict__ x,
                                                        const float *__restrict__ g,
                                                        float *__restrict__ rinv,
                                                        T *__restrict__ n1, int N, int d,
                                                        float eps, const RopeJob rj) {
  int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  if (row >= N) return;
  if (rj.tab)  // the token's rotation table entries (one lane per pair)
    for (int j = lane; j < rj.hd; j += 64) rj.tab[int64_t(row) * rj.hd + j] = rope_entry(rj, row, j);
  const T *xr = x + int64_t(row) * d;
  // fp32 scale for the controller (fp32 end to end); fp64 for the n1 the
  // projections read, rounded once to the activation dtype
  float ss = 0.f;
  double sd = 0.0;
  for (int c = lane * 8; c < d; c += 512) {
    float v[8];
    load8(xr + c, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      ss = fmaf(v[i], v[i], ss);
      sd = fma(double(v[i]), double(v[i]), sd);
    }
  }
  ss = wave_sum(ss);
  float r = 1.0f / sqrtf(ss / float(d) + eps);
  if (lane == 0) rinv[row] = r;
  if (n1) {
    sd = wave_sum(sd);
    const double rd = 1.0 / sqrt(sd / double(d) + double(eps));
    T *nr = n1 + int64_t(row) * d;
    for (int c = lane * 8; c < d; c += 512) {
      float v[8], gv[8];
      double o[8];
      load8(xr + c, v);
      load8(g + c, gv);
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = (double(v[i]) * rd) * double(gv[i]);
      store8(nr + c, o);
    }
  }
}

typedef float f32x4r __attribute__((ext_vector_type(4)));

// Split of the trunk's K = d + d_psi inputs over blocks, so that a small
// batch (decode) still spreads over the chip: K chunks are multiples of 32.
void router_split(int N, int K, int &ks, int &kchunk) {
  const int mt = (N + 63) / 64;
  int want = (512 + mt - 1) / mt;
  const int kmax = (K + 63) / 64;
  want = want < 1 ? 1 : want > kmax ? kmax : want;
  kchunk = ((K + want - 1) / want + 31) / 32 * 32;
  ks = (K + kchunk - 1) / kchunk;
}

// Partial trunk pre-activations upart[ks][N][128] = [n1 ; psi] W1^T over the
// block's K chunk, with n1 = x r g1 formed on load (fp32 MFMA 16x16x4).
// Block: 64 rows x 128 outputs, 4 waves of 16 rows; the next K step is
// fetched into registers while the current one is multiplied from LDS.
// XL: where the chunk holds inputs of x and of psi, the products with x alone
// go to xlast (the backward pass wants W1 n1 without the other terms of a1).
template <typename T, bool XL>
__global__ __launch_bounds__(256) void trunk1_kernel(const T *__restrict__ x,
                                                     const float *__restrict__ rinv,
                                                     const float *__restrict__ g1,
                                                     const float *__restrict__ psi,
                                                     const float *__restrict__ W1,
                                                     float *__restrict__ upart, int N, int d,
                                                     int dpsi, int kchunk,
                                                     float *__restrict__ xlast) {
  constexpr int BM = 64, BK = 32, LD = BK + 1;
  __shared__ float As[2][BM][LD];
  __shared__ float Bs[2][128][LD];
  const int K = d + dpsi;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int m0 = blockIdx.x * BM;
  const int kb = blockIdx.y * kchunk, ke = min(K, kb + kchunk);
  f32x4r acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = f32x4r{0.f, 0.f, 0.f, 0.f};
  const int ar = tid >> 2, ak = (tid & 3) * 8;
  const int br = tid >> 1, bk = (tid & 1) * 16;
  const int arow = m0 + ar;
  const float rr = arow < N ? rinv[arow] : 0.f;
  float ra[8], rb[16];
  auto fetch = [&](int k0) {
    // A: 8 consecutive inputs of row arow; whole 8-runs inside x use one
    // 16-byte load (d % 64 == 0, so a run never straddles x and psi)
    const int ka = k0 + ak;
    if (arow < N && ka + 8 <= ke && ka + 8 <= d) {
      float xv[8], gv[8];
      load8(x + int64_t(arow) * d + ka, xv);
      load8(g1 + ka, gv);
#pragma unroll
      for (int i = 0; i < 8; ++i) ra[i] = (xv[i] * rr) * gv[i];
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = ka + i;
        float v = 0.f;
        if (arow < N && k < ke)
          v = k < d ? (Act<T>::ld(x, int64_t(arow) * d + k) * rr) * g1[k]
                    : psi[int64_t(arow) * dpsi + (k - d)];
        ra[i] = v;
      }
    }
    // B: 16 consecutive inputs of W1 row br (K % 4 == 0: 16-byte aligned)
    const int kb0 = k0 + bk;
    if (kb0 + 16 <= ke) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float4 w = *(const float4 *)(W1 + int64_t(br) * K + kb0 + 4 * i);
        rb[4 * i] = w.x; rb[4 * i + 1] = w.y; rb[4 * i + 2] = w.z; rb[4 * i + 3] = w.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int k = kb0 + i;
        rb[i] = k < ke ? W1[int64_t(br) * K + k] : 0.f;
      }
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 8; ++i) As[buf][ar][ak + i] = ra[i];
#pragma unroll
    for (int i = 0; i < 16; ++i) Bs[buf][br][bk + i] = rb[i];
  };
  fetch(kb);
  put(0);
  __syncthreads();
  int buf = 0;
  // accumulator r of the lane: row 16 wave + 4 (lane / 16) + r, columns 16 j + lane % 16
  auto store = [&](float *out) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = m0 + 16 * wave + 4 * (lane >> 4) + r;
      if (row >= N) continue;
#pragma unroll
      for (int j = 0; j < 8; ++j) out[int64_t(row) * 128 + 16 * j + (lane & 15)] = acc[j][r];
    }
  };
  for (int k0 = kb; k0 < ke; k0 += BK) {
    if (XL && k0 == d && kb < d) store(xlast);  // (d and the chunks are multiples of BK)
    const bool more = k0 + BK < ke;
    if (more) fetch(k0 + BK);
#pragma unroll
    for (int kk = 0; kk < BK; kk += 4) {
      const float av = As[buf][16 * wave + (lane & 15)][kk + (lane >> 4)];
#pragma unroll
      for (int j = 0; j < 8; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
            av, Bs[buf][16 * j + (lane & 15)][kk + (lane >> 4)], acc[j], 0, 0, 0);
    }
    if (more) put(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  store(upart + int64_t(blockIdx.y) * N * 128);
}

// Tail, a tile of TB <= 16 tokens a block of four waves:
//   u = GELU(sum of trunk partials + b1); h = W2 u + b2; h^ = RMSNorm(h) gr;
//   z = [Wa; We; Wb] h^ + [ca; ce; cb]; argmax / top-k decisions and gates.
// A chain of short steps, so its length counts and not its arithmetic.  The
// products are taken transposed (fp32 MFMA 16x16x4, weight rows by tokens):
// wave w owns rows 32 w .. 32 w + 31 of W2 and the logit tiles w, w + 4, ...,
// and holds them in registers as the MFMA wants them (four consecutive inputs
// a lane; one 16-byte load feeds four steps), fetched from L2 before anything
// waits for the trunk.  A lane then has four consecutive outputs of one token:
// the norm is two shuffles and an exchange of four sums, and h^ and z go to LDS
// in 16 bytes.  Few blocks' worth of tokens are spread over the chip in
// smaller tiles (launch_router); the columns past TB hold whatever the LDS
// held, which no other column reads, and are not stored.  With fewer than 8
// tokens the trunk's chunks are summed by 8 / TB groups of threads, a run of
// chunks each, whose sums are added in order.
// (Weights staged in LDS by blocks of eight waves, a CU each: 20.7 us at 333
// tokens, 24 at 2000 of the 1.3B layer, 38 at 16384; so: 10, 12.9, 25.4.  A
// prefill of 333 tokens at 410M 152 -> 139 us, of 2000 after 7000 at 1.3B 727 -> 708.)
constexpr int RT_TB = 16, RT_DR = 128, RT_NZ = 112, RT_TILES = 256;
constexpr int RT_LD = RT_DR + 4, RT_ZLD = RT_NZ + 4;

template <bool TWO>  // 16 tokens: two float4 of u a thread, several tiles a block
__global__ __launch_bounds__(256, 2) void router_tail_kernel(
    const float *__restrict__ upart, int KS, const float *__restrict__ b1,
    const float *__restrict__ W2, const float *__restrict__ b2, const float *__restrict__ gr,
    const float *__restrict__ Wa, const float *__restrict__ ca, const float *__restrict__ We,
    const float *__restrict__ ce, const float *__restrict__ Wb, const float *__restrict__ cb,
    uint8_t *__restrict__ mode, uint8_t *__restrict__ bit, int32_t *__restrict__ eidx,
    float *__restrict__ egate, int N, int TB, int H, int A, int E1, int k, float eps,
    TailTap tap) {
  constexpr int DR = RT_DR, NE = TWO ? 2 : 1, NB = TWO ? 2 : 12;
  __shared__ __align__(16) float Us[RT_TB][RT_LD];   // u, then h^
  __shared__ __align__(16) float Zs[RT_TB][RT_ZLD];  // the groups' chunk sums, then z
  __shared__ __align__(16) float b2s[DR], grs[DR], bzs[RT_NZ];
  __shared__ float red[4][RT_TB];
  static_assert(8 * RT_LD <= RT_TB * RT_ZLD, "chunk sums fit");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tl = lane & 15, q4 = (lane >> 4) * 4;
  const int NZ = 3 * A + E1 + 4;
  auto zrow = [&](int z) {
    z = z < NZ ? z : NZ - 1;
    return z < 3 * A ? Wa + z * DR : z < 3 * A + E1 ? We + (z - 3 * A) * DR
                                                    : Wb + (z - 3 * A - E1) * DR;
  };
  // element (token ut, columns uc ..), group ug of the NG that share the chunks
  const int nel = 32 * (TB < 8 ? TB : 8), NG = 256 / nel;
  const int ut = (tid & (nel - 1)) >> 5, uc = (tid & 31) * 4, ug = tid / nel;
  const int per = (KS + NG - 1) / NG, sb = ug * per, se = min(KS, sb + per);
  f32x4r pre[NB][NE];
  auto load_parts = [&](int t0, int s0) {
#pragma unroll
    for (int s = 0; s < NB; ++s)
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        pre[s][e] = f32x4r{0.f, 0.f, 0.f, 0.f};
        if (s0 + s < se && ut + 8 * e < min(TB, N - t0))
          pre[s][e] = *(const f32x4r *)(upart + (int64_t(s0 + s) * N + t0 + ut + 8 * e) * DR + uc);
      }
  };
  // loads in the order in which they are waited for: the trunk's chunks, the
  // small vectors, the weights
  load_parts(blockIdx.x * TB, sb);
  __builtin_amdgcn_sched_barrier(0);
  const f32x4r b1v = {b1[uc], b1[uc + 1], b1[uc + 2], b1[uc + 3]};
  float sv[3] = {0.f, 0.f, 0.f};
  if (tid < DR) {
    sv[0] = b2[tid];
    sv[1] = gr[tid];
    if (tid < NZ) sv[2] = tid < 3 * A ? ca[tid] : tid < 3 * A + E1 ? ce[tid - 3 * A]
                                                                   : cb[tid - 3 * A - E1];
  }
  __builtin_amdgcn_sched_barrier(0);
  f32x4r w2[2][8], wz[8], wx[8];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int s = 0; s < 8; ++s)
      w2[j][s] = *(const f32x4r *)(W2 + (32 * wave + 16 * j + tl) * DR + 16 * s + q4);
  {
    const float *row = zrow(16 * wave + tl);
#pragma unroll
    for (int s = 0; s < 8; ++s) wz[s] = *(const f32x4r *)(row + 16 * s + q4);
  }
  __builtin_amdgcn_sched_barrier(0);
  if (tid < DR) {  // read behind the loop's first barrier
    b2s[tid] = sv[0];
    grs[tid] = sv[1];
    if (tid < RT_NZ) bzs[tid] = sv[2];
  }
  const int HA = H / A;  // heads per decision group
  for (int t0 = blockIdx.x * TB; t0 < N; t0 += gridDim.x * TB) {
    const int nt = min(TB, N - t0);  // this tile's tokens
    f32x4r u[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) u[e] = f32x4r{0.f, 0.f, 0.f, 0.f};
    for (int s0 = sb;;) {
#pragma unroll
      for (int s = 0; s < NB; ++s)
#pragma unroll
        for (int e = 0; e < NE; ++e) u[e] += pre[s][e];
      s0 += NB;
      if (s0 >= se) break;
      load_parts(t0, s0);
    }
    if (TWO && t0 + int(gridDim.x) * TB < N) load_parts(t0 + gridDim.x * TB, sb);
    if (!TWO && NG > 1) {  // (block-uniform)
      float *ps = &Zs[0][0];
      *(f32x4r *)(ps + (ug * TB + ut) * RT_LD + uc) = u[0];
      __syncthreads();
      if (ug == 0)
        for (int g = 1; g < NG; ++g) u[0] += *(const f32x4r *)(ps + (g * TB + ut) * RT_LD + uc);
    }
    if (ug == 0) {
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        f32x4r a = u[e] + b1v, y;
        if (tap.a1 && ut + 8 * e < nt)
          *(f32x4r *)(tap.a1 + int64_t(t0 + ut + 8 * e) * DR + uc) = a;
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = 0.5f * a[i] * (1.0f + erff(a[i] * 0.70710678118654752f));
        *(f32x4r *)&Us[ut + 8 * e][uc] = y;
      }
    }
    __syncthreads();
    // h: two accumulators per 16 rows (even and odd steps)
    f32x4r hv[2];
    {
      f32x4r acc[2][2];
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j][0] = acc[j][1] = f32x4r{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const f32x4r x = *(const f32x4r *)&Us[tl][16 * s + q4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[j][i & 1] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(w2[j][s][i], x[i], acc[j][i & 1], 0, 0, 0);
      }
      if (16 * wave + 64 < NZ) {  // the wave's second logit tile, on its way meanwhile
        const float *row = zrow(16 * wave + 64 + tl);
#pragma unroll
        for (int s = 0; s < 8; ++s) wx[s] = *(const f32x4r *)(row + 16 * s + q4);
      }
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        hv[j] = (acc[j][0] + acc[j][1]) + *(const f32x4r *)(b2s + 32 * wave + 16 * j + q4);
#pragma unroll
        for (int r = 0; r < 4; ++r) ss = fmaf(hv[j][r], hv[j][r], ss);
      }
      ss += __shfl_xor(ss, 16, 64);
      ss += __shfl_xor(ss, 32, 64);
      if (lane < 16) red[wave][lane] = ss;
    }
    __syncthreads();
    {
      const float ss = (red[0][tl] + red[1][tl]) + (red[2][tl] + red[3][tl]);
      const float r = 1.0f / sqrtf(ss / float(DR) + eps);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int n = 32 * wave + 16 * j + q4;
        const f32x4r hn = (hv[j] * r) * *(const f32x4r *)(grs + n);
        *(f32x4r *)&Us[tl][n] = hn;
        if (tl < nt) {
          if (tap.hpre) *(f32x4r *)(tap.hpre + int64_t(t0 + tl) * DR + n) = hv[j];
          if (tap.h) *(f32x4r *)(tap.h + int64_t(t0 + tl) * DR + n) = hn;
        }
      }
    }
    __syncthreads();
    auto logits = [&](int zt, const f32x4r *w) {
      f32x4r acc[2];
      acc[0] = acc[1] = f32x4r{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const f32x4r x = *(const f32x4r *)&Us[tl][16 * s + q4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[s][i], x[i], acc[i & 1], 0, 0, 0);
      }
      *(f32x4r *)&Zs[tl][16 * zt + q4] =
          (acc[0] + acc[1]) + *(const f32x4r *)(bzs + 16 * zt + q4);
    };
    static_assert(RT_NZ <= 128, "two logit tiles a wave");
    if (16 * wave < NZ) logits(wave, wz);  // (wave-uniform, no barrier inside)
    if (16 * wave + 64 < NZ) logits(wave + 4, wx);
    __syncthreads();
    if (tap.z)
      for (int it = tid; it < nt * NZ; it += 256) {
        const int tt = it / NZ, z = it - tt * NZ;
        tap.z[int64_t(t0) * NZ + it] = Zs[tt][z];
      }
    // decisions: 16 lanes per token.  Modes: heads j, j + 16, ...; argmax, first
    // maximum on ties.  Bit width and experts: lane j holds expert logits j,
    // j + 16, ... (E + 1 <= 64)
    if (4 * wave < nt) {  // wave-uniform
      const int tt = 4 * wave + (lane >> 4);
      const float *z = Zs[tt], *ze = z + 3 * A;
      const bool live = tt < nt;
      const int64_t t = t0 + tt;
      if (live)
        for (int hh = tl; hh < H; hh += 16) {
          const float *za = z + 3 * (HA == 1 ? hh : hh / HA);
          int best = 0;
          if (za[1] > za[best]) best = 1;
          if (za[2] > za[best]) best = 2;
          mode[t * H + hh] = uint8_t(best);
        }
      if (live && tl == 0) {
        const float *zb = ze + E1;
        const float z0 = zb[0], z1 = zb[1], z2 = zb[2], z3 = zb[3];
        int bb = z1 > z0 ? 1 : 0;
        float zm = z1 > z0 ? z1 : z0;
        if (z2 > zm) { bb = 2; zm = z2; }
        if (z3 > zm) bb = 3;
        bit[t] = uint8_t(bb);
      }
      // top-k by logit (softmax is monotone), ties to the lower id; the gate
      // renormalises over the selected set, null included
      float zj[4], zmax = -INFINITY;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        zj[q] = 16 * q + tl < E1 ? ze[16 * q + tl] : -INFINITY;
        zmax = fmaxf(zmax, zj[q]);
      }
      zmax = seg_max(zmax, 16);
      uint64_t open = E1 < 64 ? (1ull << E1) - 1 : ~0ull, all = open;  // not yet taken
      float tot = 0.f;
      for (int sl = 0; sl < k; ++sl) {
        float m = -INFINITY;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (open >> (16 * q + tl) & 1) m = fmaxf(m, zj[q]);
        m = seg_max(m, 16);
        uint64_t hit = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (16 * q < E1)  // uniform
            hit |= (__ballot(zj[q] == m) >> (lane & 48) & 0xffffull) << (16 * q);
        hit &= open;
        if (!hit) hit = open;  // only NaNs left: the lowest id
        open &= ~(hit & (~hit + 1));
        tot += expf(m - zmax);
      }
      const uint64_t taken = all & ~open;
      if (live)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (taken >> (16 * q + tl) & 1) {
            const int sl = __popcll(taken & ((1ull << (16 * q + tl)) - 1));
            eidx[t * k + sl] = 16 * q + tl;
            egate[t * k + sl] = expf(zj[q] - zmax) / tot;
          }
    }
    if (!TWO) return;
    __syncthreads();  // the next tile writes Us and Zs
  }
}

// The same tail for few tokens (decode), one 256-thread block per token, so
// that each step's weight reads are all in flight at once instead of a wave
// walking whole rows: thread j < 128 sums the trunk partials of column j (in
// chunk order, then b1); two threads per row of W2 (64 columns each) and
// four per logit row (32 columns each), their partial sums added by lane
// shuffles (every thread of a row ends with the same value).  fp32 either
// way; the products are summed in a different order than the MFMA tail, and
// the decisions do not depend on it above the routing margin.
constexpr int RTB_MAXKS = 48;
__global__ __launch_bounds__(256) void router_tail_blk_kernel(
    const float *__restrict__ upart, int KS, const float *__restrict__ b1,
    const float *__restrict__ W2, const float *__restrict__ b2, const float *__restrict__ gr,
    const float *__restrict__ Wa, const float *__restrict__ ca, const float *__restrict__ We,
    const float *__restrict__ ce, const float *__restrict__ Wb, const float *__restrict__ cb,
    uint8_t *__restrict__ mode, uint8_t *__restrict__ bit, int32_t *__restrict__ eidx,
    float *__restrict__ egate, int N, int H, int A, int E1, int k, float eps, TailTap tap) {
  constexpr int DR = RT_DR;
  __shared__ __align__(16) float us[DR], hs[DR], zs[RT_NZ];
  __shared__ float red[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t = blockIdx.x;  // grid = N
  const int NZ = 3 * A + E1 + 4;
  // u = GELU(sum of the KS trunk partials + b1)
  if (tid < DR) {
    float p[RTB_MAXKS];
#pragma unroll
    for (int s = 0; s < RTB_MAXKS; ++s)
      if (s < KS) p[s] = upart[(int64_t(s) * N + t) * DR + tid];
    float a = 0.f;
#pragma unroll
    for (int s = 0; s < RTB_MAXKS; ++s)
      if (s < KS) a += p[s];
    a += b1[tid];
    if (tap.a1) tap.a1[int64_t(t) * DR + tid] = a;
    us[tid] = 0.5f * a * (1.0f + erff(a * 0.70710678118654752f));
  }
  __syncthreads();
  // h = W2 u + b2, row r = tid / 2; h^ = RMSNorm(h) gr
  {
    const int r = tid >> 1, c0 = (tid & 1) * (DR / 2);
    const float4 *w = (const float4 *)(W2 + r * DR + c0);
    float4 x[DR / 8];
#pragma unroll
    for (int i = 0; i < DR / 8; ++i) x[i] = w[i];
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < DR / 8; ++i) {
      const float4 u = *(const float4 *)(us + c0 + 4 * i);
      acc = fmaf(x[i].x, u.x, acc); acc = fmaf(x[i].y, u.y, acc);
      acc = fmaf(x[i].z, u.z, acc); acc = fmaf(x[i].w, u.w, acc);
    }
    acc += __shfl_xor(acc, 1, 64);
    const float h = acc + b2[r];
    const float ssw = seg_sum((tid & 1) ? 0.f : h * h, 64);  // the wave's 32 rows
    if (lane == 0) red[wave] = ssw;
    __syncthreads();
    const float ss = (red[0] + red[1]) + (red[2] + red[3]);
    const float rr = 1.0f / sqrtf(ss / float(DR) + eps);
    const float hn = (h * rr) * gr[r];
    if ((tid & 1) == 0) {
      hs[r] = hn;
      if (tap.hpre) tap.hpre[int64_t(t) * DR + r] = h;
      if (tap.h) tap.h[int64_t(t) * DR + r] = hn;
    }
  }
  __syncthreads();
  // z = [Wa; We; Wb] h^ + [ca; ce; cb], logit row z0 + tid / 4
  for (int z0 = 0; z0 < NZ; z0 += 64) {
    const int z = z0 + (tid >> 2), c0 = (tid & 3) * (DR / 4);
    float acc = 0.f;
    if (z < NZ) {
      const float *wz = z < 3 * A ? Wa + z * DR : z < 3 * A + E1 ? We + (z - 3 * A) * DR
                                                                  : Wb + (z - 3 * A - E1) * DR;
      float4 x[DR / 16];
#pragma unroll
      for (int i = 0; i < DR / 16; ++i) x[i] = ((const float4 *)(wz + c0))[i];
#pragma unroll
      for (int i = 0; i < DR / 16; ++i) {
        const float4 u = *(const float4 *)(hs + c0 + 4 * i);
        acc = fmaf(x[i].x, u.x, acc); acc = fmaf(x[i].y, u.y, acc);
        acc = fmaf(x[i].z, u.z, acc); acc = fmaf(x[i].w, u.w, acc);
      }
    }
    acc += __shfl_xor(acc, 1, 64);
    acc += __shfl_xor(acc, 2, 64);
    if (z < NZ && (tid & 3) == 0) {
      const float bias = z < 3 * A ? ca[z] : z < 3 * A + E1 ? ce[z - 3 * A] : cb[z - 3 * A - E1];
      zs[z] = acc + bias;
      if (tap.z) tap.z[int64_t(t) * NZ + z] = zs[z];
    }
  }
  __syncthreads();
  if (wave != 0) return;  // decisions by the first wave (no barrier below)
  const int HA = H / A;
  for (int hh = lane; hh < H; hh += 64) {
    const float *za = zs + 3 * (hh / HA);
    int best = 0;
    if (za[1] > za[best]) best = 1;
    if (za[2] > za[best]) best = 2;
    mode[int64_t(t) * H + hh] = uint8_t(best);
  }
  if (lane == 0) {
    const float *zb = zs + 3 * A + E1;
    int bb = 0;
    for (int j = 1; j < 4; ++j)
      if (zb[j] > zb[bb]) bb = j;
    bit[t] = uint8_t(bb);
  }
  const float zj = lane < E1 ? zs[3 * A + lane] : -INFINITY;
  const float zmax = seg_max(zj, 64);
  uint64_t taken = 0;
  float tot = 0.f;
  for (int sl = 0; sl < k; ++sl) {
    const float cand = (lane < E1 && !(taken >> lane & 1)) ? zj : -INFINITY;
    const float m = seg_max(cand, 64);
    const uint64_t hit = __ballot(lane < E1 && !(taken >> lane & 1) && cand == m);
    const int best = __ffsll((unsigned long long)hit) - 1;
    taken |= 1ull << best;
    tot += expf(m - zmax);
  }
  if (taken >> lane & 1) {
    const int sl = __popcll(taken & lanemask_lt());
    eidx[int64_t(t) * k + sl] = lane;
    egate[int64_t(t) * k + sl] = expf(zj - zmax) / tot;
  }
}

hipError_t launch_router(const triroute_cfg &cfg, int N, const void *x, const float *psi,
                         const triroute_router_w &w, void *n1, uint8_t *mode, uint8_t *bit,
                         int32_t *eidx, float *egate, float *rinv, float *u, const RopeJob *rope,
                         hipStream_t st, TailTap tap) {
  RopeJob rj{};
  if (rope) rj = *rope;
  const int d = cfg.d_model;
  int ks, kchunk;
  router_split(N, d + cfg.d_psi, ks, kchunk);
  dim3 g1((N + 3) / 4);
  dim3 g2((N + 63) / 64, ks);
  if (cfg.act == TRIROUTE_BF16) {
    rms_norm1_kernel<bf16><<<g1, 256, 0, st>>>((const bf16 *)x, w.g1, rinv, (bf16 *)n1, N, d,
                                               cfg.rms_eps, rj);
    (tap.xlast ? trunk1_kernel<bf16, true> : trunk1_kernel<bf16, false>)<<<g2, 256, 0, st>>>(
        (const bf16 *)x, rinv, w.g1, psi, w.W1, u, N, d, cfg.d_psi, kchunk, tap.xlast);
  } else {
    rms_norm1_kernel<float><<<g1, 256, 0, st>>>((const float *)x, w.g1, rinv, (float *)n1, N, d,
                                                cfg.rms_eps, rj);
    (tap.xlast ? trunk1_kernel<float, true> : trunk1_kernel<float, false>)<<<g2, 256, 0, st>>>(
        (const float *)x, rinv, w.g1, psi, w.W1, u, N, d, cfg.d_psi, kchunk, tap.xlast);
  }
  if (N <= 256 && ks <= RTB_MAXKS) {  // a CU a token, where the vector units are the shorter way:
    // the same layers with the tiles of one token instead, 160M decode of one
    // row 68.0 -> 68.8 us, 410M of 64 rows 128.0 -> 128.6, fp32 of 128 83.4 -> 84.6
    router_tail_blk_kernel<<<dim3(N), 256, 0, st>>>(
        u, ks, w.b1, w.W2, w.b2, w.gr, w.Wa, w.ca, w.We, w.ce, w.Wb, w.cb, mode, bit, eidx, egate,
        N, cfg.n_heads, attn_groups(cfg), cfg.n_experts + 1, cfg.top_k, cfg.rms_eps, tap);
    return hipGetLastError();
  }
  // tokens per tile: the fewest (a power of two) whose tiles are at most one a
  // CU; past 8192 tokens the
  // two blocks a CU that its registers allow keep their weights for several
  int tb = 1;
  while (tb < RT_TB && (N + tb - 1) / tb > RT_TILES) tb *= 2;
  const int tiles = (N + tb - 1) / tb;
  auto *tail = tb == RT_TB ? router_tail_kernel<true> : router_tail_kernel<false>;
  tail<<<dim3(tiles < 512 ? tiles : 512), 256, 0, st>>>(
      u, ks, w.b1, w.W2, w.b2, w.gr, w.Wa, w.ca, w.We, w.ce, w.Wb, w.cb, mode, bit, eidx, egate, N,
      tb, cfg.n_heads, attn_groups(cfg), cfg.n_experts + 1, cfg.top_k, cfg.rms_eps, tap);
  return hipGetLastError();
}

hipError_t router_prepare() { return hipSuccess; }

}  // namespace tr
