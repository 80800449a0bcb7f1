// Backward pass of the relaxed controller (paper Sec. 3.4-3.7, Algorithm 1
// step 7 for the controller): from the language-model gradients of the soft
// samples y~^a, y~^b (the straight-through estimator hands the hard choice's
// gradient to them) and of the selected gates p-bar, plus the regulariser's
// own terms, to the logits, then through the whitened heads, RMSNorm(h; gr),
// the GELU trunk and the first norm to every controller weight and to x and
// psi.  The language-model part of each axis' logit gradient is divided by
// that axis' balance factor rho, which then moves towards the part's norm.
//
// Kernels, in order: the trunk and tail of the forward again (with taps of
// a1, h, h^ and z; deterministic, so the logits equal the forward's), four
// tokens a wave for the logit gradient and the chain down to da1, fp32 MFMA
// grams sum_t A_t^T B_t over fixed token chunks for the weight gradients
// (fp32 within a chunk, chunks added in order in fp64), the biases' column
// sums in fp64, the product da1 W1 with the first norm's backward in its
// epilogue, and a final kernel for the whitening, the head weights and rho.
// Every sum has a fixed order.
#include <algorithm>

#include "kernels.hpp"

namespace tr {

namespace {

constexpr int DR = 128;
__device__ __forceinline__ float gelu_f(float y) {
  return 0.5f * y * (1.0f + erff(y * 0.70710678118654752f));
}
// d GELU / dy = Phi(y) + y phi(y)
__device__ __forceinline__ float gelu_grad_f(float y) {
  return 0.5f * (1.0f + erff(y * 0.70710678118654752f)) +
         y * 0.39894228040143268f * expf(-0.5f * y * y);
}

__device__ __forceinline__ float wsum(float v) { return seg_sum(v, 64); }

struct BwdTokArgs {
  const float *Z, *a1, *hpre, *Wf;  // logits, trunk taps, head weights as applied (folded)
  const float *ya, *yb, *egate;
  const int32_t *eidx, *pos;
  const float *g_ya, *g_yb, *g_gate;
  const float *W2, *gr;
  const double *stats, *usage;  // the forward's batch statistics
  const double *rho;            // [3] or NULL (1)
  const double *lambda;         // [2] or NULL (0)
  const float *rinv;
  const float *upart, *xlast;   // the trunk's products with x: nx whole chunks, and xlast's
  int nx;
  float *dz, *dh, *da1, *u, *tgr, *lmsq;  // dz: [N][DR], zero past the logits
  float *cx;                    // [N]: factor of x in dx
  int N, H, A, E1, k, dh_, w, dkv, d;
  float inv_ta, inv_tb, zeta, alpha, beta, gamma, eps, kappa_e;
};

// What a lane needs of the batch statistics and the weights of the loss terms
// for every token: attention options, its expert, its bit option.
struct BwdConst {
  float fa[3], la[3], fe, le, fb, lb;  // usage fractions f and log P + 1 of the options
  bool ent_a, ent_e, ent_b;            // the entropy floor is active
  float ca, cf, cm;                    // lambda / dense cost (attention per key, experts, bits)
  float rho_a, rho_e, rho_b;             // balance factors the language-model parts are divided by
};
__device__ __forceinline__ BwdConst bwd_const(const BwdTokArgs &p) {
  const int lane = threadIdx.x & 63;
  const double *st = p.stats;
  BwdConst c;
  const float Df = float(st[TRIROUTE_RS_DENSE]), Dm = float(st[TRIROUTE_RS_DENSE + 1]);
  const float lam_f = p.lambda ? float(p.lambda[0]) : 0.f, lam_m = p.lambda ? float(p.lambda[1]) : 0.f;
  c.rho_a = p.rho ? float(p.rho[0]) : 1.f;
  c.rho_e = p.rho ? float(p.rho[1]) : 1.f;
  c.rho_b = p.rho ? float(p.rho[2]) : 1.f;
  for (int m = 0; m < 3; ++m) {
    c.fa[m] = float(st[TRIROUTE_RS_F_ATTN + m]);
    const float P = float(st[TRIROUTE_RS_P_ATTN + m]);
    c.la[m] = P > 0.f ? logf(P) + 1.f : 0.f;
  }
  c.fe = lane < p.E1 ? float(p.usage[lane]) : 0.f;
  const float Pe = lane < p.E1 ? float(p.usage[p.E1 + lane]) : 0.f;
  c.le = Pe > 0.f ? logf(Pe) + 1.f : 0.f;
  c.fb = lane < 4 ? float(st[TRIROUTE_RS_F_BITS + lane]) : 0.f;
  const float Pb = lane < 4 ? float(st[TRIROUTE_RS_P_BITS + lane]) : 0.f;
  c.lb = Pb > 0.f ? logf(Pb) + 1.f : 0.f;
  c.ent_a = p.zeta * logf(3.f) - float(st[TRIROUTE_RS_ENTROPY]) > 0.f;
  c.ent_e = p.zeta * logf(float(p.E1)) - float(st[TRIROUTE_RS_ENTROPY + 1]) > 0.f;
  c.ent_b = p.zeta * logf(4.f) - float(st[TRIROUTE_RS_ENTROPY + 2]) > 0.f;
  c.ca = lam_f / Df;
  c.cf = lam_f / Df * p.kappa_e;
  c.cm = lane < 4 ? lam_m / Dm * float(p.dkv) * 2.f * float(2 << lane) : 0.f;
  return c;
}

// The logit gradients of token t into dzw[TOKS r] (r < 3 A + E + 5): lane a < A:
// attention group a; lane j < E + 1: expert j; lanes 0..3: the bit options.
constexpr int TOKS = 4;
__device__ __forceinline__ void logit_grads(const BwdTokArgs &p, const BwdConst &k, int t, float *dzw) {
  const int lane = threadIdx.x & 63;
  const int NZ = 3 * p.A + p.E1 + 4, HA = p.H / p.A;
  const float *z = p.Z + int64_t(t) * NZ;
  const float rows_a = float(double(p.N) * p.A), rows = float(p.N);
  const float kf = float(p.pos[t]) + 1.f, kl = fminf(kf, float(p.w));
  float sq_a = 0.f, sq_e = 0.f, sq_b = 0.f;  // squares of the language-model parts
  // ---- attention groups
  if (lane < p.A) {
    const int a = lane;
    float y[3], gl[3], gc[3], q[3], zz[3];
    const float kap[3] = {0.f, float(HA) * 2.f * float(p.dh_) * kl, float(HA) * 2.f * float(p.dh_) * kf};
    float zm = -INFINITY;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      y[m] = p.ya[(int64_t(t) * p.A + a) * 3 + m];
      gl[m] = p.g_ya[(int64_t(t) * p.A + a) * 3 + m];
      gc[m] = k.ca * kap[m];
      zz[m] = z[3 * a + m];
      zm = fmaxf(zm, zz[m]);
    }
    float qs = 0.f;
#pragma unroll
    for (int m = 0; m < 3; ++m) { q[m] = expf(zz[m] - zm); qs += q[m]; }
    const float lse = zm + logf(qs);
    float sy_l = 0.f, sy_c = 0.f, sfp = 0.f, slp = 0.f;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      q[m] /= qs;
      sy_l += y[m] * gl[m];
      sy_c += y[m] * gc[m];
      sfp += k.fa[m] * q[m];
      slp += k.la[m] * q[m];
    }
#pragma unroll
    for (int m = 0; m < 3; ++m) {
      const float dl = p.inv_ta * y[m] * (gl[m] - sy_l);
      sq_a += dl * dl;
      float d = dl / k.rho_a + p.inv_ta * y[m] * (gc[m] - sy_c);
      d += p.alpha * 3.f / rows_a * q[m] * (k.fa[m] - sfp);
      d += p.beta * 2.f / rows_a * lse * q[m];
      if (k.ent_a) d += p.gamma / rows_a * q[m] * (k.la[m] - slp);
      dzw[TOKS * (3 * a + m)] = d;
    }
  }
  // ---- experts: the gates over the selected set, then the full softmax
  {
    const float ze = lane < p.E1 ? z[3 * p.A + lane] : -INFINITY;
    const float zmx = seg_max(ze, 64);
    const float ee = lane < p.E1 ? expf(ze - zmx) : 0.f;
    const float es = wsum(ee);
    const float pe = ee / es, lse = zmx + logf(es);
    const float sfp = wsum(k.fe * pe), slp = wsum(k.le * pe);
    // slot s on lane s: expert, gate, upstream
    const int es_ = lane < p.k ? p.eidx[int64_t(t) * p.k + lane] : -1;
    const float gs = lane < p.k ? p.egate[int64_t(t) * p.k + lane] : 0.f;
    const float gl = lane < p.k ? p.g_gate[int64_t(t) * p.k + lane] : 0.f;
    const float gc = lane < p.k && es_ != 0 ? k.cf : 0.f;
    const float sgl = wsum(gs * gl), sgc = wsum(gs * gc);
    const float sl_l = gs * (gl - sgl), sl_c = gs * (gc - sgc);
    float dl = 0.f, dc = 0.f;
    for (int s = 0; s < p.k; ++s) {
      const int e = __shfl(es_, s, 64);
      const float a_l = __shfl(sl_l, s, 64), a_c = __shfl(sl_c, s, 64);
      if (e == lane) { dl += a_l; dc += a_c; }
    }
    if (lane < p.E1) {
      sq_e += dl * dl;
      float d = dl / k.rho_e + dc;
      d += p.alpha * float(p.E1) / rows * pe * (k.fe - sfp);
      d += p.beta * 2.f / rows * lse * pe;
      if (k.ent_e) d += p.gamma / rows * pe * (k.le - slp);
      dzw[TOKS * (3 * p.A + lane)] = d;
    }
  }
  // ---- bits: y~ over (2, 4, 8, 16)
  {
    const bool on = lane < 4;
    const float zb = on ? z[3 * p.A + p.E1 + lane] : -INFINITY;
    const float y = on ? p.yb[int64_t(t) * 4 + lane] : 0.f;
    const float gl = on ? p.g_yb[int64_t(t) * 4 + lane] : 0.f;
    const float zmx = seg_max(zb, 64);
    const float ee = on ? expf(zb - zmx) : 0.f;
    const float es = wsum(ee);
    const float q = ee / es, lse = zmx + logf(es);
    const float sy_l = wsum(y * gl), sy_c = wsum(y * k.cm), sfp = wsum(k.fb * q), slp = wsum(k.lb * q);
    if (on) {
      const float dl = p.inv_tb * y * (gl - sy_l);
      sq_b += dl * dl;
      float d = dl / k.rho_b + p.inv_tb * y * (k.cm - sy_c);
      d += p.alpha * 4.f / rows * q * (k.fb - sfp);
      d += p.beta * 2.f / rows * lse * q;
      if (k.ent_b) d += p.gamma / rows * q * (k.lb - slp);
      dzw[TOKS * (3 * p.A + p.E1 + lane)] = d;
    }
  }
  const float sqa = wsum(sq_a), sqe = wsum(sq_e), sqb = wsum(sq_b);
  if (lane < 3) p.lmsq[int64_t(t) * 4 + lane] = lane == 0 ? sqa : lane == 1 ? sqe : sqb;
}

// Four tokens a wave: the two 128-wide products of the chain read every weight
// once for the four (the launch is bound by those loads from the caches: one
// token a wave took 71 us for 16384 tokens of the 1.3B layer, four 57).  A lane owns
// features lane and lane + 64 of the trunk.
__global__ __launch_bounds__(256) void relax_bwd_tok_kernel(BwdTokArgs p) {
  __shared__ __align__(16) float dzs[4][DR][TOKS];  // a wave's logit gradients, then its dh
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int t0 = (blockIdx.x * 4 + wave) * TOKS;
  if (t0 >= p.N) return;  // wave-uniform; no block barrier below
  float(*dzw)[TOKS] = dzs[wave];
  const int NZ = 3 * p.A + p.E1 + 4;
  for (int r = lane; r < DR; r += 64) *(float4 *)dzw[r] = make_float4(0.f, 0.f, 0.f, 0.f);
  __builtin_amdgcn_wave_barrier();
  const BwdConst bc = bwd_const(p);
  // (a token past the last repeats it, to the same values)
#pragma unroll
  for (int q = 0; q < TOKS; ++q) logit_grads(p, bc, min(t0 + q, p.N - 1), &dzw[0][q]);
  __builtin_amdgcn_wave_barrier();
  const int nt = min(TOKS, p.N - t0);
  for (int q = 0; q < nt; ++q)
    for (int r = lane; r < DR; r += 64) p.dz[int64_t(t0 + q) * DR + r] = dzw[r][q];
  // rows of W (two features a lane) times the four tokens' entries of v
  auto product = [&](const float *W, int n, float (&g)[TOKS][2]) {
#pragma unroll
    for (int q = 0; q < TOKS; ++q) g[q][0] = g[q][1] = 0.f;
#pragma unroll 4
    for (int r = 0; r < n; ++r) {
      const float4 v = *(const float4 *)dzw[r];
      const float w0 = W[int64_t(r) * DR + lane], w1 = W[int64_t(r) * DR + lane + 64];
      g[0][0] = fmaf(w0, v.x, g[0][0]); g[0][1] = fmaf(w1, v.x, g[0][1]);
      g[1][0] = fmaf(w0, v.y, g[1][0]); g[1][1] = fmaf(w1, v.y, g[1][1]);
      g[2][0] = fmaf(w0, v.z, g[2][0]); g[2][1] = fmaf(w1, v.z, g[2][1]);
      g[3][0] = fmaf(w0, v.w, g[3][0]); g[3][1] = fmaf(w1, v.w, g[3][1]);
    }
  };
  // ---- dh^ = W'^T dz, then RMSNorm(h; gr): h^ = h r gr
  float g[TOKS][2];
  product(p.Wf, NZ, g);
  float dh[TOKS][2];
#pragma unroll
  for (int q = 0; q < TOKS; ++q) {
    const int64_t at = int64_t(min(t0 + q, p.N - 1)) * DR + lane;
    const float h0 = p.hpre[at], h1 = p.hpre[at + 64];
    const float rr = 1.0f / sqrtf(wsum(h0 * h0 + h1 * h1) / float(DR) + p.eps);
    const float gh0 = g[q][0] * p.gr[lane], gh1 = g[q][1] * p.gr[lane + 64];
    const float dot = wsum(gh0 * h0 + gh1 * h1);
    const float c3 = rr * rr * rr * dot / float(DR);
    dh[q][0] = rr * gh0 - c3 * h0;
    dh[q][1] = rr * gh1 - c3 * h1;
    if (q < nt) {
      p.tgr[at] = g[q][0] * h0 * rr;
      p.tgr[at + 64] = g[q][1] * h1 * rr;
      p.dh[at] = dh[q][0];
      p.dh[at + 64] = dh[q][1];
    }
  }
  __builtin_amdgcn_wave_barrier();  // the logit gradients are used up
  *(float4 *)dzw[lane] = make_float4(dh[0][0], dh[1][0], dh[2][0], dh[3][0]);
  *(float4 *)dzw[lane + 64] = make_float4(dh[0][1], dh[1][1], dh[2][1], dh[3][1]);
  __builtin_amdgcn_wave_barrier();
  // sum_j dn1_j n1_j = sum_c da1_c (W1 n1)_c.  W1 n1 comes from the trunk's
  // partial products with x: as a1 - b1 - W1_psi psi it would lose its low bits
  // to a large bias or side feature (1000 times W1 n1, d 64: elements of dx were
  // off by up to 3e-4 of themselves).  Loaded ahead of the product, whose time
  // covers it (703 us the 1.3B training step of 16384 tokens, 710 behind it).
  float x[TOKS][2], y[TOKS][2];
#pragma unroll
  for (int q = 0; q < TOKS; ++q) {
    const int64_t at = int64_t(min(t0 + q, p.N - 1)) * DR + lane;
    x[q][0] = p.a1[at];
    x[q][1] = p.a1[at + 64];
    y[q][0] = p.xlast ? p.xlast[at] : 0.f;  // (an entry of da1's own: read before it is written)
    y[q][1] = p.xlast ? p.xlast[at + 64] : 0.f;
  }
  for (int s = 0; s < p.nx; ++s)
#pragma unroll
    for (int q = 0; q < TOKS; ++q) {
      const int64_t at = (int64_t(s) * p.N + min(t0 + q, p.N - 1)) * DR + lane;
      y[q][0] += p.upart[at];
      y[q][1] += p.upart[at + 64];
    }
  // ---- h = W2 u + b2: du = W2^T dh; u = GELU(a1)
  product(p.W2, DR, g);
#pragma unroll
  for (int q = 0; q < TOKS; ++q) {
    const float d0 = g[q][0] * gelu_grad_f(x[q][0]), d1 = g[q][1] * gelu_grad_f(x[q][1]);
    const float s = wsum(d0 * y[q][0] + d1 * y[q][1]);
    if (q < nt) {
      const int t = t0 + q;
      const int64_t at = int64_t(t) * DR + lane;
      p.u[at] = gelu_f(x[q][0]);
      p.u[at + 64] = gelu_f(x[q][1]);
      p.da1[at] = d0;
      p.da1[at + 64] = d1;
      const float r = p.rinv[t];
      if (lane == 0) p.cx[t] = r * r * s / float(p.d);
    }
  }
}

// Column sums of up to CS_JOBS token-major matrices in one launch (job
// blockIdx.z): part[c][i] = sum over tokens t of chunk c (CS_CHUNK tokens) of
// A[t][i], in fp64: wave w of a block adds tokens c CS_CHUNK + 64 w .. + 63
// for the block's 64 columns (lane = column), the waves are added in order.
constexpr int CS_CHUNK = 256, CS_JOBS = 5;
struct ColsumJobs {
  const float *A[CS_JOBS];
  double *part[CS_JOBS];
  float *out[CS_JOBS];
  double *out64[CS_JOBS];
  int lda[CS_JOBS], m[CS_JOBS];
};
__global__ __launch_bounds__(256) void colsum_kernel(ColsumJobs J, int N) {
  __shared__ double ws_[4][64];
  const float *A = J.A[blockIdx.z];
  const int lda = J.lda[blockIdx.z], m = J.m[blockIdx.z];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane, c = blockIdx.y;
  if (int(blockIdx.x) * 64 >= m) return;  // block-uniform
  const int t0 = c * CS_CHUNK + 64 * wave, t1 = min(N, t0 + 64);
  double s = 0;
  if (i < m) {
    // 16 loads in flight at a time, added in token order
    for (int tb = t0; tb < t1; tb += 16) {
      float v[16];
#pragma unroll
      for (int q = 0; q < 16; ++q) v[q] = A[int64_t(min(tb + q, t1 - 1)) * lda + i];  // clamped
#pragma unroll
      for (int q = 0; q < 16; ++q) s += tb + q < t1 ? double(v[q]) : 0.0;
    }
  }
  ws_[wave][lane] = s;
  __syncthreads();
  if (wave == 0 && i < m)
    J.part[blockIdx.z][int64_t(c) * m + i] =
        ((ws_[0][lane] + ws_[1][lane]) + ws_[2][lane]) + ws_[3][lane];
}

// sum over the nc chunks, in order, of part[c * ne] (16 loads in flight)
template <typename T>
__device__ __forceinline__ double chunk_sum(const T *part, int nc, int64_t ne) {
  double s = 0;
  for (int cb = 0; cb < nc; cb += 16) {
    T v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = part[int64_t(min(cb + q, nc - 1)) * ne];  // clamped
#pragma unroll
    for (int q = 0; q < 16; ++q) s += cb + q < nc ? double(v[q]) : 0.0;
  }
  return s;
}
__global__ __launch_bounds__(256) void colsum_finish_kernel(ColsumJobs J, int nc) {
  const int i = blockIdx.x * 256 + threadIdx.x, z = blockIdx.y, m = J.m[z];
  if (i >= m) return;
  const double s = chunk_sum(J.part[z] + i, nc, m);
  if (J.out[z]) J.out[z][i] = float(s);
  if (J.out64[z]) J.out64[z][i] = s;
}

typedef float f32x4m __attribute__((ext_vector_type(4)));
typedef float f32x16m __attribute__((ext_vector_type(16)));

// Grams of token-major matrices, C = A^T B: A [N][DR] fp32 (its token scaled
// by ascale, if given), B [N][n] fp32 or the activation dtype, each chunk of
// tokens to its own plane of C.  fp32 MFMA 32x32x2.  A block takes all 128
// columns of A by 64 of B, so B (the tokens' activations: most of the bytes)
// is read once and as it is stored; a wave takes 32 of the 128 rows.  32
// tokens at a time through two LDS buffers, the next ones' loads in registers
// meanwhile; rows of 32 mod 64 floats put the two token rows that a wave
// reads at once in different banks.  (64 x 64 tiles over a materialised
// [n1; psi], single-buffered: 221 us for dW1 of the 1.3B layer, 16384 tokens,
// 39 TFLOP/s, and 45 us to write [n1; psi]; now 100 us, 86 TFLOP/s.)
constexpr int GR_JOBS = 3, GR_KT = 32, GR_LA = DR + 32, GR_LB = 64 + 32;
struct GramJobs {
  const float *A[GR_JOBS];
  const void *B[GR_JOBS];
  float *C[GR_JOBS];                    // planes of [DR][ldc]
  int64_t plane[GR_JOBS];
  int n[GR_JOBS], ldc[GR_JOBS], tile[GR_JOBS + 1];  // first 64-column tile of each job
};

template <typename T>
__global__ __launch_bounds__(256) void gram_kernel(GramJobs J, const float *__restrict__ ascale,
                                                   int N, int chunk) {
  __shared__ __align__(16) float As[2][GR_KT][GR_LA], Bs[2][GR_KT][GR_LB];
  int z = 0;
  while (z + 1 < GR_JOBS && int(blockIdx.x) >= J.tile[z + 1]) ++z;
  const float *A = J.A[z];
  const T *B = (const T *)J.B[z];
  const int n = J.n[z], j0 = (int(blockIdx.x) - J.tile[z]) * 64;
  const int k_lo = blockIdx.y * chunk, k_hi = min(N, k_lo + chunk);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int at = tid >> 5, ac = 4 * (tid & 31);  // A: token at + 8 i, columns ac .. ac + 3
  const int bt = tid >> 3, bc = 8 * (tid & 7);   // B: token bt, columns j0 + bc .. + 7
  // the next step's operands stay as loaded until they are put into LDS: a
  // conversion at the load would wait for it before this step's products
  float4 ra[4];
  float sa[4];
  T rb[8];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = k0 + at + 8 * i;
      ra[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      sa[i] = 1.f;
      if (t < k_hi) {
        ra[i] = *(const float4 *)(A + int64_t(t) * DR + ac);
        if (ascale) sa[i] = ascale[t];
      }
    }
    const int t = k0 + bt;
#pragma unroll
    for (int q = 0; q < 8; ++q) rb[q] = T(0);
    if (t < k_hi) {
      const T *b = B + int64_t(t) * n + j0 + bc;
      if (n >= 64) {  // whole runs of 8, aligned; psi (n <= 32) may lie anywhere
#pragma unroll
        for (int q = 0; q < 8; q += 16 / int(sizeof(T))) *(uint4 *)(rb + q) = *(const uint4 *)(b + q);
      } else {
#pragma unroll
        for (int q = 0; q < 8; ++q)
          if (j0 + bc + q < n) rb[q] = b[q];
      }
    }
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *(float4 *)&As[buf][at + 8 * i][ac] =
          make_float4(ra[i].x * sa[i], ra[i].y * sa[i], ra[i].z * sa[i], ra[i].w * sa[i]);
    float f[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) f[q] = Act<T>::cvt(rb[q]);
    *(float4 *)&Bs[buf][bt][bc] = make_float4(f[0], f[1], f[2], f[3]);
    *(float4 *)&Bs[buf][bt][bc + 4] = make_float4(f[4], f[5], f[6], f[7]);
  };
  f32x16m acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
  fetch(k_lo);
  put(0);
  __syncthreads();
  int buf = 0;
  const int l31 = lane & 31, hi = lane >> 5;
  for (int k0 = k_lo; k0 < k_hi; k0 += GR_KT) {
    const bool more = k0 + GR_KT < k_hi;
    if (more) fetch(k0 + GR_KT);
#pragma unroll
    for (int kq = 0; kq < GR_KT; kq += 2) {
      const float a = As[buf][kq + hi][32 * wave + l31];
#pragma unroll
      for (int j = 0; j < 2; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, Bs[buf][kq + hi][32 * j + l31], acc[j], 0, 0, 0);
    }
    if (more) put(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  float *C = J.C[z] + int64_t(blockIdx.y) * J.plane[z];
  const int ldc = J.ldc[z];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int c = j0 + 32 * j + l31;
    if (c >= n) continue;
#pragma unroll
    for (int i = 0; i < 16; ++i)  // register i: row 8 (i / 4) + 4 (lane / 32) + i % 4
      C[int64_t(32 * wave + 8 * (i >> 2) + 4 * hi + (i & 3)) * ldc + c] = acc[j][i];
  }
}

// out[r][c] (r < rows, c < ld; rows ldo apart) = sum over the nc planes, in
// order, of part (fp64), times colscale[c] where the job is scaled, as fp32
constexpr int SUM_JOBS = GR_JOBS + 1;
struct SumJobs {
  const float *part[SUM_JOBS];
  float *out[SUM_JOBS];
  int64_t plane[SUM_JOBS];
  int rows[SUM_JOBS], ld[SUM_JOBS], ldo[SUM_JOBS], nc[SUM_JOBS];
  bool scaled[SUM_JOBS];
};
__global__ __launch_bounds__(256) void gram_sum_kernel(SumJobs J, const float *__restrict__ colscale) {
  const int z = blockIdx.y;
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  const int ld = J.ld[z];
  if (e >= int64_t(J.rows[z]) * ld) return;
  double s = chunk_sum(J.part[z] + e, J.nc[z], J.plane[z]);
  const int r = int(e / ld), c = int(e - int64_t(r) * ld);
  if (J.scaled[z]) s *= double(colscale[c]);
  J.out[z][int64_t(r) * J.ldo[z] + c] = float(s);
}

// [dn1; dpsi] = da1 W1 and the first norm n1 = x r g1 behind it, per tile in
// registers: dx = r g1 dn1 - cx x (cx: see relax_bwd_tok_kernel) and the sums
// over tokens of dn1 x r (dg1) in fp64, one partial per block.  A block
// takes 64 tokens (16 a wave, their da1 held in registers as MFMA operands:
// of row lane % 16, k 16 s + 4 (lane / 16) + i for MFMA (s, i)) and `tiles`
// tiles of 64 columns, W1 streaming through two LDS buffers of 64 k-rows (68
// floats a row: rows four apart fall in different banks).  Four blocks a CU
// (at 32 tokens a wave one fitted, and the kernel took 187 us instead of
// 151).  dn1 is never written: as a matrix of its own it cost 145 us to
// make, 113 us to turn into dx and 28 us to sum for dg1 (1.3B, 16384 tokens:
// 134 MB, four times through memory).
constexpr int DXT = 64, DX_LD = 68;
template <typename T>
__global__ __launch_bounds__(256, 4) void trunk_bwd_kernel(
    const float *__restrict__ da1, const float *__restrict__ W1, const T *__restrict__ x,
    const float *__restrict__ g1, const float *__restrict__ rinv, const float *__restrict__ cx,
    int N, int d, int dpsi, int tiles, float *__restrict__ dx, float *__restrict__ dpsi_out,
    double *__restrict__ dg_part) {
  __shared__ __align__(16) float Ws[2][64][DX_LD];
  __shared__ double sgs[2][4][64];  // each wave's sums of the last two tiles
  const int K1 = d + dpsi, nt = (K1 + 63) / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int t0 = blockIdx.x * DXT + 16 * wave, l15 = lane & 15, o4 = lane >> 4;
  const int ty0 = blockIdx.y * tiles, ty1 = min(nt, ty0 + tiles);
  f32x4m a[8];
  {
    const float *src = da1 + int64_t(min(t0 + l15, N - 1)) * DR + 4 * o4;
#pragma unroll
    for (int s = 0; s < 8; ++s) a[s] = *(const f32x4m *)(src + 16 * s);
  }
  // this lane's rows of a tile: tokens t0 + 4 o4 + q
  float rr[4], cc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int t = min(t0 + 4 * o4 + q, N - 1);
    rr[q] = rinv[t];
    cc[q] = cx[t];
  }
  const int wr = tid >> 4, wc = 4 * (tid & 15);  // staged k-row wr + 16 i, columns wc .. wc + 3
  float4 rw[4];
  auto fetch = [&](int ty, int half) {
    const int c = ty * 64 + wc;  // K1 is a multiple of 4: four columns are all in or all out
#pragma unroll
    for (int i = 0; i < 4; ++i)
      rw[i] = c < K1 ? *(const float4 *)(W1 + int64_t(64 * half + wr + 16 * i) * K1 + c)
                     : make_float4(0.f, 0.f, 0.f, 0.f);
  };
  auto put = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) *(float4 *)&Ws[buf][wr + 16 * i][wc] = rw[i];
  };
  // the waves' sums of tile ty, in wave order (a barrier after they were left)
  auto tile_sum = [&](int ty) {
    if (wave == 0 && ty * 64 < d) {
      const double(*q)[64] = sgs[ty & 1];
      dg_part[int64_t(blockIdx.x) * d + ty * 64 + lane] =
          ((q[0][lane] + q[1][lane]) + q[2][lane]) + q[3][lane];
    }
  };
  if (ty0 >= ty1) return;  // block-uniform
  fetch(ty0, 0);
  put(0);
  __syncthreads();
  for (int ty = ty0; ty < ty1; ++ty) {
    const int c0 = ty * 64 + l15;
    // the tile's x, in flight during its products
    T xv[4][4];
    if (ty * 64 < d) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const T *xr = x + int64_t(min(t0 + 4 * o4 + q, N - 1)) * d + c0;
#pragma unroll
        for (int j = 0; j < 4; ++j) xv[q][j] = xr[16 * j];
      }
    }
    f32x4m acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4m{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const bool more = half == 0 || ty + 1 < ty1;
      if (more) fetch(half == 0 ? ty : ty + 1, half ^ 1);
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                a[4 * half + s][q], Ws[half][16 * s + 4 * o4 + q][16 * j + l15], acc[j], 0, 0, 0);
      if (more) put(half ^ 1);
      __syncthreads();
      if (half == 0 && ty > ty0) tile_sum(ty - 1);
    }
    if (ty * 64 >= d) {  // the side features (d is a multiple of 64)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int t = t0 + 4 * o4 + q, c = c0 + 16 * j - d;
          if (t < N && c < dpsi) dpsi_out[int64_t(t) * dpsi + c] = acc[j][q];
        }
      continue;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float gj = g1[c0 + 16 * j];
      double sg = 0.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int t = t0 + 4 * o4 + q;
        const float dn = acc[j][q], xx = Act<T>::cvt(xv[q][j]);
        if (t < N) {
          dx[int64_t(t) * d + c0 + 16 * j] = rr[q] * (gj * dn) - cc[q] * xx;
          sg += double(dn * xx * rr[q]);
        }
      }
      sg += __shfl_xor(sg, 16, 64);
      sg += __shfl_xor(sg, 32, 64);
      if (o4 == 0) sgs[ty & 1][wave][l15 + 16 * j] = sg;
    }
  }
  __syncthreads();
  tile_sum(ty1 - 1);
}

// 64 columns a block, a quarter of the partials a wave, the quarters in order
__global__ __launch_bounds__(256) void dg_finish_kernel(const double *__restrict__ part, int nc, int d,
                                                        float *__restrict__ dg1) {
  __shared__ double q[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + lane, per = (nc + 3) / 4, c0 = per * wave;  // d % 64 == 0
  q[wave][lane] = c0 < nc ? chunk_sum(part + int64_t(c0) * d + i, min(per, nc - c0), d) : 0.0;
  __syncthreads();
  if (wave == 0) dg1[i] = float(((q[0][lane] + q[1][lane]) + q[2][lane]) + q[3][lane]);
}

// Head weights from the gram of (dz, h^): with whitening, z = W (h^ - mu) /
// (sd + eps) + c, so dW = (G - dc mu^T) / (sd + eps); biases dc = sum dz.
// Then rho <- (1 - m) rho + m sqrt(sum of the squares of the language-model
// parts).  One thread per head weight.
__global__ __launch_bounds__(256) void heads_final_kernel(const float *__restrict__ G,
                                                          const float *__restrict__ dc, int A, int E1,
                                                          const float *__restrict__ mu,
                                                          const float *__restrict__ sd, float weps,
                                                          float *dWa, float *dca, float *dWe, float *dce,
                                                          float *dWb, float *dcb, const double *lmsq,
                                                          double *rho, float rho_m, double *lm_norm) {
  const int NZ = 3 * A + E1 + 4;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < NZ * DR) {
    const int r = e / DR, j = e % DR;
    const int ax = r < 3 * A ? 0 : r < 3 * A + E1 ? 1 : 2;
    float v = G[e];
    if (mu) v = (v - dc[r] * mu[ax * DR + j]) / (sd[ax * DR + j] + weps);
    if (ax == 0) dWa[int64_t(r) * DR + j] = v;
    else if (ax == 1) dWe[int64_t(r - 3 * A) * DR + j] = v;
    else dWb[int64_t(r - 3 * A - E1) * DR + j] = v;
    if (j == 0) {
      if (ax == 0) dca[r] = dc[r];
      else if (ax == 1) dce[r - 3 * A] = dc[r];
      else dcb[r - 3 * A - E1] = dc[r];
    }
  }
  if (blockIdx.x == 0 && threadIdx.x < 3) {
    const double nrm = sqrt(lmsq[threadIdx.x]);
    if (lm_norm) lm_norm[threadIdx.x] = nrm;
    if (rho && rho_m > 0.f) rho[threadIdx.x] = (1.0 - rho_m) * rho[threadIdx.x] + rho_m * nrm;
  }
}

// Chunks of the gram launches: about GR_BLOCKS blocks (four a CU), at least 32
// tokens and at most `most` of them in an fp32 partial sum: 512 for the
// trunk's gram, 128 for the heads' (and dW2's, in their launch), beyond which
// the partials' rounding shows in the result.
constexpr int GR_BLOCKS = 1024, GR_MOST_X = 512, GR_MOST = 128;
int gram_chunk(int tiles, int N, int most) {
  const int want = std::max(1, GR_BLOCKS / tiles);
  const int c = ((N + want - 1) / want + GR_KT - 1) / GR_KT * GR_KT;
  return std::min(c, most);
}
int chunks_of(int N, int chunk) { return (N + chunk - 1) / chunk; }

// Layout of the partial sums, in floats: the trunk weight's gram, the small
// grams' planes, the column sums' and dg1's fp64 partials.
struct PartLayout {
  int x_tiles, x_chunk, s_chunk, nx, ns, ncs, ndg;
  size_t w1, small, cs, dg, total;
};
PartLayout part_layout(const triroute_cfg &c, int N) {
  PartLayout L;
  const size_t K1 = size_t(c.d_model + c.d_psi);
  L.x_tiles = c.d_model / 64;
  L.x_chunk = gram_chunk(L.x_tiles, N, GR_MOST_X);
  L.s_chunk = gram_chunk(5, N, GR_MOST);
  L.nx = chunks_of(N, L.x_chunk);
  L.ns = chunks_of(N, L.s_chunk);
  L.ncs = chunks_of(N, CS_CHUNK);
  L.ndg = chunks_of(N, DXT);
  size_t at = 0;
  auto take = [&](size_t n) { const size_t r = at; at += (n + 63) / 64 * 64; return r; };
  L.w1 = take(size_t(L.nx) * DR * c.d_model);
  L.small = take(size_t(L.ns) * DR * (2 * DR + c.d_psi));
  L.cs = take(2 * size_t(L.ncs) * (4 * DR + 4));
  L.dg = take(2 * size_t(L.ndg) * c.d_model);
  L.total = at;
  return L;
}

}  // namespace

size_t relax_grad_part_floats(const triroute_cfg &cfg, int N) { return part_layout(cfg, N).total; }

hipError_t launch_relax_backward(const triroute_cfg &cfg, int N, const void *x, const float *psi,
                                 const triroute_router_w &w, const float *Wf,
                                 const float *white_mu, const float *white_sd, float white_eps,
                                 const RelaxBwdJob &j, hipStream_t st) {
  const int A = attn_groups(cfg), E1 = cfg.n_experts + 1, NZ = 3 * A + E1 + 4;
  const int d = cfg.d_model, dpsi = cfg.d_psi, K1 = d + dpsi;
  const PartLayout L = part_layout(cfg, N);
  BwdTokArgs p;
  p.Z = j.z; p.a1 = j.a1; p.hpre = j.hpre; p.Wf = Wf;
  p.ya = j.y_attn; p.yb = j.y_bits; p.egate = j.egate; p.eidx = j.eidx; p.pos = j.pos;
  p.g_ya = j.g_attn; p.g_yb = j.g_bits; p.g_gate = j.g_gate;
  p.W2 = w.W2; p.gr = w.gr; p.stats = j.stats; p.usage = j.usage; p.rho = j.rho_io;
  p.lambda = j.lambda;
  p.rinv = j.rinv;
  {
    int ks, kchunk;
    router_split(N, K1, ks, kchunk);
    p.nx = dpsi > 0 ? d / kchunk : ks;
    p.upart = j.upart;
    p.xlast = dpsi > 0 && d % kchunk != 0 ? j.da1 : nullptr;
  }
  p.dz = j.dz; p.dh = j.dh; p.da1 = j.da1; p.u = j.u; p.tgr = j.tgr; p.lmsq = j.lmsq; p.cx = j.cx;
  p.N = N; p.H = cfg.n_heads; p.A = A; p.E1 = E1; p.k = cfg.top_k; p.dh_ = cfg.head_dim;
  p.w = cfg.window; p.dkv = cfg.n_kv_heads * cfg.head_dim; p.d = d;
  p.inv_ta = 1.f / j.tau_a; p.inv_tb = 1.f / j.tau_b; p.zeta = j.zeta; p.alpha = j.alpha;
  p.beta = j.beta; p.gamma = j.gamma; p.eps = cfg.rms_eps;
  p.kappa_e = 3.f * float(cfg.d_model) * float(cfg.d_ff);
  relax_bwd_tok_kernel<<<dim3((N + 4 * TOKS - 1) / (4 * TOKS)), 256, 0, st>>>(p);
  const RelaxGradOut &o = j.out;
  // biases and norm gains of the controller: column sums
  ColsumJobs cs;
  {
    const float *src[CS_JOBS] = {j.dz, j.tgr, j.dh, j.da1, j.lmsq};
    float *out[CS_JOBS] = {j.dc, o.dgr, o.db2, o.db1, nullptr};
    double *part = (double *)(j.part + L.cs);
    for (int i = 0; i < CS_JOBS; ++i) {
      cs.A[i] = src[i];
      cs.out[i] = out[i];
      cs.out64[i] = i == 4 ? j.lmsq_sum : nullptr;
      cs.lda[i] = i == 4 ? 4 : DR;
      cs.m[i] = i == 0 ? NZ : i == 4 ? 3 : DR;
      cs.part[i] = part;
      part += size_t(L.ncs) * cs.m[i];
    }
  }
  colsum_kernel<<<dim3(DR / 64, L.ncs, CS_JOBS), 256, 0, st>>>(cs, N);
  colsum_finish_kernel<<<dim3(1, CS_JOBS), 256, 0, st>>>(cs, L.ncs);
  // weight grams: (dz, h^), (dh, u) and (da1, psi), then (r da1, x) for the
  // trunk's part of W1, whose columns g1 scales at the end
  const int planew = 2 * DR + dpsi;
  float *ps = j.part + L.small, *pw = j.part + L.w1;
  GramJobs g{};
  g.A[0] = j.dz; g.B[0] = j.hh; g.C[0] = ps; g.n[0] = DR; g.ldc[0] = DR;
  g.A[1] = j.dh; g.B[1] = j.u; g.C[1] = ps + DR * DR; g.n[1] = DR; g.ldc[1] = DR;
  g.A[2] = j.da1; g.B[2] = psi; g.C[2] = ps + 2 * DR * DR; g.n[2] = dpsi; g.ldc[2] = dpsi;
  for (int i = 0; i < GR_JOBS; ++i) g.plane[i] = int64_t(DR) * planew;
  g.tile[0] = 0; g.tile[1] = 2; g.tile[2] = 4; g.tile[3] = dpsi > 0 ? 5 : 4;
  gram_kernel<float><<<dim3(g.tile[3], L.ns), 256, 0, st>>>(g, nullptr, N, L.s_chunk);
  GramJobs gx{};
  gx.A[0] = j.da1; gx.B[0] = x; gx.C[0] = pw; gx.n[0] = d; gx.ldc[0] = d; gx.plane[0] = int64_t(DR) * d;
  gx.tile[0] = 0;
  for (int i = 1; i <= GR_JOBS; ++i) gx.tile[i] = L.x_tiles;
  const dim3 xg(L.x_tiles, L.nx);
  if (cfg.act == TRIROUTE_BF16)
    gram_kernel<bf16><<<xg, 256, 0, st>>>(gx, j.rinv, N, L.x_chunk);
  else
    gram_kernel<float><<<xg, 256, 0, st>>>(gx, j.rinv, N, L.x_chunk);
  SumJobs sj{};
  sj.part[0] = ps; sj.out[0] = j.G; sj.rows[0] = NZ; sj.ld[0] = DR; sj.ldo[0] = DR;
  sj.part[1] = ps + DR * DR; sj.out[1] = o.dW2; sj.rows[1] = DR; sj.ld[1] = DR; sj.ldo[1] = DR;
  sj.part[2] = ps + 2 * DR * DR; sj.out[2] = o.dW1 + d; sj.rows[2] = dpsi > 0 ? DR : 0;
  sj.ld[2] = dpsi > 0 ? dpsi : 1; sj.ldo[2] = K1;
  sj.part[3] = pw; sj.out[3] = o.dW1; sj.rows[3] = DR; sj.ld[3] = d; sj.ldo[3] = K1;
  for (int i = 0; i < 4; ++i) {
    sj.plane[i] = i < 3 ? int64_t(DR) * planew : int64_t(DR) * d;
    sj.nc[i] = i < 3 ? L.ns : L.nx;
    sj.scaled[i] = i == 3;
  }
  gram_sum_kernel<<<dim3(unsigned((int64_t(DR) * std::max(d, DR) + 255) / 256), 4), 256, 0, st>>>(sj, w.g1);
  // [dn1; dpsi], the first norm and dg1; blocks of 64 tokens, their columns
  // split so that about four blocks a CU run
  const int mt = (N + DXT - 1) / DXT, nt = (K1 + 63) / 64;
  const int split = std::max(1, std::min(nt, (1024 + mt - 1) / mt)), tiles = (nt + split - 1) / split;
  const dim3 tg(mt, (nt + tiles - 1) / tiles);
  double *dgp = (double *)(j.part + L.dg);
  if (cfg.act == TRIROUTE_BF16)
    trunk_bwd_kernel<bf16><<<tg, 256, 0, st>>>(j.da1, w.W1, (const bf16 *)x, w.g1, j.rinv, j.cx, N, d,
                                               dpsi, tiles, o.dx, o.dpsi, dgp);
  else
    trunk_bwd_kernel<float><<<tg, 256, 0, st>>>(j.da1, w.W1, (const float *)x, w.g1, j.rinv, j.cx, N, d,
                                                dpsi, tiles, o.dx, o.dpsi, dgp);
  dg_finish_kernel<<<dim3(d / 64), 256, 0, st>>>(dgp, L.ndg, d, o.dg1);
  heads_final_kernel<<<dim3((NZ * DR + 255) / 256), 256, 0, st>>>(
      j.G, j.dc, A, E1, white_mu, white_sd, white_eps, o.dWa, o.dca, o.dWe, o.dce, o.dWb, o.dcb,
      j.lmsq_sum, j.rho_io, j.rho_m, o.lm_norm);
  return hipGetLastError();
}

}  // namespace tr
