// Surrogate network of the transmutation energy (10 -> 64 -> 64 -> 1, SiLU,
// BF16 operands on the 16x16x32 MFMA, FP32 accumulation): inference,
// normalization fitting, and training with hand-written forward/backward
// kernels and Adam on FP32 master weights.
//
// Parameter order of the flat vectors (4929 values):
//   w1[64][10], b1[64], w2[64][64], b2[64], w3[64], b3.
#include <cmath>
#include <vector>

#include "mlp_device.hpp"

namespace vc {

constexpr int OFF_W1 = 0, OFF_B1 = 640, OFF_W2 = 704, OFF_B2 = 4800, OFF_W3 = 4864, OFF_B3 = 4928;

}  // namespace vc

struct vcsgc_mlp {
  hipStream_t stream = nullptr;
  int device = 0;
  float *p = nullptr;     // FP32 master parameters [4929]
  float *g = nullptr;     // gradient [4929]
  float *m1 = nullptr, *m2 = nullptr;  // Adam moments
  __bf16 *w1b = nullptr;  // [64][32]
  __bf16 *w2b = nullptr;  // [64][64], then its transpose
  float *w3r = nullptr;   // [64] bf16-rounded w3
  float mu[10], sd[10];
  float out_mu = 0.f, out_sd = 1.f;
  int64_t adam_t = 0;
  // training scratch for batch size cap
  int64_t cap = 0;
  unsigned char *work = nullptr;
  double *red = nullptr;  // per-sample squared errors
  double *mom = nullptr;  // normalization: block totals, then mean and sd per column
  std::string err;
};

namespace vc {

MlpDev mlp_dev(const vcsgc_mlp *m) {
  MlpDev d;
  d.w1 = m->w1b;
  d.w2 = m->w2b;
  d.b1 = m->p + OFF_B1;
  d.b2 = m->p + OFF_B2;
  d.w3 = m->w3r;
  d.b3 = m->p + OFF_B3;
  for (int k = 0; k < MLP_IN; ++k) {
    d.mu[k] = m->mu[k];
    d.sd[k] = m->sd[k];
  }
  d.out_mu = m->out_mu;
  d.out_sd = m->out_sd;
  return d;
}

// bf16 copies of the weights for the MFMA operands
__global__ void k_mlp_refresh(const float *__restrict__ p, __bf16 *w1b, __bf16 *w2b, float *w3r) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < MLP_H * MLP_KP) {
    const int n = t / MLP_KP, k = t % MLP_KP;
    w1b[t] = to_bf16(k < MLP_IN ? p[OFF_W1 + n * MLP_IN + k] : 0.0f);
  }
  if (t < MLP_H * MLP_H) {
    w2b[t] = to_bf16(p[OFF_W2 + t]);
    w2b[MLP_H * MLP_H + t % MLP_H * MLP_H + t / MLP_H] = to_bf16(p[OFF_W2 + t]);
  }
  if (t < MLP_H) w3r[t] = bf16_round(p[OFF_W3 + t]);
}

hipError_t mlp_refresh(vcsgc_mlp *m) {
  k_mlp_refresh<<<16, 256, 0, m->stream>>>(m->p, m->w1b, m->w2b, m->w3r);
  return hipGetLastError();
}

// Inference on n raw descriptors (FP64, [n][10]); 16 samples per block.
__global__ void __launch_bounds__(BLOCK) k_mlp_infer(MlpDev md, int64_t n,
                                                     const double *__restrict__ desc, double *dE) {
  __shared__ __bf16 zs[16 * MLP_KP];
  __shared__ __bf16 h1[16 * MLP_H], h2[16 * MLP_H];
  __shared__ float yv[16];
  const int64_t base = (int64_t)blockIdx.x * 16;
  for (int e = threadIdx.x; e < 16 * MLP_KP; e += BLOCK) {
    const int r = e / MLP_KP, k = e % MLP_KP;
    const int64_t b = base + r;
    zs[e] = (b < n && k < MLP_IN) ? mlp_input(md, k, desc[b * MLP_IN + k]) : to_bf16(0.0f);
  }
  __syncthreads();
  mlp_block16(md, zs, h1, h2, yv);
  if (threadIdx.x < 16 && base + threadIdx.x < n)
    dE[base + threadIdx.x] = (double)(yv[threadIdx.x] * md.out_sd + md.out_mu);
}

// ---------------------------------------------------------------------------
// training
// ---------------------------------------------------------------------------
// Training runs two kernels per step, k_fwd_bwd and k_grads.  (Seventeen
// launches with every activation and error in memory as [B][64] floats, one
// thread per column for the column sums, were 2.8 ms a step at a batch of
// 4,096, 2.6 ms of it in the column sums' one-load-at-a-time chains.)  The
// arithmetic and the order of every sum are those of the plain formulation:
// products in ascending k (32 per MFMA), column sums in ascending sample.

__device__ __forceinline__ float dsilu(float a) {
  const float s = 1.0f / (1.0f + expf(-a));
  return s * (1.0f + a * (1.0f - s));
}

// Activations and errors of one batch, Bp = B rounded up to 32 samples (the
// samples past B are zero).  Errors that are summed over the samples in FP32
// are row-major [b][64]; operands of the weight-gradient products are bf16 and
// sample-contiguous [neuron][Bp], so that a lane's eight products are one
// 16-byte load.
struct MlpWork {
  float *P;    // [Bp][64] dY[b] H2[b][k]
  float *dA2;  // [Bp][64]
  float *dA1;  // [Bp][64]
  float *dY;   // [Bp]
  __bf16 *dA2t, *dA1t, *H1t;  // [64][Bp]
  __bf16 *Zt;                 // [16][Bp], rows 10.. zero
  double *red;  // per-sample squared errors [B]
  float *g;     // gradient [4929]
  int64_t Bp;
};

// bytes of workspace per padded sample, the squared errors aside
constexpr int64_t MLP_WORK_BYTES = 4 * (3 * MLP_H + 1) + 2 * (3 * MLP_H + 16);

static MlpWork carve_work(unsigned char *base, int64_t B, double *red, float *g) {
  MlpWork w;
  w.Bp = (B + 31) / 32 * 32;  // every part below is a multiple of 64 bytes
  float *f = (float *)base;
  w.P = f;
  w.dA2 = w.P + w.Bp * MLP_H;
  w.dA1 = w.dA2 + w.Bp * MLP_H;
  w.dY = w.dA1 + w.Bp * MLP_H;
  w.dA2t = (__bf16 *)(w.dY + w.Bp);
  w.dA1t = w.dA2t + w.Bp * MLP_H;
  w.H1t = w.dA1t + w.Bp * MLP_H;
  w.Zt = w.H1t + w.Bp * MLP_H;
  w.red = red;
  w.g = g;
  return w;
}

// Forward and backward pass of 16 samples per block, everything between the
// drawn samples and the errors in registers and LDS: samples 0..B-1
// (draw == 0) or Philox-drawn sample indices, with replacement (draw != 0).
// Wave v computes neurons 16 v .. 16 v + 15 of each layer; lane l holds rows
// 4 (l / 16) .. + 3 of neuron 16 v + l % 16, of which it keeps the
// pre-activations for the backward pass.  Bound by the latency of its chain
// (draw, three MFMA layers, the 64-term output sum), one block per CU and
// 9.3 us at a batch of 4,096.
__global__ void __launch_bounds__(BLOCK)
    k_fwd_bwd(int64_t n, int64_t B, const double *__restrict__ desc,
              const double *__restrict__ dE, MlpDev md, const __bf16 *__restrict__ w2t,
              uint64_t seed, uint64_t step, int draw, MlpWork w) {
  __shared__ __bf16 zs[16 * MLP_KP];
  __shared__ __bf16 h1[16 * MLP_H], da2[16 * MLP_H];
  __shared__ float h2[16 * (MLP_H + 1)];
  __shared__ float w3[MLP_H];
  __shared__ float tv[16], dy[16];
  __shared__ int64_t src[16];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r = lane & 15, kb = (lane >> 4) * 8, row0 = (lane >> 4) * 4;
  const int nn = wv * 16 + r;  // this lane's neuron
  const int64_t base = (int64_t)blockIdx.x * 16;
  const MlpFrag f = mlp_frag(md);
  bf16x8 w2c[2];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    w2c[0][q] = w2t[nn * MLP_H + kb + q];
    w2c[1][q] = w2t[nn * MLP_H + 32 + kb + q];
  }
  if (tid < MLP_H) w3[tid] = md.w3[tid];
  if (tid < 16) {
    int64_t s = base + tid;
    if (draw && s < B) {
      const U4 u = philox(seed, 0x5EEDull, step, (uint64_t)s, 0, 7);
      s = (int64_t)__umul64hi(u.v[0], (uint64_t)n);
    }
    src[tid] = base + tid < B ? s : -1;
    tv[tid] = base + tid < B ? (float)((dE[s] - (double)md.out_mu) / (double)md.out_sd) : 0.0f;
  }
  __syncthreads();
  for (int e = tid; e < 16 * MLP_KP; e += BLOCK) {
    const int b = e / MLP_KP, k = e % MLP_KP;
    const int64_t s = src[b];
    const bool in = s >= 0 && k < MLP_IN;
    zs[e] = in ? mlp_input(md, k, desc[s * MLP_IN + k]) : to_bf16(0.0f);
  }
  __syncthreads();
  const bool ok[4] = {base + row0 < B, base + row0 + 1 < B, base + row0 + 2 < B,
                      base + row0 + 3 < B};
  typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
  // column nn of four consecutive samples, sample-contiguous
  auto store_t = [&](__bf16 *dst, const bf16x4 &v) {
    *(bf16x4 *)(dst + nn * w.Bp + base + row0) = v;
  };
  float a1[4], a2[4];
  {  // layer 1
    bf16x8 a;
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q] = zs[r * MLP_KP + kb + q];
    floatx4 c = {0.f, 0.f, 0.f, 0.f};
    c = mfma16(a, f.w1, c);
    bf16x4 t;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a1[q] = c[q] + f.b1;
      const __bf16 h = to_bf16(silu(a1[q]));
      h1[(row0 + q) * MLP_H + nn] = h;
      t[q] = ok[q] ? h : to_bf16(0.0f);
    }
    store_t(w.H1t, t);
    if (wv == 0) {  // the inputs, sample-contiguous (rows 10..15 are zero)
      bf16x4 z;
#pragma unroll
      for (int q = 0; q < 4; ++q) z[q] = zs[(row0 + q) * MLP_KP + r];
      *(bf16x4 *)(w.Zt + r * w.Bp + base + row0) = z;
    }
  }
  __syncthreads();
  {  // layer 2
    floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < MLP_H; ks += 32) {
      bf16x8 a;
#pragma unroll
      for (int q = 0; q < 8; ++q) a[q] = h1[r * MLP_H + ks + kb + q];
      c = mfma16(a, ks == 0 ? f.w2a : f.w2b, c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a2[q] = c[q] + f.b2;
      h2[(row0 + q) * (MLP_H + 1) + nn] = bf16_round(silu(a2[q]));
    }
  }
  __syncthreads();
  // y = b3 + sum_k w3[k] H2[b][k]; dY = 2 (y - t) / B; squared error
  if (tid < 16) {
    float acc = md.b3[0];
    for (int k = 0; k < MLP_H; ++k) acc += w3[k] * h2[tid * (MLP_H + 1) + k];
    const float d = acc - tv[tid];
    const bool in = base + tid < B;
    dy[tid] = in ? 2.0f * d / (float)B : 0.0f;
    w.dY[base + tid] = dy[tid];
    if (in) w.red[base + tid] = (double)d * (double)d;
  }
  __syncthreads();
  {  // output-layer products and dA2[b][j] = dY[b] w3[j] SiLU'(A2[b][j])
    bf16x4 t;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int64_t e = (base + row0 + q) * MLP_H + nn;
      const float y = dy[row0 + q];
      w.P[e] = y * h2[(row0 + q) * (MLP_H + 1) + nn];
      const float v = y * w3[nn] * dsilu(a2[q]);
      w.dA2[e] = v;
      t[q] = to_bf16(v);
      da2[(row0 + q) * MLP_H + nn] = t[q];
    }
    store_t(w.dA2t, t);
  }
  __syncthreads();
  {  // dH1 = dA2 W2, dA1 = dH1 SiLU'(A1)
    floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < MLP_H; ks += 32) {
      bf16x8 a;
#pragma unroll
      for (int q = 0; q < 8; ++q) a[q] = da2[r * MLP_H + ks + kb + q];
      c = mfma16(a, w2c[ks / 32], c);
    }
    bf16x4 t;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float v = c[q] * dsilu(a1[q]);
      w.dA1[(base + row0 + q) * MLP_H + nn] = v;
      t[q] = to_bf16(v);
    }
    store_t(w.dA1t, t);
  }
}

// Adam's update of parameter t and the copies of it that the products read
struct AdamPar {
  float *p, *m1, *m2;
  __bf16 *w1b, *w2b, *w2t;
  float *w3r;
  float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const AdamPar &a, int t, float gt) {
  const float m = a.b1 * a.m1[t] + (1.0f - a.b1) * gt;
  const float v = a.b2 * a.m2[t] + (1.0f - a.b2) * gt * gt;
  a.m1[t] = m;
  a.m2[t] = v;
  const float pn = a.p[t] - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
  a.p[t] = pn;
  if (t < OFF_B1) {
    a.w1b[t / MLP_IN * MLP_KP + t % MLP_IN] = to_bf16(pn);
  } else if (t >= OFF_W2 && t < OFF_B2) {
    const int e = t - OFF_W2;
    a.w2b[e] = to_bf16(pn);
    a.w2t[e % MLP_H * MLP_H + e / MLP_H] = to_bf16(pn);
  } else if (t >= OFF_W3 && t < OFF_B3) {
    a.w3r[t - OFF_W3] = bf16_round(pn);
  }
}

// Gradients from the errors of a batch, one role per block:
//   blocks 0..19   one 16 x 16 tile (the first wave) of dW2 = dA2^T H1 (16
//                  tiles) and dW1 = dA1^T Z (4 tiles), the whole batch in one
//                  MFMA chain with GR_DEPTH steps' operands loaded together;
//   blocks 20..31  column sums of P (dW3), dA2 (db2) and dA1 (db1), GR_COLS
//                  columns each: the block streams GR_ROWS rows at a time
//                  through two LDS buffers and its first wave adds them, one
//                  column per lane;
//   block 32       db3, the sum of dY.
// The chains are serial in the sample (their order is the result's), so the
// kernel's time is the longest chain's, about 4,096 dependent FP32 additions
// at the default batch, if the operands arrive in time: one compute unit
// waits about 2 us for what it can have in flight (64 KB), so the columns are
// split over 12 blocks and the tiles over 20: 34 us at a batch of 4,096, 20
// of them the additions (three blocks of 64 columns and five of four tiles:
// 67 us).
// ADAM: the update is applied to the parameters; else the gradient is stored.
constexpr int GR_DEPTH = 16, GR_COLS = 16, GR_ROWS = 1024;
constexpr int GR_TILES = 20, GR_SUMS = 3 * MLP_H / GR_COLS, GR_BLOCKS = GR_TILES + GR_SUMS + 1;

// Sums of COLS columns of X[Bp][LD] over the first B rows, ascending, one
// column per lane of the block's first wave (lanes past COLS repeat them).
// GR_ROWS rows are loaded by the whole block while the tile before them is
// added from LDS (rows past Bp repeat the last one and are not added).
template <int COLS, int LD>
__device__ __forceinline__ float column_sums(const float *X, int64_t B, int64_t Bp, float *buf) {
  const int tid = threadIdx.x;
  constexpr int PR = COLS >= 4 ? COLS / 4 : 1;      // 16-byte pieces per row
  constexpr int RP = COLS >= 4 ? 1 : 4;             // rows per piece
  constexpr int PIECES = GR_ROWS * COLS / 4, NV = PIECES / BLOCK;
  static_assert(PIECES % BLOCK == 0 && (COLS % 4 == 0 || LD == 1), "whole pieces per thread");
  float4 v[NV];
  auto load = [&](int64_t tile) {
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = u * BLOCK + tid;
      int64_t row = tile * GR_ROWS + e / PR * RP;
      row = row < Bp ? row : Bp - RP;
      v[u] = *(const float4 *)(X + row * LD + e % PR * 4);
    }
  };
  auto store = [&](int half) {
    float4 *d = (float4 *)buf + half * PIECES;
#pragma unroll
    for (int u = 0; u < NV; ++u) d[u * BLOCK + tid] = v[u];
  };
  const int64_t tiles = (B + GR_ROWS - 1) / GR_ROWS;
  float acc = 0.f;
  load(0);
  store(0);
  __syncthreads();
  for (int64_t t = 0; t < tiles; ++t) {
    if (t + 1 < tiles) load(t + 1);
    if (tid < 64) {
      const float *s = buf + (t & 1) * PIECES * 4 + tid % COLS;
      const int64_t left = B - t * GR_ROWS;
      const int rows = left < GR_ROWS ? (int)left : GR_ROWS;
      int b = 0;
      for (; b + 32 <= rows; b += 32) {
        float x[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) x[u] = s[(b + u) * COLS];
#pragma unroll
        for (int u = 0; u < 32; ++u) acc += x[u];
      }
      for (; b < rows; ++b) acc += s[b * COLS];
    }
    if (t + 1 < tiles) store((int)((t + 1) & 1));
    __syncthreads();
  }
  return acc;
}

template <bool ADAM>
__global__ void __launch_bounds__(BLOCK) k_grads(int64_t B, MlpWork w, AdamPar ad) {
  extern __shared__ float buf[];  // [2][GR_ROWS][GR_COLS] (column sums), [2][GR_ROWS] (db3)
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  auto put = [&](int t, float gt) {
    if (ADAM)
      adam_update(ad, t, gt);
    else
      w.g[t] = gt;
  };
  if (blockIdx.x < GR_TILES) {
    if (wv) return;
    const int tile = blockIdx.x;
    const int r = lane & 15, kb = (lane >> 4) * 8;
    const bool two = tile < 16;
    const int m0 = two ? tile / 4 * 16 : (tile - 16) * 16, n0 = two ? tile % 4 * 16 : 0;
    const __bf16 *A = (two ? w.dA2t : w.dA1t) + (m0 + r) * w.Bp + kb;
    const __bf16 *Bm = (two ? w.H1t : w.Zt) + (n0 + r) * w.Bp + kb;
    floatx4 c = {0.f, 0.f, 0.f, 0.f};
    for (int64_t k0 = 0; k0 < w.Bp; k0 += 32 * GR_DEPTH) {
      bf16x8 a[GR_DEPTH], b[GR_DEPTH];
#pragma unroll
      for (int u = 0; u < GR_DEPTH; ++u) {
        const int64_t k = k0 + 32 * u < w.Bp ? k0 + 32 * u : 0;  // inside the rows
        a[u] = *(const bf16x8 *)(A + k);
        b[u] = *(const bf16x8 *)(Bm + k);
      }
#pragma unroll
      for (int u = 0; u < GR_DEPTH; ++u)
        if (k0 + 32 * u < w.Bp) c = mfma16(a[u], b[u], c);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int mm = m0 + (lane >> 4) * 4 + q, nn = n0 + r;
      if (two)
        put(OFF_W2 + mm * MLP_H + nn, c[q]);
      else if (nn < MLP_IN)
        put(OFF_W1 + mm * MLP_IN + nn, c[q]);
    }
    return;
  }
  const int sum = (int)blockIdx.x - GR_TILES;
  if (sum < GR_SUMS) {
    const int which = sum * GR_COLS / MLP_H, c0 = sum * GR_COLS % MLP_H;
    const float *X = (which == 0 ? w.P : (which == 1 ? w.dA2 : w.dA1)) + c0;
    const float acc = column_sums<GR_COLS, MLP_H>(X, B, w.Bp, buf);
    if (tid < GR_COLS) put((which == 0 ? OFF_W3 : (which == 1 ? OFF_B2 : OFF_B1)) + c0 + tid, acc);
  } else {
    const float acc = column_sums<1, 1>(w.dY, B, w.Bp, buf);
    if (tid == 0) put(OFF_B3, acc);
  }
}

// fixed-order double sum of v[0..n) into *out, divided by div (one block)
__global__ void k_dsum(int64_t n, const double *__restrict__ v, double *out, double div) {
  __shared__ double s[BLOCK];
  double acc = 0.0;
  for (int64_t k = threadIdx.x; k < n; k += BLOCK) acc = acc + v[k];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int h = BLOCK / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) s[threadIdx.x] = s[threadIdx.x] + s[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = s[0] / div;
}

// Per-column sums and sums of squares of [n][cols] doubles: block b adds the
// row groups b, b + gridDim.x, ... (BLOCK / cols rows of one coalesced read
// each, a thread keeps to one column) and leaves its totals in
// part[(b cols + c) 2 ..]; the last step adds the blocks' totals in order.
// (One block per column, reading every cols-th double, took 0.25 ms at 65,536
// samples and grew with n.)
constexpr int MOM_GRID = 256;

__global__ void __launch_bounds__(BLOCK)
    k_moments(int64_t n, int cols, const double *__restrict__ X, double *part) {
  __shared__ double s1[BLOCK], s2[BLOCK];
  const int rpb = BLOCK / cols, used = rpb * cols, t = threadIdx.x;
  double a = 0.0, b = 0.0;
  if (t < used)
    for (int64_t e = (int64_t)blockIdx.x * used + t; e < n * cols; e += (int64_t)gridDim.x * used) {
      const double v = X[e];
      a = a + v;
      b = b + v * v;
    }
  s1[t] = a;
  s2[t] = b;
  __syncthreads();
  if (t < cols) {
    for (int k = 1; k < rpb; ++k) {
      a = a + s1[k * cols + t];
      b = b + s2[k * cols + t];
    }
    part[2 * ((int64_t)blockIdx.x * cols + t)] = a;
    part[2 * ((int64_t)blockIdx.x * cols + t) + 1] = b;
  }
}

// mean and standard deviation per column (out[2 c], out[2 c + 1]) from nb
// blocks' totals; one wave per column, fixed order
__global__ void __launch_bounds__(64)
    k_moments_final(int64_t n, int cols, int nb, const double *__restrict__ part, double *out) {
  const int c = blockIdx.x, l = threadIdx.x;
  double a = 0.0, b = 0.0;
  for (int k = l; k < nb; k += 64) {
    a = a + part[2 * ((int64_t)k * cols + c)];
    b = b + part[2 * ((int64_t)k * cols + c) + 1];
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    a = a + __shfl_down(a, o);
    b = b + __shfl_down(b, o);
  }
  if (l == 0) {
    const double mean = a / (double)n;
    const double var = b / (double)n - mean * mean;
    out[2 * c] = mean;
    out[2 * c + 1] = var > 0.0 ? sqrt(var) : 0.0;
  }
}

static AdamPar adam_par(const vcsgc_mlp *m) {
  AdamPar a = {};
  a.p = m->p;
  a.m1 = m->m1;
  a.m2 = m->m2;
  a.w1b = m->w1b;
  a.w2b = m->w2b;
  a.w2t = m->w2b + MLP_H * MLP_H;
  a.w3r = m->w3r;
  return a;
}

// Forward and backward pass over a batch and its gradient (into w.g, or
// straight into Adam's update of the parameters when ad is given); the
// per-sample squared errors go to w.red.
constexpr size_t GR_LDS = 2 * sizeof(float) * GR_ROWS * GR_COLS;

static hipError_t mlp_fwd_bwd(const vcsgc_mlp *m, const MlpWork &w, int64_t n, int64_t B,
                              const double *desc, const double *dE, const MlpDev &md,
                              uint64_t seed, uint64_t step, int draw, const AdamPar *ad) {
  // every padded sample is written (the pads as zeros)
  k_fwd_bwd<<<(unsigned)(w.Bp / 16), BLOCK, 0, m->stream>>>(
      n, B, desc, dE, md, m->w2b + MLP_H * MLP_H, seed, step, draw, w);
  if (ad)
    k_grads<true><<<GR_BLOCKS, BLOCK, GR_LDS, m->stream>>>(B, w, *ad);
  else
    k_grads<false><<<GR_BLOCKS, BLOCK, GR_LDS, m->stream>>>(B, w, AdamPar{});
  return hipGetLastError();
}

// more than 64 KB of LDS per block has to be asked for
static hipError_t grads_lds() {
  hipError_t e = hipFuncSetAttribute((const void *)k_grads<true>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)GR_LDS);
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void *)k_grads<false>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)GR_LDS);
  return e;
}

hipError_t mlp_ensure_cap(vcsgc_mlp *m, int64_t B) {
  if (B <= m->cap) return hipSuccess;
  (void)hipStreamSynchronize(m->stream);
  if (m->work) (void)hipFree(m->work);
  m->work = nullptr;
  if (m->red) (void)hipFree(m->red);
  m->red = nullptr;
  m->cap = 0;
  const int64_t Bp = (B + 31) / 32 * 32;
  hipError_t e = hipMalloc((void **)&m->work, (size_t)(MLP_WORK_BYTES * Bp));
  if (e == hipSuccess) e = hipMalloc((void **)&m->red, sizeof(double) * (B + 8));
  if (e != hipSuccess) return e;
  m->cap = B;
  return hipSuccess;
}

hipError_t mlp_grad_batch(vcsgc_mlp *m, const double *desc, const double *dE, int64_t n,
                          double *loss) {
  hipError_t e = mlp_ensure_cap(m, n);
  if (e != hipSuccess) return e;
  const MlpWork w = carve_work(m->work, n, m->red, m->g);
  if ((e = mlp_fwd_bwd(m, w, n, n, desc, dE, mlp_dev(m), 0, 0, 0, nullptr)) != hipSuccess) return e;
  k_dsum<<<1, BLOCK, 0, m->stream>>>(n, m->red, m->red + m->cap, 1.0);
  double h = 0.0;
  e = hipMemcpyAsync(&h, m->red + m->cap, sizeof(double), hipMemcpyDeviceToHost, m->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  if (loss) *loss = h / (double)n;
  return e;
}

hipError_t mlp_train(vcsgc_mlp *m, const double *desc, const double *dE, int64_t n,
                     const vcsgc_train_cfg *cfg, vcsgc_train_report *rep) {
  const int64_t B = cfg->batch;
  hipError_t e = mlp_ensure_cap(m, B);
  if (e != hipSuccess) return e;
  const int64_t steps_per_epoch = (n + B - 1) / B;
  const int64_t steps = steps_per_epoch * cfg->epochs;
  const MlpDev md = mlp_dev(m);
  const MlpWork w = carve_work(m->work, B, m->red, m->g);
  AdamPar ad = adam_par(m);
  ad.lr = (float)cfg->lr;
  ad.b1 = (float)cfg->beta1;
  ad.b2 = (float)cfg->beta2;
  ad.eps = (float)cfg->eps;
  double first = -1.0, last = 0.0;
  for (int64_t st = 0; st < steps; ++st) {
    m->adam_t += 1;
    ad.c1 = 1.0f - powf((float)cfg->beta1, (float)m->adam_t);
    ad.c2 = 1.0f - powf((float)cfg->beta2, (float)m->adam_t);
    if ((e = mlp_fwd_bwd(m, w, n, B, desc, dE, md, cfg->seed, (uint64_t)st, 1, &ad)) != hipSuccess)
      return e;
    // epoch-end loss of the last batch (one read-back per epoch)
    if ((st + 1) % steps_per_epoch == 0 || st == 0) {
      k_dsum<<<1, BLOCK, 0, m->stream>>>(B, m->red, m->red + m->cap, 1.0);
      double h = 0.0;
      e = hipMemcpyAsync(&h, m->red + m->cap, sizeof(double), hipMemcpyDeviceToHost, m->stream);
      if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
      if (e != hipSuccess) return e;
      h /= (double)B;
      if (first < 0.0) first = h;
      last = h;
    }
  }
  if (rep) {
    rep->loss_first = first;
    rep->loss_last = last;
    rep->steps = steps;
  }
  return hipSuccess;
}

hipError_t mlp_forward(vcsgc_mlp *m, const double *desc, int64_t n, double *dE) {
  if (n <= 0) return hipSuccess;
  k_mlp_infer<<<(unsigned)((n + 15) / 16), BLOCK, 0, m->stream>>>(mlp_dev(m), n, desc, dE);
  return hipGetLastError();
}

hipError_t mlp_fit_normalization(vcsgc_mlp *m, const double *desc, const double *dE, int64_t n) {
  double *st = m->mom + 2 * MOM_GRID * (MLP_IN + 1);
  auto blocks = [&](int cols) {
    const int64_t rpb = BLOCK / cols, g = (n + rpb - 1) / rpb;
    return (int)(g < MOM_GRID ? g : MOM_GRID);
  };
  double *part1 = m->mom + 2 * MOM_GRID * MLP_IN;
  const int g0 = blocks(MLP_IN), g1 = blocks(1);
  k_moments<<<g0, BLOCK, 0, m->stream>>>(n, MLP_IN, desc, m->mom);
  k_moments<<<g1, BLOCK, 0, m->stream>>>(n, 1, dE, part1);
  k_moments_final<<<MLP_IN, 64, 0, m->stream>>>(n, MLP_IN, g0, m->mom, st);
  k_moments_final<<<1, 64, 0, m->stream>>>(n, 1, g1, part1, st + 2 * MLP_IN);
  double h[22];
  hipError_t e = hipGetLastError();
  if (e == hipSuccess)
    e = hipMemcpyAsync(h, st, sizeof(h), hipMemcpyDeviceToHost, m->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  if (e != hipSuccess) return e;
  for (int k = 0; k < MLP_IN; ++k) {
    m->mu[k] = (float)h[2 * k];
    m->sd[k] = h[2 * k + 1] > 1e-6 ? (float)h[2 * k + 1] : 1.0f;
  }
  m->out_mu = (float)h[20];
  m->out_sd = h[21] > 1e-9 ? (float)h[21] : 1.0f;
  return hipSuccess;
}

}  // namespace vc

// ---------------------------------------------------------------------------
// C ABI of the network
// ---------------------------------------------------------------------------
namespace {

vcsgc_status mfail(vcsgc_mlp *m, hipError_t e, const char *where) {
  if (m) m->err = std::string(where) + ": " + hipGetErrorString(e);
  return VCSGC_E_DEVICE;
}

// deterministic initial weights: uniform(-1/sqrt(fan_in), 1/sqrt(fan_in)),
// zero biases, from a 64-bit linear congruential stream
void init_params(uint64_t seed, std::vector<float> &p) {
  uint64_t x = seed * 6364136223846793005ull + 1442695040888963407ull;
  auto next = [&]() {
    x = x * 6364136223846793005ull + 1442695040888963407ull;
    return (double)(x >> 11) * 0x1p-53;
  };
  p.assign(vc::MLP_NPARAM, 0.0f);
  const double s1 = 1.0 / std::sqrt(10.0), s2 = 1.0 / std::sqrt(64.0);
  for (int k = 0; k < 640; ++k) p[vc::OFF_W1 + k] = (float)((2.0 * next() - 1.0) * s1);
  for (int k = 0; k < 4096; ++k) p[vc::OFF_W2 + k] = (float)((2.0 * next() - 1.0) * s2);
  for (int k = 0; k < 64; ++k) p[vc::OFF_W3 + k] = (float)((2.0 * next() - 1.0) * s2);
}

}  // namespace

extern "C" {

vcsgc_status vcsgc_mlp_create(uint64_t seed, hipStream_t stream, vcsgc_mlp **out) {
  if (!out) return VCSGC_E_INVALID_ARG;
  vcsgc_mlp *m = new vcsgc_mlp();
  (void)hipGetDevice(&m->device);
  m->stream = stream;
  for (int k = 0; k < 10; ++k) {
    m->mu[k] = 0.f;
    m->sd[k] = 1.f;
  }
  hipError_t e = hipMalloc((void **)&m->p, sizeof(float) * vc::MLP_NPARAM);
  if (e == hipSuccess) e = hipMalloc((void **)&m->g, sizeof(float) * vc::MLP_NPARAM);
  if (e == hipSuccess) e = hipMalloc((void **)&m->m1, sizeof(float) * vc::MLP_NPARAM);
  if (e == hipSuccess) e = hipMalloc((void **)&m->m2, sizeof(float) * vc::MLP_NPARAM);
  if (e == hipSuccess) e = hipMalloc((void **)&m->w1b, sizeof(__bf16) * 64 * 32);
  if (e == hipSuccess) e = hipMalloc((void **)&m->w2b, sizeof(__bf16) * 2 * 64 * 64);
  if (e == hipSuccess)
    e = hipMalloc((void **)&m->mom, sizeof(double) * (2 * vc::MOM_GRID * (vc::MLP_IN + 1) + 22));
  if (e == hipSuccess) e = vc::grads_lds();
  if (e == hipSuccess) e = hipMalloc((void **)&m->w3r, sizeof(float) * 64);
  std::vector<float> p;
  init_params(seed, p);
  if (e == hipSuccess)
    e = hipMemcpy(m->p, p.data(), sizeof(float) * vc::MLP_NPARAM, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemsetAsync(m->m1, 0, sizeof(float) * vc::MLP_NPARAM, stream);
  if (e == hipSuccess) e = hipMemsetAsync(m->m2, 0, sizeof(float) * vc::MLP_NPARAM, stream);
  if (e == hipSuccess) e = vc::mlp_refresh(m);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    vcsgc_mlp_destroy(m);
    return e == hipErrorOutOfMemory ? VCSGC_E_OUT_OF_MEMORY : VCSGC_E_DEVICE;
  }
  *out = m;
  return VCSGC_OK;
}

vcsgc_status vcsgc_mlp_destroy(vcsgc_mlp *m) {
  if (!m) return VCSGC_OK;
  (void)hipStreamSynchronize(m->stream);
  void *ptrs[] = {m->p, m->g, m->m1, m->m2, m->w1b, m->w2b, m->w3r, m->work, m->red, m->mom};
  for (void *q : ptrs)
    if (q) (void)hipFree(q);
  delete m;
  return VCSGC_OK;
}

vcsgc_status vcsgc_mlp_set_params(vcsgc_mlp *m, const float *params, const float *mu,
                                  const float *sd, float out_mu, float out_sd) {
  if (!m || !params || !mu || !sd || !(out_sd > 0.f)) return VCSGC_E_INVALID_ARG;
  for (int k = 0; k < 10; ++k)
    if (!(sd[k] > 0.f)) return VCSGC_E_INVALID_ARG;
  hipError_t e = hipMemcpy(m->p, params, sizeof(float) * vc::MLP_NPARAM, hipMemcpyHostToDevice);
  if (e != hipSuccess) return mfail(m, e, "set_params");
  for (int k = 0; k < 10; ++k) {
    m->mu[k] = mu[k];
    m->sd[k] = sd[k];
  }
  m->out_mu = out_mu;
  m->out_sd = out_sd;
  e = vc::mlp_refresh(m);
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  return e == hipSuccess ? VCSGC_OK : mfail(m, e, "set_params");
}

vcsgc_status vcsgc_mlp_get_params(vcsgc_mlp *m, float *params, float *mu, float *sd,
                                  float *out_mu, float *out_sd) {
  if (!m) return VCSGC_E_INVALID_ARG;
  if (params) {
    hipError_t e = hipStreamSynchronize(m->stream);
    if (e == hipSuccess)
      e = hipMemcpy(params, m->p, sizeof(float) * vc::MLP_NPARAM, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return mfail(m, e, "get_params");
  }
  for (int k = 0; k < 10; ++k) {
    if (mu) mu[k] = m->mu[k];
    if (sd) sd[k] = m->sd[k];
  }
  if (out_mu) *out_mu = m->out_mu;
  if (out_sd) *out_sd = m->out_sd;
  return VCSGC_OK;
}

vcsgc_status vcsgc_mlp_fit_normalization(vcsgc_mlp *m, const double *desc_dev,
                                         const double *dE_dev, int64_t n) {
  if (!m || !desc_dev || !dE_dev || n < 2) return VCSGC_E_INVALID_ARG;
  hipError_t e = vc::mlp_fit_normalization(m, desc_dev, dE_dev, n);
  return e == hipSuccess ? VCSGC_OK : mfail(m, e, "fit_normalization");
}

vcsgc_status vcsgc_mlp_train(vcsgc_mlp *m, const double *desc_dev, const double *dE_dev,
                             int64_t n, const vcsgc_train_cfg *cfg, vcsgc_train_report *report) {
  if (!m || !desc_dev || !dE_dev || !cfg || n < 1 || cfg->epochs < 0 || cfg->batch < 1 ||
      cfg->batch > (1 << 22) || !(cfg->lr > 0.0) || !(cfg->beta1 >= 0.0 && cfg->beta1 < 1.0) ||
      !(cfg->beta2 >= 0.0 && cfg->beta2 < 1.0) || !(cfg->eps > 0.0))
    return VCSGC_E_INVALID_ARG;
  hipError_t e = vc::mlp_train(m, desc_dev, dE_dev, n, cfg, report);
  return e == hipSuccess ? VCSGC_OK : mfail(m, e, "train");
}

vcsgc_status vcsgc_mlp_forward(vcsgc_mlp *m, const double *desc_dev, int64_t n, double *dE_dev) {
  if (!m || n < 0 || (n > 0 && (!desc_dev || !dE_dev))) return VCSGC_E_INVALID_ARG;
  hipError_t e = vc::mlp_forward(m, desc_dev, n, dE_dev);
  return e == hipSuccess ? VCSGC_OK : mfail(m, e, "forward");
}

vcsgc_status vcsgc_mlp_grad(vcsgc_mlp *m, const double *desc_dev, const double *dE_dev, int64_t n,
                            float *grad_host, double *loss) {
  if (!m || !desc_dev || !dE_dev || n < 1 || n > (1 << 22)) return VCSGC_E_INVALID_ARG;
  hipError_t e = vc::mlp_grad_batch(m, desc_dev, dE_dev, n, loss);
  if (e == hipSuccess && grad_host)
    e = hipMemcpy(grad_host, m->g, sizeof(float) * vc::MLP_NPARAM, hipMemcpyDeviceToHost);
  return e == hipSuccess ? VCSGC_OK : mfail(m, e, "grad");
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Allocation-free gradient (vcsgc_mlp_grad_noalloc).  The batch's workspace
// (activations, back-propagated errors and per-sample squared errors of at
// most VCSGC_NOALLOC_MAX_SAMPLES samples) is a fixed device array, so the
// call allocates nothing on any path; outputs go to caller device memory and
// nothing is read back.  The array's device address is looked up once per
// device (hipGetSymbolAddress) and only that address reaches the kernels.
// Every kernel of the pass writes its whole output, so nothing needs clearing
// between calls; calls that overlap on one device share the array and race.
// ---------------------------------------------------------------------------
#include <mutex>

namespace vc {

constexpr int64_t NA_MAX = VCSGC_NOALLOC_MAX_SAMPLES;
constexpr size_t NA_FLOAT_BYTES = (size_t)(NA_MAX * MLP_WORK_BYTES);
constexpr size_t NA_BYTES = NA_FLOAT_BYTES + sizeof(double) * (size_t)NA_MAX;
static_assert(NA_FLOAT_BYTES % 256 == 0, "double area aligned");

static __device__ __align__(256) unsigned char scratch[NA_BYTES];

constexpr int NA_DEVICES = 64;
static void *g_scratch[NA_DEVICES] = {};
static std::mutex g_scratch_mu;

// device address of `scratch` on `dev` (looked up once per device)
static hipError_t scratch_address(int dev, unsigned char **out) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch[dev]) {
    int cur = 0;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != dev && (e = hipSetDevice(dev)) != hipSuccess) return e;
    void *ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess) return e;
    g_scratch[dev] = ptr;
  }
  *out = (unsigned char *)g_scratch[dev];
  return hipSuccess;
}

}  // namespace vc

extern "C" vcsgc_status vcsgc_mlp_grad_noalloc(const vcsgc_mlp *m, const double *desc_dev,
                                               const double *dE_dev, int64_t n, float *grad_dev,
                                               double *loss_dev) {
  if (!m || !desc_dev || !dE_dev || !grad_dev || !loss_dev) return VCSGC_E_INVALID_ARG;
  if (n < 1 || n > VCSGC_NOALLOC_MAX_SAMPLES) return VCSGC_E_INVALID_ARG;
  if (m->device < 0 || m->device >= vc::NA_DEVICES) return VCSGC_E_INVALID_ARG;
  unsigned char *base = nullptr;
  hipError_t e = vc::scratch_address(m->device, &base);
  if (e != hipSuccess) return VCSGC_E_DEVICE;
  const vc::MlpWork w =
      vc::carve_work(base, n, (double *)(base + vc::NA_FLOAT_BYTES), grad_dev);
  e = vc::mlp_fwd_bwd(m, w, n, n, desc_dev, dE_dev, vc::mlp_dev(m), 0, 0, 0, nullptr);
  if (e != hipSuccess) return VCSGC_E_DEVICE;
  vc::k_dsum<<<1, vc::BLOCK, 0, m->stream>>>(n, w.red, loss_dev, (double)n);
  return hipGetLastError() == hipSuccess ? VCSGC_OK : VCSGC_E_DEVICE;
}
