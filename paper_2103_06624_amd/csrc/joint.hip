// Kernels of the joint optimisation of intermediate bounds (Sec. 3.3, Eq.
// opt_non_convex): per-subdomain relaxation tables refreshed from the current
// bounds, the clip of computed bounds by the root bounds, the broadcast of the
// per-layer shared variables to the rows of an intermediate-bound pass and the
// weighted reduction of the rows' gradients back onto them, and the gradient
// of the bound with respect to the intermediate bounds themselves.
#include "common.h"
#include "internal.h"

namespace cvb {

namespace {

inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

constexpr float kTie = 1e-4f;  // relative width of a tie between a computed and a root bound

// status / chord of columns [0, nd_x) of handle X (row stride nd_x) from the
// current bounds (row stride nd).  A root-unstable unsplit neuron is active
// when l >= 0, inactive when u <= 0, else unstable with its root chord index;
// every other word keeps its root value (splits decide their own neurons).
__global__ void refresh_k(uint32_t* status, const uint32_t* __restrict__ status0, float2* chord,
                          const float* __restrict__ lcur, const float* __restrict__ ucur, int B, int nd_x, int nd) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)B * nd_x) return;
  const int b = (int)(i / nd_x);
  const int c = (int)(i - (int64_t)b * nd_x);
  const uint32_t r0 = status0[i];
  uint32_t r = r0;
  float2 ch = make_float2(0.f, 0.f);
  if ((r0 & kKindMask) == kUnstable) {
    const float l = lcur[(int64_t)b * nd + c], u = ucur[(int64_t)b * nd + c];
    if (l >= 0.f) {
      r = kActive;
    } else if (u <= 0.f) {
      r = kInactive;
    } else {
      // upper chord of ReLU on [l, u] (Lemma 2.1)
      const float den = u - l;
      ch = make_float2(u / den, -u * l / den);
    }
  }
  status[i] = r;
  chord[i] = ch;
}

// layer bounds from the rows of an intermediate pass ([B][2d]: z lower
// bounds, then bounds of -z): the tighter of the computed and the root bound;
// ml / mu mark where the gradient follows the computed bound -- unless it is
// looser than the root's by more than kTie max(1, |root|) (a tie is decided
// for the computed bound, whatever the rounding)
__global__ void clip_k(const float* __restrict__ lb, int d, int off, const float* __restrict__ lroot,
                       const float* __restrict__ uroot, float* lcur, float* ucur, uint8_t* ml, uint8_t* mu, int B,
                       int nd) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)B * d) return;
  const int b = (int)(i / d);
  const int j = (int)(i - (int64_t)b * d);
  const int64_t c = (int64_t)b * nd + off + j;
  const float ln = lb[(int64_t)b * 2 * d + j], un = -lb[(int64_t)b * 2 * d + d + j];
  const float lr = lroot[c], ur = uroot[c];
  lcur[c] = fmaxf(ln, lr);
  ucur[c] = fminf(un, ur);
  ml[c] = ln >= lr - kTie * fmaxf(fabsf(lr), 1.f);
  mu[c] = un <= ur + kTie * fmaxf(fabsf(ur), 1.f);
}

// alpha' rows of the pass: row (b, k) takes the shared block of its side
// (k >= d: the upper bounds); the shared blocks of b start at aoff[b] / d
__global__ void bcast_alpha_k(float* arow, const float* __restrict__ ash, Batch bt, int d) {
  const int r = blockIdx.x;
  const int b = r / bt.m, k = r - b * bt.m;
  const int uc = bt.ucount[b];
  const float* src = ash + bt.aoff[b] / d + (k >= d ? uc : 0);
  float* dst = arow + bt.rbase[r];
  for (int c = threadIdx.x; c < uc; c += blockDim.x) dst[c] = src[c];
}

__global__ void bcast_beta_k(float* brow, const float* __restrict__ bsh, int64_t nnz, int m, int d) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= nnz * m) return;
  const int64_t t = i / m;
  const int k = (int)(i - t * m);
  brow[i] = bsh[t * 2 + (k >= d ? 1 : 0)];
}

// The reductions over a pass's rows (2 d_i of them per subdomain, thousands on
// a convolutional layer) are bound by reading the per-row entries once: [rows,
// uc] floats in rows of one subdomain, contiguous (a row's entries start at
// aoff[b] + k ucount[b]).  Each sum keeps its order, row by row: the shared
// variables steer every later iterate, and a sum in another order would turn
// into another trajectory wherever a gradient is near zero.  So a workgroup
// takes 32 columns (128-byte pieces of a row), all its threads bring chunks of
// rows into LDS, the next chunk's loads in flight, and one thread per column
// walks the chunk.  One thread per column straight over memory left 8 to 30
// workgroups on the chip, each a serial chain of loads: on the CIFAR network
// with four convolutions, at four subdomains, 598 us a launch for the alpha'
// sums and 540 us for the bounds' gradient (means over the layers), against
// 42 and 29 us so.
constexpr int kRedCols = 32;
constexpr int kRedThreads = 1024;
constexpr int kRedRows = kRedThreads / kRedCols;  // rows loaded together

// s <- fmaf(w(r), x(r), s) for r = 0 .. n - 1 in order, rows with w = 0 left out
// (0 x 0 leaves s as it is); the operands of 16 rows are read together, then
// walked.
template <class W, class X>
__device__ __forceinline__ void walk(float& s, int n, W w, X x) {
  constexpr int kU = 16;
  for (int r0 = 0; r0 < n; r0 += kU) {
    float wv[kU], xv[kU];
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      const int r = min(r0 + q, n - 1);
      wv[q] = w(r);
      xv[q] = x(r);
    }
#pragma unroll
    for (int q = 0; q < kU; ++q) {
      const float wq = r0 + q < n ? wv[q] : 0.f;
      s = fmaf(wq, wq != 0.f ? xv[q] : 0.f, s);
    }
  }
}

// shared gradient of side s of subdomain b = sum over the side's rows of
// w[row] x the row's gradient (a row of weight 0 contributes nothing)
__global__ __launch_bounds__(kRedThreads) void reduce_alpha_k(float* gash, const float* __restrict__ garow,
                                                              const float* __restrict__ w, Batch bt, int d) {
  constexpr int kQ = 7, kChunk = kRedRows * kQ;  // (two buffers within 64 KB)
  __shared__ float xs[2][kChunk][kRedCols], ws[2][kChunk];
  const int b = blockIdx.x >> 1, side = blockIdx.x & 1;
  const int uc = bt.ucount[b];
  const int c0 = blockIdx.y * kRedCols;
  if (c0 >= uc) return;  // uniform over the workgroup
  const int t = threadIdx.x % kRedCols, g = threadIdx.x / kRedCols;
  const int c = min(c0 + t, uc - 1);
  const int k0 = side * d;
  const float* const wr = w + (int64_t)b * bt.m + k0;
  const float* const gr = garow + bt.aoff[b] + (int64_t)k0 * uc + c;
  float x[kQ], wk = 0.f;
  auto load = [&](int k) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) x[q] = gr[(int64_t)min(k + q * kRedRows + g, d - 1) * uc];
    if (threadIdx.x < kChunk) wk = k + (int)threadIdx.x < d ? wr[k + threadIdx.x] : 0.f;
  };
  load(0);
  float s = 0.f;
  for (int k = 0, buf = 0; k < d; k += kChunk, buf ^= 1) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) xs[buf][q * kRedRows + g][t] = x[q];
    if (threadIdx.x < kChunk) ws[buf][threadIdx.x] = wk;
    if (k + kChunk < d) load(k + kChunk);
    __syncthreads();
    if (g == 0) {
      const int n = min(kChunk, d - k);
      walk(s, n, [&](int r) { return ws[buf][r]; }, [&](int r) { return xs[buf][r][t]; });
    }
  }
  if (g == 0 && c0 + t < uc) gash[bt.aoff[b] / d + side * uc + c] = s;
}

// the same for beta': one wave per (split, side), its rows brought into LDS
__global__ __launch_bounds__(64) void reduce_beta_k(float* gbsh, const float* __restrict__ gbrow,
                                                    const float* __restrict__ w, const int* __restrict__ split_dom,
                                                    int m, int d) {
  constexpr int kQ = 8, kChunk = 64 * kQ;
  __shared__ float xs[kChunk], ws[kChunk];
  const int64_t q0 = blockIdx.x, t = q0 >> 1;
  const int side = (int)(q0 & 1), lane = threadIdx.x;
  const float* const wr = w + (int64_t)split_dom[t] * m + side * d;
  const float* const gr = gbrow + t * m + side * d;
  float s = 0.f;
  for (int k = 0; k < d; k += kChunk) {
    float x[kQ], wk[kQ];
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int i = min(k + 64 * q + lane, d - 1);
      x[q] = gr[i];
      wk[q] = wr[i];
    }
    __syncthreads();  // the chunk before has been walked
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      xs[64 * q + lane] = x[q];
      ws[64 * q + lane] = wk[q];
    }
    __syncthreads();
    const int n = min(kChunk, d - k);
    if (lane == 0)
      walk(s, n, [&](int r) { return ws[r]; }, [&](int r) { return xs[r]; });
  }
  if (lane == 0) gbsh[q0] = s;
}

// d(sum_rows w g)/dl and /du at the currently unstable neurons of columns
// [col0, nd_x) of handle X, added into dL, dU [B][nd].  A row uses the upper
// chord u (z - l)/(u - l) where its stored A is negative; with zbar the
// adjoint's pre-activation there, the chord term A (s zbar - s l) has
// d/dl = A u (zbar - u)/(u - l)^2 and d/du = A l (l - zbar)/(u - l)^2.
// One workgroup per 32 columns of a subdomain, as above: its threads form each
// row's terms, half a wave walks the sum for l and half the one for u.
__global__ __launch_bounds__(kRedThreads) void cot_k(float* dL, float* dU, const uint32_t* __restrict__ status,
                                                     const float* __restrict__ acomp,
                                                     const float* __restrict__ zchord, const float* __restrict__ w,
                                                     const float* __restrict__ lcur, const float* __restrict__ ucur,
                                                     Batch bt, int col0, int nd_x, int nd) {
  constexpr int kQ = 4, kChunk = kRedRows * kQ;
  // a row's term is cs es[0] (for l), cs es[1] (for u)
  __shared__ float cs[kChunk][kRedCols], es[2][kChunk][kRedCols];
  const int b = blockIdx.x;
  const int t = threadIdx.x % kRedCols, g = threadIdx.x / kRedCols;
  const int c = col0 + blockIdx.y * kRedCols + t;
  const uint32_t rec = c < nd_x ? status[(int64_t)b * nd_x + c] : kInactive;
  const bool uns = (rec & kKindMask) == kUnstable;
  const int m = bt.m, uc = bt.ucount[bt.prop[b]];
  const int64_t cb = (int64_t)b * nd + c, a0 = bt.aoff[b] + (uns ? rec & kCidxMask : 0);
  const float* const wr = w ? w + (int64_t)b * m : nullptr;
  const float l = uns ? lcur[cb] : 0.f, u = uns ? ucur[cb] : 0.f;
  float a[kQ], z[kQ], wk[kQ];
  auto load = [&](int k) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int r = k + q * kRedRows + g, kr = min(r, m - 1);
      a[q] = z[q] = wk[q] = 0.f;
      if (!uns) continue;
      wk[q] = r < m ? (wr ? wr[kr] : 1.f) : 0.f;
      a[q] = acomp[a0 + (int64_t)kr * uc];
      z[q] = zchord[a0 + (int64_t)kr * uc];  // meaningful where a < 0
    }
  };
  load(0);
  float s = 0.f;
  for (int k = 0; k < m; k += kChunk) {
    __syncthreads();  // the chunk before has been walked
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int r = q * kRedRows + g;
      const bool on = wk[q] != 0.f && a[q] < 0.f;
      cs[r][t] = on ? wk[q] * a[q] : 0.f;
      es[0][r][t] = on ? u * (z[q] - u) : 0.f;
      es[1][r][t] = on ? l * (l - z[q]) : 0.f;
    }
    if (k + kChunk < m) load(k + kChunk);
    __syncthreads();
    if (g < 2) {
      const int n = min(kChunk, m - k);
#pragma unroll 16
      for (int r = 0; r < n; ++r) s = fmaf(cs[r][t], es[g][r][t], s);
    }
  }
  if (g < 2 && uns) {
    const float den = u - l;
    const float inv2 = 1.f / (den * den);
    (g == 0 ? dL : dU)[cb] += s * inv2;
  }
}

// row weights of the pass of layer (off, d): the bound cotangents where the
// computed bound is the one in use (lower rows: dL; upper rows: -dU, their
// bound being -u)
__global__ void weights_k(float* w, const float* __restrict__ dL, const float* __restrict__ dU,
                          const uint8_t* __restrict__ ml, const uint8_t* __restrict__ mu, int B, int d, int off,
                          int nd) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)B * d) return;
  const int b = (int)(i / d);
  const int j = (int)(i - (int64_t)b * d);
  const int64_t c = (int64_t)b * nd + off + j;
  w[(int64_t)b * 2 * d + j] = ml[c] ? dL[c] : 0.f;
  w[(int64_t)b * 2 * d + d + j] = mu[c] ? -dU[c] : 0.f;
}

// shared alpha' at CROWN's adaptive slope of the root bounds: block (b, side)
// fills its uc_b entries from the default-slope table adef [B][nd_x] through
// b's unstable list
__global__ void alpha_init_k(float* ash, const int* __restrict__ ulist, const int64_t* __restrict__ uoff, Batch bt,
                             int d) {
  const int b = blockIdx.x, side = blockIdx.y;
  const int uc = bt.ucount[b];
  float* dst = ash + bt.aoff[b] / d + side * uc;
  const int* src = ulist + uoff[b];
  const float* ad = bt.adef + (int64_t)b * bt.nd;
  for (int c = threadIdx.x; c < uc; c += blockDim.x) dst[c] = ad[src[c]];
}

}  // namespace

void launch_joint_alpha_init(float* ash, const int* ulist, const int64_t* uoff, const Batch& bt, int B, int d,
                             hipStream_t s) {
  if (B > 0) alpha_init_k<<<dim3(B, 2), 256, 0, s>>>(ash, ulist, uoff, bt, d);
}

void launch_joint_refresh(uint32_t* status, const uint32_t* status0, float2* chord, const float* lcur,
                          const float* ucur, int B, int nd_x, int nd, hipStream_t s) {
  const int64_t n = (int64_t)B * nd_x;
  if (n > 0) refresh_k<<<nblk(n, 256), 256, 0, s>>>(status, status0, chord, lcur, ucur, B, nd_x, nd);
}

void launch_joint_clip(const float* lb, int d, int off, const float* lroot, const float* uroot, float* lcur,
                       float* ucur, uint8_t* ml, uint8_t* mu, int B, int nd, hipStream_t s) {
  const int64_t n = (int64_t)B * d;
  if (n > 0) clip_k<<<nblk(n, 256), 256, 0, s>>>(lb, d, off, lroot, uroot, lcur, ucur, ml, mu, B, nd);
}

void launch_joint_bcast(float* arow, const float* ash, float* brow, const float* bsh, const Batch& bt, int d,
                        int64_t nnz, hipStream_t s) {
  if (bt.n_rows > 0) bcast_alpha_k<<<bt.n_rows, 256, 0, s>>>(arow, ash, bt, d);
  if (nnz > 0) bcast_beta_k<<<nblk(nnz * bt.m, 256), 256, 0, s>>>(brow, bsh, nnz, bt.m, d);
}

void launch_joint_reduce(float* gash, const float* garow, float* gbsh, const float* gbrow, const float* w,
                         const Batch& bt, int B, int d, int ucmax, const int* split_dom, int64_t nnz, hipStream_t s) {
  if (B <= 0) return;
  if (ucmax > 0)
    reduce_alpha_k<<<dim3(2 * B, nblk(ucmax, kRedCols)), kRedThreads, 0, s>>>(gash, garow, w, bt, d);
  if (nnz > 0) reduce_beta_k<<<(unsigned)(nnz * 2), 64, 0, s>>>(gbsh, gbrow, w, split_dom, bt.m, d);
}

void launch_joint_cot(float* dL, float* dU, const uint32_t* status, const float* acomp, const float* zchord,
                      const float* w, const float* lcur, const float* ucur, const Batch& bt, int col0, int nd_x,
                      int nd, int B, hipStream_t s) {
  if (B > 0 && nd_x > col0)
    cot_k<<<dim3(B, nblk(nd_x - col0, kRedCols)), kRedThreads, 0, s>>>(dL, dU, status, acomp, zchord, w, lcur, ucur,
                                                                       bt, col0, nd_x, nd);
}

void launch_joint_weights(float* w, const float* dL, const float* dU, const uint8_t* ml, const uint8_t* mu, int B,
                          int d, int off, int nd, hipStream_t s) {
  const int64_t n = (int64_t)B * d;
  if (n > 0) weights_k<<<nblk(n, 256), 256, 0, s>>>(w, dL, dU, ml, mu, B, d, off, nd);
}

}  // namespace cvb
