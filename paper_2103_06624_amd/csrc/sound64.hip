// Sound-mode evaluation of the bound in float64 (gfx950).
//
// The same recursion as the float32 kernels (Theorem 3.1, Eq. definition_A:
// Lambda(i) = A(i) D(i) + beta^T S(i), A(i-1) = Lambda(i) W(i), the constants
// A lowerb + Lambda b, and the concretisation of A(0) over the input set),
// carried out in double: the specification merged into the last layer, every
// product, the relaxation (with the chord u/(u-l), -ul/(u-l) formed in double
// from the float bounds), the constants and the concretisation.  Each kernel
// also accumulates a rigorous bound on its own float64 rounding error, per
// row (weights per neuron from the host analysis, with the unit roundoff of
// double), and the final sum subtracts it and rounds the result down to
// float: the reported bound lies below the exact bound of the same relaxation
// by that margin (about 1e-13 of the terms' magnitudes) plus one float ulp.
//
// One workgroup per batch row for the dense and convolution layers (the rows'
// inputs in LDS), on large batches up to three rows of a subdomain; one wave per row
// for the top layer.  These kernels run once per evaluation in sound
// mode, not in the optimiser's loop.
#include "common.h"
#include "internal.h"

#include <type_traits>
#include <utility>

namespace cvb {

namespace {

__device__ __forceinline__ double wave_sum_d(double x) {
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Sum over a 256-thread block, returned to thread 0 (red: 4 doubles of LDS).
__device__ __forceinline__ double block_sum_d(double x, double* red) {
  x = wave_sum_d(x);
  __syncthreads();  // red may still be read from the previous call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return threadIdx.x == 0 ? (red[0] + red[1]) + (red[2] + red[3]) : 0.0;
}

// Relaxation of one neuron in double (Lemma 2.1 cases, the split term); adds
// A lowerb + Lambda b to cst and |Lambda| sw to err; returns Lambda.
__device__ __forceinline__ double relax64(const Pass64& q, const RowInfo& ri, uint32_t rec, int64_t pc, double a,
                                          double bias, double& cst, double& err) {
  const uint32_t kind = rec & kKindMask;
  double lam = 0.0;
  if (kind == kActive) {
    lam = a;
  } else if (kind == kUnstable) {
    if (a >= 0.0) {
      const int64_t ai = ri.abase + (rec & kCidxMask);
      lam = (double)(q.alpha ? q.alpha[ai] : q.bt.adef[pc]) * a;
    } else {
      const double l = q.l[pc], u = q.u[pc];
      const double den = u - l;  // exact: both are floats
      lam = a * (u / den);
      cst += a * (-(u * l) / den);
    }
  } else if (kind == kSplit) {
    const double be = q.beta[(int64_t)(rec & kSplitMask) * q.bt.m + ri.k];
    lam = (rec & kSidePos) ? a - be : be;
  }
  cst += lam * bias;
  err += fabs(lam) * (double)q.sw[pc];
  return lam;
}

// Concretisation of one input coordinate: the box minimum, or over an l2 ball
// A x0 (with A^2 into sq).
__device__ __forceinline__ void conc64(const Pass64& q, int p, int j, double a, double& cst, double& err,
                                       double& sq) {
  const int64_t pb = (int64_t)p * q.bt.d0 + j;
  if (q.bt.l2x0) {
    cst += a * (double)q.bt.l2x0[pb];
    sq += a * a;
    return;
  }
  const double tm = fmin(a * (double)q.bt.xlo[pb], a * (double)q.bt.xhi[pb]);
  cst += tm;
  err += q.sg * fabs(tm);
}

// relax64 / conc64 over a thread's outputs j0 + 256 u (u < kC, those below
// N), in ascending j: the operands are loaded first, in two rounds of
// independent loads (the status words, then what they select), and each
// neuron then takes relax64's (conc64's) arithmetic in the same order.
template <int kC>
__device__ __forceinline__ void epi64(const Pass64& q, const RowInfo& ri, const Lay64& y, int row, int j0,
                                      const double (&a)[kC], double& cst, double& err, double& sq) {
  if (y.conc) {
    float x0[kC], x1[kC];
#pragma unroll
    for (int u = 0; u < kC; ++u) {
      const int j = j0 + 256 * u;
      x0[u] = x1[u] = 0.f;
      if (j < y.N) {
        const int64_t pb = (int64_t)ri.p * q.bt.d0 + j;
        if (q.bt.l2x0) {
          x0[u] = q.bt.l2x0[pb];
        } else {
          x0[u] = q.bt.xlo[pb];
          x1[u] = q.bt.xhi[pb];
        }
      }
    }
    // local copies, all three written back, so that neither branch updates
    // its sum through memory
    double c = cst, e = err, s2 = sq;
    if (q.bt.l2x0) {
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        if (j0 + 256 * u >= y.N) continue;
        c += a[u] * (double)x0[u];
        s2 += a[u] * a[u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        if (j0 + 256 * u >= y.N) continue;
        const double tm = fmin(a[u] * (double)x0[u], a[u] * (double)x1[u]);
        c += tm;
        e += q.sg * fabs(tm);
      }
    }
    cst = c;
    err = e;
    sq = s2;
    return;
  }
  uint32_t rec[kC];
#pragma unroll
  for (int u = 0; u < kC; ++u) {
    const int j = j0 + 256 * u;
    rec[u] = j < y.N ? q.bt.status[(int64_t)ri.b * q.bt.nd + y.layer_off + j] : 0u;
  }
  // o0: alpha (unstable, A >= 0), l (unstable, A < 0) or beta (split); o1: u
  float o0[kC], o1[kC], swv[kC], bv[kC];
#pragma unroll
  for (int u = 0; u < kC; ++u) {
    const int j = j0 + 256 * u;
    o0[u] = o1[u] = swv[u] = bv[u] = 0.f;
    if (j >= y.N) continue;
    const int64_t pc = (int64_t)ri.p * q.bt.nd + y.layer_off + j;
    swv[u] = q.sw[pc];
    bv[u] = y.bias[j];
    const uint32_t kind = rec[u] & kKindMask;
    if (kind == kUnstable) {
      if (a[u] >= 0.0) {
        o0[u] = q.alpha ? q.alpha[ri.abase + (rec[u] & kCidxMask)] : q.bt.adef[pc];
      } else {
        o0[u] = q.l[pc];
        o1[u] = q.u[pc];
      }
    } else if (kind == kSplit) {
      o0[u] = q.beta[(int64_t)(rec[u] & kSplitMask) * q.bt.m + ri.k];
    }
  }
#pragma unroll
  for (int u = 0; u < kC; ++u) {
    const int j = j0 + 256 * u;
    if (j >= y.N) continue;
    const uint32_t kind = rec[u] & kKindMask;
    const double av = a[u];
    double lam = 0.0;
    if (kind == kActive) {
      lam = av;
    } else if (kind == kUnstable) {
      if (av >= 0.0) {
        lam = (double)o0[u] * av;
      } else {
        const double l = o0[u], uu = o1[u];
        const double den = uu - l;  // exact: both are floats
        lam = av * (uu / den);
        cst += av * (-(uu * l) / den);
      }
    } else if (kind == kSplit) {
      const double be = o0[u];
      lam = (rec[u] & kSidePos) ? av - be : be;
    }
    cst += lam * (double)bv[u];
    err += fabs(lam) * (double)swv[u];
    y.out[(int64_t)row * y.ldo + j] = lam;
  }
}

// The same for kC outputs j0 + st u (u < nu) in kR rows of one subdomain,
// row0 .. row0 + nr - 1 (nr uniform over the workgroup): everything the
// epilogue reads is read ahead of the products -- what the rows share (status
// word, chord in double, weights, bias, or the box) once for all of them --
// and relax64's (conc64's) arithmetic then runs on registers, as selects.
template <int kC, int kR>
struct Epi64 {
  uint32_t rec[kC];
  float sw[kC], bias[kC], var[kR][kC];  // var: alpha (unstable) or beta (split); (concretisation: sw, bias the box)
  double2 ch[kC];

  // (loads are unconditional, outputs that do not exist read j0's operands and
  // neurons without a variable their weight: a load under a branch of its own
  // is waited for at the branch's end, one after the other)
  __device__ __forceinline__ void read(const Pass64& q, const Lay64& y, int row0, int nr, int j0, int st, int nu) {
    const int b = row0 / q.bt.m, k0 = row0 - b * q.bt.m, p = q.bt.prop[b];
    if (y.conc) {
      const float* const lo = (q.bt.l2x0 ? q.bt.l2x0 : q.bt.xlo) + (int64_t)p * q.bt.d0 + j0;
      const float* const hi = (q.bt.l2x0 ? q.bt.l2x0 : q.bt.xhi) + (int64_t)p * q.bt.d0 + j0;
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        sw[u] = lo[u < nu ? st * u : 0];
        bias[u] = hi[u < nu ? st * u : 0];
      }
      return;
    }
    const int64_t pc0 = (int64_t)p * q.bt.nd + y.layer_off + j0;
#pragma unroll
    for (int u = 0; u < kC; ++u) {
      const int d = u < nu ? st * u : 0;
      rec[u] = q.bt.status[(int64_t)b * q.bt.nd + y.layer_off + j0 + d];
      sw[u] = q.sw[pc0 + d];
      bias[u] = y.bias[j0 + d];
      ch[u] = q.chord[pc0 + d];
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int rr = r < nr ? r : 0;
      const int64_t ab = q.bt.rbase[row0 + rr];
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        const uint32_t kind = rec[u] & kKindMask;
        const int64_t pc = pc0 + (u < nu ? st * u : 0);
        const float* v = q.alpha ? q.sw + pc : q.bt.adef + pc;
        v = q.alpha && kind == kUnstable ? q.alpha + (ab + (rec[u] & kCidxMask)) : v;
        v = kind == kSplit ? q.beta + ((int64_t)(rec[u] & kSplitMask) * q.bt.m + k0 + rr) : v;
        var[r][u] = *v;
      }
    }
  }

  __device__ __forceinline__ void apply(const Pass64& q, const Lay64& y, int row0, int nr, int j0, int st, int nu,
                                        const double (&a)[kR][kC], double (&cst)[kR], double (&err)[kR],
                                        double (&sq)[kR]) const {
    if (y.conc) {
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        if (r >= nr) break;
#pragma unroll
        for (int u = 0; u < kC; ++u) {
          if (u >= nu) continue;
          const double av = a[r][u];
          if (q.bt.l2x0) {
            cst[r] += av * (double)sw[u];
            sq[r] += av * av;
          } else {
            const double tm = fmin(av * (double)sw[u], av * (double)bias[u]);
            cst[r] += tm;
            err[r] += q.sg * fabs(tm);
          }
        }
      }
      return;
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      if (r >= nr) break;
      double* const out = y.out + (int64_t)(row0 + r) * y.ldo + j0;
#pragma unroll
      for (int u = 0; u < kC; ++u) {
        const double av = a[r][u], vr = var[r][u];
        const uint32_t kind = u < nu ? rec[u] & kKindMask : kInactive;
        const bool neg = kind == kUnstable && !(av >= 0.0);
        double lam = kind == kActive ? av : 0.0;
        lam = kind == kUnstable ? (neg ? av * ch[u].x : vr * av) : lam;
        lam = kind == kSplit ? ((rec[u] & kSidePos) ? av - vr : vr) : lam;
        cst[r] += neg ? av * ch[u].y : 0.0;
        cst[r] += lam * (double)bias[u];
        err[r] += fabs(lam) * (double)sw[u];
        if (u < nu) out[st * u] = lam;
      }
    }
  }
};

// Chords of every neuron in double, u/(u-l) and -ul/(u-l) (the difference of
// two floats is exact): what relax64 forms at each use.
__global__ void chord64_k(const float* __restrict__ l, const float* __restrict__ u, double2* __restrict__ ch, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double lv = l[i], uv = u[i], den = uv - lv;
  ch[i] = den > 0.0 ? make_double2(uv / den, -(uv * lv) / den) : make_double2(0.0, 0.0);
}

// The top ReLU layer: A(L-1) = C_p W(L) in double (general specification) or
// the exact rows +-W(L) (identity specification, as float rows CW), relaxed
// (or concretised when there is no ReLU layer).  One wave per row.
__global__ __launch_bounds__(256) void top64_k(Pass64 q, Top64 t) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= q.bt.n_rows) return;
  const RowInfo ri = row_info(q.bt, row);
  double cst = 0.0, err = 0.0, sq = 0.0;
  double c0;
  const float* crow = t.C ? t.C + ((int64_t)ri.p * q.bt.m + ri.k) * t.dL : nullptr;
  if (crow) {
    c0 = 0.0;
    for (int o = 0; o < t.dL; ++o) c0 += (double)crow[o] * (double)t.bL[o];
  } else {
    c0 = (double)t.Cb[ri.p * t.cb_pstride + ri.k];
  }
  for (int j = lane; j < t.n; j += 64) {
    double a;
    if (crow) {
      a = 0.0;
      for (int o = 0; o < t.dL; ++o) a += (double)crow[o] * (double)t.WL[(int64_t)o * t.ldw + j];
    } else {
      a = (double)t.CW[ri.p * t.cw_pstride + (int64_t)ri.k * t.ldcw + j];
    }
    if (t.conc) {
      conc64(q, ri.p, j, a, cst, err, sq);
    } else {
      const int64_t pc = (int64_t)ri.p * q.bt.nd + t.layer_off + j;
      const uint32_t rec = q.bt.status[(int64_t)ri.b * q.bt.nd + t.layer_off + j];
      t.out[(int64_t)row * t.ldo + j] = relax64(q, ri, rec, pc, a, (double)t.bias[j], cst, err);
    }
  }
  cst = wave_sum_d(cst);
  err = wave_sum_d(err);
  sq = wave_sum_d(sq);
  if (lane == 0) {
    q.part[row] = cst + c0;
    q.perr[row] = err + (double)t.err0[ri.p * q.bt.m + ri.k];
    if (q.psq) q.psq[row] = sq;
  }
}

// Back-substitution through dense layer i: A(i-1)_j = sum_k Lambda(i)_k W(i)_kj
// in double, then the relaxation of layer i-1 (or the concretisation).
__global__ __launch_bounds__(256) void dense64_k(Pass64 q, Lay64 y) {
  extern __shared__ double lam_s[];
  __shared__ double red[4];
  const int row = blockIdx.x;
  const RowInfo ri = row_info(q.bt, row);
  for (int k = threadIdx.x; k < y.K; k += 256) lam_s[k] = y.in[(int64_t)row * y.ldi + k];
  __syncthreads();
  double cst = 0.0, err = 0.0, sq = 0.0;
  for (int j = threadIdx.x; j < y.N; j += 256) {
    double a = 0.0;
    for (int k = 0; k < y.K; ++k) a += lam_s[k] * (double)y.W[(int64_t)k * y.ldw + j];
    if (y.conc) {
      conc64(q, ri.p, j, a, cst, err, sq);
    } else {
      const int64_t pc = (int64_t)ri.p * q.bt.nd + y.layer_off + j;
      const uint32_t rec = q.bt.status[(int64_t)ri.b * q.bt.nd + y.layer_off + j];
      y.out[(int64_t)row * y.ldo + j] = relax64(q, ri, rec, pc, a, (double)y.bias[j], cst, err);
    }
  }
  const double c = block_sum_d(cst, red), e = block_sum_d(err, red), s2 = block_sum_d(sq, red);
  if (threadIdx.x == 0) {
    q.part[(int64_t)y.slot * q.bt.n_rows + row] = c;
    q.perr[(int64_t)y.slot * q.bt.n_rows + row] = e;
    if (q.psq) q.psq[(int64_t)y.slot * q.bt.n_rows + row] = s2;
  }
}

// The rows' sums over a workgroup's threads, to their slots: within each wave,
// then (red: 3 kR NW doubles) over its NW waves.
template <int kR, int NW>
__device__ __forceinline__ void block_out64(const Pass64& q, int slot, int row0, int nr, double (&cst)[kR],
                                            double (&err)[kR], double (&sq)[kR], double* red) {
  const int wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      cst[r] += __shfl_xor(cst[r], o, 64);
      err[r] += __shfl_xor(err[r], o, 64);
      if (q.psq) sq[r] += __shfl_xor(sq[r], o, 64);
    }
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      red[(3 * r) * NW + wid] = cst[r];
      red[(3 * r + 1) * NW + wid] = err[r];
      red[(3 * r + 2) * NW + wid] = sq[r];
    }
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 3 * nr; t += 64 * NW) {
    double v = red[NW * t];
#pragma unroll
    for (int i = 1; i < NW; ++i) v += red[NW * t + i];
    const int r = t / 3, c = t - 3 * r;
    const int64_t o = (int64_t)slot * q.bt.n_rows + row0 + r;
    if (c == 0) q.part[o] = v;
    else if (c == 1) q.perr[o] = v;
    else if (q.psq) q.psq[o] = v;
  }
}

// First row and rows (at most kR) of workgroup blockIdx.x: a subdomain's rows
// in groups of kR.
template <int kR>
__device__ __forceinline__ void row_group(int m, int* row0, int* nr) {
  const int per = (m + kR - 1) / kR, b = blockIdx.x / per, k0 = (blockIdx.x - b * per) * kR;
  *row0 = b * m + k0;
  *nr = min(kR, m - k0);
}

// The same for up to kR rows of one subdomain per workgroup, on large batches.
// In the one-row kernel a product takes a load and a conversion of its weight;
// here both serve kR rows, and Lambda, the same for every lane, is read by
// scalar loads.  100 -> 512 at 9216
// rows: 130 us in the one-row kernel, 65 here (nine rows 154, five 101: fewer
// waves fit).  Each row's sums over k keep the one-row order.
template <int kR, int NW>
__global__ __launch_bounds__(64 * NW) void dense64_rows_k(Pass64 q, Lay64 y, const double* __restrict__ in,
                                                          const float* __restrict__ W) {
  __shared__ double red[3 * kR * NW];
  int row0, nr;
  row_group<kR>(q.bt.m, &row0, &nr);
  double cst[kR], err[kR], sq[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) cst[r] = err[r] = sq[r] = 0.0;
  const double* const lam = in + (int64_t)row0 * y.ldi;  // (whole groups readable; results past nr are dropped)
  for (int j = threadIdx.x; j < y.N; j += 64 * NW) {
    Epi64<1, kR> ep;
    ep.read(q, y, row0, nr, j, 0, 1);
    double a[kR][1];
#pragma unroll
    for (int r = 0; r < kR; ++r) a[r][0] = 0.0;
#pragma unroll 8
    for (int k = 0; k < y.K; ++k) {
      const double w = (double)W[(int64_t)k * y.ldw + j];
#pragma unroll
      for (int r = 0; r < kR; ++r) a[r][0] = fma(lam[(int64_t)r * y.ldi + k], w, a[r][0]);
    }
    ep.apply(q, y, row0, nr, j, 0, 1, a, cst, err, sq);
  }
  block_out64<kR, NW>(q, y.slot, row0, nr, cst, err, sq, red);
}

// a[U] = f(U) for the constant indices U (the array stays in registers).
template <int kC, class F, int... U>
__device__ __forceinline__ void fill_seq(double (&a)[kC], F f, std::integer_sequence<int, U...>) {
  ((a[U] = f(U)), ...);
}

// A(i-1) at input position j of a conv layer (0 for j >= N): the taps with
// iy + p - ky a non-negative multiple of the stride, in ascending ky (then kx,
// then co): ky = ry, ry + s, ... and oy = oy0, oy0 - 1, ...
__device__ __forceinline__ double tap_sum64(const double* lam_s, const float* W, const ConvGeom& g, int N, int j) {
  if (j >= N) return 0.0;
  const int ci = j / (g.hi * g.wi), rem = j - ci * g.hi * g.wi;
  const int iy = rem / g.wi, ix = rem - iy * g.wi;
  const int ry = (iy + g.p) % g.s, rx = (ix + g.p) % g.s;
  const int oy0 = (iy + g.p - ry) / g.s, ox0 = (ix + g.p - rx) / g.s;
  double acc = 0.0;
  for (int ky = ry, oy = oy0; ky < g.k && oy >= 0; ky += g.s, --oy) {
    if (oy >= g.ho) continue;
    for (int kx = rx, ox = ox0; kx < g.k && ox >= 0; kx += g.s, --ox) {
      if (ox >= g.wo) continue;
#pragma unroll 8
      for (int co = 0; co < g.co; ++co)
        acc += lam_s[(co * g.ho + oy) * g.wo + ox] * (double)W[((co * g.ci + ci) * g.k + ky) * g.k + kx];
    }
  }
  return acc;
}

constexpr int kC64 = 8;  // outputs per thread per pass of the conv kernel

// The outputs of one row, with the weights W in LDS or in global memory (a
// separate instance for each, so that LDS weights are read as LDS).
template <int kC>
__device__ __forceinline__ void conv64_row(const Pass64& q, const Lay64& y, const ConvGeom& g, const RowInfo& ri,
                                           int row, const double* lam_s, const float* W, double& cst, double& err,
                                           double& sq) {
  for (int j0 = threadIdx.x; j0 < y.N; j0 += 256 * kC) {
    double a[kC];
    fill_seq(a, [&](int u) { return tap_sum64(lam_s, W, g, y.N, j0 + 256 * u); }, std::make_integer_sequence<int, kC>{});
    epi64<kC>(q, ri, y, row, j0, a, cst, err, sq);
  }
}

// The outputs of one row when the plane size hi wi divides 256 (DCI = 256 /
// (hi wi)): a thread's outputs j0 + 256 u then sit at one position, in
// channels ci0 + DCI u, and share their taps, so each Lambda value read from
// LDS serves all kC of them.  wt holds the weights in LDS as [co][ky][kx][cip]
// (input channel innermost, zero past ci).  Each output's sum keeps the order
// of tap_sum64.
template <int kC, int DCI>
__device__ __forceinline__ void conv64_row_pos(const Pass64& q, const Lay64& y, const ConvGeom& g,
                                               const RowInfo& ri, int row, const double* lam_s, const float* wt,
                                               int cip, double& cst, double& err, double& sq) {
  constexpr int hw = 256 / DCI;
  for (int j0 = threadIdx.x; j0 < y.N; j0 += 256 * kC) {
    const int ci0 = j0 / hw, pos = j0 - ci0 * hw;
    const int iy = pos / g.wi, ix = pos - iy * g.wi;
    const int ry = (iy + g.p) % g.s, rx = (ix + g.p) % g.s;
    const int oy0 = (iy + g.p - ry) / g.s, ox0 = (ix + g.p - rx) / g.s;
    double a[kC];
#pragma unroll
    for (int u = 0; u < kC; ++u) a[u] = 0.0;
    for (int ky = ry, oy = oy0; ky < g.k && oy >= 0; ky += g.s, --oy) {
      if (oy >= g.ho) continue;
      for (int kx = rx, ox = ox0; kx < g.k && ox >= 0; kx += g.s, --ox) {
        if (ox >= g.wo) continue;
        const float* wp = wt + (ky * g.k + kx) * cip + ci0;
#pragma unroll 2
        for (int co = 0; co < g.co; ++co) {
          const double l = lam_s[(co * g.ho + oy) * g.wo + ox];
          const float* w = wp + co * g.k * g.k * cip;
#pragma unroll
          for (int u = 0; u < kC; ++u) a[u] += l * (double)w[DCI * u];
        }
      }
    }
    epi64<kC>(q, ri, y, row, j0, a, cst, err, sq);
  }
}

// The outputs of one row for a 3-channel input of 1024 positions (32x32):
// N = 3072, so a thread's outputs j0 + 256 u (u < 12, one pass) sit at four
// positions j0 + 256 g, each in all three channels (u = g + 4 c).  Each
// Lambda value read from LDS serves the three channels of its position; wt
// holds the weights as [co][ky][kx][3].  Each output's sum keeps the order of
// tap_sum64, and the epilogue takes the outputs in ascending j as before.
__device__ __forceinline__ void conv64_row_rgb(const Pass64& q, const Lay64& y, const ConvGeom& g,
                                               const RowInfo& ri, int row, const double* lam_s, const float* wt,
                                               double& cst, double& err, double& sq) {
  constexpr int P = 4, C = 3, kC = P * C;
  const int j0 = threadIdx.x;
  double a[kC];
#pragma unroll
  for (int u = 0; u < kC; ++u) a[u] = 0.0;
  // one position (a compile-time gi, so that a stays in registers)
  auto position = [&](auto gic) {
    constexpr int gi = decltype(gic)::value;
    const int pos = j0 + 256 * gi;
    const int iy = pos / g.wi, ix = pos - iy * g.wi;
    const int ry = (iy + g.p) % g.s, rx = (ix + g.p) % g.s;
    const int oy0 = (iy + g.p - ry) / g.s, ox0 = (ix + g.p - rx) / g.s;
    for (int ky = ry, oy = oy0; ky < g.k && oy >= 0; ky += g.s, --oy) {
      if (oy >= g.ho) continue;
      for (int kx = rx, ox = ox0; kx < g.k && ox >= 0; kx += g.s, --ox) {
        if (ox >= g.wo) continue;
        const float* wp = wt + (ky * g.k + kx) * C;
#pragma unroll 2
        for (int co = 0; co < g.co; ++co) {
          const double l = lam_s[(co * g.ho + oy) * g.wo + ox];
          const float* w = wp + co * g.k * g.k * C;
#pragma unroll
          for (int c = 0; c < C; ++c) a[gi + P * c] += l * (double)w[c];
        }
      }
    }
  };
  position(std::integral_constant<int, 0>{});
  position(std::integral_constant<int, 1>{});
  position(std::integral_constant<int, 2>{});
  position(std::integral_constant<int, 3>{});
  epi64<kC>(q, ri, y, row, j0, a, cst, err, sq);
}

// Back-substitution through conv layer i (transposed convolution): for input
// position (ci, iy, ix), A(i-1) = sum over (co, ky, kx) with oy = (iy + pad -
// ky) / stride and ox likewise whole and inside the output plane of
// Lambda(i)[co, oy, ox] W[co, ci, ky, kx], in double.
// The weights are staged in LDS after the row when they fit (w_lds: as
// stored, or in the position-blocked layout of conv64_row_pos when the plane
// size divides 256, or of conv64_row_rgb for a 3x32x32 input), else read
// from global memory; the same values and the same order of every sum in
// every case.
template <int w_lds>
__global__ __launch_bounds__(256) void conv64_k(Pass64 q, Lay64 y, ConvGeom g) {
  extern __shared__ double lam_s[];
  __shared__ double red[4];
  const int row = blockIdx.x;
  const RowInfo ri = row_info(q.bt, row);
  float* const w_s = reinterpret_cast<float*>(lam_s + ((y.K + 1) & ~1));
  for (int k0 = threadIdx.x; k0 < y.K; k0 += 256 * 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int k = k0 + 256 * u;
      v[u] = k < y.K ? y.in[(int64_t)row * y.ldi + k] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (k0 + 256 * u < y.K) lam_s[k0 + 256 * u] = v[u];
  }
  // w_lds: 1 the weights as stored, 2 the position-blocked layout of
  // conv64_row_pos with dci = 256 / (hi wi) and cip channels, 3 that layout
  // with cip = 3 for conv64_row_rgb, 0 global memory
  const int dci = w_lds == 2 ? 256 / (g.hi * g.wi) : 0, cip = w_lds == 3 ? 3 : g.ci + dci * kC64;
  if constexpr (w_lds == 1) {
    for (int t = threadIdx.x; t < g.co * g.ci * g.k * g.k; t += 256) w_s[t] = y.W[t];
  } else if constexpr (w_lds >= 2) {
    for (int t = threadIdx.x; t < g.co * g.k * g.k * cip; t += 256) {
      const int c = t % cip, r = t / cip, kx = r % g.k, r2 = r / g.k, ky = r2 % g.k, co = r2 / g.k;
      w_s[t] = c < g.ci ? y.W[((co * g.ci + c) * g.k + ky) * g.k + kx] : 0.f;
    }
  }
  __syncthreads();
  double cst = 0.0, err = 0.0, sq = 0.0;
  if constexpr (w_lds == 3) {
    conv64_row_rgb(q, y, g, ri, row, lam_s, w_s, cst, err, sq);
  } else if constexpr (w_lds == 2) {
    if (dci == 1) conv64_row_pos<kC64, 1>(q, y, g, ri, row, lam_s, w_s, cip, cst, err, sq);
    else if (dci == 2) conv64_row_pos<kC64, 2>(q, y, g, ri, row, lam_s, w_s, cip, cst, err, sq);
    else if (dci == 4) conv64_row_pos<kC64, 4>(q, y, g, ri, row, lam_s, w_s, cip, cst, err, sq);
    else conv64_row_pos<kC64, 8>(q, y, g, ri, row, lam_s, w_s, cip, cst, err, sq);
  } else if constexpr (w_lds == 1) {
    conv64_row<kC64>(q, y, g, ri, row, lam_s, w_s, cst, err, sq);
  } else {
    conv64_row<kC64>(q, y, g, ri, row, lam_s, y.W, cst, err, sq);
  }
  const double c = block_sum_d(cst, red), e = block_sum_d(err, red), s2 = block_sum_d(sq, red);
  if (threadIdx.x == 0) {
    q.part[(int64_t)y.slot * q.bt.n_rows + row] = c;
    q.perr[(int64_t)y.slot * q.bt.n_rows + row] = e;
    if (q.psq) q.psq[(int64_t)y.slot * q.bt.n_rows + row] = s2;
  }
}

// The weights of a conv layer in double, [ky][kx][co][cip] (input channel
// innermost, zero past ci), for conv64_rows_k.
__global__ void conv64_pack_k(const float* __restrict__ W, ConvGeom g, int cip, double* __restrict__ dst) {
  const int n = g.k * g.k * g.co * cip;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < n; t += gridDim.x * blockDim.x) {
    const int c = t % cip, r = t / cip, co = r % g.co, kk = r / g.co;
    dst[t] = c < g.ci ? (double)W[(int64_t)(co * g.ci + c) * g.k * g.k + kk] : 0.0;
  }
}

// Back-substitution through conv layer i for up to kR rows of one subdomain per
// workgroup, on large batches.  The input positions whose coordinates agree modulo the stride meet
// the same taps; a wave takes 64 positions of one such class and kC input
// channels, so that every weight it needs is the same for all of its lanes and
// comes from a scalar load, already in double, and each Lambda value read from
// LDS serves kC products.  (In the one-row kernels a product takes an LDS read
// and a conversion of its weight, and a wave whose lanes are neighbours in x
// walks the taps of all classes.)  The rows lie in LDS inside a zero border, so
// no tap needs a range check.  Eight waves share the rows'
// planes (62 KB at 8x16x16: two workgroups per compute unit); four waves with
// eight channels each run 2 per SIMD and take 159 us where these take 118.
// At 9216 rows: 8x8x8 back to 8x16x16 168 us in the one-row kernel, 127 here,
// 8x16x16 to itself 202 and 158, into 3x32x32 182 and 138; what is left is the
// memory traffic (63 us of a 16x16 layer) and the phases of a workgroup that
// two of them do not overlap.  Each output's sum keeps the order of tap_sum64.
template <int kC, int kR, int NW>
__global__ __launch_bounds__(64 * NW) void conv64_rows_k(Pass64 q, Lay64 y, ConvGeom g, Geo64 z,
                                                     const double* __restrict__ in, const double* __restrict__ wt) {
  extern __shared__ __attribute__((aligned(16))) double lam_s[];
  __shared__ double red[3 * kR * NW];
  const int tid = threadIdx.x, lane = tid & 63;
  int row0, nr;
  row_group<kR>(q.bt.m, &row0, &nr);
  const int rowlen = g.co * z.plane;  // (padded row of one batch row)
  for (int t0 = tid; t0 < rowlen; t0 += 64 * NW * 4) {
    double v[kR][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int t = min(t0 + 64 * NW * u, rowlen - 1);
      const int co = __umulhi(t, z.m_plane), rem = t - co * z.plane, yy = __umulhi(rem, z.m_pw);
      const int oy = yy - z.b0, ox = rem - yy * z.pw - z.b0;
      const bool in_p = (unsigned)oy < (unsigned)g.ho && (unsigned)ox < (unsigned)g.wo;
      const int k = in_p ? (co * g.ho + oy) * g.wo + ox : 0;
#pragma unroll
      for (int r = 0; r < kR; ++r) {
        const double x = in[(int64_t)(row0 + min(r, nr - 1)) * y.ldi + k];
        v[r][u] = in_p ? x : 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (t0 + 64 * NW * u < rowlen) {
#pragma unroll
        for (int r = 0; r < kR; ++r) lam_s[r * rowlen + t0 + 64 * NW * u] = v[r][u];
      }
  }
  __syncthreads();
  double cst[kR], err[kR], sq[kR];
#pragma unroll
  for (int r = 0; r < kR; ++r) cst[r] = err[r] = sq[r] = 0.0;

  // items (class, chunk of 64 positions, channel group), dealt round the waves
  const int groups = (g.ci + kC - 1) / kC;
  int item = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int ry = 0; ry < g.s; ++ry) {
    const int iy0 = (ry + g.s - g.p % g.s) % g.s, ny = (g.hi - iy0 + g.s - 1) / g.s;
    for (int rx = 0; rx < g.s; ++rx) {
      const int ix0 = (rx + g.s - g.p % g.s) % g.s, nx = (g.wi - ix0 + g.s - 1) / g.s;
      const int np = ny > 0 && nx > 0 ? ny * nx : 0, chunks = (np + 63) >> 6, n = chunks * groups;
      for (; item < n; item += NW) {
        const int chunk = item / groups, c0 = (item - chunk * groups) * kC;
        const int e = min(chunk * 64 + lane, np - 1), ay = e / nx, ax = e - ay * nx;
        const bool ok = chunk * 64 + lane < np;
        const int iy = iy0 + g.s * ay, ix = ix0 + g.s * ax;
        const int oy0 = (iy + g.p - ry) / g.s, ox0 = (ix + g.p - rx) / g.s;
        const double* lp = lam_s + (oy0 + z.b0) * z.pw + ox0 + z.b0;
        const int hw = g.hi * g.wi, j0 = c0 * hw + iy * g.wi + ix, nu = ok ? min(kC, g.ci - c0) : 0;
        Epi64<kC, kR> ep;
        ep.read(q, y, row0, nr, j0, hw, nu);
        double a[kR][kC];
#pragma unroll
        for (int r = 0; r < kR; ++r)
#pragma unroll
          for (int c = 0; c < kC; ++c) a[r][c] = 0.0;
        for (int ky = ry, ty = 0; ky < g.k; ky += g.s, ++ty)
          for (int kx = rx, tx = 0; kx < g.k; kx += g.s, ++tx) {
            const double* const wp = wt + (int64_t)(ky * g.k + kx) * g.co * z.cip + c0;
            const double* const l0 = lp - ty * z.pw - tx;
#pragma unroll 2
            for (int co = 0; co < g.co; ++co) {
              double w[kC];
#pragma unroll
              for (int c = 0; c < kC; ++c) w[c] = wp[co * z.cip + c];
#pragma unroll
              for (int r = 0; r < kR; ++r) {
                const double l = l0[r * rowlen + co * z.plane];
#pragma unroll
                for (int c = 0; c < kC; ++c) a[r][c] = fma(l, w[c], a[r][c]);
              }
            }
          }
        ep.apply(q, y, row0, nr, j0, hw, nu, a, cst, err, sq);
      }
      item -= n;  // the next class's items follow on
    }
  }
  block_out64<kR, NW>(q, y.slot, row0, nr, cst, err, sq, red);
}

// Rows of a group: three, which every load of a weight serves, or as many as
// leave no group partly empty where a subdomain has few.  A group computes all
// its rows: at 3,000 rows, one a subdomain, 784-100-100 took 75 us in the
// one-row kernel, 100 in groups of three and takes 72 in groups of one; with
// two 131, 102 and 86 (groups of two), with four 251, 184 and 156.
int group_rows(int m) { return m == 1 ? 1 : m == 2 || m == 4 ? 2 : 3; }

template <int kR>
void launch_dense64_rows(const Pass64& q, const Lay64& y, hipStream_t s) {
  const unsigned groups = (unsigned)(q.bt.n_rows / q.bt.m * ((q.bt.m + kR - 1) / kR));
  if (y.N > 256) launch_k(dense64_rows_k<kR, 8>, groups, 512, 0, s, q, y, y.in, y.W);
  else launch_k(dense64_rows_k<kR, 4>, groups, 256, 0, s, q, y, y.in, y.W);
}

// Channels per wave item of conv64_rows_k.
int conv64_channels(const ConvGeom& g) { return g.ci <= 3 ? 3 : 4; }

template <int kC, int kR, int NW>
void launch_conv64_rows(const Pass64& q, const Lay64& y, const ConvGeom& g, const Geo64& z, hipStream_t s) {
  launch_k(conv64_rows_k<kC, kR, NW>, (unsigned)(q.bt.n_rows / q.bt.m * ((q.bt.m + kR - 1) / kR)), 64 * NW,
           (uint32_t)((size_t)kR * g.co * z.plane * sizeof(double)), s, q, y, g, z, y.in, y.w64);
}

// Round a double down to a float (the largest float <= x).
__device__ __forceinline__ float down_f(double x) {
  float f = (float)x;
  if ((double)f > x) f = nextafterf(f, -INFINITY);
  return f;
}

// lb = (sum of the constants) - (margin), rounded down to float.  The margin
// is the sum of the rounding-error partials scaled by `scale` (their own
// summation), plus, over an l2 ball, eps ||A(0)||_2 (taken as an upper bound:
// the sum of squares and the square root inflated by `ball`, which also
// covers the float64 rounding of the A(0) x0 sum, bounded by ball ||A(0)||_2
// ||x0||_2), plus the rounding of the final subtraction.
__global__ __launch_bounds__(256) void finalize64_k(Pass64 q, Fin64 f) {
  const int row = blockIdx.x * 256 + threadIdx.x;
  if (row >= q.bt.n_rows) return;
  double tot = 0.0, err = 0.0, s2 = 0.0;
  for (int t = 0; t < f.n_used; ++t) {
    tot += q.part[(int64_t)t * q.bt.n_rows + row];
    err += q.perr[(int64_t)t * q.bt.n_rows + row];
    if (q.psq) s2 += q.psq[(int64_t)t * q.bt.n_rows + row];
  }
  double margin = err * f.scale;
  if (q.psq) {
    const int p = q.bt.prop[row / q.bt.m];
    const double nrm = sqrt(s2) * (1.0 + f.ball);
    tot -= (double)q.bt.l2eps[p] * nrm;
    margin += ((double)q.bt.l2eps[p] + (double)f.x0n[p]) * nrm * f.ball;
  }
  const double d = tot - margin;
  const float lbv = down_f(d - fabs(d) * 0x1p-52 - 0x1p-1000);
  if (f.lb) f.lb[row] = lbv;
  if (f.best) f.best[row] = f.first ? lbv : fmaxf(f.best[row], lbv);
}

}  // namespace

void launch_top64(const Pass64& q, const Top64& t, hipStream_t s) {
  if (q.bt.n_rows > 0) launch_k(top64_k, (unsigned)((q.bt.n_rows + 3) / 4), 256, 0, s, q, t);
}

void launch_dense64(const Pass64& q, const Lay64& y, hipStream_t s) {
  if (q.bt.n_rows <= 0) return;
  // (the chords are there from kRows64 rows on: checked, since the kernel reads them)
  if (q.chord && q.bt.n_rows >= kRows64) {
    const int kr = group_rows(q.bt.m);
    kr == 1 ? launch_dense64_rows<1>(q, y, s) : kr == 2 ? launch_dense64_rows<2>(q, y, s) : launch_dense64_rows<3>(q, y, s);
    return;
  }
  launch_k(dense64_k, (unsigned)q.bt.n_rows, 256, (uint32_t)(y.K * sizeof(double)), s, q, y);
}

void launch_chord64(const float* l, const float* u, double2* ch, int64_t n, hipStream_t s) {
  if (n > 0) launch_k(chord64_k, (unsigned)((n + 255) / 256), 256, 0, s, l, u, ch, n);
}

size_t conv64_pack_size(const ConvGeom& g) {
  const int kc = conv64_channels(g);
  return (size_t)g.k * g.k * g.co * ((g.ci + kc - 1) / kc * kc);
}

void launch_conv64_pack(const float* W, const ConvGeom& g, double* dst, hipStream_t s) {
  const int kc = conv64_channels(g);
  launch_k(conv64_pack_k, 32, 256, 0, s, W, g, (g.ci + kc - 1) / kc * kc, dst);
}

void launch_conv64(const Pass64& q, const Lay64& y, const ConvGeom& g, hipStream_t s) {
  if (q.bt.n_rows <= 0) return;
  // (below: too few workgroups, stride classes that fill less than a wave, or no
  // second row to share a read; a 3x32x32 network at 576 rows takes 142 us by
  // rows of one and 124 by threes, at 288 rows 107 and 108; 28x28 into 5 and 8
  // channels with one row a subdomain, 3,000 rows, 117 by the one-row kernels,
  // 134 by this one on single rows and 174 on groups of three)
  if (y.w64 && q.chord && q.bt.n_rows >= kRows64 && q.bt.m > 1 && g.ho > 1 && g.wo > 1 && g.hi * g.wi >= 64 * g.s * g.s) {
    // the taps reach b0 positions before the plane and b1 after it
    Geo64 z{};
    int lo = 0, hi_y = g.ho - 1, hi_x = g.wo - 1;
    for (int r = 0; r < g.s; ++r) {
      const int i0 = (r + g.s - g.p % g.s) % g.s, taps = r < g.k ? (g.k - r + g.s - 1) / g.s : 0;
      lo = std::min(lo, (i0 + g.p - r) / g.s - std::max(0, taps - 1));
      hi_y = std::max(hi_y, (g.hi - 1 + g.p - r) / g.s);
      hi_x = std::max(hi_x, (g.wi - 1 + g.p - r) / g.s);
    }
    z.b0 = -lo;
    z.pw = z.b0 + hi_x + 1;
    z.plane = z.pw * (z.b0 + hi_y + 1);
    const int kc = conv64_channels(g);
    z.cip = (g.ci + kc - 1) / kc * kc;
    z.m_plane = (uint32_t)(((1ull << 32) + z.plane - 1) / z.plane);
    z.m_pw = (uint32_t)(((1ull << 32) + z.pw - 1) / z.pw);
    const size_t row = (size_t)g.co * z.plane * sizeof(double);
    if (3 * row <= 64 * 1024) {
      const bool two = group_rows(q.bt.m) == 2;
      if (kc == 3) two ? launch_conv64_rows<3, 2, 8>(q, y, g, z, s) : launch_conv64_rows<3, 3, 8>(q, y, g, z, s);
      else two ? launch_conv64_rows<4, 2, 8>(q, y, g, z, s) : launch_conv64_rows<4, 3, 8>(q, y, g, z, s);
      return;
    }
  }
  const size_t row_b = (size_t)((y.K + 1) & ~1) * sizeof(double), w_b = (size_t)g.co * g.ci * g.k * g.k * sizeof(float);
  const int hw = g.hi * g.wi;
  const size_t wt_b = (size_t)g.co * g.k * g.k * (g.ci + (hw > 0 ? 256 / hw : 0) * kC64) * sizeof(float);
  int w_lds = 0;
  size_t lds = row_b;
  if (hw == 1024 && g.ci == 3 && y.N == 3 * 1024 && row_b + w_b <= 48 * 1024) {
    w_lds = 3;  // the [co][ky][kx][3] layout holds the same number of weights
    lds += w_b;
  } else if (hw >= 32 && 256 % hw == 0 && y.N == g.ci * hw && row_b + wt_b <= 48 * 1024) {
    w_lds = 2;
    lds += wt_b;
  } else if (row_b + w_b <= 48 * 1024) {
    w_lds = 1;
    lds += w_b;
  }
  const unsigned nb = (unsigned)q.bt.n_rows;
  if (w_lds == 3) launch_k(conv64_k<3>, nb, 256, (uint32_t)lds, s, q, y, g);
  else if (w_lds == 2) launch_k(conv64_k<2>, nb, 256, (uint32_t)lds, s, q, y, g);
  else if (w_lds == 1) launch_k(conv64_k<1>, nb, 256, (uint32_t)lds, s, q, y, g);
  else launch_k(conv64_k<0>, nb, 256, (uint32_t)lds, s, q, y, g);
}

void launch_finalize64(const Pass64& q, const Fin64& f, hipStream_t s) {
  if (q.bt.n_rows > 0) launch_k(finalize64_k, (unsigned)((q.bt.n_rows + 255) / 256), 256, 0, s, q, f);
}

}  // namespace cvb
