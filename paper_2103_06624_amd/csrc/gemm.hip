// Back-substitution and adjoint GEMMs for dense layers on FP32 MFMA (gfx950).
//
// Both directions are computed as C[M,N] = A[M,K] * Bt[N,K]^T with both
// operands K-contiguous:
//   back-substitution  A(i-1) = Lambda(i) W(i):  A = Lambda [rows, d_i],
//                      Bt = W(i)^T stored [d_{i-1}, d_i];
//   adjoint forward    zbar(i) = zhat(i-1) W(i)^T + b(i):  A = zhat,
//                      Bt = W(i) itself [d_i, d_{i-1}].
// The epilogue applies the next step of the method to the tile in registers:
// the ReLU relaxation of the next layer (Lemma 2.1 + beta S), the box
// concretisation (Eq. beta_crown_lp), or the adjoint's relaxed forward step
// with the alpha/beta gradients.
#include "common.h"
#include "internal.h"

typedef float floatx4 __attribute__((ext_vector_type(4)));

namespace cvb {

namespace {

// 4 consecutive elements [k, k+4) of row `row` of a K-contiguous matrix
// (leading dimension ld >= K rounded up to 4, 16-byte aligned rows).  The
// address is clamped into the matrix, so the load needs no per-lane branch;
// mask4 zeroes what lies outside [0, nrows) x [0, K).  The two are separate
// so that the mask (which needs the data) runs when the slab is parked in
// LDS, not right after the load is issued.
__device__ __forceinline__ float4 ld4(const float* __restrict__ P, int ld, int row, int nrows, int k, int K) {
  const int K4 = (K + 3) & ~3;
  return *reinterpret_cast<const float4*>(P + (int64_t)min(row, nrows - 1) * ld + min(k, K4 - 4));
}

__device__ __forceinline__ float4 mask4(float4 x, int row, int nrows, int k, int K) {
  const bool rok = row < nrows;
  x.x = rok && k < K ? x.x : 0.f;
  x.y = rok && k + 1 < K ? x.y : 0.f;
  x.z = rok && k + 2 < K ? x.z : 0.f;
  x.w = rok && k + 3 < K ? x.w : 0.f;
  return x;
}

// Four consecutive 32-bit values at p (4-byte aligned), in one load.  The
// arrays it reads have room for a quad past their last entry (kSlack).
template <class T>
__device__ __forceinline__ void ld_quad(const T* __restrict__ p, T (&x)[4]) {
  static_assert(sizeof(T) == 4, "32-bit values");
  typedef uint32_t quad __attribute__((ext_vector_type(4), aligned(4)));
  const quad v = *reinterpret_cast<const quad*>(p);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const uint32_t w = v[r];
    x[r] = __builtin_bit_cast(T, w);
  }
}

// Epilogue operands of one tile, gathered before its K loop so that they land
// while the MFMAs run.  In the backward modes (TR) the MFMAs compute each 16x16
// block transposed (operands swapped: the same products, summed in the same
// order), so element (i, j, r) of a lane is row m0 + wm*WM + 16i + lane%16,
// column n0 + wn*WN + 16j + 4(lane/16) + r: a lane has one row per i and four
// neighbouring columns per j, whose status words, chords, bias and results move
// as 16-byte pieces, and one row's indices instead of four.  The epilogue's loads
// and index arithmetic, not the MFMAs, take most of these launches.  Untransposed,
// transposed, and transposed with the gathers free of branches, us with 32x32x32
// tiles:
//   100 -> 1024 relaxation at 18432 rows         97.5   89.3   81.0
//   100 -> 2048 relaxation at 9216 rows          99.7   91.2   83.2
//   200 -> 784 concretisation at 9216 rows       46.2   43.2   44.5
// The adjoint keeps row 4(lane/16) + r, column lane%16: most of its traffic is
// the packed alpha, its moments and the stored A, whose entries lie side by side
// along a row and coalesce over the 16 lanes of one (transposed, 20 iterations of
// 784-6x200-10 at 9216 rows take 6.31 ms instead of 6.02).
template <int BM, int BN, bool TR>
struct TileOps {
  static constexpr int FM = BM / 32, FN = BN / 32, NE = FM * FN * 4;
  RowInfo eri[FM][TR ? 1 : 4];
  uint32_t rec[NE];
  float2 ech[NE];
  float ecf[NE];   // alpha of an unstable neuron (relaxation: or beta of a split one)
  float ebias[FN][TR ? 4 : 1];
  float esw[NE];   // relaxation, sound mode: the neuron's rounding-error weight
  float east[NE];  // adjoint: the stored A of an unstable neuron
  float2 emo[NE];  // adjoint with Adam: the moments of an unstable neuron's alpha
  float ebe[NE];   // kFwdTop: C_p W(L)
};

// OCC > 0 asks the compiler for at least OCC waves per SIMD (registers capped
// accordingly): with OCC = 8 a 32x32 tiling of ~10^4 x 200 is resident in one
// round instead of two.  DEPTH = 2 keeps two slabs of global loads in flight
// (two register sets, loads issued two slabs before they are parked in LDS):
// a slab's MFMA work is far shorter than the load latency at these sizes.
// DEPTH >= 3 holds all of K in registers (K <= DEPTH * BK): one load latency
// per tile instead of one per slab.
// Modes: kBwdRelax, kBwdConc, kFwd (the adjoint's first layer reads x* as a
// dense operand), kFwdTop (kFwd plus the next top-layer relaxation).
template <int BM, int BN, int BK, int MODE, int OCC, int DEPTH>
__global__ __launch_bounds__(256, OCC) void gemm_nt(const float* __restrict__ A, int lda, const float* __restrict__ Bt,
                                               int ldb, int M, int N, int K, int last, Batch bt, Vars v, Epi e) {
  constexpr int LDK = BK + 4;  // padded LDS row: LDK/4 odd, conflict-free b128 reads
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int FM = WM / 16, FN = WN / 16;
  constexpr int QK = BK / 4;  // float4 per row of a slab
  constexpr int A_LD = (BM * QK + 255) / 256;  // float4 loads per thread
  constexpr int B_LD = (BN * QK + 255) / 256;
  constexpr bool TR = MODE == kBwdRelax || MODE == kBwdConc;  // lane layout: see TileOps
  using Ops = TileOps<BM, BN, TR>;
  __shared__ __attribute__((aligned(16))) float As[2][BM][LDK];
  __shared__ __attribute__((aligned(16))) float Bs[2][BN][LDK];
  __shared__ float red[2][BM];
  __shared__ float rede[2][BM];  // sound mode: the rounding-error partials

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wid = tid >> 6;
  const int wm = wid >> 1, wn = wid & 1;
  const int rsub = 4 * (lane >> 4);
  const int csub = lane & 15;

  // XCD-aware order: consecutive logical tiles (the column tiles of one row
  // tile) land on the same XCD, so they share its L2 copy of the row tile.
  const int tiles_n = (N + BN - 1) / BN;
  const int nblk = gridDim.x;
  int logical = blockIdx.x;
  if ((nblk & 7) == 0) logical = (blockIdx.x & 7) * (nblk >> 3) + (blockIdx.x >> 3);
  const int tm = logical / tiles_n, tn = logical - tm * tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;

  struct Regs {
    float4 a[A_LD], b[B_LD];
  };
  auto gload = [&](Regs& r, int k0) {
#pragma unroll
    for (int t = 0; t < A_LD; ++t) {
      const int idx = min(tid + t * 256, BM * QK - 1);
      r.a[t] = ld4(A, lda, m0 + idx / QK, M, k0 + (idx % QK) * 4, K);
    }
#pragma unroll
    for (int t = 0; t < B_LD; ++t) {
      const int idx = min(tid + t * 256, BN * QK - 1);
      r.b[t] = ld4(Bt, ldb, n0 + idx / QK, N, k0 + (idx % QK) * 4, K);
    }
  };
  // threads past the slab repeat its last float4 (same value, same address)
  auto sstore = [&](const Regs& r, int buf, int k0) {
#pragma unroll
    for (int t = 0; t < A_LD; ++t) {
      const int idx = min(tid + t * 256, BM * QK - 1);
      *reinterpret_cast<float4*>(&As[buf][idx / QK][(idx % QK) * 4]) =
          mask4(r.a[t], m0 + idx / QK, M, k0 + (idx % QK) * 4, K);
    }
#pragma unroll
    for (int t = 0; t < B_LD; ++t) {
      const int idx = min(tid + t * 256, BN * QK - 1);
      *reinterpret_cast<float4*>(&Bs[buf][idx / QK][(idx % QK) * 4]) =
          mask4(r.b[t], n0 + idx / QK, N, k0 + (idx % QK) * 4, K);
    }
  };
  auto compute = [&](floatx4 (&acc)[FM][FN], int buf) {
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      float4 fa[FM], fb[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i)
        fa[i] = *reinterpret_cast<const float4*>(&As[buf][wm * WM + i * 16 + (lane & 15)][ks + 4 * (lane >> 4)]);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        fb[j] = *reinterpret_cast<const float4*>(&Bs[buf][wn * WN + j * 16 + (lane & 15)][ks + 4 * (lane >> 4)]);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const float fx[4] = {fa[i].x, fa[i].y, fa[i].z, fa[i].w}, fy[4] = {fb[j].x, fb[j].y, fb[j].z, fb[j].w};
#pragma unroll
          for (int t = 0; t < 4; ++t)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(TR ? fy[t] : fx[t], TR ? fx[t] : fy[t], acc[i][j], 0, 0, 0);
        }
    }
  };

  auto row_of = [&](int i, int r) { return m0 + wm * WM + i * 16 + (TR ? csub : rsub + r); };
  auto col_of = [&](int j, int r) { return n0 + wn * WN + j * 16 + (TR ? rsub + r : csub); };
  auto elem = [&](int i, int j, int r) { return (i * FN + j) * 4 + r; };
  // (TR) columns of quad j that exist in row i of the lane
  auto count = [&](int i, int j) { return row_of(i, 0) < M ? min(max(N - col_of(j, 0), 0), 4) : 0; };
  // the column to read for column (j, r): itself, or inside the matrix
  auto col_in = [&](int j, int r) { return min(col_of(j, r), TR ? (N - 1) & ~3 : N - 1); };
  // what a lane reads in place of a variable that its neuron does not have
  const float* const none = reinterpret_cast<const float*>(bt.rbase);

  // The gathers of the backward modes have no branch: a load under one makes
  // every later wait count as if it had not been issued, so that waiting for
  // the first slab would wait for the gathers of the whole tile.  Lanes without
  // a column or a variable read some valid address.  (The adjoint's variables
  // stay under one: five unconditional loads per entry cost it registers, 114
  // against 92 and a wave per SIMD, 25.2 us against 22.5 at 200x200.)
  // First level: bias, row info and status records.
  auto gather1 = [&](Ops& o) {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if constexpr (TR) {
        if (MODE != kBwdConc) ld_quad(e.bias + col_in(j, 0), o.ebias[j]);
      } else {
        o.ebias[j][0] = e.bias[col_in(j, 0)];
      }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
#pragma unroll
      for (int r = 0; r < (TR ? 1 : 4); ++r) o.eri[i][r] = row_info(bt, min(row_of(i, r), M - 1));
      if constexpr (MODE != kBwdConc) {
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          if constexpr (TR) {
            uint32_t w[4];
            ld_quad(bt.status + (int64_t)o.eri[i][0].b * bt.nd + e.layer_off + col_in(j, 0), w);
#pragma unroll
            for (int r = 0; r < 4; ++r) o.rec[elem(i, j, r)] = w[r];
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
              o.rec[elem(i, j, r)] = bt.status[(int64_t)o.eri[i][r].b * bt.nd + e.layer_off + col_in(j, r)];
          }
        }
      }
    }
  };
  // Second level, which needs the status records: chord and alpha / beta, the
  // stored A for the adjoint, or the box for concretisation.
  auto gather2 = [&](Ops& o) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const int q0 = elem(i, j, 0);
        if constexpr (MODE == kBwdConc) {
          const int64_t pb = (int64_t)o.eri[i][0].p * bt.d0 + col_in(j, 0);
          float lo[4], hi[4];
          ld_quad((bt.l2x0 ? bt.l2x0 : bt.xlo) + pb, lo);
          ld_quad((bt.l2x0 ? bt.l2x0 : bt.xhi) + pb, hi);
#pragma unroll
          for (int r = 0; r < 4; ++r) o.ech[q0 + r] = make_float2(lo[r], hi[r]);
        } else if constexpr (TR) {
          const RowInfo& ri = o.eri[i][0];
          const int64_t pc0 = (int64_t)ri.p * bt.nd + e.layer_off + col_in(j, 0);
          const float* const cp = reinterpret_cast<const float*>(bt.chord + pc0);  // (zero at stable neurons)
          float c[2][4];
          ld_quad(cp, c[0]);
          ld_quad(cp + 4, c[1]);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            o.ech[q0 + r] = make_float2(c[r >> 1][2 * (r & 1)], c[r >> 1][2 * (r & 1) + 1]);
            if (r >= count(i, j)) o.rec[q0 + r] = kInactive;
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const uint32_t rec = o.rec[q0 + r], kind = rec & kKindMask;
            const float* v1 = v.alpha ? v.alpha + (ri.abase + (rec & kCidxMask)) : bt.adef + (pc0 + r);
            v1 = kind == kUnstable ? v1 : none;
            v1 = kind == kSplit ? v.beta + ((int64_t)(rec & kSplitMask) * bt.m + ri.k) : v1;
            o.ecf[q0 + r] = *v1;
          }
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int row = row_of(i, r), col = col_of(j, r), q = q0 + r;
            const RowInfo& ri = o.eri[i][r];
            o.ech[q] = o.emo[q] = make_float2(0.f, 0.f);
            o.east[q] = o.ecf[q] = 0.f;
            if (row >= M || col >= N) {
              o.rec[q] = kInactive;
              continue;
            }
            const int64_t pc = (int64_t)ri.p * bt.nd + e.layer_off + col;
            const bool uns = (o.rec[q] & kKindMask) == kUnstable;
            if (uns) o.ech[q] = bt.chord[pc];
            if (uns && !v.sat) {
              const int64_t ai = ri.abase + (o.rec[q] & kCidxMask);
              o.east[q] = v.acomp[ai];
              o.ecf[q] = v.alpha ? v.alpha[ai] : bt.adef[pc];
              if (v.adam) o.emo[q] = make_float2(v.ma[ai], v.va[ai]);
            }
            // the fused top layer: ebe holds C_p W(L) at this neuron
            if (MODE == kFwdTop) o.ebe[q] = e.cw[ri.p * e.cw_pstride + (int64_t)ri.k * e.ldcw + col_in(j, r)];
          }
        }
      }
    // (sound mode's float32 pass)
    if constexpr (MODE == kBwdRelax) {
#pragma unroll
      for (int q = 0; q < Ops::NE; ++q) o.esw[q] = 0.f;
      if (bt.sw) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            float w[4];
            ld_quad(bt.sw + (int64_t)o.eri[i][0].p * bt.nd + e.layer_off + col_in(j, 0), w);
#pragma unroll
            for (int r = 0; r < 4; ++r) o.esw[elem(i, j, r)] = w[r];
          }
      }
    }
  };
  // sum over the four lanes that share a row (lane % 16)
  auto row_sum = [&](float x) {
    x += __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
  };

  // epilogue
  auto epilogue = [&](const Ops& o, floatx4 (&acc)[FM][FN]) {
    if constexpr (TR) {
      // second per-row sum: the rounding-error bound (sound mode) or, when
      // concretising over an l2 ball, the sum of A(0)^2; with both modes on,
      // the other array's slot gets 0 (the l2 concretisation's own rounding is
      // bounded at the final sum)
      float* const p2 = MODE == kBwdConc && bt.l2x0 ? e.psq : (e.perr ? e.perr : e.psq);
      float* const pz = e.perr && e.psq ? (p2 == e.perr ? e.psq : e.perr) : nullptr;
#pragma unroll
      for (int i = 0; i < FM; ++i) {
        float cst = 0.f, cer = 0.f;
        const int row = row_of(i, 0);
        const RowInfo& ri = o.eri[i][0];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const int nv = count(i, j);
          float x[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int q = elem(i, j, r);
            const float a = acc[i][j][r];
            if (r >= nv) continue;
            if (MODE == kBwdRelax) {
              if (v.acomp && (o.rec[q] & kKindMask) == kUnstable) v.acomp[ri.abase + (o.rec[q] & kCidxMask)] = a;
              x[r] = relax_value(bt, v, ri, o.rec[q], o.ech[q], o.ecf[q], a, o.ebias[j][r], &cst);
              cer = fmaf(fabsf(x[r]), o.esw[q], cer);
            } else if (bt.l2x0) {  // l_p ball: A(0) x0 here, - eps ||A(0)||_q in the final sum
              cst = fmaf(a, o.ech[q].x, cst);
              x[r] = lp_entry(a, bt.lpq, &cer);  // x*'s direction for the adjoint
            } else {
              const float tm = conc_term(a, o.ech[q].x, o.ech[q].y);
              cst += tm;
              cer = fmaf(bt.sg, fabsf(tm), cer);
              x[r] = xstar(a > 0.f, a < 0.f, o.ech[q].x, o.ech[q].y);
            }
          }
          // (rows are padded to whole quads)
          float* const dst = MODE == kBwdRelax ? e.out + (int64_t)row * e.ldo : v.xdense ? v.xdense + (int64_t)row * v.ldx : nullptr;
          if (dst && nv > 0) *reinterpret_cast<float4*>(dst + col_of(j, 0)) = make_float4(x[0], x[1], x[2], x[3]);
        }
        cst = row_sum(cst);
        if (p2) cer = row_sum(cer);
        if (rsub == 0) {
          red[wn][wm * WM + i * 16 + csub] = cst;
          if (p2) rede[wn][wm * WM + i * 16 + csub] = cer;
        }
      }
      // combine the two column halves (wn = 0, 1) of each row, one slot per tile
      __syncthreads();
      for (int t = tid; t < BM; t += 256) {
        const int row = m0 + t;
        if (row < M) {
          e.part[(int64_t)(e.slot0 + tn) * M + row] = red[0][t] + red[1][t];
          if (p2) p2[(int64_t)(e.slot0 + tn) * M + row] = rede[0][t] + rede[1][t];
          if (pz) pz[(int64_t)(e.slot0 + tn) * M + row] = 0.f;
        }
      }
    } else if constexpr (MODE == kFwdTop) {
      // last adjoint layer inside the optimiser: Adam step, then the next
      // iteration's top-layer relaxation with the new variables
      float cst[FM][4];
#pragma unroll
      for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          cst[i][r] = 0.f;
          const int row = row_of(i, r);
          const bool rok = row < M;
          const RowInfo& ri = o.eri[i][r];
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const int col = col_of(j, r);
            const int q = elem(i, j, r);
            if (rok && col < N) {
              const float zb = e.wx0 ? fmaf(-v.l2s[row], acc[i][j][r], e.wx0[(int64_t)ri.p * N + col])
                                     : acc[i][j][r] + o.ebias[j][0];
              const int64_t pc = (int64_t)ri.p * bt.nd + e.layer_off + col;
              float vn = 0.f;
              relax_fwd_value(bt, v, ri, o.rec[q], o.ech[q], o.east[q], o.ecf[q], pc, zb, true, o.emo[q], &vn);
              const float a = o.ebe[q];
              if (v.acomp && (o.rec[q] & kKindMask) == kUnstable) v.acomp[ri.abase + (o.rec[q] & kCidxMask)] = a;
              e.top_out[(int64_t)row * e.ldo + col] = relax_value(bt, v, ri, o.rec[q], o.ech[q], vn, a, o.ebias[j][0],
                                                                  &cst[i][r]);
            }
          }
          cst[i][r] = wave_sum16(cst[i][r]);
        }
      }
      if (csub == 0) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) red[wn][wm * WM + i * 16 + rsub + r] = cst[i][r];
      }
      __syncthreads();
      for (int t = tid; t < BM; t += 256) {
        const int row = m0 + t;
        if (row < M) {
          float c = red[0][t] + red[1][t];
          if (tn == 0) {
            const RowInfo ri = row_info(bt, row);
            c += e.cb[ri.p * e.cb_pstride + ri.k];
          }
          e.part[(int64_t)(e.slot0 + tn) * M + row] = c;
          if (e.psq) e.psq[(int64_t)(e.slot0 + tn) * M + row] = 0.f;  // l2 ball: no A(0) terms here
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < FM; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = row_of(i, r);
          if (row >= M) continue;
          const RowInfo& ri = o.eri[i][r];
#pragma unroll
          for (int j = 0; j < FN; ++j) {
            const int col = col_of(j, r);
            if (col >= N) continue;
            const int q = elem(i, j, r);
            // l2 ball, first layer: W(1) x* + b(1) = (W(1) x0 + b(1)) - l2s (W(1) A(0))
            const float zb = e.wx0 ? fmaf(-v.l2s[row], acc[i][j][r], e.wx0[(int64_t)ri.p * N + col])
                                   : acc[i][j][r] + o.ebias[j][0];
            if (v.sat) {  // the network itself at x*: every layer's output is kept
              e.out[(int64_t)row * e.ldo + col] = true_relu(o.rec[q], zb, v.sat + row);
              continue;
            }
            const int64_t pc = (int64_t)ri.p * bt.nd + e.layer_off + col;
            const float zh = relax_fwd_value(bt, v, ri, o.rec[q], o.ech[q], o.east[q], o.ecf[q], pc, zb, true, o.emo[q]);
            if (!last) e.out[(int64_t)row * e.ldo + col] = zh;
          }
        }
      }
    }
  };

  const int nk = (K + BK - 1) / BK;
  constexpr int NF = DEPTH >= 3 ? DEPTH : 1;
  Ops ops;
  Regs r0, r1, rf[NF];
  floatx4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  gather1(ops);
  if (DEPTH >= 3) {
#pragma unroll
    for (int d = 0; d < NF; ++d) gload(rf[d], min(d, nk - 1) * BK);
  } else {
    gload(r0, 0);
    if (DEPTH == 2) gload(r1, min(1, nk - 1) * BK);
  }
  gather2(ops);
  if (DEPTH >= 3) {
    // slab d sits in LDS buffer d & 1; slab d + 1 waits in rf[d + 1]
    sstore(rf[0], 0, 0);
    __syncthreads();
#pragma unroll
    for (int d = 0; d < NF; ++d) {
      if (d >= nk) break;
      compute(acc, d & 1);
      if (d + 1 < NF && d + 1 < nk) sstore(rf[d + 1 < NF ? d + 1 : 0], (d + 1) & 1, (d + 1) * BK);
      __syncthreads();
    }
  } else if (DEPTH == 1) {
    sstore(r0, 0, 0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
      const int buf = kt & 1;
      if (kt + 1 < nk) gload(r0, (kt + 1) * BK);
      compute(acc, buf);
      if (kt + 1 < nk) sstore(r0, buf ^ 1, (kt + 1) * BK);
      __syncthreads();
    }
  } else {
    // entering a pair of slabs kt, kt+1: slab kt in LDS buffer 0, slab kt+1
    // in flight in r1.  Loads and stores are unconditional (slab index
    // clamped: past the end they repeat the last slab into a buffer nobody
    // reads again), so every load is consumed on every path and no load is
    // left pending where its registers are reused.
    sstore(r0, 0, 0);
    __syncthreads();
    for (int kt = 0; kt < nk; kt += 2) {
      const int k2 = min(kt + 2, nk - 1) * BK, k3 = min(kt + 3, nk - 1) * BK;
      gload(r0, k2);
      compute(acc, 0);
      sstore(r1, 1, min(kt + 1, nk - 1) * BK);
      __syncthreads();
      if (kt + 1 >= nk) break;
      gload(r1, k3);
      compute(acc, 1);
      sstore(r0, 0, k2);
      __syncthreads();
    }
  }
  epilogue(ops, acc);
}

template <int BM, int BN, int BK, int OCC, int DEPTH>
void launch_cfg(int mode, const GemmArgs& g, hipStream_t s) {
  const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  dim3 grid(tiles), block(256);
  switch (mode) {
    case kBwdRelax:
      launch_k(gemm_nt<BM, BN, BK, kBwdRelax, OCC, DEPTH>, grid, block, 0, s, g.A, g.lda, g.Bt, g.ldb, g.M, g.N, g.K,
               g.last, g.bt, g.v, g.e);
      break;
    case kBwdConc:
      launch_k(gemm_nt<BM, BN, BK, kBwdConc, OCC, DEPTH>, grid, block, 0, s, g.A, g.lda, g.Bt, g.ldb, g.M, g.N, g.K,
               g.last, g.bt, g.v, g.e);
      break;
    case kFwdTop:
      launch_k(gemm_nt<BM, BN, BK, kFwdTop, OCC, DEPTH>, grid, block, 0, s, g.A, g.lda, g.Bt, g.ldb, g.M, g.N, g.K,
               g.last, g.bt, g.v, g.e);
      break;
    default:
      launch_k(gemm_nt<BM, BN, BK, kFwd, OCC, DEPTH>, grid, block, 0, s, g.A, g.lda, g.Bt, g.ldb, g.M, g.N, g.K,
               g.last, g.bt, g.v, g.e);
      break;
  }
}

}  // namespace

const GemmCfg kGemmCfgs[kNumGemmCfgs] = {
    {64, 64, 16, 0, 1}, {64, 32, 16, 0, 1}, {32, 64, 16, 0, 1}, {128, 64, 16, 0, 1}, {128, 32, 16, 0, 1},
    {32, 32, 16, 0, 1}, {32, 32, 32, 0, 1}, {32, 32, 64, 0, 1}, {64, 32, 32, 0, 1},  {32, 64, 32, 0, 1},
    {64, 64, 32, 0, 1}, {64, 32, 64, 0, 1}, {32, 64, 64, 0, 1}, {32, 32, 16, 8, 1},  {32, 32, 32, 8, 1},
    {64, 32, 16, 6, 1}, {32, 64, 16, 6, 1}, {32, 32, 16, 8, 2}, {32, 32, 32, 8, 2},  {32, 32, 32, 0, 2},
    {64, 32, 32, 0, 2}, {32, 64, 32, 0, 2}, {64, 64, 32, 0, 2}, {64, 32, 16, 6, 2},  {32, 64, 16, 6, 2},
    {32, 32, 64, 0, 2}, {64, 32, 64, 0, 2}, {32, 64, 64, 0, 2}, {64, 64, 16, 0, 2}, {64, 32, 32, 0, 8},
    {32, 32, 32, 0, 8}, {32, 64, 32, 0, 8}, {64, 64, 32, 0, 8}, {64, 32, 64, 0, 4}, {32, 32, 64, 0, 4},
    {32, 64, 64, 0, 4}, {64, 32, 32, 4, 2}, {32, 64, 32, 4, 2}, {64, 32, 16, 4, 2}, {64, 32, 32, 4, 1}};

bool gemm_cfg_fits(int cfg, int K) {
  const GemmCfg& c = kGemmCfgs[cfg];
  return c.depth <= 2 || (K + c.bk - 1) / c.bk <= c.depth;
}

void launch_gemm(int cfg, int mode, const GemmArgs& g, hipStream_t s) {
  if (!gemm_cfg_fits(cfg, g.K)) cfg = 19;  // K too deep for an all-of-K tiling
  switch (cfg) {
    case 0: launch_cfg<64, 64, 16, 0, 1>(mode, g, s); break;
    case 1: launch_cfg<64, 32, 16, 0, 1>(mode, g, s); break;
    case 2: launch_cfg<32, 64, 16, 0, 1>(mode, g, s); break;
    case 3: launch_cfg<128, 64, 16, 0, 1>(mode, g, s); break;
    case 4: launch_cfg<128, 32, 16, 0, 1>(mode, g, s); break;
    case 5: launch_cfg<32, 32, 16, 0, 1>(mode, g, s); break;
    case 6: launch_cfg<32, 32, 32, 0, 1>(mode, g, s); break;
    case 7: launch_cfg<32, 32, 64, 0, 1>(mode, g, s); break;
    case 8: launch_cfg<64, 32, 32, 0, 1>(mode, g, s); break;
    case 9: launch_cfg<32, 64, 32, 0, 1>(mode, g, s); break;
    case 10: launch_cfg<64, 64, 32, 0, 1>(mode, g, s); break;
    case 11: launch_cfg<64, 32, 64, 0, 1>(mode, g, s); break;
    case 12: launch_cfg<32, 64, 64, 0, 1>(mode, g, s); break;
    case 13: launch_cfg<32, 32, 16, 8, 1>(mode, g, s); break;
    case 14: launch_cfg<32, 32, 32, 8, 1>(mode, g, s); break;
    case 15: launch_cfg<64, 32, 16, 6, 1>(mode, g, s); break;
    case 16: launch_cfg<32, 64, 16, 6, 1>(mode, g, s); break;
    case 17: launch_cfg<32, 32, 16, 8, 2>(mode, g, s); break;
    case 18: launch_cfg<32, 32, 32, 8, 2>(mode, g, s); break;
    case 19: launch_cfg<32, 32, 32, 0, 2>(mode, g, s); break;
    case 20: launch_cfg<64, 32, 32, 0, 2>(mode, g, s); break;
    case 21: launch_cfg<32, 64, 32, 0, 2>(mode, g, s); break;
    case 22: launch_cfg<64, 64, 32, 0, 2>(mode, g, s); break;
    case 23: launch_cfg<64, 32, 16, 6, 2>(mode, g, s); break;
    case 24: launch_cfg<32, 64, 16, 6, 2>(mode, g, s); break;
    case 25: launch_cfg<32, 32, 64, 0, 2>(mode, g, s); break;
    case 26: launch_cfg<64, 32, 64, 0, 2>(mode, g, s); break;
    case 27: launch_cfg<32, 64, 64, 0, 2>(mode, g, s); break;
    case 28: launch_cfg<64, 64, 16, 0, 2>(mode, g, s); break;
    case 29: launch_cfg<64, 32, 32, 0, 8>(mode, g, s); break;
    case 30: launch_cfg<32, 32, 32, 0, 8>(mode, g, s); break;
    case 31: launch_cfg<32, 64, 32, 0, 8>(mode, g, s); break;
    case 32: launch_cfg<64, 64, 32, 0, 8>(mode, g, s); break;
    case 33: launch_cfg<64, 32, 64, 0, 4>(mode, g, s); break;
    case 34: launch_cfg<32, 32, 64, 0, 4>(mode, g, s); break;
    case 35: launch_cfg<32, 64, 64, 0, 4>(mode, g, s); break;
    case 36: launch_cfg<64, 32, 32, 4, 2>(mode, g, s); break;
    case 37: launch_cfg<32, 64, 32, 4, 2>(mode, g, s); break;
    case 38: launch_cfg<64, 32, 16, 4, 2>(mode, g, s); break;
    default: launch_cfg<64, 32, 32, 4, 1>(mode, g, s); break;
  }
}

}  // namespace cvb
