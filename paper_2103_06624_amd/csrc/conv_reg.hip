// Conv layers with the epilogue on the matrix cores' own tile (gfx950, FP32
// MFMA 16x16x4): back-substitution (transposed convolution), concretisation
// and the adjoint's forward convolution, one batch row at a time.
//
// The same implicit GEMM D[m, n] = sum_k G[m, k] Wm[k, n] as conv.hip (its row
// and column axes are described there), in the same order of every sum over
// k.  What differs is where a result lives.  A wave owns fixed 16x16 tiles of
// D (TM of m by NTW of n) for every row of a subdomain and computes them
// transposed, so a lane holds one GEMM row m and, per column tile t, the four
// columns 4 (lane / 16) + r.  The columns are ordered (ConvReg) so that these
// are the output neurons base(lane) + plane (r + ts t): one position of the
// output plane, channels a plane apart.  The layer's epilogue (relaxation,
// concretisation, adjoint step) then runs on the accumulators, with the
// relaxation of the lane's neurons in registers for all rows of a subdomain,
// and neither an LDS copy of the output row nor a barrier stands between the
// GEMM and its epilogue.  The only barrier of a row hands over the staged
// input (two with a single input buffer).
//
// What bounds these kernels: a row's MFMAs (192 for 8 -> 8 channels k3 s1 on a
// 16x16 plane, 184 us of the 73,728 rows' 407), then instruction issue between
// a row's GEMMs (693 VALU and 240 LDS instructions per row there, where
// the subdomain-major kernel of conv.hip, which scatters the tile through LDS
// and walks the row in natural order between two barriers, issues 1,490 and
// 450) and the registers, which hold the relaxation of a lane's neurons: a
// kernel that spills loses to the older one.  Small workgroups (2 to 8 waves)
// leave several rows in flight on a CU.  Measured, us per launch, older kernel
// against this one:
//   8 -> 8 k3 s1 back-substitution, 73,728 rows          475   407
//   into a 3x32x32 input from 8 channels, 73,728 rows    483   404
//   into a 3x32x32 input from 16 channels, 9,216 rows    129    87
//   32 -> 16 k4 s2 back-substitution, 9,216 rows         307   259
//   adjoint 8 -> 8 k4 s2, 73,728 rows                    443   367
//   the same with Adam                                   461   380
//   adjoint 16 -> 32 k4 s2, 9,216 rows                   257   170
//   adjoint from x*, 3 -> 16, 9,216 rows                 191   137
//   adjoint from x*, 3 -> 8, 73,728 rows                 693   653
//   the same with Adam                                   734   718
//   adjoint 8 -> 8 k3 s1, 73,728 rows                    567   573
//   the same with Adam                                   658   744
//   8 -> 8 k4 s2 back-substitution, 73,728 rows          376   614
// (where the older kernel is the better one it is the default: conv_plan_reg).
//
// Lanes without a neuron (GEMM rows outside a polyphase class, padding
// columns) are not branched round: their buffer offsets lie past the row, so
// loads return 0 (an inactive neuron, an empty box) and stores are dropped.
#include <algorithm>

#include "common.h"
#include "internal.h"

namespace cvb {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef const uint64_t __attribute__((address_space(4)))* cword_ptr;

// s_waitcnt immediate for vmcnt(0) with the other counters left free (gfx9)
constexpr int kWaitVm0 = 0x0F70;
// waves of a workgroup at most (16 leave 128 registers)
constexpr int reg_max_waves(int mode, int ntw, int tm) { return mode == kBwdConc && ntw * tm <= 2 ? 16 : 8; }
constexpr int kRegIn = 2;       // float4s of the next row's input a thread reads ahead
constexpr int kRegWords = 8;    // sign words of the next row's x* a wave reads ahead
constexpr uint32_t kNoVar = 0x80000000u;  // no variable: past the end of every buffer
constexpr int kRsrcFlags = 0x00020000;    // raw 32-bit buffer, gfx9

// A bounds-checked view of n bytes at p: loads past the end return 0, stores
// past it are dropped.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t view(const void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, kRsrcFlags);
}
__device__ __forceinline__ uint32_t ldu(rsrc_t r, uint32_t byte) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, byte, 0, 0);
}
__device__ __forceinline__ float ldf(rsrc_t r, uint32_t byte) { return __uint_as_float(ldu(r, byte)); }
__device__ __forceinline__ void stf(float x, rsrc_t r, uint32_t byte) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, byte, 0, 0);
}

__device__ __forceinline__ float comp(const float4& v, int q) { return q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w; }

// d = bit `lane` of mask ? b : a (mask uniform across the wave)
__device__ __forceinline__ float pick_bit(float a, float b, uint64_t mask) {
  float d;
  asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(mask));
  return d;
}

// a b, and 0 where a or b is 0, also with the other one infinite or NaN: one
// instruction (the intrinsic rather than asm, so that the compiler places the
// waits for an MFMA's result)
extern "C" __device__ float cvb_fmul_legacy(float, float) __asm("llvm.amdgcn.fmul.legacy");
__device__ __forceinline__ float mul0(float a, float b) { return cvb_fmul_legacy(a, b); }

// The smaller of two products, the other one where one is NaN: fminf, which
// would first pass mul0's result through an instruction of its own.
__device__ __forceinline__ float min_num(float a, float b) {
  float d;
  asm("v_min_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// The variable code of a neuron's status word: the byte offset of an unstable
// neuron's alpha in its row's block; a split neuron's side and index with
// both top bits set; kNoVar otherwise.
__device__ __forceinline__ uint32_t var_code(uint32_t rec) {
  const uint32_t kind = rec & kKindMask;
  return kind == kUnstable ? (rec & kCidxMask) << 2 : (kind == kSplit ? rec : kNoVar);
}
__device__ __forceinline__ bool is_unstable(uint32_t vo) { return (int32_t)vo >= 0; }
__device__ __forceinline__ bool is_split(uint32_t vo) { return (vo & kKindMask) == kSplit; }

// Staged slot of input float t (as conv.hip's)
__device__ __forceinline__ int staged_at(const ConvPlan& pl, int t) {
  const int c = __umulhi((unsigned)t, pl.mgp);
  const int rem = t - c * (pl.gh * pl.gw);
  const int y = __umulhi((unsigned)rem, pl.mgw);
  return c * pl.pplane + pl.bofs + y * pl.gwp + (rem - y * pl.gw);
}

// What a launch asks of a kernel beyond its mode, fixed when it is compiled
// (kept apart so that the common passes carry neither the registers nor the
// tests of the others).  Back-substitution: kPlain, or kMargin with the
// rounding-error weights of sound mode or an l_p ball.  Adjoint: kGrad, kAdam
// or kTrue (the network itself at x*).
enum Kind { kPlain = 0, kMargin = 1, kGrad = 0, kAdam = 1, kTrue = 2 };

// An opaque copy: tests on a lane's variable codes are made where they are
// used instead of being held over the rows as a lane mask each
__device__ __forceinline__ uint32_t here(uint32_t x) {
  asm volatile("" : "+v"(x));
  return x;
}

template <int MODE, int KIND, int NTW, int TM>
constexpr int reg_occupancy() {
  constexpr int nu = NTW * TM;
  if (MODE == kBwdConc) return nu >= 4 ? 3 : 4;
  if (MODE == kBwdRelax) return nu >= 4 ? 2 : nu == 2 ? 3 : 4;
  return nu >= 2 ? 2 : 4;  // (eight numbers per neuron spill in 168 registers)
}

// NP > 0: the number of K passes (of 16) when compiled in (all column tiles in
// one wave): a lane keeps its gathers' LDS addresses in registers for every
// row, and a row's GEMM is LDS reads and MFMAs alone.  NP = 0: any K, the
// column offsets in LDS too, everything read a pass ahead.
template <int MODE, int KIND, int NTW, int TM, int NP, int RC>
__global__ __launch_bounds__(64 * reg_max_waves(MODE, NTW, TM), (reg_occupancy<MODE, KIND, NTW, TM>())) void conv_reg(
    const float* __restrict__ zin, int ldi, ConvPlan pl, int M, int last, Batch bt, Vars v, Epi e, int mu) {
  extern __shared__ float4 smem4[];
  constexpr int kWaves = reg_max_waves(MODE, NTW, TM);
  __shared__ float red[2][kWaves][2];
  constexpr bool kBwd = MODE == kBwdRelax || MODE == kBwdConc;
  constexpr int NU = TM * NTW * RC;  // neurons per lane
  const ConvReg& rp = pl.reg;
  const int m = bt.m;
  const int upb = (m + mu - 1) / mu;  // units per subdomain
  const int n_units = (M / m) * upb;
  if ((int)blockIdx.x >= n_units) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nthr = blockDim.x;
  const int n_pass = pl.kpad >> 4;

  // LDS: the staged row (rp.nbuf of them, each with a spare slot for lanes that
  // stage nothing); with NP = 0 the weights (four K steps of a lane together)
  // and the column offsets of a lane group's four K steps of a pass
  const int zpitch = (pl.dinp + 4) & ~3;
  float* const zi0 = reinterpret_cast<float*>(smem4);
  float4* const w4 = smem4 + rp.nbuf * (zpitch >> 2);
  int4* const ko = reinterpret_cast<int4*>(w4 + n_pass * rp.nt * 64);
  for (int t = tid; t < n_pass * rp.nt * 64; t += nthr) w4[t] = rp.w4[t];
  if constexpr (NP == 0) {
    for (int t = tid; t < n_pass * 4; t += nthr) {
      const int4* const k = pl.ktab + (t >> 2) * 16 + (t & 3);
      ko[t] = make_int4(k[0].x, k[4].x, k[8].x, k[12].x);
    }
  }
  for (int t = tid; t < rp.nbuf * zpitch; t += nthr) zi0[t] = 0.f;  // the borders stay zero
  if (tid < 4 * kWaves) (&red[0][0][0])[tid] = 0.f;

  // this wave's tiles: column tiles t0 .. t0 + NTW - 1 of TM consecutive tiles
  // of m; j = base + plane (r + ts t), past dout where the lane has no neuron
  const int tg = rp.nt / NTW, t0 = (wave % tg) * NTW, mt0 = (wave / tg) * TM;
  int mex[TM];
  uint32_t base[TM];  // byte offset of the lane's first neuron in a row
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const bool ok = mt0 + i < rp.n_mt;
    const int4 o = rp.ob[(ok ? mt0 + i : 0) * 64 + lane];
    mex[i] = o.x;
    base[i] = ok && o.y >= 0 ? (uint32_t)(o.y + rp.plane * rp.ts * t0) * 4u : kNoVar;
  }
  const uint32_t sp = rp.plane * 4;  // bytes between the channels of a lane
  // byte offset of the lane's neuron u = (i NTW + t) RC + r in a row
  auto off = [&](int u) { return base[u / (RC * NTW)] + sp * (uint32_t)(u % RC + rp.ts * ((u / RC) % NTW)); };
  int kr[NP > 0 ? NP : 1][4];
  if constexpr (NP > 0) {
#pragma unroll
    for (int ps = 0; ps < NP; ++ps) {
#pragma unroll
      for (int q = 0; q < 4; ++q) kr[ps][q] = pl.ktab[(4 * ps + q) * 4 + (lane >> 4)].x + (TM == 1 ? mex[0] : 0);
    }
  }

  // the staged slots of this thread's inputs (the same for every row), where
  // rows are staged by float4s
  const bool v4 = rp.v4;
  int so[kRegIn];
#pragma unroll
  for (int q = 0; q < kRegIn; ++q) {
    const int t = 4 * (tid + nthr * q);
    so[q] = MODE != kFwdX && t < pl.din ? staged_at(pl, t) : -1;
  }
  // x* of a conv first layer: word w of the row's sign planes holds the
  // lanes' inputs xt[64 w + lane]; a wave stages kRegWords of them
  // (their byte offsets in the staged row, under 64 KB, in pairs)
  uint32_t xs[kRegWords / 2];
  const int xw0 = wave * kRegWords;
  if constexpr (MODE == kFwdX) {
#pragma unroll
    for (int q = 0; q < kRegWords; ++q) {
      const uint32_t at = (uint32_t)(xw0 + q < rp.nwords ? rp.xt[(xw0 + q) * 64 + lane].x : pl.dinp) * 4u;
      xs[q >> 1] = (q & 1) ? xs[q >> 1] | (at << 16) : at;
    }
  }
  float4 in4[kRegIn];
  // the box of those inputs: in registers, or with Adam's numbers there already
  // in LDS (each lane its own entries: no barrier)
  constexpr bool kBoxLds = MODE == kFwdX && KIND == kAdam;
  float xl[kRegWords], xu[kRegWords];
  float2* const bx = reinterpret_cast<float2*>(ko + (NP == 0 ? n_pass * 4 : 0)) + xw0 * 64 + lane;
  uint64_t wp[kRegWords], wn[kRegWords];
  auto in_load = [&](int row) {
    if constexpr (MODE == kFwdX) {
      const cword_ptr p = (cword_ptr)(v.xpos + (int64_t)row * bt.w64);
      const cword_ptr n = (cword_ptr)(v.xneg + (int64_t)row * bt.w64);
#pragma unroll
      for (int q = 0; q < kRegWords; ++q) {
        const int w = min(xw0 + q, rp.nwords - 1);
        wp[q] = p[w];
        wn[q] = n[w];
      }
    } else {
      const float* const zr = zin + (int64_t)row * ldi;
      if (v4) {
#pragma unroll
        for (int q = 0; q < kRegIn; ++q)
          in4[q] = reinterpret_cast<const float4*>(zr)[min(tid + nthr * q, (pl.din >> 2) - 1)];
      } else {
#pragma unroll
        for (int q = 0; q < 4 * kRegIn; ++q)
          reinterpret_cast<float*>(in4)[q] = zr[min((int)here(tid) + nthr * q, pl.din - 1)];
      }
    }
  };
  auto box_load = [&](int p) {
    if constexpr (MODE == kFwdX) {
      const float* const l = bt.xlo + (int64_t)p * bt.d0;
      const float* const h = bt.xhi + (int64_t)p * bt.d0;
#pragma unroll
      for (int q = 0; q < kRegWords; ++q) {
        const int j = rp.xt[min(xw0 + q, rp.nwords - 1) * 64 + lane].y;
        if constexpr (kBoxLds) {
          bx[q * 64] = make_float2(l[j], h[j]);
        } else {
          xl[q] = l[j];
          xu[q] = h[j];
        }
      }
    }
  };
  auto in_store = [&](float* zi, int row) {
    if constexpr (MODE == kFwdX) {
#pragma unroll
      for (int q = 0; q < kRegWords; ++q) {
        float2 b;
        if constexpr (kBoxLds) b = bx[q * 64];
        else b = make_float2(xl[q], xu[q]);
        *reinterpret_cast<float*>(reinterpret_cast<char*>(zi) + ((q & 1) ? xs[q >> 1] >> 16 : xs[q >> 1] & 0xffffu)) =
            pick_bit(pick_bit(0.5f * (b.x + b.y), b.y, wn[q]), b.x, wp[q]);
      }
    } else {
      const float* const zr = zin + (int64_t)row * ldi;
      if (v4) {
#pragma unroll
        for (int q = 0; q < kRegIn; ++q) {
          if (so[q] < 0) continue;
          float* const z = zi + so[q];
          z[0] = in4[q].x;
          z[1] = in4[q].y;
          z[2] = in4[q].z;
          z[3] = in4[q].w;
        }
        // a row longer than the read-ahead holds
        for (int t = 4 * (tid + nthr * kRegIn); t < pl.din; t += 4 * nthr) {
          const float4 x = *reinterpret_cast<const float4*>(zr + t);
          float* const z = zi + staged_at(pl, t);
          z[0] = x.x;
          z[1] = x.y;
          z[2] = x.z;
          z[3] = x.w;
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4 * kRegIn; ++q) {
          const int t = (int)here(tid) + nthr * q;  // (its slot: computed here, not held)
          if (t < pl.din) zi[staged_at(pl, t)] = reinterpret_cast<const float*>(in4)[q];
        }
        for (int t = tid + nthr * 4 * kRegIn; t < pl.din; t += nthr) zi[staged_at(pl, t)] = zr[t];
      }
    }
  };

  // the bias of the lane's neurons (the relaxed layer's, or the adjoint's own)
  float kb[NU];
  if constexpr (MODE != kBwdConc) {
    const rsrc_t rb = view(e.bias, (int64_t)pl.dout * 4);
#pragma unroll
    for (int u = 0; u < NU; ++u) kb[u] = ldf(rb, off(u));
  }

  __syncthreads();  // before any thread stages a row over the zeroed planes
  float* zi = zi0;
  {
    const int b0 = blockIdx.x / upb;
    const int row0 = b0 * m + ((int)blockIdx.x - b0 * upb) * mu;
    in_load(row0);
    box_load(bt.prop[b0]);
    in_store(zi, row0);
  }
  __syncthreads();  // the first row is staged

  int par = 0;
  for (int unit = blockIdx.x; unit < n_units; unit += gridDim.x) {
    const int b = unit / upb;
    const int r0 = b * m + (unit - b * upb) * mu;
    const int r1 = b * m + min((unit - b * upb) * mu + mu, m);
    const int p = bt.prop[b];
    const int64_t ab0 = bt.aoff[b];
    const int uc = bt.ucount[p];
    RowInfo ri{b, r0 - b * m, p, ab0 + (int64_t)(r0 - b * m) * uc};

    // ---- the relaxation of the lane's neurons, for every row of the unit.
    // Back-substitution: Lambda = a (a >= 0 ? x : c0) + sx, constant += a c1
    // where unstable and a < 0, with x alpha of an unstable neuron and c0
    // elsewhere (1 active or split z >= 0, 0 inactive or split z < 0), c0, c1
    // an unstable neuron's chord, sx -beta (+beta) of a split z >= 0 (z < 0)
    // neuron.
    // Adjoint: zhat = x1 >= 0 ? zb x : c0 zb + c1, x1 the stored A (0 where
    // not unstable).  Concretisation: c0, c1 the input's box.  Slopes and boxes
    // multiply by mul0: a neuron of slope 0, and a lane without a neuron, take
    // nothing from an a or zb that left float32.  The operations and roundings
    // of the case analysis (common.h), the sign of a zero and 0 inf aside.
    uint32_t vo[NU];
    float c0[NU], c1[NU], x[NU], sx[NU], x1[NU], x3[NU], x4[NU];
    uint64_t any_split = 0;
    if constexpr (MODE == kBwdConc) {
      const rsrc_t rl = view((KIND == kMargin && bt.l2x0 ? bt.l2x0 : bt.xlo) + (int64_t)p * bt.d0, (int64_t)pl.dout * 4);
      const rsrc_t ru = view(bt.xhi + (int64_t)p * bt.d0, (int64_t)pl.dout * 4);
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        c0[u] = ldf(rl, off(u));
        c1[u] = ldf(ru, off(u));
      }
    } else {
      const int64_t pc0 = (int64_t)p * bt.nd + e.layer_off;
      const rsrc_t rs = view(bt.status + (int64_t)b * bt.nd + e.layer_off, (int64_t)pl.dout * 4);
      const rsrc_t rc = view(bt.chord + pc0, (int64_t)pl.dout * 8);
      const rsrc_t rd = view(bt.adef + pc0, (int64_t)pl.dout * 4);
      uint32_t rec[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const uint32_t o = off(u);
        rec[u] = ldu(rs, o);
        const uint32_t o2 = (o << 1) | (o & kNoVar);  // (a lane without a neuron stays past the end)
        c0[u] = ldf(rc, o2);
        c1[u] = ldf(rc, o2 + 4);
        x[u] = ldf(rd, o);
        if (MODE == kFwd && e.wx0) kb[u] = ldf(view(e.wx0 + (int64_t)p * e.n, (int64_t)e.n * 4), o);
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        vo[u] = var_code(rec[u]);
        const uint32_t kind = rec[u] & kKindMask;
        const bool one = kind == kActive || (kind == kSplit && (rec[u] & kSidePos));
        const bool uns = kind == kUnstable;
        c0[u] = uns ? c0[u] : (one ? 1.f : 0.f);
        c1[u] = uns ? c1[u] : 0.f;
        x[u] = uns ? x[u] : c0[u];
        sx[u] = x1[u] = x3[u] = x4[u] = 0.f;
        any_split |= __ballot(kind == kSplit);
      }
    }
    // a row's own variables: alpha (and the adjoint's stored A and Adam
    // moments) of the unstable neurons, beta of the split ones
    auto row_vars = [&]() {
      if constexpr (MODE == kBwdConc) return;
      const int64_t ub = (int64_t)uc * 4;
      if constexpr (MODE == kBwdRelax) {
        if (v.alpha) {
          const rsrc_t ra = view(v.alpha + ri.abase, ub);
#pragma unroll
          for (int u = 0; u < NU; ++u) x[u] = ldf(ra, vo[u]);
        }
        if (any_split) {
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const uint32_t c = here(vo[u]);
            if (is_split(c)) sx[u] = v.beta[(int64_t)(c & kSplitMask) * bt.m + ri.k];
          }
        }
      } else {
        if constexpr (KIND == kTrue) return;
        const rsrc_t rs = view(v.acomp + ri.abase, ub);
#pragma unroll
        for (int u = 0; u < NU; ++u) x1[u] = ldf(rs, vo[u]);
        if (KIND == kAdam || v.alpha) {
          const rsrc_t ra = view((KIND == kAdam ? v.alpha_w : v.alpha) + ri.abase, ub);
#pragma unroll
          for (int u = 0; u < NU; ++u) x[u] = ldf(ra, vo[u]);
        }
        if constexpr (KIND == kAdam) {
          const rsrc_t r3 = view(v.ma + ri.abase, ub), r4 = view(v.va + ri.abase, ub);
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            x3[u] = ldf(r3, vo[u]);
            x4[u] = ldf(r4, vo[u]);
          }
        }
      }
    };
    row_vars();
    // the next unit's first row (staged during this unit's last row)
    const int nunit = unit + gridDim.x;
    const int nb = nunit / upb;
    const int nfirst = nunit < n_units ? nb * m + (nunit - nb * upb) * mu : -1;

    for (int row = r0; row < r1; ++row, par ^= 1) {
      const int nrow = row + 1 < r1 ? row + 1 : nfirst;
      if (nrow >= 0) in_load(nrow);
      if (MODE == kFwdX && row + 1 == r1 && nrow >= 0 && bt.prop[nb] != p) box_load(bt.prop[nb]);

      // ---- the GEMM over K passes [p0, p1), into s
      auto gemm = [&](floatx4(&s)[TM][NTW], int p0, int p1) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int t = 0; t < NTW; ++t) s[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
        if constexpr (NP > 0) {
#pragma unroll
          for (int ps = 0; ps < NP; ++ps) {
            float4 bw[NTW];
#pragma unroll
            for (int t = 0; t < NTW; ++t) bw[t] = w4[(ps * NTW + t) * 64 + lane];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int i = 0; i < TM; ++i) {
                const float a = (zi0 + (TM == 1 ? 0 : mex[i]))[kr[ps][q]];
#pragma unroll
                for (int t = 0; t < NTW; ++t)
                  s[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(comp(bw[t], q), a, s[i][t], 0, 0, 0);
              }
          }
          // two passes' LDS reads ahead of the MFMAs that use them
          constexpr int kRd = NTW + 4 * TM, kMf = 4 * TM * NTW;
          __builtin_amdgcn_sched_group_barrier(0x100, (NP > 1 ? 2 : 1) * kRd, 0);
#pragma unroll
          for (int ps = 0; ps < NP; ++ps) {
            __builtin_amdgcn_sched_group_barrier(0x008, kMf, 0);
            if (ps + 2 < NP) __builtin_amdgcn_sched_group_barrier(0x100, kRd, 0);
          }
        } else {
          // one pass ahead: its gathers (at offsets read two ahead) and weights
          const int g = lane >> 4;
          int4 kn = ko[p0 * 4 + g];
          float4 bn[NTW];
          float an[TM][4];
          auto fetch = [&](int ps) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
              const float* const z = zi + mex[i];
              an[i][0] = z[kn.x];
              an[i][1] = z[kn.y];
              an[i][2] = z[kn.z];
              an[i][3] = z[kn.w];
            }
#pragma unroll
            for (int t = 0; t < NTW; ++t) bn[t] = w4[(ps * rp.nt + t0 + t) * 64 + lane];
            kn = ko[min(ps + 1, n_pass - 1) * 4 + g];
          };
          fetch(p0);
          for (int ps = p0; ps < p1; ++ps) {
            float4 bw[NTW];
            float a[TM][4];
#pragma unroll
            for (int t = 0; t < NTW; ++t) bw[t] = bn[t];
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int q = 0; q < 4; ++q) a[i][q] = an[i][q];
            fetch(min(ps + 1, n_pass - 1));
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
              for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < NTW; ++t)
                  s[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(comp(bw[t], q), a[i][q], s[i][t], 0, 0, 0);
            // the next pass's reads before this pass's MFMAs
            __builtin_amdgcn_sched_group_barrier(0x100, 4 * TM + NTW + 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4 * TM * NTW, 0);
          }
        }
      };
      floatx4 acc[TM][NTW];
      if (TM > 1 || NP > 0 || rp.ksp == 1) {
        gemm(acc, 0, n_pass);
      } else {  // chunks of the K passes, summed in order
        gemm(acc, 0, n_pass / rp.ksp);
        for (int c = 1; c < rp.ksp; ++c) {
          floatx4 part[TM][NTW];
          gemm(part, c * n_pass / rp.ksp, (c + 1) * n_pass / rp.ksp);
#pragma unroll
          for (int t = 0; t < NTW; ++t) acc[0][t] += part[0][t];
        }
      }
      float* const zn = rp.nbuf == 2 ? (zi == zi0 ? zi0 + zpitch : zi0) : zi;
      if (rp.nbuf == 1) __syncthreads();  // every wave is past this row's GEMM
      if (nrow >= 0) in_store(zn, nrow);
      // every outstanding load has long arrived: one wait here, so that the
      // compiler issues none between the epilogue's stores (a wait for a load
      // would be a wait for every store before it too)
      __builtin_amdgcn_s_waitcnt(kWaitVm0);

      // ---- the epilogue, on the accumulators
      float cst = 0.f, cer = 0.f;
      const int64_t ub = (int64_t)uc * 4;
      if constexpr (MODE == kBwdRelax) {
        const rsrc_t ro = view(e.out + (int64_t)row * e.ldo, (int64_t)pl.dout * 4);
        if (any_split) {  // the sign of a split neuron's beta: - where z >= 0
#pragma unroll
          for (int u = 0; u < NU; ++u) sx[u] = __uint_as_float(__float_as_uint(sx[u]) ^ ((vo[u] << 2) & 0x80000000u));
        }
        if (v.acomp) {
          const rsrc_t rs = view(v.acomp + ri.abase, ub);
#pragma unroll
          for (int u = 0; u < NU; ++u) stf(acc[u / (RC * NTW)][(u / RC) % NTW][u % RC], rs, vo[u]);
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) {
          const float a = acc[u / (RC * NTW)][(u / RC) % NTW][u % RC];
          // (no alpha array: x keeps the default slopes)
          const bool uns = is_unstable(vo[u]);
          const float xp = uns ? x[u] : c0[u];
          // (sx is 0 or the slope 0 or 1: one rounding either way)
          const float lam = mul0(a, a >= 0.f ? xp : c0[u]) + sx[u];
          cst = uns && !(a >= 0.f) ? fmaf(a, c1[u], cst) : cst;
          cst = fmaf(lam, kb[u], cst);
          stf(lam, ro, off(u));
          if (KIND == kMargin && bt.sw) {
            const rsrc_t rw = view(bt.sw + (int64_t)p * bt.nd + e.layer_off, (int64_t)pl.dout * 4);
            cer = fmaf(fabsf(lam), ldf(rw, off(u)), cer);
          }
        }
      } else if constexpr (MODE == kBwdConc) {
        if (KIND == kMargin && bt.l2x0) {  // l_p ball: A(0) x0 here, - eps ||A(0)||_q in the final sum
          const rsrc_t rx = view(v.xdense + (v.xdense ? (int64_t)row * v.ldx : 0), (int64_t)pl.dout * 4);
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const float a = acc[u / (RC * NTW)][(u / RC) % NTW][u % RC];
            cst = off(u) < (uint32_t)pl.dout * 4u ? fmaf(a, c0[u], cst) : cst;
            float sq = 0.f;
            const float xd = lp_entry(a, bt.lpq, &sq);
            // (a lane without a neuron: its sum of powers does not count)
            cer += off(u) < (uint32_t)pl.dout * 4u ? sq : 0.f;
            if (v.xdense) stf(xd, rx, off(u));  // x*'s direction for the adjoint
          }
        } else {
          // x* as two sign planes, a word per (tile, r): bit = lane
          int lp[2] = {0, 0}, ln[2] = {0, 0};
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const float a = acc[u / (RC * NTW)][(u / RC) % NTW][u % RC];
            // (0 inf of the upper edge: NaN, which the minimum leaves out)
            const float tm = min_num(mul0(a, c0[u]), a * c1[u]);
            cst += tm;
            if (KIND == kMargin) cer = fmaf(bt.sg, fabsf(tm), cer);
            if (v.xpos) {
              const uint64_t bp = __ballot(a > 0.f), bn = __ballot(a < 0.f);
              const bool mine = lane == u;
              lp[0] = mine ? (int)bp : lp[0];
              lp[1] = mine ? (int)(bp >> 32) : lp[1];
              ln[0] = mine ? (int)bn : ln[0];
              ln[1] = mine ? (int)(bn >> 32) : ln[1];
            }
          }
          static_assert(NU <= 64, "a lane per word");
          // (all column tiles in one wave: its words are consecutive)
          const int w0 = mt0 * rp.nt * RC;
          if (v.xpos && lane < NU && w0 + lane < rp.nwords) {
            reinterpret_cast<int2*>(v.xpos + (int64_t)row * bt.w64)[w0 + lane] = make_int2(lp[0], lp[1]);
            reinterpret_cast<int2*>(v.xneg + (int64_t)row * bt.w64)[w0 + lane] = make_int2(ln[0], ln[1]);
          }
        }
      } else {
        const float rm = MODE == kFwd && e.wx0 ? -v.l2s[row] : 1.f;
        const rsrc_t ro = view(e.out + (int64_t)row * e.ldo, (int64_t)pl.dout * 4);
        if constexpr (KIND == kTrue) {  // the network itself at x*: the exact ReLU, the splits checked
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const float zb = fmaf(rm, acc[u / (RC * NTW)][(u / RC) % NTW][u % RC], kb[u]);
            const uint32_t c = here(vo[u]);
            if (any_split && is_split(c) && ((c & kSidePos) ? zb < 0.f : zb > 0.f)) v.sat[row] = 0;
            stf(fmaxf(zb, 0.f), ro, off(u));
          }
        } else {
          float zbv[NU];
#pragma unroll
          for (int u = 0; u < NU; ++u) {
            const float zb = fmaf(rm, acc[u / (RC * NTW)][(u / RC) % NTW][u % RC], kb[u]);
            const float xp = is_unstable(vo[u]) ? x[u] : c0[u];
            const float zh = x1[u] >= 0.f ? mul0(zb, xp) : fmaf(c0[u], zb, c1[u]);
            if (!last) stf(zh, ro, off(u));
            zbv[u] = zb;
          }
          if constexpr (KIND == kAdam) {
            const rsrc_t ra = view(v.alpha_w + ri.abase, ub), r3 = view(v.ma + ri.abase, ub),
                         r4 = view(v.va + ri.abase, ub);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
              const float g = x1[u] >= 0.f ? zbv[u] * x1[u] : 0.f;
              float ma, va;
              const float xn = adam_values(g, v.lr_a, v.bc1, v.bc2, 0.f, 1.f, x[u], x3[u], x4[u], ma, va);
              stf(ma, r3, vo[u]);
              stf(va, r4, vo[u]);
              stf(xn, ra, vo[u]);
            }
          } else {
            const rsrc_t rg = view(v.galpha + ri.abase, ub);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
              stf(x1[u] >= 0.f ? zbv[u] * x1[u] : 0.f, rg, vo[u]);
              // (the joint optimisation's zbar at upper-chord neurons)
              if (v.zchord) {
                const rsrc_t rz = view(v.zchord + ri.abase, ub);
                stf(zbv[u], rz, x1[u] < 0.f ? vo[u] : kNoVar);
              }
            }
          }
          if (any_split) {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
              const uint32_t c = here(vo[u]);
              if (is_split(c)) {
                const int64_t bi = (int64_t)(c & kSplitMask) * bt.m + ri.k;
                const float gb = (c & kSidePos) ? -zbv[u] : zbv[u];
                // (a split neuron owns an alpha entry too: its gradient is 0)
                const int64_t ai = ri.abase + bt.cidx[(int64_t)p * bt.nd + e.layer_off + (off(u) >> 2)];
                if (v.gsplit) {  // the steps: split_adam_k, after the pass
                  v.gsplit[bi] = gb;
                } else if (KIND == kAdam) {
                  adam_apply(v.beta_w, v.mb, v.vb, bi, gb, v.lr_b, v.bc1, v.bc2, 0.f, INFINITY);
                  adam_apply(v.alpha_w, v.ma, v.va, ai, 0.f, v.lr_a, v.bc1, v.bc2, 0.f, 1.f);
                } else {
                  v.gbeta[bi] = gb;
                  v.galpha[ai] = 0.f;
                }
              }
            }
          }
        }
      }
      if (kBwd) {
        cst = wave_sum(cst);
        if (KIND == kMargin) cer = wave_sum(cer);
        if (lane == 0) {
          red[par][wave][0] = cst;
          if (KIND == kMargin) red[par][wave][1] = cer;
        }
      }
      if (row + 1 < r1) {
        ri.k += 1;
        ri.abase += uc;
        row_vars();
      }
      __syncthreads();  // the next row is staged; with two buffers, this row's is free
      if (kBwd && tid == 0) {
        float tot = 0.f, ter = 0.f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {  // (waves past the workgroup's: zeros)
          tot += red[par][w][0];
          if (KIND == kMargin) ter += red[par][w][1];
        }
        e.part[(int64_t)e.slot0 * M + row] = tot;
        if constexpr (KIND == kMargin) {
          // rounding-error bound, or the sum of A(0)^2 (l2 ball); with both
          // modes on, the other array's slot gets 0
          float* const p2 = MODE == kBwdConc && bt.l2x0 ? e.psq : (e.perr ? e.perr : e.psq);
          float* const pz = e.perr && e.psq ? (p2 == e.perr ? e.psq : e.perr) : nullptr;
          if (p2) p2[(int64_t)e.slot0 * M + row] = ter;
          if (pz) pz[(int64_t)e.slot0 * M + row] = 0.f;
        }
      }
      zi = zn;
    }
  }
}

// (column tiles, row tiles per wave, K passes) that are built.  The passes are
// compiled in wherever one wave holds all column tiles and there are one to six
// of them: the gathers' addresses take four registers a pass and row tile, and
// with more the kernels spill (at six, 16 bytes in back-substitution with two
// row tiles, 8 in the adjoint with Adam).  Against the loop over passes (P = 0),
// us per launch at 9,216 rows: back-substitution 8 -> 8 k3 s1 on 16x16 64.2 and
// 76.5, 12 -> 8 95.9 and 122.5, 4 -> 4 44.4 and 50.4; into 3x32x32 from 16
// channels k4 s2 86.6 and 116.5, from 12 72.6 and 96.1, from 8 k3 s2 56.6 and
// 93.6; x* into 6 channels k4 s2 77.0 and 89.2; adjoint 8 -> 6 k3 s1 68.3 and
// 77.1.  Of 60 layers drawn from generic networks the loop was faster on two,
// into 3x24x24 from 5 and 6 channels k5 s2 (47 and 56 against 54 and 62: a
// second staged row in LDS).  (Concretisation takes four row tiles with one or two passes, two with
// more: conv_plan_reg.)
#define CVB_REG_K6(X, T) X(1, T, 0) X(1, T, 1) X(1, T, 2) X(1, T, 3) X(1, T, 4) X(1, T, 5) X(1, T, 6)
#define CVB_REG_RELAX(X) CVB_REG_K6(X, 1) CVB_REG_K6(X, 2) X(2, 1, 0) X(2, 2, 0)
#define CVB_REG_CONC(X) X(1, 2, 0) X(1, 2, 3) X(1, 2, 4) X(1, 2, 5) X(1, 2, 6) X(1, 4, 0) X(1, 4, 1) X(1, 4, 2) X(2, 1, 0)
#define CVB_REG_FWDX(X) CVB_REG_K6(X, 1) CVB_REG_K6(X, 2) X(2, 1, 0)
#define CVB_REG_FWD(X) CVB_REG_K6(X, 1) CVB_REG_K6(X, 2) X(2, 1, 0)

typedef void (*reg_fn)(const float*, int, ConvPlan, int, int, Batch, Vars, Epi, int);

template <int MODE, int KIND>
reg_fn reg_kernel_kind(int ntw, int tm, int np, int rc) {
#define CVB_RK(N, T, P) \
  if (ntw == N && tm == T && np == P) \
    return MODE == kBwdConc && rc <= 3 ? conv_reg<MODE, KIND, N, T, P, MODE == kBwdConc ? 3 : 4> : conv_reg<MODE, KIND, N, T, P, 4>;
  if constexpr (MODE == kBwdRelax) {
    CVB_REG_RELAX(CVB_RK)
  } else if constexpr (MODE == kBwdConc) {
    CVB_REG_CONC(CVB_RK)
  } else if constexpr (MODE == kFwdX) {
    CVB_REG_FWDX(CVB_RK)
  } else {
    CVB_REG_FWD(CVB_RK)
  }
#undef CVB_RK
  return nullptr;
}

reg_fn reg_kernel(int mode, int kind, int ntw, int tm, int np, int rc) {
  switch (mode) {
    case kBwdRelax:
      return kind == kPlain ? reg_kernel_kind<kBwdRelax, kPlain>(ntw, tm, np, rc)
                            : reg_kernel_kind<kBwdRelax, kMargin>(ntw, tm, np, rc);
    case kBwdConc:
      return kind == kPlain ? reg_kernel_kind<kBwdConc, kPlain>(ntw, tm, np, rc)
                            : reg_kernel_kind<kBwdConc, kMargin>(ntw, tm, np, rc);
    case kFwdX:
      return kind == kGrad   ? reg_kernel_kind<kFwdX, kGrad>(ntw, tm, np, rc)
             : kind == kAdam ? reg_kernel_kind<kFwdX, kAdam>(ntw, tm, np, rc)
                             : reg_kernel_kind<kFwdX, kTrue>(ntw, tm, np, rc);
    default:
      return kind == kGrad   ? reg_kernel_kind<kFwd, kGrad>(ntw, tm, np, rc)
             : kind == kAdam ? reg_kernel_kind<kFwd, kAdam>(ntw, tm, np, rc)
                             : reg_kernel_kind<kFwd, kTrue>(ntw, tm, np, rc);
  }
}

}  // namespace

static int reg_box_bytes(const ConvReg& r) { return r.nw * kRegWords * 64 * (int)sizeof(float2); }

void conv_plan_reg(int mode, ConvPlan& pl) {
  ConvReg& r = pl.reg;
  r.grid = 0;
  if (!r.ob) return;
  r.v4 = pl.gw % 4 == 0 && pl.din % 4 == 0;
  // (column, row) tiles per wave: the first that fits the waves of a workgroup,
  // wider n first (the gathers of a row tile serve its column tiles).  A pair
  // of row tiles where back-substitution has eight of them: 428 us against
  // 467 with one tile each (8 -> 8 channels k3 s1 on 16x16, 73,728 rows); the
  // adjoint's eight numbers per neuron spill with two (653 against 618).
  static const int wide[][2] = {{2, 1}, {1, 2}, {1, 1}, {2, 2}, {1, 4}};
  static const int thin[][2] = {{2, 1}, {1, 1}, {1, 2}, {2, 2}, {1, 4}};
  // Concretisation, 19 tiles of a 32x32 input: four per wave with two K passes
  // (409 us against 442 with two; 8 -> 3 channels, 73,728 rows), two with more
  // (85 against 156; 16 -> 3 channels, 9,216 rows).
  static const int conc[][2] = {{2, 1}, {1, 4}, {1, 2}, {1, 1}, {1, 4}};
  static const int conc_k[][2] = {{2, 1}, {1, 2}, {1, 4}, {1, 1}, {1, 4}};
  const auto& cand = mode == kBwdConc ? (pl.kpad > 32 ? conc_k : conc) : mode == kBwdRelax && r.n_mt >= 8 ? wide : thin;
  r.nw = 0;
  for (const auto& c : cand) {
    if (r.nt % c[0] || (c[0] == 1 && r.nt > 1)) continue;
    const int nw = r.nt / c[0] * ((r.n_mt + c[1] - 1) / c[1]);
    if (nw > reg_max_waves(mode, c[0], c[1]) || (mode == kBwdConc && r.nt > c[0])) continue;
    if (mode == kFwdX && (r.nwords <= 0 || r.nwords > nw * kRegWords)) continue;
    if (!reg_kernel(mode, 0, c[0], c[1], 0, r.rc)) continue;
    r.ntw = c[0];
    r.tm = c[1];
    r.nw = nw;
    break;
  }
  if (!r.nw) return;
  // The default where nothing is tuned.  Register tiles win where a row is
  // large (of 2,048 neurons and more an older kernel's thread owns four and
  // walks them in natural order) and where its workgroups are so small that
  // several rows run on a CU, as long as its one chain of K passes is short;
  // in between, tiles that a row does not fill leave the matrix cores idle.
  // Back-substitution through a stride-2 layer shares its GEMM rows between the
  // classes, so that a third of a 16x16 plane's lanes have no neuron (8 -> 8 k4
  // s2 above), and the adjoint's eight numbers per neuron leave eight waves no
  // room for more of them (8 -> 8 k3 s1 with Adam): both want more neurons
  // still.  Concretisation, which holds no variables, loses to K alone.
  // Over 150 networks drawn from 1 to 4 channels on 11x13 to 32x32, 1 to 3
  // convolutions of 3 to 32 channels, k2 to k5, s1 and s2, tiles against the
  // variants at 9,216 rows, geometric mean over all layers and the layers they
  // slow by more than 3 %: this rule 1.10 and 1 of 134 (back-substitution), 1.33
  // and 2 of 80 (concretisation), 1.16 and none of 80 (x*), 1.12 and 4 of 134
  // (adjoint); tiles everywhere 1.13 and 31, 1.32 and 8, 1.12 and 21, 1.11 and
  // 31.  At 576 rows 12 of the 428 against 87.
  const bool small = r.nw * r.nt <= (mode == kBwdRelax ? 2 : 4) && pl.kpad <= (mode == kFwd ? 192 : 128);
  const bool edge = mode == kBwdRelax ? r.ts == 16 && pl.kpad >= 96 : mode == kFwd ? r.nt > 1 : true;
  const bool large = pl.dout > 2048 || (pl.dout == 2048 && edge) ||
                     (mode == kFwdX && r.tm * r.nt == 1 && pl.dout >= 1536);
  r.prefer = small || large || (mode == kBwdConc && pl.kpad <= 128);
  // K passes compiled in where that kernel exists (and adds no K chunks)
  r.np = r.ksp == 1 && r.nt == r.ntw && reg_kernel(mode, 0, r.ntw, r.tm, pl.kpad >> 4, r.rc) ? pl.kpad >> 4 : 0;
  const int w = pl.kpad * r.nt * 16 * (int)sizeof(float) + (r.np ? 0 : pl.kpad * (int)sizeof(int));
  const int z = ((pl.dinp + 4) & ~3) * (int)sizeof(float);
  // two input rows where that leaves room for 16 waves on a CU (one where the
  // gathers' addresses are fixed)
  r.nbuf = !r.np && w + 2 * z <= 160 * 1024 * r.nw / 16 ? 2 : 1;
  r.smem = w + r.nbuf * z;
  // (the adjoint's box in LDS, with Adam)
  const int smem = r.smem + (mode == kFwdX ? reg_box_bytes(r) : 0);
  if (smem > 64 * 1024) return;
  const int grid =
      resident_blocks(reinterpret_cast<const void*>(reg_kernel(mode, 1, r.ntw, r.tm, r.np, r.rc)), 64 * r.nw, smem);
  if (grid < 0) return;
  r.grid = grid;
}

int launch_conv_reg(int mode, const ConvArgs& a, hipStream_t s) {
  const ConvReg& r = a.pl.reg;
  if (r.grid <= 0 || a.M <= 0) return -1;
  const int kind = mode >= kFwdX ? (a.v.sat ? kTrue : a.v.adam ? kAdam : kGrad)
                                 : (a.bt.sw || a.bt.l2x0 || a.e.perr || a.e.psq ? kMargin : kPlain);
  // (a plan made for x* from sign planes is launched as the plain adjoint over
  // an l_p ball's dense rows)
  const reg_fn k = reg_kernel(mode, kind, r.ntw, r.tm, r.np, r.rc);
  if (!k) return -1;
  // (concretisation over an l_p ball writes no sign planes, so any kernel may
  // run it; with the norm's sum the register tiles spill: 95 us against 71
  // subdomain-major, 8 -> 3 channels, 9,216 rows)
  if (mode == kBwdConc && a.bt.l2x0 && a.pl.sd) return -1;
  const int m = a.bt.m, B = a.M / m, mu = conv_unit_rows(B, m, r.grid);
  const dim3 grid((unsigned)std::min<int64_t>((int64_t)B * ((m + mu - 1) / mu), r.grid));
  const int smem = r.smem + (mode == kFwdX && kind == kAdam ? reg_box_bytes(r) : 0);
  launch_k(k, grid, dim3(64 * r.nw), (uint32_t)smem, s, a.in, a.ldi, a.pl, a.M, a.last, a.bt, a.v, a.e, mu);
  return 0;
}

}  // namespace cvb
