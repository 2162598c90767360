// The C ABI of libcvbound: validation, device set-up, pass orchestration,
// HIP-graph capture of the optimisation loop, tile autotuning and profiling.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/cvbound.h"
#include "common.h"
#include "devmem.h"
#include "internal.h"

using namespace cvb;

namespace {

thread_local std::string g_err;

}  // namespace

int cvb::fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

namespace {

inline int r4(int d) { return (d + 3) & ~3; }
inline int r16(int d) { return (d + 15) & ~15; }
inline int r32(int d) { return (d + 31) & ~31; }

// ---------------------------------------------------------------------------
// a handle and its layers

struct DevLayer {
  int type;
  int din, dout;
  ConvGeom g;
  int ld_in, ld_out;       // padded row lengths of W and Wt (dense)
  float* W = nullptr;      // dense [dout, ld_in]; conv OIHW
  float* Wt = nullptr;     // dense [din, ld_out]
  double* W64 = nullptr;   // conv: W in conv64_rows_k's order (sound mode, large batches)
  float* bias = nullptr;   // [dout], per neuron
  ConvPlan bwd{}, fwd{};   // conv: back-substitution and forward implicit GEMMs
  ConvPlan bwd_def{}, fwd_def{};  // the same as first built (before any variant choice)
};

}  // namespace

// A property of the code and the device, asked for once (a query is a few
// microseconds, and every handle of a root pass makes ten of the same).
int cvb::resident_blocks(const void* k, int threads, int smem) {
  static std::mutex mu;
  static std::map<std::tuple<int, const void*, int, int>, int> known;
  int dev = 0, cus = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();
    return -1;
  }
  std::lock_guard<std::mutex> lk(mu);
  const auto it = known.find({dev, k, threads, smem});
  if (it != known.end()) return it->second;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k, threads, smem) != hipSuccess) {
    (void)hipGetLastError();
    return -1;
  }
  return known[{dev, k, threads, smem}] = cus * per;
}

LaunchTiming& cvb::launch_timing() {
  thread_local LaunchTiming t;
  return t;
}

namespace {

struct KStat {
  std::string name;
  double flops = 0, bytes = 0;
  hipEvent_t e0 = nullptr, e1 = nullptr;
};

struct Profiler {
  // Back-to-back launches per timed kernel: spreads the cost of the two event
  // records (a few microseconds) over several launches.
  static constexpr int kRepeat = 8;
  std::vector<KStat> recs;
  hipStream_t s;
  void begin(const std::string& name, double flops, double bytes) {
    KStat k;
    k.name = name;
    k.flops = flops;
    k.bytes = bytes;
    (void)hipEventCreate(&k.e0);
    (void)hipEventCreate(&k.e1);
    // the kernel launched next runs kRepeat times between the two events
    launch_timing() = LaunchTiming{k.e0, k.e1, kRepeat};
    recs.push_back(k);
  }
  void end() {
    LaunchTiming& t = launch_timing();
    if (t.start) {  // nothing was launched (empty range): a zero-length record
      t = LaunchTiming{};
      (void)hipEventRecord(recs.back().e0, s);
      (void)hipEventRecord(recs.back().e1, s);
    }
  }
};

struct GraphKey {
  std::vector<uintptr_t> v;
  bool operator==(const GraphKey& o) const { return v == o.v; }
};

}  // namespace

struct cv_bound {
  DevMem mem;
  // buffers whose size depends on the subdomain batch (rows, alpha entries,
  // splits), sized by capacities that only grow: cv_bound_update reuses them
  // for any batch no larger than one the handle has held
  DevMem bm;
  struct Cap {
    int B = 0;
    int64_t R = 0, na = 0, nnz = 0;
  } bcap;
  int dev = 0;  // the device the handle was built on
  int L = 0;  // layers (ReLU after 1..L-1)
  std::vector<DevLayer> layers;
  std::vector<int> dims;  // d_0..d_L
  std::vector<int> offs;  // ReLU layer offsets in the nd axis
  int P = 0, m = 0, B = 0, R = 0, nd = 0, d0 = 0, w64 = 0;
  int64_t nnz = 0, n_alpha = 0;
  int ldact = 4;
  int n_slots = 1;
  // host copies for queries
  std::vector<int> h_prop;
  std::vector<int64_t> h_aoff;
  std::vector<int> h_cidx;  // [P, nd]
  std::vector<int> h_ucount;
  std::vector<double> unst_rows_per_layer;  // sum over rows of unstable neurons per ReLU layer
  // root classes per property (kind | index in the unstable list) [P, nd], and
  // the unstable count per property and ReLU layer: what a new batch's splits
  // are checked against and its tables built from
  std::vector<uint32_t> h_kind;
  std::vector<std::vector<int>> h_ucount_layer;
  uint32_t* d_kind = nullptr;
  int *d_split_dom = nullptr, *d_split_col = nullptr;
  uint8_t* d_defer = nullptr;  // [nd] 1 on the columns of conv layers (their split steps run after the adjoint)
  bool has_conv = false;
  int8_t* d_side = nullptr;
  char* btab = nullptr;  // the batch's tables (Batch::prop, aoff, sptr, rbase, the splits), one block
  int forced_tiling = -1, forced_conv = -1;  // cv_bound_set_tiling / cv_bound_set_conv_variant
  int forced_tiles = -1;                     // cv_bound_set_conv_tiles
  int parts_req = 0;  // cv_bound_set_parts (0: two sub-batches from kPartsMinRows rows on)
  // device arrays
  Batch bt{};
  float* CW = nullptr;
  int64_t cw_pstride = 0, cb_pstride = 0;
  int ldcw = 4;
  float* Cb = nullptr;
  float* act[2] = {nullptr, nullptr};
  float* part = nullptr;
  // sound mode: per-neuron weights of the rounding-error bound, the bound's
  // per-row partials and its constant for the merged specification
  // the optimiser's fused top layer: where the last adjoint GEMM left
  // Lambda(L-1) (act buffer) and how many partial slots it filled
  int ftop_buf = 0, ftop_slots = 1;
  // l2-ball input sets: centre [P, d0], radius [P], W(1) x0 + b(1) [P, d1],
  // the A(0)^2 partials [n_slots, R] and eps / ||A(0)||_2 per row
  bool l2 = false;
  float *l2x0 = nullptr, *l2eps = nullptr, *wx0 = nullptr, *psq = nullptr, *l2s = nullptr;
  std::vector<float> hl2x0, hl2eps;  // host copies (sound mode's weights are built from them)
  float* x0n = nullptr;              // [P] ||x0_p||_2 rounded up (sound mode over balls)
  float l2fac = 1.f;
  float lpq = 2.f;  // dual exponent q of the balls (2: l2)
  bool sound = false;
  float* sw = nullptr;    // [P, nd]
  float* perr = nullptr;  // [n_slots, R]
  float* err0 = nullptr;  // [P, m]
  float sound_g = 0.f, sound_scale = 1.f;
  // the float64 evaluation of sound mode: root bounds and specification kept
  // on the device, margin weights of the float64 analysis, row buffers
  float *dl = nullptr, *du = nullptr, *dC = nullptr;
  float* sw64 = nullptr;    // [P, nd]
  float* err064 = nullptr;  // [P, m]
  double sg64 = 0.0, scale64 = 1.0, ball64 = 0.0;
  double2* chord64 = nullptr;  // [P, nd] chords in double (large batches)
  double* act64[2] = {nullptr, nullptr};
  double *part64 = nullptr, *perr64 = nullptr, *psq64 = nullptr;  // [L, R]
  // the optimiser in sound mode: each row's best float32 bound so far, the
  // variables of that iterate, and which rows the last evaluation improved
  float *gbest = nullptr, *abest = nullptr, *bbest = nullptr;
  int* improved = nullptr;
  int* ulist = nullptr;
  int64_t* uoff = nullptr;
  // gradient / optimisation buffers (allocated on first use)
  float* acomp = nullptr;
  uint64_t* xpos = nullptr;
  uint64_t* xneg = nullptr;
  float* xdense = nullptr;  // x* per row when the first layer is dense
  int ldx = 0;
  float* g_alpha = nullptr;
  float* g_beta = nullptr;
  float* adam = nullptr;  // [2 n_alpha + 2 n_beta]
  // joint optimisation of intermediate bounds: the adjoint's zbar at
  // upper-chord neurons (passes of the joint state only), and that state
  float* zchord = nullptr;
  struct Joint;
  Joint* joint = nullptr;
  // tile choice per ReLU-layer kernel: [0..L-1] back-substitution of layer i+1,
  // [L..2L-1] adjoint forward of layer i+1
  std::vector<int> cfg;
  // runs of dense layers fused by the chain kernels: the back-substitution
  // chain covers layers L-1 .. chain_lo (with the top ReLU layer), the adjoint
  // chain layers chain_lo+1 .. L-1; chain_b / chain_f select the chain (1) or
  // per-layer kernels (0) for each direction
  int chain_lo = 0;
  int chain_b = 0, chain_f = 0;
  int chain_np = 0, chain_ncw = 0, chain_rb = 0, chain_uw = 0, chain_grid = 0;  // chain geometry (plan_chain)
  // concurrent sub-batches for the optimiser: the subdomains split into
  // nparts contiguous ranges, each its own handle, graph and stream
  struct Inputs;
  std::unique_ptr<Inputs> in;  // host copy of the init arguments, to build parts
  std::vector<cv_bound*> parts;
  std::vector<int> part_dom;  // [nparts + 1] subdomain boundaries
  std::vector<hipStream_t> pstream;
  std::vector<hipEvent_t> pev;  // [nparts + 1]
  // optimisation graph
  hipStream_t cap = nullptr;
  hipGraphExec_t gexec = nullptr;
  GraphKey gkey;
  GraphKey gseen;  // arguments of the last call run without a graph
  Profiler* prof = nullptr;
};

struct cv_bound::Inputs {
  std::vector<cv_layer> layers;
  std::vector<std::vector<float>> w, b;
  int P = 0, m = 0;
  std::vector<float> xlo, xhi, C, l, u;
  std::vector<int32_t> prop;
  std::vector<int64_t> sptr;
  std::vector<int32_t> slayer, sneuron;
  std::vector<int8_t> sside;
};

namespace {

std::mutex g_tune_mu;
std::map<std::tuple<int, int, int, int>, int> g_tune;  // (mode, M, N, K) -> cfg

// Untuned choice.  32x32 tiles keep the chip full at these skinny shapes and
// leave room for four and more waves per SIMD.  Up to 256 columns a second K
// slice in flight pays where the K loop is long against the epilogue and the
// rows do not fill the chip many times over (us, one slice and two: 576 rows,
// 200x200 relaxation 6.4 and 6.1, 9,216 rows 18.0 and 17.6, but 18,432 rows 29.6
// and 30.4; K = 100 at 9,216 rows 13.0 and 13.6; adjoint 48 -> 100 8.3 and 9.5).
// Above, the operands of the epilogue are most of the traffic, and registers for
// them are worth more (relaxation 100 -> 512 at 9,216 rows: 23.9, two slices
// 25.5, 64x64x16 tiles, two waves per SIMD, 31.0).  Concretisation has the box
// alone to read: 64x64 tiles there from two and a half per CU on (16 -> 784 at 9,216
// rows 11.7 against 14.6 with 32x32x32, 100 -> 784 at 18,432 rows 44.8 against
// 51.9; 200 -> 784 at 1,152 rows 11.1 against 9.9).
int gemm_default_cfg(int mode, int M, int N, int K) {
  if (N <= 32) return 5;  // 32x32x16
  if (N <= 256)           // 32x32x32, two slices in flight or one
    return K > 256 || (K > 128 && (M <= 16384 || mode == kBwdConc)) ? 19 : 6;
  const int64_t tiles = (int64_t)((M + 63) / 64) * ((N + 63) / 64);
  return mode == kBwdConc && tiles >= 640 ? 0 : 6;  // 64x64x16, 32x32x32
}

int cfg_for(const cv_bound* h, int mode, int M, int N, int K, int fallback) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  auto it = g_tune.find({mode, M, N, K});
  return it == g_tune.end() ? fallback : it->second;
  (void)h;
}

// GEMM tiling of every dense layer in both directions: `tiling` >= 0 forces
// that one, -1 takes the tuned (else built-in) choice for each layer shape.
void assign_tiles(cv_bound* h, int tiling) {
  const int n_layers = h->L;
  h->cfg.assign(2 * n_layers, -1);
  for (int i = 1; i < n_layers; ++i) {
    if (h->layers[i - 1].type != CV_LAYER_DENSE) continue;
    const int N_b = h->dims[i - 1], K_b = h->dims[i];
    auto cfg = [&](int mode, int N, int K) {
      return tiling >= 0 ? tiling : cfg_for(h, mode, h->R, N, K, gemm_default_cfg(mode, h->R, N, K));
    };
    h->cfg[i - 1] = cfg(i - 1 >= 1 ? kBwdRelax : kBwdConc, N_b, K_b);
    h->cfg[n_layers + i - 1] = cfg(kFwd, K_b, N_b);
  }
}

// Conv kernel variants (conv_plan_variant) per layer shape and direction,
// chosen by cv_bound_autotune: (mode, rows, c_in, h_in, w_in, c_out, k, s, p).
typedef std::tuple<int, int, int, int, int, int, int, int, int> ConvKey;
std::map<ConvKey, int> g_conv_tune;

ConvKey conv_key(int mode, int rows, const ConvGeom& g) {
  return ConvKey{mode, rows, g.ci, g.hi, g.wi, g.co, g.k, g.s, g.p};
}

int conv_mode(int layer_index, bool bwd, bool first_dense) {
  (void)first_dense;
  return bwd ? (layer_index == 0 ? kBwdConc : kBwdRelax) : (layer_index == 0 ? kFwdX : kFwd);
}

// The concretisation and the adjoint's step of a conv first layer share the
// order of the sign planes: both by register tiles, or neither.
void couple_first(DevLayer& d) {
  if (!d.bwd.reg.on || !d.fwd.reg.on) d.bwd.reg.on = d.fwd.reg.on = 0;
}

// Kernel variant of every conv layer in both directions: `forced` >= 0 forces
// that variant where it can run (elsewhere the default), -1 takes the tuned
// choice for each layer shape, else the default plan; h->forced_tiles then puts
// the register tiles on every layer that has them, or on none.
void assign_conv_variants(cv_bound* h, int forced) {
  for (int i = 0; i < h->L; ++i) {
    DevLayer& d = h->layers[i];
    if (d.type != CV_LAYER_CONV2D) continue;
    for (int dir = 0; dir < 2; ++dir) {
      ConvPlan& pl = dir == 0 ? d.bwd : d.fwd;
      pl = dir == 0 ? d.bwd_def : d.fwd_def;
      const int mode = conv_mode(i, dir == 0, false);
      int v = forced;
      if (v < 0) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        auto it = g_conv_tune.find(conv_key(mode, h->R, d.g));
        v = it == g_conv_tune.end() ? -1 : it->second;
      }
      if (v >= 0) (void)conv_plan_variant(mode, pl, v);
      if (h->forced_tiles >= 0) pl.reg.on = h->forced_tiles && pl.reg.grid > 0;
    }
    if (i == 0) couple_first(d);
  }
}

constexpr int kMaxParts = 4;             // concurrent sub-batches of the optimiser, at most
// Default: two sub-batches from this many rows on, whose launches fill each
// other's tails.  One and two, 20 iterations: 784-6x200-10 at 9,216 rows 6.80 and
// 6.06 ms, at 4,608 rows 4.05 and 3.99, at 1,152 rows 2.76 and 3.11; the deep CNN
// (3x32x32, 8 channels), whose launches have long tails no more, at 73,728 rows
// 97.6 and 98.7, at 9,216 rows 14.5 and 15.2.
constexpr int kPartsMinRows = 4096;
constexpr int kChainWidth = 256;         // widest LDS-resident layer of a chain
constexpr int kLdsBytes = 160 * 1024;    // LDS per workgroup on gfx950
constexpr int kChainStaticLds = 64 * 32; // row-info table of the chain kernels (upper bound)

// Chain geometry: np = widest chained operand rounded to 32 (LDS pitch) and
// ncw rounded to 16 (output chunk); the rows divided
// evenly over one workgroup per compute unit, each padded to rb 16-row blocks
// (at most kChainRowBlocks, else more workgroups than CUs).  Returns false when it does not
// fit the LDS or the per-wave unit registers.
bool plan_chain(cv_bound* h) {
  int wmax = 4;
  for (int i = h->chain_lo; i <= h->L - 1; ++i) wmax = std::max(wmax, h->dims[i]);
  const int np = (wmax + 31) & ~31, ncw = (wmax + 15) & ~15;
  int dev = 0, ncu = 0, lds = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu <= 0)
    ncu = 256;
  if (hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || lds <= 0)
    lds = 64 * 1024;
  lds = std::min(lds, kLdsBytes);
  const int R = std::max(1, h->R);
  int grid = std::min(ncu, R);
  int rb = ((R + grid - 1) / grid + 15) / 16;
  if (rb > kChainRowBlocks) {
    rb = kChainRowBlocks;
    grid = (R + 16 * rb - 1) / (16 * rb);
  }
  if (!chain_units_fit(rb, np, ncw) || chain_smem_bytes(rb, np) + kChainStaticLds > (size_t)lds) return false;
  chain_prepare(lds - kChainStaticLds);
  h->chain_np = np;
  h->chain_rb = rb;
  h->chain_ncw = ncw;
  h->chain_uw = chain_units_per_wave(rb, ncw);
  h->chain_grid = grid;
  return true;
}

// ---------------------------------------------------------------------------
// conv layers as implicit GEMMs (ConvPlan; the kernels are in conv.hip)

constexpr int kFar = -(1 << 20);  // an offset that puts any gather or output outside its plane

struct HostPlan {
  std::vector<int4> mt, kt, nt;
  std::vector<int> ku;  // the uniform per-step part of kt (empty: kt does not split)
  std::vector<float> wm;
  ConvPlan p{};
  int M = 0, K = 0;  // GEMM rows and columns before padding
};

// Pad the tables to whole tiles and lay out Wm (value wv(k, n) for k < K,
// n < N) in MFMA operand order.
template <class F>
void plan_pad(HostPlan& o, int M, int K, int N, F wv) {
  ConvPlan& p = o.p;
  o.M = M;
  o.K = K;
  p.mpad = r16(M);
  p.kpad = r16(K);  // the kernel takes four K steps of 4 per pass
  const int tiles = (N + 15) / 16;
  p.nt = tiles <= 1 ? 1 : tiles <= 2 ? 2 : tiles <= 4 ? 4 : 8;
  o.mt.resize(p.mpad, make_int4(kFar, kFar, kFar, kFar));
  o.kt.resize(p.kpad, make_int4(kFar, kFar, 0, 0));
  o.nt.resize(p.nt * 16, make_int4(0, 0, -1, 0));
  o.wm.assign((size_t)p.kpad * p.nt * 16, 0.f);
  for (int ks = 0; ks < p.kpad / 4; ++ks)
    for (int t = 0; t < p.nt; ++t)
      for (int l = 0; l < 64; ++l) {
        const int k = ks * 4 + l / 16, n = t * 16 + l % 16;
        if (k < K && n < N) o.wm[((size_t)ks * p.nt + t) * 64 + l] = wv(k, n);
      }
}

// The split kt[4 s + q] = ku[s] + v(q) of the column offsets (v(q) = kt[q] -
// kt[0], ku[s] = kt[4 s]), when every real column obeys it and every padding
// column's tap, so placed, stays inside the staged row for every GEMM row
// (a padding column has zero weights, so any tap in range will do); else
// ku stays empty and the kernels read kt.
void plan_uniform(HostPlan& o) {
  const ConvPlan& p = o.p;
  o.ku.clear();
  if (o.K < 4) return;
  int v[4], m0 = INT32_MAX, m1 = INT32_MIN;
  for (int q = 0; q < 4; ++q) v[q] = o.kt[q].x - o.kt[0].x;
  for (int m = 0; m < p.mpad; ++m) {
    m0 = std::min(m0, o.mt[m].x);
    m1 = std::max(m1, o.mt[m].x);
  }
  std::vector<int> ku(p.kpad / 4);
  for (int s = 0; s < p.kpad / 4; ++s) {
    ku[s] = 4 * s < o.K ? o.kt[4 * s].x : ku[0];
    for (int q = 0; q < 4; ++q) {
      const int kk = 4 * s + q, off = ku[s] + v[q];
      if (kk < o.K ? o.kt[kk].x != off : (m0 + off < 0 || m1 + off >= p.dinp)) return;
    }
  }
  o.ku = ku;
}

// Turn the gather tables (row origin (y, x) in mt, column offset (dy, dx)
// and channel base in kt) into flat offsets into the staged row, whose
// channel planes get a zero border wide enough for every tap the GEMM reads.
void plan_border(HostPlan& o) {
  ConvPlan& p = o.p;
  const int plane = p.gh * p.gw, C = p.din / plane;
  int y0 = INT32_MAX, y1 = INT32_MIN, x0 = INT32_MAX, x1 = INT32_MIN, dy0 = INT32_MAX, dy1 = INT32_MIN,
      dx0 = INT32_MAX, dx1 = INT32_MIN;
  for (int m = 0; m < o.M; ++m) {
    y0 = std::min(y0, o.mt[m].x);
    y1 = std::max(y1, o.mt[m].x);
    x0 = std::min(x0, o.mt[m].y);
    x1 = std::max(x1, o.mt[m].y);
  }
  for (int k = 0; k < o.K; ++k) {
    dy0 = std::min(dy0, o.kt[k].x);
    dy1 = std::max(dy1, o.kt[k].x);
    dx0 = std::min(dx0, o.kt[k].y);
    dx1 = std::max(dx1, o.kt[k].y);
  }
  const int bly = std::max(0, -(y0 + dy0)), bhy = std::max(0, y1 + dy1 - (p.gh - 1));
  const int blx = std::max(0, -(x0 + dx0)), bhx = std::max(0, x1 + dx1 - (p.gw - 1));
  p.gwp = p.gw + blx + bhx;
  p.pplane = (p.gh + bly + bhy) * p.gwp;
  p.bofs = bly * p.gwp + blx;
  p.dinp = C * p.pplane;
  p.mgp = (unsigned)((((uint64_t)1 << 32) + plane - 1) / plane);
  p.mgw = (unsigned)((((uint64_t)1 << 32) + p.gw - 1) / p.gw);
  const int4 e0 = o.mt[0];
  for (int m = 0; m < p.mpad; ++m) {  // padding rows reuse row 0's window
    const int4 e = m < o.M ? o.mt[m] : e0;
    o.mt[m] = make_int4((e.x + bly) * p.gwp + (e.y + blx), 0, o.mt[m].z, o.mt[m].w);
  }
  for (int k = 0; k < p.kpad; ++k) {  // padding columns (zero weights) read row m's own origin
    const int4 e = o.kt[k];
    o.kt[k] = make_int4(k < o.K ? (e.z / plane) * p.pplane + e.x * p.gwp + e.y : 0, 0, 0, 0);
  }
  plan_uniform(o);
}

// Column n of a paired plan (two horizontally adjacent outputs x = 2 X + px
// per GEMM row, c channels): its (px, channel).  With 8 channels the columns
// go in groups of four, px alternating between groups -- (px 0, ch 0-3),
// (px 1, ch 0-3), (px 0, ch 4-7), (px 1, ch 4-7) -- so the 32 lanes that
// store two neighbouring column groups of a transposed MFMA tile write the
// two parities of a position: even and odd LDS banks.
inline void pair_col(int n, int c, int& px, int& ch) {
  if (c == 8) {
    px = (n >> 2) & 1;
    ch = (n & 3) | ((n >> 3) << 2);
  } else {
    px = n / c;
    ch = n % c;
  }
}

// Back-substitution through conv layer ly (transposed convolution), polyphase
// form: GEMM rows (Y, X), columns (py, px, ci), K = (co, a, b).  A stride-1
// layer with c_in <= 8 folds output pairs x = 2 X + px into a row instead:
// columns (px, ci), K = (co, a, b') with b' = kx - px in [-1, k).
void plan_convt(const cv_layer& ly, HostPlan& o) {
  const int s = ly.stride, k = ly.kernel, pad = ly.pad, ci = ly.in_c, hi = ly.in_h, wi = ly.in_w;
  const int co = ly.out_c, ho = ly.out_h, wo = ly.out_w, am = (k + s - 1) / s;
  ConvPlan& p = o.p;
  p.gh = ho;
  p.gw = wo;
  p.oh = hi;
  p.ow = wi;
  p.din = co * ho * wo;
  p.dout = ci * hi * wi;
  if (s == 1 && ci <= 8) {
    const int nX = (wi + 1) / 2, kb = k + 1, M = hi * nX, K = co * k * kb, N = 2 * ci;
    plan_pad(o, M, K, N, [&](int kk, int n) {
      int px, c;
      pair_col(n, ci, px, c);
      const int c_o = kk / (k * kb), a = (kk / kb) % k, kx = kk % kb - 1 + px;
      return kx >= 0 && kx < k ? ly.weight[(((size_t)c_o * ci + c) * k + a) * k + kx] : 0.f;
    });
    for (int m = 0; m < M; ++m) o.mt[m] = make_int4(m / nX + pad, 2 * (m % nX) + pad, m / nX + pad, m % nX);
    for (int kk = 0; kk < K; ++kk) o.kt[kk] = make_int4(-((kk / kb) % k), 1 - kk % kb, (kk / (k * kb)) * ho * wo, 0);
    for (int n = 0; n < N; ++n) {
      int px, c;
      pair_col(n, ci, px, c);
      o.nt[n] = make_int4(-pad, px, c * hi * wi, 0);
    }
    p.osy = 1;
    p.osx = 2;
    plan_border(o);
    return;
  }
  std::vector<int> k0(s), T(s);
  for (int c = 0; c < s; ++c) {
    k0[c] = (c + pad) % s;
    T[c] = (c + pad - k0[c]) / s;
  }
  auto range = [&](int n, int& lo, int& up) {
    lo = INT32_MAX;
    up = INT32_MIN;
    for (int y = 0; y < n; ++y) {
      const int Y = y / s + T[y % s];
      lo = std::min(lo, Y);
      up = std::max(up, Y);
    }
  };
  int y0, y1, x0, x1;
  range(hi, y0, y1);
  range(wi, x0, x1);
  const int nX = x1 - x0 + 1, M = (y1 - y0 + 1) * nX, K = co * am * am, N = s * s * ci;
  plan_pad(o, M, K, N, [&](int kk, int n) {
    const int c_o = kk / (am * am), a = (kk / am) % am, b = kk % am;
    const int cls = n / ci, c = n % ci, py = cls / s, px = cls % s;
    const int ky = k0[py] + s * a, kx = k0[px] + s * b;
    return ky < k && kx < k ? ly.weight[(((size_t)c_o * ci + c) * k + ky) * k + kx] : 0.f;
  });
  for (int m = 0; m < M; ++m) {
    const int Y = y0 + m / nX, X = x0 + m % nX;
    o.mt[m] = make_int4(Y, X, Y, X);
  }
  for (int kk = 0; kk < K; ++kk)
    o.kt[kk] = make_int4(-((kk / am) % am), -(kk % am), (kk / (am * am)) * ho * wo, 0);
  for (int n = 0; n < N; ++n) {
    const int cls = n / ci, c = n % ci, py = cls / s, px = cls % s;
    o.nt[n] = make_int4(py - s * T[py], px - s * T[px], c * hi * wi, 0);
  }
  p.osy = s;
  p.osx = s;
  plan_border(o);
}

// The forward convolution of ly: GEMM rows (oy, ox), K = (ci, ky, kx), N = co;
// with c_out <= 8, output pairs ox = 2 X + px share a row: columns (px, co),
// K = (ci, ky, kx') with kx' = kx + s px in [0, k + s).
void plan_conv(const cv_layer& ly, HostPlan& o) {
  const int s = ly.stride, k = ly.kernel, pad = ly.pad, ci = ly.in_c, hi = ly.in_h, wi = ly.in_w;
  const int co = ly.out_c, ho = ly.out_h, wo = ly.out_w;
  ConvPlan& p = o.p;
  p.gh = hi;
  p.gw = wi;
  p.oh = ho;
  p.ow = wo;
  p.din = ci * hi * wi;
  p.dout = co * ho * wo;
  p.osy = 1;
  if (co <= 8) {
    const int nX = (wo + 1) / 2, kf = k + s, M = ho * nX, K = ci * k * kf;
    // K index kk -> (c, ky, kx'); with k a multiple of 4 the order is (kx', c,
    // ky), ky innermost, so that the column offsets split into a per-step and
    // a per-lane part (plan_uniform); otherwise (c, ky, kx')
    const bool ky_in = k % 4 == 0;
    auto kdec = [&](int kk, int& c, int& ky, int& kx) {
      if (ky_in) {
        ky = kk % k;
        c = (kk / k) % ci;
        kx = kk / (k * ci);
      } else {
        c = kk / (k * kf);
        ky = (kk / kf) % k;
        kx = kk % kf;
      }
    };
    plan_pad(o, M, K, 2 * co, [&](int kk, int n) {
      int px, c_o, c, ky, kxf;
      pair_col(n, co, px, c_o);
      kdec(kk, c, ky, kxf);
      const int kx = kxf - px * s;
      return kx >= 0 && kx < k ? ly.weight[(((size_t)c_o * ci + c) * k + ky) * k + kx] : 0.f;
    });
    for (int m = 0; m < M; ++m) {
      const int oy = m / nX, X = m % nX;
      o.mt[m] = make_int4(oy * s - pad, 2 * X * s - pad, oy, X);
    }
    for (int kk = 0; kk < K; ++kk) {
      int c, ky, kxf;
      kdec(kk, c, ky, kxf);
      o.kt[kk] = make_int4(ky, kxf, c * hi * wi, 0);
    }
    for (int n = 0; n < 2 * co; ++n) {
      int px, c_o;
      pair_col(n, co, px, c_o);
      o.nt[n] = make_int4(0, px, c_o * ho * wo, 0);
    }
    p.osx = 2;
    plan_border(o);
    return;
  }
  const int M = ho * wo, K = ci * k * k;
  plan_pad(o, M, K, co, [&](int kk, int n) { return ly.weight[(size_t)n * K + kk]; });
  for (int m = 0; m < M; ++m) {
    const int oy = m / wo, ox = m % wo;
    o.mt[m] = make_int4(oy * s - pad, ox * s - pad, oy, ox);
  }
  for (int kk = 0; kk < K; ++kk) o.kt[kk] = make_int4((kk / k) % k, kk % k, (kk / (k * k)) * hi * wi, 0);
  for (int n = 0; n < co; ++n) o.nt[n] = make_int4(0, 0, n * ho * wo, 0);
  p.osx = 1;
  plan_border(o);
}

// The register-tile kernel's tables of a built plan (ConvReg): its columns
// reordered, the weights four K steps together.  col(t, g, r): the plan's
// column there, or -1.  Empty tables where the layer has no such order.
struct HostReg {
  std::vector<int4> ob;
  std::vector<float4> w4;
  std::vector<int2> xt;
  ConvReg r{};
};

void plan_reg(const cv_layer& ly, bool bwd, const HostPlan& o, HostReg& q) {
  const ConvPlan& p = o.p;
  const int C = bwd ? ly.in_c : ly.out_c, s = ly.stride;
  const bool poly = bwd && s == 2, pair = C <= 8 && (!bwd || s == 1);
  if (bwd && s > 2) return;
  ConvReg& r = q.r;
  r.plane = p.oh * p.ow;
  r.ts = poly ? 4 : 16;
  const int tiles = poly ? (C + 3) / 4 : pair ? 1 : (C + 15) / 16;
  r.nt = tiles <= 1 ? 1 : tiles <= 2 ? 2 : tiles <= 4 ? 4 : 8;
  if (tiles > 8) return;
  r.n_mt = p.mpad / 16;
  r.ksp = 1;
  auto column = [&](int t, int g, int rr) -> int {
    if (poly) return 4 * t + rr < C ? g * C + 4 * t + rr : -1;
    if (!pair) return 16 * t + 4 * g + rr < C ? 16 * t + 4 * g + rr : -1;
    for (int n = 0; n < 2 * C; ++n) {
      int px, ch;
      pair_col(n, C, px, ch);
      if (px == (g & 1) && ch == rr + 4 * (g >> 1)) return n;
    }
    return -1;
  };
  int cols[8 * 16];
  r.rc = 0;
  for (int t = 0; t < r.nt; ++t)
    for (int g = 0; g < 4; ++g)
      for (int rr = 0; rr < 4; ++rr) {
        const int n = cols[t * 16 + g * 4 + rr] = column(t, g, rr);
        if (n >= 0) r.rc = std::max(r.rc, rr + 1);
      }
  auto col = [&](int t, int g, int rr) { return cols[t * 16 + g * 4 + rr]; };
  r.rc = r.rc <= 3 ? 3 : 4;  // (the kernel's instances)
  r.nwords = r.n_mt * r.nt * r.rc;
  q.ob.resize((size_t)r.n_mt * 64);
  for (int m = 0; m < r.n_mt * 16; ++m)
    for (int g = 0; g < 4; ++g) {
      const int4 mo = o.mt[m];
      int at = -1;
      const int n = col(0, g, 0);
      if (n >= 0 && m < o.M) {
        const int4 ne = o.nt[n];
        const int y = p.osy * mo.z + ne.x, x = p.osx * mo.w + ne.y;
        if (y >= 0 && y < p.oh && x >= 0 && x < p.ow) at = ne.z + y * p.ow + x;
      }
      q.ob[(size_t)(m / 16) * 64 + g * 16 + m % 16] = make_int4(mo.x, at, 0, 0);
    }
  auto wv = [&](int k, int n) { return n < 0 ? 0.f : o.wm[((size_t)(k / 4) * p.nt + n / 16) * 64 + (k % 4) * 16 + n % 16]; };
  q.w4.resize((size_t)(p.kpad / 16) * r.nt * 64);
  for (int ps = 0; ps < p.kpad / 16; ++ps)
    for (int t = 0; t < r.nt; ++t)
      for (int l = 0; l < 64; ++l) {
        const int n = col(t, (l % 16) / 4, l % 4), k = ps * 16 + l / 16;
        q.w4[((size_t)ps * r.nt + t) * 64 + l] = make_float4(wv(k, n), wv(k + 4, n), wv(k + 8, n), wv(k + 12, n));
      }
}

// Weight placement and LDS bytes of a built plan.
void plan_finish(ConvPlan& p) {
  // a weight matrix over 16 KB stays in global memory (more workgroups fit per CU)
  p.wg = (size_t)p.kpad * p.nt * 16 * sizeof(float) > 16384 ? 1 : 0;
  p.smem = conv_plan_smem(p);
}

// Whether both implicit GEMMs of conv layer ly fit the LDS a workgroup uses.
bool conv_fits_lds(const cv_layer& ly) {
  HostPlan pb, pf;
  plan_convt(ly, pb);
  plan_conv(ly, pf);
  plan_finish(pb.p);
  plan_finish(pf.p);
  return pb.p.smem <= 65536 && pf.p.smem <= 65536;
}

// ---------------------------------------------------------------------------
// validation

int check_layers(const cv_layer* layers, int n, std::vector<int>& dims, bool allow_conv_last = false) {
  if (!layers || n < 1) return fail(CV_EINVAL, "need at least one layer");
  dims.assign(n + 1, 0);
  for (int i = 0; i < n; ++i) {
    const cv_layer& ly = layers[i];
    if (!ly.weight || !ly.bias) return fail(CV_EINVAL, "layer %d: null weight or bias", i + 1);
    const int64_t din = (int64_t)ly.in_c * ly.in_h * ly.in_w;
    const int64_t dout = (int64_t)ly.out_c * ly.out_h * ly.out_w;
    if (ly.in_c <= 0 || ly.in_h <= 0 || ly.in_w <= 0 || ly.out_c <= 0 || ly.out_h <= 0 || ly.out_w <= 0 ||
        din > (1 << 24) || dout > (1 << 24))
      return fail(CV_ESHAPE, "layer %d: bad sizes", i + 1);
    if (ly.type == CV_LAYER_CONV2D) {
      if (ly.kernel <= 0 || ly.stride <= 0 || ly.pad < 0) return fail(CV_ESHAPE, "layer %d: bad conv geometry", i + 1);
      if ((ly.in_h + 2 * ly.pad - ly.kernel) / ly.stride + 1 != ly.out_h ||
          (ly.in_w + 2 * ly.pad - ly.kernel) / ly.stride + 1 != ly.out_w)
        return fail(CV_ESHAPE, "layer %d: conv output size does not match", i + 1);
      // the implicit GEMMs' N axes: stride^2 c_in columns (back-substitution), c_out (forward)
      if (ly.stride > 8 || (int64_t)ly.stride * ly.stride * ly.in_c > 128 || ly.out_c > 128)
        return fail(CV_ESHAPE, "layer %d: stride^2 * c_in and c_out must be at most 128", i + 1);
      if (i < n - 1 && !conv_fits_lds(ly))
        return fail(CV_ESHAPE, "layer %d: conv rows and weights do not fit in LDS", i + 1);
      if (i == n - 1 && !allow_conv_last) return fail(CV_ESHAPE, "the last layer must be dense");
    } else if (ly.type != CV_LAYER_DENSE) {
      return fail(CV_ESHAPE, "layer %d: unknown type %d", i + 1, ly.type);
    }
    if (i == 0) dims[0] = (int)din;
    else if (din != dims[i]) return fail(CV_ESHAPE, "layer %d: input size %lld does not match %d", i + 1, (long long)din, dims[i]);
    dims[i + 1] = (int)dout;
  }
  return CV_OK;
}

bool finite_all(const float* p, int64_t n) {
  for (int64_t i = 0; i < n; ++i)
    if (!std::isfinite(p[i])) return false;
  return true;
}

// The tables of a plan, in one allocation and copy.
int upload_plan(cv_bound* h, HostPlan& o, HostReg& hr, int mode, ConvPlan& out) {
  std::vector<int4> all;
  auto put = [&](const void* src, size_t bytes) {
    const size_t at = all.size();
    all.resize(at + (bytes + 15) / 16, make_int4(0, 0, 0, 0));
    if (bytes) std::memcpy(&all[at], src, bytes);
    return at;
  };
  const size_t mt = put(o.mt.data(), o.mt.size() * sizeof(int4)), kt = put(o.kt.data(), o.kt.size() * sizeof(int4)),
               nt = put(o.nt.data(), o.nt.size() * sizeof(int4)), ku = put(o.ku.data(), o.ku.size() * sizeof(int)),
               wm = put(o.wm.data(), o.wm.size() * sizeof(float)), ob = put(hr.ob.data(), hr.ob.size() * sizeof(int4)),
               w4 = put(hr.w4.data(), hr.w4.size() * sizeof(float4)), xt = put(hr.xt.data(), hr.xt.size() * sizeof(int2));
  int4* d = nullptr;
  int rc;
  if ((rc = h->mem.upload(&d, all.data(), all.size(), nullptr))) return rc;
  out = o.p;
  out.mtab = d + mt;
  out.ktab = d + kt;
  out.ntab = d + nt;
  out.kuni = o.ku.empty() ? nullptr : reinterpret_cast<const int*>(d + ku);
  out.wm = reinterpret_cast<const float*>(d + wm);
  plan_finish(out);
  out.grid = conv_plan_grid(mode, out);
  conv_plan_sd(mode, out);
  if (hr.ob.empty()) return CV_OK;
  out.reg = hr.r;
  out.reg.ob = d + ob;
  out.reg.w4 = reinterpret_cast<const float4*>(d + w4);
  out.reg.xt = hr.xt.empty() ? nullptr : reinterpret_cast<const int2*>(d + xt);
  // a narrow output plane with a long K: the subdomain-major kernel splits the
  // K passes over its idle waves; the same chunks here, so that every variant
  // of the default path rounds alike
  if (out.sd && out.nj <= 2) {
    int& k = out.reg.ksp;
    while (2 * k * (out.mpad >> 4) <= 8 && 2 * k <= (out.kpad >> 4)) k *= 2;
  }
  conv_plan_reg(mode, out);
  out.reg.on = out.reg.grid > 0 && out.reg.prefer;
  return CV_OK;
}

// Where bit `lane` of each word of the register-tile sign planes lies in the
// staged input row of the forward plan pf, and which input it is (lanes
// without an input: the spare slot).
std::vector<int2> sign_slots(const ConvReg& r, const std::vector<int4>& ob, const ConvPlan& pf) {
  std::vector<int2> xt((size_t)r.nwords * 64, make_int2(pf.dinp, 0));
  const int plane = pf.gh * pf.gw;
  for (int mt = 0; mt < r.n_mt; ++mt)
    for (int t = 0; t < r.nt; ++t)
      for (int rr = 0; rr < r.rc; ++rr)
        for (int l = 0; l < 64; ++l) {
          const int b = ob[(size_t)mt * 64 + l].y;
          const int64_t j = b + (int64_t)r.plane * (rr + r.ts * t);
          if (b < 0 || j >= pf.din) continue;
          const int c = (int)(j / plane), y = (int)(j % plane) / pf.gw, x = (int)(j % plane) % pf.gw;
          xt[(((size_t)mt * r.nt + t) * r.rc + rr) * 64 + l] =
              make_int2(c * pf.pplane + pf.bofs + y * pf.gwp + x, (int)j);
        }
  return xt;
}

// Build the layer copies on the device.
int upload_layers(cv_bound* h, const cv_layer* layers, int n, hipStream_t s) {
  h->layers.resize(n);
  for (int i = 0; i < n; ++i) {
    const cv_layer& ly = layers[i];
    DevLayer& d = h->layers[i];
    d.type = ly.type;
    d.din = h->dims[i];
    d.dout = h->dims[i + 1];
    d.g = ConvGeom{ly.in_c, ly.in_h, ly.in_w, ly.out_c, ly.out_h, ly.out_w, ly.kernel, ly.stride, ly.pad};
    std::vector<float> bias_full(d.dout);
    if (ly.type == CV_LAYER_DENSE) {
      // zero padding: rows to multiples of 16 and the K (contiguous) axis to
      // multiples of 32, so MFMA tiles read whole blocks (and k-chunk pairs)
      // without masks
      d.ld_in = r32(d.din);
      d.ld_out = r32(d.dout);
      std::vector<float> W((size_t)r16(d.dout) * d.ld_in, 0.f), Wt((size_t)r16(d.din) * d.ld_out, 0.f);
      for (int o = 0; o < d.dout; ++o)
        for (int j = 0; j < d.din; ++j) {
          const float w = ly.weight[(size_t)o * d.din + j];
          W[(size_t)o * d.ld_in + j] = w;
          Wt[(size_t)j * d.ld_out + o] = w;
        }
      int rc = h->mem.upload(&d.W, W.data(), W.size(), s);
      if (rc) return rc;
      rc = h->mem.upload(&d.Wt, Wt.data(), Wt.size(), s);
      if (rc) return rc;
      for (int o = 0; o < d.dout; ++o) bias_full[o] = ly.bias[o];
    } else {
      const size_t nw = (size_t)ly.out_c * ly.in_c * ly.kernel * ly.kernel;
      int rc = h->mem.upload(&d.W, ly.weight, nw, s);
      if (rc) return rc;
      const int pos = ly.out_h * ly.out_w;
      for (int o = 0; o < d.dout; ++o) bias_full[o] = ly.bias[o / pos];
      if (!finite_all(ly.weight, (int64_t)nw)) return fail(CV_EINVAL, "layer %d: non-finite weight", i + 1);
      HostPlan pb, pf;
      plan_convt(ly, pb);
      plan_conv(ly, pf);
      HostReg rb, rf;
      plan_reg(ly, true, pb, rb);
      plan_reg(ly, false, pf, rf);
      if ((rc = upload_plan(h, pb, rb, i == 0 ? kBwdConc : kBwdRelax, d.bwd))) return rc;
      if (i == 0) {
        // the first layer's adjoint step reads the sign planes in the order
        // the concretisation's register tiles write them
        rf.r.nwords = 0;
        if (d.bwd.reg.grid > 0 && !rf.ob.empty()) {
          rf.xt = sign_slots(d.bwd.reg, rb.ob, pf.p);
          rf.r.nwords = rb.r.nwords;
          h->w64 = std::max(h->w64, rb.r.nwords);
        }
      }
      if ((rc = upload_plan(h, pf, rf, i == 0 ? kFwdX : kFwd, d.fwd))) return rc;
      if (i == 0) couple_first(d);
      d.bwd_def = d.bwd;
      d.fwd_def = d.fwd;
    }
    if (ly.type == CV_LAYER_DENSE && !finite_all(ly.weight, (int64_t)d.dout * d.din))
      return fail(CV_EINVAL, "layer %d: non-finite weight", i + 1);
    if (!finite_all(ly.bias, ly.out_c)) return fail(CV_EINVAL, "layer %d: non-finite bias", i + 1);
    int rc = h->mem.upload(&d.bias, bias_full.data(), bias_full.size(), s);
    if (rc) return rc;
  }
  return CV_OK;
}

// Spec source for build(): host C, or the identity [I; -I] on the last layer.
struct Spec {
  const float* C = nullptr;  // [P, m, dL] host
  bool identity = false;
};

// Every buffer of the batch pool dropped (their contents are per batch).
void release_batch(cv_bound* h) {
  h->bm.clear();
  h->act[0] = h->act[1] = nullptr;
  h->act64[0] = h->act64[1] = nullptr;
  for (float** p : {&h->part, &h->acomp, &h->xdense, &h->g_alpha, &h->g_beta, &h->adam, &h->perr, &h->gbest,
                    &h->abest, &h->bbest, &h->psq, &h->l2s, &h->zchord})
    *p = nullptr;
  for (double** p : {&h->part64, &h->perr64, &h->psq64}) *p = nullptr;
  h->xpos = h->xneg = nullptr;
  h->improved = nullptr;
  h->d_split_dom = h->d_split_col = nullptr;
  h->d_side = nullptr;
  h->btab = nullptr;
  h->bt.prop = nullptr;
  h->bt.aoff = h->bt.rbase = h->bt.sptr = nullptr;
  h->bt.status = nullptr;
  h->bcap = cv_bound::Cap{};
}

// A subdomain batch checked on the host (Sec. 3.4: independent subdomains
// bounded together): splits against each property's root-unstable neurons,
// and the tables the device needs.  Touches no device state.
struct BatchPlan {
  int B = 0;
  int64_t R = 0, nnz = 0, n_alpha = 0;
  const int32_t* dom_prop = nullptr;
  const int64_t* split_ptr = nullptr;
  const int8_t* split_side = nullptr;
  std::vector<int> split_dom, split_col;
  std::vector<int64_t> aoff;
  std::vector<double> unst;
};

int check_batch(const cv_bound* h, int B, const int32_t* dom_prop, const int64_t* split_ptr,
                const int32_t* split_layer, const int32_t* split_neuron, const int8_t* split_side, BatchPlan& bp) {
  const int P = h->P, nd = h->nd, m = h->m, n_layers = h->L;
  if (B < 0) return fail(CV_EINVAL, "n_dom must be >= 0");
  if (!split_ptr || (!dom_prop && B > 0)) return fail(CV_EINVAL, "null input pointer");
  const int64_t R = (int64_t)B * m;
  if (R > (1ll << 30)) return fail(CV_EINVAL, "too many rows (%lld)", (long long)R);
  if (split_ptr[0] != 0) return fail(CV_ESPLIT, "split_ptr[0] must be 0");
  const int64_t nnz = B > 0 ? split_ptr[B] : 0;
  if (nnz > 0 && (!split_layer || !split_neuron || !split_side)) return fail(CV_EINVAL, "null split arrays");
  bp.split_dom.assign(nnz, 0);
  bp.split_col.assign(nnz, 0);
  bp.aoff.assign(B + 1, 0);
  bp.unst.assign(std::max(1, n_layers - 1), 0.0);
  std::vector<int> seen(nd, -1);
  for (int b = 0; b < B; ++b) {
    const int p = dom_prop[b];
    if (p < 0 || p >= P) return fail(CV_EINVAL, "subdomain %d: property %d out of range", b, p);
    bp.aoff[b + 1] = bp.aoff[b] + (int64_t)m * h->h_ucount[p];
    for (int li = 0; li + 1 < n_layers; ++li) bp.unst[li] += (double)m * h->h_ucount_layer[p][li];
    const int64_t s0 = split_ptr[b], s1 = split_ptr[b + 1];
    if (s1 < s0) return fail(CV_ESPLIT, "subdomain %d: split_ptr decreases", b);
    if (s1 >= kMaxSplits) return fail(CV_ESPLIT, "more than %lld splits in total", (long long)kMaxSplits - 1);
    for (int64_t t = s0; t < s1; ++t) {
      const int ly = split_layer[t], nr = split_neuron[t];
      if (ly < 1 || ly >= n_layers) return fail(CV_ESPLIT, "split %lld: layer %d out of range", (long long)t, ly);
      if (nr < 0 || nr >= h->dims[ly]) return fail(CV_ESPLIT, "split %lld: neuron %d out of range", (long long)t, nr);
      if (split_side[t] != 1 && split_side[t] != -1)
        return fail(CV_ESPLIT, "split %lld: side must be +1 or -1", (long long)t);
      const int col = h->offs[ly - 1] + nr;
      if ((h->h_kind[(size_t)p * nd + col] & kKindMask) != kUnstable)
        return fail(CV_ESPLIT, "split %lld: neuron (%d,%d) is not root-unstable", (long long)t, ly, nr);
      if (seen[col] == b) return fail(CV_ESPLIT, "subdomain %d splits neuron (%d,%d) twice", b, ly, nr);
      seen[col] = b;
      bp.split_dom[t] = b;
      bp.split_col[t] = col;
    }
  }
  bp.B = B;
  bp.R = R;
  bp.nnz = nnz;
  bp.n_alpha = bp.aoff[B];
  bp.dom_prop = dom_prop;
  bp.split_ptr = split_ptr;
  bp.split_side = split_side;
  return CV_OK;
}

// The checked batch made h's (the caller's arrays must still be live): row and
// alpha tables, CSR split arrays, status words.  Batch-sized buffers live in
// h->bm; when the batch needs more than the pool holds the pool is
// reallocated, sized for this batch (grow: with a quarter to spare, for
// batches that grow round by round), else reused.
int set_batch(cv_bound* h, const BatchPlan& bp, bool grow, hipStream_t s) {
  const int nd = h->nd, m = h->m, n_layers = h->L;
  const int B = bp.B;
  const int64_t R = bp.R, nnz = bp.nnz;
  const int32_t* dom_prop = bp.dom_prop;
  const int64_t* split_ptr = bp.split_ptr;
  const int8_t* split_side = bp.split_side;
  const std::vector<int64_t>& aoff = bp.aoff;
  const std::vector<int>& split_dom = bp.split_dom;
  const std::vector<int>& split_col = bp.split_col;
  // ---- commit
  h->B = B;
  h->R = (int)R;
  h->nnz = nnz;
  h->h_prop.assign(dom_prop, dom_prop + B);
  h->h_aoff = aoff;
  h->n_alpha = bp.n_alpha;
  h->unst_rows_per_layer = bp.unst;
  int rc;
  cv_bound::Cap& c = h->bcap;
  if (B > c.B || R > c.R || h->n_alpha > c.na || nnz > c.nnz || !h->bt.status) {
    HIPCHK(hipStreamSynchronize(s));
    HIPCHK(hipDeviceSynchronize());  // every stream of the handle is done with the old buffers
    release_batch(h);
    auto sz = [&](int64_t n) { return grow ? n + n / 4 : n; };
    c.B = (int)sz(B);
    c.R = sz(R);
    c.na = sz(h->n_alpha);
    c.nnz = sz(nnz);
    DevMem& M = h->bm;
    uint32_t* d_status;
    // the tables lie one after the other, each from a 16-byte boundary
    if ((rc = M.alloc(&h->btab, sizeof(int) * (size_t)c.B + 2 * sizeof(int64_t) * ((size_t)c.B + 1) +
                                    sizeof(int64_t) * (size_t)c.R + (2 * sizeof(int) + 1) * (size_t)c.nnz + 7 * 16)) ||
        (rc = M.alloc(&d_status, (size_t)c.B * nd)) || (rc = M.alloc(&h->part, (size_t)std::max<int64_t>(1, c.R) * h->n_slots)))
      return rc;
    if (n_layers >= 2 && ((rc = M.alloc(&h->act[0], (size_t)c.R * h->ldact)) ||
                          (rc = M.alloc(&h->act[1], (size_t)c.R * h->ldact))))
      return rc;
    h->bt.status = d_status;
  }
  std::vector<int64_t> rbase((size_t)R);
  for (int b = 0; b < B; ++b)
    for (int k = 0; k < m; ++k) rbase[(size_t)b * m + k] = aoff[b] + (int64_t)k * h->h_ucount[dom_prop[b]];
  // one blocking copy: the host arrays may be the caller's temporaries
  std::vector<char> tab;
  auto put = [&](const void* src, size_t bytes) {
    const size_t at = tab.size();
    tab.resize(at + ((bytes + 15) & ~(size_t)15));
    if (bytes) std::memcpy(tab.data() + at, src, bytes);
    return h->btab + at;
  };
  h->bt.prop = reinterpret_cast<int*>(put(dom_prop, sizeof(int) * B));
  h->bt.aoff = reinterpret_cast<int64_t*>(put(aoff.data(), sizeof(int64_t) * (B + 1)));
  h->bt.sptr = reinterpret_cast<int64_t*>(put(split_ptr, sizeof(int64_t) * (B + 1)));
  h->bt.rbase = reinterpret_cast<int64_t*>(put(rbase.data(), sizeof(int64_t) * R));
  h->d_split_dom = reinterpret_cast<int*>(put(split_dom.data(), sizeof(int) * nnz));
  h->d_split_col = reinterpret_cast<int*>(put(split_col.data(), sizeof(int) * nnz));
  h->d_side = reinterpret_cast<int8_t*>(put(split_side, sizeof(int8_t) * nnz));
  HIPCHK(hipMemcpy(h->btab, tab.data(), tab.size(), hipMemcpyHostToDevice));
  uint32_t* status = const_cast<uint32_t*>(h->bt.status);
  launch_status_fill(status, h->d_kind, h->bt.prop, B, nd, s);
  launch_status_split(status, h->d_split_dom, h->d_split_col, h->d_side, nnz, nd, s);
  HIPCHK(hipGetLastError());
  h->bt.n_rows = h->R;
  return CV_OK;
}

int build(cv_bound* h, const cv_layer* layers, int n_layers, int P, const float* x_lo, const float* x_hi, int m,
          Spec spec, const float* l, const float* u, int B, const int32_t* dom_prop, const int64_t* split_ptr,
          const int32_t* split_layer, const int32_t* split_neuron, const int8_t* split_side, hipStream_t s) {
  if (P <= 0 || B < 0 || m <= 0) return fail(CV_EINVAL, "n_props, n_dom and m must be positive");
  if (!x_lo || !x_hi || (!spec.C && !spec.identity) || (!dom_prop && B > 0) || !split_ptr)
    return fail(CV_EINVAL, "null input pointer");
  int rc = check_layers(layers, n_layers, h->dims, spec.identity);
  if (rc) return rc;
  h->L = n_layers;
  h->P = P;
  h->m = m;
  h->d0 = h->dims[0];
  h->w64 = (h->d0 + 63) / 64;
  h->offs.assign(std::max(1, n_layers), 0);
  int nd = 0;
  for (int i = 1; i < n_layers; ++i) {
    h->offs[i - 1] = nd;
    nd += h->dims[i];
  }
  h->nd = nd;
  if (nd > 0 && (!l || !u)) return fail(CV_EINVAL, "null intermediate bounds");
  if (!finite_all(x_lo, (int64_t)P * h->d0) || !finite_all(x_hi, (int64_t)P * h->d0))
    return fail(CV_EINVAL, "non-finite input box");
  for (int64_t i = 0; i < (int64_t)P * h->d0; ++i)
    if (x_lo[i] > x_hi[i]) return fail(CV_EINVAL, "input box has x_lo > x_hi at %lld", (long long)i);
  if (nd > 0 && (!finite_all(l, (int64_t)P * nd) || !finite_all(u, (int64_t)P * nd)))
    return fail(CV_EINVAL, "non-finite intermediate bounds");
  if (spec.C && !finite_all(spec.C, (int64_t)P * m * h->dims[n_layers])) return fail(CV_EINVAL, "non-finite C");

  // ---- per-property neuron classes (Eq. definition_D: l >= 0 active, u <= 0 inactive)
  h->h_kind.assign((size_t)P * nd, 0u);
  h->h_cidx.assign((size_t)P * nd, -1);
  h->h_ucount.assign(P, 0);
  std::vector<int> ulist;
  std::vector<int64_t> uoff(P + 1, 0);
  h->h_ucount_layer.assign(P, std::vector<int>(std::max(1, n_layers - 1), 0));
  for (int p = 0; p < P; ++p) {
    uoff[p] = (int64_t)ulist.size();
    for (int j = 0; j < nd; ++j) {
      const float lo = l[(size_t)p * nd + j], up = u[(size_t)p * nd + j];
      uint32_t k = lo >= 0.f ? kActive : (up <= 0.f ? kInactive : kUnstable);
      if (k == kUnstable) {
        k |= (uint32_t)h->h_ucount[p];  // index in the property's unstable list
        h->h_cidx[(size_t)p * nd + j] = h->h_ucount[p]++;
        ulist.push_back(j);
        int li = (int)(std::upper_bound(h->offs.begin(), h->offs.begin() + (n_layers - 1), j) - h->offs.begin()) - 1;
        h->h_ucount_layer[p][li]++;
      }
      h->h_kind[(size_t)p * nd + j] = k;
    }
  }
  uoff[P] = (int64_t)ulist.size();
  // the subdomains and their splits, checked before any device work
  BatchPlan bp;
  if ((rc = check_batch(h, B, dom_prop, split_ptr, split_layer, split_neuron, split_side, bp))) return rc;

  // ---- device copies of the network and of the per-property tables
  DevMem& M = h->mem;
  M.begin();
  rc = upload_layers(h, layers, n_layers, s);
  if (rc) return rc;
  {
    std::vector<uint8_t> defer(std::max(1, nd), 0);
    for (int i = 1; i < n_layers; ++i)
      if (layers[i - 1].type == CV_LAYER_CONV2D) {
        h->has_conv = true;
        std::fill(defer.begin() + h->offs[i - 1], defer.begin() + h->offs[i - 1] + h->dims[i], (uint8_t)1);
      }
    if ((rc = M.upload(&h->d_defer, defer.data(), defer.size(), s))) return rc;
  }
  int *d_ucount, *d_cidx;
  float *d_l, *d_u, *d_xlo, *d_xhi, *d_adef;
  float2* d_chord;
  if ((rc = M.upload(&d_ucount, h->h_ucount.data(), P, s)) ||
      (rc = M.upload(&d_cidx, h->h_cidx.data(), (size_t)P * nd, s)) ||
      (rc = M.upload(&h->d_kind, h->h_kind.data(), (size_t)P * nd, s)) ||
      (rc = M.upload(&d_l, l, l ? (size_t)P * nd : 0, s)) || (rc = M.upload(&d_u, u, u ? (size_t)P * nd : 0, s)) ||
      (rc = M.upload(&d_xlo, x_lo, (size_t)P * h->d0, s)) || (rc = M.upload(&d_xhi, x_hi, (size_t)P * h->d0, s)) ||
      (rc = M.alloc(&d_adef, (size_t)P * nd)) || (rc = M.alloc(&d_chord, (size_t)P * nd)) ||
      (rc = M.upload(&h->ulist, ulist.data(), ulist.size(), s)) || (rc = M.upload(&h->uoff, uoff.data(), P + 1, s)) ||
      (rc = M.flush()))
    return rc;
  h->dl = d_l;
  h->du = d_u;
  launch_prep_chord(d_l, d_u, d_chord, d_adef, (int64_t)P * nd, s);
  HIPCHK(hipGetLastError());

  Batch& bt = h->bt;
  bt.m = m;
  bt.nd = nd;
  bt.d0 = h->d0;
  bt.w64 = h->w64;  // (as wide as the register-tile sign planes need)
  bt.ucount = d_ucount;
  bt.cidx = d_cidx;
  bt.chord = d_chord;
  bt.adef = d_adef;
  bt.xlo = d_xlo;
  bt.xhi = d_xhi;

  // ---- specification merged into the last layer: A(L-1) = C W(L), c = C b(L)
  const DevLayer& last = h->layers[n_layers - 1];
  const int dprev = h->dims[n_layers - 1];
  h->ldcw = r4(dprev);
  if (spec.identity) {
    const int d = last.dout;
    if (m != 2 * d) return fail(CV_EINVAL, "identity spec needs m = 2 d");
    if ((rc = M.alloc(&h->CW, (size_t)m * h->ldcw)) || (rc = M.alloc(&h->Cb, m))) return rc;
    launch_spec_identity(last.type == CV_LAYER_DENSE ? last.W : nullptr, last.ld_in,
                         last.type == CV_LAYER_CONV2D ? last.W : nullptr,
                         last.type == CV_LAYER_CONV2D ? &last.g : nullptr, last.bias, d, dprev, h->CW, h->ldcw, h->Cb,
                         s);
    h->cw_pstride = 0;
    h->cb_pstride = 0;
  } else {
    float* dC;
    if ((rc = M.upload(&dC, spec.C, (size_t)P * m * last.dout, s)) ||
        (rc = M.alloc(&h->CW, (size_t)P * m * h->ldcw)) || (rc = M.alloc(&h->Cb, (size_t)P * m)))
      return rc;
    h->dC = dC;
    launch_spec_merge(dC, last.W, last.ld_in, last.bias, P, m, last.dout, dprev, h->CW, h->ldcw, h->Cb, s);
    h->cw_pstride = (int64_t)m * h->ldcw;
    h->cb_pstride = m;
  }
  HIPCHK(hipGetLastError());

  // ---- workspace
  int maxd = 4;
  for (int i = 1; i < n_layers; ++i) maxd = std::max(maxd, h->dims[i]);
  h->ldact = r4(maxd);
  // the top layer takes one slot, or one per 32-column tile when it is
  // relaxed inside the optimiser's last adjoint GEMM
  h->n_slots = n_layers >= 2 && layers[n_layers - 2].type == CV_LAYER_DENSE ? std::max(1, (h->dims[n_layers - 1] + 31) / 32)
                                                                           : 1;
  for (int i = n_layers - 1; i >= 1; --i) {  // back-substitution through layer i
    const DevLayer& ly = h->layers[i - 1];
    h->n_slots += ly.type == CV_LAYER_DENSE ? (h->dims[i - 1] + 31) / 32 : 1;
  }
  // ---- the subdomains: splits checked, row tables, status words, buffers
  if ((rc = set_batch(h, bp, false, s))) return rc;
  assign_tiles(h, -1);
  assign_conv_variants(h, -1);
  // dense layers fused by the chain kernels (LDS-resident widths up to kChainWidth)
  h->chain_lo = 0;
  h->chain_b = h->chain_f = 0;
  auto chain_ok = [&](int i) {  // layer i dense with a K-dim (d_i) that fits
    return i >= 1 && h->layers[i - 1].type == CV_LAYER_DENSE && h->dims[i] <= kChainWidth;
  };
  if (n_layers >= 2 && chain_ok(n_layers - 1)) {
    int lo = n_layers - 1;
    while (lo - 1 >= 1 && chain_ok(lo - 1) && (n_layers - lo) < kChainMax) --lo;
    h->chain_lo = lo;
    // the chain is available; per-layer kernels stay the default (measured
    // faster at ~10^4 rows), cv_bound_autotune / cv_bound_set_plan choose
    if (!plan_chain(h)) h->chain_lo = 0;
  }
  HIPCHK(hipStreamSynchronize(s));
  return CV_OK;
}

// (batch-sized buffers come from the batch pool at its capacities)
int ensure_grad(cv_bound* h) {
  if (h->acomp) return CV_OK;
  int rc;
  const cv_bound::Cap& c = h->bcap;
  if ((rc = h->bm.alloc(&h->acomp, c.na)) || (rc = h->bm.alloc(&h->xpos, (size_t)c.R * h->w64)) ||
      (rc = h->bm.alloc(&h->xneg, (size_t)c.R * h->w64)))
    return rc;
  if (h->layers[0].type == CV_LAYER_DENSE && !h->xdense) {
    // the first adjoint step reads x* as a plain GEMM operand
    h->ldx = r4(h->d0);
    if ((rc = h->bm.alloc(&h->xdense, (size_t)c.R * h->ldx))) return rc;
  }
  return CV_OK;
}

int ensure_opt(cv_bound* h) {
  int rc = ensure_grad(h);
  if (rc) return rc;
  if (h->g_alpha) return CV_OK;
  const cv_bound::Cap& c = h->bcap;
  const int64_t nb = c.nnz * h->m;
  if ((rc = h->bm.alloc(&h->g_alpha, c.na)) || (rc = h->bm.alloc(&h->g_beta, nb)) ||
      (rc = h->bm.alloc(&h->adam, 2 * c.na + 2 * nb)))
    return rc;
  return CV_OK;
}

// The l_p-ball buffers of a handle: per-row |A(0)|^q partials and minimiser
// scales, and the minimiser's direction kept densely.
int ensure_ball(cv_bound* q) {
  int rc;
  const cv_bound::Cap& c = q->bcap;
  if (!q->psq && ((rc = q->bm.alloc(&q->psq, (size_t)q->n_slots * std::max<int64_t>(1, c.R))) ||
                  (rc = q->bm.alloc(&q->l2s, std::max<int64_t>(1, c.R)))))
    return rc;
  if (!q->xdense) {
    q->ldx = r4(q->d0);
    if ((rc = q->bm.alloc(&q->xdense, (size_t)std::max<int64_t>(1, c.R) * q->ldx))) return rc;
  }
  return CV_OK;
}

// ---------------------------------------------------------------------------
// sound mode: a rigorous bound on what float32 rounding can move each bound
// by, so that the reported value lb - margin lies below the bound computed in
// exact arithmetic from the same relaxation.  Host double arithmetic, every
// weight rounded up to float.  Terms, with u' = 2^-23 (twice the unit
// roundoff, so any rounding mode of the matrix cores is covered) and
// g(n) = n u' / (1 - n u'):
//   * the product A(i-1) = Lambda(i) W(i) (K = d_i terms per output for a
//     dense layer on the matrix cores; at most c_out ceil(k/s)^2 taps for a
//     transposed convolution, whose FMAs round to nearest: u'/2 there): its
//     error against the exact product, times any input of layer i (at most
//     hmax = max(u, 0) of layer i-1, or max(|x_lo|, |x_hi|) at the input), is
//     at most g(d_i) sum_k |Lambda(i)_k| v_k, v_k = sum_j |W(i)_kj| hmax_j;
//   * Lambda itself is one rounding away from A D + beta S: u' |Lambda_k| zmax_k;
//   * the float32 chord of an unstable neuron can sit below the ReLU at the
//     ends of [l, u] by at most 4u'(s zmax + |t|) (slope s, intercept t);
//     weighted by |A_k| = |Lambda_k| / s;
//   * every term added into the constant and the concretisation sum passes
//     through at most N additions (N bounded from the kernels' reduction
//     trees and the number of partial slots): G = g(N) + u' times its size,
//     |Lambda_k b_k| for the bias, |A_k t_k| for the chord intercept;
//   * the merged specification C W(L), C b(L) (formed once in float32):
//     g(d_L) (sum_o |C_o| v(L)_o + |C_o b_o|), a per-(property, row) constant.
// All but the last collapse into one weight per (property, neuron):
//   sw_k = g(d_i) v_k + u' zmax_k + G |b_k| + [unstable] (4u'(s zmax + |t|) + G |t|) / s,
// so an epilogue adds |Lambda_k| sw_k per element and G |term| per
// concretisation term; the final sum scales the margin by (1 + 2 g(N)) for
// its own rounding and rounds the result down.

float round_up_f(double x) {
  float f = (float)x;
  if ((double)f < x) f = std::nextafter(f, INFINITY);
  return f;
}

// v_k = sum_j |W_kj| hm_j for one layer (host weights)
void abs_weighted(const cv_layer& ly, const std::vector<double>& hm, std::vector<double>& v) {
  if (ly.type == CV_LAYER_DENSE) {
    for (int k = 0; k < ly.out_c; ++k) {
      double t = 0.0;
      const float* w = ly.weight + (size_t)k * ly.in_c;
      for (int j = 0; j < ly.in_c; ++j) t += std::fabs((double)w[j]) * hm[j];
      v[k] = t;
    }
    return;
  }
  for (int c = 0; c < ly.out_c; ++c)
    for (int oy = 0; oy < ly.out_h; ++oy)
      for (int ox = 0; ox < ly.out_w; ++ox) {
        double t = 0.0;
        for (int ci = 0; ci < ly.in_c; ++ci)
          for (int ky = 0; ky < ly.kernel; ++ky) {
            const int iy = oy * ly.stride - ly.pad + ky;
            if (iy < 0 || iy >= ly.in_h) continue;
            for (int kx = 0; kx < ly.kernel; ++kx) {
              const int ix = ox * ly.stride - ly.pad + kx;
              if (ix < 0 || ix >= ly.in_w) continue;
              const float w = ly.weight[(((size_t)c * ly.in_c + ci) * ly.kernel + ky) * ly.kernel + kx];
              t += std::fabs((double)w) * hm[((size_t)ci * ly.in_h + iy) * ly.in_w + ix];
            }
          }
        v[((size_t)c * ly.out_h + oy) * ly.out_w + ox] = t;
      }
}

// out = W x + b for one affine layer, in double.
void affine_host(const cv_layer& ly, const float* x, std::vector<double>& out) {
  if (ly.type == CV_LAYER_DENSE) {
    out.assign(ly.out_c, 0.0);
    for (int k = 0; k < ly.out_c; ++k) {
      double t = ly.bias[k];
      const float* w = ly.weight + (size_t)k * ly.in_c;
      for (int j = 0; j < ly.in_c; ++j) t += (double)w[j] * x[j];
      out[k] = t;
    }
    return;
  }
  out.assign((size_t)ly.out_c * ly.out_h * ly.out_w, 0.0);
  for (int c = 0; c < ly.out_c; ++c)
    for (int oy = 0; oy < ly.out_h; ++oy)
      for (int ox = 0; ox < ly.out_w; ++ox) {
        double t = ly.bias[c];
        for (int ci = 0; ci < ly.in_c; ++ci)
          for (int ky = 0; ky < ly.kernel; ++ky) {
            const int iy = oy * ly.stride - ly.pad + ky;
            if (iy < 0 || iy >= ly.in_h) continue;
            for (int kx = 0; kx < ly.kernel; ++kx) {
              const int ix = ox * ly.stride - ly.pad + kx;
              if (ix < 0 || ix >= ly.in_w) continue;
              t += (double)ly.weight[(((size_t)c * ly.in_c + ci) * ly.kernel + ky) * ly.kernel + kx] *
                   x[((size_t)ci * ly.in_h + iy) * ly.in_w + ix];
            }
          }
        out[((size_t)c * ly.out_h + oy) * ly.out_w + ox] = t;
      }
}

// Weights and constants of the margin for handle h from its host inputs
// (layers, box [P, d0], root bounds [P, nd], C [P, m, dL] unless identity).
// Over l2 balls (l2x0 [P, d0], l2eps [P] set) an input coordinate is bounded
// by |x0_j| + eps_p instead of the box, and the per-property ||x0||_2 and the
// norm's rounding factor are prepared for the final sum.
// One rounding-error analysis (the terms above) for unit roundoff up (2^-23
// for the float32 kernels, 2^-52 for the float64 evaluation) and the longest
// addition chain of the kernels' sums.
struct SoundWeights {
  std::vector<float> sw, e0;
  double G = 0, gchain = 0;
};

void sound_weights(const cv_bound* h, const cv_layer* layers, const float* x_lo, const float* x_hi, const float* l,
                   const float* u, const float* C, bool identity, const float* l2x0, const float* l2eps, double up,
                   int chain, SoundWeights& out);

// Sound mode's batch-sized buffers (float64 rows and partials, the optimiser's
// best-iterate copies), from the batch pool at its capacities.
int ensure_sound_batch(cv_bound* h) {
  int rc;
  if (h->R >= kRows64) {
    bool packed = !h->chord64;
    if (packed) {
      const int64_t n = (int64_t)h->P * std::max(h->nd, 1);
      if ((rc = h->mem.alloc(&h->chord64, n))) return rc;
      launch_chord64(h->dl, h->du, h->chord64, (int64_t)h->P * h->nd, nullptr);
    }
    for (DevLayer& ly : h->layers) {
      if (ly.type != CV_LAYER_CONV2D || ly.W64) continue;
      if ((rc = h->mem.alloc(&ly.W64, conv64_pack_size(ly.g)))) return rc;
      launch_conv64_pack(ly.W, ly.g, ly.W64, nullptr);
      packed = true;
    }
    if (packed) HIPCHK(hipStreamSynchronize(nullptr));
  }
  if (h->perr) return CV_OK;
  const cv_bound::Cap& c = h->bcap;
  const int64_t R1 = std::max<int64_t>(1, c.R), R8 = R1 + 8;  // (the last group of rows is read whole)
  const int L = h->L;
  if ((rc = h->bm.alloc(&h->perr, (size_t)R1 * h->n_slots)) ||
      (rc = h->bm.alloc(&h->act64[0], (size_t)R8 * h->ldact)) ||
      (rc = h->bm.alloc(&h->act64[1], (size_t)R8 * h->ldact)) || (rc = h->bm.alloc(&h->part64, (size_t)R1 * L)) ||
      (rc = h->bm.alloc(&h->perr64, (size_t)R1 * L)) || (rc = h->bm.alloc(&h->psq64, (size_t)R1 * L)) ||
      (rc = h->bm.alloc(&h->gbest, (size_t)R1)) || (rc = h->bm.alloc(&h->improved, (size_t)R1)) ||
      (rc = h->bm.alloc(&h->abest, (size_t)std::max<int64_t>(1, c.na))) ||
      (rc = h->bm.alloc(&h->bbest, (size_t)std::max<int64_t>(1, c.nnz * h->m))))
    return rc;
  return CV_OK;
}

int prepare_sound(cv_bound* h, const cv_layer* layers, const float* x_lo, const float* x_hi, const float* l,
                  const float* u, const float* C, bool identity, hipStream_t s, const float* l2x0 = nullptr,
                  const float* l2eps = nullptr) {
  const int L = h->L, P = h->P, nd = h->nd, d0 = h->d0;
  // the float64 evaluation keeps one row of Lambda in a workgroup's 64 KB of LDS
  for (int i = 1; i < L; ++i)
    if (h->dims[i] > 8192) return fail(CV_ESHAPE, "sound mode: layer %d is wider than 8192 neurons", i);
  const double up = std::ldexp(1.0, -23);
  auto gam = [&](double n) { return n * up / (1.0 - n * up); };
  // longest addition chain: final sum over slots (and its four-way merge),
  // plus the longest in-kernel chain (GEMM tiles: a few; top layer: two per
  // 64 neurons per lane; transposed convolutions: two per 256 outputs of a
  // row, bounded by two per input channel per 256 positions) and the
  // reduction trees (at most 64 levels)
  int chain = 0;
  if (L >= 2) chain = std::max(chain, 2 * ((h->dims[L - 1] + 63) / 64));
  for (int i = 1; i < L; ++i) {
    const cv_layer& ly = layers[i - 1];
    if (ly.type != CV_LAYER_DENSE)
      chain = std::max(chain, 2 * ly.in_c * ((ly.in_h * ly.in_w + 255) / 256));
  }
  chain += h->n_slots + 64;
  SoundWeights w32, w64;
  sound_weights(h, layers, x_lo, x_hi, l, u, C, identity, l2x0, l2eps, up, chain, w32);
  // float64 kernels: per-thread chains over a layer's outputs (at most the
  // widest layer), block trees (8 levels), the final sum over L slots
  int chain64 = 64 + L;
  for (int i = 0; i <= L; ++i) chain64 = std::max(chain64, h->dims[i] + 64 + L);
  const double up64 = std::ldexp(1.0, -52);
  sound_weights(h, layers, x_lo, x_hi, l, u, C, identity, l2x0, l2eps, up64, chain64, w64);
  int rc;
  if (!h->sw) {
    if ((rc = h->mem.alloc(&h->sw, w32.sw.size())) || (rc = h->mem.alloc(&h->err0, w32.e0.size())) ||
        (rc = h->mem.alloc(&h->sw64, w64.sw.size())) || (rc = h->mem.alloc(&h->err064, w64.e0.size())))
      return rc;
  }
  if ((rc = ensure_sound_batch(h))) return rc;
  HIPCHK(hipMemcpyAsync(h->sw, w32.sw.data(), w32.sw.size() * sizeof(float), hipMemcpyHostToDevice, s));
  HIPCHK(hipMemcpyAsync(h->err0, w32.e0.data(), w32.e0.size() * sizeof(float), hipMemcpyHostToDevice, s));
  HIPCHK(hipMemcpyAsync(h->sw64, w64.sw.data(), w64.sw.size() * sizeof(float), hipMemcpyHostToDevice, s));
  HIPCHK(hipMemcpyAsync(h->err064, w64.e0.data(), w64.e0.size() * sizeof(float), hipMemcpyHostToDevice, s));
  const double G = w32.G;
  h->sg64 = w64.G;
  h->scale64 = 1.0 + 2.0 * w64.gchain;
  // ||A(0)||_2: d0 squares summed, a square root; A(0) x0: d0 products summed
  h->ball64 = (d0 + 64) * up64 / (1.0 - (d0 + 64) * up64) + 4.0 * up64;
  (void)nd;
  (void)P;
  if (l2x0) {
    std::vector<float> x0n(P);
    for (int p = 0; p < P; ++p) {
      double t = 0.0;
      for (int j = 0; j < d0; ++j) t += (double)l2x0[(size_t)p * d0 + j] * l2x0[(size_t)p * d0 + j];
      x0n[p] = round_up_f(std::sqrt(t) * (1.0 + 1e-12));
    }
    if (!h->x0n && (rc = h->mem.alloc(&h->x0n, P))) return rc;
    HIPCHK(hipMemcpyAsync(h->x0n, x0n.data(), sizeof(float) * P, hipMemcpyHostToDevice, s));
    // sum of squares within gam(chain) relative, the square root and the
    // product each within an ulp
    h->l2fac = round_up_f((1.0 + gam(chain)) * (1.0 + 4.0 * up));
  }
  HIPCHK(hipStreamSynchronize(s));
  h->sound_g = round_up_f(G);
  h->sound_scale = round_up_f(1.0 + 2.0 * gam(chain));
  return CV_OK;
}

void sound_weights(const cv_bound* h, const cv_layer* layers, const float* x_lo, const float* x_hi, const float* l,
                   const float* u, const float* C, bool identity, const float* l2x0, const float* l2eps, double up,
                   int chain, SoundWeights& out) {
  const int L = h->L, P = h->P, m = h->m, nd = h->nd, d0 = h->d0;
  auto gam = [&](double n) { return n * up / (1.0 - n * up); };
  const double G = gam(chain) + up;
  out.G = G;
  out.gchain = gam(chain);
  std::vector<float> sw((size_t)P * std::max(nd, 1), 0.f), e0((size_t)P * m, 0.f);
  for (int p = 0; p < P; ++p) {
    std::vector<double> hm(d0);
    for (int j = 0; j < d0; ++j)
      hm[j] = l2x0 ? std::fabs((double)l2x0[(size_t)p * d0 + j]) + (double)l2eps[p]
                   : std::max(std::fabs((double)x_lo[(size_t)p * d0 + j]), std::fabs((double)x_hi[(size_t)p * d0 + j]));
    int off = 0;
    for (int i = 1; i < L; ++i) {
      const cv_layer& ly = layers[i - 1];
      const int d = h->dims[i];
      const int per = ly.type == CV_LAYER_DENSE ? 1 : ly.out_h * ly.out_w;
      // terms per output of the back-substitution product, all on the matrix
      // cores (u'): all d_i neurons for a dense layer; for a transposed
      // convolution the K axis of its polyphase GEMM, c_out ceil(k/s)^2
      const int ks = (ly.kernel + ly.stride - 1) / std::max(1, ly.stride);
      const double gk = ly.type == CV_LAYER_DENSE ? gam(d) : gam((double)ly.out_c * ks * ks);
      std::vector<double> v(d, 0.0), hn(d);
      abs_weighted(ly, hm, v);
      for (int k = 0; k < d; ++k) {
        const double lk = l[(size_t)p * nd + off + k], uk = u[(size_t)p * nd + off + k];
        const double zmax = std::max(std::fabs(lk), std::fabs(uk));
        const double bk = std::fabs((double)ly.bias[k / per]);
        double w = gk * v[k] + up * zmax + G * bk;
        if (lk < 0.0 && uk > 0.0) {
          const double sl = uk / (uk - lk), t = -uk * lk / (uk - lk);
          w += (4.0 * up * (sl * zmax + std::fabs(t)) + G * std::fabs(t)) / sl;
        }
        sw[(size_t)p * nd + off + k] = round_up_f(w);
        hn[k] = std::max(uk, 0.0);
      }
      hm.swap(hn);
      off += d;
    }
    if (!identity) {
      const cv_layer& ly = layers[L - 1];
      const int dL = h->dims[L];
      std::vector<double> vL(dL, 0.0);
      abs_weighted(ly, hm, vL);
      for (int k = 0; k < m; ++k) {
        double e = 0.0, cb = 0.0;
        for (int o = 0; o < dL; ++o) {
          const double c = C[((size_t)p * m + k) * dL + o];
          e += std::fabs(c) * vL[o] + std::fabs(c * ly.bias[o]);
          cb += c * ly.bias[o];
        }
        // 1e-30: room for any flushed denormal along the way
        e0[(size_t)p * m + k] = round_up_f(gam(dL) * e + G * std::fabs(cb) + 1e-30);
      }
    }
  }
  out.sw.swap(sw);
  out.e0.swap(e0);
}

// ---------------------------------------------------------------------------
// passes

std::string cfg_name(int cfg) {
  const GemmCfg& c = kGemmCfgs[cfg];
  return std::to_string(c.bm) + "x" + std::to_string(c.bn) + "x" + std::to_string(c.bk) +
         (c.occ ? "w" + std::to_string(c.occ) : std::string()) + (c.depth > 1 ? "d" + std::to_string(c.depth) : "");
}

Epi make_epi(const cv_bound* h) {
  Epi e{};
  e.part = h->part;
  e.perr = h->sound ? h->perr : nullptr;
  e.psq = h->l2 ? h->psq : nullptr;
  e.n_slots = h->n_slots;
  e.ldo = h->ldact;
  return e;
}

// profile name of a conv layer: channels, kernel and stride ("8-16k4s2")
std::string conv_tag(const ConvGeom& g) {
  return std::to_string(g.ci) + "-" + std::to_string(g.co) + "k" + std::to_string(g.k) + "s" + std::to_string(g.s);
}

// conv MACs of one row (taps inside the input only)
double conv_macs(const ConvGeom& g) {
  double taps = 0;
  for (int oy = 0; oy < g.ho; ++oy)
    for (int ky = 0; ky < g.k; ++ky) {
      const int iy = oy * g.s - g.p + ky;
      if (iy < 0 || iy >= g.hi) continue;
      for (int ox = 0; ox < g.wo; ++ox)
        for (int kx = 0; kx < g.k; ++kx) {
          const int ix = ox * g.s - g.p + kx;
          if (ix >= 0 && ix < g.wi) taps += 1;
        }
    }
  return taps * g.ci * g.co;
}

struct AdamStep {
  float lr_a, lr_b, bc1, bc2;
  float *ma, *va, *mb, *vb;
};

double chain_flops(const cv_bound* h) {
  double f = 0;
  for (int i = h->chain_lo; i <= h->L - 1; ++i) f += 2.0 * h->R * h->dims[i] * h->dims[i - 1];
  return f;
}

// Back-substitution of every layer plus concretisation; lb / best per row.
// skip_top: the top layer was relaxed by the previous adjoint pass (fused
// into its last GEMM): start from its Lambda(L-1) and partial slots.
int enqueue_bwd(cv_bound* h, const float* alpha, const float* beta, bool grad, float* lb, float* best, int first,
                hipStream_t s, bool skip_top = false, int* improved = nullptr) {
  const int L = h->L;
  Vars v{};
  v.alpha = alpha;
  v.beta = beta;
  v.acomp = grad ? h->acomp : nullptr;
  // x* for the adjoint: dense rows for a dense first layer, sign planes for a convolution
  // (over an l2 ball: A(0) itself, densely, whatever the first layer)
  const bool dense1 = h->layers[0].type == CV_LAYER_DENSE;
  v.xpos = grad && !dense1 && !h->l2 ? h->xpos : nullptr;
  v.xneg = grad && !dense1 && !h->l2 ? h->xneg : nullptr;
  v.xdense = grad && (dense1 || h->l2) ? h->xdense : nullptr;
  v.ldx = h->ldx;
  Profiler* pf = h->prof;
  if (h->R == 0) return CV_OK;
  int cur = 0, slot = 1, i_next = L - 1;
  if (skip_top) {
    cur = h->ftop_buf;
    slot = h->ftop_slots;
  } else if (h->chain_b && !h->sound && !h->l2 && !improved) {
    const int lo = h->chain_lo;
    ChainArgs ca{};
    ca.nl = L - lo;
    for (int i = L - 1, t = 0; i >= lo; --i, ++t) {
      const DevLayer& ly = h->layers[i - 1];
      ca.ly[t] = ChainLayer{ly.Wt, ly.ld_out, h->dims[i], h->dims[i - 1], i - 1 >= 1 ? h->layers[i - 2].bias : nullptr,
                            i - 1 >= 1 ? h->offs[i - 2] : 0};
    }
    ca.np = h->chain_np;
    ca.ncw = h->chain_ncw;
    ca.ldk = h->chain_np + 4;
    ca.rb = h->chain_rb;
    ca.uw = h->chain_uw;
    ca.grid = h->chain_grid;
    ca.CW = h->CW;
    ca.cw_pstride = h->cw_pstride;
    ca.ldcw = h->ldcw;
    ca.Cb = h->Cb;
    ca.cb_pstride = h->cb_pstride;
    ca.n_top = h->dims[L - 1];
    ca.top_off = h->offs[L - 2];
    ca.top_bias = h->layers[L - 2].bias;
    ca.conc = lo == 1;
    ca.out = h->act[0];
    ca.ldo = h->ldact;
    ca.part = h->part;
    ca.n_slots = h->n_slots;
    ca.slot = 0;
    ca.lb = lb;
    ca.best = best;
    ca.first = first;
    ca.final = lo == 1;
    ca.bt = h->bt;
    ca.v = v;
    const double rows = h->R;
    if (pf) pf->begin("chain_bwd", chain_flops(h),
                      rows * h->dims[L - 1] * 4.0 +
                          (lo == 1 && !v.xdense ? rows * h->d0 / 4.0 : rows * h->dims[lo - 1] * 4.0) +
                          (double)h->B * (h->nd - (lo >= 2 ? h->offs[lo - 2] : 0)) * 2.0);
    launch_chain_bwd(ca, s);
    if (pf) pf->end();
    if (lo == 1) {
      HIPCHK(hipGetLastError());
      return CV_OK;
    }
    i_next = lo - 1;
  } else {
    TopArgs ta{};
    ta.CW = h->CW;
    ta.cw_pstride = h->cw_pstride;
    ta.ldcw = h->ldcw;
    ta.Cb = h->Cb;
    ta.cb_pstride = h->cb_pstride;
    ta.n = h->dims[L - 1];
    ta.conc = L == 1;
    ta.err0 = h->sound ? h->err0 : nullptr;
    ta.bt = h->bt;
    ta.v = v;
    ta.e = make_epi(h);
    ta.e.slot0 = 0;
    if (L >= 2) {
      ta.e.layer_off = h->offs[L - 2];
      ta.e.bias = h->layers[L - 2].bias;
      ta.e.out = h->act[0];
    }
    if (pf) pf->begin(L == 1 ? "top_conc" : "top_relax", 0, (double)h->R * ta.n * 8);
    launch_top(ta, s);
    if (pf) pf->end();
  }
  for (int i = i_next; i >= 1; --i) {
    const DevLayer& ly = h->layers[i - 1];
    const int mode = i - 1 >= 1 ? kBwdRelax : kBwdConc;
    Epi e = make_epi(h);
    e.slot0 = slot;
    e.n = h->dims[i - 1];
    if (mode == kBwdRelax) {
      e.layer_off = h->offs[i - 2];
      e.bias = h->layers[i - 2].bias;
      e.out = h->act[cur ^ 1];
    }
    const double rows = h->R;
    const int N = h->dims[i - 1], K = h->dims[i];
    const double io = rows * K * 4.0 + (mode == kBwdRelax || v.xdense ? rows * N * 4.0 : rows * N / 4.0) +
                      (double)h->B * N * 2.0 +
                      (mode == kBwdRelax ? h->unst_rows_per_layer[i - 2] * 4.0 * (grad ? 2 : 1) : 0.0);
    if (ly.type == CV_LAYER_DENSE) {
      const int c = h->cfg[i - 1] >= 0 ? h->cfg[i - 1] : 0;
      GemmArgs g{h->act[cur], h->ldact, ly.Wt, ly.ld_out, h->R, N, K, 0, h->bt, v, e};
      if (pf) pf->begin(std::string(mode == kBwdRelax ? "gemm_bwd_relax_" : "gemm_bwd_conc_") + cfg_name(c),
                        2.0 * rows * N * K, io + (double)N * K * 4.0);
      launch_gemm(c, mode, g, s);
      if (pf) pf->end();
      slot += (N + kGemmCfgs[c].bn - 1) / kGemmCfgs[c].bn;
    } else {
      ConvArgs a{h->act[cur], h->ldact, ly.bwd, h->R, 0, h->bt, v, e};
      if (pf) pf->begin(std::string(mode == kBwdRelax ? "convt_bwd_relax_" : "convt_bwd_conc_") + conv_tag(ly.g),
                        2.0 * rows * conv_macs(ly.g), io);
      if (launch_convt_bwd(mode, a, s)) return fail(CV_ESHAPE, "unsupported conv channels");
      if (pf) pf->end();
      slot += 1;
    }
    cur ^= 1;
  }
  if (pf) pf->begin("finalize", 0, (double)h->R * (slot + 2) * 4.0);
  const L2Final l2f{h->bt.prop, h->m, h->l2eps, h->l2s, h->x0n, h->sound_g, h->l2fac, h->lpq};
  launch_finalize(h->part, h->sound ? h->perr : nullptr, h->sound_scale, h->l2 ? h->psq : nullptr, l2f, h->n_slots,
                  slot, h->R, lb, best, first, s, improved);
  if (pf) pf->end();
  HIPCHK(hipGetLastError());
  return CV_OK;
}

// Sound mode's evaluation in float64 (sound64.hip): every back-substitution
// step, relaxation and concretisation in double with its rigorous float64
// margin; lb = the bound minus the margin rounded down to float (best: the
// running maximum, first = 1 starts it).  Needs the buffers of set_sound.
int enqueue_bwd64(cv_bound* h, const float* alpha, const float* beta, float* lb, float* best, int first,
                  hipStream_t s) {
  const int L = h->L;
  if (h->R == 0) return CV_OK;
  if (!h->sw64 || !h->act64[0]) return fail(CV_EINVAL, "sound mode is off");
  Pass64 q{};
  q.bt = h->bt;
  q.l = h->dl;
  q.u = h->du;
  q.chord = h->chord64;
  q.alpha = alpha;
  q.beta = beta;
  q.sw = h->sw64;
  q.sg = h->sg64;
  q.part = h->part64;
  q.perr = h->perr64;
  q.psq = h->l2 ? h->psq64 : nullptr;
  Top64 t{};
  const DevLayer& last = h->layers[L - 1];
  if (h->dC) {
    t.C = h->dC;
    t.dL = h->dims[L];
    t.WL = last.W;
    t.ldw = last.ld_in;
    t.bL = last.bias;
  } else {
    t.CW = h->CW;
    t.cw_pstride = h->cw_pstride;
    t.ldcw = h->ldcw;
    t.Cb = h->Cb;
    t.cb_pstride = h->cb_pstride;
  }
  t.n = h->dims[L - 1];
  t.conc = L == 1;
  t.err0 = h->err064;
  if (L >= 2) {
    t.layer_off = h->offs[L - 2];
    t.bias = h->layers[L - 2].bias;
    t.out = h->act64[0];
    t.ldo = h->ldact;
  }
  launch_top64(q, t, s);
  int cur = 0;
  for (int i = L - 1; i >= 1; --i) {
    const DevLayer& ly = h->layers[i - 1];
    Lay64 y{};
    y.in = h->act64[cur];
    y.ldi = h->ldact;
    y.K = h->dims[i];
    y.N = h->dims[i - 1];
    y.W = ly.W;
    y.ldw = ly.ld_in;
    y.w64 = ly.W64;
    y.conc = i == 1;
    y.slot = L - i;
    if (i >= 2) {
      y.layer_off = h->offs[i - 2];
      y.bias = h->layers[i - 2].bias;
      y.out = h->act64[cur ^ 1];
      y.ldo = h->ldact;
    }
    if (ly.type == CV_LAYER_DENSE) launch_dense64(q, y, s);
    else launch_conv64(q, y, ly.g, s);
    cur ^= 1;
  }
  Fin64 f{};
  f.n_used = L;
  f.scale = h->scale64;
  f.ball = h->ball64;
  f.x0n = h->x0n;
  f.lb = lb;
  f.best = best;
  f.first = first;
  launch_finalize64(q, f, s);
  HIPCHK(hipGetLastError());
  return CV_OK;
}

// Adjoint forward sweep: zbar(i) = W(i) zhat(i-1) + b(i) from zhat(0) = x*,
// gradients of alpha and beta in the epilogues (or, with `ad`, the projected
// Adam step applied in place).
// Operand of forward layer i: zhat(i-1) for i > 1; at the first layer x*,
// read densely (dense first layer), from its sign planes (conv first layer,
// mode kFwdX), or over an l2 ball as A(0) itself with zbar(1) = W(1) x0 + b(1)
// - l2s (W(1) A(0)) formed in the epilogue.
void first_layer_input(cv_bound* h, int i, Vars& v, Epi& e, const float*& in, int& lda, int& mode) {
  mode = kFwd;
  lda = h->ldact;
  in = i == 1 ? nullptr : h->act[(i - 1) & 1];
  if (i != 1) return;
  if (h->l2) {
    in = h->xdense;
    lda = h->ldx;
    e.wx0 = h->wx0;
    v.l2s = h->l2s;
  } else if (h->layers[0].type == CV_LAYER_DENSE) {
    in = h->xdense;
    lda = h->ldx;
  } else {
    mode = kFwdX;
  }
}

// fuse_top (optimiser, with Adam): the last adjoint GEMM also relaxes the next
// iteration's top layer (Epi::top_out); the next back-substitution then
// starts from its output (enqueue_bwd with skip_top).
int enqueue_fwd(cv_bound* h, const float* alpha, const float* beta, float* ga, float* gb, const AdamStep* ad,
                hipStream_t s, bool fuse_top = false) {
  const int L = h->L;
  Vars v{};
  v.alpha = alpha;
  v.beta = beta;
  v.acomp = h->acomp;
  v.galpha = ga;
  v.gbeta = gb;
  v.xpos = h->xpos;
  v.xneg = h->xneg;
  v.zchord = h->zchord;
  if (ad) {
    v.adam = 1;
    v.lr_a = ad->lr_a;
    v.lr_b = ad->lr_b;
    v.bc1 = ad->bc1;
    v.bc2 = ad->bc2;
    v.alpha_w = const_cast<float*>(alpha);
    v.beta_w = const_cast<float*>(beta);
    v.ma = ad->ma;
    v.va = ad->va;
    v.mb = ad->mb;
    v.vb = ad->vb;
  }
  Profiler* pf = h->prof;
  if (h->R == 0) return CV_OK;
  // the adjoint chain starts one layer above the lowest chained layer, whose
  // input (x* or a wide conv output) goes through the per-layer kernel
  const int i_chain = h->chain_f ? h->chain_lo + 1 : L;
  for (int i = 1; i <= L - 1 && i < i_chain; ++i) {
    const DevLayer& ly = h->layers[i - 1];
    const int last = i == L - 1;
    Epi e = make_epi(h);
    e.layer_off = h->offs[i - 1];
    e.bias = ly.bias;
    e.n = h->dims[i];
    e.out = h->act[i & 1];
    int mode, lda;
    const float* in;
    first_layer_input(h, i, v, e, in, lda, mode);
    const double rows = h->R;
    const int N = h->dims[i], K = h->dims[i - 1];
    const double io = (mode == kFwdX ? rows * K / 4.0 : rows * K * 4.0) + (last ? 0.0 : rows * N * 4.0) +
                      (double)h->B * N * 2.0 + h->unst_rows_per_layer[i - 1] * 4.0 * 3;
    if (ly.type == CV_LAYER_DENSE) {
      const int c = h->cfg[L + i - 1] >= 0 ? h->cfg[L + i - 1] : 0;
      if (last && fuse_top) {
        h->ftop_buf = i & 1;  // not the input buffer act[(i - 1) & 1]
        h->ftop_slots = (N + kGemmCfgs[c].bn - 1) / kGemmCfgs[c].bn;
        e.top_out = h->act[h->ftop_buf];
        e.cw = h->CW;
        e.cw_pstride = h->cw_pstride;
        e.ldcw = h->ldcw;
        e.cb = h->Cb;
        e.cb_pstride = h->cb_pstride;
        e.slot0 = 0;
      }
      GemmArgs g{in, lda, ly.W, ly.ld_in, h->R, N, K, last, h->bt, v, e};
      if (pf) pf->begin(std::string(i == 1 ? "gemm_fwd_x_" : "gemm_fwd_") + cfg_name(c), 2.0 * rows * N * K,
                        io + (double)N * K * 4.0);
      launch_gemm(c, e.top_out ? kFwdTop : mode, g, s);
      if (pf) pf->end();
    } else {
      ConvArgs a{in, lda, ly.fwd, h->R, last, h->bt, v, e};
      // with Adam, the split neurons' steps wait for split_adam_k after the
      // pass: their reads would otherwise stall the epilogue
      if (v.adam && h->g_beta) a.v.gsplit = h->g_beta;
      if (pf) pf->begin(std::string(mode == kFwdX ? "conv_fwd_x_" : "conv_fwd_") + conv_tag(ly.g),
                        2.0 * rows * conv_macs(ly.g), io);
      if (launch_conv_fwd(mode, a, s)) return fail(CV_ESHAPE, "unsupported conv channels");
      if (pf) pf->end();
    }
  }
  if (i_chain <= L - 1) {
    const int lo = i_chain;
    ChainArgs ca{};
    ca.nl = L - lo;
    double fl = 0, unst = 0;
    for (int i = lo, t = 0; i <= L - 1; ++i, ++t) {
      const DevLayer& ly = h->layers[i - 1];
      ca.ly[t] = ChainLayer{ly.W, ly.ld_in, h->dims[i - 1], h->dims[i], ly.bias, h->offs[i - 1]};
      fl += 2.0 * h->R * h->dims[i] * h->dims[i - 1];
      unst += h->unst_rows_per_layer[i - 1];
    }
    ca.np = h->chain_np;
    ca.ncw = h->chain_ncw;
    ca.ldk = h->chain_np + 4;
    ca.rb = h->chain_rb;
    ca.uw = h->chain_uw;
    ca.grid = h->chain_grid;
    ca.from_x = 0;
    ca.in = h->act[(lo - 1) & 1];
    ca.ldi = h->ldact;
    ca.bt = h->bt;
    ca.v = v;
    const double rows = h->R;
    if (pf) pf->begin("chain_fwd", fl,
                      rows * h->dims[lo - 1] * 4.0 + (double)h->B * (h->nd - h->offs[lo - 1]) * 2.0 +
                          unst * 4.0 * (ad ? 7 : 3));
    launch_chain_fwd(ca, s);
    if (pf) pf->end();
  }
  if (v.adam && h->g_beta && h->has_conv && h->nnz > 0) {
    Vars w = v;
    w.gsplit = h->g_beta;
    if (pf) pf->begin("split_adam", 0.0, (double)h->nnz * h->m * 4.0 * 10);
    launch_split_adam(h->bt, w, h->d_split_dom, h->d_split_col, h->d_defer, h->nnz, s);
    if (pf) pf->end();
  }
  HIPCHK(hipGetLastError());
  return CV_OK;
}

// Adam moments: first / second moments of alpha and of beta (all null: the
// handle's own zeroed state).
struct AdamPtrs {
  float *ma = nullptr, *va = nullptr, *mb = nullptr, *vb = nullptr;
};

int enqueue_opt(cv_bound* h, int iters, float lr_a, float lr_b, float decay, float* alpha, float* beta,
                AdamPtrs ap, int step0, float* lb_best, float* lb_last, hipStream_t s) {
  const int64_t nb = h->nnz * h->m;
  if (!ap.ma) {
    launch_fill(h->adam, 0.f, 2 * h->n_alpha + 2 * nb, s);
    ap.ma = h->adam;
    ap.va = h->adam + h->n_alpha;
    ap.mb = h->adam + 2 * h->n_alpha;
    ap.vb = h->adam + 2 * h->n_alpha + nb;
  }
  int rc;
  // sound mode: the iterations run the plain float32 kernels, and each row's
  // best iterate is recorded (its float32 bound and its variables); the
  // reported bounds are then the float64 evaluations of that iterate and of
  // the final one (below)
  const bool snd = h->sound;
  const float* sw_saved = h->bt.sw;
  if (snd) {
    h->sound = false;
    h->bt.sw = nullptr;
  }
  float* const track = snd ? h->gbest : lb_best;
  int* const impr = snd ? h->improved : nullptr;
  // the top layer's relaxation rides on the last adjoint GEMM from the
  // second iteration on (per-layer kernels, dense top layer, no sound margin)
  const int L = h->L;
  const bool fuse = L >= 2 && h->layers[L - 2].type == CV_LAYER_DENSE && !h->chain_b && !h->chain_f && !h->sound;
  auto restore = [&]() {
    if (snd) {
      h->sound = true;
      h->bt.sw = sw_saved;
    }
  };
  for (int t = 0; t < iters; ++t) {
    if ((rc = enqueue_bwd(h, alpha, beta, true, nullptr, track, t == 0, s, fuse && t > 0, impr))) {
      restore();
      return rc;
    }
    if (snd) launch_keep_best(alpha, beta, h->abest, h->bbest, impr, h->bt, s);
    const int tt = step0 + t;
    AdamStep ad;
    ad.bc1 = (float)(1.0 - std::pow(0.9, tt + 1));
    ad.bc2 = (float)(1.0 - std::pow(0.999, tt + 1));
    const double sc = std::pow((double)decay, tt);
    ad.lr_a = (float)(lr_a * sc);
    ad.lr_b = (float)(lr_b * sc);
    ad.ma = ap.ma;
    ad.va = ap.va;
    ad.mb = ap.mb;
    ad.vb = ap.vb;
    if ((rc = enqueue_fwd(h, alpha, beta, nullptr, nullptr, &ad, s, fuse))) {
      restore();
      return rc;
    }
  }
  rc = enqueue_bwd(h, alpha, beta, false, lb_last, track, iters == 0, s, fuse && iters > 0, impr);
  if (!rc && snd) launch_keep_best(alpha, beta, h->abest, h->bbest, impr, h->bt, s);
  restore();
  if (rc) return rc;
  // sound mode: the best and the final iterates in float64 (each with its
  // rigorous float64 margin, rounded down): lb_best = the larger of the two
  if (snd && ((rc = enqueue_bwd64(h, h->abest, h->bbest, nullptr, lb_best, 1, s)) ||
              (rc = enqueue_bwd64(h, alpha, beta, lb_last, lb_best, 0, s))))
    return rc;
  HIPCHK(hipGetLastError());
  return CV_OK;
}

void drop_graph(cv_bound* h) {
  if (h->gexec) (void)hipGraphExecDestroy(h->gexec);
  h->gexec = nullptr;
  h->gkey.v.clear();
}

// The whole optimisation loop of one handle: issued directly the first time
// a set of arguments is seen, captured in a HIP graph (keyed by the
// arguments) the second time and replayed on `s` from then on.
int optimize_one(cv_bound* h, int iters, float lr_alpha, float lr_beta, float lr_decay, float* alpha, float* beta,
                 AdamPtrs ap, int step0, float* lb_best, float* lb_last, hipStream_t s) {
  int rc = ensure_opt(h);
  if (rc) return rc;
  if (h->R == 0) return CV_OK;
  GraphKey key;
  float fl[3] = {lr_alpha, lr_beta, lr_decay};
  uint32_t fb[3];
  std::memcpy(fb, fl, sizeof(fb));
  key.v = {(uintptr_t)alpha, (uintptr_t)beta, (uintptr_t)ap.ma, (uintptr_t)ap.va, (uintptr_t)ap.mb, (uintptr_t)ap.vb,
           (uintptr_t)lb_best, (uintptr_t)lb_last, (uintptr_t)iters, (uintptr_t)step0, fb[0], fb[1], fb[2]};
  if (!h->gexec || !(h->gkey == key)) {
    if (!(h->gseen == key)) {  // first time: no capture
      h->gseen = key;
      return enqueue_opt(h, iters, lr_alpha, lr_beta, lr_decay, alpha, beta, ap, step0, lb_best, lb_last, s);
    }
    drop_graph(h);
    if (!h->cap) HIPCHK(hipStreamCreateWithFlags(&h->cap, hipStreamNonBlocking));
    HIPCHK(hipStreamBeginCapture(h->cap, hipStreamCaptureModeThreadLocal));
    rc = enqueue_opt(h, iters, lr_alpha, lr_beta, lr_decay, alpha, beta, ap, step0, lb_best, lb_last, h->cap);
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamEndCapture(h->cap, &graph);
    if (rc) {
      if (graph) (void)hipGraphDestroy(graph);
      return rc;
    }
    if (e != hipSuccess) return fail(CV_EDEVICE, "graph capture failed: %s", hipGetErrorString(e));
    e = hipGraphInstantiate(&h->gexec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e != hipSuccess) {
      h->gexec = nullptr;
      return fail(CV_EDEVICE, "graph instantiation failed: %s", hipGetErrorString(e));
    }
    h->gkey = key;
  }
  HIPCHK(hipGraphLaunch(h->gexec, s));
  return CV_OK;
}

void destroy_handle(cv_bound* h);

void free_parts(cv_bound* h) {
  for (cv_bound* q : h->parts) destroy_handle(q);
  h->parts.clear();
  h->part_dom.clear();
  for (hipStream_t t : h->pstream) (void)hipStreamDestroy(t);
  h->pstream.clear();
  for (hipEvent_t e : h->pev) (void)hipEventDestroy(e);
  h->pev.clear();
}

// Split the subdomains into n contiguous ranges of (nearly) equal size, each a
// handle of its own built from the kept init arguments.
int set_parts(cv_bound* h, int n) {
  if ((int)h->parts.size() == n || (n == 1 && h->parts.empty())) return CV_OK;
  free_parts(h);
  if (n <= 1) return CV_OK;
  const cv_bound::Inputs& in = *h->in;
  h->part_dom.resize(n + 1);
  for (int i = 0; i <= n; ++i) h->part_dom[i] = (int)((int64_t)h->B * i / n);
  for (int i = 0; i < n; ++i) {
    const int b0 = h->part_dom[i], b1 = h->part_dom[i + 1];
    const int64_t s0 = in.sptr[b0];
    std::vector<int64_t> ptr(b1 - b0 + 1);
    for (int b = b0; b <= b1; ++b) ptr[b - b0] = in.sptr[b] - s0;
    std::unique_ptr<cv_bound> q(new cv_bound());
    Spec sp;
    sp.C = in.C.data();
    int rc = build(q.get(), in.layers.data(), (int)in.layers.size(), in.P, in.xlo.data(), in.xhi.data(), in.m, sp,
                   in.l.empty() ? nullptr : in.l.data(), in.u.empty() ? nullptr : in.u.data(), b1 - b0,
                   in.prop.data() + b0, ptr.data(), in.slayer.data() + s0, in.sneuron.data() + s0,
                   in.sside.data() + s0, nullptr);
    if (rc) {
      free_parts(h);
      return rc;
    }
    q->dev = h->dev;
    q->forced_tiling = h->forced_tiling;
    q->forced_conv = h->forced_conv;
    q->forced_tiles = h->forced_tiles;
    if (h->forced_tiling >= 0) assign_tiles(q.get(), h->forced_tiling);
    if (h->forced_conv >= 0 || h->forced_tiles >= 0) assign_conv_variants(q.get(), h->forced_conv);
    q->chain_b = h->chain_b ? (q->chain_lo ? 1 : 0) : 0;
    q->chain_f = h->chain_f ? (q->chain_lo && q->chain_lo + 1 <= q->L - 1 ? 1 : 0) : 0;
    h->parts.push_back(q.release());
    hipStream_t t = nullptr;
    if (hipStreamCreateWithFlags(&t, hipStreamNonBlocking) != hipSuccess) {
      free_parts(h);
      return fail(CV_EDEVICE, "stream creation failed");
    }
    h->pstream.push_back(t);
  }
  for (int i = 0; i <= n; ++i) {
    hipEvent_t e = nullptr;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      free_parts(h);
      return fail(CV_EDEVICE, "event creation failed");
    }
    h->pev.push_back(e);
  }
  // new sub-batches follow the handle's input set and sound mode
  if (h->l2) {
    for (cv_bound* q : h->parts) {
      int rc;
      if ((rc = ensure_ball(q))) return rc;
      q->l2x0 = h->l2x0;
      q->l2eps = h->l2eps;
      q->wx0 = h->wx0;
      q->l2 = true;
      q->lpq = h->lpq;
      q->bt.l2x0 = h->l2x0;
      q->bt.l2eps = h->l2eps;
      q->bt.lpq = h->lpq;
    }
  }
  if (h->sound) {
    const cv_bound::Inputs& in = *h->in;
    for (cv_bound* q : h->parts) {
      int rc = prepare_sound(q, in.layers.data(), in.xlo.data(), in.xhi.data(), in.l.data(), in.u.data(),
                             in.C.data(), false, nullptr, h->l2 ? h->hl2x0.data() : nullptr,
                             h->l2 ? h->hl2eps.data() : nullptr);
      if (rc) return rc;
      q->sound = true;
      q->bt.sw = q->sw;
      q->bt.sg = q->sound_g;
    }
  }
  return CV_OK;
}

void free_joint(cv_bound* h);

// h re-targeted to a new batch (set_batch), with everything chosen per batch
// redone: tile and conv-variant choices (they are keyed by the row count),
// the chain geometry, sound-mode and ball buffers; the optimiser graph and any
// joint state are dropped.
int update_batch(cv_bound* h, int B, const int32_t* dom_prop, const int64_t* split_ptr, const int32_t* split_layer,
                 const int32_t* split_neuron, const int8_t* split_side, hipStream_t s) {
  BatchPlan bp;
  int rc = check_batch(h, B, dom_prop, split_ptr, split_layer, split_neuron, split_side, bp);
  if (rc) return rc;
  // work still queued on any stream (the sub-batches' own ones included) may
  // read the tables about to be rewritten
  HIPCHK(hipDeviceSynchronize());
  if ((rc = set_batch(h, bp, true, s))) return rc;
  drop_graph(h);
  h->gseen = GraphKey{};
  free_joint(h);
  assign_tiles(h, h->forced_tiling);
  assign_conv_variants(h, h->forced_conv);
  if (h->chain_lo && !plan_chain(h)) {
    h->chain_lo = 0;
    h->chain_b = h->chain_f = 0;
  }
  if (h->sound && (rc = ensure_sound_batch(h))) return rc;
  if (h->l2 && (rc = ensure_ball(h))) return rc;
  return CV_OK;
}

// A new batch for h and its sub-batches (Alg. 1's rounds), keeping the
// network, properties, specifications, root bounds, input sets and modes.
int update_domains(cv_bound* h, int B, const int32_t* dom_prop, const int64_t* split_ptr, const int32_t* split_layer,
                   const int32_t* split_neuron, const int8_t* split_side, hipStream_t s) {
  int rc = update_batch(h, B, dom_prop, split_ptr, split_layer, split_neuron, split_side, s);
  if (rc) return rc;
  cv_bound::Inputs& in = *h->in;
  const int64_t nnz = B > 0 ? split_ptr[B] : 0;
  in.prop.assign(dom_prop, dom_prop + B);
  in.sptr.assign(split_ptr, split_ptr + B + 1);
  in.slayer.assign(split_layer, split_layer + nnz);
  in.sneuron.assign(split_neuron, split_neuron + nnz);
  in.sside.assign(split_side, split_side + nnz);
  in.slayer.push_back(0);  // sliced pointers stay valid for empty slices
  in.sneuron.push_back(0);
  in.sside.push_back(1);
  int n = h->parts_req > 0 ? h->parts_req : (h->R >= kPartsMinRows ? 2 : 1);
  n = std::min(n, std::max(1, B));
  if (n <= 1) {
    free_parts(h);
    return CV_OK;
  }
  if ((int)h->parts.size() != n) {
    free_parts(h);
    return set_parts(h, n);
  }
  for (int i = 0; i <= n; ++i) h->part_dom[i] = (int)((int64_t)B * i / n);
  for (int i = 0; i < n; ++i) {
    const int b0 = h->part_dom[i], b1 = h->part_dom[i + 1];
    const int64_t s0 = in.sptr[b0];
    std::vector<int64_t> ptr(b1 - b0 + 1);
    for (int b = b0; b <= b1; ++b) ptr[b - b0] = in.sptr[b] - s0;
    if ((rc = update_batch(h->parts[i], b1 - b0, in.prop.data() + b0, ptr.data(), in.slayer.data() + s0,
                           in.sneuron.data() + s0, in.sside.data() + s0, s)))
      return rc;
  }
  return CV_OK;
}

// Offsets of part i's slices in the whole batch's arrays: alpha entries,
// beta entries (split rows x m), rows.
struct PartOff {
  int64_t a0, s0, r0;
};

// Run f(part, offsets, part stream) for every part, forked from and joined
// into s.
template <class F>
int for_parts(cv_bound* h, hipStream_t s, F f) {
  const int np = (int)h->parts.size();
  HIPCHK(hipEventRecord(h->pev[np], s));
  for (int i = 0; i < np; ++i) {
    const int b0 = h->part_dom[i];
    const PartOff o{h->h_aoff[b0], h->in->sptr[b0] * h->m, (int64_t)b0 * h->m};
    HIPCHK(hipStreamWaitEvent(h->pstream[i], h->pev[np], 0));
    int rc = f(h->parts[i], o, h->pstream[i]);
    if (rc) return rc;
    HIPCHK(hipEventRecord(h->pev[i], h->pstream[i]));
    HIPCHK(hipStreamWaitEvent(s, h->pev[i], 0));
  }
  return CV_OK;
}

// Sound mode on for h and its sub-batches, the margin's weights built for the
// current input sets (boxes, or the balls set by cv_bound_set_input_l2).
int rebuild_sound(cv_bound* h, hipStream_t s) {
  const cv_bound::Inputs& in = *h->in;
  std::vector<cv_bound*> all{h};
  all.insert(all.end(), h->parts.begin(), h->parts.end());
  for (cv_bound* q : all) {
    int rc = prepare_sound(q, in.layers.data(), in.xlo.data(), in.xhi.data(), in.l.data(), in.u.data(), in.C.data(),
                           false, s, h->l2 ? h->hl2x0.data() : nullptr, h->l2 ? h->hl2eps.data() : nullptr);
    if (rc) return rc;
    q->sound = true;
    q->bt.sw = q->sw;
    q->bt.sg = q->sound_g;
    drop_graph(q);
  }
  return CV_OK;
}

void free_joint(cv_bound* h);

void destroy_handle(cv_bound* h) {
  if (!h) return;
  free_joint(h);
  free_parts(h);
  drop_graph(h);
  if (h->cap) (void)hipStreamDestroy(h->cap);
  delete h;
}

// Host copy of the init arguments (the caller's buffers may be freed after
// cv_bound_init returns).
void keep_inputs(cv_bound* h, const cv_layer* layers, int n_layers, int P, const float* x_lo, const float* x_hi,
                 int m, const float* C, const float* l, const float* u, int B, const int32_t* dom_prop,
                 const int64_t* split_ptr, const int32_t* split_layer, const int32_t* split_neuron,
                 const int8_t* split_side) {
  std::unique_ptr<cv_bound::Inputs> in(new cv_bound::Inputs());
  in->layers.assign(layers, layers + n_layers);
  in->w.resize(n_layers);
  in->b.resize(n_layers);
  for (int i = 0; i < n_layers; ++i) {
    const cv_layer& ly = layers[i];
    const size_t nw = ly.type == CV_LAYER_DENSE ? (size_t)ly.out_c * ly.in_c
                                                 : (size_t)ly.out_c * ly.in_c * ly.kernel * ly.kernel;
    in->w[i].assign(ly.weight, ly.weight + nw);
    in->b[i].assign(ly.bias, ly.bias + ly.out_c);
    in->layers[i].weight = in->w[i].data();
    in->layers[i].bias = in->b[i].data();
  }
  const int d0 = h->d0, dL = h->dims[n_layers], nd = h->nd;
  in->P = P;
  in->m = m;
  in->xlo.assign(x_lo, x_lo + (size_t)P * d0);
  in->xhi.assign(x_hi, x_hi + (size_t)P * d0);
  in->C.assign(C, C + (size_t)P * m * dL);
  if (l) in->l.assign(l, l + (size_t)P * nd);
  if (u) in->u.assign(u, u + (size_t)P * nd);
  in->prop.assign(dom_prop, dom_prop + B);
  in->sptr.assign(split_ptr, split_ptr + B + 1);
  const int64_t nnz = split_ptr[B];
  if (nnz > 0) {
    in->slayer.assign(split_layer, split_layer + nnz);
    in->sneuron.assign(split_neuron, split_neuron + nnz);
    in->sside.assign(split_side, split_side + nnz);
  }
  // sliced pointers must stay valid for empty slices
  in->slayer.push_back(0);
  in->sneuron.push_back(0);
  in->sside.push_back(1);
  h->in = std::move(in);
}

}  // namespace

// ---------------------------------------------------------------------------
// Workspace of cv_bound_grad_noalloc: one static device array per GPU, held
// until the process ends.  Its host-side name is not a device address: host
// code uses only the address hipGetSymbolAddress returns for the current
// device, resolved once per device at cv_bound_init.

constexpr size_t kScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int resolve_scratch(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return fail(CV_EDEVICE, "device %d out of range", dev);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_ptr[dev]) return CV_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p) {
    (void)hipGetLastError();
    return fail(CV_EDEVICE, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
  }
  g_scratch_ptr[dev] = p;
  return CV_OK;
}

// The gradient pass with every workspace buffer carved from the static array
// (256-byte aligned pieces): the two activation buffers, the partial slots,
// the stored A at unstable neurons, x* (sign planes and/or dense rows) and
// the sound-mode / l2-ball partials.  Every piece is written by the pass
// before it is read, so nothing needs clearing.  The handle's own buffers are
// swapped out for the launches and restored afterwards (kernel arguments are
// taken at launch).
int grad_noalloc(cv_bound* h, const float* alpha, const float* beta, float* lb, float* g_alpha, float* g_beta,
                 hipStream_t s) {
  void* base = nullptr;
  {
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    base = (h->dev >= 0 && h->dev < kMaxDevices) ? g_scratch_ptr[h->dev] : nullptr;
  }
  if (!base) return fail(CV_EDEVICE, "static workspace not resolved for device %d", h->dev);
  const size_t R = (size_t)std::max(1, h->R);
  const bool dense1 = h->layers[0].type == CV_LAYER_DENSE;
  const int ldx = r4(h->d0);
  // the register tiles' sign planes may be wider than the input: a batch that
  // fits only without them runs the first layer's older kernels
  DevLayer& first = h->layers[0];
  const int reg_b = first.bwd.reg.on, reg_f = first.fwd.reg.on, w64_reg = h->w64, w64_in = (h->d0 + 63) / 64;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += (bytes + 255) & ~(size_t)255;
    return at;
  };
  const size_t o_act0 = h->L >= 2 ? take(R * h->ldact * sizeof(float)) : 0;
  const size_t o_act1 = h->L >= 2 ? take(R * h->ldact * sizeof(float)) : 0;
  const size_t o_part = take(R * h->n_slots * sizeof(float));
  const size_t o_acomp = take((size_t)std::max<int64_t>(1, h->n_alpha) * sizeof(float));
  const bool need_xd = dense1 || h->l2;
  const size_t o_xd = need_xd ? take(R * ldx * sizeof(float)) : 0;
  const size_t o_perr = h->sound ? take(R * h->n_slots * sizeof(float)) : 0;
  const size_t o_psq = h->l2 ? take(R * h->n_slots * sizeof(float)) : 0;
  const size_t o_l2s = h->l2 ? take(R * sizeof(float)) : 0;
  const size_t before = off;
  size_t o_xpos = take(R * h->w64 * sizeof(uint64_t)), o_xneg = take(R * h->w64 * sizeof(uint64_t));
  const bool narrow = off > kScratchBytes && w64_reg > w64_in;
  if (narrow) {
    off = before;
    o_xpos = take(R * w64_in * sizeof(uint64_t));
    o_xneg = take(R * w64_in * sizeof(uint64_t));
  }
  if (off > kScratchBytes)
    return fail(CV_ENOMEM, "cv_bound_grad_noalloc: this batch needs %zu bytes of workspace, the static array holds %zu",
                off, kScratchBytes);
  unsigned char* b = static_cast<unsigned char*>(base);
  struct Saved {
    float *act0, *act1, *part, *acomp, *xdense, *perr, *psq, *l2s;
    uint64_t *xpos, *xneg;
    int ldx;
  } sv{h->act[0], h->act[1], h->part, h->acomp, h->xdense, h->perr, h->psq, h->l2s, h->xpos, h->xneg, h->ldx};
  if (h->L >= 2) {
    h->act[0] = reinterpret_cast<float*>(b + o_act0);
    h->act[1] = reinterpret_cast<float*>(b + o_act1);
  }
  h->part = reinterpret_cast<float*>(b + o_part);
  h->acomp = reinterpret_cast<float*>(b + o_acomp);
  h->xpos = reinterpret_cast<uint64_t*>(b + o_xpos);
  h->xneg = reinterpret_cast<uint64_t*>(b + o_xneg);
  if (need_xd) {
    h->xdense = reinterpret_cast<float*>(b + o_xd);
    h->ldx = ldx;
  }
  if (h->sound) h->perr = reinterpret_cast<float*>(b + o_perr);
  if (h->l2) {
    h->psq = reinterpret_cast<float*>(b + o_psq);
    h->l2s = reinterpret_cast<float*>(b + o_l2s);
  }
  if (narrow) {
    first.bwd.reg.on = first.fwd.reg.on = 0;
    h->w64 = h->bt.w64 = w64_in;
  }
  int rc = enqueue_bwd(h, alpha, beta, true, lb, nullptr, 0, s);
  if (!rc) rc = enqueue_fwd(h, alpha, beta, g_alpha, g_beta, nullptr, s);
  first.bwd.reg.on = reg_b;
  first.fwd.reg.on = reg_f;
  h->w64 = h->bt.w64 = w64_reg;
  // sound mode: the float64 bound (its buffers were allocated when sound
  // mode was switched on)
  if (!rc && h->sound) rc = enqueue_bwd64(h, alpha, beta, lb, nullptr, 0, s);
  h->act[0] = sv.act0;
  h->act[1] = sv.act1;
  h->part = sv.part;
  h->acomp = sv.acomp;
  h->xdense = sv.xdense;
  h->perr = sv.perr;
  h->psq = sv.psq;
  h->l2s = sv.l2s;
  h->xpos = sv.xpos;
  h->xneg = sv.xneg;
  h->ldx = sv.ldx;
  return rc;
}

// ===========================================================================
// ABI

namespace {

// Root bounds of every ReLU layer, one sub-network at a time (layers 1..i,
// specification [I; -I] on layer i); sound: evaluated as sound mode does (float64
// with a rigorous rounding margin, rounded outward).
int root_bounds(const cv_layer* layers, int32_t n_layers, int32_t n_props, const float* x_lo, const float* x_hi,
                float* l_out, float* u_out, bool sound, void* stream, int iters = 0, float lr_alpha = 0.f,
                float decay = 1.f) {
  if (iters < 0 || !std::isfinite(lr_alpha) || !std::isfinite(decay)) return fail(CV_EINVAL, "bad optimiser settings");
  std::vector<int> dims;
  int rc = check_layers(layers, n_layers, dims);
  if (rc) return rc;
  if (n_props <= 0 || !x_lo || !x_hi) return fail(CV_EINVAL, "bad arguments");
  int nd = 0;
  for (int i = 1; i < n_layers; ++i) nd += dims[i];
  if (nd > 0 && (!l_out || !u_out)) return fail(CV_EINVAL, "null outputs");
  hipStream_t s = (hipStream_t)stream;
  std::vector<float> lo((size_t)n_props * nd, 0.f), up((size_t)n_props * nd, 0.f);
  std::vector<int32_t> prop(n_props);
  std::vector<int64_t> sptr(n_props + 1, 0);
  for (int p = 0; p < n_props; ++p) prop[p] = p;
  int off = 0;
  DevMem mem, bm;  // device memory of one sub-network after the other
  for (int i = 1; i < n_layers; ++i) {
    // sub-network of layers 1..i with specification [I; -I] on layer i
    const int d = dims[i];
    std::vector<cv_layer> sub(layers, layers + i);
    int ndp = off;  // bounds of layers 1..i-1
    std::vector<float> lsub((size_t)n_props * std::max(1, ndp)), usub((size_t)n_props * std::max(1, ndp));
    for (int p = 0; p < n_props; ++p)
      for (int j = 0; j < ndp; ++j) {
        lsub[(size_t)p * ndp + j] = lo[(size_t)p * nd + j];
        usub[(size_t)p * ndp + j] = up[(size_t)p * nd + j];
      }
    cv_bound hb;
    hb.mem.take(mem);
    hb.bm.take(bm);
    hb.bm.keep = true;
    hb.mem.peer = &hb.bm;
    hb.bm.peer = &hb.mem;
    Spec sp;
    sp.identity = true;
    rc = build(&hb, sub.data(), i, n_props, x_lo, x_hi, 2 * d, sp, lsub.data(), usub.data(), n_props, prop.data(),
               sptr.data(), nullptr, nullptr, nullptr, s);
    if (rc) return rc;
    if (sound) {  // the bounds come from the float64 pass with its margin, rounded outward
      if ((rc = prepare_sound(&hb, sub.data(), x_lo, x_hi, lsub.data(), usub.data(), nullptr, true, s))) return rc;
      hb.sound = true;
      hb.bt.sw = hb.sw;
      hb.bt.sg = hb.sound_g;
    }
    float* dlb;
    if ((rc = hb.mem.alloc(&dlb, (size_t)hb.R))) return rc;
    if (iters > 0 && hb.n_alpha > 0) {
      // each of the 2d bounds (rows) has its own alpha' for every unstable
      // neuron below: projected Adam from CROWN's default, best iterate kept
      float *alpha, *dlast;
      if ((rc = ensure_opt(&hb)) || (rc = hb.mem.alloc(&alpha, (size_t)hb.n_alpha)) ||
          (rc = hb.mem.alloc(&dlast, (size_t)hb.R)))
        return rc;
      launch_alpha_default(alpha, hb.ulist, hb.uoff, hb.bt, s);
      if ((rc = enqueue_opt(&hb, iters, lr_alpha, 0.f, decay, alpha, nullptr, AdamPtrs{}, 0, dlb, dlast, s)))
        return rc;
    } else if ((rc = sound ? enqueue_bwd64(&hb, nullptr, nullptr, dlb, nullptr, 0, s)
                           : enqueue_bwd(&hb, nullptr, nullptr, false, dlb, nullptr, 0, s))) {
      return rc;
    }
    std::vector<float> lb(hb.R);
    HIPCHK(hipMemcpyAsync(lb.data(), dlb, (size_t)hb.R * sizeof(float), hipMemcpyDeviceToHost, s));
    HIPCHK(hipStreamSynchronize(s));
    for (int p = 0; p < n_props; ++p)
      for (int j = 0; j < d; ++j) {
        lo[(size_t)p * nd + off + j] = lb[(size_t)p * 2 * d + j];
        up[(size_t)p * nd + off + j] = -lb[(size_t)p * 2 * d + d + j];
      }
    drop_graph(&hb);
    mem.take(hb.mem);
    bm.take(hb.bm);
    off += d;
  }
  for (size_t t = 0; t < lo.size(); ++t) {
    l_out[t] = lo[t];
    u_out[t] = up[t];
  }
  return CV_OK;
}

// ---------------------------------------------------------------------------
// Joint optimisation of intermediate bounds (Sec. 3.3, Eq. opt_non_convex).
// Every subdomain's bounds of ReLU layers 2..L-1 are recomputed in each
// iteration as beta-CROWN bounds of the sub-network ending at that layer
// (specification [I; -I]), with variables alpha', beta' shared by the layer's
// neurons per bound side; they replace the root bounds where tighter and feed
// the relaxation of the final objective.  The gradient of sum g reaches
// alpha', beta' through the bounds: d g / d l, d u at each unstable neuron
// (launch_joint_cot) weighs the rows of the layer's pass, whose per-row
// gradients are summed onto the shared variables (launch_joint_reduce), and
// the pass's own bounds' gradient flows on to the layers below it.
// Each pass is a handle of its own with one "property" per subdomain, so its
// relaxation tables (status, chord) are per subdomain and are refreshed from
// the current bounds before it runs.

}  // namespace

struct JointLayer {
  cv_bound* h = nullptr;  // layers 1..i, specification [I; -I], the splits below layer i
  int i = 0, d = 0, off = 0;
  int64_t nnz = 0, n_ash = 0;
  float *arow = nullptr, *brow = nullptr, *garow = nullptr, *gbrow = nullptr;  // per-row copies
  float *ash = nullptr, *bsh = nullptr, *gash = nullptr, *gbsh = nullptr;      // shared [sum_b 2 uc_b], [nnz][2]
  float *ma = nullptr, *va = nullptr, *mb = nullptr, *vb = nullptr;            // Adam moments of ash, bsh
  float *lb = nullptr, *w = nullptr;                                           // [B][2d] row bounds, weights
  uint32_t* st0 = nullptr;  // status words at the root bounds
};

struct cv_bound::Joint {
  cv_bound* hm = nullptr;  // the final objective, one property per subdomain
  uint32_t* st0m = nullptr;
  std::vector<JointLayer> lay;
  DevMem mem;
  float *lroot = nullptr, *uroot = nullptr, *lcur = nullptr, *ucur = nullptr, *dL = nullptr, *dU = nullptr;
  uint8_t *ml = nullptr, *mu = nullptr;
  float *ga = nullptr, *gb = nullptr, *ma = nullptr, *va = nullptr, *mb = nullptr, *vb = nullptr;
  float* lb = nullptr;  // [R] bounds of the current iterate
  ~Joint() {
    destroy_handle(hm);
    for (JointLayer& q : lay) destroy_handle(q.h);
  }
};

namespace {

void free_joint(cv_bound* h) {
  delete h->joint;
  h->joint = nullptr;
}

// The conv kernels of a joint pass: its bounds feed its own relaxations, where
// a constant summed in another order is another trajectory, so
// back-substitution (and with it the first layer's sign planes) stays on the
// row-order kernels; the adjoint above the first layer, whose sums over k do
// not depend on the kernel, runs on its own plan (register tiles in one K chunk,
// as in the row-major kernel that also stores zbar).
void joint_conv_plans(cv_bound* x) {
  for (int i = 0; i < x->L; ++i) {
    DevLayer& d = x->layers[i];
    if (d.type != CV_LAYER_CONV2D) continue;
    d.bwd.reg.on = 0;
    if (i == 0) d.fwd.reg.on = 0;
    d.fwd.reg.ksp = 1;
  }
}

// The joint state of h, built from its kept init arguments on first use.
int make_joint(cv_bound* h, hipStream_t s) {
  if (h->joint) return CV_OK;
  const cv_bound::Inputs& in = *h->in;
  const int B = h->B, nd = h->nd, L = h->L, m = h->m, d0 = h->d0, dL = h->dims[L];
  if (in.l.empty()) return fail(CV_EINVAL, "joint optimisation needs the handle's root bounds");
  std::unique_ptr<cv_bound::Joint> J(new cv_bound::Joint());
  // one property per subdomain: its box, specification and root bounds
  std::vector<float> xlo((size_t)B * d0), xhi((size_t)B * d0), C((size_t)B * m * dL), lr((size_t)B * nd),
      ur((size_t)B * nd);
  std::vector<int32_t> ident(B);
  for (int b = 0; b < B; ++b) {
    const int p = in.prop[b];
    ident[b] = b;
    std::copy(in.xlo.begin() + (size_t)p * d0, in.xlo.begin() + (size_t)(p + 1) * d0, xlo.begin() + (size_t)b * d0);
    std::copy(in.xhi.begin() + (size_t)p * d0, in.xhi.begin() + (size_t)(p + 1) * d0, xhi.begin() + (size_t)b * d0);
    std::copy(in.C.begin() + (size_t)p * m * dL, in.C.begin() + (size_t)(p + 1) * m * dL, C.begin() + (size_t)b * m * dL);
    std::copy(in.l.begin() + (size_t)p * nd, in.l.begin() + (size_t)(p + 1) * nd, lr.begin() + (size_t)b * nd);
    std::copy(in.u.begin() + (size_t)p * nd, in.u.begin() + (size_t)(p + 1) * nd, ur.begin() + (size_t)b * nd);
  }
  int rc;
  J->hm = new cv_bound();
  Spec sp;
  sp.C = C.data();
  if ((rc = build(J->hm, in.layers.data(), L, B, xlo.data(), xhi.data(), m, sp, lr.data(), ur.data(), B,
                  ident.data(), in.sptr.data(), in.slayer.data(), in.sneuron.data(), in.sside.data(), s)))
    return rc;
  if (J->hm->n_alpha != h->n_alpha || J->hm->nnz != h->nnz) return fail(CV_EINVAL, "joint layout mismatch");
  cv_bound* hm = J->hm;
  joint_conv_plans(hm);
  DevMem& M = J->mem;
  const size_t bnd = (size_t)std::max(1, B * nd);
  if ((rc = ensure_grad(hm)) || (rc = hm->mem.alloc(&hm->zchord, hm->n_alpha)) ||
      (rc = M.upload(&J->lroot, lr.data(), lr.size(), s)) || (rc = M.upload(&J->uroot, ur.data(), ur.size(), s)) ||
      (rc = M.alloc(&J->lcur, bnd)) || (rc = M.alloc(&J->ucur, bnd)) || (rc = M.alloc(&J->dL, bnd)) ||
      (rc = M.alloc(&J->dU, bnd)) || (rc = M.alloc(&J->ml, bnd)) || (rc = M.alloc(&J->mu, bnd)) ||
      (rc = M.alloc(&J->ga, h->n_alpha)) || (rc = M.alloc(&J->gb, h->nnz * m)) ||
      (rc = M.alloc(&J->ma, h->n_alpha)) || (rc = M.alloc(&J->va, h->n_alpha)) ||
      (rc = M.alloc(&J->mb, h->nnz * m)) || (rc = M.alloc(&J->vb, h->nnz * m)) ||
      (rc = M.alloc(&J->lb, std::max(1, h->R))) || (rc = M.alloc(&J->st0m, (size_t)std::max(1, B * nd))))
    return rc;
  HIPCHK(hipMemcpyAsync(J->st0m, hm->bt.status, sizeof(uint32_t) * B * nd, hipMemcpyDeviceToDevice, s));
  // the pass of each intermediate layer i = 2..L-1
  for (int i = 2; i <= L - 1; ++i) {
    JointLayer q;
    q.i = i;
    q.d = h->dims[i];
    q.off = h->offs[i - 1];
    const int ndx = q.off;  // ReLU layers 1..i-1
    std::vector<float> lsub((size_t)B * ndx), usub((size_t)B * ndx);
    for (int b = 0; b < B; ++b)
      for (int c = 0; c < ndx; ++c) {
        lsub[(size_t)b * ndx + c] = lr[(size_t)b * nd + c];
        usub[(size_t)b * ndx + c] = ur[(size_t)b * nd + c];
      }
    std::vector<int64_t> ptr(B + 1, 0);
    std::vector<int32_t> sl, sn;
    std::vector<int8_t> ss;
    for (int b = 0; b < B; ++b) {
      for (int64_t t = in.sptr[b]; t < in.sptr[b + 1]; ++t)
        if (in.slayer[t] < i) {
          sl.push_back(in.slayer[t]);
          sn.push_back(in.sneuron[t]);
          ss.push_back(in.sside[t]);
        }
      ptr[b + 1] = (int64_t)sl.size();
    }
    q.nnz = ptr[B];
    sl.push_back(0);
    sn.push_back(0);
    ss.push_back(1);
    q.h = new cv_bound();
    J->lay.push_back(q);  // owned by J from here on
    JointLayer& Q = J->lay.back();
    Spec si;
    si.identity = true;
    if ((rc = build(Q.h, in.layers.data(), i, B, xlo.data(), xhi.data(), 2 * Q.d, si, lsub.data(), usub.data(), B,
                    ident.data(), ptr.data(), sl.data(), sn.data(), ss.data(), s)))
      return rc;
    cv_bound* x = Q.h;
    joint_conv_plans(x);
    Q.n_ash = x->n_alpha / Q.d;  // 2 uc_b per subdomain
    const int64_t nb = Q.nnz * 2 * Q.d;
    if ((rc = ensure_grad(x)) || (rc = x->mem.alloc(&x->zchord, x->n_alpha)) ||
        (rc = M.alloc(&Q.arow, x->n_alpha)) || (rc = M.alloc(&Q.brow, nb)) || (rc = M.alloc(&Q.garow, x->n_alpha)) ||
        (rc = M.alloc(&Q.gbrow, nb)) || (rc = M.alloc(&Q.ash, Q.n_ash)) || (rc = M.alloc(&Q.bsh, Q.nnz * 2)) ||
        (rc = M.alloc(&Q.gash, Q.n_ash)) || (rc = M.alloc(&Q.gbsh, Q.nnz * 2)) || (rc = M.alloc(&Q.ma, Q.n_ash)) ||
        (rc = M.alloc(&Q.va, Q.n_ash)) || (rc = M.alloc(&Q.mb, Q.nnz * 2)) || (rc = M.alloc(&Q.vb, Q.nnz * 2)) ||
        (rc = M.alloc(&Q.lb, std::max(1, x->R))) || (rc = M.alloc(&Q.w, std::max(1, x->R))) ||
        (rc = M.alloc(&Q.st0, (size_t)std::max(1, B * ndx))))
      return rc;
    HIPCHK(hipMemcpyAsync(Q.st0, x->bt.status, sizeof(uint32_t) * B * ndx, hipMemcpyDeviceToDevice, s));
  }
  HIPCHK(hipStreamSynchronize(s));
  h->joint = J.release();
  return CV_OK;
}

// Status / chords of pass x (its first nd_x columns) from the current bounds.
void joint_refresh(cv_bound::Joint* J, cv_bound* x, const uint32_t* st0, int nd, hipStream_t s) {
  launch_joint_refresh(const_cast<uint32_t*>(x->bt.status), st0, const_cast<float2*>(x->bt.chord), J->lcur, J->ucur,
                       x->B, x->nd, nd, s);
}

// One forward phase: every intermediate layer's bounds from the shared
// variables (with the per-row gradients of each pass when grad), then the
// final objective's bounds into lb (its gradients into J->ga, J->gb when grad).
int joint_forward(cv_bound* h, const float* alpha, const float* beta, bool grad, float* lb, float* best, int first,
                  hipStream_t s) {
  cv_bound::Joint* J = h->joint;
  const int B = h->B, nd = h->nd;
  int rc;
  for (JointLayer& q : J->lay) {
    cv_bound* x = q.h;
    joint_refresh(J, x, q.st0, nd, s);
    launch_joint_bcast(q.arow, q.ash, q.brow, q.bsh, x->bt, q.d, q.nnz, s);
    if ((rc = enqueue_bwd(x, q.arow, q.brow, grad, q.lb, nullptr, 0, s))) return rc;
    if (grad) {
      launch_fill(q.garow, 0.f, x->n_alpha, s);  // entries of neurons made stable are not written
      if ((rc = enqueue_fwd(x, q.arow, q.brow, q.garow, q.gbrow, nullptr, s))) return rc;
    }
    launch_joint_clip(q.lb, q.d, q.off, J->lroot, J->uroot, J->lcur, J->ucur, J->ml, J->mu, B, nd, s);
  }
  cv_bound* hm = J->hm;
  joint_refresh(J, hm, J->st0m, nd, s);
  if ((rc = enqueue_bwd(hm, alpha, beta, grad, lb, best, first, s))) return rc;
  if (grad) {
    launch_fill(J->ga, 0.f, h->n_alpha, s);
    if ((rc = enqueue_fwd(hm, alpha, beta, J->ga, J->gb, nullptr, s))) return rc;
  }
  HIPCHK(hipGetLastError());
  return CV_OK;
}

// The reverse phase: d(sum g)/d(l, u) from the final objective's pass, then
// layer by layer from the top: row weights, shared gradients, and the pass's
// own contribution to the bounds' gradients of the layers below it.
void joint_reverse(cv_bound* h, hipStream_t s) {
  cv_bound::Joint* J = h->joint;
  const int B = h->B, nd = h->nd, col0 = h->L > 2 ? h->dims[1] : nd;
  cv_bound* hm = J->hm;
  launch_fill(J->dL, 0.f, (int64_t)B * nd, s);
  launch_fill(J->dU, 0.f, (int64_t)B * nd, s);
  launch_joint_cot(J->dL, J->dU, hm->bt.status, hm->acomp, hm->zchord, nullptr, J->lcur, J->ucur, hm->bt, col0, nd,
                   nd, B, s);
  for (int t = (int)J->lay.size() - 1; t >= 0; --t) {
    JointLayer& q = J->lay[t];
    cv_bound* x = q.h;
    launch_joint_weights(q.w, J->dL, J->dU, J->ml, J->mu, B, q.d, q.off, nd, s);
    const int ucmax = *std::max_element(x->h_ucount.begin(), x->h_ucount.end());
    launch_joint_reduce(q.gash, q.garow, q.gbsh, q.gbrow, q.w, x->bt, B, q.d, ucmax, x->d_split_dom, q.nnz, s);
    launch_joint_cot(J->dL, J->dU, x->bt.status, x->acomp, x->zchord, q.w, J->lcur, J->ucur, x->bt, col0, x->nd, nd,
                     B, s);
  }
}

int optimize_joint(cv_bound* h, int iters, float lr_a, float lr_b, float decay, float* alpha, float* beta,
                   float* lb_best, float* lb_last, float* l_out, float* u_out, hipStream_t s) {
  int rc = make_joint(h, s);
  if (rc) return rc;
  cv_bound::Joint* J = h->joint;
  const int B = h->B, nd = h->nd;
  const int64_t nb = h->nnz * h->m;
  // fresh start of the intermediate variables and of every Adam moment
  HIPCHK(hipMemcpyAsync(J->lcur, J->lroot, sizeof(float) * B * nd, hipMemcpyDeviceToDevice, s));
  HIPCHK(hipMemcpyAsync(J->ucur, J->uroot, sizeof(float) * B * nd, hipMemcpyDeviceToDevice, s));
  for (JointLayer& q : J->lay) {
    launch_joint_alpha_init(q.ash, q.h->ulist, q.h->uoff, q.h->bt, B, q.d, s);
    launch_fill(q.bsh, 0.f, q.nnz * 2, s);
    launch_fill(q.gash, 0.f, q.n_ash, s);
    launch_fill(q.gbsh, 0.f, q.nnz * 2, s);
    for (float* z : {q.ma, q.va}) launch_fill(z, 0.f, q.n_ash, s);
    for (float* z : {q.mb, q.vb}) launch_fill(z, 0.f, q.nnz * 2, s);
  }
  for (float* z : {J->ma, J->va}) launch_fill(z, 0.f, h->n_alpha, s);
  for (float* z : {J->mb, J->vb}) launch_fill(z, 0.f, nb, s);
  for (int t = 0; t < iters; ++t) {
    if ((rc = joint_forward(h, alpha, beta, true, J->lb, lb_best, t == 0, s))) return rc;
    joint_reverse(h, s);
    const float bc1 = (float)(1.0 - std::pow(0.9, t + 1)), bc2 = (float)(1.0 - std::pow(0.999, t + 1));
    const float la = (float)(lr_a * std::pow((double)decay, t)), lb = (float)(lr_b * std::pow((double)decay, t));
    launch_adam(alpha, J->ga, J->ma, J->va, h->n_alpha, la, bc1, bc2, 0.f, 1.f, s);
    launch_adam(beta, J->gb, J->mb, J->vb, nb, lb, bc1, bc2, 0.f, INFINITY, s);
    for (JointLayer& q : J->lay) {
      launch_adam(q.ash, q.gash, q.ma, q.va, q.n_ash, la, bc1, bc2, 0.f, 1.f, s);
      launch_adam(q.bsh, q.gbsh, q.mb, q.vb, q.nnz * 2, lb, bc1, bc2, 0.f, INFINITY, s);
    }
  }
  // the final iterate, evaluated once more
  if ((rc = joint_forward(h, alpha, beta, false, lb_last ? lb_last : J->lb, lb_best, iters == 0, s))) return rc;
  if (l_out) HIPCHK(hipMemcpyAsync(l_out, J->lcur, sizeof(float) * B * nd, hipMemcpyDeviceToDevice, s));
  if (u_out) HIPCHK(hipMemcpyAsync(u_out, J->ucur, sizeof(float) * B * nd, hipMemcpyDeviceToDevice, s));
  HIPCHK(hipGetLastError());
  return CV_OK;
}

}  // namespace

extern "C" {

const char* cv_last_error(void) { return g_err.c_str(); }

int cv_bound_init(cv_bound** out, const cv_layer* layers, int32_t n_layers, int32_t n_props, const float* x_lo,
                  const float* x_hi, int32_t m, const float* C, const float* l, const float* u, int32_t n_dom,
                  const int32_t* dom_prop, const int64_t* split_ptr, const int32_t* split_layer,
                  const int32_t* split_neuron, const int8_t* split_side, void* stream) {
  if (!out) return fail(CV_EINVAL, "null handle pointer");
  *out = nullptr;
  if (!C) return fail(CV_EINVAL, "null specification");
  if (split_ptr && n_dom > 0 && split_ptr[n_dom] > 0 && (!split_layer || !split_neuron || !split_side))
    return fail(CV_EINVAL, "null split arrays");
  // no intermediate bounds given: per-layer CROWN on the GPU (as
  // cv_bound_root_bounds), computed once here for every property
  std::vector<float> lroot, uroot;
  if (!l || !u) {
    std::vector<int> dims;
    int rc0 = check_layers(layers, n_layers, dims);
    if (rc0) return rc0;
    if (n_props <= 0 || !x_lo || !x_hi) return fail(CV_EINVAL, "bad arguments");
    int nd = 0;
    for (int i = 1; i < n_layers; ++i) nd += dims[i];
    lroot.assign((size_t)n_props * std::max(nd, 1), 0.f);
    uroot.assign((size_t)n_props * std::max(nd, 1), 0.f);
    if (nd > 0 && (rc0 = root_bounds(layers, n_layers, n_props, x_lo, x_hi, lroot.data(), uroot.data(), false,
                                     stream)))
      return rc0;
    l = lroot.data();
    u = uroot.data();
  }
  std::unique_ptr<cv_bound> h(new cv_bound());
  Spec sp;
  sp.C = C;
  int rc = build(h.get(), layers, n_layers, n_props, x_lo, x_hi, m, sp, l, u, n_dom, dom_prop, split_ptr,
                 split_layer, split_neuron, split_side, (hipStream_t)stream);
  if (rc) return rc;
  // the device of this handle, and the address of its static workspace there
  HIPCHK(hipGetDevice(&h->dev));
  if ((rc = resolve_scratch(h->dev))) return rc;
  keep_inputs(h.get(), layers, n_layers, n_props, x_lo, x_hi, m, C, l, u, n_dom, dom_prop, split_ptr, split_layer,
              split_neuron, split_side);
  // large batches: two concurrent halves in the optimiser (their kernels
  // overlap each other's tails and launch gaps)
  if (h->R >= kPartsMinRows && (rc = set_parts(h.get(), 2))) return rc;
  *out = h.release();
  return CV_OK;
}

int cv_bound_sizes(const cv_bound* h, int64_t* n_alpha, int64_t* n_beta, int64_t* n_rows) {
  if (!h) return fail(CV_EINVAL, "null handle");
  if (n_alpha) *n_alpha = h->n_alpha;
  if (n_beta) *n_beta = h->nnz * h->m;
  if (n_rows) *n_rows = h->R;
  return CV_OK;
}

int64_t cv_bound_alpha_offset(const cv_bound* h, int32_t dom, int32_t row, int32_t layer, int32_t neuron) {
  if (!h || dom < 0 || dom >= h->B || row < 0 || row >= h->m || layer < 1 || layer >= h->L || neuron < 0 ||
      neuron >= h->dims[layer])
    return -1;
  const int p = h->h_prop[dom];
  const int c = h->h_cidx[(size_t)p * h->nd + h->offs[layer - 1] + neuron];
  if (c < 0) return -1;
  return h->h_aoff[dom] + (int64_t)row * h->h_ucount[p] + c;
}

int cv_bound_alpha_init(cv_bound* h, float* alpha, void* stream) {
  if (!h || (!alpha && h->n_alpha > 0)) return fail(CV_EINVAL, "null argument");
  launch_alpha_default(alpha, h->ulist, h->uoff, h->bt, (hipStream_t)stream);
  HIPCHK(hipGetLastError());
  return CV_OK;
}

// The network's own forward pass at each row's x* (left by a gradient-style
// back-substitution in xdense or the sign planes): exact ReLU, split checks
// into sat, then ub = C_p (W(L) zhat(L-1) + b(L)).  Per-layer kernels only.
int enqueue_true_fwd(cv_bound* h, float* ub, int32_t* sat, hipStream_t s) {
  const int L = h->L;
  launch_fill_i32(sat, 1, h->R, s);
  Vars v{};
  v.xpos = h->xpos;
  v.xneg = h->xneg;
  v.sat = sat;
  for (int i = 1; i <= L - 1; ++i) {
    const DevLayer& ly = h->layers[i - 1];
    Epi e = make_epi(h);
    e.layer_off = h->offs[i - 1];
    e.bias = ly.bias;
    e.n = h->dims[i];
    e.out = h->act[i & 1];
    int mode, lda;
    const float* in;
    first_layer_input(h, i, v, e, in, lda, mode);
    const int N = h->dims[i], K = h->dims[i - 1];
    if (ly.type == CV_LAYER_DENSE) {
      const int c = h->cfg[L + i - 1] >= 0 ? h->cfg[L + i - 1] : 0;
      GemmArgs g{in, lda, ly.W, ly.ld_in, h->R, N, K, 0, h->bt, v, e};
      launch_gemm(c, mode, g, s);
    } else {
      ConvArgs a{in, lda, ly.fwd, h->R, 0, h->bt, v, e};
      if (launch_conv_fwd(mode, a, s)) return fail(CV_ESHAPE, "unsupported conv channels");
    }
  }
  TopArgs ta{};
  ta.CW = h->CW;
  ta.cw_pstride = h->cw_pstride;
  ta.ldcw = h->ldcw;
  ta.Cb = h->Cb;
  ta.cb_pstride = h->cb_pstride;
  ta.n = h->dims[L - 1];
  ta.bt = h->bt;
  launch_top_dot(ta, h->act[(L - 1) & 1], h->ldact, ub, s);
  HIPCHK(hipGetLastError());
  return CV_OK;
}

int cv_bound_eval(cv_bound* h, const float* alpha, const float* beta, float* lb, void* stream) {
  if (!h || (!lb && h->R > 0) || (!alpha && h->n_alpha > 0) || (!beta && h->nnz > 0))
    return fail(CV_EINVAL, "null argument");
  hipStream_t s = (hipStream_t)stream;
  if (h->sound) return enqueue_bwd64(h, alpha, beta, lb, nullptr, 0, s);
  return enqueue_bwd(h, alpha, beta, false, lb, nullptr, 0, s);
}

int cv_bound_grad(cv_bound* h, const float* alpha, const float* beta, float* lb, float* g_alpha, float* g_beta,
                  void* stream) {
  if (!h || (!lb && h->R > 0) || (!alpha && h->n_alpha > 0) || (!beta && h->nnz > 0) || (!g_alpha && h->n_alpha > 0) ||
      (!g_beta && h->nnz > 0))
    return fail(CV_EINVAL, "null argument");
  int rc = ensure_grad(h);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  if ((rc = enqueue_bwd(h, alpha, beta, true, lb, nullptr, 0, s))) return rc;
  if ((rc = enqueue_fwd(h, alpha, beta, g_alpha, g_beta, nullptr, s))) return rc;
  return h->sound ? enqueue_bwd64(h, alpha, beta, lb, nullptr, 0, s) : CV_OK;
}

int cv_bound_grad_noalloc(cv_bound* h, const float* alpha, const float* beta, float* lb, float* g_alpha,
                          float* g_beta, void* stream) {
  if (!h || (!lb && h->R > 0) || (!alpha && h->n_alpha > 0) || (!beta && h->nnz > 0) || (!g_alpha && h->n_alpha > 0) ||
      (!g_beta && h->nnz > 0))
    return fail(CV_EINVAL, "null argument");
  if (h->R == 0) return CV_OK;
  return grad_noalloc(h, alpha, beta, lb, g_alpha, g_beta, (hipStream_t)stream);
}

int cv_bound_upper(cv_bound* h, const float* alpha, const float* beta, float* lb, float* ub, int32_t* sat,
                   void* stream) {
  if (!h || ((!ub || !sat) && h->R > 0) || (!alpha && h->n_alpha > 0) || (!beta && h->nnz > 0))
    return fail(CV_EINVAL, "null argument");
  int rc = ensure_grad(h);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (h->R == 0) return CV_OK;
  if (h->L == 1) {  // no ReLU layer: the bound is exact and attained at x*
    // ub is the network's value at x*, never lowered by the sound margin;
    // in sound mode lb is the lowered bound of a second pass
    const bool snd = h->sound;
    const Batch saved = h->bt;
    h->sound = false;
    h->bt.sw = nullptr;
    rc = enqueue_bwd(h, alpha, beta, false, ub, nullptr, 0, s);
    h->sound = snd;
    h->bt = saved;
    if (rc) return rc;
    if (lb && snd && (rc = enqueue_bwd64(h, alpha, beta, lb, nullptr, 0, s))) return rc;
    if (lb && !snd) HIPCHK(hipMemcpyAsync(lb, ub, sizeof(float) * h->R, hipMemcpyDeviceToDevice, s));
    launch_fill_i32(sat, 1, h->R, s);
    HIPCHK(hipGetLastError());
    return CV_OK;
  }
  if ((rc = enqueue_bwd(h, alpha, beta, true, lb, nullptr, 0, s))) return rc;
  if ((rc = enqueue_true_fwd(h, ub, sat, s))) return rc;
  return h->sound && lb ? enqueue_bwd64(h, alpha, beta, lb, nullptr, 0, s) : CV_OK;
}

int cv_bound_optimize(cv_bound* h, int32_t iters, float lr_alpha, float lr_beta, float lr_decay, float* alpha,
                      float* beta, float* adam_state, int32_t step0, float* lb_best, float* lb_last, void* stream) {
  if (!h || (!lb_best && h->R > 0) || (!alpha && h->n_alpha > 0) || (!beta && h->nnz > 0))
    return fail(CV_EINVAL, "null argument");
  if (iters < 0 || step0 < 0 || !std::isfinite(lr_alpha) || !std::isfinite(lr_beta) || !std::isfinite(lr_decay))
    return fail(CV_EINVAL, "bad optimiser settings");
  hipStream_t s = (hipStream_t)stream;
  if (h->R == 0) return CV_OK;
  AdamPtrs ap;
  if (adam_state) {
    const int64_t nb = h->nnz * h->m;
    ap = {adam_state, adam_state + h->n_alpha, adam_state + 2 * h->n_alpha, adam_state + 2 * h->n_alpha + nb};
  }
  const int np = (int)h->parts.size();
  if (np <= 1) return optimize_one(h, iters, lr_alpha, lr_beta, lr_decay, alpha, beta, ap, step0, lb_best, lb_last, s);
  // fork: every part waits for the caller's stream, runs on its own stream;
  // join: the caller's stream waits for every part
  return for_parts(h, s, [&](cv_bound* q, const PartOff& o, hipStream_t t) {
    AdamPtrs pq;
    if (ap.ma) pq = {ap.ma + o.a0, ap.va + o.a0, ap.mb + o.s0, ap.vb + o.s0};
    return optimize_one(q, iters, lr_alpha, lr_beta, lr_decay, alpha ? alpha + o.a0 : nullptr,
                        beta ? beta + o.s0 : nullptr, pq, step0, lb_best + o.r0, lb_last ? lb_last + o.r0 : nullptr, t);
  });
}

int cv_bound_optimize_joint(cv_bound* h, int32_t iters, float lr_alpha, float lr_beta, float lr_decay, float* alpha,
                            float* beta, float* lb_best, float* lb_last, float* l_out, float* u_out, void* stream) {
  if (!h || !h->in || (!lb_best && h->R > 0) || (!alpha && h->n_alpha > 0) || (!beta && h->nnz > 0))
    return fail(CV_EINVAL, "null argument");
  if (iters < 0 || !std::isfinite(lr_alpha) || !std::isfinite(lr_beta) || !std::isfinite(lr_decay))
    return fail(CV_EINVAL, "bad optimiser settings");
  if (h->sound) return fail(CV_EINVAL, "joint optimisation runs in plain float32 (sound mode is on)");
  if (h->l2) return fail(CV_EINVAL, "joint optimisation is over boxes (l_p balls are set)");
  if (h->R == 0) return CV_OK;
  return optimize_joint(h, iters, lr_alpha, lr_beta, lr_decay, alpha, beta, lb_best, lb_last, l_out, u_out,
                        (hipStream_t)stream);
}

int cv_bound_joint_sizes(const cv_bound* h, int32_t layer, int64_t* n_alpha_p, int64_t* n_beta_p) {
  if (!h) return fail(CV_EINVAL, "null handle");
  if (!h->joint) return fail(CV_EINVAL, "no joint state (cv_bound_optimize_joint has not run)");
  if (layer < 2 || layer > h->L - 1) return fail(CV_EINVAL, "layer must be 2..L-1");
  const JointLayer& q = h->joint->lay[layer - 2];
  if (n_alpha_p) *n_alpha_p = q.n_ash;
  if (n_beta_p) *n_beta_p = q.nnz * 2;
  return CV_OK;
}

int cv_bound_joint_vars(cv_bound* h, int32_t layer, float* alpha_p, float* beta_p, float* g_alpha_p, float* g_beta_p,
                        void* stream) {
  int64_t na = 0, nb = 0;
  int rc = cv_bound_joint_sizes(h, layer, &na, &nb);
  if (rc) return rc;
  const JointLayer& q = h->joint->lay[layer - 2];
  hipStream_t s = (hipStream_t)stream;
  const std::pair<float*, const float*> cp[] = {{alpha_p, q.ash}, {g_alpha_p, q.gash}};
  for (const auto& c : cp)
    if (c.first && na) HIPCHK(hipMemcpyAsync(c.first, c.second, sizeof(float) * na, hipMemcpyDeviceToDevice, s));
  const std::pair<float*, const float*> cb[] = {{beta_p, q.bsh}, {g_beta_p, q.gbsh}};
  for (const auto& c : cb)
    if (c.first && nb) HIPCHK(hipMemcpyAsync(c.first, c.second, sizeof(float) * nb, hipMemcpyDeviceToDevice, s));
  return CV_OK;
}

int cv_bound_set_parts(cv_bound* h, int32_t nparts) {
  if (!h) return fail(CV_EINVAL, "null handle");
  if (nparts < 1 || nparts > kMaxParts) return fail(CV_EINVAL, "nparts must be 1..%d", kMaxParts);
  h->parts_req = nparts;
  return set_parts(h, std::min<int>(nparts, std::max(1, h->B)));
}

int cv_bound_update(cv_bound* h, int32_t n_dom, const int32_t* dom_prop, const int64_t* split_ptr,
                    const int32_t* split_layer, const int32_t* split_neuron, const int8_t* split_side, void* stream) {
  if (!h || !h->in) return fail(CV_EINVAL, "null handle");
  return update_domains(h, n_dom, dom_prop, split_ptr, split_layer, split_neuron, split_side, (hipStream_t)stream);
}

int cv_bound_autotune(cv_bound* h, void* stream) {
  if (!h) return fail(CV_EINVAL, "null handle");
  hipStream_t s = (hipStream_t)stream;
  int rc = ensure_opt(h);
  if (rc) return rc;
  if (h->R == 0) return CV_OK;
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  const int L = h->L;
  for (int dir = 0; dir < 2; ++dir) {
    for (int i = 1; i < L; ++i) {
      const DevLayer& ly = h->layers[i - 1];
      if (ly.type != CV_LAYER_DENSE) continue;
      int mode, N, K;
      const float* A;
      const float* Bt;
      int ldb;
      Epi e = make_epi(h);
      Vars v{};
      v.alpha = nullptr;
      v.beta = h->g_beta;  // any valid memory: only timing matters here
      v.acomp = h->acomp;
      v.galpha = h->g_alpha;
      v.gbeta = h->g_beta;
      v.xpos = nullptr;
      v.xneg = nullptr;
      v.xdense = h->xdense;
      v.ldx = h->ldx;
      int lda = h->ldact;
      if (dir == 0) {
        mode = i - 1 >= 1 ? kBwdRelax : kBwdConc;
        N = h->dims[i - 1];
        K = h->dims[i];
        A = h->act[0];
        Bt = ly.Wt;
        ldb = ly.ld_out;
        if (mode == kBwdRelax) {
          e.layer_off = h->offs[i - 2];
          e.bias = h->layers[i - 2].bias;
          e.out = h->act[1];
        }
        e.slot0 = 1;
      } else {
        mode = kFwd;  // a dense first layer reads x* as a dense operand
        N = h->dims[i];
        K = h->dims[i - 1];
        A = i == 1 ? h->xdense : h->act[0];
        if (i == 1) lda = h->ldx;
        Bt = ly.W;
        ldb = ly.ld_in;
        e.layer_off = h->offs[i - 1];
        e.bias = ly.bias;
        e.out = h->act[1];
      }
      // the candidates need the same slot room as the worst case (BN = 32)
      float best_ms = 1e30f;
      int best = -1;
      for (int c = 0; c < kNumGemmCfgs; ++c) {
        if (!gemm_cfg_fits(c, K)) continue;
        GemmArgs g{A, lda, Bt, ldb, h->R, N, K, dir == 1 && i == L - 1, h->bt, v, e};
        for (int w = 0; w < 2; ++w) launch_gemm(c, mode, g, s);
        HIPCHK(hipEventRecord(e0, s));
        const int reps = 10;
        for (int w = 0; w < reps; ++w) launch_gemm(c, mode, g, s);
        HIPCHK(hipEventRecord(e1, s));
        HIPCHK(hipEventSynchronize(e1));
        float ms = 0;
        HIPCHK(hipEventElapsedTime(&ms, e0, e1));
        if (ms < best_ms) {
          best_ms = ms;
          best = c;
        }
      }
      h->cfg[(dir == 0 ? 0 : L) + i - 1] = best;
      std::lock_guard<std::mutex> lk(g_tune_mu);
      g_tune[{mode, h->R, N, K}] = best;
    }
  }
  // conv layers: each kernel variant timed per layer and direction on this
  // batch (the same operands as a gradient pass)
  launch_fill(h->g_alpha, 0.5f, h->n_alpha, s);
  launch_fill(h->adam, 0.f, 2 * h->n_alpha, s);
  constexpr int kCand = kNumConvVariants + 1;  // the variants and the register tiles
  static_assert(kConvTiles == kNumConvVariants, "the candidates are 0 .. kConvTiles");
  float first_ms[2][kCand];
  int first_best[2] = {-1, -1};
  for (int dir = 0; dir < 2; ++dir) {
    for (int i = 1; i < L; ++i) {
      DevLayer& ly = h->layers[i - 1];
      if (ly.type != CV_LAYER_CONV2D) continue;
      const int mode = conv_mode(i - 1, dir == 0, false);
      Epi e = make_epi(h);
      Vars v{};
      v.alpha = nullptr;
      v.beta = h->g_beta;
      v.acomp = h->acomp;
      v.galpha = h->g_alpha;
      v.gbeta = h->g_beta;
      v.xpos = h->xpos;
      v.xneg = h->xneg;
      const float* in = h->act[0];
      int last = 0;
      if (dir == 0) {
        if (mode == kBwdRelax) {
          e.layer_off = h->offs[i - 2];
          e.bias = h->layers[i - 2].bias;
          e.out = h->act[1];
        }
        e.slot0 = 1;
        e.n = h->dims[i - 1];
      } else {
        e.layer_off = h->offs[i - 1];
        e.bias = ly.bias;
        e.n = h->dims[i];
        e.out = h->act[1];
        last = i == L - 1;
      }
      const ConvPlan def = dir == 0 ? ly.bwd_def : ly.fwd_def;
      float best_ms = 1e30f;
      int best = -1;
      float times[kCand];
      std::fill(times, times + kCand, 1e30f);
      for (int var = 0; var < kCand; ++var) {
        ConvPlan pl = def;
        if (conv_plan_variant(mode, pl, var)) continue;
        ConvArgs a{in, h->ldact, pl, h->R, last, h->bt, v, e};
        // the adjoint both as the gradient runs it and as the optimiser does,
        // whose Adam numbers cost the kernels different shares of their waves
        // (8 -> 8 k3 s1 at 73,728 rows, us, tiles and subdomain-major: plain 573
        // and 567, with Adam 744 and 658)
        times[var] = 0.f;
        for (int ad = 0; ad <= dir; ++ad) {
          if (ad) {
            a.v.adam = 1;
            a.v.bc1 = a.v.bc2 = 1.f;  // (learning rates 0: the scratch values stay)
            a.v.alpha_w = h->g_alpha;
            a.v.beta_w = a.v.gsplit = h->g_beta;
            a.v.ma = a.v.mb = h->adam;
            a.v.va = a.v.vb = h->adam + h->n_alpha;
          }
          auto run = [&]() { return dir == 0 ? launch_convt_bwd(mode, a, s) : launch_conv_fwd(mode, a, s); };
          for (int w = 0; w < 2; ++w)
            if (run()) return fail(CV_ESHAPE, "unsupported conv channels");
          HIPCHK(hipEventRecord(e0, s));
          for (int w = 0; w < 5; ++w) run();
          HIPCHK(hipEventRecord(e1, s));
          HIPCHK(hipEventSynchronize(e1));
          float ms = 0;
          HIPCHK(hipEventElapsedTime(&ms, e0, e1));
          times[var] += ms;
        }
        const float ms = times[var];
        // (a first layer's register tiles are chosen for both directions together, below)
        if (ms < best_ms && !(i == 1 && var == kConvTiles)) {
          best_ms = ms;
          best = var;
        }
      }
      if (i == 1) {
        first_best[dir] = best;
        std::copy(times, times + kCand, first_ms[dir]);
        continue;
      }
      if (best >= 0) {
        std::lock_guard<std::mutex> lk(g_tune_mu);
        g_conv_tune[conv_key(mode, h->R, ly.g)] = best;
      }
    }
  }
  if (L >= 2 && h->layers[0].type == CV_LAYER_CONV2D) {
    // the first layer's two directions share the sign planes' order
    const float reg = first_ms[0][kConvTiles] + first_ms[1][kConvTiles];
    float old = 0.f;
    for (int dir = 0; dir < 2; ++dir) old += first_best[dir] >= 0 ? first_ms[dir][first_best[dir]] : 1e30f;
    for (int dir = 0; dir < 2; ++dir) {
      const int v = reg < old ? kConvTiles : first_best[dir];
      std::lock_guard<std::mutex> lk(g_tune_mu);
      if (v >= 0) g_conv_tune[conv_key(conv_mode(0, dir == 0, false), h->R, h->layers[0].g)] = v;
    }
  }
  assign_conv_variants(h, -1);
  // whole passes: fused dense chain or per-layer kernels
  if (h->chain_lo) {
    const int saved_b = h->chain_b, saved_f = h->chain_f;
    const std::vector<int> cands = {0, 1};
    for (int dir = 0; dir < 2; ++dir) {
      if (dir == 1 && h->chain_lo + 1 > L - 1) continue;  // no adjoint chain
      float best_ms = 1e30f;
      int best = dir == 0 ? saved_b : saved_f;
      for (int T : cands) {
        (dir == 0 ? h->chain_b : h->chain_f) = T;
        auto pass = [&]() {
          return dir == 0 ? enqueue_bwd(h, h->g_alpha, h->g_beta, true, nullptr, nullptr, 0, s)
                          : enqueue_fwd(h, h->g_alpha, h->g_beta, h->g_alpha, h->g_beta, nullptr, s);
        };
        for (int w = 0; w < 2; ++w)
          if ((rc = pass())) return rc;
        HIPCHK(hipEventRecord(e0, s));
        for (int w = 0; w < 5; ++w)
          if ((rc = pass())) return rc;
        HIPCHK(hipEventRecord(e1, s));
        HIPCHK(hipEventSynchronize(e1));
        float ms = 0;
        HIPCHK(hipEventElapsedTime(&ms, e0, e1));
        if (ms < best_ms) {
          best_ms = ms;
          best = T;
        }
      }
      (dir == 0 ? h->chain_b : h->chain_f) = best;
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  drop_graph(h);
  HIPCHK(hipStreamSynchronize(s));
  for (cv_bound* q : h->parts)
    if ((rc = cv_bound_autotune(q, stream))) return rc;
  return CV_OK;
}

int cv_bound_set_plan(cv_bound* h, int32_t chain_bwd, int32_t chain_fwd) {
  if (!h) return fail(CV_EINVAL, "null handle");
  auto ok = [&](int c) { return c == 0 || (c == 1 && h->chain_lo); };
  if (!ok(chain_bwd) || !ok(chain_fwd)) return fail(CV_EINVAL, "plan entries must be 0 or 1 (1 only where a chain exists)");
  if (chain_fwd && h->chain_lo + 1 > h->L - 1) return fail(CV_EINVAL, "this network has no adjoint chain");
  h->chain_b = chain_bwd;
  h->chain_f = chain_fwd;
  drop_graph(h);
  for (cv_bound* q : h->parts) {
    q->chain_b = chain_bwd && q->chain_lo ? 1 : 0;
    q->chain_f = chain_fwd && q->chain_lo && q->chain_lo + 1 <= q->L - 1 ? 1 : 0;
    drop_graph(q);
  }
  return CV_OK;
}

int32_t cv_bound_num_tilings(void) { return kNumGemmCfgs; }

int32_t cv_bound_num_conv_variants(void) { return kNumConvVariants; }

int cv_bound_set_conv_variant(cv_bound* h, int32_t variant) {
  if (!h) return fail(CV_EINVAL, "null handle");
  if (variant < -1 || variant >= kNumConvVariants)
    return fail(CV_EINVAL, "conv variant must be -1 or in [0, %d)", kNumConvVariants);
  h->forced_conv = variant;
  assign_conv_variants(h, variant);
  drop_graph(h);
  for (cv_bound* q : h->parts) {
    q->forced_conv = variant;
    assign_conv_variants(q, variant);
    drop_graph(q);
  }
  return CV_OK;
}

int cv_bound_conv_variant(const cv_bound* h, int32_t layer, int32_t dir) {
  if (!h || layer < 1 || layer > h->L || (dir != 0 && dir != 1)) return -1;
  const DevLayer& d = h->layers[layer - 1];
  if (d.type != CV_LAYER_CONV2D) return -1;
  const ConvPlan& pl = dir == 0 ? d.bwd : d.fwd;
  return pl.reg.on ? 2 : (pl.sd ? 2 : 0) + (pl.wg ? 1 : 0);
}

int cv_bound_set_conv_tiles(cv_bound* h, int32_t on) {
  if (!h) return fail(CV_EINVAL, "null handle");
  if (on < -1 || on > 1) return fail(CV_EINVAL, "conv tiles must be -1, 0 or 1");
  std::vector<cv_bound*> all{h};
  all.insert(all.end(), h->parts.begin(), h->parts.end());
  for (cv_bound* q : all) {
    q->forced_tiles = on;
    assign_conv_variants(q, q->forced_conv);
    drop_graph(q);
  }
  return CV_OK;
}

int cv_bound_conv_tiles(const cv_bound* h, int32_t layer, int32_t dir) {
  if (!h || layer < 1 || layer > h->L || (dir != 0 && dir != 1)) return -1;
  const DevLayer& d = h->layers[layer - 1];
  if (d.type != CV_LAYER_CONV2D) return -1;
  return (dir == 0 ? d.bwd : d.fwd).reg.on ? 1 : 0;
}

int cv_bound_set_tiling(cv_bound* h, int32_t tiling) {
  if (!h) return fail(CV_EINVAL, "null handle");
  if (tiling < -1 || tiling >= kNumGemmCfgs) return fail(CV_EINVAL, "tiling must be -1 or in [0, %d)", kNumGemmCfgs);
  h->forced_tiling = tiling;
  assign_tiles(h, tiling);
  drop_graph(h);
  for (cv_bound* q : h->parts) {
    q->forced_tiling = tiling;
    assign_tiles(q, tiling);
    drop_graph(q);
  }
  return CV_OK;
}

int cv_bound_set_sound(cv_bound* h, int32_t on, void* stream) {
  if (!h || !h->in) return fail(CV_EINVAL, "null handle");
  if (on != 0 && on != 1) return fail(CV_EINVAL, "sound must be 0 or 1");
  if (on && h->l2 && h->lpq != 2.f) return fail(CV_EINVAL, "sound mode supports boxes and l2 balls only");
  if (on) return rebuild_sound(h, (hipStream_t)stream);
  std::vector<cv_bound*> all{h};
  all.insert(all.end(), h->parts.begin(), h->parts.end());
  for (cv_bound* q : all) {
    q->sound = false;
    q->bt.sw = nullptr;
    drop_graph(q);
  }
  return CV_OK;
}

int cv_bound_set_input_lp(cv_bound* h, const float* x0, const float* eps, float p_norm, void* stream) {
  if (!h || !h->in) return fail(CV_EINVAL, "null handle");
  hipStream_t s = (hipStream_t)stream;
  std::vector<cv_bound*> all{h};
  all.insert(all.end(), h->parts.begin(), h->parts.end());
  if (!x0) {  // back to the box
    for (cv_bound* q : all) {
      q->l2 = false;
      q->lpq = 2.f;
      q->bt.l2x0 = nullptr;
      q->bt.l2eps = nullptr;
      drop_graph(q);
    }
    return h->sound ? rebuild_sound(h, s) : CV_OK;
  }
  if (!eps) return fail(CV_EINVAL, "null argument");
  // q = p / (p - 1) <= 4 keeps the float32 q-th powers of A(0) in range
  if (!(p_norm >= 4.f / 3.f) || !std::isfinite(p_norm)) return fail(CV_EINVAL, "p must be finite and >= 4/3");
  const float lpq = p_norm == 2.f ? 2.f : (float)((double)p_norm / ((double)p_norm - 1.0));
  if (h->sound && lpq != 2.f) return fail(CV_EINVAL, "sound mode supports boxes and l2 balls only");
  const int P = h->P, d0 = h->d0, d1 = h->dims[1];
  for (int64_t i = 0; i < (int64_t)P * d0; ++i)
    if (!std::isfinite(x0[i])) return fail(CV_EINVAL, "x0 must be finite");
  for (int p = 0; p < P; ++p)
    if (!(eps[p] >= 0.f) || !std::isfinite(eps[p])) return fail(CV_EINVAL, "eps must be finite and >= 0");
  // W(1) x0 + b(1) per property, in double, rounded once
  const cv_layer& ly1 = h->in->layers[0];
  std::vector<float> wx0((size_t)P * d1);
  std::vector<double> t;
  for (int p = 0; p < P; ++p) {
    affine_host(ly1, x0 + (size_t)p * d0, t);
    for (int j = 0; j < d1; ++j) wx0[(size_t)p * d1 + j] = (float)t[j];
  }
  int rc;
  if (!h->l2x0 && ((rc = h->mem.alloc(&h->l2x0, (size_t)P * d0)) || (rc = h->mem.alloc(&h->l2eps, P)) ||
                   (rc = h->mem.alloc(&h->wx0, (size_t)P * d1))))
    return rc;
  HIPCHK(hipMemcpyAsync(h->l2x0, x0, sizeof(float) * P * d0, hipMemcpyHostToDevice, s));
  HIPCHK(hipMemcpyAsync(h->l2eps, eps, sizeof(float) * P, hipMemcpyHostToDevice, s));
  HIPCHK(hipMemcpyAsync(h->wx0, wx0.data(), sizeof(float) * P * d1, hipMemcpyHostToDevice, s));
  HIPCHK(hipStreamSynchronize(s));
  // the sub-batches read the parent's centre, radius and W(1) x0 + b(1); each
  // handle keeps its own per-row sums and scales, and x* (A(0)) densely
  for (cv_bound* q : all) {
    if ((rc = ensure_ball(q))) return rc;
    q->l2x0 = h->l2x0;
    q->l2eps = h->l2eps;
    q->wx0 = h->wx0;
    q->l2 = true;
    q->lpq = lpq;
    q->bt.l2x0 = h->l2x0;
    q->bt.l2eps = h->l2eps;
    q->bt.lpq = lpq;
    drop_graph(q);
  }
  h->hl2x0.assign(x0, x0 + (size_t)P * d0);
  h->hl2eps.assign(eps, eps + P);
  return h->sound ? rebuild_sound(h, s) : CV_OK;
}

int cv_bound_set_input_l2(cv_bound* h, const float* x0, const float* eps, void* stream) {
  return cv_bound_set_input_lp(h, x0, eps, 2.f, stream);
}

int cv_bound_profile(cv_bound* h, const float* alpha, const float* beta, int32_t reps, cv_kernel_stat* out,
                     int32_t max_out, int32_t* n_out, void* stream) {
  if (!h || !out || !n_out || reps <= 0) return fail(CV_EINVAL, "bad argument");
  int rc = ensure_opt(h);
  if (rc) return rc;
  hipStream_t s = (hipStream_t)stream;
  Profiler pf;
  pf.s = s;
  h->prof = nullptr;
  std::vector<std::string> order;
  std::map<std::string, cv_kernel_stat> acc;
  // one untimed pass first: the first launch of each kernel loads its code
  rc = enqueue_bwd(h, alpha, beta, true, nullptr, nullptr, 0, s);
  if (!rc) rc = enqueue_fwd(h, alpha, beta, h->g_alpha, h->g_beta, nullptr, s);
  if (!rc) rc = enqueue_bwd(h, alpha, beta, false, nullptr, nullptr, 0, s);
  if (!rc && hipStreamSynchronize(s) != hipSuccess) rc = fail(CV_EDEVICE, "profile warm-up failed");
  h->prof = rc ? nullptr : &pf;
  for (int r = 0; r < reps && rc == CV_OK; ++r) {
    pf.recs.clear();
    rc = enqueue_bwd(h, alpha, beta, true, nullptr, nullptr, 0, s);
    if (!rc) rc = enqueue_fwd(h, alpha, beta, h->g_alpha, h->g_beta, nullptr, s);
    if (!rc) rc = enqueue_bwd(h, alpha, beta, false, nullptr, nullptr, 0, s);
    if (hipStreamSynchronize(s) != hipSuccess) rc = fail(CV_EDEVICE, "profile pass failed");
    std::map<std::string, int> per_rep;
    for (KStat& k : pf.recs) {
      float ms = 0;
      (void)hipEventElapsedTime(&ms, k.e0, k.e1);
      ms /= Profiler::kRepeat;
      (void)hipEventDestroy(k.e0);
      (void)hipEventDestroy(k.e1);
      if (!acc.count(k.name)) {
        cv_kernel_stat z{};
        std::snprintf(z.name, sizeof(z.name), "%s", k.name.c_str());
        acc[k.name] = z;
        order.push_back(k.name);
      }
      cv_kernel_stat& st = acc[k.name];
      st.total_ms += ms;
      if (r == 0) {
        st.launches += 1;
        st.flops += k.flops;
        st.bytes += k.bytes;
      }
    }
  }
  h->prof = nullptr;
  if (rc) return rc;
  int n = 0;
  for (const std::string& nm : order) {
    if (n < max_out) out[n] = acc[nm];
    ++n;
  }
  *n_out = n;
  return CV_OK;
}

void cv_bound_destroy(cv_bound* h) { destroy_handle(h); }

int cv_bound_root_bounds(const cv_layer* layers, int32_t n_layers, int32_t n_props, const float* x_lo,
                         const float* x_hi, float* l_out, float* u_out, void* stream) {
  return root_bounds(layers, n_layers, n_props, x_lo, x_hi, l_out, u_out, false, stream);
}

int cv_bound_root_bounds_sound(const cv_layer* layers, int32_t n_layers, int32_t n_props, const float* x_lo,
                               const float* x_hi, float* l_out, float* u_out, void* stream) {
  return root_bounds(layers, n_layers, n_props, x_lo, x_hi, l_out, u_out, true, stream);
}

int cv_bound_root_bounds_opt(const cv_layer* layers, int32_t n_layers, int32_t n_props, const float* x_lo,
                             const float* x_hi, int32_t iters, float lr_alpha, float lr_decay, int32_t sound,
                             float* l_out, float* u_out, void* stream) {
  if (sound != 0 && sound != 1) return fail(CV_EINVAL, "sound must be 0 or 1");
  return root_bounds(layers, n_layers, n_props, x_lo, x_hi, l_out, u_out, sound != 0, stream, iters, lr_alpha,
                     lr_decay);
}

}  // extern "C"
