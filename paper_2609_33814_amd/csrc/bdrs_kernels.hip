// gfx950 kernels of the Dual O-BDRS hot path.
//
// Sweep (the reduction of Algorithm 1's row and column updates, and of
// Algorithm 2's column pass).  For every output point p of one side and the
// input points q of the other side it evaluates, in base 2,
//     LSE2_p = log2 sum_q 2^{ w2_q - kappa2 ||P_p - Q_q||^2 },
//     kappa2 = log2(e) * s / eps,   w2 = log2(e) * w,
// which is LSE_q(w_q - C_pq / eps) / ln 2.  The cost is never stored: inputs
// are grouped in tiles of 64 spatially close points with centre Qc, offsets
// b_q = Q_q - Qc, and with a = P_p - Qc and the plane fit
// w2_q ~ alpha + gamma . b_q of the tile's weights the exponent expands
// exactly as
//     w2_q - kappa2 |a - b_q|^2 = base + B . b_q + A_q,
//     base = alpha - kappa2 |a|^2,  B = gamma + 2 kappa2 a,
//     A_q = w2_q - alpha - gamma . b_q - kappa2 |b_q|^2   (written by the producing epilogue),
// i.e. d FMAs and one add per entry, then one v_exp_f32 and one add.  The plain
// sweep forms the exponents on the matrix cores (sweep_split_mfma).
//
// Precision split.  The weights w grow like g / eps as the temperature falls,
// so float32 values of that size would carry absolute errors u |g| / eps.  The
// inner loop therefore only sees small numbers: A_q is the weight's residual
// from its tile's plane minus the tile-local quadratic (float32), B is formed
// in float64 before it is rounded, and the large per-(output, tile) part base
// and the lane's running shift M are kept in float64.  The summand is
// 2^{cm + B . b_q + A_q} with cm = base - M (float32).  For the entries that
// dominate an output's sum B is the exponent's slope across the tile near its
// maximum, so every float32 operand is of the order of kappa2 r^2 (r the tile
// radius) rather than of the weights' variation across the tile, which at low
// temperature is 2 kappa2 |a| r, the transport distance |a| times larger.
//
// Stability without a per-entry max: the per-(output, tile) upper bound
//     UB >= max_q exponent  (lane_bound)
// is compared with M.  Only when UB > M + 64 does the lane take the exact
// maximum of the tile first (and rescale its sum), so every summed term is at
// most 2^64 and M never exceeds the true maximum (no underflow of the leading
// terms).  Lanes of a wave hold 64 consecutive outputs in tile order, i.e.
// neighbouring points, so they agree on which tiles need the exact maximum.
//
// Each (block of 256 outputs, split of the input tiles) writes a partial
// (M, S[, N]); the finish kernels merge the splits in float64 and run the
// epilogue of Algorithm 1 (overrelaxation, momentum, packing of the next
// sweep's weights) or of Algorithm 2 (column mean costs and masses).
#include "bdrs_internal.h"

#include <hip/hip_ext.h>

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace bdrs {

namespace {

constexpr double kLog2eD = 1.4426950408889634074;
constexpr double kLn2D = 0.69314718055994530942;
// Exact-max gate: a tile whose bound exceeds the running shift by more than
// this takes its exact maximum first, so no summed term exceeds 2^64.
constexpr float kThresh = 64.0f;

// The control block in one scalar load, issued as soon as its address is known
// (read field by field under conditions it cost a chain of round trips).
typedef __attribute__((address_space(4))) const Ctrl cctrl;
struct CtrlVals {
  double eta, lam, scale;
  long long k;  // first iteration of the block
  unsigned variant;
};
__device__ __forceinline__ CtrlVals load_ctrl(const Ctrl* c) {
  cctrl* p = (cctrl*)c;
  CtrlVals v;
  v.k = p->k;
  v.variant = p->variant;
  v.eta = p->eta;
  v.lam = p->lam;
  v.scale = p->scale;
  return v;
}

// kappa2 = log2(e) s / eps at the temperature of the column update of iteration
// c.k + ahead, eta_k = eta / (lambda k + 1), or (ROW) of its row update: the
// same, or eta / k for the old kernel K^{.k} (at k = 0 one at which every cost
// term vanishes).  No branches: they would hold back the loads after them.
// Divisions with their scaling: eta, eps and the cost scale may be any finite
// positive numbers, and a quotient may leave the normal range on the way (two
// Newton steps without it gave NaN there and saved at most 0.2%: 100 iterations
// of 64x64 grids 1894 against 1898 us, 1 M points the same).
template <bool ROW>
__device__ __forceinline__ double kap2_of(const CtrlVals& c, int ahead) {
  const double k = (double)(c.k + ahead);
  double den = c.lam * k + 1.0;
  if (ROW) den = c.variant & kVarOldKernel ? (k >= 1.0 ? k : 1.0 / kFarTemperature) : den;
  return kLog2eD * c.scale / (c.eta / den);
}

// The control block with the temperature of a sweep called with its own eps
// (eps > 0): eta = eps and lambda = 0 give eps whatever k is.
__device__ __forceinline__ CtrlVals with_eps(CtrlVals c, double eps, bool own) {
  c.eta = own ? eps : c.eta;
  c.lam = own ? 0.0 : c.lam;
  c.variant = own ? 0u : c.variant;
  return c;
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Wavefront all-reductions of a double with DPP lane moves inside each row of
// 16 lanes (swap neighbours, swap pairs, mirror halves, mirror the row) and
// four readlanes across the rows; every lane receives the result.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double read_lane(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

constexpr int kDppXor1 = 0xB1;        // quad_perm(1, 0, 3, 2)
constexpr int kDppXor2 = 0x4E;        // quad_perm(2, 3, 0, 1)
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7 - i within each half row
constexpr int kDppMirror = 0x140;     // lane i <-> 15 - i within each row

__device__ __forceinline__ double wave_sum(double v) {
  v += dpp_move<kDppXor1>(v);
  v += dpp_move<kDppXor2>(v);
  v += dpp_move<kDppHalfMirror>(v);
  v += dpp_move<kDppMirror>(v);
  return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// N independent sums at once (their lane moves interleave).
template <int N>
__device__ __forceinline__ void wave_sum_n(double (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_move<kDppXor1>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_move<kDppXor2>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_move<kDppHalfMirror>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] += dpp_move<kDppMirror>(v[i]);
#pragma unroll
  for (int i = 0; i < N; ++i)
    v[i] = (read_lane(v[i], 0) + read_lane(v[i], 16)) + (read_lane(v[i], 32) + read_lane(v[i], 48));
}

// Wavefront maximum of a float (every lane receives it).
template <int CTRL>
__device__ __forceinline__ float dpp_movef(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float read_lanef(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ float wave_maxf(float v) {
  v = fmaxf(v, dpp_movef<kDppXor1>(v));
  v = fmaxf(v, dpp_movef<kDppXor2>(v));
  v = fmaxf(v, dpp_movef<kDppHalfMirror>(v));
  v = fmaxf(v, dpp_movef<kDppMirror>(v));
  return fmaxf(fmaxf(read_lanef(v, 0), read_lanef(v, 16)), fmaxf(read_lanef(v, 32), read_lanef(v, 48)));
}

__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp_move<kDppXor1>(v));
  v = fmax(v, dpp_move<kDppXor2>(v));
  v = fmax(v, dpp_move<kDppHalfMirror>(v));
  v = fmax(v, dpp_move<kDppMirror>(v));
  return fmax(fmax(read_lane(v, 0), read_lane(v, 16)), fmax(read_lane(v, 32), read_lane(v, 48)));
}

// ---------------------------------------------------------------------------
// Sweep
// ---------------------------------------------------------------------------
// Constant-address-space views of what a sweep only reads (the kernels before
// it wrote it): uniform reads compile to scalar loads whatever pointer they
// come from (kernel argument or a descriptor in memory) and whatever the kernel
// has stored before.
typedef __attribute__((address_space(4))) const float gfloat;
typedef __attribute__((address_space(4))) const double gdouble;
typedef __attribute__((address_space(4))) const int gint;
typedef __attribute__((address_space(4))) const TileRec gtile;

// Points of a tile per group: the tile data of one group (8 D offsets into
// scalar registers, 8 weights into vector registers by broadcast loads) is
// requested while the previous group is being computed.
constexpr int kGroup = 8;

// The fields of a tile record the sweep uses (dimensions < D).
template <int D>
struct TileVals {
  double alpha;
  float ctr[D], rad[D], gam[D], rho;
};

template <int D>
__device__ __forceinline__ TileVals<D> load_tile(gtile* __restrict__ rec) {
  gdouble* dp = (gdouble*)rec;
  gfloat* fp = (gfloat*)rec;
  TileVals<D> v;
  v.alpha = dp[0];
#pragma unroll
  for (int d = 0; d < D; ++d) {
    v.ctr[d] = fp[2 + d];
    v.rad[d] = fp[5 + d];
    v.gam[d] = fp[8 + d];
  }
  v.rho = fp[11];
  return v;
}

template <int D>
struct Group {
  float b[D][kGroup];
  float a[kGroup];
};

// Group g of a tile whose offsets start at offs_t ([D][64]) and weights at a_t.
template <int D>
__device__ __forceinline__ Group<D> load_group(gfloat* __restrict__ offs_t, gfloat* __restrict__ a_t, int g) {
  Group<D> r;
  gfloat* offs = offs_t + g * kGroup;
  gfloat* aq = a_t + g * kGroup;
#pragma unroll
  for (int d = 0; d < D; ++d)
#pragma unroll
    for (int u = 0; u < kGroup; ++u) r.b[d][u] = offs[d * kTile + u];
#pragma unroll
  for (int u = 0; u < kGroup; ++u) r.a[u] = aq[u];
  return r;
}

// The input side of a sweep.
struct SweepIn {
  gfloat* off;
  gfloat* A;
  gtile* tile;
  int ntiles, count;
};

__device__ __forceinline__ SweepIn sweep_in(const SideDev& s) {
  return SweepIn{(gfloat*)s.off, (gfloat*)s.A, (gtile*)s.tile, s.ntiles, s.count};
}

// What a lane keeps for its output while it sweeps: the point, the kernel's
// temperature, the wavefront's output box (all lanes, padding included: a
// larger box only loosens the coarse bound) and the skip gate's depth.
template <int D>
struct SweepOut {
  float P[D], blo[D], bhi[D];
  double kap2d, tskip;  // kappa2; depth T of the skip gate (SideDev::tskip)
  float kap2f, inv2kap;
};

// The sums of one split of one output and the shift they are relative to.
struct SplitSum {
  double M;
  float S, N, V[3];
  int J;          // slot of the term that set the shift
  int evaluated;  // input tiles this wavefront evaluated (the same on every lane)
};

// A value that is the same on every lane, held in a scalar register.
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// own: the record of the outputs' own tile, whose box (widened against the
// rounding of its centre and radius) holds the wavefront's 64 points.
template <int D, bool BATCH>
__device__ __forceinline__ SweepOut<D> sweep_out(const float (&P)[D], const TileVals<D>& own, double kap2,
                                                 double tskip) {
  SweepOut<D> o;
  o.kap2d = kap2;
  o.kap2f = (float)kap2;
  o.inv2kap = (float)(0.5 / kap2);
  o.tskip = tskip;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const float ctr = own.ctr[d], half = own.rad[d] * 1.000001f + fabsf(ctr) * 1e-6f;
    o.P[d] = P[d];
    o.blo[d] = ctr - half;
    o.bhi[d] = ctr + half;
    // batches on lines: in scalar registers, without which the sweep spills four
    // vector registers (a 3-d one spills with it, its scalar ones being full, and
    // on lines a single problem, which does not spill, takes up to 1.4% longer).
    // 100 iterations of four problems of 777 to 5100 points 3.01..3.08 -> 2.98..2.99
    // ms, of three of 9000 to 30000 points 12.77..12.82 -> 12.90..13.00 ms (at 5
    // wavefronts per SIMD instead, without spilling too, 13.10..13.17 ms)
    if (D == 1 && BATCH) {
      o.blo[d] = uniform(o.blo[d]);
      o.bhi[d] = uniform(o.bhi[d]);
    }
  }
  return o;
}

// Lower bound of the smallest skip gate of the wavefront: the minimum taken in
// float32 and moved down by more than the conversion's rounding.
__device__ __forceinline__ double gate_min(double Mlo) {
  const float m = -wave_maxf(-(float)Mlo);
  return (double)fmaf(-1e-6f, fabsf(m), m) - 1e-6;
}

// Split `split` of nsplit takes the tiles split, split + nsplit, ... (local
// index i is tile split + i nsplit), so that each split samples the whole input
// cloud: late in a solve only the tiles near an output block matter, and they
// spread over all splits instead of crowding into one wavefront's work.

// Coarse test of up to 64 tiles at once, lane l taking local tile c0 + l: an
// upper bound of the exponents of the tile's points for every output of the
// wavefront, alpha + sum_d |gamma_d| r_d + rho - kappa2 dist^2(output box,
// tile box), to be compared with the smallest running maximum of the
// wavefront.  It bounds each lane's own bound from above, so a tile it
// rejects would be skipped by the per-lane test too.  The tile index is
// clamped to a valid tile (also for an empty split).
template <int D>
__device__ __forceinline__ double coarse_of(const TileVals<D>& t, const SweepOut<D>& o) {
  float w = t.rho, g2 = 0.0f;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    w = fmaf(fabsf(t.gam[d]), t.rad[d], w);
    // gap between the boxes, shrunk by a relative 1e-5 against rounding
    const float gap =
        fmaxf(0.0f, fmaxf((t.ctr[d] - t.rad[d]) - o.bhi[d], o.blo[d] - (t.ctr[d] + t.rad[d]))) * 0.99999f;
    g2 = fmaf(gap, gap, g2);
  }
  return t.alpha + (double)fmaf(-o.kap2f, g2, w);
}

// Candidates among the local tiles c0 ... c0+63 of a split, as a bit mask.
template <int D>
__device__ __forceinline__ unsigned long long coarse_mask(const SweepIn& in, const SweepOut<D>& o, double gate,
                                                          int split, int nsplit, int c0) {
  const int t = split + (c0 + (int)(threadIdx.x & (kTile - 1))) * nsplit;
  const double cub = coarse_of<D>(load_tile<D>(in.tile + min(t, in.ntiles - 1)), o);
  return __ballot(t < in.ntiles && !(cub < gate));
}

// Warm start: the exact exponent of one remembered input point is a lower
// bound of the output's maximum over all inputs, so it is a valid shift for
// every split (a split whose terms all lie far below it adds ~nothing); it
// spares the exact-max pass on the first tile of each split.  Its loads are
// issued unconditionally at a clamped, valid index and the result is masked
// afterwards: loads under a branch would wait for their data one by one.
template <int D>
__device__ __forceinline__ void warm_start(const SweepIn& in, const SweepOut<D>& o, int j, double& M, int& J) {
  M = -INFINITY;
  J = -1;
  const int jc = min(max(j, 0), in.count - 1);
  const int tj = jc / kTile, qj = jc % kTile;
  const double al = in.tile[tj].alpha;
  const float aj = in.A[jc];
  double na = 0.0, ab = 0.0, gb = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const double ad = (double)o.P[d] - (double)in.tile[tj].ctr[d];
    const double bd = (double)in.off[((size_t)tj * D + d) * kTile + qj];
    na += ad * ad;
    ab += ad * bd;
    gb += (double)in.tile[tj].gam[d] * bd;
  }
  if (j >= 0 && j < in.count && al > -INFINITY && aj > -INFINITY) {
    M = al + (double)aj + gb + o.kap2d * (2.0 * ab - na);
    J = j;
  }
}

// Upper bound of the exponents w2_q - kappa2 |a - b_q|^2 of a tile:
// w2_q <= alpha + gamma . b_q + rho, and the concave quadratic
// gamma . b - kappa2 |a - b|^2 is maximised over the tile's box per axis.
template <int D>
__device__ __forceinline__ double lane_bound(const TileVals<D>& t, const SweepOut<D>& o, const float (&a)[D]) {
  float ubf = t.rho;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const float g = t.gam[d], rad = t.rad[d];
    const float bs = __builtin_amdgcn_fmed3f(fmaf(g, o.inv2kap, a[d]), -rad, rad);  // clamp to the box
    const float df = a[d] - bs;
    ubf = fmaf(g, bs, ubf);
    ubf = fmaf(-o.kap2f, df * df, ubf);
  }
  return t.alpha + (double)ubf;
}

// Exact maximum of a tile's exponents (relative to base) and its point.
template <int D>
__device__ __forceinline__ float tile_max(gfloat* __restrict__ offs, gfloat* __restrict__ Aq, const float (&B)[D],
                                          int& qi) {
  float tm = -INFINITY;
  qi = 0;
#pragma unroll 8
  for (int q = 0; q < kTile; ++q) {
    float z = Aq[q];
#pragma unroll
    for (int d = 0; d < D; ++d) z = fmaf(B[d], offs[d * kTile + q], z);
    if (z > tm) {
      tm = z;
      qi = q;
    }
  }
  return tm;
}

// One split of the plain sweep for one wavefront of 64 outputs, the exponents
// formed on the matrix cores.  Per chunk of up to 64 tiles the coarse test
// picks the candidates; per candidate the lane bounds its own exponents, the
// wavefront skips the tile when no lane can see it, else the whole 64 x 64
// block of exponents z_qp = cm_p + B_p . b_q + A_q is a product of inner
// dimension D + 2, taken in rank-one steps of v_mfma_f32_16x16x1 (four blocks
// of 16 outputs, 16 inputs): each step is one IEEE fused multiply-add per
// element, so the chain cm, + B_0 b_0, ..., + 1 A_q rounds exactly as the
// scalar code of the other modes does.  The chain's first step is the same for
// all inputs, so it is taken once per tile and the four quarters of the tile's
// points start from its registers.  Input operands: lane l holds point
// pt(l) of the tile, one coalesced load per coordinate, and cbsz/abid
// broadcast one quarter of them to all blocks.  Result element i is block i / 4,
// row 4 (lane / 16) + i % 4; with the two pairs of bits of the point's index in
// its quarter exchanged (pt) the lanes of quarter g of the wavefront hold the
// points q = g mod 4, in order, so each lane's running sum per output block is
// the sum over q = g mod 4 in point order, and three exchanges between the
// quarters bring the four together.
//
// Bound: the float32 VALU / matrix pipe, one for both on gfx950 (work of the
// two kinds from different wavefronts takes the sum of their times).  Measured
// cycles per wavefront instruction: fused multiply-add 4.2 (any form with three
// register operands or a scalar one), exp2 8.2, add 2.5 (4 after an exp2),
// rank-one step 2.03 per input.  So an entry takes 19.3 cycles here against
// 25.8 on the VALU for d = 3, 17.3 against 21.6 for d = 2, 15.3 against 17.4
// for d = 1; and the tile data comes by one vector load per coordinate instead
// of a chain of scalar ones.  With blocks of 32 x 32 (v_mfma_f32_32x32x1), whose
// registers leave no room for the bases, the first step was taken for each
// half: 1.5 cycles more per entry.
// Dense sweeps of 1 M points per side (d = 3): 194 ms on the VALU, 173 with halves,
// 164 with quarters; 50 iterations of two 251x251 grids (d = 2, 7% of the
// entries): 9.46, 8.31, 8.03 ms; of 30000 x 20000 points on a line: 5.19 ms on the
// VALU, 5.02 with quarters.  The next candidate's record and points are requested
// while the current one is tested and evaluated.
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

template <int D>
struct TilePts {
  float b[D], a;
};

template <int D>
__device__ __forceinline__ TilePts<D> load_points(const SweepIn& in, int t, int pt) {
  TilePts<D> v;
#pragma unroll
  for (int d = 0; d < D; ++d) v.b[d] = in.off[((size_t)t * D + d) * kTile + pt];
  v.a = in.A[(size_t)t * kTile + pt];
  return v;
}

// Exponents of 16 inputs (quarter H of the tile's points) against 64 outputs,
// from the outputs' bases.
template <int D, int H>
__device__ __forceinline__ f32x16 exponents(const TilePts<D>& q, const float (&B)[D], f32x16 z) {
#pragma unroll
  for (int d = 0; d < D; ++d) z = __builtin_amdgcn_mfma_f32_16x16x1f32(q.b[d], B[d], z, 2, H, 0);
  return __builtin_amdgcn_mfma_f32_16x16x1f32(q.a, 1.0f, z, 2, H, 0);
}

// sum_q 2^{z_q} over the tile's 64 points for the lane's own output.
template <int D>
__device__ __forceinline__ float tile_sum(const TilePts<D>& pts, const float (&B)[D], float cm) {
  f32x16 base = {};
  base = __builtin_amdgcn_mfma_f32_16x16x1f32(1.0f, cm, base, 0, 0, 0);
  // x[i]: outputs 16 i + lane % 16
  float x[4];
  f32x16 z = exponents<D, 0>(pts, B, base);
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = fast_exp2(z[4 * i]);
#pragma unroll
  for (int e = 1; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] += fast_exp2(z[4 * i + e]);
  auto add = [&](const f32x16& y) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] += fast_exp2(y[4 * i + e]);
  };
  add(exponents<D, 1>(pts, B, base));
  add(exponents<D, 2>(pts, B, base));
  add(exponents<D, 3>(pts, B, base));
  // quarter g of the wavefront holds q = g mod 4 of all four output blocks: swaps
  // between neighbouring quarters, then between the halves, bring the four sums
  // of a lane's own output together
  auto swapped_sum = [](u32x2 w) { return __uint_as_float(w[0]) + __uint_as_float(w[1]); };
  auto bits = [](float v) { return __float_as_uint(v); };
  const float u = swapped_sum(__builtin_amdgcn_permlane16_swap(bits(x[0]), bits(x[1]), false, false));
  const float v = swapped_sum(__builtin_amdgcn_permlane16_swap(bits(x[2]), bits(x[3]), false, false));
  return swapped_sum(__builtin_amdgcn_permlane32_swap(bits(u), bits(v), false, false));
}

// Exact maximum of a tile's exponents (relative to base) and its point, as
// tile_max, on the matrix cores and from the points already loaded; every lane
// of the wavefront takes part.  Equal exponents: the first point, as there.
// In clouds half of the evaluated tiles come here (on grids 1 in 100), where a
// lone wavefront waited for a chain of scalar loads, 64 compares and selects per
// lane in one chain.  50 iterations, before and after: 3-D clouds of 3000 points
// 1.30 -> 1.21 ms, of 700 and 900 points 1.68 -> 1.41 ms, 2-D of 3000 and 3500
// points 1.23 -> 1.15 ms, on a line 1.07 -> 1.02 ms.  Sweeps
// that never come here measured 0.3 to 1.8% more with the same instructions in
// their loop; so did the former maximum compiled beside this one and used from
// 131072 inputs on (where the code lies, not what it does), which was not kept.
struct MaxAt {
  float z;
  int q;
};

template <int D, int H>
__device__ __forceinline__ void max_quarter(const TilePts<D>& p, const float (&B)[D], MaxAt (&x)[4]) {
  f32x16 z = {};
  z = __builtin_amdgcn_mfma_f32_16x16x1f32(p.a, 1.0f, z, 2, H, 0);
#pragma unroll
  for (int d = 0; d < D; ++d) z = __builtin_amdgcn_mfma_f32_16x16x1f32(p.b[d], B[d], z, 2, H, 0);
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (z[4 * i + e] > x[i].z) x[i] = MaxAt{z[4 * i + e], 4 * H + e};
}

__device__ __forceinline__ MaxAt better_of(const MaxAt& a, const MaxAt& b) {
  return b.z > a.z || (b.z == a.z && b.q < a.q) ? b : a;
}

template <int D>
__device__ __forceinline__ float tile_max_mfma(const TilePts<D>& pts, const float (&B)[D], int& qi) {
  MaxAt x[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i] = MaxAt{-INFINITY, 0};
  max_quarter<D, 0>(pts, B, x);
  max_quarter<D, 1>(pts, B, x);
  max_quarter<D, 2>(pts, B, x);
  max_quarter<D, 3>(pts, B, x);
  const int g = (int)(threadIdx.x & (kTile - 1)) >> 4;  // the lane holds q = g mod 4
#pragma unroll
  for (int i = 0; i < 4; ++i) x[i].q = 4 * x[i].q + g;
  auto pair16 = [](const MaxAt& a, const MaxAt& b) {
    const u32x2 z = __builtin_amdgcn_permlane16_swap(__float_as_uint(a.z), __float_as_uint(b.z), false, false);
    const u32x2 q = __builtin_amdgcn_permlane16_swap((unsigned)a.q, (unsigned)b.q, false, false);
    return better_of(MaxAt{__uint_as_float(z[0]), (int)q[0]}, MaxAt{__uint_as_float(z[1]), (int)q[1]});
  };
  const MaxAt u = pair16(x[0], x[1]), v = pair16(x[2], x[3]);
  const u32x2 z = __builtin_amdgcn_permlane32_swap(__float_as_uint(u.z), __float_as_uint(v.z), false, false);
  const u32x2 q = __builtin_amdgcn_permlane32_swap((unsigned)u.q, (unsigned)v.q, false, false);
  const MaxAt m = better_of(MaxAt{__uint_as_float(z[0]), (int)q[0]}, MaxAt{__uint_as_float(z[1]), (int)q[1]});
  qi = m.q;
  return m.z;
}

// Exponent of a tile for a lane: slope B = gamma + 2 kappa2 a (rounded once)
// and base = alpha - kappa2 |a|^2.
template <int D>
__device__ __forceinline__ double tile_base(const TileVals<D>& t, const SweepOut<D>& o, const float (&a)[D],
                                            float (&B)[D]) {
  const double kap2x2 = 2.0 * o.kap2d;
  float na = 0.0f;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    na = fmaf(a[d], a[d], na);
    B[d] = (float)fma(kap2x2, (double)a[d], (double)t.gam[d]);
  }
  return t.alpha - o.kap2d * (double)na;
}

template <int D>
__device__ __forceinline__ SplitSum sweep_split_mfma(const SweepIn& in, const SweepOut<D>& o, int split, int nsplit,
                                                      double M, int J, unsigned long long cand) {
  const int lane = (int)(threadIdx.x & (kTile - 1));
  const int pt = (lane & 48) | ((lane & 3) << 2) | ((lane >> 2) & 3);
  SplitSum r{M, 0.0f, 0.0f, {0.0f, 0.0f, 0.0f}, J, 0};
  double Mth = M + kThresh;      // the exact-max gate, updated with M
  double Mlo = M - o.tskip;      // the skip gate, updated with M
  for (int c0 = 0; split + c0 * nsplit < in.ntiles; c0 += kTile) {
    if (c0 != 0) cand = coarse_mask<D>(in, o, gate_min(Mlo), split, nsplit, c0);
    if (!cand) continue;
    int t = split + (c0 + __builtin_ctzll(cand)) * nsplit;
    TileVals<D> cur = load_tile<D>(in.tile + t);
    TilePts<D> pts = load_points<D>(in, t, pt);
    while (cand) {
      cand &= cand - 1;
      const int tn = cand ? split + (c0 + __builtin_ctzll(cand)) * nsplit : t;  // the last re-reads itself
      const TileVals<D> nxt = load_tile<D>(in.tile + tn);
      const TilePts<D> nps = load_points<D>(in, tn, pt);
      float a[D];
#pragma unroll
      for (int d = 0; d < D; ++d) a[d] = o.P[d] - cur.ctr[d];
      const double ub = lane_bound<D>(cur, o, a);
      // every term of this tile lies below 2^-T of the running maximum on every
      // lane: the tile cannot change any sum in float32, so it is skipped, as
      // is a tile without mass (alpha = -inf)
      if (!(__all(ub < Mlo) || __double_as_longlong(cur.alpha) == (long long)0xFFF0000000000000ULL)) {
        ++r.evaluated;
        float B[D];
        const double base = tile_base<D>(cur, o, a, B);
        if (__any(ub > Mth)) {
          // exact maximum of this tile for the lanes whose bound exceeds the window
          int qi;
          const double tmd = base + (double)tile_max_mfma<D>(pts, B, qi);
          if (ub > Mth && tmd > r.M) {
            r.S *= fast_exp2((float)(r.M - tmd));
            r.M = tmd;
            Mth = r.M + kThresh;
            Mlo = r.M - o.tskip;
            r.J = t * kTile + qi;
          }
        }
        r.S += tile_sum<D>(pts, B, (float)(base - r.M));
      }
      t = tn;
      cur = nxt;
      pts = nps;
    }
  }
  return r;
}

// The same walk with every entry evaluated on the VALU: the certificate sweep
// (cost-weighted sum N) and the barycentric sweep (coordinate sums V), whose
// weighted sums need the points per entry.  The
// weights are read with broadcast vector loads (a lane-dependent zero in the
// address), which leaves the scalar path to the offsets and the candidates'
// tile records; the next group of 8 points (after a tile's last group, the
// next candidate's first) is requested before the current group is computed.
template <int D, int MODE>
__device__ __forceinline__ SplitSum sweep_split_valu(const SweepIn& in, const SweepOut<D>& o, int split,
                                                         int nsplit, double M, int J, unsigned long long cand) {
  constexpr bool CERT = MODE == kSweepCert;
  constexpr bool BARY = MODE == kSweepBary;
  static_assert(CERT || BARY, "the plain sweep is sweep_split_mfma");
  const int lane0 = (int)__builtin_amdgcn_mbcnt_lo(0u, 0u);
  SplitSum r{M, 0.0f, 0.0f, {0.0f, 0.0f, 0.0f}, J, 0};
  double Mth = M + kThresh;      // the exact-max gate, updated with M
  double Mlo = M - o.tskip;      // the skip gate, updated with M
  Group<D> grp;
  for (int c0 = 0; split + c0 * nsplit < in.ntiles; c0 += kTile) {
    if (c0 != 0) cand = coarse_mask<D>(in, o, gate_min(Mlo), split, nsplit, c0);
    if (cand) {
      const int tf = split + (c0 + __builtin_ctzll(cand)) * nsplit;
      grp = load_group<D>(in.off + (size_t)tf * D * kTile, in.A + (size_t)tf * kTile + lane0, 0);
    }
    while (cand) {
      const int t = split + (c0 + __builtin_ctzll(cand)) * nsplit;
      cand &= cand - 1;
      const TileVals<D> cur = load_tile<D>(in.tile + t);
      const int tn = cand ? split + (c0 + __builtin_ctzll(cand)) * nsplit : t;  // next candidate (the last re-reads itself)
      // tile addresses computed before any lane-dependent branch
      gfloat* __restrict__ offs_t = in.off + (size_t)t * D * kTile;
      gfloat* __restrict__ a_t = in.A + (size_t)t * kTile + lane0;
      gfloat* __restrict__ offs_n = in.off + (size_t)tn * D * kTile;
      gfloat* __restrict__ a_n = in.A + (size_t)tn * kTile + lane0;
      float a[D];
#pragma unroll
      for (int d = 0; d < D; ++d) a[d] = o.P[d] - cur.ctr[d];
      const double ub = lane_bound<D>(cur, o, a);
      // every term of this tile lies below 2^-T of the running maximum on every
      // lane: the tile cannot change any sum in float32, so it is skipped, as
      // is a tile without mass (alpha = -inf)
      if (__all(ub < Mlo) || __double_as_longlong(cur.alpha) == (long long)0xFFF0000000000000ULL) {
        grp = load_group<D>(offs_n, a_n, 0);
        continue;
      }
      ++r.evaluated;
      float B[D];
      const double base = tile_base<D>(cur, o, a, B);
      if (ub > Mth) {
        // exact maximum of this tile for the lanes whose bound exceeds the window
        int qi;
        const double tmd = base + (double)tile_max<D>(offs_t, a_t, B, qi);
        if (tmd > r.M) {
          const float sc = fast_exp2((float)(r.M - tmd));
          r.S *= sc;
          if (CERT) r.N *= sc;
          if (BARY) {
#pragma unroll
            for (int d = 0; d < D; ++d) r.V[d] *= sc;
          }
          r.M = tmd;
          Mth = r.M + kThresh;
          Mlo = r.M - o.tskip;
          r.J = t * kTile + qi;
        }
      }
      const float cm = (float)(base - r.M);
      float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
      float n0 = 0.f, n1 = 0.f;
      float vt[D];
#pragma unroll
      for (int d = 0; d < D; ++d) vt[d] = 0.0f;
#pragma unroll
      for (int g = 0; g < kTile / kGroup; ++g) {
        // request the next group (the first group of the next tile after the last)
        const Group<D> nx = (g + 1 < kTile / kGroup) ? load_group<D>(offs_t, a_t, g + 1)
                                                    : load_group<D>(offs_n, a_n, 0);
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
          float z = cm;
#pragma unroll
          for (int d = 0; d < D; ++d) z = fmaf(B[d], grp.b[d][u], z);
          z += grp.a[u];
          const float e = fast_exp2(z);
          if (g == 0 && u < 4) {
            (u == 0 ? s0 : u == 1 ? s1 : u == 2 ? s2 : s3) = e;
          } else {
            (u % 4 == 0 ? s0 : u % 4 == 1 ? s1 : u % 4 == 2 ? s2 : s3) += e;
          }
          if (CERT) {
            float c2 = 0.0f;
#pragma unroll
            for (int d = 0; d < D; ++d) {
              const float df = a[d] - grp.b[d][u];
              c2 = fmaf(df, df, c2);
            }
            if (u & 1) n1 = fmaf(c2, e, n1); else n0 = fmaf(c2, e, n0);
          }
          if (BARY) {
#pragma unroll
            for (int d = 0; d < D; ++d) vt[d] = fmaf(e, grp.b[d][u], vt[d]);
          }
        }
        grp = nx;
      }
      const float st = (s0 + s1) + (s2 + s3);
      r.S += st;
      if (CERT) r.N += n0 + n1;
      if (BARY) {
        // sum_q e_q y_q = c_t sum_q e_q + sum_q e_q b_q (points = tile centre + offset)
#pragma unroll
        for (int d = 0; d < D; ++d) r.V[d] += fmaf(cur.ctr[d], st, vt[d]);
      }
    }
  }
  return r;
}

template <int D, int MODE>
__device__ __forceinline__ SplitSum sweep_split(const SweepIn& in, const SweepOut<D>& o, int split, int nsplit,
                                                double M, int J, unsigned long long cand) {
  if constexpr (MODE == kSweepPlain) return sweep_split_mfma<D>(in, o, split, nsplit, M, J, cand);
  else return sweep_split_valu<D, MODE>(in, o, split, nsplit, M, J, cand);
}

// A split's record: the shift relative to the output's reference in float32,
// the sums rescaled by that rounding so that the record is exact.
template <typename Rec>
__device__ __forceinline__ Rec make_rec(const SplitSum& r, double Rref) {
  float dM = -INFINITY, fix = 1.0f;
  if (r.M > -INFINITY) {
    const double dd = r.M - Rref;
    dM = (float)dd;
    fix = fast_exp2((float)(dd - (double)dM));
  }
  if constexpr (sizeof(Rec) == sizeof(PartialCert)) return Rec{dM, r.S * fix, r.N * fix, r.J};
  else return Rec{dM, r.S * fix, r.J};
}

template <int MODE>
struct RecOf { typedef PartialRec type; };
template <>
struct RecOf<kSweepCert> { typedef PartialCert type; };

// Wavefronts per SIMD that a sweep's registers must leave room for (a minimum:
// the compiler may need fewer registers), as measured.  Plain: d = 3 at 5 (at 6 it
// spills, 4 is 5% slower), d = 1 and 2 at 6 (at 5 the compiler interleaves the
// quarters, which spills for d = 2 and is 3% slower).  With costs or coordinates
// at 4, where 5 to 7 come out (asking for 5 or 6 was 1 to 2% slower).
template <int D, int MODE>
constexpr int sweep_waves() {
  return MODE != kSweepPlain ? 4 : D == 3 ? 5 : 6;
}

// One block of kSweepBlock outputs (bx) against one split of the input tiles,
// its records written to memory for k_finish.
template <int D, int MODE, bool ROW, bool BATCH>
__device__ __forceinline__ void sweep_block(const LaunchCtx& c, int nsplit, double eps, int own, int kofs, int bx,
                                            int split, unsigned* __restrict__ tile_count, int slot) {
  constexpr bool BARY = MODE == kSweepBary;
  const SideDev& out = ROW ? c.rows : c.cols;
  const SideDev& ins = ROW ? c.cols : c.rows;
  const SweepIn in = sweep_in(ins);
  const Partials part = c.part;
  // arguments that are used late are loaded with the others all the same: the
  // compiler would load them where they are used, a scalar round trip each
  asm volatile("" ::"s"(ins.tskip), "s"(part.ref), "s"(part.rec), "s"(tile_count), "s"(in.off), "s"(in.A), "s"(c.ctrl));
  const int np_out = out.np;
  const int p = bx * kSweepBlock + threadIdx.x;
  const int lane = (int)(threadIdx.x & (kTile - 1));
  // everything that depends on the arguments alone is requested first: a
  // wavefront's start is round trips (these, then the warm start's gather)
  float P[D];
#pragma unroll
  for (int d = 0; d < D; ++d) P[d] = ((gfloat*)out.abs)[(size_t)d * np_out + p];
  const int j_hint = ((gint*)out.hint)[p];
  const int t = split + lane * nsplit;
  const TileVals<D> first = load_tile<D>(in.tile + min(t, in.ntiles - 1));
  // (past the last tile: padding, copies of a point of the last tile)
  const int tile = min(bx * (kSweepBlock / kTile) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kTile)),
                       out.ntiles - 1);
  const TileVals<D> own_tile = load_tile<D>((gtile*)out.tile + tile);
  const CtrlVals raw = load_ctrl(c.ctrl);
  __builtin_amdgcn_sched_barrier(0);  // all of it under way before the first wait
  const CtrlVals cv = with_eps(raw, eps, own != 0);
  const SweepOut<D> o = sweep_out<D, BATCH>(P, own_tile, kap2_of<ROW>(cv, kofs), (double)ins.tskip);
  double M;
  int J;
  warm_start<D>(in, o, j_hint, M, J);
  const double cub = coarse_of<D>(first, o);
  // the records' reference: the warm start's exponent (the same in every
  // split), 0 without one; split 0 stores it for the merge
  const double Rref = M > -INFINITY ? M : 0.0;
  if (!BARY && split == 0) part.ref[p] = Rref;
  const double gate = gate_min(M - o.tskip);  // a reduction over the wavefront: not under a lane's condition
  const unsigned long long cand = __ballot(t < in.ntiles && !(cub < gate));
  const SplitSum r = sweep_split<D, MODE>(in, o, split, nsplit, M, J, cand);
  if (tile_count && lane == 0) tile_count[slot] = (unsigned)r.evaluated;
  if constexpr (BARY) {
    PartialBary* pb = reinterpret_cast<PartialBary*>(part.rec) + (size_t)split * np_out + p;
    pb->M = r.M;
    pb->S = r.S;
    for (int d = 0; d < 3; ++d) pb->V[d] = r.V[d];
  } else {
    typedef typename RecOf<MODE>::type Rec;
    reinterpret_cast<Rec*>(part.rec)[(size_t)split * np_out + p] = make_rec<Rec>(r, Rref);
  }
}

// The direction is a template parameter, as the dimension and the mode, so that
// every argument sits at a fixed place and all of them are loaded at once.
template <int D, int MODE, bool ROW>
__global__ __launch_bounds__(kSweepBlock) __attribute__((amdgpu_waves_per_eu(sweep_waves<D, MODE>()))) void k_sweep(
    LaunchCtx c, int nsplit, double eps, int own, int kofs) {
  // blockIdx.x is the split and blockIdx.y the output block:
  // consecutive workgroups go to consecutive XCDs, so the splits of one output
  // block spread over all XCDs (a heavy output region does not load one XCD)
  // and each XCD reads the input tiles of only part of the splits (its L2
  // holds just those)
  const int slot = (blockIdx.y * gridDim.x + blockIdx.x) * (kSweepBlock / kTile) + threadIdx.x / kTile;
  sweep_block<D, MODE, ROW, false>(c, nsplit, eps, own, kofs, blockIdx.y, blockIdx.x, c.tile_count, slot);
}

// Batched sweep: block i runs work item i = (problem, block of outputs, split)
// of a list over several problems; the arithmetic per item is the same as in
// the single-problem launch.
template <int D, int MODE, bool ROW>
__global__ __launch_bounds__(kSweepBlock) __attribute__((amdgpu_waves_per_eu(sweep_waves<D, MODE>()))) void k_sweep_batch(
    const BatchItem* __restrict__ items, const LaunchCtx* __restrict__ descs, int kofs) {
  const BatchItem it = items[blockIdx.x];
  const LaunchCtx& c = descs[it.prob];
  sweep_block<D, MODE, ROW, true>(c, ROW ? c.splits_row : c.splits_col, 0.0, 0, kofs, it.blk, it.split, nullptr, 0);
}

// ---------------------------------------------------------------------------
// Finish: merge the split partials (float64) and run the epilogue.
// ---------------------------------------------------------------------------
struct Merged {
  double lse;   // natural-log LSE
  double S;     // merged shifted sum (relative to Mx)
  double N;     // merged shifted cost sum
  int J;        // input slot of the exact maximum of the winning split, or -1
};

// One split's record as the merge reads it.
struct SplitRec {
  float dM, S, N;
  int J;
};
__device__ __forceinline__ SplitRec split_rec(const PartialRec& q) { return SplitRec{q.dM, q.S, 0.0f, q.J}; }
__device__ __forceinline__ SplitRec split_rec(const PartialCert& q) { return SplitRec{q.dM, q.S, q.N, q.J}; }

template <bool CERT, typename Load, typename Meanwhile>
__device__ __forceinline__ Merged merge_splits_t(Load load, double R, int splits, Meanwhile meanwhile) {
  // The epilogue runs few waves, so its time is the number of memory round
  // trips: one pass over the split records, G of them requested together.
  // Past the last split the index is clamped to a valid record and its shift
  // gets -inf added (so its weight is 0): every loaded value is used
  // unconditionally, which keeps the loads together (a load the compiler may
  // sink under a branch waits for its data before the next one is issued).
  // Each batch is merged against the running maximum, which is raised first
  // if the batch holds a larger one (the running sums are rescaled).  Shifts
  // are relative to the output's reference R.
  constexpr int G = 16;
  float mx = -INFINITY;
  double S = 0.0, N = 0.0;
  int J = -1;
  auto batch = [&](int s0) {
    SplitRec q[G];
#pragma unroll
    for (int g = 0; g < G; ++g) q[g] = load(min(s0 + g, splits - 1));
    if (s0 == 0) meanwhile();
#pragma unroll
    for (int g = 0; g < G; ++g) q[g].dM += (s0 + g < splits) ? 0.0f : -INFINITY;
    float bm = -INFINITY;
    int bj = -1;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const bool up = q[g].dM > bm;  // the first split holding the batch maximum
      bj = up ? q[g].J : bj;
      bm = up ? q[g].dM : bm;
    }
    if (bm > mx) {  // strictly: J stays with the first split holding the maximum
      // shifts of one output differ by little: the weight is a hardware float32 exp2
      const double sc = mx == -INFINITY ? 0.0 : (double)fast_exp2(mx - bm);
      S *= sc;
      if (CERT) N *= sc;
      mx = bm;
      J = bj;
    }
    if (mx == -INFINITY) return;  // nothing so far
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const double w = (double)fast_exp2(q[g].dM - mx);  // 0 for an empty or masked split
      S += w * (double)q[g].S;
      if (CERT) N += w * (double)q[g].N;
    }
  };
  // the first batch outside the loop: at a loop header the wait counts are
  // merged conservatively, which would wait for the loads issued before it
  batch(0);
  for (int s0 = G; s0 < splits; s0 += G) batch(s0);
  Merged r{-INFINITY, 0.0, 0.0, -1};
  if (mx == -INFINITY) return r;  // empty sum
  r.S = S;
  r.N = N;
  r.J = J;
  r.lse = kLn2D * ((R + (double)mx) + log2(S));
  return r;
}

template <bool CERT, typename Meanwhile>
__device__ __forceinline__ Merged merge_splits(const Partials& pt, int splits, int np, int p, Meanwhile meanwhile) {
  const double R = pt.ref[p];
  if constexpr (CERT) {
    const PartialCert* rec = reinterpret_cast<const PartialCert*>(pt.rec) + p;
    return merge_splits_t<true>([=](int s) { return split_rec(rec[(size_t)s * np]); }, R, splits, meanwhile);
  } else {
    const PartialRec* rec = reinterpret_cast<const PartialRec*>(pt.rec) + p;
    return merge_splits_t<false>([=](int s) { return split_rec(rec[(size_t)s * np]); }, R, splits, meanwhile);
  }
}

// Packs the weights w of one tile for the sweeps: a least-squares plane
// w2 ~ alpha + gamma . b of the tile's log2 weights w2 = log2(e) w over the
// offsets b, with its largest residual rho (so w2 <= alpha + gamma . b + rho
// holds for every point of the tile, whatever the fit: the sweep turns it
// into an upper bound of its exponents), and per point
// A_p = w2_p - alpha - gamma . b_p - kappa2 |b_p|^2 in float32 (-inf on padding
// or for w = -inf), the part of the exponent that does not depend on the
// output; alpha is -inf when the tile has no mass.  Called by whole wavefronts
// (one tile each).
// Offsets of point p from its tile centre (0 past the real points); the
// epilogues request them before they wait for the split records.
// Loads at clamped (valid) addresses whatever p is, zeroed by a multiplication
// (offsets are finite) rather than a select, so that every loaded value is
// used and the loads issue together.
template <int D>
struct Offsets {
  float b[D];
};
template <int D>
__device__ __forceinline__ Offsets<D> load_offsets(const SideDev& sd, int p) {
  const int t = min(p, sd.count - 1) / kTile, q = p % kTile;
  const float* base = sd.off + (size_t)t * D * kTile + q;
  Offsets<D> o;
#pragma unroll
  for (int d = 0; d < D; ++d) o.b[d] = base[(size_t)d * kTile] * (p < sd.count ? 1.0f : 0.0f);
  return o;
}

// Geometry of the tile that the wavefront's points p belong to.
template <int D>
struct Geom {
  double mb[D], cinv[6], cnt;
};
template <int D>
__device__ __forceinline__ Geom<D> load_geom(const SideDev& sd, int p) {
  typedef __attribute__((address_space(4))) const TileGeom cgeom;  // scalar loads
  cgeom* t = (cgeom*)sd.geom + __builtin_amdgcn_readfirstlane(min(p / kTile, sd.ntiles - 1));
  Geom<D> g;
#pragma unroll
  for (int d = 0; d < D; ++d) g.mb[d] = t->mb[d];
#pragma unroll
  for (int i = 0; i < 6; ++i) g.cinv[i] = t->cinv[i];
  g.cnt = t->cnt;
  return g;
}

template <int D>
__device__ __forceinline__ void pack_weight_d(const SideDev& sd, const Geom<D>& g, int p, double w, double kap2,
                                              const Offsets<D>& bo) {
  constexpr int dim = D;
  const bool live = p < sd.count && w > -INFINITY;
  const int t = p / kTile;
  double w2 = 0.0;
  double b[D];
  float n2 = 0.0f;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    b[d] = (double)bo.b[d];
    n2 = fmaf(bo.b[d], bo.b[d], n2);
  }
  if (live) w2 = kLog2eD * w;
  if (p >= sd.ntiles * kTile) return;
  double gam[3] = {0.0, 0.0, 0.0}, alpha = -INFINITY;
  // least-squares plane through the live points of the tile (centred sums).
  // When the live points are the tile's real points (every weight finite, as
  // in the iterations: the marginals are positive), their geometry is the
  // tile's precomputed one and the fit needs only the sums of w2 and of the
  // centred offsets times w2 (the centred offsets sum to zero, so the latter
  // is the centred cross sum), all taken at once.
  const int nreal = min(kTile, sd.count - t * kTile);
  const unsigned long long real_mask = nreal >= kTile ? ~0ull : ((1ull << nreal) - 1ull);
  if (__ballot(live) == real_mask) {
    const double wl = live ? w2 : 0.0;
    double v[D + 1];
    v[0] = wl;
#pragma unroll
    for (int d = 0; d < D; ++d) v[d + 1] = live ? (b[d] - g.mb[d]) * wl : 0.0;
    wave_sum_n<D + 1>(v);
    const double mw = nreal == kTile ? v[0] * (1.0 / kTile) : v[0] / g.cnt;
    // symmetric inverse stored as xx, xy, xz, yy, yz, zz
    constexpr int kSym[3][3] = {{0, 1, 2}, {1, 3, 4}, {2, 4, 5}};
    alpha = mw;
#pragma unroll
    for (int d = 0; d < D; ++d) {
      double s = 0.0;
#pragma unroll
      for (int e = 0; e < D; ++e) s = fma(g.cinv[kSym[d][e]], v[e + 1], s);
      gam[d] = (double)(float)s;  // the sweep reads gamma as float32
      alpha -= gam[d] * g.mb[d];
    }
  } else {
    const double one = live ? 1.0 : 0.0;
    const double cnt = wave_sum(one);
    double mb[D], mw = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) mb[d] = 0.0;
    if (cnt > 0.0) {
      for (int d = 0; d < dim; ++d) mb[d] = wave_sum(one * b[d]) / cnt;
      mw = wave_sum(live ? w2 : 0.0) / cnt;
      double cbb[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, cbw[3] = {0, 0, 0};
      for (int d = 0; d < dim; ++d) {
        const double bd = live ? b[d] - mb[d] : 0.0;
        cbw[d] = wave_sum(bd * (live ? w2 - mw : 0.0));
        for (int e = 0; e <= d; ++e) {
          cbb[d][e] = wave_sum(bd * (live ? b[e] - mb[e] : 0.0));
          cbb[e][d] = cbb[d][e];
        }
      }
      // solve cbb gamma = cbw by Cramer's rule; a (near-)singular system keeps gamma = 0
      if constexpr (D == 1) {
        if (cbb[0][0] > 1e-12) gam[0] = cbw[0] / cbb[0][0];
      } else if constexpr (D == 2) {
        const double det = cbb[0][0] * cbb[1][1] - cbb[0][1] * cbb[1][0];
        if (fabs(det) > 1e-12 * (cbb[0][0] * cbb[1][1] + 1e-300)) {
          gam[0] = (cbw[0] * cbb[1][1] - cbb[0][1] * cbw[1]) / det;
          gam[1] = (cbb[0][0] * cbw[1] - cbw[0] * cbb[1][0]) / det;
        }
      } else {
        const double a00 = cbb[1][1] * cbb[2][2] - cbb[1][2] * cbb[2][1];
        const double a01 = cbb[0][2] * cbb[2][1] - cbb[0][1] * cbb[2][2];
        const double a02 = cbb[0][1] * cbb[1][2] - cbb[0][2] * cbb[1][1];
        const double det = cbb[0][0] * a00 + cbb[1][0] * a01 + cbb[2][0] * a02;
        if (fabs(det) > 1e-12 * (cbb[0][0] * cbb[1][1] * cbb[2][2] + 1e-300)) {
          const double a10 = cbb[1][2] * cbb[2][0] - cbb[1][0] * cbb[2][2];
          const double a11 = cbb[0][0] * cbb[2][2] - cbb[0][2] * cbb[2][0];
          const double a12 = cbb[0][2] * cbb[1][0] - cbb[0][0] * cbb[1][2];
          const double a20 = cbb[1][0] * cbb[2][1] - cbb[1][1] * cbb[2][0];
          const double a21 = cbb[0][1] * cbb[2][0] - cbb[0][0] * cbb[2][1];
          const double a22 = cbb[0][0] * cbb[1][1] - cbb[0][1] * cbb[1][0];
          gam[0] = (a00 * cbw[0] + a01 * cbw[1] + a02 * cbw[2]) / det;
          gam[1] = (a10 * cbw[0] + a11 * cbw[1] + a12 * cbw[2]) / det;
          gam[2] = (a20 * cbw[0] + a21 * cbw[1] + a22 * cbw[2]) / det;
        }
      }
      for (int d = 0; d < dim; ++d) gam[d] = (double)(float)gam[d];  // the sweep reads gamma as float32
      alpha = mw;
      for (int d = 0; d < dim; ++d) alpha -= gam[d] * mb[d];
    }
  }
  double res = 0.0;
  if (live) {
    res = w2 - alpha;
    for (int d = 0; d < dim; ++d) res -= gam[d] * b[d];
  }
  // the weight's residual from the plane minus the tile-local quadratic
  sd.A[p] = live ? (float)(res - kap2 * (double)n2) : -INFINITY;
  const double rho = wave_max(fabs(res));
  if ((threadIdx.x & (kTile - 1)) == 0) {
    TileRec& tr = sd.tile[t];
    tr.alpha = alpha;
    for (int d = 0; d < 3; ++d) tr.gam[d] = (float)gam[d];
    tr.rho = (float)(rho * (1.0 + 1e-6)) + 1e-3f;  // rounded up: the bound must hold
  }
}

__device__ __forceinline__ void pack_weight(const SideDev& sd, int dim, int p, double w, double kap2) {
  if (dim == 1) pack_weight_d<1>(sd, load_geom<1>(sd, p), p, w, kap2, load_offsets<1>(sd, p));
  else if (dim == 2) pack_weight_d<2>(sd, load_geom<2>(sd, p), p, w, kap2, load_offsets<2>(sd, p));
  else pack_weight_d<3>(sd, load_geom<3>(sd, p), p, w, kap2, load_offsets<3>(sd, p));
}

// Merge of the barycentric partials of output p: shift, shifted sum and the
// shifted coordinate sums, in float64.
struct MergedBary {
  double lse;   // natural-log LSE
  double V[3];  // coordinate sums relative to the merged sum
};

__device__ __forceinline__ MergedBary merge_bary(const void* __restrict__ part, int splits, int np, int p) {
  const PartialBary* pb = reinterpret_cast<const PartialBary*>(part);
  double mx = -INFINITY;
  for (int s = 0; s < splits; ++s) mx = fmax(mx, pb[(size_t)s * np + p].M);
  MergedBary r;
  double S = 0.0, V[3] = {0.0, 0.0, 0.0};
  if (mx > -INFINITY) {
    for (int s = 0; s < splits; ++s) {
      const PartialBary q = pb[(size_t)s * np + p];
      const double w = exp2(q.M - mx);
      S += w * (double)q.S;
      for (int d = 0; d < 3; ++d) V[d] += w * (double)q.V[d];
    }
  }
  r.lse = kLn2D * (mx + log2(S));
  for (int d = 0; d < 3; ++d) r.V[d] = S > 0.0 ? V[d] / S : 0.0;
  return r;
}

// What the epilogues read that does not depend on the merge.
template <int D>
struct FinishPre {
  CtrlVals cv;
  Offsets<D> bo;                   // offsets the packing needs
  double lm, s, t0, t1;            // log marginal and dual state of output p
  Geom<D> geom;                    // of the tile being packed
};

// An epilogue runs one wavefront per output tile, so its time is the number
// of memory round trips: these loads are issued before the split records are
// waited for.  Unconditional (p < np, and every array read here holds np
// entries of the output side): a load under a branch is waited for there.
// ITER: an iteration's epilogue (the others read the control block alone).
template <int D, bool ROW, bool ITER>
__device__ __forceinline__ FinishPre<D> finish_loads(const LaunchCtx& c, int p) {
  const SideDev& out = ROW ? c.rows : c.cols;
  FinishPre<D> f;
  if (!ITER) {
    f.cv = load_ctrl(c.ctrl);
    return f;
  }
  f.bo = load_offsets<D>(out, p);
  f.lm = out.logmarg[p];
  f.s = (ROW ? c.st.la : c.st.lb1)[p];
  f.t0 = f.t1 = 0.0;
  if (!ROW) {
    f.t0 = c.st.lt[0][p];
    f.t1 = c.st.lt[1][p];
  }
  f.geom = load_geom<D>(out, p);
  f.cv = load_ctrl(c.ctrl);
  return f;
}

constexpr bool finish_iterates(int kind) {
  return kind == kFinishRow || kind == kFinishCol || kind == kFinishColCert;
}

// Epilogue of output p from its merged sums (whole wavefronts, one output
// tile each).
template <int D, int kind, bool ROW>
__device__ __forceinline__ void finish_out(const LaunchCtx& c, double* __restrict__ lse_out, int p, int kofs,
                                           const Merged& mg, const FinishPre<D>& pre) {
  const SideDev& out = ROW ? c.rows : c.cols;
  const bool real = p < out.count;
  constexpr bool cert = kind == kFinishColCert;
  const double pre_lm = pre.lm, pre_s = pre.s, pre_t0 = pre.t0, pre_t1 = pre.t1;
  // the warm start of the next sweep of this side: only the iteration's own sweeps set it
  if (finish_iterates(kind) && real && mg.J >= 0) out.hint[p] = mg.J;
  const CtrlVals* ctrl = &pre.cv;
  const long long k = ctrl->k + kofs;  // this iteration: the block's first plus the offset
  const double lam = ctrl->lam;

  if constexpr (kind == kFinishLse) {
    if (real) lse_out[out.perm[p]] = mg.lse;
    return;
  }
  if constexpr (kind == kFinishPlanCol) {
    // (X^T 1)_j = beta_j sum_i K_ij alpha_i
    if (real) c.plan_col[p] = exp(c.st.lb1[p] + mg.lse);
    return;
  }
  // two-sided rounding of the state plan (Altschuler, Weed and Rigollet 2017, Algorithm 2)
  if constexpr (kind == kFinishRound1) {
    // log x_i = min(0, log r_i - log (X 1)_i)
    if (real) c.plan_row[p] = fmin(0.0, out.logmarg[p] - (c.st.la[p] + mg.lse));
    return;
  }
  if constexpr (kind == kFinishRound2) {
    // X' = diag(x) X: log y_j = min(0, log c_j - log (X'^T 1)_j); deficit c_j - y_j (X'^T 1)_j
    if (real) {
      const double lcol = c.st.lb1[p] + mg.lse;
      const double ly = fmin(0.0, out.logmarg[p] - lcol);
      c.plan_col[p] = ly;
      // nonnegative by construction; the clamp removes an ulp of rounding
      // where y_j = c_j / (X'^T 1)_j, so that every entry of G is >= 0
      c.st.mu[p] = fmax(0.0, out.marg[p] - exp(lcol + ly));
    }
    return;
  }
  if constexpr (kind == kFinishRound3) {
    // X'' = diag(x) X diag(y): row deficit r_i - (X'' 1)_i and sum_j X''_ij C_ij
    if (real) {
      const double row2 = exp(c.st.la[p] + c.plan_row[p] + mg.lse);
      c.plan_aux[p] = fmax(0.0, out.marg[p] - row2);
      c.st.pvec[p] = row2 * ctrl->scale * mg.N / mg.S;
    }
    return;
  }
  if constexpr (kind == kFinishCertOnly) {
    // Algorithm 2 for the last finished iteration k-1 (k has been advanced)
    if (real) {
      c.st.mu[p] = ctrl->scale * mg.N / mg.S;
      c.st.logs[p] = c.st.lt[(k - 1) & 1][p] + mg.lse;
    }
    return;
  }
  if constexpr (kind == kFinishRepair) {
    // p_i = A_i sum_j K_ij t_j (1 - e_j) = exp(log alpha-hat_i + LSE_i)
    c.st.pvec[p] = real ? exp(c.st.lah[p] + mg.lse) : 0.0;
    return;
  }
  if constexpr (kind == kFinishRow) {
    // row update of Algorithm 1: the unrelaxed row scaling normalises the rows to r; the
    // relaxed one mixes it with the previous relaxed scaling, weight lambda on the new one
    const double kap2 = kap2_of<false>(*ctrl, kofs);
    double colw = 0.0;
    if (real) {
      const double lah = pre_lm - mg.lse;
      c.st.lah[p] = lah;
      if (ctrl->variant & kVarDebiased) {
        // debiased row update: log a^k = theta_k log a^{k-1} + log r - LSE, theta_k = 0 (k <= 1), 1/k
        const double theta = k <= 1 ? 0.0 : 1.0 / (double)k;
        colw = theta * pre_s + lah;
        c.st.la[p] = colw;
      } else {
        // one rounded product fused into the other: fixed whatever the
        // compiler's contraction (the result is exact for lambda = 1)
        c.st.la[p] = fma(lam, lah, (1.0 - lam) * pre_s);
        colw = lah;
      }
    }
    // weights of the column sweep of the same iteration: log alpha-hat (the
    // debiased variant: its row scaling a^k)
    pack_weight_d<D>(c.rows, pre.geom, p, colw, kap2, pre.bo);
    return;
  }
  if constexpr (kind == kFinishCol || kind == kFinishColCert) {
    // column epilogue (plain or certificate)
    const int cur = (int)(k & 1), nxt = (int)((k + 1) & 1);
    double lt_next = 0.0;
    if (real) {
      const double lbh = pre_lm - mg.lse;                 // log beta-hat^k = log c - LSE
      const double lb1 = pre_s;
      const double lb = fma(lam, lbh, (1.0 - lam) * lb1);  // log beta^k (rounding as for alpha)
      if (cert) {
        // certificate statistics of the intermediate plan's column (Prop. 3, Algorithm 2):
        // its mean cost (cost-weighted over plain merged sums) and the log of its mass
        c.st.mu[p] = ctrl->scale * mg.N / mg.S;
        c.st.logs[p] = (cur ? pre_t1 : pre_t0) + mg.lse;
      }
      c.st.lbh[p] = lbh;
      c.st.lb2[p] = lb1;
      c.st.lb1[p] = lb;
      // momentum for iteration k+1: log beta-tilde^k = log beta^k + (log beta^k - log beta^{k-1}) / lambda
      lt_next = (ctrl->variant & kVarNoMomentum) ? lb : lb + (lam == 1.0 ? lb - lb1 : (lb - lb1) / lam);
      c.st.lt[nxt][p] = lt_next;
    }
    pack_weight_d<D>(c.cols, pre.geom, p, lt_next, kap2_of<true>(*ctrl, kofs + 1), pre.bo);
  }
}

// Merge of the records in memory + epilogue of one tile (bx) of 64 outputs.
// The kind is a template parameter: compiled together, the kinds of all
// dimensions were 13000 instructions, and the arguments of an iteration's
// epilogue were loaded in a chain of scalar round trips behind its branches.
template <int D, int kind, bool ROW>
__device__ __forceinline__ void finish_block(const LaunchCtx& c, int splits, double* __restrict__ lse_out, int bx,
                                             int kofs) {
  const SideDev& out = ROW ? c.rows : c.cols;
  const int p = bx * kTile + threadIdx.x;
  const int np = out.np;
  if constexpr (kind == kFinishPlanRow) {
    // state plan: (X 1)_i = alpha_i sum_j K_ij beta_j, barycentre sum_j X_ij y_j / (X 1)_i
    const MergedBary mb = merge_bary(c.part.rec, splits, np, p);
    if (p < out.count) {
      c.plan_row[p] = exp(c.st.la[p] + mb.lse);
      if (lse_out) {
        const int i = out.perm[p];
#pragma unroll
        for (int d = 0; d < D; ++d) lse_out[(size_t)i * D + d] = c.origin[d] + mb.V[d];
      }
    }
  } else {
    // the arguments of the later part loaded with the first ones, and the scalar
    // loads of the control block and the tile geometry waited for while the
    // records are under way (the compiler would issue each where it is used)
    asm volatile("" ::"s"(c.ctrl), "s"(out.geom), "s"(out.A), "s"(out.tile), "s"(out.hint), "s"(c.part.rec));
    const FinishPre<D> pre = finish_loads<D, ROW, finish_iterates(kind)>(c, p);
    // the sweeps that gathered cost-weighted sums wrote certificate records
    constexpr bool cert_rec = kind == kFinishColCert || kind == kFinishCertOnly || kind == kFinishRound3;
    const Merged mg = merge_splits<cert_rec>(c.part, splits, np, p, [&]() {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::"s"(pre.cv.k), "s"(pre.cv.lam), "s"(pre.cv.scale), "s"(pre.cv.variant));
      if constexpr (finish_iterates(kind)) {
        asm volatile("" ::"s"(pre.cv.eta), "s"(pre.geom.cnt), "s"(pre.geom.cinv[0]), "s"(pre.geom.cinv[D]));
#pragma unroll
        for (int d = 0; d < D; ++d) asm volatile("" ::"s"(pre.geom.mb[d]));
      }
    });
    finish_out<D, kind, ROW>(c, lse_out, p, kofs, mg, pre);
  }
}

template <int D, int kind, bool ROW>
__global__ __launch_bounds__(kTile) void k_finish(LaunchCtx c, int splits, double* __restrict__ lse_out, int kofs) {
  finish_block<D, kind, ROW>(c, splits, lse_out, blockIdx.x, kofs);
}

// Advances the iteration counter by n after a block of n iterations (kernels of
// the block read the block's first iteration and take their offset as an
// argument, so a captured block replays at any k).
__global__ void k_advance(Ctrl* ctrl, int n) {
  if (threadIdx.x == 0) ctrl->k += n;
}

__global__ void k_advance_batch(const LaunchCtx* __restrict__ descs, int count, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) descs[i].ctrl->k += n;
}

// Batched merge + epilogue: block i runs item i = (problem, output tile).
template <int D, int kind, bool ROW>
__global__ __launch_bounds__(kTile) void k_finish_batch(const BatchItem* __restrict__ items,
                                                        const LaunchCtx* __restrict__ descs, int kofs) {
  const BatchItem it = items[blockIdx.x];
  const LaunchCtx& c = descs[it.prob];
  finish_block<D, kind, ROW>(c, ROW ? c.splits_row : c.splits_col, nullptr, it.blk, kofs);
}

// lt and A_C of iteration k from the stored log beta^{k-1}, log beta^{k-2}.
__device__ __forceinline__ void prologue_block(const LaunchCtx& c, int bx) {
  const int p = bx * kBlock + threadIdx.x;
  if (p >= c.cols.np) return;
  const long long k = c.ctrl->k;
  const double lam = c.ctrl->lam;
  const bool real = p < c.cols.count;
  double lt = 0.0;
  if (real) {
    const double lb1 = c.st.lb1[p], lb2 = c.st.lb2[p];
    lt = (c.ctrl->variant & kVarNoMomentum) ? lb1 : lb1 + (lb1 - lb2) / lam;
    c.st.lt[k & 1][p] = lt;
  }
  const double kap2 = kap2_of<true>(load_ctrl(c.ctrl), 0);
  pack_weight(c.cols, c.dim, p, lt, kap2);
}

__global__ __launch_bounds__(kBlock) void k_prologue(LaunchCtx c) { prologue_block(c, blockIdx.x); }

// Restores both sides' weights after the sweep buffers were used otherwise: the
// first col_blocks blocks are the prologue's, the others write rows.A from log
// alpha-hat of iteration k - 1 at that iteration's temperature (none at k = 0).
// One launch for both, and the temperature from the control block, so that the
// host need not read k back first.
__global__ __launch_bounds__(kBlock) void k_repack(LaunchCtx c, int col_blocks) {
  if ((int)blockIdx.x < col_blocks) return prologue_block(c, blockIdx.x);
  const int p = (blockIdx.x - col_blocks) * kBlock + threadIdx.x;
  const long long k = c.ctrl->k - 1;
  if (p >= c.rows.np || k < 0) return;
  double eps;
  {
#pragma clang fp contract(off)  // as the host rounds it
    const double den = c.ctrl->lam * (double)k + 1.0;
    eps = c.ctrl->variant & kVarOldKernel ? (k >= 1 ? c.ctrl->eta / (double)k : c.ctrl->eta * kFarTemperature)
                                          : c.ctrl->eta / den;
  }
  const double kap2 = kLog2eD * c.ctrl->scale / eps;
  pack_weight(c.rows, c.dim, p, p < c.rows.count ? c.st.lah[p] : 0.0, kap2);
}

// A of the input side from caller weights w (original order), for bdrs_lse.
__global__ __launch_bounds__(kBlock) void k_pack(LaunchCtx c, int transpose, const double* __restrict__ w,
                                                 double eps) {
  const SideDev& in = transpose ? c.rows : c.cols;
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= in.np) return;
  const double kap2 = kLog2eD * c.ctrl->scale / eps;
  const double wv = p < in.count ? w[in.perm[p]] : 0.0;
  pack_weight(in, c.dim, p, wv, kap2);
}

// State-plan weights of the input side: log beta^{k-1} on the columns (row sums
// and barycentres), log alpha^{k-1} on the rows (column sums), at temperature eps.
__global__ __launch_bounds__(kBlock) void k_pack_state(LaunchCtx c, int transpose, double eps, int with_factors) {
  const SideDev& in = transpose ? c.rows : c.cols;
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= in.np) return;
  const double kap2 = kLog2eD * c.ctrl->scale / eps;
  const double* w = transpose ? c.st.la : c.st.lb1;
  const double* f = transpose ? c.plan_row : c.plan_col;
  double v = 0.0;
  if (p < in.count) v = with_factors ? w[p] + f[p] : w[p];
  pack_weight(in, c.dim, p, v, kap2);
}

// Marginal-error statistics of the state plan (float64): per block partial
// sums / maxima over both sides, then one block combines them in order.
// Partial layout per block: row l1, row max abs, row max rel, col l1, col max
// abs, col max rel, total mass, pad.
__global__ __launch_bounds__(kBlock) void k_plan_partial(LaunchCtx c) {
  __shared__ double sh[kBlock / kTile][8];
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int stride = gridDim.x * kBlock;
  for (int p = blockIdx.x * kBlock + threadIdx.x; p < c.rows.count; p += stride) {
    const double r = c.rows.marg[p], x = c.plan_row[p];
    const double e = fabs(x - r);
    v[0] += e;
    v[1] = fmax(v[1], e);
    v[2] = fmax(v[2], e / r);
    v[6] += x;
  }
  for (int p = blockIdx.x * kBlock + threadIdx.x; p < c.cols.count; p += stride) {
    const double cj = c.cols.marg[p];
    const double e = fabs(c.plan_col[p] - cj);
    v[3] += e;
    v[4] = fmax(v[4], e);
    v[5] = fmax(v[5], e / cj);
  }
  v[0] = wave_sum(v[0]);
  v[3] = wave_sum(v[3]);
  v[6] = wave_sum(v[6]);
  v[1] = wave_max(v[1]);
  v[2] = wave_max(v[2]);
  v[4] = wave_max(v[4]);
  v[5] = wave_max(v[5]);
  const int wv = threadIdx.x / kTile;
  if ((threadIdx.x & (kTile - 1)) == 0)
    for (int i = 0; i < 8; ++i) sh[wv][i] = v[i];
  __syncthreads();
  if (threadIdx.x < 8) {
    const int i = threadIdx.x;
    double a = sh[0][i];
    for (int w = 1; w < kBlock / kTile; ++w) a = (i == 0 || i == 3 || i == 6) ? a + sh[w][i] : fmax(a, sh[w][i]);
    c.cert_part[(size_t)blockIdx.x * 8 + i] = a;
  }
}

__global__ __launch_bounds__(kBlock) void k_plan_final(LaunchCtx c, int nblocks) {
  // all partials are requested at once and then combined in block order from
  // LDS (one by one from memory it was a round trip per block: 45 us)
  __shared__ double part[kMaxCertBlocks * 8];
  for (int i = threadIdx.x; i < nblocks * 8; i += kBlock) part[i] = c.cert_part[i];
  __syncthreads();
  if (threadIdx.x < 8) {
    const int i = threadIdx.x;
    const bool sum = i == 0 || i == 3 || i == 6;
    double a = part[i];
    for (int b = 1; b < nblocks; ++b) {
      const double x = part[b * 8 + i];
      a = sum ? a + x : fmax(a, x);
    }
    c.plan_stats[i] = a;
  }
}

// Repair weights: log t_j + log(1 - e_j), e_j = min(1, c_j / s_j) (-inf where e_j = 1).
__global__ __launch_bounds__(kBlock) void k_repair_pack(LaunchCtx c) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p >= c.cols.np) return;
  const long long k = c.ctrl->k - 1;  // the certified iteration
  double w = -INFINITY;
  if (p < c.cols.count) {
    const double s = exp(c.st.logs[p]);
    const double cj = c.cols.marg[p];
    if (s > cj) w = c.st.lt[k & 1][p] + log1p(-cj / s);
  }
  const double kap2 = kap2_of<true>(load_ctrl(c.ctrl), -1);
  pack_weight(c.cols, c.dim, p, w, kap2);
}

// ---------------------------------------------------------------------------
// Certificate reductions (float64).  Partial sums per block, then one block
// adds the partials in a fixed order (deterministic).
// slots: 0 sum r log A, 1 sum c (log B - log c), 2 sum |s - c|, 3 sum s mu,
//        4 sum s, 5 non-finite count
// ---------------------------------------------------------------------------
__device__ void block_reduce_store(double* vals, int nv, double* dst) {
  __shared__ double red[kBlock / kTile][8];
  const int lane = threadIdx.x & (kTile - 1), wid = threadIdx.x / kTile;
  for (int i = 0; i < nv; ++i) {
    const double v = wave_sum(vals[i]);
    if (lane == 0) red[wid][i] = v;
  }
  __syncthreads();
  if (threadIdx.x < nv) {
    double s = 0.0;
    for (int w = 0; w < kBlock / kTile; ++w) s += red[w][threadIdx.x];
    dst[threadIdx.x] = s;
  }
}

__device__ __forceinline__ void cert_partial_block(const LaunchCtx& c, int bx, int nb) {
  double v[6] = {0, 0, 0, 0, 0, 0};
  const int stride = nb * kBlock;
  const bool debiased = (c.ctrl->variant & kVarDebiased) != 0;
  for (int p = bx * kBlock + threadIdx.x; p < c.rows.count; p += stride) {
    // f = eps log A with A the row scaling the column update read (Prop. 3)
    const double lah = debiased ? c.st.la[p] : c.st.lah[p];
    if (!isfinite(lah)) v[5] += 1.0;
    v[0] += c.rows.marg[p] * lah;
  }
  for (int p = bx * kBlock + threadIdx.x; p < c.cols.count; p += stride) {
    const double lbh = c.st.lbh[p];
    const double cj = c.cols.marg[p];
    const double s = exp(c.st.logs[p]);
    const double mu = c.st.mu[p];
    if (!isfinite(lbh) || !isfinite(s) || !isfinite(mu)) v[5] += 1.0;
    v[1] += cj * (lbh - c.cols.logmarg[p]);
    v[2] += fabs(s - cj);
    v[3] += s * mu;
    v[4] += s;
  }
  block_reduce_store(v, 6, c.cert_part + (size_t)bx * 8);
}

__global__ __launch_bounds__(kBlock) void k_cert_partial(LaunchCtx c) { cert_partial_block(c, blockIdx.x, gridDim.x); }

__global__ __launch_bounds__(kBlock) void k_cert_partial_batch(const BatchItem* __restrict__ items,
                                                               const LaunchCtx* __restrict__ descs) {
  const BatchItem it = items[blockIdx.x];
  cert_partial_block(descs[it.prob], it.blk, descs[it.prob].cert_blocks);
}

__device__ __forceinline__ void cert_final_block(const LaunchCtx& c) {
  double v[6] = {0, 0, 0, 0, 0, 0};
  for (int b = threadIdx.x; b < c.cert_blocks; b += kBlock)
    for (int i = 0; i < 6; ++i) v[i] += c.cert_part[(size_t)b * 8 + i];
  __shared__ double tot[8];
  block_reduce_store(v, 6, tot);
  __syncthreads();
  if (threadIdx.x == 0) {
    const long long k = c.ctrl->k - 1;  // the iteration just certified
    const double eps = c.ctrl->eta / (c.ctrl->lam * (double)k + 1.0);
    const double L = eps * (tot[0] + tot[1]);                 // <r, f> + <c, g>
    const double delta = 0.5 * tot[2];                        // 1/2 ||s - c||_1
    const double costZ = tot[3];                              // sum_j s_j mu_j
    const double U = costZ + c.ctrl->omega * delta;           // Algorithm 2
    double* o = c.cert_out;
    o[0] = (double)k;
    o[1] = eps;
    o[2] = L;
    o[3] = U;
    o[4] = delta;
    o[5] = costZ;
    o[6] = tot[4];
    o[7] = tot[5];
  }
}

__global__ __launch_bounds__(kBlock) void k_cert_final(LaunchCtx c) { cert_final_block(c); }

// one block per listed problem; also copies the record into a contiguous array
__global__ __launch_bounds__(kBlock) void k_cert_final_batch(const int* __restrict__ probs,
                                                             const LaunchCtx* __restrict__ descs,
                                                             double* __restrict__ records) {
  const LaunchCtx& c = descs[probs[blockIdx.x]];
  cert_final_block(c);
  __syncthreads();
  if (threadIdx.x < kCertSlots) {
    __threadfence_block();
    records[(size_t)blockIdx.x * kCertSlots + threadIdx.x] = c.cert_out[threadIdx.x];
  }
}

// repair: sum p, sum q, sum p|x|^2, sum q|y|^2, sum p x (3), sum q y (3), sum e s mu
__global__ __launch_bounds__(kBlock) void k_repair_partial(LaunchCtx c) {
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int stride = gridDim.x * kBlock;
  const int dim = c.dim;
  for (int p = blockIdx.x * kBlock + threadIdx.x; p < c.rows.count; p += stride) {
    const double pv = c.st.pvec[p];
    double n2 = 0.0;
    for (int d = 0; d < dim; ++d) {
      const double xd = c.rows.abs[(size_t)d * c.rows.np + p];
      n2 += xd * xd;
      v[3 + d] += pv * xd;
    }
    v[0] += pv;
    v[2] += pv * n2;
  }
  block_reduce_store(v, 6, c.cert_part + (size_t)blockIdx.x * 8);
  __syncthreads();
  double w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int p = blockIdx.x * kBlock + threadIdx.x; p < c.cols.count; p += stride) {
    const double s = exp(c.st.logs[p]);
    const double cj = c.cols.marg[p];
    const double q = cj > s ? cj - s : 0.0;
    const double e = cj < s ? cj / s : 1.0;
    double n2 = 0.0;
    for (int d = 0; d < dim; ++d) {
      const double yd = c.cols.abs[(size_t)d * c.cols.np + p];
      n2 += yd * yd;
      w[3 + d] += q * yd;
    }
    w[0] += q;
    w[1] += e * s * c.st.mu[p];
    w[2] += q * n2;
  }
  block_reduce_store(w, 6, c.cert_part + ((size_t)gridDim.x + blockIdx.x) * 8);
}

__global__ __launch_bounds__(kBlock) void k_repair_final(LaunchCtx c) {
  // partial layout: [0, G) row sums, [G, 2G) column sums
  double v[6] = {0, 0, 0, 0, 0, 0}, w[6] = {0, 0, 0, 0, 0, 0};
  const int G = c.cert_blocks;
  for (int b = threadIdx.x; b < G; b += kBlock)
    for (int i = 0; i < 6; ++i) {
      v[i] += c.cert_part[(size_t)b * 8 + i];
      w[i] += c.cert_part[(size_t)(G + b) * 8 + i];
    }
  __shared__ double tv[8], tw[8];
  block_reduce_store(v, 6, tv);
  __syncthreads();
  block_reduce_store(w, 6, tw);
  __syncthreads();
  if (threadIdx.x == 0) {
    // p^T C q = s [ (sum q)(sum p|x|^2) + (sum p)(sum q|y|^2) - 2 (sum p x).(sum q y) ]
    double cross = 0.0;
    for (int d = 0; d < c.dim; ++d) cross += tv[3 + d] * tw[3 + d];
    const double pCq = c.ctrl->scale * (tw[0] * tv[2] + tv[0] * tw[2] - 2.0 * cross);
    const double delta = c.cert_out[4];
    const double costClip = tw[1];                        // sum_j e_j s_j mu_j
    double* o = c.cert_out;
    o[8] = costClip + (delta > 0.0 ? pCq / delta : 0.0);   // <C, Z^>
    o[9] = tv[0];                                         // 1^T p
    o[10] = tw[0];                                        // 1^T q
    o[11] = pCq;
  }
}

// Rounded cost: sum_i cost_i + e_r^T C e_c / ||e_r||_1 with the squared
// Euclidean closed form e_r^T C e_c = s [ (sum e_c)(sum e_r |x|^2) +
// (sum e_r)(sum e_c |y|^2) - 2 (sum e_r x).(sum e_c y) ].  Row deficits in
// plan_aux, row costs in pvec, column deficits in mu (kFinishRound3 / 2).
__global__ __launch_bounds__(kBlock) void k_round_partial(LaunchCtx c) {
  double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int stride = gridDim.x * kBlock;
  const int dim = c.dim;
  for (int p = blockIdx.x * kBlock + threadIdx.x; p < c.rows.count; p += stride) {
    const double er = c.plan_aux[p];
    double n2 = 0.0;
    for (int d = 0; d < dim; ++d) {
      const double xd = c.rows.abs[(size_t)d * c.rows.np + p];
      n2 += xd * xd;
      v[3 + d] += er * xd;
    }
    v[0] += er;
    v[1] += c.st.pvec[p];
    v[2] += er * n2;
  }
  block_reduce_store(v, 6, c.cert_part + (size_t)blockIdx.x * 8);
  __syncthreads();
  double w[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int p = blockIdx.x * kBlock + threadIdx.x; p < c.cols.count; p += stride) {
    const double ec = c.st.mu[p];
    double n2 = 0.0;
    for (int d = 0; d < dim; ++d) {
      const double yd = c.cols.abs[(size_t)d * c.cols.np + p];
      n2 += yd * yd;
      w[3 + d] += ec * yd;
    }
    w[0] += ec;
    w[2] += ec * n2;
  }
  block_reduce_store(w, 6, c.cert_part + ((size_t)gridDim.x + blockIdx.x) * 8);
}

__global__ __launch_bounds__(kBlock) void k_round_final(LaunchCtx c) {
  double v[6] = {0, 0, 0, 0, 0, 0}, w[6] = {0, 0, 0, 0, 0, 0};
  const int G = c.cert_blocks;
  for (int b = threadIdx.x; b < G; b += kBlock)
    for (int i = 0; i < 6; ++i) {
      v[i] += c.cert_part[(size_t)b * 8 + i];
      w[i] += c.cert_part[(size_t)(G + b) * 8 + i];
    }
  __shared__ double tv[8], tw[8];
  block_reduce_store(v, 6, tv);
  __syncthreads();
  block_reduce_store(w, 6, tw);
  __syncthreads();
  if (threadIdx.x == 0) {
    double dot = 0.0;
    for (int d = 0; d < c.dim; ++d) dot += tv[3 + d] * tw[3 + d];
    const double erCec = c.ctrl->scale * (tw[0] * tv[2] + tv[0] * tw[2] - 2.0 * dot);
    const double mass = tv[0];
    double* o = c.plan_stats;
    o[8] = tv[1] + (mass > 0.0 ? erCec / mass : 0.0);   // <C, G>
    o[9] = tv[1];                                       // <C, X''>
    o[10] = mass;                                       // ||e_r||_1
    o[11] = tw[0];                                      // ||e_c||_1 (equals ||e_r||_1)
  }
}

// Adds the per-wavefront tile counts of one sweep to the running total (one
// block, fixed order: profiling only).
__global__ __launch_bounds__(kBlock) void k_count_tiles(const unsigned* __restrict__ count, int n,
                                                        unsigned long long* __restrict__ total) {
  __shared__ unsigned long long part[kBlock];
  unsigned long long v = 0;
  for (int i = threadIdx.x; i < n; i += kBlock) v += count[i];
  part[threadIdx.x] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long tsum = 0;
    for (int i = 0; i < kBlock; ++i) tsum += part[i];
    *total += tsum;
  }
}

// Up to kStateVecs vectors between tile order and the caller's order in one
// launch (a state is six of them, and a launch costs more than a vector):
// out: dst[perm[p]] = src[p]; in: dst[p] = src[perm[p]] over the padded length.
__global__ void k_scatter(StateVecs v) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
#pragma unroll
  for (int i = 0; i < kStateVecs; ++i)
    if (v.dst[i] && p < v.len[i]) v.dst[i][v.perm[i][p]] = v.src[i][p];
}

__global__ void k_gather(StateVecs v) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
#pragma unroll
  for (int i = 0; i < kStateVecs; ++i)
    if (v.src[i] && p < v.len[i]) v.dst[i][p] = v.src[i][v.perm[i][p]];
}

// Hints to the caller's order (dst[perm_out[p]] = perm_in[hint[p]]) and back,
// both sides in one launch (a null pointer skips one).
__global__ void k_hints_out(SideDev rows, SideDev cols, int* __restrict__ row_hint, int* __restrict__ col_hint) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (row_hint && p < rows.count) row_hint[rows.perm[p]] = rows.hint[p] >= 0 ? cols.perm[rows.hint[p]] : -1;
  if (col_hint && p < cols.count) col_hint[cols.perm[p]] = cols.hint[p] >= 0 ? rows.perm[cols.hint[p]] : -1;
}

__global__ void k_hints_in(SideDev rows, SideDev cols, const int* __restrict__ row_hint,
                           const int* __restrict__ col_hint) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (row_hint && p < rows.np) {
    const int j = row_hint[rows.perm[p]];
    rows.hint[p] = (j >= 0 && j < cols.count) ? cols.iperm[j] : -1;
  }
  if (col_hint && p < cols.np) {
    const int j = col_hint[cols.perm[p]];
    cols.hint[p] = (j >= 0 && j < rows.count) ? rows.iperm[j] : -1;
  }
}

// Factors of a feasible plan X_ij = exp(u_i + v_j - C_ij / eps) + a_i b_j, in
// original order.  Rounded state plan (Altschuler, Weed and Rigollet 2017,
// Algorithm 2): u = log alpha + log x, v = log beta + log y, a = e_r,
// b = e_c / ||e_r||_1.  Repaired intermediate plan (proof of Prop. 3):
// u = log alpha-hat, v = log t + log e with e_j = min(1, c_j / s_j), a = p,
// b = (c - s)_+ / delta.  lt_prev: log t of the last row update (repair only).
__global__ void k_export_factors(LaunchCtx c, int repaired, const double* __restrict__ lt_prev,
                                 double* __restrict__ u, double* __restrict__ v, double* __restrict__ a,
                                 double* __restrict__ b) {
  const int p = blockIdx.x * kBlock + threadIdx.x;
  if (p < c.rows.count) {
    const int i = c.rows.perm[p];
    if (u) u[i] = repaired ? c.st.lah[p] : c.st.la[p] + c.plan_row[p];
    if (a) a[i] = repaired ? c.st.pvec[p] : c.plan_aux[p];
  }
  if (p < c.cols.count) {
    const int j = c.cols.perm[p];
    if (repaired) {
      const double ls = c.st.logs[p];
      const double delta = c.cert_out[4];
      if (v) v[j] = lt_prev[p] + fmin(0.0, c.cols.logmarg[p] - ls);
      if (b) b[j] = delta > 0.0 ? fmax(c.cols.marg[p] - exp(ls), 0.0) / delta : 0.0;
    } else {
      const double mass = c.plan_stats[10];
      if (v) v[j] = c.st.lb1[p] + c.plan_col[p];
      if (b) b[j] = mass > 0.0 ? c.st.mu[p] / mass : 0.0;
    }
  }
}

// Dense rows [row_begin, row_begin + nrows) of a factored plan, row-major in
// original order: out[(i - row_begin) n + j] = exp(u_i + v_j - kap |x_i - y_j|^2)
// (+ a_i b_j when R1), in float64 from the stored float32 coordinates.
// Bound: writes, 8 bytes per entry (the float64 exponentials need less: a
// shorter polynomial for them changed nothing), so every line is written whole:
// a row's columns are split where its memory crosses 128 bytes, not at multiples
// of kBlock, and a strip holds rows of one alignment (every period-th row;
// lead is what the first block of such rows has before the row begins).
// A thread holds y_j, v_j and b_j of its column; the first wavefront loads the
// strip's slots, coordinates and factors (one lane per row) into LDS, and every
// thread reads them from there for each row.  Consecutive blocks are neighbours
// along a row, so that the blocks in flight fill whole rows; strips of 32 rows
// leave many blocks to balance; the stores bypass the caches.
// With the call, 4096 rows of 16384 entries (537 MB; a fill takes 81 us, launch
// and wait about 20): 132 -> 110 us; of 16383 entries, which begin anywhere in a
// line: 151 -> 113 us; 3001 rows of 2477: 33.4 -> 32.8 us.  Rows split at multiples
// of kBlock instead: 182 us at 16383 entries (154 us through the caches); strips
// of 64 / 48 / 24 rows at 16384: 12 us more / the same / the same; two columns
// per thread: 3 us more.
constexpr int kEntryRows = 32;
constexpr int kLineDoubles = 16;  // 128 bytes
template <int D, bool R1>
__global__ __launch_bounds__(kBlock) void k_plan_entries(LaunchCtx c, const double* __restrict__ u,
                                                         const double* __restrict__ v,
                                                         const double* __restrict__ a,
                                                         const double* __restrict__ b, double kap,
                                                         long long row_begin, long long nrows, int skew,
                                                         int period, long long strips,
                                                         double* __restrict__ out) {
  __shared__ float sx[D][kEntryRows];
  __shared__ double su[kEntryRows], sa[kEntryRows];
  const int n = c.cols.count;
  for (long long sb = blockIdx.y; sb < strips; sb += gridDim.y) {
    const int phase = (int)(sb & (period - 1));
    const long long r0 = (sb - phase) * kEntryRows + phase;  // rows r0, r0 + period, ...
    if (r0 >= nrows) continue;                               // the whole block
    const int rows = (int)min((long long)kEntryRows, (nrows - r0 + period - 1) / period);
    const int lead = (int)((skew + r0 * n) & (kLineDoubles - 1));
    const long long jj = (long long)blockIdx.x * kBlock + threadIdx.x - lead;
    const bool col = jj >= 0 && jj < n;  // no early return: every thread reaches the barriers
    const int j = col ? (int)jj : 0;
    const int qj = c.cols.iperm[j];
    double y[D];
#pragma unroll
    for (int d = 0; d < D; ++d) y[d] = (double)c.cols.abs[(size_t)d * c.cols.np + qj];
    const double vj = v[j], bj = R1 ? b[j] : 0.0;
    __syncthreads();  // the previous strip's rows have been read
    if ((int)threadIdx.x < rows) {
      const long long i = row_begin + r0 + (long long)threadIdx.x * period;
      const int q = c.rows.iperm[i];
#pragma unroll
      for (int d = 0; d < D; ++d) sx[d][threadIdx.x] = c.rows.abs[(size_t)d * c.rows.np + q];
      su[threadIdx.x] = u[i];
      sa[threadIdx.x] = R1 ? a[i] : 0.0;
    }
    __syncthreads();
    if (!col) continue;
    double* o = out + (size_t)r0 * n + j;
    for (int t = 0; t < rows; ++t, o += (size_t)period * n) {
      double d2 = 0.0;
#pragma unroll
      for (int d = 0; d < D; ++d) {
        const double e = (double)sx[d][t] - y[d];
        d2 = fma(e, e, d2);
      }
      __builtin_nontemporal_store(exp(su[t] + vj - kap * d2) + sa[t] * bj, o);
    }
  }
}

}  // namespace

// Runs f with the dimension (1, 2, 3) as a constant.
template <typename F>
hipError_t by_dim(int dim, F f) {
  switch (dim) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_sweep_batch(const BatchItem* items, int nitems, const LaunchCtx* descs, int dim,
                              bool transpose, bool cert, int kofs, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  return by_dim(dim, [&](auto d) {
    constexpr int D = decltype(d)::value;
    auto* k = transpose ? (cert ? k_sweep_batch<D, kSweepCert, false> : k_sweep_batch<D, kSweepPlain, false>)
                        : (cert ? k_sweep_batch<D, kSweepCert, true> : k_sweep_batch<D, kSweepPlain, true>);
    hipLaunchKernelGGL(k, dim3(nitems), dim3(kSweepBlock), 0, s, items, descs, kofs);
  });
}

hipError_t launch_finish_batch(const BatchItem* items, int nitems, const LaunchCtx* descs, int dim, FinishKind kind,
                               int kofs, hipStream_t s) {
  if (nitems <= 0) return hipSuccess;
  return by_dim(dim, [&](auto d) {
    constexpr int D = decltype(d)::value;
    auto* k = kind == kFinishRow   ? k_finish_batch<D, kFinishRow, true>
              : kind == kFinishCol ? k_finish_batch<D, kFinishCol, false>
                                   : k_finish_batch<D, kFinishColCert, false>;
    hipLaunchKernelGGL(k, dim3(nitems), dim3(kTile), 0, s, items, descs, kofs);
  });
}

hipError_t launch_advance(Ctrl* ctrl, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(kTile), 0, s, ctrl, n);
  return hipGetLastError();
}

hipError_t launch_advance_batch(const LaunchCtx* descs, int count, int n, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_advance_batch, dim3((count + kBlock - 1) / kBlock), dim3(kBlock), 0, s, descs, count, n);
  return hipGetLastError();
}

hipError_t launch_cert_batch(const BatchItem* items, int nitems, const int* probs, int nprobs,
                             const LaunchCtx* descs, double* records, hipStream_t s) {
  if (nitems <= 0 || nprobs <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_cert_partial_batch, dim3(nitems), dim3(kBlock), 0, s, items, descs);
  hipLaunchKernelGGL(k_cert_final_batch, dim3(nprobs), dim3(kBlock), 0, s, probs, descs, records);
  return hipGetLastError();
}

int choose_splits(int np_out, int ntiles_in) {
  // enough (output wave, split) pairs to give every SIMD of the 256 CUs many
  // waves (skipped tiles make the work per pair uneven, so finer pairs balance
  // better), but at least 4 tiles per split so the per-split set-up stays
  // small; the partial records stay below target * 64 records plus one per
  // output
  const int out_waves = (np_out + kTile - 1) / kTile;
  int s = (BDRS_TARGET_WAVES + out_waves - 1) / out_waves;
  const int max_s = (ntiles_in + 3) / 4;
  if (s > max_s) s = max_s;
  if (s < 1) s = 1;
  const int tps = (ntiles_in + s - 1) / s;
  return (ntiles_in + tps - 1) / tps;  // splits that own at least one tile
}

static hipError_t launch_sweep_mode(const LaunchCtx& c, bool transpose, SweepMode mode, int splits, double eps_arg,
                                    int kofs) {
  const SideDev& out = transpose ? c.cols : c.rows;
  const dim3 grid(splits, out.np / kSweepBlock), block(kSweepBlock);  // x: split, y: output block (see k_sweep)
  const int own = eps_arg > 0.0 ? 1 : 0;
  return by_dim(c.dim, [&](auto d) {
    constexpr int D = decltype(d)::value;
    auto* k = mode == kSweepBary ? k_sweep<D, kSweepBary, true>
              : transpose ? (mode == kSweepCert ? k_sweep<D, kSweepCert, false> : k_sweep<D, kSweepPlain, false>)
                          : (mode == kSweepCert ? k_sweep<D, kSweepCert, true> : k_sweep<D, kSweepPlain, true>);
    if (c.ev_start && c.ev_stop)
      hipExtLaunchKernelGGL(k, grid, block, 0, c.stream, c.ev_start, c.ev_stop, 0u, c, splits, eps_arg, own, kofs);
    else
      hipLaunchKernelGGL(k, grid, block, 0, c.stream, c, splits, eps_arg, own, kofs);
  });
}

hipError_t launch_sweep(const LaunchCtx& c, bool transpose, bool cert, int splits, double eps_arg, int kofs) {
  return launch_sweep_mode(c, transpose, cert ? kSweepCert : kSweepPlain, splits, eps_arg, kofs);
}

hipError_t launch_sweep_bary(const LaunchCtx& c, int splits, double eps) {
  return launch_sweep_mode(c, false, kSweepBary, splits, eps, 0);
}

hipError_t launch_finish(const LaunchCtx& c, bool transpose, FinishKind kind, int splits, double* lse_out,
                         int kofs) {
  // one wavefront per block (one tile of outputs), so the O(n) epilogue spreads over all CUs
  const dim3 grid((transpose ? c.cols : c.rows).ntiles), block(kTile);
  // (the kinds that do not pack weights are the same for every dimension)
  const bool any_dim = !finish_iterates(kind) && kind != kFinishPlanRow;
  return by_dim(any_dim ? 1 : c.dim, [&](auto d) {
    constexpr int D = decltype(d)::value;
    void (*k)(LaunchCtx, int, double*, int) = nullptr;
    switch (kind) {
      case kFinishRow: k = k_finish<D, kFinishRow, true>; break;
      case kFinishCol: k = k_finish<D, kFinishCol, false>; break;
      case kFinishColCert: k = k_finish<D, kFinishColCert, false>; break;
      case kFinishPlanRow: k = k_finish<D, kFinishPlanRow, true>; break;
      case kFinishLse: k = transpose ? k_finish<1, kFinishLse, false> : k_finish<1, kFinishLse, true>; break;
      case kFinishRepair: k = k_finish<1, kFinishRepair, true>; break;
      case kFinishCertOnly: k = k_finish<1, kFinishCertOnly, false>; break;
      case kFinishPlanCol: k = k_finish<1, kFinishPlanCol, false>; break;
      case kFinishRound1: k = k_finish<1, kFinishRound1, true>; break;
      case kFinishRound2: k = k_finish<1, kFinishRound2, false>; break;
      case kFinishRound3: k = k_finish<1, kFinishRound3, true>; break;
    }
    hipLaunchKernelGGL(k, grid, block, 0, c.stream, c, splits, lse_out, kofs);
  });
}

hipError_t launch_prologue(const LaunchCtx& c) {
  hipLaunchKernelGGL(k_prologue, dim3(c.cols.np / kBlock), dim3(kBlock), 0, c.stream, c);
  return hipGetLastError();
}

hipError_t launch_pack(const LaunchCtx& c, bool transpose, const double* w, double eps) {
  const SideDev& in = transpose ? c.rows : c.cols;
  hipLaunchKernelGGL(k_pack, dim3(in.np / kBlock), dim3(kBlock), 0, c.stream, c, transpose ? 1 : 0, w, eps);
  return hipGetLastError();
}

hipError_t launch_repack(const LaunchCtx& c) {
  const int cols = c.cols.np / kBlock;
  hipLaunchKernelGGL(k_repack, dim3(cols + c.rows.np / kBlock), dim3(kBlock), 0, c.stream, c, cols);
  return hipGetLastError();
}

hipError_t launch_count_tiles(const LaunchCtx& c, int n) {
  if (!c.tile_count || !c.tile_total || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_count_tiles, dim3(1), dim3(kBlock), 0, c.stream, c.tile_count, n, c.tile_total);
  return hipGetLastError();
}

hipError_t launch_pack_state(const LaunchCtx& c, bool transpose, double eps, bool with_factors) {
  const SideDev& in = transpose ? c.rows : c.cols;
  hipLaunchKernelGGL(k_pack_state, dim3(in.np / kBlock), dim3(kBlock), 0, c.stream, c, transpose ? 1 : 0, eps,
                     with_factors ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_round_reduce(const LaunchCtx& c) {
  // two sets of cert_blocks x 8 partials: the certificate's buffer holds both
  hipLaunchKernelGGL(k_round_partial, dim3(c.cert_blocks), dim3(kBlock), 0, c.stream, c);
  hipLaunchKernelGGL(k_round_final, dim3(1), dim3(kBlock), 0, c.stream, c);
  return hipGetLastError();
}

hipError_t launch_plan_stats(const LaunchCtx& c) {
  // the certificate's partial buffer holds cert_blocks x 8 doubles
  hipLaunchKernelGGL(k_plan_partial, dim3(c.cert_blocks), dim3(kBlock), 0, c.stream, c);
  hipLaunchKernelGGL(k_plan_final, dim3(1), dim3(kBlock), 0, c.stream, c, c.cert_blocks);
  return hipGetLastError();
}

hipError_t launch_cert_reduce(const LaunchCtx& c) {
  hipLaunchKernelGGL(k_cert_partial, dim3(c.cert_blocks), dim3(kBlock), 0, c.stream, c);
  hipLaunchKernelGGL(k_cert_final, dim3(1), dim3(kBlock), 0, c.stream, c);
  return hipGetLastError();
}

hipError_t launch_repair_pack(const LaunchCtx& c) {
  hipLaunchKernelGGL(k_repair_pack, dim3(c.cols.np / kBlock), dim3(kBlock), 0, c.stream, c);
  return hipGetLastError();
}

hipError_t launch_repair_reduce(const LaunchCtx& c) {
  hipLaunchKernelGGL(k_repair_partial, dim3(c.cert_blocks), dim3(kBlock), 0, c.stream, c);
  hipLaunchKernelGGL(k_repair_final, dim3(1), dim3(kBlock), 0, c.stream, c);
  return hipGetLastError();
}

hipError_t launch_export_factors(const LaunchCtx& c, bool repaired, const double* lt_prev, double* u, double* v,
                                 double* a, double* b) {
  const int cnt = std::max(c.rows.count, c.cols.count);
  if (cnt <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_export_factors, dim3((cnt + kBlock - 1) / kBlock), dim3(kBlock), 0, c.stream, c,
                     repaired ? 1 : 0, lt_prev, u, v, a, b);
  return hipGetLastError();
}

hipError_t launch_plan_entries(const LaunchCtx& c, const double* u, const double* v, const double* a,
                               const double* b, double kap, long long row_begin, long long nrows, double* out) {
  if (nrows <= 0 || c.cols.count <= 0) return hipSuccess;
  // rows period apart start at the same place in a line
  int period = kLineDoubles;
  while (period > 1 && (long long)c.cols.count * (period / 2) % kLineDoubles == 0) period /= 2;
  const long long per_group = (long long)period * kEntryRows;
  const long long strips = (nrows + per_group - 1) / per_group * period;
  const int skew = (int)((uintptr_t)out / sizeof(double) % kLineDoubles);
  const long long width = (long long)c.cols.count + (period > 1 || skew ? kLineDoubles - 1 : 0);
  const dim3 grid((unsigned)((width + kBlock - 1) / kBlock), (unsigned)std::min(strips, 65535LL));
  const bool r1 = a != nullptr && b != nullptr;
  return by_dim(c.dim, [&](auto d) {
    constexpr int D = decltype(d)::value;
    auto* k = r1 ? k_plan_entries<D, true> : k_plan_entries<D, false>;
    hipLaunchKernelGGL(k, grid, dim3(kBlock), 0, c.stream, c, u, v, a, b, kap, row_begin, nrows, skew, period,
                       strips, out);
  });
}

static int longest(const StateVecs& v) {
  int n = 0;
  for (int i = 0; i < kStateVecs; ++i)
    if (v.src[i] && v.dst[i]) n = std::max(n, v.len[i]);
  return n;
}

hipError_t launch_scatter(const StateVecs& v, hipStream_t s) {
  const int n = longest(v);
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_scatter, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, v);
  return hipGetLastError();
}

hipError_t launch_gather(const StateVecs& v, hipStream_t s) {
  const int n = longest(v);
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, s, v);
  return hipGetLastError();
}

hipError_t launch_hints_out(const LaunchCtx& c, int* row_hint, int* col_hint) {
  if (!row_hint && !col_hint) return hipSuccess;
  const int n = std::max(c.rows.count, c.cols.count);
  hipLaunchKernelGGL(k_hints_out, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, c.stream, c.rows, c.cols,
                     row_hint, col_hint);
  return hipGetLastError();
}

hipError_t launch_hints_in(const LaunchCtx& c, const int* row_hint, const int* col_hint) {
  if (!row_hint && !col_hint) return hipSuccess;
  const int n = std::max(c.rows.np, c.cols.np);
  hipLaunchKernelGGL(k_hints_in, dim3((n + kBlock - 1) / kBlock), dim3(kBlock), 0, c.stream, c.rows, c.cols,
                     row_hint, col_hint);
  return hipGetLastError();
}

}  // namespace bdrs
