// Cutoff pair kernels.
//
//  * excluded volume: eq. u_ex for every pair within rc (all beads);
//  * real-space electrostatics: the bracket of eq. ewald,
//    lB z_i z_j [erf(alpha_ij r) - erf(beta r)]/r, over the charged beads only
//    (their own cell list and compacted arrays), so the transcendental-heavy
//    term costs nothing for neutral beads and the kernels never branch on
//    charge.
//
// Both work on "clusters": CI consecutive beads of the cell-sorted order
// (CI = 2, 4 or 8; spatially compact because the order is by cell), one
// wavefront per cluster, either with a neighbour list in HBM (two launches)
// or list-free (one launch, k_pair_fused):
//
//  1. k_nl_build: one wavefront per cluster.  The lanes enumerate the cell
//     columns within reach of the cluster's bounding box (culled by the exact
//     box-to-column distance, z runs clipped to the cutoff sphere), expand the
//     runs into an LDS candidate buffer, and test each candidate against every
//     bead of the cluster with the exact minimum-image distance.  A candidate
//     within rc of at least one cluster bead is appended (ballot compaction,
//     candidate order) to the cluster's list: the list is the union of the
//     beads' cutoff spheres, not a bounding-box shell.
//  2. k_nl_force: one wavefront per cluster, lanes laid out as
//     CI cluster beads x (64/CI) list entries.  Every lane evaluates its
//     (bead, entry) pair, masked by the exact cutoff test, so the hot loop has
//     no per-lane walk and no divergence beyond the mask.  Each pair is seen
//     from both ends (no scatter of forces to j); the partial forces of a bead
//     are combined with xor shuffles in a fixed order and added once to the
//     64-bit fixed-point accumulator.
//
//  k_pair_fused does both in one pass: the candidates that pass the list
//  test go to a small LDS ring instead of HBM, and every 64 of them are
//  evaluated at once with the force pass's lane layout.
//
// Lists are rebuilt every evaluation, so they need no skin.  The minimum
// image is the wrapped 32-bit difference of the fractional fixed-point
// coordinates (valid because rc <= L/2 is enforced).
//
// This header holds the device code; each pair_*.hip file compiles one part of
// it (pair type and precision), so that the parts build side by side.
#pragma once

#include <type_traits>
#include <utility>

#include "gcme_internal.h"

namespace gcme {

namespace {

// hardware 2^x (1 ulp; results below the smallest normal flush to zero,
// far below anything the single-precision sums resolve)
__device__ inline float gexp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ inline double gexp2(double x) { return exp2(x); }
__device__ inline float gexp(float x) { return expf(x); }
__device__ inline double gexp(double x) { return exp(x); }
__device__ inline float gerfc(float x) { return erfcf(x); }
__device__ inline double gerfc(double x) { return erfc(x); }
__device__ inline float gsqrt(float x) { return sqrtf(x); }
__device__ inline double gsqrt(double x) { return sqrt(x); }

// erfc(x) e^(x^2), x >= 0, in single precision by the rational
// approximation of Abramowitz and Stegun (Handbook of Mathematical
// Functions, 7.1.26): with t = 1/(1 + p x), erfc(x) = (a1 t + a2 t^2 +
// a3 t^3 + a4 t^4 + a5 t^5) e^(-x^2), absolute error at most 1.5e-7.  The
// factor e^(-x^2) is left to the caller, who needs it for the force too.
__device__ inline float erfc_scaled(float x) {
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
  return t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f),
                  0.254829592f);
}

template <typename T>
struct Series;
template <>
struct Series<float> {
  static constexpr int n = 8;
};
template <>
struct Series<double> {
  static constexpr int n = NSER;
};

constexpr int NL_WAVES = 4;    // wavefronts (clusters) per workgroup
constexpr int NL_CAND = 1024;  // LDS candidate buffer per wavefront
constexpr int NL_SEG = 128;    // LDS segment list per wavefront (two per column)

// DPP lane moves (within rows of 16 lanes, all sources valid).
template <int CTRL>
__device__ inline int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ inline float dpp_f(float v) {
  return __int_as_float(dpp_i<CTRL>(__float_as_int(v)));
}
template <int CTRL>
__device__ inline double dpp_f(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = dpp_i<CTRL>((int)b), hi = dpp_i<CTRL>((int)(b >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int DPP_ROW_ROR8 = 0x128, DPP_ROW_HALF_MIRROR = 0x141, DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E;

// Inclusive scan over the wavefront: shifts within rows of 16 lanes (lanes
// shifted in read 0), then the rows' totals broadcast into the rows after
// them -- six adds, where shuffles would take an LDS round trip each.
__device__ inline int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return v;
}

// Number of set bits of m below this lane.
__device__ inline int lanes_below(unsigned long long m) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__device__ inline uint32_t read_lane(uint32_t v, int l) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); }

// A wave-uniform float kept in a scalar register (the VALU reads it as an
// operand, so it costs no vector register).
__device__ inline float uni(float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); }

// Fixed-order sum over the block (NL_WAVES waves); result valid in thread 0.
__device__ inline double block_sum(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0) {
    for (int w = 0; w < NL_WAVES; ++w) t += sh[w];
  }
  return t;
}

__device__ inline long long to_fixed(double f, double scale, unsigned int* status) {
  double v = f * scale;
  if (!(fabs(v) < 4.0e18)) {
    atomicOr(status, (unsigned)STATUS_FORCE_OVERFLOW);
    return 0;
  }
  return (long long)llrint(v);
}

// ---------------------------------------------------------------------------
// Candidate enumeration, shared by the list build and the list-free kernel
// ---------------------------------------------------------------------------

// A cluster's geometry as wave-uniform values.  Positions are taken relative
// to the centre of the bounding box of its beads: the frame's floats are then
// as small as they can be, and with them the rounding of the separation of
// close pairs, and each is rounded once, from double (forces of the adsorption
// study's slab, whose electrode beads are stiff: 2.5e-7 off; 3.6e-7 with the
// conversion in single precision, 5.2e-7 with bead 0 for the origin; 1% of
// the kernel's time).  Cell ranges are in float relative to
// the lower corner of the centre's cell: every value is a few cells at most,
// so float carries it to ~1e-7 of a cell, and the margin in rclm keeps each
// range conservative.
struct ClusterBox {
  uint32_t u0[3];      // the centre, fixed point
  float lo[3], hi[3];  // bounding box relative to the centre
  int c0[3];           // cell of the centre
  float p0[3];         // the centre within its cell
  bool compact;        // every bead within 3 rcl of the centre
  float rcl;           // list cutoff, a hair above rc
  float rclm;          // enumeration radius: rcl plus a margin
  int clo[3], chi[3];  // cell ranges relative to c0 (absolute when whole)
  bool whole[3];       // the range spans the whole axis
};

// Smallest (largest) value over each group of CI consecutive lanes, in all of
// its lanes.
template <int CI, class Op>
__device__ inline int group_reduce(int v, Op op) {
  v = op(v, dpp_i<DPP_XOR1>(v));
  if (CI >= 4) v = op(v, dpp_i<DPP_XOR2>(v));
  if (CI >= 8) v = op(v, dpp_i<DPP_ROW_HALF_MIRROR>(v));
  return v;
}

// Sum over each group of W consecutive lanes (8 to 32), in a fixed order, in
// all of its lanes.
template <int W, typename T>
__device__ inline T group_sum(T v) {
  v += dpp_f<DPP_XOR1>(v);
  v += dpp_f<DPP_XOR2>(v);
  v += dpp_f<DPP_ROW_HALF_MIRROR>(v);
  if (W >= 16) v += dpp_f<DPP_ROW_ROR8>(v);
  if (W >= 32) v += __shfl_xor(v, 16, 64);
  return v;
}

// The geometry from the cluster's bead records, one bead per lane: lane l
// holds bead l % CI (slots beyond the cluster's beads repeat bead 0), so the
// bounding box is three lane exchanges per bound.  Receives the lane's bead
// relative to the centre (r) and its squared distance from it (nn).
template <int CI>
__device__ inline void make_box(ClusterBox& K, const uint4 me, const RepDesc& R, float r[3], float& nn) {
  const uint32_t u[3] = {me.x, me.y, me.z};
  // (the bounds as integers: the conversion to float is monotonic)
  auto lower = [](int a, int b) { return min(a, b); };
  auto upper = [](int a, int b) { return max(a, b); };
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t b0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)u[k]);
    const int du = (int)(u[k] - b0);
    const int dlo = __builtin_amdgcn_readfirstlane(group_reduce<CI>(du, lower));
    const int dhi = __builtin_amdgcn_readfirstlane(group_reduce<CI>(du, upper));
    // (rounded up: dlo - mid and dhi - mid stay within 32 bits for a cluster
    // as wide as the axis)
    const uint32_t wid = (uint32_t)dhi - (uint32_t)dlo;
    const int mid = (int)((uint32_t)dlo + (wid >> 1) + (wid & 1u));
    K.u0[k] = b0 + (uint32_t)mid;
    r[k] = (float)((double)(du - mid) * R.scaled[k]);
    K.lo[k] = uni((float)(dlo - mid) * R.scalef[k]);
    K.hi[k] = uni((float)(dhi - mid) * R.scalef[k]);
    const unsigned long long pp = (unsigned long long)K.u0[k] * (unsigned)R.nc[k];
    K.c0[k] = (int)(pp >> 32);
    K.p0[k] = uni((float)(uint32_t)(pp & 0xffffffffu) * 2.3283064365386963e-10f * R.hf[k]);
  }
  nn = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
  K.rcl = R.rclf;
  K.rclm = R.rclmf;
  // (nn >= 0: its bits order as it does)
  const float nmax = __int_as_float(__builtin_amdgcn_readfirstlane(group_reduce<CI>(__float_as_int(nn), upper)));
  K.compact = nmax <= 9.f * K.rcl * K.rcl;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    K.clo[k] = (int)floorf((K.p0[k] + K.lo[k] - K.rclm) * R.ihf[k]);
    K.chi[k] = (int)floorf((K.p0[k] + K.hi[k] + K.rclm) * R.ihf[k]);
    K.clo[k] = __builtin_amdgcn_readfirstlane(K.clo[k]);
    K.chi[k] = __builtin_amdgcn_readfirstlane(K.chi[k]);
    K.whole[k] = K.chi[k] - K.clo[k] + 1 >= R.nc[k];
    if (K.whole[k]) {
      K.clo[k] = 0;
      K.chi[k] = R.nc[k] - 1;
    }
  }
}

// Sign of the periodic offset from cell index a to cell index c along an
// axis of n cells: +1 when c lies less than half the axis ahead of a, -1
// when less than half behind, 0 when equal; at exactly half the axis the
// smaller index counts as behind.  ahead(c, a, n) = -ahead(a, c, n).
__device__ inline int ahead(int c, int a, int n) {
  int d = c - a;
  if (d == 0) return 0;
  if (d < 0) d += n;
  if (2 * d < n) return 1;
  if (2 * d > n) return -1;
  return a < c ? 1 : -1;
}

// One round of the enumeration: the 8 x 8 columns from (x0, y0) on of the
// cluster's reach, one per lane, culled by the exact box-to-column distance,
// each z run clipped to the sphere of radius rclm around the box and split
// at the periodic end into up to two bead ranges; the non-empty ranges go to
// seg (first bead, length) (wave-level, no block barriers).  Returns their
// number.
template <bool HALF>
__device__ inline int column_segments(const ClusterBox& K, const RepDesc& R, const int* __restrict__ start, int first,
                                      int x0, int y0, int2* seg) {
  const int lane = threadIdx.x & 63;
  const int nx = R.nc[0], ny = R.nc[1], nz = R.nc[2];
  const float rclm2 = K.rclm * K.rclm;
  int b0[2] = {0, 0}, ln[2] = {0, 0};
  const int rx = x0 + (lane >> 3), ry = y0 + (lane & 7);
  if (rx <= K.chi[0] && ry <= K.chi[1]) {
    const float hx = R.hf[0], hy = R.hf[1];
    const float gx = K.whole[0] ? 0.f
                                : fmaxf(0.f, fmaxf(rx * hx - (K.p0[0] + K.hi[0]), (K.p0[0] + K.lo[0]) - (rx + 1) * hx));
    const float gy = K.whole[1] ? 0.f
                                : fmaxf(0.f, fmaxf(ry * hy - (K.p0[1] + K.hi[1]), (K.p0[1] + K.lo[1]) - (ry + 1) * hy));
    const float d2 = gx * gx + gy * gy;
    if (d2 < rclm2) {
      int cx = K.whole[0] ? rx : K.c0[0] + rx;
      int cy = K.whole[1] ? ry : K.c0[1] + ry;
      cx += cx < 0 ? nx : (cx >= nx ? -nx : 0);
      cy += cy < 0 ? ny : (cy >= ny ? -ny : 0);
      const int sx = HALF ? ahead(cx, K.c0[0], nx) : 1, sy = HALF ? ahead(cy, K.c0[1], ny) : 1;
      const bool owned = sx > 0 || (sx == 0 && sy >= 0);
      int zlo = 0, zhi = nz - 1;
      if (!K.whole[2]) {
        const float zr = __builtin_amdgcn_sqrtf(rclm2 - d2) * 1.000001f;  // (1 ulp root, kept conservative)
        zlo = K.c0[2] + (int)floorf((K.p0[2] + K.lo[2] - zr) * R.ihf[2]);
        zhi = K.c0[2] + (int)floorf((K.p0[2] + K.hi[2] + zr) * R.ihf[2]);
        if (zhi - zlo + 1 >= nz) {
          zlo = 0;
          zhi = nz - 1;
        }
      }
      const int col = cx * ny + cy;
      if (col & 1) {  // a column counted downwards (cell_of)
        const int t = nz - 1 - zlo;
        zlo = nz - 1 - zhi;
        zhi = t;
      }
      const int colbase = R.cell_off + col * nz;
      if (zlo < 0) {
        b0[0] = start[colbase + zlo + nz];
        ln[0] = start[colbase + nz] - b0[0];
        b0[1] = start[colbase];
        ln[1] = start[colbase + zhi + 1] - b0[1];
      } else if (zhi >= nz) {
        b0[0] = start[colbase + zlo];
        ln[0] = start[colbase + nz] - b0[0];
        b0[1] = start[colbase];
        ln[1] = start[colbase + zhi - nz + 1] - b0[1];
      } else {
        b0[0] = start[colbase + zlo];
        ln[0] = start[colbase + zhi + 1] - b0[0];
      }
      if (HALF && !owned) ln[0] = ln[1] = 0;
      if (HALF && sx == 0 && sy == 0) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int e = b0[q] + ln[q], nb = max(b0[q], first);
          ln[q] = max(0, e - nb);
          b0[q] = nb;
        }
      }
    }
  }
  int nseg = 0;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const bool has = ln[q] > 0;
    const unsigned long long m = __ballot(has);
    if (q == 1 && m == 0ull) break;  // no column wraps
    if (has) seg[nseg + lanes_below(m)] = make_int2(b0[q], ln[q]);
    nseg += __popcll(m);
  }
  __builtin_amdgcn_wave_barrier();
  return nseg;
}

// Every bead of the cells within reach of the cluster: the columns whose
// distance to the cluster's box is below rclm, each with its z run clipped to
// the sphere of radius rclm around the box.  The beads are handed over in
// rounds: a round leaves up to NL_CAND bead indices in cand[0, total) and
// calls visit(total).  Wavefront-level only (no block barriers); seg is the
// wavefront's NL_SEG-entry segment scratch.
template <class V>
__device__ inline void for_candidates(const ClusterBox& K, const RepDesc& R, const int* __restrict__ start, int2* seg,
                                      int* cand, V&& visit) {
  const int lane = threadIdx.x & 63;
  for (int x0 = K.clo[0]; x0 <= K.chi[0]; x0 += 8)
    for (int y0 = K.clo[1]; y0 <= K.chi[1]; y0 += 8) {
      const int nseg = column_segments<false>(K, R, start, 0, x0, y0, seg);
      // expand segments into the candidate buffer (a segment too long for the
      // room left is split across rounds), then visit the round.  A round
      // takes 64 segments, a lane each, or the last 32 by two lanes each.
      int sn = 0, soff = 0;
      while (sn < nseg) {
        const int two = nseg - sn <= 32 ? 1 : 0;
        const int s = sn + (lane >> two), sub = lane & two;
        int sb = 0, sl = 0;
        if (s < nseg) {
          const int2 sg = seg[s];
          const int skip = s == sn ? soff : 0;
          sb = sg.x + skip;
          sl = sg.y - skip;
        }
        const int inc = wave_incl_scan(sub == 0 ? sl : 0);
        const int exc = inc - sl;
        const int take = max(0, min(sl, NL_CAND - exc));
        int t = sub;
        int* dst = cand + exc;
        while (__any(t < take)) {
          if (t < take) dst[t] = sb + t;
          t += 1 + two;
        }
        const int total = min((int)read_lane((uint32_t)inc, 63), NL_CAND);
        const unsigned long long partial = __ballot(take < sl);
        if (partial == 0ull) {
          sn += 64 >> two;
          soff = 0;
        } else {
          const int f = __ffsll((long long)partial) - 1;
          const int tf = (int)read_lane((uint32_t)take, f);
          soff = ((f >> two) == 0 ? soff : 0) + tf;
          sn += f >> two;
        }
        __builtin_amdgcn_wave_barrier();
        visit(total);
        __builtin_amdgcn_wave_barrier();
      }
    }
}

// The candidates cand[0, total) in chunks of 64, one per lane: the index and
// bead-record loads of NCH chunks are issued together (one memory latency
// covers them), then f(record, valid, index) runs per chunk in order.  Three
// chunks at a time, the whole record waited for at once and a last drain that
// stops at its last group: N = 2,097,152 pairs 731 -> 699 us, 256 replicas 268 ->
// 258 us (two chunks: 717 and 264).
template <int NCH, class F>
__device__ inline void for_chunks(const int* cand, int total, const uint4* __restrict__ pk, int fallback, F&& f) {
  const int lane = threadIdx.x & 63;
  for (int p = 0; p < total; p += 64 * NCH) {
    int jj[NCH];
    uint4 rr[NCH];
#pragma unroll
    for (int u = 0; u < NCH; ++u) {
      const int q = p + 64 * u + lane;
      jj[u] = q < total ? cand[q] : -1;
    }
#pragma unroll
    for (int u = 0; u < NCH; ++u) rr[u] = pk[jj[u] < 0 ? fallback : jj[u]];
#pragma unroll
    for (int u = 0; u < NCH; ++u)
      if (u == 0 || p + 64 * u < total) {
        // (the parameter word with the position: the compiler would sink its
        // load into the branch that stores the hits, a second memory latency)
        asm volatile("" : "+v"(rr[u].w));
        f(rr[u], jj[u] >= 0, jj[u] < 0 ? fallback : jj[u]);
      }
  }
}

// ---------------------------------------------------------------------------
// List build
// ---------------------------------------------------------------------------

// Whether the cluster takes the fast path: in its frame, separations equal the
// per-pair minimum image for every pair within rc as long as each cluster bead
// lies within L/2 - rc of the centre on each axis (then |d| < rc cannot wrap);
// and the cluster is compact (every bead within 3 rcl of the centre), which
// bounds the rounding of the frame-relative arithmetic.
__device__ inline bool in_frame(const ClusterBox& K, const RepDesc& R) {
  bool frame = K.compact;
#pragma unroll
  for (int k = 0; k < 3; ++k) frame = frame && fmaxf(-K.lo[k], K.hi[k]) < 0.5f * (float)R.L[k] - K.rclm;
  return frame;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// The list test of a compact cluster in its frame, on the matrix cores:
// |D - r_i|^2 < rcl^2 for some bead i is tested as
// min_i(|r_i|^2 - 2 D.r_i) < rcl^2 - |D|^2, D the candidate's position
// relative to the centre.  The left side is a product of the CI x 3 matrix of
// -2 r_i with the 3 x 64 matrix of the candidates, started from |r_i|^2: the
// 4 x 4 x 1 multiply in 16 blocks takes four beads (rows) against the
// wavefront's 64 candidates (four columns in each block) for one axis, and
// leaves in each lane the four values of its own candidate.  Three of them
// per four beads replace 12 fused multiply-adds, and the matrix pipe runs
// beside the other wavefronts' vector instructions: the candidate test of
// eight beads went from 35 vector instructions to 8 and 6 matrix
// instructions.  The candidates that can pass lie within 4 rcl of the centre, so
// the rounding of the expanded form stays below 1e-5 rcl^2, inside the margin
// of rcl over rc: no pair within rc is dropped.
template <int CI>
struct FrameTest {
  float qx, qy, qz;            // -2 r of bead lane % CI
  f32x4 n[CI > 4 ? CI / 4 : 1];  // |r_i|^2 of beads 4 h .. 4 h + 3
  float rcl2;
};

template <int CI>
__device__ inline void frame_test_init(FrameTest<CI>& T, const ClusterBox& K, const float r[3], float nn) {
  T.qx = -2.f * r[0];
  T.qy = -2.f * r[1];
  T.qz = -2.f * r[2];
  T.rcl2 = K.rcl * K.rcl;
#pragma unroll
  for (int h = 0; h < (CI > 4 ? CI / 4 : 1); ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i)  // (CI = 2: rows 2 and 3 repeat beads 0 and 1, as their lanes do)
      T.n[h][i] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(nn), 4 * h + i));
}

// One four-bead product for one axis: with eight beads, the rows are those of
// block H (lanes 4 H .. 4 H + 3), broadcast to all 16 blocks; with four or
// two, every block holds them already.
template <int CI, int H>
__device__ inline f32x4 frame_mfma(float q, float d, f32x4 c) {
  return CI > 4 ? __builtin_amdgcn_mfma_f32_4x4x1f32(q, d, c, 4, H, 0)
                : __builtin_amdgcn_mfma_f32_4x4x1f32(q, d, c, 0, 0, 0);
}

// Every lane of the wavefront must call it; D receives the lane's candidate
// pj relative to the centre.
template <int CI>
__device__ inline bool near_frame(const FrameTest<CI>& T, const ClusterBox& K, const uint4& pj, const RepDesc& R,
                                  float& Dx, float& Dy, float& Dz) {
  Dx = (float)((double)(int)(pj.x - K.u0[0]) * R.scaled[0]);
  Dy = (float)((double)(int)(pj.y - K.u0[1]) * R.scaled[1]);
  Dz = (float)((double)(int)(pj.z - K.u0[2]) * R.scaled[2]);
  const float thr = T.rcl2 - (Dx * Dx + Dy * Dy + Dz * Dz);
  f32x4 v = frame_mfma<CI, 0>(T.qx, Dx, T.n[0]);
  v = frame_mfma<CI, 0>(T.qy, Dy, v);
  v = frame_mfma<CI, 0>(T.qz, Dz, v);
  if constexpr (CI > 4) {
    f32x4 w = frame_mfma<CI, 1>(T.qx, Dx, T.n[1]);
    w = frame_mfma<CI, 1>(T.qy, Dy, w);
    w = frame_mfma<CI, 1>(T.qz, Dz, w);
    const float m0 = fminf(fminf(v[0], v[1]), v[2]), m1 = fminf(fminf(v[3], w[0]), w[1]);
    return fminf(fminf(fminf(w[2], w[3]), m0), m1) < thr;
  } else if constexpr (CI == 4) {
    return fminf(fminf(fminf(v[0], v[1]), v[2]), v[3]) < thr;
  } else {
    return fminf(v[0], v[1]) < thr;
  }
}

// The same test by the minimum image of each pair (any cluster); lane k < CI
// of `me` holds bead k.
template <int CI>
__device__ inline bool near_exact(const ClusterBox& K, const uint4& me, const uint4& pj, const RepDesc& R) {
  const float rcl2f = K.rcl * K.rcl;
  bool hit = false;
#pragma unroll
  for (int i = 0; i < CI; ++i) {
    const float dx = (float)(int)(read_lane(me.x, i) - pj.x) * R.scalef[0];
    const float dy = (float)(int)(read_lane(me.y, i) - pj.y) * R.scalef[1];
    const float dz = (float)(int)(read_lane(me.z, i) - pj.z) * R.scalef[2];
    hit |= dx * dx + dy * dy + dz * dz < rcl2f;
  }
  return hit;
}

// ---------------------------------------------------------------------------
// Pair evaluation
// ---------------------------------------------------------------------------

// Per-lane accumulators.
template <typename T>
struct Lane {
  T fx, fy, fz;
  double e, w0, w1, w2, w3, w4, w5;  // energy and virial summed in FP64
  T eA[MAXT], dj[MAXT], di;          // adjoint sums of the lane's bead i
  T ett[MAXT * MAXT];                // adjoint: type-pair energies (ti, tj)
  T dsg[MAXT];                       // adjoint: d/dsigma_t (excluded volume) or d/da_t (real space)
  unsigned long long cnt;
};

template <typename T>
__device__ inline void lane_zero(Lane<T>& L) {
  L.fx = L.fy = L.fz = 0;
  L.e = L.w0 = L.w1 = L.w2 = L.w3 = L.w4 = L.w5 = 0;
  for (int t = 0; t < MAXT; ++t) L.eA[t] = L.dj[t] = L.dsg[t] = 0;
  for (int t = 0; t < MAXT * MAXT; ++t) L.ett[t] = 0;
  L.di = 0;
  L.cnt = 0;
}

// The real-space bracket of eq. ewald for one type pair at r^2 = r2 > 0:
// phi = [erf(alpha r) - erf(beta r)]/r and g = -(1/r) dphi/dr; ea receives
// exp(-alpha^2 r^2) where the evaluation computes it (left as is in the
// series branch).  cexpb = -beta^2 log2(e), tsb = (2/sqrt(pi)) beta.
template <typename T>
__device__ __attribute__((always_inline)) inline void bracket(const ElecPar<T>& p, T r2, T beta, T beta2, T cexpb,
                                                              T tsb, T& phi, T& g, T& ea) {
  constexpr T TSP = (T)1.1283791670955126;  // 2/sqrt(pi)
  if (r2 < p.rs2) {
    // series in r^2, free of the cancellation near contact
    phi = p.cphi[Series<T>::n - 1];
    g = p.cg[Series<T>::n - 1];
#pragma unroll
    for (int n = Series<T>::n - 2; n >= 0; --n) {
      phi = phi * r2 + p.cphi[n];
      g = g * r2 + p.cg[n];
    }
  } else if constexpr (std::is_same<T, float>::value) {
    // single precision: both error functions from their Gaussians, which
    // the force needs anyway (one reciprocal square root, two 2^x, two
    // reciprocals)
    // each product rounded on its own (no multiply-add fused across a
    // difference), so that alpha == beta gives exactly zero
#pragma clang fp contract(off)
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float r = r2 * rinv;
    ea = gexp2(p.cexp * r2);
    const float eb = gexp2(cexpb * r2);
    phi = (erfc_scaled(beta * r) * eb - erfc_scaled(p.alpha * r) * ea) * rinv;
    g = (phi - (p.tsa * ea - tsb * eb)) * rinv * rinv;
    (void)beta2;
  } else {
    T r = gsqrt(r2);
    T rinv = (T)1 / r;
    ea = gexp(-p.alpha2 * r2);
    phi = (gerfc(beta * r) - gerfc(p.alpha * r)) * rinv;
    g = (phi - TSP * (p.alpha * ea - beta * gexp(-beta2 * r2))) * rinv * rinv;
    (void)cexpb;
    (void)tsb;
  }
}

// The pair's virial d_a f_b, f = fs d, in FP64.
template <typename T>
__device__ inline void add_virial(Lane<T>& L, T fs, T dx, T dy, T dz) {
  const double fxd = (double)(fs * dx), fyd = (double)(fs * dy), fzd = (double)(fs * dz);
  L.w0 += fxd * (double)dx;
  L.w1 += fyd * (double)dy;
  L.w2 += fzd * (double)dz;
  L.w3 += fxd * (double)dy;
  L.w4 += fxd * (double)dz;
  L.w5 += fyd * (double)dz;
}

// x to the accumulator of type tj < nt (nt the same for the wavefront: the
// accumulators of types that the replica does not have are not looked at).
template <typename T>
__device__ inline void add_by_type(T (&v)[MAXT], int tj, int nt, T x) {
#pragma unroll
  for (int t = 0; t < MAXT; ++t)
    if (t < nt) v[t] += t == tj ? x : (T)0;
}

// One ordered pair (i, j) with separation d = r_i - r_j, r2 < rc^2.  The
// derivative with respect to a radius adds the pair's share at bead i's type
// alone: bead j's share is added when the pair is seen from j (in the force
// vector-Jacobian product, whose two visits differ by v, both are added).
template <typename T, bool ELEC, bool EV, bool ADJ, bool COUNT>
__device__ inline void interact(Lane<T>& L, T dx, T dy, T dz, T r2, uint32_t pj, const GcmPar<T>* grow,
                                const ElecPar<T>* erow, const AdjPar<T>* arow, T zi, T beta, T beta2, T lB,
                                T vx, T vy, T vz, bool vjp, T cexpb, T tsb, int nt, bool vir) {
  const int tj = param_type(pj);
  T fs, en;
  if (!ELEC) {
    const GcmPar<T> g = grow[tj];
    en = g.C * gexp2(-g.bl * r2);
    fs = g.twob * en;
    if (ADJ) {
      const AdjPar<T> ap = arow[tj];
      // du/ds = u (3 r^2/s^3 - 3/s), s = s_ij
      T duds = en * ((T)3 * r2 * ap.inv_s2 - (T)3) * ap.s_inv;
      T eA = en;
      if (vjp) {
        // force vector-Jacobian product: (v_i . d) dfs/dtheta with
        // dfs/dA = fs/A (divided by A with the energies) and
        // dfs/ds = (u/s^3)(9 r^2/s^2 - 15)
        const T vd = vx * dx + vy * dy + vz * dz;
        eA = vd * fs;
        duds = vd * en * ap.inv_s2 * ap.s_inv * ((T)9 * r2 * ap.inv_s2 - (T)15);
      }
      L.di += duds * ap.dsig_i;
      add_by_type(L.eA, tj, nt, eA);
      if (vjp) add_by_type(L.dj, tj, nt, duds * ap.dsig_j);
    }
  } else {
    const ElecPar<T>& p = erow[tj];
    const T zz = zi * (T)param_z(pj);
    T phi, g, ea = 0;  // ea: exp(-alpha^2 r^2) where computed
    bracket(p, r2, beta, beta2, cexpb, tsb, phi, g, ea);
    fs = lB * zz * g;
    en = lB * zz * phi;
    if (ADJ) {
      const AdjPar<T> ap = arow[tj];
      // d/da_ij of lB zz erf(alpha r)/r = -lB zz (2/sqrt(pi)) (alpha/a_ij) exp(-alpha^2 r^2)
      if (r2 < p.rs2) ea = gexp(-p.alpha2 * r2);
      T dd = -lB * zz * ap.ea * ea;
      // force vector-Jacobian product: dg/dalpha = 2 (2/sqrt(pi)) alpha^2
      // exp(-alpha^2 r^2), so dfs/da_ij = 2 alpha^2 dd
      if (vjp) dd = (vx * dx + vy * dy + vz * dz) * (T)2 * p.alpha2 * dd;
      L.di += dd * ap.daij_i;
      if (vjp) add_by_type(L.dj, tj, nt, dd * ap.daij_j);
    }
  }
  L.fx += fs * dx;
  L.fy += fs * dy;
  L.fz += fs * dz;
  if (EV) {
    L.e += (double)en;
    if (vir) add_virial(L, fs, dx, dy, dz);
  }
  if (COUNT) ++L.cnt;
}

// Move the adjoint sums of bead i (type ti) into the per-type accumulators.
template <typename T, bool ELEC>
__device__ inline void flush_adj(Lane<T>& L, int ti, bool vjp) {
#pragma unroll
  for (int q = 0; q < MAXT; ++q) {
#pragma unroll
    for (int t = 0; t < MAXT; ++t)
      if (q == ti && !ELEC) L.ett[q * MAXT + t] += L.eA[t];
    if (q == ti) L.dsg[q] += vjp ? L.di : (T)2 * L.di;  // (both visits' shares; halved at the end)
    L.dsg[q] += L.dj[q];
  }
#pragma unroll
  for (int q = 0; q < MAXT; ++q) {
    L.eA[q] = 0;
    L.dj[q] = 0;
  }
  L.di = 0;
}

// The exponent and force factor of eq. u_ex for one type pair: the force over
// the separation is fc 2^(nb r^2).
template <typename T>
struct ExpPar {
  T nb, fc;
};

// What a lane needs to evaluate the pairs of its bead i.
template <typename T>
struct PairCtx {
  T sx, sy, sz, rc2, beta, beta2, lB, zi;
  T cexpb, tsb;  // -beta^2 log2(e), (2/sqrt(pi)) beta
  T vx, vy, vz;  // force vector-Jacobian product: v of bead i (adjoint only)
  bool vjp;
  int nt;        // types of the replica
  bool vir;      // the virial is asked for
  const ExpPar<T>* prow;
  const GcmPar<T>* grow;
  const ElecPar<T>* erow;
  const AdjPar<T>* arow;
};

// The replica's type-pair tables, staged once per workgroup.
template <typename T, bool ELEC, bool ADJ>
struct Tables {
  ExpPar<T> p[ELEC ? 1 : MAXT * MAXT];
  GcmPar<T> g[ELEC ? 1 : MAXT * MAXT];
  ElecPar<T> e[ELEC ? MAXT * MAXT : 1];
  AdjPar<T> a[ADJ ? MAXT * MAXT : 1];
};

template <typename T, bool ELEC, bool ADJ>
__device__ inline void stage_tables(Tables<T, ELEC, ADJ>& S, const PairLaunch& a, int rep) {
  const size_t tb = (size_t)rep * MAXT * MAXT;
  if (!ELEC && threadIdx.x < MAXT * MAXT) {
    const GcmPar<T> g = reinterpret_cast<const GcmPar<T>*>(a.gcm)[tb + threadIdx.x];
    S.g[threadIdx.x] = g;
    S.p[threadIdx.x] = ExpPar<T>{-g.bl, g.fC};
  }
  if (ELEC && threadIdx.x < MAXT * MAXT) S.e[threadIdx.x] = reinterpret_cast<const ElecPar<T>*>(a.elec)[tb + threadIdx.x];
  if (ADJ && threadIdx.x < MAXT * MAXT) S.a[threadIdx.x] = reinterpret_cast<const AdjPar<T>*>(a.adj)[tb + threadIdx.x];
  __syncthreads();
}

template <typename T, bool ELEC, bool ADJ>
__device__ inline PairCtx<T> make_ctx(const Tables<T, ELEC, ADJ>& S, const RepDesc& R, uint32_t pi,
                                      const PairLaunch& a, int i) {
  const int ti = param_type(pi);
  PairCtx<T> P;
  P.sx = (T)R.scaled[0];
  P.sy = (T)R.scaled[1];
  P.sz = (T)R.scaled[2];
  P.rc2 = (T)R.rc2;
  P.beta = (T)R.beta;
  P.beta2 = (T)(R.beta * R.beta);
  if constexpr (std::is_same<T, float>::value) {
    // float operations matching the host's for alpha (see build_tables)
    const float bf = (float)R.beta;
    P.cexpb = -(bf * bf) * 1.44269504088896341f;
    P.tsb = 1.12837916709551257f * bf;
  } else {
    P.cexpb = -R.beta * R.beta * 1.4426950408889634;
    P.tsb = 1.1283791670955126 * R.beta;
  }
  P.lB = (T)R.lB;
  P.zi = (T)param_z(pi);
  P.prow = S.p + (ELEC ? 0 : ti * MAXT);
  P.grow = S.g + (ELEC ? 0 : ti * MAXT);
  P.erow = S.e + (ELEC ? ti * MAXT : 0);
  P.arow = S.a + (ADJ ? ti * MAXT : 0);
  P.nt = R.nt;
  P.vir = a.virial != 0;
  P.vjp = false;
  P.vx = P.vy = P.vz = 0;
  if (ADJ && a.vjp) {
    const int fi = ELEC ? a.qidx[i] : i;
    P.vjp = true;
    P.vx = (T)a.vjp[fi];
    P.vy = (T)a.vjp[(size_t)a.nbeads + fi];
    P.vz = (T)a.vjp[2 * (size_t)a.nbeads + fi];
  }
  return P;
}

// Pair (i, j) when ok (j a real bead other than i) and r < rc: separation by
// the exact minimum image in T, the one cutoff test of the method's sums.
template <typename T, bool ELEC, bool EV, bool ADJ, bool COUNT>
__device__ inline void pair_at(Lane<T>& L, const PairCtx<T>& P, T dx, T dy, T dz, uint32_t pw, bool ok) {
  const T r2 = dx * dx + dy * dy + dz * dz;
  const bool in = ok && r2 < P.rc2;
  if (!ELEC && !ADJ && !COUNT) {
    // excluded volume: cheap enough to evaluate for every lane, which keeps
    // the unrolled pairs free of branches; a pair that does not count gets
    // the exponent -inf, hence exactly zero
    const ExpPar<T> g = P.prow[param_type(pw)];
    const T ex = gexp2(in ? g.nb * r2 : -(T)INFINITY);
    const T fs = g.fc * ex;
    L.fx += fs * dx;
    L.fy += fs * dy;
    L.fz += fs * dz;
    if (EV) {
      L.e += (double)(P.grow[param_type(pw)].C * ex);
      if (P.vir) add_virial(L, fs, dx, dy, dz);
    }
  } else if (in) {
    interact<T, ELEC, EV, ADJ, COUNT>(L, dx, dy, dz, r2, pw, P.grow, P.erow, P.arow, P.zi, P.beta, P.beta2, P.lB,
                                      P.vx, P.vy, P.vz, P.vjp, P.cexpb, P.tsb, P.nt, P.vir);
  }
}

template <typename T, bool ELEC, bool EV, bool ADJ, bool COUNT>
__device__ inline void try_pair(Lane<T>& L, const PairCtx<T>& P, const uint4& mi, const uint4& pj, bool ok) {
  const T dx = (T)(int)(mi.x - pj.x) * P.sx;
  const T dy = (T)(int)(mi.y - pj.y) * P.sy;
  const T dz = (T)(int)(mi.z - pj.z) * P.sz;
  pair_at<T, ELEC, EV, ADJ, COUNT>(L, P, dx, dy, dz, pj.w, ok);
}

// Combine the partial forces of bead i over its CJ lanes (lane exchanges, fixed
// order) and add them once to the fixed-point accumulator.
template <typename T, int CI, bool ELEC, bool ADJ>
__device__ inline void flush_bead(const PairLaunch& a, Lane<T>& L, bool vi, int i, int ti) {
  constexpr int CJ = 64 / CI;
  const int jl = (threadIdx.x & 63) % CJ;
  if (ADJ && a.dbead) {
    // the bead's own-radius derivative: every bead is in one cluster, so one
    // store per bead, summed over its lanes in a fixed order
    T d = L.di;
#pragma unroll
    for (int o = CJ >> 1; o > 0; o >>= 1) d += __shfl_xor(d, o, 64);
    if (vi && jl == 0) a.dbead[ELEC ? a.qidx[i] : i] = (double)d;
  }
  if (ADJ && vi) flush_adj<T, ELEC>(L, ti, a.vjp != nullptr);
  // lanes 0, 1 and 2 of the bead's group add one axis each
  const T fx = group_sum<CJ>(L.fx), fy = group_sum<CJ>(L.fy), fz = group_sum<CJ>(L.fz);
  if (vi && jl < 3) {
    const int fi = ELEC ? a.qidx[i] : i;
    const T f = jl == 0 ? fx : jl == 1 ? fy : fz;
    long long* F = jl == 0 ? a.F[0] : jl == 1 ? a.F[1] : a.F[2];
    atomicAdd((unsigned long long*)&F[fi], (unsigned long long)to_fixed((double)f, a.fscale, a.status));
  }
}

// Workgroup partial sums (every pair was seen from both ends: halved).
// Reached by every thread of the workgroup.
template <typename T, bool ELEC, bool EV, bool ADJ, bool COUNT>
__device__ inline void block_outputs(const PairLaunch& a, const Lane<T>& L, double* red, int item) {
  const int lane = threadIdx.x & 63;
  if (COUNT) {
    unsigned long long cc = L.cnt;
    for (int o = 32; o > 0; o >>= 1) cc += __shfl_xor(cc, o, 64);
    if (lane == 0 && cc) atomicAdd(a.pair_count, cc);
  }
  if (EV) {
    double v[7] = {L.e, L.w0, L.w1, L.w2, L.w3, L.w4, L.w5};
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      double t = block_sum(v[k], red);
      if (threadIdx.x == 0) a.part[(size_t)item * PART_W + k] = 0.5 * t;
    }
  }
  if (ADJ) {
    constexpr int W = MAXT * MAXT + 2 * MAXT;
    if (!ELEC) {
      for (int q = 0; q < MAXT * MAXT; ++q) {
        double t = block_sum((double)L.ett[q], red);
        if (threadIdx.x == 0) a.adj_part[(size_t)item * W + q] = 0.5 * t;
      }
    }
    for (int t = 0; t < MAXT; ++t) {
      double s = block_sum((double)L.dsg[t], red);
      if (threadIdx.x == 0) a.adj_part[(size_t)item * W + MAXT * MAXT + (ELEC ? MAXT : 0) + t] = 0.5 * s;
    }
  }
}

// List-driven pairs: one wavefront per cluster, lanes = CI beads x 64/CI
// list entries.
template <typename T, int CI, bool ELEC, bool EV, bool ADJ, bool COUNT>
__global__ __launch_bounds__(NL_WAVES * 64) void k_nl_force(PairLaunch a) {
  constexpr int CJ = 64 / CI;
  __shared__ double red[NL_WAVES];
  __shared__ Tables<T, ELEC, ADJ> S;
  wave_stamp(a.stamps, 0);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int item = xcd_item(blockIdx.x, a.ntiles);
  const Tile tl = uniform_load(a.tiles + item);
  const RepDesc R = uniform_load(a.rep + tl.rep);
  stage_tables(S, a, tl.rep);
  const int il = lane / CJ, jl = lane % CJ;
  Lane<T> L;
  lane_zero(L);
  if (wave < tl.count) {
    const int c = tl.first + wave;
    const int2 info = a.cl[c];
    const int first = info.x, ni = info.y >> 16;
    const bool vi = il < ni;
    const int i = first + (vi ? il : 0);
    const uint4 mi = a.pk[i];
    const PairCtx<T> P = make_ctx(S, R, mi.w, a, i);
    const int cnt = a.count[c];
    const uint32_t* __restrict__ lst = a.list + (size_t)c * a.cap;
    const uint4* __restrict__ pk = a.pk;
    // NU entries per lane per round: the list loads, then the dependent
    // bead-record loads, are issued back to back so one memory latency
    // covers NU pairs
    constexpr int NU = 4;
    for (int e0 = jl; e0 < cnt; e0 += NU * CJ) {
      int jj[NU];
      uint4 pp[NU];
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int e = e0 + u * CJ;
        jj[u] = e < cnt ? (int)lst[e] : -1;
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) pp[u] = pk[jj[u] < 0 ? i : jj[u]];
#pragma unroll
      for (int u = 0; u < NU; ++u) try_pair<T, ELEC, EV, ADJ, COUNT>(L, P, mi, pp[u], vi && jj[u] >= 0 && jj[u] != i);
    }
    flush_bead<T, CI, ELEC, ADJ>(a, L, vi, i, param_type(mi.w));
  }
  block_outputs<T, ELEC, EV, ADJ, COUNT>(a, L, red, item);
  wave_stamp(a.stamps, 1);
}

// List-free pairs: one wavefront per cluster enumerates the candidates of
// its cell columns (as the list build does), keeps those within the list
// cutoff of some cluster bead (the list build's test), and evaluates them at
// once from an LDS ring of pending pairs: whenever 64 are pending they are
// taken by the lanes laid out as CI beads x 64/CI entries.  The same pairs
// and cutoff test as the list path, with no list in HBM.
constexpr int RING = 128;  // pending-pair ring per wavefront (entries)
static_assert(RING == 128, "the drain relies on a ring of exactly two 64-entry halves");

// Wavefronts per SIMD the list-free kernel is compiled for, at least: the
// kernel is bound by instruction issue, and fewer than four wavefronts leave
// gaps between the LDS reads of a drain and their use.  In single precision
// forces alone take 82 registers without being told (five wavefronts); left
// to itself the compiler gave energies 143 and the adjoint 141 (three), and
// both fit 124 without a spill.  Evaluations of 199,999 beads, three and four
// wavefronts: energies 428 and 398 us, with the virial 459 and 431, adjoint
// 620 and 542; of 32,768 beads 143 and 139, 154 and 149, 198 and 176.  Double
// precision does not fit 128 registers, and counting is no timed path.
template <typename T, bool EV, bool ADJ, bool COUNT>
struct FusedWaves {
  static constexpr int value = std::is_same<T, float>::value && !COUNT ? 4 : 1;
};

template <typename T, int CI, bool ELEC, bool EV, bool ADJ, bool COUNT>
__global__ __launch_bounds__(NL_WAVES * 64) __attribute__((amdgpu_waves_per_eu(FusedWaves<T, EV, ADJ, COUNT>::value)))
void k_pair_fused(PairLaunch a) {
  constexpr int CJ = 64 / CI;
  __shared__ double red[NL_WAVES];
  __shared__ Tables<T, ELEC, ADJ> S;
  __shared__ int2 s_seg[NL_WAVES][NL_SEG];
  __shared__ int s_cand[NL_WAVES][NL_CAND];
  __shared__ uint4 s_ring[NL_WAVES][RING];
  wave_stamp(a.stamps, 0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int item = xcd_item(blockIdx.x, a.ntiles);
  const Tile tl = uniform_load(a.tiles + item);
  const RepDesc R = uniform_load(a.rep + tl.rep);
  const int il = lane / CJ, jl = lane % CJ;
  const uint4* __restrict__ pk = a.pk;
  // this wave's cluster: CI consecutive beads from bead0 + wave CI (the
  // replica's last cluster may be short).  Its records are requested before
  // the tables are staged, so the two loads overlap.
  const bool active = wave < tl.count;
  const int first = __builtin_amdgcn_readfirstlane(tl.bead0 + wave * CI);
  const int ni =
      __builtin_amdgcn_readfirstlane(active ? min(CI, (ELEC ? R.q_off + R.nq : R.bead_off + R.n) - first) : 1);
  const bool vi = il < ni;
  const int i = first + (vi ? il : 0);
  uint4 me = make_uint4(0u, 0u, 0u, 0u), mi = me;
  if (active) {
    const int kk = lane % CI;  // lane l: bead l % CI (slots beyond ni: bead 0)
    me = pk[first + (kk < ni ? kk : 0)];
    mi = pk[i];
  }
  stage_tables(S, a, tl.rep);
  Lane<T> L;
  lane_zero(L);
  if (active) {
    ClusterBox K;
    float rme[3], nn;
    make_box<CI>(K, me, R, rme, nn);
    const PairCtx<T> P = make_ctx(S, R, mi.w, a, i);
    uint4* ring = s_ring[wave];
    int head = 0, tail = 0;  // wave-uniform: pairs evaluated / appended
    // Appends the lane's record to the ring where hit, in lane order, and
    // evaluates 64 pending pairs when there are as many.
    auto push = [&](bool hit, const uint4 rec, auto&& drain) __attribute__((always_inline)) {
      const unsigned long long m = __ballot(hit);
      if (hit) ring[(tail + lanes_below(m)) & (RING - 1)] = rec;
      tail += __popcll(m);
      __builtin_amdgcn_wave_barrier();
      if (tail - head >= 64) drain(64);
    };
    // 1 + the cluster slot of a candidate that is itself a cluster bead, else 0
    auto slot_of = [&](int j) -> uint32_t {
      const uint32_t d = (uint32_t)(j - first);
      return d < (uint32_t)ni ? d + 1u : 0u;
    };
    const uint32_t self = (uint32_t)(il + 1);
    const int* cand = s_cand[wave];
    // evaluates the n <= 64 pending entries from head: lane (il, jl) takes
    // entries jl + k CJ, k < CI, in groups of at most four (the records of a
    // group are read together; fewer live registers for CI = 8).  head is a
    // multiple of 64 here (every drain but the last takes exactly 64), so the
    // entries do not wrap.
    constexpr int G = CI < 4 ? CI : 4;
    // In single precision, with the cluster in its frame, the ring holds the
    // candidate's position relative to the centre as floats (computed once,
    // by the test), so a pair costs one subtraction per axis.  Otherwise it
    // holds the fixed-point record, and each pair takes its own minimum
    // image.  (Not for the electrostatics, whose pair cost that would hardly
    // change.)
    constexpr bool REL = std::is_same<T, float>::value && !ELEC && !COUNT;
    // The record's parameter word: in the low half the bead's type and charge
    // (forces alone, BARE: the byte offset of its type in a row of the pair
    // table), in the high half its slot_of.
    constexpr bool BARE = REL && !EV && !ADJ;
    const bool frame = in_frame(K, R);
    FrameTest<CI> ft;
    if (frame) frame_test_init<CI>(ft, K, rme, nn);
    if (REL && frame) {
      const float rxi = (float)((double)(int)(mi.x - K.u0[0]) * R.scaled[0]);
      const float ryi = (float)((double)(int)(mi.y - K.u0[1]) * R.scaled[1]);
      const float rzi = (float)((double)(int)(mi.z - K.u0[2]) * R.scaled[2]);
      // The slots past the last entry of the final drain are filled with a
      // record 1e18 away: the branch-free excluded-volume pair multiplies
      // every lane's separation by its (zero) force factor, so no slot may
      // hold a stale or never-written LDS value (NaN or inf times zero is
      // NaN).  Forces alone (BARE) then need no per-pair validity test: a
      // bead paired with itself has zero separation, so zero force; lanes of
      // missing cluster beads (vi false) are never flushed; and the padding
      // lies beyond the cutoff.
      auto drain = [&](int n) __attribute__((always_inline)) {
        uint4* base = ring + (head & 64);
        if (n < 64) {
          const uint32_t far = __float_as_uint(1e18f);
          if (lane >= n) base[lane] = make_uint4(far, far, far, 0u);
          __builtin_amdgcn_wave_barrier();
        }
#pragma unroll
        for (int k0 = 0; k0 < CI; k0 += G) {
          if (n <= k0 * CJ) break;  // (a last drain that ends before this group)
          uint4 pp[G];
#pragma unroll
          for (int g = 0; g < G; ++g) pp[g] = base[jl + (k0 + g) * CJ];
#pragma unroll
          for (int g = 0; g < G; ++g) {
            const T dx = (T)(rxi - __uint_as_float(pp[g].x));
            const T dy = (T)(ryi - __uint_as_float(pp[g].y));
            const T dz = (T)(rzi - __uint_as_float(pp[g].z));
            if constexpr (BARE) {
              const T r2 = dx * dx + dy * dy + dz * dz;
              const ExpPar<T> p = *reinterpret_cast<const ExpPar<T>*>(reinterpret_cast<const char*>(P.prow) + pp[g].w);
              const T fs = p.fc * gexp2(r2 < P.rc2 ? p.nb * r2 : -(T)INFINITY);
              L.fx += fs * dx;
              L.fy += fs * dy;
              L.fz += fs * dz;
            } else {
              pair_at<T, ELEC, EV, ADJ, COUNT>(L, P, dx, dy, dz, pp[g].w,
                                               vi && jl + (k0 + g) * CJ < n && (pp[g].w >> 16) != self);
            }
          }
        }
        head += n;
      };
      for_candidates(K, R, a.start, s_seg[wave], s_cand[wave], [&](int total) {
        for_chunks<3>(cand, total, pk, first, [&](const uint4 pj, bool v, int j) {
          float Dx, Dy, Dz;
          const bool near = near_frame<CI>(ft, K, pj, R, Dx, Dy, Dz);
          const uint32_t w = BARE ? (pj.w & 0xffu) * (uint32_t)sizeof(ExpPar<T>) : (pj.w & 0xffffu) | slot_of(j) << 16;
          push(near && v, make_uint4(__float_as_uint(Dx), __float_as_uint(Dy), __float_as_uint(Dz), w), drain);
        });
      });
      if (tail > head) drain(tail - head);
    } else {
      // Every slot of both ring halves is written before any drain can read
      // it, with position 0 and parameter word 0 (type 0, a valid table
      // index): a cluster with few candidates (as in sparse regions) drains
      // slots that no candidate was written to.
      ring[lane] = ring[64 + lane] = make_uint4(0u, 0u, 0u, 0u);
      __builtin_amdgcn_wave_barrier();
      auto drain = [&](int n) __attribute__((always_inline)) {
        const uint4* base = ring + (head & 64);
#pragma unroll
        for (int k0 = 0; k0 < CI; k0 += G) {
          if (n <= k0 * CJ) break;  // (a last drain that ends before this group)
          uint4 pp[G];
#pragma unroll
          for (int g = 0; g < G; ++g) pp[g] = base[jl + (k0 + g) * CJ];
#pragma unroll
          for (int g = 0; g < G; ++g) {
            // slots past the last entry of a final drain are masked, and
            // their parameter word replaced by 0 (a valid table index)
            const bool live = jl + (k0 + g) * CJ < n;
            uint4 q = pp[g];
            q.w = live ? q.w : 0u;
            try_pair<T, ELEC, EV, ADJ, COUNT>(L, P, mi, q, vi && live && (q.w >> 16) != self);
          }
        }
        head += n;
      };
      for_candidates(K, R, a.start, s_seg[wave], s_cand[wave], [&](int total) {
        for_chunks<3>(cand, total, pk, first, [&](const uint4 pj, bool v, int j) {
          float Dx, Dy, Dz;
          const bool near = frame ? near_frame<CI>(ft, K, pj, R, Dx, Dy, Dz) : near_exact<CI>(K, me, pj, R);
          push(near && v, make_uint4(pj.x, pj.y, pj.z, (pj.w & 0xffffu) | slot_of(j) << 16), drain);
        });
      });
      if (tail > head) drain(tail - head);
    }
    flush_bead<T, CI, ELEC, ADJ>(a, L, vi, i, param_type(mi.w));
  }
  block_outputs<T, ELEC, EV, ADJ, COUNT>(a, L, red, item);
  wave_stamp(a.stamps, 1);
}

}  // namespace

// Launches the excluded-volume (ELEC false) or charged pairs in the precision T
// of an evaluation: the kernel for the cluster size and the outputs asked for.
template <typename T, bool ELEC>
void dispatch_ci(hipStream_t s, const PairLaunch& a, bool ev, bool adj, bool count);

}  // namespace gcme
