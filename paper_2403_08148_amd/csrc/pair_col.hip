// Column-cluster pair kernels (tuning half_pairs).
#include "pair_kernels.h"

namespace gcme {

namespace {

// ---------------------------------------------------------------------------
// Half-shell excluded-volume pairs
// ---------------------------------------------------------------------------
//
// One wavefront per column cluster (at most CI consecutive sorted beads of
// one cell column).  Its beads are wave-uniform; each lane takes one
// candidate of the owned columns (for_candidates<HALF>) and evaluates it
// against every cluster bead, so a pair is evaluated once and both beads
// get its force: the cluster beads' sums stay in registers until the end
// (one fixed-order lane reduction), a candidate's goes to the fixed-point
// accumulator after its chunk.  Integer accumulation keeps reruns
// bit-identical whatever the order of the atomics.

// Fixed point of a single-precision force component at `scale`, rounded to
// the nearest integer (ties to even) as llrint would: the fused multiply-add
// with 1.5 2^52 leaves the integer in the low mantissa bits.  Needs
// |f| scale < 2^51 (|f| < lim); beyond, or not finite, the status bit is set
// and 0 returned.
__device__ inline long long fixed_of(float f, double scale, float lim, unsigned int* status) {
  if (!(fabsf(f) < lim)) {
    atomicOr(status, (unsigned)STATUS_FORCE_OVERFLOW);
    return 0;
  }
  return __double_as_longlong(fma((double)f, scale, 6755399441055744.0)) - 0x4338000000000000LL;
}
__device__ inline long long fixed_of(double f, double scale, float, unsigned int* status) {
  return to_fixed(f, scale, status);
}

// a + b after exchanging the upper 32 lanes of a with the lower 32 of b
// (lanes 0-31: the sum of a over lanes l and l + 32; lanes 32-63: of b).
__device__ inline float swap32_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The same within each half for rows of 16 (rows 0, 2: a; rows 1, 3: b).
__device__ inline float swap16_sum(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ inline double swap32_sum(double a, double b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  const double p = __longlong_as_double(((long long)hi[0] << 32) | lo[0]);
  const double q = __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
  return p + q;
}
__device__ inline double swap16_sum(double a, double b) {
  const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  const double p = __longlong_as_double(((long long)hi[0] << 32) | lo[0]);
  const double q = __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
  return p + q;
}

// Sums of V per-lane values over the wavefront, in a fixed order: lanes of
// row r (lanes 16 r .. 16 r + 15) end with u[m] = the total of
// v[r V/4 + m], m < V/4.
template <typename T, int V>
__device__ inline void reduce_rows(const T (&v)[V], T (&u)[V / 4]) {
  static_assert(V % 4 == 0, "four rows");
  T w[V / 2];
#pragma unroll
  for (int m = 0; m < V / 2; ++m) w[m] = swap32_sum(v[m], v[m + V / 2]);
#pragma unroll
  for (int m = 0; m < V / 4; ++m) {
    T t = swap16_sum(w[m], w[m + V / 4]);
    t += dpp_f<DPP_ROW_ROR8>(t);
    t += dpp_f<DPP_ROW_HALF_MIRROR>(t);
    t += dpp_f<DPP_XOR1>(t);
    t += dpp_f<DPP_XOR2>(t);
    u[m] = t;
  }
}

// Pair tables of the half-shell kernels: excluded volume (-bl, fC) and C per
// type pair, or the real-space bracket's coefficients.
template <typename T, bool ELEC>
struct HalfTab {
  ExpPar<T> p[ELEC ? 1 : MAXT * MAXT];
  T c[ELEC ? 1 : MAXT * MAXT];
  ElecPar<T> e[ELEC ? MAXT * MAXT : 1];
};

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>) in
// order: a loop unrolled whatever the size of its body, so that register
// arrays indexed by the counter stay in registers.
template <class F, int... I>
__device__ __attribute__((always_inline)) inline void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// A cluster bead as the half-shell kernels read it.
template <typename T>
struct IBead {
  T x, y, z;  // relative to the centre
  int trow;   // type x MAXT: its row of the pair tables
  T q;        // charge number
};

// ELEC: the charged beads (their compacted records and cell list), the
// real-space bracket of eq. ewald in place of eq. u_ex; forces go to the
// sorted index of each charged bead.
//
// Per cluster: the owned column runs (column_segments<HALF>) are read 64
// consecutive beads at a time, one per lane; a bead within the list cutoff
// of the cluster's bounding box joins a 128-entry LDS ring of pending
// candidates, and every 64 pending candidates are evaluated at once, a lane
// per candidate against every cluster bead.  In the cluster's frame (the centre's;
// every column cluster in bulk) the ring holds the candidate's position
// relative to the centre, so a pair costs a subtraction per axis; otherwise the
// fixed-point record, and each pair takes its own minimum image.
//
// HALF false: every column within reach (both ends of each pair; no
// candidate atomics, each pair's energy and virial halved), the same ring
// and evaluation otherwise.
template <typename T, int CI, bool EV, bool ELEC, bool HALF>
__global__ __launch_bounds__(NL_WAVES * 64) void k_pair_col(PairLaunch a) {
  constexpr int NV = 3 * CI;
  __shared__ double red[NL_WAVES];
  __shared__ HalfTab<T, ELEC> S;
  __shared__ int2 s_seg[NL_WAVES][NL_SEG];
  __shared__ uint4 s_ring[NL_WAVES][RING];
  __shared__ int s_rj[NL_WAVES][RING];  // candidate index
  __shared__ int s_rf[NL_WAVES][RING];  // its force slot (sorted bead index)
  __shared__ int s_cand[NL_WAVES][NL_CAND];
  __shared__ IBead<T> s_ib[NL_WAVES][ELEC ? 1 : CI];
  wave_stamp(a.stamps, 0);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int item = xcd_item(blockIdx.x, a.ntiles);
  const Tile tl = a.tiles[item];
  const RepDesc& R = a.rep[tl.rep];
  const uint4* __restrict__ pk = a.pk;
  const int slot = tl.first + wave;
  // tl.bead0: the replica's first cluster slot
  const bool active = wave < tl.count && slot - tl.bead0 < a.hncl[tl.rep];
  int2 info = make_int2(0, 1);
  if (active) info = a.cl[slot];
  const int first = info.x, ni = info.y;
  uint4 me = make_uint4(0u, 0u, 0u, 0u);
  if (active) me = pk[first + (lane % CI < ni ? lane % CI : 0)];
  if (threadIdx.x < MAXT * MAXT) {
    const size_t tb = (size_t)tl.rep * MAXT * MAXT + threadIdx.x;
    if (ELEC) {
      S.e[threadIdx.x] = reinterpret_cast<const ElecPar<T>*>(a.elec)[tb];
    } else {
      const GcmPar<T> g = reinterpret_cast<const GcmPar<T>*>(a.gcm)[tb];
      S.p[threadIdx.x] = ExpPar<T>{-g.bl, g.fC};
      S.c[threadIdx.x] = g.C;
    }
  }
  __syncthreads();
  double e = 0, w0 = 0, w1 = 0, w2 = 0, w3 = 0, w4 = 0, w5 = 0;
  if (active) {
    ClusterBox K;
    float rme[3], nn;
    make_box<CI>(K, me, R, rme, nn);
    // the beads' fixed-point positions, wave-uniform (slots beyond ni repeat bead 0)
    uint32_t ux[CI], uy[CI], uz[CI];
#pragma unroll
    for (int k = 0; k < CI; ++k) {
      ux[k] = read_lane(me.x, k);
      uy[k] = read_lane(me.y, k);
      uz[k] = read_lane(me.z, k);
    }
    const bool frame = in_frame(K, R);
    const T sx = (T)R.scaled[0], sy = (T)R.scaled[1], sz = (T)R.scaled[2];
    const T rc2 = (T)R.rc2;
    // the real-space bracket's constants (as the cluster kernels take them)
    const T beta = (T)R.beta, beta2 = (T)(R.beta * R.beta), lB = (T)R.lB;
    T cexpb, tsb;
    if constexpr (std::is_same<T, float>::value) {
      const float bf = (float)R.beta;
      cexpb = -(bf * bf) * 1.44269504088896341f;
      tsb = 1.12837916709551257f * bf;
    } else {
      cexpb = -R.beta * R.beta * 1.4426950408889634;
      tsb = 1.1283791670955126 * R.beta;
    }
    // the cluster beads, wave-uniform: positions relative to the centre, the
    // type row of the pair tables and the charge (slots beyond ni: far from
    // everything, so the unrolled pairs need no branch; the general path
    // masks them)
    // (excluded volume: in LDS, every lane reading the same entry, which
    // keeps the kernel within three wavefronts' registers per SIMD; the
    // charged pairs' branchy bracket keeps them in registers)
    IBead<T> ib[CI];
    IBead<T>* ibl = s_ib[wave];
#pragma unroll
    for (int k = 0; k < CI; ++k) {
      const uint32_t wk = read_lane(me.w, k);
      ib[k].x = k < ni ? (T)(int)(ux[k] - K.u0[0]) * sx : (T)1e18f;
      ib[k].y = k < ni ? (T)(int)(uy[k] - K.u0[1]) * sy : (T)1e18f;
      ib[k].z = k < ni ? (T)(int)(uz[k] - K.u0[2]) * sz : (T)1e18f;
      ib[k].trow = param_type(wk) * MAXT;
      ib[k].q = (T)param_z(wk);
      if (!ELEC && lane == k) ibl[k] = ib[k];
    }
    T fx[CI], fy[CI], fz[CI];
#pragma unroll
    for (int k = 0; k < CI; ++k) fx[k] = fy[k] = fz[k] = 0;
    const float lim = (float)(2251799813685248.0 / a.fscale);  // 2^51 / scale
    const bool rel = std::is_same<T, float>::value && frame;
    uint4* ring = s_ring[wave];
    int* rj = s_rj[wave];
    int* rf = s_rf[wave];
    // every slot of the ring is written before a drain can read it
    ring[lane] = ring[64 + lane] = make_uint4(0u, 0u, 0u, 0u);
    rj[lane] = rj[64 + lane] = -1;
    rf[lane] = rf[64 + lane] = 0;
    __builtin_amdgcn_wave_barrier();
    int head = 0, tail = 0;  // wave-uniform: candidates evaluated / appended
    // n <= 64 pending candidates from head, one per lane (head is a multiple
    // of 64 here: every drain but the last takes exactly 64).  FRAME: ring
    // positions relative to the centre; MASK: the drain holds cluster beads,
    // whose pairs with the cluster count only for k < j - first.
    auto drain = [&](int n) __attribute__((always_inline)) {
      const int q = (head & 64) + lane;
      const bool valid = lane < n;
      const uint4 rec = ring[q];
      const int j = valid ? rj[q] : -1;
      const int fj = rf[q];
      const unsigned jrel = j < 0 ? 0u : (unsigned)(j - first);
      const bool intra = __ballot(j >= 0 && jrel < (unsigned)ni) != 0ull;
      auto eval = [&](auto frame_tag, auto mask_tag) __attribute__((always_inline)) {
        constexpr bool FR = decltype(frame_tag)::value, MASK = decltype(mask_tag)::value;
        T Dx = 0, Dy = 0, Dz = 0;
        if (FR) {
          if (std::is_same<T, float>::value) {
            Dx = (T)__uint_as_float(rec.x);
            Dy = (T)__uint_as_float(rec.y);
            Dz = (T)__uint_as_float(rec.z);
          } else {
            Dx = (T)(int)(rec.x - K.u0[0]) * sx;
            Dy = (T)(int)(rec.y - K.u0[1]) * sy;
            Dz = (T)(int)(rec.z - K.u0[2]) * sz;
          }
          if (!valid) Dx = Dy = Dz = (T)-1e18f;  // beyond the cutoff of every bead
        }
        const int tj = param_type(rec.w);
        const T qj = (T)param_z(rec.w);
        T gx = 0, gy = 0, gz = 0;
        bool any = false;
        static_for<CI>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          const IBead<T> bi = ELEC ? ib[k] : ibl[k];
          T dx, dy, dz;
          if (FR) {
            dx = bi.x - Dx;
            dy = bi.y - Dy;
            dz = bi.z - Dz;
          } else {
            dx = (T)(int)(ux[k] - rec.x) * sx;
            dy = (T)(int)(uy[k] - rec.y) * sy;
            dz = (T)(int)(uz[k] - rec.z) * sz;
          }
          const T r2 = dx * dx + dy * dy + dz * dz;
          bool in = r2 < rc2;
          // half shell: within the cluster, pairs (k, j) with k < j; both
          // ends: every cluster bead but the candidate itself
          if (MASK || !FR) in = in && (HALF ? jrel > (unsigned)k : jrel != (unsigned)k);
          if (!FR) in = in && k < ni && valid;
          const int ix = bi.trow + tj;
          T fs = 0, en = 0;
          if (ELEC) {
            if (in) {
              T phi, g, ea;
              bracket(S.e[ix], r2, beta, beta2, cexpb, tsb, phi, g, ea);
              const T c = lB * (bi.q * qj);
              fs = c * g;
              en = c * phi;
            }
          } else {
            const ExpPar<T> hp = S.p[ix];
            const T ex = gexp2(in ? hp.nb * r2 : -(T)INFINITY);
            fs = hp.fc * ex;
            en = EV ? S.c[ix] * ex : (T)0;
          }
          // the candidate's sum is kept with the cluster bead's sign and
          // negated once: two fused multiply-adds per axis
          fx[k] = fma(fs, dx, fx[k]);
          fy[k] = fma(fs, dy, fy[k]);
          fz[k] = fma(fs, dz, fz[k]);
          gx = fma(fs, dx, gx);
          gy = fma(fs, dy, gy);
          gz = fma(fs, dz, gz);
          any = any || in;
          if (EV) {
            const double fxd = (double)(fs * dx), fyd = (double)(fs * dy), fzd = (double)(fs * dz);
            e += (double)en;
            w0 += fxd * (double)dx;
            w1 += fyd * (double)dy;
            w2 += fzd * (double)dz;
            w3 += fxd * (double)dy;
            w4 += fxd * (double)dz;
            w5 += fyd * (double)dz;
          }
        });
        if (HALF && j >= 0 && any) {
          atomicAdd((unsigned long long*)&a.F[0][fj], (unsigned long long)fixed_of(-gx, a.fscale, lim, a.status));
          atomicAdd((unsigned long long*)&a.F[1][fj], (unsigned long long)fixed_of(-gy, a.fscale, lim, a.status));
          atomicAdd((unsigned long long*)&a.F[2][fj], (unsigned long long)fixed_of(-gz, a.fscale, lim, a.status));
        }
      };
      using TT = std::true_type;
      using FF = std::false_type;
      if (!frame)
        eval(FF{}, TT{});
      else if (intra)
        eval(TT{}, TT{});
      else
        eval(TT{}, FF{});
      head += n;
    };
    // the list cutoff around the cluster's bounding box (relative to the centre)
    const float rcl2 = K.rcl * K.rcl;
    int* cand = s_cand[wave];
    // the candidates cand[0, total), 64 per chunk (one per lane): those within
    // the list cutoff of the box join the ring
    auto filter = [&](int total) __attribute__((always_inline)) {
      // the records of FB chunks are requested together (one memory latency
      // for all of them), and the charged beads' sorted indices with them
      constexpr int FB = 4;
      for (int p0 = 0; p0 < total; p0 += 64 * FB) {
        int jj[FB], ff[FB];
        uint4 pp[FB];
#pragma unroll
        for (int u = 0; u < FB; ++u) {
          const int q = p0 + 64 * u + lane;
          jj[u] = q < total ? cand[q] : -1;
        }
#pragma unroll
        for (int u = 0; u < FB; ++u) {
          pp[u] = pk[jj[u] < 0 ? first : jj[u]];
          ff[u] = ELEC ? a.qidx[jj[u] < 0 ? first : jj[u]] : jj[u];
        }
#pragma unroll
        for (int u = 0; u < FB; ++u) {
          if (p0 + 64 * u >= total) break;
          const int j = jj[u];
          const bool valid = j >= 0;
          const uint4 pj = pp[u];
          bool hit;
          uint4 rec = pj;
          if (frame) {
            const float Dx = (float)(int)(pj.x - K.u0[0]) * R.scalef[0];
            const float Dy = (float)(int)(pj.y - K.u0[1]) * R.scalef[1];
            const float Dz = (float)(int)(pj.z - K.u0[2]) * R.scalef[2];
            const float bx = fmaxf(0.f, fmaxf(K.lo[0] - Dx, Dx - K.hi[0]));
            const float by = fmaxf(0.f, fmaxf(K.lo[1] - Dy, Dy - K.hi[1]));
            const float bz = fmaxf(0.f, fmaxf(K.lo[2] - Dz, Dz - K.hi[2]));
            hit = valid && bx * bx + by * by + bz * bz < rcl2;
            if (rel) rec = make_uint4(__float_as_uint(Dx), __float_as_uint(Dy), __float_as_uint(Dz), pj.w);
          } else {
            hit = valid && near_exact<CI>(K, me, pj, R);
          }
          const unsigned long long m = __ballot(hit);
          if (hit) {
            const int q = (tail + lanes_below(m)) & (RING - 1);
            ring[q] = rec;
            rj[q] = j;
            rf[q] = ff[u];
          }
          tail += __popcll(m);
          __builtin_amdgcn_wave_barrier();
          if (tail - head >= 64) drain(64);
          __builtin_amdgcn_wave_barrier();
        }
      }
    };
    const int wx = (K.chi[0] - K.clo[0] + 8) / 8, wy = (K.chi[1] - K.clo[1] + 8) / 8;
    for (int blk = 0; blk < wx * wy; ++blk) {
      const int nseg = column_segments<HALF>(K, R, a.start, first, K.clo[0] + blk / wy * 8, K.clo[1] + blk % wy * 8,
                                             s_seg[wave]);
      // the owned column runs packed into the candidate buffer (filtered
      // whenever it fills), so that filter chunks are full
      int pos = 0;
      for (int sg = 0; sg < nseg; ++sg) {
        const int sb = __builtin_amdgcn_readfirstlane(s_seg[wave][sg].x);
        const int sl = __builtin_amdgcn_readfirstlane(s_seg[wave][sg].y);
        for (int off = 0; off < sl;) {
          const int take = min(sl - off, NL_CAND - pos);
          for (int t = lane; t < take; t += 64) cand[pos + t] = sb + off + t;
          pos += take;
          off += take;
          __builtin_amdgcn_wave_barrier();
          if (pos == NL_CAND) {
            filter(pos);
            pos = 0;
          }
        }
      }
      if (pos > 0) filter(pos);
    }
    if (tail > head) drain(tail - head);
    // the cluster beads' sums: row r of the wavefront holds beads
    // r CI/4 .. r CI/4 + CI/4 - 1 (CI/4 beads x 3 axes per row)
    T v[NV], u[NV / 4];
#pragma unroll
    for (int k = 0; k < CI; ++k) {
      v[3 * k] = fx[k];
      v[3 * k + 1] = fy[k];
      v[3 * k + 2] = fz[k];
    }
    reduce_rows<T, NV>(v, u);
    const int row = lane >> 4, t = lane & 15;
    if (t < CI / 4) {
      T f3[3] = {0, 0, 0};
#pragma unroll
      for (int b = 0; b < CI / 4; ++b)
        if (t == b) {
          f3[0] = u[3 * b];
          f3[1] = u[3 * b + 1];
          f3[2] = u[3 * b + 2];
        }
      const int k = row * (CI / 4) + t;
      if (k < ni) {
        const int fi = ELEC ? a.qidx[first + k] : first + k;
#pragma unroll
        for (int c = 0; c < 3; ++c)
          atomicAdd((unsigned long long*)&a.F[c][fi],
                    (unsigned long long)fixed_of(f3[c], a.fscale, lim, a.status));
      }
    }
  }
  if (EV) {
    // half shell: every pair once; both ends: twice, halved
    double v7[7] = {e, w0, w1, w2, w3, w4, w5};
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      const double t = block_sum(v7[k], red);
      if (threadIdx.x == 0) a.part[(size_t)item * PART_W + k] = HALF ? t : 0.5 * t;
    }
  }
  wave_stamp(a.stamps, 1);
}

template <bool ELEC>
void launch_col(hipStream_t s, const PairLaunch& a, bool fp64, bool ev, bool half) {
  if (a.ntiles <= 0) return;
  dim3 g(a.ntiles), b(NL_WAVES * 64);
#define GCME_COL(T, CI, H)                                                        \
  do {                                                                             \
    if (ev)                                                                        \
      hipLaunchKernelGGL((k_pair_col<T, CI, true, ELEC, H>), g, b, 0, s, a);      \
    else                                                                           \
      hipLaunchKernelGGL((k_pair_col<T, CI, false, ELEC, H>), g, b, 0, s, a);     \
  } while (0)
#define GCME_COL_H(T, CI) \
  do {                    \
    if (half)             \
      GCME_COL(T, CI, true); \
    else                  \
      GCME_COL(T, CI, false); \
  } while (0)
  if (fp64) {
    if (a.ci == 8)
      GCME_COL_H(double, 8);
    else
      GCME_COL_H(double, 4);
  } else {
    if (a.ci == 8)
      GCME_COL_H(float, 8);
    else
      GCME_COL_H(float, 4);
  }
#undef GCME_COL_H
#undef GCME_COL
}

}  // namespace

void launch_pair_gcm_col(hipStream_t s, const PairLaunch& a, bool fp64, bool ev, bool half) {
  launch_col<false>(s, a, fp64, ev, half);
}

void launch_pair_elec_col(hipStream_t s, const PairLaunch& a, bool fp64, bool ev, bool half) {
  launch_col<true>(s, a, fp64, ev, half);
}

}  // namespace gcme
