// Integrators (velocity Verlet, BAOAB Langevin), output conversion and the
// fixed-order final reductions.
//
// Langevin noise: Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11) with
// counter (step, bead id, replica, 0) and key (seed, 0x67636d65); uniforms
// ((x >> 11) + 1/2) 2^-53; Box-Muller on (u0, u1) and (u2, u3).  Keying by
// the original bead id makes the noise independent of the cell ordering.
#include "gcme_internal.h"

namespace gcme {

namespace {

__device__ inline void philox4x64_10(unsigned long long x[4], unsigned long long k0, unsigned long long k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += 0x9E3779B97F4A7C15ULL;
      k1 += 0xBB67AE8584CAA73BULL;
    }
    const unsigned long long m0 = 0xD2E7470EE14C6C93ULL, m1 = 0xCA5A826395121157ULL;
    unsigned long long hi0 = __umul64hi(m0, x[0]), lo0 = m0 * x[0];
    unsigned long long hi1 = __umul64hi(m1, x[2]), lo1 = m1 * x[2];
    unsigned long long y0 = hi1 ^ x[1] ^ k0, y2 = hi0 ^ x[3] ^ k1;
    x[0] = y0;
    x[1] = lo1;
    x[2] = y2;
    x[3] = lo0;
  }
}

__device__ inline void gauss3(unsigned long long seed, unsigned long long step, unsigned long long id,
                              unsigned long long rep, double g[3]) {
  unsigned long long x[4] = {step, id, rep, 0ULL};
  philox4x64_10(x, seed, 0x67636d65ULL);
  double u[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) u[k] = ((double)(x[k] >> 11) + 0.5) * (1.0 / 9007199254740992.0);
  double r0 = sqrt(-2.0 * log(u[0])), r1 = sqrt(-2.0 * log(u[2]));
  double s1, c1, s3, c3;
  sincospi(2.0 * u[1], &s1, &c1);
  sincospi(2.0 * u[3], &s3, &c3);
  g[0] = r0 * c1;
  g[1] = r0 * s1;
  g[2] = r1 * c3;
}

__device__ inline uint32_t drift(uint32_t u, double dx, double L) {
  long long du = llrint(dx / L * 4294967296.0);
  return u + (uint32_t)du;
}

// First half of a step for one bead, from velocity v, position u and force
// f (already in force units): kick, then drift (velocity Verlet) or drift,
// Ornstein-Uhlenbeck noise, drift (BAOAB), with the noise of `step`.  A type
// of infinite mass (inverse mass 0, no noise amplitude) is held at rest.
__device__ inline void first_half(const IntLaunch& a, const RepDesc& R, int r, int t, unsigned long long step,
                                  int id, const double f[3], double v[3], uint32_t u[3]) {
  const double im = a.inv_mass[r * MAXT + t];
  const double dt = a.dt[r];
#pragma unroll
  for (int k = 0; k < 3; ++k) v[k] = im == 0.0 ? 0.0 : v[k] + 0.5 * dt * f[k] * im;
  if (a.langevin[r]) {
    double g[3];
    gauss3(a.seed, step, (unsigned long long)id, (unsigned long long)r, g);
    const double c1 = a.c1[r], c2 = a.c2s[r * MAXT + t];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      u[k] = drift(u[k], 0.5 * dt * v[k], R.L[k]);
      v[k] = c1 * v[k] + c2 * g[k];
      u[k] = drift(u[k], 0.5 * dt * v[k], R.L[k]);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) u[k] = drift(u[k], dt * v[k], R.L[k]);
  }
}

template <bool BIN>
__global__ void k_int_first(IntLaunch a, StateView A, long long* F0, long long* F1, long long* F2, CellView c,
                            int N) {
  wave_stamp(a.stamps, 0);
  const int s0 = blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = s0 < N;
  if (!BIN && !active) return;
  const int s = active ? s0 : 0;  // inactive lanes of the last wavefront only take part in the binning
  const uint32_t prm = A.param[s];
  const int r = param_rep(prm), t = param_type(prm);
  const RepDesc& R = a.rep[r];
  long long* Fk[3] = {F0, F1, F2};
  double f[3], v[3];
  uint32_t u[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    f[k] = (double)Fk[k][s] * a.fscale_inv;
    if (active) Fk[k][s] = 0;
    v[k] = A.vel[k][s];
    u[k] = A.pos[k][s];
  }
  const int id = A.id[s];
  first_half(a, R, r, t, *a.step, id, f, v, u);
  if (active) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      A.pos[k][s] = u[k];
      A.vel[k][s] = v[k];
    }
  }
  if (BIN) bin_bead(c, R, u[0], u[1], u[2], prm, s, id, active);
  wave_stamp(a.stamps, 1);
}

// The second half kick of the step just completed (as k_int_last, on the
// sorted copy B), then the first half of the next step (as k_int_first) and
// its binning, written to A.  The step counter already names the next step:
// the scan of the step's sort advanced it (one thread, where a count of the
// finished blocks would take one same-address atomic per block: 340 us per
// step at N = 2,097,152).
__global__ __launch_bounds__(BEAD_THREADS) void k_int_between(IntLaunch a, StateView B, StateView A, long long* F0,
                                                     long long* F1, long long* F2, CellView c, int N) {
  wave_stamp(a.stamps, 0);
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned long long step = *a.step;
  const bool active = s < N;
  int cid = 0;
  uint32_t prm = 0;
  if (active) {
    prm = B.param[s];
    const int r = param_rep(prm), t = param_type(prm);
    const RepDesc& R = a.rep[r];
    const double im = a.inv_mass[r * MAXT + t];
    const double dt = a.dt[r];
    long long* Fk[3] = {F0, F1, F2};
    double f[3], v[3];
    uint32_t u[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const long long fi = Fk[k][s];
      v[k] = B.vel[k][s] + 0.5 * dt * (double)fi * a.fscale_inv * im;
      f[k] = (double)fi * a.fscale_inv;
      Fk[k][s] = 0;
      u[k] = B.pos[k][s];
    }
    const int id = B.id[s];
    first_half(a, R, r, t, step, id, f, v, u);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      A.pos[k][s] = u[k];
      A.vel[k][s] = v[k];
    }
    A.param[s] = prm;
    A.id[s] = id;
    cid = cell_of(R, u[0], u[1], u[2]);
    c.cell[s] = cid;
    if (c.slot_a) c.slot_a[id] = s;
  }
  // the binning's counts, one atomic per run of equal cells in the wavefront
  count_bead(c, cid, prm, s, active);
  wave_stamp(a.stamps, 1);
}

__device__ inline double block_sum(double v, double* sh) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wid] = v;
  __syncthreads();
  double t = 0;
  if (threadIdx.x == 0) t = ((sh[0] + sh[1]) + (sh[2] + sh[3]));
  return t;
}

// Second half kick on the sorted copy B, written back to A (so the state is
// left in the order the forces are indexed in).  One tile per block.
template <bool KIN>
__global__ __launch_bounds__(256) void k_int_last(IntLaunch a, StateView B, StateView A, long long* F0,
                                                  long long* F1, long long* F2) {
  wave_stamp(a.stamps, 0);
  __shared__ double sh[4];
  const Tile tile = a.tiles[blockIdx.x];
  const bool active = (int)threadIdx.x < tile.count;
  const int n = tile.first + (active ? (int)threadIdx.x : 0);
  double ke = 0;
  if (active) {
    const uint32_t prm = B.param[n];
    const int r = tile.rep, t = param_type(prm);
    const double im = a.inv_mass[r * MAXT + t];
    const double dt = a.dt[r];
    long long* Fk[3] = {F0, F1, F2};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double v = B.vel[k][n] + 0.5 * dt * (double)Fk[k][n] * a.fscale_inv * im;
      A.vel[k][n] = v;
      A.pos[k][n] = B.pos[k][n];
      ke += im == 0.0 ? 0.0 : 0.5 * v * v / im;
    }
    A.param[n] = prm;
    A.id[n] = B.id[n];
  }
  if (KIN) {
    double t = block_sum(ke, sh);
    if (threadIdx.x == 0) {
      a.part[(size_t)blockIdx.x * PART_W + 0] = t;
      for (int k = 1; k < PART_W; ++k) a.part[(size_t)blockIdx.x * PART_W + k] = 0.0;
    }
  }
  wave_stamp(a.stamps, 1);
}

__global__ void k_gather_vjp(StateView B, const double* v, double* vs, int N) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int id = B.id[n];
#pragma unroll
  for (int k = 0; k < 3; ++k) vs[(size_t)k * N + n] = v[(size_t)k * N + id];
}

__global__ void k_bead_adj_out(StateView B, const double* dg, const double* dq, const double* self_a,
                               double* out_s, double* out_a, int N) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  const int id = B.id[n];
  const uint32_t prm = B.param[n];
  const int z = param_z(prm);
  if (out_s) out_s[id] = dg[n];
  if (out_a) out_a[id] = dq[n] + self_a[param_rep(prm) * MAXT + param_type(prm)] * (double)(z * z);
}

__global__ void k_state_out(StateView A, const RepDesc* rep, double* pos, double* vel, long long ld, int N) {
  int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  int id = A.id[s];
  const RepDesc& R = rep[param_rep(A.param[s])];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (pos) pos[k * ld + id] = (double)A.pos[k][s] * R.scaled[k];
    if (vel) vel[k * ld + id] = A.vel[k][s];
  }
}

// The same in two passes, for large systems: the state's order and the
// original one are unrelated, so every store of k_state_out is a memory line
// of its own, six per bead.  First each bead's position and velocity go to its
// place as one record each (about two lines), then the records are read and
// the arrays written in order.  N = 2,097,152: 139 us against 208 us in one pass;
// below a quarter of a million beads one launch is as fast.
constexpr int STATE_RECORD_BEADS = 262144;

__global__ void k_state_records(StateView A, uint4* pr, double* vr, int N) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= N) return;
  const int id = A.id[s];
  if (pr) pr[id] = make_uint4(A.pos[0][s], A.pos[1][s], A.pos[2][s], A.param[s]);
  if (vr) {
#pragma unroll
    for (int k = 0; k < 3; ++k) vr[3 * (size_t)id + k] = A.vel[k][s];
  }
}

__global__ void k_state_unpack(const RepDesc* rep, const uint4* pr, const double* vr, double* pos, double* vel, int N) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= N) return;
  if (pos) {
    const uint4 p = pr[n];
    const RepDesc& R = rep[param_rep(p.w)];
    pos[n] = (double)p.x * R.scaled[0];
    pos[(size_t)N + n] = (double)p.y * R.scaled[1];
    pos[2 * (size_t)N + n] = (double)p.z * R.scaled[2];
  }
  if (vel) {
#pragma unroll
    for (int k = 0; k < 3; ++k) vel[k * (size_t)N + n] = vr[3 * (size_t)n + k];
  }
}

// One thread's share of a column of the rows [lo, hi) (W doubles each): rows
// lo + first, lo + first + step, ..., four loads in flight, in a fixed order.
template <int W>
__device__ inline double row_sum(const double* part, int lo, int hi, int first, int step, int col) {
  double v[4] = {0, 0, 0, 0};
  int r = lo + first;
  for (; r + 3 * step < hi; r += 4 * step) {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] += part[(size_t)(r + u * step) * W + col];
  }
  for (int u = 0; r < hi; r += step, ++u) v[u] += part[(size_t)r * W + col];
  return (v[0] + v[1]) + (v[2] + v[3]);
}

// The energy terms, virial and parameter derivatives of the replicas: a.nb
// blocks per replica.  Eight threads take the eight columns of a row (one 64-
// byte line), a block 32 rows at a time, every slot one after another with no
// barrier between them; the blocks' sums meet in fin_part, which the last
// block of a replica to finish adds up in block order, so the result does not
// depend on which one that is.  (One block with a block sum per slot and
// column took 20 us at N = 300 and 74 us for the 12,500 rows of N = 200,000;
// now 4 and 7 us.)
__device__ inline void finalize_block(const FinalLaunch& a, int bid) {
  __shared__ double sh[4][FIN_VALUES];
  __shared__ double res[FIN_VALUES];
  __shared__ int last;
  const int r = bid / a.nb, b = bid % a.nb;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 7, first = b * 32 + (threadIdx.x >> 3), step = 32 * a.nb;
  const bool adj = a.dE_dA || a.dE_dsigma || a.dE_da;
  constexpr int W = MAXT * MAXT + 2 * MAXT;
  static_assert(W == 24 && PART_W == 8 && FIN_VALUES == 8 * (N_SLOTS + 4), "eight columns per group");
  double v[N_SLOTS + 4];
#pragma unroll
  for (int sl = 0; sl < N_SLOTS; ++sl) {
    v[sl] = 0;
    if (a.part[sl] && (sl != SLOT_KIN || a.have_kin) && col < 7)
      v[sl] = row_sum<PART_W>(a.part[sl], a.slot_off[sl][r], a.slot_off[sl][r + 1], first, step, col);
  }
  // parameter derivatives: columns 0-15 type-pair energies, 16-19 sigma
  // (excluded volume), 20-23 a (charged pairs)
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int q = g < 3 ? 0 : 1, c = (g < 3 ? 8 * g : 16) + col;
    v[N_SLOTS + g] = 0;
    if (adj && a.adj_part[q] && (g < 2 || (g == 2 ? col < MAXT : col >= MAXT)))
      v[N_SLOTS + g] = row_sum<W>(a.adj_part[q], a.adj_off[q][r], a.adj_off[q][r + 1], first, step, c);
  }
#pragma unroll
  for (int k = 0; k < N_SLOTS + 4; ++k) {
    double t = v[k];
    t += __shfl_xor(t, 8, 64);
    t += __shfl_xor(t, 16, 64);
    t += __shfl_xor(t, 32, 64);
    if (lane < 8) sh[wave][8 * k + col] = t;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < FIN_VALUES; k += 256) {
    res[k] = (sh[0][k] + sh[1][k]) + (sh[2][k] + sh[3][k]);
    if (a.nb > 1) a.fin_part[(size_t)bid * FIN_VALUES + k] = res[k];
  }
  if (a.nb > 1) {
    __threadfence();  // this block's sums before its count
    __syncthreads();
    if (threadIdx.x == 0)
      last = __hip_atomic_fetch_add(&a.fin_count[r], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == a.nb - 1;
    __syncthreads();
    if (!last) return;
    __threadfence();  // every block's sums after the count
    for (int k = threadIdx.x; k < FIN_VALUES; k += 256)
      res[k] = row_sum<FIN_VALUES>(a.fin_part, r * a.nb, (r + 1) * a.nb, 0, 1, k);
    if (threadIdx.x == 0) a.fin_count[r] = 0;  // for the next launch
  }
  __syncthreads();
  const double(*slot)[8] = reinterpret_cast<const double(*)[8]>(res);
  if (threadIdx.x == 0) {
    const double ec = a.consts[2 * r], es = a.consts[2 * r + 1];
    if (a.energy) {
      double* E = a.energy + (size_t)r * N_TERMS;
      const double e0 = slot[SLOT_GCM][0], e1 = slot[SLOT_REAL][0];
      const double e2 = slot[SLOT_RECIP][0] + slot[SLOT_EWALD][0];  // a replica has one of the two
      const double e7 = slot[SLOT_SLAB][0], e8 = slot[SLOT_BOND][0];
      E[0] = e0;
      E[1] = e1;
      E[2] = e2;
      E[3] = ec;
      E[4] = es;
      E[5] = (((e0 + e1) + (e2 + ec)) + es) + (e7 + e8);
      E[6] = a.have_kin ? slot[SLOT_KIN][0] : 0.0;
      E[7] = e7;
      E[8] = e8;
    }
  }
  if (a.virial && threadIdx.x >= 64 && threadIdx.x < 70) {
    const int k = (int)threadIdx.x - 64;
    a.virial[(size_t)r * 6 + k] =
        ((slot[SLOT_GCM][1 + k] + slot[SLOT_REAL][1 + k]) + (slot[SLOT_RECIP][1 + k] + slot[SLOT_EWALD][1 + k])) +
        (slot[SLOT_SLAB][1 + k] + slot[SLOT_BOND][1 + k]);
  }
  if (adj && threadIdx.x < MAXT * MAXT) {
    const double* ett = res + 8 * N_SLOTS;
    const double* dsg = ett + MAXT * MAXT;
    const double* dea = ett + MAXT * MAXT + 8 + MAXT;
    const int q = threadIdx.x, t = q / MAXT, u = q % MAXT;
    // unordered type-pair energy: both visiting orders
    const double E = t == u ? ett[q] : ett[t * MAXT + u] + ett[u * MAXT + t];
    const double A = a.Avals[(size_t)r * MAXT * MAXT + q];
    if (a.dE_dA) a.dE_dA[(size_t)r * MAXT * MAXT + q] = A != 0.0 ? a.adj_scale * E / A : 0.0;
    if (u == 0) {
      if (a.dE_dsigma) a.dE_dsigma[(size_t)r * MAXT + t] = a.adj_scale * dsg[t];
      if (a.dE_da) a.dE_da[(size_t)r * MAXT + t] = a.adj_scale * dea[t] + (a.vjp ? 0.0 : a.dself[(size_t)r * MAXT + t]);
    }
  }
}

// The first blocks take the final sums, the others 256 beads each.
__global__ __launch_bounds__(256) void k_outputs(OutLaunch a) {
  const int nfin = a.fin.nrep * a.fin.nb;
  if ((int)blockIdx.x < nfin) {
    finalize_block(a.fin, blockIdx.x);
    return;
  }
  const int n = ((int)blockIdx.x - nfin) * 256 + (int)threadIdx.x;
  if (n >= a.N) return;
  const int id = a.B.id[n];
  const size_t N = (size_t)a.N;
  if (a.force) {
#pragma unroll
    for (int k = 0; k < 3; ++k) a.force[k * N + id] = (double)a.F[k * N + n] * a.fscale_inv;
  }
  if (a.commit) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      a.A.pos[k][n] = a.B.pos[k][n];
      a.A.vel[k][n] = a.B.vel[k][n];
    }
    a.A.param[n] = a.B.param[n];
    a.A.id[n] = id;
  }
}

inline int nblk(long long n, int t) { return (int)((n + t - 1) / t); }

}  // namespace

void launch_int_first(hipStream_t s, const IntLaunch& a, StateView A, long long* const F[3], const CellView* bin) {
  if (bin)
    hipLaunchKernelGGL(k_int_first<true>, dim3(nblk(a.nbeads, BEAD_THREADS)), dim3(BEAD_THREADS), 0, s, a, A, F[0], F[1], F[2], *bin,
                       a.nbeads);
  else
    hipLaunchKernelGGL(k_int_first<false>, dim3(nblk(a.nbeads, BEAD_THREADS)), dim3(BEAD_THREADS), 0, s, a, A, F[0], F[1], F[2],
                       CellView{}, a.nbeads);
}

void launch_int_between(hipStream_t s, const IntLaunch& a, StateView B, StateView A, long long* const F[3],
                        const CellView& bin) {
  hipLaunchKernelGGL(k_int_between, dim3(nblk(a.nbeads, BEAD_THREADS)), dim3(BEAD_THREADS), 0, s, a, B, A, F[0], F[1], F[2], bin,
                     a.nbeads);
}

void launch_int_last(hipStream_t s, const IntLaunch& a, StateView B, StateView A, long long* const F[3], bool kin) {
  if (kin)
    hipLaunchKernelGGL(k_int_last<true>, dim3(a.ntiles), dim3(256), 0, s, a, B, A, F[0], F[1], F[2]);
  else
    hipLaunchKernelGGL(k_int_last<false>, dim3(a.ntiles), dim3(256), 0, s, a, B, A, F[0], F[1], F[2]);
}

void launch_gather_vjp(hipStream_t s, StateView B, const double* v, double* vs, int N) {
  hipLaunchKernelGGL(k_gather_vjp, dim3(nblk(N, 256)), dim3(256), 0, s, B, v, vs, N);
}

void launch_bead_adj_out(hipStream_t s, StateView B, const double* dg, const double* dq, const double* self_a,
                         double* out_sigma, double* out_a, int N) {
  hipLaunchKernelGGL(k_bead_adj_out, dim3(nblk(N, 256)), dim3(256), 0, s, B, dg, dq, self_a, out_sigma, out_a, N);
}

void launch_state_out(hipStream_t s, StateView A, const RepDesc* rep, double* pos, double* vel, uint4* pr, double* vr,
                      int N) {
  if (N >= STATE_RECORD_BEADS) {
    hipLaunchKernelGGL(k_state_records, dim3(nblk(N, 256)), dim3(256), 0, s, A, pos ? pr : nullptr, vel ? vr : nullptr, N);
    hipLaunchKernelGGL(k_state_unpack, dim3(nblk(N, 256)), dim3(256), 0, s, rep, pr, vr, pos, vel, N);
    return;
  }
  hipLaunchKernelGGL(k_state_out, dim3(nblk(N, 256)), dim3(256), 0, s, A, rep, pos, vel, N, N);
}

void launch_outputs(hipStream_t s, const OutLaunch& a) {
  const int blocks = a.fin.nrep * a.fin.nb + (a.force || a.commit ? nblk(a.N, 256) : 0);
  if (blocks > 0) hipLaunchKernelGGL(k_outputs, dim3(blocks), dim3(256), 0, s, a);
}

}  // namespace gcme
