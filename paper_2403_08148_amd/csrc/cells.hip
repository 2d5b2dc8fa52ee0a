// Cell list: wrap into fixed point, bin, scan, scatter and a deterministic
// permutation of the state into (cell, previous order) order.
//
// Positions are stored as 32-bit fractions of the box edge (u = x/L * 2^32),
// so the minimum-image separation of two beads is the wrapped 32-bit
// difference, and drift never leaves the box.  Beads of one cell are kept in
// their previous relative order (a stable counting sort), which makes every
// later sum over neighbours run in the same order on every rerun.
#include "gcme_internal.h"

namespace gcme {

namespace {

// Positions to fixed point in the state's order, with the forces cleared;
// with BIN also the binning (as k_bin) of the new positions.
template <bool BIN>
__global__ void k_ingest(const double* __restrict__ pos, long long ld, int N, const RepDesc* __restrict__ rep,
                         StateView A, long long* F, CellView c) {
  const int s0 = blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = s0 < N;
  if (!BIN && !active) return;
  const int s = active ? s0 : 0;  // (inactive lanes only take part in the binning)
  const int id = A.id[s];
  const uint32_t prm = A.param[s];
  const RepDesc& R = rep[param_rep(prm)];
  uint32_t u[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double f = pos[k * ld + id] / R.L[k];
    f -= floor(f);
    // round to the nearest 2^-32 fraction; 2^32 wraps to 0
    u[k] = (uint32_t)(unsigned long long)llrint(f * 4294967296.0);
    if (active) {
      F[(long long)k * N + s] = 0;
      A.pos[k][s] = u[k];
    }
  }
  if (BIN) bin_bead(c, R, u[0], u[1], u[2], prm, s, id, active);
}

template <typename I>
__global__ void k_fill(I* p, I v, long long n) {
  long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  long long stride = (long long)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

// The binning alone, and (F given) the forces cleared.
__global__ void k_bin(StateView A, const RepDesc* __restrict__ rep, CellView c, long long* F, int N) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = s < N;
  const int si = active ? s : 0;
  const uint32_t p = A.param[si];
  const RepDesc& R = rep[param_rep(p)];
  const int id = c.slot_a ? A.id[si] : 0;
  if (F && active) F[s] = F[(long long)N + s] = F[2LL * N + s] = 0;
  bin_bead(c, R, A.pos[0][si], A.pos[1][si], A.pos[2][si], p, s, id, active);
}

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_PER_THREAD = 4;
constexpr int SCAN_BLOCK = SCAN_THREADS * SCAN_PER_THREAD;
// up to this many scan blocks, each adds up the block sums before it itself
// (at most 2 SCAN_SUMS_MAX ints per block) instead of a k_scan_top launch
constexpr int SCAN_SUMS_MAX = 1024;

// Inclusive scan of one int per thread over a block of NT threads (a
// multiple of 64, at most 1024); sh holds NT / 64 ints.
template <int NT>
__device__ inline int block_incl_scan(int v, int* sh) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(v, o, 64);
    if (lane >= o) v += t;
  }
  __syncthreads();
  if (lane == 63) sh[wid] = v;
  __syncthreads();
  int add = 0;
  for (int w = 0; w < wid; ++w) add += sh[w];
  return v + add;
}

// The whole scan in one launch, for grids of up to SELF_SCAN_MAX cells (those
// that no bucket sort takes: larger ones, or with images): block
// b of an array (blockIdx.y 0: all beads, 1: charged beads) adds up the counts
// of all cells before its own itself, four at a time and SELF_SCAN_UNROLL
// loads in flight, and then scans its own.  Produces start (exclusive) and,
// for all beads, the scatter cursor fill = start.  It is bound by the latency
// of a load, a block scan and a store: the one-block scan it replaces took
// 4.9 us for 32,768 beads (step 80 -> 78 us), and this 3.4.  The counts read
// twice grow with the square of the grid, which sets the limit: for 96,000
// beads between walls this takes 5.0 us, and 3.3 + 5.1 and a gap in the two
// launches below; for 256 replicas (above the limit) 12.2, and 4.6 + 5.1; for
// N = 2,097,152 49, and about 20.
constexpr int SELF_SCAN_THREADS = 1024;
constexpr int SELF_SCAN_BLOCK = 4 * SELF_SCAN_THREADS;
constexpr int SELF_SCAN_UNROLL = 8;
constexpr int SELF_SCAN_MAX = 131072;

__global__ __launch_bounds__(SELF_SCAN_THREADS) void k_scan_self(CellView c) {
  constexpr int NT = SELF_SCAN_THREADS, NW = NT / 64, U = SELF_SCAN_UNROLL;
  __shared__ int s_own[NW], s_off[NW];
  const int n = c.ncells;
  const int* __restrict__ cnt = blockIdx.y == 0 ? c.counts : c.qcounts;
  int* __restrict__ st = blockIdx.y == 0 ? c.start : c.qstart;
  if (c.step && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *c.step += 1ULL;
  const int base = blockIdx.x * SELF_SCAN_BLOCK + threadIdx.x * 4;
  int v[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = base + u < n ? cnt[base + u] : 0;
  // (the blocks before this one are whole)
  const int4* __restrict__ cnt4 = reinterpret_cast<const int4*>(cnt);
  const int nb4 = blockIdx.x * NT;
  int off = 0;
  for (int i0 = threadIdx.x; i0 < nb4; i0 += U * NT) {
    int4 w[U];
#pragma unroll
    for (int u = 0; u < U; ++u) w[u] = i0 + u * NT < nb4 ? cnt4[i0 + u * NT] : make_int4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) off += (w[u].x + w[u].y) + (w[u].z + w[u].w);
  }
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int own = (v[0] + v[1]) + (v[2] + v[3]);
  int inc = own;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(inc, o, 64);
    off += __shfl_xor(off, o, 64);
    if (lane >= o) inc += t;
  }
  if (lane == 63) {
    s_own[wid] = inc;
    s_off[wid] = off;
  }
  __syncthreads();
  int run = inc - own;
#pragma unroll
  for (int w = 0; w < NW; ++w) run += s_off[w] + (w < wid ? s_own[w] : 0);
  int r[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    r[u] = run;
    run += v[u];
  }
  if (base + 4 <= n) {
    const int4 o = make_int4(r[0], r[1], r[2], r[3]);
    *reinterpret_cast<int4*>(st + base) = o;
    if (blockIdx.y == 0) *reinterpret_cast<int4*>(c.fill + base) = o;
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (base + u < n) {
        st[base + u] = r[u];
        if (blockIdx.y == 0) c.fill[base + u] = r[u];
      }
  }
  // (run of the last thread: the total)
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == NT - 1) st[n] = run;
}

__global__ void k_scan_reduce(CellView c, int nb) {
  __shared__ int sh[8];
  int b = blockIdx.x;
  int base = b * SCAN_BLOCK + threadIdx.x * SCAN_PER_THREAD;
  int s0 = 0, s1 = 0;
#pragma unroll
  for (int k = 0; k < SCAN_PER_THREAD; ++k) {
    int i = base + k;
    if (i < c.ncells) {
      s0 += c.counts[i];
      s1 += c.qcounts[i];
    }
  }
  int t0 = block_incl_scan<SCAN_THREADS>(s0, sh);
  int t1 = block_incl_scan<SCAN_THREADS>(s1, sh);
  if (threadIdx.x == SCAN_THREADS - 1) {
    c.bsum[b] = t0;
    c.bsum[nb + b] = t1;
  }
}

// One block: exclusive scan of the block sums (both arrays).
__global__ void k_scan_top(CellView c, int nb) {
  __shared__ int sh[8];
  if (c.step && threadIdx.x == 0) *c.step += 1ULL;
  for (int arr = 0; arr < 2; ++arr) {
    int* bs = c.bsum + arr * nb;
    int carry = 0;
    for (int base = 0; base < nb; base += SCAN_THREADS) {
      int i = base + threadIdx.x;
      int v = i < nb ? bs[i] : 0;
      int inc = block_incl_scan<SCAN_THREADS>(v, sh);
      if (i < nb) bs[i] = carry + inc - v;
      __shared__ int tot;
      if (threadIdx.x == SCAN_THREADS - 1) tot = inc;
      __syncthreads();
      carry += tot;
      __syncthreads();
    }
    if (threadIdx.x == 0) {
      int* st = arr == 0 ? c.start : c.qstart;
      st[c.ncells] = carry;
    }
  }
}

// Last pass: each block's scan plus its offset.  With SUMS the block adds up
// the block sums before it itself (the raw ones of k_scan_reduce; cheap
// while there are few blocks), writes the totals from the last block and
// advances the step counter, so that k_scan_top is not launched; otherwise
// k_scan_top has turned the block sums into offsets.
template <bool SUMS>
__global__ void k_scan_apply(CellView c, int nb) {
  __shared__ int sh[8];
  __shared__ int off_sh[2];
  int b = blockIdx.x;
  int base = b * SCAN_BLOCK + threadIdx.x * SCAN_PER_THREAD;
  if constexpr (SUMS) {
    if (c.step && b == 0 && threadIdx.x == 0) *c.step += 1ULL;
    int s0 = 0, s1 = 0;
    for (int k = threadIdx.x; k < b; k += SCAN_THREADS) {
      s0 += c.bsum[k];
      s1 += c.bsum[nb + k];
    }
    const int t0 = block_incl_scan<SCAN_THREADS>(s0, sh);
    __syncthreads();
    const int t1 = block_incl_scan<SCAN_THREADS>(s1, sh);
    if (threadIdx.x == SCAN_THREADS - 1) {
      off_sh[0] = t0;
      off_sh[1] = t1;
    }
    __syncthreads();
  }
  for (int arr = 0; arr < 2; ++arr) {
    const int* cnt = arr == 0 ? c.counts : c.qcounts;
    int* st = arr == 0 ? c.start : c.qstart;
    int v[SCAN_PER_THREAD];
    int tot = 0;
#pragma unroll
    for (int k = 0; k < SCAN_PER_THREAD; ++k) {
      int i = base + k;
      v[k] = i < c.ncells ? cnt[i] : 0;
      tot += v[k];
    }
    int inc = block_incl_scan<SCAN_THREADS>(tot, sh);
    const int off = SUMS ? off_sh[arr] : c.bsum[arr * nb + b];
    if (SUMS && b == nb - 1 && threadIdx.x == SCAN_THREADS - 1) st[c.ncells] = off + inc;
    int run = off + inc - tot;
#pragma unroll
    for (int k = 0; k < SCAN_PER_THREAD; ++k) {
      int i = base + k;
      if (i < c.ncells) {
        st[i] = run;
        if (arr == 0) c.fill[i] = run;
      }
      run += v[k];
    }
    __syncthreads();
  }
}

__global__ void k_scatter(CellView c, int N) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const bool active = s < N;
  const int cid = active ? c.cell[s] : 0;
  // fill holds the cell's next free slot (initialised to start by the scan)
  const int slot = run_atomic_add(c.fill, cid, active);
  // (slots outside the population cannot come from consistent counts; they
  // are dropped rather than written out of bounds)
  if (active && (unsigned)slot < (unsigned)N) c.tmp[slot] = s;
}

// Position p of the scattered array holds bead s of cell c in arbitrary
// order; its final slot is start[c] + (number of beads of c with a smaller
// previous index).  Charged beads get the same rank among charged beads.
__global__ void k_permute(StateView A, StateView B, uint4* __restrict__ bpk, CellView c, ChargedView q, int N) {
  int p = blockIdx.x * blockDim.x + threadIdx.x;
  // the counts were consumed by the scan: clear them for the next binning
  for (int k = p; k < c.ncells; k += gridDim.x * blockDim.x) {
    c.counts[k] = 0;
    c.qcounts[k] = 0;
  }
  if (p >= N) return;
  const int s = c.tmp[p];
  // bead s's own data is requested as soon as s is known, beside its cell
  const int cid = c.cell[s];
  const uint32_t prm = A.param[s];
  const uint32_t px = A.pos[0][s], py = A.pos[1][s], pz = A.pos[2][s];
  const double vx = A.vel[0][s], vy = A.vel[1][s], vz = A.vel[2][s];
  const int id = A.id[s];
  // (clamped to the population, so inconsistent counts cannot send an
  // access out of bounds)
  const int lo = max(0, c.start[cid]), hi = min(N, c.start[cid + 1]);
  const bool charged = param_z(prm) != 0;
  // the rank among the cell's beads: their indices PB at a time, then the
  // parameters of those before s (charged beads only), each batch of loads
  // issued together
  constexpr int PB = 8;
  int rank = 0, qrank = 0;
  for (int t0 = lo; t0 < hi; t0 += PB) {
    int o[PB];
#pragma unroll
    for (int u = 0; u < PB; ++u) o[u] = t0 + u < hi ? c.tmp[t0 + u] : N;
    uint32_t po[PB];
#pragma unroll
    for (int u = 0; u < PB; ++u) po[u] = charged && o[u] < s ? A.param[o[u]] : 0u;
#pragma unroll
    for (int u = 0; u < PB; ++u) {
      rank += o[u] < s;
      qrank += param_z(po[u]) != 0;
    }
  }
  const int n = lo + rank;
  if (n >= N) return;
  B.pos[0][n] = px;
  B.pos[1][n] = py;
  B.pos[2][n] = pz;
  B.vel[0][n] = vx;
  B.vel[1][n] = vy;
  B.vel[2][n] = vz;
  B.param[n] = prm;
  B.id[n] = id;
  if (c.slot_of && (unsigned)id < (unsigned)N) c.slot_of[id] = n;
  const uint4 rec = make_uint4(px, py, pz, prm);
  bpk[n] = rec;
  if (charged) {
    const int qn = c.qstart[cid] + qrank;
    if ((unsigned)qn < (unsigned)c.qstart[c.ncells]) {
      q.pk[qn] = rec;
      q.idx[qn] = n;
    }
  }
}

// The whole sort (scan, scatter and permute) in one block, for small systems,
// where the three launches and the gaps between them take longer than the
// work.  With image charges, so that no buckets serve, three launches and this:
// 500 beads 53.4 and 47.1 us a step, 1,000 57.6 and 50.9 (in FP64 62.5 and
// 56.7), 3,000 58.4 and 57.2, 4,096 59.6 and 59.5, where the line lies.  The
// cell counts of all beads (low half) and of the charged
// ones (high half) are scanned together in LDS; the scattered bead indices
// stay there too (with a mark for the charged ones), so the ranks within a
// cell are LDS reads.
constexpr int SMALL_SORT_THREADS = 1024;
constexpr int SMALL_SORT_BPT = 4;  // beads per thread
constexpr int SMALL_SORT_BEADS = SMALL_SORT_THREADS * SMALL_SORT_BPT;
constexpr int SMALL_SORT_CELLS = 32768;  // 128 KiB of LDS beside the 16 KiB of bead indices

__global__ __launch_bounds__(SMALL_SORT_THREADS) void k_sort_small(StateView A, StateView B, uint4* __restrict__ bpk,
                                                                   CellView c, ChargedView q, int N) {
  static_assert(SMALL_SORT_BEADS < 65536, "counts are packed in halves of a word");
  constexpr int NT = SMALL_SORT_THREADS, BPT = SMALL_SORT_BPT;
  __shared__ int sh[NT / 64];
  extern __shared__ __align__(16) int buf[];  // ncells packed counts, then N bead indices
  const int nc = c.ncells;
  int* tmp = buf + nc;
  if (c.step && threadIdx.x == 0) *c.step += 1ULL;
  // this thread's beads: their cells and all that is moved, requested at once
  int cid[BPT], id[BPT];
  uint32_t px[BPT], py[BPT], pz[BPT], prm[BPT];
  double vx[BPT], vy[BPT], vz[BPT];
#pragma unroll
  for (int u = 0; u < BPT; ++u) {
    const int s = threadIdx.x + u * NT;
    const bool on = s < N;
    cid[u] = on ? c.cell[s] : 0;
    prm[u] = on ? A.param[s] : 0u;
    px[u] = on ? A.pos[0][s] : 0u;
    py[u] = on ? A.pos[1][s] : 0u;
    pz[u] = on ? A.pos[2][s] : 0u;
    vx[u] = on ? A.vel[0][s] : 0.0;
    vy[u] = on ? A.vel[1][s] : 0.0;
    vz[u] = on ? A.vel[2][s] : 0.0;
    id[u] = on ? A.id[s] : 0;
  }
  for (int i = threadIdx.x; i < nc; i += NT) {
    buf[i] = c.counts[i] | c.qcounts[i] << 16;
    c.counts[i] = c.qcounts[i] = 0;  // for the next binning
  }
  __syncthreads();
  const int per = (nc + NT - 1) / NT;
  const int lo = min(nc, (int)threadIdx.x * per), hi = min(lo + per, nc);
  int sum = 0;
  for (int i = lo; i < hi; ++i) sum += buf[i];
  const int inc = block_incl_scan<NT>(sum, sh);
  int run = inc - sum;
  for (int i = lo; i < hi; ++i) {
    const int v = buf[i];
    buf[i] = run;
    run += v;
  }
  if (threadIdx.x == NT - 1) {
    c.start[nc] = inc & 0xffff;
    c.qstart[nc] = (unsigned)inc >> 16;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nc; i += NT) {
    const unsigned v = (unsigned)buf[i];
    c.start[i] = (int)(v & 0xffffu);
    c.qstart[i] = (int)(v >> 16);
  }
  __syncthreads();
  // scatter; each cell's low half counts up to the next cell's start
#pragma unroll
  for (int u = 0; u < BPT; ++u) {
    const int s = threadIdx.x + u * NT;
    if (s < N) {
      const int slot = atomicAdd(&buf[cid[u]], 1) & 0xffff;
      // (slots outside the population cannot come from consistent counts)
      if (slot < N) tmp[slot] = s | (param_z(prm[u]) != 0 ? 0x10000 : 0);
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < BPT; ++u) {
    const int s = threadIdx.x + u * NT;
    if (s >= N) continue;
    const int c0 = cid[u] > 0 ? buf[cid[u] - 1] & 0xffff : 0, c1 = min(buf[cid[u]] & 0xffff, N);
    int rank = 0, qrank = 0;
    for (int t = c0; t < c1; ++t) {
      const int o = tmp[t];
      const bool before = (o & 0xffff) < s;
      rank += before;
      qrank += before && (o & 0x10000);
    }
    const int n = c0 + rank;
    if (n >= N) continue;
    B.pos[0][n] = px[u];
    B.pos[1][n] = py[u];
    B.pos[2][n] = pz[u];
    B.vel[0][n] = vx[u];
    B.vel[1][n] = vy[u];
    B.vel[2][n] = vz[u];
    B.param[n] = prm[u];
    B.id[n] = id[u];
    if (c.slot_of && (unsigned)id[u] < (unsigned)N) c.slot_of[id[u]] = n;
    const uint4 rec = make_uint4(px[u], py[u], pz[u], prm[u]);
    bpk[n] = rec;
    if (param_z(prm[u]) != 0) {
      const int qn = (int)((unsigned)buf[cid[u]] >> 16) + qrank;
      if (qn < q.n) {
        q.pk[qn] = rec;
        q.idx[qn] = n;
      }
    }
  }
}

// The whole sort in one launch from the buckets that the binning filled, for
// grids of up to BUCKET_SORT_CELLS cells.  A block takes `per` consecutive
// cells: it adds up the counts of the cells before them itself (as
// k_scan_self), scans its own, and moves their beads: 16 lanes, a DPP row,
// hold the entries of a cell, whose ranks (beads of the cell with a smaller
// previous index) are 15 row rotations.  The counts and the length of the list
// below are cleared for the next binning by the last block to have read them.
// The beads of a cell of more than CELL_CAP are brought together in LDS, from
// its bucket and the list of those that found one full, and ranked among
// themselves; in a block with more than BUCKET_LIST of them, each wavefront
// meets those of its own cells in order by going through all N (neither in a
// fluid of some three beads a cell).
// It is bound by latency: the load of the counts, a block scan, then the loads
// and stores of a bead.  Against scan, scatter and permute, the whole sort and
// its gaps: 4,099 beads 13.0 -> 10.0 us, 32,768 15.5 -> 13.0 (ten steps 787 ->
// 746 us); steps of 8,000 beads 56 -> 51, 16,384 61 -> 56, 50,000 (18,000
// cells) 84.6 -> 82, and no gain at 80,000 (29,000 cells) and above, since
// every block reads all counts before its own.  Crowded systems of 20,000 cells,
// steps with scan, scatter and permute and with this: a dense column of 7,000
// beads in cells of 30 172 and 172 us (355 where each listed bead was compared
// with all the block's, and 2,048 had room), a spot of cells of 380 beads 195
// and 167 (232), a droplet 155 and 155 (165).
constexpr int BUCKET_SORT_THREADS = 1024;
constexpr int BUCKET_SORT_CELLS = 24576;
constexpr int BUCKET_LIST = 8192;
constexpr int BUCKET_PER_MAX = 128;  // cells of a block
// about a block per CU, of whole groups of 64 cells
constexpr int bucket_per(int ncells) { return std::max(64, ((ncells + 255) / 256 + 63) & ~63); }
static_assert(bucket_per(BUCKET_SORT_CELLS) <= BUCKET_PER_MAX && BUCKET_PER_MAX <= BUCKET_SORT_THREADS, "a thread per cell");
static_assert(CELL_CAP == 16, "a cell's bucket is one DPP row");

template <int R>
__device__ inline void row_ranks(uint32_t key, int& rank, int& qrank) {
  if constexpr (R < 16) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, 0x120 + R, 0xf, 0xf, false);  // row_ror:R
    rank += o < key;
    qrank += o < key && (o & 1u);
    row_ranks<R + 1>(key, rank, qrank);
  }
}

__device__ inline void move_bead(const StateView& A, const StateView& B, uint4* __restrict__ bpk, const CellView& c,
                                 const ChargedView& q, int N, int s, int n, int qn) {
  // (inconsistent counts cannot send an access out of bounds)
  if ((unsigned)s >= (unsigned)N || (unsigned)n >= (unsigned)N) return;
  const uint32_t prm = A.param[s];
  const uint32_t px = A.pos[0][s], py = A.pos[1][s], pz = A.pos[2][s];
  const double vx = A.vel[0][s], vy = A.vel[1][s], vz = A.vel[2][s];
  const int id = A.id[s];
  B.pos[0][n] = px;
  B.pos[1][n] = py;
  B.pos[2][n] = pz;
  B.vel[0][n] = vx;
  B.vel[1][n] = vy;
  B.vel[2][n] = vz;
  B.param[n] = prm;
  B.id[n] = id;
  if (c.slot_of && (unsigned)id < (unsigned)N) c.slot_of[id] = n;
  const uint4 rec = make_uint4(px, py, pz, prm);
  bpk[n] = rec;
  if (param_z(prm) != 0 && (unsigned)qn < (unsigned)q.n) {
    q.pk[qn] = rec;
    q.idx[qn] = n;
  }
}

__global__ __launch_bounds__(BUCKET_SORT_THREADS) void k_sort_buckets(StateView A, StateView B, uint4* __restrict__ bpk,
                                                                      CellView c, ChargedView q, int N, int per) {
  constexpr int NT = BUCKET_SORT_THREADS, NW = NT / 64, U = 4;
  __shared__ int s_own[2][NW], s_off[2][NW];
  __shared__ int s_cnt[BUCKET_PER_MAX], s_start[BUCKET_PER_MAX], s_qstart[BUCKET_PER_MAX];
  // the crowded cells' beads, cell by cell (s_seg: where a cell's begin, s_fill:
  // how many are there), and of each the cell
  __shared__ __align__(16) uint32_t s_key[BUCKET_LIST];
  __shared__ uint16_t s_cell[BUCKET_LIST];
  __shared__ int s_seg[BUCKET_PER_MAX], s_fill[BUCKET_PER_MAX];
  __shared__ int s_last, s_nlist, s_no;
  const int n = c.ncells, c0 = blockIdx.x * per;
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  if (c.step && blockIdx.x == 0 && t == 0) *c.step += 1ULL;
  if (t == 0) {
    s_nlist = 0;
    s_no = min(c.sortn[1], N);  // entries of over: read before the ticket, like the counts
  }
  // 1. the starts of this block's cells (c0 is a multiple of 64)
  const bool mine = t < per && c0 + t < n;
  const int v0 = mine ? c.counts[c0 + t] : 0, v1 = mine ? c.qcounts[c0 + t] : 0;
  const int4* __restrict__ k0 = reinterpret_cast<const int4*>(c.counts);
  const int4* __restrict__ k1 = reinterpret_cast<const int4*>(c.qcounts);
  int o0 = 0, o1 = 0;
  for (int i0 = t; i0 < c0 / 4; i0 += U * NT) {
    int4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = i0 + u * NT < c0 / 4;
      a[u] = in ? k0[i0 + u * NT] : make_int4(0, 0, 0, 0);
      b[u] = in ? k1[i0 + u * NT] : make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      o0 += (a[u].x + a[u].y) + (a[u].z + a[u].w);
      o1 += (b[u].x + b[u].y) + (b[u].z + b[u].w);
    }
  }
  int i0 = v0, i1 = v1;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int a = __shfl_up(i0, o, 64), b = __shfl_up(i1, o, 64);
    o0 += __shfl_xor(o0, o, 64);
    o1 += __shfl_xor(o1, o, 64);
    if (lane >= o) {
      i0 += a;
      i1 += b;
    }
  }
  if (lane == 63) {
    s_own[0][wid] = i0;
    s_own[1][wid] = i1;
    s_off[0][wid] = o0;
    s_off[1][wid] = o1;
  }
  // every load of what the last block clears has returned: the ticket says so,
  // and nothing of it may be read after
  __syncthreads();
  int tick = 0;
  if (t == NT - 64) tick = atomicAdd(&c.sortn[0], 1);
  int r0 = i0 - v0, r1 = i1 - v1;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    r0 += s_off[0][w] + (w < wid ? s_own[0][w] : 0);
    r1 += s_off[1][w] + (w < wid ? s_own[1][w] : 0);
  }
  if (t < per) {
    s_cnt[t] = v0;
    s_start[t] = r0;
    s_qstart[t] = r1;
    if (mine) {
      c.start[c0 + t] = r0;
      c.qstart[c0 + t] = r1;
      if (c0 + t == n - 1) {
        c.start[n] = r0 + v0;
        c.qstart[n] = r1 + v1;
      }
    }
    s_fill[t] = 0;
    if (v0 > CELL_CAP) {
      const int room = (v0 + 3) & ~3;
      const int at = s_seg[t] = atomicAdd(&s_nlist, room);
      for (int k = at + v0; k < min(at + room, BUCKET_LIST); ++k) {  // (no bead's key: after all)
        s_key[k] = 0xffffffffu;
        s_cell[k] = 0xffffu;
      }
    }
  }
  __syncthreads();
  // 2. the beads of the cells that their buckets hold
  for (int g = t >> 4; g < per; g += NT / 16) {
    const int cnt = s_cnt[g];
    if (!__any(cnt > 0)) continue;
    const bool on = cnt <= CELL_CAP && (t & 15) < cnt;
    const uint32_t key = on ? c.bucket[(size_t)(c0 + g) * CELL_CAP + (t & 15)] : 0xffffffffu;
    int rank = 0, qrank = 0;
    row_ranks<1>(key, rank, qrank);
    if (on) move_bead(A, B, bpk, c, q, N, (int)(key >> 1), s_start[g] + rank, s_qstart[g] + qrank);
  }
  // 3. the others
  const int nl = s_nlist;
  if (nl > 0 && nl <= BUCKET_LIST) {
    auto put = [&](int g, uint32_t key) {
      const int at = atomicAdd(&s_fill[g], 1);
      if (at < s_cnt[g]) {  // (as for consistent counts)
        s_key[s_seg[g] + at] = key;
        s_cell[s_seg[g] + at] = (uint16_t)g;
      }
    };
    for (int g = t >> 4; g < per; g += NT / 16)
      if (s_cnt[g] > CELL_CAP) put(g, c.bucket[(size_t)(c0 + g) * CELL_CAP + (t & 15)]);
    for (int i = t; i < s_no; i += NT) {
      const uint2 e = c.over[i];
      const uint32_t g = e.x - (uint32_t)c0;
      if (g < (uint32_t)per && s_cnt[g] > CELL_CAP) put((int)g, e.y);
    }
    __syncthreads();
    for (int i = t; i < nl; i += NT) {
      const uint32_t key = s_key[i], g = s_cell[i];
      if (g >= (uint32_t)per || s_cnt[g] <= CELL_CAP) continue;
      const int k1 = s_seg[g] + s_cnt[g];
      int rank = 0, qrank = 0;
      for (int k = s_seg[g]; k < k1; k += 4) {
        const uint4 o = *reinterpret_cast<const uint4*>(s_key + k);
        rank += (o.x < key) + (o.y < key) + (o.z < key) + (o.w < key);
        qrank += (o.x < key && (o.x & 1u)) + (o.y < key && (o.y & 1u)) + (o.z < key && (o.z & 1u)) +
                 (o.w < key && (o.w & 1u));
      }
      move_bead(A, B, bpk, c, q, N, (int)(key >> 1), s_start[g] + rank, s_qstart[g] + qrank);
    }
  } else if (nl > BUCKET_LIST) {
    // each wavefront its own cells, whose s_start count up as it meets beads
    for (int b0 = 0; b0 < N; b0 += 64 * U) {
      int cid[U];
#pragma unroll
      for (int u = 0; u < U; ++u) cid[u] = b0 + 64 * u + lane < N ? c.cell[b0 + 64 * u + lane] - c0 : -1;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = b0 + 64 * u + lane, g = cid[u];
        const bool m = (unsigned)g < (unsigned)per && (g & (NW - 1)) == wid && s_cnt[g] > CELL_CAP;
        unsigned long long left = __ballot(m);
        while (left) {
          const int gg = __builtin_amdgcn_readlane(g, __ffsll((long long)left) - 1);
          const bool take = m && g == gg;
          const bool charged = take && param_z(A.param[s]) != 0;
          const unsigned long long mm = __ballot(take), mq = __ballot(charged);
          const unsigned long long below = (1ull << lane) - 1ull;
          const int base = s_start[gg], qbase = s_qstart[gg];
          if (take) move_bead(A, B, bpk, c, q, N, s, base + __popcll(mm & below), qbase + __popcll(mq & below));
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // (every lane has read them)
          if (lane == 0) {
            s_start[gg] = base + __popcll(mm);
            s_qstart[gg] = qbase + __popcll(mq);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          left &= ~mm;
        }
      }
    }
  }
  // 4. the counts and the list's length, when every block has read them
  if (t == NT - 64) s_last = tick == (int)gridDim.x - 1;
  __syncthreads();
  if (s_last) {
    for (int i = t; i < n; i += NT) c.counts[i] = c.qcounts[i] = 0;
    if (t < 2) c.sortn[t] = 0;
  }
}

// Column clusters (see ColLaunch).  One block: the columns' cluster counts
// are staged in LDS (loads spread over the block), each thread then takes a
// contiguous run of columns, and a block scan of the runs' counts gives every
// column its first cluster slot, numbered from its replica's first slot.
// With `fill` the scan's threads write the clusters themselves (one column
// per thread at most); otherwise each column's first slot goes to colbase
// and k_col_fill writes them, one thread per column.
constexpr int COL_THREADS = 1024;
constexpr int COL_LDS_MAX = 36864;  // columns + replicas staged in LDS (144 KiB)

__global__ __launch_bounds__(COL_THREADS) void k_col_scan(ColLaunch a, bool fill) {
  __shared__ int sh[COL_THREADS / 64];
  extern __shared__ int lds[];
  int* rfirst = lds;            // [nrep]: global cluster count before each replica
  int* rend = lds + a.nrep;     // [nrep]: ... and after it
  int* cnt = lds + 2 * a.nrep;  // [ncols]: clusters per column, then their first slot
  wave_stamp(a.stamps, 0);
  const int n = a.ncols;
  const int sh_ci = __ffs(a.ci) - 1;
  // 1. the counts, four columns per thread in flight
  for (int c0 = threadIdx.x; c0 < n; c0 += 4 * COL_THREADS) {
    int lo[4], hi[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * COL_THREADS;
      lo[u] = c < n ? a.coltab[c].x : 0;
      hi[u] = c < n ? a.coltab[c + 1].x : 0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      lo[u] = a.start[lo[u]];
      hi[u] = a.start[hi[u]];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = c0 + u * COL_THREADS;
      if (c < n) cnt[c] = (hi[u] - lo[u] + a.ci - 1) >> sh_ci;
    }
  }
  __syncthreads();
  // 2. exclusive scan over contiguous runs of columns
  const int per = (n + COL_THREADS - 1) / COL_THREADS;
  const int lo = min(n, (int)threadIdx.x * per), hi = min(lo + per, n);
  int s = 0;
  for (int c = lo; c < hi; ++c) s += cnt[c];
  const int inc = block_incl_scan<COL_THREADS>(s, sh);
  int run = inc - s;
  for (int c = lo; c < hi; ++c) {
    const int v = cnt[c];
    cnt[c] = run;
    const int r = a.coltab[c].y;
    if (c == 0 || a.coltab[c - 1].y != r) rfirst[r] = run;
    run += v;
    if (c + 1 == n || a.coltab[c + 1].y != r) rend[r] = run;
  }
  __syncthreads();
  // 3. each replica's count, and the columns' first slots (or the clusters)
  for (int r = threadIdx.x; r < a.nrep; r += COL_THREADS) a.ncl[r] = rend[r] - rfirst[r];
  for (int c = threadIdx.x; c < n; c += COL_THREADS) {
    const int2 ct = a.coltab[c];
    const int slot = a.rep_base[ct.y] + cnt[c] - rfirst[ct.y];
    if (fill) {
      const int b = a.start[ct.x], e = a.start[a.coltab[c + 1].x];
      int sl = slot;
      for (int f = b; f < e; f += a.ci) a.cl[sl++] = make_int2(f, min(a.ci, e - f));
    } else {
      a.colbase[c] = slot;
    }
  }
  wave_stamp(a.stamps, 1);
}

__global__ void k_col_fill(ColLaunch a) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= a.ncols) return;
  const int b = a.start[a.coltab[c].x], e = a.start[a.coltab[c + 1].x];
  int slot = a.colbase[c];
  for (int f = b; f < e; f += a.ci) a.cl[slot++] = make_int2(f, min(a.ci, e - f));
}

inline int nblk(long long n, int t) { return (int)((n + t - 1) / t); }

}  // namespace

void launch_ingest(hipStream_t s, const double* pos_soa, int N, const RepDesc* rep, StateView A, long long* F,
                   const CellView* bin) {
  if (bin)
    hipLaunchKernelGGL(k_ingest<true>, dim3(nblk(N, 256)), dim3(256), 0, s, pos_soa, N, N, rep, A, F, *bin);
  else
    hipLaunchKernelGGL(k_ingest<false>, dim3(nblk(N, 256)), dim3(256), 0, s, pos_soa, N, N, rep, A, F, CellView{});
}

void launch_fill_i64(hipStream_t s, long long* p, long long v, long long n) {
  if (n <= 0) return;
  int b = nblk(n, 256);
  if (b > 4096) b = 4096;
  hipLaunchKernelGGL(k_fill<long long>, dim3(b), dim3(256), 0, s, p, v, n);
}

void launch_bin(hipStream_t s, StateView A, const RepDesc* rep, CellView c, long long* F, int N) {
  hipLaunchKernelGGL(k_bin, dim3(nblk(N, BEAD_THREADS)), dim3(BEAD_THREADS), 0, s, A, rep, c, F, N);
}

static void launch_scan(hipStream_t s, CellView c) {
  if (c.ncells <= SELF_SCAN_MAX) {
    hipLaunchKernelGGL(k_scan_self, dim3(nblk(c.ncells, SELF_SCAN_BLOCK), 2), dim3(SELF_SCAN_THREADS), 0, s, c);
    return;
  }
  int nb = nblk(c.ncells, SCAN_BLOCK);
  hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(SCAN_THREADS), 0, s, c, nb);
  if (nb <= SCAN_SUMS_MAX) {
    hipLaunchKernelGGL(k_scan_apply<true>, dim3(nb), dim3(SCAN_THREADS), 0, s, c, nb);
    return;
  }
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(SCAN_THREADS), 0, s, c, nb);
  hipLaunchKernelGGL(k_scan_apply<false>, dim3(nb), dim3(SCAN_THREADS), 0, s, c, nb);
}

// Buckets pay while the counts are few enough to be summed by every block and
// a cell's bucket (64 B) holds its beads: at seven beads a cell on average, the
// limit, one cell in 1,000 of an ideal gas has more than CELL_CAP.  Up to
// 1,024 beads the one-block sort, which fetches one bead a thread, is as
// short (700 beads 8.8 us against 8.9, 1,100 10.7 against 9.1, 1,536 13.0
// against 9.3, 4,000 25.5 against 9.5: the step 52 -> 47); above, it serves
// where there are no buckets.
bool bucket_sort(int N, int ncells) {
  return N > SMALL_SORT_THREADS && ncells <= BUCKET_SORT_CELLS && N <= 7LL * ncells;
}

void launch_sort(hipStream_t s, StateView A, StateView B, uint4* bpk, CellView c, ChargedView q, int N) {
  if (c.bucket) {
    const int per = bucket_per(c.ncells);
    hipLaunchKernelGGL(k_sort_buckets, dim3(nblk(c.ncells, per)), dim3(BUCKET_SORT_THREADS), 0, s, A, B, bpk, c, q, N, per);
    return;
  }
  if (N <= SMALL_SORT_BEADS && c.ncells <= SMALL_SORT_CELLS) {
    const size_t sh = ((size_t)c.ncells + N) * 4;
    if (sh > 65536) (void)hipFuncSetAttribute((const void*)k_sort_small, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
    hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(SMALL_SORT_THREADS), sh, s, A, B, bpk, c, q, N);
    return;
  }
  launch_scan(s, c);
  hipLaunchKernelGGL(k_scatter, dim3(nblk(N, BEAD_THREADS)), dim3(BEAD_THREADS), 0, s, c, N);
  hipLaunchKernelGGL(k_permute, dim3(nblk(N, BEAD_THREADS)), dim3(BEAD_THREADS), 0, s, A, B, bpk, c, q, N);
}

int col_clusters_max_entries() { return COL_LDS_MAX; }

void launch_col_clusters(hipStream_t s, const ColLaunch& a) {
  if (a.ncols <= 0) return;
  const size_t sh = ((size_t)a.ncols + 2 * (size_t)a.nrep) * 4;
  if (sh > 65536) (void)hipFuncSetAttribute((const void*)k_col_scan, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh);
  // one column per thread of the scan: it writes the clusters itself
  const bool fill = a.ncols <= COL_THREADS;
  hipLaunchKernelGGL(k_col_scan, dim3(1), dim3(COL_THREADS), sh, s, a, fill);
  if (!fill) hipLaunchKernelGGL(k_col_fill, dim3(nblk(a.ncols, 128)), dim3(128), 0, s, a);
}

}  // namespace gcme
