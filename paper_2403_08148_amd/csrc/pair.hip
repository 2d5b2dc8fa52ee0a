// The list build and the launchers of the cutoff pair kernels (device code in
// pair_kernels.h; the pair kernels themselves are compiled by pair_gcm_*.hip,
// pair_elec_*.hip and pair_col.hip).
#include "pair_kernels.h"

namespace gcme {

namespace {

// Compiled for five wavefronts per SIMD (102 VGPRs; a few spilled for CI =
// 8): the 256 batched replicas' step went 0.763 -> 0.748 ms.
template <int CI>
__global__ __launch_bounds__(NL_WAVES * 64) __attribute__((amdgpu_waves_per_eu(5))) void k_nl_build(PairLaunch a) {
  __shared__ int2 s_seg[NL_WAVES][NL_SEG];
  __shared__ int s_cand[NL_WAVES][NL_CAND];
  wave_stamp(a.stamps, 0);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int c = xcd_item(blockIdx.x, (a.ncl + NL_WAVES - 1) / NL_WAVES) * NL_WAVES + wave;
  if (c >= a.ncl) return;  // whole wavefront; no block barriers below
  const int2 info = uniform_load(a.cl + c);
  const int first = info.x, rep = info.y & 0xffff, ni = info.y >> 16;
  const RepDesc R = uniform_load(a.rep + rep);
  const uint4* __restrict__ pk = a.pk;
  const int kk = lane % CI;
  const uint4 me = pk[first + (kk < ni ? kk : 0)];
  ClusterBox K;
  float r[3], nn;
  make_box<CI>(K, me, R, r, nn);
  uint32_t* __restrict__ out = a.list + (size_t)c * a.cap;
  int nent = 0;
  // one candidate per lane; hits are appended in candidate order
  auto append = [&](bool hit, int j) {
    const unsigned long long m = __ballot(hit);
    if (hit) {
      const int idx = nent + lanes_below(m);
      if (idx < a.cap) out[idx] = (uint32_t)j;
    }
    nent += __popcll(m);
  };
  const int* cand = s_cand[wave];
  if (in_frame(K, R)) {
    FrameTest<CI> T;
    frame_test_init<CI>(T, K, r, nn);
    for_candidates(K, R, a.start, s_seg[wave], s_cand[wave], [&](int total) {
      for_chunks<2>(cand, total, pk, first, [&](const uint4 pj, bool v, int j) {
        float Dx, Dy, Dz;
        const bool near = near_frame<CI>(T, K, pj, R, Dx, Dy, Dz);
        append(near && v, j);
      });
    });
  } else {
    for_candidates(K, R, a.start, s_seg[wave], s_cand[wave], [&](int total) {
      for_chunks<2>(cand, total, pk, first,
                    [&](const uint4 pj, bool v, int j) { append(near_exact<CI>(K, me, pj, R) && v, j); });
    });
  }
  if (lane == 0) {
    a.count[c] = min(nent, a.cap);
    if (nent > a.cap) atomicOr(a.status, (unsigned)STATUS_LIST_OVERFLOW);
  }
  wave_stamp(a.stamps, 1);
}

}  // namespace

void launch_nl_build(hipStream_t s, const PairLaunch& a) {
  if (a.ncl <= 0 || a.direct) return;
  dim3 g((a.ncl + NL_WAVES - 1) / NL_WAVES), b(NL_WAVES * 64);
  switch (a.ci) {
    case 2: hipLaunchKernelGGL(k_nl_build<2>, g, b, 0, s, a); break;
    case 8: hipLaunchKernelGGL(k_nl_build<8>, g, b, 0, s, a); break;
    default: hipLaunchKernelGGL(k_nl_build<4>, g, b, 0, s, a); break;
  }
}

void launch_pair_gcm(hipStream_t s, const PairLaunch& a, bool fp64, bool ev, bool adjoint) {
  if (a.ntiles <= 0) return;
  bool count = a.pair_count != nullptr;
  if (fp64)
    dispatch_ci<double, false>(s, a, ev, adjoint, count);
  else
    dispatch_ci<float, false>(s, a, ev, adjoint, count);
}

void launch_pair_elec(hipStream_t s, const PairLaunch& a, bool fp64, bool ev, bool adjoint) {
  if (a.ntiles <= 0) return;
  if (fp64)
    dispatch_ci<double, true>(s, a, ev, adjoint, false);
  else
    dispatch_ci<float, true>(s, a, ev, adjoint, false);
}

int pair_waves_per_block() { return NL_WAVES; }

}  // namespace gcme
