// Launches of the dense and table step kernels of one workgroup size.
#pragma once
#include <cstdlib>

#include "qs_handle.h"
#include "qs_kernels.h"

namespace {

using qs_host::ptrs;

// Calls of several substeps on small batches run the motor part one substep
// ahead in a second wavefront (QS_STEP_PIPE=0/1 forces it off/on): a lone
// wavefront waits for its own instructions, and two share a substep.  Up to 1536
// workgroups (three wavefronts a SIMD) all of them are resident together; beyond,
// the last ones wait for a second turn.  us a call, one wavefront / two, of two,
// four and ten substeps:
//   4096 quads in swarms of 8    6.7 / 5.7    8.9 / 7.7   17.8 / 14.1
//   4096 in 32                   9.9 / 9.1   13.9 / 12.5  27.0 / 22.1
//   1100 workgroups of 12s      11.8 / 10.7  15.6 / 13.6  26.5 / 22.0  (table)
//   1536                        12.6 / 11.9  16.6 / 15.0  27.6 / 24.6
//   1700                        13.2 / 16.1  16.8 / 20.9  28.8 / 35.3
//   1536 of 3s                  12.1 / 11.0  15.0 / 13.5  24.7 / 20.4
//   1536 of 48s                 22.0 / 20.8  27.3 / 25.7  44.0 / 39.6
//   1421 of 1 to 64             23.8 / 22.6  30.0 / 28.3  45.9 / 42.2
//   98304 in 8                  10.3 / 9.5   13.6 / 12.2  25.9 / 22.3
//   98304 in 32                 15.8 / 15.4  20.1 / 18.8  36.3 / 36.5
//   131072 in 8                 12.2 / 14.2  14.7 / 17.9  27.1 / 30.6
//   131072 in 1                  8.1 / 7.6   10.4 / 9.7   18.0 / 16.5
//   262144 in 1                 14.5 / 14.3  18.5 / 18.4  30.4 / 30.4
bool use_step_pipe(const qs_handle* h) {
  if (const char* e = std::getenv("QS_STEP_PIPE")) return e[0] == '1';
  return h->nblk <= (h->uniform_n == 1 ? 2048 : 1536);
}

// Observation rows per staging pass.  A grid of at most 2048 workgroups
// has at most two per SIMD, which LDS never limits: the whole workgroup's
// rows in one pass (fewest synchronisations; 4096 x 8: 6.7 us per launch
// against 7.0 us in two passes).  Larger grids keep the staging area and the
// exchange tile together within 10 KiB per wavefront of the workgroup
// (160 KiB of LDS over the four wavefronts per SIMD that the step's
// registers allow), so that LDS does not hold the resident workgroups below
// what the registers allow.  At 32768 x 32 (K = 6, 64-quad workgroups, a
// 6 KiB tile) that is 16 rows per pass: ten substeps per call 40.8 -> 50.9 G
// quad-steps/s against 32 rows (13.0 KiB per workgroup, three wavefronts
// per SIMD).  QS_STAGE_ROWS=n overrides (0: every lane stores its own row).
int stage_rows(int bs, int od, int nblk) {
  static const int forced = [] {
    const char* e = std::getenv("QS_STAGE_ROWS");
    return e ? std::atoi(e) : -1;
  }();
  if (forced >= 0 && forced <= bs && (forced & (forced - 1)) == 0) return forced;
  const size_t row = (size_t)od * sizeof(float);
  const size_t tile = 2 * qs::TILE_ROWS_CO * (size_t)bs * sizeof(float);
  const size_t budget = (size_t)(bs / 64) * 10 * 1024;
  size_t cap = budget > tile ? budget - tile : 0;
  if (nblk <= 2048) cap = 48 * 1024;
  int r = bs;
  while (r > 8 && (size_t)r * row > cap) r >>= 1;
  return r;
}

// Launch one instantiation.
template <int BS, int KT, int N>
void go(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
        hipStream_t s, float* rw) {
  size_t dyn = 0;
  int stage = 0;
  if constexpr (KT >= 0) {
    stage = stage_rows(BS, h->OD, h->nblk);
    dyn = (size_t)stage * h->OD * sizeof(float);
  }
  if constexpr (BS == 64 && KT != -1) {
    // (swarms of 64 go over their partners once more for the observation, which
    // their one-wavefront kernel takes from the screen: two substeps lose,
    // 16384 quads 18.4 / 19.0 us, four gain, 26.0 / 25.3)
    if (nsub >= (N == 64 ? 4 : 2) && use_step_pipe(h)) {
      hipLaunchKernelGGL((qs::step_pipe_kernel<KT, N>), dim3(h->nblk), dim3(128), dyn, s,
                         h->d_st, h->d_par, act, goals, h->d_c, h->Q, nsub,
                         (unsigned long long)h->t, ptrs(h), obs, stage,
                         h->graph_mode ? h->d_t : nullptr, h->d_done, rw);
      return;
    }
  }
  hipLaunchKernelGGL((qs::step_kernel<BS, KT, N>), dim3(h->nblk), dim3(BS), dyn, s, h->d_st,
                     h->d_par, act, goals, h->d_c, h->Q, nsub, (unsigned long long)h->t,
                     ptrs(h), obs, stage, h->graph_mode ? h->d_t : nullptr, h->d_done, rw);
}

template <int BS, int KT>
void go_n(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
          hipStream_t s, float* rw) {
  switch (h->uniform_n) {
    case 1: go<BS, KT, 1>(h, act, nsub, goals, obs, s, rw); break;
    case 2: go<BS, KT, 2>(h, act, nsub, goals, obs, s, rw); break;
    case 4: go<BS, KT, 4>(h, act, nsub, goals, obs, s, rw); break;
    case 8: go<BS, KT, 8>(h, act, nsub, goals, obs, s, rw); break;
    case 16: go<BS, KT, 16>(h, act, nsub, goals, obs, s, rw); break;
    case 32: go<BS, KT, 32>(h, act, nsub, goals, obs, s, rw); break;
    case 64: go<BS, KT, 64>(h, act, nsub, goals, obs, s, rw); break;
    default: go<BS, KT, 0>(h, act, nsub, goals, obs, s, rw); break;
  }
}

template <int BS>
int launch_bs(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
              bool with_obs, hipStream_t s, float* rw) {
  if (!with_obs)
    go_n<BS, -2>(h, act, nsub, goals, obs, s, rw);
  else if (h->K == 6)
    go_n<BS, 6>(h, act, nsub, goals, obs, s, rw);
  else if (h->K == 0)
    go_n<BS, 0>(h, act, nsub, goals, obs, s, rw);
  else if (h->K <= qs::kSlots<qs::K_UPTO8>)
    go_n<BS, qs::K_UPTO8>(h, act, nsub, goals, obs, s, rw);
  else
    go<BS, -1, 0>(h, act, nsub, goals, obs, s, rw);
  return hipGetLastError() == hipSuccess ? QS_OK : QS_ERR_HIP;
}

}  // namespace
