// Launches of the bucketed kernel (uneven swarm sizes) of one workgroup size.
#pragma once
#include <algorithm>

#include "qs_handle.h"
#include "qs_kernels.h"

namespace {

using qs_host::ptrs;

// One launch of the bucketed kernel over items [item0, item0 + count).
template <int BS, int KT>
void go_range(qs_handle* h, int item0, int count, int grid, const float* act, int nsub,
              const float* goals, float* obs, hipStream_t s, float* rw) {
  const size_t dyn = KT >= 0 ? (size_t)qs::BUCKET_STAGE_ROWS * h->OD * sizeof(float) : 0;
  hipLaunchKernelGGL((qs::bucket_kernel<BS, KT>), dim3(std::max(grid, 1)), dim3(BS), dyn, s,
                     h->d_st, h->d_par, act, goals, h->d_c, h->Q, nsub,
                     (unsigned long long)h->t, ptrs(h), obs, item0, count,
                     h->graph_mode ? h->d_t : nullptr, h->d_done, rw);
}

template <int BS, int KT>
void go_items(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
              hipStream_t s, float* rw) {
  const int grid = h->item_grid > 0 ? std::min(h->item_grid, h->n_items) : h->n_items;
  go_range<BS, KT>(h, 0, h->n_items, grid, act, nsub, goals, obs, s, rw);
}

template <int BS>
void items_bs(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
              bool with_obs, hipStream_t s, float* rw) {
  if (!with_obs)
    go_items<BS, -2>(h, act, nsub, goals, obs, s, rw);
  else if (h->K == 6)
    go_items<BS, 6>(h, act, nsub, goals, obs, s, rw);
  else if (h->K == 0)
    go_items<BS, 0>(h, act, nsub, goals, obs, s, rw);
  else if (h->K <= qs::kSlots<qs::K_UPTO8>)
    go_items<BS, qs::K_UPTO8>(h, act, nsub, goals, obs, s, rw);
  else
    go_items<BS, -1>(h, act, nsub, goals, obs, s, rw);
}

// One launch over an item range alone (autotuner trials; not in graph
// mode).
template <int BS>
void range_bs(qs_handle* h, int item0, int count, const float* act, int nsub,
              const float* goals, float* obs, bool with_obs, hipStream_t s) {
  if (!with_obs)
    go_range<BS, -2>(h, item0, count, count, act, nsub, goals, obs, s, nullptr);
  else if (h->K == 6)
    go_range<BS, 6>(h, item0, count, count, act, nsub, goals, obs, s, nullptr);
  else if (h->K == 0)
    go_range<BS, 0>(h, item0, count, count, act, nsub, goals, obs, s, nullptr);
  else if (h->K <= qs::kSlots<qs::K_UPTO8>)
    go_range<BS, qs::K_UPTO8>(h, item0, count, count, act, nsub, goals, obs, s, nullptr);
  else
    go_range<BS, -1>(h, item0, count, count, act, nsub, goals, obs, s, nullptr);
}

}  // namespace
