// The handle behind the C ABI, and the launches that live in translation units
// of their own (the kernels' instantiations build in parallel).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "quadswarm.h"
#include "qs_checks.h"
#include "qs_device.h"

using qs::Consts;
using qs::Ptrs;

struct qs_handle {
  int dev = 0;
  int E = 0, Q = 0, Qp = 0, K = 0, OD = 0;
  int bs = 64, nblk = 0;
  int max_n = 1;      // largest swarm
  int uniform_n = 0;  // every swarm holds this many quads (power of two), else 0
  Consts c{};
  Consts* d_c = nullptr;  // device copy of c, read by every kernel
  float* d_st = nullptr;
  float* d_par = nullptr;
  uint32_t* d_sw = nullptr;
  int2* d_blk = nullptr;
  int32_t* d_qenv = nullptr;
  unsigned long long* d_contacts = nullptr;
  int* d_err = nullptr;
  int* h_err = nullptr;  // pinned
  uint64_t t = 0;
  bool record = false;
  // uneven swarm sizes: work items of the persistent bucketed launch
  std::vector<int> env_start, env_n;  // host copy of the environments
  int4* d_items = nullptr;
  int2* d_item_envs = nullptr;
  int n_items = 0;
  int item_bs = 64;      // workgroup size of the bucketed launch
  int item_grid = 0;     // persistent grid size of the shared launch (0: one workgroup per item)
  // slot sizes (bit log2 N; 16 and 32) whose items take the body with the size
  // known at compile time (all slot's places in chunks of four, through the
  // expanded screen) instead of the run-time size's: the faster one unless the
  // autotuner measures otherwise (172,943 quads of 1 to 32, ten substeps, the items
  // of 32 alone: 49.7 -> 36.9 us)
  uint32_t chunked = (1u << 4) | (1u << 5);
  // per slot size: swarms, and the times the autotuner measured for the
  // slot's items alone with each body (ns per call)
  int slot_swarms[7] = {0, 0, 0, 0, 0, 0, 0};
  float slot_ns_one[7] = {0, 0, 0, 0, 0, 0, 0};
  float slot_ns_chunked[7] = {0, 0, 0, 0, 0, 0, 0};
  bool bucketed = false;
  int items_from = 0;    // substeps a call from which it is used (fewer: the table)
  bool items_always = false;  // in every call, by QS_BUCKETED: the autotuner leaves it so
  // graph-safe substep counter
  bool graph_mode = false;
  unsigned long long* d_t = nullptr;
  unsigned int* d_done = nullptr;
  // backward passes' scratch, grown on demand: the tape of the chunk of
  // segments in flight, one checkpoint [27][Q], and the parameter gradient
  // [Q][6] of the chunks so far where there are several
  float* d_tape = nullptr;
  size_t tape_cap = 0;
  float* d_ck1 = nullptr;
  size_t ck1_cap = 0;
  float* d_gsum = nullptr;
  size_t gsum_cap = 0;
};

namespace qs_host {

inline Ptrs ptrs(qs_handle* h) {
  Ptrs p;
  p.st = h->d_st;
  p.par = h->d_par;
  p.sw = h->d_sw;
  p.blk = h->d_blk;
  p.contacts = h->record ? h->d_contacts : nullptr;
  p.err = h->d_err;
  p.Q = h->Q;
  p.items = h->d_items;
  p.item_envs = h->d_item_envs;
  return p;
}

// Dense and table launches of workgroups of 64 and 128 (qs_step64.hip,
// qs_step128.hip).
int launch_step64(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
                  bool with_obs, hipStream_t s, float* rw);
int launch_step128(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
                   bool with_obs, hipStream_t s, float* rw);

// The bucketed launch, and one over a range of its items alone (autotuner
// trials; not in graph mode) (qs_bucket64.hip, qs_bucket128.hip).
void launch_items64(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
                    bool with_obs, hipStream_t s, float* rw);
void launch_items128(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
                     bool with_obs, hipStream_t s, float* rw);
void launch_range64(qs_handle* h, int item0, int count, const float* act, int nsub,
                    const float* goals, float* obs, bool with_obs, hipStream_t s);
void launch_range128(qs_handle* h, int item0, int count, const float* act, int nsub,
                     const float* goals, float* obs, bool with_obs, hipStream_t s);

// The device address of the allocation-free entry point's scratch on device
// dev, which must be current (qs_grad.hip).
int noalloc_scratch(int dev, float** out);

}  // namespace qs_host
