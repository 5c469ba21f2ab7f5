// Bucketed launches of workgroups of 64.
#include "qs_bucket_launch.h"

void qs_host::launch_items64(qs_handle* h, const float* act, int nsub, const float* goals,
                             float* obs, bool with_obs, hipStream_t s, float* rw) {
  items_bs<64>(h, act, nsub, goals, obs, with_obs, s, rw);
}

void qs_host::launch_range64(qs_handle* h, int item0, int count, const float* act, int nsub,
                             const float* goals, float* obs, bool with_obs, hipStream_t s) {
  range_bs<64>(h, item0, count, act, nsub, goals, obs, with_obs, s);
}
