// Step and observation launches of workgroups of 128.
#include "qs_step_launch.h"

int qs_host::launch_step128(qs_handle* h, const float* act, int nsub, const float* goals,
                           float* obs, bool with_obs, hipStream_t s, float* rw) {
  return launch_bs<128>(h, act, nsub, goals, obs, with_obs, s, rw);
}
