// Differentiation entry points of the C ABI: rollouts, their reverse pass and
// the derivative of one step call.
#include <cmath>
#include <cstdlib>
#include <algorithm>
#include <mutex>

#include "qs_handle.h"
#include "qs_rollout.h"

namespace {

using qs_host::aligned;
using qs_host::outputs_overlap;
using qs_host::ptrs;

// ---- differentiable rollouts ------------------------------------------------
// Small batches run the parts of a substep on wavefronts of their own
// (forward_pipe, reverse_pipe_kernel) for as long as their workgroups are
// resident together; QS_ROLLOUT_PIPE, QS_RECOMPUTE_PIPE and QS_REVERSE_PIPE =
// 0/1 force it off/on.  The tape of handles with swarms above 32 holds no
// contact set (tape_word): their backward pass keeps one wavefront.  Measured
// over 40 substeps, us with one wavefront -> with the pipeline:
//  - forward, five wavefronts: 512 workgroups of 8: 122 -> 61, of 32:
//    216 -> 162; 1024: 126 -> 140, 214 -> 326 (a CU holds three);
//    four wavefronts at 1024: 126 -> 85, 214 -> 172; 4096 of 8: equal.  Swarms
//    of one over 200 substeps: 1536: 346 -> 297, 1792: 344 -> 324, 2048: 347 ->
//    354, over 20: 41.0 -> 42.6.  Of 8 with the penalty: 1536: 576 -> 456, 1792:
//    576 -> 509, 2048: 580 -> 563 (without: 421 -> 363, 423 -> 408, 429 -> 470);
//  - recompute (workgroups times segments): 2048: equal, 4096: 466 -> 496 with
//    the sweep behind it;
//  - reverse, two resident on a CU: 512 of 8: 210 -> 127; 1024: 275 -> 300.
int is_wide(const qs_handle* h) { return h->max_n > 32 ? 1 : 0; }
bool pipe(const qs_handle* h, const char* env, bool pays) {
  if (h->Q > 1 << 24) return false;  // a row's byte offsets are 32-bit
  if (const char* e = std::getenv(env)) return e[0] == '1';
  return pays;
}
bool use_rollout_pipe(const qs_handle* h, bool pen) {
  const int limit = h->max_n == 1 ? 1792 : h->uniform_n == 8 && pen ? 2048 : 1024;
  return pipe(h, "QS_ROLLOUT_PIPE", h->nblk <= limit);
}
bool use_noise_wave(const qs_handle* h) { return h->max_n == 1 || h->nblk <= 512; }
bool use_recompute_pipe(const qs_handle* h, int nseg) {
  return !is_wide(h) && pipe(h, "QS_RECOMPUTE_PIPE", (long long)h->nblk * nseg <= 2048);
}
bool use_reverse_pipe(const qs_handle* h) {
  return !is_wide(h) && pipe(h, "QS_REVERSE_PIPE", h->nblk <= 512);
}

template <int BS, int N, bool PEN>
void go_roll(qs_handle* h, const float* act, int ncalls, int nsub, float* ckpt, int ce, float* pen,
             float beta, hipStream_t s) {
  if constexpr (BS == 64) {
    if (use_rollout_pipe(h, PEN)) {
      constexpr int P = PEN ? qs::PEN_SUM : qs::PEN_NONE;
      if (use_noise_wave(h))
        hipLaunchKernelGGL((qs::rollout_pipe_kernel<N, PEN, true>), dim3(h->nblk),
                           dim3(64 * qs::kPipeWaves<P, true>), 0, s, h->d_c, ptrs(h), act, ncalls,
                           nsub, (unsigned long long)h->t, ckpt, ce, pen, beta);
      else
        hipLaunchKernelGGL((qs::rollout_pipe_kernel<N, PEN, false>), dim3(h->nblk),
                           dim3(64 * qs::kPipeWaves<P, false>), 0, s, h->d_c, ptrs(h), act, ncalls,
                           nsub, (unsigned long long)h->t, ckpt, ce, pen, beta);
      return;
    }
  }
  // Pairs have a kernel of their own: the table's loops take four places at a time
  // (131072 quads, 200 substeps, table / own: 435 / 405 us, with the penalty 520 /
  // 432).  Their pipeline is the table's.
  if constexpr (N == 0) {
    if (h->uniform_n == 2) {
      hipLaunchKernelGGL((qs::rollout_kernel<BS, 2, PEN>), dim3(h->nblk), dim3(BS), 0, s, h->d_c,
                         ptrs(h), act, ncalls, nsub, (unsigned long long)h->t, ckpt, ce, pen, beta);
      return;
    }
  }
  hipLaunchKernelGGL((qs::rollout_kernel<BS, N, PEN>), dim3(h->nblk), dim3(BS), 0, s, h->d_c, ptrs(h),
                     act, ncalls, nsub, (unsigned long long)h->t, ckpt, ce, pen, beta);
}

// The arrays of one backward pass: the tape of the chunk of segments in flight
// ([S][31 or 34][Q]) and the caller's state adjoint in, out ([Q][27], may be
// one array) and parameter gradient ([Q][6], accumulated).
struct AdjBuffers {
  float* tape;
  const float* gin;
  float* gout;
  qs::ParSum gpar;
};

template <int BS, int N, bool PEN>
void go_recompute(qs_handle* h, const AdjBuffers& sc, const float* ckpt, const float* act,
                  int ncalls, int ce, int nsub, uint64_t t0, const float* gpen, float beta,
                  hipStream_t s) {
  const int nseg = (ncalls + ce - 1) / ce;
  if constexpr (BS == 64) {
    if (use_recompute_pipe(h, nseg)) {
      constexpr int P = PEN ? qs::PEN_GRAD : qs::PEN_NONE;
      hipLaunchKernelGGL((qs::recompute_pipe_kernel<N, PEN>), dim3(h->nblk, nseg),
                         dim3(64 * qs::kPipeWaves<P, false>), 0, s, h->d_c, ptrs(h), ckpt, act, ncalls, ce,
                         nsub, (unsigned long long)t0, sc.tape, gpen, beta);
      return;
    }
  }
  hipLaunchKernelGGL((qs::recompute_kernel<BS, N, PEN>), dim3(h->nblk, nseg), dim3(BS), 0, s,
                     h->d_c, ptrs(h), ckpt, act, ncalls, ce, nsub, (unsigned long long)t0, sc.tape,
                     is_wide(h), use_reverse_pipe(h) && BS == 64, gpen, beta);
}

template <int BS, int N, bool PEN>
void go_reverse(qs_handle* h, const AdjBuffers& sc, const float* act, int ncalls, int nsub,
                uint64_t t0, float* gact, hipStream_t s) {
  if constexpr (BS == 64) {
    if (use_reverse_pipe(h)) {
      hipLaunchKernelGGL((qs::reverse_pipe_kernel<PEN>), dim3(h->nblk), dim3(448), 0, s, h->d_c,
                         ptrs(h), act, ncalls, nsub, sc.tape, sc.gin, sc.gout, h->uniform_n, gact, sc.gpar,
                         (unsigned long long)t0);
      return;
    }
  }
  hipLaunchKernelGGL((qs::reverse_kernel<BS, N, PEN>), dim3(h->nblk), dim3(BS), 0, s, h->d_c,
                     ptrs(h), act, ncalls, nsub, (unsigned long long)t0, sc.tape, sc.gin,
                     sc.gout, is_wide(h), gact, sc.gpar);
}

// Dispatch on (block size, uniform swarm size) for a launcher template F.
// Callers pass no penalty for swarms of one, which have none.
template <template <int, int, bool> class F, bool PEN, typename... A>
void dispatch(qs_handle* h, A... a) {
  if (h->bs == 128) {
    switch (h->uniform_n) {
      case 1: F<128, 1, false>::run(h, a...); break;
      case 8: F<128, 8, PEN>::run(h, a...); break;
      case 32: F<128, 32, PEN>::run(h, a...); break;
      default: F<128, 0, PEN>::run(h, a...); break;
    }
  } else {
    switch (h->uniform_n) {
      case 1: F<64, 1, false>::run(h, a...); break;
      case 8: F<64, 8, PEN>::run(h, a...); break;
      case 32: F<64, 32, PEN>::run(h, a...); break;
      default: F<64, 0, PEN>::run(h, a...); break;
    }
  }
}

template <int BS, int N, bool PEN>
struct RollF {
  static void run(qs_handle* h, const float* act, int ncalls, int nsub, float* ckpt, int ce,
                  float* pen, float beta, hipStream_t s) {
    go_roll<BS, N, PEN>(h, act, ncalls, nsub, ckpt, ce, pen, beta, s);
  }
};

template <int BS, int N, bool PEN>
struct RecF {
  static void run(qs_handle* h, const AdjBuffers* sc, const float* ckpt, const float* act,
                  int ncalls, int ce, int nsub, uint64_t t0, const float* gpen, float beta,
                  hipStream_t s) {
    go_recompute<BS, N, PEN>(h, *sc, ckpt, act, ncalls, ce, nsub, t0, gpen, beta, s);
  }
};

template <int BS, int N, bool PEN>
struct RevF {
  static void run(qs_handle* h, const AdjBuffers* sc, const float* act, int ncalls, int nsub,
                  uint64_t t0, float* gact, hipStream_t s) {
    go_reverse<BS, N, PEN>(h, *sc, act, ncalls, nsub, t0, gact, s);
  }
};

int grow(float** p, size_t* cap, size_t need) {
  if (need <= *cap && *p) return QS_OK;
  (void)hipFree(*p);
  *p = nullptr;
  *cap = 0;
  if (hipMalloc((void**)p, need * sizeof(float)) != hipSuccess) {
    *p = nullptr;
    return QS_ERR_NOMEM;
  }
  *cap = need;
  return QS_OK;
}

// Bytes of tape the backward pass may hold at once (QS_TAPE_BYTES overrides);
// at least one segment is always taped.
size_t tape_budget() {
  if (const char* e = std::getenv("QS_TAPE_BYTES")) {
    const long long b = std::atoll(e);
    if (b > 0) return (size_t)b;
  }
  return (size_t)8 << 30;
}

// Floats of tape one checkpoint segment needs.
size_t segment_tape_floats(const qs_handle* h, int n_calls, int nsub, int ce, bool pen) {
  return (size_t)std::min(ce, n_calls) * nsub * (pen ? qs::kTapeRows<true> : qs::kTapeRows<false>) *
         h->Q;
}

// Backward pass over n_calls calls with checkpoints every ce calls (ckpt:
// [27][Q] each); sc.tape holds G segments.  Segments are taken in chunks of G,
// last chunk first: one launch recomputes every segment of the chunk in
// parallel, one launch sweeps the chunk in reverse.
int run_adjoint(qs_handle* h, AdjBuffers sc, int G, const float* act, int n_calls,
                int nsub, int ce, const float* ckpt, uint64_t t0, const float* gpen, float beta,
                float* gact, hipStream_t s) {
  const int nseg = (n_calls + ce - 1) / ce;
  for (int hi = nseg; hi > 0; hi -= G) {
    const int g0 = std::max(0, hi - G);
    sc.gpar.first = hi == nseg;
    sc.gpar.last = g0 == 0;
    const int c0 = g0 * ce, nc = std::min(n_calls, hi * ce) - c0;
    const float* ck = ckpt + (size_t)g0 * qs::NSTATE * h->Q;
    const float* a = act + (size_t)c0 * h->Q * 4;
    float* ga = gact + (size_t)c0 * h->Q * 4;
    const uint64_t ts = t0 + (uint64_t)c0 * nsub;
    if (gpen) {
      dispatch<RecF, true>(h, &sc, ck, a, nc, ce, nsub, ts, gpen, beta, s);
      dispatch<RevF, true>(h, &sc, a, nc, nsub, ts, ga, s);
    } else {
      dispatch<RecF, false>(h, &sc, ck, a, nc, ce, nsub, ts, gpen, beta, s);
      dispatch<RevF, false>(h, &sc, a, nc, nsub, ts, ga, s);
    }
    if (hipGetLastError() != hipSuccess) return QS_ERR_HIP;
    sc.gin = sc.gout;  // the next chunk goes on from here
  }
  return QS_OK;
}

// Argument checks shared by the two forms of qs_step_backward.
int check_step_backward(const qs_handle* h, const float* d_state_in, const float* d_actions,
                        int32_t n_substeps, const float* d_gstate_out, const float* d_gstate_in,
                        const float* d_gactions, const float* d_gparams) {
  if (!h || !d_state_in || !d_actions || !d_gstate_out || !d_gstate_in || !d_gactions ||
      !d_gparams)
    return QS_ERR_NULL;
  if (n_substeps < 0) return QS_ERR_INVALID;
  if (h->c.flags & qs::F_DOWNWASH) return QS_ERR_UNSUPPORTED;
  if (!aligned(d_actions, 16) || !aligned(d_gactions, 16) || !aligned(d_state_in, 4) ||
      !aligned(d_gstate_out, 4) || !aligned(d_gstate_in, 4) || !aligned(d_gparams, 4))
    return QS_ERR_ALIGN;
  // d_gstate_in may be d_gstate_out itself (a workgroup has read its rows before it
  // writes them), not a part of it
  const size_t Q = (size_t)h->Q;
  const bool same = d_gstate_in == d_gstate_out;
  if (outputs_overlap({{d_gstate_in, Q * 108}, {d_gactions, Q * 16}, {d_gparams, Q * 24}},
                      {{d_state_in, Q * 108}, {d_actions, Q * 16},
                       {same ? nullptr : d_gstate_out, Q * 108}}))
    return QS_ERR_INVALID;
  return QS_OK;
}

// One qs_step_backward call: up to VJP_MAX_SUBSTEPS substeps in one launch; more
// through the recompute and reverse sweeps of one segment, with ck1 [27][Q]
// for the state before the call.  (us a call with eight launches -> one, for 1,
// 2 and 4 substeps: 512 x 8: 23 -> 8.4, 25 -> 11, 30 -> 17; 4096 x 8: 36 -> 9.4,
// 40 -> 13, 46 -> 19; 32768 x 8: 113 -> 25, 127 -> 34, 190 -> 75.  Five, by the
// sweeps, take 19, 26 and 93: more substeps in one launch lose to the pipelines
// in the smallest batches and to their own LDS in the largest.)
bool one_launch(const qs_handle* h, int nsub) {
  return h->bs == 64 && nsub >= 1 && nsub <= qs::VJP_MAX_SUBSTEPS;
}

template <int N>
void go_step_vjp(qs_handle* h, const AdjBuffers& b, const float* state_in, const float* act,
                 int nsub, uint64_t t0, float* gact, hipStream_t s) {
  const size_t dyn = (size_t)(nsub - 1) * qs::VJP_ROW * 64 * sizeof(float);
  hipLaunchKernelGGL((qs::step_vjp_kernel<N>), dim3(h->nblk), dim3(64), dyn, s, h->d_c, ptrs(h),
                     state_in, act, nsub, (unsigned long long)t0, b.gin, b.gout, gact, b.gpar.out);
}

int step_backward_run(qs_handle* h, float* tape, float* ck1, const float* d_state_in,
                      const float* d_actions, int32_t n_substeps, uint64_t substep_index,
                      const float* d_gstate_out, float* d_gstate_in, float* d_gactions,
                      float* d_gparams, hipStream_t s) {
  const AdjBuffers b{tape, d_gstate_out, d_gstate_in, {d_gparams, nullptr, true, true}};
  if (one_launch(h, n_substeps)) {
    switch (h->uniform_n) {
      case 1: go_step_vjp<1>(h, b, d_state_in, d_actions, n_substeps, substep_index, d_gactions, s); break;
      case 8: go_step_vjp<8>(h, b, d_state_in, d_actions, n_substeps, substep_index, d_gactions, s); break;
      case 32: go_step_vjp<32>(h, b, d_state_in, d_actions, n_substeps, substep_index, d_gactions, s); break;
      default: go_step_vjp<0>(h, b, d_state_in, d_actions, n_substeps, substep_index, d_gactions, s); break;
    }
  } else if (n_substeps > 0) {
    hipLaunchKernelGGL(qs::rows_to_fields_kernel, dim3((h->Q + 63) / 64), dim3(64), 0, s,
                       d_state_in, ck1, h->Q);
    return run_adjoint(h, b, 1, d_actions, 1, n_substeps, 1, ck1, substep_index, nullptr, 0.f,
                       d_gactions, s);
  } else {  // kernels, not memory operations, so the sequence can be captured
    hipLaunchKernelGGL(qs::fill_kernel, dim3((unsigned)((4LL * h->Q + 255) / 256)), dim3(256), 0,
                       s, d_gactions, 4LL * h->Q, 0.0f);
    const long long n = (long long)qs::NSTATE * h->Q;
    if (d_gstate_in != d_gstate_out)
      hipLaunchKernelGGL(qs::copy_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s,
                         d_gstate_out, d_gstate_in, n);
  }
  return hipGetLastError() == hipSuccess ? QS_OK : QS_ERR_HIP;
}

// ---- fixed scratch of the allocation-free entry point -------------------
// qs_step_backward_noalloc keeps its scratch in this array instead of
// allocating: 64 MiB, one copy on every device the library runs on, held
// until the process ends.  Host code never uses the array's name as an
// address (on the host it names a stand-in, not device memory): the device
// address comes from hipGetSymbolAddress, looked up once per device with
// that device current, and only that pointer is passed to kernels.
}  // namespace

constexpr size_t kNoAllocScratchFloats = (size_t)QS_NOALLOC_SCRATCH_BYTES / sizeof(float);
static __device__ __align__(256) float scratch[kNoAllocScratchFloats];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[kMaxDevices] = {};

}  // namespace

// The device address of the scratch array on device dev (which must be
// current), looked up on first use and kept.
int qs_host::noalloc_scratch(int dev, float** out) {
  if (dev < 0 || dev >= kMaxDevices) return QS_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return QS_ERR_HIP;
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return QS_OK;
}



using qs_host::noalloc_scratch;

extern "C" {

int qs_rollout(qs_handle* h, const float* d_actions, int32_t n_calls, int32_t n_substeps,
               int32_t ckpt_every, float* d_ckpt, float* d_penalty, float beta, void* stream) {
  if (!h || !d_actions) return QS_ERR_NULL;
  if (n_calls < 0 || n_substeps < 0) return QS_ERR_INVALID;
  if (d_ckpt && ckpt_every < 1) return QS_ERR_INVALID;
  if (d_penalty && !(beta > 0.f && std::isfinite(beta))) return QS_ERR_INVALID;
  if (!aligned(d_actions, 16) || (d_ckpt && !aligned(d_ckpt, 4)) ||
      (d_penalty && !aligned(d_penalty, 4)))
    return QS_ERR_ALIGN;
  if (n_calls == 0 || n_substeps == 0) return QS_OK;
  {
    const size_t Q = (size_t)h->Q, n_ck = d_ckpt ? (n_calls + ckpt_every - 1) / ckpt_every : 0;
    if (outputs_overlap({{d_ckpt, n_ck * qs::NSTATE * Q * 4}, {d_penalty, Q * 4}},
                        {{d_actions, (size_t)n_calls * Q * 16}}))
      return QS_ERR_INVALID;
  }
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  hipStream_t s = (hipStream_t)stream;
  if (h->max_n == 1) d_penalty = nullptr;  // swarms of one have no penalty
  if (d_penalty)
    dispatch<RollF, true>(h, d_actions, (int)n_calls, (int)n_substeps, d_ckpt, (int)ckpt_every,
                          d_penalty, beta, s);
  else
    dispatch<RollF, false>(h, d_actions, (int)n_calls, (int)n_substeps, d_ckpt,
                           (int)std::max(ckpt_every, 1), d_penalty, beta, s);
  if (hipGetLastError() != hipSuccess) return QS_ERR_HIP;
  h->t += (uint64_t)n_calls * (uint64_t)n_substeps;
  return QS_OK;
}

int qs_rollout_backward(qs_handle* h, const float* d_actions, int32_t n_calls,
                        int32_t n_substeps, int32_t ckpt_every, const float* d_ckpt,
                        uint64_t substep_index0, float* d_gstate, const float* d_gpenalty,
                        float beta, float* d_gactions, float* d_gparams, void* stream) {
  if (!h || !d_actions || !d_ckpt || !d_gstate || !d_gactions || !d_gparams) return QS_ERR_NULL;
  if (n_calls < 0 || n_substeps < 0 || ckpt_every < 1) return QS_ERR_INVALID;
  if (h->c.flags & qs::F_DOWNWASH) return QS_ERR_UNSUPPORTED;
  if (d_gpenalty && !(beta > 0.f && std::isfinite(beta))) return QS_ERR_INVALID;
  if (!aligned(d_actions, 16) || !aligned(d_gactions, 16) || !aligned(d_ckpt, 4) ||
      !aligned(d_gstate, 4) || !aligned(d_gparams, 4) || (d_gpenalty && !aligned(d_gpenalty, 4)))
    return QS_ERR_ALIGN;
  {
    const size_t Q = (size_t)h->Q, nc = (size_t)std::max(n_calls, 0);
    const size_t n_ck = (nc + ckpt_every - 1) / ckpt_every;
    if (outputs_overlap({{d_gactions, nc * Q * 16}, {d_gparams, Q * 24}, {d_gstate, Q * 108}},
                        {{d_actions, nc * Q * 16}, {d_ckpt, n_ck * qs::NSTATE * Q * 4},
                         {d_gpenalty, Q * 4}}))
      return QS_ERR_INVALID;
  }
  if (n_calls == 0 || n_substeps == 0) return QS_OK;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  if (h->max_n == 1) d_gpenalty = nullptr;  // swarms of one have no penalty
  hipStream_t s = (hipStream_t)stream;
  // segments per chunk: as many as fit the tape budget (also the recompute
  // grid's y extent, at most 65535), at least one
  const int nseg = (n_calls + ckpt_every - 1) / ckpt_every;
  const size_t seg = segment_tape_floats(h, n_calls, n_substeps, ckpt_every, d_gpenalty != nullptr);
  const size_t fit = tape_budget() / (seg * sizeof(float));
  const int G = (int)std::max<size_t>(1, std::min<size_t>({(size_t)nseg, fit, (size_t)65535}));
  int rc = grow(&h->d_tape, &h->tape_cap, (size_t)G * seg);
  if (rc != QS_OK) return rc;
  if (G < nseg) rc = grow(&h->d_gsum, &h->gsum_cap, (size_t)6 * h->Q);
  if (rc != QS_OK) return rc;
  const AdjBuffers b{h->d_tape, d_gstate, d_gstate, {d_gparams, h->d_gsum, true, true}};
  return run_adjoint(h, b, G, d_actions, n_calls, n_substeps, ckpt_every, d_ckpt, substep_index0,
                   d_gpenalty, beta, d_gactions, s);
}

int qs_step_backward(qs_handle* h, const float* d_state_in, const float* d_actions,
                     int32_t n_substeps, uint64_t substep_index, const float* d_gstate_out,
                     float* d_gstate_in, float* d_gactions, float* d_gparams, void* stream) {
  int rc = check_step_backward(h, d_state_in, d_actions, n_substeps, d_gstate_out, d_gstate_in,
                               d_gactions, d_gparams);
  if (rc != QS_OK) return rc;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  if (n_substeps > 0 && !one_launch(h, n_substeps)) {
    rc = grow(&h->d_tape, &h->tape_cap, segment_tape_floats(h, 1, n_substeps, 1, false));
    if (rc == QS_OK) rc = grow(&h->d_ck1, &h->ck1_cap, (size_t)qs::NSTATE * h->Q);
    if (rc != QS_OK) return rc;
  }
  return step_backward_run(h, h->d_tape, h->d_ck1, d_state_in, d_actions, n_substeps, substep_index,
                           d_gstate_out, d_gstate_in, d_gactions, d_gparams, (hipStream_t)stream);
}

int qs_step_backward_noalloc(qs_handle* h, const float* d_state_in, const float* d_actions,
                             int32_t n_substeps, uint64_t substep_index,
                             const float* d_gstate_out, float* d_gstate_in, float* d_gactions,
                             float* d_gparams, void* stream) {
  int rc = check_step_backward(h, d_state_in, d_actions, n_substeps, d_gstate_out, d_gstate_in,
                               d_gactions, d_gparams);
  if (rc != QS_OK) return rc;
  // The limit is the interface's, which callers plan by: a state, an adjoint, a
  // parameter gradient and the tape, each rounded up to 64 floats (256 bytes).
  // In use are the state and the tape, and neither where one launch does it all.
  auto part = [](size_t n) { return (n + 63) / 64 * 64; };
  const size_t Q = (size_t)h->Q;
  const size_t n_ck = part(qs::NSTATE * Q);
  const size_t n_tape = n_substeps > 0 ? part(segment_tape_floats(h, 1, n_substeps, 1, false)) : 0;
  if (2 * n_ck + part(6 * Q) + n_tape > kNoAllocScratchFloats) return QS_ERR_TOO_LARGE;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  float* base = nullptr;
  rc = noalloc_scratch(h->dev, &base);
  if (rc != QS_OK) return rc;
  return step_backward_run(h, base + n_ck, base, d_state_in, d_actions, n_substeps, substep_index,
                           d_gstate_out, d_gstate_in, d_gactions, d_gparams, (hipStream_t)stream);
}

}  // extern "C"
