// Differentiable rollouts: a multi-call forward kernel (a fresh action per
// call, checkpoints of the state, the smoothed collision penalty) and the
// backward pass: a kernel that recomputes checkpoint segments in parallel,
// taping what the reverse sweep needs of each substep, and a kernel that
// sweeps the tape in reverse.
//
// Layouts: checkpoints are field-major [27][Q], tape rows [31][Q] or, with the
// penalty, [34][Q] (coalesced per field); the state's adjoint is the caller's
// row-major [Q][27], the parameters' [Q][6]; actions and their gradients are
// [call][Q][4].
#pragma once
#include "qs_adjoint.h"

namespace qs {

// Workgroup -> quads mapping shared by the kernels (see step_kernel).
template <int BS, int N>
__device__ __forceinline__ void block_map(const Ptrs& p, int tid, int& qb, int& cnt, int& ls,
                                          int& n) {
  if constexpr (N > 0) {
    qb = blockIdx.x * BS;
    cnt = min(BS, p.Q - qb);
    ls = (tid / N) * N;
    n = N;
  } else {
    const int2 bq = p.blk[blockIdx.x];
    qb = bq.x;
    cnt = bq.y;
    const uint32_t swd = tid < cnt ? p.sw[qb + tid] : 0u;
    ls = (int)(swd >> 8);
    n = (int)(swd & 0xffu);
  }
}

__device__ __forceinline__ void load_state(const float* __restrict__ S, long long ld, int q,
                                           Quad& s) {
#pragma unroll
  for (int k = 0; k < 3; ++k) s.x[k] = S[(S_X + k) * ld + q];
#pragma unroll
  for (int k = 0; k < 3; ++k) s.v[k] = S[(S_V + k) * ld + q];
#pragma unroll
  for (int k = 0; k < 9; ++k) s.R[k] = S[(S_R + k) * ld + q];
#pragma unroll
  for (int k = 0; k < 3; ++k) s.w[k] = S[(S_W + k) * ld + q];
#pragma unroll
  for (int k = 0; k < 4; ++k) s.u[k] = S[(S_U + k) * ld + q];
#pragma unroll
  for (int k = 0; k < 4; ++k) s.e[k] = S[(S_E + k) * ld + q];
  s.fl = S[S_F * ld + q];
  s.ev = 0u;
}

__device__ __forceinline__ void store_state(float* __restrict__ S, long long ld, int q,
                                            const Quad& s) {
#pragma unroll
  for (int k = 0; k < 3; ++k) S[(S_X + k) * ld + q] = s.x[k];
#pragma unroll
  for (int k = 0; k < 3; ++k) S[(S_V + k) * ld + q] = s.v[k];
#pragma unroll
  for (int k = 0; k < 9; ++k) S[(S_R + k) * ld + q] = s.R[k];
#pragma unroll
  for (int k = 0; k < 3; ++k) S[(S_W + k) * ld + q] = s.w[k];
#pragma unroll
  for (int k = 0; k < 4; ++k) S[(S_U + k) * ld + q] = s.u[k];
#pragma unroll
  for (int k = 0; k < 4; ++k) S[(S_E + k) * ld + q] = s.e[k];
  S[S_F * ld + q] = s.fl;
}

// The same in the handle's tiles.
__device__ __forceinline__ void load_handle_state(const float* __restrict__ st, int q, Quad& s) {
  float f[NSTATE];
#pragma unroll
  for (int k = 0; k < NSTATE; ++k) f[k] = st[st_index(q, k)];
  load_state(f, 1, 0, s);
}
__device__ __forceinline__ void store_handle_state(float* __restrict__ st, int q, const Quad& s) {
  float f[NSTATE];
  store_state(f, 1, 0, s);
#pragma unroll
  for (int k = 0; k < NSTATE; ++k) st[st_index(q, k)] = f[k];
}

// A tape row: the state at the start of a substep (27 fields, the resting flag
// as part of a word, below), with the penalty its adjoint w.r.t. the position after
// the motion (3 fields), and the motor-noise draws of that substep (4 fields, for
// the reverse pipeline only: reverse_kernel draws again).  The
// recompute passes over the partners anyway, at twice the reverse sweep's occupancy
// and bound by the tape's stores, so it is the place for what the partners add; the
// sweep had passed over them again (32768 x 32, 100 substeps: recompute 3.44 -> 3.82,
// sweep 5.71 -> 4.16 ms).
//
// The quads of a workgroup lie together (kTapeRows words each), in groups of
// four fields of one quad, so that a substep writes and reads eight kilobytes in a
// row, 16 bytes a lane.  (Field by field over all quads, every wavefront went
// to thirty places megabytes apart: the same case 9.77 ms, by workgroup 9.43; the
// groups of four are equal there, and 2048 swarms of 1 to 16 go from 436 to 432 us.)
template <bool PEN>
constexpr int kTapeRows = NSTATE + 4 + (PEN ? 3 : 0);
// Fields in groups of four: u, e, R[0..3], R[4..7], R[8] and w, x and v[0]; then
// the word and the penalty's (PEN), the draws, the pair v[1..2], the word (no PEN).
template <bool PEN>
constexpr int T_DRAW = PEN ? 28 : 24;
template <bool PEN>
constexpr int T_V12 = T_DRAW<PEN> + 4;
template <bool PEN>
constexpr int T_WORD = PEN ? 24 : 30;
typedef float tape4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float tape2 __attribute__((ext_vector_type(2), aligned(4)));
// The quad's group of four, pair or word of the part of a row that holds the
// workgroup's cnt quads; group: the words of a quad before it.
template <typename T, typename F>
__device__ __forceinline__ auto& tape_at(F* part, int group, int cnt, int tid) {
  using C = typename std::conditional<std::is_const<F>::value, const T, T>::type;
  return reinterpret_cast<C*>(part + (unsigned)(group * cnt))[(unsigned)tid];
}
template <typename F>
__device__ __forceinline__ auto& tape_four(F* part, int group, int cnt, int tid) {
  return tape_at<tape4>(part, group, cnt, tid);
}
// The word: with the penalty's, the first of its group.
template <bool PEN, typename F>
__device__ __forceinline__ auto& tape_word_at(F* part, int cnt, int tid) {
  return tape_at<float>(part, T_WORD<PEN>, cnt, PEN ? 4 * tid : tid);
}

// A large batch's tape is past the caches before it is read, and then read once:
// non-temporal (32768 x 32, 100 substeps: 9.30 -> 9.10 ms; 8192 x 8, 40: 348 -> 341
// us; 32768 x 8: 982 -> 941; 131072 single quads: 425 -> 408).
template <typename T>
__device__ __forceinline__ void tape_put(T& at, T v) {
  __builtin_nontemporal_store(v, &at);
}
template <typename T>
__device__ __forceinline__ T tape_get(const T& at) {
  return __builtin_nontemporal_load(&at);
}

template <bool PEN>
__device__ __forceinline__ void tape_store_state(float* part, int cnt, int tid, const Quad& s) {
  tape_put(tape_four(part, 0, cnt, tid), tape4{s.u[0], s.u[1], s.u[2], s.u[3]});
  tape_put(tape_four(part, 4, cnt, tid), tape4{s.e[0], s.e[1], s.e[2], s.e[3]});
  tape_put(tape_four(part, 8, cnt, tid), tape4{s.R[0], s.R[1], s.R[2], s.R[3]});
  tape_put(tape_four(part, 12, cnt, tid), tape4{s.R[4], s.R[5], s.R[6], s.R[7]});
  tape_put(tape_four(part, 16, cnt, tid), tape4{s.R[8], s.w[0], s.w[1], s.w[2]});
  tape_put(tape_four(part, 20, cnt, tid), tape4{s.x[0], s.x[1], s.x[2], s.v[0]});
  tape_put(tape_at<tape2>(part, T_V12<PEN>, cnt, tid), tape2{s.v[1], s.v[2]});
}

// The state (s.fl: the word) and the penalty's adjoint (PEN).
template <bool PEN>
__device__ __forceinline__ void tape_load(const float* part, int cnt, int tid, Quad& s,
                                          float pen3[3]) {
  auto four = [&](int group) { return tape_get(tape_four(part, group, cnt, tid)); };
  const tape4 u = four(0), e = four(4), a = four(8), b = four(12), d = four(16), x = four(20);
  const tape2 v = tape_get(tape_at<tape2>(part, T_V12<PEN>, cnt, tid));
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    s.u[k] = u[k];
    s.e[k] = e[k];
    s.R[k] = a[k];
    s.R[4 + k] = b[k];
  }
  s.R[8] = d[0];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    s.w[k] = d[1 + k];
    s.x[k] = x[k];
  }
  s.v[0] = x[3];
  s.v[1] = v[0];
  s.v[2] = v[1];
  s.ev = 0u;
  if constexpr (PEN) {
    const tape4 w = four(T_WORD<PEN>);
    s.fl = w[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) pen3[k] = w[1 + k];
  } else {
    s.fl = tape_get(tape_word_at<PEN>(part, cnt, tid));
  }
}

// The word in the resting flag's field: the partners whose collision response
// the quad received in the substep, and, on the quad's own place, the resting
// flag.  Handles with swarms above 32 (wide) keep the flag alone, in bit 0,
// and the sweep finds their contacts again.
__device__ __forceinline__ float tape_word(float fl, unsigned long long resp, int me, int wide) {
  const uint32_t f = fl != 0.f ? 1u : 0u;
  return __uint_as_float(wide ? f : (uint32_t)resp | f << me);
}
__device__ __forceinline__ float word_flag(uint32_t w, int me, int wide) {
  return (wide ? w : w >> me) & 1u ? 1.f : 0.f;
}
__device__ __forceinline__ uint32_t word_resp(uint32_t w, int me, int wide) {
  return wide ? 0u : w & ~(1u << me);
}

__device__ __forceinline__ void load_params(const Ptrs& p, const Consts& c, int q, QuadPar& pp,
                                            ParAdj& pa) {
  load_forward_params(p, q, pp);
  pp.inv_m = 1.0f / pp.m;
  pp.ijx = 1.0f / pp.jx;
  pp.ijy = 1.0f / pp.jy;
  pp.ijz = 1.0f / pp.jz;
  pp.a_ns = c.ns_scale * pp.f_max;
  pa.m = pp.m;
  const v2f b = *reinterpret_cast<const v2f*>(p.par + par_index(q, P_T2W));
  pa.t2w = b[0];
  const float tau = b[1];
  pa.dlag_dtau = -(1.0f - pp.a_lag) * c.dt / (tau * tau);
}

// The action row of quad q for one call.  The multi-call kernels load it a
// call ahead, so the load's latency overlaps the previous call's substeps
// instead of stalling every call.
__device__ __forceinline__ float4 load_act(const float* act, int q) {
  return reinterpret_cast<const float4*>(act)[q];
}

// Rotor commands of an action row; a non-finite action sets the sticky
// error bit.
__device__ __forceinline__ void act_uhat(const Consts& c, const Ptrs& p, const float4& a4,
                                         float uhat[4]) {
  const bool unit = (c.flags & F_ACT_UNIT) != 0;
  uhat[0] = rotor_cmd(a4.x, unit);
  uhat[1] = rotor_cmd(a4.y, unit);
  uhat[2] = rotor_cmd(a4.z, unit);
  uhat[3] = rotor_cmd(a4.w, unit);
  if (!(isfinite(a4.x) && isfinite(a4.y) && isfinite(a4.z) && isfinite(a4.w)))
    __hip_atomic_fetch_or(p.err, ERRBIT_ACTION, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// d uhat / d a for one action component (0 where the clip is active or the
// command is zero).
__device__ __forceinline__ float duhat_da(const Consts& c, float a, float uhat) {
  if (!(uhat > 0.f)) return 0.f;
  if (c.flags & F_ACT_UNIT) return (a > 0.f && a < 1.f) ? 0.5f / uhat : 0.f;
  return (a > -1.f && a < 1.f) ? 0.25f / uhat : 0.f;
}

// ---------------------------------------------------------------------------
// Forward rollout: ncalls calls of nsub substeps from the handle's state,
// action of call k at act + k Q 4.  ckpt (optional): the state at the start
// of every ckpt_every-th call, checkpoint k at ckpt + k 27 Q.  pen
// (optional, PEN): each quad's share of the smoothed collision penalty,
// sum over substeps and env-mates of softplus(beta (d_col - d))/(2 beta).
// Bound by instruction issue, in small batches by its chain.  Four wavefronts a
// SIMD, three for swarms of 8, which then hold eight partners a chunk (with the
// penalty 168 registers; four a chunk, 142: 98304 / 262144 / 524288 quads, 50
// substeps, 160 / 274 / 473 -> 152 / 261 / 456 us) and spill nothing (without, at
// four: six registers; 118 / 196 / 340 -> 116 / 202 / 334).
// ---------------------------------------------------------------------------
template <int BS, int N, bool PEN>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(N == 8 ? 3 : 4))) void rollout_kernel(const Consts* __restrict__ cp, Ptrs p,
                                                     const float* __restrict__ act, int ncalls,
                                                     int nsub, unsigned long long t0,
                                                     float* __restrict__ ckpt, int ckpt_every,
                                                     float* __restrict__ pen, float beta) {
  __shared__ __align__(16) float sxv[2][TILE_ROWS_CO][BS];
  const Consts& c = *cp;
  const int tid = threadIdx.x;
  int qb, cnt, ls, n;
  block_map<BS, N>(p, tid, qb, cnt, ls, n);
  const bool live = tid < cnt;
  const int q = qb + (live ? tid : 0);
  const int me = tid - ls;
  const long long Q = p.Q;

  Quad s;
  QuadPar pp;
  ParAdj pa;
  if (live) {
    load_handle_state(p.st, q, s);
    load_params(p, c, q, pp, pa);
  }
  const bool pairs = N != 1 && ((c.flags & (F_COLLIDE | F_DOWNWASH)) != 0 || PEN);
  constexpr int P = PEN ? PEN_SUM : PEN_NONE;
  Pen pn;
  if constexpr (PEN) pn = make_pen(c, beta, N > 0 ? N : wave_max(live ? n : 0));
  int sidx = 0;
  float4 a_nx = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live && ncalls > 0) a_nx = load_act(act, q);
  for (int call = 0; call < ncalls; ++call) {
    const float4 a4 = a_nx;
    if (live && call + 1 < ncalls) a_nx = load_act(act + (long long)(call + 1) * Q * 4, q);
    if (ckpt && call % ckpt_every == 0 && live)
      store_state(ckpt + (long long)(call / ckpt_every) * NSTATE * Q, Q, q, s);
    float uhat[4] = {0.f, 0.f, 0.f, 0.f};
    if (live) act_uhat(c, p, a4, uhat);
    for (int sub = 0; sub < nsub; ++sub, ++sidx) {
      const unsigned long long t = t0 + (unsigned long long)sidx;
      if (live) quad_substep(c, pp, s, uhat, (uint32_t)q, t);
      if (pairs) {
        float(*tile)[BS] = sxv[sidx & 1];
        if constexpr (N == 8 && P == PEN_NONE) {
          lane_pair_pass<BS, N, true>(c, tile, s, live, ls, n, me, tid, (uint32_t)q, t);
        } else {
          constexpr bool SCREEN = N != 2;  // (one partner: no more than the exact test)
          if (live) put_tile<N, SCREEN>(tile, tid, s);
          __syncthreads();
          if (live) pair_pass<BS, N, P, SCREEN>(c, tile, s, ls, n, me, (uint32_t)q, t, &pn);
        }
      }
    }
  }
  if (live) {
    store_handle_state(p.st, q, s);
    float chk = 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) chk += s.x[k] + s.v[k] + s.w[k];
#pragma unroll
    for (int k = 0; k < 9; ++k) chk += s.R[k];
    if (!isfinite(chk))
      __hip_atomic_fetch_or(p.err, ERRBIT_STATE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (PEN) pen[q] += pn.acc[0];
  }
}

// ---------------------------------------------------------------------------
// Backward pass of a rollout, two launches per chunk of checkpoint segments
// (a segment: ce calls from one checkpoint).
//
// recompute_kernel, grid (workgroups, segments of the chunk): workgroup
// (b, g) re-runs segment g of the chunk from its checkpoint ckpt + g 27 Q
// and tapes the chunk's k-th substep in row k (the reverse sweep then re-runs
// the substep without regenerating the draws and without a pass over the
// partners).  Given the checkpoints the segments are independent, so a chunk
// is recomputed in one parallel launch.
//  act: the chunk's first call; ncalls: calls in the chunk; t0: substep
//  index of the chunk's first substep; wide: see tape_word; draws: the sweep
//  reads them from the tape; gpen: dL/d pen (PEN).
// ---------------------------------------------------------------------------
template <int BS, int N, bool PEN>
__global__ __launch_bounds__(BS) __attribute__((amdgpu_waves_per_eu(N == 8 && PEN ? 3 : 4))) void recompute_kernel(const Consts* __restrict__ cp, Ptrs p,
                                                       const float* __restrict__ ckpt,
                                                       const float* __restrict__ act, int ncalls,
                                                       int ce, int nsub, unsigned long long t0,
                                                       float* __restrict__ tape, int wide,
                                                       int draws,
                                                       const float* __restrict__ gpen,
                                                       float beta) {
  constexpr int P = PEN ? PEN_GRAD : PEN_NONE, NTAPE = kTapeRows<PEN>;
  __shared__ __align__(16) float sxv[2][PEN ? PENROW + 1 : TILE_ROWS_CO][BS];
  const Consts& c = *cp;
  const int tid = threadIdx.x;
  int qb, cnt, ls, n;
  block_map<BS, N>(p, tid, qb, cnt, ls, n);
  const bool live = tid < cnt;
  const int q = qb + (live ? tid : 0);
  const int me = tid - ls;
  const long long Q = p.Q;
  const int c0 = blockIdx.y * ce;
  const int nc = min(ce, ncalls - c0);
  const bool pairs = N != 1 && (PEN || (c.flags & (F_COLLIDE | F_DOWNWASH)) != 0);

  Quad s;
  QuadPar pp;
  ParAdj pa;
  Pen pn;
  if constexpr (PEN) {
    const float h_me = live ? -0.5f * gpen[q] : 0.f;
    sxv[0][PENROW][tid] = h_me;
    sxv[1][PENROW][tid] = h_me;
    pn = make_pen(c, beta, N > 0 ? N : wave_max(live ? n : 0), h_me);
  }
  if (live) {
    load_state(ckpt + (long long)blockIdx.y * NSTATE * Q, Q, q, s);
    load_params(p, c, q, pp, pa);
  }
  int sidx = c0 * nsub;
  float4 a_nx = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live && nc > 0) a_nx = load_act(act + (long long)c0 * Q * 4, q);
  for (int call = c0; call < c0 + nc; ++call) {
    const float4 a4 = a_nx;
    if (live && call + 1 < c0 + nc) a_nx = load_act(act + (long long)(call + 1) * Q * 4, q);
    float uhat[4] = {0.f, 0.f, 0.f, 0.f};
    if (live) act_uhat(c, p, a4, uhat);
    for (int sub = 0; sub < nsub; ++sub, ++sidx) {
      const unsigned long long t = t0 + (unsigned long long)sidx;
      float* row = tape + ((long long)sidx * Q + qb) * NTAPE;
      const float fl0 = s.fl;
      unsigned long long resp = 0ull;
      if (live) {
        tape_store_state<PEN>(row, cnt, tid, s);
        float z[4];
        quad_substep<false, Z_EXPORT>(c, pp, s, uhat, (uint32_t)q, t, nullptr, z);
        if (draws && (c.flags & F_NOISE))
          tape_four(row, T_DRAW<PEN>, cnt, tid) = tape4{z[0], z[1], z[2], z[3]};
      }
      if (pairs) {
        float(*tile)[BS] = sxv[sidx & 1];
        if constexpr (N == 8 && !PEN) {
          lane_pair_pass<BS, N, true>(c, tile, s, live, ls, n, me, tid, (uint32_t)q, t, &resp);
        } else {
          if (live) put_tile<N, true>(tile, tid, s);
          __syncthreads();
          if (live) {
            if constexpr (PEN) pn.acc[0] = pn.acc[1] = pn.acc[2] = 0.f;
            pair_pass<BS, N, P, true>(c, tile, s, ls, n, me, (uint32_t)q, t, &pn, nullptr, &resp);
          }
        }
      }
      if (live) {
        const float word = tape_word(fl0, resp, me, wide);
        if constexpr (PEN)
          tape_put(tape_four(row, T_WORD<PEN>, cnt, tid),
                   tape4{word, pn.acc[0], pn.acc[1], pn.acc[2]});
        else
          tape_put(tape_word_at<PEN>(row, cnt, tid), word);
      }
    }
  }
}

// A quad's start position, displacement, velocity and post-motion position
// from its column of an exchange tile.
template <int N, int BS>
__device__ __forceinline__ Quad tile_quad(const float (*tile)[BS], int tid) {
  Quad s;
  const float4* at = reinterpret_cast<const float4*>(&tile[XROW][0]);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    s.xo[k] = tile[k][tid];
    s.inc[k] = tile[3 + k][tid];
    s.v[k] = tile[6 + k][tid];
    if constexpr (N > 0) s.x[k] = tile[XROW + k][tid];
  }
  if constexpr (N == 0) {
    s.x[0] = at[tid].x;
    s.x[1] = at[tid].y;
    s.x[2] = at[tid].z;
  }
  return s;
}

// The contact set of a substep in the reverse sweep of handles with swarms
// above 32, whose tape does not hold it (the quad itself excluded).
template <int BS>
__device__ __forceinline__ unsigned long long mark_contacts(const Consts& c,
                                                            const float (*tile)[BS], const Quad& s,
                                                            int ls, int n, int me) {
  unsigned long long cm = 0ull;
  for_partners<BS, 0>(tile, ls, n, me, [&](int jj, const float* pj) {
    float dx, dy, dz, d2;
    cm |= pair_geom_v(c, pj, s, dx, dy, dz, d2) ? 1ull << jj : 0ull;
  });
  cm &= ~(1ull << me);
  return (c.flags & F_COLLIDE) ? cm : 0ull;
}

// Approach test of the contact set: does the quad receive a response?
template <int BS>
__device__ __forceinline__ bool any_response(const Consts& c, const float (*tile)[BS],
                                             const Quad& s, int ls, int me,
                                             unsigned long long cm) {
  bool hit = false;
  for (unsigned long long m = cm; m != 0ull; m &= m - 1ull) {
    const int jj = __builtin_ctzll(m);
    const int j = ls + jj;
    const float pj[6] = {tile[0][j], tile[1][j], tile[2][j], tile[3][j], tile[4][j], tile[5][j]};
    float dx, dy, dz, d2, nn[3], sp;
    pair_geom_v(c, pj, s, dx, dy, dz, d2);
    pair_normal<BS>(tile, s, j, jj, me, dx, dy, dz, d2, nn, sp);
    if (!(c.flags & F_APPROACH) || sp > 0.f) hit = true;
  }
  return hit;
}

// Adjoint of the collision responses of one quad (the partners in contact):
// ldv (rows 9-11 for the partners): adjoint of each quad's velocity change.
template <int BS>
__device__ __forceinline__ void response_vjp(const Consts& c, const float (*tile)[BS],
                                             const float (*ldvt)[BS], const Quad& s, int ls,
                                             int me, unsigned long long cm, const float ldv[3],
                                             float lx[3], float lv[3]) {
  for (unsigned long long m = cm; m != 0ull; m &= m - 1ull) {
    const int jj = __builtin_ctzll(m);
    const int j = ls + jj;
    const float pj[6] = {tile[0][j], tile[1][j], tile[2][j], tile[3][j], tile[4][j], tile[5][j]};
    float dx, dy, dz, d2, nn[3], sp;
    pair_geom_v(c, pj, s, dx, dy, dz, d2);
    pair_normal<BS>(tile, s, j, jj, me, dx, dy, dz, d2, nn, sp);
    if (!(c.flags & F_APPROACH) || sp > 0.f) {
      const float mu[3] = {ldv[0] - ldvt[0][j], ldv[1] - ldvt[1][j], ldv[2] - ldvt[2][j]};
      const float mn = dot3f(mu, nn);
#pragma unroll
      for (int k = 0; k < 3; ++k) lv[k] = fmaf(-mn, nn[k], lv[k]);
      if (!(d2 < 1e-12f)) {
        const float wv[3] = {tile[6][j] - s.v[0], tile[7][j] - s.v[1], tile[8][j] - s.v[2]};
        float gn[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) gn[k] = fmaf(sp, mu[k], mn * wv[k]);
        const float gnn = dot3f(gn, nn);
        const float id = rsqrtf(d2);
#pragma unroll
        for (int k = 0; k < 3; ++k) lx[k] = fmaf(gn[k] - gnn * nn[k], id, lx[k]);
      }
    }
  }
}

// A workgroup's rows of a row-major [Q][27] array (quads [qb, qb + cnt)) to or
// from LDS, words in order (one run of memory), by T threads; callers
// synchronise.  The sweeps take the adjoint from the caller's rows and put it
// back this way: converting it to fields and back, the parameters' with it,
// were four launches more (32768 x 32: 0.26 of 10.7 ms).
template <int BS, int T, bool IN, typename G>
__device__ __forceinline__ void move_rows(G* g, int qb, int cnt, float* sh, int tid) {
  G* run = g + (size_t)qb * NSTATE;
  constexpr int PER = (BS * NSTATE + T - 1) / T;
  const int total = cnt * NSTATE;
  // (the indexes of a kernel's last move are not to be shared with those of
  // its first and kept in registers between)
  asm volatile("" : "+v"(tid));
  float v[PER];  // (all reads go out before the first write)
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int i = min(tid + m * T, total - 1);
    v[m] = IN ? run[i] : sh[i];
  }
#pragma unroll
  for (int m = 0; m < PER; ++m) {
    const int i = tid + m * T;
    if (i < total) {
      if constexpr (IN) sh[i] = v[m];
      else run[i] = v[m];
    }
  }
}
__device__ __forceinline__ void get_adj(const float* row, Adj& l) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    l.x[k] = row[S_X + k];
    l.v[k] = row[S_V + k];
    l.w[k] = row[S_W + k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) l.R[k] = row[S_R + k];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    l.u[k] = row[S_U + k];
    l.e[k] = row[S_E + k];
  }
}
__device__ __forceinline__ void put_adj(float* row, const Adj& l) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    row[S_X + k] = l.x[k];
    row[S_V + k] = l.v[k];
    row[S_W + k] = l.w[k];
  }
#pragma unroll
  for (int k = 0; k < 9; ++k) row[S_R + k] = l.R[k];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    row[S_U + k] = l.u[k];
    row[S_E + k] = l.e[k];
  }
  row[S_F] = 0.f;
}

// The reverse of a substep's collision responses, by every lane of the
// workgroup: s the quads after the motion, cm the partners whose response the
// quad received (wide: found here).  tile: rows 0-8 as in the forward pass,
// 9-11 the adjoint of the collision velocity change.
template <int BS, int N>
__device__ __forceinline__ void reverse_responses(const Consts& c, float (*tile)[BS],
                                                  const Quad& s, bool live, int ls, int n, int me,
                                                  int tid, unsigned long long cm, int wide,
                                                  Adj& l) {
  // the exchange, where a quad of the workgroup received a response (rare)
  bool any = wide != 0;
  if (!any) {
    if constexpr (BS == 64) any = __ballot(cm != 0ull) != 0ull;
    else any = __syncthreads_or(cm != 0ull) != 0;
  }
  if (!any) return;
  __syncthreads();  // previous readers of the tile are done
  if (live) put_tile<N, false>(tile, tid, s);
  __syncthreads();
  bool hit = cm != 0ull;
  if constexpr (N == 0) {
    if (wide && live) {
      cm = mark_contacts<BS>(c, tile, s, ls, n, me);
      hit = any_response<BS>(c, tile, s, ls, me, cm);
    }
  }
  // the adjoint of the quad's velocity change
  float ldv[3] = {0.f, 0.f, 0.f};
  if (live && hit) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      ldv[k] = c.col_decay * l.v[k];
      l.v[k] = ldv[k];
    }
  }
  if (live) {
#pragma unroll
    for (int k = 0; k < 3; ++k) tile[9 + k][tid] = ldv[k];
  }
  __syncthreads();
  if (live) response_vjp<BS>(c, tile, tile + 9, s, ls, me, cm, ldv, l.x, l.v);
}

// Where a backward pass's parameter gradient [Q][6] goes: every chunk's share is
// summed in sum, and the total is added to the caller's array once, by the last
// chunk.  (Added chunk by chunk, each share would be rounded at the size of what
// the caller's array holds already.)
struct ParSum {
  float* out;   // the caller's
  float* sum;   // the handle's, where there are several chunks
  bool first, last;
};
__device__ __forceinline__ void add_par(const ParSum& p, int q, int k, float g) {
  const size_t i = (size_t)q * 6 + k;
  if (!p.first) g = p.sum[i] + g;
  if (p.last) p.out[i] += g;
  else p.sum[i] = g;
}

// ---------------------------------------------------------------------------
// reverse_kernel: the reverse sweep over the chunk's ncalls nsub substeps,
// last to first, from the tape; the adjoint of the state stays in
// registers for the whole chunk and the tape row of the next substep to
// process is loaded while the current one is differentiated.  It and the
// recompute wait for the tape's memory more than for their arithmetic, so the
// motor noise is drawn again instead of being stored and read: 32768 x 32, 100
// substeps with their derivative, 10.43 -> 9.77 ms.
//  gin, gout: [Q][27] dL/d(chunk end), dL/d(chunk start) (may be one array);
//  act/gact: the chunk's first call; gpar: where dL/d(m, ixx, iyy, izz, t2w,
//  tau) goes.
// ---------------------------------------------------------------------------
template <int BS, int N, bool PEN>
__global__ __launch_bounds__(BS) void reverse_kernel(const Consts* __restrict__ cp, Ptrs p,
                                                     const float* __restrict__ act, int ncalls,
                                                     int nsub, unsigned long long t0,
                                                     const float* __restrict__ tape,
                                                     const float* gin, float* gout, int wide,
                                                     float* __restrict__ gact, ParSum gpar) {
  constexpr int NTAPE = kTapeRows<PEN>;
  // the rows on their way in and out; the exchange tile between
  __shared__ __align__(16) float sh[NSTATE * BS];
  float(*tile)[BS] = reinterpret_cast<float(*)[BS]>(sh);
  const Consts& c = *cp;
  const int tid = threadIdx.x;
  int qb, cnt, ls, n;
  block_map<BS, N>(p, tid, qb, cnt, ls, n);
  const bool live = tid < cnt;
  const int q = qb + (live ? tid : 0);
  const int me = tid - ls;
  const long long Q = p.Q;
  const bool pairs = N != 1 && (c.flags & F_COLLIDE) != 0;

  Adj l;
  move_rows<BS, BS, true>(gin, qb, cnt, sh, tid);
  __syncthreads();
  if (live) get_adj(sh + tid * NSTATE, l);
  __syncthreads();
  Quad s, sn;
  float pn[3] = {0.f, 0.f, 0.f}, pen3[3];     // penalty adjoint of sn and s
  QuadPar pp;
  ParAdj pa;
  const int n_steps = ncalls * nsub;
  if (live) {
    load_params(p, c, q, pp, pa);
    const float* row = tape + ((long long)(n_steps - 1) * Q + qb) * NTAPE;
    tape_load<PEN>(row, cnt, tid, sn, pn);
  }

  // ---- reverse sweep
  float gp[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float4 a_nx = make_float4(0.f, 0.f, 0.f, 0.f);
  if (live && ncalls > 0) a_nx = load_act(act + (long long)(ncalls - 1) * Q * 4, q);
  for (int call = ncalls - 1; call >= 0; --call) {
    float uhat[4] = {0.f, 0.f, 0.f, 0.f}, gu[4] = {0.f, 0.f, 0.f, 0.f};
    const float4 a4 = a_nx;
    if (live && call > 0) a_nx = load_act(act + (long long)(call - 1) * Q * 4, q);
    if (live) act_uhat(c, p, a4, uhat);
    for (int sub = nsub - 1; sub >= 0; --sub) {
      const int k_s = call * nsub + sub;
      const unsigned long long t = t0 + (unsigned long long)k_s;
      Rec r;
      unsigned long long cm = 0ull;  // partners whose response the quad received
      if (live) {
        s = sn;
        const uint32_t word = __float_as_uint(s.fl);
        s.fl = word_flag(word, me, wide);
        cm = word_resp(word, me, wide);
#pragma unroll
        for (int k = 0; k < 3; ++k) pen3[k] = pn[k];
        if (k_s > 0) {
          const float* row = tape + ((long long)(k_s - 1) * Q + qb) * NTAPE;
          tape_load<PEN>(row, cnt, tid, sn, pn);
        }
        float z[4] = {0.f, 0.f, 0.f, 0.f};
        if (c.flags & F_NOISE) normal4(c, (uint32_t)q, t, STREAM_MOTOR, 0, z);
        quad_substep<true, Z_IMPORT>(c, pp, s, uhat, (uint32_t)q, t, &r, z);
        if constexpr (PEN) {
#pragma unroll
          for (int k = 0; k < 3; ++k) l.x[k] += pen3[k];
        }
      }
      if (pairs) reverse_responses<BS, N>(c, tile, s, live, ls, n, me, tid, cm, wide, l);
      if (live) quad_vjp(c, pp, pa, r, uhat, l, gu, gp);
    }
    if (live) {
      float4 g;
      g.x = gu[0] * duhat_da(c, a4.x, uhat[0]);
      g.y = gu[1] * duhat_da(c, a4.y, uhat[1]);
      g.z = gu[2] * duhat_da(c, a4.z, uhat[2]);
      g.w = gu[3] * duhat_da(c, a4.w, uhat[3]);
      reinterpret_cast<float4*>(gact + (long long)call * Q * 4)[q] = g;
    }
  }
  __syncthreads();
  if (live) {
    put_adj(sh + tid * NSTATE, l);
#pragma unroll
    for (int k = 0; k < 6; ++k) add_par(gpar, q, k, gp[k]);
  }
  __syncthreads();
  move_rows<BS, BS, false>(gout, qb, cnt, sh, tid);
}

// ---------------------------------------------------------------------------
// step_vjp_kernel: the derivative of one call of a few substeps in one launch
// and without a tape in memory: the substeps before the last leave their start
// state, draws and responding partners in LDS, the last one's record is still at hand when
// the sweep starts.  Same arithmetic in the same order as recompute_kernel and
// reverse_kernel, so identical results.  The conversions, fills, recompute and
// sweep were eight launches (4096 x 8, two substeps: 34.3 -> 12.8 us a call).
//  state_in, gin, gout: [Q][27]; act, gact: [Q][4]; gpar: [Q][6] accumulated;
//  dynamic LDS: VJP_ROW floats per quad and substep before the last.
// ---------------------------------------------------------------------------
constexpr int VJP_ROW = NSTATE + 4 + 2;  // state, draws, responding partners
constexpr int VJP_MAX_SUBSTEPS = 4;

template <int N>
__global__ __launch_bounds__(64) void step_vjp_kernel(const Consts* __restrict__ cp, Ptrs p,
                                                      const float* __restrict__ state_in,
                                                      const float* __restrict__ act, int nsub,
                                                      unsigned long long t0, const float* gin,
                                                      float* gout, float* __restrict__ gact,
                                                      float* __restrict__ gpar) {
  constexpr int BS = 64;
  // the rows on their way in and out; the exchange tiles between (forward rows
  // with the screen's, then the reverse's twelve)
  __shared__ __align__(16) float sh[NSTATE * BS];
  extern __shared__ float rows[];
  const Consts& c = *cp;
  const int tid = threadIdx.x;
  int qb, cnt, ls, n;
  block_map<BS, N>(p, tid, qb, cnt, ls, n);
  const bool live = tid < cnt;
  const int q = qb + (live ? tid : 0);
  const int me = tid - ls;
  const bool pairs = N != 1 && (c.flags & F_COLLIDE) != 0;
  float(*tile)[BS] = reinterpret_cast<float(*)[BS]>(sh);
  QuadPar pp;
  ParAdj pa;
  Quad s;
  Adj l;
  float4 a4 = load_act(act, q);
  move_rows<BS, BS, true>(state_in, qb, cnt, sh, tid);
  if (live) load_params(p, c, q, pp, pa);
  __syncthreads();
  if (live) load_state(sh, 1, tid * NSTATE, s);
  __syncthreads();
  move_rows<BS, BS, true>(gin, qb, cnt, sh, tid);
  __syncthreads();
  if (live) get_adj(sh + tid * NSTATE, l);
  __syncthreads();
  float uhat[4] = {0.f, 0.f, 0.f, 0.f}, gu[4] = {0.f, 0.f, 0.f, 0.f};
  float gp[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (live) act_uhat(c, p, a4, uhat);
  // the substep's in-swarm pass on sp: its responding partners
  auto responding = [&](Quad& sp, unsigned long long t) {
    unsigned long long resp = 0ull;
    if constexpr (N == 8) {
      lane_pair_pass<BS, N, true>(c, tile, sp, live, ls, n, me, tid, (uint32_t)q, t, &resp);
    } else {
      if (live) put_tile<N, true>(tile, tid, sp);
      __syncthreads();
      if (live)
        pair_pass<BS, N, PEN_NONE, true>(c, tile, sp, ls, n, me, (uint32_t)q, t, nullptr, nullptr,
                                         &resp);
      __syncthreads();
    }
    return resp;
  };
  for (int k = 0; k < nsub - 1; ++k) {
    const unsigned long long t = t0 + (unsigned long long)k;
    float* row = rows + k * VJP_ROW * BS;
    if (live) {
      store_state(row, BS, tid, s);
      float z[4] = {0.f, 0.f, 0.f, 0.f};
      quad_substep<false, Z_EXPORT>(c, pp, s, uhat, (uint32_t)q, t, nullptr, z);
#pragma unroll
      for (int i = 0; i < 4; ++i) row[(NSTATE + i) * BS + tid] = z[i];
    }
    const unsigned long long cm = pairs ? responding(s, t) : 0ull;
    row[(NSTATE + 4) * BS + tid] = __uint_as_float((uint32_t)cm);
    row[(NSTATE + 5) * BS + tid] = __uint_as_float((uint32_t)(cm >> 32));
  }
  {
    const unsigned long long t = t0 + (unsigned long long)(nsub - 1);
    Rec r;
    if (live) quad_substep<true>(c, pp, s, uhat, (uint32_t)q, t, &r);
    if (pairs) {
      Quad sp = s;
      const unsigned long long cm = responding(sp, t);
      reverse_responses<BS, N == 0 ? -1 : N>(c, tile, s, live, ls, n, me, tid, cm, 0, l);
    }
    if (live) quad_vjp(c, pp, pa, r, uhat, l, gu, gp);
  }
  for (int k = nsub - 2; k >= 0; --k) {
    const float* row = rows + k * VJP_ROW * BS;
    Rec r;
    if (live) {
      load_state(row, BS, tid, s);
      float z[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = row[(NSTATE + i) * BS + tid];
      quad_substep<true, Z_IMPORT>(c, pp, s, uhat, (uint32_t)q, t0 + (unsigned long long)k, &r, z);
    }
    if (pairs) {
      const unsigned long long cm =
          __float_as_uint(row[(NSTATE + 4) * BS + tid]) |
          (unsigned long long)__float_as_uint(row[(NSTATE + 5) * BS + tid]) << 32;
      reverse_responses<BS, N == 0 ? -1 : N>(c, tile, s, live, ls, n, me, tid, cm, 0, l);
    }
    if (live) quad_vjp(c, pp, pa, r, uhat, l, gu, gp);
  }
  __syncthreads();
  if (live) {
    float4 g;
    g.x = gu[0] * duhat_da(c, a4.x, uhat[0]);
    g.y = gu[1] * duhat_da(c, a4.y, uhat[1]);
    g.z = gu[2] * duhat_da(c, a4.z, uhat[2]);
    g.w = gu[3] * duhat_da(c, a4.w, uhat[3]);
    reinterpret_cast<float4*>(gact)[q] = g;
    put_adj(sh + tid * NSTATE, l);
#pragma unroll
    for (int k = 0; k < 6; ++k) gpar[(size_t)q * 6 + k] += gp[k];
  }
  __syncthreads();
  move_rows<BS, BS, false>(gout, qb, cnt, sh, tid);
}

// ---------------------------------------------------------------------------
// Small batches (up to 1024 workgroups of 64 quads) leave most SIMDs without a
// wavefront, and the time of a substep is the time of its dependent
// instructions.  The forward pass, the recompute and the reverse sweep then run
// the parts of a substep on wavefronts of their own, over the same 64 quads,
// with one workgroup barrier per substep; results pass through LDS rings.
//
// forward_pipe: the forward pass (TAPE false: checkpoints into out, the penalty
// summed into pen) or the recompute of a segment (TAPE: a tape row per substep
// into out, with the penalty's adjoint).
//  - the last wavefront draws the motor noise of substep i at step i (NW; where
//    the workgroups fill the chip it is left to wavefront 0, which starts);
//  - wavefront 0, at step i + 1, runs the motor part (it depends on the rotor
//    state, the action and the draws only) and hands on T and torques;
//  - wavefront 1, at step i + 2, the translation and the in-swarm pass;
//  - wavefront 2, at step i + 2, the rotation: the two need of each other only
//    what the substep before left, R's third column one way and the events
//    the other, so both answer to the events of substep i - 1 at the start of
//    substep i;
//  - with a penalty (P) wavefront 3 sums it at step i + 3 from the exchange
//    tile (it never feeds back into the motion).
// Each wavefront stores its own fields.  Same arithmetic in the same order as
// the one-wavefront kernels, so identical results.  With noise and motor, and
// translation and rotation, on one wavefront each and loads one substep ahead:
// 1024 x 8, 200 substeps, forward 222 us, now 185.
//  S: the start state (TAPE: a checkpoint; else the handle's); act: its first call; t0: its first substep.
// ---------------------------------------------------------------------------
// Loads whose address is known go out AHEAD substeps before their use: a
// substep of these pipelines is shorter than a read from HBM, which had set
// their pace at one substep ahead (1.1-1.3 us a substep whatever the stages
// did).  A value in flight cannot move between registers, so the steps are
// unrolled and each has a register set of its own.
constexpr int AHEAD = 4;

// f(i, slot) for the steps i of a wavefront's pipeline, slot = i mod A at
// compile time, and the workgroup's barrier after each.
template <int A, typename F>
__device__ __forceinline__ void pipe_steps(int n_pipe, F&& f) {
  static_assert(A == 1 || A == 4, "unrolled by one or four");
  auto step = [&](int i, auto slot) {
    if (i < n_pipe) {
      f(i, slot);
      wg_sync();
    }
  };
  for (int i = 0; i < n_pipe; i += A) {
    step(i, std::integral_constant<int, 0>{});
    if constexpr (A == 4) {
      step(i + 1, std::integral_constant<int, 1>{});
      step(i + 2, std::integral_constant<int, 2>{});
      step(i + 3, std::integral_constant<int, 3>{});
    }
  }
}

template <int P, bool NW>
constexpr int kPipeWaves = 3 + (P != PEN_NONE ? 1 : 0) + (NW ? 1 : 0);

template <int N, int P, bool TAPE, bool NW>
__device__ __forceinline__ void forward_pipe(const Consts& c, const Ptrs& p,
                                             const float* __restrict__ S,
                                             const float* __restrict__ act, int nc, int nsub,
                                             unsigned long long t0, float* __restrict__ out,
                                             int every, const float* __restrict__ gpen,
                                             float* __restrict__ pen, float beta) {
  constexpr int BS = 64, NTAPE = kTapeRows<P == PEN_GRAD>;
  constexpr int M = NW ? 1 : 0;     // step of the first substep's motor part
  __shared__ __align__(16) float sxv[2][PENROW + 1][BS];
  __shared__ float4 zring[2][BS];   // motor noise
  __shared__ float ring[2][4][BS];  // T, torques
  __shared__ float r3[2][3][BS];    // third column of R after free flight
  __shared__ uint32_t evr[2][BS];   // the substep's events
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tid = threadIdx.x & 63;
  int qb, cnt, ls, n;
  block_map<BS, N>(p, tid, qb, cnt, ls, n);
  const bool live = tid < cnt;
  const int q = qb + (live ? tid : 0);
  const int me = tid - ls;
  const long long Q = p.Q;
  const int n_steps = nc * nsub;
  const int n_pipe = n_steps + M + (P != PEN_NONE ? 2 : 1);  // steps of the pipeline
  QuadPar pp;
  ParAdj pa;
  if (live) load_params(p, c, q, pp, pa);
  constexpr bool PN = P == PEN_GRAD;
  // field f of the quad in a checkpoint of rows of Q (a 32-bit byte offset:
  // these batches stay far below 2^32 bytes a row)
  const uint32_t qo = 4u * (uint32_t)q, fo = 4u * (uint32_t)p.Q;
  auto at = [&](float* row, int f) -> float& {
    return *reinterpret_cast<float*>(reinterpret_cast<char*>(row) + (qo + (uint32_t)f * fo));
  };
  // field f of the state to start from: a checkpoint, or the handle's
  auto start = [&](int f) -> float {
    if constexpr (TAPE) return S[(long long)f * Q + q];
    else return S[st_index(q, f)];
  };
  // where the state before substep k goes (uniform: the workgroup's part of a tape
  // row, or a checkpoint), or null
  auto row_of = [&](int k) -> float* {
    if constexpr (TAPE) return out + ((long long)k * Q + qb) * NTAPE;
    const int call = k / nsub;
    if (!out || k != call * nsub || call % every != 0) return nullptr;
    return out + (long long)(call / every) * NSTATE * Q;
  };

  if (wave == 0) {
    // ---- motor part of substep i - M at step i
    float u[4], e[4];
    if (live) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        u[k] = start(S_U + k);
        e[k] = start(S_E + k);
      }
    }
    float uhat[4] = {0.f, 0.f, 0.f, 0.f};
    // each substep's action row, A substeps before its use (the recompute's
    // many workgroups hide the read, and its stores want the registers)
    constexpr int A = TAPE ? 1 : AHEAD;
    float4 aq[A];
#pragma unroll
    for (int d = 0; d < A; ++d) aq[d] = load_act(act + (long long)min(d / nsub, nc - 1) * Q * 4, q);
    int sub = 0, call_a = A / nsub, sub_a = A % nsub;  // of substeps i and i + A
    if constexpr (M > 0) wg_sync();  // step 0: no draws yet
    pipe_steps<A>(n_pipe - M, [&](int i, auto slot_c) {
      constexpr int D = decltype(slot_c)::value;
      if (i < n_steps) {
        const float4 a4 = aq[D];
        aq[D] = load_act(act + (long long)min(call_a, nc - 1) * Q * 4, q);
        if (sub == 0 && live) act_uhat(c, p, a4, uhat);
        if (live) {
          float* row = row_of(i);
          if constexpr (TAPE) {
            tape_four(row, 0, cnt, tid) = tape4{u[0], u[1], u[2], u[3]};
            tape_four(row, 4, cnt, tid) = tape4{e[0], e[1], e[2], e[3]};
          } else if (row) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              at(row, S_U + k) = u[k];
              at(row, S_E + k) = e[k];
            }
          }
          float z[4] = {0.f, 0.f, 0.f, 0.f}, zi[4] = {0.f, 0.f, 0.f, 0.f};
          if constexpr (M > 0) {
            const float4 z4 = zring[i & 1][tid];
            zi[0] = z4.x;
            zi[1] = z4.y;
            zi[2] = z4.z;
            zi[3] = z4.w;
          }
          const Drive d = motor_step<M == 0 ? Z_DRAW : Z_IMPORT>(
              c, pp, u, e, uhat, (uint32_t)q, t0 + (unsigned long long)i, z, zi);
          if (TAPE && (c.flags & F_NOISE))
            tape_four(row, T_DRAW<PN>, cnt, tid) = tape4{z[0], z[1], z[2], z[3]};
          float(*slot)[BS] = ring[i & 1];
          slot[0][tid] = d.T;
          slot[1][tid] = d.tx;
          slot[2][tid] = d.ty;
          slot[3][tid] = d.tz;
        }
        sub = sub + 1 == nsub ? 0 : sub + 1;
        sub_a = sub_a + 1 == nsub ? 0 : sub_a + 1;
        call_a += sub_a == 0 ? 1 : 0;
      }
    });
    if (!TAPE && live) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        p.st[st_index(q, S_U + k)] = u[k];
        p.st[st_index(q, S_E + k)] = e[k];
      }
    }
  } else if (wave == 1) {
    // ---- translation and in-swarm pass of substep i - M - 1 at step i
    Quad s;
    float c2[3] = {0.f, 0.f, 0.f};  // third column of R at the substep's start
    uint32_t ev = 0u;
    s.ev = 0u;
    if (live) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        s.x[k] = start(S_X + k);
        s.v[k] = start(S_V + k);
        c2[k] = start(S_R + 3 * k + 2);
      }
      s.fl = start(S_F);
    }
    const bool pairs = N != 1 && (c.flags & (F_COLLIDE | F_DOWNWASH)) != 0;
    for (int i = 0; i < M + 1; ++i) wg_sync();  // no thrust yet
    for (int k_s = 0; k_s < n_pipe - M - 1; ++k_s) {
      if (k_s < n_steps) {
        const unsigned long long t = t0 + (unsigned long long)k_s;
        float* row = row_of(k_s);
        const float fl0 = s.fl;
        unsigned long long resp = 0ull;
        float(*tile)[BS] = sxv[k_s & 1];
        if (live) {
          if constexpr (TAPE) {
            tape_four(row, 20, cnt, tid) = tape4{s.x[0], s.x[1], s.x[2], s.v[0]};
            tape_at<tape2>(row, T_V12<PN>, cnt, tid) = tape2{s.v[1], s.v[2]};
          } else if (row) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              at(row, S_X + k) = s.x[k];
              at(row, S_V + k) = s.v[k];
            }
            at(row, S_F) = s.fl;
          }
          if (k_s > 0) {
            // the events of the substep before decide what became of R
            const float(*col)[BS] = r3[(k_s - 1) & 1];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              c2[k] = (ev & SUB_REST) ? c2[k] : col[k][tid];
              c2[k] = (ev & SUB_HIT) ? (k == 2 ? 1.0f : 0.0f) : c2[k];
            }
          }
          ev = trans_step(c, pp, s, ring[k_s & 1][0][tid], c2[0], c2[1], c2[2], (uint32_t)q, t);
          if ((pairs && N != 8) || P != PEN_NONE) put_tile<N, true>(tile, tid, s);
        }
        if constexpr (N == 8) {
          if (pairs) {
            uint32_t pev = 0u;
            lane_pair_pass<BS, N, P == PEN_NONE>(c, tile, s, live, ls, n, me, tid, (uint32_t)q, t,
                                                 &resp, &pev);
            ev |= live ? pev : 0u;
          }
        } else if (pairs) {
          wave_sync();
          uint32_t pev = 0u;
          if (live)
            pair_pass<BS, N, PEN_NONE, true>(c, tile, s, ls, n, me, (uint32_t)q, t, nullptr,
                                             nullptr, &resp, &pev);
          ev |= pev;
        }
        evr[k_s & 1][tid] = ev;
        if (TAPE && live) tape_word_at<PN>(row, cnt, tid) = tape_word(fl0, resp, me, 0);
      }
      wg_sync();
    }
    if (!TAPE && live) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        p.st[st_index(q, S_X + k)] = s.x[k];
        p.st[st_index(q, S_V + k)] = s.v[k];
      }
      p.st[st_index(q, S_F)] = s.fl;
      float chk = 0.f;
#pragma unroll
      for (int k = 0; k < 3; ++k) chk += s.x[k] + s.v[k];
      if (!isfinite(chk))
        __hip_atomic_fetch_or(p.err, ERRBIT_STATE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  } else if (wave == 2) {
    // ---- rotation of substep i - M - 1 at step i
    float R[9], w[3], R0[9];
    if (live) {
#pragma unroll
      for (int k = 0; k < 9; ++k) R[k] = R0[k] = start(S_R + k);
#pragma unroll
      for (int k = 0; k < 3; ++k) w[k] = start(S_W + k);
    }
    // the events of substep k, which started from R0
    auto answer = [&](int k) {
      const uint32_t ev = evr[k & 1][tid];
      if (ev & SUB_TURNS) {
        const unsigned long long t = t0 + (unsigned long long)k;
        rot_events(c, ev, R, w, R0, (uint32_t)q, t);
        rot_pair_events(c, ev, w, (uint32_t)q, t);
      }
    };
    for (int i = 0; i < M + 1; ++i) wg_sync();  // no torques yet
    for (int k_s = 0; k_s < n_pipe - M - 1; ++k_s) {
      if (k_s < n_steps && live) {
        if (k_s > 0) answer(k_s - 1);
        float* row = row_of(k_s);
        if constexpr (TAPE) {
          tape_four(row, 8, cnt, tid) = tape4{R[0], R[1], R[2], R[3]};
          tape_four(row, 12, cnt, tid) = tape4{R[4], R[5], R[6], R[7]};
          tape_four(row, 16, cnt, tid) = tape4{R[8], w[0], w[1], w[2]};
        } else if (row) {
#pragma unroll
          for (int k = 0; k < 9; ++k) at(row, S_R + k) = R[k];
#pragma unroll
          for (int k = 0; k < 3; ++k) at(row, S_W + k) = w[k];
        }
        const float(*slot)[BS] = ring[k_s & 1];
#pragma unroll
        for (int k = 0; k < 9; ++k) R0[k] = R[k];
        rot_step(c, pp, R, w, slot[1][tid], slot[2][tid], slot[3][tid]);
#pragma unroll
        for (int k = 0; k < 3; ++k) r3[k_s & 1][k][tid] = R[3 * k + 2];
      }
      wg_sync();
    }
    if (!TAPE && live) {
      if (n_steps > 0) answer(n_steps - 1);
#pragma unroll
      for (int k = 0; k < 9; ++k) p.st[st_index(q, S_R + k)] = R[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) p.st[st_index(q, S_W + k)] = w[k];
      float chk = 0.f;
#pragma unroll
      for (int k = 0; k < 9; ++k) chk += R[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) chk += w[k];
      if (!isfinite(chk))
        __hip_atomic_fetch_or(p.err, ERRBIT_STATE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  } else if (NW && (P == PEN_NONE || wave == 4)) {
    // ---- motor noise of substep i at step i
    for (int i = 0; i < n_pipe; ++i) {
      if (i < n_steps && live && (c.flags & F_NOISE)) {
        float z[4];
        normal4(c, (uint32_t)q, t0 + (unsigned long long)i, STREAM_MOTOR, 0, z);
        zring[i & 1][tid] = make_float4(z[0], z[1], z[2], z[3]);
      }
      wg_sync();
    }
  } else if constexpr (P != PEN_NONE) {
    // ---- the penalty, or its adjoint, of substep i - M - 2 at step i
    float h_me = 0.f;
    if constexpr (P == PEN_GRAD) {
      h_me = live ? -0.5f * gpen[q] : 0.f;
      sxv[0][PENROW][tid] = h_me;
      sxv[1][PENROW][tid] = h_me;
    }
    Pen pn = make_pen(c, beta, N > 0 ? N : wave_max(live ? n : 0), h_me);
    for (int i = 0; i < M + 2; ++i) wg_sync();  // no tile yet
    for (int k_s = 0; k_s < n_steps; ++k_s) {
      if (live) {
        const float(*tile)[BS] = sxv[k_s & 1];
        const Quad so = tile_quad<N>(tile, tid);
        if constexpr (P == PEN_GRAD) pn.acc[0] = pn.acc[1] = pn.acc[2] = 0.f;
        penalty_pass<BS, N, P>(c, tile, so, ls, n, me, pn);
        if constexpr (P == PEN_GRAD) {
          float* row = row_of(k_s);
#pragma unroll
          for (int k = 0; k < 3; ++k)
            tape_at<float>(row, T_WORD<PN>, cnt, 4 * tid + 1 + k) = pn.acc[k];
        }
      }
      wg_sync();
    }
    if (P == PEN_SUM && live) pen[q] += pn.acc[0];
  }
}

template <int N, bool PEN, bool NW>
__global__ __launch_bounds__(NW ? 320 : 256) void rollout_pipe_kernel(const Consts* __restrict__ cp, Ptrs p,
                                                           const float* __restrict__ act,
                                                           int ncalls, int nsub,
                                                           unsigned long long t0,
                                                           float* __restrict__ ckpt,
                                                           int ckpt_every,
                                                           float* __restrict__ pen, float beta) {
  const Consts c = *cp;  // (a copy: kept in registers across the barriers)
  forward_pipe<N, PEN ? PEN_SUM : PEN_NONE, false, NW>(c, p, p.st, act, ncalls, nsub, t0, ckpt,
                                                   ckpt_every, nullptr, pen, beta);
}

// grid (workgroups, segments of the chunk); arguments as recompute_kernel
template <int N, bool PEN>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void recompute_pipe_kernel(const Consts* __restrict__ cp, Ptrs p,
                                                             const float* __restrict__ ckpt,
                                                             const float* __restrict__ act,
                                                             int ncalls, int ce, int nsub,
                                                             unsigned long long t0,
                                                             float* __restrict__ tape,
                                                             const float* __restrict__ gpen,
                                                             float beta) {
  const long long Q = p.Q;
  const int c0 = blockIdx.y * ce;
  const Consts c = *cp;
  forward_pipe<N, PEN ? PEN_GRAD : PEN_NONE, true, false>(
      c, p, ckpt + (long long)blockIdx.y * NSTATE * Q, act + (long long)c0 * Q * 4,
      min(ce, ncalls - c0), nsub, t0 + (unsigned long long)c0 * nsub,
      tape + (long long)c0 * nsub * kTapeRows<PEN> * Q, 1, gpen, nullptr, beta);
}

// ---------------------------------------------------------------------------
// reverse_pipe_kernel: the reverse sweep of reverse_kernel for small batches
// without swarms above 32 (see forward_pipe), on seven wavefronts.  A substep's
// re-run starts from its taped state, so no stage waits for the substep after
// it, and of the derivative only the parts that feed themselves are serial.
// Substep k passes through:
//  step i      wavefront 6: the rotor commands and their derivatives;
//  step i + 1  wavefront 0: the motor part re-run from the taped rotor state
//              and draws;
//  step i + 2  wavefront 1: the translation re-run (dL's factors and the
//              exchange tile), wavefront 2: the rotation re-run;
//  step i + 3  wavefront 5: the responses' and the translation's derivative;
//  step i + 4  wavefront 3: the rotation's;
//  step i + 5  wavefront 4: the motor's, and the action gradients.
// Wavefronts 4 to 6 share the SIMDs of the lighter ones of the first four.
// Same arithmetic in the same order as reverse_kernel, so identical results.
// The derivative, the body's re-run and the commands with the motor's on one
// wavefront each, and loads one substep ahead: 1024 x 8, 200 substeps, 241 us,
// now 185.
//  un: the uniform swarm size (a power of two) or 0 (table of sizes)
// ---------------------------------------------------------------------------
template <bool PEN>
__global__ __launch_bounds__(448) void reverse_pipe_kernel(const Consts* __restrict__ cp, Ptrs p,
                                                           const float* __restrict__ act,
                                                           int ncalls, int nsub,
                                                           const float* __restrict__ tape,
                                                           const float* gin, float* gout, int un,
                                                           float* __restrict__ gact, ParSum gpar,
                                                           unsigned long long t0) {
  constexpr int BS = 64, NTAPE = kTapeRows<PEN>;
  // rings, indexed by the substep; as many slots as steps pass from the first
  // write of one to its last read
  __shared__ float4 uring[6][2][BS];  // rotor command; its derivative w.r.t. the action
  __shared__ float4 mring[5][4][BS];  // T and torques; draws; u before, after
  __shared__ float4 tring[2][2][BS];  // F, start velocity, events
  __shared__ float4 rring[3][8][BS];  // the rotation's record
  __shared__ float tile[2][9][BS];    // start position, displacement, velocity
  __shared__ float ldvt[3][BS];       // adjoint of the collision velocity change
  __shared__ float4 aring[2][BS];     // lF, events
  __shared__ float lring[3][BS];      // lm
  __shared__ float4 bring[2][BS];     // lT, lt
  const Consts c = *cp;  // (a copy: kept in registers across the barriers)
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int tid = threadIdx.x & 63;
  int qb, cnt, ls, n;
  if (un > 0) {
    qb = blockIdx.x * BS;
    cnt = min(BS, p.Q - qb);
    ls = tid & ~(un - 1);
  } else {
    block_map<BS, 0>(p, tid, qb, cnt, ls, n);
  }
  const bool live = tid < cnt;
  const int q = qb + (live ? tid : 0);
  const int me = tid - ls;
  const long long Q = p.Q;
  const int n_steps = ncalls * nsub;
  const int n_pipe = n_steps + 5;  // steps of the pipeline
  QuadPar pp;
  ParAdj pa;
  if (live) load_params(p, c, q, pp, pa);
  // the adjoint's rows on their way in and out, where the record's ring is in
  // between
  float* sh = reinterpret_cast<float*>(&rring[0][0][0]);
  static_assert(sizeof(rring) >= NSTATE * BS * sizeof(float), "room for the rows");
  const float* my = sh + tid * NSTATE;
  float* out = sh + tid * NSTATE;
  move_rows<BS, 448, true>(gin, qb, cnt, sh, threadIdx.x);
  wg_sync();
  auto row_of = [&](int k) { return tape + ((long long)k * Q + qb) * NTAPE; };
  // the stage's substeps, last to first, each f(k); every wavefront passes
  // the same barriers
  // (with a load of substep k's row AHEAD steps before its f)
  auto loading_stages = [&](int stage, auto&& load, auto&& f) {
    if (live) {
      auto first = [&](auto slot) { load(max(n_steps - 1 - decltype(slot)::value, 0), slot); };
      first(std::integral_constant<int, 0>{});
      first(std::integral_constant<int, 1>{});
      first(std::integral_constant<int, 2>{});
      first(std::integral_constant<int, 3>{});
    }
    for (int i = 0; i < stage; ++i) wg_sync();
    pipe_steps<AHEAD>(n_pipe - stage, [&](int i, auto slot) {
      const int k = n_steps - 1 - i;
      if (k >= 0) f(k, slot, [&] { load(max(k - AHEAD, 0), slot); });
    });
  };
  auto stages = [&](int stage, auto&& f) {
    for (int i = 0; i < stage; ++i) wg_sync();
    for (int i = stage; i < n_pipe; ++i) {
      const int k = n_steps - 1 - (i - stage);
      if (k >= 0) f(k);
      wg_sync();
    }
  };

  if (wave == 0) {
    float un4[AHEAD][4], en[AHEAD][4], zn[AHEAD][4];
    loading_stages(
        1,
        [&](int k, auto slot) {
          constexpr int D = decltype(slot)::value;
          const float* row = row_of(k);
          const tape4 u4 = tape_four(row, 0, cnt, tid), e4 = tape_four(row, 4, cnt, tid);
          tape4 z4 = {0.f, 0.f, 0.f, 0.f};
          if (c.flags & F_NOISE) z4 = tape_four(row, T_DRAW<PEN>, cnt, tid);
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            un4[D][m] = u4[m];
            en[D][m] = e4[m];
            zn[D][m] = z4[m];
          }
        },
        [&](int k, auto slot, auto&& next) {
          constexpr int D = decltype(slot)::value;
          if (!live) return;
          float u[4], e[4], zi[4], z[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            u[m] = un4[D][m];
            e[m] = en[D][m];
            zi[m] = zn[D][m];
          }
          next();
          const float4 uh = uring[k % 6][0][tid];
          const float uhat[4] = {uh.x, uh.y, uh.z, uh.w};
          float4(*ms)[BS] = mring[k % 5];
          ms[2][tid] = make_float4(u[0], u[1], u[2], u[3]);
          const Drive d = motor_step<Z_IMPORT>(c, pp, u, e, uhat, (uint32_t)q,
                                               t0 + (unsigned long long)k, z, zi);
          ms[0][tid] = make_float4(d.T, d.tx, d.ty, d.tz);
          ms[1][tid] = make_float4(z[0], z[1], z[2], z[3]);
          ms[3][tid] = make_float4(u[0], u[1], u[2], u[3]);
        });
  } else if (wave == 6) {
    float4 aq[AHEAD];
    float4 uh = make_float4(0.f, 0.f, 0.f, 0.f), du = uh;
    int sub = nsub - 1, call_a = (n_steps - 1) / nsub, sub_a = nsub - 1;  // of the row to load
    loading_stages(
        0,
        [&](int, auto slot) {
          aq[decltype(slot)::value] = load_act(act + (long long)max(call_a, 0) * Q * 4, q);
          call_a -= sub_a == 0 ? 1 : 0;
          sub_a = sub_a == 0 ? nsub - 1 : sub_a - 1;
        },
        [&](int k, auto slot, auto&& next) {
          const float4 a4 = aq[decltype(slot)::value];
          if (live) {
            if (sub == nsub - 1) {  // the call's last substep comes first
              float uhat[4];
              act_uhat(c, p, a4, uhat);
              uh = make_float4(uhat[0], uhat[1], uhat[2], uhat[3]);
              du = make_float4(duhat_da(c, a4.x, uhat[0]), duhat_da(c, a4.y, uhat[1]),
                               duhat_da(c, a4.z, uhat[2]), duhat_da(c, a4.w, uhat[3]));
            }
            uring[k % 6][0][tid] = uh;
            uring[k % 6][1][tid] = du;
            next();
          }
          sub = sub == 0 ? nsub - 1 : sub - 1;
        });
  } else if (wave == 1) {
    float xn[AHEAD][3], vn[AHEAD][3], cn[AHEAD][3], fn[AHEAD];
    loading_stages(
        2,
        [&](int k, auto slot) {
          constexpr int D = decltype(slot)::value;
          const float* row = row_of(k);
          const tape4 x4 = tape_four(row, 20, cnt, tid);
          const tape2 v2 = tape_at<tape2>(row, T_V12<PEN>, cnt, tid);
#pragma unroll
          for (int m = 0; m < 3; ++m) xn[D][m] = x4[m];
          vn[D][0] = x4[3];
          vn[D][1] = v2[0];
          vn[D][2] = v2[1];
          // R[2], R[5], R[8]
          cn[D][0] = tape_at<float>(row, 8, cnt, 4 * tid + 2);
          cn[D][1] = tape_at<float>(row, 12, cnt, 4 * tid + 1);
          cn[D][2] = tape_at<float>(row, 16, cnt, 4 * tid);
          fn[D] = tape_word_at<PEN>(row, cnt, tid);
        },
        [&](int k, auto slot, auto&& next) {
          constexpr int D = decltype(slot)::value;
          if (!live) return;
          Quad s;
          s.ev = 0u;
          float c2[3], v0[3];
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            s.x[m] = xn[D][m];
            s.v[m] = v0[m] = vn[D][m];
            c2[m] = cn[D][m];
          }
          s.fl = word_flag(__float_as_uint(fn[D]), me, 0);
          next();
          const float T = mring[k % 5][0][tid].x;
          const uint32_t ev = trans_step<true>(c, pp, s, T, c2[0], c2[1], c2[2], (uint32_t)q,
                                         t0 + (unsigned long long)k);
          float(*tl)[BS] = tile[k & 1];
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            tl[m][tid] = s.xo[m];
            tl[3 + m][tid] = s.inc[m];
            tl[6 + m][tid] = s.v[m];
          }
          tring[k & 1][0][tid] = make_float4(T * c2[0], T * c2[1], T * c2[2], v0[0]);
          tring[k & 1][1][tid] = make_float4(v0[1], v0[2], __uint_as_float(ev), 0.f);
        });
  } else if (wave == 2) {
    float Rn[AHEAD][9], wn[AHEAD][3];
    auto load = [&](int k, auto slot) {
      constexpr int D = decltype(slot)::value;
      const float* row = row_of(k);
      const tape4 a = tape_four(row, 8, cnt, tid), b = tape_four(row, 12, cnt, tid),
                  d = tape_four(row, 16, cnt, tid);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        Rn[D][m] = a[m];
        Rn[D][4 + m] = b[m];
      }
      Rn[D][8] = d[0];
#pragma unroll
      for (int m = 0; m < 3; ++m) wn[D][m] = d[1 + m];
    };
    loading_stages(2, load, [&](int k, auto slot, auto&& next) {
      constexpr int D = decltype(slot)::value;
      if (!live) return;
      float R[9], w[3];
#pragma unroll
      for (int m = 0; m < 9; ++m) R[m] = Rn[D][m];
#pragma unroll
      for (int m = 0; m < 3; ++m) w[m] = wn[D][m];
      next();
      const float4 d = mring[k % 5][0][tid];
      Rec r;
      rot_step<true>(c, pp, R, w, d.y, d.z, d.w, &r);
      float4(*rs)[BS] = rring[k % 3];
      rs[0][tid] = make_float4(r.P[0], r.P[1], r.P[2], r.P[3]);
      rs[1][tid] = make_float4(r.P[4], r.P[5], r.P[6], r.P[7]);
      rs[2][tid] = make_float4(r.P[8], r.w0[0], r.w0[1], r.w0[2]);
      rs[3][tid] = make_float4(r.wdot[0], r.wdot[1], r.wdot[2], r.i0);
      rs[4][tid] = make_float4(r.w1[0], r.w1[1], r.w1[2], r.i1);
      rs[5][tid] = make_float4(r.A1[0], r.A1[1], r.A1[2], r.dp);
      rs[6][tid] = make_float4(r.c0[0], r.c0[1], r.c0[2], 0.f);
      rs[7][tid] = make_float4(r.c1[0], r.c1[1], r.c1[2], 0.f);
    });
  } else if (wave == 5) {
    // the translation's derivative
    float lx[3], lv[3], pn[AHEAD][3];
    float wn[AHEAD];
    if (live) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        lx[k] = my[S_X + k];
        lv[k] = my[S_V + k];
      }
    }
    auto load = [&](int k, auto slot) {
      constexpr int D = decltype(slot)::value;
      const float* row = row_of(k);
      if constexpr (PEN) {
        const tape4 w4 = tape_four(row, T_WORD<PEN>, cnt, tid);
        wn[D] = w4[0];
#pragma unroll
        for (int m = 0; m < 3; ++m) pn[D][m] = w4[1 + m];
      } else {
        wn[D] = tape_word_at<PEN>(row, cnt, tid);
      }
    };
    loading_stages(3, load, [&](int k, auto slot, auto&& next) {
      constexpr int D = decltype(slot)::value;
      uint32_t cm = 0u;  // partners whose response the quad received
      if (live) {
        cm = word_resp(__float_as_uint(wn[D]), me, 0);
        if constexpr (PEN) {
#pragma unroll
          for (int m = 0; m < 3; ++m) lx[m] += pn[D][m];
        }
        next();
      }
      if (__ballot(cm != 0u) != 0ull) {  // rare
        const float(*tl)[BS] = tile[k & 1];
        float ldv[3] = {0.f, 0.f, 0.f};
        if (cm != 0u) {
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            ldv[m] = c.col_decay * lv[m];
            lv[m] = ldv[m];
          }
        }
#pragma unroll
        for (int m = 0; m < 3; ++m) ldvt[m][tid] = ldv[m];
        wave_sync();
        if (cm != 0u) {
          Quad so;
#pragma unroll
          for (int m = 0; m < 3; ++m) {
            so.xo[m] = tl[m][tid];
            so.inc[m] = tl[3 + m][tid];
            so.v[m] = tl[6 + m][tid];
          }
          response_vjp<BS>(c, tl, ldvt, so, ls, me, cm, ldv, lx, lv);
        }
        wave_sync();
      }
      if (live) {
        const float4 a = tring[k & 1][0][tid], b = tring[k & 1][1][tid];
        const float F[3] = {a.x, a.y, a.z}, v0[3] = {a.w, b.x, b.y};
        float lF[3];
        lring[k % 3][tid] = vjp_trans(c, pp, __float_as_uint(b.z), F, v0, lx, lv, lF);
        aring[k & 1][tid] = make_float4(lF[0], lF[1], lF[2], b.z);
      }
    });
    if (live) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        out[S_X + k] = lx[k];
        out[S_V + k] = lv[k];
      }
      out[S_F] = 0.f;
    }
  } else if (wave == 3) {
    // the rotation's derivative
    float lR[9], lw[3], gJ[3] = {0.f, 0.f, 0.f};
    if (live) {
#pragma unroll
      for (int k = 0; k < 9; ++k) lR[k] = my[S_R + k];
#pragma unroll
      for (int k = 0; k < 3; ++k) lw[k] = my[S_W + k];
    }
    stages(4, [&](int k) {
      if (!live) return;
      const float4(*rs)[BS] = rring[k % 3];
      float4 v[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) v[m] = rs[m][tid];
      const float4 a = aring[k & 1][tid];
      Rec r;
      r.T = mring[k % 5][0][tid].x;
      r.P[0] = v[0].x; r.P[1] = v[0].y; r.P[2] = v[0].z; r.P[3] = v[0].w;
      r.P[4] = v[1].x; r.P[5] = v[1].y; r.P[6] = v[1].z; r.P[7] = v[1].w;
      r.P[8] = v[2].x; r.w0[0] = v[2].y; r.w0[1] = v[2].z; r.w0[2] = v[2].w;
      r.wdot[0] = v[3].x; r.wdot[1] = v[3].y; r.wdot[2] = v[3].z; r.i0 = v[3].w;
      r.w1[0] = v[4].x; r.w1[1] = v[4].y; r.w1[2] = v[4].z; r.i1 = v[4].w;
      r.A1[0] = v[5].x; r.A1[1] = v[5].y; r.A1[2] = v[5].z; r.dp = v[5].w;
      r.c0[0] = v[6].x; r.c0[1] = v[6].y; r.c0[2] = v[6].z;
      r.c1[0] = v[7].x; r.c1[1] = v[7].y; r.c1[2] = v[7].z;
      const float lF[3] = {a.x, a.y, a.z};
      float lt[3], lJ[3];
      const float lT = vjp_rot(c, pp, r, __float_as_uint(a.w), lF, lR, lw, lt, lJ);
      bring[k & 1][tid] = make_float4(lT, lt[0], lt[1], lt[2]);
#pragma unroll
      for (int m = 0; m < 3; ++m) gJ[m] += lJ[m];
    });
    if (live) {
#pragma unroll
      for (int k = 0; k < 9; ++k) out[S_R + k] = lR[k];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        out[S_W + k] = lw[k];
        add_par(gpar, q, 1 + k, gJ[k]);
      }
    }
  } else {
    // the motor's derivative
    float lu[4], le[4], gu[4] = {0.f, 0.f, 0.f, 0.f}, gm = 0.f, gt2w = 0.f, gtau = 0.f;
    if (live) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        lu[k] = my[S_U + k];
        le[k] = my[S_E + k];
      }
    }
    int call = ncalls - 1, sub = nsub - 1;
    stages(5, [&](int k) {
      if (sub == nsub - 1) {
#pragma unroll
        for (int m = 0; m < 4; ++m) gu[m] = 0.f;
      }
      if (live) {
        const float4(*ms)[BS] = mring[k % 5];
        const float4 z4 = ms[1][tid], u04 = ms[2][tid], u14 = ms[3][tid],
                     uh4 = uring[k % 6][0][tid];
        const float4 b = bring[k & 1][tid];
        const float z[4] = {z4.x, z4.y, z4.z, z4.w}, u0[4] = {u04.x, u04.y, u04.z, u04.w};
        const float u1[4] = {u14.x, u14.y, u14.z, u14.w}, uhat[4] = {uh4.x, uh4.y, uh4.z, uh4.w};
        const float lt[3] = {b.y, b.z, b.w};
        vjp_motor(c, pp, pa, u0, u1, z, uhat, b.x, lt, lring[k % 3][tid], lu, le, gu, gm, gt2w,
                  gtau);
        if (sub == 0) {
          const float4 da = uring[k % 6][1][tid];
          float4 g;
          g.x = gu[0] * da.x;
          g.y = gu[1] * da.y;
          g.z = gu[2] * da.z;
          g.w = gu[3] * da.w;
          reinterpret_cast<float4*>(gact + (long long)call * Q * 4)[q] = g;
        }
      }
      if (--sub < 0) {
        sub = nsub - 1;
        --call;
      }
    });
    if (live) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        out[S_U + k] = lu[k];
        out[S_E + k] = le[k];
      }
      add_par(gpar, q, 0, gm);
      add_par(gpar, q, 4, gt2w);
      add_par(gpar, q, 5, gtau);
    }
  }
  wg_sync();
  move_rows<BS, 448, false>(gout, qb, cnt, sh, threadIdx.x);
}

// ---------------------------------------------------------------------------
// Row-major [Q][27] to field-major [27][Q], 64 quads a workgroup.
__global__ __launch_bounds__(64) void rows_to_fields_kernel(const float* __restrict__ src,
                                                            float* __restrict__ dst, int Q) {
  __shared__ float sh[64 * NSTATE];
  const int tid = threadIdx.x, qb = blockIdx.x * 64, cnt = min(64, Q - qb);
  move_rows<64, 64, true>(src, qb, cnt, sh, tid);
  __syncthreads();
  if (tid < cnt) {
#pragma unroll
    for (int f = 0; f < NSTATE; ++f) dst[(size_t)f * Q + qb + tid] = sh[tid * NSTATE + f];
  }
}

__global__ void copy_kernel(const float* __restrict__ src, float* __restrict__ dst, long long n) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = src[i];
}

__global__ void fill_kernel(float* __restrict__ dst, long long n, float v) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dst[i] = v;
}

}  // namespace qs
