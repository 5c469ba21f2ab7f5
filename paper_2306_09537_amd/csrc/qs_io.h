// Kernels around the step: the graph-mode counter, the parameters, the state in
// and out of a handle, and the generator's diagnostics.
#pragma once
#include "qs_kernels.h"

namespace qs {

// Set the graph-mode counter and clear the completion counts (one
// workgroup of 64 threads).
__global__ void set_counter_kernel(unsigned long long* tdev, unsigned int* done,
                                   unsigned long long v) {
  if (blockIdx.x != 0) return;
  if (threadIdx.x == 0) __hip_atomic_exchange(tdev, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (int i = threadIdx.x; i <= DONE_SUBS; i += blockDim.x)
    __hip_atomic_exchange(done + DONE_STRIDE * i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Per-quad parameters [Q][6] (mass, ixx, iyy, izz, thrust-to-weight, tau_m)
// -> the handle's array, for environments selected by env_mask, with f_max and
// alpha_lag derived in double and rounded once (as at creation).  A row
// with a non-finite or non-positive entry is left as it was and raises the
// sticky parameter error bit.
__global__ void set_params_kernel(float* __restrict__ par, int Q,
                                  const float* __restrict__ src,
                                  const int32_t* __restrict__ qenv,
                                  const uint8_t* __restrict__ env_mask, float dt, float g,
                                  int* err) {
  const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (q >= Q) return;
  if (env_mask && env_mask[qenv[q]] == 0) return;
  float v[6];
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    v[k] = src[(size_t)q * 6 + k];
    ok = ok && isfinite(v[k]) && v[k] > 0.0f;
  }
  if (!ok) {
    __hip_atomic_fetch_or(err, ERRBIT_PARAM, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  static_assert(P_JZ == 3 && P_FMAX == 4 && P_ALAG == 5 && P_T2W == 6 && P_TAU == 7,
                "a group of four and two pairs");
  *reinterpret_cast<v4f*>(par + par_index(q, P_M)) = v4f{v[0], v[1], v[2], v[3]};
  *reinterpret_cast<v2f*>(par + par_index(q, P_FMAX)) =
      v2f{(float)(0.25 * (double)v[0] * (double)g * (double)v[4]),
          (float)(1.0 - exp(-(double)dt / (double)v[5]))};
  *reinterpret_cast<v2f*>(par + par_index(q, P_T2W)) = v2f{v[4], v[5]};
}

// The library's counter-based generator, exported for tests: for quads
// quad0 .. quad0 + n - 1 at substep t, the four Philox4x32-10 words of
// (stream, draw) into words[n][4] and, when normals is not null, the four
// N(0,1) draws built from them into normals[n][4].
__global__ void philox_debug_kernel(uint32_t key0, uint32_t key1, uint32_t stream,
                                    uint32_t draw, unsigned long long t, uint32_t quad0, int n,
                                    uint32_t* __restrict__ words, float* __restrict__ normals) {
  const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (i >= n) return;
  const uint32_t q = quad0 + (uint32_t)i;
  uint32_t r0 = q, r1 = (uint32_t)t, r2 = (uint32_t)(t >> 32), r3 = (stream << 8) | draw;
  philox4x32_10(r0, r1, r2, r3, key0, key1);
  words[4 * (size_t)i + 0] = r0;
  words[4 * (size_t)i + 1] = r1;
  words[4 * (size_t)i + 2] = r2;
  words[4 * (size_t)i + 3] = r3;
  if (normals) {
    Consts c{};
    c.key0 = key0;
    c.key1 = key1;
    float z[4];
    normal4(c, q, t, stream, draw, z);
#pragma unroll
    for (int k = 0; k < 4; ++k) normals[4 * (size_t)i + k] = z[k];
  }
}

// Row-major [Q][27] <-> the handle's tiles of 64 quads: the rows of
// a tile are one contiguous run, moved 16 bytes a lane where the caller's
// buffer allows it, as are the tile's groups, and the turn happens in
// LDS (a row stride of 27 words is odd, so neither side meets a bank
// conflict).  Bound by HBM; reading or writing the field-major side word by
// word in row order touched 27 lines per wavefront access (1,048,576 quads,
// 226 MB: state in 181 -> 36 us, state out 104 -> 45 us).
constexpr int IO_QUADS = TILE_QUADS, IO_THREADS = 256;

// Rows [q0, q0 + cnt) of src -> t.
__device__ __forceinline__ void load_rows(const float* __restrict__ src, int q0, int cnt,
                                          float* t) {
  const float* run = src + (size_t)q0 * NSTATE;
  const int total = cnt * NSTATE;
  int i0 = 0;
  if ((reinterpret_cast<uintptr_t>(run) & 15) == 0) {
    const float4* r4 = reinterpret_cast<const float4*>(run);
    for (int i = threadIdx.x; i < total >> 2; i += IO_THREADS)
      reinterpret_cast<float4*>(t)[i] = r4[i];
    i0 = total & ~3;
  }
  for (int i = i0 + threadIdx.x; i < total; i += IO_THREADS) t[i] = run[i];
}

// Canonical [Q][27] -> the handle's tiles, for environments selected by env_mask.
__global__ __launch_bounds__(IO_THREADS) void set_state_kernel(
    float* __restrict__ st, int Q, const float* __restrict__ src,
    const int32_t* __restrict__ qenv, const uint8_t* __restrict__ env_mask) {
  __shared__ __align__(16) float t[IO_QUADS * NSTATE];
  const int q0 = blockIdx.x * IO_QUADS, cnt = min(IO_QUADS, Q - q0);
  const int lane = threadIdx.x & 63;
  bool mine = lane < cnt;
  if (env_mask && mine) mine = env_mask[qenv[q0 + lane]] != 0;
  // the selected quads of the tile, the same in each of the four wavefronts
  const unsigned long long sel = __ballot(mine);
  if (sel == 0ull) return;
  if (env_mask) {  // the rows of the selected quads only
    for (int i = threadIdx.x; i < cnt * NSTATE; i += IO_THREADS)
      if (sel >> (i / NSTATE) & 1ull) t[i] = src[(size_t)q0 * NSTATE + i];
  } else {
    load_rows(src, q0, cnt, t);
  }
  __syncthreads();
  if (!mine) return;
  float* tile = st_tile(st, q0);
  const float* row = t + lane * NSTATE;
  const int g = threadIdx.x >> 6;  // the wavefront's first group; its second is g + 4
  auto put = [&](int g) {
    put_tile_four(tile, g * 4 * TILE_QUADS, lane, row[st_field(4 * g)], row[st_field(4 * g + 1)],
                  row[st_field(4 * g + 2)], row[st_field(4 * g + 3)]);
  };
  put(g);
  if (g < 2) {
    put(g + 4);
  } else if (g == 2) {
#pragma unroll
    for (int k = 0; k < 3; ++k) tile[ST_VF + 3 * lane + k] = row[st_field(24 + k)];
  }
}

// The handle's tiles -> canonical [Q][27].
__global__ __launch_bounds__(IO_THREADS) void get_state_kernel(const float* __restrict__ st,
                                                               int Q,
                                                               float* __restrict__ dst) {
  __shared__ __align__(16) float t[IO_QUADS * NSTATE];
  const int q0 = blockIdx.x * IO_QUADS, cnt = min(IO_QUADS, Q - q0);
  const int lane = threadIdx.x & 63;
  // (the private arrays are padded to whole tiles)
  const float* tile = st_tile(st, q0);
  float* row = t + lane * NSTATE;
  const int g = threadIdx.x >> 6;  // the wavefront's first group; its second is g + 4
  const v4f a = tile_four(tile, g * 4 * TILE_QUADS, lane);
  if (g < 2) {
    const v4f b = tile_four(tile, (g + 4) * 4 * TILE_QUADS, lane);
#pragma unroll
    for (int k = 0; k < 4; ++k) row[st_field(4 * g + 16 + k)] = b[k];
  } else if (g == 2) {
    const float* vf = tile + ST_VF + 3 * lane;
    const float b[3] = {vf[0], vf[1], vf[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k) row[st_field(24 + k)] = b[k];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) row[st_field(4 * g + k)] = a[k];
  __syncthreads();
  float* run = dst + (size_t)q0 * NSTATE;
  const int total = cnt * NSTATE;
  int i0 = 0;
  if ((reinterpret_cast<uintptr_t>(run) & 15) == 0) {
    float4* r4 = reinterpret_cast<float4*>(run);
    for (int i = threadIdx.x; i < total >> 2; i += IO_THREADS)
      r4[i] = reinterpret_cast<const float4*>(t)[i];
    i0 = total & ~3;
  }
  for (int i = i0 + threadIdx.x; i < total; i += IO_THREADS) run[i] = t[i];
}

}  // namespace qs
