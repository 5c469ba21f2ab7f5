// Device-side building blocks of the quadrotor-swarm step (gfx950, wave64).
//
// One lane owns one quad.  Its state lives in VGPRs for the whole call; a
// workgroup owns whole environments (never split), so the in-env pair pass
// and the nearest-neighbour search read swarm-mates' positions and
// velocities from LDS after a workgroup barrier (swarms of at most 8 take
// the neighbour candidates' positions from their lanes instead, and larger
// swarms take the neighbour keys from the last pair pass's screen).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace qs {

enum : uint32_t {
  F_ROOM = 1u, F_FLOOR = 2u, F_COLLIDE = 4u, F_NOISE = 8u, F_APPROACH = 16u, F_ACT_UNIT = 32u,
  F_DOWNWASH = 64u, F_SENSOR = 128u
};
enum : int { NSTATE = 27, NPARAM = 8 };
// clang vector types, for the non-temporal store builtin
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
// field index of a quad's state: x3 v3 R9 (row-major) w3 u4 eps4 floor
enum : int { S_X = 0, S_V = 3, S_R = 6, S_W = 15, S_U = 18, S_E = 22, S_F = 26 };
// index of the per-quad parameters (the forward reads the first six)
enum : int { P_M = 0, P_JX = 1, P_JY = 2, P_JZ = 3, P_FMAX = 4, P_ALAG = 5, P_T2W = 6, P_TAU = 7 };
// The handle's arrays hold the quads in tiles of 64, a quad's words in groups of
// four (16 bytes a lane, a tile's state 6912 bytes in a row): u, e, R[0..3],
// R[4..7], R[8] and w, x and v[0], then v[1], v[2] and the flag; the parameters in
// a group of four and two pairs, of which the forward reads the first.  Field by field over all quads a wavefront went to 33 places
// megabytes apart, and a small swarm to a part of a cache line at each.  us a call
// of one substep: 32768 x 32 108 -> 96 and 1,048,576 single quads 71 -> 68 on two
// handles in turn, 79.1 -> 79.9 and 52.4 -> 52.6 on one, whose arrays stay in the
// memory-side cache; 2,097,152 quads in swarms of 1, 8, 32 and 12: 123 -> 114,
// 195 -> 170, 202 -> 173, 272 -> 203.
constexpr int TILE_QUADS = 64;
constexpr int ST_U = 0, ST_E = 4 * 64, ST_R0 = 8 * 64, ST_R4 = 12 * 64, ST_R8W = 16 * 64,
              ST_XV = 20 * 64, ST_VF = 24 * 64;  // words before a group in the tile
__host__ __device__ constexpr int st_place(int f) {  // of field f in the order above
  return f < S_R ? f + 20 : f < S_U ? f + 2 : f < S_F ? f - 18 : 26;
}
__host__ __device__ constexpr int st_field(int place) {  // its inverse
  return place < 8 ? place + 18 : place < 20 ? place - 2 : place < 26 ? place - 20 : 26;
}
__host__ __device__ inline size_t st_index(int q, int f) {
  const int place = st_place(f), lane = q & 63;
  return (size_t)(q >> 6) * (NSTATE * TILE_QUADS) +
         (place < 24 ? (place & ~3) * TILE_QUADS + 4 * lane + (place & 3)
                     : ST_VF + 3 * lane + place - 24);
}
__host__ __device__ inline size_t par_index(int q, int k) {
  const int lane = q & 63;
  return (size_t)(q >> 6) * (NPARAM * TILE_QUADS) +
         (k < 4 ? 4 * lane + k : (k & ~1) * TILE_QUADS + 2 * lane + (k & 1));
}
// noise streams: fourth Philox counter word = stream << 8 | draw
enum : uint32_t {
  STREAM_MOTOR = 0, STREAM_WALL = 1, STREAM_PAIR = 2, STREAM_DOWNWASH = 3, STREAM_SENSOR = 4
};
// events of a call, for the reward's interaction terms
enum : uint32_t { EVF_FLOOR_HIT = 1u, EVF_WALL = 2u, EVF_CEILING = 4u, EVF_QUAD = 8u };
enum : int { ERRBIT_STATE = 1, ERRBIT_ACTION = 2, ERRBIT_PARAM = 4 };

struct Consts {
  float dt, g, arm_d, k_tau, drag, mu;
  float a_nd, ns_scale;  // motor noise: eps <- a_nd eps + ns_scale f_max z
  float rmin0, rmin1, rmin2, rmax0, rmax1, rmax2, e_wall;
  float dcol2, dcol, col_decay, col_nv, col_nw;
  uint32_t flags;
  uint32_t key0, key1;
  int32_t K;
  int32_t obs_dim;
  // downwash: -k1 (k2 dz + b1) e_z within |dxy|^2 < dw_r2, 0 < dz < dw_h
  float dw_k1, dw_k2, dw_b1, dw_r2, dw_h, dw_na, dw_nw;
  // observation sensor noise: uniform half-widths (x - goal, v), Gaussian std (omega)
  float sn_x, sn_v, sn_w;
  // reward weights: pos, vel, ori, spin, act, dact, rot, yaw, floor_hit,
  // on_floor, wall, ceiling, quad, prox, and the proximity distance
  float rw[15];
};

struct Ptrs {
  float* st;                    // private state, tiles of 64 quads (st_index)
  const float* par;             // the quads' parameters, the same (par_index)
  const uint32_t* sw;           // (env start within the block << 8) | n_e
  const int2* blk;              // [nblk] (first quad, quad count)
  unsigned long long* contacts; // a word per quad, or nullptr
  int* err;                     // sticky error bits
  int Q;                        // quad count
  const int4* items;            // uneven sizes: (slot size, first env entry, swarms, -)
  const int2* item_envs;        // uneven sizes: (first quad, size) per swarm of an item
};

// The tile words of quad q, and its group of four at word g of the tile.
__device__ __forceinline__ const float* st_tile(const float* st, int q) {
  return st + (size_t)(q >> 6) * (NSTATE * TILE_QUADS);
}
__device__ __forceinline__ float* st_tile(float* st, int q) {
  return st + (size_t)(q >> 6) * (NSTATE * TILE_QUADS);
}
__device__ __forceinline__ v4f tile_four(const float* tile, int g, int q) {
  return reinterpret_cast<const v4f*>(tile + g)[q & 63];
}
__device__ __forceinline__ void put_tile_four(float* tile, int g, int q, float a, float b, float c,
                                              float d) {
  reinterpret_cast<v4f*>(tile + g)[q & 63] = v4f{a, b, c, d};
}

// Philox4x32-10, Salmon et al. SC'11: ten rounds of two 32x32->64 products
// with a Weyl-sequence key schedule.
__device__ __forceinline__ void philox4x32_10(uint32_t& c0, uint32_t& c1, uint32_t& c2,
                                              uint32_t& c3, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint64_t pa = (uint64_t)0xD2511F53u * c0;
    const uint64_t pb = (uint64_t)0xCD9E8D57u * c2;
    const uint32_t n0 = (uint32_t)(pb >> 32) ^ c1 ^ k0;
    const uint32_t n2 = (uint32_t)(pa >> 32) ^ c3 ^ k1;
    c1 = (uint32_t)pb;
    c3 = (uint32_t)pa;
    c0 = n0;
    c2 = n2;
    k0 += 0x9E3779B9u;
    k1 += 0xBB67AE85u;
  }
}

// Uniform (2 (r >> 9) + 1) 2^-24 in (0,1): exact in float32.
__device__ __forceinline__ float u01(uint32_t r) {
  return (float)(((r >> 9) << 1) | 1u) * 5.9604644775390625e-8f;
}

// Four N(0,1) draws by Box-Muller for (quad, substep, stream, draw):
// radius sqrt(-2 ln u0) = sqrt(-2 ln2 log2 u0), angle 2 pi u1.  The hardware
// log2, sqrt and the sine/cosine of an angle given in revolutions are used
// directly: on every u = (2m + 1) 2^-24 their errors are about one ulp
// (sin/cos 1.3e-7 absolute, log2 1.2e-7 relative, near u = 1 included),
// giving draws within 6e-7 of the exact ones, at a fraction of the library
// functions' instruction count.
__device__ __forceinline__ void normal4(const Consts& c, uint32_t q, uint64_t t,
                                        uint32_t stream, uint32_t draw, float z[4]) {
  uint32_t r0 = q, r1 = (uint32_t)t, r2 = (uint32_t)(t >> 32), r3 = (stream << 8) | draw;
  philox4x32_10(r0, r1, r2, r3, c.key0, c.key1);
  constexpr float m2ln2 = -1.3862943611198906f;  // -2 ln 2
  float rad = __builtin_amdgcn_sqrtf(m2ln2 * __builtin_amdgcn_logf(u01(r0)));
  float a = u01(r1);
  z[0] = rad * __builtin_amdgcn_cosf(a);
  z[1] = rad * __builtin_amdgcn_sinf(a);
  rad = __builtin_amdgcn_sqrtf(m2ln2 * __builtin_amdgcn_logf(u01(r2)));
  a = u01(r3);
  z[2] = rad * __builtin_amdgcn_cosf(a);
  z[3] = rad * __builtin_amdgcn_sinf(a);
}

// Per-quad registers.  xo/inc are the substep's start position and
// displacement: the pair pass measures separations as
// (xo_i - xo_j) + (inc_i - inc_j), which keeps ~1e-9 m accuracy for
// centimetre gaps between quads several metres from the origin, where the
// difference of the rounded end positions would be off by ~1e-6 m.
struct Quad {
  float x[3], v[3], R[9], w[3], u[4], e[4];
  float fl;
  float xo[3], inc[3];
  uint32_t ev;  // EVF_* bits of the current call
};

struct QuadPar {
  float m, inv_m, jx, jy, jz, ijx, ijy, ijz, f_max, a_lag, a_ns;
};

// The parameters that the forward substep reads, as they are held.
__device__ __forceinline__ void load_forward_params(const Ptrs& p, int q, QuadPar& pp) {
  const v4f a = *reinterpret_cast<const v4f*>(p.par + par_index(q, P_M));
  const v2f b = *reinterpret_cast<const v2f*>(p.par + par_index(q, P_FMAX));
  pp.m = a[0];
  pp.jx = a[1];
  pp.jy = a[2];
  pp.jz = a[3];
  pp.f_max = b[0];
  pp.a_lag = b[1];
}

// Median of three unsigned words (one v_med3_u32).
__device__ __forceinline__ uint32_t umed3(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));
}

__device__ __forceinline__ float clampf(float a, float lo, float hi) {
  return fminf(fmaxf(a, lo), hi);
}

// §III-A.1: rotor-speed command from the normalised thrust action.
__device__ __forceinline__ float rotor_cmd(float a, bool unit) {
  // both maps, then a select: a branch on the flag would end the scheduling
  // region (and wait for the action load) once per rotor
  const float fu = clampf(a, 0.0f, 1.0f);
  const float fs = 0.5f * (clampf(a, -1.0f, 1.0f) + 1.0f);
  return sqrtf(unit ? fu : fs);
}

// Events of one substep of one quad.
enum : uint32_t {
  SUB_REST = 1u,      // resting on the floor
  SUB_GUARD = 2u,     // friction stopped it
  SUB_BOUNCED = 4u,   // off a wall or the ceiling
  SUB_HIT = 8u,       // hit the floor
  SUB_CLAMP = 16u,    // << axis: position held to the room
  SUB_FLIP = 128u,    // << axis: velocity mirrored
  SUB_PAIR = 1024u,   // collision response received
  SUB_DOWNWASH = 2048u,
  SUB_TURNS = SUB_REST | SUB_BOUNCED | SUB_HIT | SUB_PAIR | SUB_DOWNWASH  // those that touch R or w
};

// Intermediates of one substep kept for the reverse sweep (adjoint).
struct Rec {
  float z[4], u0[4], u1[4], P[9], w0[3], v0[3], T;
  float wdot[3], w1[3], A1[3], i0, c0[3], dp, i1, c1[3];  // i0, i1: inverse column norms
  uint32_t ev;  // SUB_*
};

// Where the motor-noise draws of a substep come from: generated (Z_DRAW),
// generated and also written to zio[4] (Z_EXPORT), or read from zio[4]
// (Z_IMPORT: the draws an earlier Z_EXPORT run saved for this quad and
// substep).
enum ZMode { Z_DRAW, Z_EXPORT, Z_IMPORT };

// Thrust and body torques of one substep: the output of the motor part.
struct Drive {
  float T, tx, ty, tz;
};

// §III-A.1 motor lag, §III-A.2 motor noise (AR(1)) and per-rotor thrust,
// §III-A X mix: updates the rotor state (u, eps) and returns the thrust and
// torques.  Depends on the rotor state, the command and the substep's draws
// only (not on position, velocity or attitude).  z: the draws (zeros
// without motor noise).
template <ZMode ZM = Z_DRAW>
__device__ __forceinline__ Drive motor_step(const Consts& c, const QuadPar& p, float u[4],
                                            float e[4], const float uhat[4], uint32_t q,
                                            uint64_t t, float z[4], float* zio = nullptr) {
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = fmaf(p.a_lag, uhat[i] - u[i], u[i]);
  if (c.flags & F_NOISE) {
    if constexpr (ZM == Z_IMPORT) {
#pragma unroll
      for (int i = 0; i < 4; ++i) z[i] = zio[i];
    } else {
      normal4(c, q, t, STREAM_MOTOR, 0, z);
    }
    if constexpr (ZM == Z_EXPORT) {
#pragma unroll
      for (int i = 0; i < 4; ++i) zio[i] = z[i];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) e[i] = fmaf(c.a_nd, e[i], p.a_ns * z[i]);
  }
  // X layout FR, BR, BL, FL
  float f[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = fmaf(p.f_max * u[i], u[i], e[i]);
  Drive d;
  d.T = (f[0] + f[1]) + (f[2] + f[3]);
  d.tx = c.arm_d * ((f[2] + f[3]) - (f[0] + f[1]));
  d.ty = c.arm_d * ((f[1] + f[2]) - (f[0] + f[3]));
  d.tz = c.k_tau * ((f[0] + f[2]) - (f[1] + f[3]));
  return d;
}

// Friction force in the plane on a quad resting on the floor under thrust F
// (static when still, kinetic when sliding).
struct Friction {
  float mu_n, fb[2], nv, nf, mag;
  bool still;
};
__device__ __forceinline__ Friction floor_friction(const Consts& c, const QuadPar& p,
                                                   const float F[3], const float v[2]) {
  Friction f;
  f.mu_n = c.mu * (p.m * c.g - F[2]);
  f.still = v[0] == 0.0f && v[1] == 0.0f;
  f.nv = f.nf = f.mag = 0.0f;
  if (f.still) {
    f.nf = sqrtf(F[0] * F[0] + F[1] * F[1]);
    const float mag = fmaxf(f.nf - f.mu_n, 0.0f);
    const float sc = f.nf > 0.0f ? mag / f.nf : 0.0f;
    f.fb[0] = sc * F[0];
    f.fb[1] = sc * F[1];
    f.mag = f.nf > 0.0f ? mag : 0.0f;
  } else {
    f.nv = sqrtf(v[0] * v[0] + v[1] * v[1]);
    const float iv = f.mu_n / f.nv;
    f.fb[0] = F[0] - iv * v[0];
    f.fb[1] = F[1] - iv * v[1];
  }
  return f;
}

// The translation of a substep in free flight from its world-frame thrust F,
// by semi-implicit Euler.  Updates x, v, xo, inc and fl of s; returns whether
// the quad rests on the floor instead: free flight is computed for every lane
// (one scheduling region) and the rare resting lane then redoes the substep
// (trans_rest) from the start values v0, fl0.
__device__ __forceinline__ bool trans_free(const Consts& c, const QuadPar& p, Quad& s,
                                           const float F[3], float v0[2], float& fl0) {
#pragma unroll
  for (int k = 0; k < 3; ++k) s.xo[k] = s.x[k];
  const bool rest = (c.flags & F_FLOOR) && s.fl != 0.0f && F[2] <= p.m * c.g;
  v0[0] = s.v[0];
  v0[1] = s.v[1];
  fl0 = s.fl;
  s.fl = 0.0f;
  const float dm = c.drag * p.inv_m;
  const float ax = fmaf(F[0], p.inv_m, -dm * s.v[0]);
  const float ay = fmaf(F[1], p.inv_m, -dm * s.v[1]);
  const float az = fmaf(F[2], p.inv_m, -dm * s.v[2]) - c.g;
  // semi-implicit Euler
  s.v[0] = fmaf(c.dt, ax, s.v[0]);
  s.v[1] = fmaf(c.dt, ay, s.v[1]);
  s.v[2] = fmaf(c.dt, az, s.v[2]);
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    s.inc[k] = c.dt * s.v[k];
    s.x[k] = fmaf(c.dt, s.v[k], s.x[k]);
  }
  return rest;
}

// §III-B.3 resting on the floor: friction in xy, no vertical motion, no
// rotation.
__device__ __forceinline__ uint32_t trans_rest(const Consts& c, const QuadPar& p, Quad& s,
                                               const float F[3], const float v0[2], float fl0) {
  uint32_t ev = SUB_REST;
  s.fl = fl0;
#pragma unroll
  for (int k = 0; k < 3; ++k) s.x[k] = s.xo[k];  // the substep's start position
  const Friction f = floor_friction(c, p, F, v0);
  s.v[0] = fmaf(c.dt, (f.fb[0] - c.drag * v0[0]) * p.inv_m, v0[0]);
  s.v[1] = fmaf(c.dt, (f.fb[1] - c.drag * v0[1]) * p.inv_m, v0[1]);
  s.v[2] = 0.0f;
  if (s.v[0] * v0[0] + s.v[1] * v0[1] < 0.0f) {
    s.v[0] = 0.0f;
    s.v[1] = 0.0f;
    ev |= SUB_GUARD;
  }
  s.inc[0] = c.dt * s.v[0];
  s.inc[1] = c.dt * s.v[1];
  s.inc[2] = 0.0f;
  s.x[0] = fmaf(c.dt, s.v[0], s.x[0]);
  s.x[1] = fmaf(c.dt, s.v[1], s.x[1]);
  return ev;
}

// Walls, ceiling and floor, after the motion.  bounced() and hit() are called
// in their rare branches, for a rotation at hand.  REC: the events the adjoint
// needs too, beside those that the rotation answers to.
template <bool REC, typename B, typename H>
__device__ __forceinline__ uint32_t trans_room(const Consts& c, Quad& s, uint32_t q, uint64_t t,
                                               B&& bounced, H&& hit) {
  uint32_t ev = 0u;
  // §III-B.2 walls and ceiling: the quad meets its mirror image
  if (c.flags & F_ROOM) {
    bool b = false;
    const float lo[2] = {c.rmin0, c.rmin1};
    const float hi[3] = {c.rmax0, c.rmax1, c.rmax2};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      // selects, not branches: hits are rare and the rest of the substep
      // stays one scheduling region
      if (k < 2) {
        const bool out = s.x[k] < lo[k];
        const bool flip = out && s.v[k] < 0.0f;
        s.x[k] = out ? lo[k] : s.x[k];
        s.inc[k] = out ? s.x[k] - s.xo[k] : s.inc[k];
        s.v[k] = flip ? -c.e_wall * s.v[k] : s.v[k];
        b = b | flip;
        s.ev |= flip ? (uint32_t)EVF_WALL : 0u;
        if constexpr (REC) ev |= (out ? SUB_CLAMP << k : 0u) | (flip ? SUB_FLIP << k : 0u);
      }
      const bool out = s.x[k] > hi[k];
      const bool flip = out && s.v[k] > 0.0f;
      s.x[k] = out ? hi[k] : s.x[k];
      s.inc[k] = out ? s.x[k] - s.xo[k] : s.inc[k];
      s.v[k] = flip ? -c.e_wall * s.v[k] : s.v[k];
      b = b | flip;
      s.ev |= flip ? (uint32_t)(k == 2 ? EVF_CEILING : EVF_WALL) : 0u;
      if constexpr (REC) ev |= (out ? SUB_CLAMP << k : 0u) | (flip ? SUB_FLIP << k : 0u);
    }
    if (b) {
      ev |= SUB_BOUNCED;
      float zv[4] = {0.f, 0.f, 0.f, 0.f};
      if (c.col_nv > 0.0f || c.col_nw > 0.0f) normal4(c, q, t, STREAM_WALL, 0, zv);
#pragma unroll
      for (int k = 0; k < 3; ++k) s.v[k] = c.col_decay * fmaf(c.col_nv, zv[k], s.v[k]);
      bounced();
    }
  }

  // §III-B.3 floor hit: stop and rest (the rotation levels the body)
  if ((c.flags & F_FLOOR) && s.x[2] < c.rmin2) {
    s.ev |= EVF_FLOOR_HIT;
    ev |= SUB_HIT;
    s.x[2] = c.rmin2;
    s.inc[2] = s.x[2] - s.xo[2];
    s.v[0] = s.v[1] = s.v[2] = 0.0f;
    s.fl = 1.0f;
    hit();
  }
  return ev;
}

// The whole translation, for a rotation kept elsewhere: from the thrust T along
// body z, the column (r2, r5, r8) of R.  Returns the substep's events.
template <bool REC = false>
__device__ __forceinline__ uint32_t trans_step(const Consts& c, const QuadPar& p, Quad& s, float T,
                                               float r2, float r5, float r8, uint32_t q,
                                               uint64_t t) {
  const float F[3] = {T * r2, T * r5, T * r8};
  float v0[2], fl0;
  uint32_t ev = 0u;
  if (trans_free(c, p, s, F, v0, fl0)) ev = trans_rest(c, p, s, F, v0, fl0);
  return ev | trans_room<REC>(c, s, q, t, [] {}, [] {});
}

// The rotation of a substep in free flight from its torques: Euler's
// equation, then R <- R + dt R [w]x with Gram-Schmidt.  REC: also record the
// intermediates the adjoint needs into *r.
template <bool REC = false>
__device__ __forceinline__ void rot_step(const Consts& c, const QuadPar& p, float R[9], float w[3],
                                         float tx, float ty, float tz, Rec* r = nullptr) {
  if constexpr (REC) {
#pragma unroll
    for (int k = 0; k < 9; ++k) r->P[k] = R[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) r->w0[k] = w[k];
  }
  // Euler's equation with the start-of-substep body rate
  const float Lx = p.jx * w[0], Ly = p.jy * w[1], Lz = p.jz * w[2];
  const float cx = w[1] * Lz - w[2] * Ly;
  const float cy = w[2] * Lx - w[0] * Lz;
  const float cz = w[0] * Ly - w[1] * Lx;
  const float wdx = (tx - cx) * p.ijx, wdy = (ty - cy) * p.ijy, wdz = (tz - cz) * p.ijz;
  w[0] = fmaf(c.dt, wdx, w[0]);
  w[1] = fmaf(c.dt, wdy, w[1]);
  w[2] = fmaf(c.dt, wdz, w[2]);
  if constexpr (REC) {
    r->wdot[0] = wdx;
    r->wdot[1] = wdy;
    r->wdot[2] = wdz;
#pragma unroll
    for (int k = 0; k < 3; ++k) r->w1[k] = w[k];
  }
  // R <- R + dt R [w]x (body rate), then Gram-Schmidt on the columns
  const float hx = c.dt * w[0], hy = c.dt * w[1], hz = c.dt * w[2];
  float c0[3], c1[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const float r0 = R[3 * k], r1 = R[3 * k + 1], r2 = R[3 * k + 2];
    c0[k] = r0 + (r1 * hz - r2 * hy);
    c1[k] = r1 + (r2 * hx - r0 * hz);
  }
  if constexpr (REC) {
#pragma unroll
    for (int k = 0; k < 3; ++k) r->A1[k] = c1[k];
  }
  const float i0 = rsqrtf(c0[0] * c0[0] + c0[1] * c0[1] + c0[2] * c0[2]);
#pragma unroll
  for (int k = 0; k < 3; ++k) c0[k] *= i0;
  const float dp = c0[0] * c1[0] + c0[1] * c1[1] + c0[2] * c1[2];
#pragma unroll
  for (int k = 0; k < 3; ++k) c1[k] = fmaf(-dp, c0[k], c1[k]);
  const float i1 = rsqrtf(c1[0] * c1[0] + c1[1] * c1[1] + c1[2] * c1[2]);
#pragma unroll
  for (int k = 0; k < 3; ++k) c1[k] *= i1;
  if constexpr (REC) {
    r->i0 = i0;
    r->i1 = i1;
    r->dp = dp;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      r->c0[k] = c0[k];
      r->c1[k] = c1[k];
    }
  }
  R[0] = c0[0]; R[3] = c0[1]; R[6] = c0[2];
  R[1] = c1[0]; R[4] = c1[1]; R[7] = c1[2];
  R[2] = c0[1] * c1[2] - c0[2] * c1[1];
  R[5] = c0[2] * c1[0] - c0[0] * c1[2];
  R[8] = c0[0] * c1[1] - c0[1] * c1[0];
}

// Heading of body x in the floor plane, its length, and what takes its place
// where the body stands on its nose.
struct Heading {
  float hx, hy, nh, kx, ky, nk;
  bool fallback;
};
__device__ __forceinline__ Heading floor_heading(float R0, float R1, float R3, float R4) {
  Heading h;
  h.hx = R0;
  h.hy = R3;
  h.nh = sqrtf(h.hx * h.hx + h.hy * h.hy);
  h.kx = R1;
  h.ky = R4;
  h.nk = sqrtf(R1 * R1 + R4 * R4);
  h.fallback = !(h.nh >= 1e-6f);
  return h;
}

// What a substep's events do to the rotation, after rot_step: rest holds the
// start attitude R0 without rotation; then a wall's kick turns the body, and a
// floor hit levels it keeping its heading.
__device__ __forceinline__ void rot_rest(float R[9], float w[3], const float R0[9]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) R[k] = R0[k];
  w[0] = w[1] = w[2] = 0.0f;
}
__device__ __forceinline__ void rot_bounced(const Consts& c, float w[3], uint32_t q, uint64_t t) {
  float zw[4] = {0.f, 0.f, 0.f, 0.f};
  if (c.col_nv > 0.0f || c.col_nw > 0.0f) normal4(c, q, t, STREAM_WALL, 1, zw);
#pragma unroll
  for (int k = 0; k < 3; ++k) w[k] = fmaf(c.col_nw, zw[k], w[k]);
}
__device__ __forceinline__ void rot_hit(float R[9], float w[3]) {
  w[0] = w[1] = w[2] = 0.0f;
  const Heading h = floor_heading(R[0], R[1], R[3], R[4]);
  float ax, ay;  // unit heading of body x in the floor plane
  if (!h.fallback) {
    ax = h.hx / h.nh;
    ay = h.hy / h.nh;
  } else {
    const float bx = h.nk > 0.0f ? h.kx / h.nk : 0.0f, by = h.nk > 0.0f ? h.ky / h.nk : 1.0f;
    ax = by;   // body x = body y x e_z
    ay = -bx;
  }
  R[0] = ax;  R[1] = -ay; R[2] = 0.0f;
  R[3] = ay;  R[4] = ax;  R[5] = 0.0f;
  R[6] = 0.0f; R[7] = 0.0f; R[8] = 1.0f;
}
__device__ __forceinline__ void rot_events(const Consts& c, uint32_t ev, float R[9], float w[3],
                                           const float R0[9], uint32_t q, uint64_t t) {
  if (ev & SUB_REST) rot_rest(R, w, R0);
  if (ev & SUB_BOUNCED) rot_bounced(c, w, q, t);
  if (ev & SUB_HIT) rot_hit(R, w);
}

// What the in-swarm pass's events do to the body rates, after rot_events: the
// noise of a collision response and of downwash.
__device__ __forceinline__ void rot_pair_events(const Consts& c, uint32_t ev, float w[3],
                                                uint32_t q, uint64_t t) {
  if ((ev & SUB_PAIR) && (c.col_nv > 0.0f || c.col_nw > 0.0f)) {
    float zw[4];
    normal4(c, q, t, STREAM_PAIR, 1, zw);
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = fmaf(c.col_nw, zw[k], w[k]);
  }
  if ((ev & SUB_DOWNWASH) && (c.dw_na > 0.0f || c.dw_nw > 0.0f)) {
    float zw[4];
    normal4(c, q, t, STREAM_DOWNWASH, 1, zw);
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = fmaf(c.dt, c.dw_nw * zw[k], w[k]);
  }
}

// The rest of a substep from its thrust and torques (not the rotor state):
// translation and rotation.  REC: also record the intermediates the adjoint
// needs into *r (the rotor fields are the caller's).
template <bool REC = false>
__device__ __forceinline__ void body_step(const Consts& c, const QuadPar& p, Quad& s,
                                          const Drive& d, uint32_t q, uint64_t t,
                                          Rec* r = nullptr) {
  if constexpr (REC) {
    r->T = d.T;
#pragma unroll
    for (int k = 0; k < 3; ++k) r->v0[k] = s.v[k];
  }
  const float F[3] = {d.T * s.R[2], d.T * s.R[5], d.T * s.R[8]};
  float v0[2], fl0, R0[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) R0[k] = s.R[k];
  uint32_t ev = 0u;
  const bool rest = trans_free(c, p, s, F, v0, fl0);
  rot_step<REC>(c, p, s.R, s.w, d.tx, d.ty, d.tz, r);
  if (rest) {
    ev = trans_rest(c, p, s, F, v0, fl0);
    rot_rest(s.R, s.w, R0);
  }
  ev |= trans_room<REC>(
      c, s, q, t, [&] { rot_bounced(c, s.w, q, t); }, [&] { rot_hit(s.R, s.w); });
  if constexpr (REC) r->ev = ev;
}

// One substep of one quad up to (not including) the in-env pair pass: the
// motor part, then the body part.  REC: also record the intermediates the
// adjoint needs into *r.
template <bool REC = false, ZMode ZM = Z_DRAW>
__device__ __forceinline__ void quad_substep(const Consts& c, const QuadPar& p, Quad& s,
                                             const float uhat[4], uint32_t q, uint64_t t,
                                             Rec* r = nullptr, float* zio = nullptr) {
  if constexpr (REC) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r->u0[i] = s.u[i];
  }
  float z[4] = {0.f, 0.f, 0.f, 0.f};
  const Drive d = motor_step<ZM>(c, p, s.u, s.e, uhat, q, t, z, zio);
  if constexpr (REC) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      r->z[i] = z[i];
      r->u1[i] = s.u[i];
    }
  }
  body_step<REC>(c, p, s, d, q, t, r);
}

// Geometry of the pair (i, j) for the in-env pass, from partner j's start
// position pj[0..2] and displacement pj[3..5] (rows 0-5 of the tile; rows
// 6-8 hold the velocities).  Returns true when the pair is in contact; then
// pair_normal gives the unit normal from j to i and sp = (v_j - v_i).n.
// Shared by the forward pass and the adjoint's recomputation so both take
// identical decisions.
// Separation from partner pj after the substep's motion and the contact
// test d^2 < d_col^2.  For the quad itself d = 0 exactly and the test is
// true: callers clear their own bit once after the partner loop instead of
// testing every partner's index.
__device__ __forceinline__ bool pair_geom_v(const Consts& c, const float pj[6], const Quad& s,
                                            float& dx, float& dy, float& dz, float& d2) {
  dx = (s.xo[0] - pj[0]) + (s.inc[0] - pj[3]);
  dy = (s.xo[1] - pj[1]) + (s.inc[1] - pj[4]);
  dz = (s.xo[2] - pj[2]) + (s.inc[2] - pj[5]);
  d2 = dx * dx + dy * dy + dz * dz;
  return d2 < c.dcol2;
}

template <int BS>
__device__ __forceinline__ void pair_normal(const float (*tile)[BS], const Quad& s, int j, int jj,
                                            int me, float dx, float dy, float dz, float d2,
                                            float n[3], float& sp) {
  if (d2 < 1e-12f) {
    n[0] = 0.f;
    n[1] = 0.f;
    n[2] = me < jj ? 1.f : -1.f;
  } else {
    const float id = rsqrtf(d2);
    n[0] = dx * id;
    n[1] = dy * id;
    n[2] = dz * id;
  }
  sp = (tile[6][j] - s.v[0]) * n[0] + (tile[7][j] - s.v[1]) * n[1] + (tile[8][j] - s.v[2]) * n[2];
}

// Smoothed collision penalty: softplus(x) = max(x, 0) + ln(1 + e^-|x|) and
// its derivative, the logistic sigmoid, from the hardware base-2 exponential,
// logarithm and reciprocal (about 1 ulp each); ln(1 + e) for e < 1e-4 from
// its series, where 1 + e would round away most of e.
__device__ __forceinline__ float softplus_hw(float x) {
  const float e = __builtin_amdgcn_exp2f(-fabsf(x) * 1.4426950408889634f);
  const float l = e < 1e-4f ? e * fmaf(-0.5f, e, 1.0f)
                            : 0.6931471805599453f * __builtin_amdgcn_logf(1.0f + e);
  return fmaxf(x, 0.f) + l;
}
__device__ __forceinline__ float sigmoid_hw(float x) {
  return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-x * 1.4426950408889634f));
}

// Workgroup barrier with the LDS fences around it, for kernels whose
// wavefronts run different code (each reaching it the same number of times).
__device__ __forceinline__ void wg_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// LDS written by some lanes of a wavefront, then read by others of the same
// wavefront.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A lane's values and their half-mirrored copies, from which the values of lane
// (lane xor D), 1 <= D <= 7, come by one data-parallel-primitive move each,
// with no LDS: quad_perm covers D = 1, 2, 3 within groups of 4 lanes;
// row_half_mirror (lane i of each group of 8 from lane 7 - i, i.e. xor 7)
// composed with one of them covers D = 4 .. 7.  Every source lane lies inside
// the destination's own group of 8, so the moves leave their unmasked form and
// fold into the subtraction that takes them.  Callers run them with every lane
// of the wavefront active (uniform control flow).
struct LaneXyz {
  float v[3], h[3];
};
template <int CTRL>
__device__ __forceinline__ float lane_move(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <int N>
__device__ __forceinline__ LaneXyz lane_xyz(float x, float y, float z) {
  constexpr int HALF_MIRROR = 0x141;
  LaneXyz p{{x, y, z}, {0.f, 0.f, 0.f}};
  if constexpr (N > 4) {
#pragma unroll
    for (int k = 0; k < 3; ++k) p.h[k] = lane_move<HALF_MIRROR>(p.v[k]);
  }
  return p;
}
template <int D>
__device__ __forceinline__ float lane_xor8(const LaneXyz& p, int k) {
  static_assert(D >= 1 && D <= 7, "partners within a group of 8 lanes");
  constexpr int QP[4] = {0xE4, 0xB1, 0x4E, 0x1B};  // quad_perm: identity, xor 1, xor 2, xor 3
  constexpr int r = D >= 4 ? (D ^ 7) : D;
  const float v = D >= 4 ? p.h[k] : p.v[k];
  if constexpr (r == 0) return v;
  else return lane_move<QP[r]>(v);
}

// compile-time booleans for generic lambdas
struct TrueT { static constexpr bool value = true; };
struct FalseT { static constexpr bool value = false; };

// Swarm size template argument of the bucketed launch's loops over a slot's
// run-time size (0: run-time sizes elsewhere).  Its body shares the kernel with
// those of the other slots, and keeps the plain screen, which needs the fewest
// registers: the expanded one put all of them past 168 (172,943 quads of 1 to
// 32, ten substeps, ten calls: 476 -> 494 us).
constexpr int SLOT_LOOP = -1;

// Contact mask of a swarm slot of N quads: 32 bits suffice up to 32 (one
// select and one OR per partner instead of two of each).
template <int N>
using PairMask = typename std::conditional<(N > 0 && N <= 32), uint32_t,
                                           unsigned long long>::type;

// Calls f(jj, pj) for every swarm-mate jj of the lane's swarm (itself
// included), in increasing jj, pj[0..5] being its start position and
// displacement from rows 0-5 of the tile and pj[6] row XR (XR < 0: none).
// N <= 0: up to three calls for the quad itself (jj == me) follow, so a pass
// must leave the quad itself out, or take nothing from it, however often it comes.
// For a compile-time swarm size the reads go out a chunk of eight partners
// at a time, ahead of the per-pair branches, so they overlap instead of
// waiting one by one.
// FEW: chunks of four in swarms of 8 too (the recompute with its penalty's
// adjoint, which is short of registers).  TAIL (N <= 0): a last chunk of less
// than four places where the wavefront's swarms all end there.
template <int BS, int N, int XR = -1, bool FEW = false, bool TAIL = false, typename T, typename F>
__device__ __forceinline__ void for_partners(T tile, int ls, int n, int me, F&& f) {
  if constexpr (N > 0) {
    // chunks of eight partners, four in swarms of 16 and more (32-quad
    // swarms: 168 -> 120 VGPRs in the step, four wavefronts per SIMD
    // instead of three)
    constexpr int CH = N < 8 ? N : (N >= 16 || FEW ? 4 : 8);
    auto chunk = [&](int j0) {
      float pj[CH][7];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
#pragma unroll
        for (int r = 0; r < 6; ++r) pj[u][r] = tile[r][ls + j0 + u];
        pj[u][6] = XR >= 0 ? tile[XR < 0 ? 0 : XR][ls + j0 + u] : 0.f;
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) f(j0 + u, pj[u]);
    };
    if constexpr (N >= 16 || (N == 8 && FEW)) {
      // large swarms: a run-time loop over the chunks keeps the registers
      // of an eight-partner body
#pragma unroll 1
      for (int j0 = 0; j0 < N; j0 += CH) chunk(j0);
    } else {
#pragma unroll
      for (int j0 = 0; j0 < N; j0 += CH) chunk(j0);
    }
  } else {
    // run-time sizes: chunks of four as well, branch-free; the places past the
    // swarm's end hold the quad itself, which no pass counts.
    // One partner at a time, every read was waited for alone:
    // 2048 swarms of 1-16, differentiated over 100 substeps, 1047 -> 917 us;
    // 4096 x 12 stepped twice and observed 15.0 -> 14.5 us.
    // TAIL, a vote for each chunk: where all of the wavefront's swarms end within
    // one, two or three more places, the last chunk holds no more than those
    // (131072 quads, 50 substeps with the penalty: swarms of 3 162 -> 157 us, of 5
    // 202 -> 178, of 6 202 -> 186, of 4, where the choice is all there is,
    // 135 -> 139).  Passes without the penalty do with less between the chunks, and
    // longer swarms lose more by the vote than short ones gain (24576 quads, 40
    // substeps with downwash: swarms of 1-64 262 us, with the vote 302, of 5 72 and 66).
    for (int j0 = 0; j0 < n; j0 += 4) {
      auto chunk = [&](auto size) {
        constexpr int CH = decltype(size)::value;
        int jj[CH];
        float pj[CH][7];
#pragma unroll
        for (int u = 0; u < CH; ++u) {
          jj[u] = j0 + u < n ? j0 + u : me;
          const int j = ls + jj[u];
#pragma unroll
          for (int r = 0; r < 6; ++r) pj[u][r] = tile[r][j];
          pj[u][6] = XR >= 0 ? tile[XR < 0 ? 0 : XR][j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < CH; ++u) f(jj[u], pj[u]);
      };
      const int left = n - j0;
      if (!TAIL || __ballot(left > 3) != 0ull) chunk(std::integral_constant<int, 4>{});
      else if (__ballot(left > 2) != 0ull) chunk(std::integral_constant<int, 3>{});
      else if (__ballot(left > 1) != 0ull) chunk(std::integral_constant<int, 2>{});
      else chunk(std::integral_constant<int, 1>{});
    }
  }
}

// Rows of the exchange tile that hold each quad's post-motion position
// (x after walls and floor) and its squared norm, written beside rows 0-8 by
// kernels whose in-swarm pass screens partners on it (pair_pass with CO).
constexpr int XROW = 9;
constexpr int XSQ = XROW + 3;
constexpr int TILE_ROWS_CO = XROW + 4;
// Positions (every coordinate, metres) within which the screen of swarms of
// 16 and 32 uses the expanded squared distance; the room of the workloads
// spans [-5, 5] x [-5, 5] x [0, 10].
constexpr float SCREEN_BOX = 10.0f;

// Swarm slots whose screen reads the squared norms.
template <int N>
constexpr bool kScreenSq = N == 0 || (N >= 16 && N <= 32);

// The screen rows of one lane: x and, for kScreenSq, |x|^2 (one expression, so
// every kernel writes the same value), or, for a padding lane, a far-away
// sentinel.  Sizes known at compile time read aligned runs of partners from a
// row (16 bytes of one coordinate of four); run-time sizes have no alignment,
// so there the four rows hold a float4 per quad, one partner a read.
template <int N, typename T>
__device__ __forceinline__ void put_screen(T tile, int tid, float x, float y, float z, float sq) {
  if constexpr (N == 0) {
    reinterpret_cast<float4*>(&tile[XROW][0])[tid] = make_float4(x, y, z, sq);
  } else {
    tile[XROW][tid] = x;
    tile[XROW + 1][tid] = y;
    tile[XROW + 2][tid] = z;
    if constexpr (kScreenSq<N>) tile[XSQ][tid] = sq;
  }
}
template <int N, typename T>
__device__ __forceinline__ void put_screen_rows(T tile, int tid, const float x[3]) {
  put_screen<N>(tile, tid, x[0], x[1], x[2], fmaf(x[2], x[2], fmaf(x[1], x[1], x[0] * x[0])));
}
template <int N, typename T>
__device__ __forceinline__ void put_screen_pad(T tile, int tid) {
  put_screen<N>(tile, tid, 1e30f, 1e30f, 1e30f, INFINITY);
}

// Calls f(jj, pj) for every swarm-mate jj (itself included), in increasing
// jj, with pj[0..2] its post-motion position from rows XROW..XROW+2 (and,
// NR = 4, pj[3] its squared norm from row XSQ), read a chunk of partners
// ahead of their arithmetic (chunk sizes as for_partners).
template <int BS, int N, int NR = 3, typename T, typename F>
__device__ __forceinline__ void for_partner_pos(T tile, int ls, int n, F&& f) {
  if constexpr (N > 0) {
    constexpr int CH = N < 8 ? N : (N >= 16 ? 4 : 8);
    auto chunk = [&](int j0) {
      float pj[CH][NR];
#pragma unroll
      for (int u = 0; u < CH; ++u) {
#pragma unroll
        for (int r = 0; r < NR; ++r) pj[u][r] = tile[XROW + r][ls + j0 + u];
      }
#pragma unroll
      for (int u = 0; u < CH; ++u) f(j0 + u, pj[u]);
    };
    if constexpr (N >= 16) {
#pragma unroll 1
      for (int j0 = 0; j0 < N; j0 += CH) chunk(j0);
    } else {
#pragma unroll
      for (int j0 = 0; j0 < N; j0 += CH) chunk(j0);
    }
  } else {
    static_assert(N == SLOT_LOOP, "run-time sizes (N = 0): screen_expanded");
    for (int j0 = 0; j0 < n; j0 += 4) {
      float pj[4][NR];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = ls + min(j0 + u, n - 1);
#pragma unroll
        for (int r = 0; r < NR; ++r) pj[u][r] = tile[XROW + r][j];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        pj[u][0] = j0 + u < n ? pj[u][0] : INFINITY;  // at infinite squared distance
        f(j0 + u, pj[u]);
      }
    }
  }
}

// Neighbour keys (§III-C, the K nearest by (d^2, index)).  A candidate at
// squared distance d2 becomes one 32-bit key: the bits of d2 (non-negative,
// so they order as the values) with the low six replaced by the partner's
// index jj within the swarm (swarms hold at most 64).  key[0..L-1] is a
// sorted list of the L smallest keys so far; a candidate enters with one min
// and L - 1 medians, all independent of each other:
// new[0] = min(old[0], x), new[k] = med3(old[k-1], x, old[k]).  The quad
// itself and non-finite distances never enter.  The list does not depend on
// the order in which candidates arrive.
constexpr uint32_t KEY_EMPTY = 0xffffffffu;
template <int L>
__device__ __forceinline__ void knn_insert(uint32_t key[L], int jj, int me, float d2) {
  const uint32_t kx = (jj != me && d2 < INFINITY)
                          ? ((__float_as_uint(d2) & ~63u) | (uint32_t)jj) : KEY_EMPTY;
  uint32_t nk[L];
  nk[0] = min(key[0], kx);
#pragma unroll
  for (int k = 1; k < L; ++k) nk[k] = umed3(key[k - 1], kx, key[k]);
#pragma unroll
  for (int k = 0; k < L; ++k) key[k] = nk[k];
}

// Squared distance from the lane's position to partner position pj[0..2]
// (one expression for the partner screen and the neighbour search, so both
// round identically).
__device__ __forceinline__ float sq_dist(const float pj[3], const float x[3]) {
  const float dx = pj[0] - x[0], dy = pj[1] - x[1], dz = pj[2] - x[2];
  return dx * dx + dy * dy + dz * dz;
}

// Expanded screen of swarms of 16 and 32 and of run-time sizes (there 49152 quads
// in swarms of 12, two substeps: 12.9 -> 12.1 us; the rollout of 2048 swarms of 1
// to 16, forward and backward over 100 substeps: 485 -> 442): mask of the partners whose
// post-motion positions lie within r of the lane's, and perhaps a few more.
// The bit is the sign of
//   e = |b|^2 + (|a|^2 - thr_x) - 2 a.b  (= |a - b|^2 - thr_x),
// three FMAs and an add per partner (|b|^2 from row XSQ, the rest once per
// lane), shifted in by one funnel shift ((acc << 1) | (e >> 31), v_alignbit):
// partner jj's bit lands at position N - 1 - jj and the mask is bit-reversed
// once.  Rounding: |e - (|a - b|^2 - thr_x)| <= 7 u ((|a| + |b|)^2 + thr_x),
// u = 2^-24.  For a lane with every |a_k| <= SCREEN_BOX and a partner within r,
// |a| + |b| <= reach = 2 sqrt(3) SCREEN_BOX + r + 1 mm, so the widening
// thr_x - r^2 = 3 err, err = 7 u (reach^2 + r^2) (+1 %), exceeds the
// rounding three times over and no such partner is dropped; a lane outside
// the box takes every partner.
template <int BS, int N>
__device__ __forceinline__ PairMask<N> screen_expanded(const float (*tile)[BS], const float x[3],
                                                       int ls, int n, float r, float r2) {
  const float reach = 2.0f * 1.7320508f * SCREEN_BOX + r + 1e-3f;
  const float err = 1.01f * 7.0f * 5.9604645e-8f * (reach * reach + r2);
  const float thr_x = r2 + 3.0f * err;
  const float na = fmaf(x[2], x[2], fmaf(x[1], x[1], fmaf(x[0], x[0], -thr_x)));
  const float a0 = -2.0f * x[0], a1 = -2.0f * x[1], a2 = -2.0f * x[2];
  auto sign_in = [&](uint32_t acc, float px, float py, float pz, float psq) {
    const float e = fmaf(a2, pz, fmaf(a1, py, fmaf(a0, px, psq + na)));
    return (uint32_t)__builtin_amdgcn_alignbit(acc, __float_as_uint(e), 31u);
  };
  if constexpr (N > 0) {
    uint32_t acc = 0u;
    for_partner_pos<BS, N, 4>(tile, ls, n, [&](int, const float* pj) {
      acc = sign_in(acc, pj[0], pj[1], pj[2], pj[3]);
    });
    return (PairMask<N>)(__builtin_bitreverse32(acc) >> (32 - N));
  } else {
    // run-time sizes: whole chunks of four (a place past the end repeats the
    // last member and is masked off), at most 32 places to a word
    const float4* at = reinterpret_cast<const float4*>(&tile[XROW][0]) + ls;
    auto word = [&](int j0, int j1) {
      uint32_t acc = 0u;
      for (int j = j0; j < j1; j += 4) {
        float4 p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u] = at[min(j + u, n - 1)];
#pragma unroll
        for (int u = 0; u < 4; ++u) acc = sign_in(acc, p[u].x, p[u].y, p[u].z, p[u].w);
      }
      const int places = (j1 - j0 + 3) & ~3;
      return __builtin_bitreverse32(acc) >> (32 - places);
    };
    unsigned long long m = word(0, min(n, 32));
    if (n > 32) m |= (unsigned long long)word(32, n) << 32;
    return m & (~0ull >> (64 - n));
  }
}
__device__ __forceinline__ float max_abs(const float x[3]) {
  return fmaxf(fabsf(x[0]), fmaxf(fabsf(x[1]), fabsf(x[2])));
}

// What a pass over the partners of a substep sums up beside the contacts:
//  PEN_SUM: the smoothed collision penalty, softplus(beta (d_col - d)) / (2 beta)
//           per partner (each quad of a pair carries half), into acc[0];
//  PEN_GRAD: its adjoint w.r.t. the quad's position,
//             d pen / d x_i = -(g_i + g_j)/2 sigmoid(beta (d_col - d)) (x_i - x_j) / d,
//           into acc[0..2].  h_me = -g_i/2, and row PENROW of the tile holds
//           -g_j/2 for the partners (halving is exact, so h_me + h_j rounds
//           as -(g_i + g_j)/2).
// Either way the sum runs in partner order.
enum PenMode { PEN_NONE = 0, PEN_SUM = 1, PEN_GRAD = 2 };
constexpr int PENROW = TILE_ROWS_CO;
struct Pen {
  float beta, hb;
  // Beyond the contact distance + 106 / beta, softplus (2^-152 before its
  // rounding) and sigmoid (1 / infinity) are exactly 0 in float32, so passes
  // over the partners within r give the same sums bit for bit.
  float r;
  int few;      // passes over the near partners pay up to this many of them; 0: never
  float h_me;
  float acc[3];
};

// n_max: the wavefront's largest swarm.  Over all partners a pass costs about
// 27 vector instructions a partner; over the near ones 10 a partner for the
// screen and 38 a near one (their reads are gathered and their index found),
// so it pays up to 0.45 n_max of them, and not at all in swarms of up to 8.
// 32768 x 32, 100 substeps with beta = 100: forward 3.27 -> 2.43 ms.
// A radius of several metres leaves nothing out; with a weight that is not
// finite every partner counts (its product with 0 is not 0).
__device__ __forceinline__ Pen make_pen(const Consts& c, float beta, int n_max, float h_me = 0.f) {
  Pen p;
  p.beta = beta;
  p.hb = 0.5f / beta;
  p.r = c.dcol + 106.0f / beta;
  p.h_me = h_me;
  p.acc[0] = p.acc[1] = p.acc[2] = 0.f;
  const bool odd = __ballot(!(fabsf(h_me) < INFINITY)) != 0ull;
  p.few = (n_max <= 8 || odd || !(p.r < 3.0f)) ? 0 : (n_max * 29) >> 6;
  return p;
}

// The largest value of the wavefront.
__device__ __forceinline__ int wave_max(int v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v = max(v, __shfl_xor(v, d, 64));
  return v;
}

template <int P>
__device__ __forceinline__ void pen_term(const Consts& c, Pen& p, bool other, float hj, float dx,
                                         float dy, float dz, float d2) {
  if constexpr (P == PEN_SUM) {
    const float sp = p.hb * softplus_hw(p.beta * (c.dcol - __builtin_amdgcn_sqrtf(d2)));
    p.acc[0] = other ? p.acc[0] + sp : p.acc[0];
  } else if constexpr (P == PEN_GRAD) {
    // the quad itself has d^2 = 0 exactly, so d^2 > 0 also leaves it out
    const float rd = __builtin_amdgcn_rsqf(d2);
    const float coef = d2 > 0.f && other
                           ? (p.h_me + hj) * sigmoid_hw(p.beta * (c.dcol - d2 * rd)) * rd
                           : 0.f;
    p.acc[0] = fmaf(coef, dx, p.acc[0]);
    p.acc[1] = fmaf(coef, dy, p.acc[1]);
    p.acc[2] = fmaf(coef, dz, p.acc[2]);
  }
}

// Contact bits (by the exact test) and penalty terms of the partners within
// p.r of the lane, two at a time so that the second one's gathered reads run
// under the first one's arithmetic.  Returns false, and has done nothing, where
// the wavefront does better over all partners.  Needs rows XROW.. of the tile.
template <int BS, int N, int P>
__device__ __forceinline__ bool near_pass(const Consts& c, const float (*tile)[BS], const Quad& s,
                                          int ls, int n, int me, Pen& p, PairMask<N>& cm) {
  using M = PairMask<N>;
  // The votes below see one wavefront.  In a table's workgroup of two, a swarm may
  // lie in both: a mate in the other one whose position or weight is not a
  // number, and so counts for everybody, would be left out.
  if constexpr (BS > 64 && N <= 0) return false;
  if (p.few == 0) return false;
  const float far = max_abs(s.x);
  const float lim = kScreenSq<N> ? SCREEN_BOX : 1000.0f;
  // (NaN included: max_abs skips it, the sum does not)
  if (__ballot(!(far <= lim && s.x[0] + s.x[1] + s.x[2] < INFINITY)) != 0ull) return false;
  M near;
  if constexpr (kScreenSq<N>) {
    near = screen_expanded<BS, N>(tile, s.x, ls, n, p.r, p.r * p.r);
  } else {
    const float w = p.r + 1e-3f, thr = w * w;
    near = 0;
    for_partner_pos<BS, N>(tile, ls, n, [&](int jj, const float* pj) {
      near |= sq_dist(pj, s.x) < thr ? (M)1 << jj : (M)0;
    });
  }
  near &= ~((M)1 << me);
  if (__ballot(__popcll((unsigned long long)near) > p.few) != 0ull) return false;
  while (near != 0) {
    int jj[2];
    jj[0] = __builtin_ctzll((unsigned long long)near);
    near &= near - 1;
    const bool two = near != 0;
    jj[1] = two ? __builtin_ctzll((unsigned long long)near) : jj[0];
    near &= near - 1;
    float pj[2][7];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int r = 0; r < 6; ++r) pj[u][r] = tile[r][ls + jj[u]];
      pj[u][6] = P == PEN_GRAD ? tile[P == PEN_GRAD ? PENROW : 0][ls + jj[u]] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      float dx, dy, dz, d2;
      const bool con = pair_geom_v(c, pj[u], s, dx, dy, dz, d2);
      cm |= con ? (M)1 << jj[u] : (M)0;
      pen_term<P>(c, p, u == 0 || two, pj[u][6], dx, dy, dz, d2);
    }
  }
  return true;
}

// Adds partner jj's collision response to the velocity change dv and its bit
// to rm, where the pair in contact responds (see pair_geom_v).
template <int BS>
__device__ __forceinline__ void pair_response(const Consts& c, const float (*tile)[BS],
                                              const Quad& s, int j, int jj, int me, float dx,
                                              float dy, float dz, float d2, float dv[3],
                                              unsigned long long& rm) {
  float nn[3], sp;
  pair_normal<BS>(tile, s, j, jj, me, dx, dy, dz, d2, nn, sp);
  if (!(c.flags & F_APPROACH) || sp > 0.f) {
#pragma unroll
    for (int k = 0; k < 3; ++k) dv[k] = fmaf(sp, nn[k], dv[k]);
    rm |= 1ull << jj;
  }
}

// The end of the in-swarm pass: the velocity change dv of the partners rm and
// the downwash kick; resp and events as in pair_pass.
__device__ __forceinline__ void pair_apply(const Consts& c, Quad& s, uint32_t q,
                                           unsigned long long t, unsigned long long rm,
                                           const float dv[3], float adw, bool dwhit,
                                           unsigned long long* resp, uint32_t* events) {
  if (resp) *resp = rm;
  uint32_t ev = 0u;
  if (rm != 0ull) {
    s.ev |= EVF_QUAD;
    ev |= SUB_PAIR;
    float zv[4] = {0.f, 0.f, 0.f, 0.f};
    if (c.col_nv > 0.0f || c.col_nw > 0.0f) normal4(c, q, t, STREAM_PAIR, 0, zv);
#pragma unroll
    for (int k = 0; k < 3; ++k) s.v[k] = c.col_decay * (s.v[k] + dv[k] + c.col_nv * zv[k]);
  }
  if (dwhit) {
    ev |= SUB_DOWNWASH;
    float za[4] = {0.f, 0.f, 0.f, 0.f};
    if (c.dw_na > 0.0f || c.dw_nw > 0.0f) normal4(c, q, t, STREAM_DOWNWASH, 0, za);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const float a = (k == 2 ? adw : 0.f) + c.dw_na * za[k];
      s.v[k] = fmaf(c.dt, a, s.v[k]);
    }
  }
  if (events) *events = ev;
  else if (ev != 0u) rot_pair_events(c, ev, s.w, q, t);
}

// In-swarm pass of one live lane after the tile (start positions,
// displacements, velocities) is written and the workgroup synchronised:
// §III-B.1 contact detection and Jacobi velocity exchange (every response
// from the pre-response velocities), the smoothed collision penalty (PEN),
// and §III-B.4 downwash from the swarm-mates above, applied as a velocity
// kick after the response.  N > 0 unrolls over the swarm slot; padding
// partners hold far-away sentinels.  Returns the contact mask.
// P (PenMode): also sum the penalty or its adjoint into *pen; with CO over
// the near partners where that pays (near_pass).  resp (optional): the
// partners whose response the quad received.  events (optional): receives the
// pass's events, and the body rates are the caller's (rot_pair_events).
// CO (tile rows XROW.. written): without penalty and downwash, partners are
// first screened on the post-motion positions with a contact distance
// widened by 1 mm, and the exact test runs for the survivors only.  The
// screen never drops a pair the exact test would mark: for positions within
// 1000 m of the origin, x differs from (start + displacement) by at most an
// ulp of 1000 (6.1e-5 m) per quad and axis, well inside the 1 mm; a lane
// further out tests every partner exactly.  So the contact set, and every
// result, is the same as without the screen.  L > 0 (swarms other than 8,
// with the screen): the screen's squared distances also enter the
// neighbour key list key[0..L-1] (knn_insert); the pass changes only
// velocities and body rates, so they are the distances of the post-pass
// positions.
template <int BS, int N, int P, bool CO = false, int L = 0>
__device__ __forceinline__ unsigned long long pair_pass(const Consts& c, const float (*tile)[BS],
                                                        Quad& s, int ls, int n, int me,
                                                        uint32_t q, unsigned long long t,
                                                        Pen* pen = nullptr,
                                                        uint32_t* key = nullptr,
                                                        unsigned long long* resp = nullptr,
                                                        uint32_t* events = nullptr) {
  static_assert(L == 0 || (CO && P == PEN_NONE), "keys from the plain screen only");
  static_assert(!CO || P != PEN_NONE || N <= 1 || N > 8, "lane_pair_pass for swarms of up to 8");
  const bool collide = (c.flags & F_COLLIDE) != 0;
  const bool dw = (c.flags & F_DOWNWASH) != 0 && s.fl == 0.0f;
  using M = PairMask<N>;
  M cm = 0;
  float adw = 0.f;
  bool dwhit = false;
  // Every partner's geometry, branch-free (contacts are rare; a branch per
  // partner would end the scheduling region and serialise the partners'
  // arithmetic): the contact set, the penalty and, when it is on (a uniform
  // choice between two loops), downwash.
  const float dw_r2 = c.dw_r2, dw_h = c.dw_h, dw_k1 = c.dw_k1, dw_k2 = c.dw_k2, dw_b1 = c.dw_b1;
  // In passes over every partner in index order (in_order), swarms of 16
  // and 32 shift the contact bits in (the sign bit of d^2 - d_col^2, for
  // numbers exactly the comparison's outcome, by one funnel shift) and
  // bit-reverse them once after the pass.
  constexpr bool ACC = N >= 16 && N <= 32;
  uint32_t acc = 0u;
  auto pair = [&](int jj, const float* pj, auto with_dw, auto in_order) {
    float dx, dy, dz, d2;
    const bool con = pair_geom_v(c, pj, s, dx, dy, dz, d2);
    if constexpr (P != PEN_NONE)
      pen_term<P>(c, *pen, P == PEN_GRAD || jj != me, pj[6], dx, dy, dz, d2);
    if constexpr (ACC && decltype(in_order)::value)
      acc = __builtin_amdgcn_alignbit(acc, __float_as_uint(d2 - c.dcol2), 31u);
    else
      cm |= con ? (M)1 << jj : (M)0;
    if constexpr (decltype(with_dw)::value) {
      // swarm-mate j above (z_j - z_i = -dz) and overlapping in xy (never
      // the quad itself: dz = 0 there)
      const bool dwc = dw & (dx * dx + dy * dy < dw_r2) & (-dz > 0.f) & (-dz < dw_h);
      adw = dwc ? adw - dw_k1 * (dw_k2 * -dz + dw_b1) : adw;
      dwhit = dwhit | dwc;
    }
  };
  constexpr int XR = P == PEN_GRAD ? PENROW : -1;
  if (c.flags & F_DOWNWASH) {
    for_partners<BS, N, XR, false, P != PEN_NONE>(
        tile, ls, n, me, [&](int jj, const float* pj) { pair(jj, pj, TrueT{}, TrueT{}); });
    if constexpr (ACC) cm = (M)(__builtin_bitreverse32(acc) >> (32 - N));
  } else if constexpr (CO && P == PEN_NONE) {
    const float dw = c.dcol + 1e-3f, thr = dw * dw;
    M cand = 0;
    bool in_box = true;  // the expanded screen's domain
    if constexpr (L == 0 && kScreenSq<N>) {
      cand = screen_expanded<BS, N>(tile, s.x, ls, n, c.dcol, c.dcol2);
      in_box = max_abs(s.x) <= SCREEN_BOX;
    } else if constexpr (N >= 16 && N <= 32) {
      // partners arrive in index order, so the mask is accumulated as
      // acc = 2 acc + bit and bit-reversed once
      uint32_t acc = 0u;
      for_partner_pos<BS, N>(tile, ls, n, [&](int jj, const float* pj) {
        const float d2 = sq_dist(pj, s.x);
        acc = acc + acc + (d2 < thr ? 1u : 0u);
        knn_insert<L>(key, jj, me, d2);
      });
      cand = (M)(__builtin_bitreverse32(acc) >> (32 - N));
    } else {
      for_partner_pos<BS, N>(tile, ls, n, [&](int jj, const float* pj) {
        const float d2 = sq_dist(pj, s.x);
        cand |= d2 < thr ? (M)1 << jj : (M)0;
        if constexpr (L > 0) knn_insert<L>(key, jj, me, d2);
      });
    }
    const bool near_origin = max_abs(s.x) <= 1000.0f;
    if (!(near_origin && in_box)) cand = (M)(n >= 64 ? ~0ull : (1ull << n) - 1ull);
    // the quad itself (distance 0) leaves the contact mask below anyway
    cand &= ~((M)1 << me);
    for (unsigned long long m = cand; m != 0ull; m &= m - 1ull) {
      const int jj = __builtin_ctzll(m);
      const int j = ls + jj;
      const float pj[6] = {tile[0][j], tile[1][j], tile[2][j], tile[3][j], tile[4][j], tile[5][j]};
      pair(jj, pj, FalseT{}, FalseT{});
    }
  } else {
    bool done = false;
    if constexpr (CO && (N <= 0 || N > 8))
      done = near_pass<BS, N, P>(c, tile, s, ls, n, me, *pen, cm);
    if (!done) {
      for_partners<BS, N, XR, P == PEN_GRAD, P != PEN_NONE>(
          tile, ls, n, me, [&](int jj, const float* pj) { pair(jj, pj, FalseT{}, TrueT{}); });
      if constexpr (ACC) cm = (M)(__builtin_bitreverse32(acc) >> (32 - N));
    }
  }
  unsigned long long cmask = collide ? (unsigned long long)(cm & ~((M)1 << me)) : 0ull;
  // The responses, for the partners in contact only, in partner order.  (The
  // sign bits shifted in above are the comparison's outcome for numbers only: a
  // partner at a distance that is none is not in contact.)
  float dv[3] = {0.f, 0.f, 0.f};
  unsigned long long rm = 0ull;
  for (unsigned long long m = cmask; m != 0ull; m &= m - 1ull) {
    const int jj = __builtin_ctzll(m);
    const int j = ls + jj;
    const float pj[6] = {tile[0][j], tile[1][j], tile[2][j], tile[3][j], tile[4][j], tile[5][j]};
    float dx, dy, dz, d2;
    const bool con = pair_geom_v(c, pj, s, dx, dy, dz, d2);
    if constexpr (ACC) {
      if (!con) cmask &= ~(1ull << jj);
    }
    if (!ACC || con) pair_response<BS>(c, tile, s, j, jj, me, dx, dy, dz, d2, dv, rm);
  }
  pair_apply(c, s, q, t, rm, dv, adw, dwhit, resp, events);
  return cmask;
}

// The exchange tile's rows of one lane.  Padding lanes are at an infinite
// distance of every position, the largest finite ones included.
template <int N, bool SCREEN, typename T>
__device__ __forceinline__ void put_tile(T tile, int tid, const Quad& s) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    tile[k][tid] = s.xo[k];
    tile[3 + k][tid] = s.inc[k];
    tile[6 + k][tid] = s.v[k];
  }
  if constexpr (SCREEN) put_screen_rows<N>(tile, tid, s.x);
}
template <typename T>
__device__ __forceinline__ void put_tile_pad(T tile, int tid) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    tile[k][tid] = INFINITY;
    tile[3 + k][tid] = 0.f;
    tile[6 + k][tid] = 0.f;
  }
}

// The in-swarm pass in slots of 2, 4 and 8 quads (aligned groups of a
// wavefront's lanes), by every lane of the wavefront: partners are screened on
// their post-motion positions (with the contact distance widened by 1 mm,
// as in pair_pass) by cross-lane moves, with no LDS, and most substeps end
// there.  Only where a lane of the wavefront finds a partner do the lanes write
// the exchange tile (PUT; otherwise the caller has) for the exact test and the
// responses, as in pair_pass, whose results these are.  Downwash passes over
// every partner.  (Screened through the tile, and tested and answered in two
// passes: forward of 1024 x 8, 200 substeps, 206 -> 183 us.)
template <int BS, int N, bool PUT>
__device__ __forceinline__ unsigned long long lane_pair_pass(
    const Consts& c, float (*tile)[BS], Quad& s, bool live, int ls, int n, int me, int tid,
    uint32_t q, unsigned long long t, unsigned long long* resp = nullptr,
    uint32_t* events = nullptr) {
  static_assert(N == 2 || N == 4 || N == 8, "aligned groups of up to 8 lanes");
  auto put = [&] {
    if constexpr (PUT) {
      if (live) put_tile<N, false>(tile, tid, s);
      else put_tile_pad(tile, tid);
    }
    wave_sync();
  };
  if (c.flags & F_DOWNWASH) {
    put();
    return live ? pair_pass<BS, N, PEN_NONE>(c, tile, s, ls, n, me, q, t, nullptr, nullptr, resp,
                                             events)
                : 0ull;
  }
  const float dw = c.dcol + 1e-3f, thr = dw * dw;
  const float x = live ? s.x[0] : INFINITY, y = live ? s.x[1] : INFINITY, z = live ? s.x[2] : INFINITY;
  // the sign of d^2 - thr as one FMA chain, shifted in: bit N - 1 - d for the
  // partner me ^ d
  const LaneXyz xyz = lane_xyz<N>(x, y, z);
  uint32_t bits = 0u;
  auto screen = [&](auto dc) {
    constexpr int D = decltype(dc)::value;
    if constexpr (D < N) {
      const float dx = lane_xor8<D>(xyz, 0) - x, dy = lane_xor8<D>(xyz, 1) - y,
                  dz = lane_xor8<D>(xyz, 2) - z;
      const float e = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, -thr)));
      bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(e), 31u);
    }
  };
  screen(std::integral_constant<int, 1>{});
  screen(std::integral_constant<int, 2>{});
  screen(std::integral_constant<int, 3>{});
  screen(std::integral_constant<int, 4>{});
  screen(std::integral_constant<int, 5>{});
  screen(std::integral_constant<int, 6>{});
  screen(std::integral_constant<int, 7>{});
  const float far = fmaxf(fabsf(x), fmaxf(fabsf(y), fabsf(z)));
  if (!(far <= 1000.0f)) bits = (1u << (N - 1)) - 1u;  // every partner
  if (!live || !(c.flags & F_COLLIDE)) bits = 0u;
  if (__ballot(bits != 0u) == 0ull) {
    if (resp) *resp = 0ull;
    if (events) *events = 0u;
    return 0ull;
  }
  put();
  if (!live) return 0ull;
  // bits by d -> bits by partner, me ^ d: each bit of me swaps places
  uint32_t m = __builtin_bitreverse32(bits) >> (32 - N);
  if (me & 1) m = ((m & 0x55u) << 1) | ((m >> 1) & 0x55u);
  if (N > 2 && (me & 2)) m = ((m & 0x33u) << 2) | ((m >> 2) & 0x33u);
  if (N > 4 && (me & 4)) m = ((m & 0x0fu) << 4) | (m >> 4);
  m &= (1u << n) - 1u;
  // exact test and response in one pass: a contact lasts some tens of
  // substeps, and the workgroup that holds one sets the launch's time
  unsigned long long cmask = 0ull, rm = 0ull;
  float dv[3] = {0.f, 0.f, 0.f};
  for (; m != 0u; m &= m - 1u) {
    const int jj = __builtin_ctz(m), j = ls + jj;
    const float pj[6] = {tile[0][j], tile[1][j], tile[2][j], tile[3][j], tile[4][j], tile[5][j]};
    float dx, dy, dz, d2;
    if (pair_geom_v(c, pj, s, dx, dy, dz, d2)) {
      cmask |= 1ull << jj;
      pair_response<BS>(c, tile, s, j, jj, me, dx, dy, dz, d2, dv, rm);
    }
  }
  pair_apply(c, s, q, t, rm, dv, 0.f, false, resp, events);
  return cmask;
}

// The penalty (or its adjoint) of one live lane alone: the P terms of
// pair_pass (same partners, same order, same arithmetic), for a wavefront
// that sums them apart from the motion.  s: the quad's start position,
// displacement and post-motion position.
template <int BS, int N, int P>
__device__ __forceinline__ void penalty_pass(const Consts& c, const float (*tile)[BS],
                                             const Quad& s, int ls, int n, int me, Pen& pen) {
  if constexpr (N <= 0 || N > 8) {
    PairMask<N> contacts = 0;
    if (near_pass<BS, N, P>(c, tile, s, ls, n, me, pen, contacts)) return;
  }
  for_partners<BS, N, P == PEN_GRAD ? PENROW : -1, false, true>(
      tile, ls, n, me, [&](int jj, const float* pj) {
        float dx, dy, dz, d2;
        pair_geom_v(c, pj, s, dx, dy, dz, d2);
        pen_term<P>(c, pen, P == PEN_GRAD || jj != me, pj[6], dx, dy, dz, d2);
      });
}

// §III-C sensor noise on the own-state part of an observation row:
// U(-sn_x, sn_x) on x - goal, U(-sn_v, sn_v) on v, N(0, sn_w^2) on omega,
// from stream SENSOR at the observation's substep index.
__device__ __forceinline__ void sensor_noise(const Consts& c, uint32_t q, unsigned long long t,
                                             float o_x[3], float o_v[3], float o_w[3]) {
#pragma unroll
  for (int draw = 0; draw < 2; ++draw) {
    uint32_t r0 = q, r1 = (uint32_t)t, r2 = (uint32_t)(t >> 32), r3 = (STREAM_SENSOR << 8) | draw;
    philox4x32_10(r0, r1, r2, r3, c.key0, c.key1);
    const float a = draw == 0 ? c.sn_x : c.sn_v;
    float* o = draw == 0 ? o_x : o_v;
    o[0] = fmaf(a, 2.0f * u01(r0) - 1.0f, o[0]);
    o[1] = fmaf(a, 2.0f * u01(r1) - 1.0f, o[1]);
    o[2] = fmaf(a, 2.0f * u01(r2) - 1.0f, o[2]);
  }
  float z[4];
  normal4(c, q, t, STREAM_SENSOR, 2, z);
#pragma unroll
  for (int k = 0; k < 3; ++k) o_w[k] = fmaf(c.sn_w, z[k], o_w[k]);
}

// §III-E reward of a call from the post-call state, the goal offset dx, the
// rotor thrusts before the call (f0) and the call's events; the proximity
// term is added by the caller per neighbour slot (reward_prox).
__device__ __forceinline__ float reward_state(const Consts& c, const Quad& s, float f_max,
                                              const float dx[3], const float f0[4]) {
  float f2 = 0.f, df2 = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float f1 = fmaf(f_max * s.u[i], s.u[i], s.e[i]);
    f2 = fmaf(f1, f1, f2);
    df2 = fmaf(f1 - f0[i], f1 - f0[i], df2);
  }
  const float* w = c.rw;
  float r = w[0] * sqrtf(dx[0] * dx[0] + dx[1] * dx[1] + dx[2] * dx[2]);
  r += w[1] * sqrtf(s.v[0] * s.v[0] + s.v[1] * s.v[1] + s.v[2] * s.v[2]);
  r += w[2] * s.R[8];
  r += w[3] * sqrtf(s.w[0] * s.w[0] + s.w[1] * s.w[1] + s.w[2] * s.w[2]);
  r += w[4] * sqrtf(f2) + w[5] * sqrtf(df2);
  r += w[6] * (s.R[0] + s.R[4] + s.R[8] - 1.0f) * 0.5f + w[7] * s.R[0];
  r += (s.ev & EVF_FLOOR_HIT) ? w[8] : 0.f;
  r += s.fl != 0.f ? w[9] : 0.f;
  r += (s.ev & EVF_WALL) ? w[10] : 0.f;
  r += (s.ev & EVF_CEILING) ? w[11] : 0.f;
  r += (s.ev & EVF_QUAD) ? w[12] : 0.f;
  return r;
}

__device__ __forceinline__ float reward_prox(const Consts& c, float rx, float ry, float rz) {
  return c.rw[13] * fmaxf(1.0f - sqrtf(rx * rx + ry * ry + rz * rz) / c.rw[14], 0.f);
}

}  // namespace qs
