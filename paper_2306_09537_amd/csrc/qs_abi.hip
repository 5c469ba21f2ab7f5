// Host side of the C ABI declared in include/quadswarm.h: argument checks,
// the handle, the environment-to-workgroup partition and the launches.
#include <initializer_list>
#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

#include "quadswarm.h"
#include "qs_handle.h"
#include "qs_io.h"

namespace {

using qs_host::aligned;
using qs_host::check_desc;
using qs_host::finite;
using qs_host::outputs_overlap;
using qs_host::overlap;
using qs_host::Span;
using qs_host::noalloc_scratch;

// Workgroup size: one wavefront (64).  It needs no barrier for the in-swarm
// exchanges (32768 x 32: 128 -> 64 made the ten-substep step 4 %, the rollout
// 6 % and the backward 3 % faster), and a workgroup's quads are one tile of the
// state.  Single quads, 128 / 64, us a call of one, four and ten substeps: 262,144
// 12.7 / 12.3, 16.9 / 17.1, 26.7 / 27.0; 524,288 26.8 / 26.7, 30.8 / 29.6, 45.2 /
// 43.3; 1,048,576 51.8 / 52.0, 56.8 / 56.1, 74.2 / 72.4; the derivative of one
// substep 50.8 / 20.7, 92 / 38, 192 / 83.
int pick_block() {
  if (const char* e = std::getenv("QS_BLOCK_SIZE")) {
    const int b = std::atoi(e);
    if (b == 64 || b == 128) return b;
  }
  return 64;
}

template <typename T>
int dalloc(T** p, size_t count) {
  if (count == 0) count = 1;
  if (hipMalloc((void**)p, count * sizeof(T)) != hipSuccess) {
    *p = nullptr;
    return QS_ERR_NOMEM;
  }
  return QS_OK;
}

void free_all(qs_handle* h) {
  (void)hipFree(h->d_st);
  (void)hipFree(h->d_par);
  (void)hipFree(h->d_sw);
  (void)hipFree(h->d_blk);
  (void)hipFree(h->d_qenv);
  (void)hipFree(h->d_contacts);
  (void)hipFree(h->d_err);
  (void)hipFree(h->d_tape);
  (void)hipFree(h->d_ck1);
  (void)hipFree(h->d_gsum);
  (void)hipFree(h->d_items);
  (void)hipFree(h->d_item_envs);
  (void)hipFree(h->d_t);
  (void)hipFree(h->d_done);
  (void)hipFree(h->d_c);
  if (h->h_err) (void)hipHostFree(h->h_err);
}

// Greedy packing of whole environments into workgroups of at most bs quads:
// the workgroup table (first quad, count) and, per quad, its swarm's start
// within the workgroup and its size.  Sets bs and the workgroup count.
int build_table(qs_handle* h, int bs) {
  std::vector<int2> blk;
  std::vector<uint32_t> sw((size_t)h->Qp, 0u);
  int cur_begin = 0, cur_cnt = 0;
  for (size_t e = 0; e < h->env_n.size(); ++e) {
    const int q0 = h->env_start[e], n = h->env_n[e];
    if (cur_cnt + n > bs) {
      blk.push_back(make_int2(cur_begin, cur_cnt));
      cur_begin = q0;
      cur_cnt = 0;
    }
    for (int i = 0; i < n; ++i) sw[(size_t)q0 + i] = ((uint32_t)(q0 - cur_begin) << 8) | (uint32_t)n;
    cur_cnt += n;
  }
  blk.push_back(make_int2(cur_begin, cur_cnt));
  (void)hipFree(h->d_blk);
  (void)hipFree(h->d_sw);
  h->d_blk = nullptr;
  h->d_sw = nullptr;
  if (hipMalloc((void**)&h->d_blk, blk.size() * sizeof(int2)) != hipSuccess ||
      hipMalloc((void**)&h->d_sw, sw.size() * sizeof(uint32_t)) != hipSuccess)
    return QS_ERR_NOMEM;
  if (hipMemcpy(h->d_blk, blk.data(), blk.size() * sizeof(int2), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(h->d_sw, sw.data(), sw.size() * sizeof(uint32_t), hipMemcpyHostToDevice) != hipSuccess)
    return QS_ERR_HIP;
  h->bs = bs;
  h->nblk = (int)blk.size();
  return QS_OK;
}

// Work items of the bucketed launch: every swarm gets a slot of the next
// power of two >= its size; slots of one size are grouped bs/slot per item.  An
// item's w field selects the chunked partner body (slot sizes in
// h->chunked).
//
// Items are ordered by the quads they serve, in runs of RUN per XCD (workgroups
// go to the eight XCDs in turn): a cache line of the state's tiles holds eight
// quads, often of several swarms, whose items then share an L2 and run at about the
// same time.  Ordered by slot size (by_size: the autotuner's trials of one slot's
// items), every XCD fetches and writes back its own part of every line: 172,943
// quads of 1 to 32, ten calls of ten substeps, 472 us; by quads in runs of 32, 128
// and 512: 444, 435 and 431; 524,289 quads of 1 to 8, one substep: 99 -> 57.
// Shorter runs keep swarms sorted by size from giving one XCD all the heavy items.
// Items of 64 places come before the others: one of them takes as long as several
// of the rest (at the end of the launch it runs alone), and as a single swarm it
// shares no more than the lines at its two ends (swarms of 1, 2, 4 .. 64, ten
// substeps, by slot size / by quads / 64 first: 131k quads 83 / 76 / 67 us, 262k
// 113 / 118 / 98, 524k 183 / 182 / 167 and with K = 9 334 / 363 / 336).
int log2i(int n) {
  int k = 0;
  while ((1 << k) < n) ++k;
  return k;
}

// Slot sizes with a second, chunked body in the bucketed kernel.
constexpr uint32_t kChunkable = (1u << 4) | (1u << 5);

int build_items(qs_handle* h, int bs, bool by_size = false) {
  std::vector<int4> items;
  std::vector<int2> envs;
  for (int k = 0; k < 7; ++k) h->slot_swarms[k] = 0;
  for (size_t e = 0; e < h->env_n.size(); ++e) ++h->slot_swarms[log2i(h->env_n[e])];
  for (int N = 64; N >= 1; N >>= 1) {
    const int per = bs / N;
    const int w = (h->chunked & kChunkable) >> log2i(N) & 1u;
    int in_item = 0;
    for (size_t e = 0; e < h->env_n.size(); ++e) {
      const int n = h->env_n[e];
      if ((1 << log2i(n)) != N) continue;
      if (in_item == 0) items.push_back(make_int4(N, (int)envs.size(), 0, w));
      envs.push_back(make_int2(h->env_start[e], n));
      items.back().z += 1;
      if (++in_item == per) in_item = 0;
    }
  }
  if (!by_size) {
    constexpr size_t RUN = 128, XCDS = 8;
    std::stable_sort(items.begin(), items.end(), [&](const int4& a, const int4& b) {
      if ((a.x == 64) != (b.x == 64)) return a.x == 64;
      return envs[(size_t)a.y].x < envs[(size_t)b.y].x;
    });
    std::vector<int4> order;
    order.reserve(items.size());
    for (size_t g = 0; g < items.size(); g += XCDS * RUN) {
      const size_t m = std::min(XCDS * RUN, items.size() - g), run = (m + XCDS - 1) / XCDS;
      for (size_t i = 0; i < run; ++i)
        for (size_t j = i; j < m; j += run) order.push_back(items[g + j]);
    }
    items.swap(order);
  }
  (void)hipFree(h->d_items);
  (void)hipFree(h->d_item_envs);
  h->d_items = nullptr;
  h->d_item_envs = nullptr;
  if (hipMalloc((void**)&h->d_items, items.size() * sizeof(int4)) != hipSuccess ||
      hipMalloc((void**)&h->d_item_envs, envs.size() * sizeof(int2)) != hipSuccess)
    return QS_ERR_NOMEM;
  if (hipMemcpy(h->d_items, items.data(), items.size() * sizeof(int4), hipMemcpyHostToDevice) !=
          hipSuccess ||
      hipMemcpy(h->d_item_envs, envs.data(), envs.size() * sizeof(int2),
                hipMemcpyHostToDevice) != hipSuccess)
    return QS_ERR_HIP;
  h->n_items = (int)items.size();
  h->item_bs = bs;
  return QS_OK;
}

// Substeps a call from which a bucketed handle takes the bucketed launch.  Fewer
// go by the table of packed workgroups: all its lanes are in use and its reads
// and writes are contiguous, but every wavefront passes over as many partners as
// its largest swarm has, each substep.  (us a call with K = 6, table against
// items.  Two substeps: 524k of 1 to 32 63 / 83.  Eight and more, slots nearly full:
// 131k of 1, 2, 4 .. 32: eight 41.7 / 35.1, sixteen 91 / 74; 524k: 113 / 109,
// 202 / 180.)  Small batches keep the table, whose substeps two wavefronts
// share (16k in thirties, eight 23.9 / 27.0; 32k of 1 to 32, ten 30.4 / 33.4;
// 65k of 1, 2 .. 32, ten 39.7 / 39.2).  Padded slots cost lanes: with a quarter
// of them empty the items lose once they need more wavefronts than the three a
// SIMD holds (524k of 1 to 32, ten substeps: 130 / 143; 131k: 53 / 48), and always
// where the swarms are small (sixteen at most: 131k in twelves 38.9 / 40.0, 524k
// 103 / 127).
int default_items_from(const qs_handle* h) {
  constexpr long long resident = 3LL * 4 * 256 * 64;  // places of 3 wavefronts on every SIMD
  if (h->Q <= 65536) return INT_MAX;
  long long places = 0;
  for (int k = 0; k < 7; ++k) places += (long long)h->slot_swarms[k] << k;
  const bool full = 10LL * h->Q >= 9 * places;
  return full || (h->max_n > 16 && places <= resident) ? 8 : INT_MAX;
}

int launch(qs_handle* h, const float* act, int nsub, const float* goals, float* obs,
           bool with_obs, hipStream_t s, float* rw = nullptr) {
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  int rc;
  if (h->bucketed && nsub >= h->items_from) {
    (h->item_bs == 128 ? qs_host::launch_items128 : qs_host::launch_items64)(
        h, act, nsub, goals, obs, with_obs, s, rw);
    rc = hipGetLastError() == hipSuccess ? QS_OK : QS_ERR_HIP;
  } else {
    rc = (h->bs == 128 ? qs_host::launch_step128 : qs_host::launch_step64)(
        h, act, nsub, goals, obs, with_obs, s, rw);
  }
  if (rc == QS_OK) h->t += (uint64_t)nsub;
  return rc;
}


// Autotuner trials: every trial starts from the saved state and substep
// counter; times come from HIP events around `reps` launches after 2 untimed
// ones.
struct Trial {
  qs_handle* h;
  const float *act, *goals;
  float* obs;
  int nsub;
  bool with_obs;
  hipStream_t s;
  float* saved;
  size_t st_bytes;
  uint64_t t_saved;
  hipEvent_t e0, e1;

  int restore() {
    h->t = t_saved;
    return hipMemcpyAsync(h->d_st, saved, st_bytes, hipMemcpyDeviceToDevice, s) == hipSuccess
               ? QS_OK : QS_ERR_HIP;
  }
  template <typename F>
  int time(F&& launch_once, float* ms_per_launch) {
    int rc = restore();
    for (int w = 0; rc == QS_OK && w < 2; ++w) rc = launch_once();
    if (rc != QS_OK) return rc;
    if (hipEventRecord(e0, s) != hipSuccess) return QS_ERR_HIP;
    const int reps = 5;
    for (int r = 0; rc == QS_OK && r < reps; ++r) rc = launch_once();
    float ms = 0.f;
    if (rc != QS_OK) return rc;
    if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
        hipEventElapsedTime(&ms, e0, e1) != hipSuccess)
      return QS_ERR_HIP;
    *ms_per_launch = ms / reps;
    return QS_OK;
  }
  int call(float* ms) {
    return time([&] { return launch(h, act, nsub, goals, obs, with_obs, s); }, ms);
  }
  int range(int item0, int count, float* ms) {
    return time([&] {
      (h->item_bs == 128 ? qs_host::launch_range128 : qs_host::launch_range64)(
          h, item0, count, act, nsub, goals, obs, with_obs, s);
      return hipGetLastError() == hipSuccess ? QS_OK : QS_ERR_HIP;
    }, ms);
  }
};

// Launch configuration of a bucketed handle: workgroup size, persistent
// grid and the slot sizes that take the chunked partner body.
struct BucketConfig {
  int bs, grid;
  uint32_t chunked;
};

int apply(qs_handle* h, hipStream_t s, const BucketConfig& c, bool by_size = false) {
  // no launch may still read the tables that are about to be rebuilt
  if (hipStreamSynchronize(s) != hipSuccess) return QS_ERR_HIP;
  h->chunked = c.chunked;
  h->item_grid = c.grid;
  return build_items(h, c.bs, by_size);
}

// Bucketed handles: (1) workgroup sizes 64 and 128 and persistent grids,
// every slot size over its swarms' own sizes; (2) per slot size with two
// bodies (16 and 32), its items alone with each body, at the workgroup size
// of (1); (3) the call with each slot size on its faster body, over the
// grids; the faster of (1) and (3) is kept.  (4) Unless QS_BUCKETED asks for items
// in every call, the call by the table: whichever launch is the faster one, calls
// of this many substeps take from now on.
int tune_buckets(Trial& tr, BucketConfig* best) {
  qs_handle* h = tr.h;
  float best_ms = 1e30f;
  int rc = QS_OK;
  const int from = h->items_from;
  h->items_from = 0;
  for (int bs : {64, 128})
    for (int g : {0, 1024, 2048, 4096}) {
      const BucketConfig c{bs, g, 0u};
      float ms = 0.f;
      if ((rc = apply(h, tr.s, c)) != QS_OK || (rc = tr.call(&ms)) != QS_OK) return rc;
      if (ms < best_ms) {
        best_ms = ms;
        *best = c;
      }
    }
  for (int k = 0; k < 7; ++k) h->slot_ns_one[k] = h->slot_ns_chunked[k] = 0.f;
  uint32_t mask = 0u;
  for (int k = 0; k < 7; ++k) {
    if (!(kChunkable >> k & 1u) || h->slot_swarms[k] == 0) continue;
    float t[2] = {0.f, 0.f};
    for (int v = 0; v < 2; ++v) {
      if ((rc = apply(h, tr.s, {best->bs, 0, v ? 1u << k : 0u}, true)) != QS_OK) return rc;
      // the slot's item range
      std::vector<int4> items((size_t)h->n_items);
      if (hipMemcpy(items.data(), h->d_items, items.size() * sizeof(int4),
                    hipMemcpyDeviceToHost) != hipSuccess)
        return QS_ERR_HIP;
      int i0 = -1, i1 = -1;
      for (int i = 0; i < h->n_items; ++i)
        if (items[(size_t)i].x == (1 << k)) {
          if (i0 < 0) i0 = i;
          i1 = i + 1;
        }
      if (i0 < 0 || (rc = tr.range(i0, i1 - i0, &t[v])) != QS_OK) return rc;
    }
    h->slot_ns_one[k] = t[0] * 1e6f;
    h->slot_ns_chunked[k] = t[1] * 1e6f;
    if (t[1] < t[0]) mask |= 1u << k;
  }
  for (int g : {0, 1024, 2048, 4096}) {
    if (mask == 0u) break;
    const BucketConfig c{best->bs, g, mask};
    float ms = 0.f;
    if ((rc = apply(h, tr.s, c)) != QS_OK || (rc = tr.call(&ms)) != QS_OK) return rc;
    if (ms < best_ms) {
      best_ms = ms;
      *best = c;
    }
  }
  if (h->items_always) return QS_OK;
  float table_ms = 0.f;
  h->items_from = INT_MAX;
  if ((rc = tr.call(&table_ms)) != QS_OK) return rc;
  h->items_from = table_ms < best_ms ? std::max(from, tr.nsub + 1) : std::min(from, tr.nsub);
  return QS_OK;
}

}  // namespace

extern "C" {

int qs_create(const qs_desc* desc, const qs_quad_params* h_params, const float* h_state0,
              qs_handle** out) {
  if (!out) return QS_ERR_NULL;
  *out = nullptr;
  if (!h_params || !h_state0) return QS_ERR_NULL;
  int rc = check_desc(desc);
  if (rc != QS_OK) return rc;
  const int E = desc->n_envs;
  const int Q = desc->env_offsets[E];
  rc = qs_host::check_quads(Q, h_params, h_state0);
  if (rc != QS_OK) return rc;

  qs_handle* h = new (std::nothrow) qs_handle();
  if (!h) return QS_ERR_NOMEM;
  if (hipGetDevice(&h->dev) != hipSuccess) {
    delete h;
    return QS_ERR_HIP;
  }
  h->E = E;
  h->Q = Q;
  h->Qp = (Q + 63) / 64 * 64;
  h->K = desc->k_neighbors;
  h->OD = 18 + 6 * h->K;
  int max_n = 1;
  for (int e = 0; e < E; ++e)
    max_n = std::max(max_n, desc->env_offsets[e + 1] - desc->env_offsets[e]);
  h->max_n = max_n;
  h->bs = pick_block();

  // constants (derived in double, rounded once)
  Consts& c = h->c;
  c.dt = desc->dt;
  c.g = desc->gravity;
  c.arm_d = (float)((double)desc->arm_length / std::sqrt(2.0));
  c.k_tau = desc->k_tau;
  c.drag = desc->drag_coef;
  c.mu = desc->floor_mu;
  c.a_nd = desc->motor_noise_decay;
  const double and_ = desc->motor_noise_decay;
  c.ns_scale = (float)((double)desc->motor_noise_std * std::sqrt(1.0 - and_ * and_));
  c.rmin0 = desc->room_min[0];
  c.rmin1 = desc->room_min[1];
  c.rmin2 = desc->room_min[2];
  c.rmax0 = desc->room_max[0];
  c.rmax1 = desc->room_max[1];
  c.rmax2 = desc->room_max[2];
  c.e_wall = desc->wall_restitution;
  c.dcol2 = (float)((double)desc->col_dist * (double)desc->col_dist);
  c.dcol = desc->col_dist;
  c.col_decay = desc->col_decay;
  c.col_nv = desc->col_noise_v;
  c.col_nw = desc->col_noise_w;
  c.flags = desc->flags;
  c.key0 = (uint32_t)desc->seed;
  c.key1 = (uint32_t)(desc->seed >> 32);
  c.K = h->K;
  c.obs_dim = h->OD;
  c.dw_k1 = desc->dw_k1;
  c.dw_k2 = desc->dw_k2;
  c.dw_b1 = desc->dw_b1;
  c.dw_r2 = (float)((double)desc->dw_radius * (double)desc->dw_radius);
  c.dw_h = desc->dw_height;
  c.dw_na = desc->dw_noise_a;
  c.dw_nw = desc->dw_noise_w;
  c.sn_x = desc->sn_x;
  c.sn_v = desc->sn_v;
  c.sn_w = desc->sn_w;
  for (int k = 0; k < 15; ++k) c.rw[k] = 0.f;
  c.rw[14] = 1.f;

  // environment -> workgroup partition (environments are never split)
  h->env_start.resize(E);
  h->env_n.resize(E);
  std::vector<int32_t> qenv((size_t)Q, 0);
  for (int e = 0; e < E; ++e) {
    const int q0 = desc->env_offsets[e], n = desc->env_offsets[e + 1] - q0;
    h->env_start[e] = q0;
    h->env_n[e] = n;
    for (int i = 0; i < n; ++i) qenv[(size_t)q0 + i] = e;
  }
  // uniform power-of-two swarms: the greedy packing is then exactly
  // "workgroup b owns quads [b bs, (b+1) bs)", which the specialised kernels use
  {
    const int n0 = desc->env_offsets[1] - desc->env_offsets[0];
    bool uni = (n0 & (n0 - 1)) == 0 && h->bs % n0 == 0;
    for (int e = 1; uni && e < E; ++e) uni = desc->env_offsets[e + 1] - desc->env_offsets[e] == n0;
    h->uniform_n = uni ? n0 : 0;
  }

  // derived per-quad parameters and the state, in tiles
  std::vector<float> par((size_t)qs::NPARAM * h->Qp, 1.0f);
  std::vector<float> st((size_t)qs::NSTATE * h->Qp, 0.0f);
  for (int q = 0; q < Q; ++q) {
    const qs_quad_params& p = h_params[q];
    par[qs::par_index(q, qs::P_M)] = p.mass;
    par[qs::par_index(q, qs::P_JX)] = p.ixx;
    par[qs::par_index(q, qs::P_JY)] = p.iyy;
    par[qs::par_index(q, qs::P_JZ)] = p.izz;
    par[qs::par_index(q, qs::P_FMAX)] =
        (float)(0.25 * (double)p.mass * (double)desc->gravity * (double)p.thrust_to_weight);
    par[qs::par_index(q, qs::P_ALAG)] =
        (float)(1.0 - std::exp(-(double)desc->dt / (double)p.motor_tau));
    par[qs::par_index(q, qs::P_T2W)] = p.thrust_to_weight;
    par[qs::par_index(q, qs::P_TAU)] = p.motor_tau;
    const float* row = h_state0 + (size_t)q * QS_STATE_DIM;
    float* tile = st.data() + (size_t)(q >> 6) * (qs::NSTATE * qs::TILE_QUADS);
    const int lane = q & 63;
    for (int g = 0; g < 6; ++g)  // the tile's groups of four, then the last three
      for (int k = 0; k < 4; ++k)
        tile[(g * qs::TILE_QUADS + lane) * 4 + k] = row[qs::st_field(4 * g + k)];
    for (int k = 0; k < 3; ++k) tile[qs::ST_VF + 3 * lane + k] = row[qs::st_field(24 + k)];
  }

  rc = QS_OK;
  if (rc == QS_OK) rc = dalloc(&h->d_st, st.size());
  if (rc == QS_OK) rc = dalloc(&h->d_par, par.size());
  if (rc == QS_OK) rc = dalloc(&h->d_qenv, qenv.size());
  if (rc == QS_OK) rc = dalloc(&h->d_contacts, (size_t)h->Qp);
  if (rc == QS_OK) rc = dalloc(&h->d_err, 1);
  if (rc == QS_OK) rc = build_table(h, h->bs);
  if (rc == QS_OK && hipMalloc((void**)&h->d_t, sizeof(unsigned long long)) != hipSuccess)
    rc = QS_ERR_NOMEM;
  if (rc == QS_OK &&
      hipMalloc((void**)&h->d_done, qs::DONE_WORDS * sizeof(unsigned int)) != hipSuccess)
    rc = QS_ERR_NOMEM;
  if (rc == QS_OK && hipMalloc((void**)&h->d_c, sizeof(Consts)) != hipSuccess) rc = QS_ERR_NOMEM;
  if (rc == QS_OK && h->uniform_n == 0) {
    const char* ev = std::getenv("QS_BUCKETED");
    h->bucketed = !(ev && ev[0] == '0');
    if (h->bucketed) rc = build_items(h, 64);
    h->items_always = ev != nullptr;
    h->items_from = ev ? 0 : default_items_from(h);
  }
  if (rc == QS_OK && hipHostMalloc((void**)&h->h_err, sizeof(int)) != hipSuccess) {
    h->h_err = nullptr;
    rc = QS_ERR_NOMEM;
  }
  if (rc == QS_OK) {
    bool ok = hipMemcpy(h->d_st, st.data(), st.size() * sizeof(float), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemcpy(h->d_par, par.data(), par.size() * sizeof(float), hipMemcpyHostToDevice) == hipSuccess;
    if (Q > 0)
      ok = ok && hipMemcpy(h->d_qenv, qenv.data(), qenv.size() * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipMemset(h->d_contacts, 0, (size_t)h->Qp * sizeof(unsigned long long)) == hipSuccess;
    ok = ok && hipMemset(h->d_err, 0, sizeof(int)) == hipSuccess;
    ok = ok && hipMemset(h->d_t, 0, sizeof(unsigned long long)) == hipSuccess;
    ok = ok && hipMemset(h->d_done, 0, qs::DONE_WORDS * sizeof(unsigned int)) == hipSuccess;
    ok = ok && hipMemcpy(h->d_c, &h->c, sizeof(Consts), hipMemcpyHostToDevice) == hipSuccess;
    ok = ok && hipDeviceSynchronize() == hipSuccess;
    if (!ok) rc = QS_ERR_HIP;
  }
  if (rc != QS_OK) {
    free_all(h);
    delete h;
    return rc;
  }
  *h->h_err = 0;
  // set-up of the allocation-free entry point's scratch address on this
  // device (its own first call retries if this lookup failed)
  float* unused = nullptr;
  (void)noalloc_scratch(h->dev, &unused);
  *out = h;
  return QS_OK;
}

int qs_destroy(qs_handle* h) {
  if (!h) return QS_OK;
  (void)hipSetDevice(h->dev);
  (void)hipDeviceSynchronize();
  free_all(h);
  delete h;
  return QS_OK;
}

int qs_sizes(const qs_handle* h, int32_t* n_quads, int32_t* n_envs, int32_t* obs_dim) {
  if (!h) return QS_ERR_NULL;
  if (n_quads) *n_quads = h->Q;
  if (n_envs) *n_envs = h->E;
  if (obs_dim) *obs_dim = h->OD;
  return QS_OK;
}

int qs_substep_index(const qs_handle* h, uint64_t* substep_index) {
  if (!h || !substep_index) return QS_ERR_NULL;
  if (h->graph_mode) {
    unsigned long long v = 0;
    if (hipSetDevice(h->dev) != hipSuccess || hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(&v, h->d_t, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess)
      return QS_ERR_HIP;
    *substep_index = v;
    return QS_OK;
  }
  *substep_index = h->t;
  return QS_OK;
}

int qs_set_graph_mode(qs_handle* h, int32_t enable, void* stream) {
  if (!h) return QS_ERR_NULL;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  hipStream_t s = (hipStream_t)stream;
  if (hipStreamSynchronize(s) != hipSuccess) return QS_ERR_HIP;
  if (enable && !h->graph_mode) {
    hipLaunchKernelGGL(qs::set_counter_kernel, dim3(1), dim3(64), 0, s, h->d_t, h->d_done,
                       (unsigned long long)h->t);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
      return QS_ERR_HIP;
    h->graph_mode = true;
  } else if (!enable && h->graph_mode) {
    unsigned long long v = 0;
    if (hipMemcpy(&v, h->d_t, sizeof(v), hipMemcpyDeviceToHost) != hipSuccess) return QS_ERR_HIP;
    h->t = v;
    h->graph_mode = false;
  }
  return QS_OK;
}

int qs_set_launch(qs_handle* h, int32_t block, int32_t grid) {
  if (!h) return QS_ERR_NULL;
  if ((block != 64 && block != 128) || grid < 0) return QS_ERR_INVALID;
  if (hipSetDevice(h->dev) != hipSuccess || hipDeviceSynchronize() != hipSuccess) return QS_ERR_HIP;
  int rc = QS_OK;
  if (h->bucketed) {
    if (block != h->item_bs) rc = build_items(h, block);
    h->item_grid = grid;
    h->items_from = 0;
  } else if (block != h->bs) {
    if (h->uniform_n > 64 || block % std::max(h->uniform_n, 1) != 0) return QS_ERR_INVALID;
    rc = build_table(h, block);
  }
  return rc;
}

int qs_set_partner_chunks(qs_handle* h, uint32_t slot_mask) {
  if (!h) return QS_ERR_NULL;
  if (slot_mask & ~kChunkable) return QS_ERR_INVALID;
  if (hipSetDevice(h->dev) != hipSuccess || hipDeviceSynchronize() != hipSuccess) return QS_ERR_HIP;
  h->chunked = slot_mask;
  return h->bucketed ? build_items(h, h->item_bs) : QS_OK;
}

int qs_launch_plan(const qs_handle* h, int32_t* plan, int32_t* n_rows) {
  if (!h || !plan || !n_rows) return QS_ERR_NULL;
  int r = 0;
  for (int k = 6; k >= 0; --k) {
    if (h->slot_swarms[k] == 0) continue;
    int32_t* row = plan + 5 * r++;
    row[0] = 1 << k;
    row[1] = h->slot_swarms[k];
    row[2] = h->bucketed && ((h->chunked & kChunkable) >> k & 1u) ? 1 : 0;
    row[3] = (int32_t)std::lround(h->slot_ns_one[k]);
    row[4] = (int32_t)std::lround(h->slot_ns_chunked[k]);
  }
  *n_rows = r;
  return QS_OK;
}

int qs_autotune(qs_handle* h, const float* d_actions, int32_t n_substeps, const float* d_goals,
                float* d_obs, int32_t* choice, void* stream) {
  if (!h || !d_actions) return QS_ERR_NULL;
  if (n_substeps < 1 || (d_goals == nullptr) != (d_obs == nullptr)) return QS_ERR_INVALID;
  if (!aligned(d_actions, 16) || (d_obs && !aligned(d_obs, 8))) return QS_ERR_ALIGN;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  if (h->graph_mode) return QS_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  // the trials must not change the simulation: every candidate starts from
  // the saved state, and the state, substep counter and sticky error word
  // are restored afterwards
  float* saved = nullptr;
  const size_t st_bytes = (size_t)qs::NSTATE * h->Qp * sizeof(float);
  if (hipMalloc((void**)&saved, st_bytes + 256) != hipSuccess) return QS_ERR_NOMEM;
  int* saved_err = reinterpret_cast<int*>(reinterpret_cast<char*>(saved) + st_bytes);
  Trial tr{h, d_actions, d_goals, d_obs, (int)n_substeps, d_obs != nullptr, s, saved, st_bytes,
           h->t, nullptr, nullptr};
  int rc = hipMemcpyAsync(saved, h->d_st, st_bytes, hipMemcpyDeviceToDevice, s) == hipSuccess &&
                   hipMemcpyAsync(saved_err, h->d_err, sizeof(int), hipMemcpyDeviceToDevice, s) ==
                       hipSuccess
               ? QS_OK : QS_ERR_HIP;
  if (rc == QS_OK && (hipEventCreate(&tr.e0) != hipSuccess || hipEventCreate(&tr.e1) != hipSuccess))
    rc = QS_ERR_HIP;
  if (rc == QS_OK) {
    if (h->bucketed) {
      BucketConfig best{h->item_bs, h->item_grid, h->chunked};
      const int from = h->items_from;
      rc = tune_buckets(tr, &best);
      if (rc != QS_OK) h->items_from = from;
      if (rc == QS_OK) rc = apply(h, s, best);
    } else if (h->uniform_n > 0) {
      // uniform power-of-two swarms: workgroup size 64 or 128
      int best_bs = h->bs;
      float best_ms = 1e30f;
      for (int bs : {64, 128}) {
        if (bs % h->uniform_n != 0) continue;
        float ms = 0.f;
        if (hipStreamSynchronize(s) != hipSuccess) { rc = QS_ERR_HIP; break; }
        if (bs != h->bs && (rc = build_table(h, bs)) != QS_OK) break;
        if ((rc = tr.call(&ms)) != QS_OK) break;
        if (ms < best_ms) {
          best_ms = ms;
          best_bs = bs;
        }
      }
      if (rc == QS_OK && hipStreamSynchronize(s) != hipSuccess) rc = QS_ERR_HIP;
      if (rc == QS_OK && best_bs != h->bs) rc = build_table(h, best_bs);
    }
  }
  if (hipMemcpyAsync(h->d_st, saved, st_bytes, hipMemcpyDeviceToDevice, s) != hipSuccess ||
      hipMemcpyAsync(h->d_err, saved_err, sizeof(int), hipMemcpyDeviceToDevice, s) != hipSuccess ||
      hipStreamSynchronize(s) != hipSuccess)
    rc = QS_ERR_HIP;
  h->t = tr.t_saved;
  if (tr.e0) (void)hipEventDestroy(tr.e0);
  if (tr.e1) (void)hipEventDestroy(tr.e1);
  (void)hipFree(saved);
  if (rc == QS_OK && choice) {
    choice[0] = h->bucketed ? h->item_bs : h->bs;
    choice[1] = h->bucketed ? h->item_grid : h->nblk;
    choice[2] = h->bucketed ? 1 : 0;
  }
  return rc;
}

int qs_step(qs_handle* h, const float* d_actions, int32_t n_substeps, void* stream) {
  if (!h || !d_actions) return QS_ERR_NULL;
  if (n_substeps < 0) return QS_ERR_INVALID;
  if (!aligned(d_actions, 16)) return QS_ERR_ALIGN;
  if (n_substeps == 0) return QS_OK;
  return launch(h, d_actions, n_substeps, nullptr, nullptr, false, (hipStream_t)stream);
}

int qs_observe(qs_handle* h, const float* d_goals, float* d_obs, void* stream) {
  if (!h || !d_goals || !d_obs) return QS_ERR_NULL;
  if (!aligned(d_goals, 4) || !aligned(d_obs, 8)) return QS_ERR_ALIGN;
  const size_t Q = (size_t)h->Q;
  if (outputs_overlap({{d_obs, Q * h->OD * 4}}, {{d_goals, Q * 12}})) return QS_ERR_INVALID;
  return launch(h, nullptr, 0, d_goals, d_obs, true, (hipStream_t)stream);
}

int qs_step_observe(qs_handle* h, const float* d_actions, int32_t n_substeps,
                    const float* d_goals, float* d_obs, void* stream) {
  if (!h || !d_actions || !d_goals || !d_obs) return QS_ERR_NULL;
  if (n_substeps < 0) return QS_ERR_INVALID;
  if (!aligned(d_actions, 16) || !aligned(d_goals, 4) || !aligned(d_obs, 8)) return QS_ERR_ALIGN;
  const size_t Q = (size_t)h->Q;
  if (outputs_overlap({{d_obs, Q * h->OD * 4}}, {{d_actions, Q * 16}, {d_goals, Q * 12}}))
    return QS_ERR_INVALID;
  return launch(h, d_actions, n_substeps, d_goals, d_obs, true, (hipStream_t)stream);
}

int qs_set_reward_weights(qs_handle* h, const float* h_w) {
  if (!h || !h_w) return QS_ERR_NULL;
  for (int k = 0; k < 15; ++k)
    if (!finite(h_w[k])) return QS_ERR_INVALID;
  if (!(h_w[14] > 0.f)) return QS_ERR_INVALID;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  // enqueued calls still read the previous weights from the device copy
  if (hipDeviceSynchronize() != hipSuccess) return QS_ERR_HIP;
  for (int k = 0; k < 15; ++k) h->c.rw[k] = h_w[k];
  if (hipMemcpy(h->d_c, &h->c, sizeof(Consts), hipMemcpyHostToDevice) != hipSuccess)
    return QS_ERR_HIP;
  return QS_OK;
}

int qs_step_observe_reward(qs_handle* h, const float* d_actions, int32_t n_substeps,
                           const float* d_goals, float* d_obs, float* d_reward, void* stream) {
  if (!h || !d_actions || !d_goals || !d_obs || !d_reward) return QS_ERR_NULL;
  if (n_substeps < 1) return QS_ERR_INVALID;
  if (!aligned(d_actions, 16) || !aligned(d_goals, 4) || !aligned(d_obs, 8) ||
      !aligned(d_reward, 4))
    return QS_ERR_ALIGN;
  const size_t Q = (size_t)h->Q;
  if (outputs_overlap({{d_obs, Q * h->OD * 4}, {d_reward, Q * 4}},
                      {{d_actions, Q * 16}, {d_goals, Q * 12}}))
    return QS_ERR_INVALID;
  return launch(h, d_actions, n_substeps, d_goals, d_obs, true, (hipStream_t)stream, d_reward);
}

int qs_get_state(qs_handle* h, float* d_state, uint64_t* substep_index, void* stream) {
  if (!h || !d_state) return QS_ERR_NULL;
  if (!aligned(d_state, 4)) return QS_ERR_ALIGN;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  hipLaunchKernelGGL(qs::get_state_kernel, dim3(h->Qp / qs::IO_QUADS), dim3(qs::IO_THREADS), 0,
                     (hipStream_t)stream, h->d_st, h->Q, d_state);
  if (hipGetLastError() != hipSuccess) return QS_ERR_HIP;
  if (substep_index) *substep_index = h->t;
  return QS_OK;
}

int qs_set_state(qs_handle* h, const float* d_state, uint64_t substep_index,
                 const uint8_t* d_env_mask, void* stream) {
  if (!h || !d_state) return QS_ERR_NULL;
  if (!aligned(d_state, 4)) return QS_ERR_ALIGN;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  hipLaunchKernelGGL(qs::set_state_kernel, dim3(h->Qp / qs::IO_QUADS), dim3(qs::IO_THREADS), 0,
                     (hipStream_t)stream, h->d_st, h->Q, d_state, h->d_qenv, d_env_mask);
  if (hipGetLastError() != hipSuccess) return QS_ERR_HIP;
  h->t = substep_index;
  if (h->graph_mode)
    hipLaunchKernelGGL(qs::set_counter_kernel, dim3(1), dim3(64), 0, (hipStream_t)stream, h->d_t,
                       h->d_done, (unsigned long long)substep_index);
  return hipGetLastError() == hipSuccess ? QS_OK : QS_ERR_HIP;
}

int qs_record_contacts(qs_handle* h, int32_t enable) {
  if (!h) return QS_ERR_NULL;
  h->record = enable != 0;
  return QS_OK;
}

int qs_debug_contacts(qs_handle* h, uint64_t* d_mask, void* stream) {
  if (!h || !d_mask) return QS_ERR_NULL;
  if (!aligned(d_mask, 8)) return QS_ERR_ALIGN;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  if (hipMemcpyAsync(d_mask, h->d_contacts, (size_t)h->Q * sizeof(uint64_t),
                     hipMemcpyDeviceToDevice, (hipStream_t)stream) != hipSuccess)
    return QS_ERR_HIP;
  return QS_OK;
}

int qs_sync(qs_handle* h, void* stream) {
  if (!h) return QS_ERR_NULL;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  hipStream_t s = (hipStream_t)stream;
  if (hipMemcpyAsync(h->h_err, h->d_err, sizeof(int), hipMemcpyDeviceToHost, s) != hipSuccess)
    return QS_ERR_HIP;
  if (hipStreamSynchronize(s) != hipSuccess) return QS_ERR_HIP;
  const int bits = *h->h_err;
  if (bits != 0) {
    *h->h_err = 0;
    if (hipMemsetAsync(h->d_err, 0, sizeof(int), s) != hipSuccess) return QS_ERR_HIP;
    if (hipStreamSynchronize(s) != hipSuccess) return QS_ERR_HIP;
    return (bits & (qs::ERRBIT_STATE | qs::ERRBIT_ACTION)) ? QS_ERR_NONFINITE : QS_ERR_INVALID;
  }
  return QS_OK;
}

int qs_set_params(qs_handle* h, const float* d_params, const uint8_t* d_env_mask, void* stream) {
  if (!h || !d_params) return QS_ERR_NULL;
  if (!aligned(d_params, 4)) return QS_ERR_ALIGN;
  if (hipSetDevice(h->dev) != hipSuccess) return QS_ERR_HIP;
  const int tb = 256;
  hipLaunchKernelGGL(qs::set_params_kernel, dim3((unsigned)((h->Q + tb - 1) / tb)), dim3(tb), 0,
                     (hipStream_t)stream, h->d_par, h->Q, d_params, h->d_qenv, d_env_mask,
                     h->c.dt, h->c.g, h->d_err);
  return hipGetLastError() == hipSuccess ? QS_OK : QS_ERR_HIP;
}

int qs_debug_philox(uint64_t seed, uint32_t noise_stream, uint32_t draw, uint64_t substep_index,
                    uint32_t quad0, int32_t n, uint32_t* d_words, float* d_normals,
                    void* stream) {
  if (!d_words) return QS_ERR_NULL;
  if (n < 0 || noise_stream > 0xffffffu || draw > 0xffu ||
      (uint64_t)quad0 + (uint64_t)n > 0x100000000ull)
    return QS_ERR_INVALID;
  if (!aligned(d_words, 4) || (d_normals && !aligned(d_normals, 4))) return QS_ERR_ALIGN;
  if (d_normals && overlap({d_words, (size_t)n * 16}, {d_normals, (size_t)n * 16}))
    return QS_ERR_INVALID;
  if (n == 0) return QS_OK;
  const int tb = 256;
  hipLaunchKernelGGL(qs::philox_debug_kernel, dim3((unsigned)((n + tb - 1) / tb)), dim3(tb), 0,
                     (hipStream_t)stream, (uint32_t)seed, (uint32_t)(seed >> 32), noise_stream,
                     draw, (unsigned long long)substep_index, quad0, (int)n, d_words, d_normals);
  return hipGetLastError() == hipSuccess ? QS_OK : QS_ERR_HIP;
}

const char* qs_error_string(int code) {
  switch (code) {
    case QS_OK: return "ok";
    case QS_ERR_NULL: return "a required pointer is NULL";
    case QS_ERR_INVALID: return "a count, size or constant is out of range";
    case QS_ERR_ENV_SIZE: return "env_offsets is not CSR or a swarm has 0 or more than 64 quads";
    case QS_ERR_HIP: return "a HIP runtime call failed";
    case QS_ERR_NONFINITE: return "a non-finite action or state value was produced on the device";
    case QS_ERR_NOMEM: return "allocation failed";
    case QS_ERR_ALIGN: return "a device pointer is misaligned";
    case QS_ERR_UNSUPPORTED: return "request not supported by this build";
    case QS_ERR_TOO_LARGE:
      return "request exceeds the fixed scratch of the allocation-free entry point";
    default: return "unknown error code";
  }
}

}  // extern "C"
