// trace_adj_queue.hip -- the adjoint of scenes with few rays per cell or few wavefronts.
//
// The coherent kernels (trace_adj.hip) sum the rays of a tile that leave one cell across
// the wavefront, cell by cell. With about two rays per cell, or a random pixel list, that
// is a serial reduction for nearly every lane (8192 random pixels of a 512 x 512 camera in
// the 128^3 room: 7553 us, against 490 us for their forward). Here a lane that leaves a cell
// puts its sums into a queue in LDS (lanes that leave one cell together and are many are
// summed first). The queue is turned, 64 entries at a time and one lane per entry, into
// corner values, which collect per voxel in a table in LDS: the chip takes 2.4e10 FP64
// atomic requests a second, of one 64-byte line each, and eight of them for every cell that
// every ray crosses would bound these scenes (256 x 256 rays in that room: 3588 us without
// the table, 1209 with).
//
// What bounds it then is the instruction stream of one wavefront (4.5 to 6 cycles per
// instruction when alone on its SIMD), so gathers are issued ahead (sharma_step_ahead, the
// rows of the next step) and the registers for it are taken: one wavefront per SIMD.
#include <algorithm>
#include <cmath>

#include "rbos_coherent.hpp"
#include "rbos_launch.hpp"

namespace rbos {

// Lanes leaving one cell at a sample are summed across the wavefront from this many on.
constexpr int QUEUE_GROUP = 8;
constexpr int QUEUE_MISSES = 3;

// Voxel sums a wavefront keeps in LDS on their way to the gradient: voxel (x, y, z) has the
// slot of its low coordinate bits, so a compact bundle of rays meets no collision; what
// does collide goes straight to the gradient. A slot that no entry touched between two
// sweeps is written out.
//
// 8 slots per axis hold a tile's cells across the view down to one ray per cell; along the
// scene's view, 16: the slots the bundle has left wait there for the sweep (8: 1776 against
// 1223 us on the 128^3 room with 256 x 256 rays). Half a chunk's steps each leave fewer
// behind: 16 gain nothing in the four-wavefront form (538, 517 us).
constexpr int QUEUE_ENTRIES = 128;
constexpr int QUEUE_ACROSS = 3, QUEUE_ALONG = 4, PIPE_ALONG = 3;  // slot bits

constexpr unsigned SLOT_FREE = 0x7fffffffu, SLOT_TOUCHED = 0x80000000u;  // voxel indices are < 2^27

template <int ALONG>
struct QueueMerge {
  static constexpr int SLOTS = 1 << (ALONG + 2 * QUEUE_ACROSS);
  static constexpr size_t BYTES = (size_t)QUEUE_ENTRIES * 36 + (size_t)SLOTS * 12;

  float acc[8];
  int key;         // record index of the lane's cell, CELL_NONE when empty
  f32x4* vals;     // LDS: 8 monomial totals per entry
  int* keys;       // LDS: the entry's cell
  double* sums;    // LDS: the table's voxel sums
  unsigned* tags;  // LDS: the slot's voxel, SLOT_FREE when free, with SLOT_TOUCHED since the last sweep
  int count;       // wave-uniform: queue entries
  int claims;      // wave-uniform: slots taken since the last sweep

  __device__ __forceinline__ QueueMerge(float* lds, int lane)
      : key(CELL_NONE), count(0), claims(0) {
    vals = reinterpret_cast<f32x4*>(lds);
    keys = reinterpret_cast<int*>(lds + 8 * QUEUE_ENTRIES);
    sums = reinterpret_cast<double*>(lds + 9 * QUEUE_ENTRIES);
    tags = reinterpret_cast<unsigned*>(sums + SLOTS);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
    for (int i = lane; i < SLOTS; i += 64) {
      sums[i] = 0.0;
      tags[i] = SLOT_FREE;
    }
    wave_lds_order();
  }

  // The last `n` (<= 64) queue entries into the table, one lane per entry: the corner values
  // of an entry's monomial totals in binary64 (one difference per axis and pair: corner 0
  // of an axis is m0 - m1, corner 1 is m1).
  __device__ __forceinline__ void insert(const SceneDev& S, int n, int lane) {
    wave_lds_order();
    count -= n;
    const bool on = lane < n;
    int took = 0;
    if (on) {
      const int i = count + lane;
      const f32x4 lo = vals[2 * i], hi = vals[2 * i + 1];
      double g[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int ax = 1; ax < 8; ax <<= 1) {
#pragma unroll
        for (int c = 0; c < 8; ++c)
          if (!(c & ax)) g[c] -= g[c | ax];
      }
      int p[3];
      cell_of_record(S, (unsigned)keys[i], p);
      // the two clamped corners per axis (apron corners repeat the edge voxel): their share
      // of the voxel index and of the slot
      unsigned v[3][2], s[3][2];
      unsigned stride = 1u;
      int shift = 0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const unsigned c0 = (unsigned)max(p[a] - 1, 0), c1 = (unsigned)min(p[a], S.n[a] - 1);
        const int bits = ALONG == QUEUE_ACROSS || a != S.view_axis ? QUEUE_ACROSS : ALONG;
        const unsigned mask = (1u << bits) - 1u;
        v[a][0] = c0 * stride;
        v[a][1] = c1 * stride;
        s[a][0] = (c0 & mask) << shift;
        s[a][1] = (c1 & mask) << shift;
        stride *= (unsigned)S.n[a];
        shift += bits;
      }
      // claim or find the slots: all eight exchanges in flight together
      unsigned t[8];
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const unsigned vox = v[0][c & 1] + v[1][(c >> 1) & 1] + v[2][c >> 2];
        t[c] = SLOT_FREE;
        __hip_atomic_compare_exchange_strong(&tags[s[0][c & 1] + s[1][(c >> 1) & 1] + s[2][c >> 2]], &t[c],
                                             vox | SLOT_TOUCHED, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_WORKGROUP);
      }
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const unsigned vox = v[0][c & 1] + v[1][(c >> 1) & 1] + v[2][c >> 2];
        const unsigned slot = s[0][c & 1] + s[1][(c >> 1) & 1] + s[2][c >> 2];
        const double x = g[c] * S.inv_dec_d;
        const bool taken = t[c] == SLOT_FREE;
        took += taken ? 1 : 0;
        if (taken || (t[c] & ~SLOT_TOUCHED) == vox) {
          __hip_atomic_fetch_add(&sums[slot], x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (t[c] == vox) tags[slot] = vox | SLOT_TOUCHED;
        } else {
          gatomic_add(S.grad + vox, x);
        }
      }
    }
    claims += wave_sum_int(took);
    wave_lds_order();
  }

  // Write out the slots that were not touched since the last sweep (all with `every`).
  __device__ __forceinline__ void sweep(const SceneDev& S, bool every, int lane) {
    wave_lds_order();
    const int n = SLOTS;
#pragma unroll 2
    for (int i = lane; i < n; i += 64) {
      const unsigned t = tags[i];
      if (t == SLOT_FREE) continue;
      if (every || !(t & SLOT_TOUCHED)) {
        gatomic_add(S.grad + (t & ~SLOT_TOUCHED), sums[i]);
        sums[i] = 0.0;
        tags[i] = SLOT_FREE;
      } else {
        tags[i] = t & ~SLOT_TOUCHED;
      }
    }
    claims = 0;
    wave_lds_order();
  }

  // The sums of the lanes in out_m (those lanes have out) become entries, and restart.
  __device__ __forceinline__ void push(const SceneDev& S, bool out, unsigned long long out_m, int lane) {
    if (count + 64 > QUEUE_ENTRIES) insert(S, 64, lane);
    // cells with many leaving lanes are summed first; the scan ends with the lanes left too
    // few, or after QUEUE_MISSES cells of few lanes
    unsigned long long pend = out_m, few = 0;
    int misses = 0;
    while (__popcll(pend) >= QUEUE_GROUP && misses < QUEUE_MISSES) {
      const int leader = __ffsll((long long)pend) - 1;
      const int cell = __builtin_amdgcn_readlane(key, leader);
      const unsigned long long group = pend & __ballot(key == cell);
      if (__popcll(group) < QUEUE_GROUP) {
        ++misses;
        few |= group;
        pend &= ~group;
        continue;
      }
      const bool mine = out && key == cell;
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = mine ? acc[k] : 0.0f;
      const float total = wave_sum8(v);
      if ((lane & 7) == 0) reinterpret_cast<float*>(vals)[8 * count + group_corner(lane)] = total;
      if (lane == 0) keys[count] = cell;
      ++count;
      pend &= ~group;
    }
    pend |= few;
    if (pend) {
      if ((pend >> lane) & 1) {
        const int i = count + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(pend >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((unsigned)pend, 0u));
        vals[2 * i] = f32x4{acc[0], acc[1], acc[2], acc[3]};
        vals[2 * i + 1] = f32x4{acc[4], acc[5], acc[6], acc[7]};
        keys[i] = key;
      }
      count += __popcll(pend);
    }
    if (out) {
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] = 0.0f;
    }
  }

  __device__ __forceinline__ void enter(const SceneDev& S, bool act, unsigned long long act_m, int k, int lane) {
    const bool out = act && k != key && key != CELL_NONE;
    const unsigned long long out_m = act_m & __ballot(k != key) & __ballot(key != CELL_NONE);
    if (out_m) push(S, out, out_m, lane);
    if (act) key = k;
  }
  __device__ __forceinline__ void take(const SceneDev& S, int, const SampleRev& R, const float w[3], float p[3]) {
    force_rev(S, R, w, p, acc);
  }

  // Entries and slots go out where the caller has its next gathers issued, so that the
  // atomics' latency runs beside the arithmetic of a step.
  __device__ __forceinline__ void ease(const SceneDev& S, int lane) {
    if (count >= 64) insert(S, 64, lane);
    if (claims >= SLOTS / 4) sweep(S, false, lane);
  }

  __device__ __forceinline__ void drain(const SceneDev& S, int lane) {
    push(S, key != CELL_NONE, __ballot(key != CELL_NONE), lane);
    while (count > 0) insert(S, min(count, 64), lane);
    sweep(S, true, lane);
  }
};

// The three samples of a step as the replay recorded them, with their cells' coefficients.
struct StepRows {
  unsigned rec[3];
  float f[3][3], c[3][8];
};

template <int DT>
__device__ __forceinline__ void load_rows(const SceneDev& S, const f32x4* row, StepRows& W) {
#pragma unroll
  for (int s = 2; s >= 0; --s) {
    const f32x4 v = row[s * 64];
    W.rec[s] = __float_as_uint(v.x);
    W.f[s][0] = v.y;
    W.f[s][1] = v.z;
    W.f[s][2] = v.w;
  }
#pragma unroll
  for (int s = 2; s >= 0; --s) fetch_cell<DT>(S, W.rec[s], W.c[s]);
}

// Nonlinear tracer, every checkpoint stride: chunks of KS steps replayed into LDS as
// recorded samples (record index and fractions), then reversed, the rows and cells of a
// step loaded one step ahead.
template <int DT, int KS>
__device__ __forceinline__ void adjoint_tile_queue(const SceneDev& S, int tile, int lane, float* lds) {
  AdjRay R;
  adjoint_ray_setup(S, tile, lane, R);
  const int q = R.q, n = R.n;
  const bool active = R.active;
  const RayBase& B = R.B;
  const bool stored = S.ckpt_k == 1;  // every step's start state is a checkpoint
  const int K = stored ? KS : S.ckpt_k;
  const int m_chunks = K / KS;
  const int nseg = wave_max_nonneg(active ? (n + K - 1) / K : 0);
  f32x4* rows = reinterpret_cast<f32x4*>(lds) + lane;
  QueueMerge<QUEUE_ALONG> M(lds + KS * 3 * 64 * 4, lane);

  // The state a chunk's replay starts from and its first samples, loaded while the chunk
  // before it (the one after it on the ray) is reversed.
  State st;
  Ahead P;
  auto load_start = [&](int step) {  // a multiple of the stride
    state_at_step(B, step, st);
    if (step == 0) {
#pragma unroll
      for (int a = 0; a < 3; ++a) { st.d[a] = 0.0f; st.e[a] = 0.0f; }
    } else {
      load_ckpt(S, q, step / S.ckpt_k - 1, st);
    }
  };
  int c0 = (nseg - 1) * K + (m_chunks - 1) * KS;  // first step of the chunk
  if (active && c0 < n && c0 >= 0 && !stored) {
    load_start(c0 / K * K);
    start_ahead<DT>(S, B, st, P);
  }
  for (; c0 >= 0; c0 -= KS) {
    const bool lane_chunk = active && c0 < n;
    if (lane_chunk) {
      const int cnt = min(KS, n - c0);
      if (stored) {
#pragma unroll 1
        for (int i = 0; i < cnt; ++i) {
          load_start(c0 + i);
          start_ahead<DT>(S, B, st, P);
          sharma_step_ahead<DT, SampleRow, NoIssue, false>(S, B, st, P, SampleRow{rows + i * 3 * 64});
        }
      } else {
#pragma unroll 1
        for (int i = c0 % K; i > 0; --i) sharma_step_ahead<DT>(S, B, st, P);
#pragma unroll 1
        for (int i = 0; i < cnt - 1; ++i) sharma_step_ahead<DT>(S, B, st, P, SampleRow{rows + i * 3 * 64});
        sharma_step_ahead<DT, SampleRow, NoIssue, false>(S, B, st, P, SampleRow{rows + (cnt - 1) * 3 * 64});
      }
    }
    const bool next = active && !stored && c0 > 0 && c0 - KS < n;
    if (next) load_start((c0 - KS) / K * K);
    StepRows cur;
    if (lane_chunk && c0 + KS - 1 < n) load_rows<DT>(S, rows + (KS - 1) * 3 * 64, cur);
#pragma unroll 1
    for (int i = KS - 1; i >= 0; --i) {
      const bool act = lane_chunk && c0 + i < n;
      SampleRev R1, R2, R3;
      float wA[3], wB[3];
      if (act) {
        sample_rev_at(S, cur.c[2], cur.rec[2], cur.f[2], R3);
        sample_rev_at(S, cur.c[1], cur.rec[1], cur.f[1], R2);
        sample_rev_at(S, cur.c[0], cur.rec[0], cur.f[0], R1);
        stage_weights(S, R.rb, R.tb, wA, wB);
      }
      if (i > 0 && lane_chunk && c0 + i - 1 < n) load_rows<DT>(S, rows + (i - 1) * 3 * 64, cur);
      if (i == 0 && next) start_ahead<DT>(S, B, st, P);
      M.ease(S, lane);
      reverse_stages(S, M, act, R1, R2, R3, wA, wB, R.rb, R.tb, lane);
    }
  }
  entry_term(S, B, B.V, active, R.tb, M, lane);
  M.drain(S, lane);
}

template <int DT, int KS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_trace_adj_queue(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles) {
  extern __shared__ float lds[];
  const int gtile = xcd_remap(blockIdx.x, total_tiles);
  const SceneDev& S = scenes[find_scene(scenes, n_scenes, gtile)];
  adjoint_tile_queue<DT, KS>(S, gtile - S.tile_begin, threadIdx.x, lds);
}

// Pixel lists beyond the four-wavefront form. The list lies on the device, so the tile's
// wavefront looks at its own pixels: in up to LIST_BUNCH cells they
// are rows of a region seen by many pixels per cell, and the coherent sweep runs. Adjoint at
// stride 3, 128^3, coherent / queue: 170 x 170 pixels of a 2048 x 1536 camera (3 or 4 cells) 733
// / 843 us, of 4096 x 3072 (2 or 3) 614 / 721, of 1024 x 768 (6 or 7) 1084 / 875; 30000 random
// pixels (a cell each) 6961 / 1408. One wavefront per SIMD at most, so its registers are free.
constexpr int LIST_BUNCH = 4;

__device__ __forceinline__ bool tile_bunched(const SceneDev& S, int tile, int lane) {
  int r, pix, smp;
  bool spread = false;
  if (tile_ray(S, tile, lane, r, pix, smp)) spread = pixels_spread(S, pix, LIST_BUNCH);
  return __ballot(spread) == 0;  // wave-uniform: the lanes with rays agree
}

template <int DT, int KS>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_trace_adj_list(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles) {
  extern __shared__ float lds[];
  const int gtile = xcd_remap(blockIdx.x, total_tiles);
  const SceneDev& S = scenes[find_scene(scenes, n_scenes, gtile)];
  const int tile = gtile - S.tile_begin, lane = threadIdx.x;
  if (!S.pixel_ids || !tile_bunched(S, tile, lane))
    adjoint_tile_queue<DT, KS>(S, tile, lane, lds);
  else if constexpr (KS == 3)
    adjoint_tile<DT, Replay::SEGMENT, 3>(S, tile, lane, lds);
  else if constexpr (KS == 4)
    adjoint_tile<DT, Replay::SEGMENT, 4>(S, tile, lane, lds);
  else if constexpr (KS == 6)
    adjoint_tile<DT, Replay::WALK, 4>(S, tile, lane, lds);
  else if (S.ckpt_k == 8)
    adjoint_tile<DT, Replay::WALK, 4>(S, tile, lane, lds);
  else if (S.ckpt_k == 1)
    adjoint_tile<DT, Replay::STORED, 4>(S, tile, lane, lds);
  else
    adjoint_tile<DT, Replay::CHUNKS, 4>(S, tile, lane, lds);
}

// With few tiles a wavefront's instruction stream is the whole time while three of four SIMDs
// idle. So a tile takes a block of four wavefronts, one per SIMD of a compute unit, each with
// its own part of the work on successive chunks of 6 or 8 steps: one replays a chunk's samples
// into LDS; one reverses the chunk after it (the adjoint of the ray alone: it leaves each
// sample's s and W); two sum the samples of the chunk after that, half of its steps each,
// every one with a queue and a table of its own. A ray's sums in a cell end where a half does, as
// they do nowhere in the form of one wavefront: there it has one binary32 sum, here two that meet
// in binary64. LDS per block: 114432 bytes in chunks of 6, 145152 in chunks of 8.
//
// Bound by the summing wavefronts' instructions (96 x 96 rays, 128^3, stride 3: 520 us; without
// their inserts 271, without any sums 260, the replay alone 247; one wavefront per tile 1098).
// 64 x 64 rays of the unit box: 182 -> 102 us; 8192 random pixels: 1082 -> 624. Three summing
// wavefronts take 446 us of the 520, but 738 for the random pixels: consecutive cells of a ray
// then more often meet in different tables, and more atomics follow.
struct ChainTerms {
  f32x4* row;  // the step's terms: sample s at row[s * 64]
  __device__ __forceinline__ void enter(const SceneDev&, bool, unsigned long long, int, int) {}
  __device__ __forceinline__ void take(const SceneDev& S, int sample, const SampleRev& R, const float w[3],
                                       float p[3]) {
    row[sample * 64] = force_terms(S, R, w, p);
  }
};

// All wavefronts of the block; orders LDS only: gathers and atomics stay in flight.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int KS>
constexpr int pipe_rows() { return KS * 3 * 64; }  // samples of a chunk
constexpr int PIPE_SUMS = 2;  // wavefronts that sum

template <int DT, int KS>
__device__ __forceinline__ void adjoint_tile_pipe(const SceneDev& S, int tile, int wave, int lane, float* lds) {
  constexpr int ROWS = pipe_rows<KS>();
  f32x4* const samples = reinterpret_cast<f32x4*>(lds) + lane;  // ring of 3 chunks
  f32x4* const terms = samples + 3 * ROWS;                      // ring of 2 chunks
  float* const entry = lds + 5 * ROWS * 4 + lane;               // the chain's last tb
  float* const queues = lds + 5 * ROWS * 4 + 3 * 64;
  AdjRay R;
  adjoint_ray_setup(S, tile, lane, R);
  const int q = R.q, n = R.n;
  const bool active = R.active;
  const RayBase& B = R.B;
  const int K = S.ckpt_k;
  // the same in every wavefront; each passes nch + 1 barriers, at the ends of rounds 0 .. nch
  const int nch = max(1, wave_max_nonneg(active ? (n + KS - 1) / KS : 0));

  if (wave == 0) {
    // reverse chunk nch - r in round r
    lds_barrier();
#pragma unroll 1
    for (int r = 1; r <= nch; ++r) {
      const int ch = nch - r;
      const int cnt = active ? min(KS, n - ch * KS) : 0;
      const f32x4* rows = samples + (r - 1) % 3 * ROWS;
      f32x4* out = terms + (r & 1) * ROWS;
      StepRows cur;
      if (KS - 1 < cnt) load_rows<DT>(S, rows + (KS - 1) * 3 * 64, cur);
#pragma unroll 1
      for (int i = KS - 1; i >= 0; --i) {
        const bool act = i < cnt;
        SampleRev R1, R2, R3;
        float wA[3], wB[3];
        if (act) {
          sample_rev_at(S, cur.c[2], cur.rec[2], cur.f[2], R3);
          sample_rev_at(S, cur.c[1], cur.rec[1], cur.f[1], R2);
          sample_rev_at(S, cur.c[0], cur.rec[0], cur.f[0], R1);
          stage_weights(S, R.rb, R.tb, wA, wB);
        }
        if (i > 0 && i - 1 < cnt) load_rows<DT>(S, rows + (i - 1) * 3 * 64, cur);
        ChainTerms M{out + i * 3 * 64};
        reverse_stages(S, M, act, R1, R2, R3, wA, wB, R.rb, R.tb, lane);
      }
      if (r == nch) {
#pragma unroll
        for (int a = 0; a < 3; ++a) entry[a * 64] = R.tb[a];
      }
      lds_barrier();
    }
    return;
  }
  if (wave == 1) {
    // replay chunk nch - 1 - r in round r
    State st;
    Ahead P;
    auto start = [&](int ch) {
      const int c0 = ch * KS, k0 = c0 / K * K;
      if (!active || c0 >= n) return;
      state_at_step(B, k0, st);
      if (k0 == 0) {
#pragma unroll
        for (int a = 0; a < 3; ++a) { st.d[a] = 0.0f; st.e[a] = 0.0f; }
      } else {
        load_ckpt(S, q, k0 / K - 1, st);
      }
      start_ahead<DT>(S, B, st, P);
    };
    start(nch - 1);
#pragma unroll 1
    for (int r = 0; r < nch; ++r) {
      const int ch = nch - 1 - r;
      const int cnt = active ? min(KS, n - ch * KS) : 0;
      f32x4* rows = samples + r % 3 * ROWS;
      if (cnt > 0) {
#pragma unroll 1
        for (int i = ch * KS % K; i > 0; --i) sharma_step_ahead<DT>(S, B, st, P);
#pragma unroll 1
        for (int i = 0; i < cnt - 1; ++i) sharma_step_ahead<DT>(S, B, st, P, SampleRow{rows + i * 3 * 64});
        sharma_step_ahead<DT, SampleRow, NoIssue, false>(S, B, st, P, SampleRow{rows + (cnt - 1) * 3 * 64});
      }
      if (ch > 0) start(ch - 1);
      lds_barrier();
    }
    lds_barrier();
    return;
  }
  // sum chunk nch + 1 - r in round r
  const int share = wave - 2;  // 0: the chunk's first steps
  QueueMerge<PIPE_ALONG> M(queues + (size_t)share * (QueueMerge<PIPE_ALONG>::BYTES / 4), lane);
  const int i0 = KS * share / PIPE_SUMS, i1 = KS * (share + 1) / PIPE_SUMS;
  lds_barrier();
  lds_barrier();
#pragma unroll 1
  for (int r = 2; r <= nch + 1; ++r) {
    const int ch = nch + 1 - r;
    const int cnt = active ? min(KS, n - ch * KS) : 0;
    const f32x4* rows = samples + (r - 2) % 3 * ROWS;
    const f32x4* in = terms + ((r - 1) & 1) * ROWS;
#pragma unroll 1
    for (int i = i1 - 1; i >= i0; --i) {
      const bool act = i < cnt;
      const unsigned long long act_m = __ballot(act);
      if (act_m == 0) continue;
      f32x4 row[3], t[3];
      if (act) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
          row[s] = rows[(i * 3 + s) * 64];
          t[s] = in[(i * 3 + s) * 64];
        }
      }
      M.ease(S, lane);
#pragma unroll
      for (int s = 2; s >= 0; --s) {
        M.enter(S, act, act_m, act ? (int)__float_as_uint(row[s].x) : 0, lane);
        if (act) {
          const float f[3] = {row[s].y, row[s].z, row[s].w};
          add_terms(f, t[s], M.acc);
        }
      }
    }
    if (r <= nch) lds_barrier();
  }
  if (share == 0) {
    const float tb[3] = {entry[0], entry[64], entry[128]};
    entry_term(S, B, B.V, active, tb, M, lane);
  }
  M.drain(S, lane);
}

template <int DT, int KS>
__global__ __launch_bounds__(64 * (2 + PIPE_SUMS)) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_trace_adj_pipe(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles) {
  extern __shared__ float lds[];
  const int gtile = xcd_remap(blockIdx.x, total_tiles);
  const SceneDev& S = scenes[find_scene(scenes, n_scenes, gtile)];
  adjoint_tile_pipe<DT, KS>(S, gtile - S.tile_begin, wave_uniform(threadIdx.x >> 6), threadIdx.x & 63, lds);
}

// Quasi-linear tracer: the line points j = 0 .. 2n are independent of each other, so a
// tile's range of them is shared out over `parts` wavefronts. The entry term is linear in
// the adjoint of the entry velocity: each part adds its own share.
template <int DT>
__device__ __forceinline__ void adjoint_tile_ql_queue(const SceneDev& S, int tile, int part, int parts, int lane,
                                                      float* lds) {
  AdjRay R;
  adjoint_ray_setup(S, tile, lane, R);
  const int n = R.n;
  const bool active = R.active;
  const RayBase& B = R.B;
  const int npts = wave_max_nonneg(active ? 2 * n + 1 : 0);
  const int j0 = (int)((long long)npts * part / parts), j1 = (int)((long long)npts * (part + 1) / parts);
  const float h = S.hf, h_6 = S.h_6;
  QueueMerge<QUEUE_ALONG> M(lds, lane);
  float pv[3] = {0.0f, 0.0f, 0.0f};  // dL/dv0 through the stage points (grid units)
  auto sample_point_j = [&](int j, Sample& P) {
    const float jf = (float)j;
    float bh[3], sm[3];
    Cell C;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      bh[a] = fmaf(jf, B.g2hi[a], B.U0hi[a]);
      sm[a] = small_part(B, a, jf, 0.0f);
    }
    locate3(S, bh, sm, C);
    P.rec = cell_index(S, C);
#pragma unroll
    for (int a = 0; a < 3; ++a) P.f[a] = C.f[a];
    fetch_cell<DT>(S, P.rec, P.c);
  };
  // samples are fetched two points ahead
  Sample P0, P1;
  if (active && j0 < j1 && j0 <= 2 * n) sample_point_j(j0, P0);
  if (active && j0 + 1 < j1 && j0 + 1 <= 2 * n) sample_point_j(j0 + 1, P1);
#pragma unroll 1
  for (int j = j0; j < j1; ++j) {
    const bool act = active && j <= 2 * n;
    SampleRev Rs;
    float w[3];
    if (act) {
      sample_rev_at(S, P0.c, P0.rec, P0.f, Rs);
      ql_force_adjoint(R, j, h, h_6, w);
#pragma unroll
      for (int a = 0; a < 3; ++a) w[a] *= S.km[a];  // dL/dK -> dL/dG
    }
    P0 = P1;
    if (active && j + 2 < j1 && j + 2 <= 2 * n) sample_point_j(j + 2, P1);
    M.ease(S, lane);
    M.enter(S, act, __ballot(act), act ? Rs.key : 0, lane);
    if (act) {
      float p[3];
      force_rev(S, Rs, w, p, M.acc);
      const float tj = (float)j * (0.5f * h);
#pragma unroll
      for (int a = 0; a < 3; ++a) pv[a] = fmaf(tj, p[a], pv[a]);
    }
  }
  float tb0[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) tb0[a] = part == 0 ? fmaf((float)n * h, R.rb[a], R.tb[a]) + pv[a] : pv[a];
  entry_term(S, B, B.V, active, tb0, M, lane);
  M.drain(S, lane);
}

template <int DT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 4))) void k_trace_adj_ql_queue(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles, int parts) {
  extern __shared__ float lds[];
  const int gtile = xcd_remap(blockIdx.x, total_tiles);
  const SceneDev& S = scenes[find_scene(scenes, n_scenes, gtile)];
  adjoint_tile_ql_queue<DT>(S, gtile - S.tile_begin, blockIdx.y, parts, threadIdx.x, lds);
}

// Steps per recorded chunk for a checkpoint stride.
static int queue_chunk(const LaunchPlan& P) {
  return P.ckpt_k == 3 || P.ckpt_k == 4 || P.ckpt_k == 6 ? P.ckpt_k : 8;
}

static size_t queue_lds(const LaunchPlan& P) {
  return (P.tracer == 1 ? 0 : (size_t)queue_chunk(P) * 3 * 64 * 16) + QueueMerge<QUEUE_ALONG>::BYTES;
}

// With every wavefront resident at once (4 per compute unit by registers, fewer by LDS), the
// nonlinear form is the faster the fewer rays share a cell: 128^3 room, stride 3, adjoint coherent
// / queue in us: 48 x 48 rays 7938 / 1105, 256 x 256 (7 rays per cell) 2464 / 1209; 48^3, 256 x 256
// (53) 398 / 375; 40^3 (76) 305 / 307; 32^3 (118) 229 / 242; 20^3 (303) 132 / 146. Where the line
// lies depends on what the coherent kernel of the stride replays: stride 4, 64^3 (30) 568 / 529,
// 48^3 (53) 351 / 372, 32^3 204 / 236; 6, 20^3 146 / 141; 1, 64^3 (21) 649 / 586, 48^3 (37) 381 /
// 418, 24^3 (150) 149 / 196; 8, 32^3 (84) 236 / 233, 24^3 (150) 167 / 170; 16, 48^3 (37) 436 / 409,
// 40^3 (54) 326 / 332, 32^3 (84) 243 / 259.
//
// At strides beyond 16 the queue forms walk from the checkpoint to every 8-step chunk, half of the
// segment on average, where the coherent kernel passes over each part of it once more: both lines
// fall with the 1.5th power of that walk. Coherent / queue, strides 16, 32, 64, 128, 256: 96^3, 176
// x 176 rays (6) 1915 / 873, 1933 / 1034, 2006 / 1315, 2143 / 1910, 2445 / 3085; 32^3, 160 x 160 (46)
// 275 / 267, 278 / 319, 291 / 402, 320 / 537; 192^3, 160 x 160 (1.3), 256: 10445 / 6921; beyond one
// residency, 224^3, 290 x 290 (3) 7025 / 4016, 7092 / 4747, 7309 / 6179, 7777 / 9054, 8709 / 14147;
// 300^3, 360 x 360 (2.7) 10374 / 7845, 10446 / 9429, 10794 / 12277, 12785 / 29734.
//
// Beyond one residency the coherent kernels' occupancy wins from about 6 rays per cell on: 192^3,
// 384 x 384 (7) 4003 / 4238; 128^3, 384 x 384 (17) 1823 / 2855. Strides 1, 8, 16, ... take 8-step
// chunks and 3 wavefronts per compute unit, so the line falls with the rounds. Stride 16: 290 x
// 290, 160^3 (6) 3394 / 2770, 224^3 (3) 7014 / 4030; 360 x 360, 224^3 (4.8) 5599 / 5693, 300^3
// (2.7) 10394 / 7872; 471 x 395 (5.5) 2693 / 3744; 4515 tiles (2.4) 5570 / 6006.
//
// The quasi-linear form shares a tile out over wavefronts while there are few: 64^3, 160 x 160
// (12) 773 / 135, 256 x 256 (30) 513 / 314, 384 x 384 (67) 478 / 712; 192^3, 384 x 384 (7) 3331 /
// 2839, 512 x 512 (13) 2974 / 5041.
//
// A pixel list's rays per cell are not known here. Lists go by queue up to one residency (see
// k_trace_adj_list; quasi-linear up to 4 tiles per compute unit), where that is the faster form
// for regions of the image and for random pixels alike, and by the coherent kernels beyond.
// Coherent / queue, 128^3: nonlinear, 1024 x 768 pixels, 240 x 240 of them (900 tiles) 1161 /
// 891, 60000 random ones of 512 x 512 5883 / 2385; 2025 tiles, 360 x 360 pixels of 2048 x 1536 906
// / 1666, of 512 x 512 2438 / 3255, random ones 4146 / 4870; 7813 tiles, random 9021 / 20272.
// Quasi-linear, 900 tiles: 658 / 401 and 5586 / 2309; 2025 tiles: 754 / 958 and 3845 / 4374; 7813
// tiles 8191 / 18159.
static bool adjoint_by_queue(const LaunchPlan& P) {
  if (P.tracer == 1) {
    const bool few = P.total_tiles <= 4 * P.n_cus;
    if (P.lists && !few) return false;
    return P.rays_per_cell < (P.total_tiles <= 2 * P.n_cus ? 64.0f : few ? 40.0f : 8.0f);
  }
  const int per_cu = std::min(4, (int)(160 * 1024 / queue_lds(P)));
  const int rounds = (P.total_tiles + per_cu * P.n_cus - 1) / (per_cu * P.n_cus);
  // steps run per step recorded, against stride 16
  const float walk = P.ckpt_k <= 16 ? 1.0f : (1.0f + 0.1f * (float)(std::min(P.ckpt_k, P.max_steps) / 8 - 1)) / 1.1f;
  const float rays_per_cell = P.rays_per_cell * walk * std::sqrt(walk);
  if (rounds <= 1) {
    if (P.lists || P.ckpt_k == 6) return true;
    return rays_per_cell < (P.ckpt_k == 1 ? 30.0f : P.ckpt_k == 3 ? 75.0f : P.ckpt_k == 8 ? 90.0f : 44.0f);
  }
  if (P.lists) return false;
  return rays_per_cell < (per_cu == 4 ? 6.0f : std::max(2.0f, 12.0f / (float)rounds));
}

// A block of the four-wavefront form takes a compute unit's LDS: as many tiles as units run at
// once, twice as many in turn. Adjoint, one wavefront per tile / four, us: 128^3 room, stride 3, 36
// tiles 1106 / 540, 256 tiles 1080 / 538, 900 tiles 1225 / 1817; stride 16, 144 tiles 1184 / 522;
// 64^3, stride 4, 256 tiles 510 / 288. Between one tile per unit and two, a second round gains
// - on fields of up to about 50^3 voxels: stride 3, 32^3, 484 tiles 244 / 213; 48^3, 289 tiles 386 / 338,
//   361 392 / 376, 484 383 / 356; but 52^3, 400 tiles 428 / 474, x-pairs, 324 tiles 460 / 495;
// - else while it is short and the rays share few cells (in brackets, rays per cell). FP32, stride 3:
//   192^3, 289 tiles (1) 1745 / 1363, 484 (1.6) 1730 / 1577; 160^3, 484 (2.2) 1425 / 1419; 128^3, 289 (2)
//   1132 / 1013, 400 (2.8) 1140 / 1082, 484 (3.4) 1119 / 1213; 96^3, 289 (3.5) 836 / 819, 361 (4.5) 838 /
//   899; 80^3, 289 (5) 683 / 709; 64^3, 289 (8) 544 / 639. The samples of longer strides and other
//   types cost the one wavefront more: stride 16, 128^3, 484 tiles 1177 / 1177; 96^3, 324 (4) 867 /
//   842; 80^3, 289 708 / 702, 324 (6) 719 / 708; 64^3, 289 564 / 660; FP16, 128^3, 400 tiles 1327 / 1170;
//   96^3, 324 962 / 914; 80^3, 289 807 / 778, 361 (6.5) 825 / 824; 64^3, 289 637 / 699; BF16 and x-pairs
//   of FP32 128^3, 400 tiles 1236 / 1112, 1252 / 1105; 80^3, 289 742 / 757, 750 / 751.
// Pixel lists on larger fields take it up to one tile per unit: 170 x 170 pixels of a 512 x 512 camera
// (452 tiles) 1209 / 2069, of 2048 x 1536 (see k_trace_adj_list) 733 / 814, 30000 random ones 1408 /
// 2172; 256 tiles 1039 / 1292, 637 / 299 and 1070 / 1152. On small fields regions gain and random
// pixels lose: 32^3, 176 x 176 of 512 x 384 258 / 197, 30000 random ones 536 / 746; 50^3 478 / 319 and
// 669 / 957. A list may be a small part of a call, and the line there is that of images. Strides
// beyond 16 stop at one tile per unit on every field, their walk is one wavefront's: stride 64,
// 192^3, 400 tiles 2872 / 3085, 96^3, 484 tiles 1315 / 1560, 144 tiles 1279 / 769; stride 256, 144 tiles
// 2944 / 2380, coherent 4472.
static bool adjoint_by_pipe(const LaunchPlan& P) {
  if (P.tracer == 1 || P.total_tiles > 2 * P.n_cus) return false;
  const float second_round = (float)P.total_tiles / (float)P.n_cus - 1.0f;
  if (second_round <= 0.0f) return true;
  if (P.ckpt_k > 16) return false;
  if (P.voxels <= 125000.0) return true;
  const float rays_per_cell = P.dtype == DT_F32 && P.ckpt_k <= 4 ? 4.0f : 7.0f;
  return !P.lists && P.rays_per_cell <= rays_per_cell && P.rays_per_cell * second_round <= 2.1f;
}

Form adjoint_form(const LaunchPlan& P) {
  if (adjoint_by_pipe(P)) return FORM_PIPE;
  if (adjoint_by_queue(P)) return FORM_QUEUE;
  return P.persistent ? FORM_PERSISTENT : FORM_GRID;
}

template <int DT, int KS>
static hipError_t launch_pipe_t(const LaunchPlan& P, hipStream_t stream) {
  const size_t lds = (size_t)pipe_rows<KS>() * 5 * 16 + 3 * 64 * 4 + PIPE_SUMS * QueueMerge<PIPE_ALONG>::BYTES;
  hipLaunchKernelGGL((k_trace_adj_pipe<DT, KS>), dim3(P.total_tiles), dim3(64 * (2 + PIPE_SUMS)), lds, stream, P.scenes,
                     P.n_scenes, P.total_tiles);
  return hipGetLastError();
}

template <int DT, int KS>
static hipError_t launch_queue_t(const LaunchPlan& P, hipStream_t stream) {
  static_assert(adj_floats_per_wave<KS == 3 ? 3 : 4>() <= KS * 3 * 64 * 4 + QUEUE_ENTRIES * 9, "the coherent sweep's LDS");
  auto* kernel = P.lists ? &k_trace_adj_list<DT, KS> : &k_trace_adj_queue<DT, KS>;
  hipLaunchKernelGGL(kernel, dim3(P.total_tiles), dim3(64), queue_lds(P), stream, P.scenes, P.n_scenes,
                     P.total_tiles);
  return hipGetLastError();
}

template <int DT>
static hipError_t launch_queue_dt(const LaunchPlan& P, hipStream_t stream) {
  if (P.tracer == 1) {
    const int parts = std::max(1, std::min(16, 8 * P.n_cus / P.total_tiles));
    hipLaunchKernelGGL(k_trace_adj_ql_queue<DT>, dim3(P.total_tiles, parts), dim3(64), queue_lds(P), stream, P.scenes,
                       P.n_scenes, P.total_tiles, parts);
    return hipGetLastError();
  }
  if (adjoint_form(P) == FORM_PIPE)
    return P.ckpt_k == 3 || P.ckpt_k == 6 ? launch_pipe_t<DT, 6>(P, stream) : launch_pipe_t<DT, 8>(P, stream);
  switch (queue_chunk(P)) {
    case 3: return launch_queue_t<DT, 3>(P, stream);
    case 4: return launch_queue_t<DT, 4>(P, stream);
    case 6: return launch_queue_t<DT, 6>(P, stream);
    default: return launch_queue_t<DT, 8>(P, stream);
  }
}

hipError_t launch_trace_adj_queue(const LaunchPlan& P, hipStream_t stream) {
  if (P.total_tiles == 0) return hipSuccess;
  switch (P.dtype) {
    case DT_F32: return launch_queue_dt<DT_F32>(P, stream);
    case DT_F16: return launch_queue_dt<DT_F16>(P, stream);
    case DT_BF16: return launch_queue_dt<DT_BF16>(P, stream);
    case DT_F32_XPAIR: return launch_queue_dt<DT_F32_XPAIR>(P, stream);
    case DT_F16_XPAIR: return launch_queue_dt<DT_F16_XPAIR>(P, stream);
    default: return launch_queue_dt<DT_BF16_XPAIR>(P, stream);
  }
}

}  // namespace rbos
