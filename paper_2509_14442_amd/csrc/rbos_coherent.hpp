// rbos_coherent.hpp -- device code of the coherent adjoint: the rays of a tile that leave one
// cell are summed across the wavefront, over recorded chunks of the sweep.
#pragma once

#include "rbos_adjoint.hpp"

namespace rbos {

// Per-lane merge of the samples' monomial coefficients by cell. A lane that leaves a cell
// parks its sums. With PARK (kernels with registers to spare), the parked sums of a cell
// are reduced across the wavefront when one of its lanes leaves a second cell (its park
// is needed again), together with those of every other lane parked in that cell: the
// tile's rays leave a cell over a few samples, so one reduction then covers most of them.
// Without, the lanes leaving cells at a sample are reduced at once.
struct Accum {
  float acc[8];
  int key;        // record index of the cell (< 2^27), CELL_NONE when empty
  float park[8];  // the sums of the last cell left
  int pkey;       // its record index, CELL_NONE when the park is free
};

__device__ __forceinline__ void accum_init(Accum& A) {
#pragma unroll
  for (int k = 0; k < 8; ++k) A.acc[k] = A.park[k] = 0.0f;
  A.key = A.pkey = CELL_NONE;
}

// Per-wavefront cache of cell totals between the wavefront reduction and the FP64
// atomics: a cell is left by the tile's rays over several steps (the bundle crosses a
// face obliquely), so its partial totals are merged here and reach the gradient once.
// Slot p holds 8 corner totals in LDS (corner a + 2b + 4c) and its key in lane p of one
// register. Slots are written out in batches every few chunks (those not touched since
// the last batch) and at the end of the tile, so the atomics' latency is exposed once per
// batch rather than once per cell (a non-returning atomic still counts in vmcnt, which the
// next load waits on). A miss with every slot taken writes one slot out at once.
// The slot masks are 32-bit (one scalar register each): the kernels run at the scalar
// register limit, and every register freed spares a reload of a scene constant.
constexpr int PEND_SLOTS = 32;
static_assert(PEND_SLOTS == 32, "slot masks are one 32-bit word, all of whose bits are slots");

struct Pending {
  float* vals;        // LDS, PEND_SLOTS * 8 floats, wave-private
  int key;            // lane p < PEND_SLOTS: key of slot p; CELL_NONE when free (always for p >= PEND_SLOTS)
  int next;           // wave-uniform: slot replaced when all are taken
  unsigned occupied;  // wave-uniform slot masks
  unsigned touched;   // slots hit or filled since the last batch write-out
};

// Add the 8 wavefront totals of cell `key` (wave_sum8's layout) to its slot, taking a
// free slot, or writing one out, when the cell has none.
__device__ __forceinline__ void cache_add(const SceneDev& S, Pending& P, int key, float total, int lane) {
  const int corner = group_corner(lane);
  const unsigned hit = (unsigned)__ballot(P.key == key);  // only lanes < PEND_SLOTS hold keys
  int slot;
  if (hit) {
    slot = __ffs((int)hit) - 1;
    if ((lane & 7) == 0) atomicAdd(&P.vals[slot * 8 + corner], total);
  } else {
    const unsigned freem = ~P.occupied;
    if (freem) {
      slot = __ffs((int)freem) - 1;
    } else {
      slot = P.next;
      P.next = (P.next + 1) & (PEND_SLOTS - 1);
      const int old = __builtin_amdgcn_readlane(P.key, slot);
      if (lane < 8)
        gatomic_add(voxel_of_corner(S, old, lane), corner_of_monomials(P.vals + slot * 8, lane) * S.inv_dec_d);
      wave_lds_order();
    }
    if ((lane & 7) == 0) P.vals[slot * 8 + corner] = total;
    if (lane == slot) P.key = key;
    P.occupied |= 1u << slot;
  }
  P.touched |= 1u << slot;
  wave_lds_order();
}

// Add the accumulators of lanes with `sel` to the cache (lanes that hold the same cell
// summed across the wavefront) and restart them. Must run with all 64 lanes active.
__device__ __forceinline__ void flush(const SceneDev& S, Accum& A, bool sel, int lane, Pending& P) {
  unsigned long long pend = __ballot(sel);
  while (pend) {
    const int leader = __ffsll((long long)pend) - 1;
    const int key = __builtin_amdgcn_readlane(A.key, leader);
    const bool mine = sel && A.key == key;
    const unsigned long long mine_m = __ballot(A.key == key);  // a single comparison: no VALU round trip
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = mine ? A.acc[k] : 0.0f;
    cache_add(S, P, key, wave_sum8(v), lane);
    pend &= ~mine_m;
  }
  if (sel) {
#pragma unroll
    for (int k = 0; k < 8; ++k) A.acc[k] = 0.0f;
  }
}

// For every cell parked by a lane with `trig`: the parks of all lanes holding that cell
// go to the cache, summed across the wavefront, and are freed. Must run with all 64
// lanes active.
__device__ __forceinline__ void flush_parks(const SceneDev& S, Accum& A, bool trig, int lane, Pending& P) {
  unsigned long long pend = __ballot(trig);
  while (pend) {
    const int leader = __ffsll((long long)pend) - 1;
    const int key = __builtin_amdgcn_readlane(A.pkey, leader);
    const bool mine = A.pkey == key;
    const unsigned long long mine_m = __ballot(A.pkey == key);  // taken before the pkey reset below
    float v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = mine ? A.park[k] : 0.0f;
    cache_add(S, P, key, wave_sum8(v), lane);
    pend &= ~mine_m;
    if (mine) A.pkey = CELL_NONE;
  }
}

// Write the slots in `which` out to the gradient and free them.
__device__ __forceinline__ void write_out(const SceneDev& S, Pending& P, unsigned which, int lane) {
  wave_lds_order();
#pragma unroll 1
  for (int q = 0; q < PEND_SLOTS * 8 / 64; ++q) {
    if (((which >> (8 * q)) & 0xffu) == 0) continue;
    const int idx = q * 64 + lane, slot = idx >> 3;
    const int key = __shfl(P.key, slot);
    if ((which >> slot) & 1u)
      gatomic_add(voxel_of_corner(S, key, idx & 7), corner_of_monomials(P.vals + slot * 8, idx & 7) * S.inv_dec_d);
  }
  wave_lds_order();
  if (lane < PEND_SLOTS && ((which >> lane) & 1u)) P.key = CELL_NONE;
  P.occupied &= ~which;
}

// Batch write-out: the slots not touched since the last one (cells the rays have left).
__device__ __forceinline__ void chunk_end(const SceneDev& S, Pending& P, int lane) {
  const unsigned stale = P.occupied & ~P.touched;
  if (stale) write_out(S, P, stale, lane);
  P.touched = 0;
}

// Lanes with act take a sample in cell `key`: a lane that enters a new cell parks the sums
// of the one it leaves (after its park has been flushed, if taken), or flushes them
// without PARK, and starts from zero. The caller then adds the sample to A.acc. act_m is
// the ballot of act, which the caller takes once for all stages of a step. The wave-uniform
// tests combine ballots of single comparisons in scalar registers: a ballot of a compound
// lane predicate is lowered through a VALU select and compare, on the latency path of
// every sample.
template <bool PARK>
__device__ __forceinline__ void enter(const SceneDev& S, Accum& A, bool act, unsigned long long act_m, int key,
                                      int lane, Pending& P) {
  const bool out = act && key != A.key && A.key != CELL_NONE;
  const unsigned long long out_m = act_m & __ballot(key != A.key) & __ballot(A.key != CELL_NONE);
  if (out_m) {
    __builtin_amdgcn_s_setprio(3);  // the merge's reduction chains first (see adjoint_tile)
    if (PARK) {
      const bool busy = out && A.pkey != CELL_NONE;
      const unsigned long long busy_m = out_m & __ballot(A.pkey != CELL_NONE);
      if (busy_m) flush_parks(S, A, busy, lane, P);
      if (out) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          A.park[k] = A.acc[k];
          A.acc[k] = 0.0f;
        }
        A.pkey = A.key;
      }
    } else {
      flush(S, A, out, lane, P);
    }
    __builtin_amdgcn_s_setprio(1);
  }
  if (act) A.key = key;
}

// Tile end: the parks, then the open accumulators, into the cache; every slot out.
__device__ __forceinline__ void drain(const SceneDev& S, Accum& A, Pending& P, int lane) {
  if (__ballot(A.pkey != CELL_NONE)) flush_parks(S, A, A.pkey != CELL_NONE, lane, P);
  flush(S, A, A.key != CELL_NONE, lane, P);
  if (P.occupied) write_out(S, P, P.occupied, lane);
}

// The merge the coherent kernels hand to reverse_stages: accumulators (and parks) per lane,
// cell totals in the wavefront's cache.
template <bool PARK>
struct CellMerge : Accum {
  Pending P;
  __device__ __forceinline__ explicit CellMerge(float* cache) : P{cache, CELL_NONE, 0, 0u, 0u} { accum_init(*this); }
  __device__ __forceinline__ void enter(const SceneDev& S, bool act, unsigned long long act_m, int k, int lane) {
    rbos::enter<PARK>(S, *this, act, act_m, k, lane, P);
  }
  __device__ __forceinline__ void take(const SceneDev& S, int, const SampleRev& R, const float w[3], float p[3]) {
    force_rev(S, R, w, p, acc);
  }
};

// How a chunk of the reverse gets its steps' states.
enum class Replay {
  STORED,   // stride 1: every step's start state is a checkpoint; nothing is replayed
  SEGMENT,  // strides 3 and 4: a segment is one chunk, replayed from its checkpoint
  WALK,     // strides 6 and 8: each chunk from the checkpoint before it, over the steps in between
  CHUNKS,   // longer strides: a pass over the segment leaves its chunks' start states
};

// The replay of a chunk keeps, for each of its steps, the record index and fractions of the
// step's three samples as the forward located them (16 bytes per sample and lane in LDS,
// sample s of step i of lane l at [(i * 3 + s) * 64 + l]). The reverse of a step then reads
// them back, issues its three cell gathers together and evaluates value, gradient and mixed
// second derivatives at exactly the forward's cells and fractions, without relocating the
// samples from the state (no stage points, no K1 / K2, no dependent gathers). Chunks of 3
// steps take 10 KB of LDS per wavefront: 4 wavefronts per SIMD, registers held to 128; chunks
// of 4 take 13 KB: 3 per SIMD.
//
// With CHUNKS the start states of a part's chunks lie in a private array (24 bytes per
// chunk, coalesced, mostly in the L2): a part's steps run twice, where replays from the
// checkpoint to every chunk's start would be quadratic in the stride.
//
// STORED needs no replay: a chunk's LDS takes the states of twice its steps, loaded together, and
// the reverse locates each step's samples from its state. Recorded samples would cost it two
// gathers and the LDS traffic for nothing: 400 x 400 rays, 128^3, 1600 us against 1675, 640 x 640,
// 192^3, 4610 against 4890, f16 4810 against 5260.
//
// Adjoint of 1M rays, against chunks of 8 (stride 6: of 6) step states in LDS, whose samples the
// reverse located again, at 3 (4) wavefronts per SIMD: 6 5360 -> 5000 us, 8 5620 -> 5370, 16 6200
// -> 5600. 512 x 512 rays, stride 16: 2910 -> 2010, since its 4096 wavefronts now reside at once.
constexpr int PART_CHUNKS = 8;  // chunks of a part: strides up to 24, in chunks of 4 up to 32, are one part

template <int CHUNK>
constexpr int chunk_floats() { return CHUNK * 3 * 64 * 4; }

template <int CHUNK>
constexpr int adj_floats_per_wave() { return chunk_floats<CHUNK>() + PEND_SLOTS * 8; }

template <int CHUNK>
constexpr int adj_waves_per_simd() { return CHUNK == 3 ? 4 : 3; }

template <int CHUNK>
constexpr bool adj_park() { return CHUNK != 3; }  // registers for the parks

// Chunks between two write-outs of the cache's stale slots: each write-out exposes its
// atomics' latency once, and at every chunk of 3 steps that cost showed (-2 % adjoint time at
// 9 steps; at 12 or more the cache fills and misses write slots out one at a time).
template <int CHUNK>
constexpr int writeout_chunks() { return CHUNK == 3 ? 3 : 2; }

// The state at a segment's first step: the entry state or the checkpoint before it.
__device__ __forceinline__ void segment_state(const SceneDev& S, int q, int seg, State& st) {
  if (seg == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) { st.d[a] = 0.0f; st.e[a] = 0.0f; }
  } else {
    load_ckpt(S, q, seg - 1, st);
  }
}

// Replay cnt > 0 steps from st, their samples into LDS; the last step only up to its third sample.
template <int DT>
__device__ __forceinline__ void record_chunk(const SceneDev& S, const RayBase& B, State& st, int cnt, f32x4* smp,
                                             int lane) {
  Sample P;
  sample_at_state<DT>(S, B, st, P);
#pragma unroll 1
  for (int i = 0; i < cnt - 1; ++i) sharma_step<DT>(S, B, st, P, SampleRow{smp + i * 3 * 64 + lane});
  sharma_step<DT, SampleRow, NoIssue, false>(S, B, st, P, SampleRow{smp + (cnt - 1) * 3 * 64 + lane});
}

// The three samples of the step from st, located as sharma_step does from the same forces.
template <int DT>
__device__ __forceinline__ void stored_samples(const SceneDev& S, const RayBase& B, const State& st, SampleRev& R1,
                                               SampleRev& R2, SampleRev& R3) {
  Sample P;
  sample_at_state<DT>(S, B, st, P);
  sample_rev_at(S, P.c, P.rec, P.f, R1);
  float bh[3], sm[3];
  Cell C;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    bh[a] = st.bh[a] + B.g2hi[a];
    sm[a] = small_part(B, a, st.jf + 1.0f, stage2_dev(S, st, a, R1.eta * R1.g[a]));
  }
  locate3(S, bh, sm, C);
  sample_rev<DT>(S, C, R2);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    bh[a] += B.g2hi[a];
    sm[a] = small_part(B, a, st.jf + 2.0f, stage3_dev(S, a, stage3_base(S, st, a), R2.eta * R2.g[a]));
  }
  locate3(S, bh, sm, C);
  sample_rev<DT>(S, C, R3);
}

// Reverse of one chunk, from the samples in LDS: steps c0 + cnt - 1 .. c0 of lanes with cnt > 0.
template <int DT, int CHUNK>
__device__ __forceinline__ void reverse_chunk(const SceneDev& S, CellMerge<adj_park<CHUNK>()>& M, const f32x4* smp, int cnt,
                                              float rb[3], float tb[3], int lane) {
  __builtin_amdgcn_s_setprio(1);
#pragma unroll  // one copy per step: 1 % faster than the rolled loop, same registers
  for (int i = CHUNK - 1; i >= 0; --i) {
    const bool act = i < cnt;
    SampleRev R1, R2, R3;
    float wA[3], wB[3];
    if (act) {
      const f32x4* row = smp + i * 3 * 64 + lane;
      const f32x4 s1 = row[0], s2 = row[64], s3 = row[128];
      const unsigned r1 = __float_as_uint(s1.x), r2 = __float_as_uint(s2.x), r3 = __float_as_uint(s3.x);
      float c1[8], c2[8], c3[8];
      fetch_cell<DT>(S, r3, c3);
      fetch_cell<DT>(S, r2, c2);
      fetch_cell<DT>(S, r1, c1);
      const float f3[3] = {s3.y, s3.z, s3.w}, f2[3] = {s2.y, s2.z, s2.w}, f1[3] = {s1.y, s1.z, s1.w};
      sample_rev_at(S, c3, r3, f3, R3);
      sample_rev_at(S, c2, r2, f2, R2);
      sample_rev_at(S, c1, r1, f1, R1);
      stage_weights(S, rb, tb, wA, wB);
    }
    reverse_stages(S, M, act, R1, R2, R3, wA, wB, rb, tb, lane);
  }
}

// Wave priority, lowest to highest: the replay (a chain of dependent gathers), the reverse
// (independent gathers, long VALU runs), the merge (serial wavefront reductions, raised in
// `enter`). Each ordering step measured -2 % adjoint time in alternating runs, whatever the
// levels.
template <int DT, Replay MODE, int CHUNK>
__device__ __forceinline__ void adjoint_tile(const SceneDev& S, int tile, int lane, float* __restrict__ lds) {
  AdjRay R;
  adjoint_ray_setup(S, tile, lane, R);
  const int q = R.q, n = R.n;
  const bool active = R.active;
  const RayBase& B = R.B;
  float* rb = R.rb;
  float* tb = R.tb;
  CellMerge<adj_park<CHUNK>()> M(lds + chunk_floats<CHUNK>());
  f32x4* smp = reinterpret_cast<f32x4*>(lds);

  if constexpr (MODE == Replay::STORED) {
    constexpr int STEPS = 2 * CHUNK;  // whose states take a chunk's LDS
    const int nch = wave_max_nonneg(active ? (n + STEPS - 1) / STEPS : 0);
    for (int ch = nch - 1; ch >= 0; --ch) {
      const int c0 = ch * STEPS;
      const int cnt = active ? min(STEPS, n - c0) : 0;
      if (cnt > 0) {
        State st[STEPS];  // all loads in flight together
#pragma unroll
        for (int i = 0; i < STEPS; ++i)
          if (i < cnt) segment_state(S, q, c0 + i, st[i]);
#pragma unroll
        for (int i = 0; i < STEPS; ++i) {
          if (i >= cnt) continue;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            lds[(i * 6 + a) * 64 + lane] = st[i].d[a];
            lds[(i * 6 + 3 + a) * 64 + lane] = st[i].e[a];
          }
        }
      }
#pragma unroll 1
      for (int i = STEPS - 1; i >= 0; --i) {
        const bool act = i < cnt;
        SampleRev R1, R2, R3;
        float wA[3], wB[3];
        if (act) {
          State st;
          state_at_step(B, c0 + i, st);
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            st.d[a] = lds[(i * 6 + a) * 64 + lane];
            st.e[a] = lds[(i * 6 + 3 + a) * 64 + lane];
          }
          stored_samples<DT>(S, B, st, R1, R2, R3);
          stage_weights(S, rb, tb, wA, wB);
        }
        reverse_stages(S, M, act, R1, R2, R3, wA, wB, rb, tb, lane);
      }
      chunk_end(S, M.P, lane);
    }
  } else if constexpr (MODE == Replay::CHUNKS) {
    const int K = S.ckpt_k;
    const int part_len = min(K, CHUNK * PART_CHUNKS);
    const int nseg = wave_max_nonneg(active ? (n + K - 1) / K : 0);
    int due = writeout_chunks<CHUNK>();
    for (int seg = nseg - 1; seg >= 0; --seg) {
      for (int p0 = ((K - 1) / part_len) * part_len; p0 >= 0; p0 -= part_len) {
        const int s0 = seg * K + p0;                            // first step of the part
        const int m = active ? min(part_len, min(K - p0, n - s0)) : 0;  // the lane's steps in it
        const int nch = wave_max_nonneg((max(m, 0) + CHUNK - 1) / CHUNK);
        float start[PART_CHUNKS][6];
        __builtin_amdgcn_s_setprio(0);
        if (m > 0) {
          State st;
          state_at_step(B, seg * K, st);
          segment_state(S, q, seg, st);
          Sample P;
          if (nch > 1 || p0 > 0) sample_at_state<DT>(S, B, st, P);
#pragma unroll 1
          for (int i = 0; i < p0; ++i) sharma_step<DT>(S, B, st, P);  // to the part's start
#pragma unroll 1
          for (int c = 0;; ++c) {
#pragma unroll
            for (int a = 0; a < 3; ++a) { start[c][a] = st.d[a]; start[c][3 + a] = st.e[a]; }
            if ((c + 1) * CHUNK >= m) break;
#pragma unroll 1
            for (int i = 0; i < CHUNK; ++i) sharma_step<DT>(S, B, st, P);
          }
        }
#pragma unroll 1
        for (int c = nch - 1; c >= 0; --c) {
          const int c0 = c * CHUNK;
          const int cnt = min(CHUNK, m - c0);
          __builtin_amdgcn_s_setprio(0);
          if (cnt > 0) {
            State st;
            state_at_step(B, s0 + c0, st);
#pragma unroll
            for (int a = 0; a < 3; ++a) { st.d[a] = start[c][a]; st.e[a] = start[c][3 + a]; }
            record_chunk<DT>(S, B, st, cnt, smp, lane);
          }
          reverse_chunk<DT, CHUNK>(S, M, smp, cnt, rb, tb, lane);
          if (--due == 0) {
            chunk_end(S, M.P, lane);
            due = writeout_chunks<CHUNK>();
          }
        }
      }
    }
  } else {
    const int nch = wave_max_nonneg(active ? (n + CHUNK - 1) / CHUNK : 0);
    for (int ch = nch - 1; ch >= 0; --ch) {
      const int c0 = ch * CHUNK;  // first step of the chunk
      const int cnt = active ? min(CHUNK, n - c0) : 0;
      __builtin_amdgcn_s_setprio(0);
      if (cnt > 0) {
        // constant for SEGMENT: with the stride read, its replay took 2 % of the adjoint more
        const int K = MODE == Replay::SEGMENT ? CHUNK : S.ckpt_k;
        const int seg = c0 / K, s0 = seg * K;
        State st;
        state_at_step(B, s0, st);
        segment_state(S, q, seg, st);
        if (MODE == Replay::WALK && c0 > s0) {
          Sample P;
          sample_at_state<DT>(S, B, st, P);
#pragma unroll 1
          for (int i = s0; i < c0; ++i) sharma_step<DT>(S, B, st, P);  // to the chunk's start
        }
        record_chunk<DT>(S, B, st, cnt, smp, lane);
      }
      reverse_chunk<DT, CHUNK>(S, M, smp, cnt, rb, tb, lane);
      if (ch % writeout_chunks<CHUNK>() == 0) chunk_end(S, M.P, lane);
    }
  }
  // v0 from the ray header again rather than held in registers through the sweep
  float V0[3] = {0.0f, 0.0f, 0.0f};
  if (active) {
#pragma unroll
    for (int a = 0; a < 3; ++a) V0[a] = gld(S.ckpt + (size_t)q + (size_t)(12 + a) * (size_t)S.ckpt_pad);
  }
  entry_term(S, B, V0, active, tb, M, lane);
  drain(S, M, M.P, lane);
}

}  // namespace rbos
