// trace_adj.hip -- Sec. 2.D: exact gradient of L_BOS with respect to eta - 1 per voxel,
// back-propagated through the wall step and every Sharma step of Eq. (1).
//
// Per wavefront (64 rays of one tile), the steps are processed from the last to the first
// in chunks of 3 or 4, aligned on the step index so that the tile's rays move through the same
// cells together. A chunk is replayed forward from a state at its start (a checkpoint, or one
// reached from there), keeping in LDS the cells and fractions of each step's three samples,
// and then reversed step by step; at stride 1 every step's state is at hand and nothing is
// replayed. Each sample's contributions are merged per lane, as monomial coefficients, while the ray
// stays in one cell; lanes that left the same cell are summed across the wavefront into a
// per-wavefront LDS cache of cell totals, which goes to the gradient with one FP64 atomic
// per corner. A wavefront lowers its issue priority while replaying and raises it while
// merging. Most loops stay rolled so the kernel fits the instruction cache; the per-ray
// geometry comes from the header the forward pass stored with the checkpoints.
#include "rbos_coherent.hpp"
#include "rbos_launch.hpp"

namespace rbos {

template <int DT, Replay MODE, int CHUNK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(adj_waves_per_simd<CHUNK>()))) void k_trace_adj(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles, int wpb, int nblocks) {
  const int wave = wave_uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int gtile = xcd_remap(blockIdx.x, nblocks) * wpb + wave;
  if (gtile >= total_tiles) return;  // whole wavefront
  const int si = find_scene(scenes, n_scenes, gtile);
  const SceneDev& S = scenes[si];
  extern __shared__ float lds[];
  adjoint_tile<DT, MODE, CHUNK>(S, gtile - S.tile_begin, lane, lds + wave * adj_floats_per_wave<CHUNK>());
}

template <int DT, Replay MODE, int CHUNK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(adj_waves_per_simd<CHUNK>()))) void k_trace_adj_persistent(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles, unsigned int* __restrict__ queues,
    const int* __restrict__ order) {
  const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const int xcd = blockIdx.x & 7;
  extern __shared__ float lds[];
  float* mine = lds + wave * adj_floats_per_wave<CHUNK>();
  for (int q = 0; q < 8; ++q) {
    const int qx = (xcd + q) & 7;
    int q_begin, q_end;
    xcd_tile_range(total_tiles, qx, q_begin, q_end);
    while (true) {
      int t = 0;
      if (lane == 0) t = (int)atomicAdd(&queues[8 + qx], 1u);
      t = wave_uniform(t) + q_begin;  // lane 0's claim (all lanes active)
      if (t >= q_end) break;
      t = wave_uniform(gld(order + t));
      const int si = find_scene(scenes, n_scenes, t);
      const SceneDev& S = scenes[si];
      adjoint_tile<DT, MODE, CHUNK>(S, t - S.tile_begin, lane, mine);
    }
  }
}

template <int DT, Replay MODE, int CHUNK>
static hipError_t launch_adj_mode(const LaunchPlan& P, hipStream_t stream) {
  const size_t lds = sizeof(float) * adj_floats_per_wave<CHUNK>() * (size_t)P.wpb;
  if (P.persistent) {
    const int grid = persistent_grid(k_trace_adj_persistent<DT, MODE, CHUNK>, P, lds);
    hipLaunchKernelGGL((k_trace_adj_persistent<DT, MODE, CHUNK>), dim3(grid), dim3(64 * P.wpb), lds, stream, P.scenes,
                       P.n_scenes, P.total_tiles, P.queues, P.tile_order);
  } else {
    int nblocks = (P.total_tiles + P.wpb - 1) / P.wpb;
    hipLaunchKernelGGL((k_trace_adj<DT, MODE, CHUNK>), dim3(nblocks), dim3(64 * P.wpb), lds, stream, P.scenes, P.n_scenes,
                       P.total_tiles, P.wpb, nblocks);
  }
  return hipGetLastError();
}

template <int DT>
__device__ __forceinline__ void adjoint_tile_ql(const SceneDev& S, int tile, int lane, float* __restrict__ cache) {
  AdjRay R;
  adjoint_ray_setup(S, tile, lane, R);
  const int n = R.n;
  const bool active = R.active;
  const RayBase& B = R.B;
  const int npts = wave_max_nonneg(active ? 2 * n + 1 : 0);
  const float h = S.hf, h_6 = S.h_6;
  CellMerge<true> M(cache);
  float pv[3] = {0.0f, 0.0f, 0.0f};  // dL/dv0 through the stage points (grid units)
#pragma unroll 1
  for (int j = 0; j < npts; ++j) {
    const bool act = active && j <= 2 * n;
    SampleRev Rs;
    float w[3];
    if (act) {
      float v[3];
      ql_force_adjoint(R, j, h, h_6, v);
      const float jf = (float)j;
      float bh[3], sm[3];
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        bh[a] = fmaf(jf, B.g2hi[a], B.U0hi[a]);
        sm[a] = small_part(B, a, jf, 0.0f);
      }
      Cell C;
      locate3(S, bh, sm, C);
      sample_rev<DT>(S, C, Rs);
#pragma unroll
      for (int a = 0; a < 3; ++a) w[a] = v[a] * S.km[a];  // dL/dK -> dL/dG
    }
    M.enter(S, act, __ballot(act), act ? Rs.key : 0, lane);
    if (act) {
      float p[3];
      force_rev(S, Rs, w, p, M.acc);
      const float tj = (float)j * (0.5f * h);
#pragma unroll
      for (int a = 0; a < 3; ++a) pv[a] = fmaf(tj, p[a], pv[a]);
    }
    if ((j & 15) == 15) chunk_end(S, M.P, lane);
  }
  float tb0[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) tb0[a] = fmaf((float)n * h, R.rb[a], R.tb[a]) + pv[a];
  entry_term(S, B, B.V, active, tb0, M, lane);
  drain(S, M, M.P, lane);
}

// Held to 80 registers for 6 wavefronts per SIMD: this latency-bound grid form runs 4 %
// faster that way, its small spill included (the persistent form gains nothing from it).
template <int DT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_trace_adj_ql(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles, int wpb, int nblocks) {
  const int wave = wave_uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int gtile = xcd_remap(blockIdx.x, nblocks) * wpb + wave;
  if (gtile >= total_tiles) return;  // whole wavefront
  const int si = find_scene(scenes, n_scenes, gtile);
  const SceneDev& S = scenes[si];
  extern __shared__ float lds[];
  adjoint_tile_ql<DT>(S, gtile - S.tile_begin, lane, lds + wave * (PEND_SLOTS * 8));
}

template <int DT>
__global__ __launch_bounds__(256) void k_trace_adj_ql_persistent(const SceneDev* __restrict__ scenes, int n_scenes,
                                                                 int total_tiles, unsigned int* __restrict__ queues,
                                                                 const int* __restrict__ order) {
  const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const int xcd = blockIdx.x & 7;
  extern __shared__ float lds[];
  float* cache = lds + wave * (PEND_SLOTS * 8);
  for (int q = 0; q < 8; ++q) {
    const int qx = (xcd + q) & 7;
    int q_begin, q_end;
    xcd_tile_range(total_tiles, qx, q_begin, q_end);
    while (true) {
      int t = 0;
      if (lane == 0) t = (int)atomicAdd(&queues[8 + qx], 1u);
      t = wave_uniform(t) + q_begin;  // lane 0's claim (all lanes active)
      if (t >= q_end) break;
      t = wave_uniform(gld(order + t));
      const int si = find_scene(scenes, n_scenes, t);
      const SceneDev& S = scenes[si];
      adjoint_tile_ql<DT>(S, t - S.tile_begin, lane, cache);
    }
  }
}

template <int DT>
static hipError_t launch_adj_ql(const LaunchPlan& P, hipStream_t stream) {
  const size_t lds = sizeof(float) * PEND_SLOTS * 8 * (size_t)P.wpb;
  if (P.persistent) {
    const int grid = persistent_grid(k_trace_adj_ql_persistent<DT>, P, lds);
    hipLaunchKernelGGL((k_trace_adj_ql_persistent<DT>), dim3(grid), dim3(64 * P.wpb), lds, stream, P.scenes,
                       P.n_scenes, P.total_tiles, P.queues, P.tile_order);
  } else {
    int nblocks = (P.total_tiles + P.wpb - 1) / P.wpb;
    hipLaunchKernelGGL((k_trace_adj_ql<DT>), dim3(nblocks), dim3(64 * P.wpb), lds, stream, P.scenes, P.n_scenes,
                       P.total_tiles, P.wpb, nblocks);
  }
  return hipGetLastError();
}

// Chunks of 4 run 3 wavefronts per SIMD with parks, chunks of 3 run 4 without: the former while
// they reside at once, and again where 16 wavefronts per compute unit leave a long second round.
// Adjoint by chunks of 4 / 3, us, at `tiles` per compute unit, 128^3 unless said:
// - stride 1: 9.8 1603 / 1738; 12.7 1896 / 1627; 16 2242 / 1722; 22 1462 / 1611 (96^3); 25 2357 /
//   2460; 25 4608 / 4721 (192^3); 32.3 2779 / 2612; 36 2858 / 2966; 46 3421 / 3385; 50 6664 / 6194
//   (192^3); 64 4750 / 4577;
// - stride 6: 11.4 1727 / 1938; 13 2137 / 1784; 17.5 2576 / 2292; 19 5110 / 5199 (192^3); 21 2548 /
//   2824; 25 2702 / 2814; 30 3061 / 2942; 36 3328 / 3271; 64 5480 / 5000;
// - stride 8: 11.4 1677 / 1985; 13 2090 / 1844; 17.5 2507 / 2422; 19 5110 / 5459 (192^3); 25 2651 /
//   2977; 30 3006 / 3172; 32 3091 / 3142, 5980 / 5691 (192^3), 7903 / 7435 (224^3); 36 3246 / 3531;
//   50 4303 / 4491; 64 5366 / 5506;
// - stride 16: 11.4 1759 / 1987; 13 2184 / 1838; 17.5 2600 / 2376; 21 2612 / 2982; 25 2801 / 2972;
//   30 3160 / 3223, 1414 / 1388 (64^3), 8010 / 7674 (224^3); 36 3495 / 3600; 39 3810 / 3854; 50
//   4601 / 4583; 64 6020 / 5600;
// - stride 32: 13 2223 / 2042; 17.5 2679 / 2606; 21 2627 / 3286; 30 3200 / 3577; 50 4694 / 5048.
static bool chunks_of_4(int stride, float tiles) {
  if (tiles <= 12.0f) return true;
  if (tiles <= 18.0f) return false;
  if (tiles <= 28.0f || stride > 16) return true;
  if (stride == 8) return tiles <= 30.5f || tiles > 33.0f;
  return (stride == 1 || stride == 16) && tiles > 33.0f && tiles <= 40.0f;
}

template <int DT>
static hipError_t launch_adj_dt(const LaunchPlan& P, hipStream_t stream) {
  if (P.tracer == 1) return launch_adj_ql<DT>(P, stream);
  const bool of4 = chunks_of_4(P.ckpt_k, (float)P.total_tiles / (float)P.n_cus);
  switch (P.ckpt_k) {
    case 1:
      return of4 ? launch_adj_mode<DT, Replay::STORED, 4>(P, stream) : launch_adj_mode<DT, Replay::STORED, 3>(P, stream);
    case 3: return launch_adj_mode<DT, Replay::SEGMENT, 3>(P, stream);
    case 4: return launch_adj_mode<DT, Replay::SEGMENT, 4>(P, stream);
    // A walk to a chunk's start takes 1.5 or 2 steps on average; a pass that leaves the starts takes
    // as many but for each segment's last chunk, which it cuts short: stride 6, 1M rays, 5000 us
    // by walks, 5200 by passes; stride 8 in chunks of 4, 5370 and 5630. Chunks of 3 do not divide
    // 8: there 3.5 steps, and the pass is the shorter way.
    case 6:
      return of4 ? launch_adj_mode<DT, Replay::WALK, 4>(P, stream) : launch_adj_mode<DT, Replay::WALK, 3>(P, stream);
    case 8:
      return of4 ? launch_adj_mode<DT, Replay::WALK, 4>(P, stream) : launch_adj_mode<DT, Replay::CHUNKS, 3>(P, stream);
  }
  return of4 ? launch_adj_mode<DT, Replay::CHUNKS, 4>(P, stream) : launch_adj_mode<DT, Replay::CHUNKS, 3>(P, stream);
}

// Processing order of the persistent adjoint. A tile's reverse sweep lasts as long as
// its longest ray, and the tiles of the per-XCD ranges differ by up to ~1.5x (rays that
// leave the box through a side face are short). Taken in index order, the long tiles
// that start last leave most wavefront slots idle at the end of the launch. Each range
// is therefore taken longest first: its tiles are counting-sorted by the forward's
// largest step count (ties in any order), so the short tiles fill the end.
__global__ __launch_bounds__(256) void k_tile_cost(const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles,
                                                   int* __restrict__ cost) {
  const int wave = wave_uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int gtile = blockIdx.x * 4 + wave;
  if (gtile >= total_tiles) return;  // whole wavefront
  const SceneDev& S = scenes[find_scene(scenes, n_scenes, gtile)];
  int r = 0, pix = 0, smp = 0, n = 0;
  if (tile_ray(S, gtile - S.tile_begin, lane, r, pix, smp)) n = max(gld(S.n_steps + r), 0);
  n = wave_max_nonneg(n);  // all 64 lanes active
  if (lane == 0) cost[gtile] = n;
}

constexpr int ORDER_KEYS = 1024;

__device__ __forceinline__ int order_key(int cost, int shift) {
  return ORDER_KEYS - 1 - min(cost >> shift, ORDER_KEYS - 1);  // longest first
}

// one block per XCD: the tiles it owns, longest first, into its range [b, e) of order
__global__ __launch_bounds__(ORDER_KEYS) void k_tile_order(const int* __restrict__ cost, int total_tiles, int shift,
                                                           int* __restrict__ order) {
  __shared__ int start[ORDER_KEYS];
  const int tid = threadIdx.x, x = blockIdx.x;
  int b, e;
  xcd_tile_range(total_tiles, x, b, e);
  start[tid] = 0;
  __syncthreads();
  for (int i = tid; i < e - b; i += ORDER_KEYS)
    atomicAdd(&start[order_key(gld(cost + xcd_tile(total_tiles, x, i)), shift)], 1);
  __syncthreads();
  // exclusive prefix sum of the key counts (Hillis-Steele)
  const int count = start[tid];
  int v = count;
  for (int d = 1; d < ORDER_KEYS; d <<= 1) {
    const int add = tid >= d ? start[tid - d] : 0;
    __syncthreads();
    v += add;
    start[tid] = v;
    __syncthreads();
  }
  start[tid] = v - count;
  __syncthreads();
  for (int i = tid; i < e - b; i += ORDER_KEYS) {
    const int t = xcd_tile(total_tiles, x, i);
    const int pos = atomicAdd(&start[order_key(gld(cost + t), shift)], 1);
    order[b + pos] = t;
  }
}

hipError_t launch_tile_order(const LaunchPlan& P, hipStream_t stream) {
  if (P.total_tiles == 0) return hipSuccess;
  hipLaunchKernelGGL(k_tile_cost, dim3((P.total_tiles + 3) / 4), dim3(256), 0, stream, P.scenes, P.n_scenes,
                     P.total_tiles, P.tile_cost);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_tile_order, dim3(8), dim3(ORDER_KEYS), 0, stream, P.tile_cost, P.total_tiles, P.order_shift,
                     P.tile_order);
  return hipGetLastError();
}

hipError_t launch_trace_adj(const LaunchPlan& P, hipStream_t stream) {
  if (P.total_tiles == 0) return hipSuccess;
  switch (P.dtype) {
    case DT_F32: return launch_adj_dt<DT_F32>(P, stream);
    case DT_F16: return launch_adj_dt<DT_F16>(P, stream);
    case DT_BF16: return launch_adj_dt<DT_BF16>(P, stream);
    case DT_F32_XPAIR: return launch_adj_dt<DT_F32_XPAIR>(P, stream);
    case DT_F16_XPAIR: return launch_adj_dt<DT_F16_XPAIR>(P, stream);
    default: return launch_adj_dt<DT_BF16_XPAIR>(P, stream);
  }
}

}  // namespace rbos
