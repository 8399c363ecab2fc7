// trace_fwd.hip -- forward ray tracing (Sec. 2.B, Eq. 1): one ray per lane, 64-ray
// tiles per wavefront, every scene of a batch in one launch.
#include <type_traits>

#include "rbos_device.hpp"
#include "rbos_launch.hpp"

namespace rbos {

// Trace one ray; writes its outputs. With checkpoints the buffer holds, component-major
// (component c of the ray at [c * ckpt_pad + ckpt_entry]): the ray header (see
// store_ray_header), then the states (d, e) before steps k, 2k, ... (6 components per
// slot).
template <int DT, bool QL, bool AHEAD>
__device__ __forceinline__ void trace_one(const SceneDev& S, int r, int pix, int smp) {
  int n = 0;
  unsigned char status = 0;
  float uvd[2] = {0.0f, 0.0f};
  bool ok = true;
  bool entered;
  RayBase B;
  Cell C;
  float e_end[3] = {0.0f, 0.0f, 0.0f};  // velocity deviation of the last state
  {
    Ray R;
    camera_ray(S, pix, smp, R.dir);
    df t_in;
    entered = box_entry(S, R.dir, t_in);
    if (entered) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        df x = dd_add(S.cam_pos[a], dd_mul(t_in, R.dir[a]));
        R.U0[a] = dd_add_f(dd_mul(dd_sub(x, S.lo[a]), S.inv_vox[a]), 0.5f);
      }
      make_base<DT>(S, R, B, C);
    }
  }
  if (!entered) {
    status |= RAY_MISSED_BOX;
  } else {
    State st;
    state_at_step(B, 0, st);
#pragma unroll
    for (int a = 0; a < 3; ++a) { st.d[a] = 0.0f; st.e[a] = 0.0f; }
    // checkpoint slot s holds the state after (s + 1) K steps
    const int q = ckpt_entry(S, r, pix, smp);
    float* ck = S.ckpt ? S.ckpt + (size_t)RAY_HEADER * S.ckpt_pad + (size_t)q : nullptr;
    const size_t slot_stride = 6 * (size_t)S.ckpt_pad;
    bool exited = false;
    std::conditional_t<AHEAD, Ahead, Sample> P;  // the next step's samples
    if constexpr (AHEAD && !QL) start_ahead<DT>(S, B, st, P);
    if constexpr (!AHEAD && !QL) sample_at_state<DT>(S, B, st, P);
    auto step = [&](auto issue) {
      if constexpr (AHEAD)
        sharma_step_ahead<DT>(S, B, st, P, NoRecord(), issue);
      else
        sharma_step<DT>(S, B, st, P, NoRecord(), issue);
    };
    // after each step: count it, stop on a non-finite state or outside the box. After a
    // Sharma step a non-finite position locates as NaN (outside), so only the velocity is
    // tested every step and the whole state once the ray stops.
    auto stop = [&]() {
      ++n;
      if (!isfinite((st.e[0] + st.e[1]) + st.e[2]) || outside_located(S, st, P.f)) {
        exited = true;
        if (!state_finite(st)) status |= RAY_NONFINITE;
      }
      return exited;
    };
    if constexpr (QL) {
      float Kc[3];  // force at the current point of the entry line
      force_at<DT>(S, C, Kc);
      while (n < S.max_steps) {
        ql_step<DT>(S, B, st, Kc);
        ++n;
        if (!state_finite(st)) {
          status |= RAY_NONFINITE;
          exited = true;
        } else if (outside_box(S, B, st)) {
          exited = true;
        }
        if (exited) break;
      }
    } else if (!ck) {
      while (n < S.max_steps) {
        step(NoIssue());
        if (stop()) break;
      }
    } else {
      // Segments of K steps; every segment after the first starts with a step whose start
      // state is stored. That step is a copy of its own with unconditional stores, issued
      // after its second gather (see NoIssue): in one loop with a branch around the stores,
      // the wait for the next gather at the branch's join would have to cover them.
      const int K = S.ckpt_k;
      int until = min(K, S.max_steps);
      while (!exited) {
        while (n < until) {
          step(NoIssue());
          if (stop()) break;
        }
        if (exited || n >= S.max_steps) break;
        step([&]() {
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            gst_stream(ck + (size_t)a * S.ckpt_pad, st.d[a]);
            gst_stream(ck + (size_t)(3 + a) * S.ckpt_pad, st.e[a]);
          }
        });
        ck += slot_stride;
        if (stop()) break;
        until = min(n - 1 + K, S.max_steps);
      }
    }
    if (!exited) status |= RAY_TRUNCATED;
#pragma unroll
    for (int a = 0; a < 3; ++a) e_end[a] = st.e[a];
    if (!(status & RAY_NONFINITE)) {
      float dX[3], s = 0.0f;
      const bool hit = wall_deflection(S, B, st, dX, &s);
      if (S.ckpt) store_ray_header(S, ckpt_entry(S, r, pix, smp), B, st, s);
      if (hit) {
        uvd[0] = dX[0] * S.wall_u_f[0] + dX[1] * S.wall_u_f[1] + dX[2] * S.wall_u_f[2];
        uvd[1] = dX[0] * S.wall_v_f[0] + dX[1] * S.wall_v_f[1] + dX[2] * S.wall_v_f[2];
      } else {
        status |= RAY_NO_WALL_HIT;
        ok = false;
      }
    } else {
      ok = false;
    }
  }
  // the undeflected camera ray's wall hit, recomputed here rather than kept live
  df dir[3], uv0[2];
  camera_ray(S, pix, smp, dir);
  const bool wall0 = wall_hit_straight(S, dir, uv0);
  if (!wall0 && !(status & RAY_NONFINITE)) {
    // the camera ray itself never reaches the wall: treat the hit as missing
    status |= RAY_NO_WALL_HIT;
    ok = false;
  }
  float u, v;
  if (ok) {
    u = dd_to_f(dd_add_f(uv0[0], uvd[0]));
    v = dd_to_f(dd_add_f(uv0[1], uvd[1]));
  } else {
    u = v = __builtin_nanf("");
    uvd[0] = uvd[1] = __builtin_nanf("");
  }
  gst(S.uv + 2 * (size_t)r, u);
  gst(S.uv + 2 * (size_t)r + 1, v);
  if (S.duv) {
    gst(S.duv + 2 * (size_t)r, uvd[0]);
    gst(S.duv + 2 * (size_t)r + 1, uvd[1]);
  }
  gst(S.n_steps + r, n);
  gst(S.status + r, status);
  if (S.wall_dir) {
    // unit direction at the wall: the exit velocity V + e (world units), or the camera
    // ray's for rays that never enter the box
    float w[3];
    if (status & RAY_NONFINITE) {
      w[0] = w[1] = w[2] = __builtin_nanf("");
    } else if (entered) {
      float n2 = 0.0f;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        w[a] = fmaf(e_end[a], S.vox[a], B.V[a]);
        n2 = fmaf(w[a], w[a], n2);
      }
      const float inv = 1.0f / sqrtf(n2);
#pragma unroll
      for (int a = 0; a < 3; ++a) w[a] *= inv;
    } else {
#pragma unroll
      for (int a = 0; a < 3; ++a) w[a] = dd_to_f(dir[a]);
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) gst(S.wall_dir + 3 * (size_t)r + a, w[a]);
  }
}

// When a step's gathers are issued: as it comes to their points, ahead, or whichever the
// wavefront's rays call for. A pixel list may be spread out, every ray in a cell of its own (16384
// to 130000 random pixels of a 512 x 512 camera, 128^3: ahead 286 to 334 us, at use 392 to 407),
// or a region of the image, whose rows stay within few cells: its gathers hit the caches, and the
// instructions that issue them ahead cost more than they hide (240 x 240 pixels of a 2048 x 1536
// camera: 307 against 254 us, of 1024 x 768: 301 and 253; 170 x 170 of 512 x 384: 287 and 256). The
// list lies on the device, so the wavefront looks for itself: rows of these regions lie in 4 to 13
// cells, the random lists' pixels in 24 to 64. The results are the same.
enum class Gathers { AT_USE, AT_USE_FEW, AHEAD, BY_WAVE };
constexpr int LIST_CELLS = 16;

// Wavefronts per SIMD the registers are held to. The Sharma step carries a sample between steps
// and takes 75 to 77 registers; held to 64 for 8 wavefronts it spills 11 to 18 of them. That pays
// for FP32 records beyond 9 tiles per compute unit (8 / 6 wavefronts, us: 900 x 900 rays, 192^3,
// stride 3 1730 / 1760; 1024 x 1024, 128^3, stride 16 1306 / 1340), and costs where wavefronts are few
// (384 x 384, 88^3 276 / 261) or samples that are decoded or gathered in parts meet checkpoint stores:
// BF16, 1024 x 1024, 128^3, stride 1 2123 / 1992, stride 3 1660 / 1643, 256 x 256, 64^3 170 / 161;
// FP16 256 x 256, 128^3 389 / 353, 1024 x 1024, stride 1 2177 / 2059; x-pairs 1894 / 1718, stride 1
// 2730 / 2114. Without checkpoints it pays for all types, 1024 x 1024, 128^3: BF16 1363 / 1373, FP16
// 1447 / 1470, x-pairs of FP32 1383 / 1416; 192^3 2005 / 2040, 2141 / 2190, 2063 / 2119; 512 x 512 (16 tiles
// per unit) alike.
template <Gathers MODE>
constexpr int fwd_waves_per_simd() {
  return MODE == Gathers::AHEAD || MODE == Gathers::BY_WAVE ? 2 : MODE == Gathers::AT_USE ? 8 : 6;
}

template <int DT, bool QL, Gathers MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(fwd_waves_per_simd<MODE>()))) void k_trace_fwd(
    const SceneDev* __restrict__ scenes, int n_scenes, int total_tiles, int wpb, int nblocks) {
  const int wave = wave_uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int gtile = xcd_remap(blockIdx.x, nblocks) * wpb + wave;
  if (gtile >= total_tiles) return;
  const int si = find_scene(scenes, n_scenes, gtile);
  const SceneDev& S = scenes[si];
  const int tile = gtile - S.tile_begin;
  int r, pix, smp;
  if (!tile_ray(S, tile, lane, r, pix, smp)) return;
  if (MODE == Gathers::BY_WAVE && S.pixel_ids && !pixels_spread(S, pix, LIST_CELLS))
    trace_one<DT, QL, false>(S, r, pix, smp);
  else
    trace_one<DT, QL, MODE == Gathers::AHEAD || MODE == Gathers::BY_WAVE>(S, r, pix, smp);
}

// Persistent form: blocks pull tiles from per-XCD queues (every 8th run of tiles), and
// steal from the other XCDs' queues once their own is drained.
template <int DT, bool QL>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(6))) void k_trace_fwd_persistent(const SceneDev* __restrict__ scenes, int n_scenes,
                                                              int total_tiles, unsigned int* __restrict__ queues) {
  const int lane = threadIdx.x & 63;
  const int xcd = blockIdx.x & 7;
  for (int q = 0; q < 8; ++q) {
    const int qx = (xcd + q) & 7;
    int q_begin, q_end;
    xcd_tile_range(total_tiles, qx, q_begin, q_end);
    while (true) {
      int t = 0;
      if (lane == 0) t = (int)atomicAdd(&queues[qx], 1u);
      t = wave_uniform(t);  // lane 0's claim (all lanes active)
      if (t >= q_end - q_begin) break;
      t = xcd_tile(total_tiles, qx, t);
      const int si = find_scene(scenes, n_scenes, t);
      const SceneDev& S = scenes[si];
      const int tile = t - S.tile_begin;
      int r, pix, smp;
      if (tile_ray(S, tile, lane, r, pix, smp)) trace_one<DT, QL, false>(S, r, pix, smp);
    }
  }
}

// Few wavefronts leave a step's gathers exposed: the kernel that issues them ahead runs, one
// wavefront per block so that they spread over the chip. The quasi-linear gathers do not wait
// for each other; more registers alone let two run together. Many wavefronts cover each
// other's gathers, the sooner the more of the field the caches hold, and the instructions
// that issue them ahead only cost. Each forward after its field's encoding, as a fit runs
// them, at use / ahead, us, 140 x 140 rays (1.3 tiles per compute unit), 256 x 256 (4) and
// 384 x 384 (9), stride 3:
// - FP32 24^3 78 / 76, 74 / 80, 93 / 98; 64^3 182 / 162, 167 / 174, 205 / 201; 96^3 277 / 231, 255 / 244,
//   296 / 290; 192^3 583 / 437, 546 / 461, 608 / 547; stride 16, 64^3 169 / 147, 151 / 144, 185 / 183;
// - x-pairs of FP32 32^3 104 / 104, 99 / 105, 126 / 131; 96^3 291 / 266, 258 / 274, 320 / 327; 192^3 617 /
//   528, 542 / 537, 645 / 633; of BF16 96^3 306 / 269, 265 / 282, 325 / 342; 192^3 646 / 532, 567 / 543, 657 / 657;
// - BF16 32^3 100 / 101, 98 / 108, 126 / 129; 96^3 279 / 260, 253 / 267, 312 / 315; 192^3 599 / 515, 548 / 525,
//   636 / 617;
// - FP16 costs more to decode still: 64^3 206 / 232, 190 / 217, 237 / 255; 192^3 652 / 743, 599 / 712, 689 /
//   758; x-pairs likewise.
// Up to two tiles per unit the next adjoint gains as well, where the checkpoints of a tile are
// in the L2 that its wavefront reads them through: 32^3, 140 x 140 rays 212 -> 202 us.
// Quasi-linear: FP32 24^3 68 / 58, 69 / 55, 85 / 78; 192^3 510 / 352, 475 / 354, 532 / 399, 512 x 512 rays
// (16) 604 / 536; FP16 64^3 166 / 133, 151 / 126, 195 / 172, 248 / 222; but BF16 64^3 131 / 124, 125 /
// 120, 167 / 160; 96^3 187 / 180, 176 / 191, 235 / 229, 306 / 331; 192^3 376 / 372, 362 / 380, 467 / 459, 606 / 635.
Form forward_form(const LaunchPlan& P) {
  int ahead;  // tiles per compute unit up to which gathers are issued ahead
  if (P.tracer == 1) {
    ahead = P.dtype != DT_BF16 ? 16 : P.voxels <= 3e5 ? 4 : 2;
  } else if (code_type(P.dtype) == DT_F16) {
    ahead = 0;
  } else {
    ahead = P.voxels >= (P.dtype == DT_F32 ? 5e5 : 3e6) ? 9 : 2;
  }
  if (P.total_tiles <= ahead * P.n_cus) return FORM_AHEAD;
  return P.persistent ? FORM_PERSISTENT : FORM_GRID;
}

template <int DT, bool QL>
static hipError_t launch_fwd_t(const LaunchPlan& P, hipStream_t stream) {
  const Form form = forward_form(P);
  if constexpr (QL || code_type(DT) != DT_F16) {  // see forward_form
    if (form == FORM_AHEAD) {
      // a compute unit with one tile waits for every gather, whatever the list
      auto* kernel = &k_trace_fwd<DT, QL, Gathers::AHEAD>;
      if constexpr (!QL) {
        if (P.lists && P.total_tiles > P.n_cus) kernel = &k_trace_fwd<DT, QL, Gathers::BY_WAVE>;
      }
      hipLaunchKernelGGL(kernel, dim3(P.total_tiles), dim3(64), 0, stream, P.scenes, P.n_scenes, P.total_tiles, 1,
                         P.total_tiles);
      return hipGetLastError();
    }
  }
  const dim3 block(64 * P.wpb);
  if (form == FORM_PERSISTENT) {
    const dim3 grid(persistent_grid(k_trace_fwd_persistent<DT, QL>, P, 0));
    hipLaunchKernelGGL((k_trace_fwd_persistent<DT, QL>), grid, block, 0, stream, P.scenes, P.n_scenes,
                       P.total_tiles, P.queues);
  } else {
    const int nblocks = (P.total_tiles + P.wpb - 1) / P.wpb;
    auto* kernel = &k_trace_fwd<DT, QL, Gathers::AT_USE>;
    if constexpr (!QL) {  // see fwd_waves_per_simd
      const bool many = DT == DT_F32 ? P.total_tiles > 9 * P.n_cus : !P.checkpoints && P.total_tiles > 16 * P.n_cus;
      if (!many) kernel = &k_trace_fwd<DT, QL, Gathers::AT_USE_FEW>;
    }
    hipLaunchKernelGGL(kernel, dim3(nblocks), block, 0, stream, P.scenes, P.n_scenes, P.total_tiles, P.wpb, nblocks);
  }
  return hipGetLastError();
}

template <int DT>
static hipError_t launch_fwd_dt(const LaunchPlan& P, hipStream_t stream) {
  return P.tracer == 1 ? launch_fwd_t<DT, true>(P, stream) : launch_fwd_t<DT, false>(P, stream);
}

hipError_t launch_trace_fwd(const LaunchPlan& P, hipStream_t stream) {
  if (P.total_tiles == 0) return hipSuccess;
  switch (P.dtype) {
    case DT_F32: return launch_fwd_dt<DT_F32>(P, stream);
    case DT_F16: return launch_fwd_dt<DT_F16>(P, stream);
    case DT_BF16: return launch_fwd_dt<DT_BF16>(P, stream);
    case DT_F32_XPAIR: return launch_fwd_dt<DT_F32_XPAIR>(P, stream);
    case DT_F16_XPAIR: return launch_fwd_dt<DT_F16_XPAIR>(P, stream);
    default: return launch_fwd_dt<DT_BF16_XPAIR>(P, stream);
  }
}

}  // namespace rbos
