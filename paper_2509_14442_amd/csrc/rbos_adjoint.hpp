// rbos_adjoint.hpp -- device code shared by the adjoint kernels: the reverse of one sample,
// one Sharma step, the ray setup and the entry term, and the wavefront reduction of cell
// sums.
#pragma once

#include <climits>

#include "rbos_device.hpp"

namespace rbos {

// Everything the reverse sweep needs about one sample.
struct SampleRev {
  float f[3];        // fraction within the cell
  int key;           // record index of the cell (cell_index)
  float g[3], H[3];  // code-unit gradient and mixed second derivatives
  float eta;         // 1 + delta
};

// A sample from its cell's 8 corner codes, record index and fractions.
__device__ __forceinline__ void sample_rev_at(const SceneDev& S, const float c[8], unsigned rec, const float f[3],
                                              SampleRev& R) {
  float q;
  trilinear_h(c, f, q, R.g, R.H);
  R.eta = fmaf(q, S.dec, S.one_plus_off);
#pragma unroll
  for (int a = 0; a < 3; ++a) R.f[a] = f[a];
  R.key = (int)rec;
}

template <int DT>
__device__ __forceinline__ void sample_rev(const SceneDev& S, const Cell& C, SampleRev& R) {
  float c[8];
  const unsigned rec = cell_index(S, C);
  fetch_cell<DT>(S, rec, c);
  sample_rev_at(S, c, rec, C.f, R);
}

// Reverse of G = force_code(P) (code units, G_a = eta dq/du_a) for its adjoint
// w = dL/dG: returns p = dL/dP (grid units) and adds the sample's contributions to
// dL/d(delta_c) for the 8 corners of its cell, times dec, to acc:
//   s = dec sum_a w_a g_a,  W_a = eta w_a,
//   p_b = s g_b + sum_{a != b} W_a H_ab,
//   dec dL/d delta_c = s w_c + sum_a W_a dw_c/du_a,
// with w_c the trilinear weight of corner c. The contributions are multilinear in the
// fractions (u, v, w) = f, so they are kept as the coefficients of the 8 monomials
// m = u^(m & 1) v^(m >> 1 & 1) w^(m >> 2): s m + sum_a W_a dm/du_a. Samples in one cell
// share the monomials' frame, so their coefficients add up; corner values follow from
// the totals (corner_of_monomials, scaled by 1 / dec). In apron cells the field is
// constant along the clamped axis (g and H vanish there); the two corners that share one
// edge voxel receive contributions that add up to the clamped-axis weights.
// force_terms returns p and (s, W); add_terms adds their coefficients.
__device__ __forceinline__ f32x4 force_terms(const SceneDev& S, const SampleRev& R, const float w[3], float p[3]) {
  const float s = S.dec * fmaf(w[0], R.g[0], fmaf(w[1], R.g[1], w[2] * R.g[2]));
  const float Wx = R.eta * w[0], Wy = R.eta * w[1], Wz = R.eta * w[2];
  // H = (H_xy, H_xz, H_yz)
  p[0] = fmaf(s, R.g[0], fmaf(Wy, R.H[0], Wz * R.H[1]));
  p[1] = fmaf(s, R.g[1], fmaf(Wx, R.H[0], Wz * R.H[2]));
  p[2] = fmaf(s, R.g[2], fmaf(Wx, R.H[1], Wy * R.H[2]));
  return f32x4{s, Wx, Wy, Wz};
}

__device__ __forceinline__ void add_terms(const float f[3], f32x4 t, float acc[8]) {
  const float s = t.x, Wx = t.y, Wy = t.z, Wz = t.w;
  const float u = f[0], v = f[1], x = f[2];
  const float m1 = fmaf(s, u, Wx);              // u:   s u + Wx
  const float m2 = fmaf(s, v, Wy);              // v:   s v + Wy
  const float m3 = fmaf(v, m1, Wy * u);         // uv:  s uv + Wx v + Wy u
  acc[0] += s;                                  // 1
  acc[1] += m1;
  acc[2] += m2;
  acc[3] += m3;
  acc[4] += fmaf(s, x, Wz);                     // w:   s w + Wz
  acc[5] = fmaf(x, m1, fmaf(Wz, u, acc[5]));    // uw:  s uw + Wx w + Wz u
  acc[6] = fmaf(x, m2, fmaf(Wz, v, acc[6]));    // vw:  s vw + Wy w + Wz v
  acc[7] = fmaf(x, m3, fmaf(Wz, u * v, acc[7]));  // uvw: s uvw + Wx vw + Wy uw + Wz uv
}

__device__ __forceinline__ void force_rev(const SceneDev& S, const SampleRev& R, const float w[3], float p[3],
                                          float acc[8]) {
  add_terms(R.f, force_terms(S, R, w, p), acc);
}

constexpr int CELL_NONE = INT_MIN;  // no cell (record indices are < 2^27)

// Corner c of a cell from its 8 monomial totals: the trilinear weight of corner
// (i, j, k) is the product over the axes of (1 - u) (bit 0) or u (bit 1), so monomial m
// enters corner c when it holds every axis set in c, with the sign (-1) per axis it holds
// beyond c. Summed in FP64.
__device__ __forceinline__ double corner_of_monomials(const float* vals, int c) {
  double g = 0.0;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    if ((m & c) == c) {
      const double t = (double)vals[m];
      g += (__popc(m & ~c) & 1) ? -t : t;
    }
  }
  return g;
}

// Sum 8 per-lane values over the 64 lanes, all eight at once: each exchange step halves
// the lanes per value and keeps the values apart (permlane32 / permlane16 swaps between
// value pairs, then one row rotation by 8), and the last three steps reduce within
// groups of 8 lanes. On return every lane of group g = lane / 8 holds the total of value
// (g & 4) | (g & 1) << 1 | (g >> 1) & 1. All 64 lanes must be active.
__device__ __forceinline__ float wave_sum8(const float v[8]) {
  float w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[k]), __float_as_uint(v[k + 4]), false, false);
    w[k] = __uint_as_float(s[0]) + __uint_as_float(s[1]);  // lanes 0-31: value k, 32-63: value k + 4
  }
  float u[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(w[2 * k]), __float_as_uint(w[2 * k + 1]), false, false);
    u[k] = __uint_as_float(s[0]) + __uint_as_float(s[1]);  // 16-lane rows: values 2k, 2k+1, 2k+4, 2k+5
  }
  const float t0 = u[0] + dpp_f<0x128>(u[0]);  // row_ror:8
  const float t1 = u[1] + dpp_f<0x128>(u[1]);
  float z = (__lane_id() & 8) ? t1 : t0;
  z += dpp_f<0xb1>(z);   // quad_perm [1,0,3,2]
  z += dpp_f<0x4e>(z);   // quad_perm [2,3,0,1]
  z += dpp_f<0x141>(z);  // row_half_mirror: completes the sum over 8 lanes
  return z;
}

__device__ __forceinline__ double* voxel_of_corner(const SceneDev& S, int key, int c) {
  int p[3];
  cell_of_record(S, (unsigned)key, p);
  // apron corners map to the edge voxel they repeat
  const int x = min(max(p[0] - 1 + (c & 1), 0), S.n[0] - 1);
  const int y = min(max(p[1] - 1 + ((c >> 1) & 1), 0), S.n[1] - 1);
  const int z = min(max(p[2] - 1 + (c >> 2), 0), S.n[2] - 1);
  return &S.grad[((size_t)z * S.n[1] + y) * S.n[0] + x];
}

// Order this lane's LDS accesses of the cache against other lanes' (the hardware runs a
// wavefront's LDS instructions in order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_order() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

// Corner of the total that lane group g = lane / 8 holds after wave_sum8.
__device__ __forceinline__ int group_corner(int lane) {
  const int g = lane >> 3;
  return (g & 4) | ((g & 1) << 1) | ((g >> 1) & 1);
}

__device__ __forceinline__ void load_ckpt(const SceneDev& S, int r, int slot, State& st) {
  const float* ck = S.ckpt + (size_t)(RAY_HEADER + slot * 6) * (size_t)S.ckpt_pad + (size_t)r;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    st.d[a] = gld(ck + (size_t)a * S.ckpt_pad);
    st.e[a] = gld(ck + (size_t)(3 + a) * S.ckpt_pad);
  }
}

// Ray setup of the adjoint: the ray of this lane, its step count and whether it carries
// a gradient, its straight-line base from the header, and the adjoint of the last state
// through the wall step X = x + s v:
//   lambda_x = lambda_X - n (v . lambda_X)/(v . n),  lambda_v = s lambda_x
// (metres; grid units multiply by the voxel size), returned as rb = dL/dd, tb = dL/de.
struct AdjRay {
  int r, q, n;  // ray, its checkpoint entry, its step count
  bool active;
  RayBase B;
  float rb[3], tb[3];
};

__device__ __forceinline__ void adjoint_ray_setup(const SceneDev& S, int tile, int lane, AdjRay& R) {
  int pix = 0;
  R.r = 0;
  R.q = 0;
  R.n = 0;
  R.active = false;
#pragma unroll
  for (int a = 0; a < 3; ++a) R.rb[a] = R.tb[a] = 0.0f;
  int smp;
  if (!tile_ray(S, tile, lane, R.r, pix, smp)) return;
  const int r = R.r;
  R.q = ckpt_entry(S, r, pix, smp);
  R.n = gld(S.n_steps + r);
  const unsigned char st = gld(S.status + r);
  const float lu = gld(S.adj_dL_duv + 2 * (size_t)r), lv = gld(S.adj_dL_duv + 2 * (size_t)r + 1);
  float ld[3] = {0.0f, 0.0f, 0.0f};  // dL/d(unit direction at the wall)
  if (S.adj_dL_ddir) {
#pragma unroll
    for (int a = 0; a < 3; ++a) ld[a] = gld(S.adj_dL_ddir + 3 * (size_t)r + a);
  }
  const bool seed = !(lu == 0.0f && lv == 0.0f) || !(ld[0] == 0.0f && ld[1] == 0.0f && ld[2] == 0.0f);
  R.active = R.n > 0 && !(st & (RAY_NO_WALL_HIT | RAY_NONFINITE | RAY_MISSED_BOX)) && seed;
  if (!R.active) return;
  float e_end[3], s;
  load_ray_header(S, R.q, R.B, e_end, s);
  float v[3], lX[3], vn = 0.0f, vl = 0.0f, v2 = 0.0f;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    v[a] = R.B.V[a] + e_end[a] * S.vox[a];
    lX[a] = lu * S.wall_u_f[a] + lv * S.wall_v_f[a];
    vn += v[a] * S.wall_n_f[a];
    vl += v[a] * lX[a];
    v2 += v[a] * v[a];
  }
  const float qv = vl / vn;
  // the direction v / |v| at the wall: its adjoint (ld - d (d . ld)) / |v| joins dL/dv
  const float inv_v = 1.0f / sqrtf(v2);
  const float dl = (v[0] * ld[0] + v[1] * ld[1] + v[2] * ld[2]) * inv_v;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float lx = lX[a] - S.wall_n_f[a] * qv;
    const float lvd = (ld[a] - v[a] * inv_v * dl) * inv_v;
    R.rb[a] = lx * S.vox[a];
    R.tb[a] = fmaf(lvd, S.vox[a], s * R.rb[a]);
  }
}

// Initial condition v0 = (1 + delta(x0)) dir: dL/d delta_c += w_c(x0) sum_a tb0_a dir_a /
// voxel_a, with tb0 = dL/dv0 in grid units and V = v0 (m per unit t). Contributions of
// lanes with `active`.
template <class Merge>
__device__ __forceinline__ void entry_term(const SceneDev& S, const RayBase& B, const float V[3], bool active,
                                           const float tb0[3], Merge& M, int lane) {
  int key0 = 0;
  float c0v[8];
  if (active) {
    Cell C0;
    locate3(S, B.U0hi, B.U0lo, C0);
    const float vn = sqrtf(V[0] * V[0] + V[1] * V[1] + V[2] * V[2]);
    float kap = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) kap = fmaf(tb0[a], (V[a] / vn) * dd_to_f(S.inv_vox[a]), kap);
    kap *= S.dec;  // the accumulators hold dec times the contributions
    // kap w_c(x0) as monomial coefficients: kap m(f)
    const float u = C0.f[0], v = C0.f[1], w = C0.f[2];
    c0v[0] = kap;
    c0v[1] = kap * u;
    c0v[2] = kap * v;
    c0v[3] = c0v[1] * v;
    c0v[4] = kap * w;
    c0v[5] = c0v[1] * w;
    c0v[6] = c0v[2] * w;
    c0v[7] = c0v[3] * w;
    key0 = (int)cell_index(S, C0);
  }
  M.enter(S, active, __ballot(active), key0, lane);
  if (active) {
#pragma unroll
    for (int k = 0; k < 8; ++k) M.acc[k] += c0v[k];
  }
}

// Reverse of one Sharma step for the state adjoints rb = dL/dd, tb = dL/de after it.
// The step (code-unit stage forces G_i at P_i, forward coefficients c_x, c_v, c_p2, c_p3)
//   P2 = x + h/2 e + c_p2 G1,  P3 = x + h e + c_p3 G2,
//   d' = x + h e + c_x (G1 + 2 G2),  e' = e + c_v (G1 + 4 G2 + G3)
// gives the force adjoints wC = dL/dG3 = c_v tb, wB = dL/dG2 = 2 c_x rb + 4 c_v tb +
// c_p3 p3, wA = dL/dG1 = c_x rb + c_v tb + c_p2 p2 (p_i = dL/dP_i from the stage's
// force_rev), and before the step rb + p3 + p2 + p1 and tb + h (rb + p3) + h/2 p2.
// stage_weights starts wA and wB from the step-end adjoints.
__device__ __forceinline__ void stage_weights(const SceneDev& S, const float rb[3], const float tb[3], float wA[3],
                                              float wB[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    wA[a] = fmaf(S.c_x[a], rb[a], S.c_v[a] * tb[a]);
    wB[a] = fmaf(S.c_x2[a], rb[a], S.c_v4[a] * tb[a]);
  }
}

// Stages C, B, A of the reverse (lanes with act), each sample's contributions into the
// accumulators of its cell; rb, tb become the adjoints before the step. The merge M takes
// the samples: M.enter(S, act, act_m, key, lane) when lanes with act (ballot act_m) come to
// a sample in cell `key`, then M.take(S, sample of the step, R, w, p) for its force_rev.
template <class Merge>
__device__ __forceinline__ void reverse_stages(const SceneDev& S, Merge& M, bool act,
                                               const SampleRev& R1, const SampleRev& R2, const SampleRev& R3,
                                               float wA[3], float wB[3], float rb[3], float tb[3], int lane) {
  float rs[3], ts[3];
  const unsigned long long act_m = __ballot(act);
  M.enter(S, act, act_m, act ? R3.key : 0, lane);
  if (act) {  // stage C
    float w[3], p[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) w[a] = S.c_v[a] * tb[a];
    M.take(S, 2, R3, w, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      rs[a] = rb[a] + p[a];
      ts[a] = fmaf(S.hf, rs[a], tb[a]);
      wB[a] = fmaf(S.c_p3[a], p[a], wB[a]);
    }
  }
  M.enter(S, act, act_m, act ? R2.key : 0, lane);
  if (act) {  // stage B
    float p[3];
    M.take(S, 1, R2, wB, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      rs[a] += p[a];
      ts[a] = fmaf(S.h_2, p[a], ts[a]);
      wA[a] = fmaf(S.c_p2[a], p[a], wA[a]);
    }
  }
  M.enter(S, act, act_m, act ? R1.key : 0, lane);
  if (act) {  // stage A
    float p[3];
    M.take(S, 0, R1, wA, p);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      rb[a] = rs[a] + p[a];
      tb[a] = ts[a];
    }
  }
}

// Quasi-linear form: the stage points lie on the entry line, at its half-step points
// j = 0 .. 2n (P(j) = U0 + j g2, g2 = V h / 2 in grid units), so the reverse needs no
// states. The state recursion is linear: with r = dL/dd and tau_k = dL/de after step k,
// r stays rb and tau_k = tb + (n - k) h rb. The force at P(j) gets the adjoint
//   even j = 2m: h (h/6 r + tau_{m+1}/6) [stage A of step m, m < n]
//                + h tau_m / 6 [stage C of step m - 1, m > 0]
//   odd  j = 2k + 1: h (h/3 r + 2/3 tau_{k+1}) [stage B of step k]
// and passes it to the 8 corner voxels and, through the point's dependence on the
// entry velocity, j h/2 times its position adjoint to dL/dv0. v = dL/dK; times S.km it is
// dL/dG, which the callers form once the point's gather is out. h and h/6 come from them too:
// read from the scene here, with km, they were six scalar loads and a wait in every point, ahead
// of its gather (1M rays: 2750 us against 2720).
__device__ __forceinline__ void ql_force_adjoint(const AdjRay& R, int j, float h, float h_6, float v[3]) {
  const int n = R.n, m = j >> 1;
  if ((j & 1) == 0) {
    const float ca = (float)(n - m - 1) * h, cc = (float)(n - m) * h;  // tau_{m+1}, tau_m
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float tA = fmaf(ca, R.rb[a], R.tb[a]), tC = fmaf(cc, R.rb[a], R.tb[a]);
      const float wa = m < n ? h * fmaf(h_6, R.rb[a], tA * (1.0f / 6.0f)) : 0.0f;
      const float wc = m > 0 ? h * (tC * (1.0f / 6.0f)) : 0.0f;
      v[a] = wa + wc;
    }
  } else {
    const float cb = (float)(n - m - 1) * h;  // tau_{m+1}
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const float tB = fmaf(cb, R.rb[a], R.tb[a]);
      v[a] = h * fmaf(h * (1.0f / 3.0f), R.rb[a], tB * (2.0f / 3.0f));
    }
  }
}

// Recorder of the replay: sample s of the step at row[s * 64].
struct SampleRow {
  f32x4* row;
  __device__ __forceinline__ void operator()(int stage, unsigned rec, const float f[3]) const {
    row[stage * 64] = f32x4{__uint_as_float(rec), f[0], f[1], f[2]};
  }
};

}  // namespace rbos
