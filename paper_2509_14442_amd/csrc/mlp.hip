// mlp.hip -- the network field of Sec. 2.D on the matrix cores: (T_nd, p, u) = MLP(xhat)
// with tanh hidden layers of 64 units, its parameter gradient for any loss given per
// point as dL/d(outputs), and the chain from dL/d(eta - 1) on the voxel grid to
// dL/dT_nd (eta - 1 = rho0 G T0 / T, T = T0 + (T_in - T0) T_nd).
//
// The 64 x 64 layers are v_mfma_f32_32x32x2f32 products (FP32 inputs and accumulation).
// The forward runs all layers of 32 points in one wavefront, the activations staying in
// registers between layers (k_mlp_forward_fused), the backward all layers of 128 points in one
// block, delta and the parameter gradient staying in registers (k_mlp_backward_fused). The
// jets of the PDE loss run layer by layer (k_jet_*, k_mlp_wgrad). Every sum over points runs
// over a fixed range per block, and a second kernel adds the blocks in order, so results do
// not depend on scheduling.
#include <hip/hip_runtime.h>

#include <atomic>

#include "mlp_launch.hpp"

namespace rbos {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// tanh x = 1 - 2 / (exp(2x) + 1), with the hardware base-2 exponential (2x / ln 2) and
// reciprocal: absolute error ~1e-7, saturating to +-1 for large |x|. The library tanhf
// costs more VALU cycles than a layer's matrix products.
__device__ __forceinline__ float tanh_fast(float x) {
  const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);
  return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e + 1.0f);
}

// Row of the 32 x 32 accumulator held in register r of a lane in half h (its column is
// the lane index mod 32).
__device__ __forceinline__ int acc_row(int r, int h) { return 8 * (r >> 2) + 4 * h + (r & 3); }

// normalised input of point p
__device__ __forceinline__ void xhat(const MlpDev& M, long long p, float x[3]) {
  if (M.points) {
#pragma unroll
    for (int a = 0; a < 3; ++a) x[a] = fmaf(M.points[3 * p + a], M.xs[a], M.xo[a]);
  } else {
    const long long q = p / M.nx;
    const int i = (int)(p - q * M.nx);
    const int j = (int)(q % M.ny);
    const int k = (int)(q / M.ny);
    x[0] = (float)(2 * i + 1) / (float)M.nx - 1.0f;
    x[1] = (float)(2 * j + 1) / (float)M.ny - 1.0f;
    x[2] = (float)(2 * k + 1) / (float)M.nz - 1.0f;
  }
}

// Fused forward: every layer of 32 points per wavefront, the activations kept in
// registers from layer to layer (each layer's are still written out for the backward
// pass). The hidden layers run transposed, C^T = W^T A^T (units as rows, points as
// columns), so that one layer's accumulators are the next layer's B operand as they
// stand: register r of the unit tile t in a lane of half h holds unit 32 t + acc_row(r, h)
// of point lane % 32, and step s = 16 t + r of the next product takes, in half h, that
// register with the weight W[32 t + acc_row(r, h)][unit] as the A operand (the two
// halves supply the two K values of the step). The block stages all weights in LDS once
// and its wavefronts loop over groups of 32 points.
constexpr int FUSED_PITCH = 72;  // LDS row pitch of a staged 64 x 64 weight matrix

__host__ __device__ constexpr int fused_lds_floats(int depth) {
  return (depth - 1) * MLP_WIDTH * FUSED_PITCH + depth * MLP_WIDTH + 3 * MLP_WIDTH + MLP_WIDTH * MLP_OUT + 8;
}

__global__ __launch_bounds__(256) void k_mlp_forward_fused(MlpDev M, float* __restrict__ act, float* __restrict__ xh,
                                                           float* __restrict__ wt, float* __restrict__ out,
                                                           float* __restrict__ T, float T0, float dT, int nblk) {
  extern __shared__ float lds[];
  const int D = M.depth;
  // W_l^T of the hidden layers for the backward pass, a layer per block. Blocks past the first
  // nblk, if the grid has any, take no points.
  const bool spare = nblk < (int)gridDim.x;
  if (!spare || (int)blockIdx.x >= nblk) {
    const int step = spare ? (int)gridDim.x - nblk : nblk;
    for (int l = 1 + (spare ? (int)blockIdx.x - nblk : (int)blockIdx.x); l < D; l += step)
      for (int e = threadIdx.x; e < MLP_WIDTH * MLP_WIDTH; e += 256)
        wt[(l - 1) * MLP_WIDTH * MLP_WIDTH + e] =
            M.params[M.off_w[l] + (e & (MLP_WIDTH - 1)) * MLP_WIDTH + (e / MLP_WIDTH)];
    if (spare) return;
  }
  float* Wh = lds;                                         // W_1 .. W_{D-1}, rows padded
  float* bh = Wh + (D - 1) * MLP_WIDTH * FUSED_PITCH;      // b_0 .. b_{D-1}
  float* W0 = bh + D * MLP_WIDTH;                          // [3][64]
  float* WD = W0 + 3 * MLP_WIDTH;                          // [64][5]
  float* bD = WD + MLP_WIDTH * MLP_OUT;                    // [5]
  const float* P = M.params;
  for (int e = threadIdx.x; e < (D - 1) * MLP_WIDTH * MLP_WIDTH; e += 256) {
    const int l = e / (MLP_WIDTH * MLP_WIDTH), k = (e / MLP_WIDTH) % MLP_WIDTH, u = e % MLP_WIDTH;
    Wh[(l * MLP_WIDTH + k) * FUSED_PITCH + u] = P[M.off_w[l + 1] + k * MLP_WIDTH + u];
  }
  for (int e = threadIdx.x; e < D * MLP_WIDTH; e += 256) bh[e] = P[M.off_b[e / MLP_WIDTH] + e % MLP_WIDTH];
  for (int e = threadIdx.x; e < 3 * MLP_WIDTH; e += 256) W0[e] = P[M.off_w[0] + e];
  for (int e = threadIdx.x; e < MLP_WIDTH * MLP_OUT; e += 256) WD[e] = P[M.off_w[D] + e];
  if (threadIdx.x < MLP_OUT) bD[threadIdx.x] = P[M.off_b[D] + threadIdx.x];
  __syncthreads();

  const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
  const long long n = M.n;
  const long long stride = (long long)nblk * 4;
  for (long long g = (long long)blockIdx.x * 4 + (threadIdx.x >> 6); g * 32 < n; g += stride) {
    const long long p = g * 32 + c;
    const bool valid = p < n;
    float x[3] = {0.0f, 0.0f, 0.0f};
    if (valid) xhat(M, p, x);
    if (valid && h == 0) *reinterpret_cast<f32x4*>(xh + p * 4) = f32x4{x[0], x[1], x[2], 0.0f};
    // a[16 t + r]: unit 32 t + acc_row(r, h) of point p
    float a[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      const int u = 32 * (i >> 4) + acc_row(i & 15, h);
      float z = bh[u];
#pragma unroll
      for (int d = 0; d < 3; ++d) z = fmaf(x[d], W0[d * MLP_WIDTH + u], z);
      a[i] = tanh_fast(z);
    }
    for (int l = 0; l < D; ++l) {
      if (l > 0) {
        const float* W = Wh + (l - 1) * MLP_WIDTH * FUSED_PITCH;
        f32x16 acc0 = {}, acc1 = {};
#pragma unroll
        for (int s = 0; s < 32; ++s) {
          const float* w = W + (32 * (s >> 4) + acc_row(s & 15, h)) * FUSED_PITCH;
          acc0 = mfma32(w[c], a[s], acc0);
          acc1 = mfma32(w[32 + c], a[s], acc1);
        }
        const float* b = bh + l * MLP_WIDTH;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          a[r] = tanh_fast(acc0[r] + b[acc_row(r, h)]);
          a[16 + r] = tanh_fast(acc1[r] + b[32 + acc_row(r, h)]);
        }
      }
      if (valid) {  // a_{l+1} [n][64]: units 32 t + 8 j + 4 h .. +3 are a[16 t + 4 j .. +3]
        float* dst = act + (size_t)l * (size_t)n * MLP_WIDTH + p * MLP_WIDTH + 4 * h;
#pragma unroll
        for (int q = 0; q < 8; ++q)
          *reinterpret_cast<f32x4*>(dst + 32 * (q >> 2) + 8 * (q & 3)) =
              f32x4{a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]};
      }
    }
    if (out || T) {
      float z[MLP_OUT];
#pragma unroll
      for (int o = 0; o < MLP_OUT; ++o) z[o] = 0.0f;
#pragma unroll
      for (int i = 0; i < 32; ++i) {
        const int u = 32 * (i >> 4) + acc_row(i & 15, h);
#pragma unroll
        for (int o = 0; o < MLP_OUT; ++o) z[o] = fmaf(a[i], WD[u * MLP_OUT + o], z[o]);
      }
#pragma unroll
      for (int o = 0; o < MLP_OUT; ++o) {  // the two halves hold the point's two unit sets
        auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(z[o]), __float_as_uint(z[o]), false, false);
        z[o] = (__uint_as_float(sw[0]) + __uint_as_float(sw[1])) + bD[o];
      }
      if (valid && h == 0) {
        if (out)
#pragma unroll
          for (int o = 0; o < MLP_OUT; ++o) out[p * MLP_OUT + o] = z[o];
        if (T) T[p] = fmaf(dT, z[0], T0);
      }
    }
  }
}

// WT_l = W_l^T for the hidden layers l = 1 .. depth - 1
__global__ __launch_bounds__(256) void k_mlp_transpose(MlpDev M, float* __restrict__ wt) {
  const int idx = blockIdx.x * 256 + threadIdx.x;
  const int l = 1 + idx / (MLP_WIDTH * MLP_WIDTH);
  if (l >= M.depth) return;
  const int e = idx % (MLP_WIDTH * MLP_WIDTH), k = e / MLP_WIDTH, j = e % MLP_WIDTH;
  wt[(l - 1) * MLP_WIDTH * MLP_WIDTH + j * MLP_WIDTH + k] = M.params[M.off_w[l] + k * MLP_WIDTH + j];
}

// Partial parameter gradient of one layer over this block's rows:
// P[m][j] = sum_i A[i][m] B[i][j] (m < 64, j < 64) and P[4096 + j] = sum_{i < bias_rows} B[i][j].
// A: the layer's input (XHAT: the first layer's, rows i < M.n the normalised position of
// point i from xh [n][4], rows i = (1 + a) M.n + p the unit vector e_a (the input's
// derivative along a in a jet); else a [nrows][64]); B: the gradient at its output, ldb
// columns of which nb are used. Four wavefronts per block: each 64-row chunk of A and B
// is staged in LDS with coalesced loads, and wavefront (mt, nt) accumulates the 32 x 32
// tile P[32 mt ..][32 nt ..] with the rows along K.
// With PROD, the same staged chunk also gives the gradient one layer down, written to
// Cout [nrows][64]: Cout = B WT (WT = W^T as 64 x 64). Wavefront (mt, nt) computes its rows
// 32 mt .. and units 32 nt .., so A and B are read from HBM once for both products.
template <bool XHAT, bool PROD>
__global__ __launch_bounds__(256) void k_mlp_wgrad(MlpDev M, const float* __restrict__ A, const float* __restrict__ B,
                                                   int ldb, int nb, float* __restrict__ partial,
                                                   long long rows_per_block, long long nrows, long long bias_rows,
                                                   const float* __restrict__ WT = nullptr,
                                                   float* __restrict__ Cout = nullptr) {
  __shared__ float As[64 * 65];
  __shared__ float Bs[64 * 65];
  __shared__ float Ws[PROD ? 64 * 65 : 1];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if constexpr (PROD) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int e = t + 256 * i;
      Ws[(e >> 6) * 65 + (e & 63)] = WT[e];
    }
  }
  const int mt = wave >> 1, nt = wave & 1;
  const int c = lane & 31, h = lane >> 5;
  const long long r0 = (long long)blockIdx.x * rows_per_block;
  const long long r1 = r0 + rows_per_block < nrows ? r0 + rows_per_block : nrows;
  f32x16 acc = {};
  float bsum = 0.0f;
  // chunk elements e = t + 256 i (row e / 64, column e % 64), loaded one chunk ahead
  float av[16], bv[16];
  auto load_chunk = [&](long long base) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int e = t + 256 * i, col = e & 63;
      const long long row = base + (e >> 6);
      av[i] = 0.0f;
      bv[i] = 0.0f;
      if (row < r1) {
        if constexpr (XHAT) {
          if (col < 3) av[i] = row < M.n ? A[row * 4 + col] : (col == (int)(row / M.n) - 1 ? 1.0f : 0.0f);
        } else {
          av[i] = A[row * MLP_WIDTH + col];
        }
        if (col < nb) bv[i] = B[row * ldb + col];
      }
    }
  };
  if (r0 < r1) load_chunk(r0);
  for (long long base = r0; base < r1; base += 64) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int e = t + 256 * i;
      As[(e >> 6) * 65 + (e & 63)] = av[i];
      Bs[(e >> 6) * 65 + (e & 63)] = bv[i];
    }
    __syncthreads();
    if (base + 64 < r1) load_chunk(base + 64);  // in flight during this chunk's products
#pragma unroll 8
    for (int s = 0; s < 32; ++s) {
      const int rr = 32 * h + s;
      const float bvv = Bs[rr * 65 + 32 * nt + c];
      acc = mfma32(As[rr * 65 + 32 * mt + c], bvv, acc);
      if (mt == 0 && base + rr < bias_rows) bsum += bvv;
    }
    if constexpr (PROD) {
      // rows 32 mt + acc_row(r, h), units 32 nt + c of B WT; K = the 64 columns of B,
      // lane half h supplying k = 32 h + s at step s
      f32x16 d = {};
#pragma unroll 8
      for (int s = 0; s < 32; ++s) {
        const int k = 32 * h + s;
        d = mfma32(Bs[(32 * mt + c) * 65 + k], Ws[k * 65 + 32 * nt + c], d);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rr = 32 * mt + acc_row(r, h);
        if (base + rr < r1) {
          Cout[(base + rr) * MLP_WIDTH + 32 * nt + c] = d[r];
        }
      }
    }
    __syncthreads();
  }
  float* P = partial + (long long)blockIdx.x * MLP_PART;
#pragma unroll
  for (int r = 0; r < 16; ++r) P[(32 * mt + acc_row(r, h)) * MLP_WIDTH + 32 * nt + c] = acc[r];
  const float other = __shfl_xor(bsum, 32);
  if (mt == 0 && h == 0) P[MLP_WIDTH * MLP_WIDTH + 32 * nt + c] = bsum + other;
}

// Fused backward: every layer of a chunk of 128 points in one block, the parameter gradient
// of every layer accumulated in registers over the block's chunks, so that the activations
// are read once and nothing else of the size of the point set is touched (a kernel per layer
// also wrote and read back each delta, 2 x 512 MB per layer at 2M points, and ran the output
// layer's 5 columns as 64).
//
// Four wavefronts carry delta_l = (delta_{l+1} W_l^T)(1 - a_l^2) down the layers, 32 points
// each, transposed as in the forward (units as rows, points as columns: the accumulators of
// one product are the B operand of the next; the rows of W_l^T, read through the vector L1,
// which holds a layer's 16 KB, are the A operand). Four others form dW_l = a_l^T delta_{l+1},
// the points along K: delta passes through LDS, [point][unit], and wavefront (mt, nt)
// accumulates the 32 x 32 tile dW_l[32 mt ..][32 nt ..] over all 128 points, a_l's rows read
// straight from memory as the A operand. Both sides take 64 products of 64 cycles per layer
// and chunk, and each SIMD holds one of each, so that one side's loads, tanh derivatives and
// LDS traffic run beside the other's products (with both products in four wavefronts of 512
// registers: 1873 us at 2M points and depth 4). The output layer (5 columns) and the first
// one (3 rows and the bias) take 16 x 16 x 4 tiles, 16 units per wavefront.
//
// Bound: the products, 0.66 ms at 2M points and depth 4; measured 1.34 ms there (a kernel per
// layer: 2.18 ms), 34 us at 4096 points (66 us), 2.60 ms at depth 8 (3.98 ms).
constexpr int BWD_POINTS = 128;  // points per chunk
constexpr int BWD_PITCH = 68;    // LDS row pitch of a delta chunk

__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// *(base + imm bytes) at a lane's byte offset, in the form the load instruction takes: a
// uniform base, one offset register for every load, and an immediate.
__device__ __forceinline__ float load_at(const float* base, unsigned lane_bytes, int imm) {
  return *(const __attribute__((address_space(1))) float*)(reinterpret_cast<const char*>(base) + (size_t)lane_bytes +
                                                           imm);
}

// 0, as a value the compiler cannot see through: loads addressed with it stay where they are
// written. Moved up to the layers before, or (the weights) out of the chunk loop, they took
// several times the registers there are.
__device__ __forceinline__ int here() {
  int zero = 0;
  asm volatile("" : "+s"(zero));
  return zero;
}

// What both sides know of the point set and of the chunk at hand.
struct BackwardSet {
  const MlpDev& M;
  const float *act, *xh, *dL, *wt;
  float* Ds;       // LDS: two delta chunks, taken in turn
  float* Xs;       // LDS: two chunks of [point][8], dL (5) and the normalised input (3), taken in turn
  int lane, wave;  // wave 0 .. 3 of its side
  long long base;  // first point of the chunk
  int rows;        // its points

  __device__ __forceinline__ const float* layer(int l) const {  // a_l of the chunk
    return act + ((size_t)(l - 1) * (size_t)M.n + (size_t)base) * MLP_WIDTH;
  }
  __device__ __forceinline__ float* delta(int buf) const { return Ds + (buf & 1) * (BWD_POINTS * BWD_PITCH); }
  __device__ __forceinline__ float* ends(int chunk) const { return Xs + (chunk & 1) * (BWD_POINTS * 8); }
};

// The side that carries delta down the layers.
template <int D>
struct DeltaSide : BackwardSet {
  int c, h;
  float wD[2][3];  // the output layer's weights as A operand: row (unit) 32 u + c, K = 2 s + h
  float dl[32];    // delta_{l+1}: unit 32 t + acc_row(r, h) of point 32 wave + c at [16 t + r]
  // Loaded ahead, past the barrier between two layers: loads return in order, and the first of
  // a layer to come from HBM would hold up all its products.
  f32x4 y[2][8];   // a_l of the lane's point, in dl's order, at [(D - l) & 1]
  float vw[3][8];  // weights of a layer's step groups, see slot
  float seed[3];   // dL of the lane's point, outputs 2 s + h
  f32x4 x;         // its normalised input

  __device__ __forceinline__ explicit DeltaSide(const BackwardSet& s) : BackwardSet(s), c(s.lane & 31), h(s.lane >> 5) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        wD[u][k] = 2 * k + h < MLP_OUT ? M.params[M.off_w[D] + (32 * u + c) * MLP_OUT + 2 * k + h] : 0.0f;
  }

  // a_l of the lane's point of a chunk (the chunk's last point past its end)
  template <int l>
  __device__ __forceinline__ void load_own(const float* a, int n_rows) {
    const float* q = a + here() + (min(32 * wave + c, n_rows - 1) * MLP_WIDTH + 4 * h);
    const f32x4* v = reinterpret_cast<const f32x4*>(q);
#pragma unroll
    for (int i = 0; i < 8; ++i) y[(D - l) & 1][i] = v[8 * (i >> 2) + 2 * (i & 3)];
  }

  // dL and the input of the lane's point of a chunk
  __device__ __forceinline__ void load_ends(long long chunk, int n_rows) {
    const long long p = chunk + min(32 * wave + c, n_rows - 1);
#pragma unroll
    for (int s = 0; s < 3; ++s) seed[s] = dL[p * MLP_OUT + (2 * s + h < MLP_OUT ? 2 * s + h : 0)];
    x = *reinterpret_cast<const f32x4*>(xh + p * 4);
  }

  // Buffer of step group g (0 .. 7) of layer l: the groups take the three in turn, through the
  // layers.
  template <int l>
  static constexpr __device__ int slot(int g) { return (2 * (D - 1 - l) + g) % 3; }

  // step group g of layer l: rows acc_row(s & 15, h) of W_l^T for the steps s = 4 g ..
  template <int l>
  __device__ __forceinline__ void load_group(int g) {
    const float* w = wt + (size_t)(l - 1) * MLP_WIDTH * MLP_WIDTH + here();
    unsigned ow = 4u * (unsigned)((32 * (g >> 2) + 8 * (g & 3) + 4 * h) * MLP_WIDTH + c);
    asm volatile("" : "+v"(ow));  // one register, not an address per load
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      vw[slot<l>(g)][2 * i] = load_at(w, ow, 256 * i);
      vw[slot<l>(g)][2 * i + 1] = load_at(w, ow, 256 * i + 128);
    }
  }

  template <int l>
  __device__ __forceinline__ void times_dtanh(const f32x16& acc0, const f32x16& acc1) {
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      const float v = y[(D - l) & 1][i >> 2][i & 3], d = i < 16 ? acc0[i & 15] : acc1[i & 15];
      dl[i] = d * (1.0f - v * v);
    }
  }

  // delta_D, and dL and the input to the other side (0 past the end)
  __device__ __forceinline__ void output_layer(int chunk) {
    const bool in = 32 * wave + c < rows;
    float* X = ends(chunk) + (32 * wave + c) * 8;
    f32x16 acc0 = {}, acc1 = {};
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      const float g = in && 2 * s + h < MLP_OUT ? seed[s] : 0.0f;
      acc0 = mfma32(wD[0][s], g, acc0);
      acc1 = mfma32(wD[1][s], g, acc1);
      if (2 * s + h < MLP_OUT) X[2 * s + h] = g;
    }
    if (h == 1) {
#pragma unroll
      for (int a = 0; a < 3; ++a) X[MLP_OUT + a] = in ? x[a] : 0.0f;
    }
    if constexpr (D > 1) {
      load_own<D - 1>(layer(D - 1), rows);
      load_group<D - 1>(0);
      load_group<D - 1>(1);
    }
    times_dtanh<D>(acc0, acc1);
  }

  // Layers l .. 1, then the next chunk's loads. A buffer of the delta is written again two
  // barriers on, when the other side has read it.
  template <int l>
  __device__ __forceinline__ void layers_from(int buf, long long next, int next_rows) {
    float* Dc = delta(buf);
#pragma unroll
    for (int q = 0; q < 8; ++q)
      *reinterpret_cast<f32x4*>(Dc + (32 * wave + c) * BWD_PITCH + 32 * (q >> 2) + 8 * (q & 3) + 4 * h) =
          f32x4{dl[4 * q], dl[4 * q + 1], dl[4 * q + 2], dl[4 * q + 3]};
    if constexpr (l == 0) {
      base = next;
      rows = next_rows;
      if (rows > 0) {
        load_own<D>(layer(D), rows);
        if (D == 1) load_ends(base, rows);
      }
      __syncthreads();
    } else {
      constexpr int below = l > 1 ? l - 1 : 1;
      __syncthreads();
      f32x16 acc0 = {}, acc1 = {};
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        __builtin_amdgcn_sched_barrier(0);  // no loads from further ahead
        if (g + 2 < 8) load_group<l>(g + 2);
        else if (l > 1) load_group<below>(g - 6);
        if (g == 5 && l > 1) load_own<below>(layer(below), rows);
        if (g == 5 && l == 1 && next_rows > 0) load_ends(next, next_rows);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc0 = mfma32(vw[slot<l>(g)][2 * i], dl[4 * g + i], acc0);
          acc1 = mfma32(vw[slot<l>(g)][2 * i + 1], dl[4 * g + i], acc1);
        }
      }
      times_dtanh<l>(acc0, acc1);
      layers_from<l - 1>(buf + 1, next, next_rows);
    }
  }
};

// The side that forms the parameter gradient. Operands over the points are 0 past the end.
// (The loads behind them run up to BWD_POINTS - 1 rows past a layer: the next layers, and ACT_TAIL
// rows that the workspace holds past the last one.)
template <int D>
struct GradSide : BackwardSet {
  int c, h, c4, k4, mt, nt;
  f32x16 dW[D > 1 ? D - 1 : 1] = {};  // hidden layers l = 1 .. D - 1 at [l - 1]
  float db[D > 1 ? D - 1 : 1] = {};
  f32x4 dWout = {}, dWin = {};
  float dbout = 0.0f;
  float va[3][8];  // rows of a layer's step groups, see slot

  __device__ __forceinline__ explicit GradSide(const BackwardSet& s)
      : BackwardSet(s), c(s.lane & 31), h(s.lane >> 5), c4(s.lane & 15), k4(s.lane >> 4), mt(s.wave >> 1),
        nt(s.wave & 1) {}

  // Buffer of a step group: the output layer's four, then eight per hidden layer, take the
  // three in turn.
  template <int l>
  static constexpr __device__ int slot(int g) { return l == D ? g % 3 : (4 + 8 * (D - 1 - l) + g) % 3; }

  // step group g of layer l: points 16 g ..
  template <int l>
  __device__ __forceinline__ void load_group(int g) {
    const float* a = layer(l) + here();
    unsigned oa = 4u * (unsigned)((16 * g + h) * MLP_WIDTH + 32 * mt + c);
    asm volatile("" : "+v"(oa));
#pragma unroll
    for (int i = 0; i < 8; ++i) va[slot<l>(g)][i] = load_at(a, oa, 512 * i);
  }

  // step group q (0 .. 3) of the output layer: points 32 q .., 4 per step
  __device__ __forceinline__ void load_output_group(int q) {
    const float* a = layer(D) + here();
    unsigned oa = 4u * (unsigned)((32 * q + k4) * MLP_WIDTH + 16 * wave + c4);
    asm volatile("" : "+v"(oa));
#pragma unroll
    for (int i = 0; i < 8; ++i) va[slot<D>(q)][i] = load_at(a, oa, 1024 * i);
  }

  // Bring a chunk's 32 KB of a_l into the L2 (a line per lane), for a later layer's loads.
  float touched = 0.0f;
  __device__ __forceinline__ void touch(int l, long long chunk, int n_rows) {
    asm volatile("" ::"v"(touched));  // the last one has arrived
    const int p = min((64 * wave + lane) >> 1, n_rows - 1);
    touched = act[((size_t)(l - 1) * (size_t)M.n + (size_t)(chunk + p)) * MLP_WIDTH + 32 * (lane & 1) + here()];
  }

  // dW_D: columns o, K = the points, units 16 wave ..
  __device__ __forceinline__ void output_layer(int chunk) {
    const float* X = ends(chunk) + (k4 * 8 + (c4 < MLP_OUT ? c4 : 0));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      __builtin_amdgcn_sched_barrier(0);
      if (q + 2 < 4) load_output_group(q + 2);
      else if (D > 1) load_group<(D > 1 ? D - 1 : 1)>(q - 2);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float gp = X[(32 * q + 4 * i) * 8];
        const float g = c4 < MLP_OUT ? gp : 0.0f;
        dWout = mfma16(32 * q + 4 * i + k4 < rows ? va[slot<D>(q)][i] : 0.0f, g, dWout);
        dbout += g;
      }
      asm volatile("" : "+v"(dWout), "+v"(dbout));
    }
  }

  template <int l>
  __device__ __forceinline__ void layers_from(int buf, int chunk, long long next, int next_rows) {
    const float* Dc = delta(buf);
    __syncthreads();
    if constexpr (l == D - 1) output_layer(chunk);
    if constexpr (l == 0) {
      const float* X = ends(chunk) + (k4 * 8 + MLP_OUT + (c4 < 3 ? c4 : 0));
      const float* Dp = Dc + (k4 * BWD_PITCH + 16 * wave + c4);
      if (next_rows > 0) {
        base = next;
        load_output_group(0);
        load_output_group(1);
      }
      // dW_0 (columns 0 .. 2) and db_0 (column 3): rows (units) 16 wave ..
#pragma unroll
      for (int s = 0; s < BWD_POINTS / 4; ++s) {
        if (s % 8 == 0) __builtin_amdgcn_sched_barrier(0);
        const float xp = X[4 * s * 8];
        const float v = c4 < 3 ? xp : c4 == 3 ? 1.0f : 0.0f;
        dWin = mfma16(Dp[4 * s * BWD_PITCH], v, dWin);
      }
      asm volatile("" : "+v"(dWin));
      rows = next_rows;
    } else {
      constexpr int below = l > 1 ? l - 1 : 1;
      const float* Dp = Dc + h * BWD_PITCH + 32 * nt + c;
      float vb[2][8];
      auto load_delta = [&](int g) {
#pragma unroll
        for (int i = 0; i < 8; ++i) vb[g & 1][i] = Dp[(16 * g + 2 * i) * BWD_PITCH];
      };
      load_delta(0);
#pragma unroll
      for (int g = 0; g < 8; ++g) {
        __builtin_amdgcn_sched_barrier(0);
        if (g + 2 < 8) load_group<l>(g + 2);
        else if (l > 1) load_group<below>(g - 6);
        if (g == 5) {  // two layers on: l - 2, or the next chunk's D and D - 1
          if (l > 2) touch(l - 2, base, rows);
          else if (next_rows > 0 && (l == 2 || D == 2)) touch(D, next, next_rows);
          else if (next_rows > 0) touch(D - 1, next, next_rows);
        }
        if (g + 1 < 8) load_delta(g + 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float b = vb[g & 1][i];
          // past the end the delta is 0: only what is not a number has to go
          dW[l - 1] = mfma32(__builtin_amdgcn_fmed3f(va[slot<l>(g)][i], -1.0f, 1.0f), b, dW[l - 1]);
          db[l - 1] += b;
        }
      }
      // computed here: the compiler put products and sums off to the end of the chunk, with
      // every operand held
      asm volatile("" : "+v"(dW[l - 1]), "+v"(db[l - 1]));
      layers_from<l - 1>(buf + 1, chunk, next, next_rows);
    }
  }

  __device__ __forceinline__ void store(float* partial, int nblk) {
    auto part = [&](int l) { return partial + ((size_t)l * nblk + blockIdx.x) * MLP_PART; };
#pragma unroll
    for (int l = 1; l < D; ++l) {
      float* P = part(l);
#pragma unroll
      for (int r = 0; r < 16; ++r) P[(32 * mt + acc_row(r, h)) * MLP_WIDTH + 32 * nt + c] = dW[l - 1][r];
      const float sum = db[l - 1] + __shfl_xor(db[l - 1], 32);
      if (mt == 0 && h == 0) P[MLP_WIDTH * MLP_WIDTH + 32 * nt + c] = sum;
    }
    dbout += __shfl_xor(dbout, 16);
    dbout += __shfl_xor(dbout, 32);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = 16 * wave + 4 * k4 + r;
      if (c4 < MLP_OUT) part(D)[u * MLP_WIDTH + c4] = dWout[r];
      if (c4 < 3) part(0)[c4 * MLP_WIDTH + u] = dWin[r];
      if (c4 == 3) part(0)[MLP_WIDTH * MLP_WIDTH + u] = dWin[r];
    }
    if (wave == 0 && k4 == 0 && c4 < MLP_OUT) part(D)[MLP_WIDTH * MLP_WIDTH + c4] = dbout;
  }
};

template <int D>
__global__ __launch_bounds__(512, 2) void k_mlp_backward_fused(MlpDev M, const float* __restrict__ act,
                                                               const float* __restrict__ xh,
                                                               const float* __restrict__ dL,
                                                               const float* __restrict__ wt,
                                                               float* __restrict__ partial, int nblk,
                                                               long long rows_per_block) {
  __shared__ __align__(16) float Ds[2 * BWD_POINTS * BWD_PITCH];
  __shared__ float Xs[2 * BWD_POINTS * 8];
  // the wavefront's index as a scalar, so that the two sides are branches and not lane masks
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long r0 = (long long)blockIdx.x * rows_per_block;
  const long long r1 = r0 + rows_per_block < M.n ? r0 + rows_per_block : M.n;
  auto rows_at = [&](long long b) { return (int)(r1 - b < BWD_POINTS ? r1 - b : BWD_POINTS); };
  const BackwardSet set{M, act, xh, dL, wt, Ds, Xs, (int)(threadIdx.x & 63), wave & 3, r0, rows_at(r0)};
  // D barriers per chunk on both sides
  int chunk = 0, buf = 0;
  if (wave < 4) {
    DeltaSide<D> side(set);
    side.template load_own<D>(side.layer(D), side.rows);
    side.load_ends(r0, side.rows);
#pragma unroll 1
    for (long long b = r0; b < r1; b += BWD_POINTS) {
      side.output_layer(chunk);
      side.template layers_from<D - 1>(buf, b + BWD_POINTS, rows_at(b + BWD_POINTS));
      buf += D;
      ++chunk;
    }
  } else {
    GradSide<D> side(set);
    side.load_output_group(0);
    side.load_output_group(1);
#pragma unroll 1
    for (long long b = r0; b < r1; b += BWD_POINTS) {
      side.template layers_from<D - 1>(buf, chunk, b + BWD_POINTS, rows_at(b + BWD_POINTS));
      buf += D;
      ++chunk;
    }
    side.store(partial, nblk);
  }
}

// dparams += sum over blocks of the partials, all layers in one launch (the packed order: W
// [fi][fo], b [fo] per layer). A block takes 16 parameters; its 16 thread groups sum the
// blocks b = g, g + 16, ..., and the groups are added in a fixed order, so the result does
// not depend on scheduling.
__global__ __launch_bounds__(256) void k_mlp_reduce(MlpDev M, const float* __restrict__ partial, int nblk,
                                                    float* __restrict__ dparams) {
  __shared__ float red[16][17];
  const int el = threadIdx.x & 15, g = threadIdx.x >> 4;
  const int e = blockIdx.x * 16 + el;
  const int total = M.off_b[M.depth] + MLP_OUT;
  float s = 0.0f;
  if (e < total) {
    int l = 0;
    while (l < M.depth && e >= M.off_w[l + 1]) ++l;
    const int fo = l == M.depth ? MLP_OUT : MLP_WIDTH, i = e - M.off_w[l];
    const int src = e < M.off_b[l] ? (i / fo) * MLP_WIDTH + i % fo : MLP_WIDTH * MLP_WIDTH + (e - M.off_b[l]);
    const float* P = partial + (size_t)l * nblk * MLP_PART + src;
#pragma unroll 8
    for (int b = g; b < nblk; b += 16) s += P[(size_t)b * MLP_PART];
  }
  red[g][el] = s;
  __syncthreads();
  if (g == 0 && e < total) {
    float t = red[0][el];
#pragma unroll
    for (int k = 1; k < 16; ++k) t += red[k][el];
    dparams[e] += t;
  }
}

__global__ __launch_bounds__(256) void k_mlp_bos_seed(long long n, const float* __restrict__ T,
                                                      const double* __restrict__ grad, double k, float* __restrict__ dL) {
  const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  if (p >= n) return;
  const double t = (double)T[p];
  dL[p * MLP_OUT] = (float)(grad[p] * (k / (t * t)));
#pragma unroll
  for (int o = 1; o < MLP_OUT; ++o) dL[p * MLP_OUT + o] = 0.0f;
}

// ------------------------------------------------------------------------------------
// Jets for the PDE residuals: per point 7 channels of every layer's activations, the
// value (c = 0), its derivative along xhat_d (c = 1 + d) and its second derivative along
// xhat_d (c = 4 + d), stored channel-major ([7][n][64]). A linear layer maps every
// channel by the same weights (the bias enters the value only); tanh maps
// (z, z_d, z_dd) to (y, t z_d, t z_dd - 2 y t z_d^2) with y = tanh z, t = 1 - y^2.
// ------------------------------------------------------------------------------------
constexpr int JET = 7;

// first layer: the input's jet is (xhat, e_d, 0); xh [n][4] as in k_mlp_forward_fused
__global__ __launch_bounds__(256) void k_jet_first(MlpDev M, float* __restrict__ aj, float* __restrict__ zj,
                                                   float* __restrict__ xh) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long p = idx >> 6;
  const int j = (int)(idx & 63);
  const long long n = M.n;
  if (p >= n) return;
  float x[3];
  xhat(M, p, x);
  if (j < 4) xh[p * 4 + j] = j < 3 ? x[j] : 0.0f;
  const float* W = M.params + M.off_w[0];
  float z = M.params[M.off_b[0] + j];
#pragma unroll
  for (int a = 0; a < 3; ++a) z = fmaf(x[a], W[a * MLP_WIDTH + j], z);
  const float y = tanh_fast(z), t = 1.0f - y * y;
  const long long e = p * MLP_WIDTH + j, ch = n * MLP_WIDTH;
  aj[e] = y;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float zd = W[d * MLP_WIDTH + j];
    aj[(1 + d) * ch + e] = t * zd;
    aj[(4 + d) * ch + e] = -2.0f * y * t * zd * zd;
    zj[d * ch + e] = zd;
    zj[(3 + d) * ch + e] = 0.0f;
  }
}

// a hidden layer on the jets: one wavefront per 32 points and direction d = blockIdx.y
// (channels 0, 1 + d, 4 + d); the value channel is written by the d = 0 wavefronts
__global__ __launch_bounds__(256) void k_jet_dense(long long n, const float* __restrict__ aj,
                                                   const float* __restrict__ W, const float* __restrict__ bias,
                                                   float* __restrict__ aj_next, float* __restrict__ zj_next) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const long long row0 = ((long long)blockIdx.x * 4 + wave) * 32;
  if (row0 >= n) return;
  const int d = blockIdx.y;
  const int c = lane & 31, h = lane >> 5;
  const long long row = row0 + c, ch = n * MLP_WIDTH;
  const int chans[3] = {0, 1 + d, 4 + d};
  f32x16 acc[3][2];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    acc[q][0] = acc[q][1] = f32x16{};
    float a[32];
    if (row < n) {
      const f32x4* pa = reinterpret_cast<const f32x4*>(aj + chans[q] * ch + row * MLP_WIDTH + 32 * h);
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const f32x4 v = pa[k];
        a[4 * k] = v.x; a[4 * k + 1] = v.y; a[4 * k + 2] = v.z; a[4 * k + 3] = v.w;
      }
    } else {
#pragma unroll
      for (int s = 0; s < 32; ++s) a[s] = 0.0f;
    }
#pragma unroll
    for (int s = 0; s < 32; ++s) {
      const float* pb = W + (32 * h + s) * MLP_WIDTH;
      acc[q][0] = mfma32(a[s], pb[c], acc[q][0]);
      acc[q][1] = mfma32(a[s], pb[32 + c], acc[q][1]);
    }
  }
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * t + c;
    const float bc = bias[col];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const long long rr = row0 + acc_row(r, h);
      if (rr < n) {
        const float y = tanh_fast(acc[0][t][r] + bc), tp = 1.0f - y * y;
        const float zd = acc[1][t][r], zdd = acc[2][t][r];
        const long long e = rr * MLP_WIDTH + col;
        if (d == 0) aj_next[e] = y;
        aj_next[(1 + d) * ch + e] = tp * zd;
        aj_next[(4 + d) * ch + e] = tp * zdd - 2.0f * y * tp * zd * zd;
        zj_next[d * ch + e] = zd;
        zj_next[(3 + d) * ch + e] = zdd;
      }
    }
  }
}

// output layer on the jets: oj [7][n][5]
__global__ __launch_bounds__(256) void k_jet_out(MlpDev M, const float* __restrict__ aj, float* __restrict__ oj) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long n = M.n;
  const long long q = idx >> 3;  // channel-major (c, p)
  const int o = (int)(idx & 7);
  if (q >= JET * n || o >= MLP_OUT) return;
  const int cch = (int)(q / n);
  const float* W = M.params + M.off_w[M.depth];
  const float* a = aj + q * MLP_WIDTH;
  float z = cch == 0 ? M.params[M.off_b[M.depth] + o] : 0.0f;
  for (int k = 0; k < MLP_WIDTH; ++k) z = fmaf(a[k], W[k * MLP_OUT + o], z);
  oj[q * MLP_OUT + o] = z;
}

// Boussinesq residuals (Sec. 2.D) in nondimensional coordinates from the output jets, the
// per-point loss g1 r_mass^2 + g2 |r_mom|^2 + g3 r_heat^2 (block partials) and its seed
// on every output channel. Outputs: T_nd, p, u_x, u_y, u_z; gravity along -z.
__global__ __launch_bounds__(256) void k_pde_seed(long long n, const float* __restrict__ oj, PdeConst P,
                                                  float* __restrict__ dj, float* __restrict__ res,
                                                  float* __restrict__ partials) {
  __shared__ float red[4];
  const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  float lp = 0.0f;
  if (p < n) {
    float v[MLP_OUT], D1[3][MLP_OUT], D2[3][MLP_OUT];
#pragma unroll
    for (int k = 0; k < MLP_OUT; ++k) {
      v[k] = oj[p * MLP_OUT + k];
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        D1[d][k] = P.s[d] * oj[((1 + d) * n + p) * MLP_OUT + k];
        D2[d][k] = P.s[d] * P.s[d] * oj[((4 + d) * n + p) * MLP_OUT + k];
      }
    }
    const float T = v[0];
    const float u[3] = {v[2], v[3], v[4]};
    float rmass = 0.0f, rmom[3], rheat = 0.0f;
#pragma unroll
    for (int d = 0; d < 3; ++d) rmass += D1[d][2 + d];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      float conv = 0.0f, lap = 0.0f;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        conv = fmaf(u[d], D1[d][2 + k], conv);
        lap += D2[d][2 + k];
      }
      rmom[k] = conv + D1[k][1] - lap * P.inv_re + (k == 2 ? -P.ri * T : 0.0f);
    }
    {
      float conv = 0.0f, lap = 0.0f;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        conv = fmaf(u[d], D1[d][0], conv);
        lap += D2[d][0];
      }
      rheat = conv - lap * P.inv_pe;
    }
    lp = P.g[0] * rmass * rmass + P.g[1] * (rmom[0] * rmom[0] + rmom[1] * rmom[1] + rmom[2] * rmom[2]) +
         P.g[2] * rheat * rheat;
    if (res) {
      res[p * 5] = rmass;
      res[p * 5 + 1] = rmom[0];
      res[p * 5 + 2] = rmom[1];
      res[p * 5 + 3] = rmom[2];
      res[p * 5 + 4] = rheat;
    }
    if (dj) {
      const float Rm = 2.0f * P.g[0] * rmass, Rh = 2.0f * P.g[2] * rheat;
      const float Rv[3] = {2.0f * P.g[1] * rmom[0], 2.0f * P.g[1] * rmom[1], 2.0f * P.g[1] * rmom[2]};
      // value channel
      dj[p * MLP_OUT] = -P.ri * Rv[2];
      dj[p * MLP_OUT + 1] = 0.0f;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        float g = Rh * D1[d][0];
#pragma unroll
        for (int k = 0; k < 3; ++k) g = fmaf(Rv[k], D1[d][2 + k], g);
        dj[p * MLP_OUT + 2 + d] = g;
      }
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        float* g1 = dj + ((1 + d) * n + p) * MLP_OUT;
        float* g2 = dj + ((4 + d) * n + p) * MLP_OUT;
        const float sd = P.s[d], sd2 = sd * sd;
        g1[0] = Rh * u[d] * sd;
        g1[1] = Rv[d] * sd;
#pragma unroll
        for (int k = 0; k < 3; ++k) g1[2 + k] = (Rv[k] * u[d] + (k == d ? Rm : 0.0f)) * sd;
        g2[0] = -Rh * sd2 * P.inv_pe;
        g2[1] = 0.0f;
#pragma unroll
        for (int k = 0; k < 3; ++k) g2[2 + k] = -Rv[k] * sd2 * P.inv_re;
      }
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) lp += __shfl_xor(lp, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = lp;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// Reverse of tanh on the jets: from G = dL/d(a channels) [7][n][64] (OUT: from the output
// seeds dj [7][n][5] through W_D^T), the layer's y = a_0 and its pre-activation
// derivatives zj [6][n][64], writes dz = dL/d(z channels) [7][n][64].
template <bool OUT>
__global__ __launch_bounds__(256) void k_jet_act_back(MlpDev M, const float* __restrict__ G,
                                                      const float* __restrict__ aj, const float* __restrict__ zj,
                                                      float* __restrict__ dz) {
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  const long long n = M.n;
  const long long p = idx >> 6;
  const int j = (int)(idx & 63);
  if (p >= n) return;
  const long long e = p * MLP_WIDTH + j, ch = n * MLP_WIDTH;
  float g[JET];
  if constexpr (OUT) {
    const float* W = M.params + M.off_w[M.depth];
#pragma unroll
    for (int c = 0; c < JET; ++c) {
      float s = 0.0f;
#pragma unroll
      for (int o = 0; o < MLP_OUT; ++o) s = fmaf(G[(c * n + p) * MLP_OUT + o], W[j * MLP_OUT + o], s);
      g[c] = s;
    }
  } else {
#pragma unroll
    for (int c = 0; c < JET; ++c) g[c] = G[c * ch + e];
  }
  const float y = aj[e], tp = 1.0f - y * y;
  float d0 = g[0] * tp;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const float zd = zj[d * ch + e], zdd = zj[(3 + d) * ch + e];
    const float gd = g[1 + d], gdd = g[4 + d];
    dz[(4 + d) * ch + e] = gdd * tp;
    dz[(1 + d) * ch + e] = gd * tp - 4.0f * gdd * y * tp * zd;
    d0 += -2.0f * y * tp * (gd * zd + gdd * zdd) - 2.0f * tp * (1.0f - 3.0f * y * y) * gdd * zd * zd;
  }
  dz[e] = d0;
}

// Boundary-type loss: per point sum_k ((out_k - target_k) / norm_k)^2 and its seed
// dL/dout_k = 2 (out_k - target_k) / norm_k^2; per-block partial sums of the loss.
__global__ __launch_bounds__(256) void k_mlp_fit_seed(long long n, const float* __restrict__ out,
                                                      const float* __restrict__ target, FitNorms inv,
                                                      float* __restrict__ dL, float* __restrict__ partials) {
  __shared__ float red[4];
  const long long p = (long long)blockIdx.x * 256 + threadIdx.x;
  float l = 0.0f;
  if (p < n) {
#pragma unroll
    for (int k = 0; k < MLP_OUT; ++k) {
      const float r = (out[p * MLP_OUT + k] - target[p * MLP_OUT + k]) * inv.v[k];
      l = fmaf(r, r, l);
      dL[p * MLP_OUT + k] = 2.0f * r * inv.v[k];
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = l;
  __syncthreads();
  if (threadIdx.x == 0 && partials) partials[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// fixed-order sum of the block partials into one value
__global__ __launch_bounds__(256) void k_sum_partials(const float* __restrict__ partials, int nblk,
                                                      float* __restrict__ result) {
  __shared__ float red[4];
  float s = 0.0f;
  for (int i = threadIdx.x; i < nblk; i += 256) s += partials[i];
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *result = (red[0] + red[1]) + (red[2] + red[3]);
}

inline size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

inline int blocks_for(long long threads) { return (int)((threads + 255) / 256); }

// blocks (four wavefronts each) of the parameter-gradient reduction over `rows` rows: one
// per 64 rows, up to two per compute unit
inline long long wgrad_blocks(long long rows) {
  const long long b = (rows + 63) / 64;
  return b < 1 ? 1 : (b > 512 ? 512 : b);
}

}  // namespace

// Rows past the activations: a backward block loads whole chunks of points (see GradSide).
constexpr size_t ACT_TAIL = BWD_POINTS - 1;

size_t mlp_work_bytes(int depth, long long n) {
  const long long nblk = wgrad_blocks(n);
  size_t b = 0;
  b += al256(sizeof(float) * ((size_t)depth * (size_t)n + ACT_TAIL) * MLP_WIDTH);
  b += al256(sizeof(float) * (size_t)depth * MLP_WIDTH * MLP_WIDTH);
  b += al256(sizeof(float) * (size_t)(depth + 1) * (size_t)nblk * MLP_PART);
  b += al256(sizeof(float) * 4 * (size_t)n);
  return b;
}

void mlp_work_carve(void* ws, int depth, long long n, MlpWork& w) {
  const long long nblk = wgrad_blocks(n);
  w.nblk = (int)nblk;
  unsigned char* p = static_cast<unsigned char*>(ws);
  w.act = reinterpret_cast<float*>(p);
  p += al256(sizeof(float) * ((size_t)depth * (size_t)n + ACT_TAIL) * MLP_WIDTH);
  w.wt = reinterpret_cast<float*>(p);
  p += al256(sizeof(float) * (size_t)depth * MLP_WIDTH * MLP_WIDTH);
  w.partial = reinterpret_cast<float*>(p);
  p += al256(sizeof(float) * (size_t)(depth + 1) * (size_t)nblk * MLP_PART);
  w.xh = reinterpret_cast<float*>(p);
}

hipError_t launch_mlp_forward(const MlpDev& M, const MlpWork& w, float* out, float* T, float T0, float dT,
                              hipStream_t stream) {
  if (M.n == 0) return hipSuccess;
  const size_t lds = sizeof(float) * (size_t)fused_lds_floats(M.depth);
  // up to 133 KB of staged weights (8 hidden layers): allow the kernel the largest size
  // once per device (safe from any thread)
  static std::atomic<int> lds_set[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64 || !lds_set[dev].load(std::memory_order_acquire)) {
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_mlp_forward_fused),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)(sizeof(float) * (size_t)fused_lds_floats(MLP_MAX_DEPTH)));
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64) lds_set[dev].store(1, std::memory_order_release);
  }
  const long long groups = (M.n + 31) / 32;
  const long long blocks = (groups + 3) / 4;
  const int nblk = (int)(blocks < 2048 ? blocks : 2048);
  // The transposed weights by blocks of their own while compute units are idle: 512 points, depth
  // 4, 25.0 -> 22.6 us. More blocks than units would run them last: 64^3 points, depth 8, 846 -> 863.
  const int grid = nblk + M.depth - 1 <= 256 ? nblk + M.depth - 1 : nblk;
  hipLaunchKernelGGL(k_mlp_forward_fused, dim3(grid), dim3(256), lds, stream, M, w.act, w.xh, w.wt, out, T,
                     T0, dT, nblk);
  return hipGetLastError();
}

template <int D>
static void launch_backward_depth(const MlpDev& M, const MlpWork& w, const float* dL_dout, int nblk, long long rows,
                                  hipStream_t stream) {
  if (M.depth == D)
    hipLaunchKernelGGL((k_mlp_backward_fused<D>), dim3(nblk), dim3(512), 0, stream, M, w.act, w.xh, dL_dout, w.wt,
                       w.partial, nblk, rows);
  else if constexpr (D > 1)
    launch_backward_depth<D - 1>(M, w, dL_dout, nblk, rows, stream);
}

static void launch_reduce(const MlpDev& M, const float* partial, int nblk, float* dparams, hipStream_t stream) {
  const int total = M.off_b[M.depth] + MLP_OUT;
  hipLaunchKernelGGL(k_mlp_reduce, dim3((total + 15) / 16), dim3(256), 0, stream, M, partial, nblk, dparams);
}

hipError_t launch_mlp_backward(const MlpDev& M, const MlpWork& w, const float* dL_dout, float* dparams,
                               hipStream_t stream) {
  if (M.n == 0) return hipSuccess;
  // whole chunks per block, on at most the blocks whose partials the workspace holds
  const long long chunks = (M.n + BWD_POINTS - 1) / BWD_POINTS;
  const long long per = (chunks + w.nblk - 1) / w.nblk;
  const int nblk = (int)((chunks + per - 1) / per);
  launch_backward_depth<MLP_MAX_DEPTH>(M, w, dL_dout, nblk, per * BWD_POINTS, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  launch_reduce(M, w.partial, nblk, dparams, stream);
  return hipGetLastError();
}

size_t mlp_jet_work_bytes(int depth, long long n) {
  const long long rows = JET * n;
  const long long nblk = wgrad_blocks(rows);
  size_t b = 0;
  b += al256(sizeof(float) * (size_t)depth * JET * (size_t)n * MLP_WIDTH);        // a jets
  b += al256(sizeof(float) * (size_t)depth * (JET - 1) * (size_t)n * MLP_WIDTH);  // z jets
  b += 2 * al256(sizeof(float) * JET * (size_t)n * MLP_OUT);                      // output jets, seeds
  b += 3 * al256(sizeof(float) * JET * (size_t)n * MLP_WIDTH);                    // dz x 2, G
  b += al256(sizeof(float) * (size_t)depth * MLP_WIDTH * MLP_WIDTH);
  b += al256(sizeof(float) * (size_t)(depth + 1) * (size_t)nblk * MLP_PART);
  b += al256(sizeof(float) * (size_t)((n + 255) / 256 + 1));
  b += al256(sizeof(float) * 4 * (size_t)n);
  return b;
}

hipError_t launch_mlp_pde(const MlpDev& M, void* ws, const PdeConst& P, float* loss, float* dparams, float* residuals,
                          hipStream_t stream) {
  const long long n = M.n;
  const int D = M.depth;
  if (n == 0) {
    if (loss) hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, stream, (const float*)nullptr, 0, loss);
    return hipGetLastError();
  }
  const long long rows = JET * n;
  const long long nblk = wgrad_blocks(rows);
  const long long rpb = ((rows + nblk - 1) / nblk + 63) / 64 * 64;
  unsigned char* q = static_cast<unsigned char*>(ws);
  auto take = [&](size_t bytes) {
    float* f = reinterpret_cast<float*>(q);
    q += al256(bytes);
    return f;
  };
  const size_t chw = sizeof(float) * (size_t)n * MLP_WIDTH;
  float* aj = take(chw * JET * D);
  float* zj = take(chw * (JET - 1) * D);
  float* oj = take(sizeof(float) * JET * (size_t)n * MLP_OUT);
  float* dj = take(sizeof(float) * JET * (size_t)n * MLP_OUT);
  float* dz[2] = {take(chw * JET), take(chw * JET)};
  float* G = take(chw * JET);
  float* wt = take(sizeof(float) * (size_t)D * MLP_WIDTH * MLP_WIDTH);
  float* partial = take(sizeof(float) * (size_t)(D + 1) * (size_t)nblk * MLP_PART);
  float* lpart = take(sizeof(float) * (size_t)((n + 255) / 256 + 1));
  float* xh = take(sizeof(float) * 4 * (size_t)n);
  auto A = [&](int l) { return aj + (size_t)(l - 1) * JET * n * MLP_WIDTH; };       // a_l jets, l = 1 .. D
  auto Z = [&](int l) { return zj + (size_t)(l - 1) * (JET - 1) * n * MLP_WIDTH; };  // z_l jets
  auto part = [&](int l) { return partial + (size_t)l * nblk * MLP_PART; };
  const unsigned tiles = (unsigned)((n + 127) / 128);
  // forward
  hipLaunchKernelGGL(k_jet_first, dim3(blocks_for(n * MLP_WIDTH)), dim3(256), 0, stream, M, A(1), Z(1), xh);
  for (int l = 1; l < D; ++l)
    hipLaunchKernelGGL(k_jet_dense, dim3(tiles, 3), dim3(256), 0, stream, n, A(l), M.params + M.off_w[l],
                       M.params + M.off_b[l], A(l + 1), Z(l + 1));
  hipLaunchKernelGGL(k_jet_out, dim3(blocks_for(rows * 8)), dim3(256), 0, stream, M, A(D), oj);
  hipLaunchKernelGGL(k_pde_seed, dim3(blocks_for(n)), dim3(256), 0, stream, n, oj, P, dparams ? dj : nullptr,
                     residuals, lpart);
  if (loss) hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, stream, lpart, blocks_for(n), loss);
  if (!dparams) return hipGetLastError();
  // reverse
  if (D > 1)
    hipLaunchKernelGGL(k_mlp_transpose, dim3(blocks_for((long long)(D - 1) * MLP_WIDTH * MLP_WIDTH)), dim3(256), 0,
                       stream, M, wt);
  hipLaunchKernelGGL((k_mlp_wgrad<false, false>), dim3((unsigned)nblk), dim3(256), 0, stream, M, A(D), dj, MLP_OUT, MLP_OUT,
                     part(D), rpb, rows, n);
  hipLaunchKernelGGL((k_jet_act_back<true>), dim3(blocks_for(n * MLP_WIDTH)), dim3(256), 0, stream, M, dj, A(D),
                     Z(D), dz[0]);
  int cur = 0;
  for (int l = D - 1; l >= 1; --l) {
    // dW_l = sum_c a_l^c^T dz_{l+1}^c (bias: value channel); G = dz_{l+1} W_l^T; dz_l
    hipLaunchKernelGGL((k_mlp_wgrad<false, true>), dim3((unsigned)nblk), dim3(256), 0, stream, M, A(l), dz[cur],
                       MLP_WIDTH, MLP_WIDTH, part(l), rpb, rows, n, wt + (size_t)(l - 1) * MLP_WIDTH * MLP_WIDTH, G);
    hipLaunchKernelGGL((k_jet_act_back<false>), dim3(blocks_for(n * MLP_WIDTH)), dim3(256), 0, stream, M, G, A(l),
                       Z(l), dz[cur ^ 1]);
    cur ^= 1;
  }
  // first layer: the input jet (xhat, e_d, 0): rows 0 .. 4n of dz_1
  hipLaunchKernelGGL((k_mlp_wgrad<true, false>), dim3((unsigned)nblk), dim3(256), 0, stream, M, xh, dz[cur], MLP_WIDTH,
                     MLP_WIDTH, part(0), rpb, 4 * n, n);
  launch_reduce(M, partial, (int)nblk, dparams, stream);
  return hipGetLastError();
}

hipError_t launch_mlp_fit_seed(long long n, const float* out, const float* target, const double* norms, float* dL_dout,
                               float* loss, float* partials, hipStream_t stream) {
  FitNorms inv;
  for (int k = 0; k < MLP_OUT; ++k) inv.v[k] = (float)(1.0 / norms[k]);
  const int nblk = blocks_for(n);
  if (n > 0)
    hipLaunchKernelGGL(k_mlp_fit_seed, dim3(nblk), dim3(256), 0, stream, n, out, target, inv, dL_dout,
                       loss ? partials : nullptr);
  if (loss) hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, stream, partials, n > 0 ? nblk : 0, loss);
  return hipGetLastError();
}

hipError_t launch_mlp_bos_seed(long long n, const float* T, const double* grad_delta, double rho0G, double T0,
                               double dT, float* dL_dout, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const double k = -rho0G * T0 * dT;
  hipLaunchKernelGGL(k_mlp_bos_seed, dim3(blocks_for(n)), dim3(256), 0, stream, n, T, grad_delta, k, dL_dout);
  return hipGetLastError();
}

}  // namespace rbos
