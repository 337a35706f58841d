// The MLP building blocks in fp32 on MFMA (gfx950): forward of the network on
// given features, and its backward to features and weights from a given
// dL/do.  (fp64 runs the thread-per-sample kernels of k_mlp.hip.)
//
// v_mfma_f32_16x16x4 adds its four products to the accumulator one after the
// other, each with one rounding (checked against a chain of fmaf, 512,000
// results equal in every bit), so a layer summed over ascending k gives each
// activation the bits that a scalar fma loop gives it: which units the ReLU
// cuts does not depend on this kernel's tiling.
//
// Layout (one wave): lane l = 16 g + c works on sample c of a group of 16.
// An A operand holds, in lane (g, r), weight row r of its tile at k = 4 s + g;
// D holds, in lane (g, c), rows 4 g + i (i = 0..3) of sample c.  The rows of a
// hidden layer's tile are handed to the MFMA in the order r -> neuron
// 4 (r % 4) + r / 4, so that register i of lane group g is neuron
// 16 m + 4 i + g, which is exactly the B operand of the next layer's step
// s = 4 m + i: activations stay in their registers from layer to layer while
// k still ascends.
//
// Measured on 2^16 samples of the 2 x 64 network with 32 inputs, against the
// thread-per-sample kernels before: forward 661 -> 20 us (41 TFLOP/s; bound by
// the one fill of the operands per workgroup and the first loads), backward
// 14,967 -> 55 us (44 TFLOP/s; before, one global atomic per sample and
// weight; now bound by LDS round trips at four waves per CU).
#include "dvnr_device.h"

namespace dvnrk {

typedef float f32x4b __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4b mma4(float a, float b, f32x4b c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Neuron (within a 16-row tile) that row r of an A operand holds.
__host__ __device__ constexpr int row_neuron(int r) { return 4 * (r % 4) + r / 4; }

template <int W, int NH>
struct BlkShape {
  static constexpr int MT = W / 16;                // 16-row tiles of a hidden layer
  static constexpr int KS = W / 4;                 // K steps over a hidden layer
  static constexpr int N_A0 = MT * 8;              // forward W_0 (inputs padded to 32)
  static constexpr int N_AH = (NH - 1) * MT * KS;  // forward W_1 ..
  static constexpr int N_FWD = N_A0 + N_AH;
  static constexpr int N_BWD = N_AH + 2 * KS;      // transposed W_1 .. and W_0
  // weight-gradient staging of one wave: dZ_k and the input of layer k, 16
  // samples a row, rows padded to 20 floats (the 16 rows of an operand read
  // then start in different banks)
  static constexpr int RS = 20;
  static constexpr int ROWS = NH * W + 32 + (NH - 1) * W;
  static constexpr size_t bytes(int slots) { return sizeof(float) * (slots * 64 + 64 + 256 + 4 * ROWS * RS); }
  // the backward operands are staged in LDS beside the forward ones where that
  // fits (3 x 64 reads them from the weights, through the caches, instead)
  static constexpr bool BWD_LDS = bytes(N_FWD + N_BWD) <= (size_t)kLdsBytes;
  static constexpr int N_LDS = BWD_LDS ? N_FWD + N_BWD : N_FWD;
  static_assert(bytes(N_LDS) <= (size_t)kLdsBytes, "a workgroup fits the LDS");
};

// Operand e (slot e / 64, lane e % 64) of the forward pass, then of the backward pass.
template <int W, int NH>
__device__ __forceinline__ float blk_operand(const float* __restrict__ w, const MlpDesc& md, int e) {
  using S = BlkShape<W, NH>;
  const int slot = e / 64, lane = e % 64, r = lane % 16, g = lane / 16;
  const int in = md.in_dim;
  if (slot < S::N_A0) {
    const int m = slot / 8, f = 4 * (slot % 8) + g;
    return f < in ? w[md.off[0] + (16 * m + row_neuron(r)) * in + f] : 0.0f;
  }
  if (slot < S::N_FWD) {
    const int q = slot - S::N_A0, k = 1 + q / (S::MT * S::KS), m = (q / S::KS) % S::MT, s = q % S::KS;
    return w[md.off[k] + (16 * m + row_neuron(r)) * W + 4 * s + g];
  }
  if (slot < S::N_FWD + S::N_AH) {
    const int q = slot - S::N_FWD, k = 1 + q / (S::MT * S::KS), m = (q / S::KS) % S::MT, s = q % S::KS;
    return w[md.off[k] + (4 * s + g) * W + 16 * m + row_neuron(r)];
  }
  const int q = slot - S::N_FWD - S::N_AH, f = 16 * (q / S::KS) + r;
  return f < in ? w[md.off[0] + (4 * (q % S::KS) + g) * in + f] : 0.0f;
}

// Forward.  A wave takes GR groups of 16 samples at once: each operand read
// from LDS feeds GR MFMAs, and the chains of the groups hide one another's
// latency.
template <int W, int NH, int GR>
__global__ __launch_bounds__(256) void k_mlp_block_fwd(MlpDesc md, int64_t n, const float* __restrict__ x,
                                                       const float* __restrict__ w, float* __restrict__ out) {
  using S = BlkShape<W, NH>;
  __shared__ float A[S::N_FWD * 64];
  __shared__ float wout[W];
  for (int e = threadIdx.x; e < S::N_FWD * 64; e += 256) A[e] = blk_operand<W, NH>(w, md, e);
  if (threadIdx.x < W) wout[threadIdx.x] = w[md.off[NH] + threadIdx.x];
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, g = lane / 16, c = lane % 16;
  const int in = md.in_dim;
  constexpr int PER = 4 * 16 * GR;  // samples of a workgroup's pass
  for (int64_t base = (int64_t)blockIdx.x * PER + wave * 16 * GR; base < n; base += (int64_t)gridDim.x * PER) {
    float xb[GR][8];
#pragma unroll
    for (int q = 0; q < GR; ++q) {
      // samples past the end read the last one and are not stored
      const float* xs = x + min(base + 16 * q + c, n - 1) * in;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const float v = xs[min(4 * s + g, in - 1)];
        xb[q][s] = 4 * s + g < in ? v : 0.0f;
      }
    }
    f32x4b h[GR][S::MT];
#pragma unroll
    for (int m = 0; m < S::MT; ++m) {
      f32x4b acc[GR];
#pragma unroll
      for (int q = 0; q < GR; ++q) acc[q] = f32x4b{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const float a = A[(m * 8 + s) * 64 + lane];
#pragma unroll
        for (int q = 0; q < GR; ++q) acc[q] = mma4(a, xb[q][s], acc[q]);
      }
#pragma unroll
      for (int q = 0; q < GR; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) h[q][m][i] = fmaxf(acc[q][i], 0.0f);
    }
#pragma unroll
    for (int k = 1; k < NH; ++k) {
      f32x4b hn[GR][S::MT];
#pragma unroll
      for (int m = 0; m < S::MT; ++m) {
        f32x4b acc[GR];
#pragma unroll
        for (int q = 0; q < GR; ++q) acc[q] = f32x4b{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < S::KS; ++s) {
          const float a = A[(S::N_A0 + ((k - 1) * S::MT + m) * S::KS + s) * 64 + lane];
#pragma unroll
          for (int q = 0; q < GR; ++q) acc[q] = mma4(a, h[q][s / 4][s % 4], acc[q]);
        }
#pragma unroll
        for (int q = 0; q < GR; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) hn[q][m][i] = fmaxf(acc[q][i], 0.0f);
      }
#pragma unroll
      for (int q = 0; q < GR; ++q)
#pragma unroll
        for (int m = 0; m < S::MT; ++m) h[q][m] = hn[q][m];
    }
#pragma unroll
    for (int q = 0; q < GR; ++q) {
      float o = 0.0f;
#pragma unroll
      for (int m = 0; m < S::MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) o += wout[16 * m + 4 * i + g] * h[q][m][i];
      o += __shfl_xor(o, 16, 64);
      o += __shfl_xor(o, 32, 64);
      const int64_t gi = base + 16 * q + c;
      if (g == 0 && gi < n) out[gi] = o;
    }
  }
}

// Backward (recomputes the forward).  Persistent workgroups of 4 waves: per
// pass each wave takes 16 samples, writes their dL/dx and stages dZ_k and the
// layer inputs in LDS as [neuron][sample]; the waves then share out the
// 16 x 16 tiles of the weight gradients and contract each over the pass's 64
// samples, so a weight's sum stays in a register until the workgroup's last
// pass and goes to memory in one atomic per workgroup (one per sample before).
template <int W, int NH>
__global__ __launch_bounds__(256, 1) void k_mlp_block_bwd(MlpDesc md, int64_t n, const float* __restrict__ x,
                                                          const float* __restrict__ w, const float* __restrict__ dout,
                                                          float* __restrict__ dx, float* __restrict__ dw) {
  using S = BlkShape<W, NH>;
  constexpr int T_ALL = 2 * S::MT + (NH - 1) * S::MT * S::MT;  // 16 x 16 tiles of all weight gradients
  constexpr int U = (T_ALL + 3) / 4;                            // tiles per wave
  extern __shared__ __align__(16) float bsm[];
  float* A = bsm;
  float* wout = A + S::N_LDS * 64;
  float* red = wout + 64;  // [4][64]: output-layer gradient of each wave
  float* stage = red + 256;
  const int64_t passes = (n + 63) / 64;
  const int64_t p0 = (int64_t)blockIdx.x * passes / gridDim.x, p1 = (int64_t)(blockIdx.x + 1) * passes / gridDim.x;
  if (p0 >= p1) return;  // the whole workgroup
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64, g = lane / 16, c = lane % 16;
  const int in = md.in_dim;
  for (int e = threadIdx.x; e < S::N_LDS * 64; e += 256) A[e] = blk_operand<W, NH>(w, md, e);
  if (threadIdx.x < W) wout[threadIdx.x] = w[md.off[NH] + threadIdx.x];
  __syncthreads();
  auto opB = [&](int slot) -> float {  // backward operand
    const int e = (S::N_FWD + slot) * 64 + lane;
    if constexpr (S::BWD_LDS)
      return A[e];
    else
      return blk_operand<W, NH>(w, md, e);
  };
  // staging rows of wave v: dZ_k from row k W, layer 0's input from NH W, layer k's (k >= 1) after it
  auto SZ = [&](int v, int k) { return stage + (v * S::ROWS + k * W) * S::RS; };
  auto SI = [&](int v, int k) {
    return stage + (v * S::ROWS + (k == 0 ? NH * W : NH * W + 32 + (k - 1) * W)) * S::RS;
  };
  auto tile_kmn = [](int t, int& k, int& m, int& j) {
    if (t < 2 * S::MT) {
      k = 0;
      m = t / 2;
      j = t % 2;
    } else {
      const int r = t - 2 * S::MT;
      k = 1 + r / (S::MT * S::MT);
      m = (r / S::MT) % S::MT;
      j = r % S::MT;
    }
  };
  f32x4b dwt[U];
#pragma unroll
  for (int u = 0; u < U; ++u) dwt[u] = f32x4b{0, 0, 0, 0};
  float dwo[S::MT][4];
#pragma unroll
  for (int m = 0; m < S::MT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) dwo[m][i] = 0.0f;
  // the features and dL/do of the next pass are in flight while this one computes
  float xn[8], dn;
  auto load_pass = [&](int64_t p) {
    const int64_t gi = min(64 * p + 16 * wave + c, n - 1);
    const float* xs = x + gi * in;
#pragma unroll
    for (int s = 0; s < 8; ++s) xn[s] = xs[min(4 * s + g, in - 1)];
    dn = dout[gi];
  };
  load_pass(p0);
#pragma unroll 1
  for (int64_t p = p0; p < p1; ++p) {
    const int64_t gi = 64 * p + 16 * wave + c;
    const bool valid = gi < n;
    float xb[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) xb[s] = (valid && 4 * s + g < in) ? xn[s] : 0.0f;
    const float d = valid ? dn : 0.0f;
    load_pass(min(p + 1, p1 - 1));
#pragma unroll
    for (int s = 0; s < 8; ++s) SI(wave, 0)[(4 * s + g) * S::RS + c] = xb[s];
    f32x4b h[NH][S::MT];
#pragma unroll
    for (int m = 0; m < S::MT; ++m) {
      f32x4b acc = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < 8; ++s) acc = mma4(A[(m * 8 + s) * 64 + lane], xb[s], acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) h[0][m][i] = fmaxf(acc[i], 0.0f);
    }
#pragma unroll
    for (int k = 1; k < NH; ++k)
#pragma unroll
      for (int m = 0; m < S::MT; ++m) {
        f32x4b acc = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < S::KS; ++s)
          acc = mma4(A[(S::N_A0 + ((k - 1) * S::MT + m) * S::KS + s) * 64 + lane], h[k - 1][s / 4][s % 4], acc);
#pragma unroll
        for (int i = 0; i < 4; ++i) h[k][m][i] = fmaxf(acc[i], 0.0f);
      }
    f32x4b dz[S::MT];
#pragma unroll
    for (int m = 0; m < S::MT; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float hv = h[NH - 1][m][i];
        dwo[m][i] += d * hv;
        dz[m][i] = hv > 0.0f ? wout[16 * m + 4 * i + g] * d : 0.0f;
      }
#pragma unroll
    for (int k = NH - 1; k >= 0; --k) {
#pragma unroll
      for (int m = 0; m < S::MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 16 * m + 4 * i + g;
          SZ(wave, k)[r * S::RS + c] = dz[m][i];
          if (k >= 1) SI(wave, k)[r * S::RS + c] = h[k - 1][m][i];
        }
      if (k >= 1) {
        f32x4b nz[S::MT];
#pragma unroll
        for (int m = 0; m < S::MT; ++m) {
          f32x4b acc = {0, 0, 0, 0};
#pragma unroll
          for (int s = 0; s < S::KS; ++s)
            acc = mma4(opB(((k - 1) * S::MT + m) * S::KS + s), dz[s / 4][s % 4], acc);
#pragma unroll
          for (int i = 0; i < 4; ++i) nz[m][i] = h[k - 1][m][i] > 0.0f ? acc[i] : 0.0f;
        }
#pragma unroll
        for (int m = 0; m < S::MT; ++m) dz[m] = nz[m];
      }
    }
    // dL/dx = W_0^T dZ_0: lane (g, c) holds features 16 j + 4 g + i of its sample
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      f32x4b acc = {0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < S::KS; ++s)
        acc = mma4(opB(S::N_AH + j * S::KS + s), dz[s / 4][s % 4], acc);
      if (valid) {
        const int f0 = 16 * j + 4 * g;
        float* o = dx + gi * in + f0;
        if (in % 4 == 0) {  // (4-byte alignment is enough for the 16-byte store)
          if (f0 < in) __builtin_memcpy(o, &acc, 16);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (f0 + i < in) o[i] = acc[i];
        }
      }
    }
    __syncthreads();  // the pass is staged
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = wave + 4 * u;
      if (t < T_ALL) {
        int k, m, j;
        tile_kmn(t, k, m, j);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float* za = SZ(v, k) + (16 * m + c) * S::RS + g;
          const float* ib = SI(v, k) + (16 * j + c) * S::RS + g;
#pragma unroll
          for (int s = 0; s < 4; ++s) dwt[u] = mma4(za[4 * s], ib[4 * s], dwt[u]);
        }
      }
    }
    __syncthreads();  // the staging may be overwritten
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = wave + 4 * u;
    if (t < T_ALL) {
      int k, m, j;
      tile_kmn(t, k, m, j);
      const int cols = k == 0 ? in : W, col = 16 * j + c;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (col < cols) unsafeAtomicAdd(&dw[md.off[k] + (16 * m + 4 * g + i) * cols + col], dwt[u][i]);
    }
  }
#pragma unroll
  for (int m = 0; m < S::MT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v = dwo[m][i];
      v += __shfl_xor(v, 1, 64);
      v += __shfl_xor(v, 2, 64);
      v += __shfl_xor(v, 4, 64);
      v += __shfl_xor(v, 8, 64);
      if (c == 0) red[wave * 64 + 16 * m + 4 * i + g] = v;
    }
  __syncthreads();
  if (threadIdx.x < W) {
    const int e = threadIdx.x;
    unsafeAtomicAdd(&dw[md.off[NH] + e], (red[e] + red[64 + e]) + (red[128 + e] + red[192 + e]));
  }
}

// Workgroups of a launch: enough for every CU to have work, few enough that a
// workgroup's weight operands serve several passes (backward: one workgroup
// fills a CU's LDS).
constexpr int kBlkFwdGrid = 1024, kBlkBwdGrid = 256;
// From this many samples on, a forward wave takes four groups at once; below,
// one group per wave spreads the samples over four times as many waves.
constexpr int64_t kBlkWide = 1 << 15;

template <int W, int NH>
static hipError_t run_block_fwd(const MlpDesc& md, int64_t n, const float* x, const float* w, float* out,
                                hipStream_t s) {
  if (n >= kBlkWide) {
    const int grid = (int)std::min<int64_t>((n + 255) / 256, kBlkFwdGrid);
    hipLaunchKernelGGL((k_mlp_block_fwd<W, NH, 4>), dim3(grid), dim3(256), 0, s, md, n, x, w, out);
  } else {
    const int grid = (int)((n + 63) / 64);
    hipLaunchKernelGGL((k_mlp_block_fwd<W, NH, 1>), dim3(grid), dim3(256), 0, s, md, n, x, w, out);
  }
  return hipGetLastError();
}

template <int W, int NH>
static hipError_t run_block_bwd(const MlpDesc& md, int64_t n, const float* x, const float* w, const float* dout,
                                float* dx, float* dw, hipStream_t s) {
  using S = BlkShape<W, NH>;
  const size_t sm = S::bytes(S::N_LDS);
  auto kern = k_mlp_block_bwd<W, NH>;
  hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
  if (e != hipSuccess) return e;
  const int grid = (int)std::min<int64_t>((n + 63) / 64, kBlkBwdGrid);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(256), sm, s, md, n, x, w, dout, dx, dw);
  return hipGetLastError();
}

#define DVNR_BLK_SHAPES(X) X(16, 1) X(16, 2) X(16, 3) X(32, 1) X(32, 2) X(32, 3) X(64, 1) X(64, 2) X(64, 3)

hipError_t launch_mlp_block_fwd(const MlpDesc& md, int64_t n, const float* feats, const float* w, float* out,
                                hipStream_t s) {
  if (n <= 0) return hipSuccess;
#define X(WW, NN) \
  if (md.width == WW && md.n_hidden == NN) return run_block_fwd<WW, NN>(md, n, feats, w, out, s);
  DVNR_BLK_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

hipError_t launch_mlp_block_bwd(const MlpDesc& md, int64_t n, const float* feats, const float* w, const float* dout,
                                float* dfeats, float* dw, hipStream_t s) {
  if (n <= 0) return hipSuccess;
#define X(WW, NN) \
  if (md.width == WW && md.n_hidden == NN) return run_block_bwd<WW, NN>(md, n, feats, w, dout, dfeats, dw, s);
  DVNR_BLK_SHAPES(X)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace dvnrk
