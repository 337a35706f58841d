// The network's forward pass for inference, one wave at a time, with the
// weight operands of the workgroup's block in LDS.
//
// Layout (MFMA 16x16xK): lane l = 16 g + c works on sample c of a group of 16
// samples.  D holds, in lane (g, c), neurons 16 m + 4 g + i (i = 0..3) of
// sample c; the order of a contraction's index is free, so the next layer's K
// steps are labelled such that each lane supplies the neurons it holds, and
// the columns of the weight operands are permuted to match.  The input layer's
// K index is 8 g + s (fp32) or 8 g + j (bf16): lane group g supplies features
// 8 g .. 8 g + 7.  With that labelling the operand of a lane is a run of
// consecutive weights of one row (8 for the input layer, 4 for a hidden one),
// so a wave loads its operands straight from the weight matrices in 8- and
// 16-byte accesses: nothing has to be arranged in LDS or by a kernel before.
#pragma once

#include "dvnr_device.h"

namespace dvnrk {

typedef __bf16 bf16x8i __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4i __attribute__((ext_vector_type(4)));
typedef float f32x4i __attribute__((ext_vector_type(4)));

// NG: lane groups that share a sample's features, 1, 2 or 4 (input widths up
// to 8, 16, 32): group g supplies features 8 (g % NG) .. + 7 of the group of
// samples it belongs to, and zeros for the others.
template <bool BF16, int W, int NH, int NG>
struct InferMlp {
  typedef typename std::conditional<BF16, bf16x8i, float>::type op_t;
  typedef typename std::conditional<BF16, __bf16, float>::type w_t;
  static constexpr int MT = W / 16;                      // 16-row tiles of a hidden layer
  static constexpr int KS_IN = BF16 ? 1 : 8;             // K steps over the inputs
  static constexpr int KS_H = BF16 ? (W + 31) / 32 : W / 4;  // K steps over a hidden layer

  // weight operands in the order eval uses them: slot m KS_IN + s of the input
  // layer, then the hidden layers'; 64 lanes each
  static constexpr int N_IN = MT * KS_IN;
  static constexpr int N_SLOTS = N_IN + (NH - 1) * MT * KS_H;

  // Operand e (slot e / 64, lane e % 64) from the block's weights w (W_1 ..
  // W_out, row-major, aligned to their elements only).
  __device__ static __forceinline__ op_t operand(const w_t* __restrict__ w, const MlpDesc& md, int e) {
    const int slot = e / 64, r = e % 16, g = (e % 64) / 16;
    if (slot < N_IN) {
      const int m = slot / KS_IN, s = slot % KS_IN, in = md.in_dim;
      const int f0 = 8 * (g % NG) + (BF16 ? 0 : s);
      const w_t* row = w + md.off[0] + (16 * m + r) * in + f0;
      if constexpr (BF16) {
        op_t v;
        if (in == 8 * NG) {
          __builtin_memcpy(&v, row, sizeof(v));
        } else {
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const w_t x = f0 < in ? row[min(j, in - 1 - f0)] : w[0];
            v[j] = f0 + j < in ? x : (w_t)0.0f;
          }
        }
        return v;
      } else {
        return f0 < in ? row[0] : 0.0f;
      }
    }
    const int q = slot - N_IN, k = 1 + q / (MT * KS_H), m = (q / KS_H) % MT, s = q % KS_H;
    const w_t* row = w + md.off[k] + (16 * m + r) * W + 4 * g;
    if constexpr (BF16) {
      op_t v;
      bf16x4i lo, hi = {0, 0, 0, 0};
      __builtin_memcpy(&lo, row + 32 * s, sizeof(lo));
      if (2 * s + 1 < MT) __builtin_memcpy(&hi, row + 32 * s + 16, sizeof(hi));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v[i] = lo[i];
        v[4 + i] = hi[i];
      }
      return v;
    } else {
      return row[16 * (s / 4) + s % 4];
    }
  }

  __device__ static __forceinline__ f32x4i mma(op_t a, op_t b, f32x4i c) {
    if constexpr (BF16)
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
    else
      return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }

  // max(x, 0), and 0 for a NaN, as fmaxf gives, but in one instruction (fmaxf
  // takes a second one to quiet a signaling NaN): the median of x, 0 and
  // infinity, which the compiler must not know to be infinity
  __device__ static __forceinline__ float relu(float x) {
    float inf = __builtin_huge_valf();
#ifdef __HIP_DEVICE_COMPILE__
    asm("" : "+s"(inf));
#endif
    return __builtin_amdgcn_fmed3f(x, 0.0f, inf);
  }

  // Network outputs of sample c of Q groups of 16 samples (in every lane group)
  // from the lanes' features.  A: the operands (LDS), in slot order, each read
  // once for the Q groups, whose chains hide one another's latency; wo: the
  // output layer's weights of the neurons that the lane holds (16 m + 4 g + i).
  template <int Q>
  __device__ static __forceinline__ void eval(const op_t* __restrict__ A, const f32x4i (&wo)[MT], int lane,
                                              const op_t (&xb)[Q][KS_IN], float (&out)[Q]) {
    f32x4i h[Q][MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      f32x4i acc[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[q] = f32x4i{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < KS_IN; ++s) {
        const op_t a = A[(m * KS_IN + s) * 64 + lane];
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] = mma(a, xb[q][s], acc[q]);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) h[q][m][i] = relu(acc[q][i]);
    }
#pragma unroll
    for (int k = 1; k < NH; ++k) {
      op_t hb[Q][KS_H];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int s = 0; s < KS_H; ++s) {
          if constexpr (BF16) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int m = 2 * s + j / 4;
              hb[q][s][j] = (__bf16)(m < MT ? h[q][m < MT ? m : 0][j % 4] : 0.0f);
            }
          } else {
            hb[q][s] = h[q][s / 4][s % 4];
          }
        }
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        f32x4i acc[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[q] = f32x4i{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS_H; ++s) {
          const op_t a = A[(N_IN + ((k - 1) * MT + m) * KS_H + s) * 64 + lane];
#pragma unroll
          for (int q = 0; q < Q; ++q) acc[q] = mma(a, hb[q][s], acc[q]);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int i = 0; i < 4; ++i) h[q][m][i] = relu(acc[q][i]);
      }
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      float o = 0.0f;
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) o += wo[m][i] * h[q][m][i];
      o += __shfl_xor(o, 16, 64);
      o += __shfl_xor(o, 32, 64);
      out[q] = o;
    }
  }

  // Outputs of NQ groups of 16 samples, in fp32 two at a time (in bf16, where
  // the operands are a sixth of the LDS reads, two spill at four waves per
  // SIMD): lane group g receives group g's (0 for g >= NQ).  SETS = 4 / NG sets of lane groups hold the
  // features xb of the groups q = set, set + SETS, ...; the other sets'
  // features enter a group's product as zeros.
  template <int NQ, int T>
  __device__ static __forceinline__ float eval_groups(const op_t* __restrict__ A, const float* __restrict__ wout,
                                                      int lane, const op_t (&xb)[T][KS_IN]) {
    constexpr int SETS = 4 / NG, Q = !BF16 && NQ >= 2 ? 2 : 1;
    static_assert(NQ == SETS * T && NQ % Q == 0, "every group's features are in one set");
    const int g = lane / 16, set = g / NG;
    f32x4i wo[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) wo[m] = *reinterpret_cast<const f32x4i*>(&wout[16 * m + 4 * g]);
    float o = 0.0f;
#pragma unroll
    for (int q0 = 0; q0 < NQ; q0 += Q) {
      __builtin_amdgcn_sched_barrier(0);  // (more groups in flight would not fit the registers)
      op_t xq[Q][KS_IN];
#pragma unroll
      for (int u = 0; u < Q; ++u)
#pragma unroll
        for (int s = 0; s < KS_IN; ++s) {
          const int q = q0 + u;
          xq[u][s] = xb[q / SETS][s];
          if constexpr (SETS > 1) {
            if (set != q % SETS) {
              if constexpr (BF16) {
#pragma unroll
                for (int j = 0; j < 8; ++j) xq[u][s][j] = (__bf16)0.0f;
              } else {
                xq[u][s] = 0.0f;
              }
            }
          }
        }
      float v[Q];
      eval<Q>(A, wo, lane, xq, v);
#pragma unroll
      for (int u = 0; u < Q; ++u)
        if (g == q0 + u) o = v[u];
    }
    return o;
  }
};

}  // namespace dvnrk
