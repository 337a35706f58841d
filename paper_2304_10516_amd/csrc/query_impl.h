// The INR at arbitrary coordinates in one kernel (gfx950): encoding by direct
// gathers and the MLP forward, without features in memory.  Two kernels:
// values at given coordinates, and direct volume rendering of one block.
//
// As in the fused decode (decode_impl.h), lane (g, c) of a wave interpolates,
// for sample c of a group of 16, the levels whose features the MFMA forward
// wants from lane group g, so features go to the matrix core in registers;
// with inputs of at most 8 or 16 features, NG = 1 or 2 lane groups share a
// sample and the others take other samples.  The eight corners are summed as
// the two-pass path does (the four with the lower x, the four with the upper
// x, then both), so both paths give the same bits.
#pragma once

#include <algorithm>
#include <type_traits>

#include "infer_mlp.h"

namespace dvnrk {

// A level's entry in LDS (lane groups work on different levels).
struct QueryLevel {
  float scale;
  int R;
  uint32_t off;    // byte offset of the level in the block's table
  int dense;
};

__device__ __forceinline__ void load_query_levels(const LevelDesc& ld, int entry_bytes, QueryLevel* lev) {
  if (threadIdx.x < kMaxLevels) {
    const int l = threadIdx.x;
    lev[l] = QueryLevel{ld.scale[l], ld.R[l], (uint32_t)ld.off[l] * (uint32_t)entry_bytes, ld.dense[l]};
  }
}

// Features of T samples at (x, y, z)[t]: levels LPG fg .. LPG fg + LPG - 1, as
// the lane's MFMA operands.  tab: the block's table (its byte size is below
// 2^32: at most 2^29 elements, see dvnr_create).
template <class M, bool BF16, typename TT, int F, int T>
__device__ __forceinline__ void query_features(const QueryLevel* __restrict__ lev, int L, uint32_t mask, int fg,
                                               const TT* __restrict__ tab, const float (&x)[T], const float (&y)[T],
                                               const float (&z)[T], typename M::op_t (&xb)[T][M::KS_IN]) {
  constexpr int LPG = 8 / F;
  constexpr int VB = F * (int)sizeof(TT);
  typedef typename std::conditional<VB % 4 == 0, uint32_t, uint16_t>::type word;
  constexpr int NW = VB / (int)sizeof(word);
  constexpr int TB = T == 1 || VB > 8 ? 1 : 2;  // samples whose gathers are in flight together
  const unsigned char* base = reinterpret_cast<const unsigned char*>(tab);
#pragma unroll
  for (int j = 0; j < LPG; ++j) {
    const int l = LPG * fg + j;
    const bool live = l < L;
    const QueryLevel q = lev[live ? l : 0];
    // (a select would be turned into a branch around each feature's sums, with
    // every gathered value live until the last one)
    const uint32_t keep = live ? ~0u : 0u;
    const uint32_t R = (uint32_t)q.R;
#pragma unroll
    for (int t0 = 0; t0 < T; t0 += TB) {
      // TB samples of a level at a time: with more loads in flight the kernel
      // spills at four waves per SIMD
      if (j + t0 > 0) __builtin_amdgcn_sched_barrier(0);
      word v[TB][8][NW];
      float w[TB][3];
      // every index and load first, so that all are in flight together
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        int ix, iy, iz;
        grid_pos(x[t0 + u], q.scale, q.R, ix, w[u][0]);
        grid_pos(y[t0 + u], q.scale, q.R, iy, w[u][1]);
        grid_pos(z[t0 + u], q.scale, q.R, iz, w[u][2]);
        // dense levels have R^3 <= T <= 2^24 entries: 24-bit products suffice
        const uint32_t d0 = __umul24(R, (uint32_t)iy + __umul24(R, (uint32_t)iz)), dz = __umul24(R, R);
        const uint32_t hy = (uint32_t)iy * 2654435761u, hz = (uint32_t)iz * 805459861u;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const uint32_t gx = (uint32_t)ix + (k & 1);
          const uint32_t ed = gx + d0 + ((k & 2) ? R : 0u) + ((k & 4) ? dz : 0u);
          const uint32_t eh =
              (gx ^ (hy + ((k & 2) ? 2654435761u : 0u)) ^ (hz + ((k & 4) ? 805459861u : 0u))) & mask;
          const uint32_t e = q.dense ? ed : eh;
          const word* p = reinterpret_cast<const word*>(base + (q.off + e * (uint32_t)VB));
#pragma unroll
          for (int i = 0; i < NW; ++i) v[u][k][i] = p[i];
        }
      }
#pragma unroll
      for (int u = 0; u < TB; ++u) {
        const float tx = w[u][0], ty = w[u][1], tz = w[u][2];
        float acc[2][F];
#pragma unroll
        for (int cx = 0; cx < 2; ++cx)
#pragma unroll
          for (int f = 0; f < F; ++f) acc[cx][f] = 0.0f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const float wk =
              ((k & 1) ? tx : 1.0f - tx) * ((k & 2) ? ty : 1.0f - ty) * ((k & 4) ? tz : 1.0f - tz);
          TT e[F];
          __builtin_memcpy(e, v[u][k], VB);
#pragma unroll
          for (int f = 0; f < F; ++f) {
            if constexpr (sizeof(TT) == 2)
              acc[k & 1][f] += wk * __half2float(e[f]);
            else
              acc[k & 1][f] += wk * e[f];
          }
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const float s = __uint_as_float(__float_as_uint(acc[0][f] + acc[1][f]) & keep);
          if constexpr (BF16)
            xb[t0 + u][0][j * F + f] = (__bf16)s;
          else
            xb[t0 + u][j * F + f] = s;
        }
      }
    }
  }
}

// out[i] = de-normalized INR of block `block` at coords[i].  A wave takes
// 16 SETS T samples.
template <bool BF16, int W, int NH, typename TT, int F, int NG, int T>
__global__ __launch_bounds__(256, BF16 ? 4 : 2) void k_query(
    LevelDesc ld, MlpDesc md, const BlockMeta* __restrict__ meta, const BlockRange* __restrict__ range, int block,
    const TT* __restrict__ table_all, const typename InferMlp<BF16, W, NH, NG>::w_t* __restrict__ wsrc, int64_t n,
    const float* __restrict__ coords, float* __restrict__ out) {
  using M = InferMlp<BF16, W, NH, NG>;
  constexpr int SETS = 4 / NG, NQ = SETS * T;  // groups of 16 samples of a wave
  __shared__ QueryLevel lev[kMaxLevels];
  __shared__ __align__(16) typename M::op_t opnd[M::N_SLOTS * 64];
  __shared__ __align__(16) float wout[W];
  const int64_t param_off = meta[block].param_off;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int g = lane / 16, c = lane % 16, set = g / NG, fg = g % NG;
  const int64_t s0 = ((int64_t)blockIdx.x * 4 + wave) * (16 * NQ);
  // the lane's coordinates (the last sample stands in past the end), in flight
  // while the operands are staged
  float x[T], y[T], z[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int64_t i = min(s0 + 16 * (set + SETS * t) + c, n - 1);
    x[t] = coords[3 * i + 0];
    y[t] = coords[3 * i + 1];
    z[t] = coords[3 * i + 2];
  }
  load_query_levels(ld, F * (int)sizeof(TT), lev);
  for (int e = threadIdx.x; e < M::N_SLOTS * 64; e += 256) opnd[e] = M::operand(wsrc + param_off, md, e);
  if (threadIdx.x < W) wout[threadIdx.x] = (float)wsrc[param_off + md.off[NH] + threadIdx.x];
  __syncthreads();
  if (s0 >= n) return;
  typename M::op_t xb[T][M::KS_IN];
  query_features<M, BF16, TT, F, T>(lev, ld.L, ld.T_mask, fg, table_all + param_off, x, y, z, xb);
  const BlockRange br = range[block];
  const float o = M::template eval_groups<NQ, T>(opnd, wout, lane, xb);
  const int64_t i = s0 + 16 * g + c;
  if (g < NQ && i < n) out[i] = o * br.range + br.vmin;
}

// out[i] = de-normalized network output of the features [level][plane][F] that
// the tile encoding wrote (samples 0 .. n - 1).  A workgroup keeps the
// operands and takes 256 samples at a time.
template <bool BF16, int W, int NH, typename TT, int F, int NG>
__global__ __launch_bounds__(256, BF16 ? 4 : 2) void k_mlp_infer(
    LevelDesc ld, MlpDesc md, const BlockMeta* __restrict__ meta, const BlockRange* __restrict__ range, int block,
    const typename InferMlp<BF16, W, NH, NG>::w_t* __restrict__ wsrc, int n,
    const typename InferMlp<BF16, W, NH, NG>::w_t* __restrict__ feat, int64_t plane, float* __restrict__ out) {
  using M = InferMlp<BF16, W, NH, NG>;
  using fe_t = typename M::w_t;
  constexpr int SETS = 4 / NG, T = NG, LPG = 8 / F;
  __shared__ __align__(16) typename M::op_t opnd[M::N_SLOTS * 64];
  __shared__ __align__(16) float wout[W];
  const int64_t param_off = meta[block].param_off;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int g = lane / 16, c = lane % 16, set = g / NG, fg = g % NG;
  const BlockRange br = range[block];
  // features of a pass: samples past the end read the last one, levels past
  // the last read level 0 and become zeros
  fe_t v[T][LPG][F];
  auto load_pass = [&](int s0) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int i = min(s0 + 16 * (set + SETS * t) + c, n - 1);
#pragma unroll
      for (int j = 0; j < LPG; ++j) {
        const int l = LPG * fg + j;
        __builtin_memcpy(v[t][j], feat + ((int64_t)(l < ld.L ? l : 0) * plane + i) * F, sizeof(v[t][j]));
      }
    }
  };
  int s0 = (blockIdx.x * 4 + wave) * 64;
  load_pass(s0);
  for (int e = threadIdx.x; e < M::N_SLOTS * 64; e += 256) opnd[e] = M::operand(wsrc + param_off, md, e);
  if (threadIdx.x < W) wout[threadIdx.x] = (float)wsrc[param_off + md.off[NH] + threadIdx.x];
  __syncthreads();
  const int step = gridDim.x * 256;
  for (; s0 < n; s0 += step) {
    typename M::op_t xb[T][M::KS_IN];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int j = 0; j < LPG; ++j)
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const fe_t x = LPG * fg + j < ld.L ? v[t][j][f] : (fe_t)0.0f;
          if constexpr (BF16)
            xb[t][0][j * F + f] = x;
          else
            xb[t][j * F + f] = x;
        }
    if (s0 + step < n) load_pass(s0 + step);
    const float o = M::template eval_groups<4, T>(opnd, wout, lane, xb);
    const int i = s0 + 16 * g + c;
    if (i < n) out[i] = o * br.range + br.vmin;
  }
}

// ---------------------------------------------------------------------------
// Direct volume rendering of one block's INR.  A wave marches the rays of 4 x 4
// pixels front to back, four samples of each ray per pass; a pass's samples are
// evaluated as above, and lane group g maps sample g through the transfer
// function before every lane composites the four in order.
//
// The rays of a wave are neighbours, so its gathers share cache lines, and a
// ray's state never leaves registers: with one launch per round of samples
// (positions, encoding, MLP, shading of 2^18 samples at a time) features and
// values went through memory and a wave shaded 64 rays one sample after the
// other: 512 x 512 pixels, 128^3 block of the 16-level, 2 x 64 model, step
// 1/256 (24 M samples), mixed precision 13.1 -> 2.05 ms, bound by the gathers
// and the VALU work of their addresses.
//
// Ray setup and sample positions use round-to-nearest operations in a fixed
// order (no contraction into FMA): the number of samples of a ray is an
// integer decided by these values.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float dot3_rn(float ax, float ay, float az, float bx, float by, float bz) {
  return fadd_nc(fadd_nc(fmul_nc(ax, bx), fmul_nc(ay, by)), fmul_nc(az, bz));
}

__device__ __forceinline__ void normalize_rn(float* v) {
  const float n = __fsqrt_rn(dot3_rn(v[0], v[1], v[2], v[0], v[1], v[2]));
#pragma unroll
  for (int a = 0; a < 3; ++a) v[a] = __fdiv_rn(v[a], n);
}

__device__ __forceinline__ void cross_rn(const float* a, const float* b, float* c) {
  c[0] = fsub_nc(fmul_nc(a[1], b[2]), fmul_nc(a[2], b[1]));
  c[1] = fsub_nc(fmul_nc(a[2], b[0]), fmul_nc(a[0], b[2]));
  c[2] = fsub_nc(fmul_nc(a[0], b[1]), fmul_nc(a[1], b[0]));
}

// Unit direction of the ray through pixel (i, j) and its intersection [t0, t1]
// with the unit cube (t0 >= 0; t1 <= t0 or a NaN: none).
__device__ __forceinline__ void pixel_ray(const RayCamera& cam, int width, int height, int i, int j, float* d,
                                          float& t0, float& t1) {
  // camera frame: f = normalize(center - eye), r = normalize(f x up), u = r x f
  float fw[3], rt[3], uu[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) fw[a] = fsub_nc(cam.center[a], cam.eye[a]);
  normalize_rn(fw);
  cross_rn(fw, cam.up, rt);
  normalize_rn(rt);
  cross_rn(rt, fw, uu);
  const float aspect = __fdiv_rn((float)width, (float)height);
  const float px = fmul_nc(
      fmul_nc(fsub_nc(__fdiv_rn(fmul_nc(2.0f, fadd_nc((float)i, 0.5f)), (float)width), 1.0f), cam.tan_h), aspect);
  const float py =
      fmul_nc(fsub_nc(1.0f, __fdiv_rn(fmul_nc(2.0f, fadd_nc((float)j, 0.5f)), (float)height)), cam.tan_h);
#pragma unroll
  for (int a = 0; a < 3; ++a) d[a] = fadd_nc(fadd_nc(fw[a], fmul_nc(px, rt[a])), fmul_nc(py, uu[a]));
  const float n = __fsqrt_rn(dot3_rn(d[0], d[1], d[2], d[0], d[1], d[2]));
#pragma unroll
  for (int a = 0; a < 3; ++a) d[a] = __fdiv_rn(d[a], n);
  // slab intersection with [0,1]^3
  t0 = 0.0f;
  t1 = INFINITY;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float inv = __fdiv_rn(1.0f, d[a]);
    const float ta = fmul_nc(fsub_nc(0.0f, cam.eye[a]), inv);
    const float tb = fmul_nc(fsub_nc(1.0f, cam.eye[a]), inv);
    t0 = fmaxf(t0, fminf(ta, tb));
    t1 = fminf(t1, fmaxf(ta, tb));
  }
}

// Sample position t_k = t0 + (k + 1/2) dt; the sample exists iff t_k < t1.
__device__ __forceinline__ float sample_t(float t0, int k, float dt) {
  return fadd_nc(t0, fmul_nc(fadd_nc((float)k, 0.5f), dt));
}

// Samples k0 .. k1 - 1 of every ray (k0, k1 multiples of 16): k0 = 0 starts the
// image, later launches go on from its (C, A).  rounds[kRenderSlots x 8 words]
// gathers, over the rays that end in this launch, the rounds of S samples that
// a ray was active for.
// COOP: the four waves of a workgroup march the same 16 rays, wave w samples
// 4 w .. 4 w + 3 of every 16 (each wave then composites all sixteen, in order):
// four times the waves for an image with few rays.
template <bool BF16, int W, int NH, typename TT, int F, int NG, bool COOP>
__global__ __launch_bounds__(256, BF16 ? 4 : 2) void k_render(
    LevelDesc ld, MlpDesc md, const BlockMeta* __restrict__ meta, const BlockRange* __restrict__ range, int block,
    const TT* __restrict__ table_all, const typename InferMlp<BF16, W, NH, NG>::w_t* __restrict__ wsrc,
    RayCamera cam, int width, int height, RenderStep rs, int k0, int k1, const float* __restrict__ tf,
    float* __restrict__ image, unsigned long long* __restrict__ rounds) {
  using M = InferMlp<BF16, W, NH, NG>;
  constexpr int SETS = 4 / NG, T = NG;
  __shared__ QueryLevel lev[kMaxLevels];
  __shared__ __align__(16) typename M::op_t opnd[M::N_SLOTS * 64];
  __shared__ __align__(16) float wout[W];
  const int64_t param_off = meta[block].param_off;
  load_query_levels(ld, F * (int)sizeof(TT), lev);
  for (int e = threadIdx.x; e < M::N_SLOTS * 64; e += 256) opnd[e] = M::operand(wsrc + param_off, md, e);
  if (threadIdx.x < W) wout[threadIdx.x] = (float)wsrc[param_off + md.off[NH] + threadIdx.x];
  __syncthreads();
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int g = lane / 16, c = lane % 16, set = g / NG, fg = g % NG;
  // a workgroup takes 8 x 8 pixels (COOP: 4 x 4)
  constexpr int TILE = COOP ? 4 : 8, KS = COOP ? 16 : 4;  // samples of a ray per pass
  __shared__ float4 col[COOP ? 2 : 1][COOP ? 16 * 16 : 1];
  const int wx = (width + TILE - 1) / TILE;
  const int i = (int)(blockIdx.x % wx) * TILE + (COOP ? 0 : (wave & 1) * 4) + (c & 3);
  const int j = (int)(blockIdx.x / wx) * TILE + (COOP ? 0 : (wave >> 1) * 4) + (c >> 2);
  const int kw = COOP ? 4 * wave : 0;
  int buf = 0;
  const bool pixel = i < width && j < height;
  float d[3], t0, t1;
  pixel_ray(cam, width, height, min(i, width - 1), min(j, height - 1), d, t0, t1);
  float C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, A = 0.0f;
  const int64_t p = (int64_t)j * width + i;
  bool done = !(pixel && t1 > t0);
  if (k0 > 0 && !done) {
    C0 = image[4 * p];
    C1 = image[4 * p + 1];
    C2 = image[4 * p + 2];
    A = image[4 * p + 3];
    done = A >= rs.alpha_stop || !(sample_t(t0, k0 - 1, rs.dt) < t1);  // it ended in an earlier launch
  }
  const bool entered = !done;
  int k_end = 0;  // sample index at which the ray was found to end
  const BlockRange br = range[block];
  const TT* tab = table_all + param_off;
  // (COOP: the waves hold the same rays in the same state, so they leave together)
  for (int k = k0; k < k1 && __any(!done); k += KS) {
    float x[T], y[T], z[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const float tk = sample_t(t0, k + kw + set + SETS * t, rs.dt);
      const bool ok = !done && tk < t1;
      x[t] = ok ? fadd_nc(cam.eye[0], fmul_nc(tk, d[0])) : 0.5f;
      y[t] = ok ? fadd_nc(cam.eye[1], fmul_nc(tk, d[1])) : 0.5f;
      z[t] = ok ? fadd_nc(cam.eye[2], fmul_nc(tk, d[2])) : 0.5f;
    }
    typename M::op_t xb[T][M::KS_IN];
    query_features<M, BF16, TT, F, T>(lev, ld.L, ld.T_mask, fg, tab, x, y, z, xb);
    const float o = M::template eval_groups<4, T>(opnd, wout, lane, xb);
    // transfer function of sample k + kw + g
    const float v = o * br.range + br.vmin;
    const float s = fminf(fmaxf((v - rs.tf_lo) * rs.tf_inv_range, 0.0f), 1.0f) * (float)(rs.n_tf - 1);
    const int ti = min((int)floorf(s), rs.n_tf - 2);
    const float w = s - (float)ti;
    const float4 a = reinterpret_cast<const float4*>(tf)[ti];
    const float4 b = reinterpret_cast<const float4*>(tf)[ti + 1];
    const float op = fminf(fmaxf(a.w + w * (b.w - a.w), 0.0f), 1.0f);
    const float alpha = 1.0f - powf(1.0f - op, rs.opacity_exp);
    const float r0 = a.x + w * (b.x - a.x), r1 = a.y + w * (b.y - a.y), r2 = a.z + w * (b.z - a.z);
    auto composite = [&](int q, float aq, float q0, float q1, float q2) {
      const bool out = !(sample_t(t0, k + q, rs.dt) < t1);
      if (!done && out) {
        done = true;
        k_end = k + q;
      }
      if (!done) {
        const float wgt = (1.0f - A) * aq;
        C0 += wgt * q0;
        C1 += wgt * q1;
        C2 += wgt * q2;
        A += wgt;
        if (A >= rs.alpha_stop) {
          done = true;
          k_end = k + q;
        }
      }
    };
    if constexpr (COOP) {
      col[buf][16 * (kw + g) + c] = make_float4(r0, r1, r2, alpha);
      __syncthreads();  // (two buffers: a wave may write the next pass before another has read this one)
#pragma unroll
      for (int q = 0; q < KS; ++q) {
        const float4 e = col[buf][16 * q + c];
        composite(q, e.w, e.x, e.y, e.z);
      }
      buf ^= 1;
    } else {
#pragma unroll
      for (int q = 0; q < KS; ++q) {
        const int from = 16 * q + c;
        composite(q, __shfl(alpha, from, 64), __shfl(r0, from, 64), __shfl(r1, from, 64), __shfl(r2, from, 64));
      }
    }
  }
  if (COOP && wave > 0) return;
  if (pixel && g == 0 && (entered || k0 == 0)) {
    image[4 * p] = C0;
    image[4 * p + 1] = C1;
    image[4 * p + 2] = C2;
    image[4 * p + 3] = A;
  }
  // rounds of the rays that ended here: one atomic per wave, over several words
  // (atomics on one address queue up)
  int cnt = g == 0 && entered && done ? k_end / rs.S + 1 : 0;
#pragma unroll
  for (int off = 1; off < 16; off <<= 1) cnt += __shfl_xor(cnt, off, 64);
  if (lane == 0 && cnt > 0)
    atomicAdd(&rounds[((blockIdx.x * 4 + wave) % kRenderSlots) * 8], (unsigned long long)cnt);
}

// ---------------------------------------------------------------------------
// Launches
// ---------------------------------------------------------------------------
// Pixels up to which four waves share a ray: below, a wave per 16 rays leaves
// SIMDs idle and the longest rays' waves finish late (16 levels, 2 x 64, mixed:
// 128^2 pixels 0.82 -> 0.56 ms, 512^2 2.07 -> 1.73 ms; 768^2 2.91 -> 3.07 ms,
// where composing 16 samples in every wave costs more than it gives).
constexpr int64_t kRenderFew = 1 << 18;
constexpr int kInferGrid = 1024;  // workgroups of the network pass over features (four per CU)

template <bool BF16, int W, int NH, typename TT, int F, int NG>
static hipError_t run_query(const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta, const BlockRange* range,
                            int block, const void* table, const void* wsrc, int64_t n, const float* coords,
                            float* out, hipStream_t s) {
  using w_t = typename InferMlp<BF16, W, NH, NG>::w_t;
  constexpr int SETS = 4 / NG;
  // few samples: as few per wave as its lane groups allow, over more waves
  if (NG > 1 && n <= kQueryFew) {
    const int64_t grid = (n + 64 * SETS - 1) / (64 * SETS);
    hipLaunchKernelGGL((k_query<BF16, W, NH, TT, F, NG, 1>), dim3((unsigned)grid), dim3(256), 0, s, ld, md, meta,
                       range, block, (const TT*)table, (const w_t*)wsrc, n, coords, out);
  } else {
    const int64_t grid = (n + 255) / 256;
    if (grid > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_query<BF16, W, NH, TT, F, NG, NG>), dim3((unsigned)grid), dim3(256), 0, s, ld, md, meta,
                       range, block, (const TT*)table, (const w_t*)wsrc, n, coords, out);
  }
  return hipGetLastError();
}

template <bool BF16, int W, int NH, typename TT, int F, int NG>
static hipError_t run_mlp_infer(const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                                const BlockRange* range, int block, const void* wsrc, int n, const void* feat,
                                int64_t plane, float* out, hipStream_t s) {
  using w_t = typename InferMlp<BF16, W, NH, NG>::w_t;
  const int grid = std::min((n + 255) / 256, kInferGrid);
  hipLaunchKernelGGL((k_mlp_infer<BF16, W, NH, TT, F, NG>), dim3(grid), dim3(256), 0, s, ld, md, meta, range, block,
                     (const w_t*)wsrc, n, (const w_t*)feat, plane, out);
  return hipGetLastError();
}

template <bool BF16, int W, int NH, typename TT, int F, int NG>
static hipError_t run_render(const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta, const BlockRange* range,
                             int block, const void* table, const void* wsrc, const RayCamera& cam, int width,
                             int height, const RenderStep& rs, int k0, int k1, const float* tf, float* image,
                             unsigned long long* rounds, hipStream_t s) {
  using w_t = typename InferMlp<BF16, W, NH, NG>::w_t;
  const bool coop = (int64_t)width * height <= kRenderFew;
  const int tile = coop ? 4 : 8;
  const int64_t grid = (int64_t)((width + tile - 1) / tile) * ((height + tile - 1) / tile);
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  if (coop)
    hipLaunchKernelGGL((k_render<BF16, W, NH, TT, F, NG, true>), dim3((unsigned)grid), dim3(256), 0, s, ld, md, meta,
                       range, block, (const TT*)table, (const w_t*)wsrc, cam, width, height, rs, k0, k1, tf, image,
                       rounds);
  else
    hipLaunchKernelGGL((k_render<BF16, W, NH, TT, F, NG, false>), dim3((unsigned)grid), dim3(256), 0, s, ld, md, meta,
                       range, block, (const TT*)table, (const w_t*)wsrc, cam, width, height, rs, k0, k1, tf, image,
                       rounds);
  return hipGetLastError();
}

// Every network and grid shape of one width (a translation unit each).
#define DVNR_QUERY_SHAPES(RUN, ...)                                                          \
  DVNR_QUERY_NH(RUN, 1, __VA_ARGS__) DVNR_QUERY_NH(RUN, 2, __VA_ARGS__) DVNR_QUERY_NH(RUN, 3, __VA_ARGS__)
#define DVNR_QUERY_NH(RUN, NN, ...)                                                           \
  if (md.n_hidden == NN) {                                                                    \
    DVNR_QUERY_F(RUN, NN, 1, __VA_ARGS__) DVNR_QUERY_F(RUN, NN, 2, __VA_ARGS__)               \
    DVNR_QUERY_F(RUN, NN, 4, __VA_ARGS__) DVNR_QUERY_F(RUN, NN, 8, __VA_ARGS__)               \
  }
#define DVNR_QUERY_F(RUN, NN, FF, ...)                              \
  if (ld.F == FF) {                                                 \
    if (md.in_dim <= 8) DVNR_QUERY_G(RUN, NN, FF, 1, __VA_ARGS__);  \
    if (md.in_dim <= 16) DVNR_QUERY_G(RUN, NN, FF, 2, __VA_ARGS__); \
    DVNR_QUERY_G(RUN, NN, FF, 4, __VA_ARGS__);                      \
  }
#define DVNR_QUERY_G(RUN, NN, FF, GG, ...)                                \
  return p == Prec::MIXED ? RUN<true, W, NN, __half, FF, GG>(__VA_ARGS__) \
                          : RUN<false, W, NN, float, FF, GG>(__VA_ARGS__)

template <int W>
hipError_t query_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta, const BlockRange* range,
                       int block, const void* table, const void* wsrc, int64_t n, const float* coords, float* out,
                       hipStream_t s) {
  DVNR_QUERY_SHAPES(run_query, ld, md, meta, range, block, table, wsrc, n, coords, out, s)
  return hipErrorInvalidValue;
}

template <int W>
hipError_t mlp_infer_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                           const BlockRange* range, int block, const void* wsrc, int n, const void* feat,
                           int64_t plane, float* out, hipStream_t s) {
  DVNR_QUERY_SHAPES(run_mlp_infer, ld, md, meta, range, block, wsrc, n, feat, plane, out, s)
  return hipErrorInvalidValue;
}

template <int W>
hipError_t render_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                        const BlockRange* range, int block, const void* table, const void* wsrc,
                        const RayCamera& cam, int width, int height, const RenderStep& rs, int k0, int k1,
                        const float* tf, float* image, unsigned long long* rounds, hipStream_t s) {
  DVNR_QUERY_SHAPES(run_render, ld, md, meta, range, block, table, wsrc, cam, width, height, rs, k0, k1, tf, image,
                    rounds, s)
  return hipErrorInvalidValue;
}

}  // namespace dvnrk
