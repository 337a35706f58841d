// Encoding backward of levels whose whole gradient table fits in LDS (gfx950).
//
// On a table of a few thousand entries a step's contributions meet on the same
// few hundred cache lines: the bin-privatized backward (k_sort.hip) adds its
// bins' boxes, or every contribution of a level whose boxes do not fit, to
// global memory, where adds to one line queue up (about 40 ns each).  Here a
// workgroup takes a chunk of a block's samples on one level, sums their
// contributions into a copy of the whole table in LDS, and adds the nonzero
// entries to the gradient at the end, in coalesced rows: a line is touched
// once per chunk instead of once per contribution.
//
// The LDS sums are 64-bit fixed point, as in the partitioned backward
// (k_scatter_part.hip; LDS float atomics run at a fraction of the rate of
// integer ones): with the chunk's largest |dL/dy| M, c contributions are
// summed in units of 2^-K with c M 2^K <= 2^62, so no sum overflows, each
// contribution is rounded far below fp32 rounding, and a chunk's sums do not
// depend on their order.  A chunk with a NaN or an infinity among its dL/dy
// adds its contributions to the gradient directly, as floats.
//
// Measured against the privatized kernel: 65,536 ordered samples on 4 levels of
// 2^11 entries x 4 features 98 -> 22 us (the finest level's boxes do not fit
// there); 4,096 samples on 4 levels of 2^12 x 2 28 -> 7 us.  Bound by the LDS
// atomics and the fixed-point conversions of a chunk, and on small steps by
// the length of its dependent passes.
#include "dvnr_device.h"

namespace dvnrk {

template <int F, int ACC, int NT>
__global__ __launch_bounds__(NT) void k_scatter_table(LevelDesc ld, int l0, int nl, int W,
                                                      const BlockMeta* __restrict__ meta,
                                                      const BlockPlan* __restrict__ plan,
                                                      const float* __restrict__ coords,
                                                      const float* __restrict__ dfeat, int64_t ls,
                                                      float* __restrict__ grad) {
  __shared__ unsigned long long acc[ACC];
  __shared__ uint32_t wmax[NT / 64];
  const int chunk = blockIdx.x % W, l = l0 + (int)(blockIdx.x / W) % nl, b = (int)(blockIdx.x / W) / nl;
  const int n = plan[b].n;
  const int a0 = (int)((int64_t)n * chunk / W), cnt = (int)((int64_t)n * (chunk + 1) / W) - a0;
  if (cnt <= 0) return;  // the whole workgroup
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int R = ld.R[l], dense = ld.dense[l];
  const float sc = ld.scale[l];
  const int nf = (dense ? R * R * R : (int)(ld.T_mask + 1)) * F;  // accumulators of the level (<= ACC)
  const int64_t base = plan[b].sample_off + a0;
  float* g = grad + meta[b].param_off + (int64_t)ld.off[l] * F;
  const float* d0 = dfeat + (int64_t)l * ls + base * F;
  for (int i = tid; i < nf; i += NT) acc[i] = 0ull;
  // largest |dL/dy| of the chunk, as bits (NaN and infinity above every number)
  uint32_t m = 0u;
  for (int i = tid; i < cnt * F; i += NT) m = max(m, __float_as_uint(d0[i]) & 0x7fffffffu);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, o, 64));
  if (lane == 0) wmax[wave] = m;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) m = max(m, wmax[i]);
  if (m == 0u) return;  // every contribution is zero
  const bool finite = m < 0x7f800000u;
  int E = 0;
  (void)frexpf(8.0f * (float)cnt * __uint_as_float(finite ? m : 0u), &E);
  const int K = max(-120, min(120, 62 - E));
  const float scale = ldexpf(1.0f, K);
  // a wave's lanes take samples from all over the chunk: neighbours of an
  // ordered sample buffer lie in one bin, and their adds would meet on the
  // same few vertices
  const int per = (cnt + 63) / 64;
  for (int i = wave; i < per; i += NT / 64) {
    const int s = lane * per + i;
    if (s >= cnt) continue;
    const float* x = coords + 3 * (base + s);
    int ix, iy, iz;
    float tx, ty, tz;
    grid_pos(x[0], sc, R, ix, tx);
    grid_pos(x[1], sc, R, iy, ty);
    grid_pos(x[2], sc, R, iz, tz);
    float d[F];
#pragma unroll
    for (int f = 0; f < F; ++f) d[f] = d0[s * F + f];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t cx = k & 1, cy = (k >> 1) & 1, cz = k >> 2;
      const uint32_t e = corner_index(dense, R, ld.T_mask, ix + cx, iy + cy, iz + cz);
      const float w = (cx ? tx : 1.0f - tx) * (cy ? ty : 1.0f - ty) * (cz ? tz : 1.0f - tz);
#pragma unroll
      for (int f = 0; f < F; ++f) {
        const float c = w * d[f];
        if (finite)
          atomicAdd(&acc[e * F + f], (unsigned long long)__float2ll_rn(c * scale));
        else
          unsafeAtomicAdd(&g[(int64_t)e * F + f], c);
      }
    }
  }
  if (!finite) return;
  __syncthreads();
  for (int i = tid; i < nf; i += NT) {
    const long long s = (long long)acc[i];
    if (s != 0) unsafeAtomicAdd(&g[i], ldexpf((float)s, -K));
  }
}

bool scatter_table_fits(const LevelDesc& ld, int l) {
  const int64_t R = ld.R[l];
  return (ld.dense[l] ? R * R * R : (int64_t)ld.T_mask + 1) * ld.F <= kTableAcc;
}

hipError_t launch_scatter_table(const LevelDesc& ld, int l0, int l1, int chunks, int n_blocks, const BlockMeta* meta,
                                const BlockPlan* plan, const float* coords, const float* dfeat, int64_t ls,
                                float* grad, hipStream_t s) {
  const int nl = l1 - l0;
  if (nl <= 0 || n_blocks <= 0) return hipSuccess;
  if (chunks < 1) return hipErrorInvalidValue;
  int64_t most = 0;  // accumulators of the largest level
  for (int l = l0; l < l1; ++l) {
    if (!scatter_table_fits(ld, l)) return hipErrorInvalidValue;
    const int64_t R = ld.R[l];
    most = std::max(most, (ld.dense[l] ? R * R * R : (int64_t)ld.T_mask + 1) * ld.F);
  }
  const int64_t grid = (int64_t)n_blocks * nl * chunks;
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  // 64 KB of accumulators: two workgroups of 512 threads share a CU; 128 KB:
  // one of 1024
#define DVNR_TAB(FF)                                                                                                 \
  case FF:                                                                                                           \
    if (most <= kTableAcc / 2)                                                                                       \
      hipLaunchKernelGGL((k_scatter_table<FF, kTableAcc / 2, 512>), dim3((unsigned)grid), dim3(512), 0, s, ld, l0,   \
                         nl, chunks, meta, plan, coords, dfeat, ls, grad);                                           \
    else                                                                                                             \
      hipLaunchKernelGGL((k_scatter_table<FF, kTableAcc, 1024>), dim3((unsigned)grid), dim3(1024), 0, s, ld, l0, nl, \
                         chunks, meta, plan, coords, dfeat, ls, grad);                                               \
    break;
  switch (ld.F) {
    DVNR_TAB(1)
    DVNR_TAB(2)
    DVNR_TAB(4)
    DVNR_TAB(8)
    default: return hipErrorInvalidValue;
  }
#undef DVNR_TAB
  return hipGetLastError();
}

}  // namespace dvnrk
