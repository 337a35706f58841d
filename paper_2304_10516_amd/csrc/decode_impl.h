// Fused decode of a block to its owned voxel grid (gfx950): voxel-center
// coordinates, hash-grid encoding and the MLP forward in one kernel.
//
// A workgroup of four waves decodes a brick of 16 x 4 x 4 voxels.  On each
// level the brick touches a small box of grid vertices (its cell origins are
// monotone in the voxel index); the workgroup loads the boxes of all levels
// into LDS (a wave takes every fourth level; consecutive lanes take
// consecutive x vertices: contiguous entries on dense levels, few aligned
// segments on hashed ones, whose x prime is 1), then every voxel interpolates
// its 8 corners from LDS: ~9 global loads per voxel instead of 128 gathers.
// A level whose box is larger than the direct gathers would be, or that no
// longer fits the LDS left, gathers directly, all lanes of a wave on one such
// level at a time.
//
// Lane (g, c) of a wave interpolates, for voxel column c, the levels whose
// features the MFMA forward wants from lane group g (features 8 g .. 8 g + 7,
// see infer_mlp.h), so features go from the interpolation to the matrix core
// in registers.  A wave's column has one x per lane, one y, and the four z of
// the brick: the cell in x and y and the four x-y weight products of a level
// are formed once for four voxels.  Narrow inputs (8 or 16 features) would
// leave three or two of the lane groups idle; there NG groups share a voxel's
// features and the others take other z.
//
// A workgroup keeps the network's operands in LDS and takes a run of bricks.
//
// The kernel is bound by VALU issue (a SIMD issues one wave instruction in
// four cycles; 90 % busy by the counters on the 256^3 grid of the 16-level,
// 2 x 64 model in mixed precision): 1,425 VALU instructions per wave of 64
// voxels, of which about 620 interpolate, 340 fill the boxes and 350 run the
// network.  With the boxes filled by every wave one level after the other (a
// barrier pair per level), a voxel's levels all in one lane, the features
// staged in LDS and the operands arranged by a kernel of its own it was 2,343:
// 0.96 -> 0.68 ms (24.8 G voxels/s), 64 uneven blocks 9.87 -> 7.76 ms, a
// 67x61x50 grid of the 4-level 1 x 16 fp32 model 21 -> 13 us.
#pragma once

#include <algorithm>
#include <climits>
#include <type_traits>

#include "infer_mlp.h"

namespace dvnrk {

constexpr int kBX = 16, kBY = 4, kBZ = 4;   // brick of 256 voxels
constexpr int kBoxMaxVerts = 2048;          // a larger box costs more than the brick's direct gathers
// Bricks of a workgroup: a run shares the operands' load, but a block of few
// bricks needs them on many workgroups (64 blocks of 7,000 bricks each: runs
// of 3 take 7.76 ms, of 1 7.65 ms).
constexpr int kDecodeRun = 8;               // at most
constexpr int kDecodeGrid = 8192;           // workgroups to keep: eight rounds of four per CU
constexpr int kOneWaveVerts = 512;          // (256: the 256^3 decode 0.71 instead of 0.68 ms)
constexpr int kDecodeLdsBytes = 40 * 1024;  // most LDS for boxes (three workgroups per CU and more)

template <typename TT> __device__ __forceinline__ float tload(const TT* p) { return (float)*p; }
template <> __device__ __forceinline__ float tload<__half>(const __half* p) { return __half2float(*p); }

// A level as the brick sees it.
struct BrickLevel {
  float scale;
  int R;
  uint32_t base;  // LDS address of grid vertex (0, 0, 0) (modulo 2^32: it may lie outside the box)
  int sy, sz;    // box strides in y and z, in bytes; sy == 0: no box, gather from the table
  int start;     // first entry of the box in LDS
  int nv;        // vertices of the box
  int dx, dy;
  int lo[3];     // box origin
};
typedef const __attribute__((address_space(3))) unsigned char lds_byte;

// The words of a table entry of VB bytes, read with the widest access that its
// alignment (VB, at most 16 bytes) allows.
typedef uint32_t u32x2d __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4d __attribute__((ext_vector_type(4)));
template <int VB>
struct EntryWords {
  typedef typename std::conditional<
      VB == 2, uint16_t,
      typename std::conditional<VB == 4, uint32_t, typename std::conditional<VB == 8, u32x2d, u32x4d>::type>::type>::type
      word;
  static constexpr int N = VB / (int)sizeof(word);
};

// Brick counts of a block and the factors that divide by them: for a < 2^31,
// a / d = umulhi(a, m) >> sh with the m and sh below (Granlund and Montgomery:
// m = ceil(2^(32 + sh) / d), sh = ceil(log2 d) - 1; d = 1 has m = 0).
struct FastDiv {
  uint32_t d, m, sh;
  __device__ __forceinline__ uint32_t div(uint32_t a) const { return m ? __umulhi(a, m) >> sh : a; }
};
struct BrickGrid {
  FastDiv nx, ny;  // bricks in x and y
  int n;           // bricks
  int per;         // bricks of one XCD's range
  int run;         // consecutive bricks of a workgroup
};

// Grid position of a voxel center (in (0, 1), so neither the clamp of
// grid_pos nor a floor of a negative number is needed): the same cell and fraction.
__device__ __forceinline__ void center_pos(float x, float scale, int R, int& i0, float& t) {
  const float p = fmul_nc(x, scale);
  i0 = min((int)p, R - 2);
  t = fsub_nc(p, (float)i0);
}

// Four waves per SIMD in mixed precision (128 registers; at three the 256^3
// decode takes 0.76 instead of 0.68 ms, at five it spills); fp32 issues 96
// MFMAs per 16 voxels and is bound by them.
template <bool BF16, int W, int NH, typename TT, int F, int NG>
__global__ __launch_bounds__(256, BF16 ? 4 : 2) void k_decode_fused(
    LevelDesc ld, MlpDesc md, const BlockMeta* __restrict__ meta, const BlockRange* __restrict__ range, int block,
    BrickGrid bg, const TT* __restrict__ table_all, const typename InferMlp<BF16, W, NH, NG>::w_t* __restrict__ wsrc,
    int box_entries, float* __restrict__ out) {
  using M = InferMlp<BF16, W, NH, NG>;
  constexpr int LPG = 8 / F;        // levels of a lane
  constexpr int SETS = 4 / NG;      // lane-group sets, each with z of its own
  constexpr int VB = F * (int)sizeof(TT);
  typedef typename EntryWords<VB>::word word;
  constexpr int NW = EntryWords<VB>::N;
  extern __shared__ __align__(16) unsigned char dsm[];
  TT* box = reinterpret_cast<TT*>(dsm);
  __shared__ BrickLevel lev[kMaxLevels];
  __shared__ unsigned large_boxes;  // levels (bits) whose boxes the waves fill together
  __shared__ unsigned no_boxes;     // levels (bits) that gather from the table
  __shared__ __align__(16) typename M::op_t opnd[M::N_SLOTS * 64];
  __shared__ __align__(16) float wout[W];

  // Workgroup w runs on XCD w % 8 (round-robin dispatch): each XCD takes a
  // contiguous range of bricks, so that the boxes neighbouring bricks share
  // stay in that XCD's L2 (L2 misses per decode of a 256^3 grid: 5.2 M ->
  // 1.9 M).  Any mapping is correct; this one only improves locality.
  const int first = (int)(blockIdx.x >> 3) * bg.run, xcd = (int)(blockIdx.x & 7);
  const int b0 = xcd * bg.per + first, b1 = min(xcd * bg.per + min(first + bg.run, bg.per), bg.n);
  if (b0 >= b1) return;  // the whole workgroup leaves before any barrier
  const BlockMeta bm = meta[block];
  const int nx = bm.dims[0], ny = bm.dims[1], nz = bm.dims[2];
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const int g = lane / 16, c = lane % 16;
  const TT* tab0 = table_all + bm.param_off;
  const BlockRange br = range[block];
  // the network's operands, once for the workgroup's bricks (visible after the first barrier)
  for (int e = threadIdx.x; e < M::N_SLOTS * 64; e += 256) opnd[e] = M::operand(wsrc + bm.param_off, md, e);
  if (threadIdx.x < W) wout[threadIdx.x] = (float)wsrc[bm.param_off + md.off[NH] + threadIdx.x];

#pragma unroll 1
  for (int brick = b0; brick < b1; ++brick) {
    const int by_ = (int)bg.nx.div((uint32_t)brick), bz_ = (int)bg.ny.div((uint32_t)by_);
    const int x0 = (brick - by_ * (int)bg.nx.d) * kBX, y0 = (by_ - bz_ * (int)bg.ny.d) * kBY, z0 = bz_ * kBZ;
    auto center = [](int i, int n) { return __fdiv_rn((float)i + 0.5f, (float)n); };
    // voxel centers: x of this lane's column, y and z of the brick's rows (lane
    // k % 4 computes row k; lanes past the grid take its last voxel)
    const float px = center(min(x0 + c, nx - 1), nx);
    const float rowy = center(min(y0 + (lane & 3), ny - 1), ny), rowz = center(min(z0 + (lane & 3), nz - 1), nz);

    // ---- the boxes, by lane l of the first wave for level l
    if (wave == 0) {
      const float ax0 = __shfl(px, 0, 64), ax1 = __shfl(px, 15, 64);
      const float ay0 = __shfl(rowy, 0, 64), ay1 = __shfl(rowy, 3, 64);
      const float az0 = __shfl(rowz, 0, 64), az1 = __shfl(rowz, 3, 64);
      const int l = min(lane, ld.L - 1);
      const int R = ld.R[l];
      const float sc = ld.scale[l];
      int lo[3], hi[3];
      float tt;
      center_pos(ax0, sc, R, lo[0], tt);
      center_pos(ax1, sc, R, hi[0], tt);
      center_pos(ay0, sc, R, lo[1], tt);
      center_pos(ay1, sc, R, hi[1], tt);
      center_pos(az0, sc, R, lo[2], tt);
      center_pos(az1, sc, R, hi[2], tt);
      const int dx = hi[0] - lo[0] + 2, dy = hi[1] - lo[1] + 2, dz = hi[2] - lo[2] + 2;
      // (each axis on its own first: the product may not fit 32 bits)
      const bool small = dx <= kBoxMaxVerts && dy <= kBoxMaxVerts && dz <= kBoxMaxVerts && dx * dy <= kBoxMaxVerts &&
                         dx * dy * dz <= kBoxMaxVerts;
      const int nv = small ? dx * dy * dz : 0;
      int end = lane < ld.L ? nv : 0;  // running sum over the levels
#pragma unroll
      for (int o = 1; o < kMaxLevels; o <<= 1) {
        const int p = __shfl_up(end, o, 64);
        if (lane >= o) end += p;
      }
      const bool boxed = lane < ld.L && small && end <= box_entries;
      const unsigned long long lg = __ballot(boxed && nv > kOneWaveVerts);
      const unsigned long long nb = __ballot(lane < ld.L && !boxed);
      if (lane == 0) {
        large_boxes = (unsigned)lg;
        no_boxes = (unsigned)nb;
      }
      if (lane < ld.L) {
        const int start = end - nv;
        BrickLevel b;
        b.scale = sc;
        b.R = R;
        b.sy = boxed ? dx * VB : 0;
        b.sz = boxed ? dx * dy * VB : 0;
        b.dx = dx;
        b.dy = dy;
        b.start = start;
        b.nv = boxed ? nv : 0;
        b.base = (uint32_t)(uintptr_t)(lds_byte*)box +
                 (uint32_t)VB * ((uint32_t)start -
                                 ((uint32_t)lo[0] + (uint32_t)dx * ((uint32_t)lo[1] + (uint32_t)dy * (uint32_t)lo[2])));
        b.lo[0] = lo[0];
        b.lo[1] = lo[1];
        b.lo[2] = lo[2];
        lev[lane] = b;
      }
    }
    __syncthreads();

    // ---- fill the boxes.  Up to kOneWaveVerts vertices are one wave's work: wave w
    // takes levels w, 7 - w, 8 + w, 15 - w (coarse and fine ones mixed); the
    // waves share larger boxes.
    const unsigned large = __builtin_amdgcn_readfirstlane(large_boxes);
    const unsigned no_box = __builtin_amdgcn_readfirstlane(no_boxes);
    auto fill_box = [&](int l, bool shared) {
      const int nv = __builtin_amdgcn_readfirstlane(lev[l].nv);
      if (nv == 0) return;
      const int dx = __builtin_amdgcn_readfirstlane(lev[l].dx), dy = __builtin_amdgcn_readfirstlane(lev[l].dy);
      const int lo0 = __builtin_amdgcn_readfirstlane(lev[l].lo[0]);
      const int lo1 = __builtin_amdgcn_readfirstlane(lev[l].lo[1]);
      const int lo2 = __builtin_amdgcn_readfirstlane(lev[l].lo[2]);
      const int start = __builtin_amdgcn_readfirstlane(lev[l].start);
      const int R = ld.R[l];
      const TT* tab = tab0 + (int64_t)ld.off[l] * F;
      const float rdx = __builtin_amdgcn_rcpf((float)dx), rdy = __builtin_amdgcn_rcpf((float)dy);
      const float hdx = 0.5f * rdx, hdy = 0.5f * rdy;
      // box vertex v -> table entry.  v = lx + dx (ly + dy lz) is split with
      // float reciprocals: (v + 1/2) / dx is at least 1/(2 dx) away from an
      // integer, and for v < kBoxMaxVerts the reciprocal's and the sum's
      // roundings move it by far less, so the truncation is exactly
      // floor(v / dx) (likewise for dy).
      auto fill = [&](auto un_tag, int v0, auto dense_tag) {
        constexpr int UN = decltype(un_tag)::value;
        constexpr bool DENSE = decltype(dense_tag)::value;
        uint32_t e[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          const int v = min(v0 + 64 * u + lane, nv - 1);
          const int q = (int)fmaf((float)v, rdx, hdx);
          const int lx = v - __mul24(q, dx);
          const int lz = (int)fmaf((float)q, rdy, hdy);
          const int ly = q - __mul24(lz, dy);
          const uint32_t gx = (uint32_t)(lo0 + lx), gy = (uint32_t)(lo1 + ly), gz = (uint32_t)(lo2 + lz);
          // dense levels have R^3 <= T <= 2^24 entries: 24-bit products suffice
          if constexpr (DENSE)
            e[u] = gx + __umul24((uint32_t)R, gy + __umul24((uint32_t)R, gz));
          else
            e[u] = (gx ^ (gy * 2654435761u) ^ (gz * 805459861u)) & ld.T_mask;
        }
        // all loads in flight together (the last vertex stands in past the box's
        // end), then the stores
        const word* tw = reinterpret_cast<const word*>(tab);
        word* bw = reinterpret_cast<word*>(box);
        word r[UN][NW];
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
          for (int w = 0; w < NW; ++w) r[u][w] = tw[e[u] * (uint32_t)NW + w];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          const int v = v0 + 64 * u + lane;
          if (v < nv)
#pragma unroll
            for (int w = 0; w < NW; ++w) bw[(start + v) * NW + w] = r[u][w];
        }
      };
      auto fill_level = [&](auto dense_tag) {
        if (shared) {
          for (int v0 = 128 * wave; v0 < nv; v0 += 512) fill(std::integral_constant<int, 2>{}, v0, dense_tag);
        } else if (nv > 128) {
          for (int v0 = 0; v0 < nv; v0 += 256) fill(std::integral_constant<int, 4>{}, v0, dense_tag);
        } else if (nv > 64) {
          fill(std::integral_constant<int, 2>{}, 0, dense_tag);
        } else {
          fill(std::integral_constant<int, 1>{}, 0, dense_tag);
        }
      };
      if (ld.dense[l])
        fill_level(std::true_type{});
      else
        fill_level(std::false_type{});
    };
    for (int p = 0; p < (ld.L + 3) / 4; ++p) {
      const int l = 4 * p + ((p & 1) ? 3 - wave : wave);
      if (l < ld.L && !((large >> l) & 1)) fill_box(l, false);
    }
    for (unsigned m = large; m != 0; m &= m - 1) fill_box(__builtin_ctz(m), true);
    __syncthreads();
    if (y0 + wave < ny) {  // (uniform over the wave)
      // ---- interpolation: lane (g, c), z = z0 + set + SETS t for t < NG
      const int set = g / NG, fg = g % NG;
      const float py = __shfl(rowy, wave, 64);
      float pz[NG];
#pragma unroll
      for (int t = 0; t < NG; ++t) pz[t] = __shfl(rowz, set + SETS * t, 64);
      typename M::op_t xb[NG][M::KS_IN];
#pragma unroll
      for (int j = 0; j < LPG; ++j) {
        const int l = LPG * fg + j;
        const bool live = l < ld.L;
        const uint32_t keep = live ? ~0u : 0u;
        if (j > 0) __builtin_amdgcn_sched_barrier(0);
        const BrickLevel& b = lev[live ? l : 0];
        const float sc = b.scale;
        const int R = b.R, sy = b.sy, sz = b.sz;
        int ix, iy;
        float tx, ty;
        center_pos(px, sc, R, ix, tx);
        center_pos(py, sc, R, iy, ty);
        float wxy[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) wxy[k] = ((k & 1) ? tx : 1.0f - tx) * ((k & 2) ? ty : 1.0f - ty);
        float acc[NG][F];
#pragma unroll
        for (int t = 0; t < NG; ++t)
#pragma unroll
          for (int f = 0; f < F; ++f) acc[t][f] = 0.0f;
        if (sy != 0) {
          const uint32_t b0 = b.base + (uint32_t)(VB * ix) + (uint32_t)__mul24(sy, iy);
#pragma unroll
          for (int t = 0; t < NG; ++t) {
            if (F >= 4 && t > 0) __builtin_amdgcn_sched_barrier(0);
            int iz;
            float tz;
            center_pos(pz[t], sc, R, iz, tz);
            const uint32_t v0 = b0 + (uint32_t)__mul24(sz, iz);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
              const float w = wxy[k & 3] * ((k & 4) ? tz : 1.0f - tz);
              typedef const __attribute__((address_space(3))) word lds_word;
              lds_word* v = (lds_word*)(uintptr_t)(v0 + ((k & 2) ? sy : 0) + ((k & 4) ? sz : 0)) + (k & 1) * NW;
              word e[NW];
#pragma unroll
              for (int i = 0; i < NW; ++i) e[i] = v[i];
              TT ev[F];
              __builtin_memcpy(ev, e, VB);
#pragma unroll
              for (int f = 0; f < F; ++f) acc[t][f] += w * tload(&ev[f]);
            }
          }
        }
#pragma unroll
        for (int t = 0; t < NG; ++t)
#pragma unroll
          for (int f = 0; f < F; ++f) {
            const float v = __uint_as_float(__float_as_uint(acc[t][f]) & keep);
            if constexpr (BF16)
              xb[t][0][j * F + f] = (__bf16)v;
            else
              xb[t][j * F + f] = v;
          }
      }

      // ---- levels without a box, one after the other: lane (g, c) gathers for
      // the voxel z = z0 + g (all lanes at work), and the lane groups that the
      // level's features belong to fetch them
      if (no_box != 0) {
        const float zg = __shfl(rowz, g, 64);
        for (unsigned m = no_box; m != 0; m &= m - 1) {
          const int l = __builtin_ctz(m), R = ld.R[l], dense = ld.dense[l];
          const float sc = ld.scale[l];
          const TT* tab = tab0 + (int64_t)ld.off[l] * F;
          int ix, iy, iz;
          float tx, ty, tz;
          center_pos(px, sc, R, ix, tx);
          center_pos(py, sc, R, iy, ty);
          center_pos(zg, sc, R, iz, tz);
          float acc[F];
#pragma unroll
          for (int f = 0; f < F; ++f) acc[f] = 0.0f;
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const float w = ((k & 1) ? tx : 1.0f - tx) * ((k & 2) ? ty : 1.0f - ty) * ((k & 4) ? tz : 1.0f - tz);
            const uint32_t e = corner_index(dense, R, ld.T_mask, ix + (k & 1), iy + ((k >> 1) & 1), iz + (k >> 2));
            word ew[NW];
#pragma unroll
            for (int i = 0; i < NW; ++i) ew[i] = reinterpret_cast<const word*>(tab)[e * (uint32_t)NW + i];
            TT ev[F];
            __builtin_memcpy(ev, ew, VB);
#pragma unroll
            for (int f = 0; f < F; ++f) acc[f] += w * tload(&ev[f]);
          }
          const int owner = l / LPG, at = l % LPG;
#pragma unroll
          for (int t = 0; t < NG; ++t)
#pragma unroll
            for (int f = 0; f < F; ++f) {
              const float v = __shfl(acc[f], 16 * (set + SETS * t) + c, 64);
#pragma unroll
              for (int j = 0; j < LPG; ++j)
                if (j == at && fg == owner) {
                  if constexpr (BF16)
                    xb[t][0][j * F + f] = (__bf16)v;
                  else
                    xb[t][j * F + f] = v;
                }
            }
        }
      }

      // ---- MLP forward of the four z
      const float o = M::template eval_groups<4, NG>(opnd, wout, lane, xb);
      // lane group g stores z = z0 + g
      if (x0 + c < nx && z0 + g < nz)
        out[((int64_t)(z0 + g) * ny + (y0 + wave)) * nx + x0 + c] = o * br.range + br.vmin;
    }
    __syncthreads();  // the boxes may be overwritten
  }
}

// Box entries that a brick of a block with these dims can need on the levels
// whose boxes are small enough (an axis of e voxels spans at most
// floor((e - 1) (R - 1) / n) + 2 cells), within the LDS budget.
static int decode_box_entries(const LevelDesc& ld, const int32_t* dims, int entry_bytes) {
  const int ext[3] = {kBX, kBY, kBZ};
  int64_t sum = 0;
  for (int l = 0; l < ld.L; ++l) {
    int64_t nv = 1;
    for (int a = 0; a < 3; ++a) {
      const int64_t e = std::min<int64_t>(ext[a], dims[a]);
      nv *= std::min<int64_t>((e - 1) * (ld.R[l] - 1) / dims[a] + 3, ld.R[l]);
    }
    if (nv <= kBoxMaxVerts) sum += nv;
  }
  return (int)std::min<int64_t>(sum, kDecodeLdsBytes / entry_bytes);
}

inline FastDiv fast_div(uint32_t d) {
  if (d == 1) return FastDiv{1, 0, 0};
  uint32_t sh = 0;
  while (((uint64_t)2 << sh) < d) ++sh;
  return FastDiv{d, (uint32_t)((((uint64_t)1 << (32 + sh)) + d - 1) / d), sh};
}

template <bool BF16, int W, int NH, typename TT, int F, int NG>
static hipError_t run_decode(const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta, const BlockRange* range,
                             int block, const int32_t* dims, const void* table, const void* wsrc, float* out,
                             hipStream_t s) {
  using w_t = typename InferMlp<BF16, W, NH, NG>::w_t;
  const int64_t bricks = (int64_t)((dims[0] + kBX - 1) / kBX) * ((dims[1] + kBY - 1) / kBY) *
                         ((dims[2] + kBZ - 1) / kBZ);
  if (bricks <= 0) return hipSuccess;
  if (bricks > 0x7fffffff - 7) return hipErrorInvalidValue;
  BrickGrid bg;
  bg.nx = fast_div((uint32_t)((dims[0] + kBX - 1) / kBX));
  bg.ny = fast_div((uint32_t)((dims[1] + kBY - 1) / kBY));
  bg.n = (int)bricks;
  bg.per = (int)((bricks + 7) / 8);
  bg.run = (int)std::max<int64_t>(1, std::min<int64_t>(kDecodeRun, bricks / kDecodeGrid));
  const int64_t grid = 8 * (((int64_t)bg.per + bg.run - 1) / bg.run);  // whole rounds of the 8 XCDs
  const int entries = decode_box_entries(ld, dims, F * (int)sizeof(TT));
  using M = InferMlp<BF16, W, NH, NG>;
  const size_t box_bytes = (size_t)entries * F * sizeof(TT);
  auto kern = k_decode_fused<BF16, W, NH, TT, F, NG>;
  if (box_bytes + sizeof(typename M::op_t) * M::N_SLOTS * 64 > 48 * 1024) {  // may pass 64 KB with the static arrays
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)box_bytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(256), box_bytes, s, ld, md, meta, range, block, bg,
                     (const TT*)table, (const w_t*)wsrc, entries, out);
  return hipGetLastError();
}

// Network shapes of one translation unit (one width each).
template <int W>
hipError_t decode_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                        const BlockRange* range, int block, const int32_t* dims, const void* table, const void* wsrc,
                        float* out, hipStream_t s) {
#define DVNR_DEC(NN, FF, GG)                                                                                       \
  return p == Prec::MIXED                                                                                          \
             ? run_decode<true, W, NN, __half, FF, GG>(ld, md, meta, range, block, dims, table, wsrc, out, s)      \
             : run_decode<false, W, NN, float, FF, GG>(ld, md, meta, range, block, dims, table, wsrc, out, s)
#define DVNR_DEC_G(NN, FF)                       \
  if (ld.F == FF) {                              \
    if (md.in_dim <= 8) DVNR_DEC(NN, FF, 1);     \
    if (md.in_dim <= 16) DVNR_DEC(NN, FF, 2);    \
    DVNR_DEC(NN, FF, 4);                         \
  }
#define DVNR_DEC_F(NN) \
  if (md.n_hidden == NN) { DVNR_DEC_G(NN, 1) DVNR_DEC_G(NN, 2) DVNR_DEC_G(NN, 4) DVNR_DEC_G(NN, 8) }
  DVNR_DEC_F(1)
  DVNR_DEC_F(2)
  DVNR_DEC_F(3)
#undef DVNR_DEC_F
#undef DVNR_DEC_G
#undef DVNR_DEC
  return hipErrorInvalidValue;
}

}  // namespace dvnrk
