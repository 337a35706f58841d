// Choice of the fused decode, query and rendering kernels by network width
// (decode_impl.h, query_impl.h; each width is compiled in translation units
// of its own).
#include "dvnr_device.h"

namespace dvnrk {

template <int W>
hipError_t decode_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                        const BlockRange* range, int block, const int32_t* dims, const void* table, const void* wsrc,
                        float* out, hipStream_t s);
template <int W>
hipError_t query_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta, const BlockRange* range,
                       int block, const void* table, const void* wsrc, int64_t n, const float* coords, float* out,
                       hipStream_t s);
template <int W>
hipError_t mlp_infer_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                           const BlockRange* range, int block, const void* wsrc, int n, const void* feat,
                           int64_t plane, float* out, hipStream_t s);
template <int W>
hipError_t render_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                        const BlockRange* range, int block, const void* table, const void* wsrc,
                        const RayCamera& cam, int width, int height, const RenderStep& rs, int k0, int k1,
                        const float* tf, float* image, unsigned long long* rounds, hipStream_t s);

#define DVNR_BY_WIDTH(FN, ...)          \
  switch (md.width) {                   \
    case 16: return FN<16>(__VA_ARGS__); \
    case 32: return FN<32>(__VA_ARGS__); \
    case 64: return FN<64>(__VA_ARGS__); \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch_decode_fused(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                               const BlockRange* range, int block, const int32_t* dims, const void* table,
                               const void* wsrc, float* out, hipStream_t s) {
  DVNR_BY_WIDTH(decode_width, p, ld, md, meta, range, block, dims, table, wsrc, out, s)
}

hipError_t launch_query(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta, const BlockRange* range,
                        int block, const void* table, const void* wsrc, int64_t n, const float* coords, float* out,
                        hipStream_t s) {
  if (n <= 0) return hipSuccess;
  DVNR_BY_WIDTH(query_width, p, ld, md, meta, range, block, table, wsrc, n, coords, out, s)
}

hipError_t launch_mlp_infer(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                            const BlockRange* range, int block, const void* wsrc, int n, const void* feat,
                            int64_t plane, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  DVNR_BY_WIDTH(mlp_infer_width, p, ld, md, meta, range, block, wsrc, n, feat, plane, out, s)
}

hipError_t launch_render(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                         const BlockRange* range, int block, const void* table, const void* wsrc,
                         const RayCamera& cam, int width, int height, const RenderStep& rs, int k0, int k1,
                         const float* tf, float* image, unsigned long long* rounds, hipStream_t s) {
  DVNR_BY_WIDTH(render_width, p, ld, md, meta, range, block, table, wsrc, cam, width, height, rs, k0, k1, tf, image,
                rounds, s)
}

}  // namespace dvnrk
