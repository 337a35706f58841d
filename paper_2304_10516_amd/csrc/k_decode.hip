// Choice of the fused decode kernel by network width (decode_impl.h; each
// width is compiled in a translation unit of its own).
#include "dvnr_device.h"

namespace dvnrk {

template <int W>
hipError_t decode_width(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                        const BlockRange* range, int block, const int32_t* dims, const void* table, const void* wsrc,
                        float* out, hipStream_t s);
extern template hipError_t decode_width<16>(Prec, const LevelDesc&, const MlpDesc&, const BlockMeta*,
                                            const BlockRange*, int, const int32_t*, const void*, const void*, float*,
                                            hipStream_t);
extern template hipError_t decode_width<32>(Prec, const LevelDesc&, const MlpDesc&, const BlockMeta*,
                                            const BlockRange*, int, const int32_t*, const void*, const void*, float*,
                                            hipStream_t);
extern template hipError_t decode_width<64>(Prec, const LevelDesc&, const MlpDesc&, const BlockMeta*,
                                            const BlockRange*, int, const int32_t*, const void*, const void*, float*,
                                            hipStream_t);

hipError_t launch_decode_fused(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                               const BlockRange* range, int block, const int32_t* dims, const void* table,
                               const void* wsrc, float* out, hipStream_t s) {
  switch (md.width) {
    case 16: return decode_width<16>(p, ld, md, meta, range, block, dims, table, wsrc, out, s);
    case 32: return decode_width<32>(p, ld, md, meta, range, block, dims, table, wsrc, out, s);
    case 64: return decode_width<64>(p, ld, md, meta, range, block, dims, table, wsrc, out, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace dvnrk
