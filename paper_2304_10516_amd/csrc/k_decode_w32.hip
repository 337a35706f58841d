// Fused decode (decode_impl.h) of networks of width 32.
#include "decode_impl.h"

namespace dvnrk {

template hipError_t decode_width<32>(Prec p, const LevelDesc& ld, const MlpDesc& md, const BlockMeta* meta,
                                     const BlockRange* range, int block, const int32_t* dims, const void* table,
                                     const void* wsrc, float* out, hipStream_t s);

}  // namespace dvnrk
