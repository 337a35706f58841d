// Queries (query_impl.h) of networks of width 32.
#include "query_impl.h"

namespace dvnrk {

template hipError_t query_width<32>(Prec, const LevelDesc&, const MlpDesc&, const BlockMeta*, const BlockRange*, int,
                                    const void*, const void*, int64_t, const float*, float*, hipStream_t);
template hipError_t mlp_infer_width<32>(Prec, const LevelDesc&, const MlpDesc&, const BlockMeta*, const BlockRange*,
                                        int, const void*, int, const void*, int64_t, float*, hipStream_t);

}  // namespace dvnrk
