// Volume rendering (query_impl.h) of networks of width 16.
#include "query_impl.h"

namespace dvnrk {

template hipError_t render_width<16>(Prec, const LevelDesc&, const MlpDesc&, const BlockMeta*, const BlockRange*, int,
                                     const void*, const void*, const RayCamera&, int, int, const RenderStep&, int, int,
                                     const float*, float*, unsigned long long*, hipStream_t);

}  // namespace dvnrk
