// Decode attention kernels with 4 wavefronts per workgroup, 4-bit codes, up to four query heads.
#include "lq_attn_mfma.h"

namespace lq {
template hipError_t launch_mfma_t<4, 4, 1>(const Shape&, const AttnParams&, const SeqArg*, dim3, hipStream_t);
}  // namespace lq
