// Merge kernels for bf16 drafter tensors with KS = 4 (the streaming passes
// are in expand_eval_bf16_ks4.hip).
#include "expand_inst.hpp"

namespace ts {
template void launch_merge_t<uint16_t, 4>(const MergeParams&, int, bool, dim3, dim3, hipStream_t);
}  // namespace ts
