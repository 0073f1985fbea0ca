// The marching kernels for float fields (march.h).
#include "march.h"

namespace lq {

void launch_march_f32(const LatDev& L, bool l23, int mode, const void* bufs, const void* q, void* F, double* partials,
                      FireDev* st, int k, void* stream) {
    launch_march_mode<float>(L, l23, mode, bufs, q, F, partials, st, k, (hipStream_t)stream);
}

void launch_march_batch_f32(bool l23, const MemberDev* mem, const BatchGroup& g, int wide, int k, void* stream) {
    if (wide) launch_batch_group<float, 1>(l23, mem, g, k, (hipStream_t)stream);
    else launch_batch_group<float, 0>(l23, mem, g, k, (hipStream_t)stream);
}

int march_blocks_per_cu_f32(bool l23, bool l4, int wide) { return blocks_per_cu_t<float>(l23, l4, wide); }

}  // namespace lq
