// The marching kernels for double fields (march.h).
#include "march.h"

namespace lq {

void launch_march_f64(const LatDev& L, bool l23, int mode, const void* bufs, const void* q, void* F, double* partials,
                      FireDev* st, int k, void* stream) {
    launch_march_mode<double>(L, l23, mode, bufs, q, F, partials, st, k, (hipStream_t)stream);
}

void launch_march_batch_f64(bool l23, const MemberDev* mem, const BatchGroup& g, int wide, int k, void* stream) {
    if (wide) launch_batch_group<double, 1>(l23, mem, g, k, (hipStream_t)stream);
    else launch_batch_group<double, 0>(l23, mem, g, k, (hipStream_t)stream);
}

int march_blocks_per_cu_f64(bool l23, bool l4, int wide, bool two) {
    if (two && l23 && !l4 && wide) return blocks_per_cu<double, true, false, 1, true>();
    return blocks_per_cu_t<double>(l23, l4, wide);
}

}  // namespace lq
