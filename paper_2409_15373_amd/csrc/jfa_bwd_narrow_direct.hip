// Jagged flash attention backward, bf16, head sizes 32 and 64: the kernels of calls without a schedule.  These have at most a 128-row
// block per compute unit, far from where shorter blocks pay: four waves per workgroup always (see narrow_block_rows(), narrow_key_rows()).
#include "jfa_bwd_narrow_kernels.h"

namespace jfa {

hipError_t launch_dq_narrow_direct(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                                   const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, void *dq,
                                   int cus, hipStream_t stream) {
    return launch_dq_narrow_waves<4, true>(q, k, v, out, dout, lse, stats, offsets, offsets_kv, causal, B, H, D, s, dq, cus, stream);
}

hipError_t launch_dkv_narrow_direct(const void *q, const void *k, const void *v, const void *dout, const float *stats, const int64_t *offsets,
                                    const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, void *dk, void *dv, int cus,
                                    hipStream_t stream) {
    return launch_dkv_narrow_waves<4, true>(q, k, v, dout, stats, offsets, offsets_q, causal, B, H, D, s, dk, dv, cus, stream);
}

}  // namespace jfa
