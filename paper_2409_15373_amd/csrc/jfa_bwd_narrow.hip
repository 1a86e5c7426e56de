// Jagged flash attention backward, bf16, head sizes 32 and 64: the kernels with four waves per workgroup, and which of them a
// call takes.  The two-wave ones (jfa_bwd_narrow_short.hip) and those without a schedule (jfa_bwd_narrow_direct.hip) are files of
// their own: each takes as long to compile as these.
#include "jfa_bwd_narrow_kernels.h"

namespace jfa {

hipError_t launch_dq_narrow(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                            const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, int block_rows,
                            void *dq, int cus, hipStream_t stream) {
    if (block_rows == kNarrowShortBlockRows)
        return launch_dq_narrow_short(q, k, v, out, dout, lse, stats, offsets, offsets_kv, causal, B, H, D, s, dq, cus, stream);
    if (block_rows != kNarrowBlockRows) return hipErrorInvalidValue;
    if (s.direct_blocks)
        return launch_dq_narrow_direct(q, k, v, out, dout, lse, stats, offsets, offsets_kv, causal, B, H, D, s, dq, cus, stream);
    return launch_dq_narrow_waves<4, false>(q, k, v, out, dout, lse, stats, offsets, offsets_kv, causal, B, H, D, s, dq, cus, stream);
}

hipError_t launch_dkv_narrow(const void *q, const void *k, const void *v, const void *dout, const float *stats, const int64_t *offsets,
                             const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, int block_rows, void *dk, void *dv,
                             int cus, hipStream_t stream) {
    if (block_rows == kNarrowShortBlockRows)
        return launch_dkv_narrow_short(q, k, v, dout, stats, offsets, offsets_q, causal, B, H, D, s, dk, dv, cus, stream);
    if (block_rows != kNarrowBlockRows) return hipErrorInvalidValue;
    if (s.direct_blocks)
        return launch_dkv_narrow_direct(q, k, v, dout, stats, offsets, offsets_q, causal, B, H, D, s, dk, dv, cus, stream);
    return launch_dkv_narrow_waves<4, false>(q, k, v, dout, stats, offsets, offsets_q, causal, B, H, D, s, dk, dv, cus, stream);
}

}  // namespace jfa
