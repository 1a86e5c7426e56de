// Pieces shared by the fp32 kernels (jfa_f32.hip on the fp32 matrix instructions, jfa_f32_split.hip on the bf16 ones).  Not part of
// the C ABI.
#pragma once
#include "jfa_common.h"
#include "jfa_mfma.h"
#include "jfa_lds.h"

namespace jfa {

// x, made anew wherever this stands: kept in registers through a stage it would be spilled
__device__ inline int not_hoisted(int x) {
    asm volatile("" : "+v"(x));
    return x;
}

// exp(x).  The argument is a difference (score minus maximum or log-sum-exp) of numbers that may be much larger than it:
// scaled in one rounding together with the subtraction, and only the difference times log2(e).  (Both sides of the difference
// times log2(e) first, one vector instruction less per score: the gradients' error was 1.3 times this at scores of standard
// deviation 1 and 1.4 times at 16.)
__device__ inline float exp_f32(float x) { return fast_exp2(x * 1.4426950408889634f); }

template <int D> __device__ inline void clear(f32x16 (&acc)[D / 32]) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[db][e] = 0.0f;
}

// Store a transposed accumulator (rows = features, column = this lane's row of the output tensor).
template <int D> __device__ inline void store_row(float *dst, const f32x16 (&acc)[D / 32], float scale, int half) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4 *>(dst + db * 32 + g * 8 + half * 4) =
                make_float4(acc[db][4 * g] * scale, acc[db][4 * g + 1] * scale, acc[db][4 * g + 2] * scale, acc[db][4 * g + 3] * scale);
}

// The workgroup's next work item into `t`, false when nothing is left; ends with a barrier, so that the stage buffers
// are free.  item: number of items taken so far.
__device__ inline bool next_item(Work &t, const SmallWork &mine, bool small, int item, const Schedule &s, const int64_t *offsets,
                                 const int64_t *offsets_other, int B, int H, WorkCursor &cursor, int64_t total, int64_t *slot) {
    if (small) {   // the workgroup's items were decoded when the schedule was built
        __syncthreads();
        return item < __builtin_amdgcn_readfirstlane(mine.count) && load_work<true>(&mine.item[item], t);
    }
    const int64_t w = fetch_item(s.counter, cursor, total, slot);
    if (w < 0) return false;
    t = decode_work(s, offsets, B, H, w, offsets_other);
    return true;
}

// The kernels on the bf16 matrix instructions (jfa_f32_split.hip): blocks of kF32SplitRows queries or kF32SplitKeyRows keys
hipError_t launch_fwd_f32_split(const float *q, const float *k, const float *v, const int64_t *offsets, const int64_t *offsets_kv, bool causal,
                                int B, int H, int D, Schedule s, float *out, float *lse, int cus, hipStream_t stream);
hipError_t launch_dq_f32_split(const float *q, const float *k, const float *v, const float *out, const float *dout, const float *lse,
                               const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s,
                               float *dq, float *delta, int cus, hipStream_t stream);
hipError_t launch_dkv_f32_split(const float *q, const float *k, const float *v, const float *dout, const float *lse, const float *delta,
                                const int64_t *offsets, const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s,
                                float *dk, float *dv, int cus, hipStream_t stream);

}  // namespace jfa
