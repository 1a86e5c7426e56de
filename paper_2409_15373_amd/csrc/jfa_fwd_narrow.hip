// Jagged flash attention forward, bf16, head sizes 32 and 64 (paper Section 2.1).
//
// Same mathematics and operand layouts as fwd_bf16_kernel: work item = (sample, head, 128 queries), four waves of 32 (short
// samples: 64 queries, two waves; see narrow_block_rows()), transposed score tile S^T = K Q^T (a lane owns one query), O^T += V^T P^T with V^T from the transposing read.
// A score costs the same vector work at every head size and a half or a quarter of the matrix work of D = 128, and the two
// hardly overlap on a SIMD (a stage of 64 keys takes a wave's SIMD 1070 clocks at D = 64, 720 at D = 32: about 44 per
// matrix instruction and 3.8 per vector instruction), so vector instructions are what bounds these sizes, and on short
// samples a tile's start-up:
//   * exponentials are taken against a reference maximum per query that is left alone while it does (the maximum over the
//     first 64 keys at first): a score is one multiply-add, one exponential and half of a conversion and of a row-sum step,
//     with no running maximum.  A stage in which a lane's 32 probabilities add up to 2^8 (kStale; so surely one with a
//     probability of 2^8, and surely none whose probabilities are all below 2^3) is taken again maximum first;
//   * stages go directly to LDS, one ahead, into unpadded swizzled buffers (jfa_narrow.h): no staging registers, no LDS
//     stores, one barrier per stage;
//   * three (D = 64) or four workgroups per compute unit, which are not in step, fill each other's start-up (one more of
//     either spills: equal on long samples, 5 % slower on short ones); the next item is claimed while the first loads
//     travel; outputs leave as whole rows; the claim and the stage are not copied over the kernel (20 KB of instructions;
//     at 42 KB, with three buffers and a copy of the stage for each, a tile's start took half as long again).
// H * D = 512, microseconds before -> now: 1024 samples of 1 to 1024 rows D = 64 1208 -> 1098, D = 32 1600 -> 1432;
// 64 samples of 4096 rows D = 64 2468 -> 2255 (975 TFLOP/s), D = 32 3328 -> 2905; 1024 of 512 rows D = 64 875 -> 786.
// (A reference fixed for the whole tile, redone where its row sum passes 2^62: D = 64 1080, 2178 and 768, D = 32 as now; but
// the largest probability of a row is then rounded to bf16 instead of 1, which shows at large scores, and values above 2^65
// can overflow.)
#include "jfa_narrow.h"

namespace jfa {

// Sum of a lane's 32 probabilities of a stage from which on the reference maximum is stale.
constexpr float kStale = 0x1p8f;

// CROSS: keys and values are the rows of a second offsets array; CAUSAL: query i sees keys 0 .. i.  See fwd_bf16_kernel.
template <int D, int W, bool CROSS, bool CAUSAL, int DIRECT>
__global__ __launch_bounds__(64 * W, D == 64 ? (W == 4 ? 3 : 2) : 4) void fwd_narrow_kernel(
    const __bf16 *__restrict__ q, const __bf16 *__restrict__ k, const __bf16 *__restrict__ v, const int64_t *__restrict__ offsets,
    const int64_t *__restrict__ offsets_kv, int B, int H, Schedule s, __bf16 *__restrict__ out, float *__restrict__ lse) {
    using N = Narrow<D>;
    constexpr int kKSteps = D / 16, kDBlocks = D / 32, kRows = 32 * W;   // kRows: queries of a tile
    __shared__ __attribute__((aligned(1024))) char st[kNwStages * N::kStage];   // buffer b: K at b * kStage, V behind it
    __shared__ typename NarrowWalk<CROSS, DIRECT>::Shared walk_mem;
    static_assert(sizeof(st) >= kInlineScratchInts * sizeof(int), "the stage buffers double as the scheduler's scratch");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const float c = 1.4426950408889634f / sqrtf((float)D);   // log2(e) / sqrt(D): exp(x / sqrt(D)) = exp2(c x)
    const float tau = 8.0f / c;                              // a factor of 2^8
    const int64_t row_stride = (int64_t)H * D;
    const int64_t sum_B = offsets[B];
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
    const NarrowAddresses<D> at(lane);
    const NarrowCopier<D, W> copier(wave, lane, row_stride);
    NarrowWalk<CROSS, DIRECT> walk(&walk_mem, s, offsets, offsets_kv, B, H, reinterpret_cast<int *>(st));

    Work t{};
    int have = walk.small && walk.next(t);
    asm volatile("" : "+s"(have));   // a first pass with 0 only claims (known to be 0, it would be a second copy of the claim)
    for (;;) {
        __syncthreads();   // every wave has read the slot, and the previous tile's use of the stage buffers is over
        const int Lq = t.len;                      // queries of the sample
        const int L = CROSS ? t.olen : t.len;      // keys of the sample
        const int64_t krow0 = CROSS ? t.orow0 : t.row0;
        const int q0 = t.block * kRows + wave * 32;   // first query of this wave
        const int i = q0 + col;                               // this lane's query; rows past the end repeat the last one
        const int iq = i < Lq ? i : Lq - 1;
        const bool wave_active = q0 < Lq;
        const int Lc = CAUSAL && (t.block + 1) * kRows < L ? (t.block + 1) * kRows : L;   // keys this tile needs
        const int n_stages = have ? (Lc + kNwStageRows - 1) / kNwStageRows : 0;
        const __bf16 *const kbase = k + krow0 * row_stride + (int64_t)t.head * D;
        const __bf16 *const vbase = v + krow0 * row_stride + (int64_t)t.head * D;
        __bf16 *const obase = out + t.row0 * row_stride + (int64_t)t.head * D;
        float *const lse_i = lse + (int64_t)t.head * sum_B + t.row0 + i;

        bf16x8 qreg[kKSteps];
        if (n_stages > 0) {
            const __bf16 *qrow = q + (t.row0 + iq) * row_stride + (int64_t)t.head * D + 8 * half;
#pragma unroll
            for (int ks = 0; ks < kKSteps; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 16 * ks);
            copier.copy(kbase, vbase, 0, L, st);
        }
        if (wave == 0) walk.claim();   // overlaps with the loads in flight
        if (CROSS && have && L == 0 && i < Lq) {   // no keys: an empty softmax, out = 0 and lse = -inf
            __bf16 *orow = obase + i * row_stride + half * (D / 2);
#pragma unroll
            for (int e = 0; e < D / 2; e += 8) *reinterpret_cast<u32x4 *>(orow + e) = u32x4{0, 0, 0, 0};
            if (half == 0) *lse_i = -INFINITY;
        }
        if (n_stages > 0) {
            f32x16 o[kDBlocks];
            float m = -INFINITY, lsum = 0.0f;   // reference maximum (raw scores) of this lane's query; its share of the row sum
#pragma unroll
            for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[db][e] = 0.0f;

            // stages whose keys all exist and, if causal, lie at or below the wave's first query need no mask; if causal, the
            // wave's 32 queries meet the diagonal in one stage and the later ones are above it
            const int n_full = (CAUSAL && q0 + 1 < L ? q0 + 1 : L) / kNwStageRows;
            const int n_mine = !wave_active ? 0 : CAUSAL ? q0 / kNwStageRows + 1 : n_stages;

            // One stage.  maximum_first: a reference that the stage's largest score exceeds by more than 2^8 is raised to it, with
            // rescaling, before the exponentials are taken (a tile's first stage sets the reference that way).  Otherwise they
            // are taken against the reference as it is; if their sum says that it may be stale, once more maximum first, and so
            // in all the tile's later stages of this wave: scores that rise that far do so again.  The flags are the same in
            // every lane.  (`raise` is false by itself in the steady stages: a test of maximum_first between the score products
            // and the exponentials keeps them from overlapping, 3 to 5 % of the kernel.)
            bool maximum_first = true;
            auto run_block = [&](const char *kt, bool raise, bool masked, int j) {
                const char *const vt = kt + N::kTile;
                f32x16 a[2];
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
#pragma unroll
                    for (int e = 0; e < 16; ++e) a[mb][e] = 0.0f;
#pragma unroll
                    for (int ks = 0; ks < kKSteps; ++ks)
                        a[mb] = mfma_32x32x16(lds_read_b128(kt + mb * 32 * N::kRow + at.row[ks]), qreg[ks], a[mb]);
                }
                if (masked) {   // keys past the end of the sample (causal: and above the diagonal)
                    const int lim = (CAUSAL && iq + 1 < L ? iq + 1 : L) - j * kNwStageRows - 4 * half;
#pragma unroll
                    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            if (mb * 32 + (e >> 2) * 8 + (e & 3) >= lim) a[mb][e] = -INFINITY;
                }
                // Probabilities, rounded to bf16 (the values the second product and the row sum use).
                u32x4 pw[4];
                float stage_sum;
                for (;;) {
                    if (raise) {
                        float mx = -INFINITY;
#pragma unroll
                        for (int e = 0; e < 16; ++e) mx = fmaxf(fmaxf(mx, a[0][e]), a[1][e]);
                        mx = pair_max(mx);
                        if (__builtin_amdgcn_ballot_w64(mx > m + tau) != 0) {
                            const float n = fmaxf(m, mx);
                            const float alpha = fast_exp2((m - n) * c);   // exp2(-inf) = 0 in the first stage
                            m = n;
                            lsum *= alpha;
#pragma unroll
                            for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
                                for (int e = 0; e < 16; ++e) o[db][e] *= alpha;
                        }
                    }
                    const float mc = m * c;
                    float part[2] = {0.0f, 0.0f};
#pragma unroll
                    for (int ts = 0; ts < 4; ++ts)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            bf16x2 pr;
                            pr[0] = (__bf16)fast_exp2(fmaf(a[ts >> 1][8 * (ts & 1) + 2 * e], c, -mc));
                            pr[1] = (__bf16)fast_exp2(fmaf(a[ts >> 1][8 * (ts & 1) + 2 * e + 1], c, -mc));
                            part[ts & 1] = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, part[ts & 1], false);
                            pw[ts][e] = __builtin_bit_cast(uint32_t, pr);
                        }
                    stage_sum = part[0] + part[1];
                    if (raise || __builtin_amdgcn_ballot_w64(!(stage_sum < kStale)) == 0) break;
                    raise = maximum_first = true;
                }
                lsum += stage_sum;
                // O^T += V^T P^T.  Slot e of a 16-key step is key 8 (e / 4) + 4 half + e % 4.
#pragma unroll
                for (int ts = 0; ts < 4; ++ts)
#pragma unroll
                    for (int db = 0; db < kDBlocks; ++db) {
                        const char *pv = vt + ts * 16 * N::kRow;
                        o[db] = mfma_32x32x16(concat(lds_read_tr16(pv + at.tr[0][db]), lds_read_tr16(pv + at.tr[1][db])), __builtin_bit_cast(bf16x8, pw[ts]), o[db]);
                    }
            };
            // The copies of stage j + 1 go into the other buffer, which stage j - 1 has released, while stage j is computed.
            auto end_stage = [&]() {
                asm volatile("" ::: "memory");
                wait_vm<0>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            };
            end_stage();   // stage 0 has landed
            // stages unmasked for every wave of the tile (a causal tile's first wave has the fewest)
            const int n_plain = (CAUSAL && t.block * kRows + 1 < L ? t.block * kRows + 1 : L) / kNwStageRows;
            for (int j = 0; j < n_stages; ++j) {
                for (; (j & 1) && j + 3 <= n_plain && !maximum_first; j += 2) {   // two steady stages at a time: buffers 1 and 0, offsets in the instructions
                    copier.template copy<true>(kbase, vbase, (j + 1) * kNwStageRows, L, st);
                    if (wave_active) run_block(st + N::kStage, false, false, j);
                    end_stage();
                    copier.template copy<true>(kbase, vbase, (j + 2) * kNwStageRows, L, st + N::kStage);
                    if (wave_active) run_block(st, false, false, j + 1);
                    end_stage();
                }
                char *const here = st + (j & 1) * N::kStage, *const other = st + (~j & 1) * N::kStage;
                if (j + 1 < n_stages) copier.copy(kbase, vbase, (j + 1) * kNwStageRows, L, other);
                if (j < n_mine) run_block(here, maximum_first, j >= n_full, j);
                if (j == 0) maximum_first = false;
                end_stage();
            }

            // ---- normalise and store: every wave is past the last stage's barrier and no copy is in flight ----
            const float l_total = pair_sum(lsum);
            if (wave_active) {
                narrow_store<D>(st + wave * 32 * N::kRow, lane, o, 1.0f / l_total, obase, row_stride, q0, Lq);
                if (i < Lq && half == 0) *lse_i = (m * c + fast_log2(l_total)) * 0.6931471805599453f;
            }
        } else {
            __syncthreads();   // the slot is written
        }
        have = walk.next(t);
        if (!have) break;
    }
}

hipError_t launch_fwd_narrow(const void *q, const void *k, const void *v, const int64_t *offsets, const int64_t *offsets_kv, bool causal,
                             int B, int H, int D, Schedule s, int block_rows, void *out, float *lse, int cus, hipStream_t stream) {
    if (causal && offsets_kv) return hipErrorInvalidValue;
#define JFA_LAUNCH_AS(DD, W, CROSS, CAUSAL, DIRECT)                                                                \
    hipLaunchKernelGGL((fwd_narrow_kernel<DD, W, CROSS, CAUSAL, DIRECT>), dim3(item_grid<fwd_narrow_kernel<DD, W, CROSS, CAUSAL, DIRECT>, W == 2 ? 2 : 1>(64 * W, B, H, s, cus)), \
                       dim3(64 * W), 0, stream, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v, offsets, offsets_kv, B, H, s, \
                       (__bf16 *)out, lse)
#define JFA_LAUNCH(DD, W, CROSS, CAUSAL)                                                                     \
    do {                                                                                                     \
        if (s.direct_blocks) JFA_LAUNCH_AS(DD, W, CROSS, CAUSAL, 1);                                         \
        else JFA_LAUNCH_AS(DD, W, CROSS, CAUSAL, 0);                                                         \
    } while (0)
#define JFA_CASE(DD, W)                                                                                      \
    case DD * 1000 + 32 * W:                                                                                 \
        if (offsets_kv) JFA_LAUNCH(DD, W, true, false);                                                      \
        else if (causal) JFA_LAUNCH(DD, W, false, true);                                                     \
        else JFA_LAUNCH(DD, W, false, false);                                                                \
        break;
// Cross attention only, and always with a schedule: see narrow_block_rows().  At D = 32 the instance that holds both walks is the faster
// as the compiler has arranged it (3000 x 4 heads, 40 queries against 250 keys, 56.9 -> 56.0 us).
#define JFA_SHORT_CASE(DD)                                                                                   \
    case DD * 1000 + kNarrowShortBlockRows:                                                                  \
        if (!offsets_kv) return hipErrorInvalidValue;                                                        \
        JFA_LAUNCH_AS(DD, 2, true, false, (DD == 32 ? kEither : 0));                                         \
        break;
    switch (D * 1000 + block_rows) {
        JFA_SHORT_CASE(32) JFA_CASE(32, 4) JFA_SHORT_CASE(64) JFA_CASE(64, 4)
        default: return hipErrorInvalidValue;
    }
#undef JFA_SHORT_CASE
#undef JFA_CASE
#undef JFA_LAUNCH
#undef JFA_LAUNCH_AS
    return hipGetLastError();
}

}  // namespace jfa
