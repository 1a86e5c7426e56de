// Jagged flash attention backward, bf16, head sizes 32 and 64 (paper Section 2.2).
//
//   P  = exp(S / sqrt(D) - lse),   dP = dO V^T,   dS = P o (dP - delta),   delta = rowsum(dO o O)
//   dV = P^T dO,   dQ = dS K / sqrt(D),   dK = dS^T Q / sqrt(D)
//
// The split and the operand layouts of dq_bf16_kernel / dkv_bf16_kernel (jfa_bwd_bf16.hip): 128 stationary rows per tile (short
// samples: 64, see narrow_block_rows()), 32 per wave, on the lanes; the other rows stream past them in stages of 64; no atomics on results.  At these head sizes a
// score's vector work is what counts (see jfa_fwd_narrow.hip), so there is as little of it as possible:
//   * dP's accumulators start at minus delta (dQ, D = 32) or, with V negated, at delta (dK / dV), the scores of the dK / dV
//     kernel at minus lse * sqrt(D): the stream's statistics are read from LDS straight into the accumulators, and P and dS
//     are one multiply (or multiply-add), one exponential, one multiply and the conversions;
//   * only stages that contain the sample's end or the diagonal mask, and those skip a block of 32 rows that no lane needs
//     (training step on 1024 samples of 1 to 1024 rows, H = 8, D = 64, 4494 -> 4446 us; 1000 of at most 20, H = 2: backward
//     50 -> 41);
//   * stages (and the stream's statistics) go directly to LDS, one ahead; gradients leave as whole rows.
// Workgroups per compute unit: dQ four at D = 32 and three at D = 64.  Its rows of the forward's output pass through LDS and,
// at D = 64, delta is subtracted from every dP, sixteen vector instructions more per block, which leaves registers for the third
// without any spilled: 1024 samples of 1 to 1024 rows, H = 8, 1401 us (1371 with empty blocks skipped; 1457 with the addend and
// 15 registers spilled, 1569 with two workgroups); 256 samples of 64 rows on average, H = 2, 570 tiles, 16.4 us (20.3 and 22.6:
// scratch memory costs a launch 4 us, and 512 places a second round); 64 samples of 4096 rows 1049 (1033).  D = 32 fits with the
// addend: subtracting is 6 to 10 % slower there.  dK / dV two at D = 64 and three at D = 32 (one more spills: 5 % slower at
// D = 64; at D = 32 2 % faster on that batch but 1 to 4 us slower a launch, for the scratch memory).
// H * D = 512, whole backward, microseconds before -> now: 1024 samples of 1 to 1024 rows D = 64 4100 -> 3290, D = 32
// 4840 -> 3850; 64 samples of 4096 rows D = 64 9000 -> 6940 (792 TFLOP/s), D = 32 10750 -> 8130.  A 32 x 32 block costs a SIMD
// about 44 clocks per matrix instruction (12 + 16) and 3.8 per vector instruction (72 + 64; 134 + 96 before).
// The dQ kernel runs first: it forms delta and -lse * sqrt(D) for its queries and leaves them in the two planes of `stats`.
#pragma once
#include "jfa_narrow.h"

namespace jfa {

// What both kernels wait for at the end of a stage: this wave's copies for the next one; then everyone's.
__device__ inline void narrow_end_stage() {
    asm volatile("" ::: "memory");
    wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// CROSS: `offsets` belongs to the queries, offsets_kv to the keys and values; CAUSAL: query i sees keys 0 .. i.
template <int D, int W, bool CROSS, bool CAUSAL, int DIRECT>
__global__ __launch_bounds__(64 * W, D == 64 ? (W == 4 ? 3 : 2) : 4) void dq_narrow_kernel(
    const __bf16 *__restrict__ q, const __bf16 *__restrict__ k, const __bf16 *__restrict__ v, const __bf16 *__restrict__ dout,
    const float *__restrict__ lse, const __bf16 *__restrict__ out_fwd, float *__restrict__ stats, const int64_t *__restrict__ offsets,
    const int64_t *__restrict__ offsets_kv, int B, int H, Schedule s, __bf16 *__restrict__ dq) {
    using N = Narrow<D>;
    constexpr int kKSteps = D / 16, kDBlocks = D / 32, kRows = 32 * W;   // kRows: stationary rows of a tile
    constexpr bool kSubtract = D == 64;   // delta is subtracted from every dP: as their sums' addend it takes sixteen registers
    __shared__ __attribute__((aligned(1024))) char st[kNwStages * N::kStage];   // buffer b: K at b * kStage, V behind it
    __shared__ typename NarrowWalk<CROSS, DIRECT>::Shared walk_mem;
    static_assert(sizeof(st) >= kInlineScratchInts * sizeof(int), "the stage buffers double as the scheduler's scratch");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const float scale = 1.0f / sqrtf((float)D);
    const float c = 1.4426950408889634f * scale;
    const int64_t row_stride = (int64_t)H * D;
    const int64_t sum_q = offsets[B];   // query rows; loaded once, a tile's first loads hang on it
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

        float l = 0.0f;
        const int64_t srow = (int64_t)t.head * sum_q + t.row0 + iq;   // this lane's query in `lse` and in a plane of `stats`
        char *const own = st + N::kStage + wave * 32 * N::kRow;   // the wave's rows of the forward's output pass through the second stage buffer
        bf16x8 qreg[kKSteps], doreg[kKSteps];
        if (have) {
            const int64_t off = (t.row0 + iq) * row_stride + (int64_t)t.head * D + 8 * half;
#pragma unroll
            for (int ks = 0; ks < kKSteps; ++ks) {
                qreg[ks] = *reinterpret_cast<const bf16x8 *>(q + off + 16 * ks);
                doreg[ks] = *reinterpret_cast<const bf16x8 *>(dout + off + 16 * ks);
            }
            l = lse[srow];
            if (wave_active) copier.copy_rows(out_fwd + t.row0 * row_stride + (int64_t)t.head * D, q0, Lq, own);
            if (n_stages > 0) copier.copy(kbase, vbase, 0, L, st);
        }
        if (wave == 0) walk.claim();   // overlaps with the loads in flight
        if (have) {
            wait_vm<0>();
            asm volatile("" ::: "memory");
            float delta = 0.0f;
#pragma unroll
            for (int ks = 0; ks < kKSteps; ++ks) {
                const bf16x8 o = lds_read_b128(own + at.row[ks]);
#pragma unroll
                for (int e = 0; e < 8; ++e) delta = fmaf((float)o[e], (float)doreg[ks][e], delta);
            }
            delta = pair_sum(delta);   // each lane of a pair has half of the row
            const float lse2 = l * 1.4426950408889634f;
            f32x16 acc[kDBlocks], ndelta;   // ndelta: the addend the dP products start from
#pragma unroll
            for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[db][e] = 0.0f;
#pragma unroll
            for (int e = 0; e < 16; ++e) ndelta[e] = kSubtract ? 0.0f : -delta;
            if (!kSubtract) asm volatile("" : "+v"(ndelta));   // sixteen real registers: the matrix product reads its addend from them

            const int n_full = (CAUSAL && q0 + 1 < L ? q0 + 1 : L) / kNwStageRows;   // unmasked stages of this wave; see the forward
            const int n_mine = !wave_active ? 0 : CAUSAL ? q0 / kNwStageRows + 1 : n_stages;
            auto run_block = [&](const char *kt, int j, bool masked) {
                const char *const vt = kt + N::kTile;
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    if (masked && mb == 1 && (CAUSAL && q0 + 32 < L ? q0 + 32 : L) - j * kNwStageRows <= 32) break;   // no key for any lane
                    __builtin_amdgcn_sched_barrier(0);   // the two blocks one after the other: side by side they spill
                    f32x16 sc, dp = ndelta;
#pragma unroll
                    for (int e = 0; e < 16; ++e) sc[e] = 0.0f;
#pragma unroll
                    for (int ks = 0; ks < kKSteps; ++ks) sc = mfma_32x32x16(lds_read_b128(kt + mb * 32 * N::kRow + at.row[ks]), qreg[ks], sc);
#pragma unroll
                    for (int ks = 0; ks < kKSteps; ++ks) dp = mfma_32x32x16(lds_read_b128(vt + mb * 32 * N::kRow + at.row[ks]), doreg[ks], dp);
                    if (masked) {   // keys past the end of the sample (causal: and above the diagonal) get P = 0
                        const int lim = (CAUSAL && iq + 1 < L ? iq + 1 : L) - j * kNwStageRows - mb * 32 - 4 * half;
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            if ((e >> 2) * 8 + (e & 3) >= lim) sc[e] = -INFINITY;
                    }
#pragma unroll
                    for (int e = 0; e < 16; ++e) dp[e] = (kSubtract ? dp[e] - delta : dp[e]) * fast_exp2(fmaf(sc[e], c, -lse2));
                    // dQ^T += K^T dS^T
#pragma unroll
                    for (int ts = 0; ts < 2; ++ts) {
                        const bf16x8 ds = pack_bf16(dp, 8 * ts);
                        const char *pk = kt + (mb * 32 + ts * 16) * N::kRow;
#pragma unroll
                        for (int db = 0; db < kDBlocks; ++db)
                            acc[db] = mfma_32x32x16(concat(lds_read_tr16(pk + at.tr[0][db]), lds_read_tr16(pk + at.tr[1][db])), ds, acc[db]);
                    }
                }
            };
            narrow_end_stage();   // stage 0 has landed and the second buffer is free
            const int n_plain = (CAUSAL && t.block * kRows + 1 < L ? t.block * kRows + 1 : L) / kNwStageRows;
            for (int j = 0; j < n_stages; ++j) {
                for (; !(j & 1) && j + 3 <= n_plain; j += 2) {   // two steady stages at a time, buffers 0 and 1: offsets in the instructions
                    copier.template copy<true>(kbase, vbase, (j + 1) * kNwStageRows, L, st + N::kStage);
                    if (wave_active) run_block(st, j, false);
                    narrow_end_stage();
                    copier.template copy<true>(kbase, vbase, (j + 2) * kNwStageRows, L, st);
                    if (wave_active) run_block(st + N::kStage, j + 1, false);
                    narrow_end_stage();
                }
                if (j + 1 < n_stages) copier.copy(kbase, vbase, (j + 1) * kNwStageRows, L, st + (~j & 1) * N::kStage);
                if (j < n_mine) run_block(st + (j & 1) * N::kStage, j, j >= n_full);
                narrow_end_stage();
            }
            // every wave is past the last stage's barrier and no copy is in flight
            if (i < Lq && half == 0) {   // stored here: at the top, the wait for the first stage would wait for these stores
                stats[srow] = delta;
                stats[(int64_t)H * sum_q + srow] = -l * sqrtf((float)D);
            }
            if (wave_active)
                narrow_store<D>(st + wave * 32 * N::kRow, lane, acc, scale, dq + t.row0 * row_stride + (int64_t)t.head * D, row_stride, q0, Lq);
        } else {
            __syncthreads();   // the slot is written
        }
        have = walk.next(t);
        if (!have) break;
    }
}

// CROSS: `offsets` belongs to the keys (the stationary rows), offsets_q to the queries that stream past them.  CAUSAL: key j is
// seen by queries j .. L - 1: the stream starts at the stage that holds the tile's first key.
template <int D, int W, bool CROSS, bool CAUSAL, int DIRECT>
__global__ __launch_bounds__(64 * W, D == 64 ? 2 : 3) void dkv_narrow_kernel(
    const __bf16 *__restrict__ q, const __bf16 *__restrict__ k, const __bf16 *__restrict__ v, const __bf16 *__restrict__ dout,
    const float *__restrict__ stats, const int64_t *__restrict__ offsets, const int64_t *__restrict__ offsets_q, int B, int H,
    Schedule s, __bf16 *__restrict__ dk, __bf16 *__restrict__ dv) {
    using N = Narrow<D>;
    constexpr int kKSteps = D / 16, kDBlocks = D / 32, kRows = 32 * W;   // kRows: stationary rows of a tile
    constexpr int kBuffer = N::kStage + 1024;   // Q, dO, then 64 x minus lse * sqrt(D) and 64 x delta (512 bytes; 1 KB keeps the alignment)
    __shared__ __attribute__((aligned(1024))) char st[kNwStages * kBuffer];
    __shared__ typename NarrowWalk<CROSS, DIRECT>::Shared walk_mem;
    static_assert(sizeof(st) >= kInlineScratchInts * sizeof(int), "the stage buffers double as the scheduler's scratch");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const float scale = 1.0f / sqrtf((float)D);
    const float c = 1.4426950408889634f * scale;
    const int64_t row_stride = (int64_t)H * D;
    const int64_t sum_q = CROSS ? offsets_q[B] : offsets[B];   // query rows; loaded once, a tile's first loads hang on it
    const NarrowAddresses<D> at(lane);
    const NarrowCopier<D, W> copier(wave, lane, row_stride);
    NarrowWalk<CROSS, DIRECT> walk(&walk_mem, s, offsets, offsets_q, B, H, reinterpret_cast<int *>(st));

    Work t{};
    int have = walk.small && walk.next(t);
    asm volatile("" : "+s"(have));   // a first pass with 0 only claims (known to be 0, it would be a second copy of the claim)
    for (;;) {
        __syncthreads();   // every wave has read the slot, and the previous tile's use of the stage buffers is over
        const int Lk = t.len;                      // keys of the sample
        const int L = CROSS ? t.olen : t.len;      // queries of the sample
        const int64_t qrow0 = CROSS ? t.orow0 : t.row0;
        const int k0 = t.block * kRows + wave * 32;   // first key of this wave
        const int j = k0 + col;                               // this lane's key; rows past the end repeat the last one
        const int jk = j < Lk ? j : Lk - 1;
        const bool wave_active = k0 < Lk;
        const int n_stages = have ? (L + kNwStageRows - 1) / kNwStageRows : 0;
        const int first = CAUSAL ? t.block * (kRows / kNwStageRows) : 0;   // first stage of the stream
        const __bf16 *const qbase = q + qrow0 * row_stride + (int64_t)t.head * D;
        const __bf16 *const dobase = dout + qrow0 * row_stride + (int64_t)t.head * D;
        // wave 0 copies the log-sum-exps of a stage, wave 1 the deltas
        const float *const stat_rows = stats + (int64_t)((wave == 0 ? H : 0) + t.head) * sum_q + qrow0;
        auto issue = [&](auto FULL, int jj, char *stage) {
            constexpr bool kFull = decltype(FULL)::value;
            copier.template copy<kFull>(qbase, dobase, jj * kNwStageRows, L, stage);
            if (wave < 2) {
                const int r = jj * kNwStageRows + lane;
                bd_dma4(stat_rows, 4u * (uint32_t)(kFull || r < L ? r : L - 1), stage + N::kStage + wave * 256);
            }
        };

        bf16x8 kreg[kKSteps], vreg[kKSteps];
        if (have) {
            const int64_t off = (t.row0 + jk) * row_stride + (int64_t)t.head * D + 8 * half;
#pragma unroll
            for (int ks = 0; ks < kKSteps; ++ks) {
                kreg[ks] = *reinterpret_cast<const bf16x8 *>(k + off + 16 * ks);
                vreg[ks] = *reinterpret_cast<const bf16x8 *>(v + off + 16 * ks);
            }
            if (n_stages > 0) issue(std::false_type{}, first, st + (first & 1) * kBuffer);
        }
        if (wave == 0) walk.claim();   // overlaps with the loads in flight
        if (have) {
#pragma unroll
            for (int ks = 0; ks < kKSteps; ++ks) {   // minus V: the accumulators end as delta - dP
                u32x4 x = __builtin_bit_cast(u32x4, vreg[ks]);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] ^= 0x80008000u;
                vreg[ks] = __builtin_bit_cast(bf16x8, x);
            }
            f32x16 acck[kDBlocks], accv[kDBlocks];
#pragma unroll
            for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) { acck[db][e] = 0.0f; accv[db][e] = 0.0f; }

            auto run_block = [&](const char *qt, int jj, bool masked) {
                const char *const dot = qt + N::kTile;
#pragma unroll
                for (int mb = 0; mb < 2; ++mb) {
                    if (masked && (mb == 1 ? L - jj * kNwStageRows <= 32 : CAUSAL && k0 - jj * kNwStageRows >= 32)) continue;   // no query for any lane
                    f32x16 sc, dp;
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float *stat = reinterpret_cast<const float *>(qt + N::kStage) + mb * 32 + g * 8 + half * 4;
                        const f32x4 l4 = *reinterpret_cast<const f32x4 *>(stat), d4 = *reinterpret_cast<const f32x4 *>(stat + 64);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { sc[4 * g + e] = l4[e]; dp[4 * g + e] = d4[e]; }
                    }
#pragma unroll
                    for (int ks = 0; ks < kKSteps; ++ks) sc = mfma_32x32x16(lds_read_b128(qt + mb * 32 * N::kRow + at.row[ks]), kreg[ks], sc);
#pragma unroll
                    for (int ks = 0; ks < kKSteps; ++ks) dp = mfma_32x32x16(lds_read_b128(dot + mb * 32 * N::kRow + at.row[ks]), vreg[ks], dp);
                    if (masked) {   // queries past the end of the sample (causal: and before this lane's key) get P = 0
                        const int r0 = jj * kNwStageRows + mb * 32 + 4 * half;
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int r = r0 + (e >> 2) * 8 + (e & 3);
                            if (r >= L || (CAUSAL && r < jk)) sc[e] = -INFINITY;
                        }
                    }
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        sc[e] = fast_exp2(sc[e] * c);
                        dp[e] *= sc[e];
                    }
                    // dV^T += dO^T P ;  dK^T += Q^T dS   (contraction over the 32 queries in two steps of 16)
#pragma unroll
                    for (int ts = 0; ts < 2; ++ts) {
                        const bf16x8 p = pack_bf16(sc, 8 * ts), ds = pack_bf16(dp, 8 * ts);
                        const int step = (mb * 32 + ts * 16) * N::kRow;
#pragma unroll
                        for (int db = 0; db < kDBlocks; ++db) {
                            accv[db] = mfma_32x32x16(concat(lds_read_tr16(dot + step + at.tr[0][db]), lds_read_tr16(dot + step + at.tr[1][db])), p, accv[db]);
                            acck[db] = mfma_32x32x16(concat(lds_read_tr16(qt + step + at.tr[0][db]), lds_read_tr16(qt + step + at.tr[1][db])), ds, acck[db]);
                        }
                    }
                }
            };
            // A stage without a mask, its two blocks of 32 queries in turn: the matrix instructions of block 0's scores and dP, of block
            // 1's, of block 0's gradients, of block 1's; block 0's vector work stands between the second, block 1's between the
            // third, two or four scores behind each matrix instruction, and operands are read kAhead matrix instructions ahead.
            // What a wave does between its own matrix instructions costs next to nothing; block by block the other waves of the SIMD had
            // to fill the gaps.  Microseconds, H * D = 512: 1024 samples of 1 to 1024 rows, D = 64, 1903 -> 1785 (causal 1293 -> 1249),
            // D = 32 2178 -> 2136; 64 of 4096 rows, D = 64, 4000 -> 3780.
            auto run_stage = [&](const char *qt) {
                constexpr int kS = 2 * kKSteps, kG = 4 * kDBlocks;   // matrix instructions of a block's scores and dP; of its gradients
                const char *const dot = qt + N::kTile;
                f32x16 sc[2], dp[2];
                u32x4 pw[2][2], dw[2][2];
                bf16x8 op[2 * kS + 2 * kG];
                auto statistics = [&](int mb) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const float *stat = reinterpret_cast<const float *>(qt + N::kStage) + mb * 32 + g * 8 + half * 4;
                        const f32x4 l4 = *reinterpret_cast<const f32x4 *>(stat), d4 = *reinterpret_cast<const f32x4 *>(stat + 64);
#pragma unroll
                        for (int e = 0; e < 4; ++e) { sc[mb][4 * g + e] = l4[e]; dp[mb][4 * g + e] = d4[e]; }
                    }
                };
                auto read = [&](int n) {
                    if (n < 2 * kS) {
                        const int mb = n / kS, i = n % kS;
                        op[n] = lds_read_b128((i & 1 ? dot : qt) + mb * 32 * N::kRow + at.row[i >> 1]);
                    } else {
                        const int mb = (n - 2 * kS) / kG, i = (n - 2 * kS) % kG, ts = i / (2 * kDBlocks), db = (i >> 1) % kDBlocks;
                        const char *t = (i & 1 ? qt : dot) + (mb * 32 + ts * 16) * N::kRow;
                        op[n] = concat(lds_read_tr16(t + at.tr[0][db]), lds_read_tr16(t + at.tr[1][db]));
                    }
                };
                auto multiply = [&](int n) {
                    if (n < 2 * kS) {
                        const int mb = n / kS, i = n % kS;
                        if (i & 1) dp[mb] = mfma_32x32x16(op[n], vreg[i >> 1], dp[mb]);
                        else sc[mb] = mfma_32x32x16(op[n], kreg[i >> 1], sc[mb]);
                    } else {
                        const int mb = (n - 2 * kS) / kG, i = (n - 2 * kS) % kG, ts = i / (2 * kDBlocks), db = (i >> 1) % kDBlocks;
                        if (i & 1) acck[db] = mfma_32x32x16(op[n], __builtin_bit_cast(bf16x8, dw[mb][ts]), acck[db]);
                        else accv[db] = mfma_32x32x16(op[n], __builtin_bit_cast(bf16x8, pw[mb][ts]), accv[db]);
                    }
                };
                auto weigh = [&](int mb, int g) {   // P and dS of queries 2 g and 2 g + 1 of this lane's sixteen
                    bf16x2 pr, dr;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const float x = fast_exp2(sc[mb][2 * g + e] * c);
                        pr[e] = (__bf16)x;
                        dr[e] = (__bf16)(dp[mb][2 * g + e] * x);
                    }
                    pw[mb][g >> 2][g & 3] = __builtin_bit_cast(uint32_t, pr);
                    dw[mb][g >> 2][g & 3] = __builtin_bit_cast(uint32_t, dr);
                };
                // D = 32 has 168 registers: a third spills, under the mask a second (12 bytes of scratch, backward of 256 x 4 heads of up to 400
                // rows 78.8 us, 77.7 without; 64 x 2 of up to 300 21.7 and 21.5; 1024 x 8 of up to 1024 1266 and 1258).
                constexpr int kAhead = D == 64 ? 3 : CAUSAL ? 1 : 2;
                statistics(0);
#pragma unroll
                for (int n = 0; n < kAhead; ++n) read(n);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int n = 0; n < 2 * kS + 2 * kG; ++n) {
                    if (n + kAhead < 2 * kS + 2 * kG) read(n + kAhead);
                    if (n == kS / 2) statistics(1);
                    multiply(n);
                    __builtin_amdgcn_sched_barrier(0);
                    if (n >= kS && n < 2 * kS) {
#pragma unroll
                        for (int u = 0; u < 8 / kS; ++u) weigh(0, (n - kS) * (8 / kS) + u);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (n >= 2 * kS && n < 2 * kS + kG) {
#pragma unroll
                        for (int u = 0; u < 8 / kG; ++u) weigh(1, (n - 2 * kS) * (8 / kG) + u);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            };
            // causal: the wave's 32 keys meet the diagonal in one stage, earlier ones are before all of them
            const int diagonal = CAUSAL ? k0 / kNwStageRows : 0;
            narrow_end_stage();   // the first stage has landed
            const int n_full = L / kNwStageRows;   // stages without the sample's end
            const int plain = CAUSAL ? first + kRows / kNwStageRows : 0;   // stages past the diagonal of every wave
            for (int jj = first; jj < n_stages; ++jj) {
                for (; !(jj & 1) && jj >= plain && jj + 3 <= n_full; jj += 2) {   // two steady stages at a time, buffers 0 and 1
                    issue(std::true_type{}, jj + 1, st + kBuffer);
                    if (wave_active) run_stage(st);
                    narrow_end_stage();
                    issue(std::true_type{}, jj + 2, st);
                    if (wave_active) run_stage(st + kBuffer);
                    narrow_end_stage();
                }
                if (jj + 1 < n_stages) issue(std::false_type{}, jj + 1, st + (~jj & 1) * kBuffer);
                if (wave_active && jj >= diagonal) run_block(st + (jj & 1) * kBuffer, jj, jj >= n_full || (CAUSAL && jj == diagonal));
                narrow_end_stage();
            }
            if (wave_active) {
                const int64_t base = t.row0 * row_stride + (int64_t)t.head * D;
                char *const region = st + wave * 32 * N::kRow;
                narrow_store<D>(region, lane, acck, -scale, dk + base, row_stride, k0, Lk);
                narrow_store<D>(region, lane, accv, 1.0f, dv + base, row_stride, k0, Lk);
            }
        } else {
            __syncthreads();   // the slot is written
        }
        have = walk.next(t);
        if (!have) break;
    }
}

// The instance for calls with a schedule: one of its own but where that for both walks, as the compiler has arranged it, is the faster (backward,
// us, one of its own and that for both: 1000 x 4 heads, 60 queries against 300 keys, D = 64, 149.4 and 146.9, 2000 x 2, 64 against 200, 113.5 and 112.1; 3000 x 4, 40
// against 250, D = 32, 159.2 and 158.7.  Own: D = 64, 1414 x 4 of up to 209 rows, 261.8 and 264.0; D = 32, 2000 x 2, 64 against 200, 80.5
// and 81.2).
template <int D, int W, bool CROSS> constexpr int kWithSchedule = CROSS && (D == 64 || W == 2) ? kEither : 0;

// Launchers for workgroups of W waves; DIRECT: calls without a schedule
template <int W, bool DIRECT>
hipError_t launch_dq_narrow_waves(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                                  const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, void *dq,
                                  int cus, hipStream_t stream) {
    if (causal && offsets_kv) return hipErrorInvalidValue;
#define JFA_LAUNCH_AS(DD, CROSS, CAUSAL, WALK)                                                                        \
    hipLaunchKernelGGL((dq_narrow_kernel<DD, W, CROSS, CAUSAL, WALK>), dim3(item_grid<dq_narrow_kernel<DD, W, CROSS, CAUSAL, WALK>, W == 2 ? 2 : 1>(64 * W, B, H, s, cus)), \
                       dim3(64 * W), 0, stream, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v, (const __bf16 *)dout, lse, \
                       (const __bf16 *)out, stats, offsets, offsets_kv, B, H, s, (__bf16 *)dq)
#define JFA_LAUNCH(DD, CROSS, CAUSAL) JFA_LAUNCH_AS(DD, CROSS, CAUSAL, (DIRECT ? 1 : kWithSchedule<DD, W, CROSS>))
#define JFA_CASE(DD)                                                                                         \
    case DD:                                                                                                 \
        if (offsets_kv) JFA_LAUNCH(DD, true, false);                                                         \
        else if constexpr (W == 2) return hipErrorInvalidValue;   /* see narrow_block_rows() */              \
        else if (causal) JFA_LAUNCH(DD, false, true);                                                        \
        else JFA_LAUNCH(DD, false, false);                                                                   \
        break;
    switch (D) {
        JFA_CASE(32) JFA_CASE(64)
        default: return hipErrorInvalidValue;
    }
#undef JFA_CASE
#undef JFA_LAUNCH
#undef JFA_LAUNCH_AS
    return hipGetLastError();
}

template <int W, bool DIRECT>
hipError_t launch_dkv_narrow_waves(const void *q, const void *k, const void *v, const void *dout, const float *stats, const int64_t *offsets,
                                   const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, void *dk, void *dv, int cus,
                                   hipStream_t stream) {
    if (causal && offsets_q) return hipErrorInvalidValue;
#define JFA_LAUNCH_AS(DD, CROSS, CAUSAL, WALK)                                                                        \
    hipLaunchKernelGGL((dkv_narrow_kernel<DD, W, CROSS, CAUSAL, WALK>), dim3(item_grid<dkv_narrow_kernel<DD, W, CROSS, CAUSAL, WALK>, W == 2 ? 2 : 1>(64 * W, B, H, s, cus)), \
                       dim3(64 * W), 0, stream, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v, (const __bf16 *)dout, stats, \
                       offsets, offsets_q, B, H, s, (__bf16 *)dk, (__bf16 *)dv)
#define JFA_LAUNCH(DD, CROSS, CAUSAL) JFA_LAUNCH_AS(DD, CROSS, CAUSAL, (DIRECT ? 1 : kWithSchedule<DD, W, CROSS>))
#define JFA_CASE(DD)                                                                                         \
    case DD:                                                                                                 \
        if (offsets_q) JFA_LAUNCH(DD, true, false);                                                          \
        else if constexpr (W == 2 && DD == 32) return hipErrorInvalidValue;   /* see narrow_key_rows() */    \
        else if (causal) JFA_LAUNCH(DD, false, true);                                                        \
        else JFA_LAUNCH(DD, false, false);                                                                   \
        break;
    switch (D) {
        JFA_CASE(32) JFA_CASE(64)
        default: return hipErrorInvalidValue;
    }
#undef JFA_CASE
#undef JFA_LAUNCH
#undef JFA_LAUNCH_AS
    return hipGetLastError();
}

}  // namespace jfa
