// Pieces shared by the direct-to-LDS kernels for head sizes 32 and 64 (jfa_fwd_narrow.hip, jfa_bwd_narrow.hip).  Not part
// of the C ABI.
#pragma once
#include "jfa_common.h"
#include "jfa_lds.h"
#include "jfa_mfma.h"

namespace jfa {

constexpr int kNwStageRows = 64;   // streamed rows per LDS stage
constexpr int kNwStages = 2;       // stage buffers; stage j lives in buffer j % 2, copies run one stage ahead

// A streamed tile: 64 rows of D bf16, unpadded, row r's 16-byte chunk ch at r * kRow + ((ch ^ swz(r)) << 4).  A 256-byte line
// of the 64-bank LDS holds two rows (D = 64) or four (D = 32).  The 16-byte row reads take 16 consecutive rows at one
// chunk index: the rows that share a position in the line (8 or 4 of them) get different chunks.  The transposing reads
// take 64 bytes of 4 consecutive rows: at D = 64 rows r and r + 2 share a position and differ in bit 2 of the chunk, i.e.
// in the 64-byte group; at D = 32 the four rows are one line.  Rows 16 apart have the same swizzle.
template <int D>
struct Narrow {
    static_assert(D == 32 || D == 64, "head sizes of these kernels");
    static constexpr int kRow = D * 2;
    static constexpr int kChunks = D / 8;
    static constexpr int kTile = kNwStageRows * kRow;
    static constexpr int kStage = 2 * kTile;                  // the two streamed tensors of a stage
    static constexpr int kRowsPerCopy = 64 / kChunks;         // one copy instruction moves 64 lanes x 16 bytes
    __device__ static inline int swz(int r) { return D == 64 ? ((r & 2) << 1) | ((r >> 2) & 3) : (r >> 2) & 3; }
};

// Lane addresses inside a tile.  row: chunk 2 ks + half of row `col` (+ 32 per block of 32 rows: add 32 * kRow).
// tr: element e of the transposing read is row 4 half + (lane & 15) / 4 + 8 h2, features 32 db + 16 ((lane >> 4) & 1) + ...
template <int D>
struct NarrowAddresses {
    int row[D / 16], tr[2][D / 32];
    __device__ inline NarrowAddresses(int lane) {
        using N = Narrow<D>;
        const int col = lane & 31, half = lane >> 5;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) row[ks] = col * N::kRow + (((2 * ks + half) ^ N::swz(col)) << 4);
        const int r = half * 4 + ((lane & 15) >> 2);
        const int chunk = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1), byte = (lane & 1) * 8;
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
                tr[h2][db] = (r + 8 * h2) * N::kRow + (((db * 4 + chunk) ^ N::swz(r + 8 * h2)) << 4) + byte;
    }
};

// Copies of a wave: one instruction moves kRowsPerCopy rows, lane l chunk l % kChunks of row l / kChunks of them.  What a lane
// fetches depends on its row modulo 16 only (the swizzle), so that the lane offsets of 16 rows are kept for the whole kernel
// and everything else is in the scalar base.  They fit 32 bits while H * D <= 2^24; wider rows take 64-bit addresses.
// Rows past the end repeat the last row (masked by the caller).
template <int D, int W>   // W: waves of the workgroup
struct NarrowCopier {
    using N = Narrow<D>;
    static constexpr int kWaveRows = kNwStageRows / W;    // rows of a stage that one wave copies
    static constexpr int kPer16 = 16 / N::kRowsPerCopy;   // instructions for 16 rows
    uint32_t off[kPer16];
    int wave, lane;
    int64_t row_stride;
    __device__ inline NarrowCopier(int wave_, int lane_, int64_t row_stride_) : wave(wave_), lane(lane_), row_stride(row_stride_) {
#pragma unroll
        for (int u = 0; u < kPer16; ++u) off[u] = lane_offset(u * N::kRowsPerCopy + lane / N::kChunks, 16);
    }
    __device__ inline int chunk_of(int r) const { return (lane % N::kChunks) ^ N::swz(r); }
    __device__ inline uint32_t lane_offset(int r, int n) const { return 2u * ((r < n ? r : n - 1) * (uint32_t)row_stride + (chunk_of(r) << 3)); }
    // `kRows` rows (a multiple of 16) from `base` on, the first `n` of which exist -> dst, laid out as rows of a tile
    template <int kRows, bool kFull>
    __device__ inline void copy16(const __bf16 *base, int n, char *dst) const {
        if (row_stride <= (1 << 24) && (kFull || n >= kRows)) {
#pragma unroll
            for (int u = 0; u < kRows / N::kRowsPerCopy; ++u) bd_dma16(base + u / kPer16 * 16 * row_stride, off[u % kPer16], dst + u * 1024);
        } else if (row_stride <= (1 << 24)) {
#pragma unroll
            for (int u = 0; u < kRows / N::kRowsPerCopy; ++u) bd_dma16(base, lane_offset(u * N::kRowsPerCopy + lane / N::kChunks, n), dst + u * 1024);
        } else {
#pragma unroll 1
            for (int u = 0; u < kRows / N::kRowsPerCopy; ++u) {
                const int r = u * N::kRowsPerCopy + lane / N::kChunks;
                dma16_lane(base + (r < n ? r : n - 1) * row_stride + (chunk_of(r) << 3), dst + u * 1024);
            }
        }
    }
    // The wave's kWaveRows rows of stage rows r0 .. r0 + 63 of the two tensors of `n` rows at `a` and `b` -> stage buffer.
    template <bool kFull = false>
    __device__ inline void copy(const __bf16 *a, const __bf16 *b, int r0, int n, char *stage) const {
        int w0 = r0 + wave * kWaveRows;          // first row of this wave
        const int left = n - w0;
        if (!kFull && left < 1) w0 = n - 1;      // behind the end: the last row, kWaveRows times
        char *const dst = stage + wave * kWaveRows * N::kRow;
        copy16<kWaveRows, kFull>(a + w0 * row_stride, left < 1 ? 1 : left, dst);
        copy16<kWaveRows, kFull>(b + w0 * row_stride, left < 1 ? 1 : left, dst + N::kTile);
    }
    // A wave's 32 rows, `first` .. of the `n` rows at `base` (first < n) -> `dst`, 32 * kRow bytes of its own
    __device__ inline void copy_rows(const __bf16 *base, int first, int n, char *dst) const {
        copy16<32, false>(base + first * row_stride, n - first, dst);
    }
};

// A workgroup's walk through its work items.  Small problems (Schedule::build_rows) are dealt statically from the schedule
// built in LDS; otherwise wave 0 claims and decodes the NEXT item while the current one's first loads travel.  The claim is
// next_work() with the queues on the lanes, at one place in the kernel: the kernels are as long as the instruction cache
// likes without it.  For batches of at most kTabCap samples and 65535 tiles the tile starts and the sample order are kept
// as 16-bit LDS copies, and decoding is a search in LDS and one trip to memory for the sample's offsets.  Where work is
// dealt without claims, filling them pays for smaller batches only: 1000 samples of at most 20 rows, H = 2, D = 32, backward
// 30.0 us with, 27.8 without; 300 of at most 300, H = 8, D = 64, cross forward 32.2 with, 34.2 without.
// DIRECT: no schedule (Schedule::direct_blocks), as kernels of their own: with one branch more here, every other call was up to 1.4 % slower
// (D = 64, forward, 1414 x 4 of up to 209 rows 95.5 us and 94.3, causal 92.3 and 91.1), and apart it has registers to spare (8 x 4
// of up to 600 rows, D = 64, forward 11.8 -> 10.7, backward 28.8 -> 27.2; 10 x 2 of up to 300, D = 32, 6.6 -> 6.2, 17.6 -> 16.4).
constexpr int kTabCapFixed = 512;
template <bool CROSS, int DIRECT>
struct NarrowWalk {
    struct Shared {
        WorkSlot slot;
        SmallWork mine;
        uint16_t start[kTabCap + 2], sample[kTabCap];
    };
    Shared *sh;
    const int64_t *offsets, *offsets_other;
    Schedule s;
    int B, H, n = 0;
    int64_t total = 0, next_static = 0;
    bool small, tabled = false, fixed_deal = false, home_done = false;
    int grid, step = 0;
    // `scratch`: kInlineScratchInts ints of LDS, free until the first item starts.  Called by every thread.
    __device__ inline NarrowWalk(Shared *sh_, const Schedule &s_, const int64_t *offsets_, const int64_t *offsets_other_, int B_, int H_,
                                 int *scratch)
        : sh(sh_), offsets(offsets_), offsets_other(offsets_other_), s(s_), B(B_), H(H_) {
        small = DIRECT == 1 || s.build_rows != 0;
        grid = (int)gridDim.x;
        asm volatile("" : "+s"(grid));   // read once: the dispatch packet it comes from is a slow place to read
        if (DIRECT == kEither ? s.direct_blocks != 0 : DIRECT != 0) {
            direct_small_work(&sh->mine, s, offsets, CROSS ? offsets_other : nullptr, H, s.build_rows);
        } else if (small) {
            build_small_work(offsets, CROSS ? offsets_other : nullptr, B, H, s.build_rows, scratch, &sh->mine);
        } else {
            const int tiles = s.tile_start[B];
            total = (int64_t)tiles * H;
            fixed_deal = s.static_only || total <= s.fixed_items * (int64_t)grid;
            const int at = fixed_deal && deal_turn(total, grid) ? grid - 1 - (int)blockIdx.x : (int)blockIdx.x;   // see deal_turn()
            next_static = at;
            step = 2 * (grid - 1 - at) + 1;
            if (!fixed_deal) {   // the first item of the home queue is assigned without a claim; see next_work()
                next_static = work_id(blockIdx.x % kXcds, blockIdx.x / kXcds);
                home_done = next_static >= total;
            }
            tabled = B <= (fixed_deal ? kTabCapFixed : kTabCap) && tiles <= 65535;
            if (tabled) {
                for (int p = threadIdx.x; p <= B; p += blockDim.x) sh->start[p] = (uint16_t)s.tile_start[p];
                for (int p = threadIdx.x; p < B; p += blockDim.x) sh->sample[p] = (uint16_t)s.order[p];
            }
            __syncthreads();   // the table is written
        }
    }
    // Next work id or -1, in every lane of wave 0.
    __device__ inline int64_t next_id() {
        if (fixed_deal || (next_static >= 0 && !home_done)) {
            const int64_t id = next_static;
            next_static = fixed_deal ? id + step : -1;
            step = 2 * grid - step;
            return id < total ? id : -1;
        }
        const int lane = threadIdx.x & 63, home = blockIdx.x % kXcds, base = grid / kXcds;
        const int y = (home + lane) % kXcds;   // lane's queue; lane 0: the home queue
        int open = home_done ? 0 : 1;          // queues to ask, a bit per lane
        for (;;) {
            if (open == 0) {   // look at all queues with plain loads, spend an atomic only on one that still shows work
                const bool more = lane < kXcds && work_id(y, base + __atomic_load_n(&s.counter[y * kCounterStride], __ATOMIC_RELAXED)) < total;
                open = (int)__builtin_amdgcn_ballot_w64(more);
                if (open == 0) return -1;   // counters only grow, so this loop ends
            }
            const int ask = __builtin_ctz(open);
            int64_t id = 0;
            if (lane == ask) id = work_id(y, base + atomicAdd(&s.counter[y * kCounterStride], 1));
            const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)id, ask), hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)id >> 32), ask);
            id = (int64_t)(((uint64_t)hi << 32) | lo);
            if (id < total) return id;
            home_done = true;
            open &= open - 1;
        }
    }
    __device__ inline void claim() {   // wave 0, every lane
        if (small) return;
        const int lane = threadIdx.x & 63;
        const int64_t w = next_id();
        WorkSlot *const slot = &sh->slot;
        if (w < 0) {
            if (lane == 0) slot->valid = 0;
            return;
        }
        int lo = 0, hi = B;   // invariant: tile_start[lo] * H <= w < tile_start[hi] * H
        while (hi - lo > 1) {
            const int step = (hi - lo + 63) / 64;
            const int idx = lo + (lane + 1) * step;
            const int probe = idx < hi ? (tabled ? sh->start[idx] : s.tile_start[idx]) : 0;
            const bool ok = idx < hi && (int64_t)probe * H <= w;   // true for a prefix of the lanes
            const int cnt = __popcll(__builtin_amdgcn_ballot_w64(ok));
            lo += cnt * step;
            hi = hi < lo + step ? hi : lo + step;
        }
        const int b = tabled ? sh->sample[lo] : s.order[lo];
        const int t0 = tabled ? sh->start[lo] : s.tile_start[lo];
        const int per_head = (tabled ? sh->start[lo + 1] : s.tile_start[lo + 1]) - t0;
        const int64_t row0 = offsets[b], end = offsets[b + 1];
        const int64_t orow0 = CROSS ? offsets_other[b] : 0, oend = CROSS ? offsets_other[b + 1] : 0;
        const int r = (int)(w - (int64_t)t0 * H);
        if (lane == 0) {
            slot->valid = 1;
            slot->sample = b;
            slot->head = r / per_head;
            slot->block = r - (r / per_head) * per_head;
            slot->len = (int)(end - row0);
            slot->row0_lo = (int)(uint32_t)row0;
            slot->row0_hi = (int)(uint32_t)((uint64_t)row0 >> 32);
            if (CROSS) {
                slot->olen = (int)(oend - orow0);
                slot->orow0_lo = (int)(uint32_t)orow0;
                slot->orow0_hi = (int)(uint32_t)((uint64_t)orow0 >> 32);
            }
        }
    }
    // The item claimed last.  A barrier separates it from the claim before it, another one must precede the next claim.
    __device__ inline bool next(Work &t) {
        if (small && n >= __builtin_amdgcn_readfirstlane(sh->mine.count)) return false;
        return load_work<CROSS>(small ? &sh->mine.item[n++] : &sh->slot, t);
    }
};

// Stores a wave's transposed 32 x D block (rows = features, column = the lane's row of the output tensor; scaled) as whole
// 64- or 128-byte row pieces, 16 bytes per lane: through `region`, 32 * kRow bytes of LDS that only this wave uses.
// `first`: index inside the sample of the block's first row, `n`: rows of the sample, `dst`: the sample's row 0.
template <int D>
__device__ inline void narrow_store(char *region, int lane, const f32x16 (&acc)[D / 32], float scale, __bf16 *dst, int64_t row_stride,
                                    int first, int n) {
    using N = Narrow<D>;
    const int col = lane & 31, half = lane >> 5;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 x;
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = (__bf16)(acc[db][4 * g + e] * scale);
            *reinterpret_cast<bf16x4 *>(region + col * N::kRow + (((db * 4 + g) ^ (col & (N::kChunks - 1))) << 4) + half * 8) = x;
        }
    // lanes read what other lanes of the wave wrote: neither the compiler nor the LDS may turn that round
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __bf16 *p = dst + (first + lane / N::kChunks) * row_stride + (lane % N::kChunks) * 8;
#pragma unroll
    for (int it = 0; it < 32 / N::kRowsPerCopy; ++it, p += N::kRowsPerCopy * row_stride) {
        const int r = it * N::kRowsPerCopy + lane / N::kChunks, ch = lane % N::kChunks;
        const u32x4 piece = *reinterpret_cast<const u32x4 *>(region + r * N::kRow + ((ch ^ (r & (N::kChunks - 1))) << 4));
        if (first + r < n) *reinterpret_cast<u32x4 *>(p) = piece;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the region may be written again (dK, then dV)
    __builtin_amdgcn_wave_barrier();
}

// Wait until at most `N` vector-memory operations and no LDS operation of this wave are pending.
template <int N>
__device__ inline void wait_vm() {
    static_assert(N >= 0 && N < 16, "low bits of the counter field");
    __builtin_amdgcn_s_waitcnt(0x0070 | N);
}

}  // namespace jfa
