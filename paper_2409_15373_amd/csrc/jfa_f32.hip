// fp32 jagged attention, forward and backward, on the fp32 matrix instructions (v_mfma_f32_32x32x2_f32): fp32 products,
// fp32 accumulation, the small-tolerance path (paper Section 2.1; the backward recomputes P from the stored log-sum-exp).
//
// Bound: the fp32 matrix pipe (a 32x32x2 instruction is 4096 flops in 64 clocks; a library product of 8192^3 reaches
// 153 TFLOP/s on this chip).  A block of 32 x 32 scores costs D / 2 instructions per product against 16 exponentials
// per lane and at most one LDS read per instruction, so vector work and LDS are far from being the limit, and what the
// shape of the kernels has to provide is occupancy of all four matrix pipes on short and ragged samples.  Hence
//   * a tile is 64 stationary rows and a stage 64 streamed rows; the four waves of a workgroup are the four 32 x 32
//     quarters of that square: wave w owns stationary rows 32 (w & 1) .. + 31 and in every stage the streamed rows
//     32 (w >> 1) .. + 31.  The two waves that share stationary rows add their results through LDS at the tile's end
//     (fixed order: deterministic).  A sample of up to 64 rows is then one step of each wave instead of two steps of two;
//   * streamed rows go to LDS directly (global_load_lds), the next stage's while the present one is multiplied, and
//     two workgroups share a compute unit (D <= 64), so that one computes while the other starts or ends a tile;
//   * for streams of a block or two a workgroup is one wave, with a 32 x 32 square and one stage: more tiles at once per compute
//     unit, nothing to add up.
// Operand layout of the instruction: lane l holds row (A) or column (B) l % 32 and contraction slot l / 32.  Slots are
// dummies: four consecutive instructions take features 8 g + 4 (l / 32) .. + 3, one 16-byte read per lane.  Scores are
// computed with the streamed rows on the accumulator's row axis and the stationary rows on its column (= lane) axis;
// accumulator register v is then the B operand of the next product's step v (streamed rows (v / 4) 8 + 4 (l / 32) + v % 4
// as its two slots), whose A operand is one element per lane of the transposed streamed tile, read row by row.
// Measured at B = 256, H = 2, D = 64, lengths uniform on [1, 512] against the former kernels (vector FMA, a row per four
// lanes, scores one by one): forward 590 -> 159 us, forward + backward 1861 -> 663 us.  Head size 128, small problems and short
// streams run here; the rest, that size with it, on the bf16 instructions (jfa_f32_split.hip, f32_form()).
#include "jfa_f32.h"

namespace jfa {

// W: waves per workgroup, four or, for short streams, one (see f32_block_rows): stationary rows per tile, streamed rows per stage
template <int W> constexpr int f32_rows() { return W == 4 ? kF32BlockRows : kF32ShortBlockRows; }
static_assert(f32_rows<4>() == 64 && f32_rows<1>() == 32, "a wave is a 32 x 32 square: all of it or a quarter");

__device__ inline f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

template <int D, int W> constexpr int f32_tile_bytes() { return f32_rows<W>() * D * 4; }
// A workgroup's stage buffers: two stages (one wave: one), each the streamed rows of one tensor and then of the other.  They
// double as the in-kernel scheduler's scratch.
template <int D, int W> constexpr int f32_stage_bytes() { return 2 * f32_tile_bytes<D, W>(); }
template <int D, int W> constexpr int f32_lds_bytes() {
    constexpr int stages = (W == 4 ? 2 : 1) * f32_stage_bytes<D, W>(), scratch = kInlineScratchInts * (int)sizeof(int);
    return stages > scratch ? stages : scratch;
}
// D = 128 needs more than 256 registers in the backward, and 128 KB of stages with four waves: one such workgroup per compute unit
template <int D> constexpr int f32_waves_per_simd() { return D <= 64 ? 2 : 1; }

// Up to this many items per workgroup are dealt from the sorted schedule without claims.  A claim is an atomic of the
// whole device, and its latency heads everything a tile does: at D <= 64 that costs more than the last tiles' imbalance
// (B = 256, H = 2, lengths to 512, 4.5 items: D = 64 forward 184 -> 158 us, backward 509 -> 495; 500
// samples of at most 100 rows, H = 8, 6 to 8 items, D = 32: 125 -> 56 and 240 -> 163).  At D = 128, with half the workgroups and
// twice the time per tile, balance is worth more (9 items: 343 -> 358), and next_work()'s own limit of four holds.
template <int D> constexpr int64_t f32_static_items() { return D <= 64 ? 16 : 0; }

// Row r, 16-byte chunk ch of a streamed tile sits at r * 4 D + ((ch ^ f32_swz(r)) << 4): the 16-byte row reads (16
// consecutive rows, one chunk) hit all 64 banks once, and so do the element reads of two rows 4 apart (D >= 64; two-way
// conflicts at D = 32, where a row is half a bank line).
template <int D> __device__ inline int f32_swz(int r) {
    return D == 32 ? (r >> 1) & 7 : ((r >> 2) & 1) << 3 | ((r >> 3) & 1) << 2 | (r & 3);
}

// What rows past a sample's end are copied from.  Their scores are masked, but a probability of 0 times a repeated row is not 0
// where that row holds an infinity.
static __device__ const __attribute__((aligned(16))) float zeros[4] = {0.0f, 0.0f, 0.0f, 0.0f};

// Copies a stage's rows r0 .. of one head (base: the sample's first row of that head; zeroes for rows past the sample's L) into
// `tile`.  A wave instruction fills 1 KB = 256 / D rows.  Addresses are made anew for every stage: kept, they take registers
// that are not there.
template <int D, int W>
__device__ inline void stage_rows(char *tile, const float *__restrict__ base, int64_t row_stride, int r0, int L, int wave, int lane) {
    constexpr int kChunks = D / 4, kOpRows = 64 / kChunks;                  // chunks per row, rows per instruction
    constexpr int kWaveRows = f32_rows<W>() / W, kOps = kWaveRows / kOpRows;   // rows and instructions per wave
    lane = not_hoisted(lane);
    const int first = r0 + kWaveRows * wave + lane / kChunks;
    const int ch = (lane % kChunks) ^ f32_swz<D>(lane / kChunks);   // the swizzle of a sum of row bits is the XOR of theirs
    const float *src = base + first * row_stride;
#pragma unroll
    for (int u = 0; u < kOps; ++u, src += kOpRows * row_stride)
        dma16_lane(first + u * kOpRows < L ? src + (ch ^ f32_swz<D>(u * kOpRows)) * 4 : zeros, tile + (wave * kOps + u) * 1024);
}

// This stage's copies have landed and every wave is done with the present stage.
__device__ inline void stage_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// A lane's stationary row as B operands: x[4 g + e] = row[8 g + 4 half + e].
template <int D> __device__ inline void load_operand(float (&x)[D / 2], const float *__restrict__ row, int half) {
#pragma unroll
    for (int g = 0; g < D / 8; ++g) {
        const float4 f = *reinterpret_cast<const float4 *>(row + 8 * g + 4 * half);
        x[4 * g] = f.x; x[4 * g + 1] = f.y; x[4 * g + 2] = f.z; x[4 * g + 3] = f.w;
    }
}

// LDS byte offsets of a lane's operand reads, relative to the first of the block's 32 streamed rows.  The swizzle makes
// the reads of one kind differ by constant bit patterns, so that one value of each is kept and every read costs one XOR;
// the empty asm keeps the XORs from being hoisted out of the stage loop into registers that are not there.
template <int D> __device__ inline int row_read_at(int col, int half) { return col * (4 * D) + ((half ^ f32_swz<D>(col)) << 4); }
template <int D> __device__ inline int element_read_at(int col, int half) {
    return half * (16 * D) + (((col >> 2) ^ f32_swz<D>(4 * half)) << 4) + (col & 3) * 4;
}

// (32 streamed rows at `block`) (stationary rows)^T; at: row_read_at.  A score's error grows with the length of the chains of
// additions it comes from, and the exponential turns it into a relative error of the probability: the D features are summed
// in four chains, as four lanes of a vector kernel would.  One chain: the gradients' error at scores of standard deviation 16
// is 1.5 (D = 32), 1.8 (64) and 2.1 times this (128); eight chains: 0.99 and 0.92 times at D = 64 and 128, time + 5 %.
// Both together, microseconds of forward and backward at B = 256, H = 2, lengths to 512: D = 32 85 + 275 -> 94 + 293,
// D = 64 179 + 503 -> 185 + 509, D = 128 324 + 1165 -> 343 + 1201.
template <int D> __device__ inline f32x16 product(const char *block, int at, const float (&x)[D / 2]) {
    constexpr int kChains = 4, kGroups = D / 8 / kChains;   // a chain's 16-byte reads
    f32x16 sum;
    at = not_hoisted(at);
#pragma unroll
    for (int ch = 0; ch < kChains; ++ch) {
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll
        for (int g = ch * kGroups; g < (ch + 1) * kGroups; ++g) {
            const float4 a = *reinterpret_cast<const float4 *>(block + (at ^ (g << 5)));
            acc = mfma_f32(a.x, x[4 * g], acc);
            acc = mfma_f32(a.y, x[4 * g + 1], acc);
            acc = mfma_f32(a.z, x[4 * g + 2], acc);
            acc = mfma_f32(a.w, x[4 * g + 3], acc);
        }
        sum = ch == 0 ? acc : sum + acc;
    }
    return sum;
}

// acc^T += (32 streamed rows at `block`)^T p, p in accumulator layout; at: element_read_at
template <int D> __device__ inline void accumulate(f32x16 (&acc)[D / 32], const char *block, int at, const f32x16 &p) {
    at = not_hoisted(at);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int r = acc_row(v, 0);   // + 4 in the other half-wave, which is in `at`
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
            acc[db] = mfma_f32(*reinterpret_cast<const float *>(block + (at ^ ((f32_swz<D>(r) ^ (8 * db)) << 4)) + r * (4 * D)), p[v], acc[db]);
    }
}

// An accumulator on its way to the wave that shares the stationary rows: 16 bytes per lane and step, no bank conflicts.
template <int D> __device__ inline void park(char *region, const f32x16 (&acc)[D / 32], int lane) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4 *>(region + ((db * 4 + g) * 64 + lane) * 16) =
                make_float4(acc[db][4 * g], acc[db][4 * g + 1], acc[db][4 * g + 2], acc[db][4 * g + 3]);
}
// acc = acc * mine + parked * theirs
template <int D> __device__ inline void merge(f32x16 (&acc)[D / 32], const char *region, int lane, float mine, float theirs) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 o = *reinterpret_cast<const float4 *>(region + ((db * 4 + g) * 64 + lane) * 16);
            acc[db][4 * g] = acc[db][4 * g] * mine + o.x * theirs;
            acc[db][4 * g + 1] = acc[db][4 * g + 1] * mine + o.y * theirs;
            acc[db][4 * g + 2] = acc[db][4 * g + 2] * mine + o.z * theirs;
            acc[db][4 * g + 3] = acc[db][4 * g + 3] * mine + o.w * theirs;
        }
}

template <int D, int W>
__global__ __launch_bounds__(64 * W, f32_waves_per_simd<D>()) void fwd_f32_kernel(
        const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
        const int64_t *__restrict__ offsets, const int64_t *__restrict__ offsets_kv, bool causal, int B, int H, Schedule s,
        float *__restrict__ out, float *__restrict__ lse) {
    constexpr int kRows = f32_rows<W>(), kCols = kRows, kTile = f32_tile_bytes<D, W>(), kStage = f32_stage_bytes<D, W>();
    __shared__ __attribute__((aligned(1024))) char sm[f32_lds_bytes<D, W>()];   // two stages of K rows, then V rows
    __shared__ float2 other_ml[2][32];   // running maximum and row sum of the waves w >= 2
    __shared__ int64_t slot;
    __shared__ SmallWork mine;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int rg = W == 4 ? wave & 1 : 0, part = W == 4 ? wave >> 1 : 0;   // group of 32 queries; half of the stage's keys
    const int row_at = row_read_at<D>(col, half), elem_at = element_read_at<D>(col, half);
    const float scale = 1.0f / sqrtf((float)D);
    const bool small = s.build_rows != 0;   // small problem: no scheduler launch has run, the schedule is built here, in LDS
    if (s.direct_blocks) direct_small_work(&mine, s, offsets, offsets_kv, H, kRows);
    else if (small) build_small_work(offsets, offsets_kv, B, H, s.build_rows, reinterpret_cast<int *>(sm), &mine);
    const int64_t total = small ? 0 : (int64_t)s.tile_start[B] * H;
    const int64_t sum_B = offsets[B];
    const int64_t row_stride = (int64_t)H * D;

    WorkCursor cursor;
    cursor.static_only = s.static_only || total <= f32_static_items<D>() * (int64_t)gridDim.x;
    Work t;   // keys: rows orow0 .. orow0 + olen - 1
    for (int item = 0; next_item(t, mine, small, item, s, offsets, offsets_kv, B, H, cursor, total, &slot); ++item) {
        const int L = t.olen;
        const int q0 = t.block * kRows + rg * 32;      // first query of the wave
        const int i = q0 + col;                        // this lane's query
        const int iq = i < t.len ? i : t.len - 1;      // rows past the end recompute the last row
        const bool active = q0 < t.len;
        // causal (self attention only): query i sees keys 0 .. i, so the tile needs the keys up to its last query
        const int Lc = causal && (t.block + 1) * kRows < L ? (t.block + 1) * kRows : L;
        const float *kbase = k + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *vbase = v + t.orow0 * row_stride + (int64_t)t.head * D;
        auto issue = [&](int j0, int buf) {
            stage_rows<D, W>(sm + buf * kStage, kbase, row_stride, j0, L, wave, lane);
            stage_rows<D, W>(sm + buf * kStage + kTile, vbase, row_stride, j0, L, wave, lane);
        };
        if (L > 0) issue(0, 0);
        float qr[D / 2];
        load_operand<D>(qr, q + (t.row0 + iq) * row_stride + (int64_t)t.head * D, half);
        f32x16 o[D / 32];
        clear<D>(o);
        float m = -INFINITY, l = 0.0f;   // running maximum of the scores; this lane's share of the row sum
        stage_barrier();
        for (int j0 = 0, buf = 0; j0 < Lc; j0 += kCols, buf ^= W == 4) {
            if (W == 4 && j0 + kCols < Lc) issue(j0 + kCols, buf ^ 1);
            const int k0 = j0 + part * 32;             // first key of the wave's block
            if (active && k0 < Lc && !(causal && k0 > q0 + 31)) {
                const char *kt = sm + buf * kStage + part * (32 * 4 * D), *vt = kt + kTile;
                f32x16 st = product<D>(kt, row_at, qr);
                if (k0 + 32 > L || (causal && k0 + 31 > q0)) {   // keys past the sample's end or above the diagonal
                    const int lim = (causal && iq + 1 < L ? iq + 1 : L) - k0;
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (acc_row(e, half) >= lim) st[e] = -INFINITY;
                }
                float mx = st[0];
#pragma unroll
                for (int e = 1; e < 16; ++e) mx = fmaxf(mx, st[e]);
                const float m_new = fmaxf(m, pair_max(mx) * scale);   // finite: every query of a block that is not skipped sees one of its keys
                const float a = exp_f32(m - m_new);   // exp(-inf) = 0 on the first block
                m = m_new;
                l *= a;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    st[e] = exp_f32(fmaf(st[e], scale, -m));
                    l += st[e];
                }
#pragma unroll
                for (int db = 0; db < D / 32; ++db)
#pragma unroll
                    for (int e = 0; e < 16; ++e) o[db][e] *= a;
                accumulate<D>(o, vt, elem_at, st);
            }
            stage_barrier();
            if (W == 1 && j0 + kCols < Lc) {   // one buffer: the other workgroups of the compute unit fill the gap
                issue(j0 + kCols, 0);
                stage_barrier();
            }
        }
        // the two waves of a group of queries have seen different keys: waves 2 and 3 hand over, waves 0 and 1 finish
        l = pair_sum(l);
        char *const region = sm + rg * (D * 128);
        if (W == 4) {
            if (part == 1) {
                park<D>(region, o, lane);
                if (half == 0) other_ml[rg][col] = make_float2(m, l);
            }
            __syncthreads();
        }
        if (part == 0 && i < t.len) {
            const float2 ml = W == 4 ? other_ml[rg][col] : make_float2(-INFINITY, 0.0f);
            const float m_all = fmaxf(m, ml.x);
            const float a = m_all > -INFINITY ? exp_f32(m - m_all) : 0.0f;      // a sample without keys: out = 0, lse = -inf
            const float b = m_all > -INFINITY ? exp_f32(ml.x - m_all) : 0.0f;
            const float l_all = l * a + ml.y * b;
            if (W == 4) merge<D>(o, region, lane, a, b);
            store_row<D>(out + (t.row0 + i) * row_stride + (int64_t)t.head * D, o, l_all > 0.0f ? 1.0f / l_all : 0.0f, half);
            if (half == 0) lse[(int64_t)t.head * sum_B + t.row0 + i] = m_all + logf(l_all);
        }
    }
}

// dQ: tile = 64 (one wave: 32) queries, stream the sample's keys.  The kernel is the first of the backward: it holds each query's dO
// row anyway, reads the matching row of the forward's output, and computes delta = rowsum(dO o O) for its own use
// and for the dK / dV kernel (no separate pass over dO and O, one launch less).
template <int D, int W>
__global__ __launch_bounds__(64 * W, f32_waves_per_simd<D>()) void dq_f32_kernel(
        const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
        const float *__restrict__ out_fwd, const float *__restrict__ dout, const float *__restrict__ lse,
        float *__restrict__ delta, const int64_t *__restrict__ offsets, const int64_t *__restrict__ offsets_kv, bool causal,
        int B, int H, Schedule s, float *__restrict__ dq) {
    constexpr int kRows = f32_rows<W>(), kCols = kRows, kTile = f32_tile_bytes<D, W>(), kStage = f32_stage_bytes<D, W>();
    __shared__ __attribute__((aligned(1024))) char sm[f32_lds_bytes<D, W>()];   // two stages of K rows, then V rows
    __shared__ int64_t slot;
    __shared__ SmallWork mine;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int rg = W == 4 ? wave & 1 : 0, part = W == 4 ? wave >> 1 : 0;   // group of 32 queries; half of the stage's keys
    const int row_at = row_read_at<D>(col, half), elem_at = element_read_at<D>(col, half);
    const float scale = 1.0f / sqrtf((float)D);
    const bool small = s.build_rows != 0;
    if (D < 128 && s.direct_blocks) direct_small_work(&mine, s, offsets, offsets_kv, H, kRows);   // D = 128: as dK / dV, which has no registers for it
    else if (small) build_small_work(offsets, offsets_kv, B, H, s.build_rows, reinterpret_cast<int *>(sm), &mine);
    const int64_t total = small ? 0 : (int64_t)s.tile_start[B] * H;
    const int64_t sum_B = offsets[B];
    const int64_t row_stride = (int64_t)H * D;

    WorkCursor cursor;
    cursor.static_only = s.static_only || total <= f32_static_items<D>() * (int64_t)gridDim.x;
    Work t;
    for (int item = 0; next_item(t, mine, small, item, s, offsets, offsets_kv, B, H, cursor, total, &slot); ++item) {
        const int L = t.olen;
        const int q0 = t.block * kRows + rg * 32;
        const int i = q0 + col;
        const int iq = i < t.len ? i : t.len - 1;
        const bool active = q0 < t.len;
        const int Lc = causal && (t.block + 1) * kRows < L ? (t.block + 1) * kRows : L;
        const float *kbase = k + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *vbase = v + t.orow0 * row_stride + (int64_t)t.head * D;
        auto issue = [&](int j0, int buf) {
            stage_rows<D, W>(sm + buf * kStage, kbase, row_stride, j0, L, wave, lane);
            stage_rows<D, W>(sm + buf * kStage + kTile, vbase, row_stride, j0, L, wave, lane);
        };
        if (L > 0) issue(0, 0);
        float qr[D / 2], dor[D / 2];
        const int64_t row = (t.row0 + iq) * row_stride + (int64_t)t.head * D;
        load_operand<D>(qr, q + row, half);
        load_operand<D>(dor, dout + row, half);
        float dot = 0.0f;
#pragma unroll
        for (int g = 0; g < D / 8; ++g) {
            const float4 f = *reinterpret_cast<const float4 *>(out_fwd + row + 8 * g + 4 * half);
            dot = fmaf(dor[4 * g], f.x, fmaf(dor[4 * g + 1], f.y, fmaf(dor[4 * g + 2], f.z, fmaf(dor[4 * g + 3], f.w, dot))));
        }
        const float delta_i = pair_sum(dot);   // the two lanes of a row hold half of its features each
        const float lse_i = lse[(int64_t)t.head * sum_B + t.row0 + iq];
        if (part == 0 && i < t.len && half == 0) delta[(int64_t)t.head * sum_B + t.row0 + i] = delta_i;
        f32x16 acc[D / 32];
        clear<D>(acc);
        stage_barrier();
        for (int j0 = 0, buf = 0; j0 < Lc; j0 += kCols, buf ^= W == 4) {
            if (W == 4 && j0 + kCols < Lc) issue(j0 + kCols, buf ^ 1);
            const int k0 = j0 + part * 32;
            if (active && k0 < Lc && !(causal && k0 > q0 + 31)) {
                const char *kt = sm + buf * kStage + part * (32 * 4 * D), *vt = kt + kTile;
                f32x16 st = product<D>(kt, row_at, qr);
                const f32x16 dp = product<D>(vt, row_at, dor);
                const bool masked = k0 + 32 > L || (causal && k0 + 31 > q0);
                const int lim = (causal && iq + 1 < L ? iq + 1 : L) - k0;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float p = exp_f32(fmaf(st[e], scale, -lse_i));
                    if (masked && acc_row(e, half) >= lim) p = 0.0f;
                    st[e] = p * (dp[e] - delta_i);
                }
                accumulate<D>(acc, kt, elem_at, st);
            }
            stage_barrier();
            if (W == 1 && j0 + kCols < Lc) {   // one buffer: the other workgroups of the compute unit fill the gap
                issue(j0 + kCols, 0);
                stage_barrier();
            }
        }
        char *const region = sm + rg * (D * 128);
        if (W == 4) {
            if (part == 1) park<D>(region, acc, lane);
            __syncthreads();
        }
        if (part == 0 && i < t.len) {
            if (W == 4) merge<D>(acc, region, lane, 1.0f, 1.0f);
            store_row<D>(dq + row, acc, scale, half);
        }
    }
}

// dK, dV: tile = 64 (one wave: 32) keys, stream the sample's queries (with their dO, lse, delta).
template <int D, int W>
__global__ __launch_bounds__(64 * W, f32_waves_per_simd<D>()) void dkv_f32_kernel(
        const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
        const float *__restrict__ dout, const float *__restrict__ lse, const float *__restrict__ delta,
        const int64_t *__restrict__ offsets,   // of the keys
        const int64_t *__restrict__ offsets_q, bool causal, int B, int H, Schedule s, float *__restrict__ dk,
        float *__restrict__ dv) {
    constexpr int kRows = f32_rows<W>(), kCols = kRows, kTile = f32_tile_bytes<D, W>(), kStage = f32_stage_bytes<D, W>();
    __shared__ __attribute__((aligned(1024))) char sm[f32_lds_bytes<D, W>()];   // two stages of Q rows, then dO rows
    __shared__ __attribute__((aligned(16))) float lse_s[2][kCols], delta_s[2][kCols];   // lse and delta of the streamed rows
    static_assert(__alignof__(lse_s) >= 16 && __alignof__(delta_s) >= 16, "read four at a time");
    __shared__ int64_t slot;
    __shared__ SmallWork mine;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int rg = W == 4 ? wave & 1 : 0, part = W == 4 ? wave >> 1 : 0;   // group of 32 keys; half of the stage's queries
    const int row_at = row_read_at<D>(col, half), elem_at = element_read_at<D>(col, half);
    const float scale = 1.0f / sqrtf((float)D);
    const bool small = s.build_rows != 0;
    if (D < 128 && s.direct_blocks) direct_small_work(&mine, s, offsets, offsets_q, H, kRows);   // at D = 128 it would make the kernel spill
    else if (small) build_small_work(offsets, offsets_q, B, H, s.build_rows, reinterpret_cast<int *>(sm), &mine);
    const int64_t total = small ? 0 : (int64_t)s.tile_start[B] * H;
    const int64_t sum_B = offsets_q ? offsets_q[B] : offsets[B];   // lse and delta are indexed by query rows
    const int64_t row_stride = (int64_t)H * D;

    WorkCursor cursor;
    cursor.static_only = s.static_only || total <= f32_static_items<D>() * (int64_t)gridDim.x;
    Work t;   // queries: rows orow0 .. orow0 + olen - 1
    for (int item = 0; next_item(t, mine, small, item, s, offsets, offsets_q, B, H, cursor, total, &slot); ++item) {
        const int L = t.olen;
        const int k0 = t.block * kRows + rg * 32;      // first key of the wave
        const int j = k0 + col;                        // this lane's key
        const int jk = j < t.len ? j : t.len - 1;
        const bool active = k0 < t.len;
        const float *qbase = q + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *obase = dout + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *lse_rows = lse + (int64_t)t.head * sum_B + t.orow0;
        const float *delta_rows = delta + (int64_t)t.head * sum_B + t.orow0;
        // causal: key j is seen by queries j .. L - 1, so the stream starts at the stage that holds the tile's first key
        const int istart = causal ? t.block * kRows : 0;
        auto issue = [&](int i0, int buf) {
            stage_rows<D, W>(sm + buf * kStage, qbase, row_stride, i0, L, wave, lane);
            stage_rows<D, W>(sm + buf * kStage + kTile, obase, row_stride, i0, L, wave, lane);
        };
        float lse_next = 0.0f, delta_next = 0.0f;      // statistics of the stage on its way (threads 0 .. 63)
        auto fetch_stats = [&](int i0) {
            if (tid < kCols) {
                const int i = i0 + tid < L ? i0 + tid : L - 1;
                lse_next = lse_rows[i];
                delta_next = delta_rows[i];
            }
        };
        auto store_stats = [&](int buf) {
            if (tid < kCols) { lse_s[buf][tid] = lse_next; delta_s[buf][tid] = delta_next; }
        };
        if (istart < L) {
            issue(istart, 0);
            fetch_stats(istart);
        }
        float kr[D / 2], vr[D / 2];
        const int64_t row = (t.row0 + jk) * row_stride + (int64_t)t.head * D;
        load_operand<D>(kr, k + row, half);
        load_operand<D>(vr, v + row, half);
        f32x16 acck[D / 32], accv[D / 32];
        clear<D>(acck);
        clear<D>(accv);
        store_stats(0);
        stage_barrier();
        for (int i0 = istart, buf = 0; i0 < L; i0 += kCols, buf ^= W == 4) {
            const bool more = i0 + kCols < L;
            if (W == 4 && more) {
                issue(i0 + kCols, buf ^ 1);
                fetch_stats(i0 + kCols);
            }
            const int r0 = i0 + part * 32;             // first query of the wave's block
            if (active && r0 < L && !(causal && r0 + 31 < k0)) {
                const char *qt = sm + buf * kStage + part * (32 * 4 * D), *ot = qt + kTile;
                f32x16 st = product<D>(qt, row_at, kr);
                f32x16 dp = product<D>(ot, row_at, vr);
                const bool masked = r0 + 32 > L || (causal && r0 < k0 + 31);
                const int lo = causal ? j - r0 : 0, hi = L - r0;   // this lane's key is seen by block rows lo .. hi - 1
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 l4 = *reinterpret_cast<const f32x4 *>(&lse_s[buf][part * 32 + g * 8 + half * 4]);
                    const f32x4 d4 = *reinterpret_cast<const f32x4 *>(&delta_s[buf][part * 32 + g * 8 + half * 4]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int r = acc_row(4 * g + e, half);
                        float p = exp_f32(fmaf(st[4 * g + e], scale, -l4[e]));
                        if (masked && (r < lo || r >= hi)) p = 0.0f;
                        st[4 * g + e] = p;
                        dp[4 * g + e] = p * (dp[4 * g + e] - d4[e]);
                    }
                }
                accumulate<D>(accv, ot, elem_at, st);
                accumulate<D>(acck, qt, elem_at, dp);
            }
            if (W == 4 && more) store_stats(buf ^ 1);
            stage_barrier();
            if (W == 1 && more) {
                issue(i0 + kCols, 0);
                fetch_stats(i0 + kCols);
                store_stats(0);
                stage_barrier();
            }
        }
        // each wave of a pair finishes one gradient: waves 0 and 1 dK, waves 2 and 3 dV
        char *const region = sm + rg * (D * 256);
        if (W == 4) {
            if (part == 0) park<D>(region, accv, lane); else park<D>(region + D * 128, acck, lane);
            __syncthreads();
        }
        if (j < t.len) {
            if (part == 0) {
                if (W == 4) merge<D>(acck, region + D * 128, lane, 1.0f, 1.0f);
                store_row<D>(dk + row, acck, scale, half);
            }
            if (W == 1 || part == 1) {
                if (W == 4) merge<D>(accv, region, lane, 1.0f, 1.0f);
                store_row<D>(dv + row, accv, 1.0f, half);
            }
        }
    }
}

hipError_t launch_fwd_f32(const float *q, const float *k, const float *v, const int64_t *offsets,
                          const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, F32Form form, float *out, float *lse,
                          int cus, hipStream_t stream) {
    if (form.split) return launch_fwd_f32_split(q, k, v, offsets, offsets_kv, causal, B, H, D, s, out, lse, cus, stream);
#define JFA_CASE(DD, W)                                                                                           \
    case DD * 1000 + f32_rows<W>():                                                                               \
        hipLaunchKernelGGL((fwd_f32_kernel<DD, W>), dim3(item_grid<fwd_f32_kernel<DD, W>>(64 * W, B, H, s, cus)), dim3(64 * W), 0, stream, \
                           q, k, v, offsets, offsets_kv, causal, B, H, s, out, lse);                              \
        break;
    switch (D * 1000 + form.rows) {
        JFA_CASE(32, 1) JFA_CASE(32, 4) JFA_CASE(64, 1) JFA_CASE(64, 4) JFA_CASE(128, 1) JFA_CASE(128, 4)
        default: return hipErrorInvalidValue;
    }
#undef JFA_CASE
    return hipGetLastError();
}

hipError_t launch_dq_f32(const float *q, const float *k, const float *v, const float *out, const float *dout, const float *lse,
                         const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, F32Form form,
                         float *dq, float *delta, int cus, hipStream_t stream) {
    if (form.split) return launch_dq_f32_split(q, k, v, out, dout, lse, offsets, offsets_kv, causal, B, H, D, s, dq, delta, cus, stream);
#define JFA_CASE(DD, W)                                                                                            \
    case DD * 1000 + f32_rows<W>():                                                                                \
        hipLaunchKernelGGL((dq_f32_kernel<DD, W>), dim3(item_grid<dq_f32_kernel<DD, W>>(64 * W, B, H, s, cus)), dim3(64 * W), 0, stream, \
                           q, k, v, out, dout, lse, delta, offsets, offsets_kv, causal, B, H, s, dq);              \
        break;
    switch (D * 1000 + form.rows) {
        JFA_CASE(32, 1) JFA_CASE(32, 4) JFA_CASE(64, 1) JFA_CASE(64, 4) JFA_CASE(128, 1) JFA_CASE(128, 4)
        default: return hipErrorInvalidValue;
    }
#undef JFA_CASE
    return hipGetLastError();
}

hipError_t launch_dkv_f32(const float *q, const float *k, const float *v, const float *dout, const float *lse, const float *delta,
                          const int64_t *offsets, const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, F32Form form,
                          float *dk, float *dv, int cus, hipStream_t stream) {
    if (form.split) return launch_dkv_f32_split(q, k, v, dout, lse, delta, offsets, offsets_q, causal, B, H, D, s, dk, dv, cus, stream);
#define JFA_CASE(DD, W)                                                                                            \
    case DD * 1000 + f32_rows<W>():                                                                                \
        hipLaunchKernelGGL((dkv_f32_kernel<DD, W>), dim3(item_grid<dkv_f32_kernel<DD, W>>(64 * W, B, H, s, cus)), dim3(64 * W), 0, stream, \
                           q, k, v, dout, lse, delta, offsets, offsets_q, causal, B, H, s, dk, dv);                \
        break;
    switch (D * 1000 + form.rows) {
        JFA_CASE(32, 1) JFA_CASE(32, 4) JFA_CASE(64, 1) JFA_CASE(64, 4) JFA_CASE(128, 1) JFA_CASE(128, 4)
        default: return hipErrorInvalidValue;
    }
#undef JFA_CASE
    return hipGetLastError();
}

}  // namespace jfa
