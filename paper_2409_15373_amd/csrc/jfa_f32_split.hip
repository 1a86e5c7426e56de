// fp32 jagged attention at head sizes 32 and 64 on the bf16 matrix instructions, forward and backward.
//
// A float is the exact sum of three bf16 numbers (24 = 3 x 8 significand bits, each the rest rounded to nearest), so a product of
// two floats is nine bf16 products, of which the three smallest stay below 2^-24 of it.  The other six cost 6 x 32 clocks per
// 32 x 32 x 16 block against 8 x 64 on the fp32 matrix instructions, and a sum of sixteen features or rows is rounded once
// instead of eight times.  Errors against 64 bits, normwise, D = 64, inputs of standard deviation 1 (the fp32 instructions' first):
// out 2.7e-7, 1.4e-7; dq 4.2e-7, 3.4e-7; dk 4.2e-7, 3.4e-7; dv 4.0e-7, 3.3e-7; scores of standard deviation 16, dq 2.0e-6, 1.7e-6.
// The last piece of a small float would lie below bf16's smallest normal number: factors are scaled by 2^24 before they are split,
// which is exact, and products by 2^-48 where they are used anyway.
//
// Bound: the matrix and vector pipes together.  Splitting a streamed row takes about as many instructions as its products, so it
// is split once per workgroup, on its way from registers to LDS, and read by four waves (or two pairs); of the products the
// smallest are summed first, and the sum over 32 streamed rows is formed apart and added to the accumulator at once (added one by
// one, the gradients' errors are 5 to 14 % above those of the fp32 instructions).  Two workgroups of four waves per compute unit:
// 206 to 252 registers.  Tried: workgroups of two waves (the splitting is then shared by half as many), dK / dV with both operands'
// planes in one wave (spills): both slower.  Microseconds at B = 256, H = 2, lengths to 512, against the fp32 instructions: D = 64
// forward 168 -> 108, backward 530 -> 327; D = 32 96 -> 70, 299 -> 212; 32 samples of 4096 rows, one head, D = 64, forward 1255 -> 782,
// backward 4115 -> 2659.  All NaN: 111 and 334; with one infinity per sample, in v, 1130 and 3930 (see "values that have no split").
#include "jfa_f32.h"
#include "jfa_narrow.h"

namespace jfa {

// ---- splitting ----
// The last of a float's 24 bits is at least 2^-149: scaled by 2^24 every piece is zero or at least 2^-125, a normal number.  (Not
// scaled, factors below 2^-110 had fewer than 24 bits: relative error 1.4e-4 at 2^-122.)  The largest factors, from 2^104 on, have
// no split then, see below.
constexpr float kSplitScale = 0x1p24f, kProductScale = 0x1p-48f;
// x[0 .. 7] -> three bf16 operands with kSplitScale x = p[0] + p[1] + p[2]
__device__ inline void split8(const float (&x)[8], bf16x8 (&p)[3]) {
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float y = x[e] * kSplitScale;
        p[0][e] = (__bf16)y;
        r[e] = y - (float)p[0][e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) { p[1][e] = (__bf16)r[e]; p[2][e] = (__bf16)(r[e] - (float)p[1][e]); }
}

// A stage: kSpRows streamed rows of two tensors, each as three bf16 planes laid out like the tiles of the narrow bf16 kernels.
constexpr int kSpRows = 32, kSpThreads = 256;
template <int D> constexpr int sp_plane() { return kSpRows * Narrow<D>::kRow; }
template <int D> constexpr int sp_tensor() { return 3 * sp_plane<D>(); }
template <int D> constexpr int sp_stage() { return 2 * sp_tensor<D>(); }

// One stage on its way through registers: every thread takes 8 consecutive features of kTasks rows.
template <int D>
struct SplitStage {
    using N = Narrow<D>;
    static constexpr int kThreads = kSpThreads, kPerTensor = kSpRows * N::kChunks, kTasks = 2 * kPerTensor / kThreads;
    static_assert(kTasks >= 1 && kPerTensor % 64 == 0, "a wave's tasks belong to one tensor");
    float x[kTasks][8];
    __device__ inline void fetch(const float *a, const float *b, int64_t row_stride, int r0, int n, int wave, int lane) {
        lane = not_hoisted(lane);
#pragma unroll
        for (int u = 0; u < kTasks; ++u) {
            const int first = u * kThreads + wave * 64;   // the wave's first task
            const int task = first % kPerTensor + lane, r = r0 + task / N::kChunks;
            const float *src = (first < kPerTensor ? a : b) + r * row_stride + task % N::kChunks * 8;
            float4 lo = make_float4(0.0f, 0.0f, 0.0f, 0.0f), hi = lo;   // rows past the end: zeroes
            if (r < n) {
                lo = *reinterpret_cast<const float4 *>(src);
                hi = *reinterpret_cast<const float4 *>(src + 4);
            }
            x[u][0] = lo.x; x[u][1] = lo.y; x[u][2] = lo.z; x[u][3] = lo.w;
            x[u][4] = hi.x; x[u][5] = hi.y; x[u][6] = hi.z; x[u][7] = hi.w;
        }
    }
    __device__ inline void store(char *stage, int wave, int lane) const {
        lane = not_hoisted(lane);
#pragma unroll
        for (int u = 0; u < kTasks; ++u) {
            const int first = u * kThreads + wave * 64, task = first % kPerTensor + lane;
            const int r = task / N::kChunks, ch = task % N::kChunks;
            char *dst = stage + (first < kPerTensor ? 0 : sp_tensor<D>()) + r * N::kRow + ((ch ^ N::swz(r)) << 4);
            bf16x8 p[3];
            split8(x[u], p);
#pragma unroll
            for (int i = 0; i < 3; ++i) *reinterpret_cast<bf16x8 *>(dst + i * sp_plane<D>()) = p[i];
        }
    }
};

// A lane's stationary row as operands: y[i][ks] holds plane i of features 16 ks + 8 half ..
template <int D> __device__ inline void load_split(bf16x8 (&y)[3][D / 16], const float *__restrict__ row, int half) {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        const float4 lo = *reinterpret_cast<const float4 *>(row + 16 * ks + 8 * half), hi = *reinterpret_cast<const float4 *>(row + 16 * ks + 8 * half + 4);
        const float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
        bf16x8 p[3];
        split8(x, p);
        y[0][ks] = p[0]; y[1][ks] = p[1]; y[2][ks] = p[2];
    }
}

// (32 streamed rows at `tile`) (stationary rows)^T / kProductScale: the small products first, so that only the last D / 16 steps round at
// the sum's own size
template <int D> __device__ inline f32x16 product(const char *tile, const NarrowAddresses<D> &at, const bf16x8 (&y)[3][D / 16]) {
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
    bf16x8 x0[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        x0[ks] = lds_read_b128(tile + at.row[ks]);
        const bf16x8 x1 = lds_read_b128(tile + sp_plane<D>() + at.row[ks]), x2 = lds_read_b128(tile + 2 * sp_plane<D>() + at.row[ks]);
        acc = mfma_32x32x16(x2, y[0][ks], acc);
        acc = mfma_32x32x16(x0[ks], y[2][ks], acc);
        acc = mfma_32x32x16(x1, y[1][ks], acc);
        acc = mfma_32x32x16(x1, y[0][ks], acc);
        acc = mfma_32x32x16(x0[ks], y[1][ks], acc);
    }
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) acc = mfma_32x32x16(x0[ks], y[0][ks], acc);
    return acc;
}

// acc^T += (32 streamed rows at `tile`)^T p / kProductScale, p in accumulator layout.  The block's own sum is formed first, small products before
// large ones, and added to acc at once: one rounding at the size of acc for 32 rows.
template <int D> __device__ inline void accumulate(f32x16 (&acc)[D / 32], const char *tile, const NarrowAddresses<D> &at, const f32x16 &p) {
    bf16x8 y[2][3];
#pragma unroll
    for (int ts = 0; ts < 2; ++ts) {
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = p[8 * ts + e];
        split8(x, y[ts]);
    }
#pragma unroll
    for (int db = 0; db < D / 32; ++db) {
        f32x16 sum;
#pragma unroll
        for (int e = 0; e < 16; ++e) sum[e] = 0.0f;
        bf16x8 x0[2];
#pragma unroll
        for (int ts = 0; ts < 2; ++ts) {
            const char *t = tile + ts * 16 * Narrow<D>::kRow;
            bf16x8 x3[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) x3[i] = concat(lds_read_tr16(t + i * sp_plane<D>() + at.tr[0][db]), lds_read_tr16(t + i * sp_plane<D>() + at.tr[1][db]));
            sum = mfma_32x32x16(x3[2], y[ts][0], sum);
            sum = mfma_32x32x16(x3[0], y[ts][2], sum);
            sum = mfma_32x32x16(x3[1], y[ts][1], sum);
            sum = mfma_32x32x16(x3[1], y[ts][0], sum);
            sum = mfma_32x32x16(x3[0], y[ts][1], sum);
            x0[ts] = x3[0];
        }
#pragma unroll
        for (int ts = 0; ts < 2; ++ts) sum = mfma_32x32x16(x0[ts], y[ts][0], sum);
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[db][e] += sum[e];
    }
}

// Everything this wave has written to LDS is there; then everyone's.  (__syncthreads() would wait for the loads in flight too.)
__device__ inline void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// ---- values that have no split ----
// An infinity is not a sum of three bf16 numbers: the rest is NaN, and NaN is what the products above make of it, and of factors
// that scaled round to infinity; scaled products of large factors may overflow.  Results that come out not finite are therefore taken
// again in plain fp32, one lane per row; the others stay as they are (a product of rows touches no other column).  Lane by lane that
// costs some ten times the wave's products; on the matrix instructions masked entries would be 0 times an infinity.
template <int D> __device__ inline void unscale(f32x16 (&acc)[D / 32]) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[db][e] *= kProductScale;
}
template <int D> __device__ inline bool all_finite(const f32x16 (&acc)[D / 32]) {
    float s = 0.0f;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) s = fmaf(acc[db][e], 0.0f, s);
    return s == 0.0f;
}
template <int D> __device__ inline void take_where_not_finite(f32x16 (&acc)[D / 32], const f32x16 (&again)[D / 32]) {
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[db][e] = fabsf(acc[db][e]) < INFINITY ? acc[db][e] : again[db][e];
}
// What a lane of this half holds of a row, in plain fp32: the features of a transposed accumulator's registers
template <int D> struct PlainRow {
    float x[D / 2];
    __device__ inline void load(const float *__restrict__ row, int half) {
#pragma unroll
        for (int g = 0; g < D / 8; ++g) {
            const float4 f = *reinterpret_cast<const float4 *>(row + g * 8 + half * 4);
            x[4 * g] = f.x; x[4 * g + 1] = f.y; x[4 * g + 2] = f.z; x[4 * g + 3] = f.w;
        }
    }
    __device__ inline bool has_nan() const {   // in either half
        bool nan = false;
#pragma unroll
        for (int d = 0; d < D / 2; ++d) nan = nan || x[d] != x[d];
        const bool other = __shfl_xor((int)nan, 32, 64);
        return nan || other;
    }
};
// R of the streamed rows r .. n - 1 at a time (the last one again behind the end): their loads are in flight together.  Two where the
// registers are there (forward with an infinity per sample, see above, 2.1 -> 1.1 ms; four, or two in dK / dV, spill in ordinary calls too).
template <int D, int R> struct PlainRows {
    const float *p[R];
    __device__ inline PlainRows(const float *__restrict__ base, int64_t row_stride, int r, int n, int half) {
#pragma unroll
        for (int u = 0; u < R; ++u) p[u] = base + (r + u < n ? r + u : n - 1) * row_stride + half * 4;
    }
    __device__ inline void dots(float (&y)[R], const PlainRow<D> &a) const {
        float s[R][4];
#pragma unroll
        for (int g = 0; g < D / 8; ++g) {
            if (g % 4 == 0) __builtin_amdgcn_sched_barrier(0);   // not all of the rows at once, for which there are no registers
#pragma unroll
            for (int u = 0; u < R; ++u) {
                const float4 f = *reinterpret_cast<const float4 *>(p[u] + g * 8);
                s[u][0] = fmaf(a.x[4 * g], f.x, g ? s[u][0] : 0.0f); s[u][1] = fmaf(a.x[4 * g + 1], f.y, g ? s[u][1] : 0.0f);
                s[u][2] = fmaf(a.x[4 * g + 2], f.z, g ? s[u][2] : 0.0f); s[u][3] = fmaf(a.x[4 * g + 3], f.w, g ? s[u][3] : 0.0f);
            }
        }
#pragma unroll
        for (int u = 0; u < R; ++u) y[u] = pair_sum((s[u][0] + s[u][1]) + (s[u][2] + s[u][3]));
    }
    // acc += the sum of x[u] row[u] over the rows that count: the others, and their x, are not looked at
    __device__ inline void add(f32x16 (&acc)[D / 32], const float (&x)[R], const bool (&counts)[R]) const {
#pragma unroll
        for (int g = 0; g < D / 8; ++g) {
            if (g % 4 == 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < R; ++u) {
                float4 f = *reinterpret_cast<const float4 *>(p[u] + g * 8);
                const float c = counts[u] ? x[u] : 0.0f;
                f.x = counts[u] ? f.x : 0.0f; f.y = counts[u] ? f.y : 0.0f; f.z = counts[u] ? f.z : 0.0f; f.w = counts[u] ? f.w : 0.0f;
                f32x16 &y = acc[g >> 2];
                const int e = 4 * (g & 3);
                y[e] = fmaf(c, f.x, y[e]); y[e + 1] = fmaf(c, f.y, y[e + 1]); y[e + 2] = fmaf(c, f.z, y[e + 2]); y[e + 3] = fmaf(c, f.w, y[e + 3]);
            }
        }
    }
};
// A NaN has no split either, but taken again it is the same NaN, and so the rows are looked through for NaN first, 32 at a time (all
// of a batch NaN, forward and backward, 31 ms -> 0.44, one NaN per sample 31 -> 0.6; the ordinary call 0.44).
// nan_row: the first (kLast: the last) of rows from .. n - 1 that holds one, n (kLast: -1) if none does; the same in every lane.
template <bool kLast> __device__ inline int nearer(int a, int b) { return kLast == (a > b) ? a : b; }
template <int D, bool kLast> struct NanScan {
    static constexpr int kLanes = D / 4, kRows = 64 / kLanes;   // lanes to a row, rows to a load
    const float *base;
    int64_t row_stride;
    int from, n, lane;
    // calls look(row, four columns' values) for 32 rows, done() after them, until it says so
    template <typename F, typename G> __device__ inline void run(F look, G done) const {
        const int blocks = (n - from + 31) / 32;
        for (int i = 0; i < blocks; ++i) {
            const int r0 = from + 32 * (kLast ? blocks - 1 - i : i) + lane / kLanes;
#pragma unroll
            for (int u = 0; u < 32 / kRows; ++u) {
                const int r = r0 + u * kRows < n ? r0 + u * kRows : n - 1;
                look(r, *reinterpret_cast<const float4 *>(base + r * row_stride + lane % kLanes * 4));
            }
            if (done()) break;
        }
    }
};
template <int D, bool kLast> __device__ inline int nan_row(const float *__restrict__ base, int64_t row_stride, int from, int n, int lane) {
    const int none = kLast ? -1 : n;
    int found = none;
    NanScan<D, kLast>{base, row_stride, from, n, lane}.run(
        [&](int r, float4 f) { if (f.x != f.x || f.y != f.y || f.z != f.z || f.w != f.w) found = nearer<kLast>(found, r); },
        [&]() { return __builtin_amdgcn_ballot_w64(found != none) != 0; });
    for (int d = 1; d < 64; d <<= 1) found = nearer<kLast>(found, __shfl_xor(found, d, 64));
    return found;
}
// The same for each column, and whether results of this lane that are not finite (columns on the accumulator's rows) may be anything
// but the NaN of a row that counts: those before `limit` (kLast: from `limit` on).
template <int D, bool kLast> __device__ inline bool values_besides_nan(const f32x16 (&acc)[D / 32], const float *__restrict__ base, int64_t row_stride,
                                                                       int from, int n, int limit, int lane) {
    using Scan = NanScan<D, kLast>;
    const int none = kLast ? -1 : n, half = lane >> 5;
    int found[4] = {none, none, none, none};   // of columns 4 (lane % kLanes) ..
    Scan{base, row_stride, from, n, lane}.run(
        [&](int r, float4 f) {
            if (f.x != f.x) found[0] = nearer<kLast>(found[0], r);
            if (f.y != f.y) found[1] = nearer<kLast>(found[1], r);
            if (f.z != f.z) found[2] = nearer<kLast>(found[2], r);
            if (f.w != f.w) found[3] = nearer<kLast>(found[3], r);
        },
        [&]() { return __builtin_amdgcn_ballot_w64(found[0] == none || found[1] == none || found[2] == none || found[3] == none) == 0; });
#pragma unroll
    for (int c = 0; c < 4; ++c)
        for (int d = Scan::kLanes; d < 64; d <<= 1) found[c] = nearer<kLast>(found[c], __shfl_xor(found[c], d, 64));
    bool any = false;
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = __shfl(found[e & 3], (db * 32 + acc_row(e, half)) >> 2, 64);
            any = any || (!(fabsf(acc[db][e]) < INFINITY) && (kLast ? row < limit : row >= limit));
        }
    return any;
}

template <int D>
__global__ __launch_bounds__(kSpThreads, 2) void fwd_split_kernel(
        const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
        const int64_t *__restrict__ offsets, const int64_t *__restrict__ offsets_kv, bool causal, int B, int H, Schedule s,
        float *__restrict__ out, float *__restrict__ lse) {
    constexpr int kRows = kF32SplitRows, kStage = sp_stage<D>(), kRowsAgain = 2;
    __shared__ __attribute__((aligned(1024))) char sm[2 * kStage];   // two stages: the planes of K, then of V
    __shared__ int64_t slot;
    __shared__ SmallWork mine;
    static_assert(sizeof(sm) >= kInlineScratchInts * sizeof(int), "the stage buffers double as the scheduler's scratch");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const NarrowAddresses<D> at(lane);
    const float scale = 1.0f / sqrtf((float)D);
    const bool small = s.build_rows != 0;   // small problem: no scheduler launch has run, the schedule is built here, in LDS
    if (small) build_small_work(offsets, offsets_kv, B, H, s.build_rows, reinterpret_cast<int *>(sm), &mine);
    const int64_t total = small ? 0 : (int64_t)s.tile_start[B] * H;
    const int64_t sum_B = offsets[B];
    const int64_t row_stride = (int64_t)H * D;

    WorkCursor cursor;
    cursor.static_only = s.static_only;
    Work t;   // keys: rows orow0 .. orow0 + olen - 1
    for (int item = 0; next_item(t, mine, small, item, s, offsets, offsets_kv, B, H, cursor, total, &slot); ++item) {
        const int L = t.olen;
        const int q0 = t.block * kRows + wave * 32;    // first query of the wave
        const int i = q0 + col;                        // this lane's query
        const int iq = i < t.len ? i : t.len - 1;      // rows past the end recompute the last row
        const bool active = q0 < t.len;
        // causal (self attention only): query i sees keys 0 .. i, so the tile needs the keys up to its last query
        const int Lc = causal && (t.block + 1) * kRows < L ? (t.block + 1) * kRows : L;
        const float *kbase = k + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *vbase = v + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *qrow = q + (t.row0 + iq) * row_stride + (int64_t)t.head * D;
        SplitStage<D> next;
        next.fetch(kbase, vbase, row_stride, 0, L, wave, lane);
        bf16x8 qr[3][D / 16];
        load_split<D>(qr, qrow, half);
        f32x16 o[D / 32];
        clear<D>(o);
        float m = -INFINITY, l = 0.0f;   // running maximum of the scores; this lane's share of the row sum
        next.store(sm, wave, lane);
        __syncthreads();
        for (int j0 = 0, buf = 0; j0 < Lc; j0 += kSpRows, buf ^= 1) {
            const bool more = j0 + kSpRows < Lc;
            if (more) next.fetch(kbase, vbase, row_stride, j0 + kSpRows, L, wave, lane);
            if (active && !(causal && j0 > q0 + 31)) {
                const char *kt = sm + buf * kStage, *vt = kt + sp_tensor<D>();
                f32x16 st = product<D>(kt, at, qr);
                if (j0 + 32 > L || (causal && j0 + 31 > q0)) {   // keys past the sample's end or above the diagonal
                    const int lim = (causal && iq + 1 < L ? iq + 1 : L) - j0;
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (acc_row(e, half) >= lim) st[e] = -INFINITY;
                }
                float mx = st[0];
#pragma unroll
                for (int e = 1; e < 16; ++e) mx = fmaxf(mx, st[e]);
                const float m_new = fmaxf(m, pair_max(mx) * (scale * kProductScale));   // finite: every query of a block that is not skipped sees one of its keys
                if (__builtin_amdgcn_ballot_w64(m_new > m) != 0) {
                    const float a = exp_f32(m - m_new);   // exp(-inf) = 0 on the first block
                    m = m_new;
                    l *= a;
#pragma unroll
                    for (int db = 0; db < D / 32; ++db)
#pragma unroll
                        for (int e = 0; e < 16; ++e) o[db][e] *= a;
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) st[e] = exp_f32(fmaf(st[e], scale * kProductScale, -m));
                l += ((st[0] + st[1]) + (st[2] + st[3])) + ((st[4] + st[5]) + (st[6] + st[7])) +
                     (((st[8] + st[9]) + (st[10] + st[11])) + ((st[12] + st[13]) + (st[14] + st[15])));
                accumulate<D>(o, vt, at, st);
            }
            if (more) next.store(sm + (buf ^ 1) * kStage, wave, lane);
            lds_barrier();
        }
        l = pair_sum(l);
        float back = kProductScale;
        if (active && __builtin_amdgcn_ballot_w64(!all_finite<D>(o) || !(l < INFINITY)) != 0) {
            unscale<D>(o);
            back = 1.0f;
            const int lim = causal && iq + 1 < L ? iq + 1 : L, seen = causal && q0 + 32 < L ? q0 + 32 : L;   // keys of this lane, of the wave
            PlainRow<D> q_row;
            q_row.load(qrow, half);
            const bool q_nan = q_row.has_nan();
            const int k_nan = nan_row<D, false>(kbase, row_stride, 0, seen, lane);
            const bool nan = q_nan || k_nan < lim, scores = !(l < INFINITY) || !(fabsf(m) < INFINITY);   // scores: all of the row is taken again
            bool again = !nan && scores;
            if (__builtin_amdgcn_ballot_w64(!nan && !scores && !all_finite<D>(o)) != 0) {
                const bool values = values_besides_nan<D, false>(o, vbase, row_stride, 0, seen, lim, lane);
                again = again || (!nan && values);
            }
            if (__builtin_amdgcn_ballot_w64(again) != 0) {
                float m2 = m, l2 = 0.0f;
                if (__builtin_amdgcn_ballot_w64(scores) != 0) {
                    float top = -INFINITY;
                    for (int j = 0; j < seen; j += kRowsAgain) {
                        float y[kRowsAgain];
                        PlainRows<D, kRowsAgain>(kbase, row_stride, j, seen, half).dots(y, q_row);
#pragma unroll
                        for (int u = 0; u < kRowsAgain; ++u)
                            if (j + u < lim) top = fmaxf(top, y[u] * scale);
                    }
                    if (scores) m2 = top;
                }
                f32x16 o2[D / 32];
                clear<D>(o2);
                for (int j = 0; j < seen; j += kRowsAgain) {
                    float p[kRowsAgain];
                    bool counts[kRowsAgain];
                    PlainRows<D, kRowsAgain>(kbase, row_stride, j, seen, half).dots(p, q_row);
#pragma unroll
                    for (int u = 0; u < kRowsAgain; ++u) {
                        p[u] = exp_f32(fmaf(p[u], scale, -m2));
                        counts[u] = j + u < lim;
                        if (counts[u]) l2 += p[u];
                    }
                    PlainRows<D, kRowsAgain>(vbase, row_stride, j, seen, half).add(o2, p, counts);
                }
                if (scores) {
                    m = m2;
                    l = l2;
#pragma unroll
                    for (int db = 0; db < D / 32; ++db) o[db] = o2[db];
                } else {
                    take_where_not_finite<D>(o, o2);
                }
            }
        }
        if (i < t.len) {   // a sample without keys: out = 0, lse = -inf
            store_row<D>(out + (t.row0 + i) * row_stride + (int64_t)t.head * D, o, l > 0.0f ? back / l : 0.0f, half);
            if (half == 0) lse[(int64_t)t.head * sum_B + t.row0 + i] = m + logf(l);
        }
    }
}

// dQ: stream the sample's keys.  The kernel is the first of the backward: it holds each query's dO row anyway, reads the matching
// row of the forward's output, and computes delta = rowsum(dO o O) for its own use and for the dK / dV kernel.
template <int D>
__global__ __launch_bounds__(kSpThreads, 2) void dq_split_kernel(
        const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
        const float *__restrict__ out_fwd, const float *__restrict__ dout, const float *__restrict__ lse,
        float *__restrict__ delta, const int64_t *__restrict__ offsets, const int64_t *__restrict__ offsets_kv, bool causal,
        int B, int H, Schedule s, float *__restrict__ dq) {
    constexpr int kRows = kF32SplitRows, kStage = sp_stage<D>(), kRowsAgain = 2;
    __shared__ __attribute__((aligned(1024))) char sm[2 * kStage];   // two stages: the planes of K, then of V
    __shared__ int64_t slot;
    __shared__ SmallWork mine;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const NarrowAddresses<D> at(lane);
    const float scale = 1.0f / sqrtf((float)D);
    const bool small = s.build_rows != 0;
    if (small) build_small_work(offsets, offsets_kv, B, H, s.build_rows, reinterpret_cast<int *>(sm), &mine);
    const int64_t total = small ? 0 : (int64_t)s.tile_start[B] * H;
    const int64_t sum_B = offsets[B];
    const int64_t row_stride = (int64_t)H * D;

    WorkCursor cursor;
    cursor.static_only = s.static_only;
    Work t;
    for (int item = 0; next_item(t, mine, small, item, s, offsets, offsets_kv, B, H, cursor, total, &slot); ++item) {
        const int L = t.olen;
        const int q0 = t.block * kRows + wave * 32;
        const int i = q0 + col;
        const int iq = i < t.len ? i : t.len - 1;
        const bool active = q0 < t.len;
        const int Lc = causal && (t.block + 1) * kRows < L ? (t.block + 1) * kRows : L;
        const float *kbase = k + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *vbase = v + t.orow0 * row_stride + (int64_t)t.head * D;
        SplitStage<D> next;
        next.fetch(kbase, vbase, row_stride, 0, L, wave, lane);
        const int64_t row = (t.row0 + iq) * row_stride + (int64_t)t.head * D;
        const int half_i = not_hoisted(half);
        float dot = 0.0f;
#pragma unroll
        for (int g = 0; g < D / 8; ++g) {
            const float4 a = *reinterpret_cast<const float4 *>(dout + row + 8 * g + 4 * half_i), f = *reinterpret_cast<const float4 *>(out_fwd + row + 8 * g + 4 * half_i);
            dot = fmaf(a.x, f.x, fmaf(a.y, f.y, fmaf(a.z, f.z, fmaf(a.w, f.w, dot))));
        }
        const float delta_i = pair_sum(dot);   // the two lanes of a row hold half of its features each
        const float lse_i = lse[(int64_t)t.head * sum_B + t.row0 + iq];
        if (i < t.len && half == 0) delta[(int64_t)t.head * sum_B + t.row0 + i] = delta_i;
        bf16x8 qr[3][D / 16], dor[3][D / 16];
        load_split<D>(qr, q + row, half_i);
        load_split<D>(dor, dout + row, half_i);
        f32x16 acc[D / 32];
        clear<D>(acc);
        next.store(sm, wave, lane);
        __syncthreads();
        for (int j0 = 0, buf = 0; j0 < Lc; j0 += kSpRows, buf ^= 1) {
            const bool more = j0 + kSpRows < Lc;
            if (more) next.fetch(kbase, vbase, row_stride, j0 + kSpRows, L, wave, lane);
            if (active && !(causal && j0 > q0 + 31)) {
                const char *kt = sm + buf * kStage, *vt = kt + sp_tensor<D>();
                f32x16 st = product<D>(kt, at, qr);
                __builtin_amdgcn_sched_barrier(0);   // one product after the other: side by side they spill
                const f32x16 dp = product<D>(vt, at, dor);
                const bool masked = j0 + 32 > L || (causal && j0 + 31 > q0);
                const int lim = (causal && iq + 1 < L ? iq + 1 : L) - j0;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float p = exp_f32(fmaf(st[e], scale * kProductScale, -lse_i));
                    if (masked && acc_row(e, half) >= lim) p = 0.0f;
                    st[e] = p * fmaf(dp[e], kProductScale, -delta_i);
                }
                __builtin_amdgcn_sched_barrier(0);
                accumulate<D>(acc, kt, at, st);
            }
            if (more) next.store(sm + (buf ^ 1) * kStage, wave, lane);
            lds_barrier();
        }
        const int lane_e = not_hoisted(lane);
        const int i_e = q0 + (lane_e & 31), half_e = lane_e >> 5, iq_e = i_e < t.len ? i_e : t.len - 1;
        const int64_t row_e = (t.row0 + iq_e) * row_stride + (int64_t)t.head * D;
        float back = scale * kProductScale;
        if (active && __builtin_amdgcn_ballot_w64(!all_finite<D>(acc)) != 0) {
            unscale<D>(acc);
            back = scale;
            const int lim = causal && iq_e + 1 < L ? iq_e + 1 : L, seen = causal && q0 + 32 < L ? q0 + 32 : L;   // keys of this lane, of the wave
            const float lse_e = lse[(int64_t)t.head * sum_B + t.row0 + iq_e];
            PlainRow<D> q_row, g_row;
            q_row.load(q + row_e, half_e);
            g_row.load(dout + row_e, half_e);
            float same[1];
            PlainRows<D, 1>(out_fwd + row_e, 0, 0, 1, half_e).dots(same, g_row);
            const float delta_e = same[0];
            const bool q_nan = q_row.has_nan(), g_nan = g_row.has_nan(), own = q_nan || g_nan || lse_e != lse_e || delta_e != delta_e;
            bool open = !own && !all_finite<D>(acc);
            if (__builtin_amdgcn_ballot_w64(open) != 0) {
                const int k_nan = nan_row<D, false>(kbase, row_stride, 0, seen, lane_e), v_nan = nan_row<D, false>(vbase, row_stride, 0, seen, lane_e);
                open = open && k_nan >= lim && v_nan >= lim;
            }
            if (__builtin_amdgcn_ballot_w64(open) != 0) {
                f32x16 again[D / 32];
                clear<D>(again);
                for (int j = 0; j < seen; j += kRowsAgain) {
                    float ds[kRowsAgain], dp[kRowsAgain];
                    bool counts[kRowsAgain];
                    PlainRows<D, kRowsAgain>(kbase, row_stride, j, seen, half_e).dots(ds, q_row);
                    PlainRows<D, kRowsAgain>(vbase, row_stride, j, seen, half_e).dots(dp, g_row);
#pragma unroll
                    for (int u = 0; u < kRowsAgain; ++u) {
                        ds[u] = exp_f32(fmaf(ds[u], scale, -lse_e)) * (dp[u] - delta_e);
                        counts[u] = j + u < lim;
                    }
                    PlainRows<D, kRowsAgain>(kbase, row_stride, j, seen, half_e).add(again, ds, counts);
                }
                take_where_not_finite<D>(acc, again);
            }
        }
        if (i_e < t.len) store_row<D>(dq + row_e, acc, back, half_e);
    }
}

// dK, dV: stream the sample's queries (with their lse, delta).  Planes of K and V and both accumulators of 32 keys do not fit one
// wave at two waves per SIMD, so a pair of waves shares them: wave A holds K, forms S and P and accumulates dV, wave B holds V,
// forms dP, takes P from A through LDS (behind a barrier in the middle of the stage: both have one product before and one
// behind it) and accumulates dK.
template <int D>
__global__ __launch_bounds__(kSpThreads, 2) void dkv_split_kernel(
        const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
        const float *__restrict__ dout, const float *__restrict__ lse, const float *__restrict__ delta,
        const int64_t *__restrict__ offsets,   // of the keys
        const int64_t *__restrict__ offsets_q, bool causal, int B, int H, Schedule s, float *__restrict__ dk,
        float *__restrict__ dv) {
    constexpr int kRows = kF32SplitKeyRows, kStage = sp_stage<D>(), kRowsAgain = 1;
    __shared__ __attribute__((aligned(1024))) char sm[2 * kStage];   // two stages: the planes of Q, then of dO
    __shared__ __attribute__((aligned(16))) float stat_s[2][2][kSpRows];   // per stage: lse of the streamed rows, then delta
    __shared__ f32x4 px[2][4][64];                                   // per pair: a 32 x 32 block of P on its way from A to B
    __shared__ int64_t slot;
    __shared__ SmallWork mine;
    static_assert(sizeof(sm) >= kInlineScratchInts * sizeof(int), "the stage buffers double as the scheduler's scratch");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int pair = wave & 1;
    const bool is_a = wave < 2;
    const NarrowAddresses<D> at(lane);
    const float scale = 1.0f / sqrtf((float)D);
    const bool small = s.build_rows != 0;
    if (small) build_small_work(offsets, offsets_q, B, H, s.build_rows, reinterpret_cast<int *>(sm), &mine);
    const int64_t total = small ? 0 : (int64_t)s.tile_start[B] * H;
    const int64_t sum_B = offsets_q ? offsets_q[B] : offsets[B];   // lse and delta are indexed by query rows
    const int64_t row_stride = (int64_t)H * D;

    WorkCursor cursor;
    cursor.static_only = s.static_only;
    Work t;   // queries: rows orow0 .. orow0 + olen - 1
    for (int item = 0; next_item(t, mine, small, item, s, offsets, offsets_q, B, H, cursor, total, &slot); ++item) {
        const int L = t.olen;
        const int k0 = t.block * kRows + pair * 32;    // first key of the pair
        const int j = k0 + col;                        // this lane's key
        const int jk = j < t.len ? j : t.len - 1;
        const bool active = k0 < t.len;
        const float *qbase = q + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *obase = dout + t.orow0 * row_stride + (int64_t)t.head * D;
        const float *lse_rows = lse + (int64_t)t.head * sum_B + t.orow0;
        const float *delta_rows = delta + (int64_t)t.head * sum_B + t.orow0;
        // causal: key j is seen by queries j .. L - 1, so the stream starts at the stage that holds the tile's first key
        const int istart = causal ? t.block * kRows : 0;
        float stat_next = 0.0f;      // a statistic of the stage on its way (threads 0 .. 63)
        SplitStage<D> next;
        auto fetch = [&](int i0) {
            next.fetch(qbase, obase, row_stride, i0, L, wave, lane);
            if (tid < 2 * kSpRows) {
                const int i = i0 + tid % kSpRows < L ? i0 + tid % kSpRows : L - 1;
                stat_next = (tid < kSpRows ? lse_rows : delta_rows)[i];
            }
        };
        auto store = [&](int buf) {
            next.store(sm + buf * kStage, wave, lane);
            if (tid < 2 * kSpRows) stat_s[buf][tid / kSpRows][tid % kSpRows] = stat_next;
        };
        if (istart < L) fetch(istart);
        bf16x8 sr[3][D / 16];   // K in wave A, V in wave B
        const int64_t row = (t.row0 + jk) * row_stride + (int64_t)t.head * D;
        load_split<D>(sr, (is_a ? k : v) + row, half);
        f32x16 acc[D / 32];     // dV in wave A, dK in wave B
        clear<D>(acc);
        if (istart < L) store(0);
        __syncthreads();
        for (int i0 = istart, buf = 0; i0 < L; i0 += kSpRows, buf ^= 1) {
            const bool more = i0 + kSpRows < L;
            if (more) fetch(i0 + kSpRows);
            const bool run = active && !(causal && i0 + 31 < k0);
            const char *qt = sm + buf * kStage, *ot = qt + sp_tensor<D>();
            f32x16 x;
            if (run) {
                x = product<D>(is_a ? qt : ot, at, sr);
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4 stat = *reinterpret_cast<const f32x4 *>(&stat_s[buf][is_a ? 0 : 1][g * 8 + half * 4]);
#pragma unroll
                    for (int e = 0; e < 4; ++e) x[4 * g + e] = is_a ? exp_f32(fmaf(x[4 * g + e], scale * kProductScale, -stat[e])) : fmaf(x[4 * g + e], kProductScale, -stat[e]);
                }
                if (is_a) {
                    if (i0 + 32 > L || (causal && i0 < k0 + 31)) {
                        const int lo = causal ? j - i0 : 0, hi = L - i0;   // this lane's key is seen by block rows lo .. hi - 1
#pragma unroll
                        for (int e = 0; e < 16; ++e) {
                            const int r = acc_row(e, half);
                            if (r < lo || r >= hi) x[e] = 0.0f;
                        }
                    }
#pragma unroll
                    for (int g = 0; g < 4; ++g) px[pair][g][lane] = f32x4{x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
                }
            }
            lds_barrier();   // P is written
            if (run) {
                if (!is_a) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 p = px[pair][g][lane];
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[4 * g + e] *= p[e];
                    }
                }
                accumulate<D>(acc, is_a ? ot : qt, at, x);
            }
            if (more) store(buf ^ 1);
            lds_barrier();
        }
        float back = is_a ? kProductScale : scale * kProductScale;
        if (active && __builtin_amdgcn_ballot_w64(!all_finite<D>(acc)) != 0) {
            unscale<D>(acc);
            back = is_a ? 1.0f : scale;
            const int from = causal ? k0 : 0, mine_from = causal ? jk : 0;   // the first query of the wave, of this lane's key
            PlainRow<D> k_row, v_row;
            k_row.load(k + row, half);
            v_row.load(v + row, half);
            const bool own_k = k_row.has_nan(), own_v = v_row.has_nan();
            bool open = !all_finite<D>(acc) && !own_k && (is_a || !own_v);
            if (__builtin_amdgcn_ballot_w64(open) != 0) {
                int stat_nan = -1;   // last query whose statistics are NaN (dV does not look at delta)
                for (int i = from + lane; i < L; i += 64) {
                    const float x = lse_rows[i], y = is_a ? 0.0f : delta_rows[i];
                    if (x != x || y != y) stat_nan = i;
                }
                for (int d = 1; d < 64; d <<= 1) stat_nan = nearer<true>(stat_nan, __shfl_xor(stat_nan, d, 64));
                const int q_nan = nan_row<D, true>(qbase, row_stride, from, L, lane);
                open = open && stat_nan < mine_from && q_nan < mine_from;
            }
            if (__builtin_amdgcn_ballot_w64(open) != 0) {   // dK takes all of a gradient's columns, dV one
                const bool values = is_a ? values_besides_nan<D, true>(acc, obase, row_stride, from, L, mine_from, lane)
                                         : nan_row<D, true>(obase, row_stride, from, L, lane) < mine_from;
                open = open && values;
            }
            if (__builtin_amdgcn_ballot_w64(open) != 0) {
                f32x16 again[D / 32];
                clear<D>(again);
                for (int i = from; i < L; i += kRowsAgain) {
                    float x[kRowsAgain], dp[kRowsAgain];
                    bool counts[kRowsAgain];
                    PlainRows<D, kRowsAgain>(qbase, row_stride, i, L, half).dots(x, k_row);
                    if (!is_a) PlainRows<D, kRowsAgain>(obase, row_stride, i, L, half).dots(dp, v_row);
#pragma unroll
                    for (int u = 0; u < kRowsAgain; ++u) {
                        const int r = i + u < L ? i + u : L - 1;
                        x[u] = exp_f32(fmaf(x[u], scale, -lse_rows[r]));
                        if (!is_a) x[u] *= dp[u] - delta_rows[r];
                        counts[u] = i + u >= mine_from && i + u < L;
                    }
                    PlainRows<D, kRowsAgain>(is_a ? obase : qbase, row_stride, i, L, half).add(again, x, counts);
                }
                take_where_not_finite<D>(acc, again);
            }
        }
        if (j < t.len) store_row<D>((is_a ? dv : dk) + row, acc, back, half);
    }
}

#define JFA_LAUNCH(KERNEL, ...)                                                                                    \
    switch (D) {                                                                                                  \
        case 32: hipLaunchKernelGGL(KERNEL<32>, dim3(persistent_grid<KERNEL<32>>(kSpThreads, cus)), dim3(kSpThreads), 0, stream, __VA_ARGS__); break; \
        case 64: hipLaunchKernelGGL(KERNEL<64>, dim3(persistent_grid<KERNEL<64>>(kSpThreads, cus)), dim3(kSpThreads), 0, stream, __VA_ARGS__); break; \
        default: return hipErrorInvalidValue;                                                                     \
    }                                                                                                             \
    return hipGetLastError();

hipError_t launch_fwd_f32_split(const float *q, const float *k, const float *v, const int64_t *offsets, const int64_t *offsets_kv, bool causal,
                                int B, int H, int D, Schedule s, float *out, float *lse, int cus, hipStream_t stream) {
    JFA_LAUNCH(fwd_split_kernel, q, k, v, offsets, offsets_kv, causal, B, H, s, out, lse)
}

hipError_t launch_dq_f32_split(const float *q, const float *k, const float *v, const float *out, const float *dout, const float *lse,
                               const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s,
                               float *dq, float *delta, int cus, hipStream_t stream) {
    JFA_LAUNCH(dq_split_kernel, q, k, v, out, dout, lse, delta, offsets, offsets_kv, causal, B, H, s, dq)
}

hipError_t launch_dkv_f32_split(const float *q, const float *k, const float *v, const float *dout, const float *lse, const float *delta,
                                const int64_t *offsets, const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s,
                                float *dk, float *dv, int cus, hipStream_t stream) {
    JFA_LAUNCH(dkv_split_kernel, q, k, v, dout, lse, delta, offsets, offsets_q, causal, B, H, s, dk, dv)
}
#undef JFA_LAUNCH

}  // namespace jfa
