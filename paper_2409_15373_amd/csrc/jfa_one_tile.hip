// Jagged flash attention, bf16, for samples of at most 128 queries and keys: a workgroup holds all of a (sample, head) and makes
// one pass over it, forward and backward.
//
// What bounds such a call is neither arithmetic nor memory but the chain of latencies that every work item starts and ends with (work
// list, offsets, rows, results), so the kernels keep it short and many of them in flight: the work item is the workgroup's index (no
// work list is built, nothing is claimed), a workgroup is a wave per 32 queries (backward: a pair of waves), and as many as LDS has
// room for share a compute unit.  The backward forms S and dP in both orientations (a query per lane for dQ, a key per lane for dK
// and dV: the accumulator is then in operand position, see jfa_mfma.h) out of the same tiles, each in a wave of its own, so that one
// kernel reads Q, K, V, dO, O once and writes all three gradients; they go to whole-row stores through tiles that have been read.
// Microseconds against the persistent kernels with their two-kernel backward (in brackets: the time to copy what a call must move,
// and a launch): 4096 samples of up to 32 rows, forward D = 64 36.4 -> 8.5 (10.2), D = 128 53.8 -> 16.0 (17.3), backward 61.3 -> 17.5
// (20.5) and 153 -> 31.0 (34.7); 3000 x 8 heads of up to 64, D = 128, 297 -> 153 (169) and 1087 -> 348 (340); 4 samples of up to 20,
// D = 64, 6.7 -> 3.9 and 12.8 -> 4.9.  One wave for both orientations of the backward: 4096 of up to 32, D = 128, 47.9.  A loop over
// items instead of a workgroup for each: its invariants take 100 registers more, 3000 x 8, D = 64, forward 77 -> 98.  P and dS of all
// of a wave's blocks kept as operands until the second barrier instead of one block at a time: 3000 x 8 of up to 64, D = 64, backward
// 180 -> 194 (D = 128, causal, the other way about: 400 -> 384, eleven registers are spilled).
#include "jfa_common.h"
#include "jfa_lds.h"
#include "jfa_mfma.h"
#include "jfa_narrow.h"
#include "jfa_bwd_dma.h"

namespace jfa {

// A tile is 32 rows of D bf16, row r's 16-byte chunk ch at r * kRow + ((ch ^ swizzle(r)) << 4): as the streamed tiles of the
// kernels for longer samples, conflict-free for the 16-byte row reads and for the transposing reads.
template <int D>
struct OneTile {
    static constexpr int kRow = D * 2, kChunks = D / 8, kTile = 32 * kRow, kKSteps = D / 16, kDBlocks = D / 32;
    static constexpr int kRowsPerCopy = 64 / kChunks, kCopies = 32 / kRowsPerCopy;   // a wave instruction moves 1 KB
    __device__ static inline int swizzle(int r) {
        if constexpr (D == 128) return swz(r);
        else return Narrow<D>::swz(r);
    }
    int lane, col, half;
    int row[kKSteps];          // chunk 2 ks + half of row `col`
    int tr[2][kDBlocks];       // transposing read: row 4 half + (lane & 15) / 4 (+ 8 for the operand's second half)
    __device__ inline OneTile() {
        lane = threadIdx.x & 63;
        col = lane & 31;
        half = lane >> 5;
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks) row[ks] = col * kRow + (((2 * ks + half) ^ swizzle(col)) << 4);
        const int r = half * 4 + ((lane & 15) >> 2), chunk = ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1), byte = (lane & 1) * 8;
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int db = 0; db < kDBlocks; ++db) tr[h2][db] = (r + 8 * h2) * kRow + (((db * 4 + chunk) ^ swizzle(r + 8 * h2)) << 4) + byte;
    }
    // the first `valid` of 32 rows of two tensors with equal offsets -> two tiles; rows past them repeat the last one
    __device__ inline void copy(const __bf16 *a, const __bf16 *b, int64_t row_stride, int valid, char *ta, char *tb) const {
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            const int r = u * kRowsPerCopy + lane / kChunks;
            const int64_t off = (r < valid ? r : valid - 1) * row_stride + (((lane % kChunks) ^ swizzle(r)) << 3);
            dma16_lane(a + off, ta + u * 1024);
            dma16_lane(b + off, tb + u * 1024);
        }
    }
    __device__ inline void fragments(bf16x8 (&f)[kKSteps], const char *tile) const {
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks) f[ks] = lds_read_b128(tile + row[ks]);
    }
    // (rows of the tile) x (rows f)^T: the tile's rows on the accumulator's rows, f's row on the lane
    __device__ inline f32x16 product(const char *tile, const bf16x8 (&f)[kKSteps]) const {
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks) acc = mfma_32x32x16(lds_read_b128(tile + row[ks]), f[ks], acc);
        return acc;
    }
    // g^T += tile^T x, x: 32 rows as two operands
    __device__ inline void accumulate(f32x16 (&g)[kDBlocks], const char *tile, const bf16x8 (&x)[2]) const {
#pragma unroll
        for (int ts = 0; ts < 2; ++ts)
#pragma unroll
            for (int db = 0; db < kDBlocks; ++db) {
                const char *t = tile + ts * 16 * kRow;
                g[db] = mfma_32x32x16(concat(lds_read_tr16(t + tr[0][db]), lds_read_tr16(t + tr[1][db])), x[ts], g[db]);
            }
    }
    __device__ inline void clear(f32x16 (&g)[kDBlocks]) const {
#pragma unroll
        for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) g[db][e] = 0.0f;
    }
    // g (this lane's column: row `col` of the result) scaled, through the wave's own tile `region` to whole rows of `dst`
    __device__ inline void store(char *region, const f32x16 (&g)[kDBlocks], float scale, __bf16 *dst, int64_t row_stride, int valid) const {
#pragma unroll
        for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bf16x4 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = (__bf16)(g[db][4 * q + e] * scale);
                *reinterpret_cast<bf16x4 *>(region + col * kRow + (((db * 4 + q) ^ swizzle(col)) << 4) + half * 8) = y;
            }
        wave_order();
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            const int r = u * kRowsPerCopy + lane / kChunks, ch = lane % kChunks;
            const u32x4 piece = *reinterpret_cast<const u32x4 *>(region + r * kRow + ((ch ^ swizzle(r)) << 4));
            if (r < valid) *reinterpret_cast<u32x4 *>(dst + r * row_stride + ch * 8) = piece;
        }
        wave_order();
    }
    __device__ inline void store_zeros(__bf16 *dst, int64_t row_stride, int valid) const {
#pragma unroll
        for (int u = 0; u < kCopies; ++u) {
            const int r = u * kRowsPerCopy + lane / kChunks;
            if (r < valid) *reinterpret_cast<u32x4 *>(dst + r * row_stride + lane % kChunks * 8) = u32x4{0, 0, 0, 0};
        }
    }
    // a wave's LDS instructions complete in order: only the compiler must keep them in it
    __device__ static inline void wave_order() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

// The workgroup's item: consecutive workgroups go to the eight dies in turn, so those of a die that follow each other take the
// heads of one sample, whose rows share cache lines, and consecutive samples go to different dies.
struct OneTileItem {
    int b, head, Lq, Lk;
    int64_t q0, k0;
    __device__ inline bool take(int64_t w, const int64_t *offsets_q, const int64_t *offsets_kv, int B, int H, int least, int most) {
        const int64_t i = w / kXcds, s = i / H * kXcds + w % kXcds;
        if (s >= B) return false;
        b = (int)s;
        head = (int)(i % H);
        q0 = offsets_q[b];
        Lq = (int)(offsets_q[b + 1] - q0);
        k0 = offsets_kv ? offsets_kv[b] : q0;
        Lk = offsets_kv ? (int)(offsets_kv[b + 1] - k0) : Lq;
        return Lq <= most && Lk <= most && (Lq > least || Lk > least);   // the others: another launch's
    }
};
static inline int64_t one_tile_items(int64_t B, int H) { return (B + kXcds - 1) / kXcds * kXcds * (int64_t)H; }

// The workgroup's LDS accesses so far are done; copies: its copies have landed, too.
template <int W, bool copies = false> __device__ inline void one_tile_barrier() {
    if (copies) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (W > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int D, int W, bool CAUSAL>
__global__ __launch_bounds__(64 * W, 2) void fwd_one_tile_kernel(const __bf16 *__restrict__ q, const __bf16 *__restrict__ k, const __bf16 *__restrict__ v,
                                                                 const int64_t *__restrict__ offsets, const int64_t *__restrict__ offsets_kv,
                                                                 int B, int H, int64_t first, int least, __bf16 *__restrict__ out, float *__restrict__ lse) {
    using T = OneTile<D>;
    __shared__ __attribute__((aligned(1024))) char kt[W][T::kTile], vt[W][T::kTile];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r0 = 32 * wave;
    const T ln;
    const int col = ln.col, half = ln.half;
    const float c = 1.4426950408889634f / sqrtf((float)D);
    const int64_t sum_B = offsets[B], row_stride = (int64_t)H * D;
    OneTileItem t;
    if (!t.take(first + blockIdx.x, offsets, offsets_kv, B, H, least, 32 * W)) return;
    const int Lq = t.Lq, Lk = t.Lk, i = r0 + col, iq = i < Lq ? i : Lq - 1;
    const int64_t kbase = (t.k0 + r0) * row_stride + (int64_t)t.head * D;
    const int64_t qbase = (t.q0 + r0) * row_stride + (int64_t)t.head * D;
    if (r0 < Lk && Lq > 0) ln.copy(k + kbase, v + kbase, row_stride, Lk - r0, kt[wave], vt[wave]);
    bf16x8 qf[T::kKSteps];
    if (r0 < Lq) {
        const __bf16 *row = q + (t.q0 + iq) * row_stride + (int64_t)t.head * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < T::kKSteps; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(row + 16 * ks);
    }
    one_tile_barrier<W, true>();
    if (Lq > 0 && Lk == 0 && r0 < Lq) {   // no keys: an empty softmax, out = 0 and lse = -inf
        ln.store_zeros(out + qbase, row_stride, Lq - r0);
        if (half == 0 && i < Lq) lse[(int64_t)t.head * sum_B + t.q0 + i] = -INFINITY;
    }
    if (Lk == 0) return;
    float m = -INFINITY, l = 0.0f;
    bf16x8 p[W][2];
    if (r0 < Lq) {
        const int lim = CAUSAL && iq + 1 < Lk ? iq + 1 : Lk;   // this lane's query sees keys 0 .. lim - 1
        f32x16 s[W];
#pragma unroll
        for (int kb = 0; kb < W; ++kb) {
            if (kb * 32 >= Lk || (CAUSAL && kb > wave)) continue;
            s[kb] = ln.product(kt[kb], qf);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                if (kb * 32 + acc_row(e, half) >= lim) s[kb][e] = -INFINITY;
                m = fmaxf(m, s[kb][e]);
            }
        }
        m = pair_max(m);
        const float mc = m * c;
#pragma unroll
        for (int kb = 0; kb < W; ++kb) {
            if (kb * 32 >= Lk || (CAUSAL && kb > wave)) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {   // the sum adds what the second product uses
                const __bf16 x = (__bf16)fast_exp2(fmaf(s[kb][e], c, -mc));
                p[kb][e >> 3][e & 7] = x;
                l += (float)x;
            }
        }
        l = pair_sum(l);
    }
    if (W > 1) one_tile_barrier<W>();   // the K tiles have been read: they carry the results
    if (r0 < Lq) {
        f32x16 o[T::kDBlocks];
        ln.clear(o);
#pragma unroll
        for (int kb = 0; kb < W; ++kb) {
            if (kb * 32 >= Lk || (CAUSAL && kb > wave)) continue;
            ln.accumulate(o, vt[kb], p[kb]);
        }
        ln.wave_order();
        ln.store(kt[wave], o, 1.0f / l, out + qbase, row_stride, Lq - r0);
        if (half == 0 && i < Lq) lse[(int64_t)t.head * sum_B + t.q0 + i] = (m * c + fast_log2(l)) * 0.6931471805599453f;
    }
}

// W pairs of waves: one of a pair has 32 queries and computes their dQ, the other 32 keys and computes their dK and dV.
template <int D, int W, bool CAUSAL>
__global__ __launch_bounds__(128 * W, 2) void bwd_one_tile_kernel(const __bf16 *__restrict__ q, const __bf16 *__restrict__ k, const __bf16 *__restrict__ v,
                                                                  const __bf16 *__restrict__ out, const __bf16 *__restrict__ dout,
                                                                  const float *__restrict__ lse, float *__restrict__ stats,   // [2, H, sum_B]
                                                                  const int64_t *__restrict__ offsets, const int64_t *__restrict__ offsets_kv,
                                                                  int B, int H, int64_t first, int least, __bf16 *__restrict__ dq, __bf16 *__restrict__ dk,
                                                                  __bf16 *__restrict__ dv) {
    using T = OneTile<D>;
    __shared__ __attribute__((aligned(1024))) char qt[W][T::kTile], gt[W][T::kTile], kt[W][T::kTile], vt[W][T::kTile];   // Q, dO, K, V
    __shared__ __attribute__((aligned(16))) float row_lse2[32 * W], row_delta[32 * W];   // lse * log2(e), delta per query
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool keys = wave >= W;
    const int tile = keys ? wave - W : wave, r0 = 32 * tile;
    const T ln;
    const int col = ln.col, half = ln.half;
    const float scale = 1.0f / sqrtf((float)D), c = 1.4426950408889634f * scale;
    const int64_t sum_B = offsets[B], row_stride = (int64_t)H * D;
    OneTileItem t;
    if (!t.take(first + blockIdx.x, offsets, offsets_kv, B, H, least, 32 * W)) return;
    const int Lq = t.Lq, Lk = t.Lk, mine = keys ? Lk : Lq;
    const int i = r0 + col;                                                                   // this lane's query or key
    const int64_t base = ((keys ? t.k0 : t.q0) + r0) * row_stride + (int64_t)t.head * D;      // of the wave's first row
    const int64_t stat = (int64_t)t.head * sum_B + t.q0 + i;
    if (Lq == 0 || Lk == 0) {   // one side is empty: the other's gradients are zero
        if (keys && r0 < Lk) {
            ln.store_zeros(dk + base, row_stride, Lk - r0);
            ln.store_zeros(dv + base, row_stride, Lk - r0);
        }
        if (!keys && r0 < Lq) {
            ln.store_zeros(dq + base, row_stride, Lq - r0);
            if (half == 0 && i < Lq) {
                stats[stat] = 0.0f;
                stats[(int64_t)H * sum_B + stat] = INFINITY;   // lse = -inf
            }
        }
        return;
    }
    if (r0 < mine) {
        if (keys) ln.copy(k + base, v + base, row_stride, Lk - r0, kt[tile], vt[tile]);
        else ln.copy(q + base, dout + base, row_stride, Lq - r0, qt[tile], gt[tile]);
    }
    if (!keys) {   // a query per lane
        bf16x8 of[T::kKSteps];
        float lse_i = 0.0f;
        if (r0 < Lq) {
            const int iq = i < Lq ? col : Lq - 1 - r0;
            const __bf16 *row = out + base + (int64_t)iq * row_stride + half * 8;
#pragma unroll
            for (int ks = 0; ks < T::kKSteps; ++ks) of[ks] = *reinterpret_cast<const bf16x8 *>(row + 16 * ks);
            lse_i = lse[(int64_t)t.head * sum_B + t.q0 + r0 + iq];
        }
        one_tile_barrier<2, true>();
        bf16x8 qf[T::kKSteps], gf[T::kKSteps];
        float delta = 0.0f;
        const float lse2 = lse_i * 1.4426950408889634f;
        if (r0 < Lq) {
            ln.fragments(qf, qt[tile]);
            ln.fragments(gf, gt[tile]);
#pragma unroll
            for (int ks = 0; ks < T::kKSteps; ++ks)
#pragma unroll
                for (int e = 0; e < 8; ++e) delta = fmaf((float)of[ks][e], (float)gf[ks][e], delta);
            delta = pair_sum(delta);
            if (half == 0) {
                row_lse2[i] = lse2;
                row_delta[i] = delta;
                if (i < Lq) {
                    stats[stat] = delta;
                    stats[(int64_t)H * sum_B + stat] = -lse_i * sqrtf((float)D);
                }
            }
        }
        one_tile_barrier<2>();   // the statistics are there
        f32x16 g[T::kDBlocks];
        ln.clear(g);
        const int lim = CAUSAL && i + 1 < Lk ? i + 1 : Lk;   // this lane's query sees keys 0 .. lim - 1
        if (r0 < Lq)
            for (int kb = 0; kb < W && kb * 32 < Lk && !(CAUSAL && kb > tile); ++kb) {
                const f32x16 s = ln.product(kt[kb], qf), dp = ln.product(vt[kb], gf);
                bf16x8 ds[2];   // dS, keys on the rows
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const float x = fast_exp2(fmaf(s[e], c, -lse2)) * (dp[e] - delta);
                    ds[e >> 3][e & 7] = (__bf16)(kb * 32 + acc_row(e, half) < lim ? x : 0.0f);
                }
                ln.accumulate(g, kt[kb], ds);
            }
        one_tile_barrier<2>();   // the tiles have been read: they carry the results
        if (r0 < Lq) ln.store(qt[tile], g, scale, dq + base, row_stride, Lq - r0);
    } else {   // a key per lane
        one_tile_barrier<2, true>();
        bf16x8 kf[T::kKSteps], vf[T::kKSteps];
        f32x16 s, dp, gk[T::kDBlocks], gv[T::kDBlocks];
        int qb = CAUSAL && W > 1 ? tile : 0;   // (causal: as many queries as keys, so that every key has one)
        if (r0 < Lk) {
            ln.fragments(kf, kt[tile]);
            ln.fragments(vf, vt[tile]);
            s = ln.product(qt[qb], kf);
            dp = ln.product(gt[qb], vf);
        }
        one_tile_barrier<2>();
        ln.clear(gk);
        ln.clear(gv);
        if (r0 < Lk)
            for (;;) {
                bf16x8 p[2], ds[2];   // P and dS, queries on the rows
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 l4 = *reinterpret_cast<const float4 *>(&row_lse2[qb * 32 + g * 8 + half * 4]);
                    const float4 d4 = *reinterpret_cast<const float4 *>(&row_delta[qb * 32 + g * 8 + half * 4]);
                    const float l[4] = {l4.x, l4.y, l4.z, l4.w}, d[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        const int e = 4 * g + x, r = qb * 32 + acc_row(e, half);
                        const bool sees = r < Lq && !(CAUSAL && r < i);
                        const float y = fast_exp2(fmaf(s[e], c, -l[x]));
                        p[e >> 3][e & 7] = (__bf16)(sees ? y : 0.0f);
                        ds[e >> 3][e & 7] = (__bf16)(sees ? y * (dp[e] - d[x]) : 0.0f);
                    }
                }
                ln.accumulate(gv, gt[qb], p);
                ln.accumulate(gk, qt[qb], ds);
                if (++qb >= W || qb * 32 >= Lq) break;
                s = ln.product(qt[qb], kf);
                dp = ln.product(gt[qb], vf);
            }
        one_tile_barrier<2>();
        if (r0 < Lk) {
            ln.store(vt[tile], gv, 1.0f, dv + base, row_stride, Lk - r0);
            ln.store(kt[tile], gk, scale, dk + base, row_stride, Lk - r0);
        }
    }
}

// One launch holds at most 2^22 workgroups (a grid's threads are counted in 32 bits).
#define JFA_ONE_TILE(KERNEL, DD, W, CAUSAL, ...) \
    hipLaunchKernelGGL((KERNEL<DD, W, CAUSAL>), dim3((unsigned)grid), dim3(threads * W), 0, stream, __VA_ARGS__)
#define JFA_ONE_TILE_CASE(KERNEL, DD, ...)                                                                       \
    case DD:                                                                                                     \
        if (rows == 32 && causal) JFA_ONE_TILE(KERNEL, DD, 1, true, __VA_ARGS__);                                \
        else if (rows == 32) JFA_ONE_TILE(KERNEL, DD, 1, false, __VA_ARGS__);                                    \
        else if (rows == 64 && causal) JFA_ONE_TILE(KERNEL, DD, 2, true, __VA_ARGS__);                           \
        else if (rows == 64) JFA_ONE_TILE(KERNEL, DD, 2, false, __VA_ARGS__);                                    \
        else if (causal) JFA_ONE_TILE(KERNEL, DD, 4, true, __VA_ARGS__);                                         \
        else JFA_ONE_TILE(KERNEL, DD, 4, false, __VA_ARGS__);                                                    \
        break;
#define JFA_ONE_TILE_CASES(KERNEL, ...)                                                                          \
    if ((rows != 32 && rows != 64 && rows != 128) || (causal && offsets_kv)) return hipErrorInvalidValue;                       \
    const int64_t items = one_tile_items(B, H), most = (int64_t)1 << 22;                                         \
    for (int64_t first = 0; first < items; first += most) {                                                      \
        const int64_t grid = items - first < most ? items - first : most;                                        \
        switch (D) {                                                                                             \
            JFA_ONE_TILE_CASE(KERNEL, 32, __VA_ARGS__) JFA_ONE_TILE_CASE(KERNEL, 64, __VA_ARGS__)                \
            JFA_ONE_TILE_CASE(KERNEL, 128, __VA_ARGS__)                                                          \
            default: return hipErrorInvalidValue;                                                                \
        }                                                                                                        \
    }                                                                                                            \
    return hipGetLastError();

hipError_t launch_fwd_one_tile(const void *q, const void *k, const void *v, const int64_t *offsets, const int64_t *offsets_kv, bool causal,
                               int64_t B, int H, int D, int least, int rows, void *out, float *lse, hipStream_t stream) {
    constexpr int threads = 64;
    JFA_ONE_TILE_CASES(fwd_one_tile_kernel, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v, offsets, offsets_kv, (int)B, H, first, least,
                       (__bf16 *)out, lse)
}

hipError_t launch_bwd_one_tile(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                               const int64_t *offsets, const int64_t *offsets_kv, bool causal, int64_t B, int H, int D, int least, int rows, void *dq,
                               void *dk, void *dv, hipStream_t stream) {
    constexpr int threads = 128;
    JFA_ONE_TILE_CASES(bwd_one_tile_kernel, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v, (const __bf16 *)out, (const __bf16 *)dout,
                       lse, stats, offsets, offsets_kv, (int)B, H, first, least, (__bf16 *)dq, (__bf16 *)dk, (__bf16 *)dv)
}
#undef JFA_ONE_TILE
#undef JFA_ONE_TILE_CASE
#undef JFA_ONE_TILE_CASES

}  // namespace jfa
