// Jagged flash attention forward, bf16, D = 128, long-sample variant (paper Section 2.1).
//
// Same mathematics and operand layouts as fwd_bf16_kernel (transposed score tile S^T = K Q^T, a lane owns
// one query, V^T through the transposing LDS read, 32 queries per wave, two waves per SIMD).  What differs:
//   * a workgroup is eight waves = 256 queries sharing each K / V stage, so the HBM/L2 -> LDS traffic per
//     flop is half that of the 128-query kernel;
//   * stages travel HBM/L2 -> LDS directly (global_load_lds_dwordx4): no staging registers, no LDS store
//     instructions.  The tiles are unpadded and XOR-swizzled on 16-byte (K) / 64-byte (V) granules so that
//     the 16-byte row reads and the transposing reads are conflict-free on the 64-bank LDS;
//   * three stage buffers each for K and V, copies two stages ahead, and a bare s_barrier with a partial vmcnt wait at the
//     end of a round (a __syncthreads() would wait for every load in flight);
//   * the two products and the exponentials of a wave are of three different 32-key blocks and are issued in turn, one
//     matrix instruction of each product and two exponentials at a time (see stage_body).  A wave's vector instructions
//     run under its own matrix instructions where they do not depend on them (16 matrix instructions with 64 vector ones
//     in between take 552 clocks, without any 524; after one another 924).  Taken phase by phase (scores, exponentials, products),
//     the two waves of a SIMD, which a barrier per stage keeps in step, are in the same phase most of the time: a
//     stage took 2 910 clocks, now 2 750, of 2 048 that its matrix instructions need (a skeleton without the row sum 2 470).  What is
//     left: the row sum's dot products, which do not overlap (5 %), LDS latency behind the barrier, the starts of tiles; and the clock
//     falls as the pipes fill: 512 x 8 bimodal to 4096, by counters, 3.90 -> 3.40 million clocks, matrix pipes 51 -> 58 % busy, but
//     1.94 -> 1.82 GHz, so that of 13 % fewer clocks 7 % are left in time.  Forward, microseconds, before -> now: 16 x 8 heads of
//     8192 rows 3640 -> 3505, causal 2140 -> 1998; 512 x 8 bimodal to 4096 2130 -> 2010, causal 1305 -> 1203; 1024 x 4 of up to
//     1024 1040 -> 990; 300 x 4 of up to 300 73.7 -> 67.5; 1024 x 4 Zipf to 1024 664 -> 636;
//   * exponentials are taken against a FIXED reference maximum per query (the maximum over the sample's
//     first 32 keys): no running maximum, no rescaling, no branch in the hot loop.  A reference below the
//     true maximum only scales numerator and denominator alike -- probabilities keep their relative
//     precision in fp32 and bf16 -- as long as nothing overflows; a row sum above 2^62 (or not finite) at the
//     end of the tile shows that it got too stale, and the workgroup then redoes the tile in the conservative
//     order (maximum first, online rescaling).  On data whose scores are of one scale this never runs.
#include "jfa_common.h"
#include "jfa_lds.h"
#include "jfa_mfma.h"

namespace jfa {

constexpr int kDmaThreads = 512;
constexpr int kDmaWaves = kDmaThreads / 64;
constexpr int kDmaBN = 64;            // keys per LDS stage
constexpr int kDmaD = 128;
constexpr int kDmaTile = kDmaBN * kDmaD * 2;   // bytes of one K or V stage in LDS
constexpr int kDmaOpsPerStage = 2 * (kDmaBN / 4) / kDmaWaves;   // DMA instructions per wave per stage (K and V)

template <int N> using IntC = std::integral_constant<int, N>;

// CROSS: the keys and values of a sample are the rows of a second offsets array (cross attention); otherwise
// offsets_kv is not looked at and the code is that of self attention.  CAUSAL (self attention only): query i attends
// to keys 0 .. i.  A tile then streams the keys up to its last query; a wave's 32 queries lie inside one 64-key stage, the
// last that it takes part in and the only one it masks, with the per-lane limit min(L, i + 1) in place of L.
// DIRECT: no schedule, the item is the workgroup's index.
template <bool CROSS, bool CAUSAL, bool DIRECT>
__global__ __launch_bounds__(kDmaThreads, 2) void fwd_bf16_dma_kernel(const __bf16 *__restrict__ q,
                                                                      const __bf16 *__restrict__ k,
                                                                      const __bf16 *__restrict__ v,
                                                                      const int64_t *__restrict__ offsets,
                                                                      const int64_t *__restrict__ offsets_kv, int B,
                                                                      int H, Schedule s, __bf16 *__restrict__ out,
                                                                      float *__restrict__ lse) {
    constexpr int D = kDmaD;
    constexpr int kKSteps = D / 16;    // 8
    constexpr int kDBlocks = D / 32;   // 4
    // stage buffers: K's three, then V's
    __shared__ __attribute__((aligned(1024))) char stages[6 * kDmaTile];
    __shared__ WorkSlot slot;   // the NEXT work item, claimed and decoded while the current one starts up
    __shared__ LdsSchedule<CROSS> tab;   // the schedule, copied once per workgroup when it fits
    __shared__ int restart;   // set by a wave whose reference maximum went stale beyond repair

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const float c = 1.4426950408889634f / sqrtf((float)D);
    const int64_t total = DIRECT ? 0 : (int64_t)s.tile_start[B] * H;
    const int64_t sum_B = offsets[B];
    const int64_t row_stride = (int64_t)H * D;
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};

    // ---- LDS read addresses (bytes inside a tile), fixed for the whole kernel ----
    // K element (row r, 16-byte chunk ch) sits at r * 256 + ((ch ^ (r & 15)) << 4).
    // Only k-step 0's address is kept; step ks is at kaddr0 ^ (ks << 5) (the XOR swizzle makes the eight differ by
    // a constant bit pattern).  Each stage rebuilds them: twelve loop-invariant addresses held in registers
    // across the stage would be the first values the register allocator spills.
    const int kaddr0 = col * 256 + ((half ^ (col & 15)) << 4);
    // V element (row r, 64-byte group g, byte b inside it) sits at r * 256 + ((g ^ (r & 3)) << 6) + b.
    // The transposing read of this lane: row = 4 half + (lane & 15) / 4 (+8 for the second half of the
    // operand, +16 per 16-key step), group = feature block db, bytes 32 * ((lane >> 4) & 1) + 8 * (lane & 3).
    // Feature block db is at vaddr0 ^ (db << 6).  Counted from K's buffer of the same number, so that the way from one
    // register to any of the three buffers fits an instruction's offset.
    int vaddr0;
    {
        const int r = half * 4 + ((lane & 15) >> 2);
        vaddr0 = 3 * kDmaTile + r * 256 + ((r & 3) << 6) + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
    }
    auto lds_addresses = [&](int (&kaddr)[kKSteps], int (&vaddr)[kDBlocks]) {
        int kb = kaddr0, vb = vaddr0;
        asm volatile("" : "+v"(kb), "+v"(vb));   // keeps the rebuilt addresses from being hoisted out of the loop
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks) kaddr[ks] = kb ^ (ks << 5);
#pragma unroll
        for (int db = 0; db < kDBlocks; ++db) vaddr[db] = vb ^ (db << 6);
    };
    // ---- DMA: one instruction moves 64 lanes x 16 bytes = 4 rows; wave w, instruction u fills rows 8 w + 4 u .. +3.
    // Lane l lands on physical chunk l & 15 of row 8 w + 4 u + (l >> 4) and so fetches the logical chunk that
    // the swizzle puts there.
    // byte offsets of this lane's DMA chunks inside a full stage (K and V differ in the swizzle).  Cross attention has no
    // registers for them and rebuilds them in every stage (kept, the kernel reloads spilled registers in its rounds: 1.7 times the time).
    uint32_t koffs[2], voffs[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int r = 8 * wave + (lane >> 4) + 4 * u, pc = lane & 15;
        koffs[u] = 2u * (uint32_t)(r * (int)row_stride + ((pc ^ (r & 15)) << 3));
        voffs[u] = 2u * (uint32_t)(r * (int)row_stride + ((pc ^ ((r & 3) << 2)) << 3));
    }
    // The keys a tile streams: first rows of K and V, number of keys of the sample, number of 64-key stages.
    struct Stream {
        const __bf16 *kbase, *vbase;
        int L, n_stages;
    };
    auto stream_of = [&](const Work &w) {
        Stream st;
        st.L = CROSS ? w.olen : w.len;
        const int64_t krow0 = CROSS ? w.orow0 : w.row0;
        const int w_tile0 = w.block * kDmaBlockRows;
        const int Lc = CAUSAL && w_tile0 + kDmaBlockRows < st.L ? w_tile0 + kDmaBlockRows : st.L;   // keys the tile needs
        st.n_stages = (Lc + kDmaBN - 1) / kDmaBN;
        st.kbase = k + krow0 * row_stride + (int64_t)w.head * D;
        st.vbase = v + krow0 * row_stride + (int64_t)w.head * D;
        return st;
    };
    bf16x8 qreg[kKSteps];
    auto load_q = [&](const Work &w) {   // the lane's query row (rows past the end of the sample repeat its last row)
        const int iw = w.block * kDmaBlockRows + wave * 32 + col;
        const __bf16 *qrow = q + (w.row0 + (iw < w.len ? iw : w.len - 1)) * row_stride + (int64_t)w.head * D + 8 * half;
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks) qreg[ks] = *reinterpret_cast<const bf16x8 *>(qrow + 16 * ks);
    };
    // The claim of the next item runs while a tile's first loads travel, and the tile cannot start before it is done:
    // with the schedule in LDS it is one atomic and a few LDS reads instead of five dependent trips to memory.
    const bool tabled = B <= kTabCap && !DIRECT;
    WorkCursor cursor;
    auto claim_next = [&](const Work &now) {   // wave 0, every lane; now: the present item
        if constexpr (DIRECT) {   // the next block of a sample that is longer than the bound admits
            Work next = now;
            next.block += s.direct_blocks;
            if (lane == 0) park_work<CROSS>(&slot, next, next.block * kDmaBlockRows < next.len);
            return;
        }
        if (!tabled) {
            claim_and_decode(&slot, s, offsets, B, H, total, cursor, CROSS ? offsets_kv : nullptr);
            return;
        }
        int64_t w = -1;
        if (lane == 0) w = next_work(s.counter, cursor, total);
        tab.decode(&slot, B, H, uniform64(w));
    };
    if constexpr (DIRECT) {
        if (tid == 0) direct_first(&slot, s, offsets, CROSS ? offsets_kv : nullptr, H, kDmaBlockRows);
    } else if (wave == 0) claim_and_decode(&slot, s, offsets, B, H, total, cursor, CROSS ? offsets_kv : nullptr);
    if (tabled) tab.fill(s, offsets, offsets_kv, B);
    __syncthreads();   // the slot and the tables are written
    Work t;
    bool have = load_work<CROSS>(&slot, t);
    while (have) {
        __syncthreads();   // every wave has read the slot before wave 0 refills it
        const Stream cur = stream_of(t);
        const int Lq = t.len;                      // queries of the sample
        const int L = cur.L;                       // keys of the sample
        const int q_tile0 = t.block * kDmaBlockRows;   // first query of the tile
        const int n_stages = cur.n_stages;
        const __bf16 *const kbase = cur.kbase;
        const __bf16 *const vbase = cur.vbase;
        if (CROSS && L == 0) {   // no keys: an empty softmax, out = 0 and lse = -inf
            if (wave == 0) claim_next(t);
            const int i = t.block * kDmaBlockRows + wave * 32 + (lane & 31);
            if (i < Lq) {
                __bf16 *orow = out + (t.row0 + i) * row_stride + (int64_t)t.head * D + (lane >> 5) * (D / 2);
#pragma unroll
                for (int e = 0; e < D / 2; e += 8) *reinterpret_cast<u32x4 *>(orow + e) = u32x4{0, 0, 0, 0};
                if (lane < 32) lse[(int64_t)t.head * sum_B + t.row0 + i] = -INFINITY;
            }
            __syncthreads();   // the slot is written
            have = load_work<CROSS>(&slot, t);
            continue;
        }

        auto issue_from = [&](const Stream &st, const __bf16 *base, char *tile, int stage, bool is_k) {
            const int L = st.L;
            const int j0 = stage * kDmaBN;
            const __bf16 *sbase = base + (int64_t)j0 * row_stride;
            if (!CROSS && j0 + kDmaBN <= L) {
#pragma unroll
                for (int u = 0; u < 2; ++u) bd_dma16(sbase, is_k ? koffs[u] : voffs[u], tile + (8 * wave + 4 * u) * 256);
            } else {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    int t_opaque = tid;
                    asm volatile("" : "+v"(t_opaque));
                    const int pc = t_opaque & 15;
                    const int r = 8 * wave + ((t_opaque >> 4) & 3) + 4 * u;
                    const int ch = is_k ? (pc ^ (r & 15)) : (pc ^ ((r & 3) << 2));
                    const int jr = j0 + r < L ? r : L - 1 - j0;   // rows past the end repeat the last key (masked later)
                    bd_dma16(sbase, 2u * (uint32_t)(jr * (int)row_stride + ch * 8), tile + (8 * wave + 4 * u) * 256);
                }
            }
        };
        auto issue = [&](const __bf16 *base, char *tile, int stage, bool is_k) { issue_from(cur, base, tile, stage, is_k); };

        const int i = t.block * kDmaBlockRows + wave * 32 + col;   // this lane's query
        const int iq = i < Lq ? i : Lq - 1;
        const bool wave_active = t.block * kDmaBlockRows + wave * 32 < Lq;

        f32x16 o[kDBlocks];
#pragma unroll
        for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
            for (int e = 0; e < 16; ++e) o[db][e] = 0.0f;
        float m = -INFINITY, mc = 0.0f, lsum = 0.0f;   // reference maximum as a dot product and as an exponent of two
        f32x16 zero;
#pragma unroll
        for (int e = 0; e < 16; ++e) zero[e] = 0.0f;

        // ---- helpers ----
        auto scores = [&](const char *tile, int mb, f32x16 &a) {
            int kaddr[kKSteps], vaddr[kDBlocks];
            lds_addresses(kaddr, vaddr);
#pragma unroll
            for (int e = 0; e < 16; ++e) a[e] = 0.0f;
            bf16x8 kop[kKSteps];
#pragma unroll
            for (int ks = 0; ks < kKSteps; ++ks) kop[ks] = lds_read_b128(tile + mb * 32 * 256 + kaddr[ks]);
#pragma unroll
            for (int ks = 0; ks < kKSteps; ++ks) a = mfma_32x32x16(kop[ks], qreg[ks], a);
        };
        auto accumulate = [&](const char *tile, int mb, const bf16x8 (&p)[2], const int (&vaddr)[kDBlocks]) {
            bf16x8 vop[2][kDBlocks];
#pragma unroll
            for (int ts = 0; ts < 2; ++ts)
#pragma unroll
                for (int db = 0; db < kDBlocks; ++db) {
                    const char *pvp = tile + (mb * 32 + ts * 16) * 256 + vaddr[db];
                    vop[ts][db] = concat(lds_read_tr16(pvp), lds_read_tr16(pvp + 8 * 256));
                }
#pragma unroll
            for (int ts = 0; ts < 2; ++ts)
#pragma unroll
                for (int db = 0; db < kDBlocks; ++db) o[db] = mfma_32x32x16(vop[ts][db], p[ts], o[db]);
        };
        // exponentials of one unit (32 keys x 32 queries) against the reference maximum; the rounded
        // probabilities are what the second product uses, so they are what the row sum adds up
        // st holds raw dot products; the softmax scale and the change to base-2 exponentials are one fp32 multiply-add per score
        auto exps = [&](const f32x16 &st, float subc, bf16x8 (&p)[2]) {
#pragma unroll
            for (int ts = 0; ts < 2; ++ts) {
                u32x4 pw;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    bf16x2 pr;
                    const float x0 = st[8 * ts + 2 * e], x1 = st[8 * ts + 2 * e + 1];
                    pr[0] = (__bf16)fast_exp2(fmaf(x0, c, -subc));
                    pr[1] = (__bf16)fast_exp2(fmaf(x1, c, -subc));
                    lsum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, lsum, false);
                    pw[e] = __builtin_bit_cast(uint32_t, pr);
                }
                p[ts] = __builtin_bit_cast(bf16x8, pw);
            }
        };
        // keys of a block from the lane's first on that the lane's query sees; accumulator register e holds key key0 + (e / 4) * 8 + 4 * half + e % 4
        auto keys_left = [&](int key0) {
            int h = half;
            asm volatile("" : "+v"(h));   // keeps the sixteen thresholds from being computed at tile start and spilled
            return (CAUSAL && iq + 1 < L ? iq + 1 : L) - key0 - 4 * h;
        };
        auto mask = [&](f32x16 &st, int key0) {   // keys past the end of the sample (causal: and above the diagonal)
            const int lim = keys_left(key0);
#pragma unroll
            for (int e = 0; e < 16; ++e)
                st[e] = (e >> 2) * 8 + (e & 3) >= lim ? -INFINITY : st[e];
        };
        auto unit_max = [&](const f32x16 &a, float mx) {
#pragma unroll
            for (int e = 0; e < 16; ++e) mx = fmaxf(mx, a[e]);
            return mx;
        };
        auto kbuf = [&](int b) { return stages + b * kDmaTile; };
        auto vbuf = [&](int b) { return stages + (3 + b) * kDmaTile; };

        // ---- the fast order, against the fixed reference maximum m ----
        // Sixteen groups over the two 32-key blocks b of a stage.  A group holds one product of each kind and a pair of
        // exponentials, none of which needs another's result: O^T += V^T P^T of stage j's block b, the scores of stage
        // j + 1's block b, and the exponentials of the block between them (stage j's block 1 beside b = 0, stage j + 1's
        // block 0 beside b = 1).  The groups are kept in this order, operand reads kAhead groups before their use.  The reference is
        // subtracted in the multiply-add of the exponent: as the score products' addend it would take sixteen registers.
        constexpr int kAhead = 2;
        f32x16 sc[2];      // scores of block 0 / 1, until their exponentials are taken
        u32x4 pw[2][2];    // rounded probabilities of block 0 / 1
        auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
        auto exp_pair = [&](const f32x16 &st, int g, u32x4 (&w)[2], auto MASKED, int lim) {   // keys 2 g and 2 g + 1 of this lane's sixteen
            bf16x2 pr;
            pr[0] = (__bf16)fast_exp2(fmaf(st[2 * g], c, -mc));
            pr[1] = (__bf16)fast_exp2(fmaf(st[2 * g + 1], c, -mc));
            uint32_t both = __builtin_bit_cast(uint32_t, pr);
            if constexpr (decltype(MASKED)::value != 0) {   // keys from lim on, counted from the lane's first, weigh nothing
                const int key = (g >> 1) * 8 + (g & 1) * 2;
                both &= key + 1 < lim ? 0xffffffffu : key < lim ? 0xffffu : 0u;
            }
            lsum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, both), ones, lsum, false);
            asm volatile("" : "+v"(both), "+v"(lsum));   // computed here, not where they are used a round later
            w[g >> 2][g & 3] = both;
        };
        auto value_operand = [&](const char *Vc, const int (&vaddr)[kDBlocks], int g) {   // group g of a stage
            const char *pvp = Vc + ((g >> 3) * 32 + ((g >> 2) & 1) * 16) * 256 + vaddr[g & 3];
            return concat(lds_read_tr16(pvp), lds_read_tr16(pvp + 8 * 256));
        };
        auto stage_body = [&](const char *Kn, const char *Vc, auto MASKED, int key_next) {   // MASKED: stage j + 1's scores
            int kaddr[kKSteps], vaddr[kDBlocks];
            lds_addresses(kaddr, vaddr);
            bf16x8 kop[2 * kKSteps], vop[2 * kKSteps];
            int lim = 0;
            if constexpr (decltype(MASKED)::value != 0) lim = keys_left(key_next);
            auto read = [&](int g) {
                kop[g] = lds_read_b128(Kn + (g >> 3) * 32 * 256 + kaddr[g & 7]);
                vop[g] = value_operand(Vc, vaddr, g);
            };
#pragma unroll
            for (int g = 0; g < kAhead; ++g) read(g);
            fence();
#pragma unroll
            for (int g = 0; g < 2 * kKSteps; ++g) {
                const int b = g >> 3, gi = g & 7;
                if (g + kAhead < 2 * kKSteps) read(g + kAhead);
                o[gi & 3] = mfma_32x32x16(vop[g], __builtin_bit_cast(bf16x8, pw[b][gi >> 2]), o[gi & 3]);
                fence();
                sc[b] = mfma_32x32x16(kop[g], qreg[gi], gi == 0 ? zero : sc[b]);
                fence();
                if (b == 0) exp_pair(sc[1], gi, pw[1], IntC<0>{}, 0);
                else exp_pair(sc[0], gi, pw[0], MASKED, lim);
                fence();
            }
        };
        // The wave's last stage: scores and block 0's probabilities are there.  two_blocks: block 1 has keys for it.
        auto last_stage = [&](const char *Vc, bool two_blocks, int key0) {
            int kaddr[kKSteps], vaddr[kDBlocks];
            lds_addresses(kaddr, vaddr);
            bf16x8 vop[2 * kKSteps];
            auto product = [&](int g) {
                o[g & 3] = mfma_32x32x16(vop[g], __builtin_bit_cast(bf16x8, pw[g >> 3][(g >> 2) & 1]), o[g & 3]);
            };
            constexpr int kEarly = CROSS ? 2 : 4;
#pragma unroll
            for (int g = 0; g < kEarly; ++g) vop[g] = value_operand(Vc, vaddr, g);
            if (two_blocks) {
                const int lim = keys_left(key0 + 32);
                fence();
#pragma unroll
                for (int g = 0; g < 2 * kKSteps; ++g) {
                    if (g + kEarly < 2 * kKSteps) vop[g + kEarly] = value_operand(Vc, vaddr, g + kEarly);
                    product(g);
                    if (g < kKSteps) exp_pair(sc[1], g, pw[1], IntC<1>{}, lim);
                    fence();
                }
            } else {
#pragma unroll
                for (int g = 0; g < kKSteps; ++g) {
                    if (g + kEarly < kKSteps) vop[g + kEarly] = value_operand(Vc, vaddr, g + kEarly);
                    product(g);
                    fence();
                }
            }
        };
        // conservative(): maximum first, rescale, then exponentials; used when a tile had to be restarted
        auto conservative = [&](int bsel, int j) {
            const char *const Kc = kbuf(bsel);
            const char *const Vc = kbuf(bsel);   // see vaddr0
            int kaddr[kKSteps], vaddr[kDBlocks];
            lds_addresses(kaddr, vaddr);
            f32x16 s0, s1;
            bf16x8 p0[2], p1[2];
            scores(Kc, 0, s0);
            scores(Kc, 1, s1);
            if (CAUSAL || (j + 1) * kDmaBN > L) { mask(s0, j * kDmaBN); mask(s1, j * kDmaBN + 32); }
            const float x = pair_max(unit_max(s1, unit_max(s0, -INFINITY)));
            const float n = fmaxf(m, x);
            const float a = fast_exp2((m - n) * c);   // 0 on the first stage
            m = n;
            lsum *= a;
#pragma unroll
            for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[db][e] *= a;
            exps(s0, n * c, p0);
            accumulate(Vc, 0, p0, vaddr);
            exps(s1, n * c, p1);
            accumulate(Vc, 1, p1, vaddr);
        };

        // ---- pass 1: three stage buffers for K and three for V, copies two stages ahead ----
        // Stage j of either lives in buffer j % 3.  Round j multiplies stage j of V and stage j + 1 of K, so the buffers free at
        // its top are K's j % 3 and V's (j + 2) % 3: the copies of K's stage j + 3 and V's stage j + 2 are sent there.  At its
        // end each wave waits until only those are outstanding (so what round j + 1 reads has landed) and meets the others
        // at a bare s_barrier.
        auto round_end = [&](bool k_ahead, bool v_ahead) {
            asm volatile("" ::: "memory");
            if (k_ahead) __builtin_amdgcn_s_waitcnt(0x0070 | kDmaOpsPerStage);            // vmcnt(K and V of one stage) lgkmcnt(0)
            else if (v_ahead) __builtin_amdgcn_s_waitcnt(0x0070 | kDmaOpsPerStage / 2);
            else __builtin_amdgcn_s_waitcnt(0x0070);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        // The stages this wave needs (causal: its 32 queries lie inside one 64-key stage, which is its last) and whether the
        // last one's second block has keys for it.
        const int n_mine = CAUSAL && (q_tile0 + wave * 32) / kDmaBN + 1 < n_stages ? (q_tile0 + wave * 32) / kDmaBN + 1 : n_stages;
        const bool two_blocks = (n_mine - 1) * kDmaBN + 32 < (CAUSAL && q_tile0 + wave * 32 + 32 < L ? q_tile0 + wave * 32 + 32 : L);
        auto issue_round = [&](int b, int j) {   // b = j % 3
            if (j + 3 < n_stages) issue(kbase, kbuf(b), j + 3, true);
            if (j + 2 < n_stages) issue(vbase, vbuf(b == 0 ? 2 : b - 1), j + 2, false);
        };
        auto round = [&](int b, auto MASKED, int j) {   // any but the wave's last
            issue_round(b, j);
            stage_body(kbuf(b == 2 ? 0 : b + 1), kbuf(b), MASKED, (j + 1) * kDmaBN);
            round_end(j + 3 < n_stages, j + 2 < n_stages);
        };

        load_q(t);
        issue(kbase, kbuf(0), 0, true);
        issue(vbase, vbuf(0), 0, false);
        if (n_stages > 1) {
            issue(kbase, kbuf(1), 1, true);
            issue(vbase, vbuf(1), 1, false);
        }
        if (wave == 0) claim_next(t);   // overlaps with the loads in flight
#pragma unroll
        for (int ks = 0; ks < kKSteps; ++ks) asm volatile("" : "+v"(qreg[ks]));   // Q loads complete here
        if (tid == 0) restart = 0;   // nobody looks at it between the barrier at the top of the loop and the next one
        // K's stage 0 has landed once at most what this wave sent after it is outstanding (on wave 0 also
        // the loads of the claim, which it has waited for itself).
        if (n_stages > 1) __builtin_amdgcn_s_waitcnt(0x0070 | (2 * kDmaOpsPerStage - kDmaOpsPerStage / 2));
        else __builtin_amdgcn_s_waitcnt(0x0070);   // and V's, the only other copies: no second wait
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (n_stages > 2) issue(kbase, kbuf(2), 2, true);
        if (wave_active) {   // reference maximum: the first 32 keys; their exponentials beside the scores of the next 32
            int kaddr[kKSteps], vaddr[kDBlocks];
            lds_addresses(kaddr, vaddr);
            constexpr int kEarly = CROSS ? 4 : kKSteps;
            bf16x8 kop[kKSteps];
            scores(kbuf(0), 0, sc[0]);
#pragma unroll
            for (int g = 0; g < kEarly; ++g) kop[g] = lds_read_b128(kbuf(0) + 32 * 256 + kaddr[g]);
            fence();
            if (n_mine == 1) mask(sc[0], 0);
            m = pair_max(unit_max(sc[0], -INFINITY));
            mc = m * c;
#pragma unroll
            for (int g = 0; g < kKSteps; ++g) {
                if (g + kEarly < kKSteps) kop[g + kEarly] = lds_read_b128(kbuf(0) + 32 * 256 + kaddr[g + kEarly]);
                sc[1] = mfma_32x32x16(kop[g], qreg[g], g == 0 ? zero : sc[1]);
                exp_pair(sc[0], g, pw[0], IntC<0>{}, 0);
                fence();
            }
        }
        // round 0 needs V's stage 0 and K's stage 1; K's stage 2 and V's stage 1 may be on their way
        if (n_stages > 1) round_end(n_stages > 2, true);
        int j = 0;
        if (wave_active) {
            for (; j + 5 <= n_mine; j += 3) {
                round(0, IntC<0>{}, j);
                round(1, IntC<0>{}, j + 1);
                round(2, IntC<0>{}, j + 2);
            }
            // One to four rounds are left, which take one copy of the code: the last but one is followed by masked scores (the others'
            // masks let everything pass), the last has its own form.
            int b = 0;
#pragma unroll 1
            for (; j + 1 < n_mine; ++j) {
                round(b, IntC<1>{}, j);
                b = b == 2 ? 0 : b + 1;
            }
            issue_round(b, j);
            last_stage(kbuf(b), two_blocks, j * kDmaBN);
            if (j + 1 < n_stages) round_end(j + 3 < n_stages, j + 2 < n_stages);
            ++j;
        }
        for (; j + 1 < n_stages; ++j) {   // rounds in which this wave only copies (the last one has nothing to copy)
            issue_round(j % 3, j);
            round_end(j + 3 < n_stages, j + 2 < n_stages);
        }
        // a row sum this large (or not finite) means the fixed reference was too far below the true maximum
        if (wave_active && __builtin_amdgcn_ballot_w64(!(lsum < 0x1p62f)) != 0 && lane == 0) restart = 1;
        __syncthreads();   // `restart` is written
        const bool again = restart != 0;

        // ---- pass 2 (never on data of one scale): the whole tile again, maximum first, two buffers ----
        if (again) {
            issue(kbase, kbuf(0), 0, true);
            issue(vbase, vbuf(0), 0, false);
            __builtin_amdgcn_s_waitcnt(0x0070);
            __syncthreads();
            m = -INFINITY;
            lsum = 0.0f;
#pragma unroll
            for (int db = 0; db < kDBlocks; ++db)
#pragma unroll
                for (int e = 0; e < 16; ++e) o[db][e] = 0.0f;
            for (int j = 0; j < n_stages; ++j) {
                if (j + 1 < n_stages) {
                    issue(kbase, kbuf((j + 1) & 1), j + 1, true);
                    issue(vbase, vbuf((j + 1) & 1), j + 1, false);
                }
                if (wave_active) conservative(j & 1, j);
                __builtin_amdgcn_s_waitcnt(0x0070);
                __syncthreads();
            }
        }

        Work nt;   // the next work item: wave 0 parked it in the slot before this tile's first barrier
        const bool have_next = load_work<CROSS>(&slot, nt);

        // ---- epilogue: normalise; transpose the wave's 32 x 128 output block through LDS, 64 features at a time, so
        // that it leaves as whole 128-byte pieces of rows (16 bytes per lane, eight rows per store instruction) instead
        // of 8-byte pieces of 32 different rows per instruction; store the log-sum-exp ----
        // The stage buffers are idle here (every wave is past the last stage's barrier and no DMA is in flight, and the
        // next tile's loads start behind the barrier at the top of the loop); wave w uses 4 KB of the third one: row r of its block at r * 128,
        // 16-byte chunk ch at (ch ^ (r & 7)) << 4.
        const float l_total = pair_sum(lsum);
        {
            char *const region = (wave < 4 ? kbuf(2) : vbuf(2)) + (wave & 3) * 4096;
            const float inv = 1.0f / l_total;
            int lane_e = lane;   // every address below derives from this copy, which the compiler cannot see
            asm volatile("" : "+v"(lane_e));   // through: otherwise they are computed at tile start and spilled
            const int col_e = lane_e & 31, half_e = lane_e >> 5;
            const int wbase = col_e * 128 + ((half_e * 8) ^ ((col_e & 7) << 4));
            const int q0 = t.block * kDmaBlockRows + wave * 32;   // first query of this wave
            __bf16 *const obase = out + (t.row0 + q0) * row_stride + (int64_t)t.head * D;
            const uint32_t lane_off = 2u * (uint32_t)((lane_e >> 3) * (int)row_stride + (lane_e & 7) * 8);
#pragma unroll
            for (int f = 0; f < 2; ++f) {   // features 64 f .. 64 f + 63
#pragma unroll
                for (int dl = 0; dl < 2; ++dl)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        bf16x4 x;
#pragma unroll
                        for (int e = 0; e < 4; ++e) x[e] = (__bf16)(o[2 * f + dl][4 * g + e] * inv);
                        *reinterpret_cast<bf16x4 *>(region + (wbase ^ (dl * 64 + g * 16))) = x;
                    }
#pragma unroll
                for (int it = 0; it < 4; ++it) {
                    const int r = it * 8 + (lane_e >> 3);
                    const u32x4 rowpiece = *reinterpret_cast<const u32x4 *>(region + r * 128 + (((lane_e & 7) ^ (r & 7)) << 4));
                    char *dst = reinterpret_cast<char *>(obase + (int64_t)it * 8 * row_stride + 64 * f) + lane_off;   // scalar base + 32-bit lane offset
                    if (q0 + r < Lq) *reinterpret_cast<u32x4 *>(dst) = rowpiece;
                }
            }
        }
        if (i < Lq && half == 0)
            lse[(int64_t)t.head * sum_B + t.row0 + i] = (m * c + fast_log2(l_total)) * 0.6931471805599453f;
        t = nt;
        have = have_next;
    }
}

hipError_t launch_fwd_bf16_dma(const void *q, const void *k, const void *v, const int64_t *offsets,
                               const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, void *out, float *lse,
                               int cus, hipStream_t stream) {
    if (D != kDmaD || (causal && offsets_kv)) return hipErrorInvalidValue;
#define JFA_LAUNCH(CROSS, CAUSAL, DIRECT)                                                                                  \
    hipLaunchKernelGGL((fwd_bf16_dma_kernel<CROSS, CAUSAL, DIRECT>), dim3(item_grid<fwd_bf16_dma_kernel<CROSS, CAUSAL, DIRECT>>(kDmaThreads, B, H, s, cus)), \
                       dim3(kDmaThreads), 0, stream, (const __bf16 *)q, (const __bf16 *)k, (const __bf16 *)v, offsets,     \
                       offsets_kv, B, H, s, (__bf16 *)out, lse)
#define JFA_FORM(CROSS, CAUSAL)                                                                                            \
    do {                                                                                                                   \
        if (s.direct_blocks) JFA_LAUNCH(CROSS, CAUSAL, true);                                                              \
        else JFA_LAUNCH(CROSS, CAUSAL, false);                                                                             \
    } while (0)
    if (offsets_kv) JFA_FORM(true, false);
    else if (causal) JFA_FORM(false, true);
    else JFA_FORM(false, false);
#undef JFA_FORM
#undef JFA_LAUNCH
    return hipGetLastError();
}

}  // namespace jfa
