// Internal declarations shared by the HIP translation units of libjfa.so (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace jfa {

// The work counters at the head of the private work table: two schedules with kXcds queues each, a counter per queue.  A claim is
// an atomic of the whole device, and those that meet on one 128-byte line are served one after the other: with all counters on
// one line a workgroup of a batch of short tiles waits some 10 us for each claim.  So every queue has a line of its own (the two
// schedules', which are never in use at the same time, share it).
// Microseconds, one line -> lines of their own, B x H, lengths: forward 512 x 8 with up to 256 targets against up to 1024 keys,
// D = 32, 163 -> 122; 1024 x 4 up to 200, D = 32, forward 119 -> 63, backward 241 -> 134, D = 64 115 -> 76 and 248 -> 206;
// 4096 x 1 up to 32, D = 64, 89 -> 58 and 162 -> 102; 1024 x 4 Zipf to 1024, D = 128, forward 708 -> 700.
constexpr int kCounterStride = 32;   // int32 words from one queue's counter to the next
// Histogram bins of the scheduler's counting sort (samples with >= kSchedBins-1 row blocks share the top bin).
constexpr int kSchedBins = 1024;

// Device view of one work schedule (see jfa_build_schedule in jfa.h for the meaning of the arrays).
struct Schedule {
    const int32_t *order;       // [B]
    const int32_t *tile_start;  // [B+1]
    int32_t *counter;           // kXcds zeroed work counters (one queue per XCD), kCounterStride words apart, bumped by the persistent workgroups
    // Small problems (see build_small_work) run without a scheduler launch: the counters are then not valid
    // and work is dealt statically (static_only); build_rows > 0 tells the kernel to build the schedule itself, in LDS, for
    // row blocks of that many rows (order and tile_start are then not looked at), 0 that the scheduler kernel has filled them.
    int build_rows = 0;
    bool static_only = false;
    int fixed_items = 4;   // up to this many items per workgroup are dealt without claims (kernels that walk with NarrowWalk)
    // Blocks of every (sample, head), each a workgroup of its own, with no schedule at all (0: there is one); see direct_blocks()
    int direct_blocks = 0;
};

// The chip has 8 accelerator dies (XCDs), each with its own L2, and workgroups are dealt to them round-robin
// by workgroup id.  Work ids are cut into groups of kWorkGroup consecutive ids -- consecutive ids are row
// blocks of the same (sample, head), which stream the same K/V -- and group g belongs to the queue of XCD
// g % 8, so the blocks that share K/V run on the die whose L2 already holds it.  A workgroup drains its own
// die's queue first and then helps the others, so the assumption about placement only affects locality.
constexpr int kXcds = 8;
constexpr int kWorkGroup = 32;
constexpr int kNumCounters = kXcds * kCounterStride;   // schedule i's counter of queue y: word y * kCounterStride + i

// Work id of local index t of queue y.
__device__ inline int64_t work_id(int y, int t) {
    return ((int64_t)(t / kWorkGroup) * kXcds + y) * kWorkGroup + t % kWorkGroup;
}

// Per-workgroup claim state (kept by the one thread that claims).
struct WorkCursor {
    bool first = true;
    bool home_done = false;
    bool static_only = false;   // the counters are not valid (schedule built in the kernel): deal statically whatever the size
    int fixed_items = 4;   // problems of at most this many items per workgroup are dealt statically
    int64_t next = -1;   // small problems: next statically assigned id
    int step = 0;        // ... and the distance to the one after it
    int grid = 0;        // gridDim.x, read once: the dispatch packet it comes from is a slow place to read
};

__device__ inline int cursor_grid(WorkCursor &cur) {
    if (cur.grid == 0) {
        int g = (int)gridDim.x;
        asm volatile("" : "+v"(g));   // a value, not a load the compiler may repeat wherever it is needed
        cur.grid = g;
    }
    return cur.grid;
}

// A deal without claims: round n of `total` items goes to the `grid` workgroups forwards (item n * grid + workgroup) or backwards
// (n * grid + grid - 1 - workgroup).  The items are sorted longest first and every other round goes backwards (whoever had the longest item
// of one gets the shortest of the next), so that the deal is even to less than an item.  The last round, which is hardly ever full, goes
// forwards: the workgroups at the front are dispatched first, and their waves come before the others' on a SIMD.  Returns whether round
// n goes backwards where (n ^ deal_turn()) & 1.  (The quotient may be one off: then the other order is dealt, by everyone.)
// Microseconds, all rounds forwards / every second one backwards from the second on / as here: D = 64, 4 x 8 heads of up to 4096 rows,
// forward 116 / 130 / 117, 16 x 4 of up to 2048, backward 151 / 148 / 139; 600 x 4 of up to 500, one in ten long, forward 39.5 / 41.9 / 39.6;
// D = 32, 300 x 3, up to 200 queries against at most 8 keys, 15.1 / 17.0 / 14.8; D = 128, 1024 x 4, 200 queries against up to 200 keys,
// backward 751 / 708 / 707; fp32, D = 64, 256 x 2 of up to 100, backward 76 / 81 / 76.  With two rounds, most items short and a few long
// the long ones go to the workgroups at the back: D = 64, 94 x 6 of up to 857, one in ten long, forward 26.5 / 23.5 / 25.3.  (A last round
// forwards from the second workgroup of each compute unit, the others as in the second column: 16 x 4 157, 4 x 8 126, 94 x 6 26.0.)
__device__ inline int deal_turn(int64_t total, int grid) {
    const int rounds = (int)((float)((int)total + grid - 1) * __builtin_amdgcn_rcpf((float)grid));
    return (rounds + 1) & 1;
}

// Next work id for this workgroup, or -1 when nothing is left.  Called by one thread.
//   * The first item is assigned statically (queue blockIdx % 8, local index blockIdx / 8): no memory traffic,
//     and on problems smaller than the grid the surplus workgroups leave at once.
//   * Further items of the home queue are claimed with one atomic add (local indices continue after the
//     static ones, hence the gridDim / 8 base; the grid is a multiple of 8).
//   * Once the home queue is empty the workgroup looks at all eight counters with plain loads and only
//     spends an atomic on a queue that still shows work.
//   * Problems of at most `fixed_items` items per workgroup skip all of this (see below).
__device__ inline int64_t next_work(int32_t *counters, WorkCursor &cur, int64_t total) {
    // Small problems are dealt without any atomics, the claim traffic would dominate the run time.
    const int grid = cursor_grid(cur);
    if (cur.static_only || total <= cur.fixed_items * (int64_t)grid) {
        const int at = deal_turn(total, grid) ? grid - 1 - (int)blockIdx.x : (int)blockIdx.x;
        cur.step = cur.next < 0 ? 2 * at + 1 : 2 * grid - cur.step;
        cur.next = cur.next < 0 ? at : cur.next + cur.step;
        return cur.next < total ? cur.next : -1;
    }
    const int home = blockIdx.x % kXcds;
    const int base = grid / kXcds;
    if (cur.first) {
        cur.first = false;
        const int64_t id = work_id(home, blockIdx.x / kXcds);
        if (id < total) return id;
        cur.home_done = true;  // ids grow with the local index: nothing later in this queue is valid either
    }
    if (!cur.home_done) {
        const int64_t id = work_id(home, base + atomicAdd(&counters[home * kCounterStride], 1));
        if (id < total) return id;
        cur.home_done = true;
    }
    for (;;) {
        int seen[kXcds];  // all eight counters in one round of independent loads
#pragma unroll
        for (int y = 0; y < kXcds; ++y) seen[y] = __atomic_load_n(&counters[y * kCounterStride], __ATOMIC_RELAXED);
        bool any = false;
#pragma unroll
        for (int d = 1; d < kXcds; ++d) {
            const int y = (home + d) % kXcds;
            int c = 0;
#pragma unroll
            for (int z = 0; z < kXcds; ++z) c = z == y ? seen[z] : c;
            if (work_id(y, base + c) >= total) continue;
            any = true;
            const int64_t id = work_id(y, base + atomicAdd(&counters[y * kCounterStride], 1));
            if (id < total) return id;
        }
        if (!any) return -1;  // counters only grow, so this loop ends
    }
}

// The work id is the same for every lane; saying so lets the tile parameters derived from it live in scalar
// registers and be fetched with scalar loads.
__device__ inline int64_t uniform64(int64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Next work id for the whole workgroup (thread 0 claims, `slot` in LDS hands it to the others), or -1.
__device__ inline int64_t fetch_item(int32_t *counters, WorkCursor &cur, int64_t total, int64_t *slot) {
    __syncthreads();
    if (threadIdx.x == 0) *slot = next_work(counters, cur, total);
    __syncthreads();
    return uniform64(*slot);
}

// One decoded work item.
struct Work {
    int sample;   // sample id b
    int head;     // head h
    int block;    // row-block index inside the sample
    int64_t row0; // offsets[b]
    int len;      // L_b
    // Cross attention: the sample's rows on the other side (the rows that stream past the block: keys for a
    // block of queries, queries for a block of keys), from a second offsets array.  Equal to row0 / len otherwise.
    int64_t orow0;
    int olen;
};

// Largest p in [0, B) with tile_start[p] * H <= w, found by one wave: 64 probes per round instead of one.
__device__ inline int find_position_wave(const int32_t *tile_start, int B, int H, int64_t w) {
    const int lane = threadIdx.x & 63;
    int lo = 0, hi = B;  // invariant: tile_start[lo]*H <= w < tile_start[hi]*H
    while (hi - lo > 1) {
        const int step = (hi - lo + 63) / 64;
        const int idx = lo + (lane + 1) * step;
        const bool ok = idx < hi && (int64_t)tile_start[idx] * H <= w;   // true for a prefix of the lanes
        const int cnt = __popcll(__builtin_amdgcn_ballot_w64(ok));
        lo += cnt * step;
        hi = hi < lo + step ? hi : lo + step;
    }
    return lo;
}

// Work item w -> (sample, head, row block).  Called by whole waves (each wave searches for itself, 64 probes per
// round: two or three dependent loads instead of log2(B)).
__device__ inline Work decode_work(const Schedule &s, const int64_t *offsets, int B, int H, int64_t w,
                                   const int64_t *offsets_other = nullptr) {
    Work t;
    const int p = find_position_wave(s.tile_start, B, H, w);   // every lane of the calling wave must be active
    const int t0 = s.tile_start[p];
    const int n = s.tile_start[p + 1] - t0;
    const int r = (int)(w - (int64_t)t0 * H);
    t.sample = s.order[p];
    t.head = r / n;
    t.block = r - t.head * n;
    t.row0 = offsets[t.sample];
    t.len = (int)(offsets[t.sample + 1] - t.row0);
    t.orow0 = t.row0;
    t.olen = t.len;
    if (offsets_other) {
        t.orow0 = offsets_other[t.sample];
        t.olen = (int)(offsets_other[t.sample + 1] - t.orow0);
    }
    return t;
}

// A decoded work item parked in LDS for the whole workgroup.
struct WorkSlot {
    int valid;   // 0: nothing left
    int sample, head, block, len;
    int row0_lo, row0_hi;
    int olen, orow0_lo, orow0_hi;   // the other side's rows (cross attention only)
};

// The schedule of a small problem, built inside the attention kernel instead of by a launch of its own (a launch and
// the scheduler kernel's chain of dependent trips to memory cost more than these problems' whole arithmetic), and
// kept in LDS: every workgroup computes the same schedule -- samples in descending order of their stream's block
// count, equal counts in sample order, the order the scheduler kernel produces (samples in their own order when there
// is at most one item per workgroup) -- and decodes from it the at most
// kSmallItems work items that the static deal gives it (one of every gridDim), so that nothing of the
// schedule is written to or read back from memory: after the one trip for the lengths, an item costs one more for
// its sample's offsets.  Lengths are fetched once, by all threads at once, into LDS; one wave then runs a counting
// sort over at most kInlineBins keys, in which the ranks inside a bin come from ballots, a scan of the block counts
// in sorted order, and the search for the workgroup's items.
// `scratch`: kInlineScratchInts ints of LDS that nothing else uses until the call returns (the kernels lend a stage
// buffer); `mine` is LDS that lasts.  Called by every thread of the workgroup; B <= kInlineCap; ends with a barrier.
constexpr int kInlineCap = 1024;
constexpr int kInlineBins = 64;
constexpr int kSmallItems = 4;
constexpr int kInlineScratchInts = 2 * kInlineBins + kInlineCap + kInlineCap / 4 + kInlineCap / 2 + kInlineCap + 4;   // 11.6 KB
struct SmallWork {
    int count;                     // items of this workgroup
    WorkSlot item[kSmallItems];
};
__device__ inline void build_small_work(const int64_t *offsets, const int64_t *offsets_other, int B, int H, int block_rows,
                                        int *scratch, SmallWork *mine) {
    int *const bins = scratch;                                    // [kInlineBins] counts, then [kInlineBins] next free positions
    int *const nblk = scratch + 2 * kInlineBins;                  // [kInlineCap] row blocks of sample b
    uint8_t *const keys = reinterpret_cast<uint8_t *>(nblk + kInlineCap);               // [kInlineCap] sort key of sample b
    uint16_t *const sorted = reinterpret_cast<uint16_t *>(nblk + kInlineCap + kInlineCap / 4);   // [kInlineCap] sample at position p
    int *const start = nblk + kInlineCap + kInlineCap / 4 + kInlineCap / 2;             // [kInlineCap + 1] first tile of position p
    for (int b = threadIdx.x; b < B; b += blockDim.x) {
        const int64_t len = offsets[b + 1] - offsets[b];
        const int64_t stream = offsets_other ? offsets_other[b + 1] - offsets_other[b] : len;
        const int64_t key = (stream + block_rows - 1) / block_rows;
        nblk[b] = (int)((len + block_rows - 1) / block_rows);
        keys[b] = (uint8_t)(key < kInlineBins - 1 ? key : kInlineBins - 1);
    }
    for (int i = threadIdx.x; i < 2 * kInlineBins; i += blockDim.x) bins[i] = 0;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        // inclusive scan of the block counts, samples taken in the order `at(p)`, into start[1 .. B]; returns the total
        auto scan_blocks = [&](auto at) {
            int carry = 0;
            if (lane == 0) start[0] = 0;
            for (int p0 = 0; p0 < B; p0 += 64) {
                const int p = p0 + lane;
                int incl = p < B ? nblk[at(p)] : 0;
                for (int d = 1; d < 64; d <<= 1) {
                    const int y = __shfl_up(incl, d, 64);
                    if (lane >= d) incl += y;
                }
                incl += carry;
                if (p < B) start[p + 1] = incl;
                carry = __shfl(incl, 63, 64);
            }
            return carry;
        };
        // 0. With at most one item per workgroup the order of the deal is of no consequence: the samples stay in their
        //    own order and the sort (steps 1 to 3, most of this function's time) is skipped.
        int blocks = scan_blocks([](int p) { return p; });
        const bool in_sample_order = (int64_t)blocks * H <= (int64_t)gridDim.x;
        if (!in_sample_order) {
        // 1. samples per key
        for (int b0 = 0; b0 < B; b0 += 64) {
            const bool valid = b0 + lane < B;
            const int key = valid ? keys[b0 + lane] : -1;
            uint64_t todo = __builtin_amdgcn_ballot_w64(valid);
            while (todo) {
                const int leader = __builtin_amdgcn_readfirstlane(__builtin_ctzll(todo));
                const int kk = __builtin_amdgcn_readlane(key, leader);
                const uint64_t same = __builtin_amdgcn_ballot_w64(key == kk);
                if (lane == leader) bins[kk] += __popcll(same);
                todo &= ~same;
            }
        }
        // 2. first position of each key, keys in descending order: lane l owns key kInlineBins - 1 - l
        {
            const int cnt = bins[kInlineBins - 1 - lane];
            int incl = cnt;
            for (int d = 1; d < 64; d <<= 1) {
                const int y = __shfl_up(incl, d, 64);
                if (lane >= d) incl += y;
            }
            bins[kInlineBins + (kInlineBins - 1 - lane)] = incl - cnt;
        }
        // 3. scatter in sample order
        for (int b0 = 0; b0 < B; b0 += 64) {
            const bool valid = b0 + lane < B;
            const int b = valid ? b0 + lane : 0;
            const int key = valid ? keys[b] : -1;
            uint64_t todo = __builtin_amdgcn_ballot_w64(valid);
            while (todo) {
                const int leader = __builtin_amdgcn_readfirstlane(__builtin_ctzll(todo));
                const int kk = __builtin_amdgcn_readlane(key, leader);
                const uint64_t same = __builtin_amdgcn_ballot_w64(key == kk);
                const int base = bins[kInlineBins + kk];
                if (key == kk) sorted[base + __popcll(same & ((1ull << lane) - 1))] = (uint16_t)b;
                if (lane == leader) bins[kInlineBins + kk] = base + __popcll(same);
                todo &= ~same;
            }
        }
        // 4. inclusive scan of the block counts in sorted order
        blocks = scan_blocks([&](int p) { return (int)sorted[p]; });
        }
        // 5. this workgroup's items: the position of each in the sorted order (64 probes per round), then, a lane per
        //    item, the sample's offsets -- the only trip to memory, all items at once
        const int64_t total = (int64_t)blocks * H;
        const int turn = deal_turn(total, (int)gridDim.x);
        int my_p = 0, my_r = 0, n_items = 0;
        for (int n = 0; n < kSmallItems; ++n) {
            const int64_t w = (int64_t)n * gridDim.x + ((n ^ turn) & 1 ? gridDim.x - 1 - blockIdx.x : blockIdx.x);
            if (w >= total) break;
            int lo = 0, hi = B;   // invariant: start[lo] * H <= w < start[hi] * H
            while (hi - lo > 1) {
                const int step = (hi - lo + 63) / 64;
                const int idx = lo + (lane + 1) * step;
                const bool ok = idx < hi && (int64_t)start[idx] * H <= w;   // true for a prefix of the lanes
                const int cnt = __popcll(__builtin_amdgcn_ballot_w64(ok));
                lo += cnt * step;
                hi = hi < lo + step ? hi : lo + step;
            }
            if (lane == n) {
                my_p = lo;
                my_r = (int)(w - (int64_t)start[lo] * H);
            }
            n_items = n + 1;
        }
        if (lane == 0) mine->count = n_items;
        if (lane < n_items) {
            const int sample = in_sample_order ? my_p : (int)sorted[my_p];
            const int per_head = start[my_p + 1] - start[my_p];
            const int64_t row0 = offsets[sample];
            WorkSlot *slot = &mine->item[lane];
            slot->valid = 1;
            slot->sample = sample;
            slot->head = my_r / per_head;
            slot->block = my_r - (my_r / per_head) * per_head;
            slot->len = (int)(offsets[sample + 1] - row0);
            slot->row0_lo = (int)(uint32_t)row0;
            slot->row0_hi = (int)(uint32_t)((uint64_t)row0 >> 32);
            const int64_t *const oo = offsets_other ? offsets_other : offsets;   // the other side's rows: the same without a second array
            const int64_t orow0 = oo[sample];
            slot->olen = (int)(oo[sample + 1] - orow0);
            slot->orow0_lo = (int)(uint32_t)orow0;
            slot->orow0_hi = (int)(uint32_t)((uint64_t)orow0 >> 32);
        }
    }
    __syncthreads();
}

// Persistent-grid size for `kernel`: every compute unit filled to the kernel's occupancy, no more
// (extra workgroups would only find the work counter exhausted).  Queried once per kernel.  AtLeast: workgroups per compute unit
// that the caller relies on (the kernel has the registers and the LDS for them; they need not be resident at the same time).
template <auto Kernel, int AtLeast = 1>
inline int persistent_grid(int threads, int cus) {
    static int per_cu = 0;  // one instance per kernel function
    if (per_cu == 0) {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, Kernel, threads, 0) != hipSuccess || n < AtLeast) n = AtLeast;
        per_cu = n;
    }
    const int grid = cus * per_cu;
    return (grid + kXcds - 1) / kXcds * kXcds;  // next_work() relies on a multiple of 8
}


// Claim the next work item and decode it into `slot`.  Called by every lane of ONE wave (the claim itself is
// made by its lane 0, whose registers hold `cur`); meant to be issued right after a tile's first loads so
// that its latency chain (atomic, search, offsets) overlaps with theirs.
__device__ inline void claim_and_decode(WorkSlot *slot, const Schedule &s, const int64_t *offsets, int B, int H,
                                        int64_t total, WorkCursor &cur, const int64_t *offsets_other = nullptr) {
    const int lane = threadIdx.x & 63;
    int64_t w = -1;
    if (lane == 0) w = next_work(s.counter, cur, total);
    w = uniform64(w);
    if (w < 0) {
        if (lane == 0) slot->valid = 0;
        return;
    }
    const int p = find_position_wave(s.tile_start, B, H, w);
    const int t0 = s.tile_start[p];
    const int n = s.tile_start[p + 1] - t0;
    const int r = (int)(w - (int64_t)t0 * H);
    const int sample = s.order[p];
    const int64_t row0 = offsets[sample];
    const int len = (int)(offsets[sample + 1] - row0);
    if (offsets_other) {
        const int64_t orow0 = offsets_other[sample];
        const int olen = (int)(offsets_other[sample + 1] - orow0);
        if (lane == 0) {
            slot->olen = olen;
            slot->orow0_lo = (int)(uint32_t)orow0;
            slot->orow0_hi = (int)(uint32_t)((uint64_t)orow0 >> 32);
        }
    }
    if (lane == 0) {
        slot->valid = 1;
        slot->sample = sample;
        slot->head = r / n;
        slot->block = r - (r / n) * n;
        slot->len = len;
        slot->row0_lo = (int)(uint32_t)row0;
        slot->row0_hi = (int)(uint32_t)((uint64_t)row0 >> 32);
    }
}

// The reverse of load_work, by one lane.  (CROSS: see there.)
template <bool CROSS>
__device__ inline void park_work(WorkSlot *slot, const Work &t, bool valid) {
    slot->valid = valid;
    slot->sample = t.sample;
    slot->head = t.head;
    slot->block = t.block;
    slot->len = t.len;
    slot->row0_lo = (int)(uint32_t)t.row0;
    slot->row0_hi = (int)(uint32_t)((uint64_t)t.row0 >> 32);
    if (CROSS) {
        slot->olen = t.olen;
        slot->orow0_lo = (int)(uint32_t)t.orow0;
        slot->orow0_hi = (int)(uint32_t)((uint64_t)t.orow0 >> 32);
    }
}

// Without a schedule (Schedule::direct_blocks) a workgroup's item is its index: a block of a (sample, head); `mine` is filled by one
// lane.  A sample that is longer than the bound admits has its further blocks done by the same workgroups, up to kSmallItems each.
// The kernels' walks stay as they are: decoded there, as scalars, the items of calls with a schedule took up to 0.4 us longer to start.
// The bf16 kernels of long samples at D = 128 have instances of their own for it: chosen at run time, the two walks side by side cost both of
// them registers.  One instance and two, us: without a schedule 8 x 4 of up to 600 rows forward 18.5 -> 17.8, backward 51.0 -> 48.6 (cross
// 21.1 -> 19.5, 48.6 -> 46.2); with one, 300 x 4 of up to 300 63.4 -> 62.8, 224 -> 221; cross, 512 x 8, 256 queries against bimodal keys to
// 4096, 287 -> 281, 1070 -> 1057.  See launch_bwd_dkv_dma() for the two forms that keep one.
__device__ inline void direct_first(WorkSlot *slot, const Schedule &s, const int64_t *offsets, const int64_t *offsets_other, int H, int block_rows) {
    const int per_sample = H * s.direct_blocks, b = (int)blockIdx.x / per_sample, r = (int)blockIdx.x - b * per_sample;
    const int64_t *const oo = offsets_other ? offsets_other : offsets;
    Work t;
    t.sample = b;
    t.head = r / s.direct_blocks;
    t.block = r - t.head * s.direct_blocks;
    t.row0 = offsets[b];
    t.len = (int)(offsets[b + 1] - t.row0);
    t.orow0 = oo[b];
    t.olen = (int)(oo[b + 1] - t.orow0);
    park_work<true>(slot, t, t.block * block_rows < t.len);
}
__device__ inline void direct_small_work(SmallWork *mine, const Schedule &s, const int64_t *offsets, const int64_t *offsets_other, int H, int block_rows) {
    if (threadIdx.x == 0) {
        direct_first(&mine->item[0], s, offsets, offsets_other, H, block_rows);
        int n = mine->item[0].valid;
        while (n && n < kSmallItems && (mine->item[n - 1].block + s.direct_blocks) * block_rows < mine->item[0].len) {
            mine->item[n] = mine->item[n - 1];
            mine->item[n++].block += s.direct_blocks;
        }
        mine->count = n;
    }
    __syncthreads();
}
// Kernels with instances of their own for calls without a schedule have a template argument DIRECT: 1 without, 0 with one, kEither: as
// the call says (Schedule::direct_blocks).
constexpr int kEither = -1;
template <auto Kernel, int AtLeast = 1>
inline int item_grid(int threads, int B, int H, const Schedule &s, int cus) {
    return s.direct_blocks ? B * H * s.direct_blocks : persistent_grid<Kernel, AtLeast>(threads, cus);
}

// A workgroup's LDS copy of a schedule of at most kTabCap samples (position p of the sorted order: first tile,
// sample, rows): decoding a claimed work id then costs a few LDS reads instead of a chain of dependent global loads.
// Declare it __shared__; CROSS adds the other side's rows.
constexpr int kTabCap = 1024;
template <bool CROSS>
struct LdsSchedule {
    int32_t start[kTabCap + 1];
    int32_t sample[kTabCap], len[kTabCap], row0[kTabCap][2];
    int32_t olen[CROSS ? kTabCap : 1], orow0[CROSS ? kTabCap : 1][2];

    // Called by every thread of the workgroup, B <= kTabCap; a barrier must follow before decode().
    __device__ void fill(const Schedule &s, const int64_t *offsets, const int64_t *offsets_other, int B) {
        for (int p = threadIdx.x; p <= B; p += blockDim.x) start[p] = s.tile_start[p];
        for (int p = threadIdx.x; p < B; p += blockDim.x) {
            const int b = s.order[p];
            const int64_t r0 = offsets[b];
            sample[p] = b;
            len[p] = (int)(offsets[b + 1] - r0);
            row0[p][0] = (int)(uint32_t)r0;
            row0[p][1] = (int)(uint32_t)((uint64_t)r0 >> 32);
            if (CROSS) {
                const int64_t o0 = offsets_other[b];
                olen[p] = (int)(offsets_other[b + 1] - o0);
                orow0[p][0] = (int)(uint32_t)o0;
                orow0[p][1] = (int)(uint32_t)((uint64_t)o0 >> 32);
            }
        }
    }

    // Work id w (the same in every lane; < 0: nothing left) -> slot.  Called by every lane of one wave.
    __device__ void decode(WorkSlot *slot, int B, int H, int64_t w) const {
        const int lane = threadIdx.x & 63;
        if (w < 0) {
            if (lane == 0) slot->valid = 0;
            return;
        }
        int lo = 0, hi = B;   // invariant: start[lo] * H <= w < start[hi] * H
        while (hi - lo > 1) {
            const int step = (hi - lo + 63) / 64;
            const int idx = lo + (lane + 1) * step;
            const bool ok = idx < hi && (int64_t)start[idx] * H <= w;   // true for a prefix of the lanes
            const int cnt = __popcll(__builtin_amdgcn_ballot_w64(ok));
            lo += cnt * step;
            hi = hi < lo + step ? hi : lo + step;
        }
        if (lane == 0) {
            const int t0 = start[lo];
            const int n = start[lo + 1] - t0;
            const int r = (int)(w - (int64_t)t0 * H);
            slot->valid = 1;
            slot->sample = sample[lo];
            slot->head = r / n;
            slot->block = r - (r / n) * n;
            slot->len = len[lo];
            slot->row0_lo = row0[lo][0];
            slot->row0_hi = row0[lo][1];
            if (CROSS) {
                slot->olen = olen[lo];
                slot->orow0_lo = orow0[lo][0];
                slot->orow0_hi = orow0[lo][1];
            }
        }
    }
};

// Read the parked work item into scalar registers; returns false when nothing is left.  CROSS: the slot also holds
// the other side's rows.
template <bool CROSS = false>
__device__ inline bool load_work(const WorkSlot *slot, Work &t) {
    if (__builtin_amdgcn_readfirstlane(slot->valid) == 0) return false;
    t.sample = __builtin_amdgcn_readfirstlane(slot->sample);
    t.head = __builtin_amdgcn_readfirstlane(slot->head);
    t.block = __builtin_amdgcn_readfirstlane(slot->block);
    t.len = __builtin_amdgcn_readfirstlane(slot->len);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane(slot->row0_lo);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane(slot->row0_hi);
    t.row0 = (int64_t)(((uint64_t)hi << 32) | lo);
    t.orow0 = t.row0;
    t.olen = t.len;
    if (CROSS) {
        t.olen = __builtin_amdgcn_readfirstlane(slot->olen);
        const uint32_t olo = (uint32_t)__builtin_amdgcn_readfirstlane(slot->orow0_lo);
        const uint32_t ohi = (uint32_t)__builtin_amdgcn_readfirstlane(slot->orow0_hi);
        t.orow0 = (int64_t)(((uint64_t)ohi << 32) | olo);
    }
    return true;
}

// ---- launchers (each enqueues on `stream` and returns the launch status; `cus` = compute units of the device) ----

// Scheduler: fills order / tile_start of one or two schedules (jobs[0 .. n_jobs - 1]) of B samples and zeroes `n_counters`
// counters.  Blocks of block_rows rows are counted over `offsets`; samples are ordered by the length of the rows that
// stream past a block (offsets_other: cross attention; nullptr: the sample's own length).
struct ScheduleJob {
    const int64_t *offsets, *offsets_other;
    int block_rows;
    int32_t *order, *tile_start;
    int skip_rows = 0;   // samples with no more rows than this (on both sides) get no blocks: another kernel does them
};
hipError_t launch_schedules(const ScheduleJob *jobs, int n_jobs, int B, int32_t *counters, int n_counters, hipStream_t stream);
hipError_t launch_check_offsets(const int64_t *offsets, int B, int64_t max_len, int *flags, hipStream_t stream);

// Blocks per (sample, head) where every block that the bound on the lengths admits gets a workgroup of its own (those past a sample's
// end leave at once) and there is no schedule; 0: there is one.  As long as there is a compute unit for each, nothing is to be
// balanced and the schedule (a launch, or a sort in every workgroup) is all there is to save.  Fp32, microseconds of the kernels, with
// and without a schedule: four samples of up to 64 rows, D = 32, forward 8.7 and 7.5, with backward 28.7 and 25.1; 8 x 2 of up to 600,
// D = 64, 35.9 and 33.9, 147 and 141; 16 x 1 bimodal to 1000, D = 128, 93.9 and 92.1.  With more blocks than compute units the order, longest
// first, is worth more: 300 x 2 of up to 100, D = 64, 32.9 and 35.3, 110 and 143; 2000 x 4 bimodal to 128, D = 128, 375 and 629.
// bf16, D = 128, more than 256 rows: 8 x 4 of up to 600, forward 31.5 and 23.5, causal 30.1 and 20.2, with backward 98 and 84.5; 12 x 1 of up
// to 1884 60.4 and 50.1, 194 and 174; 4 x 4 of 4096 140 and 127, 612 and 596.
// D = 64: 5 x 2 of up to 300 12.4 and 10.9, 40.9 and 36.4; 8 x 4 of up to 600 17.0 and 15.9, 57.9 and 53.3; with two blocks per compute
// unit 20 x 3 Zipf to 700 loses, 18.3 and 19.7, 65 and 73.  (The bf16 figures with one kernel for both; those of their own take another 6 to 9 %
// off the calls without a schedule at D = 32 and 64, 4 to 11 % at D = 128.)
inline int direct_blocks(int64_t B, int64_t max_len, int H, int block_rows, int cus) {
    const int64_t blocks = (max_len + block_rows - 1) / block_rows;
    return blocks > 0 && blocks <= cus && B <= cus && B * H * blocks <= cus ? (int)blocks : 0;
}

// fp32 path
// Rows per block (and per streamed stage) of an fp32 kernel, which is its workgroup size: 64 rows are four waves, the quarters
// of a 64 x 64 square, 32 rows one wave.  Where at most 32 rows stream past a block two or three of the four waves have nothing
// to do; up to 64 rows single waves that are not in step still fill a compute unit better, if there are enough of them
// (`many`: more tiles than are dealt in the kernel).  Four waves -> one, microseconds, D = 128, backward: 4096 samples of at
// most 20 rows 538 -> 163, of at most 48 605 -> 434, 2000 x 2 heads of at most 64 621 -> 475; four samples of at most 64 41 -> 53.
constexpr int kF32BlockRows = 64, kF32ShortBlockRows = 32;
inline int f32_block_rows(int64_t max_streamed, bool many) {
    return max_streamed <= 32 || (many && max_streamed <= 64) ? kF32ShortBlockRows : kF32BlockRows;
}
// How an fp32 kernel runs: on the bf16 matrix instructions (split operands, jfa_f32_split.hip: head sizes 32 and 64) or on the fp32
// ones, and its rows per block.  A wave of the former has 32 stationary rows to itself and a stage of 32 streamed rows is split
// once per workgroup; the latter have the four waves share a 64 x 64 square, which fills the chip with fewer tiles and wastes
// less of a short stream.  Fp32 -> split instructions, microseconds:
//   forward, dQ: a workgroup per compute unit and SIMD pair has to find a tile: 32 x 2 heads of up to 256 rows, D = 64, forward 17 -> 22,
//   64 x 4 of up to 512 87 -> 69.  Streams of at most 64 rows: 2000 x 2 heads 54 -> 81.  Up to 128 rows: D = 32, 500 x 8 heads of
//   up to 100, 56 -> 61; D = 64 100 -> 81, but 200 x 2 heads, 200 queries against up to 100 keys (most of them few), 30 -> 34:
//   there with twice the tiles.  The tiles are counted from the bound on the lengths: where most samples are short they are few and a long
//   sample's tile of 128 rows is longer than one of 64.  D = 64, forward and backward, lengths uniform / one in ten long: 17 x 6 of up to
//   1132 (918 tiles at most) 155 -> 106 and 498 -> 329 / 54 -> 72 and 165 -> 165; 64 x 4 of up to 300 (768) 43 -> 36 and 128 -> 91 / 25 -> 33
//   and 71 -> 65; 128 x 4 of up to 500 (2048) 152 -> 109 and 476 -> 321 / 48 -> 45 and 141 -> 106;
//   dK / dV as the queries' kernels: a probability is exp(score - lse), and where one score is most of the log-sum-exp their errors
//   cancel only if both come from the same arithmetic.  (Split alone, behind the other forward: backward of 32 x 2 heads of up to
//   256 rows, D = 64, 53 -> 48, but at scores of standard deviation 16, D = 32, dV's error is twice that of either arithmetic alone.)
constexpr int kF32SplitRows = 128, kF32SplitKeyRows = 64;
struct F32Form { bool split; int rows; };
inline F32Form f32_form(int D, int64_t B, int64_t max_len, int H, int64_t max_streamed, bool many, int cus) {
    const double tiles = (double)B * (double)((max_len + kF32SplitRows - 1) / kF32SplitRows) * H;   // at most
    const bool worth = tiles > 2.0 * cus && (max_streamed > 128 || (D == 64 && max_streamed > 64 && tiles > 4.0 * cus));
    if (D <= 64 && max_len > 64 && worth) return {true, kF32SplitRows};
    return {false, f32_block_rows(max_streamed, many)};
}
inline F32Form f32_key_form(const F32Form &queries, int64_t max_streamed, bool many) {
    if (queries.split) return {true, kF32SplitKeyRows};
    return {false, f32_block_rows(max_streamed, many)};
}
// The same on the fp32 matrix instructions, where a call whose samples have one block each at most needs no schedule either, as long as
// its items fit one launch (a grid's threads are counted in 32 bits): streams are short, and the workgroups are dealt as places get free.  300 x 2 of up to 64 rows, D = 64, 23.3 -> 20.0,
// with backward 87.5 -> 76; 2000 x 4 of up to 30, D = 32, 38.2 -> 24.4, 106 -> 93; 4000 x 4 of up to 20, D = 128, forward 206 -> 170; cross,
// forward, up to 30 queries against up to 64 keys, one sample in ten long, 3000 x 4, D = 64, 66.4 -> 60.6, D = 128 146 -> 134.  Against up to 128
// keys the order matters again: up to 64 queries, one in ten long on both sides, 2000 x 4, D = 128, 330 -> 349, 3000 x 4, D = 64, 225 -> 232.
constexpr int64_t kF32DirectItems = (int64_t)1 << 22;
inline int f32_direct_blocks(const F32Form &form, int64_t B, int64_t max_len, int H, int64_t max_streamed, int cus) {
    if (form.split) return 0;
    if (max_len > 0 && max_len <= form.rows && max_streamed <= 64 && B <= kF32DirectItems && B * H <= kF32DirectItems) return 1;
    return direct_blocks(B, max_len, H, form.rows, cus);
}
// Cross attention: offsets = the queries' offsets, offsets_kv = the keys' (nullptr: the same array); schedules are
// built over the stationary side's offsets (s, s_dq: queries; s_dkv: keys).
// causal (self attention only, offsets_kv == nullptr): row i attends to rows 0 .. i of its sample.
// form: f32_form() of the queries or f32_key_form(); the kernel's schedule is built with its rows.
hipError_t launch_fwd_f32(const float *q, const float *k, const float *v, const int64_t *offsets,
                          const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, F32Form form, float *out, float *lse,
                          int cus, hipStream_t stream);
hipError_t launch_dq_f32(const float *q, const float *k, const float *v, const float *out, const float *dout, const float *lse,
                         const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, F32Form form,
                         float *dq, float *delta, int cus, hipStream_t stream);
// (offsets: the keys'; offsets_q: the queries', nullptr where they are the same)
hipError_t launch_dkv_f32(const float *q, const float *k, const float *v, const float *dout, const float *lse, const float *delta,
                          const int64_t *offsets, const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, F32Form form,
                          float *dk, float *dv, int cus, hipStream_t stream);
// (the dQ kernel of every path runs first and computes delta[h, row] = sum_d dout * out for the kernels after it)

// bf16 attention where no sample has more than kOneTileRows queries or keys (jfa_one_tile.hip): no schedule, every item a workgroup.
// Its rows: 32, 64 or 128, at least the longest length (0: longer ones).  Every call that fits takes these kernels.  Up to 64 rows, of
// 117 shapes (B 4 to 20000, H 1 to 8, all head sizes, self, causal, cross), none is slower than in the kernels for longer samples, the
// few-query ones included (4 samples of up to 20 rows, cross, D = 128, backward 9.4 -> 6.3 us); up to 128, of 126 one is slower than in
// two-wave 64-row tiles (D = 64, cross, 2048 x 4 heads, one sample in ten long on each side, backward 153 -> 165), none than in 128-row
// ones.  Microseconds, forward and backward, lengths uniform: 500 samples of up to 90 rows, D = 128, 14.7 -> 9.6, 50 -> 23; 2000 x 2 of
// up to 128, D = 64, 53 -> 34, 118 -> 103; D = 128 82 -> 56, 322 -> 173.
constexpr int kOneTileRows = 128;
inline int one_tile_rows(int64_t max_len, int64_t max_len_kv) {
    const int64_t longest = max_len > max_len_kv ? max_len : max_len_kv;
    return longest > kOneTileRows ? 0 : longest > 64 ? 128 : longest > 32 ? 64 : 32;
}
// Whether a call of 128 rows is made in two launches, samples of at most 64 rows first: in a workgroup for 128 rows half of the waves
// and half of the LDS would be idle for them.  In large batches that is worth a launch and a second look at every sample: backward,
// 2048 x 4 heads, one sample in ten long, D = 64 119 -> 77 us, D = 32 58 -> 49 (cross, where fewer are short on both sides, 74 -> 76);
// 2000 x 2, uniform, 101 -> 97, D = 128 169 -> 175.  Forward 2048 x 8 of up to 100 rows, geometric, D = 64 93 -> 84, 2000 x 2 34 -> 37;
// D = 32 45 -> 47, cross, D = 128, 177 -> 181.
inline bool one_tile_twice(bool backward, bool cross, int D, int64_t B, int H, int rows, int cus) {
    const int64_t items = B * H;
    if (rows != 128) return false;
    return backward ? items >= 32 * (int64_t)cus && (D >= 64 || !cross) : items >= 64 * (int64_t)cus && D >= 64 && !cross;
}
// least: samples with no more rows than this on both sides are left out
hipError_t launch_fwd_one_tile(const void *q, const void *k, const void *v, const int64_t *offsets, const int64_t *offsets_kv, bool causal,
                               int64_t B, int H, int D, int least, int rows, void *out, float *lse, hipStream_t stream);
hipError_t launch_bwd_one_tile(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                               const int64_t *offsets, const int64_t *offsets_kv, bool causal, int64_t B, int H, int D, int least, int rows,
                               void *dq, void *dk, void *dv, hipStream_t stream);
// Batches with longer samples: those of at most 64 rows may go to these kernels all the same (returns 64; 0: none do) while the
// others' schedules skip them.  What that gains is in the lengths, which the host does not know; the launch and a look at every
// sample cost some 5 us.  The line lies where lengths uniform on [1, max_len], of which few are short, lose nothing.  Self attention,
// microseconds, all in the other kernels -> split:
//   D = 128, 1024 x 4 heads, up to 250 rows: uniform, forward 169 -> 166, backward 627 -> 607; geometric (mean 64) 86 -> 75, 323 -> 261;
//   up to 600: uniform 469 -> 466, 1554 -> 1553; geometric 127 -> 94, 383 -> 282; one in ten long 158 -> 116, 483 -> 362.  512 x 4 of up
//   to 250, uniform: 85 -> 88, 340 -> 338.
//   D = 64 (these samples' tiles are cheaper in the other kernels), 2048 x 8 heads of up to 250: uniform 311 -> 299, 842 -> 825, one in
//   ten long 148 -> 80, 372 -> 230; of up to 600, uniform 935 -> 944, 2748 -> 2768.  1024 x 4 of up to 250, uniform: 85 -> 88, 243 -> 241.
//   D = 32, 2048 x 8 of up to 250, Zipf lengths, backward 436 -> 468.  Cross attention, both sides uniform (fewer samples are short on
//   both), D = 128, 1024 x 4 of up to 600: 444 -> 453, 1395 -> 1409.
inline int short_sample_rows(bool cross, int D, int64_t B, int64_t max_len, int H, int cus) {
    const int64_t items = B * H;
    const bool worth = D == 128 ? items >= 16 * (int64_t)cus : D == 64 && max_len <= 256 && items >= 64 * (int64_t)cus;
    return !cross && worth ? 64 : 0;
}

// bf16 attention, register-staged kernels (D = 128, short samples)
constexpr int kFwdBlockRows = 128;
constexpr int kBwdBlockRows = 128;
// Items per workgroup that the forward takes without claims.  A claim heads a tile here, its latency is not hidden, and the streams are
// short; in the backward, twice as long a tile, balance is worth more.  Microseconds with 4 and 16, forward and backward: 1024 x 4, up to
// 200 queries against up to 200 keys 131 and 130, 467 and 474; 512 x 4 of up to 130 on both sides 55 and 47, 159 and 161; 600 x 4 heads of
// up to 250 rows 102 and 99, 377 and 390, causal 97 and 93, 341 and 356; 900 x 4 of up to 250 143 and 144, 544 and 554; but 200 queries
// against up to 200 keys 192 and 197.
constexpr int kShortFixedItems = 16;
// In all bf16 launchers `offsets` belongs to the rows the schedule `s` was built over (queries for the forward and
// dQ, keys for dK / dV) and the second array to the rows that stream past them (cross attention; nullptr: the same).
// causal: self attention in which row i attends to rows 0 .. i of its sample (not together with a second array).
hipError_t launch_fwd_bf16(const void *q, const void *k, const void *v, const int64_t *offsets,
                           const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, void *out, float *lse,
                           int cus, hipStream_t stream);
hipError_t launch_dkv_bf16(const void *q, const void *k, const void *v, const void *dout, const float *lse,
                           const float *delta, const int64_t *offsets, const int64_t *offsets_q, bool causal, int B, int H,
                           int D, Schedule s, void *dk, void *dv, int cus, hipStream_t stream);
// out != nullptr: the kernel computes delta = rowsum(dO o O) itself and stores it in `delta` (launch it before the
// dK / dV kernel); out == nullptr: `delta` has been filled before.
hipError_t launch_dq_bf16(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse,
                          float *delta, const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H,
                          int D, Schedule s, void *dq, int cus, hipStream_t stream);

// bf16 attention for D = 32 and 64 at every length.  The dQ launch comes first and fills `stats` [2, H, sum_B]
// (delta, -lse * sqrt(D)) for the dK / dV launch.
// Rows of a tile: 128 (four waves) or 64 (two).  With short samples most waves of a 128-row tile have no rows but take registers
// and places; two-wave workgroups put more tiles on a compute unit at once, and a stage's copies on fewer waves, which long
// streams pay for.  (Where both sides are short the whole sample is one tile, see one_tile_rows().)  Microseconds, 128 -> 64 rows:
// 1024 x 4, 32 queries against at most 200 keys, D = 64, forward 44 -> 36; but 1024 x 4 of at most 200 rows on both sides 77 -> 103,
// backward 206 -> 272, and four samples of 4096 keys with 32 queries 53 -> 60; in small problems (see small_problem()) 0.5 more.
constexpr int kNarrowBlockRows = 128, kNarrowShortBlockRows = 64;
inline int narrow_block_rows(int64_t max_len, int64_t max_streamed, bool small) {
    return max_len <= 64 && max_streamed <= 256 && !small ? kNarrowShortBlockRows : kNarrowBlockRows;
}
// Items per workgroup up to which work is dealt without claims.  Longest items first and every other round backwards, such a
// deal is even to less than an item; a claim costs a short item more than that.  Long items gain nothing from it, and it parts the
// blocks that share streamed rows.  Microseconds with 4 and with 16 items: 1024 x 8 of at most 100 rows, D = 32, forward 84 and 53,
// backward 172 and 126; 500 x 8, 200 queries against at most 100 keys, 58 and 40, 112 and 89; 300 x 8 Zipf to 300, D = 64, 68 and 62;
// but 1024 x 2 of at most 500, D = 32, 83 and 88, 190 and 207; 512 x 8, 256 targets against 1024 keys, D = 32, 122 and 145.
inline int narrow_fixed_items(int64_t max_streamed) { return max_streamed <= 384 ? 16 : 4; }
hipError_t launch_dq_narrow(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                            const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, int block_rows,
                            void *dq, int cus, hipStream_t stream);
hipError_t launch_dkv_narrow(const void *q, const void *k, const void *v, const void *dout, const float *stats, const int64_t *offsets,
                             const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, int block_rows, void *dk, void *dv,
                             int cus, hipStream_t stream);
hipError_t launch_dq_narrow_short(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                                  const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, void *dq,
                                  int cus, hipStream_t stream);
hipError_t launch_dkv_narrow_short(const void *q, const void *k, const void *v, const void *dout, const float *stats, const int64_t *offsets,
                                   const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, void *dk, void *dv, int cus,
                                   hipStream_t stream);
hipError_t launch_dq_narrow_direct(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse, float *stats,
                                   const int64_t *offsets, const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, void *dq,
                                   int cus, hipStream_t stream);
hipError_t launch_dkv_narrow_direct(const void *q, const void *k, const void *v, const void *dout, const float *stats, const int64_t *offsets,
                                    const int64_t *offsets_q, bool causal, int B, int H, int D, Schedule s, void *dk, void *dv, int cus,
                                    hipStream_t stream);
hipError_t launch_fwd_narrow(const void *q, const void *k, const void *v, const int64_t *offsets, const int64_t *offsets_kv, bool causal,
                             int B, int H, int D, Schedule s, int block_rows, void *out, float *lse, int cus, hipStream_t stream);

// bf16 attention, direct-to-LDS kernels (D = 128, long samples; work items are blocks of kDmaBlockRows rows)
constexpr int kDmaBlockRows = 256;
hipError_t launch_fwd_bf16_dma(const void *q, const void *k, const void *v, const int64_t *offsets,
                               const int64_t *offsets_kv, bool causal, int B, int H, int D, Schedule s, void *out, float *lse,
                               int cus, hipStream_t stream);
// The dQ launch has to come first: with `out` given (the forward's output) it computes delta = rowsum(dout o out) and
// -lse * sqrt(D) itself and leaves them in `delta` [2, H, sum_B] for the dK / dV kernel.
hipError_t launch_bwd_dq_dma(const void *q, const void *k, const void *v, const void *out, const void *dout, const float *lse,
                             float *delta, const int64_t *offsets, const int64_t *offsets_other, bool causal, int B, int H,
                             int D, Schedule s, void *dq, int cus, hipStream_t stream);

// dK and dV of self attention in one kernel (pairs of waves share 32 keys; work items are blocks of kDkvBlockRows keys);
// `stats` is the [2, H, sum_B] buffer the dQ launch has filled.
constexpr int kDkvBlockRows = 128;
// Cross attention with at most 32 queries per sample, D = 128: a forward kernel bound by reading K and V once, and the
// whole backward (statistics, dQ, dK, dV) in one kernel and one pass over K and V.  `sched`: only `order` (the samples by their number of 32-key blocks, longest
// first; nullptr = sample order), `counter` and `static_only` are used; a work item is a whole (sample, head).
constexpr int kFewqRows = 32;
hipError_t launch_fwd_cross_fewq(const void *q, const void *k, const void *v, const int64_t *offsets_q,
                                 const int64_t *offsets_kv, int B, int H, int D, Schedule sched, void *out, float *lse, int cus,
                                 hipStream_t stream);
hipError_t launch_bwd_cross_fewq(const void *q, const void *k, const void *v, const void *out, const void *dout,
                                 const float *lse, float *stats, const int64_t *offsets_q, const int64_t *offsets_kv, int B,
                                 int H, int D, Schedule sched, void *dq, void *dk, void *dv, int cus, hipStream_t stream);
hipError_t launch_bwd_dkv_dma(const void *q, const void *k, const void *v, const void *dout, const float *stats,
                              const int64_t *offsets, const int64_t *offsets_other, bool causal, int B, int H, int D, Schedule s, void *dk,
                              void *dv, int cus,
                              hipStream_t stream);

// Unfused jagged attention (Table 1): offsets of the jagged square array, then the three operators.
hipError_t launch_square_offsets(const int64_t *offsets, int B, int64_t *sq, hipStream_t stream);
hipError_t launch_unfused_scores(const void *q, const void *k, const int64_t *offsets, const int64_t *sq, int B, int H,
                                 int D, Schedule s, float scale, float *scores, int cus, hipStream_t stream);
hipError_t launch_unfused_softmax_bwd(const float *probs, const int64_t *offsets, const int64_t *sq, int B, int H,
                                      Schedule s, float scale, float *dprobs, int cus, hipStream_t stream);
hipError_t launch_unfused_apply_t(const float *X, const void *x, const int64_t *offsets, const int64_t *sq, int B, int H,
                                  int D, Schedule s, void *out, int cus, hipStream_t stream);
hipError_t launch_unfused_softmax(const int64_t *offsets, const int64_t *sq, int B, int H, Schedule s, float *scores,
                                  int cus, hipStream_t stream);
hipError_t launch_unfused_apply(const float *probs, const void *v, const int64_t *offsets, const int64_t *sq, int B,
                                int H, int D, Schedule s, void *out, int cus, hipStream_t stream);

// Whether an operator stores its rows past the L2 (non-temporal): where the tensor, at most B * max_len rows, is larger than the
// memory-side cache.  Of a smaller one the next operator finds more in the caches: 168 samples of up to 309 rows, D = T = 128, five
// operators: 48.7 us, stored past the L2 49.8; padding and back, 66 samples of up to 3787 rows of 320 bytes, 32.1, past it 33.1.
inline bool past_l2(int64_t B, int64_t max_len, int64_t row_bytes) { return (double)B * (double)max_len * (double)row_bytes > 256e6; }
// A template parameter: given both stores behind a runtime flag the compiler makes them one and drops the hint.
template <bool kPast, typename V> __device__ inline void store_streaming(V *dst, V x) {
    if constexpr (kPast) __builtin_nontemporal_store(x, dst);
    else *dst = x;
}

// Jagged <-> padded-dense conversion (Section 2.2); rows are row_chunks 16-byte chunks long.
hipError_t launch_convert(bool to_dense, const void *src, void *dst, const int64_t *offsets, int B, int64_t max_len,
                          int64_t row_chunks, uint32_t pad, int cus, hipStream_t stream);

// Jagged feature operators (Table 1); `counter` is one work counter, cleared by the launcher where the kernel looks at it.
hipError_t launch_jagged_dense_bmm(const void *x, const void *w, const int64_t *offsets, int B, int64_t max_len, int D, int T,
                                   int32_t *counter, void *out, int cus, hipStream_t stream);
hipError_t launch_jagged_jagged_bmm(const void *x, const void *y, const int64_t *offsets, int B, int D, int T,
                                    int32_t *counter, void *out, int cus, hipStream_t stream);
hipError_t launch_jagged_softmax(bool backward, const void *a, const void *b, const int64_t *offsets, int B, int64_t max_len, int D,
                                 int32_t *counter, void *out, int cus, hipStream_t stream);

}  // namespace jfa
