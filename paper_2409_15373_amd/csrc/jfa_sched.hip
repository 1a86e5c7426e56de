// Offsets-driven work scheduler: turns the jagged tensor's offsets array (paper Section 2) into a
// table of (sample, row-block) tiles, longest samples first, so that the persistent attention
// kernels hand out exactly the non-padded work and short samples leave no idle workgroups.
#include "jfa_common.h"

namespace jfa {

constexpr int kSchedThreads = 1024;

// Inclusive scan of one int per thread across the workgroup (kSchedThreads threads).
__device__ inline int block_inclusive_scan(int x, int *wave_sums) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) wave_sums[wave] = x;
    __syncthreads();
    if (wave == 0) {
        int s = lane < kSchedThreads / 64 ? wave_sums[lane] : 0;
        for (int d = 1; d < kSchedThreads / 64; d <<= 1) {
            const int y = __shfl_up(s, d, 64);
            if (lane >= d) s += y;
        }
        if (lane < kSchedThreads / 64) wave_sums[lane] = s;
    }
    __syncthreads();
    const int base = wave > 0 ? wave_sums[wave - 1] : 0;
    __syncthreads();
    return x + base;
}

// offsets_other (cross attention, else nullptr): the offsets of the rows that stream past a block.  Blocks are
// counted over `offsets`, but a block's cost grows with the length of the stream, so samples are ordered by that.
// One workgroup per schedule: the two of a backward are built side by side in one launch (4 us less on training steps of
// 426 and 621 us; within the noise of steps of 4 ms).
// What bounds it is a chain of trips to memory.  A batch of at most kSchedKept samples makes one: a thread's lengths stay in
// registers from the histogram to the scatter, and the sorted block counts go through LDS to the scan.
constexpr int kSchedPerThread = 4;
constexpr int kSchedKept = kSchedThreads * kSchedPerThread;
template <bool kKept>
__global__ __launch_bounds__(kSchedThreads) void schedule_kernel(ScheduleJob job0, ScheduleJob job1, int B,
                                                                 int32_t *__restrict__ counters, int n_counters) {
    const ScheduleJob &job = blockIdx.x == 0 ? job0 : job1;
    const int64_t *__restrict__ const offsets = job.offsets;
    const int64_t *__restrict__ const offsets_other = job.offsets_other;
    const int block_rows = job.block_rows, skip_rows = job.skip_rows;
    int32_t *__restrict__ const order = job.order;
    int32_t *__restrict__ const tile_start = job.tile_start;
    __shared__ int hist[kSchedBins];    // samples per bin, then the bin's first position in `order`
    __shared__ int cursor[kSchedBins];  // next free slot of each bin
    __shared__ int wave_sums[kSchedThreads / 64];
    __shared__ int carry;
    __shared__ int sorted_blocks[kKept ? kSchedKept : 1];   // row blocks of the sample at a position (otherwise parked in tile_start[pos + 1])
    const int tid = threadIdx.x;

    // a sample's sort key, the row-block count of the stream (of the sample itself in self attention), and its row blocks
    // (a sample's length fits 31 bits everywhere: a 32-bit division, a quarter of a 64-bit one's instructions)
    auto length = [&](const int64_t *o, int b) { return (int)(o[b + 1] - o[b]); };
    auto blocks_of = [&](int len) { return len > 0 ? (int)(((uint32_t)len + (uint32_t)block_rows - 1) / (uint32_t)block_rows) : 0; };
    auto look = [&](int b, int &bin, int &n) {
        const int len = length(offsets, b), other = offsets_other ? length(offsets_other, b) : len;
        const bool skip = len <= skip_rows && other <= skip_rows;
        const int key = skip ? 0 : blocks_of(other);
        n = skip ? 0 : blocks_of(len);
        bin = key < kSchedBins - 1 ? key : kSchedBins - 1;
    };
    int bins[kSchedPerThread], blocks[kSchedPerThread];
    if (kKept) {
#pragma unroll
        for (int u = 0; u < kSchedPerThread; ++u) {
            const int b = tid + u * kSchedThreads;
            bins[u] = blocks[u] = 0;
            if (b < B) look(b, bins[u], blocks[u]);
        }
    }
    for (int i = tid; i < n_counters; i += kSchedThreads) counters[i] = 0;
    for (int i = tid; i < kSchedBins; i += kSchedThreads) { hist[i] = 0; cursor[i] = 0; }
    __syncthreads();

    // calls f(sample, bin, row blocks) for this thread's samples
    auto for_samples = [&](auto f) {
        if (kKept) {
#pragma unroll
            for (int u = 0; u < kSchedPerThread; ++u)
                if (tid + u * kSchedThreads < B) f(tid + u * kSchedThreads, bins[u], blocks[u]);
        } else {
            for (int b = tid; b < B; b += kSchedThreads) {
                int bin, n;
                look(b, bin, n);
                f(b, bin, n);
            }
        }
    };
    // 1. histogram of the sort key
    for_samples([&](int, int bin, int) { atomicAdd(&hist[bin], 1); });
    __syncthreads();

    // 2. bins in descending order: first position of bin i = number of samples in bins above i.
    //    Thread t scans bin (kSchedBins-1-t), so an exclusive prefix over t is a suffix sum over bins.
    {
        const int bin = kSchedBins - 1 - tid;
        const int cnt = hist[bin];
        const int incl = block_inclusive_scan(cnt, wave_sums);
        hist[bin] = incl - cnt;
    }
    __syncthreads();

    // 3. scatter samples to their bin
    for_samples([&](int b, int bin, int n) {
        const int pos = hist[bin] + atomicAdd(&cursor[bin], 1);
        order[pos] = b;
        if (kKept) sorted_blocks[pos] = n;
        else tile_start[pos + 1] = n;
    });
    if (tid == 0) { tile_start[0] = 0; carry = 0; }
    __syncthreads();

    // 4. inclusive scan of the sorted block counts into tile_start[1..B]
    for (int base = 0; base < B; base += kSchedThreads) {
        const int i = base + tid;
        const int x = i < B ? (kKept ? sorted_blocks[i] : tile_start[i + 1]) : 0;
        const int incl = block_inclusive_scan(x, wave_sums) + carry;
        if (i < B) tile_start[i + 1] = incl;
        __syncthreads();
        if (tid == kSchedThreads - 1) carry = incl;
        __syncthreads();
    }
}

__global__ void check_offsets_kernel(const int64_t *__restrict__ offsets, int B, int64_t max_len, int *flags) {
    int f = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && offsets[0] != 0) f |= 1;
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < B; b += gridDim.x * blockDim.x) {
        const int64_t len = offsets[b + 1] - offsets[b];
        if (len < 0) f |= 2;
        if (len > max_len) f |= 4;
    }
    if (f) atomicOr(flags, f);
}

hipError_t launch_schedules(const ScheduleJob *jobs, int n_jobs, int B, int32_t *counters, int n_counters, hipStream_t stream) {
    if (B <= kSchedKept)
        hipLaunchKernelGGL(schedule_kernel<true>, dim3(n_jobs), dim3(kSchedThreads), 0, stream, jobs[0], jobs[n_jobs - 1], B, counters, n_counters);
    else
        hipLaunchKernelGGL(schedule_kernel<false>, dim3(n_jobs), dim3(kSchedThreads), 0, stream, jobs[0], jobs[n_jobs - 1], B, counters, n_counters);
    return hipGetLastError();
}

hipError_t launch_check_offsets(const int64_t *offsets, int B, int64_t max_len, int *flags, hipStream_t stream) {
    const int grid = B / 256 + 1 < 1024 ? B / 256 + 1 : 1024;
    hipLaunchKernelGGL(check_offsets_kernel, dim3(grid), dim3(256), 0, stream, offsets, B, max_len, flags);
    return hipGetLastError();
}

}  // namespace jfa
