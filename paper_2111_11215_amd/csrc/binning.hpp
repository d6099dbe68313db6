// Counting sort of samples by grid cell, shared by the fine and the coarse
// stage: ranks within a cell while the samples' wavefronts count them, then a
// device-wide exclusive scan of the counts.
#pragma once

#include "common.hpp"

namespace {

constexpr int kScanPer = 8192;   // elements per block of the device-wide scan

// Rank of this lane's sample among the samples of its cell.  Lanes hold
// consecutive samples, so equal cells form runs; each run's first lane adds
// the run length to the cell's count with one atomic, and the run shares the
// returned base.  All 64 lanes must call it; lanes with ok == false take part
// in the vote only.
__device__ __forceinline__ int run_rank(int cell, bool ok, int lane, int* __restrict__ counts) {
    const int prev = __shfl_up(cell, 1, 64);
    const bool head = !ok || lane == 0 || prev != cell;
    const uint64_t heads = __ballot(head);
    const uint64_t upto = (lane == 63) ? ~0ull : ((2ull << lane) - 1);
    const uint64_t le = heads & upto;
    const int leader = 63 - __clzll(static_cast<long long>(le));
    const uint64_t gt = heads & ~upto;
    const int next = gt ? __ffsll(static_cast<long long>(gt)) - 1 : 64;
    int rbase = 0;
    if (ok && lane == leader) rbase = atomicAdd(counts + cell, next - lane);
    rbase = __shfl(rbase, leader, 64);
    return rbase + lane - leader;
}

__global__ __launch_bounds__(256) void fill_int_kernel(int* __restrict__ p, int64_t n, int v) {
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[i] = v;
}

// Device-wide exclusive scan of int32 counts in three passes.
__device__ __forceinline__ int block_excl_scan_1024(int v, int* sh, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) sh[wave] = incl;
    __syncthreads();
    int woff = 0, tot = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) woff += sh[w];
        tot += sh[w];
    }
    __syncthreads();
    *total = tot;
    return woff + incl - v;
}

// Eight consecutive counts of one thread (zero past n); 32-byte aligned.
__device__ __forceinline__ void load8(const int* __restrict__ in, int64_t base, int64_t n, int v[8]) {
    if (base + 8 <= n) {
        const int4 a = *reinterpret_cast<const int4*>(in + base);
        const int4 b = *reinterpret_cast<const int4*>(in + base + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
        for (int u = 0; u < 8; ++u) v[u] = base + u < n ? in[base + u] : 0;
    }
}

__global__ __launch_bounds__(1024) void scan_block_sums_kernel(const int* __restrict__ in, int64_t n,
                                                               long long* __restrict__ bsum) {
    __shared__ int sh[16];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanPer + threadIdx.x * 8;
    int v8[8];
    load8(in, base, n, v8);
    int v = 0;
    for (int u = 0; u < 8; ++u) v += v8[u];
    int tot;
    block_excl_scan_1024(v, sh, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// Exclusive scan of the counts: each workgroup adds the totals of all the
// workgroups before it (read from bsum, summed in the workgroup) to its own
// in-workgroup scan.
__global__ __launch_bounds__(1024) void scan_apply_kernel(const int* __restrict__ in, int64_t n,
                                                          const long long* __restrict__ bsum, int* __restrict__ out) {
    __shared__ int sh[16];
    __shared__ long long sp[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    long long pre = 0;
    for (int b = threadIdx.x; b < static_cast<int>(blockIdx.x); b += 1024) pre += bsum[b];
    for (int off = 32; off > 0; off >>= 1) pre += __shfl_xor(pre, off, 64);
    if (lane == 0) sp[wave] = pre;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanPer + threadIdx.x * 8;
    int v[8];
    load8(in, base, n, v);
    int loc = 0;
    for (int u = 0; u < 8; ++u) loc += v[u];
    int tot;
    const int ex = block_excl_scan_1024(loc, sh, &tot);   // its barriers also publish sp
    long long blk = 0;
    for (int w = 0; w < 16; ++w) blk += sp[w];
    int run = static_cast<int>(blk) + ex;
    int o[8];
    for (int u = 0; u < 8; ++u) {
        o[u] = run;
        run += v[u];
    }
    if (base + 8 <= n) {
        *reinterpret_cast<int4*>(out + base) = make_int4(o[0], o[1], o[2], o[3]);
        *reinterpret_cast<int4*>(out + base + 4) = make_int4(o[4], o[5], o[6], o[7]);
    } else {
        for (int u = 0; u < 8; ++u)
            if (base + u < n) out[base + u] = o[u];
    }
}

// Scratch bytes of run_cell_scan over n counts.
inline size_t cell_scan_bytes(int64_t n) { return static_cast<size_t>((n + kScanPer - 1) / kScanPer + 1) * 8; }

// Exclusive scan of n counts into starts.
inline int32_t run_cell_scan(const int* counts, int64_t n, void* scratch, int* starts, hipStream_t s) {
    const int nb = static_cast<int>((n + kScanPer - 1) / kScanPer);
    long long* bsum = static_cast<long long*>(scratch);
    DVGO_LAUNCH(K_CELL_SCAN, scan_block_sums_kernel, dim3(nb), dim3(1024), 0, s, counts, n, bsum);
    DVGO_LAUNCH(K_CELL_SCAN, scan_apply_kernel, dim3(nb), dim3(1024), 0, s, counts, n, bsum, starts);
    return dvgo::launch_status();
}

}  // namespace
