// Device-side meeting points for the resident kernels of libdsq: kernels that keep a whole (small) problem in the
// registers of one launch, one workgroup per worker row and 4096-column chunk, and exchange what Algorithm 1 makes a
// worker know about other columns and other workers (a vector's range, its k-th magnitude, the neighbours' messages)
// through device memory between phases.  At the size of the paper's own experiment (8 workers, 272,474 parameters)
// a step is bound by launches, not by bytes: the compressors that need such a property of the whole vector took
// 4 to 12 launches and as many round trips of the state through memory.
//
// Waiting inside a kernel needs every workgroup of the launch to be running.  Three things see to it that every wait
// ends, whatever else the GPU is doing:
//   * a resident plan is only made if its workgroups fill at most half of what the GPU holds at once, and ds_step only
//     takes it while the streams that such handles step on fit next to each other (Seat in dsq_api.hip);
//   * the first meeting (meet_or_part) has a time limit, and its outcome is decided on ONE word: either all arrive
//     (from then on every workgroup runs, and later meetings end), or one workgroup's limit passes first and
//     all part.  Nothing but scratch memory has been written by then;
//   * after parting, the workgroup that leaves last (leave()) -- it waits for nobody -- does the whole step alone.
//
// Data exchanged inside a launch is written and read with relaxed atomics of agent scope: the XCDs' L2 caches are
// not coherent for plain accesses before a kernel ends.  A wave waits for its stores (drain) before its workgroup
// counts as arrived.
//
// Measured on MI355X: a meeting of 536 workgroups of 256 threads takes 1.85 us with 32 arrival counters and 32 flags,
// 9.2 us with one counter that everybody polls, and a kernel boundary at least 2.5 us plus the loads that bring the
// state back into registers.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

#include "dsq_internal.h"

namespace dsq {
namespace {

constexpr uint32_t kMeetGroups = 32;                        // arrival counters and flags of one meeting
constexpr uint32_t kMeetLine = 64;                          // words between them: 256 bytes
constexpr uint32_t kMeetWords = (1 + 2 * kMeetGroups) * kMeetLine;   // root | arrival counters | flags
constexpr uint32_t kPartBit = 0x80000000u;                  // in a flag: called off
constexpr unsigned long long kPartRoot = 1ull << 63;        // in a root
// Ticks of the 100 MHz clock: 10 ms.  About what the step costs one workgroup alone (8 workers x 272,474 parameters: norm-rescaled
// 4.5 ms, GSpar 10 to 15, top-k 17), so that a wait that would have ended soon is not given up for something dearer.
constexpr uint64_t kMeetPatience = 1'000'000;

template <typename V> __device__ __forceinline__ V agent_load(const V* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename V> __device__ __forceinline__ void agent_store(V* p, V v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ uint32_t agent_add(uint32_t* p, uint32_t v) { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// All of this wave's stores have reached memory.
__device__ __forceinline__ void drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ uint32_t meet_members(uint32_t blocks, uint32_t g) { return (blocks - g + kMeetGroups - 1) / kMeetGroups; }
__device__ __forceinline__ uint32_t meet_groups(uint32_t blocks) { return blocks < kMeetGroups ? blocks : kMeetGroups; }

// Counts this workgroup in and waits for the others; called by all threads.  The words are never cleared: `epoch` launches
// have come this way before, so each counter stands at epoch times its arrivals.  MAY_PART: returns false if `patience`
// ran out for some workgroup before all had arrived -- the same answer in every workgroup.  CLOSING: the last meeting
// of a launch; the workgroup that completes it advances the epoch and the step counter, which all have read by then.
template <bool MAY_PART, bool CLOSING>
__device__ __forceinline__ bool meet(uint32_t* w, uint32_t blocks, unsigned long long epoch, uint64_t patience, unsigned long long* epoch_cell = nullptr,
                                     unsigned long long* t_ptr = nullptr) {
    __shared__ uint32_t verdict;
    drain();
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t g = blockIdx.x % kMeetGroups, groups = meet_groups(blocks);
        const uint32_t now = (uint32_t)(epoch + 1ull) & ~kPartBit;
        const unsigned long long complete = groups * (epoch + 1ull);
        unsigned long long* root = reinterpret_cast<unsigned long long*>(w);
        uint32_t* flags = w + (size_t)(1 + kMeetGroups) * kMeetLine;
        if (agent_add(w + (size_t)(1 + g) * kMeetLine, 1u) + 1u == meet_members(blocks, g) * (uint32_t)(epoch + 1ull)) {
            if (__hip_atomic_fetch_add(root, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1ull == complete) {
                // the last group, and nobody has called it off
                for (uint32_t q = 0; q < groups; ++q) agent_store(flags + (size_t)q * kMeetLine, now);
                if constexpr (CLOSING) {
                    agent_store(epoch_cell, epoch + 1ull);
                    __hip_atomic_fetch_add(t_ptr, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);     // one step taken
                }
            }
        }
        const uint64_t since = MAY_PART ? __builtin_amdgcn_s_memrealtime() : 0;
        bool called_off = false;
        uint32_t v;
        while (((v = agent_load(flags + (size_t)g * kMeetLine)) & ~kPartBit) != now) {
            if (MAY_PART && !called_off && __builtin_amdgcn_s_memrealtime() - since >= patience) {
                called_off = true;
                // only while it is neither called off nor complete (the mark must not stay behind on a complete root)
                unsigned long long old = agent_load(root);
                while (old < complete && !__hip_atomic_compare_exchange_strong(root, &old, old | kPartRoot, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {}
                if (old < complete)
                    for (uint32_t q = 0; q < groups; ++q) agent_store(flags + (size_t)q * kMeetLine, now | kPartBit);
            }
            __builtin_amdgcn_s_sleep(1);
        }
        verdict = v & kPartBit;
    }
    __syncthreads();
    return verdict == 0u;
}

// After parting: counts this workgroup out (the finished-workgroup cells behind the step counter, as the tile kernel uses
// them); true in the one workgroup that leaves last.  Called by all threads.
__device__ __forceinline__ bool leave(unsigned long long* t_ptr, uint32_t blocks) {
    __shared__ uint32_t is_last;
    drain();                                                // flags this workgroup has set land before it counts itself out
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t last = 0;
        const uint32_t cell = blockIdx.x & 63u;
        const unsigned long long members = (blocks >> 6) + (cell < (blocks & 63u) ? 1u : 0u);
        unsigned long long* cnt = t_ptr + 32ull * (1 + cell);
        if (__hip_atomic_fetch_add(cnt, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == members - 1ull) {
            __hip_atomic_store(cnt, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long cells = blocks < 64u ? blocks : 64u;
            if (__hip_atomic_fetch_add(t_ptr + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == cells - 1ull) {
                __hip_atomic_store(t_ptr + 1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = 1u;
            }
        }
        is_last = last;
    }
    __syncthreads();
    return is_last != 0u;
}

// The step that one workgroup did alone is done: puts the words of all `meetings` where the next launch expects them
// and advances the epoch and the step counter.
__device__ __forceinline__ void close_alone(uint32_t* w, uint32_t meetings, uint32_t blocks, unsigned long long epoch, unsigned long long* epoch_cell,
                                            unsigned long long* t_ptr) {
    const uint32_t groups = meet_groups(blocks);
    for (uint32_t q = threadIdx.x; q < meetings * groups; q += blockDim.x) {
        uint32_t* one = w + (size_t)(q / groups) * kMeetWords;
        const uint32_t g = q % groups;
        agent_store(one + (size_t)(1 + g) * kMeetLine, meet_members(blocks, g) * (uint32_t)(epoch + 1ull));
        if (g == 0) agent_store(reinterpret_cast<unsigned long long*>(one), groups * (epoch + 1ull));
    }
    if (threadIdx.x == 0) {
        agent_store(epoch_cell, epoch + 1ull);
        __hip_atomic_fetch_add(t_ptr, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Sum over a wave of 64 in the order of the balanced adjacent-pairs tree, on the DPP cross-lane path (a shuffle through
// LDS takes several times as long per level): row_shr 1, 2, 4, 8 fold each row of 16 lanes into its last lane,
// row_bcast15 and row_bcast31 fold the rows; lanes without a source add zero.  The result is uniform.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add_f64(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROW_MASK, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, ROW_MASK, 0xF, false);
    return v + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double wave_tree_f64(double v) {
    v = dpp_add_f64<0x111, 0xF>(v);
    v = dpp_add_f64<0x112, 0xF>(v);
    v = dpp_add_f64<0x114, 0xF>(v);
    v = dpp_add_f64<0x118, 0xF>(v);
    v = dpp_add_f64<0x142, 0xA>(v);
    v = dpp_add_f64<0x143, 0xC>(v);
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), 63);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_max_f32(float v) {
    return fmaxf(v, __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), CTRL, ROW_MASK, 0xF, false)));
}
__device__ __forceinline__ float wave_max_f32(float v) {
    v = dpp_max_f32<0x111, 0xF>(v);
    v = dpp_max_f32<0x112, 0xF>(v);
    v = dpp_max_f32<0x114, 0xF>(v);
    v = dpp_max_f32<0x118, 0xF>(v);
    v = dpp_max_f32<0x142, 0xA>(v);
    v = dpp_max_f32<0x143, 0xC>(v);
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_add_u32(uint32_t v) {
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_u32(uint32_t v) {                  // inclusive prefix sums over the lanes
    v = dpp_add_u32<0x111, 0xF>(v);
    v = dpp_add_u32<0x112, 0xF>(v);
    v = dpp_add_u32<0x114, 0xF>(v);
    v = dpp_add_u32<0x118, 0xF>(v);
    v = dpp_add_u32<0x142, 0xA>(v);
    v = dpp_add_u32<0x143, 0xC>(v);
    return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_u32(v), 63); }

// The part of the state that one workgroup of a resident kernel keeps in registers: 4096 columns of a worker row, sixteen
// columns of a thread in four quads of adjacent ones.
constexpr int kResThreads = 256;
constexpr int kResIters = 4;
constexpr int kResChunk = 4 * kResThreads * kResIters;
constexpr int kResNear = 4;                                 // neighbours whose index and coefficient are fetched ahead

template <typename Args>                                    // L2Args or TopkArgs
struct ResidentChunk {
    const Args& a;
    const uint32_t nchunks;
    int row = 0;
    uint32_t chunk = 0;
    int e0 = 0, e1 = 0;
    int near[kResNear];
    float near_coef[kResNear];
    float4 xh[kResIters], v[kResIters];

    __device__ __forceinline__ ResidentChunk(const Args& a_, uint32_t nchunks_) : a(a_), nchunks(nchunks_) {}

    __device__ __forceinline__ uint64_t column(int it) const { return (uint64_t)chunk * kResChunk + (uint64_t)it * (4 * kResThreads) + 4u * threadIdx.x; }
    __device__ __forceinline__ size_t place() const { return (size_t)row * nchunks + chunk; }

    __device__ __forceinline__ void locate(uint32_t which) {   // rows one after the other
        __syncthreads();                                    // the shared memory of the chunk before is free
        row = (int)(which / nchunks);
        chunk = which % nchunks;
        e0 = a.rowptr[row];
        e1 = a.rowptr[row + 1];
#pragma unroll
        for (int u = 0; u < kResNear; ++u) {
            near[u] = a.col[e0 + u < e1 ? e0 + u : e0];
            near_coef[u] = a.coef[e0 + u < e1 ? e0 + u : e0];
        }
    }

    // Algorithm 1, line 5, for the sixteen columns of every thread of chunk `which`
    __device__ __forceinline__ void load(uint32_t which) {
        locate(which);
        const float* xr = a.x + (uint64_t)row * a.ld;
        const float* dr = a.delta + (uint64_t)row * a.ld;
        const float* gr = a.g + (uint64_t)row * a.g_ld;
        float4 g[kResIters];
#pragma unroll
        for (int it = 0; it < kResIters; ++it) {
            const uint64_t col = column(it);
            xh[it] = *reinterpret_cast<const float4*>(xr + col);
            v[it] = *reinterpret_cast<const float4*>(dr + col);
            g[it] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (col < a.N) g[it] = *reinterpret_cast<const float4*>(gr + col);
        }
#pragma unroll
        for (int it = 0; it < kResIters; ++it) {
            const uint64_t col = column(it);
            if (col + 3 >= a.N) {                           // whatever lies behind column N-1 is not a gradient
                if (col + 1 >= a.N) g[it].y = 0.f;
                if (col + 2 >= a.N) g[it].z = 0.f;
                g[it].w = 0.f;
            }
            xh[it].x = fmaf(-a.gamma, g[it].x, xh[it].x); v[it].x = xh[it].x + v[it].x;
            xh[it].y = fmaf(-a.gamma, g[it].y, xh[it].y); v[it].y = xh[it].y + v[it].y;
            xh[it].z = fmaf(-a.gamma, g[it].z, xh[it].z); v[it].z = xh[it].z + v[it].z;
            xh[it].w = fmaf(-a.gamma, g[it].w, xh[it].w); v[it].w = xh[it].w + v[it].w;
        }
    }

    // The thread's index as a value the compiler knows nothing about: what is derived from it is worked out where it is
    // needed, and addresses are not kept in registers from one end of the kernel to the other.
    static __device__ __forceinline__ uint32_t thread_here() {
        uint32_t t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    }

    __device__ __forceinline__ void store(int it, uint32_t thread) const {
        const uint64_t at = (uint64_t)row * a.ld + (uint64_t)chunk * kResChunk + (uint32_t)it * (4 * kResThreads) + 4u * thread;
        *reinterpret_cast<float4*>(a.x + at) = xh[it];
        *reinterpret_cast<float4*>(a.delta + at) = v[it];
    }

    // One workgroup does everything: what it has written in this phase is there for the next.
    __device__ __forceinline__ void phase_end() const {
        drain();
        __syncthreads();
    }
};

// The smallest number of pieces of `size` that a memory of `whole` can hold with no room left for one more, whatever lies
// or lay between them: gaps of up to size - step on either side of each.
inline uint64_t sure_pieces(uint64_t whole, uint64_t size, uint64_t step) {
    const uint64_t gap = size - step;
    return whole <= gap ? 0 : (whole - gap + size + gap - 1) / (size + gap);
}

// The part of the current device that `blocks` workgroups of a resident kernel fill, in units of 1 / kWholeDevice and rounded
// up; 0 if a resident plan is not made: more than half of what an empty device holds at once.  The whole is what the device
// holds for sure, next to anything that ends by itself: registers and LDS are given out in one piece each, and where other
// kernels' waves have come and gone between them five waves of 96 registers need not fit into the 512 of a SIMD, three
// do.  (Two kernels of 536 workgroups started together with a third kernel whose waves take 80 registers did not fit on the
// 256 compute units in 24 of 30 attempts; on an otherwise idle device they do.)
template <typename K>
uint32_t resident_share(K kernel, int threads, uint64_t blocks) {
    int per_cu = 0, cus = 0, lds = 0, dev = 0;
    hipFuncAttributes attr{};
    if (hipGetDevice(&dev) != hipSuccess || hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
        hipFuncGetAttributes(&attr, reinterpret_cast<const void*>(kernel)) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, dev) != hipSuccess || per_cu < 1 || cus < 1) {
        (void)hipGetLastError();
        return 0;
    }
    constexpr uint64_t kRegisters = 512, kRegisterStep = 8;   // of a SIMD, per lane; a workgroup has a wave on each of four
    const uint64_t regs = ((uint64_t)(attr.numRegs > 0 ? attr.numRegs : 1) + kRegisterStep - 1) / kRegisterStep * kRegisterStep;
    uint64_t sure = sure_pieces(kRegisters, regs, kRegisterStep);
    if (attr.sharedSizeBytes > 0) {
        const uint64_t pieces = sure_pieces((uint64_t)lds, (uint64_t)attr.sharedSizeBytes, 1);
        sure = pieces < sure ? pieces : sure;
    }
    if (sure > (uint64_t)per_cu) sure = (uint64_t)per_cu;
    const uint64_t whole = sure * (uint64_t)cus;
    if (2 * blocks > (uint64_t)per_cu * (uint64_t)cus || blocks > whole) return 0;
    return (uint32_t)((blocks * kWholeDevice + whole - 1) / whole);
}

}  // namespace
}  // namespace dsq
