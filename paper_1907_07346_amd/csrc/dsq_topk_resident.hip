// Small problems of the sparsifying operators of libdsq (gfx950): a whole step of Algorithm 1 in one launch, xh and v in
// registers from the only read of x, g and delta to the only write of x and delta (see dsq_resident.h for the meetings).
//
// Top-k:
//   collect   xh, v; the keys (magnitudes) of the chunk that reach the row's guess `tlo` of the threshold, in column order
//             -> LDS and scratch; a count of them by their distance from tlo -> the row's window in device memory
//   meeting   (may part)
//   select    every workgroup of a row finds the window's bin that holds the threshold and looks the bin's few keys up
//             among the row's collected ones: the exact threshold tau and the ties that belong to the set, with no second
//             exchange.  If the guess caught too few or too many, and where k is too large for the keys to be exchanged,
//             the workgroups of the row run a radix select instead: 11 + 10 + 10 bits, LDS histograms added up in
//             device memory, a row meeting per level and one more for the chunks' counts
//   emit      the chunk's pairs, in column order -> scratch
//   meeting
//   finish    the neighbours' pairs of the chunk are added up in LDS: delta = v - C[v], x = xh + eta sum_j a_ij C[v_j];
//             the chunk's own pairs go to their place in the message, which follows from the counts of the chunks before
//
// With two or three workgroups on a compute unit a wave issues an instruction every 8 to 12 cycles, so 1000 of them are
// 4 to 5 us: what bounds the kernel, next to the meetings and four round trips to memory, is the number of instructions.
// Gathering all the row's keys in LDS and a histogram over them in every workgroup took 10 us, and records per thread
// (which of its sixteen columns a neighbour sends) instead of the LDS sum 11 us, where the present forms take
// 4.4 and 3.7.  8 workers x 272,474 parameters, k = 1 %: the kernel 22 us (load 3.8, collect 2, the meetings 2 each), the loop
// with the state complete after every step 26, and 61 in the fourteen launches it takes otherwise.
#include <new>

#include "dsq_internal.h"
#include "dsq_resident.h"
#include "dsq_topk_common.h"

namespace dsq {

namespace {

constexpr uint32_t RS_SLOT = 128;                             // collected keys of a chunk that are exchanged: two per lane
constexpr uint32_t RS_WINDOW = 2048;                          // bins of the window above tlo
constexpr uint32_t RS_INSIDE = 64;                            // keys of one bin that are looked up: a lane for each
constexpr uint32_t RS_MAX_CHUNKS = 1024;                      // chunks per row: four per thread
constexpr int RS_AHEAD = 18;                                  // chunks whose keys a wave asks for together
constexpr int RS_WAVES = kResThreads / 64;
constexpr int RS_LEVELS = 3;
constexpr int RS_LEVEL_BINS = 2048;

struct SparseScratch {
    TopkRow* rows;                // n
    uint32_t* meetings;           // two meetings of all workgroups (dsq_resident.h) ...
    unsigned long long* epoch;    // ... and the number of launches so far
    uint32_t* reach;              // n x nchunks: keys of the chunk that reach tlo
    uint32_t* keys;               // n x nchunks x RS_SLOT: the keys, if they are that few
    uint32_t* window;             // n x RS_WINDOW: keys per bin of 2^shift above tlo; zero between launches
    uint32_t* split;              // n x nchunks: radix select: keys equal to the threshold
    uint32_t* row_arrivals;       // n x kMeetLine: row meetings, counted and never cleared
    uint32_t* row_hist;           // n x RS_LEVELS x RS_LEVEL_BINS, zero between launches
    uint32_t* sent;               // n x nchunks: pairs of the chunk ...
    uint64_t* pairs;              // n x nchunks x kResChunk: ... (column in the chunk | value << 32), in column order
    double* csum;                 // GSpar: n x nchunks tree sums of |v| over the chunks
    uint32_t* overflow;           // GSpar: set once a row kept more than its message holds
    uint32_t nchunks;
    uint32_t expected;            // workgroups the first meeting waits for: all, and without patience one more than there are,
                                  // so that it is called off whichever way they arrive (tests of what follows)
    uint32_t gather;              // 1: keys are exchanged; 0: the radix select is always taken
    uint32_t deep;                // 1: two pairs of a neighbour per thread are asked for together, not one
};

struct SparseLaunch {             // the kernel's one argument
    TopkArgs a;
    SparseScratch s;
    uint64_t patience;            // of the first meeting
};

struct SparseShared {
    union {
        float acc[kResChunk];                                 // finish()
        uint32_t level[RS_LEVEL_BINS];                        // radix select
        struct {
            uint16_t reach[RS_MAX_CHUNKS];                    // select_gathered()
            uint32_t key[RS_INSIDE], chunk[RS_INSIDE];
        };
    };
    uint2 mine[RS_SLOT];                                      // the chunk's collected elements: column in the chunk, value
    uint32_t own[kResChunk / 32];                             // columns this worker sends
    uint32_t wave_a[RS_WAVES], wave_b[RS_WAVES];
    double sweep[kResIters * RS_WAVES];                       // GSpar
    uint32_t res[4];
    uint32_t listed;
};

// The same in all threads, which the compiler is told here: a scalar branch keeps nothing of its other side in registers.
__device__ __forceinline__ bool uniform(bool b) { return __builtin_amdgcn_readfirstlane(b ? 1 : 0) != 0; }

// The sum over the workgroup, in every thread; `slot` is free again after the caller's next barrier.
__device__ __forceinline__ uint32_t group_sum_u32(uint32_t v, uint32_t* slot) {
    const uint32_t s = wave_sum_u32(v);
    if ((threadIdx.x & 63) == 0) slot[threadIdx.x >> 6] = s;
    __syncthreads();
    uint32_t tot = 0;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) tot += slot[w];
    return tot;
}

struct SparseResident : ResidentChunk<TopkArgs> {
    using Chunk = ResidentChunk<TopkArgs>;
    const SparseScratch& s;
    SparseShared& sh;

    __device__ __forceinline__ SparseResident(const TopkArgs& a_, const SparseScratch& s_, SparseShared& sh_) : Chunk(a_, s_.nchunks), s(s_), sh(sh_) {}

    __device__ __forceinline__ float value(int it, int c) const { return c == 0 ? v[it].x : c == 1 ? v[it].y : c == 2 ? v[it].z : v[it].w; }

    // The sixteen columns of a thread as bits 4 it + c: those that exist ...
    __device__ __forceinline__ uint32_t existing() const {
        const uint32_t left = (uint32_t)a.N - chunk * (uint32_t)kResChunk;        // columns from the chunk's first on
        if (left >= (uint32_t)kResChunk) return 0xFFFFu;                          // uniform
        uint32_t m = 0;
        const uint32_t thread = Chunk::thread_here();
#pragma unroll
        for (int it = 0; it < kResIters; ++it)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if ((uint32_t)it * (4 * kResThreads) + 4u * thread + (uint32_t)c < left) m |= 1u << (4 * it + c);
        return m;
    }
    // ... and those of them for which `f(key)` holds.
    template <typename F>
    __device__ __forceinline__ uint32_t mask_of(F f) const {
        uint32_t m = 0;
#pragma unroll
        for (int it = 0; it < kResIters; ++it)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                uint32_t key;                                 // key_of(), worked out anew in every walk: sixteen registers fewer
                asm volatile("v_and_b32 %0, 0x7fffffff, %1" : "=v"(key) : "v"(value(it, c)));
                if (f(key)) m |= 1u << (4 * it + c);
            }
        return m & existing();
    }
    // Calls f(bit number) for the set bits of a mask; the sixteen tests are made here and not kept from another walk
    // (as lane masks they would take 32 scalar registers).
    template <typename F>
    static __device__ __forceinline__ void for_bits(uint32_t mask, F f) {
        asm volatile("" : "+v"(mask));
#pragma unroll
        for (int b = 0; b < 16; ++b)
            if (mask & (1u << b)) f(b);
    }

    // The column of bit b inside the chunk.
    static __device__ __forceinline__ uint32_t offset_of(int b, uint32_t thread) { return (uint32_t)(b >> 2) * (4 * kResThreads) + 4u * thread + (uint32_t)(b & 3); }

    // Where the set bits of the workgroup's masks stand in column order: the four quads of a thread lie 1024 columns apart.
    struct Ranks {
        uint32_t before[kResIters];                           // set bits in front of this thread's quad `it`
        uint32_t total;
    };
    __device__ __forceinline__ Ranks ranks(uint32_t mask) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const uint32_t lo = (uint32_t)__popc(mask & 0xFu) | (uint32_t)__popc(mask & 0xF0u) << 16;       // at most 1024 in a workgroup
        const uint32_t hi = (uint32_t)__popc(mask & 0xF00u) | (uint32_t)__popc(mask & 0xF000u) << 16;
        const uint32_t ilo = wave_inclusive_u32(lo), ihi = wave_inclusive_u32(hi);
        __syncthreads();                                      // the words may still be read
        if (lane == 63) { sh.wave_a[wave] = ilo; sh.wave_b[wave] = ihi; }
        __syncthreads();
        uint32_t blo = ilo - lo, bhi = ihi - hi, tlo = 0, thi = 0;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) {
            if (w < wave) { blo += sh.wave_a[w]; bhi += sh.wave_b[w]; }
            tlo += sh.wave_a[w];
            thi += sh.wave_b[w];
        }
        Ranks r;
        uint32_t run = 0;
        r.before[0] = blo & 0xFFFFu;
        run += tlo & 0xFFFFu;
        r.before[1] = run + (blo >> 16);
        run += tlo >> 16;
        r.before[2] = run + (bhi & 0xFFFFu);
        run += thi & 0xFFFFu;
        r.before[3] = run + (bhi >> 16);
        run += thi >> 16;
        r.total = run;
        return r;
    }

    // Only the first `allowed` of the workgroup's set bits, in column order.
    __device__ __forceinline__ uint32_t first_bits(uint32_t mask, uint32_t allowed) {
        Ranks r = ranks(mask);
        uint32_t kept = 0;
        for_bits(mask, [&](int b) {
            if (r.before[b >> 2]++ < allowed) kept |= 1u << b;
        });
        return kept;
    }

    // The chunk's pairs for everybody: the elements of the mask in column order.
    __device__ __forceinline__ void emit_mask(uint32_t mask) {
        Ranks r = ranks(mask);
        uint64_t* out = s.pairs + place() * kResChunk;
        const uint32_t thread = Chunk::thread_here();
        for_bits(mask, [&](int b) {
            agent_store(out + r.before[b >> 2]++, (uint64_t)offset_of(b, thread) | (uint64_t)__float_as_uint(value(b >> 2, b & 3)) << 32);
        });
        if (threadIdx.x == 0) agent_store(s.sent + place(), r.total);
    }

    // What the neighbours send of the chunk, weighted and added up in LDS, the columns this worker sends, and the message.
    // CAPPED (GSpar): a row's message holds `cap` pairs behind its header, what a row keeps beyond them is not sent; returns
    // the pairs this row keeps.
    template <bool CAPPED>
    __device__ __forceinline__ uint32_t sum_neighbours(uint32_t cap) {
        static_assert(RS_WAVES == kResNear, "a wave per neighbour");
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const size_t row0 = (size_t)row * nchunks;
        uint32_t ahead = 0, kept = 0;                         // pairs of the row in the chunks before this one, and in all
        if constexpr (!CAPPED)
            for (uint32_t c = threadIdx.x; c < chunk; c += kResThreads) ahead += agent_load(s.sent + row0 + c);
        uint64_t* out = reinterpret_cast<uint64_t*>(a.msg + (uint64_t)row * a.k * 8) + (CAPPED ? 1 : 0);
        const uint32_t col0 = chunk * (uint32_t)kResChunk;
        bool cleared = false;
        for (int eb = e0; eb < e1; eb += kResNear) {          // ascending neighbour index, own index included
            uint64_t pair[kResNear], next[kResNear] = {};
            uint32_t count[kResNear];
            int nbs[kResNear];
#pragma unroll
            for (int u = 0; u < kResNear; ++u) {              // a pair per thread of each, or two, whether there are that many or not
                nbs[u] = eb == e0 ? near[u] : eb + u < e1 ? a.col[eb + u] : row;
                const size_t at = (size_t)nbs[u] * nchunks + chunk;
                count[u] = agent_load(s.sent + at);
                pair[u] = agent_load(s.pairs + at * kResChunk + threadIdx.x);
                if (s.deep) next[u] = agent_load(s.pairs + at * kResChunk + kResThreads + threadIdx.x);
            }
            if constexpr (CAPPED) {
                const int nb = wave == 0 ? nbs[0] : wave == 1 ? nbs[1] : wave == 2 ? nbs[2] : nbs[3];
                uint32_t before = 0, all = 0;
                for (uint32_t c = lane; c < nchunks; c += 64) {
                    const uint32_t one = agent_load(s.sent + (size_t)nb * nchunks + c);
                    before += c < chunk ? one : 0u;
                    all += one;
                }
                before = wave_sum_u32(before);
                all = wave_sum_u32(all);
                __syncthreads();                              // the words may still be read
                if (lane == 0) { sh.wave_a[wave] = before; sh.wave_b[wave] = all; }
            }
            if (!cleared) {                                   // uniform
                if constexpr (!CAPPED) __syncthreads();       // the words may still be read
#pragma unroll
                for (int it = 0; it < kResIters; ++it) reinterpret_cast<float4*>(sh.acc)[it * kResThreads + threadIdx.x] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (threadIdx.x < kResChunk / 32) sh.own[threadIdx.x] = 0u;
                if constexpr (!CAPPED) ahead = group_sum_u32(ahead, sh.wave_a);   // (its barrier)
            }
            if constexpr (CAPPED) __syncthreads();
            cleared = true;
#pragma unroll
            for (int u = 0; u < kResNear; ++u) {
                if (eb + u < e1) {                            // uniform
                    const float w = eb == e0 ? near_coef[u] : a.coef[eb + u];
                    const bool own = nbs[u] == row;
                    uint32_t n = count[u];
                    if constexpr (CAPPED) {
                        const uint32_t before = sh.wave_a[u], all = sh.wave_b[u];
                        if (own) { ahead = before; kept = all; }
                        if (all > cap) {
                            const uint32_t room = before < cap ? cap - before : 0u;
                            n = n < room ? n : room;
                        }
                    }
                    auto add = [&](uint32_t p, uint64_t one) {
                        const uint32_t q = (uint32_t)one & (uint32_t)(kResChunk - 1);
                        sh.acc[q] = fmaf(w, __uint_as_float((uint32_t)(one >> 32)), sh.acc[q]);
                        if (own) {
                            atomicOr(&sh.own[q >> 5], 1u << (q & 31));
                            out[ahead + p] = one + col0;      // the column's word does not overflow: N < 2^22
                        }
                    };
                    if (threadIdx.x < n) add(threadIdx.x, pair[u]);
                    const uint32_t held = s.deep ? 2u * kResThreads : (uint32_t)kResThreads;
                    if (s.deep && threadIdx.x + kResThreads < n) add(threadIdx.x + kResThreads, next[u]);
                    if (__builtin_amdgcn_readfirstlane(n) > held) {
                        const uint64_t* from = s.pairs + ((size_t)nbs[u] * nchunks + chunk) * kResChunk;
                        for (uint32_t p = threadIdx.x + held; p < n; p += kResThreads) add(p, agent_load(from + p));
                    }
                    __syncthreads();
                }
            }
        }
        return kept;
    }

    // Lines 6 and 9, after sum_neighbours().
    __device__ __forceinline__ void finish() {
        const uint32_t thread = Chunk::thread_here();
#pragma unroll
        for (int it = 0; it < kResIters; ++it) {
            const float4 sum = reinterpret_cast<const float4*>(sh.acc)[(uint32_t)it * kResThreads + thread];
            const uint32_t sent = sh.own[(uint32_t)it * (kResThreads / 8) + (thread >> 3)] >> (4u * (thread & 7u));
            xh[it].x = fmaf(a.eta, sum.x, xh[it].x + 0.f); xh[it].y = fmaf(a.eta, sum.y, xh[it].y + 0.f);
            xh[it].z = fmaf(a.eta, sum.z, xh[it].z + 0.f); xh[it].w = fmaf(a.eta, sum.w, xh[it].w + 0.f);
            if (sent & 1u) v[it].x = 0.f;                     // delta = v - C[v] = 0 where v was sent
            if (sent & 2u) v[it].y = 0.f;
            if (sent & 4u) v[it].z = 0.f;
            if (sent & 8u) v[it].w = 0.f;
            Chunk::store(it, thread);
        }
    }

    // ---- the whole step by one workgroup, after parting: column by column, with few registers (inlined next to the
    // registers of the usual way, more of them made the kernel spill 150) -----------------------------------------
    __device__ __forceinline__ float model_at(uint64_t j) const { return fmaf(-a.gamma, a.g[(uint64_t)row * a.g_ld + j], a.x[(uint64_t)row * a.ld + j]); }
    __device__ __forceinline__ float value_at(uint64_t j) const { return model_at(j) + a.delta[(uint64_t)row * a.ld + j]; }

    // The number of threads before this one for which `b` holds; *total: of all.
    __device__ __forceinline__ uint32_t rank_of(bool b, uint32_t* total) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const unsigned long long m = __ballot(b);
        __syncthreads();                                      // the words may still be read
        if (lane == 0) sh.wave_a[wave] = (uint32_t)__popcll(m);
        __syncthreads();
        uint32_t before = (uint32_t)__popcll(m & ((1ull << lane) - 1ull)), all = 0;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) {
            if (w < wave) before += sh.wave_a[w];
            all += sh.wave_a[w];
        }
        *total = all;
        return before;
    }

    // The pairs of the chunk; send(j, v) is called for 256 columns at a time, by all threads, with j in ascending order.
    template <typename F>
    __device__ __forceinline__ void emit_alone(F send) {
        uint64_t* out = s.pairs + place() * kResChunk;
        uint32_t done = 0;
        for (uint32_t off = threadIdx.x; off < (uint32_t)kResChunk; off += kResThreads) {
            const uint64_t j = (uint64_t)chunk * kResChunk + off;
            const float val = j < a.N ? value_at(j) : 0.f;
            uint32_t total;
            const bool take = send(j, val);
            const uint32_t at = done + rank_of(take, &total);
            if (take) agent_store(out + at, (uint64_t)off | (uint64_t)__float_as_uint(val) << 32);
            done += total;
        }
        if (threadIdx.x == 0) agent_store(s.sent + place(), done);
    }

    __device__ __forceinline__ void finish_alone() {
        for (uint32_t off = threadIdx.x; off < (uint32_t)kResChunk; off += kResThreads) {
            const uint64_t j = (uint64_t)chunk * kResChunk + off;
            if (j >= a.N) break;                              // padding columns stay zero
            const float model = model_at(j), val = value_at(j);
            a.x[(uint64_t)row * a.ld + j] = fmaf(a.eta, sh.acc[off], model + 0.f);
            a.delta[(uint64_t)row * a.ld + j] = (sh.own[off >> 5] >> (off & 31u)) & 1u ? 0.f : val;
        }
    }

    // The keys of the row's chunks meet: all its workgroups are running, so every wait ends.
    __device__ __forceinline__ void meet_row(uint32_t& target) const {
        drain();
        __syncthreads();
        target += nchunks;
        if (threadIdx.x == 0) {
            uint32_t* word = s.row_arrivals + (size_t)row * kMeetLine;
            agent_add(word, 1u);
            while ((int32_t)(agent_load(word) - target) < 0) __builtin_amdgcn_s_sleep(1);
        }
        __syncthreads();
    }

    // The bin where the count from the top crosses `need` (1 <= need <= the sum of all bins); res: [0] the bin, [1] how many
    // to take inside it, [2] elements in it.
    template <int NB>
    __device__ __forceinline__ void find_bin(const uint32_t* h, uint32_t need) {
        constexpr int PER = NB / kResThreads;
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        uint32_t mine[PER], sum = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            mine[q] = h[NB - 1 - ((int)threadIdx.x * PER + q)];
            sum += mine[q];
        }
        const uint32_t inc = wave_inclusive_u32(sum);
        if (lane == 63) sh.wave_a[wave] = inc;
        __syncthreads();
        uint32_t above = inc - sum;
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w)
            if (w < wave) above += sh.wave_a[w];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            if (above < need && need <= above + mine[q]) {
                sh.res[0] = (uint32_t)(NB - 1 - ((int)threadIdx.x * PER + q));
                sh.res[1] = need - above;
                sh.res[2] = mine[q];
            }
            above += mine[q];
        }
        __syncthreads();
    }
};

struct TopkResident : SparseResident {
    using SparseResident::SparseResident;
    uint32_t tlo = 0, shift = 0, row_target = 0;              // read before the first meeting, replaced after it
    uint32_t tau = 0, r_tie = 0;
    uint32_t eq_before = 0;                                   // keys equal to tau in the row's chunks before this one
    uint32_t collected = 0;                                   // keys of the row that reached tlo
    uint32_t here = 0;                                        // ... and of this chunk
    uint32_t tied = 0, tau_old = 0;                           // the last step's threshold had many equal keys; the threshold
    uint32_t equal = 0;                                       // keys of the row that equal tau, as far as known
    bool radix = false;

    // Asked for ahead of the state itself.
    __device__ __forceinline__ void expect(uint32_t which) {
        const uint32_t r = which / nchunks;
        tlo = s.rows[r].tlo;
        shift = s.rows[r].shift;
        tied = s.rows[r].tied;
        tau_old = s.rows[r].tau_prev;
        row_target = agent_load(s.row_arrivals + (size_t)r * kMeetLine);     // no row meets before all have read it
    }

    __device__ __forceinline__ void collect() {
        if (tied != 0u) { publish_split(tau_old); return; }  // uniform over the row
        const uint32_t mask = mask_of([&](uint32_t key) { return key >= tlo; });
        Ranks r = ranks(mask);
        here = __builtin_amdgcn_readfirstlane(r.total);
        if (s.gather != 0u && here <= RS_SLOT) {              // uniform
            const uint32_t thread = Chunk::thread_here();
            for_bits(mask, [&](int b) { sh.mine[r.before[b >> 2]++] = make_uint2(offset_of(b, thread), __float_as_uint(value(b >> 2, b & 3))); });
            __syncthreads();
            if (threadIdx.x < here) {
                const uint32_t key = sh.mine[threadIdx.x].y & 0x7FFFFFFFu, bin = (key - tlo) >> shift;
                agent_store(s.keys + place() * RS_SLOT + threadIdx.x, key);
                if (bin < RS_WINDOW) agent_add(s.window + (size_t)row * RS_WINDOW + bin, 1u);
            }
        }
        if (threadIdx.x == 0) agent_store(s.reach + place(), here);
    }

    // The threshold from the row's collected keys; false if they do not hold it or are not all there.  All workgroups of a
    // row see the same numbers, so they all take the same way.
    __device__ __forceinline__ bool select_gathered() {
        if (tied != 0u) return false;
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const size_t first = (size_t)row * nchunks;
        const bool guessed = s.gather != 0u && tlo != 0xFFFFFFFFu;               // uniform
        const uint32_t per = (nchunks + kResThreads - 1) / kResThreads;           // chunks per thread, at most 4
        uint32_t cnt[4];
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t c = per * threadIdx.x + q;
            cnt[q] = (q < per && c < nchunks) ? agent_load(s.reach + first + c) : 0u;
        }
        // eight bins of the window and two keys of each of RS_AHEAD chunks per lane, asked for before the counts are needed
        constexpr int BINS = RS_WINDOW / kResThreads;
        uint64_t bins[BINS / 2] = {}, two[RS_AHEAD] = {};
        auto ask = [&](uint32_t c0) {
#pragma unroll
            for (int b = 0; b < RS_AHEAD; ++b) {
                const uint32_t c = c0 + (uint32_t)(RS_WAVES * b);
                if (c < nchunks) two[b] = agent_load(reinterpret_cast<const uint64_t*>(s.keys + (first + c) * RS_SLOT) + lane);
            }
        };
        if (guessed) {
#pragma unroll
            for (int q = 0; q < BINS / 2; ++q) bins[q] = agent_load(reinterpret_cast<const uint64_t*>(s.window + (size_t)row * RS_WINDOW) + threadIdx.x * (BINS / 2) + q);
            ask((uint32_t)wave);
        }
        uint32_t sum = 0, most = 0, binned = 0;
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) { sum += cnt[q]; most = cnt[q] > most ? cnt[q] : most; }
#pragma unroll
        for (int q = 0; q < BINS / 2; ++q) binned += (uint32_t)bins[q] + (uint32_t)(bins[q] >> 32);
        sum = wave_sum_u32(sum) | (__any(most > RS_SLOT) ? 0x80000000u : 0u);     // the sum is below 2^23
        const uint32_t inc = wave_inclusive_u32(binned);
        __syncthreads();                                      // the words may still be read from collect()
        if (lane == 63) { sh.wave_a[wave] = sum; sh.wave_b[wave] = inc; }
        if (threadIdx.x == 0) { sh.listed = 0u; sh.res[2] = 0u; }
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
            if (q < per && per * threadIdx.x + q < nchunks) sh.reach[per * threadIdx.x + q] = (uint16_t)cnt[q];
        __syncthreads();
        collected = 0;
        uint32_t over = 0, below = inc - binned;              // keys in the bins below this thread's
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) {
            if (w < wave) below += sh.wave_b[w];
            over |= sh.wave_a[w] >> 31;
            collected += sh.wave_a[w] & 0x7FFFFFFFu;
        }
        collected = __builtin_amdgcn_readfirstlane(collected);
        const uint32_t k = (uint32_t)a.k;
        if (!guessed || __builtin_amdgcn_readfirstlane(over) != 0u || collected < k) return false;   // uniform over the row
        const uint32_t unsent = collected - k;                // collected keys below the threshold: the bin where the count passes it
        if (below <= unsent && unsent < below + binned) {
#pragma unroll
            for (int q = 0; q < BINS; ++q) {
                const uint32_t n = (uint32_t)(bins[q / 2] >> (32 * (q & 1)));
                if (below <= unsent && unsent < below + n) {
                    sh.res[0] = threadIdx.x * BINS + (uint32_t)q;
                    sh.res[1] = below + n - unsent;           // how many to take inside it
                    sh.res[2] = n;
                }
                below += n;
            }
        }
        __syncthreads();
        const uint32_t inside = __builtin_amdgcn_readfirstlane(sh.res[2]), need = sh.res[1];
        if (inside == 0u || inside > RS_INSIDE) return false; // beyond the window; more equal keys than are looked up
        const uint32_t lo = tlo + (sh.res[0] << shift), span = 1u << shift;
        for (uint32_t c0 = (uint32_t)wave;;) {
#pragma unroll
            for (int b = 0; b < RS_AHEAD; ++b) {
                const uint32_t c = c0 + (uint32_t)(RS_WAVES * b);
                if (c < nchunks) {                            // uniform
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const uint32_t key = (uint32_t)(two[b] >> (32 * half));
                        if (key - lo < span && (uint32_t)(2 * lane + half) < sh.reach[c]) {
                            const uint32_t at = atomicAdd(&sh.listed, 1u);
                            sh.key[at] = key;
                            sh.chunk[at] = c;
                        }
                    }
                }
            }
            c0 += (uint32_t)(RS_WAVES * RS_AHEAD);
            if (c0 >= nchunks) break;
            ask(c0);
        }
        __syncthreads();
        // every wave for itself: a lane per key of the bin
        const uint32_t key = (uint32_t)lane < inside ? sh.key[lane] : 0u;
        uint32_t gt = 0, eq = 0;
        for (uint32_t q = 0; q < inside; ++q) {
            const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)key, (int)q);
            gt += other > key;
            eq += other == key;
        }
        const bool hit = (uint32_t)lane < inside && gt < need && need <= gt + eq;            // all keys equal to tau
        const unsigned long long hits = __ballot(hit);
        const int at = __ffsll((long long)hits) - 1;
        tau = (uint32_t)__builtin_amdgcn_readlane((int)key, at);
        r_tie = need - (uint32_t)__builtin_amdgcn_readlane((int)gt, at);
        eq_before = (uint32_t)__popcll(__ballot(hit && sh.chunk[lane] < chunk));
        return true;
    }

    // The collected elements that are sent; two of them per lane of one wave, in column order.
    __device__ __forceinline__ void emit_gathered() {
        if (threadIdx.x >= 64) return;
        const int lane = threadIdx.x;
        const unsigned long long below = (1ull << lane) - 1ull;
        uint64_t* out = s.pairs + place() * kResChunk;
        uint32_t done = 0, ties = eq_before;
#pragma unroll
        for (int half = 0; half < (int)RS_SLOT / 64; ++half) {
            const uint32_t p = 64u * half + lane;
            const uint2 e = sh.mine[p];
            const uint32_t key = p < here ? e.y & 0x7FFFFFFFu : 0u;
            const unsigned long long tied = __ballot(p < here && key == tau);
            const bool send = p < here && (key > tau || (key == tau && ties + (uint32_t)__popcll(tied & below) < r_tie));
            const unsigned long long m = __ballot(send);
            if (send) agent_store(out + done + (uint32_t)__popcll(m & below), (uint64_t)e.x | (uint64_t)e.y << 32);
            done += (uint32_t)__popcll(m);
            ties += (uint32_t)__popcll(tied);
        }
        if (lane == 0) agent_store(s.sent + place(), done);
    }

    static __device__ __forceinline__ constexpr int level_shift(int l) { return l == 0 ? 20 : l == 1 ? 10 : 0; }
    __device__ __forceinline__ void clear_level() {
        __syncthreads();
        for (int b = threadIdx.x; b < RS_LEVEL_BINS; b += kResThreads) sh.level[b] = 0u;
        __syncthreads();
    }
    __device__ __forceinline__ void add_level(int l, uint32_t prefix) {
        const int shift = level_shift(l);
        const uint32_t bins = l == 0 ? 2048u : 1024u;
        for_bits(existing(), [&](int b) {
            const uint32_t key = key_of(value(b >> 2, b & 3));
            if (l == 0 || (key >> (shift + 10)) == prefix) atomicAdd(&sh.level[(key >> shift) & (bins - 1u)], 1u);
        });
    }
    __device__ __forceinline__ void find_level(int l, uint32_t& prefix, uint32_t& need) {
        find_bin<RS_LEVEL_BINS>(sh.level, need);              // the upper half is empty from level 1 on
        prefix = l == 0 ? sh.res[0] : prefix << 10 | sh.res[0];
        need = sh.res[1];
    }
    // Keys of the chunk above and equal to t.
    __device__ __forceinline__ void publish_split(uint32_t t) {
        const uint32_t gt = (uint32_t)__popc(mask_of([&](uint32_t key) { return key > t; }));
        const uint32_t eq = (uint32_t)__popc(mask_of([&](uint32_t key) { return key == t; }));
        __syncthreads();
        const uint32_t both = group_sum_u32(eq | gt << 16, sh.wave_a);           // at most 4096 of each
        if (threadIdx.x == 0) agent_store(s.split + place(), both);
    }
    // ... of all chunks: keys above (in the row), equal (in the row), equal in the chunks before this one.
    __device__ __forceinline__ uint32_t gather_split() {
        uint32_t gt = 0, eq = 0, before = 0;
        for (uint32_t c = threadIdx.x; c < nchunks; c += kResThreads) {
            const uint32_t both = agent_load(s.split + (size_t)row * nchunks + c);
            gt += both >> 16;
            eq += both & 0xFFFFu;
            before += c < chunk ? both & 0xFFFFu : 0u;
        }
        __syncthreads();
        gt = group_sum_u32(gt, sh.wave_a);
        equal = group_sum_u32(eq, sh.wave_b);
        __syncthreads();
        eq_before = group_sum_u32(before, sh.wave_a);
        return gt;
    }

    // Many equal keys at the threshold (columns that are all zero, saturated values): the threshold is often the one of the
    // step before, which the chunks' counts tell at once.  Else these rows go through the radix select.
    __device__ __forceinline__ bool select_tied() {
        if (tied == 0u) return false;
        const uint32_t k = (uint32_t)a.k, gt = gather_split();
        if (!(gt < k && k <= gt + equal)) return false;
        tau = tau_old;
        r_tie = k - gt;
        return true;
    }

    // Exact for any k and any values: every workgroup of the row takes part.
    __device__ __forceinline__ void select_radix() {
        uint32_t prefix = 0, need = (uint32_t)a.k;
        radix = true;
        for (int l = 0; l < RS_LEVELS; ++l) {
            uint32_t* hist = s.row_hist + ((size_t)row * RS_LEVELS + l) * RS_LEVEL_BINS;
            const int bins = l == 0 ? 2048 : 1024;
            clear_level();
            add_level(l, prefix);
            __syncthreads();
            for (int b = threadIdx.x; b < bins; b += kResThreads)
                if (sh.level[b]) agent_add(hist + b, sh.level[b]);
            meet_row(row_target);
            for (int b = threadIdx.x; b < bins; b += kResThreads) sh.level[b] = agent_load(hist + b);
            __syncthreads();
            find_level(l, prefix, need);
        }
        tau = prefix;
        r_tie = need;
        equal = sh.res[2];
        eq_before = 0;
        if (__builtin_amdgcn_readfirstlane(equal) == need) return;   // all of them are sent
        publish_split(tau);
        meet_row(row_target);
        (void)gather_split();
    }

    __device__ __forceinline__ void select_alone() {
        uint32_t prefix = 0, need = (uint32_t)a.k;
        for (int l = 0; l < RS_LEVELS; ++l) {
            clear_level();
            for (uint64_t j = threadIdx.x; j < a.N; j += kResThreads) {
                const uint32_t key = key_of(value_at(j));
                if (l == 0 || (key >> (level_shift(l) + 10)) == prefix) atomicAdd(&sh.level[(key >> level_shift(l)) & (l == 0 ? 2047u : 1023u)], 1u);
            }
            __syncthreads();
            find_level(l, prefix, need);
        }
        tau = prefix;
        r_tie = need;
    }
    __device__ __forceinline__ void step_alone(uint32_t blocks) {
        uint32_t ties = 0;                                    // in the row so far
        for (uint32_t i = 0; i < blocks; ++i) {
            locate(i);
            if (chunk == 0) {
                select_alone();
                tlo = s.rows[row].tlo;
                keep_book(true);
                clear_counts();
                ties = 0;
            }
            emit_alone([&](uint64_t j, float val) {
                const bool in = j < a.N, tied = in && key_of(val) == tau;
                uint32_t total;
                const uint32_t rank = ties + rank_of(tied, &total);
                ties += total;
                return (in && key_of(val) > tau) || (tied && rank < r_tie);
            });
        }
        phase_end();
        for (uint32_t i = 0; i < blocks; ++i) {
            locate(i);
            (void)sum_neighbours<false>(0);
            finish_alone();
        }
    }

    __device__ __forceinline__ void emit_masked() {
        uint32_t mask = mask_of([&](uint32_t key) { return key > tau; });
        const uint32_t ties = mask_of([&](uint32_t key) { return key == tau; });
        const uint32_t quota = r_tie > eq_before ? r_tie - eq_before : 0u;        // ties of this chunk that belong to the set
        if (__syncthreads_or(ties != 0u)) mask |= first_bits(ties, quota);
        emit_mask(mask);
    }

    // The guess of the next step.  exact: a radix select found the threshold, not the keys counted while v was formed.
    __device__ __forceinline__ void keep_book(bool exact) {
        if (chunk != 0 || threadIdx.x != 0) return;
        TopkRow r = s.rows[row];
        r.tau = tau;
        r.r_tie = r_tie;
        r.total = (uint32_t)a.k;
        r.tlo_used = tlo;
        r.cand_total = collected;
        // the number of keys above tlo is exact, whether they could be gathered or not: it always serves the next guess
        r.cand_mode = (tlo != 0xFFFFFFFFu && collected >= (uint32_t)a.k) ? 1u : 0u;
        r.tlo = next_candidate_threshold(r, tau, (uint32_t)a.k);
        r.cand_mode = exact ? 0u : 1u;                        // from here on what ds_topk_candidate_rows reports
        r.tied = equal > RS_INSIDE ? 1u : 0u;
        // the forecast lies in the window's second quarter or so: 512 to 1023 bins above tlo
        const uint32_t dist = r.forecast > r.tlo ? r.forecast - r.tlo : 1u;
        r.shift = dist >= 1024u ? 22u - (uint32_t)__clz((int)dist) : 0u;
        r.tau_prev = tau;
        s.rows[row] = r;
    }

    // The row's counts are zero again for the next launch (all its workgroups are done with them).
    __device__ __forceinline__ void clear_counts() const {
        if (chunk != 0) return;
        if (s.gather != 0u)
            for (uint32_t b = threadIdx.x; b < RS_WINDOW; b += kResThreads) agent_store(s.window + (size_t)row * RS_WINDOW + b, 0u);
        if (!radix) return;
        for (int b = threadIdx.x; b < RS_LEVELS * RS_LEVEL_BINS; b += kResThreads) agent_store(s.row_hist + (size_t)row * RS_LEVELS * RS_LEVEL_BINS + b, 0u);
    }
};

__global__ void __launch_bounds__(kResThreads, 5) topk_resident(SparseLaunch launch) {
    __shared__ SparseShared sh;
    const TopkArgs& a = launch.a;
    const SparseScratch& s = launch.s;
    const uint32_t blocks = gridDim.x;
    const unsigned long long epoch = *s.epoch;
    TopkResident op(a, s, sh);
    op.expect(blockIdx.x);
    op.load(blockIdx.x);
    op.collect();
    if (!uniform(meet<true, false>(s.meetings, s.expected, epoch, launch.patience))) {
        if (!uniform(leave(a.t_ptr, blocks))) return;
        op.step_alone(blocks);
        close_alone(s.meetings, 2, blocks, epoch, s.epoch, a.t_ptr);
        return;
    }
    if (uniform(op.select_gathered())) {
        op.emit_gathered();
    } else {
        if (!uniform(op.select_tied())) op.select_radix();
        op.emit_masked();
    }
    op.keep_book(op.radix);
    (void)meet<false, true>(s.meetings + kMeetWords, blocks, epoch, 0, s.epoch, a.t_ptr);
    (void)op.sum_neighbours<false>(0);
    op.finish();
    op.clear_counts();
}

// GSpar:
//   measure   xh, v; the chunk's sum of |v|                                                        -> scratch
//   meeting   (may part)
//   mark      every workgroup of a row puts lambda = k / sum |v| together for itself; the chunk's kept elements, in column
//             order                                                                                -> scratch
//   meeting
//   finish    as for top-k; the message's header and the zeros behind it by the workgroups of chunk 0
// 8 workers x 272,474 parameters, 10 % kept, the state complete after every step: 25.2 us (kernel 25.2 under the profiler); the eight launches it
// takes otherwise: 47 us.
struct GsparResident : SparseResident {
    using SparseResident::SparseResident;
    uint32_t t_lo = 0;                                        // the step's counter, read before it is advanced
    float lambda = 0.f;

    __device__ __forceinline__ uint32_t room() const { return (uint32_t)a.k - 1u; }   // pairs a message holds

    __device__ __forceinline__ void measure() {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int it = 0; it < kResIters; ++it) {              // padding columns hold v = 0
            const double sw = wave_tree_f64(((double)fabsf(v[it].x) + (double)fabsf(v[it].y)) + ((double)fabsf(v[it].z) + (double)fabsf(v[it].w)));
            if (lane == 0) sh.sweep[it * RS_WAVES + wave] = sw;   // sweep index = column order
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            double t[kResIters * RS_WAVES];
#pragma unroll
            for (int q = 0; q < kResIters * RS_WAVES; ++q) t[q] = sh.sweep[q];
#pragma unroll
            for (int len = kResIters * RS_WAVES; len > 1; len >>= 1)
#pragma unroll
                for (int q = 0; q < len / 2; ++q) t[q] = t[2 * q] + t[2 * q + 1];
            agent_store(s.csum + place(), t[0]);
        }
    }

    // The tree continued over the row's chunks (at most 1024 of them: four leaves per thread, the missing ones zero; with
    // up to 256 of them one leaf per thread is the same tree).
    __device__ __forceinline__ void row_lambda() {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        const uint32_t per = nchunks <= (uint32_t)kResThreads ? 1u : 4u;          // uniform
        double leaf[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            const uint32_t c = per * threadIdx.x + q;
            if (q < per && c < nchunks) leaf[q] = agent_load(s.csum + (size_t)row * nchunks + c);
        }
        const double part = wave_tree_f64((leaf[0] + leaf[1]) + (leaf[2] + leaf[3]));
        __syncthreads();                                      // the words may still be read
        if (lane == 0) sh.sweep[wave] = part;
        __syncthreads();
        const double sum = (sh.sweep[0] + sh.sweep[1]) + (sh.sweep[2] + sh.sweep[3]);
        lambda = (sum > 0.0) ? (float)((double)a.k_expected / sum) : 0.f;
    }

    __device__ __forceinline__ void mark() {
        uint32_t mask = 0;
#pragma unroll
        for (int it = 0; it < kResIters; ++it) mask |= gs_keep4(a, row, column(it), t_lo, lambda, v[it]) << (4 * it);
        emit_mask(mask);
    }

    // What ds_topk_candidate_rows reports: v has stayed in registers, unless one workgroup did the step.
    __device__ __forceinline__ void keep_book(bool alone) {
        if (chunk == 0 && threadIdx.x == 0) s.rows[row].gs_mode = alone ? 0u : 1u;
    }

    // The header, and zeros behind a message shorter than the last one.
    __device__ __forceinline__ void close_message(uint32_t kept) {
        if (chunk != 0) return;                               // uniform
        const uint32_t count = kept < room() ? kept : room(), last = s.rows[row].gs_total;
        uint2* mrow = reinterpret_cast<uint2*>(a.msg + (uint64_t)row * a.k * 8);
        for (uint32_t p = count + threadIdx.x; p < last; p += kResThreads) mrow[1 + p] = make_uint2(0u, 0u);
        __syncthreads();                                      // every thread has read gs_total
        if (threadIdx.x == 0) {
            mrow[0] = make_uint2(count, 0u);
            s.rows[row].gs_total = count;
            if (kept > room()) atomicOr(s.overflow, 1u);
        }
    }

    __device__ __forceinline__ void step_alone(uint32_t blocks) {
        for (uint32_t i = 0; i < blocks; ++i) {               // every workgroup has measured before it left
            locate(i);
            if (chunk == 0) {
                row_lambda();
                keep_book(true);
            }
            emit_alone([&](uint64_t j, float val) {
                uint32_t rnd[4];
                philox4x32_10((uint32_t)(j >> 2), (uint32_t)row, t_lo, kGsparStreamTag, a.seed_lo, a.seed_hi, rnd);
                const uint32_t word = (j & 3) == 0 ? rnd[0] : (j & 3) == 1 ? rnd[1] : (j & 3) == 2 ? rnd[2] : rnd[3];
                return j < a.N && (float)(word >> 8) * (1.0f / 16777216.0f) < lambda * fabsf(val);
            });
        }
        phase_end();
        for (uint32_t i = 0; i < blocks; ++i) {
            locate(i);
            const uint32_t kept = sum_neighbours<true>(room());
            finish_alone();
            close_message(kept);
        }
    }
};

__global__ void __launch_bounds__(kResThreads, 5) gspar_resident(SparseLaunch launch) {
    __shared__ SparseShared sh;
    const TopkArgs& a = launch.a;
    const SparseScratch& s = launch.s;
    const uint32_t blocks = gridDim.x;
    const unsigned long long epoch = *s.epoch;
    GsparResident op(a, s, sh);
    op.t_lo = (uint32_t)*a.t_ptr;
    op.load(blockIdx.x);
    op.measure();
    if (!uniform(meet<true, false>(s.meetings, s.expected, epoch, launch.patience))) {
        if (!uniform(leave(a.t_ptr, blocks))) return;
        op.step_alone(blocks);
        close_alone(s.meetings, 2, blocks, epoch, s.epoch, a.t_ptr);
        return;
    }
    op.row_lambda();
    op.mark();
    op.keep_book(false);
    (void)meet<false, true>(s.meetings + kMeetWords, blocks, epoch, 0, s.epoch, a.t_ptr);
    const uint32_t kept = op.sum_neighbours<true>(op.room());
    op.finish();
    op.close_message(kept);
}
static_assert(sizeof(SparseShared) <= 31 * 1024, "five workgroups share the 160 KB of a compute unit");

}  // namespace

struct SparseResidentState {
    SparseScratch s{};
    Slab slab;                    // holds all of the scratch
    bool gspar = false;
    uint64_t patience = 0;
};

void sparse_resident_destroy(SparseResidentState* st) {
    if (!st) return;
    st->slab.drop();
    delete st;
}

uint32_t sparse_resident_share(const ds_config& cfg) {
    const uint64_t nchunks = (cfg.N + kResChunk - 1) / kResChunk, blocks = (uint64_t)cfg.n * nchunks;
    if (nchunks > RS_MAX_CHUNKS) return 0;
    return cfg.comp.kind == DS_COMP_GSPAR ? resident_share(gspar_resident, kResThreads, blocks) : resident_share(topk_resident, kResThreads, blocks);
}

ds_status sparse_resident_create(const ds_config& cfg, bool impatient, TopkRow* rows, uint32_t* overflow, SparseResidentState** out) {
    SparseResidentState* st = new (std::nothrow) SparseResidentState();
    if (!st) return DS_ENOMEM;
    st->patience = impatient ? 0 : kMeetPatience;
    SparseScratch& s = st->s;
    st->gspar = cfg.comp.kind == DS_COMP_GSPAR;
    s.rows = rows;
    s.overflow = overflow;
    s.nchunks = (uint32_t)((cfg.N + kResChunk - 1) / kResChunk);
    s.expected = (uint32_t)cfg.n * s.nchunks + (impatient ? 1u : 0u);
    const size_t n = (size_t)cfg.n, all = n * s.nchunks;
    // about 1.6 k keys are collected; a chunk's have to fit in its slot with room for an uneven row
    s.gather = cfg.comp.k * kResChunk <= cfg.N * (RS_SLOT / 2) ? 1u : 0u;
    s.deep = cfg.comp.k * kResChunk > cfg.N * (uint64_t)(kResThreads * 3 / 4) ? 1u : 0u;   // most chunks send more pairs than there are threads
    const bool ok = st->slab.make([&](Slab& m) {
        m.place(s.meetings, 2 * kMeetWords);
        m.place(s.epoch, 1);
        m.place(s.window, st->gspar ? 0 : n * RS_WINDOW);
        m.place(s.row_arrivals, st->gspar ? 0 : n * kMeetLine);
        m.place(s.row_hist, st->gspar ? 0 : n * RS_LEVELS * RS_LEVEL_BINS);
        const size_t zero = m.bytes;                          // at the first launch
        m.place(s.reach, all);
        m.place(s.split, all);
        m.place(s.sent, all);
        m.place(s.csum, st->gspar ? all : 0);
        m.place(s.keys, st->gspar ? 0 : all * RS_SLOT);
        m.place(s.pairs, all * kResChunk);
        return zero;
    });
    if (!ok) {                                                // (the caller waits for the memset)
        (void)hipGetLastError();
        sparse_resident_destroy(st);
        return DS_ENOMEM;
    }
    *out = st;
    return DS_OK;
}

ds_status sparse_resident_step(SparseResidentState* st, const TopkArgs& a, hipStream_t stream) {
    const dim3 grid(st->s.nchunks * (uint32_t)a.n), block(kResThreads);
    const SparseLaunch launch{a, st->s, st->patience};
    if (st->gspar) hipLaunchKernelGGL(gspar_resident, grid, block, 0, stream, launch);
    else           hipLaunchKernelGGL(topk_resident, grid, block, 0, stream, launch);
    return hipGetLastError() == hipSuccess ? DS_OK : DS_EHIP;
}

}  // namespace dsq
