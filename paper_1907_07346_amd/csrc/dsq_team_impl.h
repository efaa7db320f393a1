// The block compressors for more workers than one workgroup holds: the rows of a tile split over a team of workgroups.
//
// The fused tile kernel (dsq_tile_impl.h) keeps x - gamma g of all n rows of a tile in the registers of one workgroup from
// phase 1 to the gossip phase.  Where a wave would own more rows than its registers hold it forms them a second time (28 bytes
// per element instead of 20), and where there are few tiles a handful of workgroups walk through all rows one after
// the other while the rest of the chip is idle.  Here the rows of a tile are split over `parts` workgroups, which run phase 1
// on their rows, meet, fetch the codes of the neighbours that other workgroups of the team encoded from their messages, and
// finish their rows from registers: 20 bytes per element and the messages, once, for any number of rows.
//
// The meeting.  A workgroup claims its part before it stores anything, arrives when the part's messages are in memory, and waits only
// after that, for its own tile.  What it waits for is work that a running workgroup has claimed, or a part that nobody has
// claimed yet because the GPU has no room for another workgroup, whatever fills it: after `team_patience` the waiting
// workgroup claims such parts itself, with its own rows parked in x, and the workgroup that comes too late for its part leaves.
// So every wait ends even if a single workgroup at a time can run, and no launch needs the others out of the way.
#pragma once

#include "dsq_resident.h"
#include "dsq_tile_impl.h"

namespace dsq {
namespace {

constexpr uint32_t kTeamParts = 64;                          // most parts a tile is split into
// Device memory of a handle: a line with the number of launches so far, then per tile a line with the number of arrivals so far
// and, for each part, the number of the last launch that claimed it.
constexpr uint32_t kTeamLine = 32;                           // 64-bit words: 256 bytes
static_assert((kTeamParts + 1) / 2 + 1 <= 2 * kTeamLine && kTeamCellBytes == 2 * kTeamLine * sizeof(unsigned long long), "an arrival counter and the claims");
// Waves per SIMD that the registers are rationed for.  A workgroup of eight waves has two on each: three workgroups on a compute unit up to two
// sweeps, two with four, one with eight.  (No scratch but 12 bytes a thread with four rows of two sweeps and 28 with two or four rows of
// four.  Rationed for seven, which is three workgroups too, the kernels of one and two sweeps spilled half as many scalars again and took longer, us a
// step at 4 bits: 100 x 100,000, blocks of 256, 53.8 and 50.8, 256 x 262,144 269 and 263; blocks of 512, 64 x 16,384 11.7 and 10.8, 100 x 2,621 9.9
// and 10.0.)
constexpr int team_waves(int sweeps) { return sweeps <= 2 ? 6 : sweeps == 4 ? 4 : 2; }
constexpr uint32_t kNoSlot = 0xFFFFFFFFu;
// Ticks of the 100 MHz clock: 50 us, many times what a part takes.
constexpr uint64_t kTeamPatience = 5'000;

template <int KIND, int BITS, int B, int SW, int NW, int RPW>
struct Team {
    using T = Tile<KIND, BITS, B, SW, NW>;
    static constexpr int THREADS = NW * kWave;
    static constexpr int ROW_WORDS = T::ROW_CODE_BYTES / 4;
    static constexpr int BLOCK_WORDS = B * BITS / 32;

    struct __align__(16) Shared {
        unsigned long long goal, taken;
        uint32_t listed, next, complete, mine;
    };

    // LDS: [Shared][codes and decode units, as in the tile kernel, of the part's own rows and of those it fetches][W - I of the
    // part's rows: rowptr, col, coef][slot of every row][rows to fetch].  (All of it dynamic: a kernel with static LDS as well may
    // not ask for the last of the 160 KB.)
    static constexpr size_t lds_bytes(int n, int rows, int slots, int edges) {
        return sizeof(Shared) + (size_t)(rows + slots) * (T::ROW_CODE_BYTES + T::BPT * sizeof(float)) + ((size_t)rows + 1 + 2 * (size_t)edges + n + slots) * 4;
    }

    const TeamArgs& a;
    Shared& sh;
    const int lane, wave;
    uint8_t* codes;
    float* units;
    int32_t* rowptr;
    int32_t* col;
    float* coef;
    uint32_t* slot_of;
    uint32_t* list;
    uint64_t tile = 0, col0 = 0;
    uint32_t launch = 0;                                     // the number of this launch

    __device__ __forceinline__ Team(const TeamArgs& a_, uint8_t* lds)
        : a(a_), sh(*reinterpret_cast<Shared*>(lds)), lane(threadIdx.x & (kWave - 1)), wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
        codes = lds + sizeof(Shared);
        units = reinterpret_cast<float*>(codes + (size_t)(a.team_rows + a.team_slots) * T::ROW_CODE_BYTES);
        rowptr = reinterpret_cast<int32_t*>(units + (size_t)(a.team_rows + a.team_slots) * T::BPT);
        col = rowptr + a.team_rows + 1;
        coef = reinterpret_cast<float*>(col + a.team_edges);
        slot_of = reinterpret_cast<uint32_t*>(coef + a.team_edges);
        list = slot_of + a.n;
    }

    __device__ __forceinline__ unsigned long long* cell() const { return a.team_cells + (tile + 1) * (2 * kTeamLine); }
    __device__ __forceinline__ uint32_t* claim_cell(uint32_t part) const { return reinterpret_cast<uint32_t*>(cell() + kTeamLine / 2) + part; }
    __device__ __forceinline__ bool claim(uint32_t part) const {
        return __hip_atomic_exchange(claim_cell(part), launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != launch;
    }
    __device__ __forceinline__ int first_row(uint32_t part) const { return (int)part * a.team_rows; }
    __device__ __forceinline__ int end_row(uint32_t part) const { return min(a.n, ((int)part + 1) * a.team_rows); }
    __device__ __forceinline__ unsigned long long arrive() {
        return __hip_atomic_fetch_add(cell(), 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // The first part of the tile that nobody has claimed.  (Called by one thread.)
    __device__ __forceinline__ uint32_t unclaimed() const {
        uint32_t part = 0;
        while (part < a.team_parts && agent_load(claim_cell(part)) == launch) ++part;
        return part;
    }

    // Called by one thread: false if a part of the tile has not been claimed when the patience ends.
    __device__ __forceinline__ bool wait() {
        const uint64_t since = __builtin_amdgcn_s_memrealtime();
        while (agent_load(cell()) < sh.goal) {
            if (__builtin_amdgcn_s_memrealtime() - since >= a.team_patience && unclaimed() < a.team_parts) return false;
            __builtin_amdgcn_s_sleep(1);
        }
        return true;
    }

    // Gives the neighbours of the part's rows that are not its own a slot each.  Called by all threads.
    __device__ __forceinline__ void mark(int row0, int row1, int edges) {
        for (int e = threadIdx.x; e < edges; e += THREADS) {
            const int nb = col[e];
            if ((nb < row0 || nb >= row1) && atomicCAS(&slot_of[nb], kNoSlot, kNoSlot - 1u) == kNoSlot) {
                const uint32_t at = atomicAdd(&sh.listed, 1u);
                if (at < (uint32_t)a.team_slots) list[at] = (uint32_t)nb;
                slot_of[nb] = (uint32_t)a.team_rows + at;
            }
        }
    }

    // The listed rows' codes and decode units, from their messages into LDS where phase 1 puts its own.
    __device__ __forceinline__ void fetch(int row0, int row1, int edges) {
        for (int e = threadIdx.x; e < edges; e += THREADS) {  // from here on `col` says where a neighbour's codes are
            const int nb = col[e];
            col[e] = nb >= row0 && nb < row1 ? nb - row0 : (int)slot_of[nb];
        }
        const uint32_t rows = sh.listed, words = rows * ROW_WORDS;
        constexpr int AHEAD = 8;
        for (uint32_t w0 = threadIdx.x; w0 < words; w0 += AHEAD * THREADS) {
            uint32_t got[AHEAD];
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const uint32_t at = w0 + u * THREADS, w = at % ROW_WORDS;
                got[u] = 0u;                                  // what phase 1 leaves for columns behind the last one
                if (at < words) {
                    const uint8_t* row = a.msg + (uint64_t)list[at / ROW_WORDS] * a.msg_row_bytes;
                    const uint64_t block = col0 / B + w / BLOCK_WORDS, first = block * B;
                    const uint64_t left = first < a.N ? a.N - first : 0, m = left < (uint64_t)B ? left : (uint64_t)B;
                    if (w % BLOCK_WORDS < (m * BITS + 31) / 32)
                        got[u] = agent_load(reinterpret_cast<const uint32_t*>(row + block * T::MSG_BLOCK_BYTES + 4) + w % BLOCK_WORDS);
                }
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const uint32_t at = w0 + u * THREADS;
                if (at < words) reinterpret_cast<uint32_t*>(codes + (size_t)a.team_rows * T::ROW_CODE_BYTES)[at] = got[u];
            }
        }
        for (uint32_t q = threadIdx.x; q < rows * T::BPT; q += THREADS) {
            const uint64_t block = col0 / B + q % T::BPT;
            float unit = 0.f;
            if (block * B < a.N) {
                unit = agent_load(reinterpret_cast<const float*>(a.msg + (uint64_t)list[q / T::BPT] * a.msg_row_bytes + block * T::MSG_BLOCK_BYTES));
                if constexpr (KIND == DS_COMP_QUANT_MAXABS) unit = unit / (float)T::L;
            }
            units[a.team_rows * T::BPT + q] = unit;
        }
    }

    __device__ __forceinline__ float* x_of(int i) const { return a.x + (uint64_t)i * a.ld + col0 + 4 * lane; }

    // Has the part's row `own` a neighbour outside [row0, row1)?
    __device__ __forceinline__ bool far(int own, int row0, int row1) const {
        bool some = false;
        for (int e = rowptr[own] + lane; e < rowptr[own + 1]; e += kWave) some |= col[e] < row0 || col[e] >= row1;
        return __any(some);
    }

    template <bool FULL, typename F>
    __device__ __forceinline__ void gossip(int own, int row0, F slot, const float4 (&xh)[SW]) const {
        const int e0 = __builtin_amdgcn_readfirstlane(rowptr[own]), e1 = __builtin_amdgcn_readfirstlane(rowptr[own + 1]);
        T::template gossip_edges<FULL>(a, row0 + own, col0, lane, codes, units, e0, e1, slot, coef, xh);
    }

    // The same from the messages in memory, for a row whose x - gamma g waits in x.
    __device__ __forceinline__ void gossip_parked(int i) const {
        float4 xh[SW];
#pragma unroll
        for (int s = 0; s < SW; ++s) xh[s] = ld4(x_of(i) + s * kSweep);
        T::template gossip_from_messages<false, true>(a, i, col0, lane, xh);
#pragma unroll
        for (int s = 0; s < SW; ++s) st4(x_of(i) + s * kSweep, xh[s]);
    }

    template <bool FULL>
    __device__ __forceinline__ void run(uint32_t part) {
        const int row0 = first_row(part), row1 = end_row(part);
        const int e0 = a.rowptr[row0], edges = a.rowptr[row1] - e0;
        // A graph that replaced the one this launch was made for may be too large for its LDS: then the rows are finished from memory.
        const bool fits = edges <= a.team_edges;              // uniform
        // W - I of the part's rows is asked for first and put into LDS behind phase 1
        int32_t ptr_ahead = 0, col_ahead = 0;
        float coef_ahead = 0.f;
        if ((int)threadIdx.x <= row1 - row0) ptr_ahead = a.rowptr[row0 + threadIdx.x] - e0;
        if ((int)threadIdx.x < edges) { col_ahead = a.col[e0 + threadIdx.x]; coef_ahead = a.coef[e0 + threadIdx.x]; }
        float4 xh[RPW][SW];
        {
            float4 xv[SW], gv[SW], dv[SW];                    // asked for while the claim is under way
            const int i = row0 + wave;
            if (i < row1) T::template load_row<FULL>(a, i, col0, lane, xv, gv, dv);
            if (threadIdx.x == 0) sh.mine = claim(part) ? 1u : 0u;
            __syncthreads();
            if (!sh.mine) return;
            if (i < row1) T::template compress_loaded<FULL, false, 3>(a, i, wave, col0, lane, xv, gv, dv, codes, units, xh[0]);
        }
#pragma unroll
        for (int r = 1; r < RPW; ++r) {
            const int i = row0 + wave + r * NW;
            if (i < row1) T::template compress_row<FULL, false, 3>(a, i, wave + r * NW, col0, lane, codes, units, xh[r]);
        }
        if (fits) {
            if ((int)threadIdx.x <= row1 - row0) rowptr[threadIdx.x] = ptr_ahead;
            if ((int)threadIdx.x < edges) { col[threadIdx.x] = col_ahead; coef[threadIdx.x] = coef_ahead; }
            for (int e = threadIdx.x + THREADS; e < edges; e += THREADS) { col[e] = a.col[e0 + e]; coef[e] = a.coef[e0 + e]; }
        }
        drain();
        __syncthreads();
        // every tile's counter grows by `team_parts` a launch
        if (threadIdx.x == 0) sh.goal = (arrive() / a.team_parts + 1ull) * a.team_parts;
        // rows whose neighbours are all here need not wait
        uint32_t later = 0;
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            const int own = wave + r * NW;
            if (row0 + own < row1) {
                if (!fits || far(own, row0, row1)) later |= 1u << r;
                else gossip<FULL>(own, row0, [&](int e) { return __builtin_amdgcn_readfirstlane(col[e]) - row0; }, xh[r]);
            }
        }
        if (fits) mark(row0, row1, edges);
        if (threadIdx.x == 0) sh.complete = wait() ? 1u : 0u;
        __syncthreads();
        const bool complete = sh.complete != 0u;
        if (complete && fits && sh.listed <= (uint32_t)a.team_slots) {       // uniform
            fetch(row0, row1, edges);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < RPW; ++r)
                if (later >> r & 1u)
                    gossip<FULL>(wave + r * NW, row0, [&](int e) { return __builtin_amdgcn_readfirstlane(col[e]); }, xh[r]);
            return;
        }
#pragma unroll
        for (int r = 0; r < RPW; ++r)
            if (later >> r & 1u) {
#pragma unroll
                for (int s = 0; s < SW; ++s) st4(x_of(row0 + wave + r * NW) + s * kSweep, xh[r][s]);
            }
        unsigned long long taken = 0;
        if (!complete) taken = help();
        for (int r = 0; r < RPW; ++r)
            if (later >> r & 1u) gossip_parked(row0 + wave + r * NW);
        for (uint32_t p = 0; p < a.team_parts; ++p) {
            if (!(taken >> p & 1ull)) continue;
            for (int i = first_row(p) + wave; i < end_row(p); i += NW) gossip_parked(i);
        }
    }

    // The parts of this tile that nobody has claimed are taken by this workgroup; a part's x - gamma g waits in x.  Returns, when
    // the tile is complete, which parts that were.
    __device__ __forceinline__ unsigned long long help() {
        if (threadIdx.x == 0) sh.taken = 0ull;
        for (;;) {
            __syncthreads();
            if (threadIdx.x == 0) {
                sh.next = kTeamParts;
                while (agent_load(cell()) < sh.goal) {
                    const uint32_t part = unclaimed();
                    if (part < a.team_parts && claim(part)) {
                        sh.next = part;
                        sh.taken |= 1ull << part;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __syncthreads();
            const uint32_t part = __builtin_amdgcn_readfirstlane(sh.next);
            if (part == kTeamParts) return sh.taken;
            for (int i = first_row(part) + wave; i < end_row(part); i += NW) {
                float4 xh[SW];
                T::template compress_row<false, false, 3>(a, i, i - first_row(part), col0, lane, codes, units, xh);
#pragma unroll
                for (int s = 0; s < SW; ++s) st4(x_of(i) + s * kSweep, xh[s]);
            }
            drain();
            __syncthreads();
            if (threadIdx.x == 0) (void)arrive();
        }
    }
};

template <int KIND, int BITS, int B, int SW, int NW, int RPW>
__global__ void __launch_bounds__(NW* kWave, team_waves(SW)) team_tile_kernel(TeamArgs a) {
    using M = Team<KIND, BITS, B, SW, NW, RPW>;
    extern __shared__ __align__(16) uint8_t lds[];
    a.msg += (a.t_ptr[0] & 1ull) * a.msg_half;                // a handle of the row-streaming plan has two message buffers
    M m(a, lds);
    const unsigned long long block = (unsigned long long)blockIdx.y * gridDim.x + blockIdx.x;
    m.tile = block / a.team_parts;
    m.col0 = m.tile * M::T::TC;
    m.launch = (uint32_t)a.team_cells[0] + 1u;
    const uint32_t part = (uint32_t)(block % a.team_parts);
    if (m.col0 < a.N && (part == 0 || !a.team_solo)) {         // the last row of a two-dimensional grid may have spare workgroups
        for (int q = threadIdx.x; q < a.n; q += M::THREADS) m.slot_of[q] = kNoSlot;
        if (threadIdx.x == 0) m.sh.listed = 0u;
        if (m.col0 + M::T::TC <= a.N) m.template run<true>(part);
        else                          m.template run<false>(part);
    }
    __syncthreads();                                          // every wave has read the step counter and the number of the launch
    const unsigned long long blocks = (unsigned long long)gridDim.x * gridDim.y;
    step_counter_bump<KIND, BITS, B, SW, NW>(a, block, blocks, a.msg_half ? 0 : -1, nullptr, a.team_cells);
}

template <int KIND, int BITS, int B, int SW, int NW, int RPW>
void launch_team(const TeamArgs& args, hipStream_t stream) {
    using M = Team<KIND, BITS, B, SW, NW, RPW>;
    TeamArgs a = args;
    a.team_parts = (uint32_t)((a.n + a.team_rows - 1) / a.team_rows);
    const uint64_t tiles = (a.N + M::T::TC - 1) / M::T::TC;
    const uint64_t want = tiles * a.team_parts, max_x = 0xFFFFFFFFull / (NW * kWave);
    const unsigned gx = (unsigned)(want < max_x ? want : max_x);
    const unsigned gy = (unsigned)((want + gx - 1) / gx);
    const size_t lds = M::lds_bytes(a.n, a.team_rows, a.team_slots, a.team_edges);
    auto kern = team_tile_kernel<KIND, BITS, B, SW, NW, RPW>;
    static unsigned long long asked = 0;
    raise_lds_limit(reinterpret_cast<const void*>(kern), lds, asked);
    hipLaunchKernelGGL(kern, dim3(gx, gy), dim3(NW * kWave), lds, stream, a);
}

template <int KIND, int BITS, int B, int SW, int RPW>
void add_team_plan(int n, const char* name, std::vector<TilePlan>& plans) {
    constexpr int NW = 8;
    if constexpr (RPW * SW <= 16) {
        const int parts = (n + NW * RPW - 1) / (NW * RPW);
        if (parts < 2 || parts > (int)kTeamParts) return;
        TilePlan p;
        p.name = name;
        p.launch_team = &launch_team<KIND, BITS, B, SW, NW, RPW>;
        p.tile_cols = SW * kSweep;
        p.waves = NW;
        p.rows_per_wave = RPW;
        p.sweeps = SW;
        p.team = true;
        p.team_rows = (n + parts - 1) / parts;               // the parts are as even as they can be
        p.lds = &Team<KIND, BITS, B, SW, NW, RPW>::lds_bytes;
        plans.push_back(p);
    }
}

// The shapes that split n rows over more than one workgroup, those with the most rows in a workgroup first.
template <int KIND, int BITS, int B>
void team_plans_for_block(int n, std::vector<TilePlan>& plans) {
    constexpr int SW = B <= kSweep ? 1 : B / kSweep;
    add_team_plan<KIND, BITS, B, SW, 4>(n, "tile/team/8w/4rows", plans);
    add_team_plan<KIND, BITS, B, SW, 2>(n, "tile/team/8w/2rows", plans);
    add_team_plan<KIND, BITS, B, SW, 1>(n, "tile/team/8w/1row", plans);
}

template <int KIND, int BITS>
void team_plans_for_kind(int block, int n, std::vector<TilePlan>& plans) {
    switch (block) {
        case 64:   return team_plans_for_block<KIND, BITS, 64>(n, plans);
        case 128:  return team_plans_for_block<KIND, BITS, 128>(n, plans);
        case 256:  return team_plans_for_block<KIND, BITS, 256>(n, plans);
        case 512:  return team_plans_for_block<KIND, BITS, 512>(n, plans);
        case 1024: return team_plans_for_block<KIND, BITS, 1024>(n, plans);
        case 2048: return team_plans_for_block<KIND, BITS, 2048>(n, plans);
        default: return;
    }
}

}  // namespace
}  // namespace dsq
