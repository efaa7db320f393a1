// Internal declarations shared by the host side and the kernel launchers of libdsq.
// Nothing here is part of the C ABI (that is include/dsq.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "dsq.h"

namespace dsq {

constexpr int kWave = 64;                 // gfx950 wavefront
constexpr int kSweep = 4 * kWave;         // columns one wave covers with one float4 per lane
constexpr uint64_t kPitchAlign = 4096;    // x / delta row pitch: N rounded up to this many floats ...
constexpr uint64_t kPitchSkew = 2560;     // ... plus 10 KB, so that rows do not sit a power of two apart: with all rows
                                          // of a column tile in flight at once, HBM channel hashing made a 16 MiB pitch
                                          // 12 % slower than this one on MI355X (measured, 64 rows x 4 Mi columns)
constexpr int kMinBlock = 64, kMaxBlock = 2048;
constexpr uint32_t kWholeDevice = 1u << 16;   // see topk_resident_share
constexpr size_t kStepCells = 32 * 65;    // 64-bit cells behind the step counter (see TileArgs::t_ptr)

// Host-side description of W - I in CSR form (diagonal always present, columns ascending).
struct Graph {
    std::vector<int32_t> rowptr, col;
    std::vector<float> w;      // W_ij as given / built
    std::vector<float> coef;   // a_ij = W_ij - I_ij in fp32 (the coefficients of Algorithm 1, line 9)
    int max_degree = 0;        // entries per row, diagonal included
};

// Many device arrays in one allocation: the same list is placed twice, for the sizes and for the addresses.  (An allocation
// or a memset takes 10 us or so of making a handle, and a state made for one launch has 25 arrays.)
struct Slab {
    static constexpr size_t kPage = 2u << 20;             // large arrays start where an allocation of their own would
    uint8_t* base = nullptr;
    size_t bytes = 0;
    template <typename T>
    void place(T*& p, size_t count) {
        const size_t size = count * sizeof(T), step = size >= kPage ? kPage : 256;
        bytes = (bytes + step - 1) / step * step;
        if (base) p = reinterpret_cast<T*>(base + bytes);
        bytes += (size + 255) / 256 * 256;
    }
    // `list(slab)` places the arrays and returns how many bytes from the start on have to be zero.
    template <typename F>
    bool make(F list) {
        bytes = 0;
        size_t zero = list(*this);
        if (hipMalloc(&base, bytes) != hipSuccess) { base = nullptr; return false; }
        bytes = 0;
        zero = list(*this);
        return hipMemset(base, 0, zero) == hipSuccess;
    }
    void drop() {
        if (base) (void)hipFree(base);
        base = nullptr;
    }
};

// Validation and topology construction (pure host code, usable without a GPU).
ds_status validate_config(const ds_config* cfg, std::string& err, std::string* warn);
ds_status build_graph(const ds_config* cfg, Graph& g, std::string& err);
uint64_t message_row_bytes(const ds_config* cfg);

constexpr uint64_t kTeamCellBytes = 512;  // see TeamArgs::team_cells

// Arguments of the fused tile kernels (block quantiser / sign / identity).
struct TileArgs {
    float* x;                  // n x ld
    float* delta;              // n x ld
    const float* g;            // n x g_ld
    uint8_t* msg;              // n x msg_row_bytes
    const int32_t* rowptr;     // device CSR of W - I: rowptr (n+1), col (nnz) and coef (nnz, fp32 bits)
    const int32_t* col;        // are ONE contiguous array in that order (the tile kernel copies it whole)
    const float* coef;
    uint64_t ld, g_ld, N, msg_row_bytes;
    int n, nnz;                // workers; stored entries of W - I
    uint32_t stay;             // fused kernels: of 64 groups of tiles, those whose x and delta stay in the memory-side cache (stays())
    float gamma, eta;
    uint32_t seed_lo, seed_hi;
    // row-streaming variant only:
    const uint8_t* msg_prev;           // the previous step's messages: set by the kernels themselves (msg holds two
    uint64_t msg_half;                 // buffers of msg_half bytes; step t writes half t & 1 and reads the other)
    uint32_t* pending;                 // 1: the previous step's gossip sum has not been added to x yet
    uint32_t known;                    // flush: 1 if the host knows that it has not; 0: the kernel looks at `pending`
    // random sparsifier only:
    const uint32_t* keep_off;          // n x nsweeps: kept values before each 256-column sweep inside its group of 16
    const uint32_t* keep_group_off;    // n x ngroups: values the row's message holds before each group
    uint32_t* keep_raw;                // 2 x n x nsweeps: kept elements per sweep; half [t & 1] belongs to step t
    uint64_t nsweeps, ngroups;         // ceil(N / 256), ceil(nsweeps / 16)
    uint32_t keep_thr;                 // an element is kept iff the top 24 bits of its random word are below this
    uint32_t msg_cap;                  // values a row's message has room for
    unsigned long long* t_ptr;         // kStepCells 64-bit cells in device memory.  [0]: the step counter t, read by
                                       // the kernel and advanced by its last workgroup to finish, so that a captured
                                       // HIP graph of ds_step keeps moving along the random stream on replay.
                                       // [1]: finished first-level cells; [2]: random sparsifier: the step whose keep
                                       // counts are in keep_raw (~0 if none); [3]: row-streaming variant: a gossip sum is
                                       // pending; [4]: row-streaming variant: the message buffer (0 / 1) the last step
                                       // wrote; [16]: tile queue of the kernels whose workgroups walk over tiles (next tile
                                       // to hand out, counted from the grid size); [32 (1+c)], c < 64: finished
                                       // workgroups with blockIdx % 64 == c.
                                       // Cells [1], [16] and [32 (1+c)] are zero between launches.
};

// Teams of workgroups (dsq_team_impl.h).  (Apart from the others: every launch copies what its kernel is given, and a caller of small steps
// waits for that: 8 x 4,645 through ds_step_static, whose kernel was given all of this and TileArgs too, 8.05 us a call and 7.9 with GivenStep.)
struct TeamArgs : TileArgs {
    unsigned long long* team_cells;    // kTeamCellBytes for the launch and for each tile: counters that are never set back
    uint64_t team_patience;            // ticks a workgroup waits before it looks for parts nobody has claimed
    uint32_t team_parts;               // workgroups that share a tile (set by the launch) ...
    int team_rows;                     // ... the rows of each, ...
    int team_slots, team_edges;        // ... the neighbours it has room to fetch, and the entries of W - I it has room for
    uint32_t team_solo;                // tests: one workgroup of each tile works, and finds the other parts unclaimed
};

// The fused tile kernel without anything in device memory beside the caller's arrays (t_ptr and rowptr are nullptr): what the launch
// copies ...
struct GivenGraph {
    uint32_t t;                        // the step's number, low word
    int topo, torus_rows, torus_cols;  // DS_TOPO_RING or DS_TOPO_TORUS2D: each workgroup works W - I out for itself
};
struct GivenStep : GivenGraph {
    float* x;
    float* delta;
    const float* g;
    uint8_t* msg;
    uint64_t ld, g_ld, N, msg_row_bytes;
    int n, nnz;
    float gamma, eta;
    uint32_t seed_lo, seed_hi;
};
// ... and what the kernel makes of it.
struct GivenTileArgs : TileArgs, GivenGraph {};

// A compiled variant of the fused tile kernel, chosen once at init.
struct TilePlan {
    const char* name = "";
    void (*launch)(const TileArgs&, int rows_per_wave, hipStream_t) = nullptr;
    void (*launch_team)(const TeamArgs&, hipStream_t) = nullptr;                            // in its place where the rows of a tile are split
    void (*launch_given)(const GivenStep&, int rows_per_wave, hipStream_t) = nullptr;   // nullptr: not built for this shape
    int tile_cols = 0;         // columns per workgroup
    int waves = 0;             // waves per workgroup
    int rows_per_wave = 0;     // rows each wave owns (held in registers when the variant says so)
    int sweeps = 0;            // 256-column sweeps per tile
    bool looped = false;       // a wave owns more rows than its registers hold and forms them twice
    // Row-streaming variant (no LDS exchange, so no limit on n): a step leaves x = x - gamma g and its gossip sum
    // to the next step's pass, which decodes the neighbours' codes from the previous messages; `flush` adds a
    // pending sum now.
    bool streaming = false;
    void (*flush)(const TileArgs&, hipStream_t) = nullptr;
    // The rows of a tile are split over several workgroups: see TeamArgs.
    bool team = false;
    int team_rows = 0, team_slots = 0, team_edges = 0;
    size_t (*lds)(int n, int rows, int slots, int edges) = nullptr;
};

// Random sparsifier: makes sure the kept-element counts of this step's 256-column sweeps are in keep_raw (the tile
// kernel of the previous step normally left them there; otherwise they are recounted from the random words) and
// turns them into message offsets: local_off (n x nsweeps, = TileArgs::keep_off of the tile launch that follows)
// inside groups of 16 sweeps, group_tot (n x ngroups, = TileArgs::keep_group_off) across the groups.  Writes
// the per-row count into the message header (prev_count, n words, remembers it so that stale values behind a
// shorter message are cleared) and raises *overflow if a row keeps more than msg_cap values.
void launch_keep_offsets(const TileArgs& a, uint32_t* local_off, uint32_t* group_tot, uint32_t* prev_count, uint32_t* overflow,
                         hipStream_t stream);
uint64_t rand_sparse_capacity(uint64_t N, uint64_t k);

// The row-streaming plan of a block compressor (quantiser or sign); false if the compressor has none.
bool stream_plan(const ds_config& cfg, TilePlan& plan);

// The shapes that split the rows of a tile over several workgroups, most rows per workgroup first; none where one holds them all
// or a tile has too many.
void team_plans(const ds_config& cfg, const Graph& graph, std::vector<TilePlan>& plans);
// Makes the shape's LDS large enough for the graph; false, and the shape as it was, if there is not that much.
bool fit_team(const Graph& graph, TilePlan& plan);
extern const uint64_t kTeamPatienceTicks;
constexpr size_t kMaxLds = 160 * 1024;    // of a workgroup

// Lists the variants that fit (n, compressor), best guess first; returns false with `err` set if none does.
bool choose_tile_plans(const ds_config& cfg, int nnz, std::vector<TilePlan>& plans, std::string& err);

// ---- top-k path ---------------------------------------------------------------------------------
struct TopkArgs {
    float* x;
    float* delta;
    const float* g;
    uint8_t* msg;              // n x k pairs (u32 index, f32 value)
    const int32_t* rowptr;
    const int32_t* col;
    const float* coef;
    uint64_t ld, g_ld, N, k;   // k: pairs from one row's message to the next (top-k: the k of the operator; GSpar: the
                               // capacity plus the header pair)
    int n;
    float gamma, eta;
    unsigned long long* t_ptr;  // step counter in device memory (advanced once per step)
    uint32_t known;            // flush: 1 if the host knows that a tail is pending; 0: the kernels look at the device's mark
    // GSpar only:
    uint64_t k_expected;       // the operator's k (expected kept elements)
    uint32_t seed_lo, seed_hi; // key of the mask's random stream
};

struct TopkState;              // device scratch of the radix select (histograms, per-chunk counts)
// The part of the current device, in units of 1 / kWholeDevice, that the kernel which takes a whole step in one launch
// (dsq_topk_resident.hip) fills; 0 if the problem is not small enough for it.
uint32_t topk_resident_share(const ds_config& cfg);
// resident: steps may take that kernel; impatient: its first meeting calls itself off at once (tests of what follows then).
ds_status topk_create(const ds_config& cfg, uint64_t ld, bool resident, bool impatient, TopkState** out, std::string& err);
void topk_destroy(TopkState* s);
// one_launch: with that kernel (the state has to be made for it), else with the launches that large problems take.
ds_status topk_step(TopkState* s, const TopkArgs& a, bool one_launch, hipStream_t stream);
// Unless the state is made for one launch, topk_step leaves the sparse part of the gossip update of x to the next step's first pass;
// topk_flush applies it now (no-op if nothing is pending).  Call before x is read or replaced, with the
// buffers, mixing matrix and eta the last step ran with (a.g is not used).  unseen: a step of the handle has been captured, so
// what is pending is not known here (a graph may have been replayed).
ds_status topk_flush(TopkState* s, const TopkArgs& a, bool unseen, hipStream_t stream);
// Number of rows whose last step selected from the candidate slots (the fast path).
ds_status topk_candidate_rows(TopkState* s, hipStream_t stream, uint32_t* count);
// GSpar: true if a row has kept more elements than its message has room for in some step since the handle was made.
ds_status gspar_overflowed(TopkState* s, hipStream_t stream, bool* overflowed);

// ---- norm-rescaled b-bit path (DS_COMP_QUANT_L2NORM) ----------------------------------------------
struct L2Args {
    float* x;
    float* delta;
    const float* g;
    uint8_t* msg;              // n rows of [f32 norm][code words]
    const int32_t* rowptr;
    const int32_t* col;
    const float* coef;
    uint64_t ld, g_ld, N, msg_row_bytes;
    uint64_t msg_half;         // msg holds two buffers of this many bytes; a step writes the one the last step did not
                               // (0, one buffer, where nothing is left to the next step: states made for one launch)
    int n;
    float gamma, eta;
    unsigned long long* t_ptr;  // step cells in device memory: [0] the step counter (advanced once per step), [4] the
                                // message buffer (0 / 1) the last completed step wrote, [5] rows finished in the
                                // step's last kernel (zero between launches)
    uint32_t known;             // flush: what the device's mark of a pending tail holds, if the host knows; 0: the kernels look
};

struct L2State;                // device scratch: per-row scales, per-chunk partial reductions
// As for the top-k path.
uint32_t l2q_resident_share(const ds_config& cfg);
ds_status l2q_create(const ds_config& cfg, uint64_t ld, bool resident, bool impatient, L2State** out, std::string& err);
void l2q_destroy(L2State* s);
ds_status l2q_step(L2State* s, const L2Args& a, bool one_launch, hipStream_t stream);
// Unless the state is made for one launch, l2q_step leaves delta = v - C[v] and the gossip update of x to the next step's first pass;
// l2q_flush applies them now (no-op if nothing is pending).  Call before the state is read or replaced, with
// the buffers, mixing matrix and eta the last step ran with (a.g is not used).
ds_status l2q_flush(L2State* s, const L2Args& a, bool unseen, hipStream_t stream);
// Number of rows whose last step kept the codes its first pass wrote speculatively (no second dense pass).
ds_status l2q_speculated_rows(L2State* s, hipStream_t stream, uint32_t* count);

// Device twin of the deterministic host gradient generator (harness aid).
ds_status launch_workload_gradient(const ds_workload& w, uint64_t t, const float* x, uint64_t x_ld, float* g, uint64_t g_ld,
                                   hipStream_t stream);

}  // namespace dsq
