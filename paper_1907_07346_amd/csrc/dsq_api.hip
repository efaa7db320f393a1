// C ABI of libdsq: handle life cycle, state transfer and the ds_step dispatcher.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <new>

#include "dsq_internal.h"

struct ds_handle {
    ds_config cfg{};
    dsq::Graph graph;
    uint64_t ld = 0;                 // row pitch of x and delta, in floats
    uint64_t msg_row_bytes = 0;
    uint64_t msg_half = 0;           // row-streaming variant: bytes of one of the two message buffers (else 0)
    uint64_t t = 0;
    bool stepped = false;
    int device = 0;
    hipStream_t last_stream = nullptr;
    float* x = nullptr;
    float* delta = nullptr;
    uint8_t* msg = nullptr;
    int32_t* d_rowptr = nullptr;
    int32_t* d_col = nullptr;
    float* d_coef = nullptr;
    unsigned long long* d_t = nullptr;   // kStepCells cells; d_t[0]: the step counter t, read and advanced by the
                                         // step's kernels; the rest: the tile kernel's finished-workgroup counters
    dsq::TilePlan tile;
    std::vector<dsq::TilePlan> tile_candidates;
    dsq::TilePlan team;                  // row-streaming plan: what takes a step whole (no team: nothing does)
    unsigned long long* d_team = nullptr;    // arrival counters of the team kernels
    bool impatient = false;              // ... whose workgroups then look for parts nobody works on at once (tests)
    // Steps since x and delta were last asked for, and how many there were between the last two times.
    uint64_t run = 0, period = 1;
    bool complete = true;                // x and delta are complete once everything enqueued has run
    enum { kFree, kWhole, kStreamed } captured = kFree;   // how the steps go that a graph may replay unseen, and all others with them
    bool unseen = false;                 // a step has been captured: graphs may run steps that are not counted here
    bool asked = false;                  // x and delta were lent since the last step, and not seen to be lent inside a capture
    bool completes = false;              // no step leaves anything to the next one (a graph relies on it: see ds_step)
    dsq::TopkState* topk = nullptr;
    dsq::L2State* l2q = nullptr;
    bool resident = false;               // steps may take one launch ...
    uint32_t share = 0;                  // ... whose workgroups wait for each other and fill this part of the GPU
    int seat = -1;                       // row of g_seats this handle holds, and the stream it holds it for
    hipStream_t seat_stream = nullptr;
    uint32_t* d_keep = nullptr;          // random sparsifier, one allocation: n x nsweeps offsets inside groups,
                                         // n x ngroups group offsets, n previous counts, one overflow flag,
                                         // 2 x n x nsweeps raw counts (steps of even / odd t)
    uint64_t nsweeps = 0, ngroups = 0;
    std::string err;
    std::string plan_name;
};

namespace {

ds_status fail(ds_handle* h, ds_status st, const std::string& msg) {
    if (h) h->err = msg;
    return st;
}

ds_status hip_fail(ds_handle* h, hipError_t e, const char* what) {
    return fail(h, e == hipErrorOutOfMemory ? DS_ENOMEM : DS_EHIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define DSQ_HIP(h, call)                                              \
    do {                                                              \
        hipError_t e_ = (call);                                       \
        if (e_ != hipSuccess) return hip_fail((h), e_, #call);        \
    } while (0)

// ---- who may step in one launch --------------------------------------------------------------------
// The workgroups of a resident kernel (dsq_resident.h) wait for each other, so all of them have to be running at some
// time.  Launches on one stream follow each other; those on several share the GPU, and where they are more than it holds each
// can keep the last workgroups of the others out, until the patience of one ends and one workgroup does that step alone:
// three handles of 8 workers x 272,474 parameters that started their steps together on three streams took 14.6 ms for it
// (norm-rescaled codes; top-k 27.8, GSpar 25.6), and 0.08 ms (0.15, 0.15) in the launches of large problems.  So a stream
// on which handles step in one launch has a seat, of the largest share any of them takes, and a handle whose stream
// finds no room takes those launches.  A handle gives its seat up when it steps on another
// stream and when it is destroyed.  Not seen from here: other processes, graphs replayed on streams of their own, and
// streams that may not use every compute unit; there the meeting's patience decides.
constexpr int kSeats = 64;
struct Seat {
    int device, handles;                 // handles == 0: free
    hipStream_t stream;
    uint32_t share;
};
Seat g_seats[kSeats];
std::mutex g_seats_lock;

void leave_seat_locked(ds_handle* h) {
    if (h->seat >= 0) g_seats[h->seat].handles -= 1;         // the share stays until the last one leaves
    h->seat = -1;
}

void take_seat(ds_handle* h, hipStream_t stream) {
    std::lock_guard<std::mutex> hold(g_seats_lock);
    leave_seat_locked(h);
    int at = -1, spare = -1;
    uint32_t others = 0;
    for (int q = 0; q < kSeats; ++q) {
        const Seat& s = g_seats[q];
        if (s.handles == 0) spare = q;
        else if (s.device != h->device) continue;
        else if (s.stream == stream) at = q;
        else others += s.share;
    }
    const uint32_t share = at >= 0 && g_seats[at].share > h->share ? g_seats[at].share : h->share;
    if (others + share > dsq::kWholeDevice || (at < 0 && spare < 0)) return;
    if (at < 0) g_seats[at = spare] = Seat{h->device, 0, stream, 0};
    g_seats[at].handles += 1;
    g_seats[at].share = share;
    h->seat = at;
    h->seat_stream = stream;
}

// May this step of the handle be one launch?
bool seated(ds_handle* h, hipStream_t stream) {
    if (!h->resident) return false;
    if (h->share == 0) return true;                          // its workgroups never wait
    static thread_local char own_stream;                     // hipStreamPerThread is one name for a stream of every thread
    if (stream == hipStreamPerThread) stream = reinterpret_cast<hipStream_t>(&own_stream);
    if (h->seat < 0 || h->seat_stream != stream) take_seat(h, stream);
    return h->seat >= 0;
}

void release(ds_handle* h) {
    if (!h) return;
    if (h->seat >= 0) {
        std::lock_guard<std::mutex> hold(g_seats_lock);
        leave_seat_locked(h);
    }
    if (h->topk) dsq::topk_destroy(h->topk);
    if (h->l2q) dsq::l2q_destroy(h->l2q);
    if (h->x) (void)hipFree(h->x);
    if (h->delta) (void)hipFree(h->delta);
    if (h->msg) (void)hipFree(h->msg);
    if (h->d_rowptr) (void)hipFree(h->d_rowptr);   // d_col and d_coef point into the same allocation
    if (h->d_t) (void)hipFree(h->d_t);
    if (h->d_team) (void)hipFree(h->d_team);
    if (h->d_keep) (void)hipFree(h->d_keep);
    delete h;
}


dsq::TileArgs tile_args(const ds_handle* h, const float* g_dev, uint64_t g_ld);

// Kernel arguments of the top-k and the norm-rescaled paths, always from the handle's CURRENT buffers, mixing
// matrix and rates (a flush after ds_set_mixing must not see the device addresses of the matrix it replaced).
dsq::TopkArgs topk_args(const ds_handle* h, const float* g_dev, uint64_t g_ld) {
    dsq::TopkArgs a{};
    a.x = h->x; a.delta = h->delta; a.g = g_dev; a.msg = h->msg;
    a.rowptr = h->d_rowptr; a.col = h->d_col; a.coef = h->d_coef;
    a.ld = h->ld; a.g_ld = g_ld; a.N = h->cfg.N; a.k = h->cfg.comp.k; a.n = h->cfg.n;
    a.gamma = h->cfg.gamma; a.eta = h->cfg.eta; a.t_ptr = h->d_t;
    if (h->cfg.comp.kind == DS_COMP_GSPAR) {               // rows of [header pair][capacity pairs]
        a.k = h->msg_row_bytes / 8;
        a.k_expected = h->cfg.comp.k;
        a.seed_lo = (uint32_t)h->cfg.seed; a.seed_hi = (uint32_t)(h->cfg.seed >> 32);
    }
    return a;
}

dsq::L2Args l2_args(const ds_handle* h, const float* g_dev, uint64_t g_ld) {
    dsq::L2Args a{};
    a.x = h->x; a.delta = h->delta; a.g = g_dev; a.msg = h->msg;
    a.rowptr = h->d_rowptr; a.col = h->d_col; a.coef = h->d_coef;
    a.ld = h->ld; a.g_ld = g_ld; a.N = h->cfg.N; a.msg_row_bytes = h->msg_row_bytes; a.n = h->cfg.n;
    a.msg_half = h->msg_half;
    a.gamma = h->cfg.gamma; a.eta = h->cfg.eta; a.t_ptr = h->d_t;
    return a;
}

// Is the stream being captured into a graph?  (What cannot be found out counts as yes.)
bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// Does a step leave part of itself to the next one?  (A state made for one launch never does.)
bool defers(const ds_handle* h) { return h->tile.streaming || ((h->topk || h->l2q) && !h->resident); }

// Three paths (top-k, norm-rescaled codes, the row-streaming block kernels) leave the tail of a step to the next step's first pass;
// this applies it now, on the stream of the last step.
ds_status apply_deferred(ds_handle* h) {
    if (h->topk) return dsq::topk_flush(h->topk, topk_args(h, nullptr, 0), h->unseen, h->last_stream);
    if (h->l2q) return dsq::l2q_flush(h->l2q, l2_args(h, nullptr, 0), h->unseen, h->last_stream);
    if (h->tile.streaming && h->stepped) {
        // (A graph that begins with this call: its steps go the way of the steps so far, whole only if nothing is pending before it either.)
        if (h->unseen && h->captured == ds_handle::kFree)
            h->captured = h->team.team && h->complete && h->period == 1 ? ds_handle::kWhole : ds_handle::kStreamed;
        if (h->complete && h->captured != ds_handle::kStreamed) return DS_OK;
        dsq::TileArgs a = tile_args(h, nullptr, 0);
        a.known = h->unseen ? 0u : 1u;
        h->tile.flush(a, h->last_stream);
        h->complete = true;
        return hipGetLastError() == hipSuccess ? DS_OK : DS_EHIP;
    }
    return DS_OK;
}

// The same for whoever looks at x and delta or changes them.  Callers that replace W, gamma or eta call it BEFORE the
// replacement: the tail belongs to the values the step ran with.
ds_status flush_deferred(ds_handle* h) {
    // A flush that is captured runs in every replay, whatever is pending then: it has to be in the graph, and to look at the device's mark.
    if (defers(h) && h->stepped && !h->unseen) h->unseen = capturing(h->last_stream);
    if (h->run) h->period = h->run;
    h->run = 0;
    return apply_deferred(h);
}

// The 64ths of the fused kernel's tiles whose x and delta stay in the memory-side cache: as many as fit into 192 MB of it beside the
// messages, which go through it too.  Only in steps that follow one another: a caller that asks for x after every step reads
// it, and draws the next gradient, in between, and plain loads that find nothing there are the slower ones (256 workers x 272,474 after a
// pass over another state 313 us, non-temporal 286).
// (us a step of a run, with nothing staying and so: 8 x 2,097,152 at 4 bits 66 and 54, 16 x 2,097,152 121 and 108; sign, 8 x 25,557,032 722
// and 675; 16 x 11,173,962 at 2 bits 637 and 616; 64 x 4,194,304 at 4 bits, whose messages are 134 MB, 1009 and 973, with twice as much
// staying 1007 and three times 1064.)
// Where the line lies depends on what is smaller being in a cache either way: x and delta of 72 MiB (8 x 1,179,648: 4 bits 39.7 and 33.2, 2
// bits 39.6 and 35.2, 8 bits 41.9 and 38, sign 40 and 36; 64 MiB in 24 rows: 31.2 and 33, 32.5 and 34.7, 33.8 and 33.8, 31.8 and 31.1), of 128
// for the random sparsifier (24 x 696,320 75.8 and 74.8, x 524,288 56.2 and 56.9).  Signs, whose pass has little else to do, also where the
// L2s hold most of it (8 x 262,144 8.4 and 7.3, 24 x 86,016 9.7 and 9.0, 8 x 393,216 12.5 and 11.5; but 8 x 524,288 15.6 and 17.1, 24 x
// 40,960 5.7 and 6.0), and uncompressed values always: their messages are stored past the caches (8 x 16,384 4.4 and 4.3, x 262,144 10.0 and
// 9.1, x 1,048,576 37 and 33, x 2,097,152 75 and 63).
bool state_stays(int kind, uint64_t bytes) {
    if (kind == DS_COMP_IDENTITY) return true;
    if (kind == DS_COMP_SIGN_MEANABS && bytes >= (12ull << 20) && bytes <= (28ull << 20)) return true;
    return bytes >= (kind == DS_COMP_RAND_SPARSE ? 128ull << 20 : 72ull << 20);
}
uint32_t stay_share(const ds_handle* h) {
    if (h->run <= 1 && h->period <= 1) return 0;
    constexpr uint64_t room = 192ull << 20;
    const uint64_t state = (uint64_t)h->cfg.n * h->cfg.N * 8;
    const uint64_t messages = h->cfg.comp.kind == DS_COMP_IDENTITY ? 0 : h->msg_row_bytes * (uint64_t)h->cfg.n;
    if (messages >= room || !state_stays(h->cfg.comp.kind, state)) return 0;
    return (uint32_t)std::min<uint64_t>(64, (room - messages) * 64 / state);
}

dsq::TileArgs tile_args(const ds_handle* h, const float* g_dev, uint64_t g_ld) {
    dsq::TileArgs a{};
    a.x = h->x; a.delta = h->delta; a.g = g_dev; a.msg = h->msg;
    a.rowptr = h->d_rowptr; a.col = h->d_col; a.coef = h->d_coef;
    a.ld = h->ld; a.g_ld = g_ld; a.N = h->cfg.N; a.msg_row_bytes = h->msg_row_bytes;
    a.n = h->cfg.n; a.nnz = (int)h->graph.col.size();
    a.gamma = h->cfg.gamma; a.eta = h->cfg.eta;
    a.seed_lo = (uint32_t)h->cfg.seed; a.seed_hi = (uint32_t)(h->cfg.seed >> 32); a.t_ptr = h->d_t;
    a.msg_half = h->msg_half;
    a.stay = stay_share(h);
    a.pending = reinterpret_cast<uint32_t*>(h->d_t + 3);        // cell 3: the row-streaming variant's pending flag
    if (h->cfg.comp.kind == DS_COMP_RAND_SPARSE) {
        a.keep_off = h->d_keep;
        a.keep_group_off = h->d_keep + (size_t)h->cfg.n * h->nsweeps;
        a.keep_raw = h->d_keep + (size_t)h->cfg.n * (h->nsweeps + h->ngroups) + h->cfg.n + 1;
        a.nsweeps = h->nsweeps;
        a.ngroups = h->ngroups;
        a.keep_thr = (uint32_t)((h->cfg.comp.k << 24) / h->cfg.N);        // floor(k 2^24 / N) <= 2^24
        a.msg_cap = (uint32_t)((h->msg_row_bytes - 4) / 4);
    }
    return a;
}

void launch_plan(const ds_handle* h, const dsq::TilePlan& plan, const float* g_dev, uint64_t g_ld, hipStream_t stream) {
    const dsq::TileArgs args = tile_args(h, g_dev, g_ld);
    if (!plan.team) return plan.launch(args, plan.rows_per_wave, stream);
    dsq::TeamArgs a{};
    static_cast<dsq::TileArgs&>(a) = args;
    a.team_cells = h->d_team;
    a.team_patience = h->impatient ? 0 : dsq::kTeamPatienceTicks;
    a.team_solo = h->impatient ? 1u : 0u;
    a.team_rows = plan.team_rows;
    a.team_slots = plan.team_slots;
    a.team_edges = plan.team_edges;
    plan.launch_team(a, stream);
}

// Row pitch candidates (floats added to N rounded up to kPitchAlign).  A tile kernel has all n rows
// of a column window in flight at once, so how the row pitch falls on the HBM channel hash decides
// up to 12 % of the achieved bandwidth, and the best pitch differs between shapes and GPUs.  ds_init
// times the real kernel on the (still all-zero) state for each candidate and keeps the fastest.
const uint64_t kPitchCandidates[] = {0, 2560, 4096, 6656, 8192, 12288};
constexpr uint64_t kMaxPitchSkew = 12288;

// Arrival counters for the narrowest tiles of any candidate.
size_t team_bytes(const ds_handle* h) {
    uint64_t tiles = 0;
    auto most = [&](const dsq::TilePlan& p) {
        if (!p.team) return;
        const uint64_t t = (h->cfg.N + p.tile_cols - 1) / p.tile_cols;
        tiles = t > tiles ? t : tiles;
    };
    for (const dsq::TilePlan& p : h->tile_candidates) most(p);
    most(h->tile);
    most(h->team);
    return tiles ? (size_t)(tiles + 1) * dsq::kTeamCellBytes : 0;
}

// Times `plan` at the current h->ld on the all-zero state (3 launches, twice, after a warm-up); < 0 on failure.
float time_plan(ds_handle* h, const dsq::TilePlan& plan, const float* g, hipEvent_t e0, hipEvent_t e1) {
    if (plan.team && hipMemset(h->d_team, 0, team_bytes(h)) != hipSuccess) return -1.f;   // another plan's parts may be another number
    launch_plan(h, plan, g, h->ld, nullptr);
    float best = 1e30f;
    for (int rep = 0; rep < 2; ++rep) {                        // the better of two timings: less noise in the choice
        (void)hipEventRecord(e0, nullptr);
        for (int r = 0; r < 3; ++r) launch_plan(h, plan, g, h->ld, nullptr);
        (void)hipEventRecord(e1, nullptr);
        float ms = 0.f;
        if (hipGetLastError() != hipSuccess) return -1.f;      // a launch that was refused would look fast
        if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess) return -1.f;
        best = ms < best ? ms : best;
    }
    return best;
}

// Picks the launch shape (at the default pitch) and then the row pitch for it by timing the real
// kernel.  Returns the chosen skew and sets h->tile; leaves x, delta and the messages zeroed.
uint64_t autotune(ds_handle* h, uint64_t base_ld, size_t state_bytes, size_t msg_bytes) {
    float* g = nullptr;
    if (hipMalloc(&g, state_bytes) != hipSuccess) { (void)hipGetLastError(); return dsq::kPitchSkew; }
    hipEvent_t e0, e1;
    bool ok = hipMemset(g, 0, state_bytes) == hipSuccess && hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess;
    uint64_t best_skew = dsq::kPitchSkew;
    if (ok) {
        float best_ms = 1e30f;
        h->ld = base_ld + dsq::kPitchSkew;
        // A later candidate (or, below, another pitch) must win by 2 % to be taken: differences below that are
        // timing noise, and a choice that flips between near-equal candidates from run to run makes measurements
        // hard to compare.
        for (const dsq::TilePlan& plan : h->tile_candidates) {
            const float ms = time_plan(h, plan, g, e0, e1);
            if (ms < 0.f) { ok = false; break; }
            if (ms < 0.98f * best_ms) { best_ms = ms; h->tile = plan; }
        }
        for (uint64_t skew : kPitchCandidates) {
            if (!ok) break;
            if (skew == dsq::kPitchSkew) continue;             // timed above
            h->ld = base_ld + skew;
            const float ms = time_plan(h, h->tile, g, e0, e1);
            if (ms < 0.f) { ok = false; break; }
            if (ms < 0.98f * best_ms) { best_ms = ms; best_skew = skew; }
        }
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    (void)hipDeviceSynchronize();
    (void)hipFree(g);
    (void)hipMemset(h->x, 0, state_bytes);
    (void)hipMemset(h->delta, 0, state_bytes);
    (void)hipMemset(h->msg, 0, msg_bytes ? msg_bytes : 4);
    (void)hipMemset(h->d_t, 0, dsq::kStepCells * sizeof(unsigned long long));   // the timed launches advanced t
    (void)hipMemset(h->d_t + 2, 0xFF, sizeof(unsigned long long));              // ... and no keep counts are valid
    if (h->d_team) (void)hipMemset(h->d_team, 0, team_bytes(h));
    (void)hipDeviceSynchronize();
    if (!ok) h->tile = h->tile_candidates.front();
    return ok ? best_skew : dsq::kPitchSkew;
}

// Is the row-streaming variant the faster one where the fused kernel would serve too?  It can be where the fused kernel's
// waves own more rows than they hold in registers (every shape ends at 64 rows), and a tile of 512 columns or more makes those
// rows a serial chain of 2 KB loads, formed twice.  Measured with the state complete after every step over 65 .. 800 workers,
// blocks of 512 .. 2048, all codes and circulant graphs (3100 points), as streaming's time in units of the fused kernel's:
//   up to 128 tiles, half of the compute units have no tile: 0.1 to 0.99 for any graph, but 1.07 at the line itself where there are
//     fewer than 96 workers with nine neighbours each (112 tiles: 0.96);
//   beyond 512 tiles from 192 workers on the fused kernel's time is that of whole waves of 256 tiles and streaming's that of
//     the tiles, which decode the neighbours from memory: with up to 5 neighbours (own included) 0.75 to 1.00 while the
//     last wave leaves a sixteenth of them all free (one point of 544 at 1.03) and up to 1.12 when it is full; with 9, 0.79
//     to 0.99 while three sixteenths are free; with 17 up to 1.22.  256 workers x 272,474, torus, 4 bits: 412
//     us fused, 345 streaming (246 back to back).  Such a handle takes a step whole where that is faster: whole_steps_faster.
// In between, and with blocks of up to 256 columns (100 x 100,000 at 4 bits: 52 us fused, 65 streaming), nothing is left to the next step.
// The graph is the one the handle is made with: a later ds_set_mixing changes no plan.
bool streams_faster(const ds_config& cfg, uint64_t entries) {
    if (cfg.comp.kind != DS_COMP_QUANT_MAXABS && cfg.comp.kind != DS_COMP_SIGN_MEANABS) return false;
    if (cfg.n <= 64 || cfg.comp.block < 512) return false;
    const uint64_t n = (uint64_t)cfg.n, tiles = (cfg.N + cfg.comp.block - 1) / cfg.comp.block;
    const bool near = entries <= 5 * n;
    if (tiles <= 128) return tiles <= 112 || n >= 96 || near;
    if (tiles <= 512 || n < 192 || entries > 9 * n) return false;
    return 16 * tiles <= (near ? 15u : 13u) * ((tiles + 255) / 256 * 256);
}

// The team shape for a handle: most rows in a workgroup while there are two workgroups per compute unit, or four where a lane
// holds sixteen float4 of x - gamma g.  (4 bits, blocks of 512, rows in a workgroup 8 / 16 / 32, state complete after every step: 100 workers x
// 2,621 10.8 / 13.6 / 17.4 us, 256 x 16,384 29.3 / 24.4 / 26.3, 256 x 262,144 319 / 277 / 271.)
dsq::TilePlan best_team(const std::vector<dsq::TilePlan>& teams, const ds_config& cfg) {
    for (const dsq::TilePlan& p : teams) {
        const uint64_t tiles = (cfg.N + p.tile_cols - 1) / p.tile_cols, parts = (cfg.n + p.team_rows - 1) / p.team_rows;
        if (tiles * parts >= (p.rows_per_wave * p.sweeps > 8 ? 1024u : 512u)) return p;
    }
    return teams.empty() ? dsq::TilePlan() : teams.back();
}

// A handle of the row-streaming plan whose x is read after every step: is the step in one launch faster than the streaming pass and
// the gossip sum on its own?  4 bits, blocks of 512: 100 workers x 41,943 26.1 us and 26.9, 280 x 3,744 15.1 and 13.1, 280 x 59,918 80
// and 91, 256 x 272,474 293 and 345; blocks of 2048, which leave one workgroup or two to a compute unit: 100 x 167,772 94 and 92, x 671,088
// 292 and 332.
bool whole_steps_faster(const ds_config& cfg, const dsq::TilePlan& stream) {
    return (uint64_t)cfg.n * cfg.N >= (stream.sweeps == 8 ? 32ull << 20 : 8ull << 20);
}

// Is it faster than the fused kernel of shape `fused`?  Where that forms its rows twice: 100 x 671,088 357 us fused, 265 as teams; 256 x
// 1,024 61 and 12.  Not where there is a workgroup for nearly every compute unit, so that one round of them does all tiles, and the second
// forming reads the memory-side cache (x and g of 112 MiB at most together).  Fused in units of the best shape of teams, 4 bits, 155 to 256 tiles:
// tiles of one sweep, 120 to 220 workers 0.82 to 1.06, 256 workers 0.99 to 1.11; of eight sweeps, 36 to 48 workers 0.86 to 1.01 from 175 tiles on
// (1.08 to 1.18 below), 56 to 72 workers 0.95 to 1.11.  Of two sweeps 80 workers 0.99 to 1.17, 140 to 256 1.08 to 1.32, and of four 48 workers 0.98 to
// 1.14, 100 to 140 1.07 to 1.21: teams there.  1.02 to 1.45 at 280 to 400 tiles and 1.04 to 1.60 at 100 to 150, all of them.  Where registers hold
// the rows, only if there are few tiles of many rows: 64 x 16,384 (32 tiles) 19 and 11, 48 x 87,381 (171 tiles) 18 and 25; not for tiles of one
// sweep, whose sixteen-wave shape takes 7 to 8 us (9 as teams).
bool teams_faster(const ds_config& cfg, const dsq::TilePlan& fused) {
    const uint64_t tiles = (cfg.N + fused.tile_cols - 1) / fused.tile_cols;
    const bool cached = (uint64_t)cfg.n * cfg.N <= (28u << 20);              // x and g fit in the memory-side cache
    if (fused.looped) return !((fused.sweeps == 1 || fused.sweeps == 8) && tiles >= 160 && tiles <= 256 && cached);
    return cfg.n > 32 && fused.sweeps >= 2 && tiles <= 64;
}

// Diagnostics (off the hot path); fp64 accumulation.  The three sums of a workgroup are added to one of kDiagCells cells of
// `out`, 128 bytes apart, which the host adds up: with one cell the additions of up to 4096 workgroups follow one another, and took longer
// than the rest where the workers are few (the whole call, 8 x 131,072: 53 us and now 33; 3 x 349,525: 83 and now 43).
constexpr int kDiagCells = 64, kDiagStride = 16;
__device__ __forceinline__ void add_diagnostics(double cons, double dsq_, double mixed, double (*part)[4], double* out) {
    double v[3] = {cons, dsq_, mixed};
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o);
        if (lane == 0) part[q][wave] = v[q];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        const double tot = part[threadIdx.x][0] + part[threadIdx.x][1] + part[threadIdx.x][2] + part[threadIdx.x][3];
        atomicAdd(&out[(blockIdx.x % kDiagCells) * kDiagStride + threadIdx.x], tot);
    }
}

// n rows of C columns at a time in LDS, so that x and delta are read once: the deviations from the mean and the mixed
// errors, which need all rows of a column, come from there.  A quad of columns per lane; the C/4 lanes of a row side by
// side, 1024/C rows in flight per load of the workgroup, the next tile's asked for while a tile is summed up.  Bound by HBM: the whole
// call, 64 workers x 4 Mi columns on a torus (2.1 GB), 516 us (the kernel 490), without the look-ahead 575; 8 x 8 Mi 203 and 264; 256 x
// 272,474 226 and 256.  (The kernel below, which reads x twice and delta once more for every neighbour, mostly past the caches: 1595.)
// LDS: [x: n x C][delta: n x C][column sums: 1024/C x C, then the means: C][rowptr n+1][col nnz][coef nnz]
constexpr int kDiagGraphWords = 4096;
constexpr size_t diagnostics_lds(int n, int C, size_t nnz) {
    return (size_t)n * C * 8 + (size_t)1024 * 8 + (size_t)C * 8 + ((size_t)n + 1 + 2 * nnz) * 4;
}
template <int C>
__global__ void __launch_bounds__(256) diagnostics_tile_kernel(const float* x, const float* delta, uint64_t ld,
                                                               uint64_t tiles, int n, int nnz, const int32_t* __restrict__ graph, float eta,
                                                               double* __restrict__ out) {
    constexpr int LANES = C / 4, SIDE = 256 / LANES;             // lanes per row, rows side by side
    extern __shared__ __align__(16) uint8_t lds[];
    __shared__ double part[3][4];
    float4* lx = reinterpret_cast<float4*>(lds);
    float4* ldel = lx + (size_t)n * LANES;
    double* sums = reinterpret_cast<double*>(ldel + (size_t)n * LANES);       // SIDE x C
    double* means = sums + SIDE * C;
    int32_t* rowptr = reinterpret_cast<int32_t*>(means + C);
    const int32_t* col = rowptr + n + 1;
    const float* coef = reinterpret_cast<const float*>(col + nnz);
    for (int q = threadIdx.x; q < n + 1 + 2 * nnz; q += 256) rowptr[q] = graph[q];
    const int quad = threadIdx.x % LANES, side = threadIdx.x / LANES;
    double cons = 0.0, dsq_ = 0.0, mixed = 0.0;
    constexpr int OWN = 4;                                       // rows of a thread, at most
    float4 xs[OWN], ds[OWN];
    auto ask = [&](uint64_t tile) {                              // padding columns are zero: they add nothing
        const uint64_t j = tile * C + 4u * quad;
#pragma unroll
        for (int u = 0; u < OWN; ++u) {
            const int i = side + u * SIDE;
            if (i < n) {
                xs[u] = *reinterpret_cast<const float4*>(x + (uint64_t)i * ld + j);
                ds[u] = *reinterpret_cast<const float4*>(delta + (uint64_t)i * ld + j);
            }
        }
    };
    if (blockIdx.x < tiles) ask(blockIdx.x);
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        double sum[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < OWN; ++u) {
            const int i = side + u * SIDE;
            if (i < n) {
                lx[i * LANES + quad] = xs[u];
                ldel[i * LANES + quad] = ds[u];
                sum[0] += (double)xs[u].x; sum[1] += (double)xs[u].y; sum[2] += (double)xs[u].z; sum[3] += (double)xs[u].w;
                dsq_ += (double)ds[u].x * (double)ds[u].x + (double)ds[u].y * (double)ds[u].y + (double)ds[u].z * (double)ds[u].z + (double)ds[u].w * (double)ds[u].w;
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);                      // vmcnt(0): so that no load below waits for the one before it
        if (tile + gridDim.x < tiles) ask(tile + gridDim.x);     // in flight while this tile is summed up ...
        asm volatile("" ::: "memory");                           // ... and not asked for where they are used
#pragma unroll
        for (int c = 0; c < 4; ++c) sums[side * C + 4 * quad + c] = sum[c];
        __syncthreads();
        if (threadIdx.x < C) {
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < SIDE; ++q) s += sums[q * C + threadIdx.x];
            means[threadIdx.x] = s / n;
        }
        __syncthreads();
        const double m[4] = {means[4 * quad], means[4 * quad + 1], means[4 * quad + 2], means[4 * quad + 3]};
        for (int i = side; i < n; i += SIDE) {
            const float4 xv = lx[i * LANES + quad];
            const double d0 = (double)xv.x - m[0], d1 = (double)xv.y - m[1], d2 = (double)xv.z - m[2], d3 = (double)xv.w - m[3];
            cons += d0 * d0 + d1 * d1 + d2 * d2 + d3 * d3;
            double w0 = 0.0, w1 = 0.0, w2 = 0.0, w3 = 0.0;
            for (int e = rowptr[i]; e < rowptr[i + 1]; ++e) {
                const float4 dv = ldel[col[e] * LANES + quad];
                const double w = (double)coef[e];
                w0 += w * (double)dv.x; w1 += w * (double)dv.y; w2 += w * (double)dv.z; w3 += w * (double)dv.w;
            }
            w0 *= (double)eta; w1 *= (double)eta; w2 *= (double)eta; w3 *= (double)eta;
            mixed += w0 * w0 + w1 * w1 + w2 * w2 + w3 * w3;
        }
        __syncthreads();                                         // the tile is used up
    }
    add_diagnostics(cons, dsq_, mixed, part, out);
}

// Any n: a thread walks all rows of its columns (grid-stride).
__global__ void __launch_bounds__(256) diagnostics_kernel(const float* __restrict__ x, const float* __restrict__ delta, uint64_t ld,
                                                          uint64_t N, int n, const int32_t* __restrict__ rowptr,
                                                          const int32_t* __restrict__ col, const float* __restrict__ coef,
                                                          float eta, double* __restrict__ out) {
    __shared__ double part[3][4];
    double cons = 0.0, dsq_ = 0.0, mixed = 0.0;
    for (uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x; j < N; j += (uint64_t)gridDim.x * 256) {
        double sum = 0.0;
        for (int i = 0; i < n; ++i) {
            const double xv = x[(uint64_t)i * ld + j];
            const double dv = delta[(uint64_t)i * ld + j];
            sum += xv;
            dsq_ += dv * dv;
        }
        const double mean = sum / n;
        for (int i = 0; i < n; ++i) {                           // second pass: no cancellation
            const double dev = (double)x[(uint64_t)i * ld + j] - mean;
            cons += dev * dev;
            double m = 0.0;
            for (int e = rowptr[i]; e < rowptr[i + 1]; ++e) m += (double)coef[e] * (double)delta[(uint64_t)col[e] * ld + j];
            m *= (double)eta;
            mixed += m * m;
        }
    }
    add_diagnostics(cons, dsq_, mixed, part, out);
}

// Plain streaming copy, one 16-byte non-temporal load and store per lane, one-shot grid: the
// yardstick for the HBM bandwidth a trivial kernel reaches.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(256) copy_kernel(f32x4* __restrict__ dst, const f32x4* __restrict__ src, uint64_t n4) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n4) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

// The access mix of ds_step without its arithmetic: three 16-byte non-temporal loads and two stores per lane,
// in place (x += g, delta += g): what a streaming kernel of this shape reaches on the same GPU.
__global__ void __launch_bounds__(256) stream_3r2w_kernel(f32x4* __restrict__ x, f32x4* __restrict__ d, const f32x4* __restrict__ g, uint64_t n4) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n4) {
        const f32x4 gv = __builtin_nontemporal_load(g + i);
        const f32x4 xv = __builtin_nontemporal_load(x + i);
        const f32x4 dv = __builtin_nontemporal_load(d + i);
        __builtin_nontemporal_store(xv + gv, x + i);
        __builtin_nontemporal_store(dv + gv, d + i);
    }
}

// The same for the DCD-PSGD step, which has no second state array: two loads, one store.
__global__ void __launch_bounds__(256) stream_2r1w_kernel(f32x4* __restrict__ x, const f32x4* __restrict__ g, uint64_t n4) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n4) {
        const f32x4 gv = __builtin_nontemporal_load(g + i);
        const f32x4 xv = __builtin_nontemporal_load(x + i);
        __builtin_nontemporal_store(xv + gv, x + i);
    }
}

constexpr int kStaticMaxWorkers = 1024;                       // ds_step_static: what its declaration promises (nothing in the kernel ends there)

}  // namespace

extern "C" {

ds_status ds_step_static(const ds_config* cfg, float* x_dev, float* delta_dev, uint64_t ld, const float* g_dev, uint64_t g_ld,
                         void* msg_dev, uint64_t t, void* hip_stream, char* errbuf, uint64_t errbuf_len) {
    std::string err, warn;
    auto fail_with = [&](ds_status st, const std::string& m) {
        if (errbuf && errbuf_len) std::snprintf(errbuf, (size_t)errbuf_len, "%s", m.c_str());
        return st;
    };
    if (dsq::validate_config(cfg, err, &warn) != DS_OK) return fail_with(DS_EINVAL, err);
    const int kind = cfg->comp.kind;
    if (cfg->algo != DS_ALGO_DEEPSQUEEZE) return fail_with(DS_EINVAL, "ds_step_static serves Algorithm 1 (DS_ALGO_DEEPSQUEEZE) only");
    if (kind != DS_COMP_QUANT_MAXABS && kind != DS_COMP_SIGN_MEANABS && kind != DS_COMP_IDENTITY)
        return fail_with(DS_EINVAL, "ds_step_static serves the block quantiser, the sign compressor and the identity only "
                                    "(the other compressors need scratch memory in proportion to N)");
    if (cfg->topo != DS_TOPO_RING && cfg->topo != DS_TOPO_TORUS2D)
        return fail_with(DS_EINVAL, "ds_step_static builds W on the device: DS_TOPO_RING or DS_TOPO_TORUS2D only");
    if (cfg->n > kStaticMaxWorkers) return fail_with(DS_EINVAL, "ds_step_static serves up to 1024 workers");
    if (!x_dev || !delta_dev || !g_dev || !msg_dev) return fail_with(DS_EINVAL, "a device pointer is NULL");
    if ((ld & 3) || ld < (cfg->N + dsq::kPitchAlign - 1) / dsq::kPitchAlign * dsq::kPitchAlign)
        return fail_with(DS_EINVAL, "ld must be a multiple of 4 and at least N rounded up to a multiple of 4096");
    if (g_ld < cfg->N || (g_ld & 3)) return fail_with(DS_EINVAL, "g_ld must be >= N and a multiple of 4");
    if ((reinterpret_cast<uintptr_t>(x_dev) | reinterpret_cast<uintptr_t>(delta_dev) | reinterpret_cast<uintptr_t>(g_dev)) & 15)
        return fail_with(DS_EINVAL, "x_dev, delta_dev and g_dev must be 16-byte aligned");
    if (reinterpret_cast<uintptr_t>(msg_dev) & 3) return fail_with(DS_EINVAL, "msg_dev must be 4-byte aligned");
    const int deg = cfg->topo == DS_TOPO_RING ? 3 : 5;
    const int nnz = deg * cfg->n;
    static thread_local std::vector<dsq::TilePlan> plans;     // (kept for its memory only: a list per call)
    plans.clear();
    if (!dsq::choose_tile_plans(*cfg, nnz, plans, err)) return fail_with(DS_EINVAL, err);
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return fail_with(DS_EHIP, "no current HIP device");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // One launch: the kernel takes the step number by value and works the graph out for itself.  (A kernel of its own that
    // put both into device memory took 2.4 us and a second launch of a 12.4 us call: 8 workers x 4,645 parameters.)
    dsq::GivenStep a{};
    a.x = x_dev; a.delta = delta_dev; a.g = g_dev; a.msg = static_cast<uint8_t*>(msg_dev);
    a.ld = ld; a.g_ld = g_ld; a.N = cfg->N; a.msg_row_bytes = dsq::message_row_bytes(cfg);
    a.n = cfg->n; a.nnz = nnz;
    a.gamma = cfg->gamma; a.eta = cfg->eta;
    a.seed_lo = (uint32_t)cfg->seed; a.seed_hi = (uint32_t)(cfg->seed >> 32);
    a.t = (uint32_t)t;
    a.topo = cfg->topo; a.torus_rows = cfg->torus_rows; a.torus_cols = cfg->torus_cols;
    const dsq::TilePlan& plan = plans.front();
    if (!plan.launch_given) return fail_with(DS_EINVAL, "internal: the first launch shape has no form that is given its graph");
    plan.launch_given(a, plan.rows_per_wave, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail_with(DS_EHIP, std::string("launching the step failed: ") + hipGetErrorString(e));
    if (errbuf && errbuf_len) std::snprintf(errbuf, (size_t)errbuf_len, "%s", warn.c_str());
    return DS_OK;
}

ds_status ds_workload_gradient(const ds_workload* w, uint64_t t, const float* x_dev, uint64_t x_ld, float* g_dev,
                               uint64_t g_ld, void* hip_stream) {
    if (!w || !g_dev || w->n < 1 || w->N < 1 || w->N > 0xFFFFFFF0ull || g_ld < w->N) return DS_EINVAL;
    if (w->kind < DS_GRAD_NORMAL || w->kind > DS_GRAD_QUADRATIC || !std::isfinite(w->scale)) return DS_EINVAL;
    if (w->kind == DS_GRAD_QUADRATIC && (!x_dev || x_ld < w->N)) return DS_EINVAL;
    return dsq::launch_workload_gradient(*w, t, x_dev, x_ld, g_dev, g_ld, static_cast<hipStream_t>(hip_stream));
}

ds_status ds_bench_stream(void* x_dev, void* delta_dev, const void* g_dev, uint64_t bytes, void* hip_stream) {
    if (!x_dev || !g_dev || (bytes & 15) ||
        ((reinterpret_cast<uintptr_t>(x_dev) | reinterpret_cast<uintptr_t>(delta_dev) | reinterpret_cast<uintptr_t>(g_dev)) & 15))
        return DS_EINVAL;
    const uint64_t n4 = bytes / 16;
    if (n4 == 0) return DS_OK;
    if (n4 > 0xFFFFFF00ull) return DS_EINVAL;
    if (!delta_dev) {
        hipLaunchKernelGGL(stream_2r1w_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                           static_cast<f32x4*>(x_dev), static_cast<const f32x4*>(g_dev), n4);
        return hipGetLastError() == hipSuccess ? DS_OK : DS_EHIP;
    }
    hipLaunchKernelGGL(stream_3r2w_kernel, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<f32x4*>(x_dev), static_cast<f32x4*>(delta_dev), static_cast<const f32x4*>(g_dev), n4);
    return hipGetLastError() == hipSuccess ? DS_OK : DS_EHIP;
}

ds_status ds_bench_copy(void* dst_dev, const void* src_dev, uint64_t bytes, void* hip_stream) {
    if (!dst_dev || !src_dev || (bytes & 15) || ((reinterpret_cast<uintptr_t>(dst_dev) | reinterpret_cast<uintptr_t>(src_dev)) & 15))
        return DS_EINVAL;
    const uint64_t n4 = bytes / 16;
    if (n4 == 0) return DS_OK;
    if (n4 > 0xFFFFFF00ull) return DS_EINVAL;              // one work-item per 16 bytes, fewer than 2^32 of them
    const unsigned blocks = (unsigned)((n4 + 255) / 256);
    hipLaunchKernelGGL(copy_kernel, dim3(blocks), dim3(256), 0, static_cast<hipStream_t>(hip_stream),
                       static_cast<f32x4*>(dst_dev), static_cast<const f32x4*>(src_dev), n4);
    return hipGetLastError() == hipSuccess ? DS_OK : DS_EHIP;
}

ds_status ds_init(const ds_config* cfg, ds_handle** out) { return ds_init_ex(cfg, nullptr, nullptr, 0, out); }

ds_status ds_init_ex(const ds_config* cfg, const ds_plan_request* plan, char* errbuf, uint64_t errbuf_len, ds_handle** out) {
    if (errbuf && errbuf_len) errbuf[0] = 0;
    if (!out) return DS_EINVAL;
    *out = nullptr;
    ds_handle* h = new (std::nothrow) ds_handle();
    if (!h) return DS_ENOMEM;
    auto bail = [&](ds_status st, const std::string& why) {
        if (errbuf && errbuf_len) std::snprintf(errbuf, (size_t)errbuf_len, "%s", why.c_str());
        release(h);
        return st;
    };
    ds_plan_request want{};                                 // all automatic
    want.tile_plan = -1; want.pitch_skew = -1; want.autotune = 1;
    if (plan) {
        want = *plan;
        if (want.variant < 0 || want.variant > 3) return bail(DS_EINVAL, "plan: variant must be 0 (automatic), 1 (row-streaming), 2 (no resident kernel) or 3 (resident kernel without patience)");
        if (want.pitch_skew < -1 || want.pitch_skew > (int64_t)kMaxPitchSkew || (want.pitch_skew > 0 && (want.pitch_skew & 3)))
            return bail(DS_EINVAL, "plan: pitch_skew must be -1 (automatic) or a multiple of 4 up to 12288");
    }

    std::string err, warn;
    if (dsq::validate_config(cfg, err, &warn) != DS_OK) return bail(DS_EINVAL, err);
    h->cfg = *cfg;
    if (dsq::build_graph(cfg, h->graph, err) != DS_OK) return bail(DS_EINVAL, err);
    h->cfg.W_rowptr = nullptr; h->cfg.W_col = nullptr; h->cfg.W_val = nullptr;   // the copy lives in graph
    const uint64_t base_ld = (cfg->N + dsq::kPitchAlign - 1) / dsq::kPitchAlign * dsq::kPitchAlign;
    h->ld = base_ld + kMaxPitchSkew;                       // allocation pitch; the working pitch is fixed below
    h->msg_row_bytes = dsq::message_row_bytes(cfg);

    const bool sparse_pairs = cfg->comp.kind == DS_COMP_TOPK || cfg->comp.kind == DS_COMP_GSPAR;   // (column, value) messages
    const bool tiled = !sparse_pairs && cfg->comp.kind != DS_COMP_QUANT_L2NORM;
    // small problems of these compressors: a whole step in one launch
    if (sparse_pairs || cfg->comp.kind == DS_COMP_QUANT_L2NORM) h->share = want.variant == 2 ? 0 : sparse_pairs ? dsq::topk_resident_share(*cfg) : dsq::l2q_resident_share(*cfg);
    h->resident = h->share != 0;
    if (want.variant == 3) h->share = 0;                   // the first meeting is called off at once: nothing waits
    if (sparse_pairs) {
        h->plan_name = cfg->comp.kind == DS_COMP_GSPAR ? (h->resident ? "gspar/resident" : "gspar/sift-scan-write") : h->resident ? "topk/resident" : "topk/radix-select";
    } else if (cfg->comp.kind == DS_COMP_QUANT_L2NORM) {
        h->plan_name = h->resident ? "l2norm/resident" : "l2norm/speculative-codes";
        if (!h->resident) h->msg_half = (uint64_t)cfg->n * h->msg_row_bytes;     // the first pass writes codes while the old ones are still read
    } else {
        // The row-streaming variant of the block compressors on request; it is also what serves a number of workers whose
        // codes do not fit in LDS, and what is faster for some sizes (streams_faster)
        dsq::TilePlan sp;
        const bool can_stream = dsq::stream_plan(h->cfg, sp);
        const bool fits = dsq::choose_tile_plans(h->cfg, (int)h->graph.col.size(), h->tile_candidates, err);
        const bool many_rows = want.tile_plan < 0 && streams_faster(*cfg, h->graph.col.size());
        std::vector<dsq::TilePlan> teams;
        if (can_stream && (!fits || want.variant == 1 || many_rows)) {
            h->tile_candidates.assign(1, sp);
            h->msg_half = (uint64_t)cfg->n * h->msg_row_bytes;
            dsq::team_plans(h->cfg, h->graph, teams);
            if (want.tile_plan > 0 && (size_t)want.tile_plan <= teams.size()) h->team = teams[(size_t)want.tile_plan - 1];
            else if (want.tile_plan != 0 && whole_steps_faster(*cfg, sp)) h->team = best_team(teams, *cfg);
        } else if (!fits) {
            return bail(DS_EINVAL, err);
        } else {
            dsq::team_plans(h->cfg, h->graph, teams);
            const size_t pinnable = h->tile_candidates.size() + teams.size();
            if (want.tile_plan >= 0 && (size_t)want.tile_plan < pinnable)
                for (const dsq::TilePlan& p : teams) h->tile_candidates.push_back(p);
            else if (!teams.empty() && teams_faster(*cfg, h->tile_candidates.front()))
                h->tile_candidates.assign(1, best_team(teams, *cfg));
        }
        h->impatient = want.variant == 3;
        h->tile = h->tile_candidates.front();
        // a pinned candidate launch shape (tests walk through all of them; an index past the end leaves the choice automatic)
        if (!h->tile.streaming && want.tile_plan >= 0 && (size_t)want.tile_plan < h->tile_candidates.size()) {
            h->tile = h->tile_candidates[(size_t)want.tile_plan];
            h->tile_candidates.assign(1, h->tile);
        }
    }

    hipError_t e = hipGetDevice(&h->device);
    if (e != hipSuccess) return bail(DS_EHIP, std::string("no HIP device: ") + hipGetErrorString(e));
    const size_t state_bytes = (size_t)cfg->n * h->ld * sizeof(float);
    const size_t nnz = h->graph.col.size();
    const size_t msg_bytes = (size_t)cfg->n * h->msg_row_bytes * (h->msg_half ? 2 : 1);
    // rowptr | col | coef as one contiguous array of 32-bit words
    hipError_t errs[5] = {
        hipMalloc(&h->x, state_bytes), hipMalloc(&h->delta, state_bytes), hipMalloc(&h->msg, msg_bytes ? msg_bytes : 4),
        hipMalloc(&h->d_rowptr, (cfg->n + 1 + 2 * nnz) * sizeof(int32_t)), hipMalloc(&h->d_t, dsq::kStepCells * sizeof(unsigned long long))};
    for (hipError_t ee : errs)
        if (ee != hipSuccess) { (void)hipGetLastError(); return bail(ee == hipErrorOutOfMemory ? DS_ENOMEM : DS_EHIP, std::string("hipMalloc: ") + hipGetErrorString(ee)); }
    h->d_col = h->d_rowptr + cfg->n + 1;
    h->d_coef = reinterpret_cast<float*>(h->d_col + nnz);
    bool ok = hipMemset(h->x, 0, state_bytes) == hipSuccess && hipMemset(h->delta, 0, state_bytes) == hipSuccess &&
              hipMemset(h->msg, 0, msg_bytes ? msg_bytes : 4) == hipSuccess &&
              hipMemset(h->d_t, 0, dsq::kStepCells * sizeof(unsigned long long)) == hipSuccess &&
              hipMemset(h->d_t + 2, 0xFF, sizeof(unsigned long long)) == hipSuccess &&   // tag of the keep counts: none yet
              hipMemcpy(h->d_rowptr, h->graph.rowptr.data(), (cfg->n + 1) * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(h->d_col, h->graph.col.data(), nnz * sizeof(int32_t), hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(h->d_coef, h->graph.coef.data(), nnz * sizeof(float), hipMemcpyHostToDevice) == hipSuccess &&
              hipDeviceSynchronize() == hipSuccess;
    if (!ok) return bail(DS_EHIP, "device initialisation failed");
    if (const size_t bytes = team_bytes(h)) {
        if (hipMalloc(&h->d_team, bytes) != hipSuccess || hipMemset(h->d_team, 0, bytes) != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
            (void)hipGetLastError();
            return bail(DS_ENOMEM, "allocating the arrival counters failed");
        }
    }
    if (cfg->comp.kind == DS_COMP_RAND_SPARSE) {
        h->nsweeps = (cfg->N + dsq::kSweep - 1) / dsq::kSweep;
        h->ngroups = (h->nsweeps + 15) / 16;
        const size_t words = (size_t)cfg->n * (3 * h->nsweeps + h->ngroups) + (size_t)cfg->n + 1;
        if (hipMalloc(&h->d_keep, words * sizeof(uint32_t)) != hipSuccess || hipMemset(h->d_keep, 0, words * sizeof(uint32_t)) != hipSuccess ||
            hipDeviceSynchronize() != hipSuccess) {
            return bail(DS_ENOMEM, "allocating the random sparsifier's offsets failed");
        }
    }

    // working row pitch: pinned by the caller, or timed per candidate for large tile-kernel problems; everything
    // else takes the default
    uint64_t skew = dsq::kPitchSkew;
    if (want.pitch_skew >= 0) {
        skew = (uint64_t)want.pitch_skew;
    } else if (want.autotune && tiled && !h->tile.streaming && (uint64_t)cfg->n * cfg->N >= (32ull << 20)) {
        skew = autotune(h, base_ld, state_bytes, msg_bytes);
    }
    h->ld = base_ld + skew;
    if (tiled)
        h->plan_name = std::string(cfg->algo == DS_ALGO_DCD_PSGD ? "dcd/" : cfg->algo == DS_ALGO_CHOCO_SGD ? "choco/" : "") + h->tile.name + "/" +
                       std::to_string(h->tile.sweeps) + "sweeps";
    h->plan_name += "/pitch+" + std::to_string(skew);

    if (sparse_pairs) {
        const ds_status st = dsq::topk_create(h->cfg, h->ld, h->resident, want.variant == 3, &h->topk, err);
        if (st != DS_OK) return bail(st, err);
    }
    if (cfg->comp.kind == DS_COMP_QUANT_L2NORM) {
        const ds_status st = dsq::l2q_create(h->cfg, h->ld, h->resident, want.variant == 3, &h->l2q, err);
        if (st != DS_OK) return bail(st, err);
    }
    h->err = warn;
    if (errbuf && errbuf_len) std::snprintf(errbuf, (size_t)errbuf_len, "%s", warn.c_str());
    *out = h;
    return DS_OK;
}

ds_status ds_step(ds_handle* h, const float* g_dev, uint64_t g_ld, void* hip_stream) {
    if (!h) return DS_EINVAL;
    if (!g_dev) return fail(h, DS_EINVAL, "g_dev is NULL");
    if (g_ld < h->cfg.N || (g_ld & 3)) return fail(h, DS_EINVAL, "g_ld must be >= N and a multiple of 4");
    if (reinterpret_cast<uintptr_t>(g_dev) & 15) return fail(h, DS_EINVAL, "g_dev must be 16-byte aligned");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != h->device)
        return fail(h, DS_ESTATE, "the current HIP device is not the one the handle was created on");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // Some plans leave part of a step to be done when x and delta are asked for, and whether there is such a part is known here only
    // as long as no graph runs steps.
    if (defers(h) && (!h->unseen || h->asked)) {
        const bool captured = capturing(stream);
        h->unseen |= captured;
        // Was x lent for the graph that this step is part of?  On the stream of the last step that would have been seen; on another one, or
        // with no step before it, the lending found nothing to enqueue, or enqueued it outside the graph.  Then the replays have to
        // find x complete as they begin: this step completes it itself, and so do all others that may come in between.
        if (h->asked && captured && (!h->stepped || h->last_stream != stream)) h->completes = true;
    }
    h->asked = false;

    h->run += 1;
    if (h->topk) {
        const ds_status st = dsq::topk_step(h->topk, topk_args(h, g_dev, g_ld), seated(h, stream), stream);
        if (st != DS_OK) return fail(h, st, "launching the sparsifying step failed");
    } else if (h->cfg.comp.kind == DS_COMP_QUANT_L2NORM) {
        const ds_status st = dsq::l2q_step(h->l2q, l2_args(h, g_dev, g_ld), seated(h, stream), stream);
        if (st != DS_OK) return fail(h, st, "launching the norm-rescaled step failed");
    } else {
        if (h->cfg.comp.kind == DS_COMP_RAND_SPARSE) {
            const dsq::TileArgs a = tile_args(h, g_dev, g_ld);
            uint32_t* groups = h->d_keep + (size_t)h->cfg.n * h->nsweeps;
            uint32_t* prev = groups + (size_t)h->cfg.n * h->ngroups;
            dsq::launch_keep_offsets(a, h->d_keep, groups, prev, prev + h->cfg.n, stream);
        }
        if (h->tile.streaming) {
            // Where x is read after every step, a step is taken whole; where several follow one another, each leaves its gossip
            // sum to the next one's pass, which reads x anyway.  A step that is captured may be replayed between any others:
            // the way of the first one that is captured is the way of all that follow, and that of a graph of steps alone, whose
            // replays may follow one another, is to stream (256 x 272,474: 246 us a replay, whole 291).
            const bool able = h->team.team && h->complete;
            bool whole = able && h->run == 1 && h->period == 1;
            if (h->captured == ds_handle::kFree && h->unseen) h->captured = able && h->completes ? ds_handle::kWhole : ds_handle::kStreamed;
            if (h->captured != ds_handle::kFree) whole = h->captured == ds_handle::kWhole;
            const dsq::TilePlan& plan = whole ? h->team : h->tile;
            launch_plan(h, plan, g_dev, g_ld, stream);
            h->complete = whole;
        } else {
            launch_plan(h, h->tile, g_dev, g_ld, stream);
        }
    }
    DSQ_HIP(h, hipGetLastError());
    h->t += 1;
    h->stepped = true;
    h->last_stream = stream;
    if (h->completes && apply_deferred(h) != DS_OK) return fail(h, DS_EHIP, "applying the tail of the step failed");
    return DS_OK;
}

ds_status ds_set_mixing(ds_handle* h, const int32_t* W_rowptr, const int32_t* W_col, const float* W_val) {
    if (!h) return DS_EINVAL;
    ds_config probe = h->cfg;
    probe.topo = DS_TOPO_CSR;
    probe.W_rowptr = W_rowptr; probe.W_col = W_col; probe.W_val = W_val;
    std::string err;
    if (dsq::validate_config(&probe, err, nullptr) != DS_OK) return fail(h, DS_EINVAL, err);
    dsq::Graph g;
    if (dsq::build_graph(&probe, g, err) != DS_OK) return fail(h, DS_EINVAL, err);
    const size_t nnz = g.col.size();
    dsq::TilePlan tile = h->tile, team = h->team;
    if (!h->topk && !h->l2q && !h->tile.streaming) {
        // the launch shape was chosen for the old graph; the new CSR only has to fit in LDS next to the codes
        std::vector<dsq::TilePlan> plans;
        if (!dsq::choose_tile_plans(h->cfg, (int)nnz, plans, err)) return fail(h, DS_EINVAL, err);
        if (tile.team && !dsq::fit_team(g, tile)) tile = plans.front();
    }
    // (Where graphs may run whole steps all others have to be whole too: with the LDS of the old W, and rows that need more finished from memory.)
    if (team.team && !dsq::fit_team(g, team) && h->captured != ds_handle::kWhole) team = dsq::TilePlan();
    // a deferred tail belongs to the old W: apply it first
    if (flush_deferred(h) != DS_OK) return fail(h, DS_EHIP, "applying the deferred tail of the last step failed");
    DSQ_HIP(h, hipStreamSynchronize(h->last_stream));
    // same number of stored entries: overwrite in place, so that the device addresses (and a HIP graph captured
    // from ds_step with them) stay valid
    const bool in_place = nnz == h->graph.col.size();
    int32_t* packed = h->d_rowptr;
    if (!in_place) DSQ_HIP(h, hipMalloc(&packed, (h->cfg.n + 1 + 2 * nnz) * sizeof(int32_t)));
    hipError_t e = hipMemcpy(packed, g.rowptr.data(), (h->cfg.n + 1) * sizeof(int32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(packed + h->cfg.n + 1, g.col.data(), nnz * sizeof(int32_t), hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(packed + h->cfg.n + 1 + nnz, g.coef.data(), nnz * sizeof(float), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (!in_place) (void)hipFree(packed);
        return hip_fail(h, e, "hipMemcpy(W)");
    }
    if (!in_place) (void)hipFree(h->d_rowptr);
    h->d_rowptr = packed;
    h->d_col = packed + h->cfg.n + 1;
    h->d_coef = reinterpret_cast<float*>(h->d_col + nnz);
    h->graph = g;
    h->tile = tile;
    h->team = team;
    h->cfg.topo = DS_TOPO_CSR;
    return DS_OK;
}

ds_status ds_set_rates(ds_handle* h, float gamma, float eta) {
    if (!h) return DS_EINVAL;
    if (!std::isfinite(gamma) || !std::isfinite(eta)) return fail(h, DS_EINVAL, "gamma and eta must be finite");
    // a deferred tail was computed for the old eta
    if (flush_deferred(h) != DS_OK) return fail(h, DS_EHIP, "applying the deferred tail of the last step failed");
    h->cfg.gamma = gamma;
    h->cfg.eta = eta;
    h->err = (eta > 0.5f) ? "warning: eta > 1/2, outside the range of the paper's Theorem 1 (W_eff may not be PSD)" : "";
    return DS_OK;
}

// Dense host array <-> pitched device rows.  Rows of more than 1 GiB go one by one (2-D copies of such widths
// are not something every runtime version handles).
static hipError_t copy_rows(void* dst, size_t dst_pitch, const void* src, size_t src_pitch, size_t row_bytes, int rows, hipMemcpyKind kind) {
    if (row_bytes <= (1ull << 30)) return hipMemcpy2D(dst, dst_pitch, src, src_pitch, row_bytes, rows, kind);
    for (int i = 0; i < rows; ++i) {
        const hipError_t e = hipMemcpy(static_cast<char*>(dst) + (size_t)i * dst_pitch, static_cast<const char*>(src) + (size_t)i * src_pitch,
                                       row_bytes, kind);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

ds_status ds_read_state(ds_handle* h, float* x_host, float* delta_host) {
    if (!h) return DS_EINVAL;
    if (!x_host && !delta_host) return fail(h, DS_EINVAL, "nothing to read");
    if (flush_deferred(h) != DS_OK) return fail(h, DS_EHIP, "applying the deferred tail of the last step failed");
    DSQ_HIP(h, hipStreamSynchronize(h->last_stream));
    const size_t row = h->cfg.N * sizeof(float), pitch = h->ld * sizeof(float);
    if (x_host) DSQ_HIP(h, copy_rows(x_host, row, h->x, pitch, row, h->cfg.n, hipMemcpyDeviceToHost));
    if (delta_host) DSQ_HIP(h, copy_rows(delta_host, row, h->delta, pitch, row, h->cfg.n, hipMemcpyDeviceToHost));
    return DS_OK;
}

ds_status ds_write_state(ds_handle* h, const float* x_host, const float* delta_host, uint64_t t) {
    if (!h) return DS_EINVAL;
    if (flush_deferred(h) != DS_OK) return fail(h, DS_EHIP, "applying the deferred tail of the last step failed");
    DSQ_HIP(h, hipStreamSynchronize(h->last_stream));
    const size_t row = h->cfg.N * sizeof(float), pitch = h->ld * sizeof(float);
    if (x_host) DSQ_HIP(h, copy_rows(h->x, pitch, x_host, row, row, h->cfg.n, hipMemcpyHostToDevice));
    if (delta_host) DSQ_HIP(h, copy_rows(h->delta, pitch, delta_host, row, row, h->cfg.n, hipMemcpyHostToDevice));
    const unsigned long long t64 = t;
    DSQ_HIP(h, hipMemcpy(h->d_t, &t64, sizeof(t64), hipMemcpyHostToDevice));
    DSQ_HIP(h, hipDeviceSynchronize());
    h->t = t;
    return DS_OK;
}

// Plans with two message buffers (row-streaming block kernels, norm-rescaled codes): a step leaves the number of
// the buffer it wrote in cell 4 of the step cells.  The caller has synchronised.
static ds_status last_message_buffer(ds_handle* h, uint8_t** out) {
    *out = h->msg;
    if (!h->msg_half) return DS_OK;
    unsigned long long half = 0;
    DSQ_HIP(h, hipMemcpy(&half, h->d_t + 4, sizeof(half), hipMemcpyDeviceToHost));
    if (half & 1ull) *out = h->msg + h->msg_half;
    return DS_OK;
}

ds_status ds_read_messages(ds_handle* h, void* host_buf, uint64_t cap, uint64_t* bytes) {
    if (!h) return DS_EINVAL;
    if (!h->stepped) return fail(h, DS_ESTATE, "no step has been taken yet");
    const uint64_t total = h->msg_row_bytes * (uint64_t)h->cfg.n;
    if (bytes) *bytes = total;
    if (!host_buf || cap < total) return fail(h, DS_EINVAL, "message buffer too small");
    DSQ_HIP(h, hipStreamSynchronize(h->last_stream));
    uint8_t* src = nullptr;
    if (last_message_buffer(h, &src) != DS_OK) return DS_EHIP;
    DSQ_HIP(h, hipMemcpy(host_buf, src, total, hipMemcpyDeviceToHost));
    if (h->cfg.comp.kind == DS_COMP_GSPAR) {
        bool over = false;
        if (dsq::gspar_overflowed(h->topk, h->last_stream, &over) != DS_OK) return DS_EHIP;
        if (over) return fail(h, DS_ESTATE, "a worker kept more elements than its message has room for: the messages since then are cut short");
    }
    if (h->d_keep) {
        uint32_t overflow = 0;
        DSQ_HIP(h, hipMemcpy(&overflow, h->d_keep + (size_t)h->cfg.n * (h->nsweeps + h->ngroups) + h->cfg.n, sizeof(overflow), hipMemcpyDeviceToHost));
        if (overflow) return fail(h, DS_ESTATE, "a worker kept more values than its message has room for (x and delta are unaffected)");
    }
    return DS_OK;
}

ds_status ds_state_ptrs(ds_handle* h, float** x_dev, float** delta_dev, uint64_t* ld) {
    if (!h) return DS_EINVAL;
    // top-k keeps the sparse part of the last gossip update pending; complete x before lending it
    if (defers(h)) h->asked = !(h->stepped && capturing(h->last_stream));
    if (flush_deferred(h) != DS_OK) return fail(h, DS_EHIP, "applying the deferred tail of the last step failed");
    if (x_dev) *x_dev = h->x;
    if (delta_dev) *delta_dev = h->delta;
    if (ld) *ld = h->ld;
    return DS_OK;
}

ds_status ds_message_ptr(ds_handle* h, void** msg_dev, uint64_t* bytes) {
    if (!h) return DS_EINVAL;
    uint8_t* src = h->msg;
    if (h->msg_half) {                                       // which of the two buffers is the last step's: ask the device
        DSQ_HIP(h, hipStreamSynchronize(h->last_stream));
        if (last_message_buffer(h, &src) != DS_OK) return DS_EHIP;
    }
    if (msg_dev) *msg_dev = src;
    if (bytes) *bytes = h->msg_row_bytes * (uint64_t)h->cfg.n;
    return DS_OK;
}

ds_status ds_diagnostics(ds_handle* h, double* out4) {
    if (!h || !out4) return DS_EINVAL;
    if (flush_deferred(h) != DS_OK) return fail(h, DS_EHIP, "applying the deferred tail of the last step failed");
    DSQ_HIP(h, hipStreamSynchronize(h->last_stream));
    double* d_out = nullptr;
    double cells[kDiagCells * kDiagStride];
    DSQ_HIP(h, hipMalloc(&d_out, sizeof(cells)));
    hipError_t e = hipMemset(d_out, 0, sizeof(cells));
    if (e == hipSuccess) {
        const size_t nnz = h->graph.col.size();
        const bool graph_fits = (size_t)h->cfg.n + 1 + 2 * nnz <= (size_t)kDiagGraphWords;
        // 64 columns a tile up to 64 rows, 16 up to 256: 32 KB for the rows either way, so that three workgroups or more
        // share a compute unit and one's loads run beside another's sums
        auto tiles = [&](int C) { return (h->cfg.N + C - 1) / C; };
        auto grid = [](uint64_t t) { return dim3((unsigned)(t < 4096 ? t : 4096)); };
        const uint64_t want = (h->cfg.N + 255) / 256;
        const unsigned blocks = (unsigned)(want < (1u << 20) ? want : (1u << 20));
        if (graph_fits && h->cfg.n <= 64)
            hipLaunchKernelGGL(diagnostics_tile_kernel<64>, grid(tiles(64)), dim3(256), diagnostics_lds(h->cfg.n, 64, nnz), nullptr, h->x, h->delta,
                               h->ld, tiles(64), h->cfg.n, (int)nnz, h->d_rowptr, h->cfg.eta, d_out);
        else if (graph_fits && h->cfg.n <= 256)
            hipLaunchKernelGGL(diagnostics_tile_kernel<16>, grid(tiles(16)), dim3(256), diagnostics_lds(h->cfg.n, 16, nnz), nullptr, h->x, h->delta,
                               h->ld, tiles(16), h->cfg.n, (int)nnz, h->d_rowptr, h->cfg.eta, d_out);
        else
            hipLaunchKernelGGL(diagnostics_kernel, dim3(blocks), dim3(256), 0, nullptr, h->x, h->delta, h->ld, h->cfg.N, h->cfg.n,
                               h->d_rowptr, h->d_col, h->d_coef, h->cfg.eta, d_out);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpy(cells, d_out, sizeof(cells), hipMemcpyDeviceToHost);
    (void)hipFree(d_out);
    if (e != hipSuccess) return hip_fail(h, e, "ds_diagnostics");
    for (int q = 0; q < 3; ++q) {
        double sum = 0.0;
        for (int c = 0; c < kDiagCells; ++c) sum += cells[c * kDiagStride + q];
        out4[q] = sum;
    }
    out4[3] = (double)(h->msg_row_bytes * (uint64_t)h->cfg.n);
    return DS_OK;
}

ds_status ds_topk_candidate_rows(ds_handle* h, uint32_t* count) {
    if (!h || !count) return DS_EINVAL;
    *count = 0;
    if (!h->topk && !h->l2q) return DS_OK;
    if (!h->stepped) return fail(h, DS_ESTATE, "no step has been taken yet");
    if (h->l2q) return dsq::l2q_speculated_rows(h->l2q, h->last_stream, count);
    return dsq::topk_candidate_rows(h->topk, h->last_stream, count);
}

uint64_t ds_step_count(const ds_handle* h) {
    // the device counter is the authority: replays of a captured graph advance it without the host seeing them
    if (!h) return 0;
    unsigned long long t64 = h->t;
    if (hipStreamSynchronize(h->last_stream) == hipSuccess)
        (void)hipMemcpy(&t64, h->d_t, sizeof(t64), hipMemcpyDeviceToHost);
    return t64;
}

const char* ds_plan_name(const ds_handle* h) { return h ? h->plan_name.c_str() : ""; }

const char* ds_last_error(const ds_handle* h) { return h ? h->err.c_str() : "handle is NULL"; }

void ds_destroy(ds_handle* h) {
    if (!h) return;
    (void)hipDeviceSynchronize();
    release(h);
}

}  // extern "C"
