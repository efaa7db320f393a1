// What the two forms of the sparsifying step of libdsq share -- the chain of launches for large problems
// (dsq_topk_kernels.hip) and the one launch for small ones (dsq_topk_resident.hip): a worker row's book-keeping, the
// order of magnitudes, the keep decisions of GSpar and the guess of the next step's threshold.
#pragma once

#include "dsq_internal.h"
#include "dsq_philox.h"

namespace dsq {

struct TopkRow {
    uint32_t prefix1, need1;   // full mode: level-1 bin holding the threshold; how many to take inside it
    uint32_t prefix2, need2;   // full mode: 22-bit prefix of the threshold key; how many to take among its matches
    uint32_t tau, r_tie;       // threshold key; number of elements with key == tau to take (lowest indices)
    uint32_t total;            // number of selected elements found by the scan (must equal k)
    uint32_t tlo;              // candidate threshold key for the next first pass (0xffffffff: collect nothing)
    uint32_t cand_mode;        // 1: this step's select runs on the candidate slots
    uint32_t overflow;         // a slot overflowed in this step's first pass
    uint32_t cand_total;       // candidates collected in this step
    uint32_t tlo_used;         // the threshold this step's first pass collected with
    uint32_t tau_prev;         // threshold key of the previous step (0xffffffff: none yet)
    uint32_t bin_lo;           // candidate mode: first key of the histogram bin that holds the threshold
    uint32_t bin_need;         //                 how many elements to take inside that bin
    uint32_t list_count;       //                 elements of that bin listed so far by topk_bin_collect
    float drift_prev;          // last step's movement of |tau| as a float (for the forecast of the next threshold)
    uint32_t forecast;         // the threshold the next step is expected to have
    uint32_t shift;            // one-launch form: the next step counts candidates in bins of 2^shift keys above tlo
    uint32_t tied;             // one-launch form: more keys equal the threshold than are looked up one by one
    float lambda;              // GSpar: this step's k / sum |v|
    float lambda_hi;           // GSpar: the upper bound the NEXT first pass collects with (0: none)
    uint32_t gs_mode;          // GSpar: 1 = this step's kept elements are among those its first pass collected
    uint32_t gs_need_count;    // GSpar: chunks of the row that must decide from v itself (0: gs_count_dense has nothing to do)
    uint32_t gs_need_write;    // GSpar: chunks that kept more than a slot holds (0: gs_write_dense has nothing to do)
    uint32_t gs_total;         // GSpar: pairs in the row's last message (what a shorter message must clear behind it)
};

// The one-launch form of a step, on the rows of the state that owns it.
struct SparseResidentState;
uint32_t sparse_resident_share(const ds_config& cfg);
// impatient: the kernel's first meeting calls itself off at once (tests of what follows then).
ds_status sparse_resident_create(const ds_config& cfg, bool impatient, TopkRow* rows, uint32_t* overflow, SparseResidentState** out);
void sparse_resident_destroy(SparseResidentState* st);
ds_status sparse_resident_step(SparseResidentState* st, const TopkArgs& a, hipStream_t stream);

namespace {

constexpr float TK_TARGET = 1.6f;            // candidates aimed at, in units of k
constexpr int BINS1 = 2048, SHIFT1 = 20;     // level 1: key bits 30..20

__device__ __forceinline__ uint32_t key_of(float v) { return __float_as_uint(v) & 0x7FFFFFFFu; }

constexpr uint32_t kGsparStreamTag = 0x47535052u;            // GSpar: 4th counter word of the mask's random stream

// The keep decisions of four adjacent columns of worker `row`.
__device__ __forceinline__ uint32_t gs_keep4(const TopkArgs& a, int row, uint64_t j, uint32_t t_lo, float lambda, const float4& v) {
    uint32_t rnd[4];
    philox4x32_10((uint32_t)(j >> 2), (uint32_t)row, t_lo, kGsparStreamTag, a.seed_lo, a.seed_hi, rnd);
    const float vv[4] = {v.x, v.y, v.z, v.w};
    uint32_t keep = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float p = lambda * fabsf(vv[c]);
        const float u = (float)(rnd[c] >> 8) * (1.0f / 16777216.0f);
        if (j + c < a.N && u < p) keep |= 1u << c;
    }
    return keep;
}

// ---- where to collect candidates in the next step ------------------------------------------------
// Near the threshold the number of keys above a level falls roughly exponentially with the level.  With
// d = tau - tlo the distance that caught ratio * k candidates this step, d* = d ln(target) / ln(ratio) would
// have caught target * k; the next level is (forecast of the next tau) - d*.  The forecast is made on |tau|
// as a float (keys are only piecewise linear in the magnitude: the slope halves at every power of two): the
// last movement repeated, or three quarters of it while the movement still changes by more than a quarter
// from step to step (early in a run delta grows fast and then settles).  Without usable candidates (full
// mode) a fixed distance of two million keys (a quarter of a binade) is taken.  Only speed depends on this
// guess; a bad one sends the row through the exact full path.
__device__ __forceinline__ uint32_t next_candidate_threshold(TopkRow& r, uint32_t tau, uint32_t k, float target = TK_TARGET) {
    const float d0 = 2.f * (float)(1u << SHIFT1);
    float dist = d0;
    if (r.cand_mode && r.cand_total > k && tau > r.tlo_used) {
        const float ratio = (float)r.cand_total / (float)k;
        dist = (float)(tau - r.tlo_used) * (logf(target) / logf(ratio));
        dist = fminf(fmaxf(dist, 65536.f), 4.f * d0);
    }
    const float mag = __uint_as_float(tau);
    float move = 0.f, next = mag;
    if (r.tau_prev != 0xFFFFFFFFu) {
        move = mag - __uint_as_float(r.tau_prev);
        const bool steady = fabsf(move - r.drift_prev) <= 0.25f * fabsf(move);
        next = mag + (steady ? move : 0.75f * move);
        if (!(next > 0.f) || !(next < 3.0e38f)) next = mag;
    }
    r.drift_prev = move;
    r.forecast = __float_as_uint(next);
    const float t = (float)__float_as_uint(next) - dist;
    return t > 0.f ? (uint32_t)t : 0u;
}

}  // namespace
}  // namespace dsq
