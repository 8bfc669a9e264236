// Declarations shared by the library's translation units (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "csketch.h"

namespace cs {

// What kernels receive by value: cs_params without the visit lists (kernel arguments are
// limited to 4 KB); a list travels separately to the one kernel that reads it.
struct KParams {
    uint32_t r, c, c_pow2, flags;
    uint64_t seed;
    uint64_t a[CS_MAX_R], b[CS_MAX_R];
    uint64_t as[CS_MAX_R], bs[CS_MAX_R];
    cs_row_plan plan[CS_MAX_R];
};
static_assert(offsetof(cs_params, visit) == sizeof(KParams), "KParams is the head of cs_params");
inline const KParams& kparams(const cs_params* p) { return *reinterpret_cast<const KParams*>(p); }

// Dispatch on the (odd) row count and on "c is a power of two" so that the hash state of all
// rows lives in registers and loops over rows are unrolled.
#define CS_DISPATCH_R(p, CALL)                                                     \
    do {                                                                           \
        const bool pow2__ = (p)->c_pow2 != 0;                                      \
        switch ((p)->r) {                                                          \
            case 1: if (pow2__) { CALL(1, true); } else { CALL(1, false); } break;   \
            case 3: if (pow2__) { CALL(3, true); } else { CALL(3, false); } break;   \
            case 5: if (pow2__) { CALL(5, true); } else { CALL(5, false); } break;   \
            case 7: if (pow2__) { CALL(7, true); } else { CALL(7, false); } break;   \
            case 9: if (pow2__) { CALL(9, true); } else { CALL(9, false); } break;   \
            case 11: if (pow2__) { CALL(11, true); } else { CALL(11, false); } break; \
            case 13: if (pow2__) { CALL(13, true); } else { CALL(13, false); } break; \
            case 15: if (pow2__) { CALL(15, true); } else { CALL(15, false); } break; \
            default: return CS_EINVAL;                                             \
        }                                                                          \
    } while (0)

constexpr int kMaxBatch = 32;   // workers per launch of the batched update kernels

// kernel argument block: worker w's table and vector
struct LatticePtrs {
    float* S[kMaxBatch];
    const float* g[kMaxBatch];
};

// True when the stride-aligned traversal is used for vectors of length d with this sketch
// (power-of-two c, a stride found for every row, d large enough to fill tiles).
bool lattice_applies(const cs_params* p, int64_t d);

int launch_accumulate_lattice(const cs_params* p, const LatticePtrs& ptrs, int nw, int64_t d,
                              int64_t i0, float scale, hipStream_t stream);
// hist (or null) is cleared and receives the counts of est by magnitude bin
int launch_estimate_lattice(const cs_params* p, const float* S, int64_t d, int64_t i0,
                            float* est, float* rows, uint64_t* hist, hipStream_t stream);
// hist[b] = number of t < d with (bits(est[t]) & 0x7fffffff) >> 20 == b, b < 2048 (cs_topk.hip);
// the _zero form only clears the 2048 counters
int launch_magnitude_hist_zero(uint64_t* hist, hipStream_t stream);
int launch_magnitude_hist(const float* est, int64_t d, uint64_t* hist, hipStream_t stream);
int launch_hash_range_lattice(const cs_params* p, int64_t i0, int64_t n, uint32_t* bucket,
                              int8_t* sign, hipStream_t stream);

bool lds_table_applies(const cs_params* p, int64_t d);   // the update of a bundle hash by hash, in LDS (cs_kernels.hip)

// Walk-order update of a worker bundle T = float[ceil(W/8)][r][c][8] (cs_walk.hip).
bool walk_applies(const cs_params* p, int64_t d);
// fold = true: T is one table float[r][c] and receives the sum over the W workers
// (all_rows_listed(p, d) must hold for launch_accumulate_walk, anyc_update_applies for the other).
// launches, here and below: kernel launches are added up there instead of made (T, g_w unused)
bool all_rows_listed(const cs_params* p, int64_t d);
int launch_accumulate_walk(const cs_params* p, float* T, int W, const float* const* g_w,
                           int64_t d, int64_t i0, float scale, bool fold, hipStream_t stream, int* launches = nullptr);
// one vector along visit lists, any column count (one_applies(p, d) must hold); S = float[r][c][cell_floats]
bool one_applies(const cs_params* p, int64_t d);
int launch_accumulate_one(const cs_params* p, float* S, int cell_floats, const float* g, int64_t d,
                          int64_t i0, float scale, hipStream_t stream, int* launches = nullptr);
// The update along visit lists into a workspace of running sums, one group of workers after the other or, of short
// vectors, several in a launch, and what lies where in a group's: row j's sums [pieces][piece_floats], piece_floats = residues (rounded up to whole wavefronts) x running sums x
// lanes of a walker.
struct SumsRow {
    uint64_t at, residues, piece_floats;
    uint32_t pieces, ncell, log_run;
};
struct SumsPlan {
    uint64_t floats;             // of one group
    SumsRow row[CS_MAX_R];
};
bool sums_apply(const cs_params* p, int64_t d);
int sums_lanes(int W);           // lanes of a walker (1, 2, 4, 8) with W workers, the same in all groups of 8
int sums_groups(const cs_params* p, int W, int64_t d);   // groups of 8 workers that a launch takes, of W workers
// workers: of the whole update (every launch of it has the same plan); nw: of this launch, up to 8 `groups`; g_w null: the plan only.
// sums_floats: from one group's sums to the next
int launch_accumulate_sums(const cs_params* p, float* sums, uint64_t sums_floats, int workers, int groups, int nw,
                           const float* const* g_w, int64_t d, float scale, SumsPlan& plan, hipStream_t stream);
// the same along visit lists for column counts that are not a power of two
bool anyc_visits_apply(const cs_params* p, int64_t d);
bool anyc_update_applies(const cs_params* p, int64_t d, int W);
bool anyc_visits_serve_query(const cs_params* p, int64_t d);
bool anyc_query_needs_scratch(const cs_params* p, int64_t d);    // ... and is the only form for this length
int launch_accumulate_anyc(const cs_params* p, float* T, int W, const float* const* g_w,
                           int64_t d, int64_t i0, float scale, bool fold, hipStream_t stream, int* launches = nullptr);
int launch_estimate_anyc(const cs_params* p, const float* S, int64_t d, int64_t i0, float* est,
                         float* rows, uint64_t* hist, hipStream_t stream);
bool walk_takes_median(const cs_params* p, int64_t d);            // fuse_last is the faster way
int launch_estimate_walk(const cs_params* p, const float* S, int64_t d, int64_t i0,
                         float* est, float* rows, bool fuse_last, uint64_t* hist, hipStream_t stream);
int launch_bundle_zero(float* T, int64_t n, hipStream_t stream);
int launch_bundle_merge(float* dst, float beta, const float* T, int groups, float alpha,
                        int64_t cells, hipStream_t stream);
int launch_bundle_merge_momentum(float* St, float* Su, float* Sv, const float* T, int groups, float alpha,
                                 float rho, int64_t cells, hipStream_t stream);
int launch_bundle_merge16(float* dst, float beta, const uint16_t* T16, int groups, float alpha,
                          int64_t cells, int fmt, hipStream_t stream);

}  // namespace cs
