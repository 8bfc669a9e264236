// Alg. 4 update in two passes: running sums along visit lists into a workspace (cs_walk.hip), then every table cell
// gathered from the sums that belong to it.
//
// A walker of the list update ends with two to four sums per residue, and adding them into the
// table is one atomic request per sum to a random cell: the memory-side atomic unit takes 21 to 24 G requests/s,
// and the worker tables of a large sketch (168 MB per 8 workers at 5 x 2^20) are pushed out of the memory-side
// cache by the streams, so that a request also reads and writes its block.  Written to the workspace in the order
// in which they are computed the same sums are whole contiguous lines.  Which residues start in which cell
// depends on the hash constants alone, so it is laid out once (the index: for every row the residues in the order
// of their cells), and a thread per cell reads the two to five sums that are its own, adds them in a fixed
// order, and writes the cell: the tables need no clearing, no atomics, the result does not depend on
// the order of execution, and the merge over workers and the momentum, which read every cell, come along.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "cs_device.h"
#include "cs_internal.h"
#include "csketch.h"

namespace cs {

namespace {

// the index: row j has start[c + 1] (the first of a cell's residues), then those residues
struct IndexRows {
    uint64_t at[CS_MAX_R];       // words before row j's start
    uint64_t words;
    uint64_t residues[CS_MAX_R];
};

IndexRows index_rows(const cs_params* p) {
    IndexRows x{};
    for (uint32_t j = 0; j < p->r; ++j) {
        x.residues[j] = p->visit[j].gmax;
        x.at[j] = x.words;
        x.words += p->c + 1 + x.residues[j];
    }
    return x;
}

template <bool POW2>
__global__ void __launch_bounds__(kBlock) k_index_count(KParams p, IndexRows rows, uint32_t* __restrict__ index) {
    const uint32_t j = blockIdx.y;
    uint32_t* start = index + rows.at[j];
    const Columns col = columns_of<POW2>(p.c);
    const uint64_t stride = static_cast<uint64_t>(gridDim.x) * kBlock;
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x; i < rows.residues[j]; i += stride)
        atomicAdd(&start[bucket_of<POW2>(hash_state(p.a[j], p.b[j], i), col)], 1u);
}

// counts -> the end of every cell's residues; a workgroup per row
__global__ void __launch_bounds__(1024) k_index_scan(KParams p, IndexRows rows, uint32_t* __restrict__ index) {
    uint32_t* start = index + rows.at[blockIdx.x];
    __shared__ uint32_t part[1024];
    const uint32_t per = (p.c + 1023) / 1024, lo = threadIdx.x * per;
    const uint32_t hi = lo + per < p.c ? lo + per : p.c;
    uint32_t sum = 0;
    for (uint32_t b = lo; b < hi; ++b) sum += start[b];
    part[threadIdx.x] = sum;
    __syncthreads();
    for (uint32_t off = 1; off < 1024; off <<= 1) {
        const uint32_t other = threadIdx.x >= off ? part[threadIdx.x - off] : 0u;
        __syncthreads();
        part[threadIdx.x] += other;
        __syncthreads();
    }
    uint32_t end = part[threadIdx.x] - sum;
    for (uint32_t b = lo; b < hi; ++b) {
        end += start[b];
        start[b] = end;
    }
    if (threadIdx.x == 0) start[p.c] = static_cast<uint32_t>(rows.residues[blockIdx.x]);
}

// SIGNS: an entry is twice the coordinate, and one more where its sign is -1
template <bool POW2, bool SIGNS>
__global__ void __launch_bounds__(kBlock) k_index_fill(KParams p, IndexRows rows, uint32_t* __restrict__ index) {
    const uint32_t j = blockIdx.y;
    uint32_t* start = index + rows.at[j];
    uint32_t* residue = start + p.c + 1;
    const Columns col = columns_of<POW2>(p.c);
    const uint64_t stride = static_cast<uint64_t>(gridDim.x) * kBlock;
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * kBlock + threadIdx.x; i < rows.residues[j]; i += stride) {
        uint32_t entry = static_cast<uint32_t>(i);
        if constexpr (SIGNS) entry = 2u * entry | sign_flip_of(hash_state(p.as[j], p.bs[j], i)) >> 31;
        residue[atomicSub(&start[bucket_of<POW2>(hash_state(p.a[j], p.b[j], i), col)], 1u) - 1u] = entry;
    }
}

// A cell's residues in ascending order, so that sums have one order.  Cells of up to kShortCell residues by a thread
// each, which inserts one after the other; those of more (narrow tables: 5 x 64 over 20 million coordinates has 51 000 in
// a cell, where insertion would be 10^9 dependent steps) by a workgroup each, whose n log^2 n / 2 comparisons are independent
// within a pass.
constexpr uint32_t kShortCell = 32;
__global__ void __launch_bounds__(kBlock) k_index_sort(uint32_t c, IndexRows rows, uint32_t* __restrict__ index) {
    uint32_t* start = index + rows.at[blockIdx.y];
    uint32_t* residue = start + c + 1;
    const uint32_t b = blockIdx.x * kBlock + threadIdx.x;
    if (b >= c) return;
    const uint32_t lo = start[b], hi = start[b + 1];
    if (hi - lo > kShortCell) return;
    for (uint32_t e = lo + 1; e < hi; ++e) {
        const uint32_t x = residue[e];
        uint32_t at = e;
        for (; at > lo && residue[at - 1] > x; --at) residue[at] = residue[at - 1];
        residue[at] = x;
    }
}

// Bitonic merges of runs of 2, 4, ... with every comparison towards ascending order (the first pass of a merge takes the
// upper run backwards), so that places from n on, which would hold the largest values, are never touched.
constexpr uint32_t kLongBlock = 1024;
__global__ void __launch_bounds__(kLongBlock) k_index_sort_long(uint32_t c, uint32_t cells, IndexRows rows, uint32_t* index) {
    const uint32_t* start = index + rows.at[blockIdx.y];
    const uint32_t b0 = blockIdx.x * cells, b1 = b0 + cells < c ? b0 + cells : c;      // cells <= kLongBlock of a workgroup
    const uint32_t mine = b0 + threadIdx.x;
    if (!__syncthreads_or(mine < b1 && start[mine + 1] - start[mine] > kShortCell)) return;
    for (uint32_t b = b0; b < b1; ++b) {
        const uint32_t n = start[b + 1] - start[b];
        if (n <= kShortCell) continue;
        uint32_t* x = index + rows.at[blockIdx.y] + c + 1 + start[b];
        uint32_t logn = 0;
        while ((1ull << logn) < n) ++logn;
        const uint32_t pairs = 1u << (logn - 1);
        for (uint32_t run = 1; run <= logn; ++run) {
            for (uint32_t step = run; step-- > 0;) {   // partners 2^step apart
                const uint32_t low = (1u << step) - 1u;
                for (uint32_t t = threadIdx.x; t < pairs; t += kLongBlock) {
                    const uint32_t first = ((t & ~low) << 1) | (t & low);
                    const uint32_t other = step + 1 == run ? first ^ ((2u << step) - 1u) : first + low + 1u;
                    if (other < n) {
                        const uint32_t u = x[first], v = x[other];
                        if (u > v) {
                            x[first] = v;
                            x[other] = u;
                        }
                    }
                }
                __syncthreads();
            }
        }
    }
}

struct GatherRow {
    uint64_t index_at, at, piece_floats;
    uint32_t residues, pieces, ncell, log_run;
};
struct GatherArgs {
    const uint32_t* index;
    const float* sums;           // of the first group
    uint64_t group_floats;       // from one group's sums to the next
    float* T;                    // the first group's table, or null
    float* S_t;                  // or null: the merge of all groups (they must be all there are)
    float* S_u;                  // or null: momentum and error accumulation behind it
    float* S_v;
    float alpha, rho;
    int32_t groups;
    uint32_t r, c;
    GatherRow row[CS_MAX_R];
};

typedef float vec4f __attribute__((ext_vector_type(4)));

// kCellLanes lanes per cell: one where there are cells enough to fill the chip, more where there are few, each
// with many sums (a short vector's chains of visits are cut into pieces, every one with sums of its own).  WL = lanes
// of a walker: the workers whose sums lie together.  Each lane has the reads of kAhead sums in flight.
// The merge is accumulated in binary64 and rounded once, as in k_bundle_merge.
template <int WL, int kCellLanes>
__global__ void __launch_bounds__(kBlock) k_gather_sums(GatherArgs a) {
    constexpr int kAhead = WL == 8 ? 4 : 8;
    constexpr int kCells = kBlock / kCellLanes;        // of a workgroup
    const uint32_t j = blockIdx.y, part = threadIdx.x % kCellLanes;
    const uint32_t b = blockIdx.x * kCells + threadIdx.x / kCellLanes;
    if (b >= a.c) return;                              // (all lanes of a cell together)
    const GatherRow& row = a.row[j];
    const uint32_t* start = a.index + row.index_at;
    const uint32_t* residue = start + a.c + 1;
    constexpr int kWalkers = 64 / WL;                  // of a wavefront
    // the residues whose running sum q belongs to this cell: entry t of them all, upto[q - 1] <= t < upto[q], is
    // residue[from[q] + t]
    uint32_t from[4], upto[4], n = 0;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
        from[q] = 0;
        if (q < row.ncell) {
            const uint32_t first = (b - q) & (a.c - 1u);
            const uint32_t lo = start[first];
            uint32_t hi = start[first + 1];
            hi = hi < row.residues ? hi : row.residues;
            from[q] = lo - n;
            n += hi > lo ? hi - lo : 0u;
        }
        upto[q] = n;
    }
    const uint32_t items = n * row.pieces;
    double total = 0.0;
    const float* sums = a.sums + row.at;
    for (int g = 0; g < a.groups; ++g, sums += a.group_floats) {
        float cell[WL];
#pragma unroll
        for (int w = 0; w < WL; ++w) cell[w] = 0.0f;
        for (uint32_t t0 = part; t0 < items; t0 += kAhead * kCellLanes) {
            float x[kAhead][WL];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const uint32_t t = t0 + u * kCellLanes;
                const uint32_t piece = row.pieces == 1 ? 0u : t / n, e = t - piece * n;
                const uint32_t q = (e >= upto[0] ? 1u : 0u) + (e >= upto[1] ? 1u : 0u) + (e >= upto[2] ? 1u : 0u);
                const uint32_t base = e < upto[0] ? from[0] : e < upto[1] ? from[1] : e < upto[2] ? from[2] : from[3];
                uint32_t i = t < items ? residue[base + e] : ~0u;
                const bool there = i < row.residues;   // (not: no more items, or an index of another sketch)
                i = there ? i : 0u;
                // [wavefront][m][walker]: residue i is m = i mod 2^log_run of walker i / 2^log_run
                const uint32_t m = i & ((1u << row.log_run) - 1u), walker = i >> row.log_run;
                const uint32_t slot = (((walker / kWalkers) << row.log_run) + m) * kWalkers + walker % kWalkers;
                const float* src = sums + (there ? piece : 0u) * row.piece_floats +
                                   (static_cast<uint64_t>(slot) * row.ncell + (there ? q : 0u)) * WL;
#pragma unroll
                for (int w = 0; w < WL; ++w) x[u][w] = 0.0f;
                if (there) {
                    if constexpr (WL >= 4) {
#pragma unroll
                        for (int w = 0; w < WL; w += 4) {
                            const vec4f v = *reinterpret_cast<const vec4f*>(src + w);
#pragma unroll
                            for (int l = 0; l < 4; ++l) x[u][w + l] = v[l];
                        }
                    } else {
#pragma unroll
                        for (int w = 0; w < WL; ++w) x[u][w] = src[w];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
#pragma unroll
                for (int w = 0; w < WL; ++w) cell[w] += x[u][w];
        }
        if constexpr (kCellLanes > 1) {
#pragma unroll
            for (int off = 1; off < kCellLanes; off <<= 1)
#pragma unroll
                for (int w = 0; w < WL; ++w) cell[w] += __shfl_xor(cell[w], off);
        }
        if (a.T && part == 0) {
            static_assert(CS_BUNDLE_GROUP == 8, "a cell of a bundle is two pieces of 16 bytes");
            vec4f* dst = reinterpret_cast<vec4f*>(a.T + ((static_cast<uint64_t>(g) * a.r + j) * a.c + b) * CS_BUNDLE_GROUP);
            vec4f u[2];
#pragma unroll
            for (int w = 0; w < CS_BUNDLE_GROUP; ++w) u[w / 4][w % 4] = w < WL ? cell[w < WL ? w : 0] : 0.0f;
            dst[0] = u[0];
            dst[1] = u[1];
        }
        if (a.S_t) {
#pragma unroll
            for (int w = 0; w < WL; ++w) total += static_cast<double>(cell[w]);
        }
    }
    if (a.S_t && part == 0) {
        const uint64_t t = static_cast<uint64_t>(j) * a.c + b;
        const float st = static_cast<float>(static_cast<double>(a.alpha) * total);
        a.S_t[t] = st;
        if (a.S_u) {
            const float u = a.rho * a.S_u[t] + st;
            a.S_u[t] = u;
            a.S_v[t] = a.S_v[t] + u;
        }
    }
}

// lanes per cell: about 2^18 lanes in all (16 from 4096 cells on: 7 x 1024, 108 000 coordinates, 7 workers, the whole update
// with 4, 16, 64: 20.7, 19.3, 22.6 us; 5 x 512, 20 sums a cell: within 4 %)
template <int WL>
int launch_gather(const cs_params* p, const GatherArgs& a, hipStream_t stream) {
    const uint64_t cells = static_cast<uint64_t>(p->r) * p->c;
    auto grid = [&](unsigned per) { return dim3((p->c + per - 1) / per, p->r); };
    if (cells >= (1u << 17)) k_gather_sums<WL, 1><<<grid(kBlock), kBlock, 0, stream>>>(a);
    else if (cells >= (1u << 15)) k_gather_sums<WL, 4><<<grid(kBlock / 4), kBlock, 0, stream>>>(a);
    else if (cells >= (1u << 12)) k_gather_sums<WL, 16><<<grid(kBlock / 16), kBlock, 0, stream>>>(a);
    else k_gather_sums<WL, 64><<<grid(kBlock / 64), kBlock, 0, stream>>>(a);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

// of the residues (power-of-two columns) or, SIGNS, of whole coordinates
template <bool POW2, bool SIGNS>
int launch_index_build(const cs_params* p, const IndexRows& rows, uint32_t* index, hipStream_t stream) {
    const int rc = launch_bundle_zero(reinterpret_cast<float*>(index), static_cast<int64_t>(rows.words), stream);
    if (rc != CS_OK) return rc;
    const dim3 grid(2048, p->r), cells((p->c + kBlock - 1) / kBlock, p->r);
    k_index_count<POW2><<<grid, kBlock, 0, stream>>>(kparams(p), rows, index);
    k_index_scan<<<p->r, 1024, 0, stream>>>(kparams(p), rows, index);
    k_index_fill<POW2, SIGNS><<<grid, kBlock, 0, stream>>>(kparams(p), rows, index);
    k_index_sort<<<cells, kBlock, 0, stream>>>(p->c, rows, index);
    uint32_t per = (p->c + 2047) / 2048;               // cells of a workgroup: one of a narrow table
    per = per < kLongBlock ? per : kLongBlock;
    k_index_sort_long<<<dim3((p->c + per - 1) / per, p->r), kLongBlock, 0, stream>>>(p->c, per, rows, index);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

// Groups of workers are taken as many at a time as the workspace holds; with one batch the merge and the momentum
// come from it, else they read the tables afterwards.
int launch_bundle_sketch(const cs_params* p, float* T, int W, const float* const* g_w, int64_t d, float scale,
                         const uint32_t* index, float* ws, uint64_t ws_floats, float* S_t, float alpha,
                         float* S_u, float* S_v, float rho, hipStream_t stream) {
    const IndexRows rows = index_rows(p);
    const int groups = (W + CS_BUNDLE_GROUP - 1) / CS_BUNDLE_GROUP, lanes = sums_lanes(W);
    const uint64_t table = static_cast<uint64_t>(p->r) * p->c * CS_BUNDLE_GROUP;
    SumsPlan plan;
    const int together = sums_groups(p, W, d);
    int rc = launch_accumulate_sums(p, nullptr, 0, W, together, 0, nullptr, d, scale, plan, stream);
    if (rc != CS_OK) return rc;
    const uint64_t at_once = ws_floats / plan.floats;
    if (at_once == 0) return CS_EWORKSPACE;
    GatherArgs a{};
    a.index = index;
    a.sums = ws;
    a.group_floats = plan.floats;
    a.alpha = alpha;
    a.rho = rho;
    a.r = p->r;
    a.c = p->c;
    for (uint32_t j = 0; j < p->r; ++j) {
        const SumsRow& s = plan.row[j];
        a.row[j] = GatherRow{rows.at[j], s.at, s.piece_floats, static_cast<uint32_t>(s.residues), s.pieces, s.ncell, s.log_run};
    }
    for (int g0 = 0; g0 < groups; g0 += a.groups) {
        a.groups = static_cast<uint64_t>(groups - g0) < at_once ? groups - g0 : static_cast<int>(at_once);
        for (int g = g0; g < g0 + a.groups; g += together) {
            const int end = g + together < g0 + a.groups ? g + together : g0 + a.groups;
            const int w0 = g * CS_BUNDLE_GROUP, w1 = W < end * CS_BUNDLE_GROUP ? W : end * CS_BUNDLE_GROUP;
            rc = launch_accumulate_sums(p, ws + (g - g0) * a.group_floats, a.group_floats, W, together, w1 - w0, g_w + w0, d,
                                        scale, plan, stream);
            if (rc != CS_OK) return rc;
        }
        a.T = T ? T + g0 * table : nullptr;
        if (a.groups == groups) {
            a.S_t = S_t;
            a.S_u = S_u;
            a.S_v = S_v;
        }
        switch (lanes) {
            case 1: rc = launch_gather<1>(p, a, stream); break;
            case 2: rc = launch_gather<2>(p, a, stream); break;
            case 4: rc = launch_gather<4>(p, a, stream); break;
            default: rc = launch_gather<8>(p, a, stream);
        }
        if (rc != CS_OK) return rc;
        if (a.groups == groups) return CS_OK;
    }
    if (!S_t) return CS_OK;
    const int64_t cells = static_cast<int64_t>(p->r) * p->c;
    if (S_u) return launch_bundle_merge_momentum(S_t, S_u, S_v, T, groups, alpha, rho, cells, stream);
    return launch_bundle_merge(S_t, 0.0f, T, groups, alpha, cells, stream);
}

// ---------------------------------------------------------------------------------------
// The update of short vectors cell by cell: for every row the coordinates in the order of their cells are laid out
// once, with their signs, and a cell is the sum of its coordinates' values, read where they lie.  The vectors of a
// group stay in L2 meanwhile.  One launch writes the tables, their merge and the momentum: no clearing, no
// atomics, and the same bits in every run.
// ---------------------------------------------------------------------------------------
constexpr int kListVectors = 256;    // of a launch: their addresses are kernel arguments

struct ListArgs {
    const uint32_t* lists;
    float* T;                        // or null
    float* S_t;                      // or null; S_u, S_v or null: as in GatherArgs
    float* S_u;
    float* S_v;
    float scale, alpha, rho;
    uint32_t r, c, d;
    uint32_t b0;                     // the launch's first column
    int32_t W, slices;
    const float* g[kListVectors];
};

// L lanes of a cell (8 to 64) share out its coordinates; `slices` wavefronts share out the groups of 8 workers.
// SHARES > 0 (S_t alone): the workers are summed coordinate by coordinate, in binary64 and rounded once, before a cell is: values
// that cancel between workers leave no rounding of their own size in it.  The slices share out a cell's coordinates too, and
// where there are more lanes than coordinates, SHARES lanes (1 or 4) a coordinate's workers.
// us, sums of every worker's cell / of the coordinates first (this) / a launch for the workers' sum more: 5 x 40, d = 784, 4
// workers 3.9 / 3.3 / 5.6, 100 workers 7.7 / 5.5 / 10.7; 5 x 64, 5000, 32 workers 7.0 / 6.4 / 7.2 (8.4 with one slice); 3 x 33,
// 2000, 100 workers 8.8 / 7.1 / 10.7 (13.0 with one lane a coordinate).
template <int L, int SHARES>
__global__ void __launch_bounds__(kBlock) k_sum_lists(ListArgs a) {
    static_assert(L >= CS_BUNDLE_GROUP, "a lane per worker of a group");
    constexpr bool FOLD = SHARES > 0;
    constexpr int kCells = 64 / L, kWaves = kBlock / 64;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int slice = wave % a.slices;
    const uint32_t j = blockIdx.y, part = lane % L, set = wave / a.slices;
    const uint32_t b = a.b0 + (blockIdx.x * (kWaves / a.slices) + set) * kCells + lane / L;
    const bool in = b < a.c;
    const uint32_t* start = a.lists + static_cast<uint64_t>(j) * (a.c + 1ull + a.d);
    const uint32_t* entry = start + a.c + 1;
    uint32_t lo = 0, n = 0;
    if (in) {
        lo = start[b];
        uint32_t hi = start[b + 1];
        hi = hi < a.d ? hi : a.d;
        n = hi > lo ? hi - lo : 0u;
    }
    const uint64_t at = static_cast<uint64_t>(j) * a.c + b;
    const bool writes = in && part == 0 && slice == 0 && a.S_t;
    float old_u = 0.0f, old_v = 0.0f;
    if (writes && a.S_u) {
        old_u = a.S_u[at];
        old_v = a.S_v[at];
    }
    // after the exchange below a lane has the sum of this worker of a group
    const uint32_t mine = (part & 1u) * 4 + (part >> 1 & 1u) * 2 + (part >> 2 & 1u);
    double total = 0.0;
    const int groups = (a.W + CS_BUNDLE_GROUP - 1) / CS_BUNDLE_GROUP;
    if constexpr (FOLD) {
        float v = 0.0f;
        constexpr int kStep = L / SHARES;
        const int share = part % SHARES, w0 = share * a.W / SHARES, w1 = (share + 1) * a.W / SHARES;
        for (uint32_t t = slice * kStep + part / SHARES; t < n; t += a.slices * kStep) {
            const uint32_t e = entry[lo + t];
            if (e >> 1 >= a.d) continue;               // (lists of another sketch)
            double sum = 0.0;
            int w = w0;
            for (; w + CS_BUNDLE_GROUP <= w1; w += CS_BUNDLE_GROUP) {
                float x[CS_BUNDLE_GROUP];
#pragma unroll
                for (int q = 0; q < CS_BUNDLE_GROUP; ++q) x[q] = a.g[w + q][e >> 1];
#pragma unroll
                for (int q = 0; q < CS_BUNDLE_GROUP; ++q) sum += static_cast<double>(x[q]);
            }
#pragma unroll 4
            for (; w < w1; ++w) sum += static_cast<double>(a.g[w][e >> 1]);
#pragma unroll
            for (int off = 1; off < SHARES; off *= 2) sum += __shfl_xor(sum, off);       // (lanes of one coordinate: in step)
            v += apply_sign(static_cast<float>(static_cast<double>(a.alpha) * sum), e << 31);
        }
#pragma unroll
        for (int off = SHARES; off < L; off *= 2) v += __shfl_xor(v, off);
        total = static_cast<double>(v);
    } else
    for (int g = slice; g < groups; g += a.slices) {
        const int nw = a.W - g * CS_BUNDLE_GROUP < CS_BUNDLE_GROUP ? a.W - g * CS_BUNDLE_GROUP : CS_BUNDLE_GROUP;
        float v[CS_BUNDLE_GROUP];
        const float* const* vec = a.g + g * CS_BUNDLE_GROUP;
#pragma unroll
        for (int w = 0; w < CS_BUNDLE_GROUP; ++w) v[w] = 0.0f;
        auto add = [&](auto whole) {
            constexpr int kAhead = 2;
            for (uint32_t t = part; t < n; t += kAhead * L) {
                float x[kAhead][CS_BUNDLE_GROUP];
                uint32_t flip[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const uint32_t e = t + u * L < n ? entry[lo + t + u * L] : ~0u;
                    const bool there = e >> 1 < a.d;   // (not: no more entries, or lists of another sketch)
                    const uint32_t i = there ? e >> 1 : 0u;
                    flip[u] = e << 31;
#pragma unroll
                    for (int w = 0; w < CS_BUNDLE_GROUP; ++w) {
                        x[u][w] = 0.0f;
                        if ((decltype(whole)::value || w < nw) && there) x[u][w] = vec[w][i];
                    }
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u)
#pragma unroll
                    for (int w = 0; w < CS_BUNDLE_GROUP; ++w) v[w] += apply_sign(x[u][w], flip[u]);
            }
        };
        if (nw == CS_BUNDLE_GROUP) add(std::true_type());
        else add(std::false_type());
        // 8 sums of L lanes -> one sum of each lane
#pragma unroll
        for (int m = CS_BUNDLE_GROUP / 2, off = 1; m > 0; m /= 2, off *= 2) {
            const bool upper = (part & off) != 0;
#pragma unroll
            for (int q = 0; q < m; ++q) {
                const float keep = upper ? v[q + m] : v[q], give = upper ? v[q] : v[q + m];
                v[q] = keep + __shfl_xor(give, off);
            }
        }
#pragma unroll
        for (int off = CS_BUNDLE_GROUP; off < L; off *= 2) v[0] += __shfl_xor(v[0], off);
        const float sum = static_cast<int>(mine) < nw ? a.scale * v[0] : 0.0f;
        if (a.T && in && part < CS_BUNDLE_GROUP)
            a.T[((static_cast<uint64_t>(g) * a.r + j) * a.c + b) * CS_BUNDLE_GROUP + mine] = sum;
        total += static_cast<double>(sum);
    }
    if (!a.S_t) return;
    if constexpr (!FOLD) {
#pragma unroll
        for (int off = 1; off < CS_BUNDLE_GROUP; off *= 2) total += __shfl_xor(total, off);
    }
    if (a.slices > 1) {
        __shared__ double totals[kWaves][kCells];
        if (part == 0) totals[wave][lane / L] = total;
        __syncthreads();
        for (int q = 1; slice == 0 && q < a.slices; ++q) total += totals[wave + q][lane / L];
    }
    if (writes) {
        const float st = static_cast<float>((FOLD ? static_cast<double>(a.scale) : static_cast<double>(a.alpha)) * total);
        a.S_t[at] = st;
        if (a.S_u) {
            const float u = a.rho * old_u + st;
            a.S_u[at] = u;
            a.S_v[at] = old_v + u;
        }
    }
}

IndexRows list_rows(const cs_params* p, int64_t d) {
    IndexRows x{};
    for (uint32_t j = 0; j < p->r; ++j) {
        x.residues[j] = static_cast<uint64_t>(d);
        x.at[j] = x.words;
        x.words += p->c + 1 + x.residues[j];
    }
    return x;
}

bool params_ok(const cs_params* p) {
    return p && p->r >= 1 && p->r <= CS_MAX_R && (p->r & 1u) && p->c >= 1 && p->c <= (1u << 31);
}

}  // namespace

}  // namespace cs

using namespace cs;

// Where the two passes take less time than clearing, requests and merge (us, update with merge and momentum: requests / two
// passes):
//  * up to 4 workers, where a request carries 4 to 16 bytes and costs what one of 32 does: 1 worker, d = 2 M, 5 x 65 536:
//    65 / 32; 2 workers, 25 M, 5 x 2^19: 332 / 254; 2 workers, 100 M, 5 x 2^20: 936 / 791; 4 workers, 2^20, 5 x 2^15: 46 / 34;
//    unless the vectors take long to read and the requests little beside that (requests at 24 G/s, reads at 5 TB/s).
//    3 workers, 23 M, 3 x 65 536 (0.23 of the reads): 178 / 209; 18 M, 3 x 32 768 (0.40): 164 / 154; with 4 workers also from 130
//    coordinates per column on, whatever the requests: 9 M, 5 x 16 384 (0.43): 132 / 150; 9.4 M, 15 x 65 536 (0.69): 474 / 511;
//    against 7.1 M, 5 x 65 536 (0.44): 144 / 131; 20 M, 3 x 2^19 (0.59): 257 / 231; 60 M, 5 x 2^20 (0.64): 1121 / 1013;
//  * up to 16 workers and short vectors, whose time is requests, and three launches where one does: 14 workers, 40 000, 5 x 64:
//    53 / 33; 16 workers, 300 000, 5 x 4096: 49 / 39; 16 workers, 2^20, 5 x 2^15: 113 / 98; not with up to 8 rows (one launch of
//    requests)
//     - from r d = 5 million on with fewer than 2^15 columns, whose few requests hide behind the reads: 11 workers, 2.2 M,
//       5 x 4096: 112 / 135; 12 workers, 1.4 M, 5 x 8192: 90 / 104;
//     - from 130 000 to 600 000 with fewer than 400 coordinates per column, where launches are half of the time: 5 workers,
//       76 000, 7 x 1024: 15.7 / 20.1; 15 workers, 47 000, 7 x 1024: 26 / 29;
//    of 758 drawn shapes of 5 to 16 workers that leaves 562 to the two passes, ahead by 8 % on average (up to 1.7 times), 48 of
//    them behind by more than 3 %; 18 of the others would have been ahead by more than 5 %;
//  * 2 to 16 workers not with 64 columns, fewer than 200 coordinates per column and more than 0.4 sums per coordinate and row: a
//    cell gathers hundreds of sums: 2 workers, 11 000, 5 x 64: 16 / 21; 11 workers, 10 800, 5 x 64: 29 / 41;
//  * long vectors with tables that the memory-side cache does not hold beside them: 8 workers, 100 M, 5 x 2^20: 3284 / 3208;
//    16 workers, 50 M, 5 x 2^19: 2963 / 2895; even at 25 M (1121 / 1118).
// W = 0, a single vector into a table: against cs_sketch_zero and cs_sketch_accumulate, whose lattice form sends a request per
// 8 to 15 coordinates.  Ahead from r d = 10 million on where the lists keep few sums: 5 x 65 536, d = 2.6 M, 0.14 sums per
// coordinate and row: 51 / 33; 15 x 32 768, 1.3 M, 0.17: 112 / 75; 15 x 65 536, 1.8 M, 0.26: 101 / 144; 5 x 4096,
// 460 000: 15 / 17; more than 8 rows, a launch more, from 16 million on: 15 x 8192, 800 000: 39 / 50; 1.1 M: 72 / 60.
static bool sums_pay(const cs_params* p, int32_t W, int64_t d) {
    double sums = 0.0;
    for (uint32_t j = 0; j < p->r; ++j) sums += static_cast<double>(p->visit[j].ncell) * static_cast<double>(p->visit[j].gmax);
    const double rd = static_cast<double>(p->r) * static_cast<double>(d), per_column = static_cast<double>(d) / p->c;
    if (W == 0) return rd >= (p->r > 8 ? 1.6e7 : 1e7) && sums <= 0.2 * rd;
    if (W > 1 && W <= 16 && p->c <= 64 && per_column < 200.0 && sums > 0.4 * rd) return false;
    if (W <= 4) {
        const double read_ns = 4.0 * rd * W / 5000.0;
        return read_ns < 1e5 || (sums / 24.0 >= 0.33 * read_ns && (W < 4 || per_column < 130.0));
    }
    if (W <= 16 && rd <= 1e7) {
        if (p->r > 8) return true;
        if (rd >= 5e6) return p->c >= (1u << 15);
        return rd < 1.3e5 || rd > 6e5 || per_column >= 400.0;
    }
    return W <= 64 && d >= 32'000'000 && static_cast<uint64_t>(p->r) * p->c * CS_BUNDLE_GROUP * sizeof(float) >= (64u << 20);
}

extern "C" int cs_update_index_bytes(const cs_params* p, int32_t W, int64_t d, size_t* bytes) {
    if (!params_ok(p) || W < 0 || d < 0 || !bytes) return CS_EINVAL;
    *bytes = sums_pay(p, W, d) && sums_apply(p, d) ? index_rows(p).words * sizeof(uint32_t) : 0;
    return CS_OK;
}

extern "C" int cs_update_index_build(const cs_params* p, int64_t d, void* index, size_t bytes, void* stream) {
    if (!params_ok(p) || d < 0 || !index || reinterpret_cast<uintptr_t>(index) % 4 != 0) return CS_EINVAL;
    if (!sums_apply(p, d)) return CS_EINVAL;
    if (bytes < index_rows(p).words * sizeof(uint32_t)) return CS_EWORKSPACE;
    return launch_index_build<true, false>(p, index_rows(p), static_cast<uint32_t*>(index), static_cast<hipStream_t>(stream));
}

extern "C" int cs_update_workspace_bytes(const cs_params* p, int32_t W, int64_t d, size_t* bytes) {
    if (!params_ok(p) || W < 1 || d < 0 || !bytes) return CS_EINVAL;
    *bytes = 0;
    if (!sums_apply(p, d)) return CS_OK;
    SumsPlan plan;
    const int rc = launch_accumulate_sums(p, nullptr, 0, W, sums_groups(p, W, d), 0, nullptr, d, 1.0f, plan, nullptr);
    *bytes = plan.floats * sizeof(float) * ((W + CS_BUNDLE_GROUP - 1) / CS_BUNDLE_GROUP);
    return rc;
}

extern "C" int cs_bundle_sketch(const cs_params* p, float* T, int32_t W, const float* const* g_w, int64_t d,
                                float scale, const void* index, size_t index_bytes, void* ws, size_t ws_bytes,
                                float* S_t, float alpha, float* S_u, float* S_v, float rho, void* stream) {
    int64_t floats;
    int rc = cs_bundle_floats(p, W, &floats);
    if (rc != CS_OK || d < 0 || !g_w || !index || !ws) return CS_EINVAL;
    if ((!T && (W > CS_BUNDLE_GROUP || !S_t)) || (!S_u != !S_v) || (S_u && !S_t)) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!g_w[w]) return CS_EINVAL;
    if (reinterpret_cast<uintptr_t>(T) % 16 != 0 || reinterpret_cast<uintptr_t>(ws) % 16 != 0 ||
        reinterpret_cast<uintptr_t>(index) % 4 != 0) return CS_EINVAL;
    if (!sums_apply(p, d)) return CS_EINVAL;
    if (index_bytes < index_rows(p).words * sizeof(uint32_t)) return CS_EWORKSPACE;
    return launch_bundle_sketch(p, T, W, g_w, d, scale, static_cast<const uint32_t*>(index), static_cast<float*>(ws),
                                ws_bytes / sizeof(float), S_t, alpha, S_u, S_v, rho, static_cast<hipStream_t>(stream));
}

// Where the lists take less time than what else there is, by figures of 1300 shapes; us, others / lists.  Lists take 4 us
// and three things that partly overlap (the root of their squares comes closest: it picks the faster way for all but 9 of 509
// shapes that have no visit lists, within 4 %):
//  * values: r d W at 250 G/s while the vectors lie in L2 (d W up to a million; 200 at 1.4, 180 at 4, 110 at 8 million);
//  * a cell's chain: 64 lanes and two entries of each at once, so that a cell of n coordinates is n / 128 rounds of a load
//    that waits for another, 0.6 us each, 1.1 with 8 workers, and 1.0 and 2.2 where vectors and lists are more than L2 holds;
//  * the cells of a wide table, 45 ps each and group of workers (14 in a launch that clears or merges).
// Against
//  * visit lists of a power of two of columns, 13 to 16 us and 1.3 a million values, 2.7 with many groups of workers: 7 x 512,
//    18 231, 8 workers (1.0 million) 13.9 / 7.0; 7 x 512, 65 729, 5 workers (2.3) 15.5 / 13.0; 7 x 2048, 73 440, 5 workers
//    (2.6) 16.1 / 14.3; 5 x 512, 33 053, 42 workers (6.9) 30.7 / 32; with more than 8 rows, two launches: 15 x 1024,
//    78 577, 4 workers (4.7) 29 / 23; few columns: 3 x 64, 400 000 37 / 34, 600 000 40 / 50, 10^6 42 / 131; 3 x 256, 400 000
//    18 / 12, 10^6 22 / 38; 5 x 128, 600 000 25 / 38; wide: 3 x 2^18, 78 644 68 / 38; 3 x 2^20, 30 000 53 / 118;
//  * visit lists of other column counts: 7 x 2561, 217 913, 1 worker (1.5) 38.6 / 10; 5 x 853, 379 355, 2 workers (3.8)
//    26.4 / 19; 3 x 847, 229 277, 7 workers (4.8, 1.6 million in the vectors) 20.4 / 24; 15 x 2277, 237 944, 3 workers (10.7)
//    58.7 / 47; few columns: 5 x 90, 600 000 50 / 52; 7 x 90 100 / 56; 3 x 100, 10^6 62 / 87;
//  * requests of every coordinate into tables in LDS (lds_table_applies): 3 x 63, 100 000 21 / 12, 4 workers 22 / 16; 3 x 33,
//    100 000, 4 workers 21 / 25; 3 x 33, 10^6 46 / 244, 4 workers 78 / 348; 15 x 33, 100 000, 32 workers 292 / 205;
//    15 x 16, 400 000 63 / 192; or in memory: 7 x 32, 1947, 109 workers 35.8 / 10.3; 5 x 1913, 64 779 24.9 / 5.4;
//    3 x 500 001, 500 002 103 / 74, 150 001 54 / 73; 3 x 1 000 001, 1000 42 / 99.
// W = 0, one vector and one table: the lattice form of a power of two of columns, 5 x 16 384, 81 921 8.1 / 6.6, 400 000 x 3 x
// 64 162 / 34, 5 x 65 536, 131 073 11 / 17; requests to few cells, 3 x 63, 4 million 6690 / 522; 3 x 200 001, 60 001 19 / 28.
static bool lists_pay(const cs_params* p, int32_t W, int64_t d) {
    const double r = p->r, c = p->c, n = static_cast<double>(d), workers = W > 0 ? W : 1;
    const double vectors = n * workers, values = vectors * r, cells = r * c * ceil(workers / CS_BUNDLE_GROUP);
    const double per_cell = n / c;
    const bool beyond_l2 = n * (workers + r / 4) > 1e6;
    if (vectors > 4e6) return false;
    const double eight = workers < 8.0 ? workers : 8.0;
    const double chain = per_cell / 128.0 * (0.55 + 0.07 * eight + (beyond_l2 ? 0.3 + 0.1 * eight : 0.0));
    const double lists = 4.0 + sqrt(chain * chain + pow(45e-6 * cells, 2) + pow(values / 250e3, 2));
    const double direct = 5.0 + 4.0 * r + 2e-6 * cells + r * n * (c < 250.0 ? 8.0 / c : 0.032) * 1e-3;   // one vector, hash by hash
    if (walk_applies(p, d)) {
        if (W == 0 && c > n) return lists <= direct;   // (the lattice form is no better there)
        if (W == 0 ? cells > 1.5e5 : c > 4.0 * n || per_cell > (beyond_l2 ? 1600.0 : 6400.0)) return false;
        return values <= (p->r > 8 ? (W > 16 ? 7e6 : 5e6) : W > 16 ? 5.5e6 : 3e6);
    }
    if (anyc_update_applies(p, d, static_cast<int>(workers))) {
        if (W > 0 && per_cell > (p->r > 5 ? 8000.0 : 6400.0)) return false;
        return vectors <= 1.2e6 && values <= (p->r > 8 ? 1e7 : 5e6);
    }
    double others = direct;
    if (W > 0 && lds_table_applies(p, d)) others = 10.0 + r + r * n * (5.0 + 5.0 * workers) * 1e-6;
    else if (W > 0)                                    // (a launch for every 32 workers)
        others = 6.0 + 4.0 * ceil(workers / 32.0) + 14e-6 * cells + cells / c * n * (c < 208.0 ? 10.0 / c : 0.048) * 1e-3;
    return lists <= others;
}

extern "C" int cs_cell_lists_bytes(const cs_params* p, int32_t W, int64_t d, size_t* bytes) {
    if (!params_ok(p) || W < 0 || d < 0 || !bytes) return CS_EINVAL;
    *bytes = 0;
    if (d >= 1 && d < (1ll << 30) && W <= kListVectors && lists_pay(p, W, d)) *bytes = list_rows(p, d).words * sizeof(uint32_t);
    return CS_OK;
}

extern "C" int cs_cell_lists_build(const cs_params* p, int64_t d, void* lists, size_t bytes, void* stream) {
    if (!params_ok(p) || d < 1 || d >= (1ll << 30) || !lists || reinterpret_cast<uintptr_t>(lists) % 4 != 0) return CS_EINVAL;
    const IndexRows rows = list_rows(p, d);
    if (bytes < rows.words * sizeof(uint32_t)) return CS_EWORKSPACE;
    uint32_t* out = static_cast<uint32_t*>(lists);
    hipStream_t s = static_cast<hipStream_t>(stream);
    return p->c_pow2 ? launch_index_build<true, true>(p, rows, out, s) : launch_index_build<false, true>(p, rows, out, s);
}

extern "C" int cs_bundle_sketch_lists(const cs_params* p, float* T, int32_t W, const float* const* g_w, int64_t d,
                                      float scale, const void* lists, size_t bytes, float* S_t, float alpha, float* S_u,
                                      float* S_v, float rho, void* stream) {
    if (!params_ok(p) || W < 1 || W > kListVectors || d < 1 || d >= (1ll << 30) || !g_w || !lists) return CS_EINVAL;
    if ((!T && !S_t) || (!S_u != !S_v) || (S_u && !S_t)) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!g_w[w]) return CS_EINVAL;
    if (reinterpret_cast<uintptr_t>(lists) % 4 != 0) return CS_EINVAL;
    if (bytes < list_rows(p, d).words * sizeof(uint32_t)) return CS_EWORKSPACE;
    ListArgs a{};
    a.lists = static_cast<const uint32_t*>(lists);
    a.T = T;
    a.S_t = S_t;
    a.S_u = S_u;
    a.S_v = S_v;
    a.scale = scale;
    a.alpha = alpha;
    a.rho = rho;
    a.r = p->r;
    a.c = p->c;
    a.d = static_cast<uint32_t>(d);
    a.W = W;
    for (int w = 0; w < W; ++w) a.g[w] = g_w[w];
    const int groups = (W + CS_BUNDLE_GROUP - 1) / CS_BUNDLE_GROUP;
    const bool fold = !T && W > 1;
    a.slices = fold ? 1 : groups >= 4 ? 4 : groups >= 2 ? 2 : 1;
    // about 65 536 lanes in all, and not more than 8 coordinates for each
    const double want = 65536.0 / (static_cast<double>(p->r) * p->c * a.slices), each = static_cast<double>(d) / (8.0 * p->c);
    int L = 8;
    while (L < 64 && L < (want > each ? want : each)) L *= 2;
    int shares = fold ? 1 : 0;
    if (fold) {
        const double per_cell = static_cast<double>(d) / p->c;
        const bool idle = per_cell <= 64.0;            // up to four wavefronts of a cell, where they have work:
        while (L == 64 && a.slices < 4 && 64.0 * a.slices < want && (idle ? W >= 16 : 64.0 * a.slices < per_cell)) a.slices *= 2;
        if (W >= 16 && (a.slices == 4 ? idle : 4.0 * per_cell <= L)) shares = 4;     // four lanes for each coordinate
    }
    const uint32_t cells = kBlock / L / a.slices;      // of a workgroup
    hipStream_t s = static_cast<hipStream_t>(stream);
    constexpr uint32_t kListBlocks = 1u << 22;         // workgroups of a launch: one of 2^32 threads is refused
    for (; a.b0 < p->c; a.b0 += cells * kListBlocks) { // (cells <= 32, c <= 2^31: no overflow)
        const uint32_t blocks = (p->c - a.b0 - 1) / cells + 1;
        const dim3 grid(blocks < kListBlocks ? blocks : kListBlocks, p->r);
        auto launch = [&](auto lanes) {
            constexpr int N = decltype(lanes)::value;
            if (shares == 4) k_sum_lists<N, 4><<<grid, kBlock, 0, s>>>(a);
            else if (shares) k_sum_lists<N, 1><<<grid, kBlock, 0, s>>>(a);
            else k_sum_lists<N, 0><<<grid, kBlock, 0, s>>>(a);
        };
        switch (L) {
            case 8: launch(std::integral_constant<int, 8>()); break;
            case 16: launch(std::integral_constant<int, 16>()); break;
            case 32: launch(std::integral_constant<int, 32>()); break;
            default: launch(std::integral_constant<int, 64>());
        }
        if (hipGetLastError() != hipSuccess) return CS_EHIP;
    }
    return CS_OK;
}
