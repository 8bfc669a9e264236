// Alg. 4 update for a bundle of workers (power-of-two column counts), and the bundle-wide
// elementwise kernels.
//
// Done naively the update is one atomic add per coordinate, row and worker, and this machine
// executes fp32 atomics at the memory side at a fixed ~21-24 G requests per second (measured,
// whatever the table size; a request is one aligned 64-byte block touched by one instruction).  Three facts cut the requests by a factor of ~300, after
// which the kernel is bound by reading the vectors:
//
//  1. The bucket hash is affine modulo p = 2^61 - 1, so moving s coordinates on moves a
//     coordinate through a row by an amount that depends on s only.  The host lists offsets for
//     which that amount is a fraction of a cell (cs_row_plan: one stride and its multiples;
//     cs_visit_plan: every such offset below the vector length), and a lane visits its
//     coordinates in that order, keeping running sums in registers: one per coordinate,
//     flushed when the cell changes, in the stride walk (k_accumulate_walk); two to four per
//     coordinate, flushed once at the very end, with a visit list (k_accumulate_visits, the
//     kernel that normally runs).
//  2. All workers use the same hash functions, so in the bundle layout T[w/8][j][b][w%8] the
//     sums of 8 workers for one cell are 32 contiguous bytes: 8 lanes (one per worker) flush
//     them as one request.
//  3. Every row needs its own visiting order, so a group's vectors are read once per row; the
//     rows of a group run in one launch.
//
// Work decomposition for row j: the residues below the stride (or below the largest gap of the
// list) are cut into chunks of RUN consecutive coordinates; a "walker" owns one chunk and
// visits it at every listed offset.  A wavefront holds 64 / WL walkers of WL lanes each, lane
// wl of a walker serving worker wl of the group.  Every hash value is evaluated exactly
// (incremental form of the definition), so results are the same sums as in any other order,
// up to fp32 rounding order.
//
// Data movement per visit: the 64 x RUN tile (64 runs = walkers x workers, RUN floats each) is
// requested as contiguous pieces by neighbouring lanes and transposed through LDS so that every
// lane gets its own run; cell and sign of a walker's RUN coordinates are told once per walker, and its lanes take
// them from wavefront masks (visit lists) or from LDS (stride walk).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "cs_device.h"
#include "cs_internal.h"
#include "csketch.h"

namespace cs {

namespace {

constexpr int kGroup = CS_BUNDLE_GROUP;  // workers per bundle group
constexpr int kWalkWaves = 2;             // wavefronts per workgroup of the 8-worker stride walk
// ... and of the 8-worker list kernel: they share a table of visits.  (2: d = 6.5 M, 5 x 2^17 196 us for 184, d = 11 M
// 313 for 304, d = 25 M, 7 x 2^19 1098 for 1075, d = 10^8 the same.)
constexpr int kWavesPerGroupOf8 = 4;

// Vectors are addressed as global memory explicitly: the pointers pass through an LDS table,
// and a generic ("flat") load would count against the LDS counter as well and force the
// hardware to drain both before any data can be used.
typedef const __attribute__((address_space(1))) float* gfloat_ptr;
typedef float vec4f __attribute__((ext_vector_type(4)));
typedef vec4f __attribute__((aligned(4))) vec4f_u;           // 16 bytes at any dword address
typedef const __attribute__((address_space(1))) vec4f_u* gvec4_ptr;

struct WalkArgs {
    const float* g[kGroup];      // vectors of the workers of this group
    float* T;                    // the group's table, float[r][c][kGroup]
    int32_t js[CS_MAX_R];        // sketch rows of this launch; blockIdx.y picks one
    int32_t nw;                  // workers in this group (<= kGroup)
    int64_t d, i0;
    float scale;
};

// WL  = lanes per walker = workers served together (1, 2, 4 or 8);
// RUN = consecutive coordinates per walker and visit (16 or 32).
// A wavefront holds WPW = 64 / WL walkers on neighbouring chunks of RUN residues, so one visit
// reads WPW * RUN * 4 contiguous bytes of every worker's vector (512 bytes for WL = 8,
// RUN = 16: measured to stream at 5.7 TB/s, against 4.5 TB/s with 256-byte and
// 3.5 TB/s with 128-byte pieces).
// NWAVE = wavefronts per workgroup; they work on neighbouring sets of walkers at about the same
// time (nothing is shared and nothing is synchronised between them), which widens the
// contiguous stretch of every vector that is being read at one moment.
template <int WL, int RUN, int NWAVE>
__global__ void __launch_bounds__(64 * NWAVE) k_accumulate_walk(KParams p, WalkArgs a) {
    constexpr int WPW = 64 / WL;                       // walkers per wavefront
    constexpr int PPL = RUN / WL > 0 ? RUN / WL : 1;   // hash values each lane computes
    constexpr int kStride = RUN + 1;                   // padded LDS row of the value tile
    constexpr int kPieces = RUN / 4;                   // 16-byte pieces per run
    constexpr int kRunsPerPass = 64 / kPieces;
    constexpr int kPasses = kPieces;                   // 64 runs / kRunsPerPass
    static_assert(WL * PPL == RUN || WL > RUN, "every coordinate of a walker gets a hash lane");
    __shared__ float tile_lds_all[NWAVE][64 * kStride];
    __shared__ uint32_t hash_lds_all[NWAVE][2][WPW * RUN];   // (bucket | sign), this and previous visit
    __shared__ gfloat_ptr gptr_lds_all[NWAVE][kGroup];

    const int lane = threadIdx.x & 63;
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wavefront-uniform
    float* tile_lds = tile_lds_all[wq];
    uint32_t (*hash_lds)[WPW * RUN] = hash_lds_all[wq];
    gfloat_ptr* gptr_lds = gptr_lds_all[wq];
    const int j = a.js[blockIdx.y];
    const int h = lane / WL, wl = lane % WL;           // my walker, my worker slot
    if (lane < kGroup) gptr_lds[lane] = (gfloat_ptr)a.g[lane < a.nw ? lane : 0];
    __builtin_amdgcn_wave_barrier();

    const int64_t D = static_cast<int64_t>(p.plan[j].Dw);
    const uint64_t ADb = p.plan[j].ADw, ADs = p.plan[j].ADws;
    const int64_t chunks = (D + RUN - 1) / RUN;
    const int64_t nwaves = (chunks + WPW - 1) / WPW;
    const uint32_t mask = p.c - 1u;
    const int64_t d = a.d;
    float* __restrict__ Tcol = a.T + static_cast<size_t>(j) * p.c * kGroup + wl;

    // loader role: piece m4 of runs r0, r0 + kRunsPerPass, ...; run rho = worker * WPW + walker,
    // so that one load instruction covers neighbouring walkers (contiguous bytes) of few workers
    const int m4 = (lane % kPieces) * 4, r0 = lane / kPieces;
    // hash role: values m0 .. m0 + PPL - 1 of my walker
    const int m0 = (wl * PPL) % RUN;
    const bool hash_duty = wl * PPL < RUN;

    // Workgroups are dealt to the 8 XCDs round-robin; giving XCD x the x-th eighth of the
    // walkers makes each XCD (and its L2) stream through its own contiguous part of every
    // vector.  gridDim.x is a multiple of 8.
    const int64_t ngroups = (nwaves + NWAVE - 1) / NWAVE;      // workgroup-sized sets of walkers
    const int64_t per_xcd = (ngroups + 7) / 8;
    const int64_t xcd_first = static_cast<int64_t>(blockIdx.x & 7) * per_xcd;
    for (int64_t k = blockIdx.x >> 3; k < per_xcd; k += gridDim.x >> 3) {
        const int64_t wv = (xcd_first + k) * NWAVE + wq;
        if (xcd_first + k >= ngroups || wv >= nwaves) break;
        const int64_t chunk0 = wv * WPW;               // first walker's chunk
        const int64_t my_off = (chunk0 + h) * RUN;     // my walker's residue offset in [0, Dw)
        // hash state of coordinate i0 + my_off + m0 (visit n = 0)
        uint64_t yb = hash_state(p.a[j], p.b[j], static_cast<uint64_t>(a.i0 + my_off + m0));
        uint64_t ys = hash_state(p.as[j], p.bs[j], static_cast<uint64_t>(a.i0 + my_off + m0));

        float acc[RUN];                                // running sum of the cell each coordinate is in
#pragma unroll
        for (int m = 0; m < RUN; ++m) acc[m] = 0.0f;

        // All pieces are requested back to back without a branch in between (a piece that is
        // not wholly inside its run reads a safe address and is discarded); runs cut short by
        // the end of the vector or of the residue range are patched up afterwards, which only
        // the last visit or the last chunk ever needs.
        float4 pre[kPasses];
        auto load_visit = [&](int64_t nD) {
            bool any_partial = false;
#pragma unroll
            for (int q = 0; q < kPasses; ++q) {
                const int rho = q * kRunsPerPass + r0;
                const int rw = rho / WPW, rh = rho % WPW;     // worker-major: neighbouring lanes, neighbouring walkers
                const int64_t off = (chunk0 + rh) * RUN;           // residue offset of that run
                const int64_t rel = nD + off;
                int64_t len = D - off;
                if (d - rel < len) len = d - rel;
                if (rw >= a.nw) len = 0;
                const bool full = m4 + 4 <= len;
                const bool part = !full && m4 < len;
                const gfloat_ptr base = gptr_lds[rw < kGroup ? rw : 0];
                const gfloat_ptr src = full ? base + rel + m4 : base;
                const vec4f u = *(gvec4_ptr)src;
                pre[q] = full ? make_float4(u.x, u.y, u.z, u.w) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                any_partial |= part;
            }
            if (__builtin_amdgcn_ballot_w64(any_partial) != 0) {
#pragma unroll
                for (int q = 0; q < kPasses; ++q) {
                    const int rho = q * kRunsPerPass + r0;
                    const int rw = rho / WPW, rh = rho % WPW;     // worker-major: neighbouring lanes, neighbouring walkers
                    const int64_t off = (chunk0 + rh) * RUN;
                    const int64_t rel = nD + off;
                    int64_t len = D - off;
                    if (d - rel < len) len = d - rel;
                    if (rw >= a.nw) len = 0;
                    if (m4 + 4 > len && m4 < len) {
                        const gfloat_ptr src = gptr_lds[rw < kGroup ? rw : 0] + rel + m4;
                        pre[q].x = src[0];
                        if (m4 + 1 < len) pre[q].y = src[1];
                        if (m4 + 2 < len) pre[q].z = src[2];
                    }
                }
            }
        };

        int64_t nD = 0;
        int par = 0;                                   // which hash buffer holds this visit
        load_visit(nD);
        while (nD + chunk0 * RUN < d) {
            // values: registers -> LDS (run-major); each lane then reads its own run
#pragma unroll
            for (int q = 0; q < kPasses; ++q) {
                const int rho = q * kRunsPerPass + r0;
                float* dst = tile_lds + ((rho % WPW) * WL + rho / WPW) * kStride + m4;
                dst[0] = pre[q].x;
                dst[1] = pre[q].y;
                dst[2] = pre[q].z;
                dst[3] = pre[q].w;
            }
            // hashes of this visit: PPL consecutive coordinates from my state; the first visit
            // also fills the "previous" buffer, so that nothing looks like a left cell
            if (hash_duty) {
                uint64_t tb = yb, ts = ys;
#pragma unroll
                for (int q = 0; q < PPL; ++q) {
                    const uint32_t pk = ((static_cast<uint32_t>(tb) - 1u) & mask) | sign_flip_of(ts);
                    hash_lds[par][h * RUN + m0 + q] = pk;
                    if (nD == 0) hash_lds[par ^ 1][h * RUN + m0 + q] = pk;
                    if (q + 1 < PPL) {
                        tb = hash_advance(tb, p.a[j]);
                        ts = hash_advance(ts, p.as[j]);
                    }
                }
            }
            yb = hash_advance(yb, ADb);
            ys = hash_advance(ys, ADs);
            __builtin_amdgcn_wave_barrier();
            const float* my_run = tile_lds + lane * kStride;
            const uint32_t* now = hash_lds[par] + h * RUN;
            const uint32_t* before = hash_lds[par ^ 1] + h * RUN;
#pragma unroll
            for (int m = 0; m < RUN; ++m) {
                const uint32_t pk = now[m];
                const uint32_t cell = pk & 0x7fffffffu;
                const uint32_t was = before[m] & 0x7fffffffu;
                if (cell != was) {                         // left the cell: send its sum
                    if (acc[m] != 0.0f)
                        atomic_add_noret(Tcol + static_cast<size_t>(was) * kGroup, acc[m]);
                    acc[m] = 0.0f;
                }
                acc[m] += apply_sign(a.scale * my_run[m], pk & 0x80000000u);
            }
            __builtin_amdgcn_wave_barrier();
            // The next visit's loads are issued after this visit's atomics: the memory counter
            // retires in order, so the wait for those loads at the top of the loop also covers
            // the (older) atomics.
            nD += D;
            par ^= 1;
            if (nD + chunk0 * RUN < d) load_visit(nD);
        }
        // the cells the walkers ended in (buffer of the last visit)
        const uint32_t* last = hash_lds[par ^ 1] + h * RUN;
#pragma unroll
        for (int m = 0; m < RUN; ++m)
            if (acc[m] != 0.0f)
                atomic_add_noret(Tcol + static_cast<size_t>(last[m] & 0x7fffffffu) * kGroup, acc[m]);
        __builtin_amdgcn_wave_barrier();
    }
}

// one launch: the rows a.js[0 .. nrows-1] of one group of workers (blockIdx.y = row of the set)
template <int WL, int RUN, int NWAVE>
int launch_walk(const cs_params* p, const WalkArgs& a, int nrows, hipStream_t stream) {
    constexpr int WPW = 64 / WL;
    int64_t most = 1;
    for (int q = 0; q < nrows; ++q) {
        const int64_t chunks = (static_cast<int64_t>(p->plan[a.js[q]].Dw) + RUN - 1) / RUN;
        const int64_t nwaves = (chunks + WPW - 1) / WPW;
        const int64_t ngroups = (nwaves + NWAVE - 1) / NWAVE;
        if (ngroups > most) most = ngroups;
    }
    const int64_t cap = 256 * 64 / NWAVE;
    int64_t gx = most < cap ? most : cap;
    gx = (gx + 7) / 8 * 8;                   // the kernel deals workgroups to XCDs in eights
    const dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>(nrows));
    k_accumulate_walk<WL, RUN, NWAVE><<<grid, 64 * NWAVE, 0, stream>>>(kparams(p), a);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

// ---------------------------------------------------------------------------------------
// The same update along a visit list (cs_visit_plan) instead of a single stride.
//
// The list s_0 = 0 < s_1 < ... holds every offset whose bucket advance is below a bound of
// ncell - 1 cells, so whatever a lane meets at i + s_k lies in one of the NC = ncell cells
// that start at the cell of i.  A lane therefore keeps NC running sums per coordinate of its
// run for the whole kernel and sends each to memory exactly once at the end: NC atomic
// requests per RUN-residue and worker group for the entire vector, and none inside the loop.
// Visit k covers [s_k, s_k + gap_k); the walker that owns residues [off, off + RUN) takes part
// in it when off < gap_k, so lanes own the residues below the largest gap.  Loads, the LDS
// transpose and the roles of lanes are those of the stride walk above.
// ---------------------------------------------------------------------------------------
struct VisitArgs {
    uint32_t K;                  // visits
    int32_t j;                   // sketch row
    uint32_t pieces;             // the visits are shared out among this many wavefronts
    uint32_t blocks;             // workgroups of one piece
    uint64_t gmax;
    uint64_t a, b, as, bs;       // hash constants of row j
    uint64_t at;                 // floats of the workspace before those of this row's sums
    uint64_t gap[4];
    uint32_t ncell;              // running sums of a coordinate
    uint32_t code[CS_MAX_VISITS / 16];
};
// The rows of a sketch are updated by one launch: their serial chains of visits overlap, and there
// are fewer launch tails.  Row q has the workgroups first[q] .. first[q] + blocks * pieces - 1: the
// rows of one sketch differ in gmax and in pieces by a factor of 30, so that a grid of
// (most blocks, rows, most pieces) is nearly all empty workgroups for a short vector (32 000 for 2 500
// at d = 30 403, c = 256, which took most of 19 us).
constexpr int kRowsPerLaunch = 8;
// Groups of workers of short vectors go into one launch too (groups_at_once).
constexpr int kGroupsPerLaunch = 32;
// Neighbouring sets of walkers that go to the same XCD (the kernel deals sets to XCDs in blocks
// of this many, so that an XCD reads a few KB of contiguous addresses per visit).  Five, not a
// power of two: with 4 sets of 2 wavefronts an XCD's block is exactly 4 KB of every vector, each
// XCD then keeps meeting the same addresses modulo 32 KB, and the update measured 1 % slower
// (1, 2, 4, 16: slower; 3, 5, 6, 8: within 0.5 % of each other).
// Whole rounds of 8 XCDs x 5 sets leave workgroups empty, most of them where rows of a few sets are
// cut into many pieces; a launch that would have more than kRoundsUpTo workgroups for that deals rows of less
// than a round singly, a workgroup per set (15 rows, c = 128, d = 11 475: 7160 workgroups for 560 sets,
// 13.9 us a launch of 8 workers for 10.2).  Smaller launches keep the rounds: neighbouring sets share
// cache lines (7 rows, c = 512, d = 12 494, 1480 workgroups for 608 sets: 0.6 us less than dealt singly).
constexpr int kVisitSetBlock = 5;
constexpr uint32_t kVisitRound = 8 * kVisitSetBlock;
constexpr unsigned kRoundsUpTo = 2048;
// the set that turn vi of a row with `blocks` workgroups stands for, and the first set of its round
__device__ __forceinline__ int64_t visit_set(int64_t vi, uint32_t blocks) {
    const int64_t slot = vi >> 3;
    return blocks < kVisitRound ? vi : ((slot / kVisitSetBlock) * 8 + (vi & 7)) * kVisitSetBlock + slot % kVisitSetBlock;
}
__device__ __forceinline__ int64_t visit_round(int64_t vi, uint32_t blocks) {
    return blocks < kVisitRound ? vi : (vi >> 3) / kVisitSetBlock * kVisitRound;
}
struct VisitRows {
    uint32_t first[kRowsPerLaunch];              // ~0: no such row
    VisitArgs row[kRowsPerLaunch];
    __device__ __forceinline__ const VisitArgs& at(unsigned y) const { return row[y]; }
};
// The list of one row when the column count is not a power of two (cs_anyc_plan): the gaps visit
// by visit.  The hash advances (a_j gap_k) mod p and (a'_j gap_k) mod p do not travel with it:
// every workgroup computes them once into LDS, so that several rows' lists fit into the 4 KB of
// kernel arguments and share a launch.
struct VisitGaps {
    uint32_t K;
    int32_t j;
    uint32_t pieces, blocks;
    uint64_t gmax;
    uint64_t a, b, as, bs;
    uint32_t omega;              // running sums: omega cells from the first one, omega more after a wrap
    uint32_t pc;                 // p mod c: how far back a wrap past p sets the bucket
    uint32_t gap[CS_ANYC_MAX_VISITS];
};
constexpr int kAnycRowsPerLaunch = 6;
template <int ROWS>
struct VisitGapsRowsOf {
    uint32_t first[ROWS];                        // ~0: no such row
    VisitGaps row[ROWS];
    __device__ __forceinline__ const VisitGaps& at(unsigned y) const { return row[y]; }
};
typedef VisitGapsRowsOf<kAnycRowsPerLaunch> VisitGapsRows;
// a row less leaves room for the vectors of 8 groups
constexpr int kAnycRowsOfGroups = 5, kAnycGroups = 8;
typedef VisitGapsRowsOf<kAnycRowsOfGroups> VisitGapsRowsGroups;
static_assert(sizeof(VisitGapsRows) + 128 <= 4096, "the lists of a launch and its other arguments are kernel arguments");
// (blockIdx.y is the group of a launch of several)
template <int GROUPS>
struct VisitWorkersOf {
    float* T;                    // the first group's table, float[r][c][kGroup]; with `fold` one table float[r][c]
    int64_t d, i0;
    uint32_t c;
    int32_t nw;                  // workers of all groups of the launch
    float scale;
    int32_t fold;                // != 0: the workers' sums of a cell are added up across the lanes
                                 // of a walker and leave as one 4-byte request into a single table
    uint32_t at_once;            // workgroups that the chip holds at a time (set by the launch): see walks_down
    float* sums;                 // PARTIAL: where the first group's running sums go
    uint64_t table_floats, sums_floats;          // from one group's to the next
    const float* g[GROUPS * kGroup];             // vectors of the workers
};
typedef VisitWorkersOf<kGroupsPerLaunch> VisitWorkers;
// what fits beside the lists of LIST
template <typename LIST>
using WorkersBeside = VisitWorkersOf<std::is_same<LIST, VisitRows>::value             ? kGroupsPerLaunch
                                     : std::is_same<LIST, VisitGapsRowsGroups>::value ? kAnycGroups
                                                                                      : 1>;
static_assert(sizeof(VisitRows) + sizeof(VisitWorkers) <= 4096, "kernel arguments");
static_assert(sizeof(VisitGapsRowsGroups) + sizeof(VisitWorkersOf<kAnycGroups>) <= 4096, "kernel arguments");


typedef float vec2f __attribute__((ext_vector_type(2)));
typedef vec2f __attribute__((aligned(4))) vec2f_u;            // 8 bytes at any dword address
typedef const __attribute__((address_space(1))) vec2f_u* gvec2_ptr;

// N consecutive floats from global memory at any dword address, as the widest requests
template <int N>
__device__ __forceinline__ void load_floats(gfloat_ptr src, float (&out)[N]) {
    static_assert(N == 2 || N % 4 == 0, "pieces of 2, 4, 8 or 16 floats");
    if constexpr (N == 2) {
        const vec2f u = *(gvec2_ptr)src;
        out[0] = u.x;
        out[1] = u.y;
    } else {
#pragma unroll
        for (int t = 0; t < N; t += 4) {
            const vec4f u = *(gvec4_ptr)(src + t);
            out[t] = u.x;
            out[t + 1] = u.y;
            out[t + 2] = u.z;
            out[t + 3] = u.w;
        }
    }
}

// the row that this workgroup works for
template <typename LIST>
__device__ __forceinline__ unsigned row_of_block(const LIST& rows) {
    constexpr int N = sizeof(rows.first) / sizeof(rows.first[0]);
    unsigned q = 0;
#pragma unroll
    for (int t = 1; t < N; ++t) q += blockIdx.x >= rows.first[t] ? 1u : 0u;
    return q;
}

// ---------------------------------------------------------------------------------------
// What a visit does to the hashes of a coordinate, told by two comparisons.
//
// Visit k is at offset s_k, and with A = (a s_k) mod p the bucket hash of i + s_k is x + A, less p if
// x >= p - A, where x is that of i.  A is the same for every coordinate, so the bucket moves on by A mod c,
// and by p mod c back in the second case (one cell further if c is a power of two, for p = -1 mod c):
// one of two cells, and which one is the comparison of x with p - 1 - A.  The sign hash likewise: its
// parity is that of x' plus that of A', inverted after a wrap.  So a lane keeps the top 32 bits of x and x' of
// its coordinates and compares them with the top 32 bits of the visit's two thresholds (bits 29..60);
// where they are equal the lower bits would decide, and the visit is hashed by the definition
// instead (once in 2^31 coordinates and visits).  Against carrying two 61-bit states per coordinate from visit
// to visit this takes 10 vector operations per coordinate and visit for about 25.
//
// Only the two sums of one value of A mod c are in registers at a time; the others wait in LDS.
// ---------------------------------------------------------------------------------------
constexpr int kTopShift = 29;                          // 61-bit hash value -> its top 32 bits
__device__ __forceinline__ uint32_t top_of(uint64_t y) { return static_cast<uint32_t>((y - 1) >> kTopShift); }
// x wraps on an advance by A when it is above p - 1 - A
__device__ __forceinline__ uint32_t threshold_of(uint64_t A) { return static_cast<uint32_t>((kP61 - 1 - A) >> kTopShift); }

// A visit.  x: threshold of the bucket hash, y: of the sign hash, z: offset, w: bits 0..28 its gap (residues
// that take part), bit 29 the parity of A', bits 30-31 A mod c (the running sum of a coordinate that does not
// wrap), or 3 where that is none of the sums that are kept.
// WIDE (more than four running sums): z has the third bit of A mod c in bit 31, and `none` is 7.
constexpr uint32_t kGapMask = (1u << 29) - 1u;
template <bool WIDE>
__device__ __forceinline__ uint32_t place_of(uint4 e) { return WIDE ? e.z & 0x7fffffffu : e.z; }
template <bool WIDE>
__device__ __forceinline__ uint32_t sum_of_visit(uint4 e) { return e.w >> 30 | (WIDE ? e.z >> 31 << 2 : 0u); }
template <bool WIDE>
constexpr uint32_t kNoSum = WIDE ? 7u : 3u;
constexpr int64_t kStepsMaxD = 1ll << 29;              // offsets and gaps of longer vectors do not fit

// Offsets and gaps of the visits of a list, by the lanes of a wavefront together.  A power-of-two list has four gaps
// and a 2-bit code per visit: the offset of a visit is how often each code comes before it, counted word by word
// and summed up over the words once.  Other lists have their gaps one by one.
struct VisitPlaces {
    uint32_t codes, before;      // my word of the list; numbers of the codes 1, 2, 3 in the words before it, 10 bits each
    __device__ __forceinline__ static uint32_t numbers(uint32_t w) {
        const uint32_t lo = w & 0x55555555u, hi = w >> 1 & 0x55555555u;
        return static_cast<uint32_t>(__builtin_popcount(lo & ~hi)) | static_cast<uint32_t>(__builtin_popcount(hi & ~lo)) << 10 |
               static_cast<uint32_t>(__builtin_popcount(lo & hi)) << 20;
    }
    __device__ __forceinline__ void init(const VisitArgs& v) {
        static_assert(CS_MAX_VISITS == 512, "32 words, numbers below 2^10");
        const uint32_t lane = threadIdx.x & 63;
        codes = lane < CS_MAX_VISITS / 16 ? v.code[lane] : 0u;
        uint32_t upto = numbers(codes);
#pragma unroll
        for (uint32_t off = 1; off < CS_MAX_VISITS / 16; off <<= 1) {
            const uint32_t other = __shfl_up(upto, off);
            upto += lane >= off ? other : 0u;
        }
        before = upto - numbers(codes);
    }
    // offset (at most kStepsMaxD) and gap (at most kGapMask) of visit k, which may differ between the lanes
    __device__ __forceinline__ void at(const VisitArgs& v, uint32_t k, uint32_t& s, uint32_t& gap) const {
        const uint32_t w = __shfl(codes, k >> 4), bits = 2u * (k & 15u);
        const uint32_t n = __shfl(before, k >> 4) + numbers(w & ((1u << bits) - 1u));
        const uint32_t n1 = n & 1023u, n2 = n >> 10 & 1023u, n3 = n >> 20;
        uint64_t x = v.gap[0] * (k - n1 - n2 - n3) + v.gap[1] * n1 + v.gap[2] * n2 + v.gap[3] * n3;
        s = static_cast<uint32_t>(x < kStepsMaxD ? x : kStepsMaxD);
        const uint32_t code = w >> bits & 3u;
        x = code == 0u ? v.gap[0] : code == 1u ? v.gap[1] : code == 2u ? v.gap[2] : v.gap[3];
        gap = static_cast<uint32_t>(x < kGapMask ? x : kGapMask);
    }
    __device__ __forceinline__ void init(const VisitGaps&) {}
    // (the lanes ask for neighbouring visits, the first lane for the first)
    __device__ __forceinline__ void at(const VisitGaps& v, uint32_t k, uint32_t& s, uint32_t& gap) const {
        const uint32_t lane = threadIdx.x & 63, base = __builtin_amdgcn_readfirstlane(k);
        auto gap_of = [&](uint32_t t) { return v.gap[t] < kGapMask ? v.gap[t] : kGapMask; };
        gap = k < v.K ? gap_of(k) : 0u;
        uint64_t sum = 0;                              // of the gaps before the first lane's visit
        for (uint32_t t = lane; t < base; t += 64) sum += gap_of(t);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
        uint64_t upto = gap;                           // of the gaps from there up to mine
#pragma unroll
        for (uint32_t off = 1; off < 64; off <<= 1) {
            const uint64_t other = __shfl_up(upto, off);
            upto += lane >= off ? other : 0u;
        }
        sum += upto - gap;
        s = static_cast<uint32_t>(sum < kStepsMaxD ? sum : kStepsMaxD);
    }
};

// The way of a workgroup through its visits: the workgroups that the chip holds at a time begin together, take about the same
// time and so pass over the vectors side by side.  The first such round walks down from the last visit, the
// next up, and so on: every round begins where the round before ended, on what the memory-side cache (256 MB) still holds of
// that, and the first on the end of vectors that a pass before wrote in order (dense state).  Us a step, all
// rounds up / in turn: 5 x 2^18, 11 M, 8 workers, dense 778 / 764 (in turn, rounds of half the size 784), 7 x 2^19, 25 M, 256 workers
// 34 580 / 33 400 (rounds of two thirds 35 260, of four thirds 34 130), 15 x 180 000, 90 M, 4 workers 6500 / 6350, 5 x 2^20, 10^8,
// 32 workers 13 640 / 13 520.  The more of the vectors the cache holds, the more of a round's reads it answers.  (Of 55 drawn updates
// 0.7 % in the mean, 3 to 5 % in a fifth of them, and two slower: 5 x 2^18, 27 M, 24 workers 2060 / 2190, 3 x 2^19, 20 M, 8 workers
// 386 / 403.)  Launches of several groups of workers count by blockIdx.x alone: their groups read other vectors.
__device__ __forceinline__ bool walks_down(uint32_t at_once) { return (blockIdx.x / at_once & 1u) == 0; }

// The visits k0 .. k1 - 1, by all wavefronts of the workgroup, the last one first with `down`; returns how many of them are
// not `none`.  within: A mod c must be below it.
template <bool POW2, int NWAVE, bool WIDE = false, typename ARGS>
__device__ __forceinline__ uint32_t fill_visit_steps(uint4* steps, const VisitPlaces& places, const ARGS& v, uint32_t k0,
                                                     uint32_t k1, const Columns& col, uint32_t within, bool down) {
    __shared__ uint32_t count[CS_MAX_VISITS / 64];
    const uint32_t lane = threadIdx.x & 63, wq = threadIdx.x >> 6;
    const uint32_t chunks = (k1 - k0 + 63) / 64;
    for (uint32_t chunk = wq; chunk < chunks; chunk += NWAVE) {
        const uint32_t k = k0 + chunk * 64 + lane;
        uint32_t s, gap;
        places.at(v, k, s, gap);
        const uint64_t A = mulmod_p(v.a, s), As = mulmod_p(v.as, s);
        const uint32_t cell = bucket_of<POW2>(A + 1, col);
        const uint32_t q = cell < within ? cell : kNoSum<WIDE>;
        const uint32_t listed = __builtin_popcountll(__builtin_amdgcn_ballot_w64(k < k1 && q < kNoSum<WIDE>));
        if (lane == 0) count[chunk] = listed;
        if (k < k1)
            steps[down ? k1 - 1 - k : k - k0] =
                make_uint4(threshold_of(A), threshold_of(As), WIDE ? s | q >> 2 << 31 : s,
                           gap | static_cast<uint32_t>(As & 1u) << 29 | q << 30);
    }
    __syncthreads();
    uint32_t listed = 0;
    for (uint32_t ch = 0; ch < chunks; ++ch) listed += count[ch];
    return __builtin_amdgcn_readfirstlane(listed);
}

// The visits of steps[0 .. n) that are not `3` and that residues from first_res on take part in, one after the other: a list with one
// short and one long gap leaves most walkers with few of its visits (K = 277, gaps 243 885 and 1 495 226:
// 66 for five residues in six), and looking at 64 visits at once finds the next without stepping through the others.
template <bool WIDE = false>
struct VisitCursor {
    const uint4* steps;
    uint64_t todo;                                      // visits base .. base + 63 that are left
    uint32_t base, n;
    uint32_t first_res, d;
    __device__ __forceinline__ void look() {
        const uint32_t k = base + (threadIdx.x & 63);
        const uint4 e = steps[k < n ? k : 0];
        todo = __builtin_amdgcn_ballot_w64(k < n && sum_of_visit<WIDE>(e) < kNoSum<WIDE> && (e.w & kGapMask) > first_res &&
                                          place_of<WIDE>(e) + first_res < d);
    }
    __device__ __forceinline__ VisitCursor(const uint4* steps_, uint32_t n_, uint32_t first_res_, uint32_t d_)
        : steps(steps_), base(0), n(n_), first_res(first_res_), d(d_) { look(); }
    // the next visit, or ~0u
    __device__ __forceinline__ uint32_t next() {
        while (todo == 0) {
            if (base + 64 >= n) return ~0u;
            base += 64;
            look();
        }
        const uint32_t k = base + static_cast<uint32_t>(__builtin_ctzll(todo));
        todo &= todo - 1;
        return k;
    }
};

// LIST = VisitRows (power-of-two column counts: three gaps and 2-bit codes, the ncell cells of a
// coordinate are neighbours) or VisitGapsRows (any column count: gaps one by one, ncell = 2 omega cells of which
// the second half lies p mod c cells back).
//
// One lane of a walker tells cell and sign of RUN / WL of the walker's coordinates, and the comparisons of a
// wavefront are two masks per coordinate of a lane, from which every lane takes the bits of its walker.
// The NC >= ncell sums of a coordinate stay in registers; the two that a visit adds to are `plain` and `wrapped`, the
// others are moved there when the visits come to another value of A mod c, so that the additions are written once.
// All of a coordinate leave together at the end: sent one by one as they are complete, its cells, which are
// neighbours, were fetched and written back by the memory-side cache once each (d = 10^8, 8 workers, 5 x 2^20: 3455 us).
// Measured against records of sign and masks in LDS, two 61-bit states per pair of coordinates, and a turn for every
// visit of the list (us, update alone): d = 6.5 M, 8 workers, 5 x 2^17 206 -> 184; 6.5 M, 5 x 180 000 268 -> 246; 11 M,
// 5 x 2^18 317 -> 304; 3 M, 2 workers, 3 x 2^15 48 -> 42; 90 M, 4 workers, 15 x 180 000 4177 -> 4074; 10^8, 8 workers,
// 5 x 2^20 3260 -> 3156; 25 M, 7 x 2^19 1068 -> 1075; 40 M, 5 x 2^19 1116 -> 1143 (lists whose walkers nearly all take part
// in nearly all visits have nothing to skip; the whole update by either way 1163 -> 1178 at 40 M, a step 1617 -> 1638).
// Bound: reads.  By the counters a launch at 10^8 reads 16.5 GB (16.0 GB and the cache lines that two wavefronts share) and
// moves 16.9 with its requests, 17.1 with its sums to the workspace, at 5.6 to 5.8 TB/s; without requests or sums it takes
// 2690 us, 6.1 TB/s.  Sums waiting in
// LDS instead of registers: 10^8 3130, 25 M 1131; four wavefronts in step by a barrier per visit: 11 M 293, 10^8 3269.
// PARTIAL (power-of-two columns): the sums go to a workspace instead of being added to the table (cs_index.hip).
// PAIRS: two neighbouring cells of a bundle leave as one request (with RUN = 16 a kernel of its own, which is not for `fold`).
template <int WL, int RUN, int NWAVE, int NC, bool PARTIAL, bool PAIRS, typename LIST>
__global__ void __launch_bounds__(64 * NWAVE)
k_accumulate_visits(LIST rows, WorkersBeside<LIST> a) {
    constexpr bool POW2 = std::is_same<LIST, VisitRows>::value;
    const unsigned row = row_of_block(rows);
    const auto& v = rows.at(row);
    const uint32_t piece = (blockIdx.x - rows.first[row]) / v.blocks;
    const uint32_t block = (blockIdx.x - rows.first[row]) % v.blocks;
    constexpr int WPW = 64 / WL;                       // walkers per wavefront
    constexpr int PPL = RUN / WL;                      // coordinates whose hashes a lane looks at
    constexpr int SPAN = WPW * RUN;                    // residues a wavefront owns
    constexpr int kStride = RUN + 1;
    static_assert(WL <= 8 && WL * PPL == RUN, "every coordinate of a walker gets a hash lane");
    // PAIRS: two neighbouring cells of a bundle are one aligned 64-byte block when the lower one is even, and leave as one request
    // then: on average ncell / 2 + 1/2 requests per residue instead of ncell.  For that the sums go through LDS.
    static_assert(!PAIRS || (!PARTIAL && POW2), "neighbouring cells");
    // Per wavefront: the value tile (one padded row per lane), the walkers' first cells and signs
    __shared__ float tile_lds_all[NWAVE][64 * kStride];
    __shared__ uint32_t first_lds_all[NWAVE][SPAN];
    // the visits of my piece, behind them the sums that wait, [][RUN][64] per wavefront
    extern __shared__ uint4 steps[];

    const int lane = threadIdx.x & 63;
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wavefront-uniform
    float* tile_lds = tile_lds_all[wq];
    uint32_t* first_lds = first_lds_all[wq];
    const int h = lane / WL, wl = lane % WL;
    const uint32_t group = blockIdx.y;
    const float* const* vectors = a.g + group * kGroup;
    const int nw = a.nw - static_cast<int>(group) * kGroup < kGroup ? a.nw - static_cast<int>(group) * kGroup : kGroup;
    const bool live = wl < nw;                          // my worker exists
    float* const T = a.T + group * a.table_floats;

    const int64_t chunks = (static_cast<int64_t>(v.gmax) + RUN - 1) / RUN;
    const int64_t nwaves = (chunks + WPW - 1) / WPW;
    const uint32_t mask = a.c - 1u;
    const Columns col = columns_of<POW2>(a.c);
    const uint32_t d = static_cast<uint32_t>(a.d);
    const bool fold = !(PAIRS && RUN == 16) && a.fold != 0;
    const size_t cell_floats = fold ? 1 : kGroup;      // floats from one cell to the next
    float* __restrict__ Tcol = fold ? T + static_cast<size_t>(v.j) * a.c
                                    : T + static_cast<size_t>(v.j) * a.c * kGroup + wl;
    uint32_t ncell, omega;                             // running sums, and the values of A mod c that they cover
    if constexpr (POW2) {
        ncell = v.ncell;
        omega = ncell - 1;
    } else {
        omega = v.omega;
        ncell = 2 * omega;
    }
    // the cell of running sum q of a coordinate that started in cell `first`
    auto cell_of_sum = [&](uint32_t first, uint32_t q) -> uint32_t {
        if constexpr (POW2) {
            return (first + q) & mask;
        } else {
            const uint32_t c = a.c;
            // (the half of the sums that wrapped past p begins at NC / 2, also in rows that use fewer)
            const uint32_t x = q < NC / 2 ? first + q : first + (q - NC / 2) + (c - v.pc);
            return x >= c ? x - c : x;
        }
    };
    const int m0 = wl * PPL;                           // hash role: coordinates m0 .. m0 + PPL - 1
    float* my_row = tile_lds + lane * kStride;         // consumer role: my walker's run of my worker
    // loader role: floats lspan .. lspan + kPer - 1 of the wavefront's span of one worker at a time;
    // they belong to walker lspan / RUN and go to that walker's row of the worker.  Requests are 16
    // bytes or more per lane: where a worker's span is shorter than 64 of them, kShare workers
    // share a request (8 workers and RUN = 16: two, 512 bytes of each; against 8-byte
    // pieces the same time with half the load instructions and 16 VGPRs fewer).
    constexpr int kShare = SPAN >= 256 ? 1 : 256 / SPAN;
    constexpr int kLoads = WL / kShare;                // load instructions per visit
    constexpr int kPer = SPAN >= 256 ? SPAN / 64 : 4;  // floats per lane and instruction
    constexpr int kLanesPerWorker = 64 / kShare;
    static_assert(kLoads * kShare == WL && kPer <= RUN, "whole requests, each within one run");
    const int part = lane / kLanesPerWorker;
    const int lspan = (lane % kLanesPerWorker) * kPer;
    float* tile_dst = tile_lds + ((lspan / RUN) * WL + part) * kStride + lspan % RUN;
    constexpr int kRowStep = kShare * kStride;         // tile rows between my loads
    gfloat_ptr src_of[kLoads];                         // where load instruction w of this lane reads, at residue 0
#pragma unroll
    for (int w = 0; w < kLoads; ++w) {
        const int from = w * kShare + part;
        src_of[w] = (gfloat_ptr)vectors[from < nw ? from : 0] + lspan;
    }
    // Walkers with small residues take part in every visit, those with large ones only in
    // the visits with the largest gap, so the sets of walkers are dealt to the XCDs in short
    // blocks rather than as eight long ranges: every XCD gets the same mix.
    const int64_t ngroups = (nwaves + NWAVE - 1) / NWAVE;
    // my piece of the chain of visits: k0 .. k1 - 1
    const uint32_t k0 = v.K * piece / v.pieces, k1 = v.K * (piece + 1) / v.pieces;
    VisitPlaces places;
    places.init(v);
    const uint32_t listed = fill_visit_steps<POW2, NWAVE>(steps, places, v, k0, k1, col, omega, walks_down(a.at_once));
    for (int64_t vi = block; ; vi += v.blocks) {
        if (visit_round(vi, v.blocks) >= ngroups) break;
        const int64_t set = visit_set(vi, v.blocks);
        const int64_t wv = set * NWAVE + wq;
        if (set >= ngroups || wv >= nwaves) continue;
        const uint32_t first_res = static_cast<uint32_t>(wv * SPAN);   // first residue of this wavefront's walkers
        const uint32_t* first = first_lds + h * RUN;

        // Requests of a visit.  `room` = residues from first_res on that belong
        // to the visit and exist; when the whole span does, every piece is whole and needs no
        // check (one wavefront-uniform base per worker plus a fixed lane offset).  Otherwise
        // pieces are cut where the visit or the vector ends, and missing values count as 0.
        float pre[kLoads][kPer];
        auto load_visit = [&](uint32_t s, uint32_t w) {
            const uint32_t in_gap = (w & kGapMask) - first_res, in_vec = d - s - first_res;
            const uint32_t room = in_gap < in_vec ? in_gap : in_vec;
            if (room >= SPAN) {
#pragma unroll
                for (int l = 0; l < kLoads; ++l) load_floats<kPer>(src_of[l] + (first_res + s), pre[l]);
            } else {
                const int len = static_cast<int>(room) - lspan;    // of my piece: >= kPer whole, <= 0 none
#pragma unroll
                for (int l = 0; l < kLoads; ++l) {
                    const gfloat_ptr src = src_of[l] + (first_res + s);
#pragma unroll
                    for (int t = 0; t < kPer; ++t) pre[l][t] = 0.0f;
                    if (len >= kPer) {
                        load_floats<kPer>(src, pre[l]);
                    } else {
#pragma unroll
                        for (int t = 0; t < kPer; ++t)
                            if (t < len) pre[l][t] = src[t];
                    }
                }
            }
        };
        uint32_t xb[PPL], xs[PPL];                     // top bits of the hashes at my walker's residues
        {
            uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(a.i0 + first_res + h * RUN + m0));
            uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(a.i0 + first_res + h * RUN + m0));
#pragma unroll
            for (int q = 0; q < PPL; ++q) {
                xb[q] = top_of(yb);
                xs[q] = top_of(ys);
                first_lds[h * RUN + m0 + q] = bucket_of<POW2>(yb, col) | sign_flip_of(ys);
                if (q + 1 < PPL) {
                    yb = hash_advance(yb, v.a);
                    ys = hash_advance(ys, v.as);
                }
            }
        }
        // sums of the coordinates whose bucket hash did not wrap and of those whose did, for visits with
        // A mod c = cur; their signs less that of the residue itself
        float plain[RUN], wrapped[RUN];
        uint32_t cur = 0;
#pragma unroll
        for (int m = 0; m < RUN; ++m) plain[m] = wrapped[m] = 0.0f;
        // The other sums.  Power-of-two c, where neighbouring cells share a sum: sum q is in other[q mod 2] (two on is
        // the one that comes for it; other[0] if there are three), else those of the other value of A mod c.
        float other[NC > 2 ? NC - 2 : 1][RUN];
#pragma unroll
        for (int t = 0; t < NC - 2; ++t)
#pragma unroll
            for (int m = 0; m < RUN; ++m) other[t][m] = 0.0f;
        auto move_to = [&](uint32_t q) {
            if (cur == q) return;
            if constexpr (!POW2) {
                if constexpr (NC > 2) {
#pragma unroll
                    for (int m = 0; m < RUN; ++m) {
                        const float p = plain[m], w = wrapped[m];
                        plain[m] = other[0][m];
                        wrapped[m] = other[1][m];
                        other[0][m] = p;
                        other[1][m] = w;
                    }
                }
                cur = q;
            } else if constexpr (NC > 2) {
                while (cur != q) {
                    const bool up = cur < q, second = NC > 3 && (up ? cur == 1u : cur == 2u);    // of other[]
#pragma unroll
                    for (int m = 0; m < RUN; ++m) {
                        const float o0 = other[0][m], o1 = other[NC - 3][m], lower = plain[m], upper = wrapped[m];
                        const float in = second ? o1 : o0, out = up ? lower : upper;
                        other[NC - 3][m] = second ? out : o1;
                        other[0][m] = second ? o0 : out;
                        plain[m] = up ? upper : in;
                        wrapped[m] = up ? in : lower;
                    }
                    cur = up ? cur + 1 : cur - 1;
                }
            }
        };
        VisitCursor<> cursor(steps, k1 - k0, first_res, d);
        uint32_t k = cursor.next();                    // the visit whose values are on their way
        uint4 e = steps[k == ~0u ? 0u : k];
        if (k != ~0u) load_visit(__builtin_amdgcn_readfirstlane(e.z), __builtin_amdgcn_readfirstlane(e.w));
        uint32_t k_next = cursor.next();
        uint4 e_next = steps[k_next == ~0u ? 0u : k_next];
        while (k != ~0u) {
            const uint32_t w = __builtin_amdgcn_readfirstlane(e.w);
            move_to(w >> 30);
#pragma unroll
            for (int l = 0; l < kLoads; ++l)
#pragma unroll
                for (int t = 0; t < kPer; ++t) tile_dst[l * kRowStep + t] = pre[l][t];
            // request the next visit as soon as the registers of this one are free, to fly while
            // this one is looked at and added up
            if (k_next != ~0u) load_visit(__builtin_amdgcn_readfirstlane(e_next.z), __builtin_amdgcn_readfirstlane(e_next.w));
            uint64_t flips[PPL], wraps[PPL];           // lane h WL + l: coordinate l PPL + q of walker h
            bool unsure = false;
#pragma unroll
            for (int q = 0; q < PPL; ++q) {
                flips[q] = __builtin_amdgcn_ballot_w64(xs[q] > e.y);
                wraps[q] = __builtin_amdgcn_ballot_w64(xb[q] > e.x);
                unsure |= xs[q] == e.y || xb[q] == e.x;
            }
            if (__builtin_amdgcn_ballot_w64(unsure) != 0) {
                // the lower bits decide: whole hash values against whole thresholds
                const uint64_t A = mulmod_p(v.a, e.z), As = mulmod_p(v.as, e.z);
                uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(a.i0 + first_res + h * RUN + m0));
                uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(a.i0 + first_res + h * RUN + m0));
#pragma unroll
                for (int q = 0; q < PPL; ++q) {
                    flips[q] = __builtin_amdgcn_ballot_w64(ys > kP61 - As);
                    wraps[q] = __builtin_amdgcn_ballot_w64(yb > kP61 - A);
                    yb = hash_advance(yb, v.a);
                    ys = hash_advance(ys, v.as);
                }
            }
            {
                // the bits of my walker: bit l of word q is coordinate l PPL + q
                uint32_t flip[PPL], wrap[PPL];
                const uint64_t odd = (w >> 29 & 1u) != 0 ? ~0ull : 0ull;
#pragma unroll
                for (int q = 0; q < PPL; ++q) {
                    const uint64_t f = flips[q] ^ odd;
                    const uint32_t shift = static_cast<uint32_t>(h * WL) & 31u;
                    flip[q] = (lane < 32 ? static_cast<uint32_t>(f) : static_cast<uint32_t>(f >> 32)) >> shift;
                    wrap[q] = (lane < 32 ? static_cast<uint32_t>(wraps[q]) : static_cast<uint32_t>(wraps[q] >> 32)) >> shift;
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int m = 0; m < RUN; ++m) {
                    const int l = m / PPL, q = m % PPL;
                    const uint32_t bits = __float_as_uint(my_row[m]) ^ ((flip[q] << (31 - l)) & 0x80000000u);
                    const uint32_t to = static_cast<uint32_t>(static_cast<int32_t>(wrap[q] << (31 - l)) >> 31);
                    plain[m] += __uint_as_float(bits & ~to);
                    wrapped[m] += __uint_as_float(bits & to);
                    // keeps the LDS reads of later coordinates from being hoisted over the sums
                    // of earlier ones, which would cost a register per read in flight
                    if (m % 4 == 3) __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_wave_barrier();
            k = k_next;
            e = e_next;
            k_next = cursor.next();
            e_next = steps[k_next == ~0u ? 0u : k_next];
        }
        // every sum in its place: plain, wrapped = sums 0 and 1 (0 and omega)
        move_to(0);
        auto sum_of = [&](int q, int m) -> float {
            if constexpr (POW2) return q == 0 ? plain[m] : q == 1 ? wrapped[m] : other[q > 1 && q - 2 < NC - 2 ? q - 2 : 0][m];
            else return q == 0 ? plain[m] : q == NC / 2 ? wrapped[m] : other[q > 1 && NC > 2 ? 1 : 0][m];
        };
        if constexpr (PARTIAL) {
            // [piece][wavefront][m][walker][running sum][worker]: the sums of a residue are neighbours, as the cells are
            // that they belong to
            float* dst = a.sums + group * a.sums_floats + v.at + (static_cast<uint64_t>(piece) * nwaves + wv) * (SPAN * WL) * ncell + h * ncell * WL + wl;
#pragma unroll
            for (int m = 0; m < RUN; ++m) {
                const uint32_t flip = first[m] & 0x80000000u;
#pragma unroll
                for (int q = 0; q < NC; ++q)
                    if (q < static_cast<int>(ncell))
                        dst[(m * WPW * ncell + q) * WL] = live ? apply_sign(a.scale * sum_of(q, m), flip) : 0.0f;
            }
        } else if (PAIRS && !fold) {
            // The sums of a residue take the slots of those blocks in LDS (an even first cell: slots 0 .. ncell-1, an
            // odd one: 1 .. ncell), and a block then leaves as one request.
            constexpr int kSlots = (NC + 2) / 2 * 2;
#pragma unroll
            for (int m = 0; m < RUN; ++m) {
                const uint32_t f = first[m], odd = f & 1u;
                float* dst = tile_lds + h * (kSlots * WL) + wl;
#pragma unroll
                for (int q = 0; q < kSlots; ++q) {
                    // slot q holds sum q (even first cell) or q - 1 (odd)
                    const float even_v = q < NC ? sum_of(q < NC ? q : 0, m) : 0.0f;
                    const float odd_v = q > 0 && q - 1 < NC ? sum_of(q > 0 && q - 1 < NC ? q - 1 : 0, m) : 0.0f;
                    dst[q * WL] = live ? apply_sign(odd ? odd_v : even_v, f & 0x80000000u) : 0.0f;
                }
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int t = 0; t < kSlots; ++t) {     // WPW * kSlots * WL items, 64 at a time
                    const uint32_t item = t * 64 + lane;
                    const uint32_t of = item / (kSlots * WL), slot = item / WL % kSlots, from = item % WL;
                    const float sum = tile_lds[item];
                    const uint32_t cell0 = first_lds[of * RUN + m] & 0x7ffffffeu;
                    if (sum != 0.0f)
                        atomic_add_noret(T + (static_cast<size_t>(v.j) * a.c + ((cell0 + slot) & mask)) * kGroup + from,
                                         a.scale * sum);
                }
                __builtin_amdgcn_wave_barrier();
            }
        } else {
#pragma unroll
            for (int m = 0; m < RUN; ++m) {
                const uint32_t f = first[m], flip = f & 0x80000000u;
#pragma unroll
                for (int q = 0; q < NC; ++q) {
                    float x = live ? sum_of(q, m) : 0.0f;
                    if (fold) {                        // the WL lanes of my walker hold the workers' sums of a cell
#pragma unroll
                        for (int off = 1; off < WL; off <<= 1) x += __shfl_xor(x, off);
                        if (wl != 0) x = 0.0f;
                    }
                    if (x != 0.0f)
                        atomic_add_noret(Tcol + static_cast<size_t>(cell_of_sum(f & 0x7fffffffu, q)) * cell_floats,
                                         apply_sign(a.scale * x, flip));
                }
            }
        }
        // Visits whose cells are not kept (which cannot be with a list built by cs_params_init: a wrong list costs
        // time, never correctness): hashed by the definition, straight into memory.
        if (!PARTIAL && listed < k1 - k0) {
            const gfloat_ptr of_mine = (gfloat_ptr)vectors[live ? wl : 0];
            for (uint32_t t = 0; t < k1 - k0; ++t) {
                if (__builtin_amdgcn_readfirstlane(steps[t].w) >> 30 < 3u) continue;
                const uint32_t s = __builtin_amdgcn_readfirstlane(steps[t].z), gap = __builtin_amdgcn_readfirstlane(steps[t].w) & kGapMask;
                if (gap <= first_res || s + first_res >= d) continue;
                const uint32_t in_gap = gap - first_res, in_vec = d - s - first_res;
                const int len = static_cast<int>(in_gap < in_vec ? in_gap : in_vec) - h * RUN;     // of my walker's run
                const uint32_t at = s + first_res + h * RUN;
                uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(a.i0 + at));
                uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(a.i0 + at));
                for (int m = 0; m < RUN && m < len; ++m) {
                    const float val = live ? apply_sign(a.scale * of_mine[at + m], sign_flip_of(ys)) : 0.0f;
                    if (val != 0.0f)
                        atomic_add_noret(Tcol + static_cast<size_t>(bucket_of<POW2>(yb, col)) * cell_floats, val);
                    yb = hash_advance(yb, v.a);
                    ys = hash_advance(ys, v.as);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// Pieces that the chains of visits of a launch are cut into, each walked by wavefronts of its own.
// A wavefront makes its visits one after the other, visit_ns each when the chip is not full, and
// every piece sends its own requests (requests[q] per piece of row q) at 24 G/s: the common
// length of the pieces with the smallest sum of the two is taken.  stream_ns: what the launch
// takes to read its vectors in any case, so that long vectors, which fill the chip, stay whole.
constexpr uint32_t kMaxPieces = 32;
template <typename LIST>
void choose_pieces(LIST& rows, int nrows, const double* requests, double visit_ns, double stream_ns, int groups = 1) {

    uint32_t longest = 1;
    for (int q = 0; q < nrows; ++q) longest = rows.row[q].K > longest ? rows.row[q].K : longest;
    double best = 1e300, best_len = longest;
    for (double len = longest; len >= 3.0; len *= 0.8) {
        double cost = len * visit_ns > stream_ns ? len * visit_ns : stream_ns;
        if (groups > 1) cost += 0.5 * len * visit_ns;
        for (int q = 0; q < nrows; ++q) cost += ceil(rows.row[q].K / len) * requests[q] / 24.0;
        if (cost < best) { best = cost; best_len = len; }
    }
    for (int q = 0; q < nrows; ++q) {
        const double n = ceil(rows.row[q].K / best_len);
        rows.row[q].pieces = n < 1.0 ? 1u : n > kMaxPieces ? kMaxPieces : static_cast<uint32_t>(n);
    }
}

// A turn of the walkers of 8 (4, 2) workers with RUN = 8 and with RUN = 16, and of a wavefront per vector.  (The
// planner, which knows neither the workers nor the run length that a launch will have, prices a
// turn at 900 ns.)
// (priced as RUN = 8, chains of 316 visits of 4 workers stayed whole: d = 22.4 M, c = 65 536, 738 us a step for 596)
// (of 2 to 8 vectors: priced at 650, as with the chip full, 805 timings of drawn shapes take 3 % more in the mean, and a single table's requests
// at one or two for all of a residue's sums 2 %)
constexpr double kVisitNs8 = 700.0, kVisitNs16 = 1300.0, kVisitNsOne = 500.0;
constexpr double kStreamBytesPerNs = 5000.0;

// The same for a group of workers; true = RUN = 8.  requests8, requests16: what a residue of each row
// sends with either run length.
// RUN = 16 with few wavefronts leaves most of the chip idle (1024 SIMDs): RUN = 8 then gives twice as
// many, each with half the work per visit, which is what a short vector's time consists of.  Up to 2048 wavefronts, and with
// a power of two of columns up to 3 million coordinates twice that, four times with 8 lanes a walker (us, 16 / 8: 5 x 131 072,
// 2.55 M, 5 workers 115 / 98; 5 x 32 768, 563 996, 6 workers 39 / 34; 15 x 4096, 608 341, 6 workers 80 / 73; 7 x 16 384, 1.8 M,
// 3 workers 61 / 56; but 5 x 131 072, 9.9 M, 4 workers 166 / 196, 5 x 65 536, 7.2 M, 9 workers 287 / 335).
template <int WL, typename LIST>
bool choose_run8(LIST& rows, int nrows, const double* requests8, const double* requests16, int64_t d, double stream_ns,
                 int groups = 1) {
    choose_pieces(rows, nrows, requests8, kVisitNs8, stream_ns, groups);
    int64_t waves = 0;                                   // with RUN = 16
    for (int q = 0; q < nrows; ++q) waves += static_cast<int64_t>(rows.row[q].gmax) * WL / 1024 * rows.row[q].pieces;
    constexpr bool pow2 = std::is_same<LIST, VisitRows>::value;
    if (groups > 1 || waves < 2048 || (pow2 && d < 3'000'000 && waves < (WL == 8 ? 8192 : 4096))) return true;
    choose_pieces(rows, nrows, requests16, kVisitNs16, stream_ns);
    return false;
}

void fill_visit_args(const cs_params* p, uint32_t j, const cs_visit_plan& vp, VisitArgs& v) {
    v.K = vp.K;
    v.j = static_cast<int32_t>(j);
    v.gmax = vp.gmax;
    v.a = p->a[j]; v.b = p->b[j]; v.as = p->as[j]; v.bs = p->bs[j];
    v.ncell = vp.ncell;
    for (int t = 0; t < 4; ++t) v.gap[t] = vp.gap[t];
    for (int t = 0; t < CS_MAX_VISITS / 16; ++t) v.code[t] = vp.code[t];
}

void fill_visit_args(const cs_params* p, uint32_t j, VisitArgs& v) { fill_visit_args(p, j, p->visit[j], v); }

// Workgroups of a launch of nrows rows whose gmax and pieces are set; fills in `blocks` and `first`.
template <int WL, int RUN, int NWAVE, typename LIST>
unsigned visits_grid(LIST& rows, int nrows) {
    constexpr int WPW = 64 / WL;
    constexpr int N = sizeof(rows.first) / sizeof(rows.first[0]);
    auto lay_out = [&](bool singly) -> unsigned {
        unsigned total = 0;
        for (int q = 0; q < nrows; ++q) {
            const int64_t chunks = (static_cast<int64_t>(rows.row[q].gmax) + RUN - 1) / RUN;
            const int64_t nwaves = (chunks + WPW - 1) / WPW;
            const int64_t ngroups = (nwaves + NWAVE - 1) / NWAVE;
            const int64_t cap = 256 * 64 / NWAVE;              // enough to fill the chip several times over
            int64_t n = ngroups < cap ? ngroups : cap;
            // the kernel deals sets to the 8 XCDs in blocks of kVisitSetBlock: whole rounds, so that
            // no workgroup takes a second set
            if (!singly || n >= kVisitRound) n = (n + kVisitRound - 1) / kVisitRound * kVisitRound;
            rows.row[q].blocks = static_cast<uint32_t>(n);
            rows.first[q] = total;
            total += rows.row[q].blocks * rows.row[q].pieces;
        }
        return total;
    };
    unsigned total = lay_out(false);
    if (total > kRoundsUpTo) total = lay_out(true);
    for (int q = nrows; q < N; ++q) rows.first[q] = ~0u;
    return total;
}

// Visits of the longest piece of a launch's lists
template <typename LIST>
uint32_t most_steps(const LIST& rows, int nrows) {
    uint32_t most = 1;
    for (int q = 0; q < nrows; ++q) {
        const uint32_t n = (rows.row[q].K + rows.row[q].pieces - 1) / rows.row[q].pieces;
        most = n > most ? n : most;
    }
    return most;
}

// Workgroups of a kernel that the chip holds at a time.  The runtime works it out from the kernel's registers and LDS, and is asked
// once for each of the last kLdsSizes amounts of LDS: sketches of more rows than a launch takes, and programs with several
// sketches, go through a few in turn.  (Us of host work a call, asked at every launch / with one amount known / so: 15 x 4096, two
// launches 9.5 / 9.2 / 9.0; 5 x 4096, one 6.2 / 5.9 / 5.9.)
constexpr unsigned kLdsSizes = 8;
template <auto KERNEL>
uint32_t workgroups_at_once(int threads, size_t lds) {
    static std::atomic<uint64_t> known[kLdsSizes];     // LDS, workgroups; 0 = none yet
    static std::atomic<unsigned> oldest{0};
    for (const auto& one : known) {
        const uint64_t k = one.load(std::memory_order_relaxed);
        if (k != 0 && k >> 32 == lds) return static_cast<uint32_t>(k);
    }
    int per_cu = 0, device = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, KERNEL, threads, lds) != hipSuccess || per_cu < 1 ||
        hipGetDevice(&device) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus < 1) {
        (void)hipGetLastError();
        return 256u;                                   // (an order of visits like any other; asked again next time)
    }
    const uint32_t n = static_cast<uint32_t>(cus) * static_cast<uint32_t>(per_cu);
    known[oldest.fetch_add(1, std::memory_order_relaxed) % kLdsSizes].store(static_cast<uint64_t>(lds) << 32 | n,
                                                                            std::memory_order_relaxed);
    return n;
}

// one launch: rows that all have at most ncell running sums, of the groups of workers that `a` holds
template <int WL, int RUN, int NWAVE, bool PAIRS16 = false, typename LIST>
int launch_visits_run(LIST& rows, WorkersBeside<LIST> a, int nrows, uint32_t ncell, hipStream_t stream) {
    const dim3 grid(visits_grid<WL, RUN, NWAVE>(rows, nrows), (a.nw + kGroup - 1) / kGroup), block(64 * NWAVE);
    const size_t lds = most_steps(rows, nrows) * sizeof(uint4);
    constexpr bool pow2 = std::is_same<LIST, VisitRows>::value;
    constexpr bool partial = pow2 && WL > 1;           // running sums: power-of-two columns
    constexpr bool pairs = pow2 && (RUN == 8 || PAIRS16);
    if (!(a.sums ? partial : a.T != nullptr) || (PAIRS16 && (a.sums || a.fold))) return CS_EINVAL;
    auto launch = [&](auto nc) {
        constexpr int NC = decltype(nc)::value;
        auto with = [&](auto sums) {
            constexpr bool to_sums = decltype(sums)::value;
            constexpr auto kernel = k_accumulate_visits<WL, RUN, NWAVE, NC, to_sums, pairs && !to_sums, LIST>;
            a.at_once = workgroups_at_once<kernel>(64 * NWAVE, lds);
            kernel<<<grid, block, lds, stream>>>(rows, a);
        };
        if constexpr (partial && !PAIRS16) {
            if (a.sums) return with(std::true_type());
        }
        with(std::false_type());
    };
    if (ncell == 2) launch(std::integral_constant<int, 2>());
    else if (ncell == 4) launch(std::integral_constant<int, 4>());
    else if constexpr (pow2) launch(std::integral_constant<int, 3>());
    else return CS_EINVAL;
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

// ---------------------------------------------------------------------------------------
// The update of one vector (one worker, or the workers' vectors summed beforehand), or of a few that the
// memory-side cache holds together, along visit lists: a wavefront per vector.
//
// Nothing is shared between the lanes of a wavefront, so a lane owns 4 neighbouring residues: a visit
// is one 16-byte load, 8 comparisons and 8 masked additions in registers, and a
// wavefront reads 1 KB of contiguous addresses.  Loads of the next kOneAhead visits are in flight; every
// request is one whole load, at the vector's last four values where its own would lie beyond, so that
// the wait for a visit's values counts the loads behind them.  The sums of a residue that the present visits do not add to wait
// in LDS.  A workgroup has SETS sets of WL wavefronts, of which each takes another vector over the same residues; at the end the
// sums of all WL vectors, which lie in neighbouring cells of the bundle, are brought to
// neighbouring lanes, so that they leave as one request (an aligned 64-byte block touched by an
// instruction is one).  The workgroup shares one table of visits; launches of one vector with fewer than
// kOneFewWaves wavefronts have workgroups of one, which spread them over more CUs (us, 4 / 1: 21 wavefronts, 3 x 512,
// d = 203 680 16.9 / 12.8; 138, 5 x 707, 326 476 41.8 / 29.2; 269, 5 x 2048, 304 889 17.3 / 14.7; 338, 5 x 2401, 224 320
// 24.8 / 26.0; 642, 5 x 2641, 747 318 36.7 / 41.7; two launches of 16 000, 15 x 131 072, 31 M 536 / 572).
// Measured, one vector (update alone, in us; with two 61-bit states per coordinate and a load for every visit of the list, taken
// part in or not -> now): d = 73 M, 5 x 2^20 468 -> 326; d = 25 M, 5 x 2^19 176 -> 137; d = 11 M, 5 x 2^18 102 -> 74;
// d = 73 M, 5 x 180 000 492 -> 445; with waits for one visit's values at a time 338 -> 325, 126 -> 122, 73 -> 72, 434 -> 435 (of
// another machine).  Bound: the requests at the end (without them 216, 92, 43 and 227 us, which
// is the five reads, 1.46 GB at 73 M by the counters too, at 6.8 TB/s; with them 1.63 GB at 4.8), 64 bytes each and 21 G/s, so that
// for one vector a residue's sums cost one or two however many they are: along lists of its own with up to CS_VECTOR_CELLS of them
// 73 M takes 250, 25 M, 5 x 2^20 149 (250 before).  With more than 4 sums a CU holds 12 to 16 wavefronts instead of 24, so
// that each has a load more on its way.  2 and 4 loads ahead and 2
// and 8 wavefronts per workgroup, with up to 4 sums: within 4 % either way.
// Several vectors: against k_accumulate_visits, whose lanes are walkers times workers, the comparisons are made once per vector
// instead of once per walker, but no value goes through LDS, four times as many wavefronts have a quarter of the work
// each, and 24 of them on a CU have 72 KB of reads in flight instead of 48.  The memory-side cache answers that with 6.4 TB/s for
// 5.6 (d = 6.5 M, 8 workers, 5 x 2^17: 1.04 GB in 162 us for 185), memory does not: see vectors_pay.
// ---------------------------------------------------------------------------------------
constexpr int kOneRun = 4;
constexpr int kOneAhead = 3;
constexpr int64_t kOneFewWaves = 300;

// PARTIAL: the sums go to a workspace, [piece][residue][running sum][worker], instead of being added to the table
// (cs_index.hip).
template <int WL, int SETS, int NC, bool PARTIAL, typename LIST>
__global__ void __launch_bounds__(64 * WL * SETS)
k_accumulate_vectors(LIST rows, WorkersBeside<LIST> a) {
    constexpr bool WIDE = NC > 4;
    constexpr bool POW2 = std::is_same<LIST, VisitRows>::value;
    constexpr int SPAN = 64 * kOneRun, kRow = SPAN + 4, kAhead = WIDE ? kOneAhead + 1 : kOneAhead;
    const unsigned row = row_of_block(rows);
    const auto& v = rows.at(row);
    const uint32_t piece = (blockIdx.x - rows.first[row]) / v.blocks;
    const uint32_t block = (blockIdx.x - rows.first[row]) % v.blocks;
    const int lane = threadIdx.x & 63;
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wavefront-uniform
    const int worker = wq % WL, set = wq / WL;
    extern __shared__ uint4 steps[];                   // the visits of my piece
    __shared__ __attribute__((aligned(16))) float sums_lds[SETS][WL][NC][kRow];
    __shared__ uint32_t first_lds[PARTIAL ? 1 : SETS][SPAN];           // first cell of a residue
    float (*parked)[kRow] = sums_lds[set][worker];
    uint32_t* first = first_lds[PARTIAL ? 0 : set];
    const uint32_t group = blockIdx.y;
    const int nw = a.nw - static_cast<int>(group) * kGroup < kGroup ? a.nw - static_cast<int>(group) * kGroup : kGroup;
    const bool live = worker < nw;
    const gfloat_ptr g = (gfloat_ptr)a.g[group * kGroup + (live ? worker : 0)];
    const int64_t i0 = a.i0;
    const uint32_t c = a.c, mask = c - 1u, d = static_cast<uint32_t>(a.d);
    const Columns col = columns_of<POW2>(c);
    const float scale = a.scale;
    const bool fold = a.fold != 0;
    const uint32_t cell_floats = fold ? 1u : static_cast<uint32_t>(kGroup);
    uint32_t ncell, omega;                             // running sums, and the values of A mod c that they cover
    if constexpr (POW2) {
        ncell = v.ncell;
        omega = ncell - 1;
    } else {
        omega = v.omega;
        ncell = 2 * omega;
    }
    auto cell_of_sum = [&](uint32_t first, uint32_t q) -> uint32_t {
        if constexpr (POW2) {
            return (first + q) & mask;
        } else {
            const uint32_t x = q < omega ? first + q : first + (q - omega) + (c - v.pc);
            return x >= c ? x - c : x;
        }
    };
    float* const Tj = PARTIAL ? nullptr : a.T + group * a.table_floats + static_cast<uint64_t>(v.j) * c * cell_floats;
    const int64_t nwaves = (static_cast<int64_t>(v.gmax) + SPAN - 1) / SPAN;
    const int64_t nsets = (nwaves + SETS - 1) / SETS;
    const uint32_t k0 = v.K * piece / v.pieces, k1 = v.K * (piece + 1) / v.pieces;
    VisitPlaces places;
    places.init(v);
    const uint32_t listed = fill_visit_steps<POW2, WL * SETS, WIDE>(steps, places, v, k0, k1, col, omega, walks_down(a.at_once));
    const uint32_t last4 = d - kOneRun;

    // sets of neighbouring wavefronts go to one XCD, as in k_accumulate_visits
    for (int64_t vi = block; ; vi += v.blocks) {
        if (visit_round(vi, v.blocks) >= nsets) break;
        const int64_t wv = visit_set(vi, v.blocks) * SETS + set;
        const uint32_t wave_res = static_cast<uint32_t>(wv * SPAN);
        const uint32_t my_res = wave_res + lane * kOneRun;
        if (live && wv < nwaves) {
            uint32_t xb[kOneRun], xs[kOneRun];              // top bits of the hashes at my residues
            uint32_t signs = 0;                             // bit m: the sign of residue m is -1
            {
                uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0 + my_res));
                uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(i0 + my_res));
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) {
                    xb[m] = top_of(yb);
                    xs[m] = top_of(ys);
                    signs |= (sign_flip_of(ys) >> 31) << m;
                    yb = hash_advance(yb, v.a);
                    ys = hash_advance(ys, v.as);
                }
            }
            struct Step {                                   // a visit that was requested
                vec4f x;
                uint32_t tb, ts, s, w, q;                   // the step, as in steps[k]
                uint32_t k;                                 // ~0u for none
            };
            VisitCursor<WIDE> cursor(steps, k1 - k0, wave_res, d);
            auto request = [&](Step& st) {
                st.k = cursor.next();
                const uint4 e = steps[st.k == ~0u ? 0u : st.k];
                st.tb = e.x;
                st.ts = e.y;
                st.s = __builtin_amdgcn_readfirstlane(place_of<WIDE>(e));
                st.q = __builtin_amdgcn_readfirstlane(sum_of_visit<WIDE>(e));
                st.w = __builtin_amdgcn_readfirstlane(e.w);
                uint32_t at = st.s + my_res;
                at = at < last4 ? at : last4;
                st.x = *(gvec4_ptr)(g + at);
            };
            // of the residues from wave_res on, how many take part in the visit and exist in the vector (> 0)
            auto room_of = [&](uint32_t s, uint32_t w) -> uint32_t {
                const uint32_t in_gap = (w & kGapMask) - wave_res, in_vec = d - s - wave_res;
                return in_gap < in_vec ? in_gap : in_vec;
            };
            // x: four values read at min(s + my_res, last4)  ->  those of my residues, 0 for the missing ones
            auto cut = [&](vec4f x, uint32_t s, uint32_t room) -> vec4f {
                const int len = static_cast<int>(room) - lane * kOneRun;
                const int over = static_cast<int>(s + my_res) - static_cast<int>(last4);
                const float in[kOneRun] = {x.x, x.y, x.z, x.w};
                float out[kOneRun];
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) {
                    float val = over <= 0 ? in[m] : 0.0f;
#pragma unroll
                    for (int t = m + 1; t < kOneRun; ++t) val = over == t - m ? in[t] : val;
                    out[m] = m < len ? val : 0.0f;
                }
                return vec4f{out[0], out[1], out[2], out[3]};
            };
            // sums of the coordinates whose bucket hash did not wrap and of those whose did, for visits with
            // A mod c = cur; their signs less that of the residue itself
            float plain[kOneRun], wrapped[kOneRun];
            uint32_t cur = 0;
#pragma unroll
            for (int m = 0; m < kOneRun; ++m) plain[m] = wrapped[m] = 0.0f;
            auto park = [&](uint32_t q, const float (&x)[kOneRun]) {
                vec4f u;
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) u[m] = x[m];
                *reinterpret_cast<vec4f*>(&parked[q][lane * kOneRun]) = u;
            };
            auto fetch = [&](uint32_t q, float (&x)[kOneRun]) {
                const vec4f u = *reinterpret_cast<const vec4f*>(&parked[q][lane * kOneRun]);
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) x[m] = u[m];
            };
#pragma unroll
            for (int q = 0; q < NC; ++q)
                *reinterpret_cast<vec4f*>(&parked[q][lane * kOneRun]) = vec4f{0.0f, 0.0f, 0.0f, 0.0f};
            auto move_to = [&](uint32_t q) {                // (neighbouring cells share a sum: power-of-two c)
                const uint32_t step = POW2 ? 1 : omega;
                park(cur, plain);
                park(cur + step, wrapped);
                fetch(q, plain);
                fetch(q + step, wrapped);
                cur = q;
            };
            auto add_up = [&](Step& st) {
                const uint32_t room = room_of(st.s, st.w);
                vec4f x = st.x;
                if (room < SPAN) x = cut(x, st.s, room);
                if (cur != st.q) move_to(st.q);
                uint64_t flips[kOneRun], wraps[kOneRun], unsure = 0;
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) {
                    flips[m] = __builtin_amdgcn_ballot_w64(xs[m] > st.ts);
                    wraps[m] = __builtin_amdgcn_ballot_w64(xb[m] > st.tb);
                    unsure |= __builtin_amdgcn_ballot_w64(xb[m] == st.tb) | __builtin_amdgcn_ballot_w64(xs[m] == st.ts);
                }
                if (__builtin_expect(unsure != 0, 0)) {
                    // the lower bits decide: whole hash values against whole thresholds
                    const uint64_t A = mulmod_p(v.a, st.s), As = mulmod_p(v.as, st.s);
                    uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0 + my_res));
                    uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(i0 + my_res));
#pragma unroll
                    for (int m = 0; m < kOneRun; ++m) {
                        flips[m] = __builtin_amdgcn_ballot_w64(ys > kP61 - As);
                        wraps[m] = __builtin_amdgcn_ballot_w64(yb > kP61 - A);
                        yb = hash_advance(yb, v.a);
                        ys = hash_advance(ys, v.as);
                    }
                }
                const uint64_t odd = (st.w >> 29 & 1u) != 0 ? ~0ull : 0ull;
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) {
                    const float val = __builtin_amdgcn_inverse_ballot_w64(flips[m] ^ odd) ? -x[m] : x[m];
                    const bool wrap = __builtin_amdgcn_inverse_ballot_w64(wraps[m]);
                    plain[m] += wrap ? 0.0f : val;
                    wrapped[m] += wrap ? val : 0.0f;
                }
            };
            Step st[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) request(st[u]);
            // (a buffer is refilled where it was read: moving a value that is still on its way would
            // wait for it)
            // (a break from every turn: where the turns meet again before the end is known, the wait for the oldest
            // values becomes one for all that are on their way)
            static_assert(kAhead == 3 || kAhead == 4, "a turn for each");
            for (;;) {
                if (st[0].k == ~0u) break;
                add_up(st[0]);
                request(st[0]);
                if (st[1].k == ~0u) break;
                add_up(st[1]);
                request(st[1]);
                if (st[2].k == ~0u) break;
                add_up(st[2]);
                request(st[2]);
                if constexpr (kAhead > 3) {
                    if (st[kAhead - 1].k == ~0u) break;
                    add_up(st[kAhead - 1]);
                    request(st[kAhead - 1]);
                }
            }
            park(cur, plain);
            park(cur + (POW2 ? 1 : omega), wrapped);
#pragma unroll
            for (int q = 0; q < NC; ++q) {                  // the signs of the residues
                float x[kOneRun];
                fetch(q, x);
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) x[m] = apply_sign(x[m], (signs >> m) << 31);
                park(q, x);
            }
        }
        if constexpr (!PARTIAL) {
            if (worker == 0) {
                uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0 + my_res));
#pragma unroll
                for (int m = 0; m < kOneRun; ++m) {
                    first[lane * kOneRun + m] = bucket_of<POW2>(yb, col);
                    yb = hash_advance(yb, v.a);
                }
            }
        }
        if constexpr (WL > 1) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
        if (wv < nwaves) {
            const uint32_t tid = worker * 64 + lane;
            if constexpr (PARTIAL) {
                float* dst = a.sums + group * a.sums_floats + v.at + (static_cast<uint64_t>(piece) * nwaves + wv) * SPAN * ncell * WL;
                auto write = [&](auto n) {             // (a division by a constant where all sums are used)
                    for (uint32_t item = tid; item < SPAN * WL * n; item += 64 * WL) {
                        const uint32_t w = item % WL, t = item / WL;
                        dst[item] = static_cast<int>(w) < nw ? scale * sums_lds[set][w][t % n][t / n] : 0.0f;
                    }
                };
                if (ncell == NC) write(std::integral_constant<uint32_t, NC>());
                else write(ncell);
            } else if (fold) {
                for (uint32_t item = tid; item < SPAN * NC; item += 64 * WL) {
                    const uint32_t res = item / NC, q = item % NC;     // (a sum that is not used is 0)
                    float x[WL];
#pragma unroll
                    for (int w = 0; w < WL; ++w) x[w] = w < nw ? sums_lds[set][w][q][res] : 0.0f;
#pragma unroll
                    for (int off = 1; off < WL; off <<= 1)
#pragma unroll
                        for (int w = 0; w + off < WL; w += 2 * off) x[w] += x[w + off];
                    if (x[0] != 0.0f) atomic_add_noret(Tj + cell_of_sum(first[res], q), scale * x[0]);
                }
            } else {
#pragma unroll 1
                for (uint32_t item = tid; item < SPAN * WL * NC; item += 64 * WL) {
                    const uint32_t w = item % WL, t = item / WL, res = t / NC, q = t % NC;
                    const float sum = static_cast<int>(w) < nw ? sums_lds[set][w][q][res] : 0.0f;
                    if (sum != 0.0f)
                        atomic_add_noret(Tj + static_cast<size_t>(cell_of_sum(first[res], q)) * kGroup + w, scale * sum);
                }
            }
        }
        // visits whose cells are not kept (never with a list of cs_params_init): hashed by the definition,
        // straight into memory
        if (!PARTIAL && listed < k1 - k0 && live && wv < nwaves) {
            for (uint32_t k = 0; k < k1 - k0; ++k) {
                const uint32_t s = __builtin_amdgcn_readfirstlane(place_of<WIDE>(steps[k])), w = __builtin_amdgcn_readfirstlane(steps[k].w);
                if (sum_of_visit<WIDE>(steps[k]) < kNoSum<WIDE> || (w & kGapMask) <= my_res || s + my_res >= d) continue;
                const uint32_t in_gap = (w & kGapMask) - my_res, in_vec = d - s - my_res;
                const uint32_t len = in_gap < in_vec ? in_gap : in_vec;
                const uint32_t at = s + my_res;
                uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0 + at));
                uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(i0 + at));
                for (uint32_t m = 0; m < kOneRun && m < len; ++m) {
                    const float val = apply_sign(scale * g[at + m], sign_flip_of(ys));
                    if (val != 0.0f)
                        atomic_add_noret(Tj + static_cast<size_t>(bucket_of<POW2>(yb, col)) * cell_floats + (fold ? 0 : worker), val);
                    yb = hash_advance(yb, v.a);
                    ys = hash_advance(ys, v.as);
                }
            }
        }
        if constexpr (WL > 1) __syncthreads();
        else __builtin_amdgcn_wave_barrier();
    }
}

// One launch of k_accumulate_vectors: n rows whose pieces are chosen, with at most ncell running sums.
template <int WL, bool PARTIAL, typename LIST>
int launch_vectors(LIST& rows, WorkersBeside<LIST> a, int n, uint32_t ncell, hipStream_t stream) {
    auto launch = [&](auto sets, auto nc) -> int {
        constexpr int SETS = decltype(sets)::value, NC = decltype(nc)::value;
        const dim3 grid(visits_grid<1, kOneRun, SETS>(rows, n), (a.nw + kGroup - 1) / kGroup);
        const size_t lds = most_steps(rows, n) * sizeof(uint4);
        constexpr auto kernel = k_accumulate_vectors<WL, SETS, NC, PARTIAL, LIST>;
        a.at_once = workgroups_at_once<kernel>(64 * WL * SETS, lds);
        kernel<<<grid, 64 * WL * SETS, lds, stream>>>(rows, a);
        return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
    };
    auto with = [&](auto sets) -> int {
        if (ncell == 2) return launch(sets, std::integral_constant<int, 2>());
        if (ncell == 4) return launch(sets, std::integral_constant<int, 4>());
        if constexpr (std::is_same<LIST, VisitRows>::value) {
            if (ncell == 3) return launch(sets, std::integral_constant<int, 3>());
            if constexpr (WL == 1 && !PARTIAL) {
                if (ncell > 4 && ncell <= 6) return launch(sets, std::integral_constant<int, 6>());
                if (ncell > 6 && ncell <= CS_VECTOR_CELLS) return launch(sets, std::integral_constant<int, CS_VECTOR_CELLS>());
            }
        }
        return CS_EINVAL;
    };
    if (!PARTIAL && !a.T) return CS_EINVAL;
    if constexpr (WL == 1) {
        int64_t waves = 0;
        for (int q = 0; q < n; ++q) waves += (static_cast<int64_t>(rows.row[q].gmax) + 64 * kOneRun - 1) / (64 * kOneRun);
        if (waves < kOneFewWaves) return with(std::integral_constant<int, 1>());
    }
    return with(std::integral_constant<int, WL >= 4 ? 1 : 4 / WL>());
}

// A wavefront per vector is the faster way for 2 to 8 vectors that the memory-side cache (256 MB) holds, or nearly (us, update with
// merge, lanes for workers / wavefronts for vectors): 5 x 2^17, 6.5 M, 8 workers 201 / 178, 9 M 267 / 238; 5 x 2^18, 14 M
// 390 / 435; 7 x 65 536, 15.4 M 544 / 575; 4 workers and less, up to 480 MB: 5 x 2^17, 10 M, 4 workers 167 / 148, 5 x 2^18,
// 30 M 437 / 422; 5 x 2^19, 40 M, 2 workers 371 / 287.  Less so where a residue takes part in few visits, so that what a workgroup
// does once (its table of visits, the sums at its end) is much of it, and in short vectors: 5 x 8192, 300 000, 8 workers 25 / 34;
// 5 x 16 384, 600 000 33 / 38; 7 x 65 536, 5 M (23 visits) 207 / 212; 7 x 2^17, 5 M, 4 workers (14) 192 / 203.  Several groups of 8 in
// a launch: 5 x 8192, 300 000, 64 workers 126 / 140.
// And where few residues make a round or two of workgroups of 5 to 8 vectors, the last of them nearly empty (the update alone):
// 3 x 8192, 1.5 M, 8 workers (41 000 residues) 37 / 47; 3 x 4096, 2 M, 5 workers (26 000) 39 / 45; but 3 x 4096, 1.3 M, 8 workers
// (62 000) 32 / 28; in launches of 5 rows and more 5 x 8192, 2.7 M, 8 workers (107 000) 74 / 83, 3.7 M, 6 workers (122 000) 83 / 100; but
// 2.1 M, 6 workers (197 000) 56 / 52, 5 x 16 384, 5.1 M, 8 workers (220 000) 145 / 130.  With sums to a workspace: 3 x 4096, 1.3 M, 8
// workers 30 / 35, 7 x 8192, 2 M, 4 workers (187 000) 48 / 52; but 3 x 65 536, 5.4 M, 4 workers (241 000) 63 / 59, 3 x 16 384, 2.6 M,
// 3 workers (139 000) 35 / 29.  Of 300 timings of drawn shapes that it leaves, 12 % faster in the mean, 15 are behind by 3 to 10 % (7 x
// 8192, 2.4 M, 8 workers 93 / 101; 5 x 16 384, 3 M, 3 workers 50 / 54; 7 x 16 384, 5.7 M, 2 workers, to a workspace 80 / 85).
// workers_of_sums: those of an update whose sums go to a workspace; `vectors` are a walker's lanes then.
template <typename LIST>
bool vectors_pay(const LIST& rows, int n, int64_t d, int vectors, int groups, int workers_of_sums = 0) {
    double residues = 0.0;
    for (int q = 0; q < n; ++q) residues += static_cast<double>(rows.row[q].gmax);
    const double bytes = 4.0 * static_cast<double>(d) * vectors;
    if (groups != 1 || d < 1'200'000 || bytes > (vectors > 4 ? 3.4e8 : 4.8e8)) return false;
    if (workers_of_sums > 0) {
        if (workers_of_sums > 3 && residues < 200e3) return false;
    } else if (vectors > 4 && residues < (vectors > 5 && n >= 5 ? 150e3 : 50e3)) {
        return false;
    }
    return n * static_cast<double>(d) >= 25.0 * residues;
}
// The rate at which the cache is read
constexpr double kCachedBytesPerNs = 6400.0;

// In runs of 16 pairs cost a turn through LDS for every coordinate of a walker, with two sums half of it for nothing, and
// 9 to 16 registers, with 3 sums of 8 workers the fourth wavefront of a SIMD.  They pay for it where requests are much of
// the launch: of up to 4 workers, whose requests are 8 or 16 bytes, in rows of 4 MB and more, which one XCD's L2 does not hold, and
// in long vectors.  Us, one by one / in pairs: 7 x 131 072, 4.2 M, 2 workers 143 / 116; 5 x 2^19, 17 M, 4 workers 413 / 358; 5 x
// 131 072, 5.1 M, 8 workers 177 / 155; 5 x 2^19, 11 M, 16 workers 755 / 699; 7 x 65 536, 15.8 M, 8 workers 606 / 574; 7 x 2^19, 25 M,
// 256 workers, whose 10 M requests a launch of 8 workers end each round, a step 33 450 / 32 870.  But 5 x 32 768, 1.65 M, 6 workers
// 118 / 132; 7 x 32 768, 4.7 M, 6 workers 172 / 211; 7 x 65 536, 4.2 M, 5 workers 152 / 171; two sums: 5 x 32 768, 3.5 M, 6
// workers 104 / 120, 3 x 65 536, 21.9 M, 24 workers 1080 / 1154, 5 x 131 072, 32 M, 4 workers 430 / 446, and 5 x 2^18, 8 M, 2
// workers 220 / 197.  What it leaves behind is up to 7 % (3 x 131 072, 16.8 M, 8 workers 261 / 280).
bool pairs_pay(uint32_t ncell, uint32_t c, int workers, int64_t d) {
    if (ncell == 2) return workers <= 4 && d < 64 * static_cast<int64_t>(c);
    return workers <= 4 || c >= 1u << 17 || d >= 12'000'000;
}

template <int WL, int NWAVE>
int launch_visits(const cs_params* p, const VisitWorkers& a, const uint32_t* js, int nrows,
                  uint32_t ncell, hipStream_t stream) {
    if (ncell < 2 || ncell > 4) return CS_EINVAL;
    VisitRows rows{};
    // every sum is a request, but those of the two cells of an aligned block of a bundle are one where they leave in pairs
    double requests8[kRowsPerLaunch], requests16[kRowsPerLaunch];
    const int groups = (a.nw + kGroup - 1) / kGroup;
    const bool pairs16 = a.fold == 0 && pairs_pay(ncell, p->c, a.nw, a.d);
    for (int q = 0; q < nrows; ++q) {
        const cs_visit_plan& vp = p->visit[js[q]];
        fill_visit_args(p, js[q], rows.row[q]);
        const double residues = static_cast<double>(vp.gmax) * groups, paired = 0.5 * vp.ncell + 0.5;
        requests8[q] = (a.fold ? vp.ncell : paired) * residues;
        requests16[q] = (pairs16 ? paired : vp.ncell) * residues;
    }
    const double stream_ns = 4.0 * static_cast<double>(a.d) * a.nw * nrows / kStreamBytesPerNs;
    if constexpr (WL > 1) {
        if (vectors_pay(rows, nrows, a.d, a.nw, groups)) {
            choose_pieces(rows, nrows, requests8, kVisitNsOne, stream_ns * kStreamBytesPerNs / kCachedBytesPerNs);
            return launch_vectors<WL, false>(rows, a, nrows, ncell, stream);
        }
    }
    const bool run8 = choose_run8<WL>(rows, nrows, requests8, requests16, a.d, stream_ns, groups);
    if (run8) return launch_visits_run<WL, 8, 1>(rows, a, nrows, ncell, stream);
    if (pairs16) return launch_visits_run<WL, 16, NWAVE, true>(rows, a, nrows, ncell, stream);
    return launch_visits_run<WL, 16, NWAVE>(rows, a, nrows, ncell, stream);
}

// the visit list of row j serves vectors of length d
bool list_serves(const cs_params* p, uint32_t j, int64_t d) {
    const cs_visit_plan& vp = p->visit[j];
    if ((p->flags & CS_FLAG_NO_VISIT_LIST) != 0 || vp.K == 0) return false;
    if (vp.ncell < 2 || vp.ncell > 4 || vp.K > CS_MAX_VISITS || d > kStepsMaxD) return false;   // (lists end at 2^28)
    return static_cast<uint64_t>(d) <= vp.cover;
}

// ... and (unless any_cost) is expected to take less time than the stride walk.  Up to a quarter above the walk that is
// the launch of the walk more: us, 8 workers unless said, such a row by the walk / its list, priced 1.02 to 1.13 times the walk,
// 7 x 2^19, 25 M 1075 / 1025, 2 workers 506 / 469; 7 x 65 536, 22 M 849 / 801; 5 x 2^20, 18 M 853 / 776, 25 M 1044 / 974; 15 x
// 65 536, 25 M 2083 / 1995, 2 workers 734 / 601.  Where other rows walk in any case, such a row lengthens their launch
// only by a longer chain of visits (a shorter stride) than theirs: 15 x 2^20, 48 M, 5 workers 6220 / 5011 (a stride of
// 30 751 beside 118 023); but behind a longer chain 15 x 2^20, 18 M, 5 workers 3467 / 3606, 61 M 5692 / 5778; 15 x 2^18,
// 100 M, 3 workers 4722 / 4891.
bool visits_apply(const cs_params* p, uint32_t j, int64_t d, bool any_cost = false) {
    const cs_visit_plan& vp = p->visit[j];
    auto dear = [](const cs_visit_plan& v) { return v.cost > v.cost_walk + v.cost_walk / 4; };
    if (!list_serves(p, j, d)) return false;
    if (any_cost || vp.cost < vp.cost_walk) return true;
    if (dear(vp)) return false;
    for (uint32_t q = 0; q < p->r; ++q)
        if ((!list_serves(p, q, d) || dear(p->visit[q])) && p->plan[q].Dw <= p->plan[j].Dw) return false;
    return true;
}

// Groups of 8 workers that share a launch, `most` at most.  A launch of one group of short vectors is a chain of visits
// that leaves most of the chip idle, 15 to 30 us however little it reads; together they read at the rate of long vectors.
// With runs of 8, chains cut as if half a chain came on top of the reads, us (requests and merge, one group at a time / together):
// 5 x 1024, d = 79 230, 240 workers 356 / 104; 7 x 128, 20 344, 122 workers 174 / 55; 5 x 2048, 446 435, 66 workers 222 / 105
// (318 where the chains were not cut, 174 in runs of 16); 15 x 2048, 767 209, 236 workers 2388 / 1806; 5 x 8192, 1.2 M, 92
// workers 522 / 308; 3 x 65 536, 3.3 M, 205 workers 1844 / 1345; other column counts: 15 x 793, 95 678, 122 workers
// 1163 / 239; 5 x 2109, 332 923, 144 workers 417 / 216.  Up to 1.6 GB of reads a group (other column counts 1.2): from there
// the tables of several groups push each other out of the memory-side cache (5 x 131 072, 23 M, 26 workers, two together
// 2167 / 2296; 3 x 262 144, 18 M, 1112 / 1148; 7 x 131 072, 9.4 M 742 / 784; 3 x 58 719, 17 M, six together 2182 / 2372; but 3 x
// 65 536, 16.9 M 1250 / 989).
int groups_at_once(const cs_params* p, int64_t d, int most = kGroupsPerLaunch) {
    const double n = 1e10 / (32.0 * static_cast<double>(d) * p->r);
    return n < (p->c_pow2 ? 6.0 : 8.0) ? 1 : n > most ? most : static_cast<int>(n);
}
// The workers of the next launch, of `left`.  Up to 4 workers that are left over share the launch of the others, with idle
// lanes, while that reads less than 0.3 GB a group (7 x 2048, 725 668, 11 workers 74 / 66; but 5 x 131 072, 3.2 M, 9 workers
// 198 / 208, 3 x 32 768, 11 M, 9 workers 253 / 288).
int workers_of_launch(const cs_params* p, int64_t d, int left, int at_once) {
    if (at_once == 1 || left <= kGroup) return left < kGroup ? left : kGroup;
    if (left > at_once * kGroup) return at_once * kGroup;
    const int tail = left % kGroup;
    return tail <= kGroup / 2 && 32.0 * static_cast<double>(d) * p->r > 3e8 ? left - tail : left;
}

void fill_visit_gaps(const cs_params* p, uint32_t j, VisitGaps& v) {
    const cs_anyc_plan& vp = p->anyc[j];
    v.K = vp.K;
    v.j = static_cast<int32_t>(j);
    v.gmax = vp.gmax;
    v.a = p->a[j]; v.b = p->b[j]; v.as = p->as[j]; v.bs = p->bs[j];
    v.omega = vp.omega;
    v.pc = static_cast<uint32_t>(kP61 % p->c);
    for (uint32_t k = 0; k < vp.K; ++k) v.gap[k] = vp.gap[k];
}

// The rows of an any-c sketch in the launches that take them: rows with the same number of
// running sums (omega = 1 or 2) together, up to `at_once` per launch, the longest lists
// first; where `mixed` (all but the update of one vector) and one launch takes all rows, all of them together,
// with the sums of omega = 2: one tail instead of two, and the row or two of the other kind do not fill the chip by
// themselves (us, two launches / one: 5 x 180 000, 6.5 M, 2 workers 198 / 177, 8 workers 249 / 227; 5 x 333 333, 30 M, 8
// workers 1030 / 993; 3 x 180 001, 17 M, 2 workers 392 / 328, 8 workers 444 / 443; 3 x 200 001, 9 M, 8 workers 197 / 166; query with counts 5 x
// 180 000, 6.5 M 84 / 75, 5 x 250 001, 12 M 143 / 139, 5 x 400 003, 9 M 145 / 134, 5 x 70 001, 2.3 M 67 / 68).
// fn(rows, n, omega) is called per launch.
template <typename FN>
int for_each_anyc_launch(const cs_params* p, uint32_t nrows_of_sketch, FN fn, int at_once = kAnycRowsPerLaunch,
                         bool mixed = false) {
    mixed = mixed && nrows_of_sketch <= static_cast<uint32_t>(at_once);
    for (uint32_t omega = 1; omega <= 2; ++omega) {
        uint32_t order[CS_MAX_R], most = 0;
        int n = 0;
        for (uint32_t j = 0; j < nrows_of_sketch; ++j) {
            if (!mixed && p->anyc[j].omega != omega) continue;
            most = p->anyc[j].omega > most ? p->anyc[j].omega : most;
            int at = n++;
            for (; at > 0 && p->anyc[order[at - 1]].K < p->anyc[j].K; --at) order[at] = order[at - 1];
            order[at] = j;
        }
        for (int q0 = 0; q0 < n; q0 += at_once) {
            const int m = n - q0 < at_once ? n - q0 : at_once;
            const int rc = fn(order + q0, m, most);
            if (rc != CS_OK) return rc;
        }
        if (mixed) break;
    }
    return CS_OK;
}

// one launch: rows js[0 .. n) (of at most that omega) of one group of workers, each along
// its list for any column count
template <int WL, int NWAVE>
int launch_visits_anyc(const cs_params* p, const VisitWorkersOf<1>& a, const uint32_t* js, int n,
                       uint32_t omega, hipStream_t stream) {
    VisitGapsRows rows{};
    double requests[kAnycRowsPerLaunch];
    for (int q = 0; q < n; ++q) {
        fill_visit_gaps(p, js[q], rows.row[q]);
        requests[q] = 2.0 * rows.row[q].omega * static_cast<double>(rows.row[q].gmax);
    }
    const double stream_ns = 4.0 * static_cast<double>(a.d) * a.nw * n / kStreamBytesPerNs;
    if constexpr (WL > 1) {
        // (with 6 to 8 workers and few coordinates per column the requests are too much of it: 5 x 180 000, 6.5 M, 8 workers 245 /
        // 245, 3 x 88 897, 4.3 M 86 / 89, 3 x 126 461, 3 M 129 / 131; but 5 x 65 723, 2.5 M, 5 workers 127 / 115, 3 x 32 571,
        // 8.5 M, 8 workers 153 / 144)
        const bool wide = a.nw > 5 && a.d < 64 * static_cast<int64_t>(a.c);
        if (p->r <= kAnycRowsPerLaunch && !wide && vectors_pay(rows, n, a.d, a.nw, 1)) {
            choose_pieces(rows, n, requests, kVisitNsOne, stream_ns * kStreamBytesPerNs / kCachedBytesPerNs);
            return launch_vectors<WL, false>(rows, a, n, 2 * omega, stream);
        }
    }
    if (choose_run8<WL>(rows, n, requests, requests, a.d, stream_ns))
        return launch_visits_run<WL, 8, 1>(rows, a, n, 2 * omega, stream);
    return launch_visits_run<WL, 16, NWAVE>(rows, a, n, 2 * omega, stream);
}

}  // namespace

// Every row has a list for this column count and vector length.
static bool anyc_all_listed(const cs_params* p, int64_t d) {
    if (p->c_pow2 || d > kStepsMaxD || (p->flags & CS_FLAG_NO_VISIT_LIST) != 0) return false;
    for (uint32_t j = 0; j < p->r; ++j) {
        const cs_anyc_plan& vp = p->anyc[j];
        if (vp.K == 0 || vp.K > CS_ANYC_MAX_VISITS || (vp.omega != 1 && vp.omega != 2)) return false;
        if (static_cast<uint64_t>(d) > vp.cover) return false;
    }
    return true;
}
// ... and by its own estimate the list beats one request per coordinate.
bool anyc_visits_apply(const cs_params* p, int64_t d) {
    if (!anyc_all_listed(p, d)) return false;
    for (uint32_t j = 0; j < p->r; ++j)
        if (p->anyc[j].cost >= p->anyc[j].cost_direct) return false;
    return true;
}

// The update of W workers follows the lists where the rows together are estimated to gain (one bad list of 5 x 46 897, d =
// 1.8 M, 97 workers, is 9 % above its requests and the other four take a quarter of theirs).  Groups that share launches
// wait for each other's chains of visits only once, so that their requests (24 G/s) and reads (5 TB/s) count and a chain.
bool anyc_update_applies(const cs_params* p, int64_t d, int W) {
    if (!anyc_all_listed(p, d)) return false;
    double lists = 0.0, direct = 0.0, requests = 0.0;
    for (uint32_t j = 0; j < p->r; ++j) {
        lists += static_cast<double>(p->anyc[j].cost);
        direct += static_cast<double>(p->anyc[j].cost_direct);
        requests += 2.0 * p->anyc[j].omega * static_cast<double>(p->anyc[j].gmax);
    }
    if (lists < direct) return true;
    const int groups = (W + kGroup - 1) / kGroup;
    if (groups == 1 || groups_at_once(p, d, kAnycGroups) == 1) return false;
    const double coordinates = static_cast<double>(p->r) * static_cast<double>(d);
    return 15000.0 + groups * (requests / 24.0 + 32.0 * coordinates / kStreamBytesPerNs) < groups * coordinates / 21.0;
}

// The query follows the lists where its r launches are worth it. Below d = 1.5 million they are not (us of
// the query of one vector, r gathers per coordinate against the lists: 0.7M x 15 rows 60 / 99, 2M x 5 rows
// 62 / 52, 2M x 15 rows 145 / 116, 4M x 5 rows 101 / 58, 6.5M x 5 rows 149 / 85, 2.2M x 3 rows 50 / 31; the
// shortest with narrow tables about even: 2.1M x 3 rows of 9001 columns, lists of up to 135 visits, 43 / 46).
bool anyc_visits_serve_query(const cs_params* p, int64_t d) {
    return anyc_visits_apply(p, d) && d >= 3 * (static_cast<int64_t>(1) << 19) &&
           d * static_cast<int64_t>(p->r - 1) >= (static_cast<int64_t>(1) << 22);
}
// Up to here r gathers per coordinate do as well where the caller has no scratch.
bool anyc_query_needs_scratch(const cs_params* p, int64_t d) {
    return anyc_visits_serve_query(p, d) && d * static_cast<int64_t>(p->r - 1) >= (static_cast<int64_t>(1) << 26);
}

// Per group of 8 workers one launch for up to kAnycRowsPerLaunch rows: every row has its own
// visiting order, so the group's vectors are read once per row (where the direct form reads them
// once in all but sends d requests per row to the atomic unit, which is what bounds it); rows
// that share a launch overlap their serial chains of visits and have one tail.
int launch_accumulate_anyc(const cs_params* p, float* T, int W, const float* const* g_w,
                           int64_t d, int64_t i0, float scale, bool fold, hipStream_t stream, int* launches) {
    const size_t row_floats = static_cast<size_t>(p->c) * kGroup;
    const int at_once = groups_at_once(p, d, kAnycGroups);
    for (int w0 = 0, nw; w0 < W; w0 += nw) {
        nw = workers_of_launch(p, d, W - w0, at_once);
        const bool one = nw == 1 && one_applies(p, d);
        if (launches) {
            if (one) launch_accumulate_one(p, nullptr, kGroup, nullptr, d, i0, scale, stream, launches);
            else for_each_anyc_launch(p, p->r, [&](const uint32_t*, int, uint32_t) { ++*launches; return CS_OK; },
                                      nw > kGroup ? kAnycRowsOfGroups : kAnycRowsPerLaunch, true);
            continue;
        }
        float* Tg = fold ? T : T + static_cast<size_t>(w0 / kGroup) * p->r * row_floats;
        if (nw > kGroup) {
            VisitWorkersOf<kAnycGroups> vw{};
            for (int w = 0; w < nw; ++w) vw.g[w] = g_w[w0 + w];
            vw.T = Tg;
            vw.d = d;
            vw.i0 = i0;
            vw.c = p->c;
            vw.nw = nw;
            vw.scale = scale;
            vw.fold = fold ? 1 : 0;
            vw.table_floats = fold ? 0 : p->r * row_floats;
            const int groups = (nw + kGroup - 1) / kGroup;
            const int rc = for_each_anyc_launch(p, p->r, [&](const uint32_t* js, int n, uint32_t omega) {
                VisitGapsRowsGroups rows{};
                double requests[kAnycRowsOfGroups];
                for (int q = 0; q < n; ++q) {
                    fill_visit_gaps(p, js[q], rows.row[q]);
                    requests[q] = 2.0 * rows.row[q].omega * static_cast<double>(rows.row[q].gmax) * groups;
                }
                choose_pieces(rows, n, requests, kVisitNs8, 4.0 * static_cast<double>(d) * nw * n / kStreamBytesPerNs, groups);
                return launch_visits_run<8, 8, 1>(rows, vw, n, 2 * omega, stream);
            }, kAnycRowsOfGroups, true);
            if (rc != CS_OK) return rc;
            continue;
        }
        if (one) {
            const int rc = launch_accumulate_one(p, Tg, fold ? 1 : kGroup, g_w[w0], d, i0, scale, stream);
            if (rc != CS_OK) return rc;
            continue;
        }
        VisitWorkersOf<1> vw{};
        for (int w = 0; w < nw; ++w) vw.g[w] = g_w[w0 + w];
        vw.T = Tg;
        vw.d = d;
        vw.i0 = i0;
        vw.c = p->c;
        vw.nw = nw;
        vw.scale = scale;
        vw.fold = fold ? 1 : 0;
        const int rc = for_each_anyc_launch(p, p->r, [&](const uint32_t* js, int n, uint32_t omega) {
            if (nw > 4) return launch_visits_anyc<8, kWavesPerGroupOf8>(p, vw, js, n, omega, stream);
            if (nw > 2) return launch_visits_anyc<4, 1>(p, vw, js, n, omega, stream);
            if (nw > 1) return launch_visits_anyc<2, 1>(p, vw, js, n, omega, stream);
            return launch_visits_anyc<1, 1>(p, vw, js, n, omega, stream);
        }, kAnycRowsPerLaunch, true);
        if (rc != CS_OK) return rc;
    }
    return CS_OK;
}

bool walk_applies(const cs_params* p, int64_t d) {
    if (!p->c_pow2 || p->c < 64 || d < 4096) return false;
    for (uint32_t j = 0; j < p->r; ++j)
        if (p->plan[j].Dw <= 1) return false;
    return true;
}

// every row of the sketch has a visit list for vectors of length d (what the folded form of
// the update needs: only the list kernel adds the workers up before it writes; a list that the
// time model likes less than the stride walk is used all the same)
bool all_rows_listed(const cs_params* p, int64_t d) {
    if (!walk_applies(p, d)) return false;
    for (uint32_t j = 0; j < p->r; ++j)
        if (!visits_apply(p, j, d, true)) return false;
    return true;
}

// the list that one vector takes in row j
static const cs_visit_plan& vector_list(const cs_params* p, uint32_t j, int64_t d) {
    const cs_visit_plan& own = p->vector[j].list;
    const bool serves = own.K != 0 && own.K <= CS_MAX_VISITS && own.ncell >= 2 && own.ncell <= CS_VECTOR_CELLS &&
                        static_cast<uint64_t>(d) <= own.cover;
    return serves ? own : p->visit[j];
}

// The lists serve the update of one vector: every row has one that covers d, and all of them
// together send fewer requests than the lattice form (about one per 8 to 15 coordinates).  Lists of its own count where one launch
// takes all rows, and with more than 5 rows for less (us, lattice / lists: 3 x 2^20, 5.2 M 99 / 68, 10.5 M 139 / 72; 5 x 2^20,
// 4.2 M 142 / 129, 8.4 M 218 / 134; 7 x 2^20, 8.4 M 294 / 240, but 6.3 M 228 / 237; 15 x 65 536, 1 M 71 / 106; 15 x 2^18, 5.2 M
// 315 / 410).
bool one_applies(const cs_params* p, int64_t d) {
    double residues = 0.0, own = 0.0;
    if (p->c_pow2) {
        if (!all_rows_listed(p, d)) return false;
        for (uint32_t j = 0; j < p->r; ++j) {
            const cs_visit_plan& vp = vector_list(p, j, d);
            residues += static_cast<double>(p->visit[j].gmax);
            own += static_cast<double>(vp.gmax) * (vp.ncell > 4 ? (vp.ncell + 15) / 19.2 : 1.0);
        }
    } else {
        if (!anyc_visits_apply(p, d)) return false;
        for (uint32_t j = 0; j < p->r; ++j) residues += static_cast<double>(p->anyc[j].gmax);
        own = residues;
    }
    const double most = static_cast<double>(p->r) * static_cast<double>(d) / 8.0;
    return 1.2 * residues <= most || (p->r <= kRowsPerLaunch && 1.2 * own <= (p->r > 5 ? 0.85 : 1.0) * most);
}

// S = float[r][c][cell_floats]: the table itself (1) or one worker's slot of a bundle (kGroup)
int launch_accumulate_one(const cs_params* p, float* S, int cell_floats, const float* g, int64_t d,
                          int64_t i0, float scale, hipStream_t stream, int* launches) {
    auto cut = [&](auto& rows, int n, double more) {   // the chains of n rows into pieces
        double requests[kRowsPerLaunch];
        for (int q = 0; q < n; ++q) requests[q] = (1.2 + more) * static_cast<double>(rows.row[q].gmax);
        const double stream_ns = 4.0 * static_cast<double>(d) * n / kStreamBytesPerNs;
        choose_pieces(rows, n, requests, kVisitNsOne, stream_ns);
    };
    auto fill = [&](auto& a) {
        a.g[0] = g;
        a.T = S;
        a.d = d;
        a.i0 = i0;
        a.c = p->c;
        a.nw = 1;
        a.scale = scale;
        a.fold = cell_floats == 1 ? 1 : 0;
    };
    if (!p->c_pow2)
        return for_each_anyc_launch(p, p->r, [&](const uint32_t* js, int n, uint32_t omega) {
            if (launches) {
                ++*launches;
                return static_cast<int>(CS_OK);
            }
            VisitGapsRows rows{};
            for (int q = 0; q < n; ++q) fill_visit_gaps(p, js[q], rows.row[q]);
            cut(rows, n, 0.0);
            VisitWorkersOf<1> a{};
            fill(a);
            return launch_vectors<1, false>(rows, a, n, 2 * omega, stream);
        });
    uint32_t order[CS_MAX_R], ncell = 2;
    for (uint32_t j = 0; j < p->r; ++j) {              // the longest lists first
        const cs_visit_plan& vp = vector_list(p, j, d);
        if (vp.ncell > ncell) ncell = vp.ncell;
        int at = static_cast<int>(j);
        for (; at > 0 && vector_list(p, order[at - 1], d).K < vp.K; --at) order[at] = order[at - 1];
        order[at] = j;
    }
    for (uint32_t q0 = 0; q0 < p->r; q0 += kRowsPerLaunch) {
        const int n = p->r - q0 < kRowsPerLaunch ? static_cast<int>(p->r - q0) : kRowsPerLaunch;
        VisitRows rows{};
        for (int q = 0; q < n; ++q) fill_visit_args(p, order[q0 + q], vector_list(p, order[q0 + q], d), rows.row[q]);
        cut(rows, n, ncell > 4 ? (ncell - 4) / 16.0 : 0.0);
        VisitWorkers a{};
        fill(a);
        const int rc = launch_vectors<1, false>(rows, a, n, ncell, stream);
        if (rc != CS_OK) return rc;
    }
    return CS_OK;
}

// ---------------------------------------------------------------------------------------
// The update into a workspace of running sums instead of a table (cs_index.hip gathers them): what
// the rows of one group of workers write and where.
// ---------------------------------------------------------------------------------------
namespace {

// Every visit of the rows' lists moves a coordinate by fewer cells than it has running sums, which is what the
// kernels rely on when the sums are all they write.  (Lists of cs_params_init do.)
bool lists_hold(const cs_params* p) {
    auto mulmod = [](uint64_t a, uint64_t b) {
        const unsigned __int128 t = static_cast<unsigned __int128>(a) * b;
        return reduce_p((static_cast<uint64_t>(t) & kP61) + static_cast<uint64_t>(t >> 61));
    };
    for (uint32_t j = 0; j < p->r; ++j) {
        const cs_visit_plan& vp = p->visit[j];
        uint64_t advance[4], s = 0, A = 0;
        for (int t = 0; t < 4; ++t) {
            if (vp.gap[t] >= static_cast<uint64_t>(kStepsMaxD)) return false;
            advance[t] = mulmod(p->a[j], vp.gap[t]);
        }
        for (uint32_t k = 0; k < vp.K; ++k) {
            if ((A & (p->c - 1)) + 1 >= vp.ncell) return false;
            const uint32_t code = (vp.code[k / 16] >> (2 * (k % 16))) & 3u;
            if ((s += vp.gap[code]) > static_cast<uint64_t>(kStepsMaxD)) return false;
            A += advance[code];
            A = A >= kP61 ? A - kP61 : A;
        }
    }
    return true;
}

// The rows of one launch: pieces and run length are chosen, their places in the workspace taken, and, with
// `run`, the launch is made.
template <int WL>
int partial_rows(VisitRows& rows, VisitWorkers& a, int n, int workers, int groups, SumsPlan& plan, hipStream_t stream) {
    double writes[kRowsPerLaunch];
    uint32_t most = 2;
    for (int q = 0; q < n; ++q) {
        const VisitArgs& v = rows.row[q];
        most = v.ncell > most ? v.ncell : most;
        // a running sum costs as many requests of 1/24 ns as four times its bytes written and read would take to stream
        // (one to eight times: within 3 % of each other, but for d = 60 789, W = 11, 5 x 1024: 32.8, 29.8, 28.4, 27.9 us)
        writes[q] = 24.0 * 32.0 * WL * v.ncell * static_cast<double>(v.gmax) / kStreamBytesPerNs * groups;
    }
    const double stream_ns = 4.0 * static_cast<double>(a.d) * WL * n / kStreamBytesPerNs * groups;
    int log_run = 0;                                   // (a wavefront per vector: the sums lie in the order of the residues)
    const bool vectors = WL == 1 || vectors_pay(rows, n, a.d, WL, groups, workers);
    if (WL == 1) choose_pieces(rows, n, writes, kVisitNsOne, stream_ns);
    else if (vectors) choose_pieces(rows, n, writes, kVisitNsOne, stream_ns * kStreamBytesPerNs / kCachedBytesPerNs);
    else log_run = choose_run8<WL>(rows, n, writes, writes, a.d, stream_ns, groups) ? 3 : 4;
    const uint64_t span = vectors ? 64 * kOneRun : 64u / WL << log_run;
    for (int q = 0; q < n; ++q) {
        VisitArgs& v = rows.row[q];
        SumsRow& out = plan.row[v.j];
        v.at = out.at = plan.floats;
        out.residues = v.gmax;
        out.piece_floats = (v.gmax + span - 1) / span * span * WL * v.ncell;
        out.pieces = v.pieces;
        out.ncell = v.ncell;
        out.log_run = log_run;
        plan.floats += out.piece_floats * v.pieces;
    }
    if (a.nw == 0) return CS_OK;
    if (vectors) return launch_vectors<WL, true>(rows, a, n, most, stream);
    if constexpr (WL > 1) {
        if (log_run == 3) return launch_visits_run<WL, 8, 1>(rows, a, n, most, stream);
        return launch_visits_run<WL, 16, WL == 8 ? kWavesPerGroupOf8 : 1>(rows, a, n, most, stream);
    }
    return CS_EINVAL;
}

template <int WL>
int partial_group(const cs_params* p, VisitWorkers& a, int workers, int groups, SumsPlan& plan, hipStream_t stream) {
    uint32_t order[CS_MAX_R];
    for (uint32_t j = 0; j < p->r; ++j) {              // the longest lists first
        int at = static_cast<int>(j);
        for (; at > 0 && p->visit[order[at - 1]].K < p->visit[j].K; --at) order[at] = order[at - 1];
        order[at] = j;
    }
    for (uint32_t q0 = 0; q0 < p->r; q0 += kRowsPerLaunch) {
        const int n = p->r - q0 < kRowsPerLaunch ? static_cast<int>(p->r - q0) : kRowsPerLaunch;
        VisitRows rows{};
        for (int q = 0; q < n; ++q) fill_visit_args(p, order[q0 + q], rows.row[q]);
        const int rc = partial_rows<WL>(rows, a, n, workers, groups, plan, stream);
        if (rc != CS_OK) return rc;
    }
    return CS_OK;
}

}  // namespace

// Power-of-two columns only: the two sums of a residue of another sketch belong to cells far apart, so that reading
// them by cell fetches a block for each (5 x 180 000, d = 6.5 M, 8 workers: update 181 us and gathering 78, for
// 255 with requests to the table).
bool sums_apply(const cs_params* p, int64_t d) {
    if (!p->c_pow2 || !walk_applies(p, d)) return false;
    for (uint32_t j = 0; j < p->r; ++j)
        if (!visits_apply(p, j, d)) return false;
    return lists_hold(p);
}

int sums_lanes(int W) { return W > 4 ? 8 : W > 2 ? 4 : W; }

// Groups of a launch of W workers
int sums_groups(const cs_params* p, int W, int64_t d) {
    const int all = (W + kGroup - 1) / kGroup, most = groups_at_once(p, d);
    return all < most ? all : most;
}

// g_w null: the plan only
int launch_accumulate_sums(const cs_params* p, float* sums, uint64_t sums_floats, int workers, int groups, int nw,
                           const float* const* g_w, int64_t d, float scale, SumsPlan& plan, hipStream_t stream) {
    plan = SumsPlan{};
    VisitWorkers a{};
    for (int w = 0; g_w && w < nw; ++w) a.g[w] = g_w[w];
    a.sums = sums;
    a.sums_floats = sums_floats;
    a.d = d;
    a.c = p->c;
    a.nw = g_w ? nw : 0;
    a.scale = scale;
    switch (sums_lanes(workers)) {
        case 1: return partial_group<1>(p, a, workers, groups, plan, stream);
        case 2: return partial_group<2>(p, a, workers, groups, plan, stream);
        case 4: return partial_group<4>(p, a, workers, groups, plan, stream);
        default: return partial_group<8>(p, a, workers, groups, plan, stream);
    }
}

// fold: T is one table float[r][c] that receives the sum over all W workers (all_rows_listed
// must hold); otherwise T is the bundle and every worker has its own slot.
int launch_accumulate_walk(const cs_params* p, float* T, int W, const float* const* g_w,
                           int64_t d, int64_t i0, float scale, bool fold, hipStream_t stream, int* launches) {
    if (fold && !all_rows_listed(p, d)) return CS_EINVAL;
    const size_t row_floats = static_cast<size_t>(p->c) * kGroup;
    uint32_t along_lists = 0;
    for (uint32_t j = 0; j < p->r; ++j) along_lists += visits_apply(p, j, d, fold) ? 1 : 0;
    const bool listed_all = along_lists == p->r;
    const bool one = W % kGroup == 1 && listed_all && one_applies(p, d);   // a group of one worker: a single vector
    const int at_once = listed_all ? groups_at_once(p, d) : 1;
    for (int w0 = 0, nw; w0 < W; w0 += nw) {
        nw = workers_of_launch(p, d, W - w0, at_once);
        if (launches) {                                // (one vector: as many launches of as many rows)
            *launches += static_cast<int>(along_lists + kRowsPerLaunch - 1) / kRowsPerLaunch + (listed_all ? 0 : 1);
            continue;
        }
        float* Tg = fold ? T : T + static_cast<size_t>(w0 / kGroup) * p->r * row_floats;
        if (nw == 1 && one) {
            const int rc = launch_accumulate_one(p, Tg, fold ? 1 : kGroup, g_w[w0], d, i0, scale, stream);
            if (rc != CS_OK) return rc;
            continue;
        }
        VisitWorkers vw{};
        for (int w = 0; w < nw; ++w) vw.g[w] = g_w[w0 + w];
        vw.T = Tg;
        vw.d = d;
        vw.i0 = i0;
        vw.c = p->c;
        vw.nw = nw;
        vw.scale = scale;
        vw.fold = fold ? 1 : 0;
        vw.table_floats = fold ? 0 : p->r * row_floats;
        // All rows with a visit list go into one launch (per 8 rows), compiled for the largest
        // number of running sums among them: a row that needs fewer simply never touches the
        // extra ones.  One launch overlaps the rows' serial chains of visits and has one tail.
        // Rows with the longest lists go first: workgroups are started in order, so the launch
        // then ends on the wavefronts that live shortest and the chip drains quickly (measured
        // against the rows in index order: 1.5 % at d = 100 M with 5 rows, 4 % at d = 25 M
        // with 7; the opposite order costs as much again).
        uint32_t ncell = 2;
        uint32_t listed[CS_MAX_R];
        int nlisted = 0;
        for (uint32_t j = 0; j < p->r; ++j) {
            if (!visits_apply(p, j, d, fold)) continue;
            if (p->visit[j].ncell > ncell) ncell = p->visit[j].ncell;
            int at = nlisted++;
            for (; at > 0 && p->visit[listed[at - 1]].K < p->visit[j].K; --at) listed[at] = listed[at - 1];
            listed[at] = j;
        }
        for (int q0 = 0; q0 < nlisted; q0 += kRowsPerLaunch) {
            const int nrows = nlisted - q0 < kRowsPerLaunch ? nlisted - q0 : kRowsPerLaunch;
            const uint32_t* js = listed + q0;
            int rc;
            if (nw > 4) rc = launch_visits<8, kWavesPerGroupOf8>(p, vw, js, nrows, ncell, stream);
            else if (nw > 2) rc = launch_visits<4, 1>(p, vw, js, nrows, ncell, stream);
            else if (nw > 1) rc = launch_visits<2, 1>(p, vw, js, nrows, ncell, stream);
            else rc = launch_visits<1, 1>(p, vw, js, nrows, ncell, stream);
            if (rc != CS_OK) return rc;
        }
        // the other rows: stride walk, all in one launch, the longest chains of visits
        // (smallest strides) first
        WalkArgs a{};
        a.nw = nw;                               // (one group: not all rows are listed)
        for (int w = 0; w < nw && w < kGroup; ++w) a.g[w] = g_w[w0 + w];
        a.T = Tg;
        a.d = d;
        a.i0 = i0;
        a.scale = scale;
        int nwalked = 0;
        for (uint32_t j = 0; j < p->r; ++j) {
            if (visits_apply(p, j, d, fold)) continue;
            int at = nwalked++;
            for (; at > 0 && p->plan[a.js[at - 1]].Dw > p->plan[j].Dw; --at) a.js[at] = a.js[at - 1];
            a.js[at] = static_cast<int32_t>(j);
        }
        if (nwalked > 0) {
            int rc;
            if (nw > 4) rc = launch_walk<8, 16, kWalkWaves>(p, a, nwalked, stream);
            else if (nw > 2) rc = launch_walk<4, 16, 1>(p, a, nwalked, stream);
            else if (nw > 1) rc = launch_walk<2, 16, 1>(p, a, nwalked, stream);
            else rc = launch_walk<1, 16, 1>(p, a, nwalked, stream);
            if (rc != CS_OK) return rc;
        }
    }
    return CS_OK;
}

// ---------------------------------------------------------------------------------------
// Alg. 4 estimate, walk order: rows[j][i] = s_j(i) S[j][h_j(i)] for every coordinate.
//
// The same stride serves the query.  A visit moves every hash on by the same A = (a n Dw) mod p, so a coordinate that
// began in cell b is in cell b + A mod c, or one further where its hash wrapped past p, which a comparison with p - A tells
// (as in the update along lists, with whole hash values here: there is nothing left to be unsure of); the sign is
// that of the first visit, turned by the parity of A' and by a wrap.  A mod c is the same for the whole
// wavefront and moves by one cell in ~1/sigma visits, so a lane keeps the four neighbouring cells ahead of
// each coordinate, which are one 16-byte load, and loads again after three such steps (~30 visits).  The
// 64 lanes of a wavefront own 64 neighbouring chunks of 4 residues, so every visit writes 1 KB of contiguous output, 16
// bytes per lane.  A second kernel takes the median over rows, or the walk of the last row does.
// Against two 61-bit states a coordinate, moved on at each visit, and a gather whenever a coordinate leaves its cell
// (some of a wavefront's 256 does at nearly every visit), with the accesses of load_values below, the whole query with counts, us: 4 M
// x 5 rows of 65 536 columns 56 -> 47; 6.5 M, 5 x 2^17 77 -> 59; 6.5 M, 15 x 65 536 204 -> 157; 11 M, 5 x 2^18 117 -> 91; 25 M,
// 5 x 2^19 232 -> 205; 25 M, 7 x 2^19 342 -> 276; 50 M, 3 x 2^18 276 -> 226; 10^8, 5 x 2^20 939 -> 733.  Bound: the scratch, and the
// first gathers of long rows, whose residues (2 to 4 million a row) each fetch a line of a table that L2 does not
// hold (10^8: 350 us for rows 0 .. 3, 290 without those loads).
// ---------------------------------------------------------------------------------------
namespace {

// Coordinates per lane and visit.  Four: a lane's values are one 16-byte piece of output, so no
// transpose is needed.
constexpr int kQRun = 4;

// A short vector leaves a row with few chunks (Dw / 256 wavefronts) and a long serial chain
// of visits each; the chain is then cut into n segments that separate wavefronts walk, at the price of one more gather
// per lane and segment.  Row j has the workgroups first[j] .. first[j] + n[j] across[j] - 1 of a launch of rows 0 ..
// (the strides of one sketch differ by a factor of 300, so that a grid of (most chunks, rows, most segments) is nearly all
// empty workgroups, which start at 4 to 5 a nanosecond: 68 800 of 5 x 2^15 at d = 2^20, where 10 000 have work).
struct RowSegments {
    int n[CS_MAX_R];
    uint32_t across[CS_MAX_R];   // a multiple of 8: blockIdx.x & 7 stays the XCD
    uint32_t first[CS_MAX_R];    // ~0: no such row
};

constexpr int kQWave = 64 * kQRun;                     // residues of a wavefront
constexpr int kQLine = 32;                             // floats of a line of memory
// How the scratch is written.  What the memory-side cache (256 MB) holds, the stride walk writes and reads with ordinary
// accesses: pieces of 1 KB that begin anywhere are written at 5.8 TB/s then, and at 3.8 with nontemporal stores, which do not put
// together in L2 a line that two wavefronts write in part each.  A larger scratch goes to memory, where such a line
// costs about four times a whole one (400 MB: pieces anywhere 4.4 TB/s ordinary and 3.7 nontemporal, pieces on lines
// 5.1; 1.6 GB: 4.0, 3.4, 5.4), and ordinary accesses push the sketch out of L2 (query of 5 rows of 100 M on lines, ordinary /
// nontemporal: 995 / 845 us).  With LINES, then, a wavefront also works out the 32 residues behind its own and writes the
// 256 that begin on a line (one short part at each visit's ends), past the caches.  Where that pays for the quarter more
// arithmetic, by r d (us, ordinary pieces anywhere / lines): 11M x 5 rows 92 / 104, 16M x 5 143 / 130, 12M x 7
// 139 / 142, 16M x 7 194 / 172, 6.5M x 15 157 / 171, 9M x 15 225 / 225, 25M x 15 717 / 583.  Lists (other column counts), whose accesses are
// all nontemporal (ordinary: 2M x 5 rows of 41 111 columns 38 / 41, 30M x 5 280 / 300): 17M x 5 184 / 201, 22M x 5 214 / 209,
// 30M x 5 280 / 258, 10M x 15 339 / 360, 20M x 15 627 / 570, 90M x 15 2439 / 2136.
constexpr uint32_t kManyRows = 7;
constexpr int64_t kWalkLinesFrom = 75000000, kWalkLinesFromMany = 120000000;
constexpr int64_t kLinesFrom = 110000000, kLinesFromMany = 200000000;
template <bool NT>
__device__ __forceinline__ vec4f load_values(const float* p) {
    if (NT) return __builtin_nontemporal_load(reinterpret_cast<const vec4f_u*>(p));
    return *reinterpret_cast<const vec4f_u*>(p);
}
template <bool NT>
__device__ __forceinline__ void store_values(float* p, vec4f u) {
    if (NT) __builtin_nontemporal_store(u, reinterpret_cast<vec4f_u*>(p));
    else *reinterpret_cast<vec4f_u*>(p) = u;
}
// RF = 0: rows[j][i] for the rows j = blockIdx.y.  RF = R (the row count): the walk of the last
// row, which instead of storing its values reads those of rows 0 .. R-2 at the same coordinates
// and writes their median, est[i] -- the last row never goes through memory.
// HIST (with RF > 0): the kernel also counts the estimates it writes by the top 11 bits of their
// magnitude (bits 30..20 of the binary32 pattern) into hist[2048], which is the first
// histogram of the selection that follows (Sec. 5.2: query every coordinate, keep the
// largest): one read of est less.  Counts are kept per workgroup in LDS and added to hist at
// the end; a workgroup of kHistWaves wavefronts shares one set of counters (8 KB), so that LDS
// does not limit how many wavefronts a CU holds.
constexpr int kHistWaves = 4;
// The last row's wavefronts alone do not fill the chip, and a visit is one round of loads: where the next visit's are under way
// meanwhile (us of the query, without / with): 3 rows, 9.8 M, vectors of 8 workers read before it 67 / 57; 16 M 85.5 / 84; 32 M 165 / 161;
// 5 rows, 6.5 M, 8 workers 72.6 / 64.8, 11.2 M 106 / 97, 14.7 M 137 / 125, one worker 13.9 M 143 / 135, but 5 x 65 536, 6.7 M 66.5 / 67.9.
// The registers of more rows cost a wavefront a SIMD: 7 rows of 12 M 138 / 142, 17 M 191 / 201; and 5 rows past the caches find memory
// busy as it is: 17 M 137 / 143, 27 M 199 / 206.
constexpr bool query_reads_ahead(int RF, bool LINES) { return RF == 3 || (RF == 5 && !LINES); }
template <int RF, bool HIST, bool LINES>
__global__ void __launch_bounds__(HIST ? 64 * kHistWaves : 64)
k_row_values_walk(KParams p, RowSegments segs, const float* __restrict__ S, int64_t d, int64_t i0,
                  float* __restrict__ rows, float* __restrict__ est,
                  unsigned long long* __restrict__ hist) {
    static_assert(kQRun == 4, "one 16-byte piece per lane");
    static_assert(!HIST || RF > 0, "only the kernel that writes est can count it");
    constexpr int NW = HIST ? kHistWaves : 1;          // wavefronts per workgroup
    constexpr int kOwn = kQRun + (LINES ? 1 : 0);
    constexpr bool kAhead = query_reads_ahead(RF, LINES);
    const int lane = threadIdx.x & 63;
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int j = RF ? RF - 1 : 0;
    if (RF == 0)
#pragma unroll
        for (int q = 1; q < CS_MAX_R; ++q) j += blockIdx.x >= segs.first[q] ? 1 : 0;
    const int nseg = segs.n[j];
    const uint32_t block = blockIdx.x - (RF ? 0u : segs.first[j]), across = RF ? gridDim.x / nseg : segs.across[j];
    const uint32_t seg = block / across, bx = block % across;
    // the counters that a later kernel of the query adds to are cleared here: a launch less
    if (RF == 0 && hist && blockIdx.x == 0)
        for (int t = threadIdx.x; t < 2048; t += 64) hist[t] = 0;
    __shared__ uint32_t lh[HIST ? 2048 : 1];
    __shared__ __align__(16) float turn_all[LINES ? NW : 1][LINES ? kQWave + kQLine : 4];
    float* turn = turn_all[LINES ? wq : 0];
    if (HIST) {
        for (int t = threadIdx.x; t < 2048; t += 64 * NW) lh[t] = 0;
        __syncthreads();
    }
    auto tally = [&](float v) {
        if (HIST) atomicAdd(&lh[(__float_as_uint(v) & 0x7fffffffu) >> 20], 1u);
    };
    const int64_t D = static_cast<int64_t>(p.plan[j].Dw);
    const int64_t visits = (d + D - 1) / D;
    const int64_t nD0 = visits * seg / nseg * D;                 // my segment of the chain
    const int64_t nD1 = visits * (seg + 1) / nseg * D;
    const uint64_t ADb = p.plan[j].ADw, ADs = p.plan[j].ADws;
    const uint64_t Ab = p.a[j], As = p.as[j];
    const int64_t nwaves = (D + kQWave - 1) / kQWave;
    const uint32_t mask = p.c - 1u;
    const bool down = (static_cast<uint32_t>(ADb) & mask) > mask / 2;      // the stride leads to lower cells
    const float* __restrict__ Sj = S + static_cast<size_t>(j) * p.c;
    float* __restrict__ out = rows + static_cast<size_t>(j) * d;
    // floats from the last line boundary to the coordinate 0 that I write
    const uint32_t line0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(RF ? est : out) / sizeof(float)) % kQLine;

    const int64_t per_xcd = (nwaves + 7) / 8;
    const int64_t xcd_first = static_cast<int64_t>(bx & 7) * per_xcd;
    for (int64_t k = static_cast<int64_t>(bx >> 3) * NW + wq; k < per_xcd; k += static_cast<int64_t>(across >> 3) * NW) {
        const int64_t wv = xcd_first + k;
        if (wv >= nwaves) break;
        const int64_t wave_off = wv * kQWave;                    // residue offsets in [0, Dw): of the wavefront
        const int64_t my_off = wave_off + lane * kQRun;          // and mine
        // my residues: four neighbours, and with LINES one of the kQLine that follow the wavefront's
        uint64_t yb[kOwn], ys[kOwn];                             // hash states at the segment's first visit
        yb[0] = hash_state(Ab, p.b[j], static_cast<uint64_t>(i0 + nD0 + my_off));
        ys[0] = hash_state(As, p.bs[j], static_cast<uint64_t>(i0 + nD0 + my_off));
#pragma unroll
        for (int m = 1; m < kQRun; ++m) {
            yb[m] = hash_advance(yb[m - 1], Ab);
            ys[m] = hash_advance(ys[m - 1], As);
        }
        if constexpr (LINES) {
            yb[kQRun] = hash_state(Ab, p.b[j], static_cast<uint64_t>(i0 + nD0 + wave_off + kQWave + lane % kQLine));
            ys[kQRun] = hash_state(As, p.bs[j], static_cast<uint64_t>(i0 + nD0 + wave_off + kQWave + lane % kQLine));
        }
        // Values of four neighbouring cells of every coordinate, times the sign at the first visit, in the order in which
        // the stride leads through them; the coordinate is in the first or the second.
        float win[kOwn][4];
        uint32_t q = 0, left = 0;                                // cells moved on by; cells behind the second one
        auto load_cells = [&]() {
            const uint32_t lowest = down ? q - 2u : q;
            uint32_t f[kOwn];
            bool edge = false;
#pragma unroll
            for (int m = 0; m < kOwn; ++m) {
                f[m] = (static_cast<uint32_t>(yb[m]) - 1u + lowest) & mask;
                edge |= f[m] > mask - 3u;
            }
            const bool some_edge = __builtin_amdgcn_ballot_w64(edge) != 0;
#pragma unroll
            for (int m = 0; m < kOwn; ++m) {
                vec4f u;
                if (!some_edge) {
                    u = *reinterpret_cast<const vec4f_u*>(Sj + f[m]);
                } else {                                         // a row's last cells are followed by its first
                    u.x = Sj[f[m]];
                    u.y = Sj[(f[m] + 1u) & mask];
                    u.z = Sj[(f[m] + 2u) & mask];
                    u.w = Sj[(f[m] + 3u) & mask];
                }
                const uint32_t flip = sign_flip_of(ys[m]);
                win[m][0] = apply_sign(down ? u.w : u.x, flip);
                win[m][1] = apply_sign(down ? u.z : u.y, flip);
                win[m][2] = apply_sign(down ? u.y : u.z, flip);
                win[m][3] = apply_sign(down ? u.x : u.w, flip);
            }
            left = 2;
        };
        load_cells();
        uint64_t A = 0, As_n = 0;                                // how far the visit moves every hash on
        auto there = [&](int64_t nD) { return nD < nD1 && nD + wave_off < d; };
        // with LINES the wavefront writes from its first whole line on, and on into the line of its last residue
        auto skipped = [&](int64_t nD) -> uint32_t {
            return LINES ? (0u - (line0 + static_cast<uint32_t>(nD + wave_off))) % kQLine : 0u;
        };
        // The other rows' values of two visits (a buffer for each of two turns: moving a value that is on its way would
        // wait for it).  kAhead: where a lane's four do not exist, four that do, which it does not use.
        constexpr int kTurns = kAhead ? 2 : 1;
        [[maybe_unused]] vec4f others[kTurns][RF > 1 ? RF - 1 : 1];
        [[maybe_unused]] auto request = [&](vec4f (&other)[RF > 1 ? RF - 1 : 1], int64_t nD) {
            const int64_t at = nD + my_off + skipped(nD), last = d - kQRun;
            const float* from = rows + (at < last ? at : last);
#pragma unroll
            for (int z = 0; z < RF - 1; ++z) other[z] = load_values<LINES>(from + static_cast<size_t>(z) * d);
        };
        if constexpr (kAhead) {
            if (there(nD0)) request(others[0], nD0);
        }
        for (int64_t nD = nD0; there(nD);) {
#pragma unroll
            for (int buf = 0; buf < kTurns; ++buf, nD += D) {
                if (buf > 0 && !there(nD)) break;
                // residues from wave_off on that exist
                const int64_t in_gap = D - wave_off, in_vec = d - nD - wave_off;
                const int64_t room = in_gap < in_vec ? in_gap : in_vec;
                const int len = static_cast<int>(room < kQWave + kQLine ? room : kQWave + kQLine);
                const uint32_t t = skipped(nD);
                const int my_len = len - static_cast<int>(t) - lane * kQRun;      // of the 4 that I write: >= 4 all, <= 0 none
                const int64_t at = nD + my_off + t;
                [[maybe_unused]] vec4f (&other)[RF > 1 ? RF - 1 : 1] = others[buf];     // the other rows' values, requested early
                if constexpr (kAhead) {
                    // (behind the last visit of mine the present one's again, which are in L2: nothing is read for no one)
                    request(others[buf ^ 1], there(nD + D) ? nD + D : nD);
                } else if constexpr (RF > 1) {
                    if (my_len >= kQRun) {
#pragma unroll
                        for (int z = 0; z < RF - 1; ++z)
                            other[z] = load_values<LINES>(rows + static_cast<size_t>(z) * d + at);
                    }
                }
                if ((static_cast<uint32_t>(A) & mask) != q) {
                    const uint32_t q_new = static_cast<uint32_t>(A) & mask;
                    const uint32_t by = (down ? q - q_new : q_new - q) & mask;
                    q = q_new;
                    if (by == 1 && left > 0) {
#pragma unroll
                        for (int m = 0; m < kOwn; ++m) {
                            win[m][0] = win[m][1];
                            win[m][1] = win[m][2];
                            win[m][2] = win[m][3];
                        }
                        --left;
                    } else {
                        load_cells();
                    }
                }
                const uint64_t wraps = kP61 - A, flips = kP61 - As_n;    // a state above them passes p
                const bool odd = (As_n & 1u) != 0;
                float o[kOwn];
#pragma unroll
                for (int m = 0; m < kOwn; ++m) {
                    const float x = (yb[m] > wraps) != down ? win[m][1] : win[m][0];
                    o[m] = (ys[m] > flips) != odd ? -x : x;
                }
                A += ADb;
                A = A >= kP61 ? A - kP61 : A;
                As_n += ADs;
                As_n = As_n >= kP61 ? As_n - kP61 : As_n;
                vec4f mine;
                mine.x = o[0]; mine.y = o[1]; mine.z = o[2]; mine.w = o[3];
                [[maybe_unused]] float head = 0.0f;
                if constexpr (LINES) {
                    *reinterpret_cast<vec4f*>(turn + lane * kQRun) = mine;
                    if (lane < kQLine) turn[kQWave + lane] = o[kQRun];
                    __builtin_amdgcn_wave_barrier();
                    mine = *reinterpret_cast<const vec4f_u*>(turn + t + lane * kQRun);
                    head = turn[lane % kQLine];
                    __builtin_amdgcn_wave_barrier();
                }
                // the visit's first residues, before its first whole line
                const bool heads = LINES && wave_off == 0 && lane < static_cast<int>(t) && lane < len;
                if constexpr (RF > 0) {
                    float* dst = est + at;
                    if (my_len >= kQRun) {
                        float vx[RF], vy[RF], vz[RF], vw[RF];
#pragma unroll
                        for (int z = 0; z < RF - 1; ++z) {
                            vx[z] = other[z].x; vy[z] = other[z].y; vz[z] = other[z].z; vw[z] = other[z].w;
                        }
                        vx[RF - 1] = mine.x; vy[RF - 1] = mine.y; vz[RF - 1] = mine.z; vw[RF - 1] = mine.w;
                        vec4f u;
                        float med[4];
                        medians_odd<RF>(vx, vy, vz, vw, med);
                        u.x = med[0]; u.y = med[1]; u.z = med[2]; u.w = med[3];
                        store_values<LINES>(dst, u);
                        tally(u.x); tally(u.y); tally(u.z); tally(u.w);
                    } else {
                        for (int m = 0; m < kQRun; ++m) {
                            if (m >= my_len) break;
                            float v[RF];
#pragma unroll
                            for (int z = 0; z < RF - 1; ++z) v[z] = rows[static_cast<size_t>(z) * d + at + m];
                            v[RF - 1] = mine[m];
                            const float med = median_odd<RF>(v);
                            dst[m] = med;
                            tally(med);
                        }
                    }
                    if (heads) {
                        float v[RF];
#pragma unroll
                        for (int z = 0; z < RF - 1; ++z) v[z] = rows[static_cast<size_t>(z) * d + nD + lane];
                        v[RF - 1] = head;
                        const float med = median_odd<RF>(v);
                        est[nD + lane] = med;
                        tally(med);
                    }
                    continue;
                }
                // the wavefront's 64 pieces are 1 KB of contiguous rows[j][i]
                float* dst = out + at;
                if (my_len >= kQRun) {
                    store_values<LINES>(dst, mine);
                } else if (my_len > 0) {
                    dst[0] = mine.x;
                    if (my_len > 1) dst[1] = mine.y;
                    if (my_len > 2) dst[2] = mine.z;
                }
                if (heads) out[nD + lane] = head;
            }
        }
    }
    if (HIST) {
        __syncthreads();
        for (int t = threadIdx.x; t < 2048; t += 64 * NW) {
            const uint32_t n = lh[t];
            if (n) atomicAdd(&hist[t], static_cast<unsigned long long>(n));
        }
    }
}


// ---------------------------------------------------------------------------------------
// Alg. 4 estimate along a visit list, for column counts that are not a power of two.
//
// The list that serves the update serves the query: whatever a lane meets at i + s_k lies in
// one of the NC = 2 omega cells that the cell of i fixes, so the lane fetches those NC cell
// values once, with the sign of i, keeps them in registers, and for the rest of the vector picks one of them per
// visit by the two comparisons of the update -- no gather and no hash inside the loop.  (Without a list the query is r
// random gathers per coordinate from a table that L2 does not hold: ~80 G gathers/s.  For power-of-two column
// counts the stride walk above does the same job and balances its load better.)
// A lane owns 4 neighbouring residues below the largest gap, a wavefront 256, and every visit
// writes 1 KB of contiguous rows[j][i] (RF = 0) or, for the last row (RF = R), reads the other
// rows' values there, takes the median and writes est, with HIST counted by magnitude as in the stride walk.  A
// coordinate outside the NC cells cannot occur with a list from cs_params_init; such visits (and those that the
// comparisons cannot tell) are hashed by the definition, value by value, and gathered from the table.
// What bounds it is the scratch: r - 1 rows written and read, est written.  With two 61-bit hash states per
// residue moved on at each visit, and the counts of magnitudes in a pass of their own, the query took 2960 us for
// 15 rows of 90 M (10.4 GB of traffic: 1.7 ms at 6.2 TB/s) and 744 us for 5 rows of 73 M; now 2236 and 569.
// ---------------------------------------------------------------------------------------
constexpr int kQueryWaves = 4;                         // wavefronts per workgroup: one table of visits, one set of counters
template <int RF, int NC, bool HIST, bool LINES>
__global__ void __launch_bounds__(64 * kQueryWaves)
k_row_values_visits(VisitGapsRows vr, const float* __restrict__ S, uint32_t c, int64_t d, int64_t i0,
                    float* __restrict__ rows, float* __restrict__ est, unsigned long long* __restrict__ hist, int nseg) {
    static_assert(kQRun == 4, "one 16-byte piece per lane");
    static_assert(NC == 2 || NC == 4, "omega = 1 or 2");
    static_assert(!HIST || RF > 0, "only the kernel that writes est can count it");
    constexpr int kOwn = kQRun + (LINES ? 1 : 0);
    const int lane = threadIdx.x & 63;
    const int wq = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const VisitGaps& v = vr.row[blockIdx.y];           // the rows of a launch run side by side
    const int j = v.j;
    // the counters that a later kernel of the query adds to are cleared here: a launch less
    if (RF == 0 && hist && blockIdx.x == 0 && blockIdx.y == 0 && blockIdx.z == 0)
        for (int t = threadIdx.x; t < 2048; t += 64 * kQueryWaves) hist[t] = 0;
    __shared__ uint32_t lh[HIST ? 2048 : 1];
    if (HIST)
        for (int t = threadIdx.x; t < 2048; t += 64 * kQueryWaves) lh[t] = 0;
    auto tally = [&](float x) {
        if (HIST) atomicAdd(&lh[(__float_as_uint(x) & 0x7fffffffu) >> 20], 1u);
    };
    __shared__ uint4 steps[CS_ANYC_MAX_VISITS];
    __shared__ __align__(16) float turn_all[LINES ? kQueryWaves : 1][LINES ? kQWave + kQLine : 4];
    float* turn = turn_all[LINES ? wq : 0];
    const Columns col = columns_of<false>(c);
    const float* __restrict__ Sj = S + static_cast<size_t>(j) * c;
    float* __restrict__ out = rows + static_cast<size_t>(j) * d;
    // floats from the last line boundary to the coordinate 0 that I write
    const uint32_t line0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(RF ? est : out) / sizeof(float)) % kQLine;
    const uint32_t omega = v.omega, pc = v.pc;
    auto cell_of_sum = [&](uint32_t first, uint32_t q) -> uint32_t {
        // (the half that wrapped past p begins at NC / 2, also in rows that use fewer)
        const uint32_t x = q < NC / 2 ? first + q : first + (q - NC / 2) + (c - pc);
        return x >= c ? x - c : x;
    };
    // A launch with few rows leaves the chip half empty and waits on its longest chain of
    // visits, so the chains are cut into nseg pieces walked by separate workgroups (blockIdx.z).
    const uint32_t k0 = v.K * blockIdx.z / nseg, k1 = v.K * (blockIdx.z + 1) / nseg;
    VisitPlaces places;
    places.init(v);
    fill_visit_steps<false, kQueryWaves>(steps, places, v, k0, k1, col, omega, false);          // (a barrier in it: lh is clear)
    const uint32_t d32 = static_cast<uint32_t>(d);
    const int64_t nwaves = (static_cast<int64_t>(v.gmax) + 64 * kQRun - 1) / (64 * kQRun);
    const int64_t nsets = (nwaves + kQueryWaves - 1) / kQueryWaves;
    const int64_t per_xcd = (nsets + 7) / 8;
    const int64_t xcd_first = static_cast<int64_t>(blockIdx.x & 7) * per_xcd;
    for (int64_t kk = blockIdx.x >> 3; kk < per_xcd; kk += gridDim.x >> 3) {
        const int64_t wv = (xcd_first + kk) * kQueryWaves + wq;
        if (xcd_first + kk >= nsets || wv >= nwaves) break;
        const uint32_t wave_res = static_cast<uint32_t>(wv * 64 * kQRun);    // first residue of the wavefront
        const uint32_t my_res = wave_res + lane * kQRun;
        // my residues: four neighbours, and with LINES one of the kQLine that follow the wavefront's
        uint32_t xb[kOwn], xs[kOwn];                   // top bits of their hashes
        float cellv[kOwn][NC];
        {
            uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0 + my_res));
            uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(i0 + my_res));
#pragma unroll
            for (int m = 0; m < kOwn; ++m) {
                if (LINES && m == kQRun) {
                    yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0 + wave_res + kQWave + lane % kQLine));
                    ys = hash_state(v.as, v.bs, static_cast<uint64_t>(i0 + wave_res + kQWave + lane % kQLine));
                }
                xb[m] = top_of(yb);
                xs[m] = top_of(ys);
                const uint32_t first = bucket_of<false>(yb, col);
#pragma unroll
                for (int n = 0; n < NC; ++n) cellv[m][n] = apply_sign(Sj[cell_of_sum(first, n)], sign_flip_of(ys));
                yb = hash_advance(yb, v.a);
                ys = hash_advance(ys, v.as);
            }
        }
        for (uint32_t k = 0; k < k1 - k0; ++k) {
            const uint4 e = steps[k];
            const uint32_t s = __builtin_amdgcn_readfirstlane(e.z), w = __builtin_amdgcn_readfirstlane(e.w);
            if ((w & kGapMask) <= wave_res || s + wave_res >= d32) continue;
            // residues from wave_res on that take part in this visit and exist in the vector
            const uint32_t in_gap = (w & kGapMask) - wave_res, in_vec = d32 - s - wave_res;
            const int len = static_cast<int>(in_gap < in_vec ? in_gap : in_vec);
            // with LINES the wavefront writes from its first whole line on, and on into the line of its last residue
            const uint32_t t = LINES ? (0u - (line0 + s + wave_res)) % kQLine : 0u;
            const int my_len = len - static_cast<int>(t) - lane * kQRun;      // of the 4 that I write: >= 4 all, <= 0 none
            const size_t at = static_cast<size_t>(s) + wave_res + t + lane * kQRun;
            [[maybe_unused]] vec4f other[RF > 1 ? RF - 1 : 1];
            if constexpr (RF > 1) {
                if (my_len >= kQRun) {
#pragma unroll
                    for (int q = 0; q < RF - 1; ++q)
                        other[q] = load_values<true>(rows + static_cast<size_t>(q) * d + at);
                }
            }
            bool flip[kOwn], wrap[kOwn], unsure = false;
#pragma unroll
            for (int m = 0; m < kOwn; ++m) {
                flip[m] = xs[m] > e.y;
                wrap[m] = xb[m] > e.x;
                unsure |= xb[m] == e.x || xs[m] == e.y;
            }
            const bool odd = (w >> 29 & 1u) != 0, second = NC > 2 && w >> 30 == 1u;
            float o[kOwn];
#pragma unroll
            for (int m = 0; m < kOwn; ++m) {
                float plain = cellv[m][0], wrapped = cellv[m][NC / 2];
                if (NC > 2) {
                    plain = second ? cellv[m][NC / 2 - 1] : plain;
                    wrapped = second ? cellv[m][NC - 1] : wrapped;
                }
                const float x = wrap[m] ? wrapped : plain;
                o[m] = flip[m] != odd ? -x : x;
            }
            if (w >> 30 == 3u || __builtin_amdgcn_ballot_w64(unsure) != 0) {
                uint64_t yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0) + (LINES ? static_cast<size_t>(s) + my_res : at));
                uint64_t ys = hash_state(v.as, v.bs, static_cast<uint64_t>(i0) + (LINES ? static_cast<size_t>(s) + my_res : at));
#pragma unroll
                for (int m = 0; m < kOwn; ++m) {
                    if (LINES && m == kQRun) {
                        yb = hash_state(v.a, v.b, static_cast<uint64_t>(i0) + s + wave_res + kQWave + lane % kQLine);
                        ys = hash_state(v.as, v.bs, static_cast<uint64_t>(i0) + s + wave_res + kQWave + lane % kQLine);
                    }
                    if (LINES || m < my_len) o[m] = apply_sign(Sj[bucket_of<false>(yb, col)], sign_flip_of(ys));
                    yb = hash_advance(yb, v.a);
                    ys = hash_advance(ys, v.as);
                }
            }
            vec4f mine;
            mine.x = o[0]; mine.y = o[1]; mine.z = o[2]; mine.w = o[3];
            [[maybe_unused]] float head = 0.0f;
            if constexpr (LINES) {
                *reinterpret_cast<vec4f*>(turn + lane * kQRun) = mine;
                if (lane < kQLine) turn[kQWave + lane] = o[kQRun];
                __builtin_amdgcn_wave_barrier();
                mine = *reinterpret_cast<const vec4f_u*>(turn + t + lane * kQRun);
                head = turn[lane % kQLine];
                __builtin_amdgcn_wave_barrier();
            }
            // the visit's first residues, before its first whole line
            const bool heads = LINES && wave_res == 0 && lane < static_cast<int>(t) && lane < len;
            if constexpr (RF > 0) {
                if (my_len >= kQRun) {
                    float vx[RF], vy[RF], vz[RF], vw[RF];
#pragma unroll
                    for (int q = 0; q < RF - 1; ++q) {
                        vx[q] = other[q].x; vy[q] = other[q].y; vz[q] = other[q].z; vw[q] = other[q].w;
                    }
                    vx[RF - 1] = mine.x; vy[RF - 1] = mine.y; vz[RF - 1] = mine.z; vw[RF - 1] = mine.w;
                    vec4f u;
                    float med[4];
                    medians_odd<RF>(vx, vy, vz, vw, med);
                    u.x = med[0]; u.y = med[1]; u.z = med[2]; u.w = med[3];
                    store_values<true>(est + at, u);
                    tally(u.x); tally(u.y); tally(u.z); tally(u.w);
                } else {
                    for (int m = 0; m < kQRun; ++m) {
                        if (m >= my_len) break;
                        float f[RF];
#pragma unroll
                        for (int q = 0; q < RF - 1; ++q) f[q] = rows[static_cast<size_t>(q) * d + at + m];
                        f[RF - 1] = mine[m];
                        const float med = median_odd<RF>(f);
                        est[at + m] = med;
                        tally(med);
                    }
                }
                if (heads) {
                    float f[RF];
#pragma unroll
                    for (int q = 0; q < RF - 1; ++q) f[q] = rows[static_cast<size_t>(q) * d + s + lane];
                    f[RF - 1] = head;
                    const float med = median_odd<RF>(f);
                    est[static_cast<size_t>(s) + lane] = med;
                    tally(med);
                }
            } else {
                float* dst = out + at;
                if (my_len >= kQRun) {
                    store_values<true>(dst, mine);
                } else if (my_len > 0) {
                    dst[0] = mine.x;
                    if (my_len > 1) dst[1] = mine.y;
                    if (my_len > 2) dst[2] = mine.z;
                }
                if (heads) out[static_cast<size_t>(s) + lane] = head;
            }
        }
    }
    if (HIST) {
        __syncthreads();
        for (int t = threadIdx.x; t < 2048; t += 64 * kQueryWaves) {
            const uint32_t n = lh[t];
            if (n) atomicAdd(&hist[t], static_cast<unsigned long long>(n));
        }
    }
}

}  // namespace

// The query along the rows' visit lists for any column count: rows 0 .. r-2 into the scratch,
// up to kAnycRowsPerLaunch rows per launch (one row's wavefronts alone fill a third to two
// thirds of the chip, and every launch has the tail of its longest chain of visits), then the
// last row together with the median.
// hist (or null): cleared, and receives the counts of est by magnitude bin.  3 rows or more (anyc_visits_serve_query).
int launch_estimate_anyc(const cs_params* p, const float* S, int64_t d, int64_t i0, float* est,
                         float* rows, uint64_t* hist, hipStream_t stream) {
    unsigned long long* h = reinterpret_cast<unsigned long long*>(hist);
    auto grid_x = [](uint64_t gmax) {
        const int64_t span = 64 * kQRun * kQueryWaves;
        const int64_t nsets = (static_cast<int64_t>(gmax) + span - 1) / span;
        const int64_t cap = 256 * 64 / kQueryWaves;
        const int64_t gx = nsets < cap ? nsets : cap;
        return static_cast<unsigned>((gx + 7) / 8 * 8);
    };
    unsigned long long* clear = h;                     // by the first launch
    // pieces per chain of a launch: enough wavefronts for about two per SIMD slot of the chip,
    // at least 8 visits per piece
    auto pieces = [](uint64_t waves, uint32_t shortest_list) {
        int64_t n = static_cast<int64_t>((16384 + waves - 1) / (waves > 0 ? waves : 1));
        if (n > shortest_list / 8) n = shortest_list / 8;
        if (n > 16) n = 16;
        return static_cast<unsigned>(n < 1 ? 1 : n);
    };
    const bool lines = static_cast<int64_t>(p->r) * d >= (p->r > kManyRows ? kLinesFromMany : kLinesFrom);
    const uint32_t last = p->r - 1;
    VisitGapsRows vr{};
    const int rc = for_each_anyc_launch(p, last, [&](const uint32_t* js, int n, uint32_t omega) {
        uint64_t most = 0, waves = 0;
        uint32_t shortest = CS_ANYC_MAX_VISITS;
        for (int q = 0; q < n; ++q) {
            fill_visit_gaps(p, js[q], vr.row[q]);
            const cs_anyc_plan& vp = p->anyc[js[q]];
            if (vp.gmax > most) most = vp.gmax;
            waves += (vp.gmax + 64 * kQRun - 1) / (64 * kQRun);
            if (vp.K < shortest) shortest = vp.K;
        }
        const unsigned nseg = pieces(waves, shortest);
        const dim3 grid(grid_x(most), static_cast<unsigned>(n), nseg);
        auto launch = [&](auto nc, auto lines) {
            k_row_values_visits<0, decltype(nc)::value, false, decltype(lines)::value><<<grid, 64 * kQueryWaves, 0, stream>>>(
                vr, S, p->c, d, i0, rows, est, clear, static_cast<int>(nseg));
        };
        using std::integral_constant;
        if (omega == 1 && lines) launch(integral_constant<int, 2>(), std::true_type());
        else if (omega == 1) launch(integral_constant<int, 2>(), std::false_type());
        else if (lines) launch(integral_constant<int, 4>(), std::true_type());
        else launch(integral_constant<int, 4>(), std::false_type());
        clear = nullptr;
        return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
    }, kAnycRowsPerLaunch, true);
    if (rc != CS_OK) return rc;
    fill_visit_gaps(p, last, vr.row[0]);
    const uint32_t omega_last = p->anyc[last].omega;
    const unsigned nseg_last = pieces((p->anyc[last].gmax + 64 * kQRun - 1) / (64 * kQRun), p->anyc[last].K);
    const dim3 gx(grid_x(p->anyc[last].gmax), 1, nseg_last);
#define CS_LASTQ(R_, NC_, H_) \
    if (lines) k_row_values_visits<R_, NC_, H_, true><<<gx, 64 * kQueryWaves, 0, stream>>>(vr, S, p->c, d, i0, rows, est, h, static_cast<int>(nseg_last)); \
    else k_row_values_visits<R_, NC_, H_, false><<<gx, 64 * kQueryWaves, 0, stream>>>(vr, S, p->c, d, i0, rows, est, h, static_cast<int>(nseg_last))
#define CS_LASTR(R_)                                                                                 \
    case R_:                                                                                         \
        if (omega_last == 1 && h) { CS_LASTQ(R_, 2, true); }                                         \
        else if (omega_last == 1) { CS_LASTQ(R_, 2, false); }                                        \
        else if (h) { CS_LASTQ(R_, 4, true); }                                                       \
        else { CS_LASTQ(R_, 4, false); }                                                             \
        break;
    switch (p->r) {
        CS_LASTR(3) CS_LASTR(5) CS_LASTR(7) CS_LASTR(9) CS_LASTR(11) CS_LASTR(13) CS_LASTR(15)
        default: return CS_EINVAL;
    }
#undef CS_LASTR
#undef CS_LASTQ
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

// Whether the last row's walk takes the median itself (launch_estimate_walk), or all rows go into the scratch and the
// caller takes it.  The scratch traffic it saves (write and read of one row) has to outweigh a second, narrower
// launch, and the other rows' values at places of one row's order, one piece of each, are read more slowly than in a
// row.  Query with counts, us, apart / fused: 5 rows 1.5 M 33 / 35, 4 M 47 / 48, 6.5 M 61 / 59, 11 M 104 / 91; 3 rows of
// 10 M 61 / 58; but 7 rows of 12 M 139 / 166, 15 of 6.5 M 158 / 196.
static bool walk_in_lines(const cs_params* p, int64_t d) {
    return d * static_cast<int64_t>(p->r) >= (p->r > kManyRows ? kWalkLinesFromMany : kWalkLinesFrom);
}
bool walk_takes_median(const cs_params* p, int64_t d) {
    return walk_in_lines(p, d) || (p->r <= 5 && d >= 5'000'000);
}

// hist: cleared; with fuse_last it also receives the counts of est by magnitude bin.
int launch_estimate_walk(const cs_params* p, const float* S, int64_t d, int64_t i0,
                         float* est, float* rows, bool fuse_last, uint64_t* hist, hipStream_t stream) {
    // Segments of the chains of visits: about 2048 wavefronts per row, of at least 4 visits; where the scratch goes to
    // memory up to 16 384 wavefronts of at least 16 (us, 2048 / 4096 / 8192: 16 M x 5 rows 141 / 130 / 149, 40 M 320 / 291 / 292,
    // 100 M 844 / 770 / 748, 16 384 737).
    const bool lines = walk_in_lines(p, d);
    const int64_t most_waves = lines ? 16384 : 2048, least_visits = lines ? 16 : 4;
    RowSegments segs{};
    uint32_t total = 0, before_last = 0;
    for (uint32_t j = 0; j < CS_MAX_R; ++j) segs.first[j] = ~0u;
    for (uint32_t j = 0; j < p->r; ++j) {
        const int64_t Dw = static_cast<int64_t>(p->plan[j].Dw);
        const int64_t nwaves = ((Dw + kQRun - 1) / kQRun + 63) / 64;
        const int64_t visits = (d + Dw - 1) / Dw;
        int64_t n = most_waves / nwaves;
        if (n > visits / least_visits) n = visits / least_visits;
        if (n < 1) n = 1;
        if (n > 1024) n = 1024;
        segs.n[j] = static_cast<int>(n);
        segs.across[j] = static_cast<uint32_t>(((nwaves < 256 * 64 ? nwaves : 256 * 64) + 7) / 8 * 8);
        segs.first[j] = before_last = total;
        total += segs.across[j] * static_cast<uint32_t>(n);
    }
    unsigned long long* h = reinterpret_cast<unsigned long long*>(hist);
    if (!fuse_last) {
        if (lines) k_row_values_walk<0, false, true><<<total, 64, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h);
        else k_row_values_walk<0, false, false><<<total, 64, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h);
        return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
    }
    // rows 0 .. r-2 into the scratch, then the last row together with the median
    if (p->r > 1) {
        if (lines) k_row_values_walk<0, false, true><<<before_last, 64, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h);
        else k_row_values_walk<0, false, false><<<before_last, 64, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h);
    } else if (h) {
        const int rc = launch_magnitude_hist_zero(hist, stream);
        if (rc != CS_OK) return rc;
    }
    const uint32_t last = p->r - 1, nlast = static_cast<uint32_t>(segs.n[last]), grid = segs.across[last] * nlast;
    const uint32_t hgrid = ((segs.across[last] + kHistWaves - 1) / kHistWaves + 7) / 8 * 8 * nlast;
#define CS_LAST(R_)                                                                                    \
    case R_:                                                                                           \
        if (h && lines) k_row_values_walk<R_, true, true><<<hgrid, 64 * kHistWaves, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h); \
        else if (h) k_row_values_walk<R_, true, false><<<hgrid, 64 * kHistWaves, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h); \
        else if (lines) k_row_values_walk<R_, false, true><<<grid, 64, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h);  \
        else k_row_values_walk<R_, false, false><<<grid, 64, 0, stream>>>(kparams(p), segs, S, d, i0, rows, est, h);  \
        break;
    switch (p->r) {
        CS_LAST(1) CS_LAST(3) CS_LAST(5) CS_LAST(7) CS_LAST(9) CS_LAST(11) CS_LAST(13) CS_LAST(15)
        default: return CS_EINVAL;
    }
#undef CS_LAST
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

// ---------------------------------------------------------------------------------------
// bundle-wide elementwise kernels
// ---------------------------------------------------------------------------------------
namespace {

__global__ void __launch_bounds__(kBlock) k_bundle_zero(float4* __restrict__ T4, int64_t n4,
                                                        float* __restrict__ T, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    for (int64_t t = t0; t < n4; t += stride) T4[t] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (int64_t t = n4 * 4 + t0; t < n; t += stride) T[t] = 0.0f;
}

// one thread per cell: adds the 8 slots of every group (32 contiguous bytes per group, and
// neighbouring lanes read neighbouring cells, so every load instruction is coalesced).
// The sum over workers is accumulated in binary64 and rounded to binary32 once, together with
// alpha and beta.  A binary32 running sum of W values of similar size loses up to log2(W) bits
// on cells that hold a heavy coordinate; with momentum and error feedback kept as sketches
// that loss is fed back every step and grows (measured at W = 256: the state cells drift
// past 1e-5 of their operands within 8 steps).  The kernel waits on its reads either way.
__global__ void __launch_bounds__(kBlock)
k_bundle_merge(float* __restrict__ dst, float beta, const float4* __restrict__ T4, int groups,
               float alpha, int64_t cells) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < cells; t += stride) {
        double s = 0.0;
        for (int g = 0; g < groups; ++g) {
            const float4* src = T4 + (static_cast<size_t>(g) * cells + t) * (kGroup / 4);
#pragma unroll
            for (int q = 0; q < kGroup / 4; ++q) {
                const float4 u = src[q];
                s += (static_cast<double>(u.x) + static_cast<double>(u.y)) +
                     (static_cast<double>(u.z) + static_cast<double>(u.w));
            }
        }
        const double base = (beta == 0.0f) ? 0.0 : static_cast<double>(beta) * static_cast<double>(dst[t]);
        dst[t] = static_cast<float>(base + static_cast<double>(alpha) * s);
    }
}

// The merge together with the momentum and error accumulation of Alg. 3 that follow it:
// S_t = alpha * sum, S_u = rho S_u + S_t, S_v += S_u in one pass (S_t is not read again, and
// one launch of 4.7 us goes).
__global__ void __launch_bounds__(kBlock)
k_bundle_merge_momentum(float* __restrict__ St, float* __restrict__ Su, float* __restrict__ Sv,
                        const float4* __restrict__ T4, int groups, float alpha, float rho, int64_t cells) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < cells; t += stride) {
        double s = 0.0;
        for (int g = 0; g < groups; ++g) {
            const float4* src = T4 + (static_cast<size_t>(g) * cells + t) * (kGroup / 4);
#pragma unroll
            for (int q = 0; q < kGroup / 4; ++q) {
                const float4 u = src[q];
                s += (static_cast<double>(u.x) + static_cast<double>(u.y)) +
                     (static_cast<double>(u.z) + static_cast<double>(u.w));
            }
        }
        const float st = static_cast<float>(static_cast<double>(alpha) * s);
        const float u = rho * Su[t] + st;
        St[t] = st;
        Su[t] = u;
        Sv[t] = Sv[t] + u;
    }
}

// the same merge from a bundle stored in 16 bits per cell: one 16-byte load per group and cell
template <int FMT>
__global__ void __launch_bounds__(kBlock)
k_bundle_merge16(float* __restrict__ dst, float beta, const uint4* __restrict__ T16, int groups,
                 float alpha, int64_t cells) {
    static_assert(kGroup == 8, "8 cells of 16 bits are one 16-byte load");
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < cells; t += stride) {
        double s = 0.0;
        for (int g = 0; g < groups; ++g) {
            const uint4 q = T16[static_cast<size_t>(g) * cells + t];
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int h = 0; h < 4; h += 2)
                s += (static_cast<double>(from_16<FMT>(static_cast<uint16_t>(w[h]))) +
                      static_cast<double>(from_16<FMT>(static_cast<uint16_t>(w[h] >> 16)))) +
                     (static_cast<double>(from_16<FMT>(static_cast<uint16_t>(w[h + 1]))) +
                      static_cast<double>(from_16<FMT>(static_cast<uint16_t>(w[h + 1] >> 16))));
        }
        const double base = (beta == 0.0f) ? 0.0 : static_cast<double>(beta) * static_cast<double>(dst[t]);
        dst[t] = static_cast<float>(base + static_cast<double>(alpha) * s);
    }
}

}  // namespace

int launch_bundle_merge16(float* dst, float beta, const uint16_t* T16, int groups, float alpha,
                          int64_t cells, int fmt, hipStream_t stream) {
    int64_t b = (cells + kBlock - 1) / kBlock;
    if (b > 256 * 16) b = 256 * 16;
    const uint4* src = reinterpret_cast<const uint4*>(T16);
    if (fmt == CS_FMT_BF16)
        k_bundle_merge16<0><<<static_cast<unsigned>(b), kBlock, 0, stream>>>(dst, beta, src, groups, alpha, cells);
    else
        k_bundle_merge16<1><<<static_cast<unsigned>(b), kBlock, 0, stream>>>(dst, beta, src, groups, alpha, cells);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

int launch_bundle_merge_momentum(float* St, float* Su, float* Sv, const float* T, int groups, float alpha,
                                 float rho, int64_t cells, hipStream_t stream) {
    int64_t b = (cells + kBlock - 1) / kBlock;
    if (b > 256 * 32) b = 256 * 32;
    k_bundle_merge_momentum<<<static_cast<unsigned>(b), kBlock, 0, stream>>>(
        St, Su, Sv, reinterpret_cast<const float4*>(T), groups, alpha, rho, cells);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

int launch_bundle_zero(float* T, int64_t n, hipStream_t stream) {
    const bool aligned = reinterpret_cast<uintptr_t>(T) % 16 == 0;
    const int64_t n4 = aligned ? n / 4 : 0;
    int64_t b = (n / 4 + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > 256 * 16) b = 256 * 16;
    k_bundle_zero<<<static_cast<unsigned>(b), kBlock, 0, stream>>>(reinterpret_cast<float4*>(T),
                                                                   n4, T, n);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

int launch_bundle_merge(float* dst, float beta, const float* T, int groups, float alpha,
                        int64_t cells, hipStream_t stream) {
    int64_t b = (cells + kBlock - 1) / kBlock;
    if (b > 256 * 32) b = 256 * 32;
    k_bundle_merge<<<static_cast<unsigned>(b), kBlock, 0, stream>>>(
        dst, beta, reinterpret_cast<const float4*>(T), groups, alpha, cells);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

}  // namespace cs
