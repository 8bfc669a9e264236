// heavy_hitters_topk: the selection half of Sec. 5.2 of the paper, where every coordinate is
// queried and the k estimates of largest magnitude are kept.
//
// Exact radix select on the 31-bit magnitude key  bits(est) & 0x7fffffff  (monotone in |est|
// for IEEE binary32): three histograms (11 + 10 + 10 bits) find the key theta of the
// k-th largest magnitude and how many entries equal to theta are still needed; an ordered
// compaction then emits, in ascending index order, every index with key > theta plus the
// lowest-index entries with key == theta.  Everything is integer work, so the result is a
// deterministic function of est.
//
// Launches.  A launch costs about 4.7 us on this machine however little it does, and a selection
// written as one kernel per pass (clear, histogram, find, compact, ..., count, scan, write) spent
// 50 of its 70 us on them.  There are three now:
//   k_topk_hist0     the first histogram, when the caller does not bring it (the estimate kernel
//                    can fill it as it writes est);
//   k_topk_compact   every workgroup finds the bin of the k-th largest key in that histogram; only
//                    entries in that bin or above can be selected, and with k << d they are a
//                    small multiple of k: they are copied, block by block in index order, into a
//                    candidate list.  The one full read of est;
//   k_topk_finish    the two remaining histograms, the count and the ordered write over the list.
// A selection from at most kSmall entries is one launch of one workgroup that holds every key in
// LDS (k_topk_small).
//
// k_topk_finish does the same with the candidates when there are at most kSmall of them: its first
// workgroups, up to 8, all find the key and each writes a share, the others return.  Longer lists, and inputs that do not fit
// the list (many equal magnitudes, k close to d: decided on the device), are shared out among
// the workgroups: the work is cut into 4 phases of T tasks, T workgroups draw tasks in order
// from a counter, and before it starts a task it waits until every task of the phase before is
// done.  Those were drawn earlier, by workgroups that are running and themselves wait for earlier
// tasks only, so every wait ends whatever part of the grid is resident -- as long as the counters are
// this call's alone.  Overlapping calls on one workspace, or a kept workspace that was never
// cleared, break that; a wait whose phase makes no progress any more is therefore given up, and
// the call then ends with indices and values that show it (k_topk_finish, `abandon`).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "cs_device.h"
#include "cs_internal.h"
#include "csketch.h"

namespace cs {

constexpr int kBins = 2048;           // bins of the first histogram
constexpr int kItems = 4;             // consecutive elements per thread and load
constexpr int kSelBlock = 1024;       // threads of the workgroups that select
constexpr int kSelWaves = kSelBlock / 64;
constexpr int kKeep = 32;             // keys per thread that a single-workgroup selection keeps in LDS (128 KB)
constexpr int64_t kSmall = static_cast<int64_t>(kSelBlock) * kKeep;
constexpr int64_t kQueryChooseHashes = CS_QUERY_CHOOSE_CELLS;
// Workgroups that read est in one pass.  512 of 512 threads keep 32 KB of reads in flight on every
// CU; more of them only add to the atomic adds on one address at their end (12 ns each, one
// after the other: with 3200 workgroups those were 38 of the compaction's 39 us at d = 6.5 M).
constexpr int kScanBlock = 512;
constexpr int kScanWaves = kScanBlock / 64;
constexpr int kMaxSegs = 512;
constexpr int kStage = 8192;          // candidates one block can hold in LDS for its chunk
constexpr int kFinishBlocks = 256;
// Workgroups that share a short list out among them (k_topk_finish), and the items of each at least.
constexpr uint32_t kShares = 8, kShareItems = 2048;
// Polls of a phase's counter, without a task of that phase ending in between, after which a wait is
// given up: 1.4 s (a poll sleeps 512 cycles and reads memory, 0.33 us measured), plus one poll per
// 16 entries of a task, forty times what a task with the chip to itself takes.
constexpr uint32_t kIdlePolls = 1u << 22;

// workspace layout (all 8-byte aligned); the candidate list follows the struct.  `hist[1..2]` and
// everything from `ticket` to `heavy` are zero when a selection starts and are left zero when it ends.
struct TopkWs {
    uint64_t hist[3][kBins];
    uint32_t prefix;                // bin of the k-th largest key in the first histogram
    uint32_t failed;                // != 0: the candidate list could not be built, est is read instead
    uint64_t k_rem;                 // how many entries of that bin are wanted
    uint32_t ticket;                // next task to draw
    uint32_t exits;                 // workgroups that are through
    uint32_t done[4];               // finished tasks per phase
    uint32_t ncand;                 // candidates appended so far
    uint32_t heavy;                 // selected entries that passed the threshold (KeyHeavymix)
    uint64_t gt[kMaxSegs];          // per segment (or task): entries with key > theta
    uint64_t eq[kMaxSegs];          // per segment (or task): entries with key == theta
    uint32_t seg_base[kMaxSegs];    // block b's candidates are cand[seg_base[b] .. + seg_count[b])
    uint32_t seg_count[kMaxSegs];
};
constexpr size_t kCandBytes = sizeof(int64_t) + sizeof(float);   // index and value of a candidate

// candidates worth providing for: a few times k, never a large part of d.  When k itself is a
// few per cent of d (the P k candidates of Alg. 3 with P in the tens) the list is sized more
// tightly: the entries of the k-th largest key's bin and above are k plus that bin's own
// population, at most a few tenths of k for magnitudes that fall off smoothly (a bin is an
// eighth of a binade wide); should they not fit, est itself is read again on the device.
__host__ inline int64_t candidate_capacity_for(int64_t d, int64_t k) {
    const int64_t roomy = 8 * k + 65536;
    if (roomy <= d / 4) return roomy;
    const int64_t tight = 3 * k + 65536;
    return tight <= d / 5 ? tight : 0;
}

// Selection keys (31 bits, larger = selected first; equal keys: lower index first).
// KeyMagnitude: the magnitude bits of the estimate (top-k by |est|).
struct KeyMagnitude {
    __device__ __forceinline__ void init() {}
    __device__ __forceinline__ uint32_t operator()(float v, int64_t) const {
        return __float_as_uint(v) & 0x7fffffffu;
    }
};
// KeyHeavymix (Alg. 1 steps 3-4): a coordinate is heavy when est^2 >= l2sq / k (binary32
// estimate, squared and compared in binary64: the product of two binary32 values is exact
// there).  Heavy coordinates get bit 30 plus the top 30 magnitude bits, so they come before
// every other coordinate and, should more than k be heavy, in order of magnitude; the others
// get the top 30 bits of a counter-based random word -- the (i+1)-th output of SplitMix64
// started at `seed` -- so the k - |H| of them with the largest words are a uniform draw
// without replacement.
struct KeyHeavymix {
    const double* l2sq;       // device: the norm estimate of cs_sketch_l2sq
    double k;
    uint64_t seed;
    double theta;
    __device__ __forceinline__ void init() { theta = *l2sq / k; }
    __device__ __forceinline__ bool heavy(float v) const {
        return static_cast<double>(v) * static_cast<double>(v) >= theta;
    }
    __device__ __forceinline__ uint32_t operator()(float v, int64_t i) const {
        if (heavy(v)) return 0x40000000u | ((__float_as_uint(v) & 0x7fffffffu) >> 1);
        uint64_t z = seed + (static_cast<uint64_t>(i) + 1u) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        return static_cast<uint32_t>(z >> 34);
    }
};

__global__ void __launch_bounds__(kBlock) k_topk_clear(TopkWs* ws) {
    for (int t = threadIdx.x; t < 3 * kBins; t += kBlock) (&ws->hist[0][0])[t] = 0;
    if (threadIdx.x == 0) {
        ws->ticket = 0;
        ws->exits = 0;
        for (int q = 0; q < 4; ++q) ws->done[q] = 0;
        ws->failed = 0;
        ws->ncand = 0;
        ws->heavy = 0;
    }
}

// v plus the value that the DPP control hands this lane (0 where it hands none, or in rows outside the mask)
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t add_from_lane(uint64_t v) {
    const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(v)), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(static_cast<uint32_t>(v >> 32)), CTRL, ROWS, 0xf, false);
    return v + (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32 | static_cast<uint32_t>(lo));
}
// inclusive sums over each row of 16 lanes: row_shr:1, 2, 4, 8
__device__ __forceinline__ uint64_t row_inclusive_sum(uint64_t v) {
    v = add_from_lane<0x111, 0xf>(v);
    v = add_from_lane<0x112, 0xf>(v);
    v = add_from_lane<0x114, 0xf>(v);
    return add_from_lane<0x118, 0xf>(v);
}
__device__ __forceinline__ uint64_t read_lane(uint64_t v, int lane) {
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v)), lane));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v >> 32)), lane));
    return static_cast<uint64_t>(hi) << 32 | lo;
}

// Sum of v over the threads before this one in a workgroup of WAVES wavefronts; *total receives
// the sum over all threads.  `lds` holds one word per wavefront; the workgroup is in step on return, and all of it calls.
// A selection is a chain of four to six of these by one workgroup, whose 16 wavefronts share four SIMDs: what bounds it is
// their instructions.  Shifts within the register file (row_shr, then row_bcast:15 into rows 1 and 3, row_bcast:31 into
// rows 2 and 3) and one scan of the wavefronts' sums by lanes, instead of shuffles through LDS and a loop over the sums in
// every thread, us of a selection: d = 784 8.6 / 6.5, d = 5000 11.9 / 10.0, d = 60 789 (shared out) 25.5 / 19.8, d = 6.5 M, k =
// 5000 32.5 / 30.6, d = 90 M, k = 320 000 136 / 128.
template <int WAVES>
__device__ __forceinline__ uint64_t block_exclusive_sum(uint64_t v, uint64_t* lds, uint64_t* total) {
    static_assert(WAVES <= 16, "the wavefronts' sums are one row of lanes");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    uint64_t inc = row_inclusive_sum(v);
    inc = add_from_lane<0x142, 0xa>(inc);
    inc = add_from_lane<0x143, 0xc>(inc);
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    const uint64_t mine = lane < WAVES ? lds[lane] : 0;
    __syncthreads();
    const uint64_t sums = row_inclusive_sum(mine);
    *total = read_lane(sums, WAVES - 1);
    return read_lane(sums - mine, wave) + inc - v;
}

// The bin of a histogram (PER consecutive bins per thread, cnt[] of mine) that holds the k_rem-th entry counted from the top; *rem =
// how many of that bin's entries are wanted, *all: it has no more than those.  All threads of the workgroup get the answer
// through `found`, and wait twice: `sums` (a word per wavefront) and `found` are for nothing else before and after.
template <int WAVES, int PER, typename COUNT>
__device__ __forceinline__ void find_bin_once(const COUNT (&cnt)[PER], uint64_t k_rem, uint64_t* sums, uint64_t* found,
                                              uint32_t* bin, uint64_t* rem, bool* all) {
    static_assert(WAVES <= 16, "the wavefronts' sums are one row of lanes");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    uint64_t mine = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) mine += cnt[q];
    uint64_t inc = row_inclusive_sum(mine);
    inc = add_from_lane<0x142, 0xa>(inc);
    inc = add_from_lane<0x143, 0xc>(inc);
    if (lane == 63) sums[wave] = inc;
    __syncthreads();
    const uint64_t of_wave = lane < WAVES ? sums[lane] : 0;
    const uint64_t upto = row_inclusive_sum(of_wave);
    uint64_t acc = read_lane(upto, WAVES - 1) - (read_lane(upto - of_wave, wave) + inc);   // entries in bins above mine
    if (acc < k_rem && k_rem <= acc + mine) {      // true for exactly one thread
#pragma unroll
        for (int q = PER - 1; q >= 0; --q) {
            if (acc < k_rem && k_rem <= acc + cnt[q]) {
                found[0] = static_cast<uint64_t>(threadIdx.x) * PER + q;
                found[1] = (k_rem - acc) << 1 | (k_rem - acc == cnt[q] ? 1u : 0u);
            }
            acc += cnt[q];
        }
    }
    __syncthreads();
    *bin = static_cast<uint32_t>(found[0]);
    *rem = found[1] >> 1;
    *all = (found[1] & 1u) != 0;
}

// ... in buffers that the next step may use.
template <int WAVES, int PER, typename COUNT>
__device__ __forceinline__ void find_bin(const COUNT (&cnt)[PER], uint64_t k_rem, uint64_t* sums, uint64_t* found, uint32_t* bin,
                                         uint64_t* rem) {
    bool all;
    find_bin_once<WAVES>(cnt, k_rem, sums, found, bin, rem, &all);
    __syncthreads();
}

template <bool VEC>
__device__ __forceinline__ void load_items(const float* __restrict__ est, int64_t base, int64_t d,
                                           float (&v)[kItems], int& nvalid) {
    // base = index of this thread's first element
    if (VEC && base + kItems <= d) {
        const float4 q = *reinterpret_cast<const float4*>(est + base);
        v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
        nvalid = kItems;
        return;
    }
    nvalid = 0;
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        if (base + q < d) { v[q] = est[base + q]; nvalid = q + 1; } else { v[q] = 0.0f; }
    }
}

// First histogram: hist_out[key >> 20] += 1 over est (2048 bins).  Magnitudes crowd into a few bins
// (same exponent), and lanes that hit the same LDS word are served one after the other: a
// workgroup keeps kCopies histograms and lane l adds into copy l mod kCopies.
template <bool VEC, typename KEY>
__global__ void __launch_bounds__(kScanBlock)
k_topk_hist0(const float* __restrict__ est, int64_t d, uint64_t* __restrict__ hist_out, KEY kf) {
    kf.init();
    constexpr int kCopies = 4;
    __shared__ uint32_t lh_all[kCopies][kBins];
    for (int t = threadIdx.x; t < kCopies * kBins; t += kScanBlock) (&lh_all[0][0])[t] = 0;
    __syncthreads();
    uint32_t* lh = lh_all[threadIdx.x % kCopies];
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kScanBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x; t * kItems < d; t += 2 * stride) {
        float v[2][kItems];
        int n[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) load_items<VEC>(est, (t + u * stride) * kItems, d, v[u], n[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int q = 0; q < kItems; ++q)
                if (q < n[u]) atomicAdd(&lh[kf(v[u][q], (t + u * stride) * kItems + q) >> 20], 1u);
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kBins; t += kScanBlock) {
        uint32_t v = 0;
#pragma unroll
        for (int q = 0; q < kCopies; ++q) v += lh_all[q][t];
        if (v) atomicAdd(reinterpret_cast<unsigned long long*>(&hist_out[t]),
                         static_cast<unsigned long long>(v));
    }
}

// The candidate list.  Block b scans its chunk of est and keeps, in index order, every entry whose
// key lies in the bin of the k-th largest key or above.  Each wavefront takes a consecutive part of
// the chunk, 1024 entries at a time (four loads in flight), and stages its candidates in its own
// part of LDS (their places come from wavefront ballots, no barrier inside the loop); the block
// then appends them to the list as one segment, whose place comes from a single atomic add.
// Segments lie in the list in the order the blocks finished; (seg_base[b], seg_count[b]) lets
// k_topk_finish put them in block order, i.e. in index order.  A wavefront whose part holds more
// candidates than it can stage counts them all and reads its part once more to write them (k of
// 4 % of d and more: at d = 90 M, k = 3.6 M this kernel takes 105 us for 75 and k_topk_finish, which had to read
// est three times when such a list was given up, 180 for 570).
// A list that would exceed `cap` raises ws->failed.
template <bool VEC, typename KEY>
__global__ void __launch_bounds__(kScanBlock)
k_topk_compact(const float* __restrict__ est, int64_t d, int64_t chunk, TopkWs* ws,
               const uint64_t* __restrict__ hist0, uint64_t k, uint32_t cap,
               int64_t* __restrict__ cand_idx, float* __restrict__ cand_val, KEY kf) {
    kf.init();
    constexpr int kWaveStage = kStage / kScanWaves;
    constexpr int kWaveTile = 64 * kItems;
    constexpr int kTiles = 4;
    __shared__ uint32_t st_off[kStage];
    __shared__ float st_val[kStage];
    __shared__ uint64_t scan[kScanWaves], found[2];
    __shared__ uint32_t wave_n[kScanWaves];
    __shared__ uint32_t seg[2];                     // base, ok
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t lo = static_cast<int64_t>(blockIdx.x) * chunk;
    const int64_t hi = (lo + chunk < d) ? lo + chunk : d;
    const int64_t part = (chunk / kScanWaves + kWaveTile - 1) / kWaveTile * kWaveTile;
    const int64_t wlo = lo + wave * part;
    const int64_t whi = (wlo + part < hi) ? wlo + part : hi;
    float v[kTiles][kItems];                        // the first tiles of my part are on their way while the bin is found
    int n[kTiles];
    auto load_tiles = [&](int64_t tile) {
#pragma unroll
        for (int u = 0; u < kTiles; ++u)
            load_items<VEC>(est, tile + static_cast<int64_t>(lane) * kItems + u * kWaveTile, whi, v[u], n[u]);
    };
    load_tiles(wlo);
    uint32_t bin0;
    {
        constexpr int per = kBins / kScanBlock;
        uint64_t cnt[per], rem;
#pragma unroll
        for (int q = 0; q < per; ++q) cnt[q] = hist0[threadIdx.x * per + q];
        find_bin<kScanWaves>(cnt, k, scan, found, &bin0, &rem);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            ws->prefix = bin0;
            ws->k_rem = rem;
        }
    }
    uint32_t* my_off = st_off + wave * kWaveStage;
    float* my_val = st_val + wave * kWaveStage;
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));   // lanes before mine
    // candidates of my part so far, the same in every lane of the wavefront.  The first kWaveStage are
    // staged; with `direct` (second reading) all go to the list from `at` on.
    uint32_t got = 0;
    auto take = [&](const float (&v)[kItems], int nvalid, int64_t base, bool direct, uint32_t at) {
        bool f[kItems];
        bool any = false;
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            f[q] = q < nvalid && (kf(v[q], base + q) >> 20) >= bin0;
            any |= f[q];
        }
        if (__builtin_amdgcn_ballot_w64(any) == 0) return;
        uint32_t before = 0, total = 0;
#pragma unroll
        for (int q = 0; q < kItems; ++q) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(f[q]);
            before += __builtin_popcountll(m & below);
            total += __builtin_popcountll(m);
        }
        uint32_t pos = got + before;
        got += total;
        if (!direct && got > static_cast<uint32_t>(kWaveStage)) return;
#pragma unroll
        for (int q = 0; q < kItems; ++q)
            if (f[q]) {
                if (direct) {
                    cand_idx[at + pos] = base + q;
                    cand_val[at + pos] = v[q];
                } else {
                    my_off[pos] = static_cast<uint32_t>(base + q - lo);
                    my_val[pos] = v[q];
                }
                ++pos;
            }
    };
    auto read_part = [&](bool direct, uint32_t at) {
        for (int64_t tile = wlo; tile < whi; tile += kTiles * kWaveTile) {
            if (direct || tile != wlo) load_tiles(tile);
            const int64_t b0 = tile + static_cast<int64_t>(lane) * kItems;
#pragma unroll
            for (int u = 0; u < kTiles; ++u) take(v[u], n[u], b0 + u * kWaveTile, direct, at);
        }
    };
    read_part(false, 0u);
    if (lane == 0) wave_n[wave] = got;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t total = 0;
        for (int w = 0; w < kScanWaves; ++w) total += wave_n[w];
        uint32_t base = 0;
        bool ok = true;
        if (total) {
            base = atomicAdd(&ws->ncand, total);
            ok = static_cast<uint64_t>(base) + total <= cap;
        }
        if (!ok) atomicOr(&ws->failed, 1u);
        ws->seg_base[blockIdx.x] = base;
        ws->seg_count[blockIdx.x] = ok ? total : 0u;
        seg[0] = base;
        seg[1] = ok ? 1u : 0u;
    }
    __syncthreads();
    if (seg[1] == 0u) return;
    uint32_t at = seg[0];
    for (int w = 0; w < wave; ++w) at += wave_n[w];
    if (got > static_cast<uint32_t>(kWaveStage)) {
        got = 0;
        read_part(true, at);
        return;
    }
    for (uint32_t t = lane; t < got; t += 64) {
        cand_idx[at + t] = lo + my_off[t];
        cand_val[at + t] = my_val[t];
    }
}

// where a selection goes
struct SelOut {
    int64_t* idx;                   // k indices, ascending
    float* val;                     // their values, or null
    const int64_t* remap;           // null, or: idx[slot] = remap[i] instead of i
    unsigned long long* n_heavy;    // null, or: how many of the selected keys have bit 30 set
    int64_t k;
    __device__ __forceinline__ void put(uint64_t slot, int64_t i, float v) const {
        if (slot >= static_cast<uint64_t>(k)) return;
        idx[slot] = remap ? remap[i] : i;
        if (val) val[slot] = v;
    }
};

// LDS of a selection by one workgroup (of the 160 KB that a CU has)
struct SmallLds {
    uint32_t key[kSmall];
    uint32_t hist[kBins];
    uint64_t mask_gt[kKeep * kSelWaves], mask_eq[kKeep * kSelWaves];   // flags of 64 items each, in memory order
    uint64_t before[kKeep * kSelWaves];       // flags set before those 64 (low word: gt, high word: eq)
    uint64_t seg[kMaxSegs];                   // (selected before segment b) - (flags before its first item)
    uint64_t scan[kSelWaves], found[2];
    uint64_t bin_sums[3][kSelWaves];          // find_bin_once, a set for each histogram
    uint64_t bin[3][2];
    uint32_t heavy;
};
static_assert(sizeof(SmallLds) <= 160 * 1024, "the LDS of a CU");

// Selection among n <= kSmall items by one workgroup of kSelBlock threads that keeps their keys in
// LDS: the remaining histograms in LDS, then one ballot per 64 items and kind (greater than
// theta, equal to it) from which the number of flags before any item can be read, so that an
// item's slot needs no second pass.  Items come in `nseg` segments, contiguous in memory but in any
// order; segment b precedes segment b + 1 in index order and holds the indices of
// [b seg_len, (b + 1) seg_len).  DIRECT: the items are est itself (index = position, one segment)
// and the first histogram is taken here as well.
// KEYED: their keys are in LDS already, each written by the thread that reads it here
// Of `shares` workgroups that all call this on the same items, this one (`share`) writes the items of its part and returns how
// many of its threads' items were heavy; with one, *out.n_heavy is written here.
template <bool DIRECT, bool KEYED, typename KEY>
__device__ __forceinline__ uint32_t select_in_workgroup(SmallLds& s, const float* __restrict__ val,
                                                    const int64_t* __restrict__ idx, uint32_t n,
                                                    uint32_t bin0, uint64_t k_rem,
                                                    const uint32_t* __restrict__ seg_base,
                                                    const uint32_t* __restrict__ seg_count, int nseg,
                                                    uint32_t seg_tiles, const SelOut& out, const KEY& kf, uint32_t share = 0,
                                                    uint32_t shares = 1) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kAhead = 4;                       // items of a thread whose index and value are on their way
    const uint32_t rounds = (n + kSelBlock - 1) / kSelBlock;
    const uint32_t from = rounds * share / shares * kSelBlock, upto = rounds * (share + 1) / shares * kSelBlock;
    const uint32_t end = upto < n ? upto : n;
    int64_t at[kAhead];
    float x[kAhead];
    auto load_ahead = [&](uint32_t p0) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const uint32_t p = p0 + q * kSelBlock < end ? p0 + q * kSelBlock : p0;
            at[q] = DIRECT ? static_cast<int64_t>(p) : idx[p];
            x[q] = val[p];
        }
    };
    // What comes last is on its way from here on.
    uint32_t base = 0, cnt_seg = 0;
    if constexpr (!DIRECT)
        if (tid < nseg) { base = seg_base[tid]; cnt_seg = seg_count[tid]; }
    if (!KEYED && from + tid < end) load_ahead(from + tid);
    for (int t = tid; t < kBins; t += kSelBlock) s.hist[t] = 0;
    if constexpr (!KEYED)
#pragma unroll 8
        for (uint32_t p = tid; p < n; p += kSelBlock) s.key[p] = kf(val[p], DIRECT ? static_cast<int64_t>(p) : idx[p]);
    // (a thread reads back only keys that it wrote itself)
    __syncthreads();
    // The histogram of a pass is cleared by the threads that read it, for the next one; with a bin whose entries are all
    // wanted the rest of the bits has nothing to decide: theta is then the key below that bin's first, none equal to it
    // is wanted.  us of k_topk_finish, with all passes, seven waits in each and one workgroup for the write / so: d = 2^20, k = 1000
    // 7.6 / 6.1; 11 M, k = 10 000 28.1 / 22.9; k_estimate_choose, 7 x 40, d = 784 11.1 / 9.6.
    bool all_of_bin = false;
    if constexpr (DIRECT) {
#pragma unroll 4
        for (uint32_t p = tid; p < n; p += kSelBlock) atomicAdd(&s.hist[s.key[p] >> 20], 1u);
        __syncthreads();
        const uint32_t cnt[2] = {s.hist[2 * tid], s.hist[2 * tid + 1]};
        s.hist[2 * tid] = s.hist[2 * tid + 1] = 0;
        find_bin_once<kSelWaves>(cnt, k_rem, s.bin_sums[0], s.bin[0], &bin0, &k_rem, &all_of_bin);
    }
    uint32_t theta = bin0;
    int shift = 20;                                 // of theta
#pragma unroll
    for (int pass = 1; pass <= 2; ++pass) {         // bits 19..10, then 9..0
        if (all_of_bin && theta != 0) break;
        shift -= 10;
        uint32_t* hist = s.hist + (DIRECT ? 0 : (pass - 1) * 1024);
#pragma unroll 4
        for (uint32_t p = tid; p < n; p += kSelBlock) {
            const uint32_t key = s.key[p];
            if ((key >> (shift + 10)) == theta) atomicAdd(&hist[(key >> shift) & 1023u], 1u);
        }
        __syncthreads();
        const uint32_t cnt[1] = {hist[tid]};
        if (DIRECT) hist[tid] = 0;
        uint32_t bin;
        find_bin_once<kSelWaves>(cnt, k_rem, s.bin_sums[pass], s.bin[pass], &bin, &k_rem, &all_of_bin);
        theta = (theta << 10) | bin;
    }
    if (shift > 0) {
        theta = (theta << shift) - 1u;
        k_rem = 0;
    }
    const uint64_t need_eq = k_rem;
    const int groups = static_cast<int>((n + 63) / 64);       // of 64 items
    for (int t = wave; t < groups; t += kSelWaves) {
        const uint32_t p = t * 64 + lane;
        const bool in = p < n;
        const uint32_t key = in ? s.key[p] : 0u;
        const uint64_t g = __builtin_amdgcn_ballot_w64(in && key > theta);
        const uint64_t e = __builtin_amdgcn_ballot_w64(in && key == theta);
        if (lane == 0) {
            s.mask_gt[t] = g;
            s.mask_eq[t] = e;
        }
    }
    if (tid == 0) s.heavy = 0;
    __syncthreads();
    auto counts = [&](int t) -> uint64_t {          // low word: gt, high word: eq
        return static_cast<uint64_t>(__builtin_popcountll(s.mask_gt[t])) |
               (static_cast<uint64_t>(__builtin_popcountll(s.mask_eq[t])) << 32);
    };
    uint64_t all;
    {
        static_assert(kKeep * kSelWaves <= kSelBlock && kMaxSegs <= kKeep * kSelWaves, "one group of 64 items per thread");
        const uint64_t mine = tid < groups ? counts(tid) : 0;
        const uint64_t b = block_exclusive_sum<kSelWaves>(mine, s.scan, &all);
        if (tid < groups) s.before[tid] = b;
    }
    __syncthreads();
    auto flags_before = [&](uint32_t p) -> uint64_t {   // of items [0, p)
        const uint32_t t = p >> 6, r = p & 63u;
        if (static_cast<int>(t) >= groups) return all;
        const uint64_t low = r ? (~0ull >> (64 - r)) : 0ull;
        return s.before[t] + (static_cast<uint64_t>(__builtin_popcountll(s.mask_gt[t] & low)) |
                              (static_cast<uint64_t>(__builtin_popcountll(s.mask_eq[t] & low)) << 32));
    };
    if constexpr (!DIRECT) {                        // two 32-bit counters side by side, modulo 2^32 each
        const uint64_t f0 = cnt_seg ? flags_before(base) : 0, f1 = cnt_seg ? flags_before(base + cnt_seg) : 0;
        const uint64_t b = block_exclusive_sum<kSelWaves>(f1 - f0, s.scan, &all);
        if (tid < nseg)
            s.seg[tid] = static_cast<uint32_t>(static_cast<uint32_t>(b) - static_cast<uint32_t>(f0)) |
                         (static_cast<uint64_t>(static_cast<uint32_t>(b >> 32) - static_cast<uint32_t>(f0 >> 32)) << 32);
        __syncthreads();
    }
    uint32_t heavy = 0;
    for (uint32_t p0 = from + tid; p0 < end; p0 += kAhead * kSelBlock) {
        if (KEYED || p0 != from + tid) load_ahead(p0);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const uint32_t p = p0 + q * kSelBlock;
            if (p >= end) break;
            const uint32_t key = s.key[p];
            const bool is_gt = key > theta, is_eq = key == theta;
            if (!(is_gt || is_eq)) continue;
            const uint64_t f = flags_before(p);
            uint32_t g = static_cast<uint32_t>(f), e = static_cast<uint32_t>(f >> 32);
            if constexpr (!DIRECT) {
                const uint64_t sg = s.seg[static_cast<uint32_t>(at[q] >> 10) / seg_tiles];
                g += static_cast<uint32_t>(sg);
                e += static_cast<uint32_t>(sg >> 32);
            }
            if (is_gt || e < need_eq) {
                out.put(static_cast<uint64_t>(g) + (e < need_eq ? e : need_eq), at[q], x[q]);
                heavy += key >> 30;
            }
        }
    }
    if (out.n_heavy) {
        if (heavy) atomicAdd(&s.heavy, heavy);
        __syncthreads();
        if (tid == 0 && shares == 1) *out.n_heavy = s.heavy;
    }
    return out.n_heavy ? s.heavy : 0u;
}

template <typename KEY>
__global__ void __launch_bounds__(kSelBlock)
k_topk_small(const float* __restrict__ est, uint32_t d, SelOut out, KEY kf) {
    kf.init();
    __shared__ SmallLds s;
    select_in_workgroup<true, false>(s, est, nullptr, d, 0u, static_cast<uint64_t>(out.k), nullptr, nullptr, 1, 1u, out, kf);
}

// Query and selection of a short vector by the workgroup that selects: estimates go to est and their keys straight into LDS.
// A step that short waits for the host, 6 us a call.  The hashes, 2 r per coordinate, are then one CU's work, so that r d is
// bounded by kQueryChooseHashes, where the kernels alone take as long either way: us from a graph, two launches / one, at 6144 (in
// brackets at 3000 to 4500), 40 columns: 1 row 14.0 / 14.0 (11.0 / 10.1); 3 10.8 / 11.1 (10.4 / 9.9); 5 11.0 / 10.5; 7 11.5 / 11.2;
// 9 12.3 / 12.4 (12.2 / 10.5); 11 13.2 / 13.4; 13 15.8 / 12.3; 15 16.0 / 13.8; 64 columns, no division: 0.4 to 2 less for the one.
// Beyond: 5 rows, d = 2000 13.0 / 13.4, 3276 14.1 / 16.7; 15, 800 18.4 / 22.4.
template <int R, bool POW2>
__global__ void __launch_bounds__(kSelBlock)
k_estimate_choose(KParams p, const float* __restrict__ S, uint32_t d, float* est, SelOut out) {
    __shared__ SmallLds s;
    const KeyMagnitude kf{};
    const Columns col = columns_of<POW2>(p.c);
    for (uint32_t t = threadIdx.x; t < d; t += kSelBlock) {
        const float v = estimate_at<R, POW2>(p, col, S, t);
        est[t] = v;
        s.key[t] = kf(v, static_cast<int64_t>(t));
    }
    // (est is read back by the threads that wrote it)
    select_in_workgroup<true, true>(s, est, nullptr, d, 0u, static_cast<uint64_t>(out.k), nullptr, nullptr, 1, 1u, out, kf);
}

// values that other workgroups of the launch wrote or added to: read past this XCD's caches
template <typename T>
__device__ __forceinline__ T load_shared(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void store_shared(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The rest of a selection, see the head of this file.  `listed`: a candidate list was asked for (it
// is used unless ws->failed says that it could not be built).  Phases of the shared form: 0 and 1
// the histograms of bits 19..10 and 9..0, 2 the counts of greater and equal entries per segment
// (per task when est is read), 3 the ordered write, whose starting slots are a scan of those counts.
template <bool VEC, typename KEY>
__global__ void __launch_bounds__(kSelBlock)
k_topk_finish(const float* __restrict__ est, int64_t d, TopkWs* ws, const uint64_t* __restrict__ hist0,
              bool listed, int nseg, uint32_t seg_tiles, const int64_t* __restrict__ cand_idx,
              const float* __restrict__ cand_val, SelOut out, KEY kf) {
    kf.init();
    __shared__ SmallLds s;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool from_list = listed && ws->failed == 0;
    const uint32_t n = from_list ? ws->ncand : 0u;
    if (from_list && n <= kSmall) {
        // Finding theta and counting take a workgroup 4 us and the slots and the write, 100 instructions an item, several times
        // that: every workgroup of up to kShares finds and counts, and writes its share.
        const uint32_t most = (n + kShareItems - 1) / kShareItems, shares = most < kShares ? most < 1 ? 1 : most : kShares;
        if (blockIdx.x >= shares) return;
        const uint32_t heavy = select_in_workgroup<false, false>(s, cand_val, cand_idx, n, ws->prefix, ws->k_rem, ws->seg_base,
                                                                 ws->seg_count, nseg, seg_tiles, out, kf, blockIdx.x, shares);
        if (tid != 0) return;
        if (shares > 1) {                              // the last one through puts the workspace back as it was
            if (heavy) __hip_atomic_fetch_add(&ws->heavy, heavy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (atomicAdd(&ws->exits, 1u) + 1 != shares) return;
            if (out.n_heavy) *out.n_heavy = load_shared(&ws->heavy);
            ws->exits = 0;
            ws->heavy = 0;
        }
        ws->ncand = 0;
        return;
    }
    // 4096 entries per task: a phase is then one load per thread.  What the phases hand on (the
    // histograms, the counts) is written and read with device-scope atomic accesses only, so no
    // cache has to be written back or invalidated in between: a task's accesses are complete
    // when its wavefronts have waited for them, and then it is counted as done.
    const int64_t items = from_list ? static_cast<int64_t>(n) : d;
    int64_t want = (items + 4095) / 4096;
    if (want > static_cast<int64_t>(gridDim.x)) want = gridDim.x;
    if (from_list && want > nseg) want = nseg;
    const uint32_t tasks = static_cast<uint32_t>(want);
    // Segments of the list that are long on the average are worked through by a whole workgroup, short
    // ones by a wavefront each (a workgroup has two or three of them, so that most of its wavefronts
    // would stand by while long ones are read 64 candidates at a time).  Lists of 3.6 M, 2.6 M and 1.6 M
    // candidates: this kernel takes 105, 100 and 85 us for 180, 170 and 125; a few hundred per segment
    // take two or three turns either way.
    const bool long_segments = n > 512u * static_cast<uint32_t>(nseg);
    if (blockIdx.x >= tasks) return;
    __shared__ uint32_t drawn;
    const int64_t est_chunk = ((d + tasks - 1) / tasks + 4095) / 4096 * 4096;
    const int64_t idle_polls = kIdlePolls + est_chunk / 16;
    __shared__ uint32_t finished;
    auto wait_for = [&](int phase) -> bool {        // every task of that phase is done; false: given up
        if (tid == 0) {
            uint32_t seen = load_shared(&ws->done[phase]);
            for (int64_t idle = 0; seen < tasks && idle < idle_polls; ++idle) {
                __builtin_amdgcn_s_sleep(8);
                const uint32_t now = load_shared(&ws->done[phase]);
                if (now != seen) idle = 0;
                seen = now;
            }
            finished = seen;
        }
        __syncthreads();
        return finished >= tasks;
    };
    // No selection came about (see the head of this file): indices that are in range, so that what
    // reads through them stays inside its vectors, and values that nobody takes for estimates.
    auto abandon = [&]() {
        for (int64_t t = tid; t < out.k; t += kSelBlock) out.put(static_cast<uint64_t>(t), t, __uint_as_float(0x7fc00000u));
        if (tid == 0 && out.n_heavy) *out.n_heavy = 0;
    };
    auto finish_task = [&](int phase) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) __hip_atomic_fetch_add(&ws->done[phase], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // the bins found so far: prefix of `bits` key bits and entries still wanted (every workgroup
    // finds them again from the finished histograms)
    uint32_t prefix = 0;
    uint64_t k_rem = static_cast<uint64_t>(out.k);
    int known = 0;                                  // histograms already looked at
    auto know = [&](int upto) {
        for (; known < upto; ++known) {
            uint32_t bin;
            if (known == 0) {
                const uint64_t cnt[2] = {hist0[2 * tid], hist0[2 * tid + 1]};
                find_bin<kSelWaves>(cnt, k_rem, s.scan, s.found, &bin, &k_rem);
                prefix = bin;
            } else {
                const uint64_t cnt[1] = {load_shared(&ws->hist[known][tid])};
                find_bin<kSelWaves>(cnt, k_rem, s.scan, s.found, &bin, &k_rem);
                prefix = (prefix << 10) | bin;
            }
        }
    };
    bool gave_up = false;
    for (;;) {
        if (tid == 0) drawn = atomicAdd(&ws->ticket, 1u);
        __syncthreads();
        const uint32_t ticket = drawn;
        __syncthreads();
        if (ticket >= 4 * tasks) break;
        const int phase = static_cast<int>(ticket / tasks);
        const uint32_t t = ticket - phase * tasks;
        if (phase > 0 && !wait_for(phase - 1)) {
            gave_up = true;
            break;
        }
        know(phase < 2 ? phase + 1 : 3);
        const int64_t lo = static_cast<int64_t>(t) * est_chunk;
        const int64_t hi = lo + est_chunk < d ? lo + est_chunk : d;
        const int seg0 = static_cast<int>(static_cast<int64_t>(nseg) * t / tasks);
        const int seg1 = static_cast<int>(static_cast<int64_t>(nseg) * (t + 1) / tasks);
        if (phase < 2) {
            const int shift = phase == 0 ? 10 : 0;
            s.hist[tid] = 0;
            __syncthreads();
            auto tally = [&](uint32_t key) {
                if ((key >> (shift + 10)) == prefix) atomicAdd(&s.hist[(key >> shift) & 1023u], 1u);
            };
            if (from_list) {
                for (uint32_t p = t * kSelBlock + tid; p < n; p += tasks * kSelBlock) tally(kf(cand_val[p], cand_idx[p]));
            } else {
                for (int64_t tile = lo; tile < hi; tile += kSelBlock * kItems) {
                    float v[kItems];
                    int nvalid;
                    const int64_t base = tile + static_cast<int64_t>(tid) * kItems;
                    load_items<VEC>(est, base, hi, v, nvalid);
#pragma unroll
                    for (int q = 0; q < kItems; ++q)
                        if (q < nvalid) tally(kf(v[q], base + q));
                }
            }
            __syncthreads();
            const uint32_t v = s.hist[tid];
            if (v) atomicAdd(reinterpret_cast<unsigned long long*>(&ws->hist[phase + 1][tid]),
                             static_cast<unsigned long long>(v));
        } else if (phase == 2) {
            if (from_list && long_segments) {       // the workgroup together, one segment after the other
                for (int b = seg0; b < seg1; ++b) {
                    const uint32_t base = ws->seg_base[b], cnt = ws->seg_count[b];
                    uint64_t c = 0, total;          // low word: greater, high word: equal
#pragma unroll 4
                    for (uint32_t p = tid; p < cnt; p += kSelBlock) {
                        const uint32_t key = kf(cand_val[base + p], cand_idx[base + p]);
                        c += (key > prefix ? 1ull : 0ull) | (key == prefix ? 1ull << 32 : 0ull);
                    }
                    block_exclusive_sum<kSelWaves>(c, s.scan, &total);
                    if (tid == 0) {
                        store_shared(&ws->gt[b], static_cast<uint64_t>(static_cast<uint32_t>(total)));
                        store_shared(&ws->eq[b], total >> 32);
                    }
                }
            } else if (from_list) {                 // one wavefront per segment
                for (int b = seg0 + wave; b < seg1; b += kSelWaves) {
                    const uint32_t base = ws->seg_base[b], cnt = ws->seg_count[b];
                    uint32_t n_gt = 0, n_eq = 0;
                    for (uint32_t p = lane; p < cnt; p += 64) {
                        const uint32_t key = kf(cand_val[base + p], cand_idx[base + p]);
                        n_gt += key > prefix ? 1u : 0u;
                        n_eq += key == prefix ? 1u : 0u;
                    }
#pragma unroll
                    for (int off = 32; off > 0; off >>= 1) {
                        n_gt += __shfl_down(n_gt, off, 64);
                        n_eq += __shfl_down(n_eq, off, 64);
                    }
                    if (lane == 0) {
                        store_shared(&ws->gt[b], static_cast<uint64_t>(n_gt));
                        store_shared(&ws->eq[b], static_cast<uint64_t>(n_eq));
                    }
                }
            } else {
                uint64_t n_gt = 0, n_eq = 0, sum_gt, sum_eq;
                for (int64_t tile = lo; tile < hi; tile += kSelBlock * kItems) {
                    float v[kItems];
                    int nvalid;
                    const int64_t base = tile + static_cast<int64_t>(tid) * kItems;
                    load_items<VEC>(est, base, hi, v, nvalid);
#pragma unroll
                    for (int q = 0; q < kItems; ++q) {
                        if (q >= nvalid) break;
                        const uint32_t key = kf(v[q], base + q);
                        n_gt += key > prefix ? 1u : 0u;
                        n_eq += key == prefix ? 1u : 0u;
                    }
                }
                block_exclusive_sum<kSelWaves>(n_gt, s.scan, &sum_gt);
                block_exclusive_sum<kSelWaves>(n_eq, s.scan, &sum_eq);
                if (tid == 0) {
                    store_shared(&ws->gt[t], sum_gt);
                    store_shared(&ws->eq[t], sum_eq);
                }
            }
        } else {
            const uint64_t need_eq = k_rem;
            uint32_t heavy = 0;
            // one tile of the workgroup: kItems consecutive items per thread, g greater and e equal
            // ones before the tile (moved on past it); at(q) is the index of the thread's q-th item
            auto write_tile = [&](const float (&v)[kItems], int nvalid, uint64_t& g, uint64_t& e, auto at) {
                uint64_t c = 0;                     // low word: greater, high word: equal
#pragma unroll
                for (int q = 0; q < kItems; ++q) {
                    if (q >= nvalid) break;
                    const uint32_t key = kf(v[q], at(q));
                    c += (key > prefix ? 1ull : 0ull) | (key == prefix ? 1ull << 32 : 0ull);
                }
                uint64_t total;
                const uint64_t before = block_exclusive_sum<kSelWaves>(c, s.scan, &total);
                if (c) {
                    uint64_t my_g = g + static_cast<uint32_t>(before), my_e = e + (before >> 32);
#pragma unroll
                    for (int q = 0; q < kItems; ++q) {
                        if (q >= nvalid) break;
                        const uint32_t key = kf(v[q], at(q));
                        const bool is_gt = key > prefix, is_eq = key == prefix;
                        if (is_gt || (is_eq && my_e < need_eq)) {
                            out.put(my_g + (my_e < need_eq ? my_e : need_eq), at(q), v[q]);
                            heavy += key >> 30;
                        }
                        my_g += is_gt;
                        my_e += is_eq;
                    }
                }
                g += static_cast<uint32_t>(total);
                e += total >> 32;
            };
            if (from_list) {
                // slots before each segment: a scan over all of them
                uint64_t all;
                const bool in = tid < nseg;
                const uint64_t g0 = block_exclusive_sum<kSelWaves>(in ? load_shared(&ws->gt[tid]) : 0, s.scan, &all);
                const uint64_t e0 = block_exclusive_sum<kSelWaves>(in ? load_shared(&ws->eq[tid]) : 0, s.scan, &all);
                if (in) { s.mask_gt[tid] = g0; s.mask_eq[tid] = e0; }
                __syncthreads();
                const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));   // lanes before mine
                for (int b = seg0; long_segments && b < seg1; ++b) {
                    uint64_t g = s.mask_gt[b], e = s.mask_eq[b];
                    const uint32_t base = ws->seg_base[b], cnt = ws->seg_count[b];
                    for (uint32_t p0 = 0; p0 < cnt; p0 += kSelBlock * kItems) {
                        float v[kItems];
                        int64_t i[kItems];
                        int nvalid = 0;
                        const uint32_t p = p0 + tid * kItems;
#pragma unroll
                        for (int q = 0; q < kItems; ++q) {
                            if (p + q < cnt) {
                                v[q] = cand_val[base + p + q];
                                i[q] = cand_idx[base + p + q];
                                nvalid = q + 1;
                            } else {
                                v[q] = 0.0f;
                                i[q] = 0;
                            }
                        }
                        write_tile(v, nvalid, g, e, [&](int q) { return i[q]; });
                    }
                }
                for (int b = seg0 + wave; !long_segments && b < seg1; b += kSelWaves) {
                    uint64_t g = s.mask_gt[b], e = s.mask_eq[b];
                    const uint32_t base = ws->seg_base[b], cnt = ws->seg_count[b];
                    for (uint32_t p0 = 0; p0 < cnt; p0 += 64) {
                        const uint32_t p = p0 + lane;
                        bool is_gt = false, is_eq = false;
                        int64_t i = 0;
                        float v = 0.0f;
                        uint32_t key = 0;
                        if (p < cnt) {
                            i = cand_idx[base + p];
                            v = cand_val[base + p];
                            key = kf(v, i);
                            is_gt = key > prefix;
                            is_eq = key == prefix;
                        }
                        const uint64_t m_gt = __builtin_amdgcn_ballot_w64(is_gt);
                        const uint64_t m_eq = __builtin_amdgcn_ballot_w64(is_eq);
                        const uint64_t my_g = g + __builtin_popcountll(m_gt & below);
                        const uint64_t my_e = e + __builtin_popcountll(m_eq & below);
                        if (is_gt || (is_eq && my_e < need_eq)) {
                            out.put(my_g + (my_e < need_eq ? my_e : need_eq), i, v);
                            heavy += key >> 30;
                        }
                        g += __builtin_popcountll(m_gt);
                        e += __builtin_popcountll(m_eq);
                    }
                }
            } else {
                uint64_t g, e;                      // greater / equal entries before the tile
                {
                    uint64_t all_g, all_e;
                    const bool in = tid < static_cast<int>(t);
                    block_exclusive_sum<kSelWaves>(in ? load_shared(&ws->gt[tid]) : 0, s.scan, &all_g);
                    block_exclusive_sum<kSelWaves>(in ? load_shared(&ws->eq[tid]) : 0, s.scan, &all_e);
                    g = all_g;
                    e = all_e;
                }
                for (int64_t tile = lo; tile < hi; tile += kSelBlock * kItems) {
                    float v[kItems];
                    int nvalid;
                    const int64_t base = tile + static_cast<int64_t>(tid) * kItems;
                    load_items<VEC>(est, base, hi, v, nvalid);
                    write_tile(v, nvalid, g, e, [&](int q) { return base + q; });
                }
            }
            if (out.n_heavy && heavy) atomicAdd(&ws->heavy, heavy);
        }
        finish_task(phase);
    }
    if (gave_up) abandon();
    // the last workgroup to leave puts the workspace back as it was; every count of a finished task
    // has arrived by then
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) drawn = atomicAdd(&ws->exits, 1u);
    __syncthreads();
    if (drawn + 1 != tasks) return;
    if (tid == 0) finished = load_shared(&ws->done[3]);
    __syncthreads();
    const bool whole = finished == tasks;
    if (!whole && !gave_up) abandon();
    for (int t = tid; t < 2 * kBins; t += kSelBlock) (&ws->hist[1][0])[t] = 0;
    if (tid == 0) {
        if (out.n_heavy && whole) *out.n_heavy = load_shared(&ws->heavy);
        ws->ticket = 0;
        ws->exits = 0;
        for (int q = 0; q < 4; ++q) ws->done[q] = 0;
        ws->failed = 0;
        ws->ncand = 0;
        ws->heavy = 0;
    }
}

// Alg. 1 step 1: out[1 + j] = sum_b S[j][b]^2, one workgroup of 1024 threads per row, binary64
// sums in a fixed order (each thread a strided share in four independent chains, then a tree
// over the workgroup), 16-byte loads when the row allows.  A workgroup alone on its CU waits for its loads: with one of a
// thread in flight 5 x 180 000 took 16.7 us, with eight 10.4.
constexpr int kSumBlock = 1024;
constexpr int kSumAhead = 8;         // loads of a thread in flight
__global__ void __launch_bounds__(kSumBlock)
k_row_sumsq(const float* __restrict__ S, uint32_t c, double* __restrict__ out) {
    __shared__ double part[kSumBlock];
    const float* row = S + static_cast<size_t>(blockIdx.x) * c;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    uint32_t done = 0;
    if (reinterpret_cast<uintptr_t>(row) % 16 == 0) {
        const uint32_t n4 = c / 4;
        const float4* row4 = reinterpret_cast<const float4*>(row);
        auto add = [&](const float4& u) {
            a0 += static_cast<double>(u.x) * static_cast<double>(u.x);
            a1 += static_cast<double>(u.y) * static_cast<double>(u.y);
            a2 += static_cast<double>(u.z) * static_cast<double>(u.z);
            a3 += static_cast<double>(u.w) * static_cast<double>(u.w);
        };
        uint32_t q = threadIdx.x;
        for (; static_cast<uint64_t>(q) + (kSumAhead - 1) * kSumBlock < n4; q += kSumAhead * kSumBlock) {
            float4 u[kSumAhead];
#pragma unroll
            for (int e = 0; e < kSumAhead; ++e) u[e] = row4[q + e * kSumBlock];
#pragma unroll
            for (int e = 0; e < kSumAhead; ++e) add(u[e]);
        }
        for (; q < n4; q += kSumBlock) add(row4[q]);
        done = n4 * 4;
    }
    uint64_t b = done + threadIdx.x;
    for (; b + (kSumAhead - 1) * kSumBlock < c; b += kSumAhead * kSumBlock) {
        float u[kSumAhead];
#pragma unroll
        for (int e = 0; e < kSumAhead; ++e) u[e] = row[b + e * kSumBlock];
#pragma unroll
        for (int e = 0; e < kSumAhead; ++e) a0 += static_cast<double>(u[e]) * static_cast<double>(u[e]);
    }
    for (; b < c; b += kSumBlock) a0 += static_cast<double>(row[b]) * static_cast<double>(row[b]);
    part[threadIdx.x] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    for (int off = kSumBlock / 2; off > 0; off >>= 1) {
        if (static_cast<int>(threadIdx.x) < off) part[threadIdx.x] += part[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[1 + blockIdx.x] = part[0];
}

// out[0] = median of out[1 .. r] (r odd, <= CS_MAX_R): insertion sort by one thread
__global__ void k_median_of_rows(double* out, int r) {
    double v[CS_MAX_R];
    for (int j = 0; j < r; ++j) {
        double x = out[1 + j];
        int q = j;
        while (q > 0 && v[q - 1] > x) { v[q] = v[q - 1]; --q; }
        v[q] = x;
    }
    out[0] = v[r / 2];
}

__global__ void __launch_bounds__(kBlock) k_hist_zero(uint64_t* hist) {
    for (int t = threadIdx.x; t < kBins; t += kBlock) hist[t] = 0;
}

int launch_magnitude_hist_zero(uint64_t* hist, hipStream_t stream) {
    k_hist_zero<<<1, kBlock, 0, stream>>>(hist);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

// workgroups of the first histogram (more of them only add to the atomic adds at their end)
static unsigned hist0_grid(int64_t d) {
    const int64_t b = (d + kScanBlock * kItems * 2 - 1) / (kScanBlock * kItems * 2);
    return static_cast<unsigned>(b < kMaxSegs ? (b < 1 ? 1 : b) : kMaxSegs);
}

int launch_magnitude_hist(const float* est, int64_t d, uint64_t* hist, hipStream_t stream) {
    if (reinterpret_cast<uintptr_t>(est) % 16 == 0)
        k_topk_hist0<true, KeyMagnitude><<<hist0_grid(d), kScanBlock, 0, stream>>>(est, d, hist, KeyMagnitude{});
    else
        k_topk_hist0<false, KeyMagnitude><<<hist0_grid(d), kScanBlock, 0, stream>>>(est, d, hist, KeyMagnitude{});
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

}  // namespace cs

using namespace cs;

extern "C" int cs_topk_workspace_bytes(int64_t d, int64_t k, size_t* bytes) {
    if (!bytes || d < 1 || k < 1 || k > d) return CS_EINVAL;
    *bytes = sizeof(TopkWs) + static_cast<size_t>(candidate_capacity_for(d, k)) * kCandBytes;
    return CS_OK;
}

// the k entries with the largest keys, ascending by index (see the header of this file).
// hist0: device uint64[2048], the histogram of key >> 20 over est, when the caller has it.
template <typename KEY, bool VEC>
static void enqueue_selection(const float* est, int64_t d, const uint64_t* hist0, const SelOut& out,
                              TopkWs* ws, int64_t cap, bool listed, bool clean, hipStream_t s, KEY kf) {
    int64_t* cand_idx = reinterpret_cast<int64_t*>(ws + 1);
    float* cand_val = reinterpret_cast<float*>(cand_idx + cap);
    if (!clean || !hist0) k_topk_clear<<<1, kBlock, 0, s>>>(ws);   // (hist[0] is not left clear)
    if (!hist0) {
        k_topk_hist0<VEC, KEY><<<hist0_grid(d), kScanBlock, 0, s>>>(est, d, ws->hist[0], kf);
        hist0 = ws->hist[0];
    }
    // chunks of whole KiB-tiles, at most kMaxSegs of them
    const int64_t tiles = (d + 1023) / 1024;
    const int64_t want = (tiles + 3) / 4 < kMaxSegs ? (tiles + 3) / 4 : kMaxSegs;   // >= 4096 entries each
    const int64_t seg_tiles = (tiles + want - 1) / want, chunk = seg_tiles * 1024;
    const int nseg = static_cast<int>((d + chunk - 1) / chunk);
    if (listed)
        k_topk_compact<VEC, KEY><<<nseg, kScanBlock, 0, s>>>(est, d, chunk, ws, hist0, static_cast<uint64_t>(out.k),
                                                             static_cast<uint32_t>(cap), cand_idx, cand_val, kf);
    k_topk_finish<VEC, KEY><<<kFinishBlocks, kSelBlock, 0, s>>>(est, d, ws, hist0, listed, nseg,
                                                                static_cast<uint32_t>(seg_tiles), cand_idx, cand_val,
                                                                out, kf);
}

template <typename KEY>
static int select_largest(const float* est, int64_t d, const uint64_t* hist0, const SelOut& out,
                          void* workspace, size_t ws_bytes, hipStream_t s, KEY kf, bool clean = false) {
    const int64_t k = out.k;
    if (d < 1 || k < 1 || k > d || !est || !out.idx || !workspace) return CS_EINVAL;
    if (reinterpret_cast<uintptr_t>(workspace) % 8 != 0) return CS_EINVAL;
    if (hist0 && reinterpret_cast<uintptr_t>(hist0) % 8 != 0) return CS_EINVAL;
    if (ws_bytes < sizeof(TopkWs)) return CS_EWORKSPACE;
    if (d <= kSmall) {
        k_topk_small<KEY><<<1, kSelBlock, 0, s>>>(est, static_cast<uint32_t>(d), out, kf);
        return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
    }
    TopkWs* ws = static_cast<TopkWs*>(workspace);
    // The candidate list takes what the workspace holds beyond the struct, up to what is worth
    // having; it is used when that is at least 2 k + 4096 entries (the k-th largest key's own
    // bin has to fit beside the k entries above it) and clearly less than d.
    int64_t cap = static_cast<int64_t>((ws_bytes - sizeof(TopkWs)) / kCandBytes);
    if (cap > candidate_capacity_for(d, k)) cap = candidate_capacity_for(d, k);
    if (cap > 0xffffffffll) cap = 0xffffffffll;
    const bool listed = cap >= 2 * k + 4096;
    if (reinterpret_cast<uintptr_t>(est) % 16 == 0)
        enqueue_selection<KEY, true>(est, d, hist0, out, ws, cap, listed, clean, s, kf);
    else
        enqueue_selection<KEY, false>(est, d, hist0, out, ws, cap, listed, clean, s, kf);
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

extern "C" int cs_heavy_hitters_topk(const float* est, int64_t d, int64_t k,
                                     const uint64_t* hist_or_null, int64_t* idx_out,
                                     float* val_out, void* workspace, size_t ws_bytes,
                                     void* stream) {
    return select_largest(est, d, hist_or_null, SelOut{idx_out, val_out, nullptr, nullptr, k}, workspace, ws_bytes,
                          reinterpret_cast<hipStream_t>(stream), KeyMagnitude{});
}

// A workspace that its owner keeps for one stream of selections is cleared once, here; every
// selection leaves it clear, so that cs_heavy_hitters_topk_kept needs no launch for that.
extern "C" int cs_topk_workspace_clear(void* workspace, size_t ws_bytes, void* stream) {
    if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 8 != 0) return CS_EINVAL;
    if (ws_bytes < sizeof(TopkWs)) return CS_EWORKSPACE;
    k_topk_clear<<<1, kBlock, 0, reinterpret_cast<hipStream_t>(stream)>>>(static_cast<TopkWs*>(workspace));
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

extern "C" int cs_heavy_hitters_topk_kept(const float* est, int64_t d, int64_t k,
                                          const uint64_t* hist_or_null, int64_t* idx_out,
                                          float* val_out, void* workspace, size_t ws_bytes,
                                          void* stream) {
    return select_largest(est, d, hist_or_null, SelOut{idx_out, val_out, nullptr, nullptr, k}, workspace, ws_bytes,
                          reinterpret_cast<hipStream_t>(stream), KeyMagnitude{}, true);
}

// ---------------------------------------------------------------------------------------
// The selection for callers that cannot allocate: its workspace is an array in the library's
// own device image.  Every GPU holds its own copy at its own address, so the address is asked
// for once per device (with that device current) and kept; host code never passes the array's
// name to a kernel.
// ---------------------------------------------------------------------------------------
constexpr size_t kStaticCandidates = 131072;     // room for a candidate list: selections up to k ~ 60 000 read est twice
static __device__ __align__(256) unsigned char
    scratch[(sizeof(cs::TopkWs) + kStaticCandidates * cs::kCandBytes + 255) / 256 * 256];

static int static_scratch(void** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptr_of_device[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return CS_EHIP;
    if (dev < 0 || dev >= kMaxDevices) return CS_EINVAL;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of_device[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return CS_EHIP;
        ptr_of_device[dev] = ptr;
    }
    *out = ptr_of_device[dev];
    return CS_OK;
}

extern "C" int cs_heavy_hitters_topk_static(const float* est, int64_t d, int64_t k,
                                            int64_t* idx_out, float* val_out, void* stream) {
    if (d > CS_TOPK_STATIC_MAX_D) return CS_ELIMIT;
    void* ws = nullptr;
    const int rc = static_scratch(&ws);
    if (rc != CS_OK) return rc;
    return select_largest(est, d, nullptr, SelOut{idx_out, val_out, nullptr, nullptr, k}, ws, sizeof(scratch),
                          reinterpret_cast<hipStream_t>(stream), KeyMagnitude{});
}

extern "C" int cs_sketch_estimate_topk(const cs_params* p, const float* S, int64_t d, float* est, int64_t k, int64_t* idx_out,
                                       float* val_out, void* stream) {
    if (!p || !S || !est || !idx_out || k < 1 || d < 1 || k > d) return CS_EINVAL;
    if (p->r == 0 || p->r > CS_MAX_R || (p->r & 1u) == 0 || p->c == 0 || p->c > (1u << 31)) return CS_EINVAL;
    if (d > kSmall || d * p->r > kQueryChooseHashes) return CS_ELIMIT;
    const SelOut out{idx_out, val_out, nullptr, nullptr, k};
#define CALL(R_, P2_)                                                                                       \
    k_estimate_choose<R_, P2_><<<1, kSelBlock, 0, reinterpret_cast<hipStream_t>(stream)>>>(                  \
        kparams(p), S, static_cast<uint32_t>(d), est, out)
    CS_DISPATCH_R(p, CALL);
#undef CALL
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

extern "C" int cs_sketch_l2sq(const cs_params* p, const float* S, double* out, void* stream) {
    if (!p || !S || !out) return CS_EINVAL;
    if (p->r == 0 || p->r > CS_MAX_R || (p->r & 1u) == 0 || p->c == 0) return CS_EINVAL;
    if (reinterpret_cast<uintptr_t>(out) % 8 != 0) return CS_EINVAL;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    k_row_sumsq<<<p->r, kSumBlock, 0, s>>>(S, p->c, out);
    k_median_of_rows<<<1, 1, 0, s>>>(out, static_cast<int>(p->r));
    return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP;
}

extern "C" int cs_heavymix_select(const float* est, int64_t d, int64_t k, const double* l2sq,
                                  uint64_t rng_seed, int64_t* idx_out, float* val_out,
                                  int64_t* n_heavy, void* workspace, size_t ws_bytes,
                                  void* stream) {
    if (!l2sq || reinterpret_cast<uintptr_t>(l2sq) % 8 != 0) return CS_EINVAL;
    if (n_heavy && reinterpret_cast<uintptr_t>(n_heavy) % 8 != 0) return CS_EINVAL;
    return select_largest(est, d, nullptr,
                          SelOut{idx_out, val_out, nullptr, reinterpret_cast<unsigned long long*>(n_heavy), k},
                          workspace, ws_bytes, reinterpret_cast<hipStream_t>(stream),
                          KeyHeavymix{l2sq, static_cast<double>(k), rng_seed, 0.0});
}

extern "C" int cs_select_exact_topk(const int64_t* cand, const float* x, int64_t n, int64_t k,
                                    int64_t* idx_out, float* val_out, void* workspace,
                                    size_t ws_bytes, void* stream) {
    if (!cand) return CS_EINVAL;
    // positions of the k largest |x| (ascending), written as the coordinates they stand for; cand
    // is ascending, so the result is ascending too
    return select_largest(x, n, nullptr, SelOut{idx_out, val_out, cand, nullptr, k}, workspace, ws_bytes,
                          reinterpret_cast<hipStream_t>(stream), KeyMagnitude{});
}
