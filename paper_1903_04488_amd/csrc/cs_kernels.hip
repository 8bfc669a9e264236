// Kernels and C ABI of the Count Sketch hot path (gfx950).  See include/csketch.h for what
// every entry point computes and which passage of the paper defines it.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "cs_device.h"
#include "cs_internal.h"
#include "csketch.h"
#include "csketch_probe.h"

namespace cs {

// ---------------------------------------------------------------------------------------
// launch helpers
// ---------------------------------------------------------------------------------------
inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

inline int launch_status() { return hipGetLastError() == hipSuccess ? CS_OK : CS_EHIP; }

inline bool params_ok(const cs_params* p) {
    return p && p->r >= 1 && p->r <= CS_MAX_R && (p->r & 1u) && p->c >= 1 && p->c <= (1u << 31);
}

// number of workgroups for a grid-stride kernel over n items: enough to fill 256 CUs a few
// times over, never more than the items need.
inline unsigned grid_for(int64_t n, int per_block = kBlock, int max_blocks = 256 * 16) {
    int64_t b = (n + per_block - 1) / per_block;
    if (b < 1) b = 1;
    if (b > max_blocks) b = max_blocks;
    return static_cast<unsigned>(b);
}

// Workgroups of the kernels that hash every coordinate, with `slots` threads that take a coordinate each (of `groups` such
// grids): 8 coordinates a thread, which share its first states, or one where that would be under 128 workgroups: short
// vectors wait on chains of hashes and gathers (us, 8 a thread / one; query: 15 x 257, d = 12 001 22.4 / 10.4; 15 x 2001,
// 150 003 24.9 / 17.4; 5 x 257, 12 001 7.1 / 5.2; 15 x 8193, 500 007 35.9 / 36.9; tables of 4 workers: 5 x 64, 3000 7.8 / 6.0;
// 5 x 129, 5000 8.5 / 5.8).  Numbers between are no better: query of 5 x 8193, 700 001 16.6 with 8, 16.1 with 2, 18.2 with 5.
// `below`: the query of up to 5 rows that lie in L1 has gathers to wait for only up to 96 (5 x 709, d = 180 001 6.9 / 6.3, 200 001
// 7.0 / 7.3; 3 x 257, 200 001 4.9 / 5.3; but 5 x 6605, 200 001 8.0 / 7.4; 7 x 709 9.3 / 9.3).
inline unsigned grid_of_hashes(int64_t d, int slots, int64_t groups = 1, int64_t below = 128) {
    const bool few = d / (slots * 8) < below / groups;
    return grid_for(d, few ? slots : slots * 8, 256 * 8);
}

// Tables of several groups of workers with few columns and many coordinates for each: their requests wait for one another at
// the same few cells, the longer the more of them are sent at once (us, tables with 8 coordinates a thread / one, in brackets
// coordinates a column: 17 workers, 5 x 32, d = 7895 (247) 15.6 / 22.3; 127, 7 x 33, 7541 (229) 63 / 107; 153, 3 x 33, 2533 (77)
// 38 / 40; 132, 5 x 33, 2223 (67) 41 / 37; 152, 3 x 91, 6663 (73) 62 / 55; 10, 15 x 99, 11 843 (120) 26.3 / 29.0; 106, 15 x 69,
// 4348 (63) 97 / 109; 184, 15 x 81, 2088 (26) 107 / 94; one group, 7 workers, 5 x 33, 6029 (183) 12.7 / 12.7).
inline bool crowded_cells(const cs_params* p, int64_t d, int64_t groups) {
    return groups > 1 && p->c < 128 && d >= static_cast<int64_t>(p->r > 8 ? 50 : p->c < 80 ? 75 : 100) * p->c;
}

// ---------------------------------------------------------------------------------------
// hash parity hooks
// ---------------------------------------------------------------------------------------
template <bool POW2>
__global__ void __launch_bounds__(kBlock)
k_hash_list(KParams p, const int64_t* __restrict__ idx, int64_t n,
            uint32_t* __restrict__ bucket, int8_t* __restrict__ sign) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride) {
        const uint64_t i = static_cast<uint64_t>(idx[t]);
        for (uint32_t j = 0; j < p.r; ++j) {
            const uint64_t yb = hash_state(p.a[j], p.b[j], i);
            const uint64_t ys = hash_state(p.as[j], p.bs[j], i);
            bucket[static_cast<size_t>(j) * n + t] = bucket_of<POW2>(yb, col);
            sign[static_cast<size_t>(j) * n + t] = sign_flip_of(ys) ? -1 : 1;
        }
    }
}

// Streaming hash state of all R rows for one thread: start at coordinate `first`, then step
// by `stride` coordinates at a time.
template <int R>
struct RowStates {
    uint64_t yb[R], ys[R];    // y-form states of the bucket and sign hashes
    uint64_t Ab[R], As[R];    // (a_j * stride) mod p, (a'_j * stride) mod p

    __device__ __forceinline__ void init(const KParams& p, uint64_t first, uint64_t stride) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            yb[j] = hash_state(p.a[j], p.b[j], first);
            ys[j] = hash_state(p.as[j], p.bs[j], first);
            Ab[j] = mulmod_p(p.a[j], stride);
            As[j] = mulmod_p(p.as[j], stride);
        }
    }
    __device__ __forceinline__ void advance() {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            yb[j] = hash_advance(yb[j], Ab[j]);
            ys[j] = hash_advance(ys[j], As[j]);
        }
    }
};

template <int R, bool POW2>
__global__ void __launch_bounds__(kBlock)
k_hash_range(KParams p, int64_t i0, int64_t n, uint32_t* __restrict__ bucket,
             int8_t* __restrict__ sign) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (t >= n) return;
    RowStates<R> st;
    st.init(p, static_cast<uint64_t>(i0 + t), static_cast<uint64_t>(stride));
    for (; t < n; t += stride) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            bucket[static_cast<size_t>(j) * n + t] = bucket_of<POW2>(st.yb[j], col);
            sign[static_cast<size_t>(j) * n + t] = sign_flip_of(st.ys[j]) ? -1 : 1;
        }
        st.advance();
    }
}

// ---------------------------------------------------------------------------------------
// sketch_accumulate: Alg. 4 update over a dense vector
// ---------------------------------------------------------------------------------------
using BatchPtrs = LatticePtrs;

// One thread per coordinate, grid-stride; the gradient is read coalesced, the r updates go
// out as fp32 atomics.  With NW > 1 the same hash values serve NW workers.
template <int R, bool POW2>
__global__ void __launch_bounds__(kBlock)
k_accumulate(KParams p, BatchPtrs ptrs, int nw, int64_t d, int64_t i0, float scale) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (t >= d) return;
    RowStates<R> st;
    st.init(p, static_cast<uint64_t>(i0 + t), static_cast<uint64_t>(stride));
    const uint32_t c = p.c;
    for (; t < d; t += stride) {
        uint32_t cell[R], flip[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            cell[j] = static_cast<uint32_t>(j) * c + bucket_of<POW2>(st.yb[j], col);
            flip[j] = sign_flip_of(st.ys[j]);
        }
        for (int w = 0; w < nw; ++w) {
            const float v = scale * ptrs.g[w][t];
            float* S = ptrs.S[w];
#pragma unroll
            for (int j = 0; j < R; ++j)
                atomic_add_noret(S + cell[j], apply_sign(v, flip[j]));
        }
        st.advance();
    }
}

// Update of a worker bundle for any sketch shape.  Eight neighbouring lanes form a slot that
// takes one coordinate; lane q of the slot carries worker q of the group (blockIdx.y), so the
// slot's 8 updates of a cell T[group][j][b][0..8) are 32 contiguous bytes and leave the
// wavefront as ONE memory request per row instead of one per worker: the atomic unit, which
// bounds this kernel, sees W/8 times fewer requests than with one table per worker.  The 8
// lanes of a slot evaluate the same hashes; that work is hidden behind the atomics.
struct GroupedVectors {
    const float* g[kMaxBatch];   // worker w of the launch; group = w / 8
};

template <int R, bool POW2>
__global__ void __launch_bounds__(kBlock)
k_accumulate_cells(KParams p, GroupedVectors vec, int nw, float* __restrict__ T, int64_t d,
                   int64_t i0, float scale) {
    constexpr int kSlots = kBlock / CS_BUNDLE_GROUP;
    const int q = threadIdx.x % CS_BUNDLE_GROUP;
    const int w = blockIdx.y * CS_BUNDLE_GROUP + q;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kSlots;
    int64_t t = static_cast<int64_t>(blockIdx.x) * kSlots + threadIdx.x / CS_BUNDLE_GROUP;
    if (t >= d || w >= nw) return;
    const float* g = nullptr;
#pragma unroll
    for (int u = 0; u < CS_BUNDLE_GROUP; ++u)
        if (q == u) g = vec.g[blockIdx.y * CS_BUNDLE_GROUP + u];
    const uint32_t c = p.c;
    float* Tq = T + static_cast<size_t>(blockIdx.y) * R * c * CS_BUNDLE_GROUP + q;
    const Columns col = columns_of<POW2>(c);
    RowStates<R> st;
    st.init(p, static_cast<uint64_t>(i0 + t), static_cast<uint64_t>(stride));
    for (; t < d; t += stride) {
        const float v = scale * g[t];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const size_t cell = static_cast<size_t>(j) * c + bucket_of<POW2>(st.yb[j], col);
            atomic_add_noret(Tq + cell * CS_BUNDLE_GROUP, apply_sign(v, sign_flip_of(st.ys[j])));
        }
        st.advance();
    }
}

// The same update when one group's whole table fits in LDS (R * c * 8 floats <= 64 KB): a
// workgroup adds into a private copy with LDS atomics and sends every non-zero cell to memory
// once at the end.  Only narrow tables gain.  Measured per coordinate and row: through memory
// max(10 / c, 0.05) ns (few columns are a hot spot for the memory-side atomic unit), through
// LDS 0.045 ns plus ~10 us per launch for clearing and sending the copy; beyond ~200 columns
// the memory path is as fast as LDS float atomics.
constexpr uint32_t kLdsCells = 2048;      // R * c at most: 64 KB of LDS for 8 workers
constexpr uint32_t kLdsColumns = 128;     // c at most

bool lds_table_applies(const cs_params* p, int64_t d) {
    return !(p->flags & CS_FLAG_NO_LDS_TABLE) && p->c <= kLdsColumns &&
           static_cast<uint64_t>(p->r) * p->c <= kLdsCells &&
           d >= static_cast<int64_t>(2048) * p->c / p->r;
}

template <int R, bool POW2>
__global__ void __launch_bounds__(kBlock)
k_accumulate_cells_lds(KParams p, GroupedVectors vec, int nw, float* __restrict__ T, int64_t d,
                       int64_t i0, float scale) {
    extern __shared__ float part[];       // [R][c][8]
    constexpr int kSlots = kBlock / CS_BUNDLE_GROUP;
    const uint32_t c = p.c;
    const int floats = static_cast<int>(R * c * CS_BUNDLE_GROUP);
    for (int x = threadIdx.x; x < floats; x += kBlock) part[x] = 0.0f;
    __syncthreads();
    const int q = threadIdx.x % CS_BUNDLE_GROUP;
    const int w = blockIdx.y * CS_BUNDLE_GROUP + q;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kSlots;
    int64_t t = static_cast<int64_t>(blockIdx.x) * kSlots + threadIdx.x / CS_BUNDLE_GROUP;
    if (t < d && w < nw) {
        const float* g = nullptr;
#pragma unroll
        for (int u = 0; u < CS_BUNDLE_GROUP; ++u)
            if (q == u) g = vec.g[blockIdx.y * CS_BUNDLE_GROUP + u];
        const Columns col = columns_of<POW2>(c);
        RowStates<R> st;
        st.init(p, static_cast<uint64_t>(i0 + t), static_cast<uint64_t>(stride));
        for (; t < d; t += stride) {
            const float v = scale * g[t];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const uint32_t cell = static_cast<uint32_t>(j) * c + bucket_of<POW2>(st.yb[j], col);
                __hip_atomic_fetch_add(part + cell * CS_BUNDLE_GROUP + q,
                                       apply_sign(v, sign_flip_of(st.ys[j])), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            st.advance();
        }
    }
    __syncthreads();
    float* Tg = T + static_cast<size_t>(blockIdx.y) * floats;
    for (int x = threadIdx.x; x < floats; x += kBlock) {
        const float v = part[x];
        if (v != 0.0f) atomic_add_noret(Tg + x, v);     // NaN compares unequal: it is sent
    }
}

template <bool POW2>
__global__ void __launch_bounds__(kBlock)
k_accumulate_sparse(KParams p, float* __restrict__ S, const int64_t* __restrict__ idx,
                    const float* __restrict__ val, int64_t n, float scale) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride) {
        const uint64_t i = static_cast<uint64_t>(idx[t]);
        const float v = scale * val[t];
        for (uint32_t j = 0; j < p.r; ++j) {
            const uint64_t yb = hash_state(p.a[j], p.b[j], i);
            const uint64_t ys = hash_state(p.as[j], p.bs[j], i);
            atomic_add_noret(S + static_cast<size_t>(j) * p.c + bucket_of<POW2>(yb, col),
                             apply_sign(v, sign_flip_of(ys)));
        }
    }
}

// ---------------------------------------------------------------------------------------
// Alg. 4 update with order-independent sums: every contribution is rounded once to a multiple
// of 2^-F and added as a 64-bit integer, so a table does not depend on how the additions were
// scheduled (a debugging and checkpointing aid; the float kernels above are the product path)
// ---------------------------------------------------------------------------------------
// scale * g * 2^F as an integer, ties to even; the product of two binary32 numbers and a power
// of two is exact in binary64, so the one rounding is the one to an integer.  False (and no
// contribution) when the value is not finite or not below 2^62 in magnitude.
__device__ __forceinline__ bool fixed_of(float g, double scale_2F, long long* q) {
    const double x = static_cast<double>(g) * scale_2F;
    if (!(fabs(x) < 0x1p62)) return false;
    *q = __double2ll_rn(x);
    return true;
}

__device__ __forceinline__ void fixed_add(long long* acc, long long q, bool negative) {
    atomicAdd(reinterpret_cast<unsigned long long*>(acc),
              static_cast<unsigned long long>(negative ? -q : q));
}

// lanes that dropped a coordinate: one atomic per wavefront that saw any
__device__ __forceinline__ void count_dropped(unsigned long long* dropped, unsigned long long mine) {
    if (dropped == nullptr) return;
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(dropped, mine);
}

template <int R, bool POW2>
__global__ void __launch_bounds__(kBlock)
k_fixed_accumulate(KParams p, long long* __restrict__ acc, const float* __restrict__ g, int64_t d,
                   int64_t i0, double scale_2F, unsigned long long* __restrict__ dropped) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    unsigned long long bad = 0;
    if (t < d) {
        RowStates<R> st;
        st.init(p, static_cast<uint64_t>(i0 + t), static_cast<uint64_t>(stride));
        for (; t < d; t += stride) {
            long long q;
            if (fixed_of(g[t], scale_2F, &q)) {
#pragma unroll
                for (int j = 0; j < R; ++j)
                    fixed_add(acc + static_cast<size_t>(j) * p.c + bucket_of<POW2>(st.yb[j], col), q,
                              sign_flip_of(st.ys[j]) != 0u);
            } else {
                ++bad;
            }
            st.advance();
        }
    }
    count_dropped(dropped, bad);
}

template <bool POW2>
__global__ void __launch_bounds__(kBlock)
k_fixed_accumulate_sparse(KParams p, long long* __restrict__ acc, const int64_t* __restrict__ idx,
                          const float* __restrict__ val, int64_t n, double scale_2F,
                          unsigned long long* __restrict__ dropped) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    unsigned long long bad = 0;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride) {
        const uint64_t i = static_cast<uint64_t>(idx[t]);
        long long q;
        if (!fixed_of(val[t], scale_2F, &q)) {
            ++bad;
            continue;
        }
        for (uint32_t j = 0; j < p.r; ++j) {
            const uint64_t yb = hash_state(p.a[j], p.b[j], i);
            const uint64_t ys = hash_state(p.as[j], p.bs[j], i);
            fixed_add(acc + static_cast<size_t>(j) * p.c + bucket_of<POW2>(yb, col), q,
                      sign_flip_of(ys) != 0u);
        }
    }
    count_dropped(dropped, bad);
}

// S = binary32( binary64(acc) * 2^-F * alpha ): the integer to binary64 (exact below 2^53), an
// exact scaling, one multiplication rounded in binary64, one rounding to binary32.
__global__ void __launch_bounds__(kBlock)
k_fixed_to_float(const long long* __restrict__ acc, int64_t n, double inv_2F, double alpha,
                 float* __restrict__ S) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride) {
        const double cell = __ll2double_rn(acc[t]) * inv_2F;
        S[t] = __double2float_rn(cell * alpha);
    }
}

// ---------------------------------------------------------------------------------------
// table-wide elementwise kernels: zero, merge, axpby, momentum
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kBlock) k_fill_zero(float* __restrict__ S, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride)
        S[t] = 0.0f;
}

constexpr int kMaxMerge = 128;   // source tables per launch of the merge kernel

struct MergePtrs {
    const float* src[kMaxMerge];
};

// dst = beta * dst + alpha * (src[0] + src[1] + ...), the sum taken in ascending order in
// binary64 and the result rounded to binary32 once (see k_bundle_merge for why).  Bound by the read of the tables: with one
// 4-byte load of a thread in flight at a time 16 tables of 5 x 2^18 took 24.4 us in a step; 16-byte pieces (VEC: dst and
// every source on 16 bytes) of kMergeAhead tables in flight 20.6, and 14.8 on tables that the memory-side cache holds.
constexpr int kMergeAhead = 8;

template <bool VEC>
__global__ void __launch_bounds__(kBlock)
k_merge(float* __restrict__ dst, float beta, MergePtrs ptrs, int nw, float alpha, int64_t n) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    const double a = static_cast<double>(alpha);
    const int64_t n4 = VEC ? n / 4 : 0;
    for (int64_t t = t0; t < n4; t += stride) {
        double s[4] = {-0.0, -0.0, -0.0, -0.0};        // (the one number that leaves the first table's zeros their sign)
        f4 base = {0.0f, 0.0f, 0.0f, 0.0f};
        if (beta != 0.0f) base = reinterpret_cast<const f4*>(dst)[t];
        auto add = [&](auto count, int w) {
            constexpr int N = decltype(count)::value;
            f4 u[N];
#pragma unroll
            for (int q = 0; q < N; ++q) u[q] = reinterpret_cast<const f4*>(ptrs.src[w + q])[t];
#pragma unroll
            for (int q = 0; q < N; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[e] += static_cast<double>(u[q][e]);
        };
        int w = 0;
        for (; w + kMergeAhead <= nw; w += kMergeAhead) add(std::integral_constant<int, kMergeAhead>{}, w);
        for (; w + 2 <= nw; w += 2) add(std::integral_constant<int, 2>{}, w);
        if (w < nw) add(std::integral_constant<int, 1>{}, w);
        f4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double kept = beta == 0.0f ? 0.0 : static_cast<double>(beta) * static_cast<double>(base[e]);
            o[e] = static_cast<float>(kept + a * s[e]);
        }
        reinterpret_cast<f4*>(dst)[t] = o;
    }
    for (int64_t t = 4 * n4 + t0; t < n; t += stride) {
        double s = static_cast<double>(ptrs.src[0][t]);
#pragma unroll 4
        for (int w = 1; w < nw; ++w) s += static_cast<double>(ptrs.src[w][t]);
        const double base = (beta == 0.0f) ? 0.0 : static_cast<double>(beta) * static_cast<double>(dst[t]);
        dst[t] = static_cast<float>(base + a * s);
    }
}

__global__ void __launch_bounds__(kBlock)
k_axpby(float* __restrict__ y, float a, const float* __restrict__ x, float b, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride) {
        const float by = (b == 0.0f) ? 0.0f : b * y[t];
        y[t] = a * x[t] + by;
    }
}

// cells that are NaN or infinite: exponent bits all ones
__global__ void __launch_bounds__(kBlock)
k_count_nonfinite(const float* __restrict__ S, int64_t n, unsigned long long* __restrict__ count) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    unsigned long long mine = 0;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride)
        mine += (__float_as_uint(S[t]) & 0x7f800000u) == 0x7f800000u ? 1u : 0u;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_down(mine, off, 64);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(count, mine);
}

__global__ void k_clear_count(unsigned long long* count) { *count = 0; }

__global__ void __launch_bounds__(kBlock)
k_momentum(float* __restrict__ Su, float* __restrict__ Sv, const float* __restrict__ St,
           float rho, int64_t n) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride) {
        const float u = rho * Su[t] + St[t];
        Su[t] = u;
        Sv[t] = Sv[t] + u;
    }
}

// ---------------------------------------------------------------------------------------
// sketch_estimate: Alg. 4 estimate
// ---------------------------------------------------------------------------------------
template <int R, bool POW2>
__global__ void __launch_bounds__(kBlock)
k_estimate(KParams p, const float* __restrict__ S, int64_t d, int64_t i0,
           float* __restrict__ est) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    if (t >= d) return;
    RowStates<R> st;
    st.init(p, static_cast<uint64_t>(i0 + t), static_cast<uint64_t>(stride));
    const uint32_t c = p.c;
    for (; t < d; t += stride) {
        float v[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const float cellv = S[static_cast<size_t>(j) * c + bucket_of<POW2>(st.yb[j], col)];
            v[j] = apply_sign(cellv, sign_flip_of(st.ys[j]));
        }
        // (up to 7 rows the sort, which needs no look for a NaN, lets more gathers overlap: 5 x 8193, d = 700 001 16.2 us for 16.9)
        est[t] = R <= 7 ? median_by_sort<R>(v) : median_odd<R>(v);
        st.advance();
    }
}

template <int R, bool POW2>
__global__ void __launch_bounds__(kBlock)
k_estimate_sparse(KParams p, const float* __restrict__ S, const int64_t* __restrict__ idx,
                  int64_t n, float* __restrict__ out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const Columns col = columns_of<POW2>(p.c);
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride) {
        const uint64_t i = static_cast<uint64_t>(idx[t]);
        float v[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const uint64_t yb = hash_state(p.a[j], p.b[j], i);
            const uint64_t ys = hash_state(p.as[j], p.bs[j], i);
            v[j] = apply_sign(S[static_cast<size_t>(j) * p.c + bucket_of<POW2>(yb, col)],
                              sign_flip_of(ys));
        }
        out[t] = median_odd<R>(v);
    }
}

// Error feedback, S -= sketch of the estimates at idx, for one or two tables (blockIdx.y) with the
// same hashes.  All estimates are taken from the table as it is on entry.  Up to kFeedbackSmall
// coordinates one workgroup per table does both halves, a barrier between them, in one launch
// (two tables: four launches of 4 to 5 us before); more are a launch per half.
struct FeedbackTables {
    float* S[2];
    float* val[2];
};
constexpr int kFeedbackBlock = 512;
constexpr int64_t kFeedbackSmall = 4 * kFeedbackBlock;

// threads t0, t0 + stride, ... of a table
template <int R, bool POW2>
__device__ __forceinline__ void feedback_estimates(const KParams& p, const float* S, float* val, const int64_t* __restrict__ idx,
                                                   int64_t n, int64_t t0, int64_t stride) {
    const Columns col = columns_of<POW2>(p.c);
    for (int64_t t = t0; t < n; t += stride) val[t] = estimate_at<R, POW2>(p, col, S, static_cast<uint64_t>(idx[t]));
}

template <int R, bool POW2>
__device__ __forceinline__ void feedback_subtract(const KParams& p, float* S, const float* val, const int64_t* __restrict__ idx,
                                                  int64_t n, int64_t t0, int64_t stride) {
    const Columns col = columns_of<POW2>(p.c);
    for (int64_t t = t0; t < n; t += stride) {
        const uint64_t i = static_cast<uint64_t>(idx[t]);
        const float v = -val[t];
#pragma unroll
        for (int j = 0; j < R; ++j)
            atomic_add_noret(S + static_cast<size_t>(j) * p.c + bucket_of<POW2>(hash_state(p.a[j], p.b[j], i), col),
                             apply_sign(v, sign_flip_of(hash_state(p.as[j], p.bs[j], i))));
    }
}

// PHASES: 1 the estimates, 2 the subtraction, 3 both (one workgroup per table)
template <int R, bool POW2, int PHASES>
__global__ void __launch_bounds__(kFeedbackBlock)
k_feedback(KParams p, FeedbackTables tab, const int64_t* __restrict__ idx, int64_t n) {
    float* S = tab.S[blockIdx.y];
    float* val = tab.val[blockIdx.y];
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kFeedbackBlock;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kFeedbackBlock + threadIdx.x;
    if (PHASES & 1) feedback_estimates<R, POW2>(p, S, val, idx, n, t0, stride);
    if (PHASES == 3) __syncthreads();
    if (PHASES & 2) feedback_subtract<R, POW2>(p, S, val, idx, n, t0, stride);
}

// ---------------------------------------------------------------------------------------
// gather_exact: second round
// ---------------------------------------------------------------------------------------
// A thread's loads are random lines of memory, W of them: what bounds it is how many are in flight.  One after the
// other (32 workers a launch, 256 threads a workgroup) k = 10 000 of 32 workers, d = 25 M, took 24.5 us; kGatherAhead
// at once, in workgroups of one wavefront, which find more CUs, 11.4.  The sum is taken in the same order.
constexpr int kMaxGather = 256;      // vectors a launch: 2 KB of kernel arguments
constexpr int kGatherBlock = 64;
constexpr int kGatherAhead = 16;
struct GatherPtrs {
    const float* vec[kMaxGather];
};

// s plus the values at i, in ascending order of the vectors
__device__ __forceinline__ float gather_add(float s, const GatherPtrs& ptrs, int nw, int64_t i) {
    int w = 0;
    for (; w + kGatherAhead <= nw; w += kGatherAhead) {
        float u[kGatherAhead];
#pragma unroll
        for (int q = 0; q < kGatherAhead; ++q) u[q] = __builtin_nontemporal_load(ptrs.vec[w + q] + i);
#pragma unroll
        for (int q = 0; q < kGatherAhead; ++q) s += u[q];
    }
    // (what is left, four at a time: the common numbers of workers are multiples of four)
    for (; w + 4 <= nw; w += 4) {
        float u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) u[q] = __builtin_nontemporal_load(ptrs.vec[w + q] + i);
#pragma unroll
        for (int q = 0; q < 4; ++q) s += u[q];
    }
    for (; w < nw; ++w) s += __builtin_nontemporal_load(ptrs.vec[w] + i);
    return s;
}

__global__ void __launch_bounds__(kGatherBlock)
k_gather(GatherPtrs ptrs, int nw, const int64_t* __restrict__ idx, int64_t k, float alpha,
         float* __restrict__ out, int first_chunk, int last_chunk) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kGatherBlock;
    for (int64_t n = static_cast<int64_t>(blockIdx.x) * kGatherBlock + threadIdx.x; n < k; n += stride) {
        const float s = gather_add(first_chunk ? 0.0f : out[n], ptrs, nw, idx[n]);
        out[n] = last_chunk ? alpha * s : s;
    }
}

// The second round beside the feedback of a pair of tables: both start from idx and neither reads what the other writes,
// and a launch of either is one chain of dependent loads.  SMALL (up to kFeedbackSmall coordinates): workgroups 0 and 1 are
// the whole feedback of a table each, the others gather, 64 coordinates by their first wavefront.  Otherwise workgroups of
// one wavefront in three equal parts, the gather and the tables' estimates; the subtraction is k_feedback's.
// us, one launch more / this: 7 x 40, k = 2, 4 vectors 8.1 / 6.3; 5 x 2^15, k = 1000, 4 20.9 / 18.7; 5 x 2^17, k = 5000, 8 15.9 /
// 11.4; 5 x 2^18, k = 10 000, 32 23.7 / 18.7.
template <int R, bool POW2, bool SMALL>
__global__ void __launch_bounds__(SMALL ? kFeedbackBlock : kGatherBlock)
k_gather_feedback(KParams p, FeedbackTables tab, GatherPtrs ptrs, int nw, const int64_t* __restrict__ idx, int64_t k,
                  float alpha, float* __restrict__ out) {
    const unsigned part = SMALL ? 1 : gridDim.x / 3;                     // workgroups of a table
    const unsigned first = 2 * part;                                     // that gathers
    if (blockIdx.x >= first) {
        if (SMALL && threadIdx.x >= kGatherBlock) return;
        const int64_t stride = static_cast<int64_t>(gridDim.x - first) * kGatherBlock;
        for (int64_t n = static_cast<int64_t>(blockIdx.x - first) * kGatherBlock + threadIdx.x; n < k; n += stride)
            out[n] = alpha * gather_add(0.0f, ptrs, nw, idx[n]);
        return;
    }
    const unsigned which = blockIdx.x / part;
    constexpr int block = SMALL ? kFeedbackBlock : kGatherBlock;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x - which * part) * block + threadIdx.x;
    const int64_t stride = static_cast<int64_t>(part) * block;
    feedback_estimates<R, POW2>(p, tab.S[which], tab.val[which], idx, k, t0, stride);
    if constexpr (SMALL) {
        __syncthreads();
        feedback_subtract<R, POW2>(p, tab.S[which], tab.val[which], idx, k, t0, stride);
    }
}
static_assert(sizeof(KParams) + sizeof(FeedbackTables) + sizeof(GatherPtrs) + 128 <= 4096, "kernel arguments");

// out = alpha * (sum of W vectors), added up in binary64 and rounded once.  Folded workers are
// summed before they are sketched: the sketch is linear, W d floats are then read once
// instead of r times.  Bound by that read; 4 vectors' 16-byte pieces are in flight per thread.
// More vectors than one launch takes: later launches add their share, scaled like the first's (so that
// nothing overflows that alpha times the whole sum does not).
constexpr int kMaxSum = 256;
struct SumPtrs {
    const float* x[kMaxSum];
};

template <bool VEC>
__global__ void __launch_bounds__(kBlock)
k_vectors_sum(SumPtrs ptrs, int nw, int64_t d, float alpha, float* __restrict__ out, int first_launch) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    int64_t done = 0;
    if (VEC) {
        const int64_t n4 = d / 4;
        for (int64_t t = t0; t < n4; t += stride) {
            double s[4] = {0.0, 0.0, 0.0, 0.0};
            auto add = [&](const f4& u) {
                s[0] += static_cast<double>(u.x); s[1] += static_cast<double>(u.y);
                s[2] += static_cast<double>(u.z); s[3] += static_cast<double>(u.w);
            };
            f4 base = {0.0f, 0.0f, 0.0f, 0.0f};
            if (!first_launch) base = reinterpret_cast<const f4*>(out)[t];
            int w = 0;
            for (; w + 4 <= nw; w += 4) {
                f4 u[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    u[q] = __builtin_nontemporal_load(reinterpret_cast<const f4*>(ptrs.x[w + q]) + t);
#pragma unroll
                for (int q = 0; q < 4; ++q) add(u[q]);
            }
            for (; w < nw; ++w) add(__builtin_nontemporal_load(reinterpret_cast<const f4*>(ptrs.x[w]) + t));
            const double a = static_cast<double>(alpha);
            f4 o;
            o.x = static_cast<float>(base.x + a * s[0]); o.y = static_cast<float>(base.y + a * s[1]);
            o.z = static_cast<float>(base.z + a * s[2]); o.w = static_cast<float>(base.w + a * s[3]);
            reinterpret_cast<f4*>(out)[t] = o;
        }
        done = n4 * 4;
    }
    for (int64_t t = done + t0; t < d; t += stride) {
        const double base = first_launch ? 0.0 : static_cast<double>(out[t]);
        double s = 0.0;
#pragma unroll 4
        for (int w = 0; w < nw; ++w) s += static_cast<double>(ptrs.x[w][t]);
        out[t] = static_cast<float>(base + static_cast<double>(alpha) * s);
    }
}

template <int FMT>
__global__ void __launch_bounds__(kBlock)
k_quantize16(const float* __restrict__ x, int64_t n, uint16_t* __restrict__ out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride)
        out[t] = to_16<FMT>(x[t]);
}

template <int FMT>
__global__ void __launch_bounds__(kBlock)
k_dequantize16(const uint16_t* __restrict__ q, int64_t n, float* __restrict__ out) {
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; t < n; t += stride)
        out[t] = from_16<FMT>(q[t]);
}

// The momentum and error-accumulation steps of Alg. 3 with dense per-worker state:
// u = rho u + g (one fused multiply-add), v = v + u.  blockIdx.y = worker; 20 bytes of
// traffic per coordinate, 16-byte accesses when the three vectors are 16-byte aligned.
// Bound: memory, read and write in turn (a copy reaches 5.0 TB/s).
// u and g, which nothing reads before the next step, go past the caches where u, v and g of all workers are more than the
// memory-side cache (256 MB) keeps beside a step's tables, estimates and scratch: what it holds at the end is then v, which the
// update reads next, from its end.  Where it keeps them, the next step finds u there.  us of this pass / of the pass with update
// and query, through the caches and past them: 22 MB 9.6 / 60.7 and 10.3 / 61.6; 42 MB 14.2 / 60.5 and 16.3 / 62.5; 112 MB 31.1 /
// 108.0 and 32.6 / 109.5; 141 MB 38.4 / 106.2 and 40.4 / 108.2; 161 MB 42.5 / 154.4 and 42.5 / 153.3; 199 MB 51.6 / 166.0 and 51.3 /
// 162.2; 245 MB 75.0 / 265.6 and 64.7 / 253.3; 877 MB 262 / 486 and 220 / 433; 11 M, 8 workers (1.06 GB) 342 / 759 and 289 /
// 701; v past them too: the same.
constexpr double kDensePastBytes = 1.5e8;
inline bool dense_goes_past(int W, int64_t d) { return 12.0 * W * static_cast<double>(d) > kDensePastBytes; }
struct DensePtrs {
    float* u[kMaxBatch];
    float* v[kMaxBatch];
    const float* g[kMaxBatch];
};

// PAST: u and g go past the caches (dense_goes_past).
template <bool VEC, bool PAST>
__global__ void __launch_bounds__(kBlock)
k_dense_momentum(DensePtrs ptrs, int64_t d, float rho) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    auto load = [](const f4* p) { return PAST ? __builtin_nontemporal_load(p) : *p; };
    float* __restrict__ u = ptrs.u[blockIdx.y];
    float* __restrict__ v = ptrs.v[blockIdx.y];
    const float* __restrict__ g = ptrs.g[blockIdx.y];
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    int64_t done = 0;
    if (VEC) {
        const int64_t n4 = d / 4;
        for (int64_t t = t0; t < n4; t += stride) {
            f4 uu = load(reinterpret_cast<f4*>(u) + t), vv = reinterpret_cast<f4*>(v)[t];
            const f4 gg = load(reinterpret_cast<const f4*>(g) + t);
            uu.x = __fmaf_rn(rho, uu.x, gg.x); uu.y = __fmaf_rn(rho, uu.y, gg.y);
            uu.z = __fmaf_rn(rho, uu.z, gg.z); uu.w = __fmaf_rn(rho, uu.w, gg.w);
            vv.x += uu.x; vv.y += uu.y; vv.z += uu.z; vv.w += uu.w;
            if (PAST) __builtin_nontemporal_store(uu, reinterpret_cast<f4*>(u) + t);
            else reinterpret_cast<f4*>(u)[t] = uu;
            reinterpret_cast<f4*>(v)[t] = vv;
        }
        done = n4 * 4;
    }
    for (int64_t t = done + t0; t < d; t += stride) {
        const float un = __fmaf_rn(rho, u[t], g[t]);
        u[t] = un;
        v[t] += un;
    }
}

// Measurement aid: a plain streaming read of the workers' vectors, the access that every
// HBM-bound kernel here is compared with.  blockIdx.y = worker; 16-byte loads, two in flight
// per thread, when the vectors are 16-byte aligned; the sum of everything read is added to
// out[0] (one atomic per workgroup, a few thousand per launch) so that the loads cannot be
// dropped.
struct ProbePtrs {
    const float* x[kMaxBatch];
};

template <bool VEC>
__global__ void __launch_bounds__(kBlock)
k_probe_stream_read(ProbePtrs ptrs, int64_t d, float* __restrict__ out) {
    const float* __restrict__ x = ptrs.x[blockIdx.y];
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    const int64_t t0 = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
    float acc = 0.0f;
    int64_t done = 0;
    if (VEC) {
        const float4* __restrict__ x4 = reinterpret_cast<const float4*>(x);
        const int64_t n4 = d / 4;
        int64_t t = t0;
        for (; t + stride < n4; t += 2 * stride) {
            const float4 p = x4[t], q = x4[t + stride];
            acc += ((p.x + p.y) + (p.z + p.w)) + ((q.x + q.y) + (q.z + q.w));
        }
        if (t < n4) {
            const float4 p = x4[t];
            acc += (p.x + p.y) + (p.z + p.w);
        }
        done = n4 * 4;
    }
    for (int64_t t = done + t0; t < d; t += stride) acc += x[t];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    __shared__ float part[kBlock / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float s = 0.0f;
#pragma unroll
        for (int q = 0; q < kBlock / 64; ++q) s += part[q];
        atomic_add_noret(out, s);                       // one per workgroup
    }
}

// Alg. 3 last step: u, v <- 0 on the coordinates of the update, for every worker
__global__ void __launch_bounds__(kBlock)
k_dense_mask(DensePtrs ptrs, const int64_t* __restrict__ idx, int64_t k) {
    float* __restrict__ u = ptrs.u[blockIdx.y];
    float* __restrict__ v = ptrs.v[blockIdx.y];
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock;
    for (int64_t n = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x; n < k; n += stride) {
        const int64_t i = idx[n];
        u[i] = 0.0f;
        v[i] = 0.0f;
    }
}

}  // namespace cs

using namespace cs;

// =========================================================================================
// C ABI
// =========================================================================================
extern "C" int cs_hash_debug(const cs_params* p, const int64_t* idx, int64_t n,
                             uint32_t* bucket, int8_t* sign, void* stream) {
    if (!params_ok(p) || n < 0) return CS_EINVAL;
    if (n == 0) return CS_OK;
    if (!idx || !bucket || !sign) return CS_EINVAL;
    if (p->c_pow2)
        k_hash_list<true><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(kparams(p), idx, n, bucket, sign);
    else
        k_hash_list<false><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(kparams(p), idx, n, bucket, sign);
    return launch_status();
}

extern "C" int cs_hash_debug_range(const cs_params* p, int64_t i0, int64_t n,
                                   uint32_t* bucket, int8_t* sign, void* stream) {
    if (!params_ok(p) || n < 0 || i0 < 0 || i0 > (int64_t)kP61 - n) return CS_EINVAL;
    if (n == 0) return CS_OK;
    if (!bucket || !sign) return CS_EINVAL;
    if (lattice_applies(p, n)) return launch_hash_range_lattice(p, i0, n, bucket, sign, as_stream(stream));
    // a small grid on purpose: every thread takes several strided steps
    const unsigned grid = grid_for(n, kBlock * 8, 64);
#define CALL(R_, P2_) \
    k_hash_range<R_, P2_><<<grid, kBlock, 0, as_stream(stream)>>>(kparams(p), i0, n, bucket, sign)
    CS_DISPATCH_R(p, CALL);
#undef CALL
    return launch_status();
}

extern "C" int cs_sketch_zero(const cs_params* p, float* S, void* stream) {
    if (!params_ok(p) || !S) return CS_EINVAL;
    const int64_t n = static_cast<int64_t>(p->r) * p->c;
    k_fill_zero<<<grid_for(n), kBlock, 0, as_stream(stream)>>>(S, n);
    return launch_status();
}

static int accumulate_direct(const cs_params* p, const BatchPtrs& ptrs, int nw, int64_t d,
                             int64_t i0, float scale, void* stream) {
    // at least ~8 coordinates per thread so the per-thread hash set-up is amortised
    const unsigned grid = grid_for(d, kBlock * 8, 256 * 8);
#define CALL(R_, P2_)                                                                      \
    k_accumulate<R_, P2_><<<grid, kBlock, 0, as_stream(stream)>>>(kparams(p), ptrs, nw, d, i0, scale)
    CS_DISPATCH_R(p, CALL);
#undef CALL
    return launch_status();
}

static int accumulate_launch(const cs_params* p, const BatchPtrs& ptrs, int nw, int64_t d,
                             int64_t i0, float scale, void* stream) {
    if (lattice_applies(p, d))
        return launch_accumulate_lattice(p, ptrs, nw, d, i0, scale, as_stream(stream));
    return accumulate_direct(p, ptrs, nw, d, i0, scale, stream);
}

extern "C" int cs_sketch_accumulate(const cs_params* p, float* S, const float* g, int64_t d,
                                    int64_t i0, float scale, void* stream) {
    if (!params_ok(p) || d < 0 || i0 < 0 || i0 > (int64_t)kP61 - d) return CS_EINVAL;
    if (d == 0) return CS_OK;
    if (!S || !g) return CS_EINVAL;
    // The lattice form is the better one for short vectors: its time is about 5 us plus that of r d
    // coordinates at 250 to 400 G/s, while a list's chains of visits and their requests take 35 to 45 us from
    // r d = 5 million on and 10 to 30 below.  Lists / lattice, us: 31 / 19 (5 x 8192, d = 1.1 M), 45 / 40
    // (3 x 32 768, 3.9 M), 61 / 72 (5 x 65 536, 4.0 M), 48 / 65 (5 x 16 384, 3.5 M), 466 / 1162 (5 x 2^20, 73 M).
    // Of 67 shapes with r d of 7 to 18 million the lattice is ahead in 36 of the 38 below 12 million (by up to
    // 1.5 times, behind by 4 % at most), the two take turns up to 15, and lists are ahead from there.
    constexpr int64_t kOneFrom = 15000000;
    const bool short_vector = lattice_applies(p, d) && static_cast<int64_t>(p->r) * d < kOneFrom;
    if (!short_vector && one_applies(p, d)) return launch_accumulate_one(p, S, 1, g, d, i0, scale, as_stream(stream));
    BatchPtrs ptrs{};
    ptrs.S[0] = S;
    ptrs.g[0] = g;
    return accumulate_launch(p, ptrs, 1, d, i0, scale, stream);
}

static int64_t bundle_groups(int32_t W) { return (static_cast<int64_t>(W) + CS_BUNDLE_GROUP - 1) / CS_BUNDLE_GROUP; }

static bool bundle_ok(const cs_params* p, int32_t W) {
    return params_ok(p) && W >= 1 &&
           static_cast<uint64_t>(p->r) * p->c * static_cast<uint64_t>(bundle_groups(W)) * CS_BUNDLE_GROUP < (1ull << 40);
}

extern "C" int cs_bundle_floats(const cs_params* p, int32_t W, int64_t* n) {
    if (!bundle_ok(p, W) || !n) return CS_EINVAL;
    *n = static_cast<int64_t>(p->r) * p->c * bundle_groups(W) * CS_BUNDLE_GROUP;
    return CS_OK;
}

extern "C" int cs_bundle_zero(const cs_params* p, float* T, int32_t W, void* stream) {
    if (!bundle_ok(p, W) || !T) return CS_EINVAL;
    return launch_bundle_zero(T, static_cast<int64_t>(p->r) * p->c * bundle_groups(W) * CS_BUNDLE_GROUP,
                              as_stream(stream));
}

extern "C" int cs_sketch_accumulate_bundle(const cs_params* p, float* T, int32_t W,
                                           const float* const* g_w, int64_t d, int64_t i0,
                                           float scale, void* stream) {
    if (!bundle_ok(p, W) || d < 0 || i0 < 0 || i0 > (int64_t)kP61 - d) return CS_EINVAL;
    if (!T || !g_w) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!g_w[w] && d > 0) return CS_EINVAL;
    if (d == 0) return CS_OK;
    if (walk_applies(p, d)) return launch_accumulate_walk(p, T, W, g_w, d, i0, scale, false, as_stream(stream));
    if (anyc_update_applies(p, d, W)) return launch_accumulate_anyc(p, T, W, g_w, d, i0, scale, false, as_stream(stream));
    // any other sketch: a slot of 8 lanes per coordinate, one lane per worker of a group
    const size_t group_floats = static_cast<size_t>(p->r) * p->c * CS_BUNDLE_GROUP;
    constexpr int kSlots = kBlock / CS_BUNDLE_GROUP;
    for (int w0 = 0; w0 < W; w0 += kMaxBatch) {
        const int nw = (W - w0 < kMaxBatch) ? (W - w0) : kMaxBatch;
        GroupedVectors vec{};
        for (int w = 0; w < nw; ++w) vec.g[w] = g_w[w0 + w];
        float* T0 = T + (w0 / CS_BUNDLE_GROUP) * group_floats;
        // at least ~8 coordinates per lane so the per-lane hash set-up is amortised
        const int groups = (nw + CS_BUNDLE_GROUP - 1) / CS_BUNDLE_GROUP;
        const dim3 grid(crowded_cells(p, d, groups) ? grid_for(d, kSlots * 8, 256 * 8) : grid_of_hashes(d, kSlots, groups),
                        static_cast<unsigned>(groups));
        if (lds_table_applies(p, d)) {
            const dim3 lgrid(grid_for(d, kSlots * 8, 512), grid.y);
            const size_t lds = static_cast<size_t>(p->r) * p->c * CS_BUNDLE_GROUP * sizeof(float);
#define CALL(R_, P2_)                                                                      \
    k_accumulate_cells_lds<R_, P2_><<<lgrid, kBlock, lds, as_stream(stream)>>>(kparams(p), vec, nw, \
                                                                               T0, d, i0, scale)
            CS_DISPATCH_R(p, CALL);
#undef CALL
        } else {
#define CALL(R_, P2_)                                                                      \
    k_accumulate_cells<R_, P2_><<<grid, kBlock, 0, as_stream(stream)>>>(kparams(p), vec, nw, T0, d, \
                                                                        i0, scale)
            CS_DISPATCH_R(p, CALL);
#undef CALL
        }
        if (launch_status() != CS_OK) return CS_EHIP;
    }
    return CS_OK;
}

extern "C" int cs_sketch_accumulate_sum(const cs_params* p, float* S, int32_t W,
                                        const float* const* g_w, int64_t d, int64_t i0,
                                        float scale, void* stream) {
    if (!params_ok(p) || W < 1 || d < 0 || i0 < 0 || i0 > (int64_t)kP61 - d) return CS_EINVAL;
    if (!S || !g_w) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!g_w[w] && d > 0) return CS_EINVAL;
    if (d == 0) return CS_OK;
    if (W == 1) return cs_sketch_accumulate(p, S, g_w[0], d, i0, scale, stream);
    // along visit lists the 8 workers of a group are added up in registers and a cell receives
    // one request per group; everything else adds worker by worker into the same table
    if (all_rows_listed(p, d)) return launch_accumulate_walk(p, S, W, g_w, d, i0, scale, true, as_stream(stream));
    if (anyc_update_applies(p, d, W)) return launch_accumulate_anyc(p, S, W, g_w, d, i0, scale, true, as_stream(stream));
    for (int w0 = 0; w0 < W; w0 += kMaxBatch) {
        const int nw = (W - w0 < kMaxBatch) ? (W - w0) : kMaxBatch;
        BatchPtrs ptrs{};
        for (int w = 0; w < nw; ++w) {
            ptrs.S[w] = S;
            ptrs.g[w] = g_w[w0 + w];
        }
        const int rc = accumulate_launch(p, ptrs, nw, d, i0, scale, stream);
        if (rc != CS_OK) return rc;
    }
    return CS_OK;
}

extern "C" int cs_bundle_update_launches(const cs_params* p, int32_t W, int64_t d, int32_t* n) {
    if (!bundle_ok(p, W) || d < 0 || !n) return CS_EINVAL;
    *n = 0;
    if (d == 0) return CS_OK;
    if (walk_applies(p, d)) return launch_accumulate_walk(p, nullptr, W, nullptr, d, 0, 1.0f, false, nullptr, n);
    if (anyc_update_applies(p, d, W)) return launch_accumulate_anyc(p, nullptr, W, nullptr, d, 0, 1.0f, false, nullptr, n);
    *n = static_cast<int32_t>((static_cast<int64_t>(W) + kMaxBatch - 1) / kMaxBatch);
    return CS_OK;
}

extern "C" int cs_bundle_merge(const cs_params* p, float* dst, float beta, const float* T,
                               int32_t W, float alpha, void* stream) {
    if (!bundle_ok(p, W) || !dst || !T) return CS_EINVAL;
    if (reinterpret_cast<uintptr_t>(T) % 16 != 0) return CS_EINVAL;
    return launch_bundle_merge(dst, beta, T, static_cast<int>(bundle_groups(W)), alpha,
                               static_cast<int64_t>(p->r) * p->c, as_stream(stream));
}

extern "C" int cs_bundle_merge_momentum(const cs_params* p, float* S_t, float* S_u, float* S_v, const float* T,
                                        int32_t W, float alpha, float rho, void* stream) {
    if (!bundle_ok(p, W) || !S_t || !S_u || !S_v || !T) return CS_EINVAL;
    if (reinterpret_cast<uintptr_t>(T) % 16 != 0) return CS_EINVAL;
    return launch_bundle_merge_momentum(S_t, S_u, S_v, T, static_cast<int>(bundle_groups(W)), alpha, rho,
                                        static_cast<int64_t>(p->r) * p->c, as_stream(stream));
}

extern "C" int cs_quantize16(const float* x, int64_t n, uint16_t* out, int32_t fmt, void* stream) {
    if (n < 0 || (fmt != CS_FMT_BF16 && fmt != CS_FMT_F16)) return CS_EINVAL;
    if (n == 0) return CS_OK;
    if (!x || !out) return CS_EINVAL;
    if (fmt == CS_FMT_BF16) k_quantize16<0><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(x, n, out);
    else k_quantize16<1><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(x, n, out);
    return launch_status();
}

extern "C" int cs_dequantize16(const uint16_t* q, int64_t n, float* out, int32_t fmt, void* stream) {
    if (n < 0 || (fmt != CS_FMT_BF16 && fmt != CS_FMT_F16)) return CS_EINVAL;
    if (n == 0) return CS_OK;
    if (!q || !out) return CS_EINVAL;
    if (fmt == CS_FMT_BF16) k_dequantize16<0><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(q, n, out);
    else k_dequantize16<1><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(q, n, out);
    return launch_status();
}

extern "C" int cs_bundle_merge16(const cs_params* p, float* dst, float beta, const uint16_t* T16,
                                 int32_t W, float alpha, int32_t fmt, void* stream) {
    if (!bundle_ok(p, W) || !dst || !T16) return CS_EINVAL;
    if (fmt != CS_FMT_BF16 && fmt != CS_FMT_F16) return CS_EINVAL;
    if (reinterpret_cast<uintptr_t>(T16) % 16 != 0) return CS_EINVAL;
    return launch_bundle_merge16(dst, beta, T16, static_cast<int>(bundle_groups(W)), alpha,
                                 static_cast<int64_t>(p->r) * p->c, fmt, as_stream(stream));
}

extern "C" int cs_sketch_accumulate_batch(const cs_params* p, float* const* S_w,
                                          const float* const* g_w, int32_t W, int64_t d,
                                          int64_t i0, float scale, void* stream) {
    if (!params_ok(p) || W < 1 || d < 0 || i0 < 0 || i0 > (int64_t)kP61 - d) return CS_EINVAL;
    if (!S_w || !g_w) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!S_w[w] || (!g_w[w] && d > 0)) return CS_EINVAL;
    if (d == 0) return CS_OK;
    for (int w0 = 0; w0 < W; w0 += kMaxBatch) {
        const int nw = (W - w0 < kMaxBatch) ? (W - w0) : kMaxBatch;
        BatchPtrs ptrs{};
        for (int w = 0; w < nw; ++w) {
            ptrs.S[w] = S_w[w0 + w];
            ptrs.g[w] = g_w[w0 + w];
        }
        const int rc = accumulate_launch(p, ptrs, nw, d, i0, scale, stream);
        if (rc != CS_OK) return rc;
    }
    return CS_OK;
}

extern "C" int cs_sketch_accumulate_sparse(const cs_params* p, float* S, const int64_t* idx,
                                           const float* val, int64_t n, float scale,
                                           void* stream) {
    if (!params_ok(p) || n < 0) return CS_EINVAL;
    if (n == 0) return CS_OK;
    if (!S || !idx || !val) return CS_EINVAL;
    if (p->c_pow2)
        k_accumulate_sparse<true><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(kparams(p), S, idx, val, n, scale);
    else
        k_accumulate_sparse<false><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(kparams(p), S, idx, val, n, scale);
    return launch_status();
}

static bool fixed_args_ok(const cs_params* p, const void* acc, int32_t frac_bits) {
    return params_ok(p) && acc && frac_bits >= 0 && frac_bits <= CS_FIXED_MAX_FRAC_BITS;
}

extern "C" int cs_fixed_accumulate(const cs_params* p, int64_t* acc, const float* g, int64_t d,
                                   int64_t i0, float scale, int32_t frac_bits, int64_t* dropped,
                                   void* stream) {
    if (!fixed_args_ok(p, acc, frac_bits) || d < 0 || i0 < 0 || (d > 0 && !g)) return CS_EINVAL;
    if (d == 0) return CS_OK;
    const double scale_2F = ldexp(static_cast<double>(scale), frac_bits);
    auto* a = reinterpret_cast<long long*>(acc);
    auto* bad = reinterpret_cast<unsigned long long*>(dropped);
#define CS_CALL(R_, P2_) \
    k_fixed_accumulate<R_, P2_><<<grid_for(d), kBlock, 0, as_stream(stream)>>>(kparams(p), a, g, d, i0, scale_2F, bad)
    CS_DISPATCH_R(p, CS_CALL);
#undef CS_CALL
    return launch_status();
}

extern "C" int cs_fixed_accumulate_sparse(const cs_params* p, int64_t* acc, const int64_t* idx,
                                          const float* val, int64_t n, float scale,
                                          int32_t frac_bits, int64_t* dropped, void* stream) {
    if (!fixed_args_ok(p, acc, frac_bits) || n < 0 || (n > 0 && (!idx || !val))) return CS_EINVAL;
    if (n == 0) return CS_OK;
    const double scale_2F = ldexp(static_cast<double>(scale), frac_bits);
    auto* a = reinterpret_cast<long long*>(acc);
    auto* bad = reinterpret_cast<unsigned long long*>(dropped);
    if (p->c_pow2)
        k_fixed_accumulate_sparse<true><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(kparams(p), a, idx, val, n, scale_2F, bad);
    else
        k_fixed_accumulate_sparse<false><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(kparams(p), a, idx, val, n, scale_2F, bad);
    return launch_status();
}

extern "C" int cs_fixed_to_float(const cs_params* p, const int64_t* acc, int32_t frac_bits,
                                 float alpha, float* S, void* stream) {
    if (!fixed_args_ok(p, acc, frac_bits) || !S) return CS_EINVAL;
    const int64_t n = static_cast<int64_t>(p->r) * p->c;
    k_fixed_to_float<<<grid_for(n), kBlock, 0, as_stream(stream)>>>(
        reinterpret_cast<const long long*>(acc), n, ldexp(1.0, -frac_bits),
        static_cast<double>(alpha), S);
    return launch_status();
}

extern "C" int cs_sketch_merge(const cs_params* p, float* dst, float beta,
                               const float* const* src, int32_t W, float alpha, void* stream) {
    if (!params_ok(p) || !dst || !src || W < 1) return CS_EINVAL;
    bool vec = reinterpret_cast<uintptr_t>(dst) % 16 == 0;
    for (int w = 0; w < W; ++w) {
        if (!src[w] || (W > 1 && src[w] == dst)) return CS_EINVAL;
        vec = vec && reinterpret_cast<uintptr_t>(src[w]) % 16 == 0;
    }
    const int64_t n = static_cast<int64_t>(p->r) * p->c;
    // More sources than one launch takes: later launches add their share on top (beta = 1).
    for (int w0 = 0; w0 < W; w0 += kMaxMerge) {
        const int nw = (W - w0 < kMaxMerge) ? (W - w0) : kMaxMerge;
        MergePtrs ptrs{};
        for (int w = 0; w < nw; ++w) ptrs.src[w] = src[w0 + w];
        const float b = w0 == 0 ? beta : 1.0f;
        if (vec) k_merge<true><<<grid_for((n + 3) / 4), kBlock, 0, as_stream(stream)>>>(dst, b, ptrs, nw, alpha, n);
        else k_merge<false><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(dst, b, ptrs, nw, alpha, n);
        if (launch_status() != CS_OK) return CS_EHIP;
    }
    return CS_OK;
}

extern "C" int cs_sketch_axpby(const cs_params* p, float* y, float a, const float* x, float b,
                               void* stream) {
    if (!params_ok(p) || !y || !x) return CS_EINVAL;
    const int64_t n = static_cast<int64_t>(p->r) * p->c;
    k_axpby<<<grid_for(n), kBlock, 0, as_stream(stream)>>>(y, a, x, b, n);
    return launch_status();
}

extern "C" int cs_sketch_count_nonfinite(const cs_params* p, const float* S, int64_t* count,
                                         void* stream) {
    if (!params_ok(p) || !S || !count || reinterpret_cast<uintptr_t>(count) % 8 != 0) return CS_EINVAL;
    const int64_t n = static_cast<int64_t>(p->r) * p->c;
    unsigned long long* out = reinterpret_cast<unsigned long long*>(count);
    k_clear_count<<<1, 1, 0, as_stream(stream)>>>(out);
    k_count_nonfinite<<<grid_for(n), kBlock, 0, as_stream(stream)>>>(S, n, out);
    return launch_status();
}

extern "C" int cs_sketch_momentum(const cs_params* p, float* S_u, float* S_v, const float* S_t,
                                  float rho, void* stream) {
    if (!params_ok(p) || !S_u || !S_v || !S_t) return CS_EINVAL;
    const int64_t n = static_cast<int64_t>(p->r) * p->c;
    k_momentum<<<grid_for(n), kBlock, 0, as_stream(stream)>>>(S_u, S_v, S_t, rho, n);
    return launch_status();
}

extern "C" int cs_estimate_workspace_bytes(const cs_params* p, int64_t d, size_t* bytes) {
    if (!params_ok(p) || d < 0 || !bytes) return CS_EINVAL;
    // the stride-aligned path stores the r signed cells of every coordinate before the median
    *bytes = (lattice_applies(p, d) || anyc_query_needs_scratch(p, d))
                 ? sizeof(float) * static_cast<size_t>(p->r) * static_cast<size_t>(d) : 0;
    return CS_OK;
}

extern "C" int cs_estimate_scratch_bytes(const cs_params* p, int64_t d, size_t* bytes) {
    const int rc = cs_estimate_workspace_bytes(p, d, bytes);
    if (rc == CS_OK && *bytes == 0 && anyc_visits_serve_query(p, d))
        *bytes = sizeof(float) * static_cast<size_t>(p->r) * static_cast<size_t>(d);
    return rc;
}

static int estimate_all(const cs_params* p, const float* S, int64_t d, int64_t i0, float* est,
                        uint64_t* hist, void* rows_ws, size_t ws_bytes, void* stream) {
    if (lattice_applies(p, d)) {
        const size_t need = sizeof(float) * static_cast<size_t>(p->r) * static_cast<size_t>(d);
        if (!rows_ws || reinterpret_cast<uintptr_t>(rows_ws) % 4 != 0) return CS_EINVAL;
        if (ws_bytes < need) return CS_EWORKSPACE;
        return launch_estimate_lattice(p, S, d, i0, est, static_cast<float*>(rows_ws), hist, as_stream(stream));
    }
    // the kernels below do not count what they write: one more read of est
    auto counted = [&](int rc) -> int {
        if (rc != CS_OK || !hist) return rc;
        rc = launch_magnitude_hist_zero(hist, as_stream(stream));
        return rc != CS_OK ? rc : launch_magnitude_hist(est, d, hist, as_stream(stream));
    };
    if (anyc_visits_serve_query(p, d)) {
        const size_t need = sizeof(float) * static_cast<size_t>(p->r) * static_cast<size_t>(d);
        const bool room = rows_ws && reinterpret_cast<uintptr_t>(rows_ws) % 4 == 0 && ws_bytes >= need;
        if (room) return launch_estimate_anyc(p, S, d, i0, est, static_cast<float*>(rows_ws), hist, as_stream(stream));
        // (shorter vectors go without scratch as well)
        if (anyc_query_needs_scratch(p, d))
            return !rows_ws || reinterpret_cast<uintptr_t>(rows_ws) % 4 != 0 ? CS_EINVAL : CS_EWORKSPACE;
    }
    const bool in_l1 = p->r <= 5 && static_cast<uint64_t>(p->r) * p->c <= (1u << 14);
    const unsigned grid = grid_of_hashes(d, kBlock, 1, in_l1 ? 96 : 128);
#define CALL(R_, P2_) \
    k_estimate<R_, P2_><<<grid, kBlock, 0, as_stream(stream)>>>(kparams(p), S, d, i0, est)
    CS_DISPATCH_R(p, CALL);
#undef CALL
    return counted(launch_status());
}

extern "C" int cs_sketch_estimate(const cs_params* p, const float* S, int64_t d, int64_t i0,
                                  float* est, uint64_t* hist_or_null, void* rows_ws,
                                  size_t ws_bytes, void* stream) {
    if (!params_ok(p) || d < 0 || i0 < 0 || i0 > (int64_t)kP61 - d) return CS_EINVAL;
    if (hist_or_null && reinterpret_cast<uintptr_t>(hist_or_null) % 8 != 0) return CS_EINVAL;
    if (d > 0 && (!S || !est)) return CS_EINVAL;
    if (d == 0) return hist_or_null ? launch_magnitude_hist_zero(hist_or_null, as_stream(stream)) : CS_OK;
    return estimate_all(p, S, d, i0, est, hist_or_null, rows_ws, ws_bytes, stream);
}

extern "C" int cs_sketch_estimate_sparse(const cs_params* p, const float* S, const int64_t* idx,
                                         int64_t n, float* out, void* stream) {
    if (!params_ok(p) || n < 0) return CS_EINVAL;
    if (n == 0) return CS_OK;
    if (!S || !idx || !out) return CS_EINVAL;
#define CALL(R_, P2_) \
    k_estimate_sparse<R_, P2_><<<grid_for(n), kBlock, 0, as_stream(stream)>>>(kparams(p), S, idx, n, out)
    CS_DISPATCH_R(p, CALL);
#undef CALL
    return launch_status();
}

extern "C" int cs_gather_exact(const float* const* vec, int32_t W, const int64_t* idx, int64_t k,
                               float alpha, float* out, void* stream) {
    if (!vec || W < 1 || k < 0) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!vec[w]) return CS_EINVAL;
    if (k == 0) return CS_OK;
    if (!idx || !out) return CS_EINVAL;
    for (int w0 = 0; w0 < W; w0 += kMaxGather) {
        const int nw = (W - w0 < kMaxGather) ? (W - w0) : kMaxGather;
        GatherPtrs ptrs{};
        for (int w = 0; w < nw; ++w) ptrs.vec[w] = vec[w0 + w];
        const unsigned grid = grid_for(k, kGatherBlock, 256 * 32);
        k_gather<<<grid, kGatherBlock, 0, as_stream(stream)>>>(ptrs, nw, idx, k, alpha, out, w0 == 0, w0 + nw == W);
        if (launch_status() != CS_OK) return CS_EHIP;
    }
    return CS_OK;
}

extern "C" int cs_vectors_sum(const float* const* x_w, int32_t W, int64_t d, float alpha, float* out,
                              void* stream) {
    if (!x_w || W < 1 || d < 0 || !out) return CS_EINVAL;
    const uintptr_t o = reinterpret_cast<uintptr_t>(out), bytes = sizeof(float) * static_cast<uintptr_t>(d);
    bool vec = o % 16 == 0;
    for (int w = 0; w < W; ++w) {
        const uintptr_t x = reinterpret_cast<uintptr_t>(x_w[w]);
        if (!x_w[w] || x_w[w] == out || (x < o ? o - x : x - o) < bytes) return CS_EINVAL;
        vec = vec && reinterpret_cast<uintptr_t>(x_w[w]) % 16 == 0;
    }
    if (d == 0) return CS_OK;
    for (int w0 = 0; w0 < W; w0 += kMaxSum) {
        const int nw = (W - w0 < kMaxSum) ? (W - w0) : kMaxSum;
        SumPtrs ptrs{};
        for (int w = 0; w < nw; ++w) ptrs.x[w] = x_w[w0 + w];
        const unsigned grid = grid_for(vec ? (d + 3) / 4 : d, kBlock, 256 * 32);
        if (vec) k_vectors_sum<true><<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, nw, d, alpha, out, w0 == 0);
        else k_vectors_sum<false><<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, nw, d, alpha, out, w0 == 0);
        if (launch_status() != CS_OK) return CS_EHIP;
    }
    return CS_OK;
}

extern "C" int cs_dense_momentum(float* const* u_w, float* const* v_w, const float* const* g_w,
                                 int32_t W, int64_t d, float rho, void* stream) {
    if (!u_w || !v_w || !g_w || W < 1 || d < 0) return CS_EINVAL;
    bool vec = true;
    for (int w = 0; w < W; ++w) {
        if (!u_w[w] || !v_w[w] || !g_w[w]) return CS_EINVAL;
        vec = vec && (reinterpret_cast<uintptr_t>(u_w[w]) | reinterpret_cast<uintptr_t>(v_w[w]) |
                      reinterpret_cast<uintptr_t>(g_w[w])) % 16 == 0;
    }
    if (d == 0) return CS_OK;
    const bool past = dense_goes_past(W, d);
    for (int w0 = 0; w0 < W; w0 += kMaxBatch) {
        const int nw = (W - w0 < kMaxBatch) ? (W - w0) : kMaxBatch;
        DensePtrs ptrs{};
        for (int w = 0; w < nw; ++w) {
            ptrs.u[w] = u_w[w0 + w];
            ptrs.v[w] = v_w[w0 + w];
            ptrs.g[w] = g_w[w0 + w];
        }
        const dim3 grid(grid_for(vec ? (d + 3) / 4 : d, kBlock, 2048), static_cast<unsigned>(nw));
        if (vec && past) k_dense_momentum<true, true><<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, d, rho);
        else if (vec) k_dense_momentum<true, false><<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, d, rho);
        else k_dense_momentum<false, false><<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, d, rho);
        if (launch_status() != CS_OK) return CS_EHIP;
    }
    return CS_OK;
}

extern "C" int cs_probe_stream_read(const float* const* x_w, int32_t W, int64_t d, float* out,
                                    void* stream) {
    if (!x_w || W < 1 || d < 0 || !out) return CS_EINVAL;
    bool vec = true;
    for (int w = 0; w < W; ++w) {
        if (!x_w[w]) return CS_EINVAL;
        vec = vec && reinterpret_cast<uintptr_t>(x_w[w]) % 16 == 0;
    }
    if (d == 0) return CS_OK;
    for (int w0 = 0; w0 < W; w0 += kMaxBatch) {
        const int nw = (W - w0 < kMaxBatch) ? (W - w0) : kMaxBatch;
        ProbePtrs ptrs{};
        for (int w = 0; w < nw; ++w) ptrs.x[w] = x_w[w0 + w];
        // about 4096 workgroups per launch, shared out among the workers
        const dim3 grid(grid_for(vec ? (d + 3) / 4 : d, kBlock * 2, (4096 + nw - 1) / nw),
                        static_cast<unsigned>(nw));
        if (vec) k_probe_stream_read<true><<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, d, out);
        else k_probe_stream_read<false><<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, d, out);
        if (launch_status() != CS_OK) return CS_EHIP;
    }
    return CS_OK;
}

extern "C" int cs_dense_mask(float* const* u_w, float* const* v_w, int32_t W, const int64_t* idx,
                             int64_t k, void* stream) {
    if (!u_w || !v_w || W < 1 || k < 0) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!u_w[w] || !v_w[w]) return CS_EINVAL;
    if (k == 0) return CS_OK;
    if (!idx) return CS_EINVAL;
    for (int w0 = 0; w0 < W; w0 += kMaxBatch) {
        const int nw = (W - w0 < kMaxBatch) ? (W - w0) : kMaxBatch;
        DensePtrs ptrs{};
        for (int w = 0; w < nw; ++w) {
            ptrs.u[w] = u_w[w0 + w];
            ptrs.v[w] = v_w[w0 + w];
        }
        const dim3 grid(grid_for(k), static_cast<unsigned>(nw));
        k_dense_mask<<<grid, kBlock, 0, as_stream(stream)>>>(ptrs, idx, k);
        if (launch_status() != CS_OK) return CS_EHIP;
    }
    return CS_OK;
}

static int feedback_tables(const cs_params* p, const FeedbackTables& tab, unsigned ntab, const int64_t* idx,
                           int64_t k, void* stream) {
    if (k <= kFeedbackSmall) {
        const dim3 grid(1, ntab);
#define CALL(R_, P2_) k_feedback<R_, P2_, 3><<<grid, kFeedbackBlock, 0, as_stream(stream)>>>(kparams(p), tab, idx, k)
        CS_DISPATCH_R(p, CALL);
#undef CALL
        return launch_status();
    }
    const dim3 grid(grid_for(k, kFeedbackBlock), ntab);
#define CALL(R_, P2_)                                                                                            \
    do {                                                                                                         \
        k_feedback<R_, P2_, 1><<<grid, kFeedbackBlock, 0, as_stream(stream)>>>(kparams(p), tab, idx, k);          \
        k_feedback<R_, P2_, 2><<<grid, kFeedbackBlock, 0, as_stream(stream)>>>(kparams(p), tab, idx, k);          \
    } while (0)
    CS_DISPATCH_R(p, CALL);
#undef CALL
    return launch_status();
}

extern "C" int cs_sketch_feedback(const cs_params* p, float* S, const int64_t* idx, int64_t k,
                                  float* val, void* stream) {
    if (!params_ok(p) || k < 0) return CS_EINVAL;
    if (k == 0) return CS_OK;
    if (!S || !idx || !val) return CS_EINVAL;
    return feedback_tables(p, FeedbackTables{{S, S}, {val, val}}, 1, idx, k, stream);
}

extern "C" int cs_sketch_feedback_pair(const cs_params* p, float* S_v, float* S_u, const int64_t* idx, int64_t k,
                                       float* val_v, float* val_u, void* stream) {
    if (!params_ok(p) || k < 0) return CS_EINVAL;
    if (k == 0) return CS_OK;
    if (!S_v || !S_u || !idx || !val_v || !val_u || S_v == S_u || val_v == val_u) return CS_EINVAL;
    return feedback_tables(p, FeedbackTables{{S_v, S_u}, {val_v, val_u}}, 2, idx, k, stream);
}

extern "C" int cs_gather_feedback(const cs_params* p, const float* const* vec, int32_t W, const int64_t* idx, int64_t k,
                                  float alpha, float* out, float* S_v, float* S_u, float* val_v, float* val_u, void* stream) {
    if (!params_ok(p) || !vec || W < 1 || k < 0) return CS_EINVAL;
    for (int w = 0; w < W; ++w)
        if (!vec[w]) return CS_EINVAL;
    if (k == 0) return CS_OK;
    if (!idx || !out || !S_v || !S_u || !val_v || !val_u || S_v == S_u) return CS_EINVAL;
    if (val_v == val_u || out == val_v || out == val_u) return CS_EINVAL;
    if (W > kMaxGather) {
        const int rc = cs_gather_exact(vec, W, idx, k, alpha, out, stream);
        return rc != CS_OK ? rc : cs_sketch_feedback_pair(p, S_v, S_u, idx, k, val_v, val_u, stream);
    }
    const FeedbackTables tab{{S_v, S_u}, {val_v, val_u}};
    GatherPtrs ptrs{};
    for (int w = 0; w < W; ++w) ptrs.vec[w] = vec[w];
    const unsigned part = grid_for(k, kGatherBlock, 256 * 8);
    if (k <= kFeedbackSmall) {
#define CALL(R_, P2_)                                                                                               \
    k_gather_feedback<R_, P2_, true><<<2 + part, kFeedbackBlock, 0, as_stream(stream)>>>(kparams(p), tab, ptrs, W, idx, k, \
                                                                                        alpha, out)
        CS_DISPATCH_R(p, CALL);
#undef CALL
        return launch_status();
    }
    const dim3 grid(grid_for(k, kFeedbackBlock), 2);
#define CALL(R_, P2_)                                                                                                   \
    do {                                                                                                                \
        k_gather_feedback<R_, P2_, false><<<3 * part, kGatherBlock, 0, as_stream(stream)>>>(kparams(p), tab, ptrs, W, idx, k, \
                                                                                           alpha, out);                \
        k_feedback<R_, P2_, 2><<<grid, kFeedbackBlock, 0, as_stream(stream)>>>(kparams(p), tab, idx, k);                 \
    } while (0)
    CS_DISPATCH_R(p, CALL);
#undef CALL
    return launch_status();
}
