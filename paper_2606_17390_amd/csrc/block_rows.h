// block_rows.h -- the product of a node-block matrix (rows 3I+a of a node
// consecutive, one list of node columns per node) with a vector, as the
// Krylov solve and the multigrid take it, in two forms with the same
// epilogues.
//
// staged, for large levels, bound by HBM (1.09 GB of float values per pass at
// 10^6 nodes): a workgroup takes the rows of 32 consecutive nodes (16 for FP64
// values), whose values are one contiguous piece of the matrix, copies them to
// LDS by fully coalesced loads, fetches the columns and vector entries
// meanwhile, and then sums from LDS with 8 (16) lanes per node.  Lanes that
// load the 3x3 blocks of their rows straight from memory, 12 bytes every 12
// bytes from three rows, reached 4.5 TB/s however they were pipelined, split
// or mapped to XCDs (254 us per product; 222 us with one round per workgroup);
// the staged form reaches 6.0 TB/s (190 us), a plain read of the same bytes
// 6.7.  It wants one chunk per workgroup: 240 us on a grid of 2048 that
// strides.
//
// direct, for small levels, bound by latency: 32 lanes per node, lane k the
// blocks k, k + 32, ..., so that more workgroups share the few rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fem {

constexpr int kRowLanes = 32;

// v + (v of the lane with bit 0 / 1 / 2 / 3 of its index flipped), by DPP:
// the lanes of a group that the earlier steps have made equal may be taken in
// any order, so quad permutations and mirrors do.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
    return v + __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
// Sum over the 32 lanes of a group, the same bits in every lane (each step
// adds the same two values in either order; the result is that of an xor
// butterfly).
__device__ __forceinline__ double sum32(double v) {
    v = dpp_add<0xB1>(v);   // quad_perm 1 0 3 2
    v = dpp_add<0x4E>(v);   // quad_perm 2 3 0 1
    v = dpp_add<0x141>(v);  // row_half_mirror
    v = dpp_add<0x140>(v);  // row_mirror
    return v + __shfl_xor(v, 16, 32);
}

// Sum over the 8 or 16 lanes of a group, the same bits in every lane.
template <int LN>
__device__ __forceinline__ double sum_lanes(double v) {
    static_assert(LN == 8 || LN == 16, "8 or 16 lanes");
    v = dpp_add<0xB1>(v);
    v = dpp_add<0x4E>(v);
    v = dpp_add<0x141>(v);
    if (LN == 16) v = dpp_add<0x140>(v);
    return v;
}

// Epilogues: E::Data E::load(I, l) fetches what node I's epilogue needs
// (l = min(lane, 2)); E::finish(I, lane, data, s) gets the node's three sums
// in every lane of its group, once per node.

template <typename RV>
constexpr int kStagedNodes = sizeof(RV) == 4 ? 32 : 16;  // 31 KB of LDS

// One 256-thread workgroup's chunks of y = A x, staged (kernels that call it
// hold themselves to four waves per SIMD).  A chunk larger than
// the buffer (more than 27 blocks per node on average) is read in place.
template <typename RV, typename E>
__device__ __forceinline__ void block_rows_staged(int32_t n, const int32_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ ncol, const RV* __restrict__ val,
                                                  const double* __restrict__ x, E& epi) {
    constexpr int NC = kStagedNodes<RV>, LN = 256 / NC, kCap = NC * 243, U = (kCap + 255) / 256, NB = 32 / LN;
    __shared__ RV sv[kCap];
    const int tid = (int)threadIdx.x, g = tid / LN, l = tid % LN;
    for (int64_t base = (int64_t)blockIdx.x * NC; base < n; base += (int64_t)gridDim.x * NC) {
        const int64_t last = min(base + NC, (int64_t)n);
        const int32_t b0 = row_ptr[3 * base], cnt = row_ptr[3 * last] - b0;
        const bool fits = cnt > 0 && cnt <= kCap;
        const int64_t I = min(base + g, last - 1);
        const int32_t bs = row_ptr[3 * I], len = row_ptr[3 * I + 1] - bs, deg = len / 3;
        RV st[U];
        if (fits) {
            const char* __restrict__ p = reinterpret_cast<const char*>(val + b0);
            int t = tid;
            asm volatile("" : "+v"(t));  // keep the 31 offsets from living across chunks
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t at = (uint32_t)min(u * 256 + t, cnt - 1) * (uint32_t)sizeof(RV);
                st[u] = *reinterpret_cast<const RV*>(p + at);
            }
        }
        // the lane's first NB blocks (past the row's end: its last one, not used)
        int32_t J[NB];
        double X[NB][3];
#pragma unroll
        for (int u = 0; u < NB; ++u) {
            J[u] = ncol[bs / 9 + max(min(l + u * LN, deg - 1), 0)];
            J[u] = deg > 0 ? J[u] : 0;
        }
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int c = 0; c < 3; ++c) X[u][c] = x[3 * (int64_t)J[u] + c];
        const typename E::Data data = epi.load(I, min(l, 2));
        __syncthreads();  // the previous chunk has been read
        if (fits) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u * 256 + tid < kCap) sv[u * 256 + tid] = st[u];
        }
        __syncthreads();
        double s[3] = {0.0, 0.0, 0.0};
        auto add = [&](const RV* p, double x0, double x1, double x2) {
#pragma unroll
            for (int a = 0; a < 3; ++a)
                s[a] += (double)p[a * len] * x0 + (double)p[a * len + 1] * x1 + (double)p[a * len + 2] * x2;
        };
        if (fits) {
            const RV* p = sv + (bs - b0);
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (l + u * LN < deg) add(p + 3 * (l + u * LN), X[u][0], X[u][1], X[u][2]);
            for (int32_t k = l + 32; k < deg; k += LN) {
                const int64_t j = 3 * (int64_t)ncol[bs / 9 + k];
                add(p + 3 * k, x[j], x[j + 1], x[j + 2]);
            }
        } else {
            const RV* __restrict__ p = val + bs;
            for (int32_t k = l; k < deg; k += LN) {
                const int64_t j = 3 * (int64_t)ncol[bs / 9 + k];
                add(p + 3 * k, x[j], x[j + 1], x[j + 2]);
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) s[a] = sum_lanes<LN>(s[a]);
        if (base + g < n) epi.finish(I, l, data, s);
    }
}

// The same, direct.
template <typename RV, typename E>
__device__ __forceinline__ void block_rows_direct(int32_t n, const int32_t* __restrict__ row_ptr,
                                                  const int32_t* __restrict__ ncol, const RV* __restrict__ val,
                                                  const double* __restrict__ x, E& epi) {
    const int g = (int)(threadIdx.x >> 5), l = (int)(threadIdx.x & (kRowLanes - 1));
    for (int64_t base = (int64_t)blockIdx.x * 8; base < n; base += (int64_t)gridDim.x * 8) {
        const int64_t I = base + g;
        if (I >= n) return;
        const int32_t bs = row_ptr[3 * I], len = row_ptr[3 * I + 1] - bs, deg = len / 3;
        const typename E::Data data = epi.load(I, min(l, 2));
        double s[3] = {0.0, 0.0, 0.0};
        for (int32_t k = l; k < deg; k += kRowLanes) {
            const int64_t J = ncol[bs / 9 + k];
            const double x0 = x[3 * J], x1 = x[3 * J + 1], x2 = x[3 * J + 2];
            const RV* __restrict__ v = val + bs + 3 * k;
#pragma unroll
            for (int a = 0; a < 3; ++a)
                s[a] += (double)v[(int64_t)a * len] * x0 + (double)v[(int64_t)a * len + 1] * x1 +
                        (double)v[(int64_t)a * len + 2] * x2;
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) s[a] = sum32(s[a]);
        epi.finish(I, l, data, s);
    }
}

// Nodes above which the staged form is taken: below, its chunks are too few
// to fill the chip and the direct form's 8 nodes per workgroup finish sooner.
constexpr int32_t kStagedMin = 32768;

// Workgroups of a product over n nodes, at most cap.
inline unsigned row_blocks(int64_t n, bool staged, int nodes, unsigned cap) {
    const int64_t nb = staged ? (n + nodes - 1) / nodes : (n + 7) / 8;
    return (unsigned)(nb < (int64_t)cap ? nb : (int64_t)cap);
}

template <typename RV, bool STAGED, typename E>
__device__ __forceinline__ void block_rows(int32_t n, const int32_t* __restrict__ row_ptr,
                                           const int32_t* __restrict__ ncol, const RV* __restrict__ val,
                                           const double* __restrict__ x, E& epi) {
    if constexpr (STAGED) block_rows_staged<RV>(n, row_ptr, ncol, val, x, epi);
    else block_rows_direct<RV>(n, row_ptr, ncol, val, x, epi);
}

}  // namespace fem
