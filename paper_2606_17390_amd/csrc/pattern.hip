// pattern.hip -- CSR pattern of the global tangent from the connectivity
// (App. E, Alg. E1: the pattern is fixed for a mesh, so it is built once and
// the element matrices are later scattered straight into its value array).
//
// Steps, all on the device:
//   1. node -> element incidence: an atomic counter per node gives each entry
//      of conn its place among the node's entries, a scan the node's start;
//   2. per node, the sorted unique list of nodes sharing an element (<= 64):
//      a wave sorts the 64 candidates of up to 8 incident elements across its
//      lanes and keeps the first of equal ones;
//   3. row_ptr from a scan of the neighbour counts (rows of one node have
//      equal length 3*deg);
//   4. col_idx rows, elem_rank (position of node J in node I's list) and the
//      incidence in ascending order, written by the same wave.
// The call that fills col_idx takes row_ptr from the caller and does step 1
// and the sort of step 2 only.
#include <hip/hip_runtime.h>

#include "fem_internal.h"

namespace fem {
namespace {

constexpr int kMaxNbr = 64;
constexpr int kScanThreads = 256;
constexpr int kScanItems = 8;
constexpr int kScanChunk = kScanThreads * kScanItems;

constexpr int kCountPer = 4;  // conn entries per thread of the incidence kernels

enum { ERR_RANGE = 1, ERR_ORPHAN = 2, ERR_DEGREE = 4 };

// Bound by the atomics, which are done at the memory side (3.9 M of them take
// 87 us): a workgroup counts its 4096 entries in an LDS hash table first, and
// adds once per distinct node (a third of the entries or fewer where elements
// next to each other follow each other).  pos keeps an entry's place among its node's
// entries, so that fill_incidence needs no atomics.  517,000 nodes, 3.9 M
// entries: 87 us, and 128 us for an atomic fill; 55 us (69 us with 2048
// entries, 88 us with 1024) and 26 us now.
constexpr int kCountThreads = 1024;
constexpr int kCountSlots = 8192;  // 2^13, at most half full

__global__ __launch_bounds__(kCountThreads) void count_incidence(const int32_t* __restrict__ conn,
                                                                 int64_t n_entries, int32_t n_nodes,
                                                                 int32_t* __restrict__ cnt,
                                                                 int32_t* __restrict__ pos,
                                                                 int32_t* __restrict__ err) {
    __shared__ int32_t skey[kCountSlots];
    __shared__ int32_t scnt[kCountSlots];
    const int64_t base = (int64_t)blockIdx.x * (kCountThreads * kCountPer) + threadIdx.x;
    int32_t n[kCountPer], place[kCountPer];
    int slot[kCountPer];
#pragma unroll
    for (int u = 0; u < kCountPer; ++u) {
        const int64_t i = base + (int64_t)kCountThreads * u;
        n[u] = i < n_entries ? conn[i] : -2;
    }
    for (int t = (int)threadIdx.x; t < kCountSlots; t += kCountThreads) {
        skey[t] = -1;
        scnt[t] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCountPer; ++u) {
        place[u] = 0;
        slot[u] = -1;
        if (n[u] == -2 && base + (int64_t)kCountThreads * u >= n_entries) continue;
        if (n[u] < 0 || n[u] >= n_nodes) {
            atomicOr(err, ERR_RANGE);
            continue;
        }
        int h = (int)(((uint32_t)n[u] * 2654435761u) >> 19);
        while (true) {
            const int32_t was = atomicCAS(&skey[h], -1, n[u]);
            if (was == -1 || was == n[u]) break;
            h = (h + 1) & (kCountSlots - 1);
        }
        slot[u] = h;
        place[u] = atomicAdd(&scnt[h], 1);
    }
    __syncthreads();
    for (int t = (int)threadIdx.x; t < kCountSlots; t += kCountThreads)
        if (skey[t] >= 0) scnt[t] = atomicAdd(&cnt[skey[t]], scnt[t]);  // now the first place of this workgroup
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kCountPer; ++u)
        if (slot[u] >= 0) pos[base + (int64_t)kCountThreads * u] = scnt[slot[u]] + place[u];
}

// Workgroups of an XCD take one contiguous eighth of conn: the entries of
// elements next to each other, which share nodes, meet in one L2.
__global__ __launch_bounds__(256) void fill_incidence(const int32_t* __restrict__ conn, int64_t n_entries,
                                                      int64_t n_chunk, int32_t n_nodes,
                                                      const int64_t* __restrict__ inc_ptr,
                                                      const int32_t* __restrict__ pos, int32_t* __restrict__ inc) {
    const int64_t base = ((int64_t)(blockIdx.x & 7) * n_chunk + (blockIdx.x >> 3)) * (256 * kCountPer) + threadIdx.x;
#pragma unroll
    for (int u = 0; u < kCountPer; ++u) {
        const int64_t i = base + 256 * u;
        if (i >= n_entries) continue;
        const int32_t n = conn[i];
        if (n < 0 || n >= n_nodes) continue;
        inc[inc_ptr[n] + pos[i]] = (int32_t)i;  // conn entry 8e + local index
    }
}

// Sorted unique neighbour list of node n (n included).  Returns the count or
// -1 if it exceeds kMaxNbr.
__device__ int node_neighbours(int32_t n, const int32_t* __restrict__ conn, const int64_t* __restrict__ inc_ptr,
                               const int32_t* __restrict__ inc, int32_t* nb) {
    int cnt = 0;
    for (int64_t k = inc_ptr[n]; k < inc_ptr[n + 1]; ++k) {
        const int64_t e = inc[k] >> 3;
        for (int j = 0; j < 8; ++j) {
            const int32_t v = conn[e * 8 + j];
            // insertion into the sorted list
            int pos = cnt;
            while (pos > 0 && nb[pos - 1] > v) --pos;
            if (pos > 0 && nb[pos - 1] == v) continue;
            if (cnt == kMaxNbr) return -1;
            for (int t = cnt; t > pos; --t) nb[t] = nb[t - 1];
            nb[pos] = v;
            ++cnt;
        }
    }
    return cnt;
}

// ---- kNodes nodes per wave, one after the other (a node with more than 8
// incident elements takes the serial node_neighbours in lane 0)

constexpr int kPatWaves = 4;  // waves per workgroup
constexpr int kNodes = 8;     // nodes per wave

template <int CTRL>
__device__ inline uint32_t dpp(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xf, 0xf, true);
}
// the value of lane ^ M
template <int M>
__device__ inline uint32_t lane_xor(uint32_t x, int lane) {
    if constexpr (M == 1) return dpp<0xB1>(x);        // quad_perm 1 0 3 2
    else if constexpr (M == 2) return dpp<0x4E>(x);   // quad_perm 2 3 0 1
    else if constexpr (M == 3) return dpp<0x1B>(x);   // quad_perm 3 2 1 0
    else if constexpr (M == 7) return dpp<0x141>(x);  // row_half_mirror
    else if constexpr (M == 15) return dpp<0x140>(x); // row_mirror
    else if constexpr (M == 8) return dpp<0x128>(x);  // row_ror:8
    else if constexpr (M < 7) return dpp<0x141>(lane_xor<7 ^ M>(x, lane));
    else if constexpr (M < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)x, (M << 10) | 0x1f);
    else return (uint32_t)__builtin_amdgcn_ds_bpermute((lane ^ M) << 2, (int)x);
}
// min where bound is 0, max where it is ~0: the median of the three
__device__ inline uint32_t min_or_max(uint32_t x, uint32_t y, uint32_t bound) {
    const uint32_t lo = x < y ? x : y, hi = x < y ? y : x;
    const uint32_t m = hi < bound ? hi : bound;
    return lo > m ? lo : m;
}
template <int J>
__device__ inline uint32_t merge_down(uint32_t x, const uint32_t (&bound)[6], int lane) {
    if constexpr (J > 0) {
        x = min_or_max(x, lane_xor<J>(x, lane), bound[__builtin_ctz(J)]);
        return merge_down<J / 2>(x, bound, lane);
    } else {
        return x;
    }
}
template <int K>
__device__ inline uint32_t merge_up(uint32_t x, const uint32_t (&bound)[6], int lane) {
    if constexpr (K <= 64) {
        x = min_or_max(x, lane_xor<K - 1>(x, lane), bound[__builtin_ctz(K) - 1]);
        return merge_up<2 * K>(merge_down<K / 4>(x, bound, lane), bound, lane);
    } else {
        return x;
    }
}

// FILL false: neighbour counts of kNodes nodes.  FILL true: column indices of
// the nodes' rows, the elem_rank entries of every (element, local index) pair
// that is one of the nodes, and (out != NULL) their incidence in ascending
// order.
//
// Bound by vector instructions: the bitonic sort of one 32-bit node number per
// lane takes 21 exchanges of two instructions each (a DPP move and a median of
// three; mirrored first steps, so that all merges ascend and 18 of the 21
// partners are DPP patterns).  A lane finds its candidate's place by a binary
// search of the sorted list in LDS.  The loads of the kNodes nodes are in
// flight together, three dependent loads per wave and not per node, and an
// XCD's workgroups take one contiguous eighth of the nodes, whose conn rows and
// elem_rank lines then stay in one L2.  517,000 nodes: counts 250 us and fill
// 307 us + 51 us (incidence by a thread per node) with a sort of 64-bit
// (node, lane) pairs by LDS permutes, one node per wave; 55 us and 179 us now
// (0.50 GB written; 88 us without the columns, 140 us without elem_rank).
template <bool FILL>
__global__ __launch_bounds__(64 * kPatWaves) void node_pass(
    int32_t n_nodes, int64_t n_chunk, const int32_t* __restrict__ conn, const int64_t* __restrict__ inc_ptr,
    const int32_t* __restrict__ inc, int32_t* __restrict__ deg_out, int32_t* __restrict__ err,
    const int32_t* __restrict__ row_ptr, int32_t* __restrict__ col_idx, uint8_t* __restrict__ rank,
    int32_t* __restrict__ out_ptr, int32_t* __restrict__ out) {
    __shared__ int32_t snb[kPatWaves][kMaxNbr];
    __shared__ int32_t scol[kPatWaves][3 * kMaxNbr];
    __shared__ uint32_t scand[kPatWaves][kNodes * 64];
    const int w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    const int64_t n0 =
        (((int64_t)(blockIdx.x & 7) * n_chunk + (blockIdx.x >> 3)) * kPatWaves + w) * kNodes;
    if (n0 >= n_nodes) return;  // the whole wave; no workgroup barrier below
    // lane (m, q): the q-th incident entry of node n0 + m
    const int m = lane >> 3, q = lane & 7;
    int64_t k0 = 0;
    int32_t cnt = 0, row0 = 0, entry = INT32_MAX;
    if (n0 + m < n_nodes) {
        k0 = inc_ptr[n0 + m];
        cnt = (int32_t)(inc_ptr[n0 + m + 1] - k0);
        if constexpr (FILL) row0 = row_ptr[3 * (n0 + m)];
    }
    if (q < cnt) entry = inc[k0 + q];
    const int nn = (int)(n_nodes - n0 < kNodes ? n_nodes - n0 : kNodes);

    // lane (q, j) = (m, q): node j of the q-th incident element, for each node
    uint32_t cand[kNodes];
#pragma unroll
    for (int t = 0; t < kNodes; ++t) {
        const int32_t e = __builtin_amdgcn_ds_bpermute((8 * t + m) << 2, entry);
        cand[t] = ~0u;
        if (e != INT32_MAX) cand[t] = (uint32_t)conn[(int64_t)(e & ~7) + q];
    }
#pragma unroll
    for (int t = 0; t < kNodes; ++t) scand[w][64 * t + lane] = cand[t];
    uint32_t bound[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) bound[t] = (lane >> t) & 1 ? ~0u : 0u;

    if constexpr (FILL) {
        if (out) {
            if (n0 + m < n_nodes && q == 0) out_ptr[n0 + m] = (int32_t)k0;
            if (n0 + nn == n_nodes && lane == 0) out_ptr[n_nodes] = (int32_t)inc_ptr[n_nodes];
            const uint32_t x = (uint32_t)entry;
            const int place = (lane_xor<1>(x, lane) < x) + (lane_xor<2>(x, lane) < x) + (lane_xor<3>(x, lane) < x) +
                              (lane_xor<4>(x, lane) < x) + (lane_xor<5>(x, lane) < x) + (lane_xor<6>(x, lane) < x) +
                              (lane_xor<7>(x, lane) < x);
            if (cnt <= 8) {
                if (q < cnt) out[k0 + place] = entry;
            } else if (q == 0) {
                for (int64_t k = k0; k < k0 + cnt; ++k) {
                    const int32_t v = inc[k];
                    int64_t p = k;
                    while (p > k0 && out[p - 1] > v) {
                        out[p] = out[p - 1];
                        --p;
                    }
                    out[p] = v;
                }
            }
        }
    }

    // the three rows of node n0 + t: 9 deg columns in a row
    auto write_columns = [&](int t, int deg) {
        int32_t* row = col_idx + __builtin_amdgcn_readlane(row0, 8 * t);
        const int len = 3 * deg;
        for (int b = 0; b < 3 * len; b += 256) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int u = b + 64 * k + lane;
                if (u < 3 * len) row[u] = scol[w][u - (u >= len ? len : 0) - (u >= 2 * len ? len : 0)];
            }
        }
        wave_sync();
    };

    int32_t my_deg = 0;  // lane t: of node n0 + t
    uint32_t more = 0;   // the nodes with more than 8 elements
    // no load in this loop: one would make the wave wait for the stores of the node before
#pragma unroll 1
    for (int t = 0; t < nn; ++t) {
        if (__builtin_amdgcn_readlane(cnt, 8 * t) > 8) {
            more |= 1u << t;
            continue;
        }
        const uint32_t own = scand[w][64 * t + lane];
        const uint32_t x = merge_up<2>(own, bound, lane);
        const uint32_t prev = dpp<0x138>(x);  // wave_shr:1
        const bool first = x != ~0u && (lane == 0 || prev != x);
        const uint64_t mask = __ballot(first);
        const int deg = __popcll(mask);
        if (lane == t) my_deg = deg;
        if constexpr (FILL) {
            const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (lane >= deg) snb[w][lane] = INT32_MAX;
            if (first) {
                snb[w][below] = (int32_t)x;
#pragma unroll
                for (int b = 0; b < 3; ++b) scol[w][3 * below + b] = 3 * (int32_t)x + b;
            }
            wave_sync();
            const int32_t e = __builtin_amdgcn_ds_bpermute((8 * t + m) << 2, entry);
            if (e != INT32_MAX) {
                const int32_t v = (int32_t)own;
                int p = 0;
#pragma unroll
                for (int step = 32; step > 0; step >>= 1)
                    if (snb[w][p + step - 1] < v) p += step;
                rank[(int64_t)e * 8 + q] = (uint8_t)p;
            }
            write_columns(t, deg);
        }
    }
    while (more) {
        const int t = __builtin_ctz(more);
        more &= more - 1;
        const int64_t k0t = inc_ptr[n0 + t], k1t = inc_ptr[n0 + t + 1];
        int s = 0;
        if (lane == 0) s = node_neighbours((int32_t)(n0 + t), conn, inc_ptr, inc, snb[w]);
        wave_sync();
        const int deg = __builtin_amdgcn_readfirstlane(s);
        if (lane == t) my_deg = deg;
        if constexpr (FILL) {
            if (deg <= 0) continue;  // reported by the counting call
            if (lane < deg)
                for (int b = 0; b < 3; ++b) scol[w][3 * lane + b] = 3 * snb[w][lane] + b;
            wave_sync();
            for (int64_t k = k0t + m; k < k1t; k += 8) {
                const int32_t e = inc[k];
                const int32_t v = conn[(int64_t)(e & ~7) + q];
                int lo = 0, hi = deg - 1;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (snb[w][mid] < v) lo = mid + 1;
                    else hi = mid;
                }
                rank[(int64_t)e * 8 + q] = (uint8_t)lo;
            }
            write_columns(t, deg);
        }
    }
    if constexpr (!FILL) {
        if (lane < nn) {
            if (my_deg < 0) {
                atomicOr(err, ERR_DEGREE);
                my_deg = 0;
            } else if (my_deg == 0) {
                atomicOr(err, ERR_ORPHAN);
            }
            deg_out[n0 + lane] = my_deg;
        }
    }
}

__global__ void node_columns(int32_t n_nodes, const int32_t* __restrict__ conn, const int64_t* __restrict__ inc_ptr,
                             const int32_t* __restrict__ inc, const int32_t* __restrict__ row_ptr,
                             int32_t* __restrict__ col_idx) {
    int32_t n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= n_nodes) return;
    int32_t nb[kMaxNbr];
    const int c = node_neighbours(n, conn, inc_ptr, inc, nb);
    if (c <= 0) return;
    for (int a = 0; a < 3; ++a) {
        int32_t* row = col_idx + row_ptr[3 * n + a];
        for (int k = 0; k < c; ++k) {
            row[3 * k + 0] = 3 * nb[k] + 0;
            row[3 * k + 1] = 3 * nb[k] + 1;
            row[3 * k + 2] = 3 * nb[k] + 2;
        }
    }
}

// node -> conn-entry incidence in ascending order (deterministic assembly),
// for a caller that asks for no elem_rank
__global__ void write_incidence(int32_t n_nodes, const int64_t* __restrict__ inc_ptr,
                                const int32_t* __restrict__ inc, int32_t* __restrict__ out_ptr,
                                int32_t* __restrict__ out) {
    const int32_t n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n > n_nodes) return;
    out_ptr[n] = (int32_t)inc_ptr[n];
    if (n == n_nodes) return;
    const int64_t b = inc_ptr[n], e = inc_ptr[n + 1];
    for (int64_t k = b; k < e; ++k) {
        const int32_t v = inc[k];
        int64_t p = k;
        while (p > b && out[p - 1] > v) {
            out[p] = out[p - 1];
            --p;
        }
        out[p] = v;
    }
}

// also puts the error flags beside the total, for one read of both
__global__ void write_row_ptr(int32_t n_nodes, const int32_t* __restrict__ deg, int64_t* __restrict__ dscan,
                              const int32_t* __restrict__ err, int32_t* __restrict__ row_ptr) {
    int32_t n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n > n_nodes) return;
    if (n == n_nodes) {
        row_ptr[3 * (int64_t)n_nodes] = (int32_t)(9 * dscan[n_nodes]);
        dscan[n_nodes + 1] = *err;
        return;
    }
    const int64_t base = 9 * dscan[n];
    const int32_t dg = deg[n];
    for (int a = 0; a < 3; ++a) row_ptr[3 * (int64_t)n + a] = (int32_t)(base + 3 * a * dg);
}

// ---- exclusive scan of int32 -> int64 (out has n+1 entries; out[n] = total)

__global__ void scan_block_sums(const int32_t* __restrict__ in, int64_t n, int64_t* __restrict__ bsum) {
    __shared__ int64_t sh[kScanThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk;
    int64_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = base + (int64_t)threadIdx.x * kScanItems + k;
        if (i < n) s += in[i];
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = kScanThreads / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = sh[0];
}

// single workgroup: exclusive scan of nb block sums in place
__global__ void scan_block_offsets(int64_t* __restrict__ bsum, int64_t nb) {
    __shared__ int64_t sh[1024];
    const int64_t per = (nb + 1023) / 1024;
    const int64_t b0 = (int64_t)threadIdx.x * per;
    int64_t s = 0;
    for (int64_t k = 0; k < per; ++k)
        if (b0 + k < nb) s += bsum[b0 + k];
    sh[threadIdx.x] = s;
    __syncthreads();
    // Hillis-Steele inclusive scan over the 1024 thread totals
    for (int off = 1; off < 1024; off <<= 1) {
        int64_t v = ((int)threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += v;
        __syncthreads();
    }
    int64_t run = sh[threadIdx.x] - s;
    for (int64_t k = 0; k < per; ++k)
        if (b0 + k < nb) {
            const int64_t v = bsum[b0 + k];
            bsum[b0 + k] = run;
            run += v;
        }
}

__global__ void scan_apply(const int32_t* __restrict__ in, int64_t n, const int64_t* __restrict__ boff,
                           int64_t* __restrict__ out) {
    __shared__ int64_t sh[kScanThreads];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
    int64_t v[kScanItems];
    int64_t s = 0;
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = (base + k < n) ? in[base + k] : 0;
        s += v[k];
    }
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        int64_t t = ((int)threadIdx.x >= off) ? sh[threadIdx.x - off] : 0;
        __syncthreads();
        sh[threadIdx.x] += t;
        __syncthreads();
    }
    int64_t run = boff[blockIdx.x] + sh[threadIdx.x] - s;
    for (int k = 0; k < kScanItems; ++k) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
        if (base + k == n - 1) out[n] = run;
    }
}

hipError_t exclusive_scan(const int32_t* in, int64_t n, int64_t* out, int64_t* bsum, hipStream_t s) {
    if (n == 0) {
        return zero_bytes(out, sizeof(int64_t), s);
    }
    const int64_t nb = (n + kScanChunk - 1) / kScanChunk;
    hipLaunchKernelGGL(scan_block_sums, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, bsum);
    hipLaunchKernelGGL(scan_block_offsets, dim3(1), dim3(1024), 0, s, bsum, nb);
    hipLaunchKernelGGL(scan_apply, dim3((unsigned)nb), dim3(kScanThreads), 0, s, in, n, bsum, out);
    return hipGetLastError();
}

struct PatternWs {
    int32_t* cnt;      // [n_nodes + 1], the last one the error flags
    int64_t* inc_ptr;  // [n_nodes + 1]
    int32_t* pos;      // [8 n_elems] place of a conn entry among its node's
    int32_t* inc;      // [8 n_elems]
    int32_t* deg;      // [n_nodes]
    int64_t* dscan;    // [n_nodes + 2], the last one the error flags
    int64_t* bsum;     // scan block sums
    int32_t* err;      // = cnt + n_nodes
};

template <typename C>
void carve_pattern(C& c, int32_t n_nodes, int32_t n_elems, PatternWs* w) {
    const size_t nb = ((size_t)n_nodes + kScanChunk) / kScanChunk + 1;
    auto cnt = c.template take<int32_t>((size_t)n_nodes + 1);
    auto ip = c.template take<int64_t>((size_t)n_nodes + 1);
    auto pos = c.template take<int32_t>((size_t)n_elems * 8 + 1);
    auto inc = c.template take<int32_t>((size_t)n_elems * 8 + 1);
    auto deg = c.template take<int32_t>((size_t)n_nodes + 1);
    auto ds = c.template take<int64_t>((size_t)n_nodes + 2);
    auto bs = c.template take<int64_t>(nb);
    if (w) *w = PatternWs{cnt, ip, pos, inc, deg, ds, bs, cnt + n_nodes};
}

// take<> of the counter returns void; adapt so the same carving code runs
struct CountAdapter {
    WsCounter cnt;
    template <typename T>
    T* take(size_t n) {
        cnt.take<T>(n);
        return nullptr;
    }
};

// Step 1.
int build_incidence(const fem_mesh* m, const PatternWs& w, hipStream_t s) {
    const int64_t ne8 = (int64_t)m->n_elems * 8;
    const int32_t nn = m->n_nodes;
    FEM_HIP_CHECK(zero_bytes(w.cnt, sizeof(int32_t) * ((size_t)nn + 1), s));
    const int64_t per = kCountThreads * kCountPer, n_chunk = ((ne8 + 256 * kCountPer - 1) / (256 * kCountPer) + 7) / 8;
    if (ne8 > 0)
        hipLaunchKernelGGL(count_incidence, dim3((unsigned)((ne8 + per - 1) / per)), dim3(kCountThreads), 0, s,
                           m->conn, ne8, nn, w.cnt, w.pos, w.err);
    FEM_HIP_CHECK(exclusive_scan(w.cnt, nn, w.inc_ptr, w.bsum, s));
    if (ne8 > 0)
        hipLaunchKernelGGL(fill_incidence, dim3((unsigned)(8 * n_chunk)), dim3(256), 0, s, m->conn, ne8, n_chunk, nn,
                           w.inc_ptr, w.pos, w.inc);
    FEM_HIP_CHECK(hipGetLastError());
    return FEM_OK;
}

// Workgroups of node_pass: 8 contiguous ranges of n_chunk workgroups.
int64_t node_chunk(int32_t n_nodes) {
    const int64_t per = kPatWaves * kNodes;
    return ((n_nodes + per - 1) / per + 7) / 8;
}

}  // namespace
}  // namespace fem

using namespace fem;

extern "C" size_t fem_csr_workspace_bytes(int32_t n_nodes, int32_t n_elems) {
    if (n_nodes < 0 || n_elems < 0) return 0;
    CountAdapter c;
    carve_pattern(c, n_nodes, n_elems, (PatternWs*)nullptr);
    return c.cnt.used + 256;
}

extern "C" int fem_csr_pattern(const fem_mesh* mesh, fem_csr* csr, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (!mesh || !csr) return set_error(FEM_EINVAL, "fem_csr_pattern: mesh and csr must not be NULL");
    if (mesh->n_nodes < 0 || mesh->n_elems < 0)
        return set_error(FEM_EINVAL, "fem_csr_pattern: negative sizes");
    if ((mesh->n_elems > 0 && !mesh->conn) || !csr->row_ptr)
        return set_error(FEM_EINVAL, "fem_csr_pattern: conn and row_ptr must not be NULL");
    if ((int64_t)mesh->n_nodes * 3 >= INT32_MAX || (int64_t)mesh->n_elems * 8 >= INT32_MAX)
        return set_error(FEM_EOVERFLOW, "fem_csr_pattern: 3*n_nodes or 8*n_elems does not fit in int32");
    hipStream_t s = (hipStream_t)stream;
    const size_t need = fem_csr_workspace_bytes(mesh->n_nodes, mesh->n_elems);
    if (!ws || ws_bytes < need)
        return set_error(FEM_ENOMEM, "fem_csr_pattern: workspace of %zu bytes required, %zu given", need, ws_bytes);
    WsCarver c(ws, ws_bytes);
    PatternWs w;
    carve_pattern(c, mesh->n_nodes, mesh->n_elems, &w);
    csr->n_rows = 3 * mesh->n_nodes;
    int rc = build_incidence(mesh, w, s);
    if (rc) return rc;
    const int T = 256;
    const int32_t nn = mesh->n_nodes;
    const int64_t n_chunk = node_chunk(nn);
    const dim3 grid((unsigned)(8 * n_chunk)), block(64 * kPatWaves);
    if (!csr->col_idx) {
        if (nn > 0)
            hipLaunchKernelGGL((node_pass<false>), grid, block, 0, s, nn, n_chunk, mesh->conn, w.inc_ptr, w.inc,
                               w.deg, w.err, (const int32_t*)nullptr, (int32_t*)nullptr, (uint8_t*)nullptr,
                               (int32_t*)nullptr, (int32_t*)nullptr);
        FEM_HIP_CHECK(exclusive_scan(w.deg, nn, w.dscan, w.bsum, s));
        hipLaunchKernelGGL(write_row_ptr, dim3((unsigned)((nn + 1 + T - 1) / T)), dim3(T), 0, s, nn, w.deg, w.dscan,
                           w.err, csr->row_ptr);
        FEM_HIP_CHECK(hipGetLastError());
        int64_t report[2] = {0, 0};
        FEM_HIP_CHECK(hipMemcpyAsync(report, w.dscan + nn, sizeof report, hipMemcpyDeviceToHost, s));
        FEM_HIP_CHECK(hipStreamSynchronize(s));
        const int64_t total = report[0], err = report[1];
        if (err & ERR_RANGE) return set_error(FEM_EMESH, "fem_csr_pattern: node index out of range in conn");
        if (err & ERR_DEGREE) return set_error(FEM_EMESH, "fem_csr_pattern: a node has more than 64 neighbours");
        if (err & ERR_ORPHAN) return set_error(FEM_EMESH, "fem_csr_pattern: a node belongs to no element");
        if (9 * total >= (int64_t)INT32_MAX)
            return set_error(FEM_EOVERFLOW, "fem_csr_pattern: nnz = %lld does not fit in int32", (long long)(9 * total));
        csr->nnz = 9 * total;
        return FEM_OK;
    }
    const bool inc_out = csr->node_elem_ptr && csr->node_elem;
    if (csr->elem_rank && nn > 0) {
        hipLaunchKernelGGL((node_pass<true>), grid, block, 0, s, nn, n_chunk, mesh->conn, w.inc_ptr, w.inc,
                           (int32_t*)nullptr, (int32_t*)nullptr, csr->row_ptr, csr->col_idx, csr->elem_rank,
                           inc_out ? csr->node_elem_ptr : nullptr, inc_out ? csr->node_elem : nullptr);
    } else {
        if (nn > 0)
            hipLaunchKernelGGL(node_columns, dim3((unsigned)((nn + T - 1) / T)), dim3(T), 0, s, nn, mesh->conn,
                               w.inc_ptr, w.inc, csr->row_ptr, csr->col_idx);
        if (inc_out)
            hipLaunchKernelGGL(write_incidence, dim3((unsigned)((nn + 1 + T - 1) / T)), dim3(T), 0, s, nn, w.inc_ptr,
                               w.inc, csr->node_elem_ptr, csr->node_elem);
    }
    FEM_HIP_CHECK(hipGetLastError());
    return FEM_OK;
}
