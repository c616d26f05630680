// Device-side building blocks: wave64 / workgroup reductions and the
// row-compressed sparse product with L lanes per row.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "pdhg_internal.hpp"

namespace pdhg {

// The value `off` lanes up (off a power of two), for the lanes that a
// reduction towards the lowest lane of an aligned group of 2 off lanes uses;
// the others get something unspecified.  Register moves (DPP within a row of
// 16 lanes, the row and half swaps across rows) instead of __shfl_xor's trips
// through the LDS unit: a tree over 64 lanes has six of them in a row, and the
// kernels that use it are bound by such chains (with the step scalars formed
// early, pdhg_kernels.hpp: 4-6% of a step on LPs of up to 240,000 entries).
template <int off>
__device__ __forceinline__ int lane_up(int v)
{
    static_assert(off == 1 || off == 2 || off == 4 || off == 8 || off == 16 || off == 32, "a step of a tree over 64 lanes");
    if constexpr (off == 32) return (int)__builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
    else if constexpr (off == 16) return (int)__builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
    else return __builtin_amdgcn_update_dpp(0, v, 0x100 + off, 0xf, 0xf, true); // row_shl: lane i reads lane i + off
}

template <int off>
__device__ __forceinline__ float lane_up(float v)
{
    return __int_as_float(lane_up<off>(__float_as_int(v)));
}

template <int off>
__device__ __forceinline__ double lane_up(double v)
{
    return __hiloint2double(lane_up<off>(__double2hiint(v)), lane_up<off>(__double2loint(v)));
}

// Sum over a group of L consecutive lanes (L a power of two <= 64), in the
// group's lowest lane, by a fixed tree (halves added pairwise), so the result
// is deterministic.
template <int L, typename T>
__device__ __forceinline__ T group_sum(T v)
{
    if constexpr (L > 32) v += lane_up<32>(v);
    if constexpr (L > 16) v += lane_up<16>(v);
    if constexpr (L > 8) v += lane_up<8>(v);
    if constexpr (L > 4) v += lane_up<4>(v);
    if constexpr (L > 2) v += lane_up<2>(v);
    if constexpr (L > 1) v += lane_up<1>(v);
    return v;
}

template <int L>
__device__ __forceinline__ double group_max(double v)
{
    if constexpr (L > 32) v = fmax(v, lane_up<32>(v));
    if constexpr (L > 16) v = fmax(v, lane_up<16>(v));
    if constexpr (L > 8) v = fmax(v, lane_up<8>(v));
    if constexpr (L > 4) v = fmax(v, lane_up<4>(v));
    if constexpr (L > 2) v = fmax(v, lane_up<2>(v));
    if constexpr (L > 1) v = fmax(v, lane_up<1>(v));
    return v;
}

// in lane 0
__device__ __forceinline__ double wave_sum(double v) { return group_sum<64>(v); }
__device__ __forceinline__ double wave_max(double v) { return group_max<64>(v); }

// Workgroup reduction of NQ values (sum, or max where is_max bit q is set);
// thread 0 receives the results.  Uses kBlock/64 LDS slots per quantity.
template <int NQ>
__device__ __forceinline__ void block_reduce(double (&v)[NQ], unsigned is_max_mask)
{
    __shared__ double lds[NQ][kBlock / 64];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; q++) {
        v[q] = ((is_max_mask >> q) & 1u) ? wave_max(v[q]) : wave_sum(v[q]);
        if (lane == 0) lds[q][wid] = v[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NQ; q++) {
            double acc = lds[q][0];
            for (int w = 1; w < kBlock / 64; w++)
                acc = ((is_max_mask >> q) & 1u) ? fmax(acc, lds[q][w]) : acc + lds[q][w];
            v[q] = acc;
        }
    }
    __syncthreads();
}

// Workgroups are dispatched round-robin over the 8 XCDs (bid % 8).  Map them
// so that every XCD works on one contiguous range of logical blocks: rows
// that gather the same cache lines then meet in the same L2.
__device__ __forceinline__ int xcd_range_block(int bid, int nblk)
{
    const int x = bid & 7, q = nblk >> 3, r = nblk & 7;
    const int base = x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q;
    return base + (bid >> 3);
}

// The mapping of a single LP's launches.  Up to kXcdChunkMin workgroups
// (a launch whose workgroups are resident together) take the contiguous
// ranges above.  A larger launch runs in many rounds, and with ranges each
// XCD would own one region of the matrix: where the rows change kind along
// the matrix (the node-balance, then the capacity rows of a multicommodity
// LP) the XCDs get unequal work.  There chunks of kXcdChunk logical blocks
// are dealt round-robin to the XCDs instead: neighbouring rows still share an
// L2 within a chunk, and every region spreads over all 8 XCDs.  A tail of
// fewer than 8 chunks keeps the dispatch order.  (The batch engine keeps the
// ranges: one LP's tiles then stay in one L2.)
constexpr int kXcdChunk = 16;
constexpr int kXcdChunkMin = 8192;

__device__ __forceinline__ int xcd_block(int bid, int nblk)
{
    if (nblk < kXcdChunkMin) return xcd_range_block(bid, nblk);
    const int full = nblk / (8 * kXcdChunk) * (8 * kXcdChunk);
    if (bid >= full) return bid;
    const int x = bid & 7, k = bid >> 3;
    return ((k / kXcdChunk) * 8 + x) * kXcdChunk + k % kXcdChunk;
}

// One lane's share of a row's product: the terms e = beg+lane, beg+lane+L, ...
// below end, accumulated in that order, in rounds of U.  A lane's share is a
// chain of loads (index, then operand); a round's gathers go out together,
// and before they are waited for the next round's index and value loads, so a
// round costs one gather's latency and the index loads hide behind it.
// Positions past the end reload the last entry; their terms are not added.
// What is compared is the entries left, never a position ahead of the end: a
// model may hold 2^31 - 1 entries, and such a position would wrap.
template <int L, int U, typename ACC, typename I, typename VM, typename VX>
__device__ __forceinline__ ACC lane_rounds(int beg, int end, int lane, const I *__restrict__ idx,
                                           const VM *__restrict__ val, const VX *__restrict__ x)
{
    ACC acc = 0;
    int left = end - beg - lane;
    if (left <= 0) return acc;
    int e = beg + lane;
    I i[U];
    VM v[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int k = e + (u * L < left ? u * L : left - 1);
        i[u] = idx[k];
        v[u] = val[k];
    }
    for (;;) {
        VX g[U];
        ACC w[U];
#pragma unroll
        for (int u = 0; u < U; u++) g[u] = x[i[u]];
#pragma unroll
        for (int u = 0; u < U; u++) w[u] = (ACC)v[u];
        if (!__builtin_amdgcn_ballot_w64(left <= (2 * U - 1) * L)) { // a full round for every lane of the wave still here
            e += U * L;
            left -= U * L;
#pragma unroll
            for (int u = 0; u < U; u++) i[u] = idx[e + u * L];
#pragma unroll
            for (int u = 0; u < U; u++) v[u] = val[e + u * L];
#pragma unroll
            for (int u = 0; u < U; u++) acc += w[u] * (ACC)g[u];
            continue;
        }
        if (__builtin_amdgcn_ballot_w64(left > U * L)) {
#pragma unroll
            for (int u = 0; u < U; u++) {
                const int k = e + ((U + u) * L < left ? (U + u) * L : left - 1);
                i[u] = idx[k];
                v[u] = val[k];
            }
        }
        acc += w[0] * (ACC)g[0];
#pragma unroll
        for (int u = 1; u < U; u++)
            if (u * L < left) acc += w[u] * (ACC)g[u];
        if (left <= U * L) return acc;
        e += U * L;
        left -= U * L;
    }
}

// The same in rounds of four and a last one of up to three entries, one after
// another: fewer instructions than the rounds above.
template <int L, typename ACC, typename I, typename VM, typename VX>
__device__ __forceinline__ ACC lane_short(int beg, int end, int lane, const I *__restrict__ idx,
                                          const VM *__restrict__ val, const VX *__restrict__ x)
{
    ACC acc = 0;
    int left = end - beg - lane;
    for (; left > 3 * L; left -= 4 * L) {
        const int e = end - left;
        I i[4];
        VM v[4];
        VX g[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            i[u] = idx[e + u * L];
            v[u] = val[e + u * L];
        }
#pragma unroll
        for (int u = 0; u < 4; u++) g[u] = x[i[u]];
#pragma unroll
        for (int u = 0; u < 4; u++) acc += (ACC)v[u] * (ACC)g[u];
    }
    if (left > 0) {
        const int e = end - left, c1 = L < left ? e + L : e, c2 = 2 * L < left ? e + 2 * L : e;
        const I i0 = idx[e], i1 = idx[c1], i2 = idx[c2];
        const ACC v0 = (ACC)val[e], v1 = (ACC)val[c1], v2 = (ACC)val[c2];
        const ACC g0 = (ACC)x[i0], g1 = (ACC)x[i1], g2 = (ACC)x[i2];
        acc += v0 * g0;
        if (L < left) acc += v1 * g1;
        if (2 * L < left) acc += v2 * g2;
    }
    return acc;
}

// Rounds of eight where a row of the wave has more than four entries a lane:
// fewer waits in a chain; at most four entries: rounds of four, as the other
// four loads would repeat the last entry.  Per iteration on transportation
// LPs (fp64 / mixed), rounds of four -> this rule: 200x500 7.33 / 6.97 -> 6.94
// / 6.55 us, 1000x2500 46.8 / 35.6 -> 46.9 / 33.6; 2000x5000 228.7 / 159.2 ->
// 225.8 / 158.9 in the solve, 16.3 / 12.8 -> 16.2 / 12.6 in the push (12.9
// with rounds of eight alone: its sink rows have three entries a lane).
// Where no row has more than one entry a lane, one round of one, as the other
// three would fetch the row's last entry: planted 3,000 x 8,000 (5 and 13
// entries) with 64 lanes 10.3 / 9.0 -> 8.7 / 8.4 us.  Lanes with rows of their
// own, or two a row, end in different rounds wherever a row of the wave is
// short, and instructions count: there one round after another, 3,000 x 8,000
// with one lane 11.5 / 10.3 -> 9.7 / 8.7, power-law 2,000 x 8,000 28.7 / 26.5 ->
// 22.2 / 21.0; rows of 150 and 225 entries keep the rounds (56.8 against 63).
template <int L, typename ACC, typename I, typename VM, typename VX>
__device__ __forceinline__ ACC lane_dot(int beg, int end, int lane, const I *__restrict__ idx,
                                        const VM *__restrict__ val, const VX *__restrict__ x)
{
    if (L <= 2 && __builtin_amdgcn_ballot_w64(end - beg <= 32 * L)) return lane_short<L, ACC>(beg, end, lane, idx, val, x);
    if (__builtin_amdgcn_ballot_w64(end - beg > 4 * L)) return lane_rounds<L, 8, ACC>(beg, end, lane, idx, val, x);
    if (L >= 16 && !__builtin_amdgcn_ballot_w64(end - beg > L)) return lane_rounds<L, 1, ACC>(beg, end, lane, idx, val, x);
    return lane_rounds<L, 4, ACC>(beg, end, lane, idx, val, x);
}

// Row-compressed product out[r] = sum_e val[e] * x[idx[e]] over rows r < rows,
// L lanes per row, accumulation in ACC.  One group of L lanes walks a row with
// stride L (coalesced for L >= 2 on long rows, one lane per row when L = 1).
template <int L, typename VM, typename VX, typename ACC, typename VO>
__global__ __launch_bounds__(kBlock) void k_spmv(int rows, const int *__restrict__ ptr,
                                                 const int *__restrict__ idx, const VM *__restrict__ val,
                                                 const VX *__restrict__ x, VO *__restrict__ out)
{
    const int64_t g = (int64_t)xcd_block(blockIdx.x, gridDim.x) * kBlock + threadIdx.x;
    const int64_t row = g / L;
    const int lane = (int)(g % L);
    if (row >= rows) return;
    const int beg = ptr[row], end = ptr[row + 1];
    ACC acc = lane_dot<L, ACC>(beg, end, lane, idx, val, x);
    acc = group_sum<L>(acc);
    if (lane == 0) out[row] = (VO)acc;
}

// Launch k_spmv with the lane count chosen at run time.
template <typename VM, typename VX, typename ACC, typename VO>
inline void spmv(hipStream_t st, int lanes, int rows, const int *ptr, const int *idx, const VM *val,
                 const VX *x, VO *out)
{
    if (rows <= 0) return;
    const int64_t threads = (int64_t)rows * lanes;
    const int grid = (int)((threads + kBlock - 1) / kBlock);
#define PDHG_SPMV_CASE(LL)                                                                       \
    case LL:                                                                                     \
        hipLaunchKernelGGL((k_spmv<LL, VM, VX, ACC, VO>), dim3(grid), dim3(kBlock), 0, st, rows, \
                           ptr, idx, val, x, out);                                               \
        break;
    switch (lanes) {
        PDHG_SPMV_CASE(1)
        PDHG_SPMV_CASE(2)
        PDHG_SPMV_CASE(4)
        PDHG_SPMV_CASE(8)
        PDHG_SPMV_CASE(16)
        PDHG_SPMV_CASE(32)
    default:
        PDHG_SPMV_CASE(64)
    }
#undef PDHG_SPMV_CASE
}

__device__ __forceinline__ bool is_inf_lo(double v) { return v <= -1e20; }
__device__ __forceinline__ bool is_inf_up(double v) { return v >= 1e20; }

} // namespace pdhg
