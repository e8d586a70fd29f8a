// Sum of the records of every output row (SEGMENT, TABLE), FP32 and FP64.
#pragma once

#include <algorithm>

#include "tile_common.h"

namespace spt {

#ifndef SPT_RED_UB
#define SPT_RED_UB 8
#endif
constexpr int kRedThreads = 256;

// Records sorted by row.  Every lane group sums the runs of equal row of
// `chunk` consecutive records (8 record loads in flight per lane); a run that
// lies inside the chunk is stored.  A run that crosses chunks of one
// workgroup is put together in LDS: each group leaves the part of the run
// that entered from its left, and the group where the run began (or the
// workgroup's first) adds the parts up to the run's end.  Only runs that
// cross the workgroup's own edges are added atomically (out was zeroed), so
// chunks can be short without more contention on the rows of many records:
// with atomics at every chunk's edge, chunks of 64 to 512 records took 21 us
// for 1000 records of rank 16 (one serial chain) and sums over short chunks
// 17 ms instead of 13.6 for the rank-64 sweep.
// The roundings of an FP32 sum: a round's records are added up before they
// join the run's sum, and the parts of a run over several groups in FP64.
// FP64 sums throughout took 4.34 instead of 4.21 ms for an all-mode sweep (rank
// 32, 3 modes, 100M nonzeros); this takes 4.21 ms and as long as one chain.
template <class Real, int VEC>
__global__ __launch_bounds__(kRedThreads) void k_reduce_records(const uint64_t *__restrict__ srow,
                                                                const uint32_t *__restrict__ sidx,
                                                                const Real *__restrict__ rec_val, int64_t P, int R,
                                                                int chunk, int64_t rows, Real *__restrict__ out) {
    constexpr int UB = SPT_RED_UB;
    constexpr int kHead = 1, kThrough = 2;
    __shared__ Real part[kRedThreads * VEC];  // per lane: its columns of the run that entered from the left
    __shared__ int flag[kRedThreads];           // per group: kHead: such a run; kThrough: it also leaves to the right
    const LaneGroup lg = lane_group<VEC>(R);
    const int NG = kRedThreads / 64 * lg.per_wave, g = lg.g, c = lg.col;
    const int64_t c0 = ((int64_t)blockIdx.x * NG + g) * chunk;
    const int64_t c1 = lg.on ? min(c0 + chunk, P) : 0;
    const bool work = c0 < c1;
    Real acc[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[v] = 0;
    Real few[VEC] = {};  // the open run's records of this round, not yet in acc
    auto fold = [&]() {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            acc[v] += few[v];
            few[v] = 0;
        }
    };
    uint64_t cur = 0, after = ~0ull;
    bool began = true;  // the open run began in this chunk
    Real *mine = part + (g * lg.G + lg.j) * VEC;
    auto emit = [&](uint64_t r, bool whole) {
        if (r >= (uint64_t)rows) return;  // sentinel records of unused slots
        Real *o = out + (int64_t)r * R + c;
        if (whole) {
            Real x[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) x[v] = acc[v];
            store_vec<VEC>(o, x);
        } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v)
                if (c + v >= VEC * lg.j) unsafeAtomicAdd(o + v, acc[v]);  // not the columns repeated from the neighbour
        }
    };
    // a run that is over: stored, or handed to the group where it began
    int my_flag = 0;
    auto close = [&]() {
        fold();
        if (began) {
            emit(cur, true);
        } else if (g == 0) {
            emit(cur, false);
        } else {
            store_vec<VEC>(mine, acc);
            my_flag = kHead;
        }
    };
    if (work) {
        const uint64_t before = c0 > 0 ? srow[c0 - 1] : ~0ull;
        if (c1 < P) after = srow[c1];
        cur = srow[c0];
        began = cur != before;
        for (int64_t q = c0; q < c1; q += UB) {
            uint64_t r[UB];
            Real x[UB][VEC];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                const bool ok = q + u < c1;
                r[u] = ok ? srow[q + u] : ~0ull;
                // sidx null: the records are already grouped by row (identity order)
                const int64_t ri = ok ? (sidx ? (int64_t)sidx[q + u] : q + u) : 0;
                if (ok) {
                    load_vec_any<VEC>(rec_val + ri * R + c, x[u]);
                } else {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) x[u][v] = 0;
                }
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                if (q + u < c1) {
                    if (r[u] != cur) {
                        close();
                        cur = r[u];
                        began = true;
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            acc[v] = 0;
                            few[v] = x[u][v];
                        }
                    } else {
#pragma unroll
                        for (int v = 0; v < VEC; ++v) few[v] += x[u][v];
                    }
                }
            }
            fold();
        }
        if (cur != after) {
            close();
        } else if (!began && g > 0) {  // one run over the whole chunk and past both of its ends
            store_vec<VEC>(mine, acc);
            my_flag = kHead | kThrough;
        }
    }
    if (lg.on && lg.j == 0) flag[g] = my_flag;
    __syncthreads();
    // the open run of the group where it began (the workgroup's first group
    // stands in for what began before it): add the parts to its right
    if (work && cur == after && (began || g == 0)) {
        bool ended = false;
        double sum[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) sum[v] = (double)acc[v];
        for (int k = g + 1; k < NG; ++k) {
            const Real *p = part + (k * lg.G + lg.j) * VEC;
#pragma unroll
            for (int v = 0; v < VEC; ++v) sum[v] += (double)p[v];
            if (!(flag[k] & kThrough)) {
                ended = true;
                break;
            }
        }
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] = (Real)sum[v];
        emit(cur, began && ended);
    }
}

template <class Real, int V>
spt_status launch_reduce_v(const uint64_t *srow, const uint32_t *sidx, const Real *rec_val, int64_t P, int R,
                           int64_t rows, Real *out, hipStream_t s) {
    const int groups = kRedThreads / 64 * (64 / ((R + V - 1) / V));  // LaneGroup
    // About 512 records to a workgroup, at least 8 (one round of loads) to a
    // group: all-mode sweeps at 16 / 32 / 64 / 512 records per group took
    // 13.69 / 13.48 / 13.46 / 13.64 ms at rank 64 and 6.6M records a mode (16
    // groups), 4.43 / 4.46 / 4.53 / 4.59 ms at rank 32 and 5M (32 groups); at
    // 8 / 16 / 64 87 / 92 / 128 us at rank 16 and 1000 records (64 groups).  Few
    // records: the shortest chunks, which leave the most groups.
    int chunk = std::max(8, (512 / groups + 7) & ~7);
    while (chunk > 8 && P / chunk < 4096) chunk -= 8;
    const int64_t per_block = groups * (int64_t)chunk;
    const int64_t blocks = (P + per_block - 1) / per_block;
    hipLaunchKernelGGL((k_reduce_records<Real, V>), dim3((unsigned)blocks), dim3(kRedThreads), 0, s, srow, sidx, rec_val,
                       P, R, chunk, rows, out);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

// 16 bytes of columns a lane; FP64 rows of more than 128 columns need 32 for a wave to hold them.
template <class Real>
spt_status launch_reduce(const uint64_t *srow, const uint32_t *sidx, const Real *rec_val, int64_t P, int R, int64_t rows,
                         Real *out, hipStream_t s) {
    constexpr int V = 16 / (int)sizeof(Real);
    if (P <= 0) return SPT_OK;
    if (R < V) return launch_reduce_v<Real, 1>(srow, sidx, rec_val, P, R, rows, out, s);
    if (R <= 64 * V) return launch_reduce_v<Real, V>(srow, sidx, rec_val, P, R, rows, out, s);
    return launch_reduce_v<Real, 4>(srow, sidx, rec_val, P, R, rows, out, s);
}

}  // namespace spt
