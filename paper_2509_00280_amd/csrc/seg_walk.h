// The walk of the SEGMENT kernels over a staged tile, shared by the FP32 and
// FP64 kernels: which lanes take which nonzeros, and how the partial sums of
// one output row come together.
//
// A tile's nonzeros stand in LDS in row-grouped order; a run is the stretch of
// one output row.  Every lane group takes an equal stretch of positions,
// whatever runs begin and end in it, sums a run at a time in registers and
// stores it as the run's record when it ends.  The part of a run that entered
// from the left goes to the group in which it began, through shuffles within a
// wave and LDS between waves, which stores the record.  So all groups make the
// same number of steps at every rank and every skew, and a tile has one record
// for each of its rows.
// Groups that took whole pieces of at most 64 nonzeros of a row instead, dealt
// longest first, waited for the longest: at rank 16 a 4096-nonzero tile has 16
// nonzeros for each of its 256 groups and pieces of 64.  All-mode sweeps in
// pieces and in equal shares: 20k nonzeros, rank 16 73.8 / 59.1 us; 3M, 4
// modes, rank 10 942 / 869 us; 5M, 5 modes, rank 25 807 / 730 us; 100M, 3
// modes, rank 32 4.42 / 4.21 ms; 150M, 4 modes, rank 64 (16 lanes a group, rows
// from the LDS cache) 13.65 / 13.56 ms.
#pragma once

#include "tile_common.h"

namespace spt {

// Bytes of LDS the walk takes over from the staged tile: every lane's part and every group's flag.
__host__ __device__ constexpr size_t walk_lds_bytes(int nt, size_t lane_bytes = 16) { return nt * (lane_bytes + 4); }

// Run starts, 32 positions of a tile each: bit p says that a run begins there
// (x), and the starts of the tile before them (y).  The plan holds T / 32 of
// these per tile.
typedef spt_u2 RunWord;

// A lane group's share [q0, q1) of a tile, and what it needs of the run starts,
// read ahead of the barrier behind the staging: its first run, whether that
// begins at q0 and whether its last ends at q1, and the starts behind q0 in the
// first 64 positions (more than a share has at up to 64 columns' lanes).
struct WalkShare {
    int q0, q1, run;
    bool began, ended;
    uint32_t bits[2];
    const RunWord *words;  // the tile's
};

template <int T>
__device__ __forceinline__ uint32_t run_bits(const RunWord *words, int q) {  // starts of positions [q, q + 32)
    const int w = q >> 5;
    return __builtin_amdgcn_alignbit(words[min(w + 1, T / 32 - 1)].x, words[min(w, T / 32 - 1)].x, q & 31);
}

// step: positions that a step of the walk takes.  Unless TIGHT, all words of
// the run starts are asked for at once; one after the other, as they are
// needed, they are four round trips to memory at every tile's start, but cost
// fewer registers on the way.  TIGHT are the 4-mode kernels of one tensor, the
// widest that are held to 64 VGPRs: all-mode sweeps without and with it, here
// and at the walk's end, 13.61 / 12.57 ms (150M nonzeros, rank 64) and 837 / 798
// us (3M, rank 10).  It cost the 3-mode kernel (100M, rank 32: 4.07 / 4.12 ms
// here, 4.07 / 4.09 at the end) and the batched kernels, which are held to 128
// VGPRs (32 decompositions 31.0 / 31.8 ms).  The kernel for up to 3 modes, which
// runs two, spills as well and would gain (10M, rank 16: 201 / 189 us), but
// shares the 3-mode kernel's form.
template <int NT, int T, bool TIGHT>
__device__ __forceinline__ WalkShare walk_share(const LaneGroup &lg, int cnt, int step, const RunWord *words) {
    const int NG = NT / 64 * lg.per_wave;
    const int each = ((cnt + NG - 1) / NG + step - 1) / step * step;
    WalkShare ws;
    ws.q0 = min(lg.g * each, cnt);
    ws.q1 = lg.on ? min(ws.q0 + each, cnt) : ws.q0;
    ws.words = words;
    const int w = ws.q0 >> 5;
    const RunWord first = words[min(w, T / 32 - 1)];
    if constexpr (!TIGHT) {
        const uint32_t second = words[min(w + 1, T / 32 - 1)].x, third = words[min(w + 2, T / 32 - 1)].x;
        const uint32_t end = words[min(ws.q1 >> 5, T / 32 - 1)].x;
        ws.run = (int)(first.y + __popc(first.x & (0xFFFFFFFFu >> (31 - (ws.q0 & 31))))) - 1;
        ws.began = (first.x >> (ws.q0 & 31)) & 1u;
        ws.ended = ws.q1 >= cnt || ((end >> (ws.q1 & 31)) & 1u);
        ws.bits[0] = __builtin_amdgcn_alignbit(second, first.x, ws.q0 & 31) & ~1u;
        ws.bits[1] = __builtin_amdgcn_alignbit(third, second, ws.q0 & 31);
        asm volatile("" : "+v"(ws.run), "+v"(ws.bits[0]), "+v"(ws.bits[1]));  // made here, before the words pile up
    } else {
        auto at = [&](int q) {  // the second word only where it is needed
            const int sh = q & 31;
            const uint32_t lo = words[min(q >> 5, T / 32 - 1)].x, hi = words[min((q >> 5) + 1, T / 32 - 1)].x;
            return sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
        };
        ws.run = (int)(first.y + __popc(first.x & (0xFFFFFFFFu >> (31 - (ws.q0 & 31))))) - 1;
        ws.began = (first.x >> (ws.q0 & 31)) & 1u;
        ws.ended = ws.q1 >= cnt || (at(ws.q1) & 1u);
        ws.bits[0] = at(ws.q0) & ~1u;
        ws.bits[1] = at(ws.q0 + 32);
    }
    return ws;
}

// UB staged words of 4 or 8 bytes at p (aligned to all of them) in one read
template <int UB, class Word>
__device__ __forceinline__ void load_words(const Word *p, Word (&x)[UB]) {
    static_assert(UB == 1 || UB == 2, "one or two");
    if constexpr (UB == 2) {
        typedef Word pair __attribute__((ext_vector_type(2)));
        const pair t = *reinterpret_cast<const pair *>(p);
        x[0] = t.x;
        x[1] = t.y;
    } else {
        x[0] = p[0];
    }
}

// Walk the first cnt positions of a staged tile (every thread of the workgroup
// calls, after the barrier behind the staging).  product(q, p, x) forms the
// products of the positions q + u, u < UB, for this lane's columns, up to the
// last factor: p[u][:] * x[u][:], which the sum takes in one fma; q is a
// multiple of UB, and the staging fills positions from cnt on to the next
// multiple with anything that can be read.
// rec[k] is the record of the tile's run k; records have ld columns (R..ld-1
// are zeroed).  Reads stay inside the tile and no record at or beyond rec_cap
// is written, whatever the plan holds.
template <class Real, int NT, int T, int VEC, int UB, bool TIGHT, int FAR, class Product>
__device__ __forceinline__ void run_walk(const LaneGroup &lg, const WalkShare &ws, int R, int cnt, int nruns,
                                         const uint32_t *__restrict__ rec, uint32_t rec_cap,
                                         Real *__restrict__ rec_val, int ld, char *lds, const Product &product) {
    constexpr uint32_t kNone = 0xFFFFFFFFu;  // no record: a store to it is dropped
    const int q0 = ws.q0, q1 = ws.q1;
    const spt_i4 slots = word_rsrc(rec, (uint32_t)nruns);
    const RowView<Real, FAR != kNear> out(rec_val, ld, rec_cap);
    // a sum for each nonzero of a step: chains of additions UB times shorter
    Real acc[UB][VEC], part[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) part[v] = 0;
    auto clear = [&]() {
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[u][v] = 0;
    };
    auto gather_sums = [&]() {  // the sums of the step's slots into the first
#pragma unroll
        for (int u = 1; u < UB; ++u)
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[0][v] += acc[u][v];
    };
    clear();
    // The records of the open run and of the next: the load of a run's record
    // is one run ahead of its use, and the gathers of a later step are waited
    // for behind it anyway.  Short runs make nearly every step of a wave end
    // some group's run, so the end of a run is kept to a dozen instructions: a
    // lookup of the record among the group's lanes, 64-bit addresses and a
    // branch around a run's sums took 3.59 instead of 3.04 ms for an all-mode
    // sweep in FP64 (rank 16, 20M nonzeros), 4.21 instead of 4.12 ms in FP32
    // (rank 32, 100M), 13.59 instead of 13.38 ms (rank 64, 150M).
    int next_at = (ws.run + 1) * 4;
    uint32_t cur = kNone, next = 0;
    bool began = ws.began, open = false;
    bool through = false;  // a run entered from the left and leaves to the right
    auto store_end = [&](const LaneGroup &lg) {
        out.template store<VEC>(cur, lg.col, acc[0]);
        if (ld > R) {  // zeros to the row's end
            if (VEC == 4 && ld - R >= 4) {
                const Real z[VEC] = {};
                for (int c = R + VEC * lg.j; c < ld; c += VEC * lg.G) out.template store<VEC>(cur, min(c, ld - VEC), z);
            } else {
                const Real z[1] = {0};
                for (int c = R + lg.j; c < ld; c += lg.G) out.template store<1>(cur, c, z);
            }
        }
    };
    auto write = [&]() { store_end(lg); };
    auto keep_part = [&]() {  // the run that entered from the left
#pragma unroll
        for (int v = 0; v < VEC; ++v) part[v] = acc[0][v];
    };
    if (q0 < q1) {
        if (began) cur = spt_word_load(slots, ws.run * 4, 0, 0);
        next = spt_word_load(slots, next_at, 0, 0);
        for (int qb = q0; qb < q1; qb += 32) {
            const int n = min(32, q1 - qb);
            uint32_t bits = qb == q0 ? ws.bits[0] : qb == q0 + 32 ? ws.bits[1] : run_bits<T>(ws.words, qb);
            for (int i = 0; i < n; i += UB) {
                Real p[UB][VEC], x[UB][VEC];
                product(qb + i, p, x);
                // One nonzero a step (5 modes): wait for the gathers here.  Left
                // to itself the compiler waits behind the end of a run, and so
                // for its store too (765 instead of 744 us at rank 25, 5M
                // nonzeros); with two a step the registers cost more than that
                // (rank 64, 4 modes, 150M nonzeros: 13.79 instead of 13.39 ms).
                if constexpr (UB == 1) {
#pragma unroll
                    for (int v = 0; v < VEC; ++v) asm volatile("" : "+v"(p[0][v]), "+v"(x[0][v]));
                }
#pragma unroll
                for (int u = 0; u < UB; ++u) {
                    if (bits & (1u << u)) {  // a run begins: the open one is over
                        gather_sums();
                        if (!began) {
                            keep_part();
                            began = true;
                        }
                        write();
                        clear();
                        cur = next;
                        next_at += 4;
                        next = spt_word_load(slots, next_at, 0, 0);
                    }
                    if (u == 0 || i + u < n)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) acc[u][v] = fma(p[u][v], x[u][v], acc[u][v]);
                }
                bits >>= UB;
            }
        }
        gather_sums();
        if (!began) {
            keep_part();
            through = !ws.ended;
        } else if (ws.ended) {
            write();
        } else {
            open = true;
        }
    }
    // TIGHT: the lane group worked out anew.  Its numbers, and the addresses made
    // from them, would otherwise be held across the walk in spills, which reach
    // HBM (40 bytes a thread were 10 of 18 bytes written per nonzero).
    int tid = threadIdx.x;
    LaneGroup tail = lg;
    if constexpr (TIGHT) {
        asm volatile("" : "+v"(tid));
        tail = lane_group<VEC>(R, tid);
    }
    // A run over many groups: the parts of a wave's groups are joined by halves,
    // the waves' then one after the other, so a run over a whole tile takes
    // log2(groups of a wave) + 16 additions.  One for every group, 1023 of them at
    // ranks up to 4, lost up to 246 roundings of FP32, and took 331 us for 5M
    // nonzeros of one row (rank 4, 3 modes) instead of 62; 24 rows 78 / 60 us, an
    // all-mode sweep of 3M nonzeros at rank 10 (4 modes) 859 / 803 us, of 150M at
    // rank 64 12.88 / 12.55 ms.  The run's first group takes the joined parts
    // from LDS: through a shuffle they cost 0.7% of a sweep at rank 32 (100M).
    const int lane = tid & 63, wave = tid >> 6, groups_end = tail.per_wave * tail.G;
    for (int d = tail.G; d < groups_end; d *= 2) {
        const bool in = through && lane + d < groups_end;
        if (!__any(in)) break;
        const bool beyond = __shfl((int)through, lane + d, 64);
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const Real y = __shfl(part[v], lane + d, 64);
            if (in) part[v] += y;
        }
        if (in) through = beyond;  // of the groups joined so far
    }
    __syncthreads();  // the staged tile is done with
    Real *parts = reinterpret_cast<Real *>(lds);
    int *flags = reinterpret_cast<int *>(parts + NT * VEC);
    if (tail.on) {
        store_vec<VEC>(parts + (tail.g * tail.G + tail.j) * VEC, part);
        if (tail.j == 0) flags[tail.g] = through;
    }
    __syncthreads();
    if (open) {
        int m = tail.g + 1, w = wave + (lane + tail.G < groups_end ? 1 : 2);
        for (;;) {  // ends at the latest in the last wave, whose last group's run ends with it
            const Real *p = parts + (m * tail.G + tail.j) * VEC;
#pragma unroll
            for (int v = 0; v < VEC; ++v) acc[0][v] += p[v];
            if (!flags[m] || w >= NT / 64) break;
            m = w * tail.per_wave;
            ++w;
        }
        store_end(tail);
    }
}

}  // namespace spt
