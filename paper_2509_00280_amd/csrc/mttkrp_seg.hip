// SEGMENT strategy of mode-n MTTKRP (Section II-B, Fig. 2) on gfx950.
//
// A workgroup of NT threads owns a tile of T = 4 NT consecutive nonzeros of
// the key-ordered stream.  Conflicts on output rows are resolved by
// regrouping the tile by output row: the run of every row is summed in
// registers (a segmented reduction over equal output index, seg_walk.h) and
// written as one record (R floats) with plain stores; the records are summed
// per row afterwards (mttkrp_table.hip).  No atomics on the main path.
//
// Plan (once per tensor and mode, the hashing stage below): an LDS hash of
// the tile's output rows (T slots, linear probing, CAS), one block scan of
// packed (nonzeros << 16 | occupied) per slot, giving every nonzero its
// position in row-grouped order, the positions where runs begin, and the
// (tile, row) pairs, one to a run.  The pairs are then sorted by row across
// the tensor (or the batch), which lays the records out grouped by row and
// gives every record its row.
//
// Call (the planned kernel): coalesced non-temporal loads of keys, values and
// plan positions; the non-output coordinates are decoded from the bit runs
// held in VGPRs and scattered once to LDS in row-grouped order; lane groups
// (LaneGroup) walk equal shares of it, gather the N-1 factor rows of each
// nonzero with buffer loads, form v * Hadamard and sum.  No hashing, atomics
// or scans over nonzeros at run time.
//
// Row-cached call (4096-nonzero tiles, 2..4 modes): the tile dictionaries
// (per mode, each tile's distinct rows most frequent first, and each
// nonzero's index in that list) replace the key decode; the first cap rows
// of every non-output mode's list are copied to LDS and a nonzero reads its
// factor row there when its index is below cap.
#include <algorithm>
#include <atomic>

#include "seg_walk.h"

namespace spt {

namespace {

constexpr int kPiece = 64;  // nonzeros per piece, the measure of spt_mttkrp_noalloc's limit
constexpr int kSegpThreads4096 = 1024;  // threads of the MTTKRP kernel on 4096-nonzero tiles

// The budget that decides which tile sizes a tensor of nmodes modes may use
// (seg_tile_ok): nm - 1 coordinates and a value of 4 bytes, the plan passes'
// hash table of 8 and 2 more per position.  The kernels need less; the sizes
// on offer are part of the plan's interface and stay.
__host__ __device__ inline size_t seg_lds_bytes(int T, int nmodes) {
    return (size_t)(nmodes - 1) * T * 4 + (size_t)T * 4 + (size_t)T * 4 + (size_t)(T + 4) * 4 + (size_t)T * 2;
}

// LDS of the planned kernel: crdg[nm - 1][T] and valg[T].
__host__ __device__ inline size_t segp_lds_bytes(int T, int nmodes) {
    return (size_t)(nmodes - 1) * T * 4 + (size_t)T * 4;
}

struct SegLds {
    uint32_t *hkey;
    uint32_t *hcnt;
    uint32_t *bits;
};

// LDS of the plan's counting and emission passes: hkey[T], hcnt[T + 4] and
// the run starts, T / 32 words.
__host__ __device__ inline size_t seg_plan_lds_bytes(int T) { return (size_t)T * 8 + 16 + (size_t)T / 8; }

__device__ __forceinline__ SegLds seg_carve_plan(char *p, int T) {
    SegLds L;
    L.hkey = (uint32_t *)p;
    L.hcnt = L.hkey + T;
    L.bits = L.hcnt + T + 4;
    return L;
}

// Hash one tile by output row.  After return: hkey[s] = row of slot s, hcnt[s]
// = (first position of slot s) << 16 | (occupied slots before s), hcnt[T] =
// (nonzeros << 16) | distinct rows, and sr[u] = slot << 16 | rank within the
// slot of this thread's nonzero u (e = threadIdx.x + u NT).
template <int NT>
__device__ __forceinline__ int seg_hash(const MttkrpArgs &a, int64_t tile, const SegLds &L, const CodecRegs &cr,
                                        uint32_t *wsum, uint32_t (&sr)[4]) {
    constexpr int T = 4 * NT;
    const int tid = threadIdx.x;
    const int64_t base = tile * (int64_t)T;
    const int64_t rem = a.nnz - base;
    const int cnt = rem < T ? (int)rem : T;
    for (int i = tid; i < T; i += NT) {
        L.hkey[i] = kNoRow;
        L.hcnt[i] = 0;
    }
    uint32_t w[4][4];
    const int nwords = 2 * a.codec.key_words;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + u * NT;
        uint64_t klo = 0, khi = 0;
        if (e < cnt) {
            klo = __builtin_nontemporal_load(a.lo + base + e);
            if (nwords == 4) khi = __builtin_nontemporal_load(a.hi + base + e);
        }
        w[u][0] = (uint32_t)klo;
        w[u][1] = (uint32_t)(klo >> 32);
        w[u][2] = (uint32_t)khi;
        w[u][3] = (uint32_t)(khi >> 32);
    }
    uint32_t rowv[4] = {0, 0, 0, 0};
#pragma unroll
    for (int word = 0; word < 4; ++word) {
        if (word < nwords) {
            const int r0 = __builtin_amdgcn_readlane(cr.rb, a.mode * 5 + word);
            const int r1 = __builtin_amdgcn_readlane(cr.rb, a.mode * 5 + word + 1);
            for (int r = r0; r < r1; ++r) {
                const uint32_t d = run_desc(cr, r);
                const uint32_t kpos = (d >> 8) & 31u, cpos = (d >> 16) & 31u, len = d >> 24;
#pragma unroll
                for (int u = 0; u < 4; ++u) rowv[u] |= __builtin_amdgcn_ubfe(w[u][word], kpos, len) << cpos;
            }
        }
    }
    __syncthreads();  // hash cleared
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + u * NT;
        sr[u] = 0;
        if (e < cnt) {
            const uint32_t row = rowv[u];
            uint32_t s = mix_hash(row) & (uint32_t)(T - 1);
            for (;;) {
                const uint32_t prev = atomicCAS(&L.hkey[s], kNoRow, row);
                if (prev == kNoRow || prev == row) break;
                s = (s + 1) & (uint32_t)(T - 1);
            }
            sr[u] = (s << 16) | atomicAdd(&L.hcnt[s], 1u);
        }
    }
    __syncthreads();
    return cnt;
}

// (count << 16 | occupied) per slot, then one exclusive scan (see seg_hash)
template <int NT>
__device__ __forceinline__ void seg_scan(const SegLds &L, int cnt, uint32_t *wsum) {
    constexpr int T = 4 * NT;
    for (int i = threadIdx.x; i < T; i += NT) {
        const uint32_t c = L.hcnt[i];
        L.hcnt[i] = (c << 16) | (c > 0 ? 1u : 0u);
    }
    __syncthreads();
    block_scan_lds(L.hcnt, T, NT, wsum);
    if (threadIdx.x == 0) {
        // totals: elements = cnt; distinct rows = prefix of the last slot plus its own
        const uint32_t pk = L.hcnt[T - 1];
        L.hcnt[T] = ((uint32_t)cnt << 16) | ((pk & 0xFFFFu) + ((uint32_t)cnt > (pk >> 16) ? 1u : 0u));
    }
    __syncthreads();
}

// The part of the output that a tile's workgroup zeroes for the record
// reduction that follows: slice i of `of` of n floats.
struct ZeroSlice {
    float *p;
    int64_t n, i, of;
};

// The uncached walk over crdg[no][T] (row-grouped factor rows) and valg[T].
// With at most 5 modes every nonzero slot of a step reads all its coordinates
// from LDS first, then issues every factor-row gather, then waits once; with
// more modes the gathers go mode by mode.  NFIX > 0: the tensor has exactly
// NFIX modes (no run-time mode test between the gathers, which would otherwise
// make the compiler wait for one mode's rows before the next mode's gathers
// are issued).
__host__ __device__ constexpr int segp_step(int nmax) { return nmax <= 4 ? 2 : 1; }  // nonzeros of a step
template <int NT, int T, int VEC, int NMAX, int NFIX, bool TIGHT, int FAR>
__device__ __forceinline__ void segp_walk(const MttkrpArgs &a, char *lds, const LaneGroup &lg, const WalkShare &ws,
                                          int cnt, int64_t k0, int nruns, float *__restrict__ rec_val, int ld) {
    constexpr int NO = NMAX - 1;  // non-output modes at most
    constexpr int UB = segp_step(NMAX);
    static_assert(NFIX == 0 || NFIX == NMAX, "a fixed mode count is the maximum");
    const int R = a.rank, mode = a.mode, no = NFIX ? NFIX - 1 : a.nmodes - 1;
    const uint32_t *crdg = reinterpret_cast<const uint32_t *>(lds);
    const float *valg = reinterpret_cast<const float *>(crdg + (size_t)no * T);
    const int c = lg.col;
    // factor of the o-th non-output mode as a row buffer
    RowView<float, FAR == kFarAll> fb[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int k = o + (o >= mode);
        fb[o] = o < no ? RowView<float, FAR == kFarAll>(a.f[k], R, a.frows[k])
                       : RowView<float, FAR == kFarAll>(nullptr, R, 0u);
    }
    auto product = [&](int q, float (&p)[UB][VEC], float (&last)[UB][VEC]) {
        float x[UB];
        load_words<UB>(valg + q, x);
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int v = 0; v < VEC; ++v) p[u][v] = x[u];
        if (NFIX == 0 && no == 0)  // one mode: the empty product
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int v = 0; v < VEC; ++v) last[u][v] = 1.f;
        if constexpr (NO <= 4) {
            uint32_t row[NO][UB];
#pragma unroll
            for (int o = 0; o < NO; ++o)
                if (o < no) load_words<UB>(crdg + o * T + q, row[o]);
            float xv[NO][UB][VEC];
#pragma unroll
            for (int o = 0; o < NO; ++o)
                if (o < no)
#pragma unroll
                    for (int u = 0; u < UB; ++u) fb[o].template load<VEC>(row[o][u], c, xv[o][u]);
#pragma unroll
            for (int o = 0; o < NO; ++o)
                if (o < no)
#pragma unroll
                    for (int u = 0; u < UB; ++u)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            if (o == 0) last[u][v] = xv[0][u][v];
                            else p[u][v] *= xv[o][u][v];
                        }
        } else {
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (o < no) {
                    float xv[UB][VEC];
#pragma unroll
                    for (int u = 0; u < UB; ++u) fb[o].template load<VEC>(crdg[o * T + q + u], c, xv[u]);
#pragma unroll
                    for (int u = 0; u < UB; ++u)
#pragma unroll
                        for (int v = 0; v < VEC; ++v) {
                            if (o == 0) last[u][v] = xv[u][v];
                            else p[u][v] *= xv[u][v];
                        }
                }
            }
        }
    };
    run_walk<float, NT, T, VEC, UB, TIGHT, FAR>(lg, ws, R, cnt, nruns, a.pl_rec + k0, (uint32_t)a.rec_cap, rec_val, ld,
                                                lds, product);
}

// Planned SEGMENT kernel.  The plan holds, per nonzero, its position in the
// tile's row-grouped order (u16), per position whether a run begins there
// (one bit) and per run its record, with the records of one row contiguous.
// A tile is staged by one scatter of values and non-output coordinates to
// their positions; there is no hashing and no scan over nonzeros at run time.
// Records of ld floats go to rec_val.
template <int NT, int T, int VEC, int NMAX, int NFIX, bool TIGHT, int FAR>
__device__ __forceinline__ void segp_tile(const MttkrpArgs &a, int64_t tile, char *lds,
                                          float *__restrict__ rec_val, int ld, const ZeroSlice &zero) {
    constexpr int PER = T / NT;  // nonzeros staged per thread
    static_assert(PER * NT == T && PER >= 1 && PER <= 8, "tile must be 1..8 nonzeros per thread");
    const int nm = NFIX ? NFIX : a.nmodes, mode = a.mode, tid = threadIdx.x;
    uint32_t *crdg = (uint32_t *)lds;
    float *valg = (float *)(crdg + (size_t)(nm - 1) * T);
    const CodecRegs cr = load_codec_regs(a.codec);
    const int64_t k0 = a.pl_off[tile];
    const int nruns = (int)min<int64_t>(a.pl_off[tile + 1] - k0, T);
    const LaneGroup lg = lane_group<VEC>(a.rank);
    const int64_t base = tile * (int64_t)T;
    const int64_t rem = a.nnz - base;
    const int cnt = rem < T ? (int)rem : T;
    const int nwords = 2 * a.codec.key_words;
    uint32_t w[PER][4];
    float v[PER];
    int ps[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int e = tid + u * NT;
        uint64_t klo = 0, khi = 0;
        float x = 0.f;
        int q = 0;
        if (e < cnt) {
            klo = __builtin_nontemporal_load(a.lo + base + e);
            if (nwords == 4) khi = __builtin_nontemporal_load(a.hi + base + e);
            x = __builtin_nontemporal_load(a.vals + base + e);
            q = a.pl_pos[base + e] & (T - 1);  // a position inside the tile
        }
        w[u][0] = (uint32_t)klo;
        w[u][1] = (uint32_t)(klo >> 32);
        w[u][2] = (uint32_t)khi;
        w[u][3] = (uint32_t)(khi >> 32);
        v[u] = x;
        ps[u] = q;
    }
    const WalkShare ws = walk_share<NT, T, TIGHT>(lg, cnt, segp_step(NMAX), a.pl_start + tile * (T / 32));
    zero_slice(zero.p, zero.n, zero.i, zero.of);  // while the loads above are in flight
    // decode the non-output coordinates and scatter them with the values
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
        if (k < nm && k != mode) {
            uint32_t x[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) x[u] = 0;
#pragma unroll
            for (int word = 0; word < 4; ++word) {
                if (word < nwords) {
                    const int r0 = __builtin_amdgcn_readlane(cr.rb, k * 5 + word);
                    const int r1 = __builtin_amdgcn_readlane(cr.rb, k * 5 + word + 1);
                    for (int r = r0; r < r1; ++r) {
                        const uint32_t d = run_desc(cr, r);
                        const uint32_t kpos = (d >> 8) & 31u, cpos = (d >> 16) & 31u, len = d >> 24;
#pragma unroll
                        for (int u = 0; u < PER; ++u) x[u] |= __builtin_amdgcn_ubfe(w[u][word], kpos, len) << cpos;
                    }
                }
            }
            const int o = k - (k > mode);
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (tid + u * NT < cnt) crdg[o * T + ps[u]] = x[u];
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (tid + u * NT < cnt) valg[ps[u]] = v[u];
    if (tid < nm && cnt < T) {  // the other half of an odd last step: row 0, value 0
        if (tid < nm - 1) crdg[tid * T + cnt] = 0;
        else valg[cnt] = 0.f;
    }
    __syncthreads();
    segp_walk<NT, T, VEC, NMAX, NFIX, TIGHT, FAR>(a, lds, lg, ws, cnt, k0, nruns, rec_val, ld);
}

__device__ __forceinline__ ZeroSlice out_slice(const MttkrpArgs &a, int64_t tile, int64_t ntiles) {
    return ZeroSlice{a.out, (int64_t)a.frows[a.mode] * a.rank, tile, ntiles};
}

template <int NT, int T, int VEC, int NMAX, int NFIX, int FAR>
__global__ __launch_bounds__(NT, NMAX <= 5 && FAR != kFarAll ? 8 : 4) void k_mttkrp_segp(MttkrpArgs a, int64_t ntiles) {
    extern __shared__ __align__(16) char lds[];
    const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
    if (tile >= ntiles) return;
    segp_tile<NT, T, VEC, NMAX, NFIX, NMAX == 4 && FAR != kFarAll, FAR>(a, tile, lds, a.rec_val, a.rank,
                                                                       out_slice(a, tile, ntiles));
}

// ---------------------------------------------------------------- row cache
// Tile dictionary (mode-agnostic, tiles of kDictTile nonzeros in key order):
// for every mode k, a tile's distinct mode-k rows, most frequent first, and
// per nonzero the index of its row in that list.  The linearized order keeps
// a tile inside a small sub-box of the index space, so a tile touches few
// distinct rows of every mode (a few hundred per 4096 nonzeros on the ratings
// tensor) and each of them many times.

// Build one mode's dictionary: one workgroup per tile hashes the tile's
// mode-a.mode rows, buckets them by count (64 buckets, counts >= 63 in the
// first), and writes row[off[tile] + i] (i-th most frequent row) and
// slot[e] = i for every nonzero e.  off comes from the counting pass (its
// distinct rows per tile).
template <int NT, int NMAX>
__global__ __launch_bounds__(NT) void k_emit_dict(MttkrpArgs a, const int64_t *__restrict__ off,
                                                  uint32_t *__restrict__ row_out, uint16_t *__restrict__ slot_out) {
    constexpr int T = 4 * NT;
    constexpr int NBK = 64;
    extern __shared__ __align__(16) char lds[];
    __shared__ uint32_t bucket[NBK];
    uint32_t *hkey = (uint32_t *)lds;
    uint32_t *hcnt = hkey + T;
    const int tid = threadIdx.x;
    const int64_t tile = blockIdx.x;
    const int64_t base = tile * (int64_t)T;
    const int64_t rem = a.nnz - base;
    const int cnt = rem < T ? (int)rem : T;
    const int64_t d0 = off[tile], d1 = off[tile + 1];
    for (int i = tid; i < T; i += NT) {
        hkey[i] = kNoRow;
        hcnt[i] = 0;
    }
    if (tid < NBK) bucket[tid] = 0;
    const CodecRegs cr = load_codec_regs(a.codec);
    const int nwords = 2 * a.codec.key_words;
    uint32_t rowv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + u * NT;
        uint32_t w[4] = {0, 0, 0, 0};
        if (e < cnt) {
            const uint64_t klo = a.lo[base + e];
            const uint64_t khi = nwords == 4 ? a.hi[base + e] : 0ull;
            w[0] = (uint32_t)klo;
            w[1] = (uint32_t)(klo >> 32);
            w[2] = (uint32_t)khi;
            w[3] = (uint32_t)(khi >> 32);
        }
        rowv[u] = decode_mode(cr, a.mode, nwords, w);
    }
    __syncthreads();  // hash cleared
    uint32_t hs[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + u * NT;
        hs[u] = 0;
        if (e < cnt) {
            const uint32_t r = rowv[u];
            uint32_t h = mix_hash(r) & (uint32_t)(T - 1);
            for (;;) {
                const uint32_t prev = atomicCAS(&hkey[h], kNoRow, r);
                if (prev == kNoRow || prev == r) break;
                h = (h + 1) & (uint32_t)(T - 1);
            }
            atomicAdd(&hcnt[h], 1u);
            hs[u] = h;
        }
    }
    __syncthreads();
    auto bucket_of = [](uint32_t c) { return c >= (uint32_t)(NBK - 1) ? 0u : (uint32_t)(NBK - 1) - c; };
    for (int i = tid; i < T; i += NT)
        if (hkey[i] != kNoRow) atomicAdd(&bucket[bucket_of(hcnt[i])], 1u);
    __syncthreads();
    if (tid == 0) {
        uint32_t run = 0;
        for (int b = 0; b < NBK; ++b) {
            const uint32_t c = bucket[b];
            bucket[b] = run;
            run += c;
        }
    }
    __syncthreads();
    for (int i = tid; i < T; i += NT) {
        if (hkey[i] != kNoRow) {
            const uint32_t d = atomicAdd(&bucket[bucket_of(hcnt[i])], 1u);
            if (d0 + d < d1) row_out[d0 + d] = hkey[i];
            hcnt[i] = d;  // the slot now holds its row's dictionary index
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + u * NT;
        if (e < cnt) slot_out[base + e] = (uint16_t)hcnt[hs[u]];
    }
}

// Floats of one cached row: a slot for every lane of a group (see LaneGroup),
// so that each lane reads its columns as one aligned vector at any rank.
__host__ __device__ inline int cached_row_floats(int R) { return R < 4 ? R : (R + 3) & ~3; }

// LDS of the row-cached kernel: crdg[nm - 1][T], valg[T], then the cache of
// cap rows per non-output mode.
__host__ __device__ inline size_t segd_lds_bytes(int T, int nmodes, int cap, int R) {
    return segp_lds_bytes(T, nmodes) + (size_t)(nmodes - 1) * cap * cached_row_floats(R) * 4;
}

// Row-cached form of segp_tile (tiles of kDictTile nonzeros).  Staging reads
// no keys: per nonzero the value, its plan position and its dictionary index
// in every non-output mode.  The first cap rows of each non-output mode's
// tile dictionary are copied to LDS; a nonzero whose index is below cap
// reads its factor row there, any other reads it from HBM/L2 by its global
// row.
template <int NT, int T, int VEC, int NMAX, int NFIX, bool TIGHT, int FAR>
__device__ __forceinline__ void segd_tile(const MttkrpArgs &a, int64_t tile, int64_t ntiles, char *lds) {
    constexpr int PER = T / NT;
    constexpr int NO = NMAX - 1;
    static_assert(PER * NT == T && NMAX <= 4, "row cache: 4 modes at most");
    const int nm = NFIX ? NFIX : a.nmodes, mode = a.mode, tid = threadIdx.x, no = nm - 1;
    const int R = a.rank, cap = a.d_cap;
    uint32_t *crdg = (uint32_t *)lds;
    float *valg = (float *)(crdg + (size_t)no * T);
    float *cache = valg + T;
    const int64_t k0 = a.pl_off[tile];
    const int nruns = (int)min<int64_t>(a.pl_off[tile + 1] - k0, T);
    const int64_t base = tile * (int64_t)T;
    const int64_t rem = a.nnz - base;
    const int cnt = rem < T ? (int)rem : T;
    const LaneGroup lg = lane_group<VEC>(R);
    constexpr int UB = 2;
    // every thread stages PER consecutive nonzeros: one 16-byte load of
    // values and one 8-byte load per u16 stream (tiles start at multiples of
    // T, so the vectors are aligned); the last tile's ragged end goes element
    // by element
    static_assert(PER == 4, "row-cached staging loads 4 nonzeros per thread");
    const int e0 = tid * PER;
    float v[PER];
    uint32_t q[PER];
    uint32_t sl[NO][PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        v[u] = 0.f;
        q[u] = 0;
#pragma unroll
        for (int o = 0; o < NO; ++o) sl[o][u] = 0;
    }
    if (e0 + PER <= cnt) {
        const spt_f4 x = __builtin_nontemporal_load(reinterpret_cast<const spt_f4 *>(a.vals + base + e0));
        const spt_u2 w = __builtin_nontemporal_load(reinterpret_cast<const spt_u2 *>(a.pl_pos + base + e0));
        v[0] = x.x;
        v[1] = x.y;
        v[2] = x.z;
        v[3] = x.w;
        q[0] = w.x & 0xFFFFu;
        q[1] = w.x >> 16;
        q[2] = w.y & 0xFFFFu;
        q[3] = w.y >> 16;
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            if (o < no) {
                const spt_u2 d = __builtin_nontemporal_load(reinterpret_cast<const spt_u2 *>(a.d_slot[o] + base + e0));
                sl[o][0] = d.x & 0xFFFFu;
                sl[o][1] = d.x >> 16;
                sl[o][2] = d.y & 0xFFFFu;
                sl[o][3] = d.y >> 16;
            }
        }
    } else {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = e0 + u;
            if (e < cnt) {
                v[u] = a.vals[base + e];
                q[u] = a.pl_pos[base + e];
#pragma unroll
                for (int o = 0; o < NO; ++o)
                    if (o < no) sl[o][u] = a.d_slot[o][base + e];
            }
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) q[u] &= (uint32_t)(T - 1);  // a position inside the tile
    const WalkShare ws = walk_share<NT, T, TIGHT>(lg, cnt, UB, a.pl_start + tile * (T / 32));
    {
        const ZeroSlice z = out_slice(a, tile, ntiles);
        zero_slice(z.p, z.n, z.i, z.of);  // while the loads above are in flight
    }
    // copy the cached rows: the first min(distinct, cap) of each dictionary
    int64_t dbase[NO];
    int dn[NO], dlast[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        dbase[o] = 0;
        dn[o] = 0;
        dlast[o] = 0;
        if (o < no) {
            dbase[o] = a.d_off[o][tile];
            const int64_t d = a.d_off[o][tile + 1] - dbase[o];  // distinct rows of the tile
            dn[o] = (int)min<int64_t>(d, (int64_t)cap);
            dlast[o] = (int)max<int64_t>(d - 1, 0);
        }
    }
    const int RS = cached_row_floats(R), slots = RS / VEC;
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        if (o < no) {
            const float *f = a.f[o + (o >= mode)];
            const uint32_t *dr = a.d_row[o] + dbase[o];
            float *cb = cache + (size_t)o * cap * RS;
            for (int i = tid; i < dn[o] * slots; i += NT) {
                const int sidx = i / slots, jj = i - sidx * slots;
                float x[VEC];
                load_vec_any<VEC>(f + (size_t)dr[sidx] * R + (VEC == 4 ? min(4 * jj, R - 4) : jj), x);
                store_vec<VEC>(cb + (size_t)sidx * RS + VEC * jj, x);
            }
        }
    }
    // scatter: cached rows by their byte offset in LDS, the others by global
    // row with kDictMiss set.  The global rows of all PER nonzeros are loaded
    // before the first LDS store, so the thread waits for them once.
    const uint32_t cache_off = (uint32_t)(reinterpret_cast<const char *>(cache) - lds);
    uint32_t grow[NO][PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            grow[o][u] = 0;
            if (o < no && e0 + u < cnt) grow[o][u] = a.d_row[o][dbase[o] + min(sl[o][u], (uint32_t)dlast[o])];
        }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (e0 + u < cnt) {
            valg[q[u]] = v[u];
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (o < no) {
                    const uint32_t si = min(sl[o][u], (uint32_t)dlast[o]);
                    crdg[o * T + q[u]] = (int)si < dn[o] ? cache_off + ((uint32_t)(o * cap) + si) * (uint32_t)(RS * 4)
                                                         : (grow[o][u] | kDictMiss);
                }
            }
        }
    }
    if (tid <= no && cnt < T) {  // the other half of an odd last step: a cached row, value 0
        if (tid < no) crdg[tid * T + cnt] = cache_off;
        else valg[cnt] = 0.f;
    }
    __syncthreads();
    // the largest entry a cached row can have: the last slot of the last mode
    const uint32_t lim = cache_off + ((uint32_t)(no * cap) - 1u) * (uint32_t)(RS * 4);
    // A crdg entry is either the byte offset in LDS of a cached row or, with
    // kDictMiss set, a global row.  Every lane first reads LDS (a miss reads
    // the last cached row: its entry, flag set, clamps to lim), then the
    // misses load their rows globally into the same registers.  A global load
    // into the registers of an LDS read waits for that read; with all LDS
    // reads of the step issued first the loads wait for one LDS round trip,
    // and no branch splits hits from misses.
    RowView<float, FAR == kFarAll> fb[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int k = o + (o >= mode);
        fb[o] = o < no ? RowView<float, FAR == kFarAll>(a.f[k], R, a.frows[k])
                       : RowView<float, FAR == kFarAll>(nullptr, R, 0u);
    }
    const char *mine = lds + lg.j * VEC * 4;  // this lane's columns of the row at offset 0
    auto product = [&](int q0, float (&p)[UB][VEC], float (&last)[UB][VEC]) {
        uint32_t row[NO][UB];
        float x[UB];
        load_words<UB>(valg + q0, x);
#pragma unroll
        for (int o = 0; o < NO; ++o)
            if (o < no) load_words<UB>(crdg + o * T + q0, row[o]);
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int v = 0; v < VEC; ++v) p[u][v] = x[u];
        float xv[NO][UB][VEC];
        // every index read of the step is issued before anything waits for
        // one (the scheduler may not hoist a use between them)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < NO; ++o)
#pragma unroll
            for (int u = 0; u < UB; ++u)
                if (o < no) load_vec<VEC>(reinterpret_cast<const float *>(mine + min(row[o][u], lim)), xv[o][u]);
#pragma unroll
        for (int o = 0; o < NO; ++o)
            if (o < no)
#pragma unroll
                for (int u = 0; u < UB; ++u)
                    if (row[o][u] & kDictMiss) fb[o].template load<VEC>(row[o][u] & ~kDictMiss, lg.col, xv[o][u]);
#pragma unroll
        for (int o = 0; o < NO; ++o)
            if (o < no)
#pragma unroll
                for (int u = 0; u < UB; ++u)
#pragma unroll
                    for (int v = 0; v < VEC; ++v) {
                        if (o == 0) last[u][v] = xv[0][u][v];
                        else p[u][v] *= xv[o][u][v];
                    }
    };
    run_walk<float, NT, T, VEC, UB, TIGHT, FAR>(lg, ws, R, cnt, nruns, a.pl_rec + k0, (uint32_t)a.rec_cap, a.rec_val, R,
                                                lds, product);
}

// Bounded to 64 VGPRs, which leaves two workgroups of 16 waves to a CU: left to
// itself the compiler takes 72 to 82 and one workgroup; the few spills lie
// outside the steps.
template <int NT, int T, int VEC, int NMAX, int NFIX, int FAR>
__global__ __launch_bounds__(NT, FAR == kFarAll ? 4 : 8) void k_mttkrp_segd(MttkrpArgs a, int64_t ntiles) {
    extern __shared__ __align__(16) char lds[];
    const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
    if (tile >= ntiles) return;
    segd_tile<NT, T, VEC, NMAX, NFIX, NMAX == 4 && FAR != kFarAll, FAR>(a, tile, ntiles, lds);
}

// Batched: tile `it` of the whole batch belongs to the last item whose
// first_tile <= it.
__device__ __forceinline__ int seg_item_of(const SegItem *__restrict__ items, int count, int64_t it) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].first_tile <= it) lo = mid;
        else hi = mid - 1;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// Every tensor's records start at its rec_base in the batch's record array,
// its rows at row_base of the concatenated output (records of the whole batch
// stay grouped by row: tensors are laid out in order).
// Persistent: a grid sized to the resident workgroups pulls the batch's tiles
// (T = 4 NT nonzeros each, over all tensors in order) from the counter
// *next_tile, zero at launch, until the counter passes total_tiles.  A
// workgroup's tiles only increase, so it finds each tile's tensor by moving
// forward from the last one.
// 3 and 4 modes take the walk of their mode count, all of whose gathers are in
// flight together, without a branch round each.  Bounded to 128 VGPRs (two
// workgroups of 8 waves to a CU): at 64, 72 and 80, with 4, 3 and 3
// workgroups, the spills cost more than the waves bring (32 members of 10k to
// 5M nonzeros, ranks 16 and 32, 10 iterations: 40.5, 40.9 and 36.3 ms, here
// 31.7, and 33.0 with one walk for all mode counts at 72).
template <int NT, int VEC, int NMAX, int NFIX, int FAR>
__global__ __launch_bounds__(NT, 4) void k_mttkrp_segp_batched(const SegItem *__restrict__ items, int count,
                                                            int64_t total_tiles, float *__restrict__ rec_val, int ld,
                                                            unsigned long long *__restrict__ next_tile,
                                                            float *__restrict__ out, int64_t out_floats) {
    extern __shared__ __align__(16) char lds[];
    __shared__ int64_t s_tile;
    int b = 0;
    for (;;) {
        if (threadIdx.x == 0) s_tile = (int64_t)atomicAdd(next_tile, 1ull);
        __syncthreads();  // also: every wave is done with the previous tile's LDS
        // the same for all lanes, and known to be: an item's fields stay in scalar registers
        const int64_t it = (int64_t)__builtin_amdgcn_readfirstlane((int)s_tile) & 0xFFFFFFFFll |
                           (int64_t)__builtin_amdgcn_readfirstlane((int)(s_tile >> 32)) << 32;
        __syncthreads();  // every thread has read s_tile before it is replaced
        if (it >= total_tiles) break;
        while (b + 1 < count && items[b + 1].first_tile <= it) ++b;
        const SegItem &item = items[b];
        const ZeroSlice zero{out, out_floats, it, total_tiles};
        float *rv = rec_val + item.rec_base * ld;
        if (NMAX == 4 && NFIX == 0 && item.a.nmodes == 4)
            segp_tile<NT, 4 * NT, VEC, 4, 4, false, FAR>(item.a, it - item.first_tile, lds, rv, ld, zero);
        else if (NMAX == 4 && NFIX == 0 && item.a.nmodes == 3)
            segp_tile<NT, 4 * NT, VEC, 3, 3, false, FAR>(item.a, it - item.first_tile, lds, rv, ld, zero);
        else
            segp_tile<NT, 4 * NT, VEC, NMAX, NFIX, false, FAR>(item.a, it - item.first_tile, lds, rv, ld, zero);
    }
}

// The plan of one tile: positions to pos (the tensor's), run starts to start
// (the tile's words), and the row (row_base + row) of every run, in position
// order, to pair_key at gpair.
template <int NT>
__device__ __forceinline__ void emit_tile(const MttkrpArgs &a, int64_t tile, char *lds, uint32_t *wsum,
                                          uint16_t *__restrict__ pos, RunWord *__restrict__ start, int64_t gpair,
                                          int64_t row_base, uint64_t *__restrict__ pair_key) {
    constexpr int T = 4 * NT;
    const SegLds L = seg_carve_plan(lds, T);
    const CodecRegs cr = load_codec_regs(a.codec);
    for (int i = threadIdx.x; i < T / 32; i += NT) L.bits[i] = 0;
    uint32_t sr[4];
    const int cnt = seg_hash<NT>(a, tile, L, cr, wsum, sr);
    seg_scan<NT>(L, cnt, wsum);
    const int64_t base = tile * (int64_t)T;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + u * NT;
        if (e < cnt) pos[base + e] = (uint16_t)((L.hcnt[sr[u] >> 16] >> 16) + (sr[u] & 0xFFFFu));
    }
    for (int i = threadIdx.x; i < T; i += NT) {
        const uint32_t pk = L.hcnt[i];
        if (L.hkey[i] != kNoRow) {
            pair_key[gpair + (pk & 0xFFFFu)] = (uint64_t)(row_base + L.hkey[i]);
            const uint32_t p = pk >> 16;
            atomicOr(&L.bits[p >> 5], 1u << (p & 31));
        }
    }
    __syncthreads();
    // 32 positions a word, and the starts before it: a scan by the first wave
    if (threadIdx.x < 64) {
        constexpr int NW = T / 32, PER = (NW + 63) / 64;
        const int lane = threadIdx.x;
        uint32_t w[PER], c = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            w[i] = lane * PER + i < NW ? L.bits[lane * PER + i] : 0u;
            c += __popc(w[i]);
        }
        uint32_t x = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        uint32_t run = x - c;
#pragma unroll
        for (int i = 0; i < PER; ++i)
            if (lane * PER + i < NW) {
                RunWord r;
                r.x = w[i];
                r.y = run;
                start[lane * PER + i] = r;
                run += __popc(w[i]);
            }
    }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_emit_plan(MttkrpArgs a, const int64_t *__restrict__ pair_off,
                                                  uint16_t *__restrict__ pos, RunWord *__restrict__ start,
                                                  uint64_t *__restrict__ pair_key) {
    extern __shared__ __align__(16) char lds[];
    __shared__ uint32_t wsum[NT / 64];
    const int64_t tile = blockIdx.x;
    emit_tile<NT>(a, tile, lds, wsum, pos, start + tile * (4 * NT / 32), pair_off[tile], 0, pair_key);
}

// Batched emission: item b's plan arrays come in its args (pl_pos, pl_start);
// gpair_off gives each global tile's first pair in the batch-wide array; pair
// keys are rows of the concatenated output (row_base + row).
template <int NT>
__global__ __launch_bounds__(NT) void k_emit_plan_batched(const SegItem *__restrict__ items, int count,
                                                          const int64_t *__restrict__ gpair_off,
                                                          uint64_t *__restrict__ pair_key) {
    extern __shared__ __align__(16) char lds[];
    __shared__ uint32_t wsum[NT / 64];
    const int64_t it = blockIdx.x;
    const int b = seg_item_of(items, count, it);
    const SegItem &item = items[b];
    const MttkrpArgs &a = item.a;
    const int64_t tile = it - item.first_tile;
    emit_tile<NT>(a, tile, lds, wsum, const_cast<uint16_t *>(a.pl_pos),
                  const_cast<RunWord *>(a.pl_start) + tile * (4 * NT / 32), gpair_off[it], item.row_base, pair_key);
}

// Item of the batch-wide pair or record g: the last whose rec_base <= g.
__device__ __forceinline__ int seg_item_of_record(const SegItem *__restrict__ items, int count, int64_t g) {
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].rec_base <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The sorted pairs of a batch: record j (its row sorted[j] of the concatenated
// output, its run idx[j]) becomes record j - rec_base of its tensor.
__global__ __launch_bounds__(256) void k_plan_records_batched(const SegItem *__restrict__ items, int count,
                                                              const uint64_t *__restrict__ sorted,
                                                              const uint32_t *__restrict__ idx, int64_t n) {
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
        const SegItem &item = items[seg_item_of_record(items, count, j)];
        const_cast<uint64_t *>(item.a.pl_rec_row)[j - item.rec_base] = sorted[j] - (uint64_t)item.row_base;
        const_cast<uint32_t *>(item.a.pl_rec)[(int64_t)idx[j] - item.rec_base] = (uint32_t)(j - item.rec_base);
    }
}

// Rows of a batch's records in its concatenated output.
__global__ __launch_bounds__(256) void k_record_rows_batched(const SegItem *__restrict__ items, int count, int64_t n,
                                                             uint64_t *__restrict__ rows) {
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256) {
        const SegItem &item = items[seg_item_of_record(items, count, j)];
        rows[j] = item.a.pl_rec_row[j - item.rec_base] + (uint64_t)item.row_base;
    }
}

// rec[idx[j]] = j: the record of the run that sorted to place j
__global__ __launch_bounds__(256) void k_plan_records(const uint32_t *__restrict__ idx, uint32_t *__restrict__ rec,
                                                      int64_t n) {
    for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n; j += (int64_t)gridDim.x * 256)
        rec[idx[j]] = (uint32_t)j;
}

// pieces of at most kPiece nonzeros | distinct rows << 32 of a hashed tile
template <int NT>
__device__ __forceinline__ void count_tile(const MttkrpArgs &a, int64_t tile, char *lds, uint32_t *wsum, int64_t *out) {
    constexpr int T = 4 * NT;
    __shared__ uint32_t total[2];
    if (threadIdx.x < 2) total[threadIdx.x] = 0;
    const SegLds L = seg_carve_plan(lds, T);
    const CodecRegs cr = load_codec_regs(a.codec);
    uint32_t sr[4];
    (void)seg_hash<NT>(a, tile, L, cr, wsum, sr);
    uint32_t np = 0, d = 0;
    for (int i = threadIdx.x; i < T; i += NT) {
        const uint32_t c = L.hcnt[i];
        np += (c + kPiece - 1) / kPiece;
        d += c > 0;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        np += __shfl_down(np, off, 64);
        d += __shfl_down(d, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&total[0], np);
        atomicAdd(&total[1], d);
    }
    __syncthreads();
    if (threadIdx.x == 0) *out = (int64_t)total[0] | ((int64_t)total[1] << 32);
}

// Pieces and distinct rows of every tile (the plan's counting pass).
template <int NT>
__global__ __launch_bounds__(NT) void k_count_pieces(MttkrpArgs a, int64_t *__restrict__ out) {
    extern __shared__ __align__(16) char lds[];
    __shared__ uint32_t wsum[NT / 64];
    count_tile<NT>(a, blockIdx.x, lds, wsum, out + blockIdx.x);
}

template <int NT>
__global__ __launch_bounds__(NT) void k_count_pieces_batched(const SegItem *__restrict__ items, int count,
                                                             int64_t *__restrict__ out) {
    extern __shared__ __align__(16) char lds[];
    __shared__ uint32_t wsum[NT / 64];
    const int64_t it = blockIdx.x;
    const int b = seg_item_of(items, count, it);
    count_tile<NT>(items[b].a, it - items[b].first_tile, lds, wsum, out + it);
}

template <int NT, int T, int NMAX, int NFIX, int VEC, int FAR>
spt_status launch_seg_k(const MttkrpArgs &a, int64_t ntiles, hipStream_t s) {
    if constexpr (T == kDictTile && NMAX <= 4) {
        if (a.d_cap > 0) {
            const size_t lds = segd_lds_bytes(T, a.nmodes, a.d_cap, a.rank);
            hipLaunchKernelGGL((k_mttkrp_segd<NT, T, VEC, NMAX, NFIX, FAR>), dim3((unsigned)ntiles), dim3(NT), lds, s, a,
                               ntiles);
            SPT_HIP(hipGetLastError());
            return SPT_OK;
        }
    }
    const size_t lds = std::max(segp_lds_bytes(T, a.nmodes), walk_lds_bytes(NT));
    hipLaunchKernelGGL((k_mttkrp_segp<NT, T, VEC, NMAX, NFIX, FAR>), dim3((unsigned)ntiles), dim3(NT), lds, s, a, ntiles);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

}  // namespace

// What a call on `a` reads or writes (records of ld columns) beyond the 4 GiB
// that a structured buffer's 32-bit offsets reach (RowView): rows past them
// would come around to the array's start.  Records get there where labels are
// in no order (150M nonzeros of rank 64, shuffled, modes 1 and 2), so those
// kernels are the others but for the records' addresses: 5.23 and 5.62 ms a
// call, 7.65 and 7.97 in the general kernel with 64-bit addresses throughout.
// Factors that large take that one (FP64, 20M rows of rank 32, 20M nonzeros:
// 1.58 and 1.11 ms for the modes that gather them; 2.67 and 1.94 with one column
// a lane and one nonzero in flight).
SegFar seg_far(const MttkrpArgs &a, int ld, size_t item) {
    for (int k = 0; k < a.nmodes; ++k)
        if (k != a.mode && (uint64_t)a.frows[k] * a.rank * item > kBufferBytes) return kFarAll;
    return (uint64_t)a.rec_cap * ld * item > kBufferBytes ? kFarRecords : kNear;
}

// tile sizes served: 1024 (256 threads), 2048 (512), 4096 (1024 threads)
bool seg_tile_ok(int tile, int nmodes) {
    if (tile != 1024 && tile != 2048 && tile != 4096) return false;
    return seg_lds_bytes(tile, nmodes) <= 160 * 1024 - 1024 && segp_lds_bytes(tile, nmodes) <= 160 * 1024 - 1024;
}

spt_status launch_emit_plan(const MttkrpArgs &a, const int64_t *pair_off, uint16_t *pos, spt_u2 *start,
                            uint64_t *pair_key, hipStream_t s) {
    const int64_t ntiles = (a.nnz + a.tile - 1) / a.tile;
    if (ntiles == 0) return SPT_OK;
    if (!seg_tile_ok(a.tile, a.nmodes)) return fail(SPT_E_INVALID_ARG, "segment: tile does not fit LDS");
    const dim3 g((unsigned)ntiles);
    const size_t lds = seg_plan_lds_bytes(a.tile);
    if (a.tile == 1024) hipLaunchKernelGGL(k_emit_plan<256>, g, dim3(256), lds, s, a, pair_off, pos, start, pair_key);
    else if (a.tile == 2048) hipLaunchKernelGGL(k_emit_plan<512>, g, dim3(512), lds, s, a, pair_off, pos, start, pair_key);
    else hipLaunchKernelGGL(k_emit_plan<1024>, g, dim3(1024), lds, s, a, pair_off, pos, start, pair_key);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_plan_records(const uint32_t *idx, uint32_t *rec, int64_t n, hipStream_t s) {
    if (n == 0) return SPT_OK;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_plan_records, dim3((unsigned)g), dim3(256), 0, s, idx, rec, n);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_count_pieces(const MttkrpArgs &a, int64_t *counts, hipStream_t s) {
    const int64_t ntiles = (a.nnz + a.tile - 1) / a.tile;
    if (ntiles == 0) return SPT_OK;
    if (!seg_tile_ok(a.tile, a.nmodes)) return fail(SPT_E_INVALID_ARG, "segment: tile does not fit LDS");
    const dim3 g((unsigned)ntiles);
    const size_t lds = seg_plan_lds_bytes(a.tile);
    if (a.tile == 1024) hipLaunchKernelGGL(k_count_pieces<256>, g, dim3(256), lds, s, a, counts);
    else if (a.tile == 2048) hipLaunchKernelGGL(k_count_pieces<512>, g, dim3(512), lds, s, a, counts);
    else hipLaunchKernelGGL(k_count_pieces<1024>, g, dim3(1024), lds, s, a, counts);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

namespace {
// 3, 4 and 5 modes get a kernel with the mode count fixed; others, and factors
// past the reach of a structured buffer, a general one
template <int NT, int T, int VEC, int FAR>
spt_status launch_seg_nm(const MttkrpArgs &a, int64_t ntiles, hipStream_t s) {
    const int nm = a.nmodes;
    if (nm == 3) return launch_seg_k<NT, T, 3, 3, VEC, FAR>(a, ntiles, s);
    if (nm == 4) return launch_seg_k<NT, T, 4, 4, VEC, FAR>(a, ntiles, s);
    if (nm == 5) return launch_seg_k<NT, T, 5, 5, VEC, FAR>(a, ntiles, s);
    return nm < 3 ? launch_seg_k<NT, T, 3, 0, VEC, FAR>(a, ntiles, s) : launch_seg_k<NT, T, 8, 0, VEC, FAR>(a, ntiles, s);
}

template <int NT, int T, int VEC>
spt_status launch_seg_far(const MttkrpArgs &a, int64_t ntiles, hipStream_t s) {
    return a.nmodes <= 4 ? launch_seg_k<NT, T, 4, 0, VEC, kFarAll>(a, ntiles, s)
                         : launch_seg_k<NT, T, 8, 0, VEC, kFarAll>(a, ntiles, s);
}

template <int NT, int T>
spt_status launch_seg_tile(const MttkrpArgs &a, int64_t ntiles, hipStream_t s) {
    const SegFar far = seg_far(a, a.rank, sizeof(float));
    if (a.rank < 4) return far == kNear ? launch_seg_nm<NT, T, 1, kNear>(a, ntiles, s) : launch_seg_far<NT, T, 1>(a, ntiles, s);
    if (far == kNear) return launch_seg_nm<NT, T, 4, kNear>(a, ntiles, s);
    return far == kFarRecords ? launch_seg_nm<NT, T, 4, kFarRecords>(a, ntiles, s) : launch_seg_far<NT, T, 4>(a, ntiles, s);
}
}  // namespace

spt_status launch_emit_dict(const MttkrpArgs &a, const int64_t *off, uint32_t *rows, uint16_t *slots, hipStream_t s) {
    const int64_t ntiles = (a.nnz + kDictTile - 1) / kDictTile;
    if (ntiles == 0) return SPT_OK;
    constexpr int NT = kDictTile / 4;
    const size_t lds = (size_t)kDictTile * 8;
    hipLaunchKernelGGL((k_emit_dict<NT, 8>), dim3((unsigned)ntiles), dim3(NT), lds, s, a, off, rows, slots);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

int dict_cap(int nmodes, int rank) {
    if (nmodes < 2 || nmodes > 4) return 0;
    const size_t fixed = segp_lds_bytes(kDictTile, nmodes);
    if (fixed >= kDictLdsBudget) return 0;
    const size_t cap = (kDictLdsBudget - fixed) / ((size_t)(nmodes - 1) * cached_row_floats(rank) * 4);
    return cap >= (size_t)kDictMinCap ? (int)std::min<size_t>(cap, kDictTile) : 0;
}

spt_status launch_mttkrp_seg(const MttkrpArgs &a, hipStream_t s) {
    const int64_t ntiles = (a.nnz + a.tile - 1) / a.tile;
    if (ntiles == 0) return SPT_OK;
    if (!seg_tile_ok(a.tile, a.nmodes)) return fail(SPT_E_INVALID_ARG, "segment: tile does not fit LDS");
    if (!a.pl_pos || !a.pl_off || !a.pl_start || !a.pl_rec) return fail(SPT_E_INVALID_ARG, "segment: no plan");
    if (a.tile == 1024) return launch_seg_tile<256, 1024>(a, ntiles, s);
    if (a.tile == 2048) return launch_seg_tile<512, 2048>(a, ntiles, s);
    return launch_seg_tile<kSegpThreads4096, 4096>(a, ntiles, s);
}

namespace {
template <int NT, int NMAX, int NFIX, int VEC, int FAR>
spt_status launch_segb_k(const SegItem *items, int count, int64_t total_tiles, float *rec_val,
                         int ld, unsigned long long *next_tile, float *out, int64_t out_floats, hipStream_t s) {
    const size_t lds = std::max(segp_lds_bytes(4 * NT, NMAX), walk_lds_bytes(NT));
    static std::atomic<int> per_cu{0};  // resident workgroups per CU (fixed per instantiation: its LDS is)
    int pc = per_cu.load(std::memory_order_relaxed);
    if (pc == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &pc, reinterpret_cast<const void *>(&k_mttkrp_segp_batched<NT, VEC, NMAX, NFIX, FAR>), NT, lds) !=
                hipSuccess ||
            pc < 1) {
            (void)hipGetLastError();  // not a failure of this call: one resident workgroup per CU is assumed
            pc = 1;
        }
        per_cu.store(pc, std::memory_order_relaxed);
    }
    const int64_t grid = std::min<int64_t>(total_tiles, (int64_t)pc * device_cus());
    spt_status st = launch_fill_zero(reinterpret_cast<float *>(next_tile), 2, s);  // the tile counter
    if (st != SPT_OK) return st;
    hipLaunchKernelGGL((k_mttkrp_segp_batched<NT, VEC, NMAX, NFIX, FAR>), dim3((unsigned)grid), dim3(NT), lds, s, items,
                       count, total_tiles, rec_val, ld, next_tile, out, out_floats);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

template <int NT, int VEC, int FAR>
spt_status launch_segb_t(const SegItem *items, int count, int64_t total_tiles, const BatchShape &b, float *rec_val,
                         unsigned long long *next_tile, float *out, int64_t out_floats, hipStream_t s) {
    auto go = [&](auto launch) { return launch(items, count, total_tiles, rec_val, b.ld, next_tile, out, out_floats, s); };
    if (b.nmodes_min == 3 && b.nmodes_max == 3) return go(launch_segb_k<NT, 3, 3, VEC, FAR>);
    return b.nmodes_max <= 4 ? go(launch_segb_k<NT, 4, 0, VEC, FAR>) : go(launch_segb_k<NT, 8, 0, VEC, FAR>);
}

template <int NT>
spt_status launch_segb_n(const SegItem *items, int count, int64_t total_tiles, const BatchShape &b, float *rec_val,
                         unsigned long long *next_tile, float *out, int64_t out_floats, hipStream_t s) {
    auto go = [&](auto launch) { return launch(items, count, total_tiles, b, rec_val, next_tile, out, out_floats, s); };
    if (!b.vec4) return b.far == kNear ? go(launch_segb_t<NT, 1, kNear>) : go(launch_segb_t<NT, 1, kFarAll>);
    if (b.far == kNear) return go(launch_segb_t<NT, 4, kNear>);
    return b.far == kFarRecords ? go(launch_segb_t<NT, 4, kFarRecords>) : go(launch_segb_t<NT, 4, kFarAll>);
}

}  // namespace

bool seg_batch_fits(int nmodes_max, int tile) { return seg_tile_ok(tile, nmodes_max); }

spt_status launch_emit_plan_batched(const SegItem *items, int count, int64_t total_tiles, int nmodes_max, int tile,
                                    const int64_t *gpair_off, uint64_t *pair_key, hipStream_t s) {
    if (total_tiles == 0) return SPT_OK;
    if (!seg_batch_fits(nmodes_max, tile)) return fail(SPT_E_INVALID_ARG, "batch plan: tile does not fit LDS");
    const dim3 g((unsigned)total_tiles);
    const size_t lds = seg_plan_lds_bytes(tile);
    if (tile == 1024) hipLaunchKernelGGL(k_emit_plan_batched<256>, g, dim3(256), lds, s, items, count, gpair_off, pair_key);
    else if (tile == 2048) hipLaunchKernelGGL(k_emit_plan_batched<512>, g, dim3(512), lds, s, items, count, gpair_off, pair_key);
    else hipLaunchKernelGGL(k_emit_plan_batched<1024>, g, dim3(1024), lds, s, items, count, gpair_off, pair_key);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_plan_records_batched(const SegItem *items, int count, const uint64_t *sorted, const uint32_t *idx,
                                       int64_t n, hipStream_t s) {
    if (n == 0) return SPT_OK;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_plan_records_batched, dim3((unsigned)g), dim3(256), 0, s, items, count, sorted, idx, n);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_record_rows_batched(const SegItem *items, int count, int64_t n, uint64_t *rows, hipStream_t s) {
    if (n == 0) return SPT_OK;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_record_rows_batched, dim3((unsigned)g), dim3(256), 0, s, items, count, n, rows);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_count_pieces_batched(const SegItem *items, int count, int64_t total_tiles, int nmodes_max, int tile,
                                       int64_t *counts, hipStream_t s) {
    if (total_tiles == 0) return SPT_OK;
    if (!seg_batch_fits(nmodes_max, tile)) return fail(SPT_E_INVALID_ARG, "batch plan: tile does not fit LDS");
    const dim3 g((unsigned)total_tiles);
    const size_t lds = seg_plan_lds_bytes(tile);
    if (tile == 1024) hipLaunchKernelGGL(k_count_pieces_batched<256>, g, dim3(256), lds, s, items, count, counts);
    else if (tile == 2048) hipLaunchKernelGGL(k_count_pieces_batched<512>, g, dim3(512), lds, s, items, count, counts);
    else hipLaunchKernelGGL(k_count_pieces_batched<1024>, g, dim3(1024), lds, s, items, count, counts);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_mttkrp_seg_batched(const SegItem *items, int count, int64_t total_tiles, const BatchShape &b,
                                     float *rec_val, unsigned long long *next_tile, float *out, int64_t out_floats,
                                     hipStream_t s) {
    if (total_tiles == 0) return SPT_OK;
    if (b.ld > 64) return fail(SPT_E_INVALID_ARG, "batched MTTKRP: rank above 64");
    if (!seg_batch_fits(b.nmodes_max, b.tile)) return fail(SPT_E_INVALID_ARG, "batched MTTKRP: tile does not fit LDS");
    if (!next_tile) return fail(SPT_E_INVALID_ARG, "batched MTTKRP: no tile counter");
    auto go = [&](auto launch) { return launch(items, count, total_tiles, b, rec_val, next_tile, out, out_floats, s); };
    return b.tile == 1024 ? go(launch_segb_n<256>) : b.tile == 2048 ? go(launch_segb_n<512>) : go(launch_segb_n<1024>);
}

}  // namespace spt
