// Linearized-tensor construction on gfx950 (Section III-C, problem formulation):
// bit deposit of every coordinate into an l(p)-bit key, then a stable LSD radix
// sort of (key, input index) over the l(p) significant bits, then the value
// gather and the FP64 sum of squares.
//
// Radix sort design (one pass per 8-bit digit, tiles of 8 elements a thread):
//   hist    : per tile, a 256-bin digit histogram in LDS (the first pass's comes
//             with the bit deposit)
//   scan    : one workgroup per digit scans the tiles' counts (digit-major array)
//   scatter : each wave ranks a contiguous span of the tile stably on its own
//             (ballots order equal digits by lane, the wave's LDS counters carry
//             them across rounds), one barrier merges the waves' counts, then the
//             tile is regrouped by digit in LDS and runs of equal digit are written
//             contiguously so global stores coalesce.  Keys and indices go through
//             the same LDS one after the other.  The last pass also moves the
//             values and sums their squares.
// Bound by memory: a pass over 30M 64-bit keys moves 720 MB in 177 us and its
// histogram reads 240 MB in 52 us (4.1 and 4.6 TB/s; a copy reaches 4.8).  With
// 256 threads and 55 KB of LDS to a 4096-element tile, tiles dealt round the
// dies, masks built from 64-bit selects and the values gathered by a launch of
// their own the passes took 242 and 72 us and the gather 575 us.
#include "tile_common.h"

namespace spt {

namespace {

constexpr int kThreads = 256;

// Tiles of the sort: threads of a workgroup and elements of each.  A large
// tile writes longer runs of equal digit (8192 elements: 256 bytes of keys), a
// small one has more workgroups and a shorter chain in each.  Encode, export
// and decode at tiles of 512 x 4 / 512 x 8 / 1024 x 8: 200k elements (3 key
// bytes) 184 / 200 / 234 us, 5M (8) 574 / 539 / 564 us, 30M (8) 3.29 / 2.96 /
// 2.80 ms; 128-bit keys (10 bytes) 1M 326 / 334 / 439 us, 6M 949 / 937 / 1254
// us, 20M 3.55 / 3.10 / 3.71 ms (1024 x 8 does not fit 64 VGPRs there).
struct RadixTile {
    int threads, items;
};
constexpr RadixTile kRadixSmall = {512, 4};
template <int KW>
constexpr RadixTile kRadixLarge = {KW == 2 ? 512 : 1024, 8};
constexpr int64_t kRadixLargeFrom = 4 << 20;

constexpr RadixTile radix_tile(int key_words, int64_t n) {
    return n < kRadixLargeFrom ? kRadixSmall : key_words == 2 ? kRadixLarge<2> : kRadixLarge<1>;
}

int64_t radix_tiles(int64_t n, RadixTile t) { return (n + t.threads * t.items - 1) / (t.threads * t.items); }

struct DimsArg {
    uint32_t d[kMaxModes];
};

// What the host reads back after an encode.
struct EncodeResult {
    int bad;  // out-of-range nonzeros
    int pad;
    unsigned long long first;  // smallest of them << 8 | its mode
    double norm_x2;
};

// Bins of a tile's histogram in LDS: one set for every four waves.
template <int THREADS>
struct TileHist {
    static constexpr int kSets = THREADS / 256;
    uint32_t h[kSets][256];
};

template <int THREADS>
__device__ __forceinline__ void hist_store(const TileHist<THREADS> &t, uint32_t *counts, int64_t b, int nblocks) {
    const int tid = threadIdx.x;
    if (tid < 256) {
        uint32_t x = 0;
#pragma unroll
        for (int w = 0; w < TileHist<THREADS>::kSets; ++w) x += t.h[w][tid];
        counts[(int64_t)tid * nblocks + b] = x;
    }
}

// key = interleave(coords), the histogram of the first digit, and the nonzeros
// out of range.  Each thread takes kDepositU nonzeros per round: all their
// coordinates are loaded before any key is formed, and every bit run of the
// codec is applied to all of them.
constexpr int kDepositU = 4;
template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS, 8) void k_deposit(const uint32_t *__restrict__ coords, int64_t nnz, DimsArg dims,
                                                     Codec codec, uint64_t *__restrict__ lo,
                                                     uint64_t *__restrict__ hi, EncodeResult *__restrict__ res,
                                                     uint32_t *__restrict__ counts, int nblocks) {
    __shared__ TileHist<THREADS> hist;
    const CodecRegs cl = load_codec_regs(codec);
    const int nm = codec.nmodes, tid = threadIdx.x;
    const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
    hist.h[tid >> 8][tid & 255] = 0;
    __syncthreads();
#pragma unroll 1
    for (int round = 0; round < ITEMS / kDepositU; ++round) {
        const int64_t e0 = b * (THREADS * ITEMS) + round * (THREADS * kDepositU) + tid;
        uint32_t c[kMaxModes][kDepositU];
#pragma unroll
        for (int n = 0; n < kMaxModes; ++n)
#pragma unroll
            for (int u = 0; u < kDepositU; ++u) {
                const int64_t e = e0 + u * THREADS;
                c[n][u] = 0;
                if (n < nm && e < nnz) c[n][u] = __builtin_nontemporal_load(coords + (int64_t)n * nnz + e);
            }
        uint32_t w[kDepositU][4];
#pragma unroll
        for (int u = 0; u < kDepositU; ++u) w[u][0] = w[u][1] = w[u][2] = w[u][3] = 0;
#pragma unroll
        for (int n = 0; n < kMaxModes; ++n) {
            if (n < nm) {
#pragma unroll
                for (int u = 0; u < kDepositU; ++u) {
                    const int64_t e = e0 + u * THREADS;
                    if (e < nnz && c[n][u] >= dims.d[n]) {
                        atomicAdd(&res->bad, 1);
                        atomicMin(&res->first, ((unsigned long long)e << 8) | (unsigned)n);
                    }
                }
#pragma unroll
                for (int word = 0; word < 4; ++word) {
                    const int r0 = __builtin_amdgcn_readlane(cl.rb, n * 5 + word);
                    const int r1 = __builtin_amdgcn_readlane(cl.rb, n * 5 + word + 1);
                    for (int r = r0; r < r1; ++r) {
                        const uint32_t d = run_desc(cl, r);
                        const uint32_t kpos = (d >> 8) & 31u, cpos = (d >> 16) & 31u, len = d >> 24;
#pragma unroll
                        for (int u = 0; u < kDepositU; ++u) w[u][word] |= __builtin_amdgcn_ubfe(c[n][u], cpos, len) << kpos;
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kDepositU; ++u) {
            const int64_t e = e0 + u * THREADS;
            if (e < nnz) {
                lo[e] = (uint64_t)w[u][0] | ((uint64_t)w[u][1] << 32);
                if (codec.key_words == 2) hi[e] = (uint64_t)w[u][2] | ((uint64_t)w[u][3] << 32);
                atomicAdd(&hist.h[tid >> 8][w[u][0] & 255u], 1u);
            }
        }
    }
    __syncthreads();
    hist_store<THREADS>(hist, counts, b, nblocks);
}

template <int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS) void k_radix_hist(const uint64_t *__restrict__ keys, int64_t n, int shift,
                                                        uint32_t *__restrict__ counts, int nblocks) {
    __shared__ TileHist<THREADS> hist;
    const int tid = threadIdx.x;
    const int64_t b = xcd_remap(blockIdx.x, gridDim.x), base = b * (THREADS * ITEMS) + tid;
    uint64_t k[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t e = base + i * THREADS;
        k[i] = e < n ? keys[e] : 0;
    }
    hist.h[tid >> 8][tid & 255] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (base + i * THREADS < n) atomicAdd(&hist.h[tid >> 8][(uint32_t)(k[i] >> shift) & 255u], 1u);
    __syncthreads();
    hist_store<THREADS>(hist, counts, b, nblocks);
}

// Exclusive scan of counts[d * nblocks + b] over b for one digit d per
// workgroup, kScanItems counts a thread: all of a digit's counts in one or two
// rounds (30M elements: 3662 tiles).
constexpr int kScanItems = 8;
constexpr int kScanThreads = 512;
__global__ __launch_bounds__(kScanThreads) void k_radix_scan(uint32_t *__restrict__ counts, int nblocks,
                                                             uint32_t *__restrict__ totals) {
    __shared__ uint32_t wsum[2][kScanThreads / 64];
    const int d = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t *row = counts + (int64_t)d * nblocks;
    uint32_t carry = 0;
    for (int b0 = 0, p = 0; b0 < nblocks; b0 += kScanThreads * kScanItems, p ^= 1) {
        const int b = b0 + tid * kScanItems;
        uint32_t v[kScanItems], sum = 0;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) v[i] = b + i < nblocks ? row[b + i] : 0u;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) sum += v[i];
        uint32_t x = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, 64);
            if (lane >= off) x += y;
        }
        if (lane == 63) wsum[p][wave] = x;
        __syncthreads();
        uint32_t all = 0, base = carry + x - sum;
#pragma unroll
        for (int w = 0; w < kScanThreads / 64; ++w) {
            if (w < wave) base += wsum[p][w];
            all += wsum[p][w];
        }
        carry += all;
#pragma unroll
        for (int i = 0; i < kScanItems; ++i) {
            if (b + i < nblocks) row[b + i] = base;
            base += v[i];
        }
    }
    if (tid == 0) totals[d] = carry;
}

// The values that go with the last pass: vout[dst] = vin[idx], and the sum of
// their squares per tile.
struct ValsArg {
    const float *in;
    float *out;
    double *partials;
};

// One pass of the sort.  `key` is the key word that holds the digit, `other`
// the other word of a 128-bit key.
template <int KW, int THREADS, int ITEMS>
__global__ __launch_bounds__(THREADS, THREADS == 1024 ? 8 : 4) void k_radix_scatter(
    const uint64_t *__restrict__ in_key, const uint64_t *__restrict__ in_other, const uint32_t *__restrict__ in_idx,
    uint64_t *__restrict__ out_key, uint64_t *__restrict__ out_other, uint32_t *__restrict__ out_idx, int64_t n,
    int shift, const uint32_t *__restrict__ counts, const uint32_t *__restrict__ totals, int nblocks, ValsArg vals) {
    constexpr int TILE = THREADS * ITEMS;
    constexpr int WAVES = THREADS / 64;
    constexpr int WSPAN = 64 * ITEMS;  // consecutive elements ranked by one wave
    static_assert(TILE <= (1 << 16), "positions in 16 bits");
    __shared__ __align__(16) char xchg[TILE * 8];  // the tile, one array after the other
    __shared__ uint16_t wcnt[WAVES][256];          // per wave and digit: count, then first position in the tile
    __shared__ uint32_t delta[256];                // per digit: output position - position in the tile
    __shared__ uint32_t wsum[2][4];
    __shared__ double wsq[WAVES];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t base = b * TILE;
    const int64_t wbase = base + (int64_t)wave * WSPAN;

    // every load of the wave's span is issued before the ranking waits for one
    // (past the end: the last element again, which takes no part)
    uint64_t key[ITEMS];
    uint32_t idx[ITEMS], dr[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) key[i] = in_key[min(wbase + i * 64 + lane, n - 1)];
    if (in_idx) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) idx[i] = in_idx[min(wbase + i * 64 + lane, n - 1)];
    } else {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) idx[i] = (uint32_t)(wbase + i * 64 + lane);
    }
    uint32_t total = 0, before_tile = 0;
    if (tid < 256) {
        total = totals[tid];
        before_tile = counts[(int64_t)tid * nblocks + b];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) wcnt[wave][lane * 4 + i] = 0;

    // Rank within the wave: equal digits of one round are ordered by lane
    // (ballots), rounds in order through the wave's own LDS counters.  The
    // counter update of a digit's first lane takes the value read by the whole
    // wave, so no other wave and no barrier is involved.
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool valid = wbase + i * 64 + lane < n;
        const uint32_t d = (uint32_t)(key[i] >> shift) & 255u;
        const uint64_t all = __ballot(valid);
        uint32_t plo = (uint32_t)all, phi = (uint32_t)(all >> 32);  // the lanes of the same digit
#pragma unroll
        for (int bit = 0; bit < 8; ++bit) {
            const uint32_t set = (uint32_t)((int32_t)(d << (31 - bit)) >> 31);
            const uint64_t m = __ballot(set != 0);
            plo &= ~((uint32_t)m ^ set);
            phi &= ~((uint32_t)(m >> 32) ^ set);
        }
        const uint32_t before = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0));
        const uint32_t old = wcnt[wave][d];
        if (valid && before == 0) wcnt[wave][d] = (uint16_t)(old + __popc(plo) + __popc(phi));
        dr[i] = d | ((old + before) << 8);
        __builtin_amdgcn_sched_barrier(0);  // one round's masks at a time: 64 VGPRs
    }
    __syncthreads();
    uint64_t other[ITEMS];  // not held while ranking, which needs the registers
    if (KW == 2) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) other[i] = in_other[min(wbase + i * 64 + lane, n - 1)];
    }

    // digit d of this tile starts at local; wave w's part of it follows the
    // parts of waves 0..w-1
    uint32_t sum = 0, x = 0, xt = 0;
    if (tid < 256) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) sum += wcnt[w][tid];
        x = sum;
        xt = total;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, 64), yt = __shfl_up(xt, off, 64);
            if (lane >= off) {
                x += y;
                xt += yt;
            }
        }
        if (lane == 63) {
            wsum[0][wave] = x;
            wsum[1][wave] = xt;
        }
    }
    __syncthreads();
    if (tid < 256) {
        uint32_t local = x - sum, digit = xt - total;
#pragma unroll
        for (int w = 0; w < 3; ++w)
            if (w < wave) {
                local += wsum[0][w];
                digit += wsum[1][w];
            }
        delta[tid] = digit + before_tile - local;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const uint32_t c = wcnt[w][tid];
            wcnt[w][tid] = (uint16_t)local;
            local += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        dr[i] = wcnt[wave][dr[i] & 255u] + (dr[i] >> 8);
        if (wbase + i * 64 + lane < n) ((uint64_t *)xchg)[dr[i]] = key[i];
    }
    __syncthreads();

    // runs of equal digit are contiguous in LDS and in the output
    const int cnt = (int)((n - base) < TILE ? (n - base) : TILE);
    uint32_t dst[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int q = tid + i * THREADS;
        dst[i] = 0;
        if (q < cnt) {
            const uint64_t k = ((const uint64_t *)xchg)[q];
            dst[i] = delta[(uint32_t)(k >> shift) & 255u] + (uint32_t)q;
            out_key[dst[i]] = k;
        }
    }
    if (KW == 2) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (wbase + i * 64 + lane < n) ((uint64_t *)xchg)[dr[i]] = other[i];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i)
            if (tid + i * THREADS < cnt) out_other[dst[i]] = ((const uint64_t *)xchg)[tid + i * THREADS];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (wbase + i * 64 + lane < n) ((uint32_t *)xchg)[dr[i]] = idx[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (tid + i * THREADS < cnt) {
            idx[i] = ((const uint32_t *)xchg)[tid + i * THREADS];
            out_idx[dst[i]] = idx[i];
        }
    if (!vals.in) return;
    float v[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) v[i] = tid + i * THREADS < cnt ? vals.in[idx[i]] : 0.f;
    double acc = 0.0;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
        if (tid + i * THREADS < cnt) {
            vals.out[dst[i]] = v[i];
            acc += (double)v[i] * (double)v[i];
        }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if (lane == 0) wsq[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        acc = 0.0;
        for (int w = 0; w < WAVES; ++w) acc += wsq[w];
        vals.partials[b] = acc;
    }
}

// out[j] = src[idx[j]] (32-bit words)
__global__ __launch_bounds__(kThreads) void k_gather_u32(const uint32_t *__restrict__ src, const uint32_t *__restrict__ idx,
                                                         uint32_t *__restrict__ out, int64_t n) {
    for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < n; j += (int64_t)gridDim.x * kThreads)
        out[j] = src[idx[j]];
}

// kDecodeU nonzeros a thread: all key words are loaded before the first is
// taken apart, and every bit run of the codec is applied to all of them.  30M
// nonzeros of 3 modes (600 MB): 155 us, one nonzero a thread took 466 us.
constexpr int kDecodeU = 8;
__global__ __launch_bounds__(kThreads) void k_decode(const uint64_t *__restrict__ lo, const uint64_t *__restrict__ hi,
                                                     int64_t nnz, Codec codec, uint32_t *__restrict__ coords) {
    const CodecRegs cl = load_codec_regs(codec);
    const int nwords = 2 * codec.key_words;
    const int64_t e0 = (int64_t)blockIdx.x * (kThreads * kDecodeU) + threadIdx.x;
    uint32_t w[kDecodeU][4];
#pragma unroll
    for (int u = 0; u < kDecodeU; ++u) {
        const int64_t e = e0 + u * kThreads;
        const uint64_t a = e < nnz ? lo[e] : 0;
        const uint64_t b = nwords == 4 && e < nnz ? hi[e] : 0;
        w[u][0] = (uint32_t)a;
        w[u][1] = (uint32_t)(a >> 32);
        w[u][2] = (uint32_t)b;
        w[u][3] = (uint32_t)(b >> 32);
    }
    for (int n = 0; n < codec.nmodes; ++n) {
        uint32_t x[kDecodeU] = {};
#pragma unroll
        for (int word = 0; word < 4; ++word) {
            if (word < nwords) {
                const int r0 = __builtin_amdgcn_readlane(cl.rb, n * 5 + word);
                const int r1 = __builtin_amdgcn_readlane(cl.rb, n * 5 + word + 1);
                for (int r = r0; r < r1; ++r) {
                    const uint32_t d = run_desc(cl, r);
#pragma unroll
                    for (int u = 0; u < kDecodeU; ++u)
                        x[u] |= __builtin_amdgcn_ubfe(w[u][word], (d >> 8) & 31u, d >> 24) << ((d >> 16) & 31u);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kDecodeU; ++u) {
            const int64_t e = e0 + u * kThreads;
            if (e < nnz) __builtin_nontemporal_store(x[u], coords + (int64_t)n * nnz + e);
        }
    }
}

constexpr int kExportU = 8;
template <int KW>
__global__ __launch_bounds__(kThreads) void k_export_keys(const uint64_t *__restrict__ lo, const uint64_t *__restrict__ hi,
                                                          int64_t nnz, uint64_t *__restrict__ keys) {
    const int64_t e0 = (int64_t)blockIdx.x * (kThreads * kExportU) + threadIdx.x;
    uint64_t a[kExportU], b[kExportU];
#pragma unroll
    for (int u = 0; u < kExportU; ++u) {
        const int64_t e = e0 + u * kThreads;
        a[u] = e < nnz ? lo[e] : 0;
        b[u] = KW == 2 && e < nnz ? hi[e] : 0;
    }
#pragma unroll
    for (int u = 0; u < kExportU; ++u) {
        const int64_t e = e0 + u * kThreads;
        if (e < nnz) {
            keys[KW * e] = a[u];
            if (KW == 2) keys[KW * e + 1] = b[u];
        }
    }
}

__global__ void k_init_result(EncodeResult *r) {
    r->bad = 0;
    r->pad = 0;
    r->first = ~0ull;
    r->norm_x2 = 0.0;
}

__global__ __launch_bounds__(kThreads) void k_sum_f64(const double *__restrict__ parts, int n, double *__restrict__ out) {
    __shared__ double ws[4];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += kThreads) acc += parts[i];
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_down(acc, off, 64);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = ws[0] + ws[1] + ws[2] + ws[3];
}

int grid_for(int64_t n, int per_block, int cap) {
    int64_t g = (n + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

__global__ void k_iota(uint32_t *p, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x)
        p[e] = (uint32_t)e;
}

struct SortBufs {
    uint64_t *lo[2], *hi[2];  // the keys' buffers; the input is in [0]
    uint32_t *idx[2];
    uint32_t *counts, *totals;
};

// `passes` passes of the stable LSD sort; pass p reads the buffers [p & 1] (the
// first makes the indices) and writes the others.  counted: the first digit's
// histograms are there.
template <int KW, int THREADS, int ITEMS>
spt_status sort_passes_t(const SortBufs &B, int64_t n, int passes, bool counted, const ValsArg &vals, hipStream_t s) {
    const int nblocks = (int)radix_tiles(n, {THREADS, ITEMS});
    for (int p = 0; p < passes; ++p) {
        const int bit = 8 * p, from = p & 1, to = from ^ 1, shift = bit % 64;
        const bool in_lo = bit < 64;
        const uint64_t *key = in_lo ? B.lo[from] : B.hi[from], *other = in_lo ? B.hi[from] : B.lo[from];
        uint64_t *key2 = in_lo ? B.lo[to] : B.hi[to], *other2 = in_lo ? B.hi[to] : B.lo[to];
        if (p > 0 || !counted)
            hipLaunchKernelGGL((k_radix_hist<THREADS, ITEMS>), dim3(nblocks), dim3(THREADS), 0, s, key, n, shift, B.counts, nblocks);
        hipLaunchKernelGGL(k_radix_scan, dim3(256), dim3(kScanThreads), 0, s, B.counts, nblocks, B.totals);
        hipLaunchKernelGGL((k_radix_scatter<KW, THREADS, ITEMS>), dim3(nblocks), dim3(THREADS), 0, s, key, other,
                           p ? B.idx[from] : (const uint32_t *)nullptr, key2, other2, B.idx[to], n, shift, B.counts,
                           B.totals, nblocks, p == passes - 1 ? vals : ValsArg{});
        SPT_HIP(hipGetLastError());
    }
    return SPT_OK;
}

template <int KW>
spt_status sort_passes(const SortBufs &B, int64_t n, int passes, hipStream_t s) {
    if (n >= kRadixLargeFrom)
        return sort_passes_t<KW, kRadixLarge<KW>.threads, kRadixLarge<KW>.items>(B, n, passes, false, ValsArg{}, s);
    return sort_passes_t<KW, kRadixSmall.threads, kRadixSmall.items>(B, n, passes, false, ValsArg{}, s);
}

template <int KW, int THREADS, int ITEMS>
spt_status deposit_sort_t(const Tensor *t, const uint32_t *coords, const SortBufs &B, int passes, EncodeResult *res,
                          const ValsArg &vals, hipStream_t s) {
    const int nblocks = (int)radix_tiles(t->nnz, {THREADS, ITEMS});
    DimsArg dims{};
    for (int k = 0; k < t->nmodes; ++k) dims.d[k] = (uint32_t)t->dims[k];
    hipLaunchKernelGGL((k_deposit<THREADS, ITEMS>), dim3(nblocks), dim3(THREADS), 0, s, coords, t->nnz, dims, t->codec,
                       B.lo[0], B.hi[0], res, B.counts, nblocks);
    SPT_HIP(hipGetLastError());
    // keys whose coordinates were out of range are still valid bit patterns,
    // so sorting them is harmless; the caller's check rejects the tensor.
    return sort_passes_t<KW, THREADS, ITEMS>(B, t->nnz, passes, true, vals, s);
}

template <int KW>
spt_status deposit_sort(const Tensor *t, const uint32_t *coords, const SortBufs &B, int passes, EncodeResult *res,
                        const ValsArg &vals, hipStream_t s) {
    if (t->nnz >= kRadixLargeFrom)
        return deposit_sort_t<KW, kRadixLarge<KW>.threads, kRadixLarge<KW>.items>(t, coords, B, passes, res, vals, s);
    return deposit_sort_t<KW, kRadixSmall.threads, kRadixSmall.items>(t, coords, B, passes, res, vals, s);
}

}  // namespace

spt_status launch_encode(Tensor *t, const uint32_t *coords, const float *vals, hipStream_t s) {
    const int64_t n = t->nnz;
    const size_t n1 = n > 0 ? (size_t)n : 1;
    const bool wide = t->key_words == 2;
    t->lo = t->hi = nullptr;
    t->vals = nullptr;
    t->perm = nullptr;
    t->norm_x2 = 0.0;
    // at least one pass: without key bits it leaves the input's order
    const int passes = n > 0 ? std::max(1, (t->lp + 7) / 8) : 0, last = passes & 1;
    const size_t tiles = (size_t)radix_tiles((int64_t)n1, radix_tile(t->key_words, n));
    SortBufs B{};
    EncodeResult *res = (EncodeResult *)dev_alloc(sizeof(EncodeResult), s);
    float *vout = (float *)dev_alloc(sizeof(float) * n1, s);
    double *partials = (double *)dev_alloc(sizeof(double) * tiles, s);
    bool ok = res && vout && partials;
    for (int i = 0; i < 2 && ok; ++i) {
        if (i == 0 || passes > 0) ok = (B.lo[i] = (uint64_t *)dev_alloc(sizeof(uint64_t) * n1, s)) != nullptr;
        if (ok && wide && (i == 0 || passes > 0)) ok = (B.hi[i] = (uint64_t *)dev_alloc(sizeof(uint64_t) * n1, s)) != nullptr;
        if (ok && (i == last || passes > 1)) ok = (B.idx[i] = (uint32_t *)dev_alloc(sizeof(uint32_t) * n1, s)) != nullptr;
    }
    if (ok && passes > 0) ok = (B.counts = (uint32_t *)dev_alloc(sizeof(uint32_t) * 256 * tiles, s)) &&
                               (B.totals = (uint32_t *)dev_alloc(sizeof(uint32_t) * 256, s));
    auto release_sort = [&](bool result) {  // result: the tensor's own buffers too
        for (int i = 0; i < 2; ++i)
            if (i != last || result) {
                dev_free(B.lo[i], s);
                dev_free(B.hi[i], s);
                dev_free(B.idx[i], s);
            }
        dev_free(B.counts, s);
        dev_free(B.totals, s);
        if (result) dev_free(vout, s);
        dev_free(res, s);
        dev_free(partials, s);
    };
    if (!ok) {
        release_sort(true);
        return fail(SPT_E_OOM, "encode: device allocation failed");
    }
    hipLaunchKernelGGL(k_init_result, dim3(1), dim3(1), 0, s, res);
    if (n > 0) {
        const ValsArg v{vals, vout, partials};
        const spt_status st = wide ? deposit_sort<2>(t, coords, B, passes, res, v, s)
                                   : deposit_sort<1>(t, coords, B, passes, res, v, s);
        if (st != SPT_OK) {
            release_sort(true);
            return st;
        }
        hipLaunchKernelGGL(k_sum_f64, dim3(1), dim3(kThreads), 0, s, partials, (int)tiles, &res->norm_x2);
        SPT_HIP(hipGetLastError());
    }
    EncodeResult h{};
    SPT_HIP(hipMemcpyAsync(&h, res, sizeof(h), hipMemcpyDeviceToHost, s));
    SPT_HIP(hipStreamSynchronize(s));
    if (h.bad != 0) {
        release_sort(true);
        return fail(SPT_E_INDEX_RANGE, std::to_string(h.bad) + " coordinate(s) out of range; first at nonzero " +
                                           std::to_string(h.first >> 8) + ", mode " + std::to_string(h.first & 255));
    }
    release_sort(false);
    t->lo = B.lo[last];
    t->hi = B.hi[last];
    t->vals = vout;
    t->perm = B.idx[last];
    t->norm_x2 = h.norm_x2;
    return SPT_OK;
}

spt_status launch_decode(const Tensor *t, uint32_t *coords, hipStream_t s) {
    if (t->nnz == 0) return SPT_OK;
    hipLaunchKernelGGL(k_decode, dim3((unsigned)((t->nnz + kThreads * kDecodeU - 1) / (kThreads * kDecodeU))),
                       dim3(kThreads), 0, s, t->lo, t->hi, t->nnz, t->codec, coords);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_gather_u32(const uint32_t *src, const uint32_t *idx, uint32_t *out, int64_t n, hipStream_t s) {
    if (n == 0) return SPT_OK;
    hipLaunchKernelGGL(k_gather_u32, dim3(grid_for(n, kThreads, 16384)), dim3(kThreads), 0, s, src, idx, out, n);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_export(const Tensor *t, uint64_t *keys, hipStream_t s) {
    if (t->nnz == 0) return SPT_OK;
    const dim3 g((unsigned)((t->nnz + kThreads * kExportU - 1) / (kThreads * kExportU)));
    if (t->key_words == 2)
        hipLaunchKernelGGL(k_export_keys<2>, g, dim3(kThreads), 0, s, t->lo, t->hi, t->nnz, keys);
    else
        hipLaunchKernelGGL(k_export_keys<1>, g, dim3(kThreads), 0, s, t->lo, t->hi, t->nnz, keys);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

// Enough for n keys and for fewer (whose tiles may be smaller).
size_t sort_ws_counts(int64_t n) {
    const int64_t small = radix_tiles(std::min(n, kRadixLargeFrom), kRadixSmall);
    return 256 * (size_t)(std::max(radix_tiles(n, radix_tile(1, n)), small) + 1);
}

// Stable LSD radix sort of n keys over their low nbits bits in caller-owned
// buffers: keys and keys2 (n each) ping-pong, idx_a / idx_b (n each) receive
// the input index of every sorted key, counts holds sort_ws_counts(n) words.
// *sorted_out / *idx_out point at the buffers holding the result.
spt_status sort_u64_keys_ws(uint64_t *keys, uint64_t *keys2, uint32_t *idx_a, uint32_t *idx_b, uint32_t *counts,
                            int64_t n, int nbits, uint64_t **sorted_out, uint32_t **idx_out, hipStream_t s) {
    const int passes = n > 0 ? (nbits + 7) / 8 : 0, last = passes & 1;
    SortBufs B{{keys, keys2}, {nullptr, nullptr}, {idx_b, idx_a}, counts + 256, counts};
    *sorted_out = B.lo[last];
    *idx_out = passes ? B.idx[last] : idx_a;
    if (n <= 0) return SPT_OK;
    if (passes) return sort_passes<1>(B, n, passes, s);
    hipLaunchKernelGGL(k_iota, dim3(grid_for(n, kThreads, 65536)), dim3(kThreads), 0, s, idx_a, n);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

}  // namespace spt
