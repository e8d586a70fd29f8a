// Mode-n MTTKRP in FP64 (Section II-B, Fig. 2) at the paper's own precision
// (FP64 values, factors and accumulation, 64-bit keys; Section IV-A).
//
// It runs the tensor's SEGMENT plan (positions of every nonzero in its tile's
// row-grouped order, runs of one output row, records laid out grouped by
// row), which does not depend on the value type:
//  1. a workgroup of T/4 threads stages one tile of the key-ordered stream:
//     keys are decoded to the non-output coordinates, which are scattered with
//     the FP64 values to their plan positions in LDS;
//  2. lane groups of ceil(R / 2) lanes, two columns each (LaneGroup), walk
//     equal shares of the tile (seg_walk.h): they gather the N-1 factor rows
//     of each nonzero in 16-byte loads, all of a step's before the first is
//     needed, form v * Hadamard(rows) and sum run by run;
//  3. each run is stored as one FP64 record at its plan-given slot; a second
//     kernel sums the records of every row (records.h).
// Bound by the vector memory path as the FP32 kernel, at twice the bytes a
// row.  One column a lane, one nonzero in flight and whole pieces of up to 64
// nonzeros to a group took 6.12 ms for an all-mode sweep (rank 16, 20M
// nonzeros, 3 modes; 1.48 ms a mode and 0.41 ms for the records' sum), this
// 3.04 ms.
#include "records.h"
#include "seg_walk.h"

namespace spt {

namespace {

__host__ __device__ inline size_t f64_lds_bytes(int T, int nmodes) {
    const size_t staged = (size_t)(nmodes - 1) * T * 4 + (size_t)T * 8;
    return staged > walk_lds_bytes(T / 4, 4 * sizeof(double)) ? staged : walk_lds_bytes(T / 4, 4 * sizeof(double));
}

struct FactorsF64 {
    const double *f[kMaxModes];
};

template <int NT, int VEC, int NMAX, int NFIX, int FAR>
__global__ __launch_bounds__(NT) void k_mttkrp_seg_f64(MttkrpArgs a, const double *__restrict__ vals64, int64_t ntiles,
                                                       FactorsF64 F, double *__restrict__ rec_val,
                                                       double *__restrict__ out) {
    constexpr int T = 4 * NT, NO = NMAX - 1, UB = NMAX <= 4 && VEC <= 2 ? 2 : 1;
    extern __shared__ __align__(16) char lds[];
    const int64_t tile = xcd_remap(blockIdx.x, gridDim.x);
    if (tile >= ntiles) return;
    const int nm = NFIX ? NFIX : a.nmodes, no = nm - 1, mode = a.mode, tid = threadIdx.x, R = a.rank;
    double *valg = (double *)lds;
    uint32_t *crdg = (uint32_t *)(valg + T);
    const CodecRegs cr = load_codec_regs(a.codec);
    const int64_t base = tile * (int64_t)T;
    const int64_t rem = a.nnz - base;
    const int cnt = rem < T ? (int)rem : T;
    const int nwords = 2 * a.codec.key_words;
    const int64_t k0 = a.pl_off[tile];
    const int nruns = (int)min<int64_t>(a.pl_off[tile + 1] - k0, T);
    uint32_t w[4][4];
    double v[4];
    int ps[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + u * NT;
        uint64_t klo = 0, khi = 0;
        v[u] = 0.0;
        ps[u] = 0;
        if (e < cnt) {
            klo = __builtin_nontemporal_load(a.lo + base + e);
            if (nwords == 4) khi = __builtin_nontemporal_load(a.hi + base + e);
            v[u] = __builtin_nontemporal_load(vals64 + base + e);
            ps[u] = a.pl_pos[base + e] & (T - 1);  // a position inside the tile
        }
        w[u][0] = (uint32_t)klo;
        w[u][1] = (uint32_t)(klo >> 32);
        w[u][2] = (uint32_t)khi;
        w[u][3] = (uint32_t)(khi >> 32);
    }
    const LaneGroup lg = lane_group<VEC>(R);
    const WalkShare ws = walk_share<NT, T, false>(lg, cnt, UB, a.pl_start + tile * (T / 32));
    // while the loads above are in flight
    zero_slice((float *)out, 2 * (int64_t)a.frows[mode] * R, tile, ntiles);
#pragma unroll
    for (int k = 0; k < NMAX; ++k) {
        if (k < nm && k != mode) {
            uint32_t x[4] = {0, 0, 0, 0};
#pragma unroll
            for (int word = 0; word < 4; ++word) {
                if (word < nwords) {
                    const int r0 = __builtin_amdgcn_readlane(cr.rb, k * 5 + word);
                    const int r1 = __builtin_amdgcn_readlane(cr.rb, k * 5 + word + 1);
                    for (int r = r0; r < r1; ++r) {
                        const uint32_t d = run_desc(cr, r);
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            x[u] |= __builtin_amdgcn_ubfe(w[u][word], (d >> 8) & 31u, d >> 24) << ((d >> 16) & 31u);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (tid + u * NT < cnt) crdg[(k - (k > mode)) * T + ps[u]] = x[u];
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (tid + u * NT < cnt) valg[ps[u]] = v[u];
    if (tid < nm && cnt < T) {  // the other half of an odd last step: row 0, value 0
        if (tid < no) crdg[tid * T + cnt] = 0;
        else valg[cnt] = 0.0;
    }
    __syncthreads();
    RowView<double, FAR == kFarAll> fb[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int k = o + (o >= mode);
        fb[o] = o < no ? RowView<double, FAR == kFarAll>(F.f[k], R, a.frows[k])
                       : RowView<double, FAR == kFarAll>(nullptr, R, 0u);
    }
    const int c = lg.col;
    auto product = [&](int q0, double (&p)[UB][VEC], double (&last)[UB][VEC]) {
        uint32_t row[NO][UB];
        double xv[NO][UB][VEC], x[UB];
        load_words<UB>(valg + q0, x);
#pragma unroll
        for (int o = 0; o < NO; ++o)
            if (o < no) load_words<UB>(crdg + o * T + q0, row[o]);
#pragma unroll
        for (int u = 0; u < UB; ++u)
#pragma unroll
            for (int q = 0; q < VEC; ++q) p[u][q] = x[u];
        if (NFIX == 0 && no == 0)  // one mode: the empty product
#pragma unroll
            for (int u = 0; u < UB; ++u)
#pragma unroll
                for (int q = 0; q < VEC; ++q) last[u][q] = 1.0;
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
                    for (int q = 0; q < VEC; ++q) {
                        if (o == 0) last[u][q] = xv[0][u][q];
                        else p[u][q] *= xv[o][u][q];
                    }
    };
    run_walk<double, NT, T, VEC, UB, false, FAR>(lg, ws, R, cnt, nruns, a.pl_rec + k0, (uint32_t)a.rec_cap, rec_val, R,
                                                 lds, product);
}

__global__ __launch_bounds__(256) void k_gather_f64(const double *__restrict__ src, const uint32_t *__restrict__ idx,
                                                    double *__restrict__ dst, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        dst[i] = src[idx[i]];
}

template <int NT, int VEC, int NMAX, int NFIX, int FAR>
spt_status launch_f64_k(const MttkrpArgs &a, const double *vals64, const FactorsF64 &F, int64_t ntiles, double *rec_val,
                        double *out, hipStream_t s) {
    hipLaunchKernelGGL((k_mttkrp_seg_f64<NT, VEC, NMAX, NFIX, FAR>), dim3((unsigned)ntiles), dim3(NT),
                       f64_lds_bytes(4 * NT, a.nmodes), s, a, vals64, ntiles, F, rec_val, out);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

template <int NT, int VEC, int FAR>
spt_status launch_f64_n(const MttkrpArgs &a, const double *vals64, const FactorsF64 &F, int64_t ntiles, double *rec_val,
                        double *out, hipStream_t s) {
    auto go = [&](auto launch) { return launch(a, vals64, F, ntiles, rec_val, out, s); };
    if constexpr (FAR == kFarAll) {
        return a.nmodes <= 4 ? go(launch_f64_k<NT, VEC, 4, 0, FAR>) : go(launch_f64_k<NT, VEC, 8, 0, FAR>);
    } else {
        if (a.nmodes == 3) return go(launch_f64_k<NT, VEC, 3, 3, FAR>);
        if (a.nmodes == 4) return go(launch_f64_k<NT, VEC, 4, 4, FAR>);
        if (a.nmodes == 5) return go(launch_f64_k<NT, VEC, 5, 5, FAR>);
        return a.nmodes < 3 ? go(launch_f64_k<NT, VEC, 3, 0, FAR>) : go(launch_f64_k<NT, VEC, 8, 0, FAR>);
    }
}

template <int NT>
spt_status launch_f64_t(const MttkrpArgs &a, const double *vals64, const FactorsF64 &F, int64_t ntiles, double *rec_val,
                        double *out, hipStream_t s) {
    auto go = [&](auto launch) { return launch(a, vals64, F, ntiles, rec_val, out, s); };
    const SegFar far = seg_far(a, a.rank, sizeof(double));
    if (a.rank < 2) return far == kNear ? go(launch_f64_n<NT, 1, kNear>) : go(launch_f64_n<NT, 1, kFarAll>);
    if (a.rank <= 128)
        return far == kNear ? go(launch_f64_n<NT, 2, kNear>)
                            : far == kFarRecords ? go(launch_f64_n<NT, 2, kFarRecords>) : go(launch_f64_n<NT, 2, kFarAll>);
    // two columns a lane would be more than a wave
    return far == kNear ? go(launch_f64_n<NT, 4, kNear>)
                        : far == kFarRecords ? go(launch_f64_n<NT, 4, kFarRecords>) : go(launch_f64_n<NT, 4, kFarAll>);
}

}  // namespace

bool f64_tile_ok(int tile, int nmodes) {
    return (tile == 1024 || tile == 2048 || tile == 4096) && f64_lds_bytes(tile, nmodes) <= 160 * 1024 - 1024;
}

spt_status launch_mttkrp_seg_f64(const MttkrpArgs &a, const double *vals64, const double *const *F,
                                 double *rec_val, double *out, hipStream_t s) {
    const int64_t ntiles = (a.nnz + a.tile - 1) / a.tile;
    if (ntiles == 0) return SPT_OK;
    if (!f64_tile_ok(a.tile, a.nmodes)) return fail(SPT_E_INVALID_ARG, "mttkrp_f64: tile does not fit LDS");
    if (!a.pl_pos || !a.pl_off || !a.pl_start || !a.pl_rec) return fail(SPT_E_INVALID_ARG, "mttkrp_f64: no plan");
    if (a.rank > 256) return fail(SPT_E_INVALID_ARG, "mttkrp_f64: rank above 256");
    FactorsF64 f{};
    for (int k = 0; k < a.nmodes; ++k) f.f[k] = F[k];
    if (a.tile == 1024) return launch_f64_t<256>(a, vals64, f, ntiles, rec_val, out, s);
    if (a.tile == 2048) return launch_f64_t<512>(a, vals64, f, ntiles, rec_val, out, s);
    return launch_f64_t<1024>(a, vals64, f, ntiles, rec_val, out, s);
}

spt_status launch_reduce_records_f64(const uint64_t *srow, const double *rec, int64_t P, int R, int64_t rows,
                                     double *out, hipStream_t s) {
    return launch_reduce<double>(srow, nullptr, rec, P, R, rows, out, s);
}

spt_status launch_gather_f64(const double *src, const uint32_t *idx, double *dst, int64_t n, hipStream_t s) {
    if (n == 0) return SPT_OK;
    const int64_t g = std::min<int64_t>((n + 255) / 256, 65536);
    hipLaunchKernelGGL(k_gather_f64, dim3((unsigned)g), dim3(256), 0, s, src, idx, dst, n);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

}  // namespace spt
