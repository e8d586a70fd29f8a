// Dense FP64 steps of CP-ALS on gfx950 (the ALS update that Section II-B
// defers to Kolda and Bader):
//   gram        G = C^T C for an I x R FP32 matrix: FP32 values widened to FP64
//               (products exact) and accumulated by v_mfma_f64_16x16x4_f64;
//               only the upper block triangle is computed and mirrored.
//   solve_prep  one workgroup: V = Hadamard product of the other Grams,
//               Cholesky V = L L^T with a ridge retry, W = V^-1, column norms of
//               M W from the quadratic form lambda_r^2 = (W (M^T M) W)_rr,
//               S = W diag(1/lambda).
//   apply       C = fp32(M S) by 16-row tiles (FP64 MFMA), with the fit's inner
//               product sum M .* C * lambda fused in.
//   fit         |Xhat|^2 = lambda^T (Hadamard of all Grams) lambda and the fit.
#include <algorithm>
#include <utility>

#include "spt_internal.h"

namespace spt {

namespace {

constexpr int kThreads = 256;

typedef double double4_t __attribute__((ext_vector_type(4)));

int gram_nb(int R) { return (R + 15) / 16; }
// 16 x 16 tiles of the upper block triangle; a partial Gram is that many tiles of 256 doubles, row-major inside
__host__ __device__ constexpr int gram_tiles(int nb) { return nb * (nb + 1) / 2; }

// Row slices (workgroups, one partial each) of the Gram kernel: 256 rows each,
// two rounds of rows for each of its 8 waves at rank 64, up to the number of
// workgroups that are resident at once (80 KB of LDS at rank 64: 2 per CU).
constexpr int kGramRows = 256;
constexpr int kGramMaxSlices = 512;
// A Gram of at most this many slices is left to its reader to add up.
constexpr int kGramDirect = 4;
int gram_slices_single(int64_t rows) {
    return (int)std::max<int64_t>(1, std::min<int64_t>((rows + kGramRows - 1) / kGramRows, kGramMaxSlices));
}

// Partial Gram of the rows [r0, r1) (r0 a multiple of 4) of a row-major FP32
// matrix, by a workgroup of 8 waves.  Wave w takes row groups of 4 rows w, w +
// 8, ..., UNR of them at a time, and accumulates every upper tile with FP64
// MFMA (A[m][k] from lane m + 16 k, B[k][n] from lane n + 16 k, D[m][n] in
// lane n + 16 (m % 4), element m / 4).  The waves' tiles are added in a fixed
// order in three steps of LDS.  Bound by load latency before the matrix cores
// (one v_mfma_f64_16x16x4 a tile and 4 rows, 10 tiles at rank 64), so the next
// UNR groups are loaded, as FP32, while the present ones are multiplied.
// With one group in flight and one wave after the other adding its tiles, 100k
// rows at rank 64 took 29 us, and 20 to add up the partials (5 now).
constexpr int kGramThreads = 512;
template <int NB>
constexpr int gram_unr() { return NB <= 2 ? 4 : 2; }

template <int NB>
__device__ __forceinline__ void gram_slice(const float *__restrict__ C, int ld, int R, int64_t r0, int64_t r1,
                                           double *__restrict__ out) {
    constexpr int NT = gram_tiles(NB), NWAVE = kGramThreads / 64, UNR = gram_unr<NB>();
    __shared__ double red[NWAVE / 2][NT * 256];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, kr = lane >> 4, cc = lane & 15;
    double4_t acc[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[i] = (double4_t){0.0, 0.0, 0.0, 0.0};
    float cur[UNR][NB], nxt[UNR][NB];
    auto load = [&](float (&x)[UNR][NB], int64_t row0) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int64_t row = row0 + (int64_t)u * 4 * NWAVE + kr;
            const float *rp = C + row * ld;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int c = b * 16 + cc;
                x[u][b] = (row < r1 && c < R) ? rp[c] : 0.f;
            }
        }
    };
    constexpr int64_t step = (int64_t)4 * NWAVE * UNR;
    int64_t row0 = r0 + 4 * wave;
    load(cur, row0);
    for (; row0 < r1; row0 += step) {
        load(nxt, row0 + step);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            double v[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) v[b] = (double)cur[u][b];
            int t = 0;
#pragma unroll
            for (int pb = 0; pb < NB; ++pb)
#pragma unroll
                for (int qb = pb; qb < NB; ++qb, ++t)
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[pb], v[qb], acc[t], 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b) cur[u][b] = nxt[u][b];
    }
    if (wave >= NWAVE / 2) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave - NWAVE / 2][t * 256 + e * 64 + lane] = acc[t][e];
    }
    __syncthreads();
    if (wave < NWAVE / 2) {
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double &d = red[wave][t * 256 + e * 64 + lane];
                d = acc[t][e] + d;
            }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NT * 256; e += kGramThreads) out[e] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
}

template <int NB>
__global__ __launch_bounds__(kGramThreads) void k_gram_partial(const float *__restrict__ C, int64_t rows, int R,
                                                               double *__restrict__ work) {
    const int64_t per = ((rows + gridDim.x - 1) / gridDim.x + 3) / 4 * 4;
    const int64_t r0 = blockIdx.x * per;
    gram_slice<NB>(C, R, R, r0, min(r0 + per, rows), work + (size_t)blockIdx.x * gram_tiles(NB) * 256);
}

// Batched: slice gs of the launch belongs to the last item whose first_slice <= gs.
template <int NB>
__global__ __launch_bounds__(kGramThreads) void k_gram_batched_partial(const GramItem *__restrict__ items, int count,
                                                                      double *__restrict__ work) {
    const int64_t gs = blockIdx.x;
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].first_slice <= gs) lo = mid;
        else hi = mid - 1;
    }
    const GramItem &it = items[__builtin_amdgcn_readfirstlane(lo)];
    const int64_t r0 = (gs - it.first_slice) * kGramSliceRows;
    gram_slice<NB>(it.C, it.ld, it.rank, r0, min(it.rows, r0 + kGramSliceRows),
                   work + (size_t)gs * gram_tiles(NB) * 256);
}

// G = the sum of a Gram's slices, mirrored: a workgroup adds 32 of their
// elements, 8 threads to an element (every 8th slice each, then in order).
constexpr int kGramSumElems = 32;
__device__ __forceinline__ void gram_sum(const double *__restrict__ work, int64_t nslices, int nb, int R,
                                         double *__restrict__ G) {
    constexpr int W = kThreads / kGramSumElems;
    __shared__ double red[W][kGramSumElems];
    const int stride = gram_tiles(nb) * 256;
    const int x = threadIdx.x % kGramSumElems, y = threadIdx.x / kGramSumElems;
    const int e = blockIdx.x * kGramSumElems + x;
    double s = 0.0;
    if (e < stride) {
        int64_t k = y;
        for (; k + 7 * W < nslices; k += 8 * W) {
            double v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = work[(size_t)(k + i * W) * stride + e];
#pragma unroll
            for (int i = 0; i < 8; ++i) s += v[i];
        }
        for (; k < nslices; k += W) s += work[(size_t)k * stride + e];
    }
    red[y][x] = s;
    __syncthreads();
    if (y == 0 && e < stride) {
#pragma unroll
        for (int i = 1; i < W; ++i) s += red[i][x];
        int t = e >> 8, pb = 0;
        while (t >= nb - pb) t -= nb - pb, ++pb;
        const int p = pb * 16 + ((e >> 4) & 15), q = (pb + t) * 16 + (e & 15);
        if (p < R && q < R) {
            G[p * R + q] = s;
            if (t > 0) G[q * R + p] = s;
        }
    }
}

__global__ __launch_bounds__(kThreads) void k_gram_sum(const double *__restrict__ work, int nslices, int nb, int R,
                                                       double *__restrict__ G) {
    gram_sum(work, nslices, nb, R, G);
}

__global__ __launch_bounds__(kThreads) void k_gram_sum_batched(const GramItem *__restrict__ items, int nb,
                                                               const double *__restrict__ work) {
    const GramItem &it = items[blockIdx.y];
    gram_sum(work + (size_t)it.first_slice * gram_tiles(nb) * 256, it.nslices, nb, it.rank, it.G);
}

// Element (i, j) of the Gram that the solve reads: whole, or still in a few slices.
__device__ __forceinline__ double gram_at(const GramRef &g, int nb, int R, int i, int j) {
    if (g.slices == 0) return g.p[i * R + j];
    if (i / 16 > j / 16) {
        const int x = i;
        i = j;
        j = x;
    }
    const int pb = i / 16, stride = gram_tiles(nb) * 256;
    const double *p = g.p + (pb * nb - pb * (pb - 1) / 2 + j / 16 - pb) * 256 + (i & 15) * 16 + (j & 15);
    double s = 0.0;
    for (int k = 0; k < g.slices; ++k) s += p[(size_t)k * stride];
    return s;
}

// ------------------------------------------------------------------ solve preparation
// One workgroup; R <= 64, padded to RP = 16 nb by an identity block (V) and
// zeros (Gm).  W = V^-1 from the Cholesky factor V = L L^T, in 16 x 16 blocks.
// What bounds it is one serial chain: R pivots, each a reciprocal square root
// that the next one waits for.  So that chain alone runs in one wave, in
// registers (a diagonal block factored and inverted at once, 16 pivots, no
// barrier), and everything else is FP64 MFMA tiles of other waves beside it:
// per block column k two barriers, the first behind the diagonal block (X_kk =
// L_kk^-1) and the sums that do not need it, the second behind what does:
//   T_ki = V_ki - sum_{p<k} L_kp L_ip^T,   L_ik^T = X_kk T_ki      (i > k)
//   D_kj = sum_{j<=p<k} L_kp X_pj,         X_kj   = -X_kk D_kj     (j < k)
// with X = L^-1, then W = X^T X.  An MFMA result D[m][n] sits in lane n + 16
// (m % 4), element m / 4, which is where the next product wants it as its
// right operand: no result moves between the two.
// One element sweep with a barrier per pivot, as it was, took 84 / 51 / 31 / 16
// us at rank 64 / 48 / 32 / 16.
constexpr int kSolveThreads = 512;
constexpr int kSolveLd = 66;  // doubles: rows 4 banks apart, so that 16 rows of one column do not collide

__device__ __forceinline__ double lane_f64(double x, int lane) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), lane);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), lane);
    return __hiloint2double(hi, lo);
}

// lane J of each row of 16 lanes to the whole row
template <int J>
__device__ __forceinline__ double row_bcast_f64(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x150 + J, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x150 + J, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// Pivot J of a 16 x 16 block held by one wave in MFMA result layout (lane n +
// 16 q: column n, rows 4 e + q): b the symmetric block, x the inverse of its
// factor so far (identity at first).  c = column J as it is: rows i > J lose
// c_i c_n / d from b and c_i x[J][n] / d from x, row J of x is scaled by 1 / l.
// The pivot's reciprocal square root is the hardware estimate and two Newton
// steps, which gives 1 / l and 1 / d without a square root or a divide.
template <int J>
__device__ __forceinline__ void solve_pivot(double (&b)[4], double (&x)[4], int n, int q, bool &ok) {
    constexpr int E = J / 4, Q = J % 4;
    const double d = lane_f64(b[E], J + 16 * Q);
    ok = ok && d > 0.0 && isfinite(d);
    double r = __builtin_amdgcn_rsq(d);
    r = r * (1.5 - 0.5 * d * r * r);
    r = r * (1.5 - 0.5 * d * r * r);
    const double id = r * r;
    double c[4];
    c[0] = row_bcast_f64<J>(b[0]);
    c[1] = row_bcast_f64<J>(b[1]);
    c[2] = row_bcast_f64<J>(b[2]);
    c[3] = row_bcast_f64<J>(b[3]);
    const double cn = __shfl(b[E], n + 16 * Q, 64);  // b is symmetric: its row J is its column J
    const double xn = __shfl(x[E], n + 16 * Q, 64);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double ci = 4 * e + q > J ? c[e] : 0.0;
        b[e] -= ci * cn * id;
        x[e] -= ci * xn * id;
    }
    if (q == Q) x[E] *= r;
}

template <int... J>
__device__ __forceinline__ void solve_pivots(double (&b)[4], double (&x)[4], int n, int q, bool &ok,
                                             std::integer_sequence<int, J...>) {
    (solve_pivot<J>(b, x, n, q, ok), ...);
}

// acc + sign * X Y^T over 16 columns, X and Y 16 x 16 blocks of row-major LDS matrices
__device__ __forceinline__ double4_t mfma_abt(const double *X, const double *Y, double4_t acc, int lane) {
    const int r = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int k = 0; k < 16; k += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[r * kSolveLd + k + kq], Y[r * kSolveLd + k + kq], acc, 0, 0, 0);
    return acc;
}

// acc + X Y over 16 columns of X
__device__ __forceinline__ double4_t mfma_ab(const double *X, const double *Y, double4_t acc, int lane) {
    const int r = lane & 15, kq = lane >> 4;
#pragma unroll
    for (int k = 0; k < 16; k += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[r * kSolveLd + k + kq], Y[(k + kq) * kSolveLd + r], acc, 0, 0, 0);
    return acc;
}

// X^T Y over the rows [k0, k1) of two row-major LDS matrices (16-column blocks at X and Y)
__device__ __forceinline__ double4_t mfma_atb(const double *X, const double *Y, int k0, int k1, int lane) {
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    const int r = lane & 15, kq = lane >> 4;
    for (int k = k0; k < k1; k += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[(k + kq) * kSolveLd + r], Y[(k + kq) * kSolveLd + r], acc, 0, 0, 0);
    return acc;
}

__device__ __forceinline__ void solve_prep_body(const double *__restrict__ grams, int nmodes, int mode, int R,
                                                const GramRef &gram_m, double *__restrict__ S,
                                                double *__restrict__ lambda, int *__restrict__ status,
                                                double *__restrict__ gram_new) {
    constexpr int LD = kSolveLd;
    __shared__ double A[64 * LD];
    __shared__ double B[64 * LD];
    __shared__ double Xs[64 * LD];
    __shared__ double lam_s[64];
    __shared__ int failed;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int nb = (R + 15) / 16, RP = nb * 16, RR = R * R;
    const int n = lane & 15, q = lane >> 4;
    // V = Hadamard product of the Grams of every mode except `mode` -> A
    for (int e = tid; e < RP * RP; e += kSolveThreads) {
        const int i = e / RP, j = e - i * RP;
        double v = i == j ? 1.0 : 0.0;
        if (i < R && j < R) {
            v = 1.0;
            for (int k = 0; k < nmodes; ++k)
                if (k != mode) v *= grams[(size_t)k * RR + i * R + j];
        }
        A[i * LD + j] = v;
    }
    if (tid == 0) failed = 0;
    __syncthreads();
    int attempt = 0;
    for (; attempt < 4; ++attempt) {
        double ridge = 0.0;
        if (attempt > 0) {
            double trace = 0.0;
            for (int i = 0; i < R; ++i) trace += A[i * LD + i];
            ridge = 1e-12 * trace / R * pow(1e3, (double)(attempt - 1));
        }
        // the ridge goes on the diagonal blocks only, as they are read
        for (int k = 0; k < nb; ++k) {
            double4_t acc = {0.0, 0.0, 0.0, 0.0};
            const int panel = nb - 1 - k;                    // tiles i > k
            const bool is_panel = wave >= 1 && wave <= panel;
            const bool is_inv = wave > panel && wave < nb;   // tiles j < k
            const int t = is_panel ? k + wave : wave - 1 - panel;  // i or j
            if (wave == 0) {
                for (int p = 0; p < k; ++p) acc = mfma_abt(B + k * 16 * LD + p * 16, B + k * 16 * LD + p * 16, acc, lane);
                double b[4], x[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int i = 4 * e + q, gi = k * 16 + i;
                    double v = A[gi * LD + k * 16 + n];
                    if (i == n && gi < R) v += ridge;
                    b[e] = v - acc[e];
                    x[e] = i == n ? 1.0 : 0.0;
                }
                bool ok = true;
                solve_pivots(b, x, n, q, ok, std::make_integer_sequence<int, 16>{});
                if (!ok && lane == 0) failed = 1;
#pragma unroll
                for (int e = 0; e < 4; ++e) Xs[(k * 16 + 4 * e + q) * LD + k * 16 + n] = x[e];
            } else if (is_panel) {
                for (int p = 0; p < k; ++p) acc = mfma_abt(B + k * 16 * LD + p * 16, B + t * 16 * LD + p * 16, acc, lane);
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] = A[(k * 16 + 4 * e + q) * LD + t * 16 + n] - acc[e];
            } else if (is_inv) {
                for (int p = t; p < k; ++p) acc = mfma_ab(B + k * 16 * LD + p * 16, Xs + p * 16 * LD + t * 16, acc, lane);
            }
            __syncthreads();
            if (failed) break;
            if (is_panel || is_inv) {
                double4_t r = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    r = __builtin_amdgcn_mfma_f64_16x16x4f64(Xs[(k * 16 + n) * LD + k * 16 + 4 * s + q], acc[s], r, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (is_panel) B[(t * 16 + n) * LD + k * 16 + 4 * e + q] = r[e];  // L_ik, transposed back
                    else Xs[(k * 16 + 4 * e + q) * LD + t * 16 + n] = -r[e];
                }
            }
            __syncthreads();
        }
        if (!failed) break;
        __syncthreads();  // every wave has read the flag
        if (tid == 0) failed = 0;
        __syncthreads();
    }
    if (attempt == 4) {
        if (tid == 0) *status = -1;
        return;
    }
    // Gm over V (which no wave reads any more); W = X^T X = V^-1 into B
    for (int e = tid; e < RP * RP; e += kSolveThreads) {
        const int i = e / RP, j = e - i * RP;
        A[i * LD + j] = i < R && j < R ? gram_at(gram_m, nb, R, i, j) : 0.0;
    }
    auto tiles = [&](auto product, double *dst) {
        for (int t = wave; t < nb * nb; t += kSolveThreads / 64) {
            const int ti = t / nb, tj = t - ti * nb;
            const double4_t acc = product(ti, tj);
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[(ti * 16 + 4 * e + q) * LD + tj * 16 + n] = acc[e];
        }
        __syncthreads();
    };
    // X is lower triangular: its blocks above the diagonal were never written
    tiles([&](int ti, int tj) { return mfma_atb(Xs + ti * 16, Xs + tj * 16, max(ti, tj) * 16, RP, lane); }, B);
    // Tm = Gm W into Xs, then P = W Tm = W Gm W into A (Gm and W are symmetric)
    tiles([&](int ti, int tj) { return mfma_atb(A + ti * 16, B + tj * 16, 0, RP, lane); }, Xs);
    tiles([&](int ti, int tj) { return mfma_atb(B + ti * 16, Xs + tj * 16, 0, RP, lane); }, A);
    // lambda_r^2 = P[r][r]
    for (int r = tid; r < R; r += kSolveThreads) {
        const double s2 = A[r * LD + r];
        const double l = s2 > 0.0 ? sqrt(s2) : 0.0;
        lam_s[r] = l > 0.0 ? l : 1.0;
        lambda[r] = lam_s[r];
    }
    __syncthreads();
    // The Gram of the new factor C = M S without reading C: C^T C = S^T Gm S,
    // and with S = W diag(1/lambda), W symmetric, its (p, q) entry is
    // P[p][q] / (lambda_p lambda_q).  FP64 throughout, so it is the Gram of
    // the exact product rather than of C rounded to FP32.  Only the other
    // modes' Grams were read above, so the slot of `mode` may be overwritten.
    for (int e = tid; e < RR; e += kSolveThreads) {
        const int i = e / R, j = e - i * R;
        if (gram_new) gram_new[e] = A[i * LD + j] / (lam_s[i] * lam_s[j]);
        S[e] = B[i * LD + j] / lam_s[j];
    }
    if (tid == 0) *status = attempt;
}

__global__ __launch_bounds__(kSolveThreads) void k_solve_prep(const double *__restrict__ grams, int nmodes, int mode, int R,
                                                              GramRef gram_m, double *__restrict__ S,
                                                              double *__restrict__ lambda, int *__restrict__ status,
                                                              double *__restrict__ gram_new) {
    solve_prep_body(grams, nmodes, mode, R, gram_m, S, lambda, status, gram_new);
}

__global__ __launch_bounds__(kSolveThreads) void k_solve_prep_batched(const SolveItem *__restrict__ items, int mode) {
    const SolveItem &it = items[blockIdx.x];
    solve_prep_body(it.grams, it.nmodes, mode, it.rank, GramRef{it.gram_m, 0}, it.S, it.lambda, it.status + mode,
                    it.gram_new);
}

// ------------------------------------------------------------------ apply
// C = M S on FP64 MFMA for 16-row tiles t = t0, t0 + dt, ... < t1, one at a
// time per wave, S (RP x RP) in LDS.  The k index of v_mfma_f64_16x16x4_f64 is
// only summed over, so step j takes columns kq KS + j (KS = RP / 4) for lane
// quarter kq: every lane holds KS contiguous values of its row of M, and the
// next tile's are loaded while this one is multiplied.  Bound by the matrix
// cores and by bringing S to LDS, which several tiles of a wave share.  Rows
// of S in LDS lie so that the four quarters' rows fall on both halves of the
// banks.  Also the fit's inner product sum_rc M[r][c] C[r][c] lambda[c].
// 100k rows at rank 64: 38 us with a workgroup for every 4 tiles, rank 48
// padded to 64 and all four quarters on the same banks.
template <int NB>
struct ApplyShape {
    static constexpr int RP = NB * 16, KS = RP / 4;
    static constexpr int LD = NB == 1 ? 20 : NB == 2 ? 34 : NB == 3 ? 52 : 65;  // LD KS = 16 (mod 32)
};

template <int NB>
__device__ __forceinline__ void apply_tiles(const float *__restrict__ M, int ldm, int64_t rows, int R,
                                            const double *__restrict__ S, float *__restrict__ C,
                                            const double *__restrict__ lambda, double *__restrict__ inner_out,
                                            int64_t t0, int64_t dt, int64_t t1) {
    constexpr int RP = ApplyShape<NB>::RP, KS = ApplyShape<NB>::KS, LD = ApplyShape<NB>::LD;
    __shared__ double sS[RP * LD];
    __shared__ double red[kThreads / 64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int mrow = lane & 15, kq = lane >> 4;
    const bool vec_ok = R == RP && (ldm & 3) == 0 && ((uintptr_t)M & 15u) == 0;
    auto load = [&](float (&a)[KS], int64_t t) {
        const int64_t row = t * 16 + mrow;
        if (vec_ok && t < t1 && row < rows) {
            // the lane's KS values are contiguous and 16-byte aligned: vector loads
            const float4 *mp = reinterpret_cast<const float4 *>(M + row * ldm + kq * KS);
#pragma unroll
            for (int j = 0; j < KS / 4; ++j) {
                const float4 v = mp[j];
                a[4 * j] = v.x;
                a[4 * j + 1] = v.y;
                a[4 * j + 2] = v.z;
                a[4 * j + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                const int c = kq * KS + j;
                a[j] = (t < t1 && row < rows && c < R) ? M[row * ldm + c] : 0.f;
            }
        }
    };
    float a[KS], nxt[KS];
    load(a, t0);
    for (int e = tid; e < RP * RP; e += kThreads) {
        const int p = e / RP, q = e % RP;
        sS[p * LD + q] = (p < R && q < R) ? S[p * R + q] : 0.0;
    }
    __syncthreads();
    double inner = 0.0;
    for (int64_t t = t0; t < t1; t += dt) {
        load(nxt, t + dt);
        double4_t acc[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) acc[cb] = (double4_t){0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            const double av = (double)a[j];
            const double *srow = sS + (kq * KS + j) * LD + mrow;  // B[k][n] = S[k][cb 16 + n], n = lane & 15
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, srow[cb * 16], acc[cb], 0, 0, 0);
        }
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t row = t * 16 + 4 * e + kq;
                const int c = cb * 16 + mrow;
                if (row < rows && c < R) {
                    const float v = (float)acc[cb][e];
                    C[row * R + c] = v;
                    if (inner_out) inner += (double)M[row * ldm + c] * (double)v * lambda[c];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < KS; ++j) a[j] = nxt[j];
    }
    if (inner_out) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) inner += __shfl_down(inner, off, 64);
        if (lane == 0) red[wave] = inner;
        __syncthreads();
        if (tid == 0) {
            double sum = 0.0;
            for (int w = 0; w < kThreads / 64; ++w) sum += red[w];
            *inner_out = sum;
        }
    }
}

template <int NB>
__global__ __launch_bounds__(kThreads) void k_apply(const float *__restrict__ M, int64_t rows, int R,
                                                    const double *__restrict__ S, float *__restrict__ C,
                                                    const double *__restrict__ lambda,
                                                    double *__restrict__ inner_partials) {
    apply_tiles<NB>(M, R, rows, R, S, C, lambda, inner_partials ? inner_partials + blockIdx.x : nullptr,
                    (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6), (int64_t)gridDim.x * (kThreads / 64),
                    (rows + 15) / 16);
}

// Batched: block `g` belongs to the last item whose first_block <= g and takes kApplyBatchRows rows of it.
constexpr int kApplyBatchRows = 128;
template <int NB>
__global__ __launch_bounds__(kThreads) void k_apply_batched(const ApplyItem *__restrict__ items, int count) {
    const int64_t g = blockIdx.x;
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].first_block <= g) lo = mid;
        else hi = mid - 1;
    }
    const ApplyItem &it = items[__builtin_amdgcn_readfirstlane(lo)];
    const int64_t b = g - it.first_block;
    apply_tiles<NB>(it.M, it.ldm, it.rows, it.rank, it.S, it.C, it.lambda, it.inner ? it.inner + b : nullptr,
                    b * (kApplyBatchRows / 16) + (threadIdx.x >> 6), kThreads / 64,
                    min((b + 1) * (kApplyBatchRows / 16), (it.rows + 15) / 16));
}

// ------------------------------------------------------------------ fit
// One workgroup: R^2 products and up to 1024 partial sums, so as wide as it gets.
constexpr int kFitThreads = 1024;
__device__ __forceinline__ void fit_body(const double *__restrict__ grams, int nmodes, int R,
                                         const double *__restrict__ lambda,
                                         const double *__restrict__ inner_partials, int nparts, double norm_x2,
                                         double *__restrict__ out) {
    __shared__ double red[2][kFitThreads / 64];
    const int tid = threadIdx.x;
    const int RR = R * R;
    double xh = 0.0;
    for (int e = tid; e < RR; e += kFitThreads) {
        double v = 1.0;
        for (int k = 0; k < nmodes; ++k) v *= grams[(size_t)k * RR + e];
        xh += lambda[e / R] * v * lambda[e % R];
    }
    double in = 0.0;
    for (int i = tid; i < nparts; i += kFitThreads) in += inner_partials[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        xh += __shfl_down(xh, off, 64);
        in += __shfl_down(in, off, 64);
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = xh;
        red[1][tid >> 6] = in;
    }
    __syncthreads();
    if (tid == 0) {
        double nxh = 0.0, inner = 0.0;
        for (int w = 0; w < kFitThreads / 64; ++w) {
            nxh += red[0][w];
            inner += red[1][w];
        }
        double r2 = norm_x2 + nxh - 2.0 * inner;
        if (r2 < 0.0) r2 = 0.0;
        out[0] = 1.0 - sqrt(r2) / sqrt(norm_x2);
        out[1] = nxh;
        out[2] = inner;
    }
}

__global__ __launch_bounds__(kFitThreads) void k_fit(const double *__restrict__ grams, int nmodes, int R,
                                                  const double *__restrict__ lambda,
                                                  const double *__restrict__ inner_partials, int nparts,
                                                  double norm_x2, double *__restrict__ out,
                                                  const int *__restrict__ status, AlsReport *report, int number) {
    fit_body(grams, nmodes, R, lambda, inner_partials, nparts, norm_x2, out);
    if (threadIdx.x == 0) {
        report->fit = out[0];
        for (int k = 0; k < nmodes; ++k) report->status[k] = status[k];
        __hip_atomic_store(&report->number, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ __launch_bounds__(kFitThreads) void k_fit_batched(const FitItem *__restrict__ items) {
    const FitItem &it = items[blockIdx.x];
    fit_body(it.grams, it.nmodes, it.rank, it.lambda, it.inner, it.nparts, it.norm_x2, it.out);
}

// out[1] must hold |Xhat|^2 from k_fit; writes out[0] (fit) and out[3] (residual^2).
__device__ __forceinline__ void fit_direct_body(const double *__restrict__ parts, int64_t nparts, double norm_x2,
                                                double *__restrict__ out) {
    __shared__ double red[2][4];
    const int tid = threadIdx.x;
    double a = 0.0, b = 0.0;
    for (int64_t i = tid; i < nparts; i += kThreads) {
        a += parts[2 * i];
        b += parts[2 * i + 1];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_down(a, off, 64);
        b += __shfl_down(b, off, 64);
    }
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = a;
        red[1][tid >> 6] = b;
    }
    __syncthreads();
    if (tid == 0) {
        const double res = red[0][0] + red[0][1] + red[0][2] + red[0][3];
        const double hat = red[1][0] + red[1][1] + red[1][2] + red[1][3];
        double off_support = out[1] - hat;  // model mass on the zero cells
        if (off_support < 0.0) off_support = 0.0;
        const double r2 = res + off_support;
        out[0] = 1.0 - sqrt(r2) / sqrt(norm_x2);
        out[3] = r2;
    }
}

__global__ __launch_bounds__(kThreads) void k_fit_direct(const double *__restrict__ parts, int nparts, double norm_x2,
                                                         double *__restrict__ out) {
    fit_direct_body(parts, nparts, norm_x2, out);
}

__global__ __launch_bounds__(kThreads) void k_fit_direct_batched(const FitDirectItem *__restrict__ items) {
    const FitDirectItem &it = items[blockIdx.x];
    fit_direct_body(it.parts, it.nparts, it.norm_x2, it.out);
}

}  // namespace

size_t gram_work_bytes(int64_t rows, int rank) {
    return (size_t)gram_slices_single(rows) * gram_tiles(gram_nb(rank)) * 256 * sizeof(double);
}

spt_status launch_gram(const float *C, int64_t rows, int rank, double *G, double *work, size_t work_bytes,
                       GramRef *ref, hipStream_t s) {
    if (rank > 64) return fail(SPT_E_INVALID_ARG, "gram: rank above 64");
    if (gram_work_bytes(rows, rank) > work_bytes) return fail(SPT_E_INVALID_ARG, "gram: workspace too small");
    const int nb = gram_nb(rank), slices = gram_slices_single(rows);
    const dim3 g((unsigned)slices), b(kGramThreads);
    if (nb == 1) hipLaunchKernelGGL(k_gram_partial<1>, g, b, 0, s, C, rows, rank, work);
    else if (nb == 2) hipLaunchKernelGGL(k_gram_partial<2>, g, b, 0, s, C, rows, rank, work);
    else if (nb == 3) hipLaunchKernelGGL(k_gram_partial<3>, g, b, 0, s, C, rows, rank, work);
    else hipLaunchKernelGGL(k_gram_partial<4>, g, b, 0, s, C, rows, rank, work);
    if (ref && slices <= kGramDirect) {
        *ref = GramRef{work, slices};
    } else {
        hipLaunchKernelGGL(k_gram_sum, dim3(gram_tiles(nb) * 256 / kGramSumElems), dim3(kThreads), 0, s, work, slices, nb,
                           rank, G);
        if (ref) *ref = GramRef{G, 0};
    }
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_solve_prep(const double *grams, int nmodes, int mode, int rank, const GramRef &gram_m, double *S,
                             double *lambda, int *status_out, double *gram_new, hipStream_t s) {
    if (rank > 64) return fail(SPT_E_INVALID_ARG, "solve: rank above 64");
    hipLaunchKernelGGL(k_solve_prep, dim3(1), dim3(kSolveThreads), 0, s, grams, nmodes, mode, rank, gram_m, S, lambda,
                       status_out, gram_new);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

// 4 waves of 16-row tiles a block; from 1024 blocks on (4 per CU at rank 64's
// 33 KB of LDS) every wave takes the same number of tiles.
constexpr int64_t kApplyMaxBlocks = 1024;
int apply_blocks(int64_t rows) {
    const int64_t quads = ((rows + 15) / 16 + 3) / 4;
    const int64_t each = std::max<int64_t>(1, (quads + kApplyMaxBlocks - 1) / kApplyMaxBlocks);
    return (int)std::max<int64_t>(1, (quads + each - 1) / each);
}

spt_status launch_apply(const float *M, int64_t rows, int rank, const double *S, float *C, const double *lambda,
                        double *inner_partials, hipStream_t s) {
    const dim3 g((unsigned)apply_blocks(rows)), b(kThreads);
    const int nb = gram_nb(rank);
    if (nb == 1) hipLaunchKernelGGL(k_apply<1>, g, b, 0, s, M, rows, rank, S, C, lambda, inner_partials);
    else if (nb == 2) hipLaunchKernelGGL(k_apply<2>, g, b, 0, s, M, rows, rank, S, C, lambda, inner_partials);
    else if (nb == 3) hipLaunchKernelGGL(k_apply<3>, g, b, 0, s, M, rows, rank, S, C, lambda, inner_partials);
    else hipLaunchKernelGGL(k_apply<4>, g, b, 0, s, M, rows, rank, S, C, lambda, inner_partials);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_fit(const double *grams, int nmodes, int rank, const double *lambda, const double *inner_partials,
                      int nparts, double norm_x2, double *out, const int *status, AlsReport *report, int number,
                      hipStream_t s) {
    hipLaunchKernelGGL(k_fit, dim3(1), dim3(kFitThreads), 0, s, grams, nmodes, rank, lambda, inner_partials, nparts, norm_x2,
                       out, status, report, number);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_fit_direct_batched(const FitDirectItem *items, int count, hipStream_t s) {
    if (count <= 0) return SPT_OK;
    hipLaunchKernelGGL(k_fit_direct_batched, dim3((unsigned)count), dim3(kThreads), 0, s, items);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_fit_direct(const double *resid_partials, int nparts, double norm_x2, double *out, hipStream_t s) {
    hipLaunchKernelGGL(k_fit_direct, dim3(1), dim3(kThreads), 0, s, resid_partials, nparts, norm_x2, out);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

int64_t gram_slices(int64_t rows) { return std::max<int64_t>(1, (rows + kGramSliceRows - 1) / kGramSliceRows); }

size_t gram_batched_ws_bytes(int64_t total_slices, int rmax) {
    return (size_t)std::max<int64_t>(total_slices, 1) * gram_tiles(gram_nb(rmax)) * 256 * sizeof(double);
}

spt_status launch_gram_batched(const GramItem *items, int count, int64_t total_slices, int rmax, double *work,
                               hipStream_t s) {
    if (count == 0 || total_slices == 0) return SPT_OK;
    if (rmax > 64) return fail(SPT_E_INVALID_ARG, "gram: rank above 64");
    const int nb = gram_nb(rmax);
    const dim3 g((unsigned)total_slices), b(kGramThreads);
    if (nb == 1) hipLaunchKernelGGL(k_gram_batched_partial<1>, g, b, 0, s, items, count, work);
    else if (nb == 2) hipLaunchKernelGGL(k_gram_batched_partial<2>, g, b, 0, s, items, count, work);
    else if (nb == 3) hipLaunchKernelGGL(k_gram_batched_partial<3>, g, b, 0, s, items, count, work);
    else hipLaunchKernelGGL(k_gram_batched_partial<4>, g, b, 0, s, items, count, work);
    for (int c0 = 0; c0 < count; c0 += 65535) {  // grid rows
        const int c = std::min(count - c0, 65535);
        hipLaunchKernelGGL(k_gram_sum_batched, dim3(gram_tiles(nb) * 256 / kGramSumElems, c), dim3(kThreads), 0, s,
                           items + c0, nb, work);
    }
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_solve_prep_batched(const SolveItem *items, int count, int mode, hipStream_t s) {
    if (count == 0) return SPT_OK;
    hipLaunchKernelGGL(k_solve_prep_batched, dim3(count), dim3(kSolveThreads), 0, s, items, mode);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

int apply_batch_rows() { return kApplyBatchRows; }

spt_status launch_apply_batched(const ApplyItem *items, int count, int64_t total_blocks, int rmax, hipStream_t s) {
    if (total_blocks == 0) return SPT_OK;
    const dim3 g((unsigned)total_blocks), b(kThreads);
    const int nb = gram_nb(rmax);
    if (nb == 1) hipLaunchKernelGGL(k_apply_batched<1>, g, b, 0, s, items, count);
    else if (nb == 2) hipLaunchKernelGGL(k_apply_batched<2>, g, b, 0, s, items, count);
    else if (nb == 3) hipLaunchKernelGGL(k_apply_batched<3>, g, b, 0, s, items, count);
    else hipLaunchKernelGGL(k_apply_batched<4>, g, b, 0, s, items, count);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

spt_status launch_fit_batched(const FitItem *items, int count, hipStream_t s) {
    if (count == 0) return SPT_OK;
    hipLaunchKernelGGL(k_fit_batched, dim3(count), dim3(kFitThreads), 0, s, items);
    SPT_HIP(hipGetLastError());
    return SPT_OK;
}

}  // namespace spt
