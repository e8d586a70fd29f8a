// Device helpers shared by the MTTKRP kernels.
#pragma once

#include "spt_internal.h"

namespace spt {

// Workgroups are dealt round-robin over the 8 XCDs.  Each XCD gets runs of
// kXcdChunk consecutive work indices (its L2 sees the key-order locality
// inside a run), and the runs of the 8 XCDs interleave over the whole index
// range, so a heavy stretch of the tensor is shared by all XCDs instead of
// landing on one (one contiguous eighth per XCD left the last XCD running
// 1.5x longer than the first on skewed tensors).  A bijection on [0, nwg):
// the indices past the last full round of 8 runs map to themselves.
constexpr int64_t kXcdChunk = 64;
__device__ __forceinline__ int64_t xcd_remap(int64_t b, int64_t nwg) {
    const int64_t full = (nwg / (8 * kXcdChunk)) * (8 * kXcdChunk);
    if (b >= full) return b;
    const int64_t x = b & 7, j = b >> 3;
    return ((j / kXcdChunk) * 8 + x) * kXcdChunk + (j % kXcdChunk);
}

template <int VEC>
__device__ __forceinline__ void load_vec(const float *p, float (&x)[VEC]) {
    if constexpr (VEC == 4) {
        const float4 t = *reinterpret_cast<const float4 *>(p);
        x[0] = t.x;
        x[1] = t.y;
        x[2] = t.z;
        x[3] = t.w;
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) x[q] = p[q];
    }
}

typedef float spt_f4 __attribute__((ext_vector_type(4)));
// Four floats at any 4-byte boundary (a row of a rank that is no multiple of
// 4): global memory takes them as one 16-byte access all the same.
typedef float spt_f4u __attribute__((ext_vector_type(4), aligned(4)));

template <int VEC>
__device__ __forceinline__ void load_vec_any(const float *p, float (&x)[VEC]) {
    if constexpr (VEC == 4) {
        const spt_f4u t = *reinterpret_cast<const spt_f4u *>(p);
        x[0] = t.x;
        x[1] = t.y;
        x[2] = t.z;
        x[3] = t.w;
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) x[q] = p[q];
    }
}

// two doubles likewise
typedef double spt_d2u __attribute__((ext_vector_type(2), aligned(8)));

template <int VEC>
__device__ __forceinline__ void load_vec_any(const double *p, double (&x)[VEC]) {
    if constexpr (VEC % 2 == 0) {
#pragma unroll
        for (int q = 0; q < VEC; q += 2) {
            const spt_d2u t = *reinterpret_cast<const spt_d2u *>(p + q);
            x[q] = t.x;
            x[q + 1] = t.y;
        }
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) x[q] = p[q];
    }
}

template <int VEC>
__device__ __forceinline__ void store_vec(double *p, const double (&x)[VEC]) {
    if constexpr (VEC % 2 == 0) {
#pragma unroll
        for (int q = 0; q < VEC; q += 2) {
            const spt_d2u t = {x[q], x[q + 1]};
            *reinterpret_cast<spt_d2u *>(p + q) = t;
        }
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) p[q] = x[q];
    }
}

template <int VEC>
__device__ __forceinline__ void store_vec(float *p, const float (&x)[VEC]) {
    if constexpr (VEC == 4) {
        const spt_f4u t = {x[0], x[1], x[2], x[3]};
        *reinterpret_cast<spt_f4u *>(p) = t;
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) p[q] = x[q];
    }
}

// Lane groups of the walk: a record's R columns are owned by G consecutive
// lanes of one wave, 64 / G groups to a wave (the lanes left over sit the walk
// out).  VEC 4 (R >= 4): G = ceil(R / 4) lanes of 4 columns each; the last
// lane takes the row's last 4 columns, so at a rank that is no multiple of 4
// it repeats up to 3 columns of its neighbour with the same values instead of
// idling or masking.  VEC 1 (R < 4): one column a lane.
// Packing by ceil(R / 4) and not by the next power of two (and, at ranks that
// are no multiple of 4, instead of one column a lane over the whole wave) puts
// more nonzeros in flight per wave for the same row bytes.  All-mode sweeps,
// before and after: rank 25, 5 modes, 5M nonzeros 6.97 / 0.88 ms (with the
// 5-mode walk that issues all gathers of a step at once); rank 10, 4 modes, 3M
// nonzeros 2.78 / 1.11 ms; ranks 32 and 64, where the groups are the same
// lanes as before, 4.53 / 4.55 and 13.65 / 13.62 ms.
struct LaneGroup {
    int G, per_wave, j, col;  // lanes per group, groups per wave, lane in the group, first column
    int g;                    // group in the workgroup
    bool on;
};
template <int VEC>
__device__ __forceinline__ LaneGroup lane_group(int R, int tid) {
    LaneGroup q;
    q.G = VEC > 1 ? (R + VEC - 1) / VEC : R;
    q.per_wave = 64 / q.G;
    const int lane = tid & 63, w = tid >> 6, gl = lane / q.G;
    q.j = lane - gl * q.G;
    q.col = VEC > 1 ? min(VEC * q.j, R - VEC) : q.j;
    q.g = w * q.per_wave + gl;
    q.on = gl < q.per_wave;
    return q;
}
template <int VEC>
__device__ __forceinline__ LaneGroup lane_group(int R) {
    return lane_group<VEC>(R, threadIdx.x);
}

// Zeroes slice `i` of `of` of an array of n floats (16-byte aligned, or null): a kernel
// whose workgroups wait on other things clears the output of the kernel that
// follows it on the way, which costs that launch and not its bytes.
__device__ __forceinline__ void zero_slice(float *__restrict__ p, int64_t n, int64_t i, int64_t of) {
    if (!p) return;
    const int64_t per = ((n + of - 1) / of + 3) & ~int64_t(3);
    const int64_t a = i * per, b = min(a + per, n);
    const spt_f4 z = {0.f, 0.f, 0.f, 0.f};
    for (int64_t e = a + 4 * (int64_t)threadIdx.x; e < b; e += 4 * (int64_t)blockDim.x) {
        if (e + 4 <= b) {
            __builtin_nontemporal_store(z, reinterpret_cast<spt_f4 *>(p + e));
        } else {
            for (int64_t k = e; k < b; ++k) p[k] = 0.f;
        }
    }
}

// A factor matrix seen as a structured buffer whose records are its rows
// (stride R floats): a gather passes the row index and the column's byte
// offset straight to the load, with no address arithmetic, and rows past
// `rows` read as zero.  The descriptor is wave-uniform (SGPRs); R <= 4095.
// The hardware forms the byte offset of a row in 32 bits: for arrays up to
// kBufferBytes (RowView has the others).
typedef int spt_i4 __attribute__((ext_vector_type(4)));
typedef uint32_t spt_u4 __attribute__((ext_vector_type(4)));
__device__ spt_f4 spt_row_load4(spt_i4 rsrc, int vindex, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.struct.buffer.load.v4f32");
__device__ float spt_row_load1(spt_i4 rsrc, int vindex, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.struct.buffer.load.f32");

__device__ uint32_t spt_word_load(spt_i4 rsrc, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.raw.buffer.load.i32");
__device__ void spt_row_store4(spt_f4 x, spt_i4 rsrc, int vindex, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.struct.buffer.store.v4f32");
__device__ void spt_row_store1(float x, spt_i4 rsrc, int vindex, int voffset, int soffset, int aux) __asm(
    "llvm.amdgcn.struct.buffer.store.f32");

// n 32-bit words, the same for all lanes; reads past them give 0
__device__ __forceinline__ spt_i4 word_rsrc(const uint32_t *base, uint32_t n) {
    const uint64_t p = (uint64_t)base;
    return spt_i4{__builtin_amdgcn_readfirstlane((int)(uint32_t)p),
                  __builtin_amdgcn_readfirstlane((int)((uint32_t)(p >> 32) & 0xFFFFu)),
                  __builtin_amdgcn_readfirstlane((int)(n * 4)), 0x00020000};
}

__device__ __forceinline__ spt_i4 row_rsrc(const float *base, int R, uint32_t rows) {
    const uint64_t p = (uint64_t)base;
    spt_i4 r;
    r.x = (int)(uint32_t)p;
    r.y = (int)(((uint32_t)(p >> 32) & 0xFFFFu) | ((uint32_t)(R * 4) << 16));  // base[47:32] | stride
    r.z = (int)rows;                                                            // records
    r.w = 0x00020000;                                                           // 32-bit data format
    return r;
}

template <int VEC>
__device__ __forceinline__ void load_row_vec(spt_i4 rsrc, uint32_t row, int col, float (&x)[VEC]) {
    if constexpr (VEC == 4) {
        const spt_f4 t = spt_row_load4(rsrc, (int)row, col * 4, 0, 0);
        x[0] = t.x;
        x[1] = t.y;
        x[2] = t.z;
        x[3] = t.w;
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) x[q] = spt_row_load1(rsrc, (int)row, (col + q) * 4, 0, 0);
    }
}

// the same for FP64 rows
__device__ __forceinline__ spt_i4 row_rsrc(const double *base, int R, uint32_t rows) {
    return row_rsrc(reinterpret_cast<const float *>(base), 2 * R, rows);
}

template <int VEC>
__device__ __forceinline__ void load_row_vec(spt_i4 rsrc, uint32_t row, int col, double (&x)[VEC]) {
    if constexpr (VEC % 2 == 0) {
#pragma unroll
        for (int q = 0; q < VEC; q += 2) {
            const spt_f4 t = spt_row_load4(rsrc, (int)row, (col + q) * 8, 0, 0);
            x[q] = __hiloint2double(__float_as_int(t.y), __float_as_int(t.x));
            x[q + 1] = __hiloint2double(__float_as_int(t.w), __float_as_int(t.z));
        }
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) {
            const float lo = spt_row_load1(rsrc, (int)row, (col + q) * 8, 0, 0);
            const float hi = spt_row_load1(rsrc, (int)row, (col + q) * 8 + 4, 0, 0);
            x[q] = __hiloint2double(__float_as_int(hi), __float_as_int(lo));
        }
    }
}

// Rows past the buffer's are not written.
template <int VEC>
__device__ __forceinline__ void store_row_vec(spt_i4 rsrc, uint32_t row, int col, const float (&x)[VEC]) {
    if constexpr (VEC == 4) {
        spt_row_store4(spt_f4{x[0], x[1], x[2], x[3]}, rsrc, (int)row, col * 4, 0, 0);
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) spt_row_store1(x[q], rsrc, (int)row, (col + q) * 4, 0, 0);
    }
}

template <int VEC>
__device__ __forceinline__ void store_row_vec(spt_i4 rsrc, uint32_t row, int col, const double (&x)[VEC]) {
    if constexpr (VEC % 2 == 0) {
#pragma unroll
        for (int q = 0; q < VEC; q += 2)
            spt_row_store4(spt_f4{__int_as_float(__double2loint(x[q])), __int_as_float(__double2hiint(x[q])),
                                  __int_as_float(__double2loint(x[q + 1])), __int_as_float(__double2hiint(x[q + 1]))},
                           rsrc, (int)row, (col + q) * 8, 0, 0);
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) {
            spt_row_store1(__int_as_float(__double2loint(x[q])), rsrc, (int)row, (col + q) * 8, 0, 0);
            spt_row_store1(__int_as_float(__double2hiint(x[q])), rsrc, (int)row, (col + q) * 8 + 4, 0, 0);
        }
    }
}

// A row-major matrix of `rows` rows of R values as the walk reads or writes it:
// a structured buffer or, FAR, 64-bit addresses.  Rows past the last read as
// zeros or as the last row (FAR), and are not written.
template <class Real, bool FAR>
struct RowView {
    spt_i4 r;
    __device__ __forceinline__ RowView() {}
    __device__ __forceinline__ RowView(const Real *p, int R, uint32_t rows) : r(row_rsrc(p, R, rows)) {}
    template <int VEC>
    __device__ __forceinline__ void load(uint32_t row, int col, Real (&x)[VEC]) const {
        load_row_vec<VEC>(r, row, col, x);
    }
    template <int VEC>
    __device__ __forceinline__ void store(uint32_t row, int col, const Real (&x)[VEC]) const {
        store_row_vec<VEC>(r, row, col, x);
    }
};

template <class Real>
struct RowView<Real, true> {
    const Real *p;
    int R;
    uint32_t rows;
    __device__ __forceinline__ RowView() {}
    __device__ __forceinline__ RowView(const Real *q, int ld, uint32_t n) : p(q), R(ld), rows(n) {}
    template <int VEC>
    __device__ __forceinline__ void load(uint32_t row, int col, Real (&x)[VEC]) const {
        load_vec_any<VEC>(p + (size_t)min(row, rows - 1) * R + col, x);
    }
    template <int VEC>
    __device__ __forceinline__ void store(uint32_t row, int col, const Real (&x)[VEC]) const {
        if (row < rows) store_vec<VEC>(const_cast<Real *>(p) + (size_t)row * R + col, x);
    }
};

// The codec held in VGPRs: lane l of every wave keeps run descriptors l,
// l + 64 and l + 128 and the run bound rb[l / 5][l % 5].  Decoding reads them
// with v_readlane at wave-uniform indices: no memory access, no LDS wait.
struct CodecRegs {
    uint32_t r0, r1, r2, rb;
};

__device__ __forceinline__ CodecRegs load_codec_regs(const Codec &c) {
    const int lane = threadIdx.x & 63;
    CodecRegs cr;
    cr.r0 = lane < c.nruns ? c.run[lane] : 0u;
    cr.r1 = lane + 64 < c.nruns ? c.run[lane + 64] : 0u;
    cr.r2 = lane + 128 < c.nruns ? c.run[lane + 128] : 0u;
    cr.rb = lane < kMaxModes * 5 ? (uint32_t)(&c.rb[0][0])[lane] : 0u;
    return cr;
}

__device__ __forceinline__ uint32_t run_desc(const CodecRegs &cr, int r) {
    if (r < 64) return __builtin_amdgcn_readlane(cr.r0, r);
    if (r < 128) return __builtin_amdgcn_readlane(cr.r1, r - 64);
    return __builtin_amdgcn_readlane(cr.r2, r - 128);
}

// Coordinate of mode k from the four 32-bit words of one key.  A descriptor
// d packs word | kpos << 8 | cpos << 16 | len << 24 (len <= 31).
__device__ __forceinline__ uint32_t decode_mode(const CodecRegs &cr, int k, int nwords, const uint32_t (&w)[4]) {
    uint32_t x = 0;
#pragma unroll
    for (int word = 0; word < 4; ++word) {
        if (word < nwords) {
            const int r0 = __builtin_amdgcn_readlane(cr.rb, k * 5 + word);
            const int r1 = __builtin_amdgcn_readlane(cr.rb, k * 5 + word + 1);
            for (int r = r0; r < r1; ++r) {
                const uint32_t d = run_desc(cr, r);
                x |= __builtin_amdgcn_ubfe(w[word], (d >> 8) & 31u, d >> 24) << ((d >> 16) & 31u);
            }
        }
    }
    return x;
}

// In-place exclusive scan of n u32 values in LDS by a block of nthreads
// (n a multiple of nthreads); wsum holds one entry per wave.
__device__ __forceinline__ void block_scan_lds(uint32_t *a, int n, int nthreads, uint32_t *wsum) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = n / nthreads;
    uint32_t *p = a + tid * per;
    uint32_t local = 0;
    for (int i = 0; i < per; ++i) local += p[i];
    uint32_t x = local;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint32_t run = x - local;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    for (int i = 0; i < per; ++i) {
        const uint32_t v = p[i];
        p[i] = run;
        run += v;
    }
    __syncthreads();
}

__device__ __forceinline__ uint32_t mix_hash(uint32_t r) {
    r ^= r >> 16;
    r *= 0x7feb352dU;
    r ^= r >> 15;
    return r;
}

}  // namespace spt
