// Epilogues of the projection kernels (gemm.hip, f32.hip).
#pragma once

#include <type_traits>

#include "common.h"
#include "launch.h"

namespace mtp {

// ---------------------------------------------------------------- epilogues
// An epilogue stores 4 consecutive n of one row m.  Its operands come in
// three groups, so that a kernel storing many (m, n) issues their loads
// ahead of its stores:
//   RowKey  row_key(m)   one per output row (EpiQKV: its sequence and position)
//   RowPre  row(key)     one per output row (EpiQKV: its cache page, a load
//                        that depends on the key: all keys of a kernel's rows
//                        are loaded before any of these)
//   ColPre  col(n)       one per 4-column group (the biases)
//   ElemPre elem(m, n)   one per 4 outputs (EpiResid: the residual values)
//   store(rp, cp, ep, m, n, v, split, nvalid)
// A load that follows a store it may alias cannot move above it, and vmcnt
// counts stores as well as loads, so an epilogue that loads inside each
// store4 waits one full memory round trip per store (32-64 per wave in the
// large kernel).  The loads take clamped, valid m and n (the callers pass
// m < M and n < N or the last valid ones); only the stores are guarded.
// ok(rp) says whether a row is stored at all (EpiQKV: not a padding row);
// store<true> may assume it is, so that a kernel whose wave holds only such
// rows issues the same stores on every lane (a lane-dependent branch around
// a store leaves the compiler unable to count the stores in flight, and it
// then waits for all of them before the next one).
struct EpiNoPre {};

template <class Epi>
__device__ __forceinline__ void epi_store4(const Epi& e, int m, int n, const float (&v)[4], int split, int nvalid) {
    e.template store<false>(e.row(e.row_key(m)), e.col(n), e.elem(m, n), m, n, v, split, nvalid);
}

__device__ __forceinline__ uint32_t epi_pk2(float a, float b) {
    return bf16x2_bits(a, b);
}

template <typename KVT>
struct EpiQKV {
    float* q;            // [M][d] queries (fp32)
    const float* bias;   // [3d]
    const RowInfo* rows;
    KVView kv;
    int d;
    using RowKey = RowInfo;
    struct RowPre { int page, pos; };        // pos < 0: a padding row (no cache write)
    using ColPre = float4;
    using ElemPre = EpiNoPre;
    __device__ __forceinline__ RowKey row_key(int m) const { return rows[m]; }
    // the page stays as loaded (nothing computed from it before the stores)
    __device__ __forceinline__ RowPre row(const RowKey& ri) const {
        const int pos = max(ri.pos, 0), seq = max(ri.seq, 0);
        return RowPre{kv.block_table[(size_t)seq * kv.max_pages_per_seq + (pos >> kv.page_shift)], ri.pos};
    }
    __device__ __forceinline__ ColPre col(int n) const { return *reinterpret_cast<const float4*>(bias + n); }
    __device__ __forceinline__ ElemPre elem(int, int) const { return {}; }
    __device__ __forceinline__ bool ok(const RowPre& rp) const { return rp.pos >= 0; }
    // every caller's wave holds 16 consecutive columns inside one section
    // (d is a multiple of 64), so the section is wave-uniform
    template <bool ROWS_OK>
    __device__ __forceinline__ void store(const RowPre& rp, const ColPre& bv, const ElemPre&, int m, int n,
                                          const float (&v)[4], int, int) const {
        const float r0 = v[0] + bv.x, r1 = v[1] + bv.y, r2 = v[2] + bv.z, r3 = v[3] + bv.w;
        const int sec = __builtin_amdgcn_readfirstlane((n >= d) + (n >= 2 * d));   // q, k or v
        if (sec == 0) {
            *reinterpret_cast<float4*>(q + (size_t)m * d + n) = make_float4(r0, r1, r2, r3);
            return;
        }
        if (!ROWS_OK && rp.pos < 0) return;
        const int c = n - sec * d;
        const int slot = rp.pos & (kv.page_size - 1);
        KVT* blk = reinterpret_cast<KVT*>(kv.pool) + kv_page_block(kv, rp.page, sec - 1, c >> 6);
        if constexpr (sizeof(KVT) == 2) {
            if (sec == 2) {   // transposed V block: [dim][slot]
                bf16_t* vt = blk + (size_t)(c & 63) * kv.page_size + slot;
                vt[0] = f32_to_bf16(r0);
                vt[kv.page_size] = f32_to_bf16(r1);
                vt[2 * kv.page_size] = f32_to_bf16(r2);
                vt[3 * kv.page_size] = f32_to_bf16(r3);
                return;
            }
            *reinterpret_cast<uint2*>(blk + (size_t)slot * MTP_HEAD_DIM + (c & 63)) =
                make_uint2(epi_pk2(r0, r1), epi_pk2(r2, r3));
        } else {
            *reinterpret_cast<float4*>(blk + (size_t)slot * MTP_HEAD_DIM + (c & 63)) = make_float4(r0, r1, r2, r3);
        }
    }
};

template <typename OutT>
struct EpiGelu {
    OutT* out;
    const float* bias;
    int ldo;
    int pk;               // bf16 output in fragment order (K = ldo)
    using RowKey = EpiNoPre;
    using RowPre = EpiNoPre;
    using ColPre = float4;
    using ElemPre = EpiNoPre;
    __device__ __forceinline__ RowKey row_key(int) const { return {}; }
    __device__ __forceinline__ RowPre row(const RowKey&) const { return {}; }
    __device__ __forceinline__ ColPre col(int n) const { return *reinterpret_cast<const float4*>(bias + n); }
    __device__ __forceinline__ ElemPre elem(int, int) const { return {}; }
    __device__ __forceinline__ bool ok(const RowPre&) const { return true; }
    template <bool ROWS_OK>
    __device__ __forceinline__ void store(const RowPre&, const ColPre& bv, const ElemPre&, int m, int n,
                                          const float (&v)[4], int, int) const {
        const float r[4] = {gelu_erf(v[0] + bv.x), gelu_erf(v[1] + bv.y), gelu_erf(v[2] + bv.z), gelu_erf(v[3] + bv.w)};
        OutT* p = out + (pk ? frag_off(m, n, ldo) : (size_t)m * ldo + n);
        if constexpr (sizeof(OutT) == 2) {
            *reinterpret_cast<uint2*>(p) = make_uint2(epi_pk2(r[0], r[1]), epi_pk2(r[2], r[3]));
        } else {
            *reinterpret_cast<float4*>(p) = make_float4(r[0], r[1], r[2], r[3]);
        }
    }
};

struct EpiPartial {
    float* part;          // [split][M][ldo]
    int ldo;
    size_t split_stride;  // elements between splits
    using RowKey = EpiNoPre;
    using RowPre = EpiNoPre;
    using ColPre = EpiNoPre;
    using ElemPre = EpiNoPre;
    __device__ __forceinline__ RowKey row_key(int) const { return {}; }
    __device__ __forceinline__ RowPre row(const RowKey&) const { return {}; }
    __device__ __forceinline__ ColPre col(int) const { return {}; }
    __device__ __forceinline__ ElemPre elem(int, int) const { return {}; }
    __device__ __forceinline__ bool ok(const RowPre&) const { return true; }
    template <bool ROWS_OK>
    __device__ __forceinline__ void store(const RowPre&, const ColPre&, const ElemPre&, int m, int n,
                                          const float (&v)[4], int split, int) const {
        *reinterpret_cast<float4*>(part + split * split_stride + (size_t)m * ldo + n) =
            make_float4(v[0], v[1], v[2], v[3]);
    }
};

// h[m][n..n+3] += product + bias: the residual stream updated in place by a
// projection with no K split (every (m, n) belongs to one workgroup, so the
// read-modify-write is race free); the same association as resid_ln_kernel.
struct EpiResid {
    float* h;             // [M][ldh]
    const float* bias;    // [N]
    int ldh;
    using RowKey = EpiNoPre;
    using RowPre = EpiNoPre;
    using ColPre = float4;
    using ElemPre = float4;
    __device__ __forceinline__ RowKey row_key(int) const { return {}; }
    __device__ __forceinline__ RowPre row(const RowKey&) const { return {}; }
    __device__ __forceinline__ ColPre col(int n) const { return *reinterpret_cast<const float4*>(bias + n); }
    __device__ __forceinline__ ElemPre elem(int m, int n) const {
        return *reinterpret_cast<const float4*>(h + (size_t)m * ldh + n);
    }
    __device__ __forceinline__ bool ok(const RowPre&) const { return true; }
    template <bool ROWS_OK>
    __device__ __forceinline__ void store(const RowPre&, const ColPre& bv, const ElemPre& x, int m, int n,
                                          const float (&v)[4], int, int) const {
        *reinterpret_cast<float4*>(h + (size_t)m * ldh + n) =
            make_float4(x.x + (v[0] + bv.x), x.y + (v[1] + bv.y), x.z + (v[2] + bv.z), x.w + (v[3] + bv.w));
    }
};

struct EpiLogits {
    float* out;           // [M][ldo]
    const float* bias;    // [N]
    int ldo;
    int N;
    using RowKey = EpiNoPre;
    using RowPre = EpiNoPre;
    using ColPre = float4;
    using ElemPre = EpiNoPre;
    __device__ __forceinline__ RowKey row_key(int) const { return {}; }
    __device__ __forceinline__ RowPre row(const RowKey&) const { return {}; }
    __device__ __forceinline__ ColPre col(int n) const {
        return make_float4(bias[min(n, N - 1)], bias[min(n + 1, N - 1)], bias[min(n + 2, N - 1)], bias[min(n + 3, N - 1)]);
    }
    __device__ __forceinline__ ElemPre elem(int, int) const { return {}; }
    __device__ __forceinline__ bool ok(const RowPre&) const { return true; }
    template <bool ROWS_OK>
    __device__ __forceinline__ void store(const RowPre&, const ColPre& bv, const ElemPre&, int m, int n,
                                          const float (&v)[4], int, int nvalid) const {
        float* p = out + (size_t)m * ldo + n;
        const float b[4] = {bv.x, bv.y, bv.z, bv.w};
        for (int i = 0; i < nvalid; ++i) p[i] = v[i] + b[i];
    }
};

}  // namespace mtp
