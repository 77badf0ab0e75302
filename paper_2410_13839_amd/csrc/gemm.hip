// GEMM kernels of the decoder trunk and the fused K-head projection.
//
// All products are "NT": C[m][n] = sum_k X[m][k] * W[n][k], with X the
// activations ([M][K], row-major) and W a Linear weight ([N][K], row-major),
// so both operands are K-contiguous.  Outputs go through an epilogue functor
// that receives 4 consecutive n of one row m.
//
//  * gemm_med_bf16: M <= 256 (decode rows of the batched path, the heads).
//    A weight stream (M = 128 rows is ~128 flop per weight byte, below the
//    MFMA / HBM ridge), so W fragments go straight from HBM into MFMA
//    registers (no LDS round trip), 16 waves per workgroup split the K range,
//    each wave loading its own activation fragments from L2 (no LDS staging:
//    no two waves read the same k), and one LDS reduction over the waves
//    precedes the epilogue.  The grid is sized so every CU streams.
//  * gemm_big_bf16: M > 256 (prefill, NAR).  256 x 256 tiles on MFMA with
//    both operands streamed global -> LDS in fragment order.
// The fp32 model's products are in f32.hip.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "epilogue.h"
#include "launch.h"

namespace mtp {

// ---------------------------------------------------------------- medium bf16
// Workgroup (x, y, z) = (NT 16-column tiles, 16*MT-row group, K split).  Wave
// w takes k steps w, w + 16, ... of its split (32 k per step), up to MAXST at
// a time, all loads of a round in flight together: NT weight fragments
// (packed order, each one contiguous 1 KB wave load) and one 16 x 32
// activation fragment per row tile, which serves all NT column tiles (the
// activations are re-read from L2 once per column group, so wider groups
// cut that traffic).  Rows beyond M read the last valid row and column tiles
// beyond N the last valid tile; neither is stored.  The wave index is made
// scalar so the step guards are uniform branches.
constexpr int GM_NW = 16;

template <int MT, int NT, int MAXST, int XP, class Epi>
__global__ __launch_bounds__(64 * GM_NW) void gemm_med_bf16(const bf16_t* __restrict__ X, int ldx, int M,
                                                            const bf16_t* __restrict__ W, int N, int K,
                                                            int k_per_split, Epi epi) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int ntiles = (N + 15) >> 4;
    const int nt0 = blockIdx.x * NT;
    const int m0 = blockIdx.y * 16 * MT;
    const int split = blockIdx.z;
    const int kb = split * k_per_split;
    const int nsteps = k_per_split >> 5;
    const bf16_t* wp[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
        wp[j] = W + ((size_t)min(nt0 + j, ntiles - 1) * (K >> 5) + (kb >> 5)) * 512 + lane * 8;
    // XP: X in fragment order (one contiguous 1 KB block per row tile and k
    // step, rows padded to 16), else row-major
    const bf16_t* xp[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        if (XP) {
            const int t = min(m0 / 16 + mt, (M - 1) >> 4);
            xp[mt] = X + ((size_t)t * (K >> 5) + (kb >> 5)) * 512 + lane * 8;
        } else {
            const int m = min(m0 + 16 * mt + r, M - 1);
            xp[mt] = X + (size_t)m * ldx + kb + g * 8;
        }
    }
    f32x4_t acc[NT][MT];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) acc[j][mt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    for (int s0 = wave; s0 < nsteps; s0 += GM_NW * MAXST) {
        uint4 wv[MAXST][NT];
        uint4 xv[MAXST][MT];
#pragma unroll
        for (int u = 0; u < MAXST; ++u) {
            const int ss = s0 + GM_NW * u;
            if (ss < nsteps) {
#pragma unroll
                for (int j = 0; j < NT; ++j) wv[u][j] = *reinterpret_cast<const uint4*>(wp[j] + (size_t)ss * 512);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
                    xv[u][mt] = *reinterpret_cast<const uint4*>(xp[mt] + (XP ? (size_t)ss * 512 : (size_t)ss * 32));
            }
        }
#pragma unroll
        for (int u = 0; u < MAXST; ++u) {
            if (s0 + GM_NW * u < nsteps) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        acc[j][mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, wv[u][j]),
                                                                             __builtin_bit_cast(bf16x8_t, xv[u][mt]),
                                                                             acc[j][mt], 0, 0, 0);
            }
        }
    }

    // one output item (4 columns of one row) per thread: its epilogue
    // operands load while the waves' sums go through LDS
    static_assert(NT * MT * 64 <= 64 * GM_NW, "one epilogue item per thread");
    const int t = threadIdx.x;
    const int jm = min(t >> 6, NT * MT - 1), l = t & 63;
    const int j = jm / MT, mt = jm - j * MT;
    const int m = m0 + 16 * mt + (l & 15);
    const int n = (nt0 + j) * 16 + 4 * (l >> 4);
    const int mc = min(m, M - 1), nc = n < N ? n : ((N - 1) & ~3);
    const typename Epi::RowPre rp = epi.row(epi.row_key(mc));
    const typename Epi::ColPre cp = epi.col(nc);
    const typename Epi::ElemPre ep = epi.elem(mc, nc);
    __shared__ f32x4_t red[GM_NW][NT * MT][64];
#pragma unroll
    for (int j2 = 0; j2 < NT; ++j2)
#pragma unroll
        for (int mt2 = 0; mt2 < MT; ++mt2) red[wave][j2 * MT + mt2][lane] = acc[j2][mt2];
    __syncthreads();
    if (t < NT * MT * 64) {
        f32x4_t s = red[0][jm][l];
#pragma unroll
        for (int w = 1; w < GM_NW; ++w) s += red[w][jm][l];
        if (m < M && n < N) {
            const float v[4] = {s[0], s[1], s[2], s[3]};
            epi.template store<false>(rp, cp, ep, m, n, v, split, min(4, N - n));
        }
    }
}

// Column tiles per workgroup: two, so every activation fragment serves two
// weight fragments (the activations are re-read once per workgroup), with
// the LDS reduction holding 16 waves x NT x MT tiles (at most 8).
constexpr int GM_NT = 2;

template <int MT, int XP, class Epi>
static void launch_med(hipStream_t st, const bf16_t* X, int ldx, int M, const bf16_t* W, int N, int K, int splits,
                       Epi epi) {
    constexpr int NT = GM_NT;
    static_assert(NT * MT <= 8, "LDS reduction");
    const int kps = K / splits;
    const int per_wave = ((kps >> 5) + GM_NW - 1) / GM_NW;   // k steps per wave
    dim3 grid(((N + 15) / 16 + NT - 1) / NT, (M + 16 * MT - 1) / (16 * MT), splits);
    dim3 block(64 * GM_NW);
    // one round of loads holds at most MAXST x (NT + MT) fragments per wave
    constexpr int CAP = NT * MT >= 8 ? 2 : 4;
    if (per_wave <= 1)
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, 1, XP, Epi>), grid, block, 0, st, X, ldx, M, W, N, K, kps, epi);
    else if (per_wave == 2 || CAP == 2)
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, 2, XP, Epi>), grid, block, 0, st, X, ldx, M, W, N, K, kps, epi);
    else if (per_wave == 3)
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, 3, XP, Epi>), grid, block, 0, st, X, ldx, M, W, N, K, kps, epi);
    else
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, CAP, XP, Epi>), grid, block, 0, st, X, ldx, M, W, N, K, kps, epi);
}

template <int MT, class Epi>
static void launch_med_x(hipStream_t st, const bf16_t* X, int ldx, int M, const bf16_t* W, int N, int K, int splits,
                         int xpk, Epi epi) {
    if (xpk) launch_med<MT, 1>(st, X, ldx, M, W, N, K, splits, epi);
    else launch_med<MT, 0>(st, X, ldx, M, W, N, K, splits, epi);
}

// ---------------------------------------------------------------- large bf16
// M > 256 (prefill, NAR).  Tiles of BM rows x BN columns (256 x 256 and
// 256 x 128 with 8 waves in a 2 x 4 grid, each wave owning 128 x BN/4
// outputs as 8 x BN/64 v_mfma_f32_16x16x32_bf16 tiles; 128 x 128 with 4
// waves in a 2 x 2 grid, 64 x 64 outputs each, for products too small to
// give the CUs enough of the larger tiles).  Both
// operands are in fragment order (activations written so by their producers,
// weights packed at load), so a 16 x 32 fragment is one contiguous 1 KB; it
// travels global -> LDS by one global_load_lds_dwordx4 per wave (lane l's 16
// bytes land at byte 16 l, the order the MFMA operand read wants: every
// ds_read_b128 is conflict free) with no register staging.  K advances 32 per
// stage through NS = 4 LDS stages, NS - 1 of them in flight while one is
// consumed.  Each stage buffer is its own LDS object and the stage loop is
// unrolled by NS, so the compiler's LDS-DMA waits see which buffer a read
// touches.  Workgroups are numbered so that the ones sharing an XCD (the
// dispatcher deals workgroups to the 8 XCDs in turn) take neighbouring tiles
// of one row band, which they share through that XCD's L2.
constexpr int GB_NS = 4;

__device__ __forceinline__ constexpr int vmcnt_imm(int n) {
    // s_waitcnt immediate: vmcnt = n, expcnt and lgkmcnt not waited on
    return (n & 15) | (((n >> 4) & 3) << 14) | (7 << 4) | (15 << 8);
}

// Workgroup barrier without the memory fence __syncthreads() adds: that
// fence waits for every outstanding global load, the stages still in flight
// included.  The explicit vmcnt wait before it covers the stage consumed.
__device__ __forceinline__ void gb_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int BM, int BN, int NWV, class Epi>
__global__ __launch_bounds__(64 * NWV) void gemm_big_bf16(const bf16_t* __restrict__ X, int M,
                                                          const bf16_t* __restrict__ W, int N, int K, int k_per_split,
                                                          int tiles_m, int tiles_n, Epi epi) {
    constexpr int FM = BM / 16, FN = BN / 16;   // 16-row fragments of a stage
    constexpr int NF = FM + FN;                 // fragments per stage (one 32-k step)
    constexpr int NL = NF / NWV;                // global_load_lds per wave per stage
    constexpr int WGN = NWV / 2;                // waves along n (two along m)
    constexpr int WFM = FM / 2, WFN = FN / WGN; // fragments per wave
    static_assert(NF % NWV == 0 && (WFM == 8 || WFM == 4) && WFN >= 1, "tile shape");
    typedef __attribute__((address_space(3))) void lds_void;
    __shared__ __attribute__((aligned(1024))) bf16_t s0[NF * 512];
    __shared__ __attribute__((aligned(1024))) bf16_t s1[NF * 512];
    __shared__ __attribute__((aligned(1024))) bf16_t s2[NF * 512];
    __shared__ __attribute__((aligned(1024))) bf16_t s3[NF * 512];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave - wm * WGN;
    // tiles of this workgroup: XCD x (= bid % 8) takes the x-th eighth of the
    // tiles in row-band order (n fastest), and its workgroups take them in
    // turn (workgroup j of the XCD: tiles j, j + wgx, ...), so the ones in
    // flight on an XCD are neighbours in a row band
    const int ntile = tiles_m * tiles_n;
    const int bid = blockIdx.x;
    const int per = (ntile + 7) >> 3;
    const int wgx = gridDim.x >> 3;             // workgroups per XCD
    const int t_end = min(((bid & 7) + 1) * per, ntile);
    int t = (bid & 7) * per + (bid >> 3);
    if (t >= t_end) return;                     // uniform: whole workgroup
    const int mfr_last = ((M + 15) >> 4) - 1, nfr_last = ((N + 15) >> 4) - 1;
    const int split = blockIdx.y;
    const int ks0 = (split * k_per_split) >> 5; // first 32-k step
    const int nst = k_per_split >> 5;
    const int K32 = K >> 5;

    // fragment f of a stage: f < FM is activation rows 16 f.., else weight
    // rows 16 (f - FM)..; wave w issues f = w, w + NWV, ...
    int mfr0 = 0, nfr0 = 0;                     // first 16-row fragment of each operand
    const bf16_t* src[NL];
    auto set_tile = [&](int tt) {
        const int tm = tt / tiles_n, tn = tt - tm * tiles_n;
        mfr0 = tm * FM;
        nfr0 = tn * FN;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int f = wave + NWV * i;
            const bf16_t* base;
            if (f < FM) base = X + (size_t)min(mfr0 + f, mfr_last) * K32 * 512;
            else base = W + (size_t)min(nfr0 + f - FM, nfr_last) * K32 * 512;
            src[i] = base + (size_t)ks0 * 512 + lane * 8;
        }
    };
    set_tile(t);
    auto issue = [&](bf16_t* buf, int st) {
#pragma unroll
        for (int i = 0; i < NL; ++i)
            __builtin_amdgcn_global_load_lds((const void*)(src[i] + (size_t)st * 512),
                                             (lds_void*)(buf + (wave + NWV * i) * 512), 16, 0, 0);
    };

    f32x4_t acc[WFN][WFM];
#pragma unroll
    for (int i = 0; i < WFN; ++i)
#pragma unroll
        for (int j = 0; j < WFM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    // Operand reads are ds_read_b128 in asm: the compiler cannot tell the
    // stage being read from the stages the LDS DMA is still filling and would
    // wait for every load in flight before each read.  The stage read is
    // complete (the vmcnt wait and barrier before it).  Each asm block issues
    // its reads and waits for them itself, so its outputs are valid when it
    // ends whatever the compiler does with the registers afterwards.
    auto compute = [&](const bf16_t* buf) {
        const uint32_t lb = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16_t*)buf + lane * 16;
        const uint32_t la = lb + (FM + wn * WFN) * 1024, lbm = lb + wm * WFM * 1024;
        bf16x8_t a[WFN], b[WFM];
        static_assert((WFN == 8 || WFN == 4 || WFN == 2), "operand counts");
        if constexpr (WFN == 8) {
            asm volatile(
                "ds_read_b128 %0, %8 offset:0\n\tds_read_b128 %1, %8 offset:1024\n\t"
                "ds_read_b128 %2, %8 offset:2048\n\tds_read_b128 %3, %8 offset:3072\n\t"
                "ds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %8 offset:5120\n\t"
                "ds_read_b128 %6, %8 offset:6144\n\tds_read_b128 %7, %8 offset:7168\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(a[4]), "=&v"(a[5]), "=&v"(a[6]),
                  "=&v"(a[7])
                : "v"(la)
                : "memory");
        } else if constexpr (WFN == 4) {
            asm volatile(
                "ds_read_b128 %0, %4 offset:0\n\tds_read_b128 %1, %4 offset:1024\n\t"
                "ds_read_b128 %2, %4 offset:2048\n\tds_read_b128 %3, %4 offset:3072\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3])
                : "v"(la)
                : "memory");
        } else {
            asm volatile(
                "ds_read_b128 %0, %2 offset:0\n\tds_read_b128 %1, %2 offset:1024\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(a[0]), "=&v"(a[1])
                : "v"(la)
                : "memory");
        }
        if constexpr (WFM == 8) {
            asm volatile(
                "ds_read_b128 %0, %8 offset:0\n\tds_read_b128 %1, %8 offset:1024\n\t"
                "ds_read_b128 %2, %8 offset:2048\n\tds_read_b128 %3, %8 offset:3072\n\t"
                "ds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %8 offset:5120\n\t"
                "ds_read_b128 %6, %8 offset:6144\n\tds_read_b128 %7, %8 offset:7168\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3]), "=&v"(b[4]), "=&v"(b[5]), "=&v"(b[6]),
                  "=&v"(b[7])
                : "v"(lbm)
                : "memory");
        } else {
            asm volatile(
                "ds_read_b128 %0, %4 offset:0\n\tds_read_b128 %1, %4 offset:1024\n\t"
                "ds_read_b128 %2, %4 offset:2048\n\tds_read_b128 %3, %4 offset:3072\n\t"
                "s_waitcnt lgkmcnt(0)"
                : "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
                : "v"(lbm)
                : "memory");
        }
#pragma unroll
        for (int i = 0; i < WFN; ++i)
#pragma unroll
            for (int j = 0; j < WFM; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    };

    // prologue: stages 0 .. NS-2 in flight
    if (0 < nst) issue(s0, 0);
    if (1 < nst) issue(s1, 1);
    if (2 < nst) issue(s2, 2);
    const int r = lane & 15, g = lane >> 4;
    for (bool later = false;; later = true) {
        // step st: wait for stage st (the NS-2 later stages may stay in
        // flight; on a later tile the first step waits for everything, the
        // previous tile's output stores included), barrier (stage st visible
        // to all waves, and every wave is done with the buffer stage st +
        // NS - 1 refills), refill, consume
#define GB_STEP(BUF, NEXT, U)                                                          \
        {                                                                              \
            const int st = st0 + (U);                                                  \
            if (st < nst) {                                                            \
                if (later && st == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));        \
                else if (st + 2 < nst) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * NL));  \
                else if (st + 1 < nst) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NL));      \
                else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                         \
                gb_barrier();                                                          \
                if (st + GB_NS - 1 < nst) issue(NEXT, st + GB_NS - 1);                 \
                compute(BUF);                                                          \
            }                                                                          \
        }
        for (int st0 = 0; st0 < nst; st0 += GB_NS) {
            GB_STEP(s0, s3, 0)
            GB_STEP(s1, s0, 1)
            GB_STEP(s2, s1, 2)
            GB_STEP(s3, s2, 3)
        }
#undef GB_STEP
        // the next tile's first stages go out before this tile's outputs are
        // stored, once every wave is done reading the stage buffers
        const int em0 = mfr0, en0 = nfr0;
        const int t_next = t + wgx;
        const bool more = t_next < t_end;      // uniform
        if (more) {
            gb_barrier();
            set_tile(t_next);
            if (0 < nst) issue(s0, 0);
            if (1 < nst) issue(s1, 1);
            if (2 < nst) issue(s2, 2);
        }
        // epilogue: lane (r, g) of tile (i, j) holds outputs n = 4 g .. 4 g + 3
        // of weight fragment i, row m = r of activation fragment j.  The
        // rows' operands load once; each column fragment's operands load
        // while the previous fragment's outputs are stored, so a wave waits
        // about WFN + 1 memory round trips, not one per store.  A wave whose
        // outputs all lie inside the product (and whose rows are all stored)
        // stores without guards.
        int em[WFM], emc[WFM];
        typename Epi::RowKey rk[WFM];
        typename Epi::RowPre rp[WFM];
        bool rows_ok = true;
#pragma unroll
        for (int j = 0; j < WFM; ++j) {
            em[j] = (em0 + wm * WFM + j) * 16 + r;
            emc[j] = min(em[j], M - 1);
            rk[j] = epi.row_key(emc[j]);
        }
#pragma unroll
        for (int j = 0; j < WFM; ++j) rp[j] = epi.row(rk[j]);
#pragma unroll
        for (int j = 0; j < WFM; ++j) rows_ok = rows_ok && epi.ok(rp[j]);
        const bool inside = (em0 + wm * WFM + WFM) * 16 <= M && (en0 + wn * WFN + WFN) * 16 <= N;   // uniform
        const bool fast = inside && __all(rows_ok);
        // column operands (biases) go out one fragment ahead; per-output
        // operands (the residual values) one fragment at a time, after the
        // previous fragment's stores, for want of registers (the 128 of the
        // accumulators are still live)
        typename Epi::ColPre cp[2];
        typename Epi::ElemPre ep[WFM];
        auto col_n = [&](int i) {
            const int n = (en0 + wn * WFN + i) * 16 + 4 * g;
            return n < N ? n : ((N - 1) & ~3);
        };
        auto store_all = [&](auto guarded) {
            constexpr bool GUARD = decltype(guarded)::value;
            cp[0] = epi.col(col_n(0));
#pragma unroll
            for (int j = 0; j < WFM; ++j) ep[j] = epi.elem(emc[j], col_n(0));
#pragma unroll
            for (int i = 0; i < WFN; ++i) {
                if (i + 1 < WFN) cp[(i + 1) & 1] = epi.col(col_n(i + 1));
                const int n = (en0 + wn * WFN + i) * 16 + 4 * g;
#pragma unroll
                for (int j = 0; j < WFM; ++j) {
                    const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
                    if (!GUARD) {
                        epi.template store<true>(rp[j], cp[i & 1], ep[j], em[j], n, v, split, 4);
                    } else if (em[j] < M && n < N) {
                        epi.template store<false>(rp[j], cp[i & 1], ep[j], em[j], n, v, split, min(4, N - n));
                    }
                }
                if (i + 1 < WFN) {
#pragma unroll
                    for (int j = 0; j < WFM; ++j) ep[j] = epi.elem(emc[j], col_n(i + 1));
                }
            }
        };
        if (fast) store_all(std::false_type{});
        else store_all(std::true_type{});
#pragma unroll
        for (int i = 0; i < WFN; ++i)
#pragma unroll
            for (int j = 0; j < WFM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        if (!more) break;
        t = t_next;
    }
}

template <int BM, int BN, int NWV, class Epi>
static hipError_t launch_big(hipStream_t st, const bf16_t* X, int M, const bf16_t* W, int N, int K, int splits,
                             Epi epi) {
    const int kps = K / splits;
    if (kps % 32) return hipErrorInvalidValue;
    const int tm = (M + BM - 1) / BM, tn = (N + BN - 1) / BN;
    const int ntile = tm * tn;
    // the tile numbering deals eighths of the tiles to the XCDs; each XCD
    // gets at most as many workgroups as it holds at once (its CUs times the
    // workgroups per CU the LDS stages allow), and those take its tiles in
    // turn, so a workgroup's next tile streams in while it stores the last
    static int n_cu = 0;
    if (n_cu == 0) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 8)
            v = 256;
        n_cu = v;
    }
    constexpr int lds_kb = GB_NS * (BM / 16 + BN / 16);   // 1 KB per fragment per stage
    const int per_cu = lds_kb <= 80 ? 2 : 1;               // 160 KB of LDS per CU
    const int per_xcd = std::min((ntile + 7) / 8, std::max(1, n_cu / 8) * per_cu);
    dim3 grid(8 * per_xcd, splits);
    hipLaunchKernelGGL((gemm_big_bf16<BM, BN, NWV, Epi>), grid, dim3(64 * NWV), 0, st, X, M, W, N, K, kps, tm, tn, epi);
    return hipGetLastError();
}

// ------------------------------------------------------------------ launchers
// Tile of the large-M kernel for an M x N product (M > 256): 256 x 256 when
// that gives at least 128 tiles (half the CUs), 256 x 128 when that gives
// 192, else 128 x 128 when that gives 96 (64 for a split-K product, whose
// K splits multiply the workgroups), else 256 x 128 when that gives 64;
// otherwise {0, 0}: the product is too small for any and goes to the medium
// kernel (64-row groups, one workgroup per 32 columns).  Measured at M =
// 325 and 1,075: 72-81 tiles of 128 x 128 without K splits lose to the
// medium kernel, 96 and more win against it and against 256 x 128.
struct BigTile { int bm, bn; };
static int tile_count(int M, int N, int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); }
static BigTile big_tile(int M, int N, bool splittable) {
    if (tile_count(M, N, 256, 256) >= 128) return {256, 256};
    if (tile_count(M, N, 256, 128) >= 192) return {256, 128};
    if (tile_count(M, N, 128, 128) >= (splittable ? 64 : 96)) return {128, 128};
    if (tile_count(M, N, 256, 128) >= 64) return {256, 128};
    return {0, 0};
}
template <class Epi>
static hipError_t launch_bf16(hipStream_t st, const bf16_t* X, int ldx, int M, const bf16_t* W, int N, int K,
                              int splits, int xpk, Epi epi) {
    if (splits < 1 || K % (32 * splits)) return hipErrorInvalidValue;
    if (M <= 16) {
        launch_med_x<1>(st, X, ldx, M, W, N, K, splits, xpk, epi);
    } else if (M <= 32) {
        launch_med_x<2>(st, X, ldx, M, W, N, K, splits, xpk, epi);
    } else {
        const BigTile bt = big_tile(M, N, std::is_same<Epi, EpiPartial>::value);
        if (bt.bm == 0) {
            launch_med_x<4>(st, X, ldx, M, W, N, K, splits, xpk, epi);
        } else {
            if (!xpk) return hipErrorInvalidValue;   // large products take fragment-order activations only
            if (bt.bm == 128) return launch_big<128, 128, 4>(st, X, M, W, N, K, splits, epi);
            return bt.bn == 256 ? launch_big<256, 256, 8>(st, X, M, W, N, K, splits, epi)
                                : launch_big<256, 128, 8>(st, X, M, W, N, K, splits, epi);
        }
    }
    return hipGetLastError();
}

// Whether an M x N bf16 product takes the large-M kernel (the prefill and
// NAR trunk), where a residual projection updates the residual stream in its
// epilogue (EPI_RESID) instead of writing split-K partial sums.
int gemm_resid_in_place(int M, int N) {
    return M > 256 && big_tile(M, N, false).bm != 0;
}

// Workgroups of one split-K-able (partial-sum) bf16 launch for M rows and N
// columns before K splitting.
int gemm_tiles(int M, int N) {
    const int groups = ((N + 15) / 16 + GM_NT - 1) / GM_NT;
    if (M <= 32) return groups;
    const BigTile bt = M <= 256 ? BigTile{0, 0} : big_tile(M, N, true);
    if (bt.bm == 0) return groups * ((M + 63) / 64);
    return tile_count(M, N, bt.bm, bt.bn);
}

hipError_t gemm(hipStream_t st, const GemmArgs& a) {
    if (a.dtype != 1) return gemm_f32(st, a);
    const bf16_t* X = (const bf16_t*)a.X;
    const bf16_t* W = (const bf16_t*)a.W;
    switch (a.epi) {
    case EPI_QKV:
        return launch_bf16(st, X, a.ldx, a.M, W, a.N, a.K, 1, a.xpk, EpiQKV<bf16_t>{a.q, a.bias, a.rows, a.kv, a.d});
    case EPI_GELU:
        return launch_bf16(st, X, a.ldx, a.M, W, a.N, a.K, 1, a.xpk,
                           EpiGelu<bf16_t>{(bf16_t*)a.out, a.bias, a.ldo, a.opk});
    case EPI_PARTIAL:
        return launch_bf16(st, X, a.ldx, a.M, W, a.N, a.K, a.splits, a.xpk,
                           EpiPartial{(float*)a.out, a.ldo, a.split_stride});
    case EPI_RESID:
        // large-M bf16 products only, no K split
        if (a.splits != 1 || !gemm_resid_in_place(a.M, a.N) || a.N % 4) return hipErrorInvalidValue;
        return launch_bf16(st, X, a.ldx, a.M, W, a.N, a.K, 1, a.xpk, EpiResid{(float*)a.out, a.bias, a.ldo});
    case EPI_LOGITS:
        return launch_bf16(st, X, a.ldx, a.M, W, a.N, a.K, 1, a.xpk, EpiLogits{(float*)a.out, a.bias, a.ldo, a.N});
    }
    return hipErrorInvalidValue;
}

}  // namespace mtp
