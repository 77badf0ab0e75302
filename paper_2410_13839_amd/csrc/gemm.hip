// GEMM kernels of the decoder trunk and the fused K-head projection.
//
// All products are "NT": C[m][n] = sum_k X[m][k] * W[n][k], with X the
// activations ([M][K], row-major) and W a Linear weight ([N][K], row-major),
// so both operands are K-contiguous.  Outputs go through an epilogue functor
// that receives 4 consecutive n of one row m.
//
//  * gemm_med_bf16: M <= 192 (decode rows of the batched path, the heads),
//    and more rows while its workgroups fit one round of the CUs (pick_tile).
//    A weight stream (M = 128 rows is ~128 flop per weight byte, below the
//    MFMA / HBM ridge), so W fragments go straight from HBM into MFMA
//    registers (no LDS round trip), 16 waves per workgroup split the K range,
//    each wave loading its own activation fragments from L2 (no LDS staging:
//    no two waves read the same k), and one LDS reduction over the waves
//    precedes the epilogue.  The grid is sized so every CU streams.
//  * gemm_pp_bf16, gemm_duo_bf16: the other products (prefill, NAR).  Tiles on
//    MFMA with both operands streamed global -> LDS in fragment order.
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

template <int MT, int NT, int MAXST, class Epi>
__global__ __launch_bounds__(64 * GM_NW) void gemm_med_bf16(const bf16_t* __restrict__ X, int M,
                                                            const bf16_t* __restrict__ W, int N, int K,
                                                            int k_per_split, Epi epi) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
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
    // X in fragment order: one contiguous 1 KB block per row tile and k step, rows padded to 16
    const bf16_t* xp[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int t = min(m0 / 16 + mt, (M - 1) >> 4);
        xp[mt] = X + ((size_t)t * (K >> 5) + (kb >> 5)) * 512 + lane * 8;
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
                for (int mt = 0; mt < MT; ++mt) xv[u][mt] = *reinterpret_cast<const uint4*>(xp[mt] + (size_t)ss * 512);
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
//
// Row tiles MT of a workgroup (med_rows): the fewest (1, 2, 4) that keep the
// launch within one workgroup per CU.  A workgroup of fewer rows pulls fewer
// activations through its CU and reduces less in LDS, and its weights are in
// the XCD's L2 or the memory-side cache from another row group; a second round
// of workgroups costs more than both save.  Weights cold, MT = 1 / 2 / 4 (us):
// 32 x 3072 x 1024 4.1 / 4.9 / 5.3, 32 x 4096 x 1024 4.3 / 4.9 / 5.5, 64 x 3072
// x 1024 - / 4.8 / 6.0, 64 x 4096 x 1024 - / 4.9 / 6.1; past 256 workgroups 32
// x 6144 x 1536 7.2 / 6.6 / 7.5, 128 x 4096 x 1024 - / 6.9 / 6.1.  A split-K
// product counts four splits: 32 x 1024 x 1024 2.8 (MT = 1, 4 splits) against
// 3.0 (MT = 2, 8 splits), 32 x 1536 x 6144 7.6 (MT = 1, 2 splits) against 6.7
// (MT = 2, 4 splits).
constexpr int GM_NT = 2;
static int med_groups(int N) { return ((N + 15) / 16 + GM_NT - 1) / GM_NT; }
static int med_rows(int M, int N, bool splittable) {
    const int most = M <= 16 ? 1 : M <= 32 ? 2 : 4;
    int mt = 1;
    while (mt < most && med_groups(N) * ((M + 16 * mt - 1) / (16 * mt)) * (splittable ? 4 : 1) > 256) mt *= 2;
    return mt;
}

template <int MT, class Epi>
static void launch_med(hipStream_t st, const bf16_t* X, int M, const bf16_t* W, int N, int K, int splits, Epi epi) {
    constexpr int NT = GM_NT;
    static_assert(NT * MT <= 8, "LDS reduction");
    const int kps = K / splits;
    const int per_wave = ((kps >> 5) + GM_NW - 1) / GM_NW;   // k steps per wave
    dim3 grid(((N + 15) / 16 + NT - 1) / NT, (M + 16 * MT - 1) / (16 * MT), splits);
    dim3 block(64 * GM_NW);
    // one round of loads holds at most MAXST x (NT + MT) fragments per wave
    constexpr int CAP = NT * MT >= 8 ? 2 : 4;
    if (per_wave <= 1)
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, 1, Epi>), grid, block, 0, st, X, M, W, N, K, kps, epi);
    else if (per_wave == 2 || CAP == 2)
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, 2, Epi>), grid, block, 0, st, X, M, W, N, K, kps, epi);
    else if (per_wave == 3)
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, 3, Epi>), grid, block, 0, st, X, M, W, N, K, kps, epi);
    else
        hipLaunchKernelGGL((gemm_med_bf16<MT, NT, CAP, Epi>), grid, block, 0, st, X, M, W, N, K, kps, epi);
}

// ---------------------------------------------------------------- large bf16
// Products of more than 192 rows (prefill, NAR): tiles of BM rows x BN columns, 16 x 16 x 32 MFMA.  Both operands are in fragment order
// (activations written so by their producers, weights packed at load), so a
// 16 x 32 fragment is one contiguous 1 KB; it travels global -> LDS by one
// global_load_lds_dwordx4 per wave (lane l's 16 bytes land at byte 16 l, the
// order the MFMA operand read wants: every ds_read_b128 is conflict free) with
// no register staging.  K advances 32 per stage through NS = 4 LDS stages, NS
// - 1 of them in flight while one is consumed.  Workgroups are numbered so
// that the ones sharing an XCD (the dispatcher deals workgroups to the 8 XCDs
// in turn) take neighbouring tiles of one row band, which they share through
// that XCD's L2.
//
// Two kernels: gemm_pp_bf16 (256 columns, eight waves in two groups that take
// turns at LDS and the matrix cores) and gemm_duo_bf16 (64 or 128 columns, four
// waves, two or three workgroups per CU).
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

// Outputs of a wave's WFN x WFM fragments, from activation fragment mf and
// weight fragment nf on.
template <int WFM, int WFN, class Epi>
__device__ __forceinline__ void store_tile(const f32x4_t (&acc)[WFN][WFM], const Epi& epi, int mf, int nf, int M, int N,
                                           int split, int r, int g) {
    // epilogue: lane (r, g) of tile (i, j) holds outputs n = 4 g .. 4 g + 3
    // of weight fragment i, row m = r of activation fragment j.  The
    // rows' operands load once; each column fragment's operands load
    // while the previous fragment's outputs are stored, so a wave does not
    // wait a memory round trip per store.  A wave whose
    // outputs all lie inside the product (and whose rows are all stored)
    // stores without guards.
    int em[WFM], emc[WFM];
    typename Epi::RowKey rk[WFM];
    typename Epi::RowPre rp[WFM];
    bool rows_ok = true;
#pragma unroll
    for (int j = 0; j < WFM; ++j) {
        em[j] = (mf + j) * 16 + r;
        emc[j] = min(em[j], M - 1);
        rk[j] = epi.row_key(emc[j]);
    }
#pragma unroll
    for (int j = 0; j < WFM; ++j) rp[j] = epi.row(rk[j]);
#pragma unroll
    for (int j = 0; j < WFM; ++j) rows_ok = rows_ok && epi.ok(rp[j]);
    const bool inside = (mf + WFM) * 16 <= M && (nf + WFN) * 16 <= N;   // uniform
    const bool fast = inside && __all(rows_ok);
    // column operands (biases) and per-output operands (the residual
    // values) go out one fragment ahead of the stores; the latter in two sets
    // of registers, which the operands of the product have left free (one set,
    // a round trip per fragment: the 10678 x 1024 x 4096 product with the
    // residual took 97 us, with two 87 us)
    typename Epi::ColPre cp[2];
    typename Epi::ElemPre ep[2][WFM];
    auto col_n = [&](int i) {
        const int n = (nf + i) * 16 + 4 * g;
        return n < N ? n : ((N - 1) & ~3);
    };
    auto store_all = [&](auto guarded) {
        constexpr bool GUARD = decltype(guarded)::value;
        cp[0] = epi.col(col_n(0));
#pragma unroll
        for (int j = 0; j < WFM; ++j) ep[0][j] = epi.elem(emc[j], col_n(0));
#pragma unroll
        for (int i = 0; i < WFN; ++i) {
            if (i + 1 < WFN) {
                cp[(i + 1) & 1] = epi.col(col_n(i + 1));
#pragma unroll
                for (int j = 0; j < WFM; ++j) ep[(i + 1) & 1][j] = epi.elem(emc[j], col_n(i + 1));
            }
            const int n = (nf + i) * 16 + 4 * g;
#pragma unroll
            for (int j = 0; j < WFM; ++j) {
                const float v[4] = {acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]};
                if (!GUARD) {
                    epi.template store<true>(rp[j], cp[i & 1], ep[i & 1][j], em[j], n, v, split, 4);
                } else if (em[j] < M && n < N) {
                    epi.template store<false>(rp[j], cp[i & 1], ep[i & 1][j], em[j], n, v, split, min(4, N - n));
                }
            }
        }
    };
    if (fast) store_all(std::false_type{});
    else store_all(std::true_type{});
}

// The operand fragments of one 32-k step of a wave: WFN of the weights at LDS
// byte address pa, WFM of the activations at pb, 1 KB each.  One asm block
// issues the reads and waits for them: the compiler cannot tell the stage
// being read from those the LDS DMA is filling, and would wait for them too.
template <int WFN, int WFM>
__device__ __forceinline__ void pp_read(bf16x8_t (&a)[WFN], bf16x8_t (&b)[WFM], uint32_t pa, uint32_t pb) {
    static_assert((WFN == 4 && WFM >= 4 && WFM <= 8) || (WFN == 2 && (WFM == 2 || WFM == 4)), "fragments per wave");
#define PP_A2 "ds_read_b128 %0, %[pa] offset:0\n\tds_read_b128 %1, %[pa] offset:1024\n\t"
#define PP_A                                                                                       \
    PP_A2                                                                                          \
    "ds_read_b128 %2, %[pa] offset:2048\n\tds_read_b128 %3, %[pa] offset:3072\n\t"                 \
    "ds_read_b128 %4, %[pb] offset:0\n\tds_read_b128 %5, %[pb] offset:1024\n\t"                    \
    "ds_read_b128 %6, %[pb] offset:2048\n\tds_read_b128 %7, %[pb] offset:3072\n\t"
#define PP_B4 "ds_read_b128 %8, %[pb] offset:4096\n\t"
#define PP_B5 "ds_read_b128 %9, %[pb] offset:5120\n\t"
#define PP_B6 "ds_read_b128 %10, %[pb] offset:6144\n\t"
#define PP_B7 "ds_read_b128 %11, %[pb] offset:7168\n\t"
#define PP_W "s_waitcnt lgkmcnt(0)"
#define PP_O                                                                                                     \
    "=&v"(a[0]), "=&v"(a[1]), "=&v"(a[2]), "=&v"(a[3]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3])
#define PP_I [pa] "v"(pa), [pb] "v"(pb)
    if constexpr (WFN == 2 && WFM == 2)
        asm volatile(PP_A2 "ds_read_b128 %2, %[pb] offset:0\n\tds_read_b128 %3, %[pb] offset:1024\n\t" PP_W
                     : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0]), "=&v"(b[1]) : PP_I : "memory");
    else if constexpr (WFN == 2)
        asm volatile(PP_A2 "ds_read_b128 %2, %[pb] offset:0\n\tds_read_b128 %3, %[pb] offset:1024\n\t"
                     "ds_read_b128 %4, %[pb] offset:2048\n\tds_read_b128 %5, %[pb] offset:3072\n\t" PP_W
                     : "=&v"(a[0]), "=&v"(a[1]), "=&v"(b[0]), "=&v"(b[1]), "=&v"(b[2]), "=&v"(b[3]) : PP_I : "memory");
    else if constexpr (WFM == 4) asm volatile(PP_A PP_W : PP_O : PP_I : "memory");
    else if constexpr (WFM == 5) asm volatile(PP_A PP_B4 PP_W : PP_O, "=&v"(b[4]) : PP_I : "memory");
    else if constexpr (WFM == 6) asm volatile(PP_A PP_B4 PP_B5 PP_W : PP_O, "=&v"(b[4]), "=&v"(b[5]) : PP_I : "memory");
    else if constexpr (WFM == 7)
        asm volatile(PP_A PP_B4 PP_B5 PP_B6 PP_W : PP_O, "=&v"(b[4]), "=&v"(b[5]), "=&v"(b[6]) : PP_I : "memory");
    else
        asm volatile(PP_A PP_B4 PP_B5 PP_B6 PP_B7 PP_W
                     : PP_O, "=&v"(b[4]), "=&v"(b[5]), "=&v"(b[6]), "=&v"(b[7]) : PP_I : "memory");
#undef PP_A2
#undef PP_A
#undef PP_B4
#undef PP_B5
#undef PP_B6
#undef PP_B7
#undef PP_W
#undef PP_O
#undef PP_I
}

// Waits until at most `left` stages of NL loads each are in flight (left <= MOST).
template <int MOST, int NL>
__device__ __forceinline__ void wait_stages(int left) {
    static_assert(MOST * NL < 64, "vmcnt");
    if constexpr (MOST == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    else if (left >= MOST) __builtin_amdgcn_s_waitcnt(vmcnt_imm(MOST * NL));
    else wait_stages<MOST - 1, NL>(left);
}

// Tiles of 32 WFM rows x 32 WFN columns, four waves in a 2 x 2 grid, WGS
// workgroups per CU (NS stages of KS 32-k steps each, at most 160 / WGS KB):
// nothing keeps the workgroups of a CU in step, so one multiplies while another
// reads its operands, starts or stores a tile.  That makes it the kernel for
// products whose epilogue moves more than their operands (the residual read
// and written, few tiles per CU; 128 columns): 10678 x 1024 x 4096 with the
// residual 85.9 us (192 rows) against 87.4 with gemm_pp_bf16, 6720 x 1024 x
// 4096 63.9 (128 rows) against 68.7; and for products of few tiles.
//
// With few tiles what bounds it is a workgroup's serial chain per stage
// (barrier, operand reads, multiplies: ~700 clocks per 32-k step of a lone
// 128 x 128 tile, 400 of a 64 x 64 one, whatever the number of stages in
// flight: 8 stages measured as 4 do), so such products take smaller tiles,
// three workgroups per CU, and 64 x 64 tiles 64 k per stage, half the
// barriers.  Weights cold, 128 x 128 / 128 x 64 / 64 x 64 (us): 325 x 3072 x
// 1024 14.7 / 11.5 / 8.7, 325 x 4096 x 1024 16.2 / 12.4 / 10.5, 1075 x 3072 x
// 1024 16.2 / 15.0 / 16.7, 1075 x 4096 x 1024 21.2 / 18.4 / 21.2.
//
// mfast: tiles are numbered rows first, so an XCD's tiles are neighbours in a
// column band: each weight is then read by one XCD and the activations by all,
// the smaller traffic when there are fewer rows than columns (1075 x 4096 x
// 1024, 128 x 64: 18.4 against 20.7 us).
template <int WFM, int WFN, int KS, int NS, int WGS, class Epi>
__global__ __launch_bounds__(256, WGS) void gemm_duo_bf16(const bf16_t* __restrict__ X, int M, const bf16_t* __restrict__ W,
                                                    int N, int K, int k_per_split, int tiles_m, int tiles_n, int mfast,
                                                    Epi epi) {
    constexpr int NWV = 4;
    constexpr int FM = 2 * WFM, FN = 2 * WFN;   // 16-row fragments of a 32-k step
    constexpr int NF = (FM + FN) * KS;          // of a stage: row fragments, KS steps each, then columns'
    constexpr int NL = (NF + NWV - 1) / NWV;    // global_load_lds per wave per stage (the last ones may repeat)
    static_assert(NS * NF * WGS <= 160, "LDS");
    __shared__ __attribute__((aligned(1024))) bf16_t stage[NS * NF * 512];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // tiles of this workgroup: XCD x (= bid % 8) takes the x-th eighth of the
    // tiles in row-band order (n fastest; or in column-band order), and its
    // workgroups take them in turn (workgroup j of the XCD: tiles j, j + wgx,
    // ...), so the ones in flight on an XCD are neighbours in a band
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
    const int nst = k_per_split / (32 * KS);
    const int K32 = K >> 5;
    const uint32_t base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16_t*)stage + lane * 16;
    const int r = lane & 15, g = lane >> 4;
    int mfr0 = 0, nfr0 = 0;
    const bf16_t* src[NL];
    int dst[NL];
    auto set_tile = [&](int tt) {
        const int td = mfast ? tiles_m : tiles_n;
        const int th = tt / td, tl = tt - th * td;
        const int tm = mfast ? tl : th, tn = mfast ? th : tl;
        mfr0 = tm * FM;
        nfr0 = tn * FN;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int fk = min(wave + NWV * i, NF - 1);
            const int f = fk / KS;
            const bf16_t* b;
            if (f < FM) b = X + (size_t)min(mfr0 + f, mfr_last) * K32 * 512;
            else b = W + (size_t)min(nfr0 + f - FM, nfr_last) * K32 * 512;
            src[i] = b + (size_t)(ks0 + fk % KS) * 512 + lane * 8;
            dst[i] = fk * 512;
        }
    };
    typedef __attribute__((address_space(3))) void lds_void;
    auto issue = [&](int st, int bi) {
        bf16_t* buf = stage + bi * (NF * 512);
#pragma unroll
        for (int i = 0; i < NL; ++i)
            __builtin_amdgcn_global_load_lds((const void*)(src[i] + (size_t)st * (512 * KS)), (lds_void*)(buf + dst[i]), 16, 0, 0);
    };
    auto issue_first = [&]() {
#pragma unroll
        for (int s = 0; s < NS - 1; ++s)
            if (s < nst) issue(s, s);
    };
    set_tile(t);
    issue_first();
    bool later = false;
    while (true) {
        f32x4_t acc[WFN][WFM];
#pragma unroll
        for (int i = 0; i < WFN; ++i)
#pragma unroll
            for (int j = 0; j < WFM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        int bi = 0;
        for (int st = 0; st < nst; ++st) {
            // wait for stage st (the later ones may stay in flight; on a later
            // tile the first step waits for everything, the previous tile's
            // output stores included), barrier (stage st visible to all waves,
            // and every wave is done with the buffer that the next issue
            // refills), refill, consume
            if (later && st == 0) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            else wait_stages<NS - 2, NL>(nst - 1 - st);
            gb_barrier();
            const int bn = bi == 0 ? NS - 1 : bi - 1;
            if (st + NS - 1 < nst) issue(st + NS - 1, bn);
            const uint32_t lb = base + bi * (NF * 1024);
            bf16x8_t a[WFN * KS], b[WFM * KS];
            pp_read<WFN * KS, WFM * KS>(a, b, lb + (FM + wn * WFN) * (KS * 1024), lb + wm * WFM * (KS * 1024));
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int u = 0; u < KS; ++u)
#pragma unroll
                for (int i = 0; i < WFN; ++i)
#pragma unroll
                    for (int j = 0; j < WFM; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i * KS + u], b[j * KS + u], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
            bi = bi + 1 == NS ? 0 : bi + 1;
        }
        // the next tile's first stages go out before this tile's outputs are
        // stored, once every wave is done reading the stage buffers
        gb_barrier();
        const int em0 = mfr0 + wm * WFM, en0 = nfr0 + wn * WFN;
        t += wgx;
        const bool more = t < t_end;            // uniform
        if (more) {
            set_tile(t);
            issue_first();
        }
        store_tile<WFM, WFN>(acc, epi, em0, en0, M, N, split, r, g);
        if (!more) break;
        later = true;
    }
}

// At least 192 tiles of 128 x 256 (wide_tiles): eight waves, tiles of BM = 32
// WFM rows x 256 columns (WFM = 4 .. 8, so that a product's tiles fill whole
// rounds of the CUs; see pick_tile).
//
// What bounds a tile of this size is LDS bandwidth against the matrix cores:
// a 32-k step of 256 x 256 reads 96 KB of operands from LDS and lets 32 KB of
// DMA in (1024 clocks at 128 bytes a clock) while its MFMAs take 1024 clocks
// a SIMD, so the two have to run beside each other all the time.  With all
// waves in step (read, then multiply, a barrier per stage) they take turns,
// and the matrix cores were busy 56% of the time.  Here the two row groups of
// four waves (one wave of each on every SIMD) run one barrier apart: while
// one group reads its operands and asks for a later stage, the other
// multiplies, with the higher wave priority.  Measured, fp32 output, against
// the same tile in step: 10678 x 3072 x 1024 78.6 -> 69.7 us (964 TFLOP/s),
// 10678 x 1024 x 4096 106.8 -> 78.9 us, 73.9 us with 192-row tiles (1.21
// PFLOP/s).  Weights straight from global memory into registers instead of
// LDS, a column-major tile order and a start in K of its own for each
// workgroup all measured the same within 2%, or slower.
//
// A stage is landed for everyone once every wave has waited for its own DMA
// of it and a barrier has passed: each wave waits at the end of the phase in
// which it reads the stage before, one barrier ahead of the first reader.  A
// buffer is refilled (stage st + 3 into that of st - 1) by a group that is
// reading stage st; the other group is then multiplying st - 1 or later and
// has read it.
template <int WFM, class Epi>
__global__ __launch_bounds__(512) void gemm_pp_bf16(const bf16_t* __restrict__ X, int M, const bf16_t* __restrict__ W,
                                                    int N, int K, int k_per_split, int tiles_m, int tiles_n, Epi epi) {
    constexpr int NWV = 8, WFN = 4;
    constexpr int FM = 2 * WFM, FN = 4 * WFN;   // 16-row fragments of a stage (one 32-k step)
    constexpr int NF = FM + FN;
    constexpr int NL = (NF + NWV - 1) / NWV;    // global_load_lds per wave per stage (the last ones may repeat)
    __shared__ __attribute__((aligned(1024))) bf16_t stage[GB_NS * NF * 512];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;    // wm: the group
    // tiles of this workgroup, as in gemm_duo_bf16
    const int ntile = tiles_m * tiles_n;
    const int bid = blockIdx.x;
    const int per = (ntile + 7) >> 3;
    const int wgx = gridDim.x >> 3;
    const int t_end = min(((bid & 7) + 1) * per, ntile);
    int t = (bid & 7) * per + (bid >> 3);
    if (t >= t_end) return;                     // uniform: whole workgroup
    const int mfr_last = ((M + 15) >> 4) - 1, nfr_last = ((N + 15) >> 4) - 1;
    const int split = blockIdx.y;
    const int ks0 = (split * k_per_split) >> 5;
    const int nst = k_per_split >> 5;
    const int K32 = K >> 5;
    const uint32_t base = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) bf16_t*)stage + lane * 16;
    const int r = lane & 15, g = lane >> 4;

    int mfr0 = 0, nfr0 = 0;
    const bf16_t* src[NL];
    int dst[NL];
    auto set_tile = [&](int tt) {
        const int tm = tt / tiles_n, tn = tt - tm * tiles_n;
        mfr0 = tm * FM;
        nfr0 = tn * FN;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int f = min(wave + NWV * i, NF - 1);
            const bf16_t* b;
            if (f < FM) b = X + (size_t)min(mfr0 + f, mfr_last) * K32 * 512;
            else b = W + (size_t)min(nfr0 + f - FM, nfr_last) * K32 * 512;
            src[i] = b + (size_t)ks0 * 512 + lane * 8;
            dst[i] = f * 512;
        }
    };
    typedef __attribute__((address_space(3))) void lds_void;
    auto issue = [&](int st) {
        bf16_t* buf = stage + (st % GB_NS) * (NF * 512);
#pragma unroll
        for (int i = 0; i < NL; ++i)
            __builtin_amdgcn_global_load_lds((const void*)(src[i] + (size_t)st * 512), (lds_void*)(buf + dst[i]), 16, 0, 0);
    };
    // the wait for this wave's part of the first stage: with the two later
    // stages in flight, or for everything
    auto issue_first = [&]() {
#pragma unroll
        for (int s = 0; s < GB_NS - 1; ++s)
            if (s < nst) issue(s);
    };
    set_tile(t);
    issue_first();
    bool later = false;
    while (true) {
        f32x4_t acc[WFN][WFM];
#pragma unroll
        for (int i = 0; i < WFN; ++i)
#pragma unroll
            for (int j = 0; j < WFM; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        // (on a later tile the previous one's output stores are in the count)
        if (!later && nst >= GB_NS - 1) __builtin_amdgcn_s_waitcnt(vmcnt_imm((GB_NS - 2) * NL));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        gb_barrier();
        if (wm == 1) gb_barrier();              // the second group runs one barrier behind
        for (int st = 0; st < nst; ++st) {
            // reading phase
            const uint32_t lb = base + (st % GB_NS) * (NF * 1024);
            bf16x8_t a[WFN], b[WFM];
            if (st + GB_NS - 1 < nst) issue(st + GB_NS - 1);
            pp_read<WFN, WFM>(a, b, lb + (FM + wn * WFN) * 1024, lb + wm * WFM * 1024);
            if (st + 3 < nst) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * NL));
            else if (st + 2 < nst) __builtin_amdgcn_s_waitcnt(vmcnt_imm(NL));
            else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
            gb_barrier();
            // multiplying phase
            __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int i = 0; i < WFN; ++i)
#pragma unroll
                for (int j = 0; j < WFM; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            gb_barrier();
        }
        if (wm == 0) gb_barrier();              // every wave is past its last read here
        // the next tile's first stages go out before this tile's outputs are stored
        const int em0 = mfr0 + wm * WFM, en0 = nfr0 + wn * WFN;
        t += wgx;
        const bool more = t < t_end;            // uniform
        if (more) {
            set_tile(t);
            issue_first();
        }
        store_tile<WFM, WFN>(acc, epi, em0, en0, M, N, split, r, g);
        if (!more) break;
        later = true;
    }
}

// Compute units of the current device (256 where that cannot be asked).
static int cu_count() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v < 8)
            v = 256;
        return v;
    }();
    return n;
}

// The tile numbering deals eighths of the tiles to the XCDs; each XCD gets at
// most as many workgroups as it holds at once (its CUs times the workgroups
// per CU that the LDS stages allow), and those take its tiles in turn, so a
// workgroup's next tile streams in while it stores the last.
template <int WFM, int WFN, int KS, int NS, int WGS, class Epi>
static hipError_t launch_duo(hipStream_t st, const bf16_t* X, int M, const bf16_t* W, int N, int K, int splits,
                             bool mfast, Epi epi) {
    const int kps = K / splits;
    if (kps % (32 * KS)) return hipErrorInvalidValue;
    const int tm = (M + 32 * WFM - 1) / (32 * WFM), tn = (N + 32 * WFN - 1) / (32 * WFN);
    const int per_xcd = std::min((tm * tn + 7) / 8, cu_count() / 8 * WGS);
    hipLaunchKernelGGL((gemm_duo_bf16<WFM, WFN, KS, NS, WGS, Epi>), dim3(8 * per_xcd, splits), dim3(256), 0, st, X, M, W, N, K,
                       kps, tm, tn, mfast ? 1 : 0, epi);
    return hipGetLastError();
}
template <int WFM, class Epi>
static hipError_t launch_pp(hipStream_t st, const bf16_t* X, int M, const bf16_t* W, int N, int K, int splits,
                            Epi epi) {
    const int kps = K / splits;
    if (kps % 32) return hipErrorInvalidValue;
    const int tm = (M + 32 * WFM - 1) / (32 * WFM), tn = (N + 255) / 256;
    const int per_xcd = std::min((tm * tn + 7) / 8, cu_count() / 8);
    hipLaunchKernelGGL((gemm_pp_bf16<WFM, Epi>), dim3(8 * per_xcd, splits), dim3(512), 0, st, X, M, W, N, K, kps, tm, tn,
                       epi);
    return hipGetLastError();
}

// ------------------------------------------------------------------ launchers
// Tile of an M x N product; rows 0: the medium kernel.
//
// The eight-wave kernel (256 columns) needs one CU a tile and costs about as
// much for a tile of 128 rows on a few CUs as on all: with fewer than 192
// tiles of 128 x 256 (three quarters of the CUs) the four-wave kernel's tiles
// are faster (weights cold: 1075 x 4096 x 1024, 144 against 576 tiles, 22.9
// against 18.2 us; from 6720 rows and 1024 columns on, 212 tiles, the larger
// ones win).  The row count is the one with the least rounds x rows: the
// workgroups take tiles in rounds, and a last round costs as much as a full
// one (6720 x 3072 x 1024, 27 x 12 tiles of 256 rows, 1.27 rounds: 59.9 us; 42
// x 12 of 160, 1.97 rounds: 50.9 us; 10678 x 1024 x 4096, one round either
// way: 256 rows 78.9, 192 rows 73.9 us).  32 rows are added for what a round
// costs whatever its tiles.
//
// Below that, 64 x 64 while all its workgroups are resident at once (three per
// CU), else 128 x 64 (fewer than 768 tiles here): a second round costs more
// than the smaller tile saves (1075 x 4096 x 1024, 1088 tiles of 64 x 64, 21.2
// us, 128 x 64 18.4; 700 x 4096 x 1024, 704 tiles of 64 x 64, 14.5 us, 128 x 64
// 15.3; 128 x 128, one to two workgroups per CU, 21.2 and 17.5).  A split-K
// product of a long K with more than 256 tiles of 64 x 64 takes 128 x 64 and two
// splits (1075 x 1024 x 4096: 21.8 us; 64 x 64 22.4 unsplit or split; at K =
// 1024 8.2 against 9.4 with 64 x 64 unsplit), from K = 8192 on with more than
// 192 (512 x 2048 x 8192, 256 tiles: 26.1 us in four splits, 64 x 64 29.1).
//
// The medium kernel for up to 192 rows (128 x 3072 x 1024: 6.0 us, 64 x 64
// 9.0), and past them where its workgroups fit one round of the CUs (256 x 2048
// x 512: 4.2 us, 64 x 64 6.2; 320 x 1536 x 512 4.7 against 6.2, 512 x 1024 x 256
// 3.8 against 5.0; with more, 320 x 2048 x 512 6.5 against 6.1) and, with as
// many K splits as the round has room for, the K of each is at most 3072 (with
// the residual pass that follows: 325 x 1024 x 1024 unsplit 8.7 us, 64 x 64 in
// two splits 9.6; 256 x 1024 x 4096 in two 10.8 against 11.4; 512 x 768 x 3072
// unsplit 12.7 against 12.8; 320 x 1024 x 4096 unsplit 14.5 against 13.6).
struct BigTile { int rows; int cols; };
static int tile_count(int M, int N, int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); }
// The row count with the least rounds x (rows + 32) over `slots` workgroups.
static int best_rows(int M, int N, int bn, int slots, int most) {
    int best = 0, best_cost = 0;
    for (int bm = most; bm >= 128; bm -= 32) {
        const int cost = (tile_count(M, N, bm, bn) + slots - 1) / slots * (bm + 32);
        if (best == 0 || cost < best_cost) {
            best = bm;
            best_cost = cost;
        }
    }
    return best;
}
static bool wide_tiles(int M, int N) { return M > 192 && tile_count(M, N, 128, 256) >= 192; }
static BigTile pick_tile(int M, int N, int K, bool splittable) {
    if (M <= 192) return {0, 0};
    if (wide_tiles(M, N)) return {best_rows(M, N, 256, cu_count(), 256), 256};
    const int wgs = med_groups(N) * ((M + 63) / 64);
    int s = 1;
    while (splittable && wgs * 2 * s <= 256) s *= 2;
    if (wgs <= 256 && K / s <= 3072) return {0, 0};
    const int t64 = tile_count(M, N, 64, 64), slots = 3 * cu_count();
    const int split_slots = K < 2048 ? slots : K < 8192 ? cu_count() : cu_count() * 3 / 4;
    // (64 k per stage; split-K products have K splits of whole stages, see gemm_splits)
    if (t64 <= (splittable ? split_slots : slots)) return {64, 64};
    return {128, 64};
}
template <class Epi>
static hipError_t launch_bf16(hipStream_t st, const GemmArgs& a, int splits, Epi epi) {
    constexpr bool split = std::is_same<Epi, EpiPartial>::value;
    const bf16_t* X = (const bf16_t*)a.X;
    const bf16_t* W = (const bf16_t*)a.W;
    const int M = a.M, N = a.N, K = a.K;
    // activations in fragment order; K is a model width, a multiple of 256
    if (!a.xpk || K % 64 || splits < 1 || K % (32 * splits)) return hipErrorInvalidValue;
    if constexpr (std::is_same<Epi, EpiResid>::value) {
        // (the residual epilogue's operands leave no registers for 256 rows)
        if (!gemm_resid_in_place(M, N)) return hipErrorInvalidValue;
        switch (wide_tiles(M, N) ? best_rows(M, N, 128, 2 * cu_count(), 224) : 128) {
        case 128: return launch_duo<4, 4, 1, 4, 2>(st, X, M, W, N, K, splits, false, epi);
        case 160: return launch_duo<5, 4, 1, 4, 2>(st, X, M, W, N, K, splits, false, epi);
        case 192: return launch_duo<6, 4, 1, 4, 2>(st, X, M, W, N, K, splits, false, epi);
        default: return launch_duo<7, 4, 1, 3, 2>(st, X, M, W, N, K, splits, false, epi);
        }
    } else {
        const BigTile bt = pick_tile(M, N, K, split);
        const bool mfast = M <= N;
        if (bt.rows == 0) {
            switch (med_rows(M, N, split)) {
            case 1: launch_med<1>(st, X, M, W, N, K, splits, epi); break;
            case 2: launch_med<2>(st, X, M, W, N, K, splits, epi); break;
            default: launch_med<4>(st, X, M, W, N, K, splits, epi); break;
            }
            return hipGetLastError();
        }
        if (bt.cols == 64) {
            if (bt.rows == 64) return launch_duo<2, 2, 2, 3, 3>(st, X, M, W, N, K, splits, mfast, epi);
            return launch_duo<4, 2, 1, 4, 3>(st, X, M, W, N, K, splits, mfast, epi);
        }
        switch (bt.rows) {
        case 128: return launch_pp<4>(st, X, M, W, N, K, splits, epi);
        case 160: return launch_pp<5>(st, X, M, W, N, K, splits, epi);
        case 192: return launch_pp<6>(st, X, M, W, N, K, splits, epi);
        case 224: return launch_pp<7>(st, X, M, W, N, K, splits, epi);
        default: return launch_pp<8>(st, X, M, W, N, K, splits, epi);
        }
    }
}

// Whether an M x N bf16 product takes the large-M tiles (the prefill and
// NAR trunk), where a residual projection updates the residual stream in its
// epilogue (EPI_RESID) instead of writing split-K partial sums.
// From wide tiles on, and where 64 x 64 tiles no longer fit one round (then with
// 128 x 128): 84 layers of 4300 rows, d 1024, 20.1 ms against 21.5 with partial sums, 5375
// rows 23.0 against 24.6, 3225 rows 16.6 either way; below, partial sums (2600
// rows: 78 us of products and residual passes a layer against 84).
int gemm_resid_in_place(int M, int N) {
    return M > 256 && (wide_tiles(M, N) || tile_count(M, N, 64, 64) > 3 * cu_count());
}

// K splits (a power of two, at most `most`) of a partial-sum product.
//
// The medium kernel: up to one workgroup per CU, each split at least 256 k
// (325 x 1024 x 1024, 192 workgroups: 4.7 us unsplit, 6.5 in two; 32 x 1024 x
// 1024 2.8 in four, 3.0 in eight; 32 x 1536 x 6144, 48 workgroups: 6.7 in four,
// 6.9 in eight).  Tiles: up to two workgroups per CU, each split at least 512 k
// (325 x 1024 x 4096, 96 tiles: 10.4 us in four, 10.8 in eight; 576 x 1024 x
// 1024, 144 tiles: 6.6 in two, 7.2 in four).  The residual pass that follows
// reads every split.
int gemm_splits(int M, int N, int K, int most) {
    const BigTile bt = pick_tile(M, N, K, true);
    const int mt = med_rows(M, N, true);
    const int wgs = bt.rows == 0 ? med_groups(N) * ((M + 16 * mt - 1) / (16 * mt)) : tile_count(M, N, bt.rows, bt.cols);
    const int limit = bt.rows == 0 ? 256 : 2 * cu_count() + cu_count() / 4, least = bt.rows == 0 ? 256 : 512;
    const int unit = bt.rows == 64 ? 64 : 32;    // whole stages
    int s = 1;
    while (2 * s <= most && wgs * 2 * s <= limit && K % (unit * 2 * s) == 0 && K / (2 * s) >= least) s *= 2;
    return s;
}

hipError_t gemm(hipStream_t st, const GemmArgs& a) {
    if (a.dtype != 1) return gemm_f32(st, a);
    switch (a.epi) {
    case EPI_QKV: return launch_bf16(st, a, 1, EpiQKV<bf16_t>{a.q, a.bias, a.rows, a.kv, a.d});
    case EPI_GELU: return launch_bf16(st, a, 1, EpiGelu<bf16_t>{(bf16_t*)a.out, a.bias, a.ldo, a.opk});
    case EPI_PARTIAL: return launch_bf16(st, a, a.splits, EpiPartial{(float*)a.out, a.ldo, a.split_stride});
    case EPI_RESID:
        // large-M bf16 products only, no K split
        if (a.splits != 1 || !gemm_resid_in_place(a.M, a.N) || a.N % 4) return hipErrorInvalidValue;
        return launch_bf16(st, a, 1, EpiResid{(float*)a.out, a.bias, a.ldo});
    case EPI_LOGITS: return launch_bf16(st, a, 1, EpiLogits{(float*)a.out, a.bias, a.ldo, a.N});
    }
    return hipErrorInvalidValue;
}

}  // namespace mtp
