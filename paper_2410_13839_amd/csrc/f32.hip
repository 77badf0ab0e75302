// Products of the fp32 model (weights, activations and KV cache in fp32) on
// the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: full float32 multiply
// and accumulate, no reduced-precision inputs).
//
// Same "NT" product as gemm.hip: C[m][n] = sum_k X[m][k] W[n][k], both
// operands row-major and K-contiguous.
//
// What bounds it: the fp32 model is small (d 256: 0.8-1 MB of weights per
// product), so a decode step is a chain of launches each a memory round trip
// long.  One workgroup therefore owns 16 columns and 16 * MT rows with the
// whole K, split over its 16 waves: every wave asks for all its weight and
// activation chunks at once (float4 per lane, no LDS staging: no two waves
// share a k), and one LDS reduction over the waves ends the product.
// The former kernel (16 x 64 tiles staged through LDS 32 k at a time, one
// round trip per 32 k) took 20 us a launch at K = 256 and 80 us at K = 1024
// (2 rows, d 256); this one 4.6-5.4 and 5.7 us, of which 1.8 us are the launch.
//
// A lane's float4 is four consecutive k of one row (lane r + 16 g: row r, k =
// 4 g .. 4 g + 3); the four instructions of a chunk take one component each,
// so an instruction's four k are 4 apart, alike in both operands.
//
// Input modes (XM): 0 the rows as they are; 1 LayerNorm of the residual rows
// (at most 16 of them: wave w takes row w's statistics while the product's
// operands are in flight); 2 the final LayerNorm of each sequence's last
// pending row (the heads), or of its kept row hz when it ran none.  With the
// LayerNorm in the consumer and the residual added in the producer (EpiResid,
// every output belongs to one workgroup) a layer is five launches instead of
// seven plus the key-split merge: the decode step of the 2-layer d 256 model
// went from 335 to 61 us.
#include <algorithm>

#include "common.h"
#include "epilogue.h"
#include "launch.h"
#include "wave.h"

namespace mtp {

namespace {
constexpr int GF_NW = 16;      // waves, splitting K
constexpr int GF_MAXQ = 8;     // float4 chunks of a row per lane in the LayerNorm modes (d <= 2048)

struct F32Args {
    const float* X; int ldx; int M;
    const float* W; int N; int K;
    int k_per_split;
    // LayerNorm modes (K = d = ldx)
    const float* g; const float* beta;
    const SeqState* st; int Q;     // XM 2
    float* hz;                     // XM 2: [M][K]
};

// XM 2: where sequence b's row comes from
__device__ __forceinline__ const float* final_row(const F32Args& a, int b, bool* pending) {
    const int pl = a.Q > 0 ? a.st[b].pend_len : 0;
    *pending = pl > 0;
    return pl > 0 ? a.X + (size_t)(b * a.Q + pl - 1) * a.ldx : a.hz + (size_t)b * a.K;
}
}  // namespace

template <int MT, int MAXST, int XM, class Epi>
__global__ __launch_bounds__(64 * GF_NW) void gemm_f32_kernel(F32Args a, Epi epi) {
    static_assert(XM == 0 || MT == 1, "LayerNorm rows: one per wave");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16 * MT;
    const int split = blockIdx.z, kb = split * a.k_per_split;
    const int nsteps = a.k_per_split >> 4;             // 16 k each
    __shared__ float s_stat[2][16];
    __shared__ f32x4_t red[GF_NW][MT][64];

    // wave mt < MT stores row tile mt, 4 columns of one row per lane; its
    // epilogue operands (for the cache: the row's position, then its page) are
    // asked for first, so that they cost no round trip after the product
    const int mt = min(wave, MT - 1);
    const int m = m0 + 16 * mt + r, n = n0 + 4 * g;
    const int mc = min(m, a.M - 1), nc = n < a.N ? n : ((a.N - 1) & ~3);
    const typename Epi::RowKey rk = epi.row_key(mc);
    const typename Epi::ColPre cp = epi.col(nc);
    const typename Epi::ElemPre ep = epi.elem(mc, nc);
    typename Epi::RowPre rp{};

    const float* wp = a.W + (size_t)min(n0 + r, a.N - 1) * a.K + kb + 4 * g;
    const float* xp[MT];
#pragma unroll
    for (int j = 0; j < MT; ++j) {
        const int mj = min(m0 + 16 * j + r, a.M - 1);
        if constexpr (XM == 2) {
            bool unused;
            xp[j] = final_row(a, mj, &unused) + 4 * g;
        } else {
            xp[j] = a.X + (size_t)mj * a.ldx + kb + 4 * g;
        }
    }
    f32x4_t acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float mean = 0.f, rstd = 0.f;
    // LayerNorm modes: wave w's row for the statistics (K is a multiple of 256)
    const int row = min(wave, a.M - 1);
    bool pending = false;
    f32x4_t x[GF_MAXQ];
    if constexpr (XM != 0) {
        const float* hp = XM == 2 ? final_row(a, row, &pending) : a.X + (size_t)row * a.ldx;
#pragma unroll
        for (int j = 0; j < GF_MAXQ; ++j) {
            x[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if (256 * j < a.K) x[j] = *reinterpret_cast<const f32x4_t*>(hp + 4 * (lane + 64 * j));
        }
    }

    for (int s0 = wave; s0 < nsteps; s0 += GF_NW * MAXST) {   // (LayerNorm modes: K >= 256, every wave has a step)
        f32x4_t wv[MAXST], xv[MAXST][MT], gv[MAXST], bv[MAXST];
#pragma unroll
        for (int u = 0; u < MAXST; ++u) {
            const int ss = min(s0 + GF_NW * u, nsteps - 1);     // clamped: no branch around the loads
            wv[u] = *reinterpret_cast<const f32x4_t*>(wp + 16 * ss);
#pragma unroll
            for (int j = 0; j < MT; ++j) xv[u][j] = *reinterpret_cast<const f32x4_t*>(xp[j] + 16 * ss);
            if constexpr (XM != 0) {
                gv[u] = *reinterpret_cast<const f32x4_t*>(a.g + 16 * ss + 4 * g);
                bv[u] = *reinterpret_cast<const f32x4_t*>(a.beta + 16 * ss + 4 * g);
            }
        }
        if (s0 == wave) rp = epi.row(rk);
        if constexpr (XM != 0) {
            if (s0 == wave) {                            // first round (uniform over the workgroup)
                float s = 0.f;
#pragma unroll
                for (int j = 0; j < GF_MAXQ; ++j) s += (x[j][0] + x[j][1]) + (x[j][2] + x[j][3]);
                const float mu = wave_sum64(s) / (float)a.K;
                float v = 0.f;
#pragma unroll
                for (int j = 0; j < GF_MAXQ; ++j)
                    if (256 * j < a.K) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) { const float t = x[j][i] - mu; v = fmaf(t, t, v); }
                    }
                const float rs = rsqrtf(wave_sum64(v) / (float)a.K + 1e-5f);
                if (lane == 0) {
                    s_stat[0][wave] = mu;
                    s_stat[1][wave] = rs;
                }
                if constexpr (XM == 2) {
                    // the row stays the sequence's last one (no workgroup reads
                    // hz of a sequence that has a pending row)
                    if (blockIdx.x == 0 && pending && wave < a.M) {
#pragma unroll
                        for (int j = 0; j < GF_MAXQ; ++j)
                            if (256 * j < a.K)
                                *reinterpret_cast<f32x4_t*>(a.hz + (size_t)row * a.K + 4 * (lane + 64 * j)) = x[j];
                    }
                }
                __syncthreads();
                mean = s_stat[0][r];
                rstd = s_stat[1][r];
            }
        }
#pragma unroll
        for (int u = 0; u < MAXST; ++u) {
            if (s0 + GF_NW * u < nsteps) {               // uniform
#pragma unroll
                for (int j = 0; j < MT; ++j) {
                    f32x4_t y = xv[u][j];
                    if constexpr (XM != 0) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) y[i] = (y[i] - mean) * rstd * gv[u][i] + bv[u][i];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[u][i], y[i], acc[j], 0, 0, 0);
                }
            }
        }
    }

#pragma unroll
    for (int i = 0; i < MT; ++i) red[wave][i][lane] = acc[i];
    __syncthreads();
    if (wave < MT) {
        f32x4_t s = red[0][mt][lane];
#pragma unroll
        for (int w = 1; w < GF_NW; ++w) s += red[w][mt][lane];
        if (m < a.M && n < a.N) {
            const float v[4] = {s[0], s[1], s[2], s[3]};
            epi.template store<false>(rp, cp, ep, m, n, v, split, min(4, a.N - n));
        }
    }
}

namespace {
// Rows per workgroup: 16 * MT, more of them where the rows are there, so that
// a weight chunk serves more rows.  MAXST: chunks per wave in flight.
template <int MT, int XM, class Epi>
void go(hipStream_t st, const F32Args& a, int splits, Epi epi) {
    const dim3 grid((a.N + 15) / 16, (a.M + 16 * MT - 1) / (16 * MT), splits), block(64 * GF_NW);
    const int per_wave = (a.k_per_split / 16 + GF_NW - 1) / GF_NW;
    if (per_wave <= 1) hipLaunchKernelGGL((gemm_f32_kernel<MT, 1, XM, Epi>), grid, block, 0, st, a, epi);
    else if (per_wave == 2) hipLaunchKernelGGL((gemm_f32_kernel<MT, 2, XM, Epi>), grid, block, 0, st, a, epi);
    else hipLaunchKernelGGL((gemm_f32_kernel<MT, 4, XM, Epi>), grid, block, 0, st, a, epi);
}

template <class Epi>
hipError_t launch(hipStream_t st, const GemmArgs& g, Epi epi) {
    F32Args a{};
    a.X = (const float*)g.X; a.ldx = g.ldx; a.M = g.M;
    a.W = (const float*)g.W; a.N = g.N; a.K = g.K;
    const int splits = g.epi == EPI_PARTIAL ? g.splits : 1;
    if (splits < 1 || g.K % (16 * splits) || g.M < 1) return hipErrorInvalidValue;
    a.k_per_split = g.K / splits;
    if (g.xm != 0) {
        if (!gemm_f32_ln_ok(g.M, g.K) || g.ldx != g.K || splits != 1) return hipErrorInvalidValue;
        a.g = g.ln_g; a.beta = g.ln_b; a.st = g.st; a.Q = g.Q; a.hz = g.hz;
        if (g.xm == 1) go<1, 1>(st, a, 1, epi);
        else go<1, 2>(st, a, 1, epi);
    } else if (g.M <= 16) {
        go<1, 0>(st, a, splits, epi);
    } else if (g.M <= 32) {
        go<2, 0>(st, a, splits, epi);
    } else {
        go<4, 0>(st, a, splits, epi);
    }
    return hipGetLastError();
}
}  // namespace

// Whether the product takes its rows' LayerNorm itself (GemmArgs::xm): one
// wave per row, and a row of at most GF_MAXQ float4 per lane.
bool gemm_f32_ln_ok(int M, int K) { return M <= GF_NW && K % 256 == 0 && K <= 256 * GF_MAXQ; }

hipError_t gemm_f32(hipStream_t st, const GemmArgs& a) {
    switch (a.epi) {
    case EPI_QKV: return launch(st, a, EpiQKV<float>{a.q, a.bias, a.rows, a.kv, a.d});
    case EPI_GELU: return launch(st, a, EpiGelu<float>{(float*)a.out, a.bias, a.ldo, 0});
    case EPI_PARTIAL: return launch(st, a, EpiPartial{(float*)a.out, a.ldo, a.split_stride});
    case EPI_RESID:
        if (a.N % 4) return hipErrorInvalidValue;
        return launch(st, a, EpiResid{(float*)a.out, a.bias, a.ldo});
    case EPI_LOGITS: return launch(st, a, EpiLogits{(float*)a.out, a.bias, a.ldo, a.N});
    }
    return hipErrorInvalidValue;
}

}  // namespace mtp
