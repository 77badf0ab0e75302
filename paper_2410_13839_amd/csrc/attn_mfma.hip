// Attention for the bf16 cache on MFMA: decode (attn_dec_kernel) and prefill
// (attn_prefill_fa_kernel), flash-style online softmax with every key product on
// the matrix cores and the probabilities kept in registers.
#include <math.h>

#include "attn_dec.h"
#include "common.h"
#include "launch.h"
#include "wave.h"

namespace mtp {

namespace {
__device__ __forceinline__ uint32_t pk2(float a, float b) {
    return bf16x2_bits(a, b);
}
}  // namespace

// Decode attention (attn_dec.h): one workgroup per (sequence, head, key
// split) of NW waves.
template <int NW, int PD>
__global__ __launch_bounds__(64 * NW) void attn_dec_kernel(AttnMfmaArgs p) {
    attn_dec_body<NW, PD, 16, false>(p, blockIdx.x, blockIdx.y, blockIdx.z, gridDim.y, FrontSync{});
}

template <int NW, int PD>
static hipError_t attn_dec_go_pd(hipStream_t st, const AttnMfmaArgs& a) {
    const size_t lds = (size_t)NW * 16 * 64 * sizeof(float);    // attn_dec_body's s_acc at QN = 16
    static bool attr_set = false;
    if (!attr_set && lds > 48 * 1024) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_dec_kernel<NW, PD>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess) return err;
        attr_set = true;
    }
    hipLaunchKernelGGL((attn_dec_kernel<NW, PD>), dim3(a.n_tiles, a.kv.n_heads, a.n_splits), dim3(64 * NW), lds, st, a);
    return hipGetLastError();
}

// Ring depth: two 16-key groups per wave once a split holds that many, for
// 16-wave workgroups (one per CU); smaller workgroups keep one group in
// flight per wave and gain more waves per CU instead (at batch 32: 684 vs
// 695 us per decode step).
template <int NW>
static hipError_t attn_dec_go(hipStream_t st, const AttnMfmaArgs& a) {
    const int groups = (a.split_len + 16 * NW - 1) / (16 * NW);
    if (groups >= 2 && NW == 16) return attn_dec_go_pd<NW, 2>(st, a);
    return attn_dec_go_pd<NW, 1>(st, a);
}

// Prefill attention, flash style (bf16 cache, 16-key pages): one workgroup
// per (64-row query tile, head) of G groups of 4 waves; wave w of a group owns
// the tile's query rows 16 w .. 16 w + 15 and runs over the group's blocks of 64
// keys (four pages; group i takes blocks i, i + G, ...).
// Each block's K rows and V^T rows are staged once in LDS for the four waves
// (double-buffered: the next block's loads sit in registers while the
// current one is consumed; keys past the context are zeroed in V^T, whose
// products with a zero probability must not meet a NaN):
//   S^T[key][q] = K[key][:] . Q[q][:]       16 x 16 x 32 MFMA, 2 k steps per
//                                          16-key tile; Q is pre-scaled by
//                                          log2(e) / 8, so exp2 applies
//   O^T[dim][q] += V^T[dim][key] P^T[key][q] 16 x 16 x 32 MFMA whose 32-deep
//                                          k index takes keys 4 g .. 4 g + 3
//                                          of two 16-key tiles: lane (r, g)'s
//                                          P^T operand is then exactly its own
//                                          S^T values after exp2.
// Causal, or bidirectional (every row sees its sequence's ctx_len keys) with
// p.bidir.  Rows of the tile past its row count compute and are not stored.
//
// What bounds it with many workgroups is vector issue: a block's 16 exponentials
// a lane take as long as its MFMAs.  The softmax around them is kept small: the
// products start from -m (the reference the exponentials subtract) instead of
// zero, m moves only when a score exceeds it by 8 (2^8 in float32 sums and bf16
// probabilities of unchanged relative precision; a ballot decides, the lanes'
// maxima are combined only then), and the row sums stay per lane until the end.
// V^T is staged in the order its operand reads want, 16 bytes a lane.
// With few workgroups it is one wave's chain per block (1.5 us), so two groups
// share the keys (G = 2) and are merged through LDS at the end.
// Measured, 16 heads, before and after (us; the parts: softmax and two groups,
// a head's tiles on one XCD, scalar page addresses): 8 utterances of 6720 rows,
// bidirectional, 83.5 -> 75.2 -> 71.5 -> 63.5; one of 1075 rows 28.2 -> 22.3 ->
// 21.7 -> 20.7; causal, 32 prompts of 10678 rows 49.2 -> 48.7 -> 44.7 -> 42.4,
// one of 325 rows 10.4 -> 9.0 -> 8.0 -> 7.6.
// Workgroup barrier for LDS hand-offs: waits for this wave's LDS operations
// only, so global loads issued for later blocks stay in flight across it
// (__syncthreads() would wait for them too).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int G>
__global__ __launch_bounds__(256 * G) void attn_prefill_fa_kernel(AttnMfmaArgs p) {
    constexpr int KP = 72;                       // padded staged row (bf16): 144 B
    constexpr float MSTEP = 8.0f;                // scores above m before it moves (log2 units)
    __shared__ __attribute__((aligned(16))) bf16_t s_stage[G][4][64 * KP];
    // tiles of one head on one XCD (the dispatcher deals workgroups to the 8
    // XCDs in turn), whose L2 then holds the head's keys for all of them
    int head, tix;
    if ((p.kv.n_heads & 7) == 0) {
        const int j = blockIdx.x >> 3, hq = j / p.n_tiles;
        head = (blockIdx.x & 7) + 8 * hq;
        tix = j - hq * p.n_tiles;
    } else {
        head = blockIdx.x / p.n_tiles;
        tix = blockIdx.x - head * p.n_tiles;
    }
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);   // uniform per wave
    const int tid = threadIdx.x & 255, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    bf16_t (*sk)[64 * KP] = &s_stage[grp][0];    // two buffers [key][dim]
    // two buffers [dim][key]: 32-key half hf, then the operand's order: key 4 g
    // + e of 16-key tile 2 hf + t at 32 hf + 8 g + 4 t + e
    bf16_t (*sv)[64 * KP] = &s_stage[grp][2];
    const int r = lane & 15, g = lane >> 4;
    const int2 tile = p.tiles[tix];
    const int row0 = tile.x, nrows = tile.y;
    if (nrows <= 0) return;                      // uniform over the workgroup
    const int b = p.rows[row0].seq;
    const int pos0 = p.rows[row0].pos;
    const bool bidir = p.bidir != 0;
    const int kend = bidir ? p.st[b].ctx_len : pos0 + nrows;
    const int nblk = (kend + 63) >> 6;
    const bf16_t* pool = reinterpret_cast<const bf16_t*>(p.kv.pool);
    // the sequence's pages up to the last block, looked up once into LDS (a
    // load whose address waits on a page-table load would also wait for the
    // loads of the block in flight before it)
    extern __shared__ int s_pg[];
    const int npg = min(p.kv.max_pages_per_seq, nblk * 4);
    for (int i = threadIdx.x; i < npg; i += 256 * G) s_pg[i] = p.kv.block_table[(size_t)b * p.kv.max_pages_per_seq + i];
    __syncthreads();

    // Two register sets (A, B): a block's loads go out two blocks before its
    // compute (one block of compute hid too little of the load latency).
    // Thread t moves the 16-byte chunks t and t + 256 of the block's four
    // 2 KB K blocks and of its four 2 KB V^T blocks; the chunks are plain
    // variables (arrays of them ended up in scratch memory).
    // (a wave's 64 chunks lie in one page, so the page and the address of its
    // block are scalar)
    const bf16_t* kvb = pool + kv_page_block(p.kv, 0, 0, head) + (tid & 127) * 8;
    const size_t vt_off = (size_t)p.kv.n_heads * 16 * MTP_HEAD_DIM;      // V^T block after the K block
    const size_t pg_str = 2 * vt_off;                                    // page after page
#define MTP_FA_GLOAD1(KR, VR, I, BLK)                                                             \
    {                                                                                             \
        const int pg = (wave >> 1) + 2 * (I);                                                     \
        const size_t o = __builtin_amdgcn_readfirstlane(s_pg[min((BLK) * 4 + pg, npg - 1)]) * pg_str; \
        KR = *reinterpret_cast<const uint4*>(kvb + o);                                            \
        VR = *reinterpret_cast<const uint4*>(kvb + o + vt_off);                                   \
    }
#define MTP_FA_SSTORE1(KR, VR, I, BUF, BLK)                                                       \
    {                                                                                             \
        const int c = tid + 256 * (I), pg = c >> 7, w = c & 127;                                  \
        /* K chunk w: slot w / 8, dims 8 (w % 8) ..; V^T chunk w: dim w / 2, keys 8 (w % 2) .. */ \
        *reinterpret_cast<uint4*>(&sk[BUF][(pg * 16 + (w >> 3)) * KP + (w & 7) * 8]) = KR;        \
        uint4 v = VR;                                                                             \
        const int k0 = (BLK) * 64 + pg * 16 + (w & 1) * 8;                                        \
        if (k0 + 8 > kend) { /* keys past the context: zero */                                    \
            uint32_t m[4];                                                                        \
            _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                       \
                const uint32_t lo = k0 + 2 * j < kend ? 0x0000FFFFu : 0u;                         \
                const uint32_t hi = k0 + 2 * j + 1 < kend ? 0xFFFF0000u : 0u;                     \
                m[j] = lo | hi;                                                                   \
            }                                                                                     \
            v = make_uint4(v.x & m[0], v.y & m[1], v.z & m[2], v.w & m[3]);                       \
        }                                                                                         \
        bf16_t* vd = &sv[BUF][(w >> 1) * KP + (pg >> 1) * 32 + (w & 1) * 16 + (pg & 1) * 4];      \
        *reinterpret_cast<uint2*>(vd) = make_uint2(v.x, v.y);                                     \
        *reinterpret_cast<uint2*>(vd + 8) = make_uint2(v.z, v.w);                                 \
    }
    uint4 kA0, kA1, vA0, vA1, kB0, kB1, vB0, vB1;
    auto gloadA = [&](int blk) { MTP_FA_GLOAD1(kA0, vA0, 0, blk) MTP_FA_GLOAD1(kA1, vA1, 1, blk) };
    auto gloadB = [&](int blk) { MTP_FA_GLOAD1(kB0, vB0, 0, blk) MTP_FA_GLOAD1(kB1, vB1, 1, blk) };
    auto sstoreA = [&](int buf, int blk) { MTP_FA_SSTORE1(kA0, vA0, 0, buf, blk) MTP_FA_SSTORE1(kA1, vA1, 1, buf, blk) };
    auto sstoreB = [&](int buf, int blk) { MTP_FA_SSTORE1(kB0, vB0, 0, buf, blk) MTP_FA_SSTORE1(kB1, vB1, 1, buf, blk) };
#undef MTP_FA_GLOAD1
#undef MTP_FA_SSTORE1

    // every stage issues its loads and its LDS stores, the last ones of a
    // clamped (repeated) block into a buffer nobody reads: with conditional
    // ones the compiler's wait counts become the conservative merge of both
    // paths and wait for the newest loads too
    gloadA(min(grp, nblk - 1));
    gloadB(min(grp + G, nblk - 1));
    bf16x8_t qf[2];
    {
        const float sc = 0.18033688011112042f;   // log2(e) / sqrt(64)
        const float* qp = p.q + (size_t)(row0 + min(16 * wave + r, nrows - 1)) * p.ldq + head * 64 + g * 8;
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
            const float4 x = *reinterpret_cast<const float4*>(qp + 32 * h2);
            const float4 y = *reinterpret_cast<const float4*>(qp + 32 * h2 + 4);
            qf[h2] = __builtin_bit_cast(bf16x8_t, make_uint4(pk2(x.x * sc, x.y * sc), pk2(x.z * sc, x.w * sc),
                                                             pk2(y.x * sc, y.y * sc), pk2(y.z * sc, y.w * sc)));
        }
    }
    const int qpos = pos0 + 16 * wave + r;       // this lane's query position
    const int qlast = pos0 + 16 * wave + 15;     // the wave's last query position
    // m_run: the row's reference (-infinity before its first visible key), the
    // same in the four lanes of a row; l_run: this lane's share of the row sum
    float m_run = -INFINITY, l_run = 0.f;
    f32x4_t acc[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) acc[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};

    auto compute = [&](int buf, int blk) {
        const int kb0 = blk * 64;
        if (blk < nblk && (bidir || kb0 <= qlast)) {   // uniform per wave: some key of the block is visible
            const bf16_t* K = sk[buf];
            const bf16_t* VT = sv[buf];
            const bool unseen = m_run == -INFINITY;
            const float c0 = unseen ? 0.f : -m_run;
            f32x4_t sc4[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16_t* kr = K + (16 * t + r) * KP + 8 * g;
                sc4[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(kr), qf[0],
                                                                 f32x4_t{c0, c0, c0, c0}, 0, 0, 0);
                sc4[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<const bf16x8_t*>(kr + 32), qf[1],
                                                                 sc4[t], 0, 0, 0);
            }
            if (kb0 + 64 > kend || (!bidir && kb0 + 63 > pos0 + 16 * wave)) {   // uniform per wave
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int key = kb0 + 16 * t + 4 * g + e;
                        const bool ok = key < kend && (bidir || key <= qpos);
                        sc4[t][e] = ok ? sc4[t][e] : -INFINITY;
                    }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int t = 0; t < 4; ++t)
                mx = fmaxf(mx, fmaxf(fmaxf(sc4[t][0], sc4[t][1]), fmaxf(sc4[t][2], sc4[t][3])));
            if (__any(mx > (unseen ? -INFINITY : MSTEP))) {   // uniform: some row's reference moves
                mx = xor16_max(mx);
                mx = xor32_max(mx);
                // (a row with no visible key yet keeps m = -infinity and subtracts 0)
                const float dm = unseen ? (mx == -INFINITY ? 0.f : mx) : fmaxf(mx, 0.f);
                const float scale = unseen ? 1.f : __builtin_amdgcn_exp2f(-dm);   // unseen: sums are still 0
                m_run = unseen ? mx : m_run + dm;
                l_run *= scale;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) acc[dt] *= scale;
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e) sc4[t][e] -= dm;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
#pragma unroll
                for (int e = 0; e < 4; ++e) sc4[t][e] = __builtin_amdgcn_exp2f(sc4[t][e]);
                l_run += (sc4[t][0] + sc4[t][1]) + (sc4[t][2] + sc4[t][3]);
            }
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                const int t0 = 2 * pr, t1 = 2 * pr + 1;
                const bf16x8_t pf = __builtin_bit_cast(
                    bf16x8_t, make_uint4(pk2(sc4[t0][0], sc4[t0][1]), pk2(sc4[t0][2], sc4[t0][3]),
                                         pk2(sc4[t1][0], sc4[t1][1]), pk2(sc4[t1][2], sc4[t1][3])));
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) {
                    const bf16x8_t vf = *reinterpret_cast<const bf16x8_t*>(VT + (16 * dt + r) * KP + 32 * pr + 8 * g);
                    acc[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf, acc[dt], 0, 0, 0);
                }
            }
        }
    };
    sstoreA(0, min(grp, nblk - 1));
    lds_barrier();
    // (every group runs the first group's number of rounds: the barriers are
    // the workgroup's)
    for (int b0 = 0; b0 < nblk; b0 += 2 * G) {
        // block blk in LDS buffer 0, the group's next one in registers B
        const int blk = b0 + grp;
        gloadA(min(blk + 2 * G, nblk - 1));
        compute(0, blk);
        sstoreB(1, min(blk + G, nblk - 1));
        lds_barrier();
        if (b0 + G >= nblk) break;               // uniform over the workgroup
        // block blk + G in LDS buffer 1, the one after it in registers A
        gloadB(min(blk + 3 * G, nblk - 1));
        compute(1, blk + G);
        sstoreA(0, min(blk + 2 * G, nblk - 1));
        lds_barrier();
    }
    l_run = xor16_sum(l_run);
    l_run = xor32_sum(l_run);
    if constexpr (G == 2) {
        // the second group's rows through LDS (its stage buffers, which its
        // waves are done with after the loop's last barrier)
        float* sm = reinterpret_cast<float*>(s_stage[1]) + (wave * 64 + lane);
        constexpr int ST = 256;                  // floats between values: consecutive lanes, consecutive words
        static_assert(18 * ST * 4 <= (int)sizeof(s_stage[1]), "merge area");
        if (grp == 1) {
            sm[0] = m_run;
            sm[ST] = l_run;
#pragma unroll
            for (int dt = 0; dt < 4; ++dt)
#pragma unroll
                for (int e = 0; e < 4; ++e) sm[(2 + 4 * dt + e) * ST] = acc[dt][e];
        }
        __syncthreads();
        if (grp == 1) return;
        // (the first group has seen the sequence's first key, so m_run is finite)
        const float m1 = sm[0], m = fmaxf(m_run, m1);
        const float s0 = __builtin_amdgcn_exp2f(m_run - m), s1 = __builtin_amdgcn_exp2f(m1 - m);
        l_run = l_run * s0 + sm[ST] * s1;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[dt][e] = acc[dt][e] * s0 + sm[(2 + 4 * dt + e) * ST] * s1;
    }

    // O = O^T / l: lane (r, g) holds dims 16 dt + 4 g .. + 3 of query row r
    const int q = 16 * wave + r;
    if (q < nrows) {
        const float inv = 1.0f / l_run;
        const int row = row0 + q;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const int col = head * 64 + 16 * dt + 4 * g;
            const uint2 o = make_uint2(pk2(acc[dt][0] * inv, acc[dt][1] * inv), pk2(acc[dt][2] * inv, acc[dt][3] * inv));
            *reinterpret_cast<uint2*>(p.out + (p.packed ? frag_off(row, col, p.ldo) : (size_t)row * p.ldo + col)) = o;
        }
    }
}

hipError_t attention_mfma(hipStream_t st, const AttnMfmaArgs& a) {
    if (a.split_len < 32 || a.n_splits < 1 || a.n_splits > 64 || a.kv.page_size != 16) return hipErrorInvalidValue;
    if (a.mode == 0) {
        // decode: pending chunk of at most 16 rows per sequence
        if (a.Q < 1 || a.Q > 16 || a.qt < a.Q || a.split_len % 16) return hipErrorInvalidValue;
        // waves per workgroup: at most one per 16-key group of a split, and
        // few enough that the whole grid is resident at once (16 waves per CU
        // at this kernel's register count)
        const int grid = a.n_tiles * a.kv.n_heads * a.n_splits;
        const int nw_split = a.split_len >= 256 ? 16 : (a.split_len >= 128 ? 8 : 4);
        const int nw_grid = grid <= 256 ? 16 : (grid <= 512 ? 8 : 4);
        const int nw = nw_split < nw_grid ? nw_split : nw_grid;
        if (nw == 16) return attn_dec_go<16>(st, a);
        if (nw == 8) return attn_dec_go<8>(st, a);
        return attn_dec_go<4>(st, a);
    }
    // prefill: tiles of at most 64 rows, one split
    if (a.n_splits != 1 || a.qt != MTP_PREFILL_ROWS) return hipErrorInvalidValue;
    // dynamic LDS: one page number per page of a sequence
    const size_t lds = (size_t)a.kv.max_pages_per_seq * sizeof(int);
    if (lds > 48 * 1024) return hipErrorInvalidValue;
    // two groups a workgroup while those are resident at once (two per CU):
    // 1075 bidirectional rows of 16 heads, 272 workgroups, 28.2 us with one
    // group and the longer softmax, 22.3 us with two
    if (a.n_tiles * a.kv.n_heads <= 512)
        hipLaunchKernelGGL(attn_prefill_fa_kernel<2>, dim3(a.n_tiles * a.kv.n_heads), dim3(512), lds, st, a);
    else
        hipLaunchKernelGGL(attn_prefill_fa_kernel<1>, dim3(a.n_tiles * a.kv.n_heads), dim3(256), lds, st, a);
    return hipGetLastError();
}

}  // namespace mtp
