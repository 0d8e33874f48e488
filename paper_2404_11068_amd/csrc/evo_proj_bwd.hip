// evo_proj_bwd.hip -- backward of the fused LayerNorm + batched projections,
// gfx950.
//
// With y = LN(x) (saved by the forward as bf16) and upstream gradients
// dout_p of the P projections:
//
//   dY      = sum_p dout_p W_p          [R, C]   (dy_kernel, MFMA)
//   dx, dln = LayerNorm backward of dY           (dy_kernel's epilogue)
//   dW_p    = dout_p^T y                [HD, C]  (dw_kernel, MFMA, per token chunk)
//   dbias_p = sum over tokens of dout_p          (same kernel, a ones operand)
//
// followed by a fixed-order sum of the per-chunk dW / dbias partials.  In
// both products the contraction runs along an axis that is not contiguous in
// one operand (features of W in dY, tokens in dW), so those operands are
// staged in LDS and read with the transposing LDS read (ds_read_b64_tr_b16),
// which yields the MFMA fragment directly.
#include <stdlib.h>

#include "evo_frag.h"
#include "evo_kernels.h"

namespace evo {
namespace {

// Row padding (bf16 elements) of the LDS tiles read with the transposing LDS
// read.  Per 32 lanes that read takes 64 contiguous bytes from each of four
// consecutive rows; it is conflict-free when the four rows fall in distinct
// 64-byte groups of the 64 four-byte banks.  With 32 elements of padding the
// row stride is 16 or 48 dwords past a multiple of 64 for every width used
// here but 32 (which keeps a two-way conflict).  Padding by 8 left two-way
// conflicts on every read: 6.4M conflict cycles per call at 32768 tokens x
// 256 channels, against 0.13M now.
constexpr int kLdsPad = 32;

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// workgroups of the weight-gradient pass (about one per CU)
inline int proj_bwd_dw_wgs() {
    static const int v = [] {
        const char *e = getenv("EVO_PROJ_DW_WGS");
        const int x = e ? atoi(e) : 0;
        return x >= 8 && x <= 65536 ? x : 256;
    }();
    return v;
}

// features per workgroup of the weight-gradient pass: 64, or 128 when C = 64
// (at least eight 32x32 output tiles, one per wave).  A block lies inside one
// projection (FB divides HD) or covers whole projections (HD divides FB, FB
// divides P*HD); 32 always qualifies (HD is a multiple of 32).
inline int proj_bwd_fb(int C, int HD, int P) {
    const int want = C == 64 ? 128 : 64;
    for (int fb = want; fb > 32; fb /= 2)
        if (HD % fb == 0 || (fb % HD == 0 && (P * HD) % fb == 0)) return fb;
    return 32;
}

// tokens per workgroup of the dY pass: 128 (at 64 channels eight 32 x 32 tiles,
// one per wave), at 256 channels fewer, down to the same eight tiles, while the
// workgroups would leave CUs idle.  At 128 channels always 64: with 128, two workgroups no longer share a CU (100000 tokens x 128:
// backward 88.5 -> 79.6 us, as a plain layer 44.7 -> 39.5); at 256 channels 64
// would read the weight twice as often (32768 x 256: 77.5 against 69.8 us).
inline int dy_block_tokens(int64_t R, int C) {
    if (C < 256) return C == 128 ? 64 : 128;
    int tm = 128;
    while (tm > 32 && (R + tm - 1) / tm < 256) tm /= 2;
    return tm;
}

// a wave-uniform pointer, moved to scalar registers
__device__ __forceinline__ const char *uniform_ptr(const char *p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char *)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ const void *dout_ptr(const PjBwdArgs &a, int p) {
    return p == 0 ? a.dout0 : p == 1 ? a.dout1 : p == 2 ? a.dout2 : a.dout3;
}

// ---------------------------------------------------------------------------
// dY of TM tokens x all C channels per workgroup of eight waves, and with a
// LayerNorm its backward in the epilogue: dx of the tokens and one partial row
// of dln_w | dln_b.  The waves form a WT x WC grid over the tokens and channels,
// MT x MC tiles of 32 x 32 each (two by two at 128 tokens x 256 channels: a
// fragment read from LDS then serves two products).  The contraction runs over
// stages of 64 features; both operands of a stage go through LDS
// (double-buffered): the dout rows [TM][64], 16-byte chunk c of row r at
// c ^ akey(r), read back as row fragments, and the weight rows [64][C], read
// back with the transposing read.  Global loads are issued four stages ahead
// into a ring of register stages, in one in-order stream (the memory counter
// retires loads in issue order, so a wait for one load is a wait for every
// older one).
//
// The LayerNorm epilogue takes dY through LDS in fp32 to whole rows (C/8 lanes a row),
// so it is not rounded to bf16 on its way into the LayerNorm backward, and
// neither dY (33 MB written and read at 32768 x 256) nor a second kernel is
// left.  32768 x 256, F 1024 (kernel trace, minima): dY 32.3 + LayerNorm
// backward 11.7 + its reduction 3.9 us -> 36.6 us; the whole backward 80.6 -> 70 us.
template <int C, int TM>
struct DyCfg {
    static constexpr int NW = 8, NT = 64 * NW, KC = 64;
    static constexpr int TT = TM / 32, CT = C / 32;
    static constexpr int WT = CT >= 8 ? (TT >= 4 ? 2 : 1) : CT == 4 ? 2 : 4;  // token groups of waves
    static constexpr int WC = NW / WT;
    static constexpr int MT = TT / WT, MC = CT / WC;
    static_assert(MT >= 1 && MC >= 1 && MT * WT == TT && MC * WC == CT, "wave grid");
    static constexpr int WSTR = C + kLdsPad;      // weight stage row stride (elements)
    static constexpr int LW = KC * WSTR, LA = TM * KC;
    static constexpr int OSTR = C + 4;            // row stride of the fp32 dY tile (floats)
    static constexpr int NRED = 2 * C * NW;       // dln partials of the waves (floats)
    static constexpr int LDS_STAGE = 2 * (LW + LA) * 2, LDS_OUT = (TM * OSTR + NRED) * 4;
    template <bool LN> static constexpr int LDS = !LN || LDS_STAGE > LDS_OUT ? LDS_STAGE : LDS_OUT;
};

// Chunk swizzle of the dout rows (128 bytes, eight 16-byte chunks): reading one
// chunk of 16 consecutive rows, and writing four chunks of four consecutive
// rows (consecutive lanes on one row's 64 bytes, so that a load's lanes share
// cache lines), touch every bank once.
__device__ __forceinline__ int akey(int r) {
    const int j = (r >> 1) & 7;
    return ((j & 1) << 2) | (j >> 1);
}

// v from another lane of the same 16-lane row, chosen by a DPP control word
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
// sum over LPR consecutive lanes (8, 16 or 32), left in each of them
template <int LPR>
__device__ __forceinline__ float row_sum(float v) {
    v += dpp<0xB1>(v);                               // quad_perm [1,0,3,2]
    v += dpp<0x4E>(v);                               // quad_perm [2,3,0,1]
    v += dpp<0x141>(v);                              // row_half_mirror
    if constexpr (LPR >= 16) v += dpp<0x140>(v);     // row_mirror
    if constexpr (LPR >= 32) v += __shfl_xor(v, 16, 64);
    return v;
}

template <int C, int TM, bool LN, int NR>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void dy_kernel(PjBwdArgs a,
                                                                                     float *__restrict__ part_ln) {
    using G = DyCfg<C, TM>;
    constexpr int NT = G::NT, KC = G::KC, MT = G::MT, MC = G::MC, WSTR = G::WSTR;
    constexpr int NA = (TM * KC / 8 + NT - 1) / NT;  // dout 16-byte chunks per thread and stage
    constexpr int NWL = KC * C / 8 / NT;             // weight 16-byte chunks per thread and stage
    static_assert(NWL * NT == KC * C / 8, "stage split");
    __shared__ __attribute__((aligned(16))) char lds[G::template LDS<LN>];
    uint16_t *const st = (uint16_t *)lds;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int wt = wave / G::WC, wc = wave % G::WC;
    const int64_t row0 = (int64_t)blockIdx.x * TM;
    int64_t nrows = a.R - row0;
    nrows = nrows < TM ? nrows : TM;
    const int F = a.P * a.HD;
    const int NS = (F + KC - 1) / KC;
    const rsrc_t rW = make_buf(a.W, (uint32_t)F * C * 2u);

    // dout chunk j of this thread: half hf of the stage (32 features, all in
    // one projection), token row r, 16-byte column c4 of the half
    int a_r[NA], a_c4[NA], a_hf[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int idx = tid + j * NT;
        a_hf[j] = __builtin_amdgcn_readfirstlane(idx / (TM * 4));
        const int ii = idx % (TM * 4);
        a_r[j] = ii >> 2;
        a_c4[j] = ii & 3;
    }
    const uint32_t ablk = (uint32_t)nrows * a.HD * 2u;
    const int64_t aoff = row0 * a.HD * 2;
    auto load_stage = [&](int s, u32x4 (&ra)[NA], u32x4 (&rw)[NWL]) {
#pragma unroll
        for (int j = 0; j < NA; ++j) {
            // projection and feature offset of the half (scalar)
            const int f = s * KC + 32 * a_hf[j];
            const int p = (f >= a.HD) + (f >= 2 * a.HD) + (f >= 3 * a.HD);
            const bool in = f < F && a_hf[j] < 2;
            const char *base = uniform_ptr((const char *)dout_ptr(a, in ? p : 0) + aoff);
            const rsrc_t ro = make_buf(base, __builtin_amdgcn_readfirstlane(in ? ablk : 0u));
            ra[j] = bload16(ro, (uint32_t)(a_r[j] * a.HD + (f - p * a.HD) + 8 * a_c4[j]) * 2u);
        }
#pragma unroll
        for (int j = 0; j < NWL; ++j) {  // weight rows s*KC .. (rows past F read as zeros)
            const int idx = tid + j * NT;
            const int rr = idx / (C / 8), c8 = idx % (C / 8);
            rw[j] = bload16(rW, (uint32_t)((s * KC + rr) * C + c8 * 8) * 2u);
        }
    };
    auto store_stage = [&](int buf, const u32x4 (&ra)[NA], const u32x4 (&rw)[NWL]) {
        uint16_t *wl = st + buf * (G::LW + G::LA);
        uint16_t *al = wl + G::LW;
#pragma unroll
        for (int j = 0; j < NA; ++j)
            if (a_hf[j] < 2) *(u32x4 *)&al[a_r[j] * KC + 8 * ((4 * a_hf[j] + a_c4[j]) ^ akey(a_r[j]))] = ra[j];
#pragma unroll
        for (int j = 0; j < NWL; ++j) {
            const int idx = tid + j * NT;
            const int rr = idx / (C / 8), c8 = idx % (C / 8);
            *(u32x4 *)&wl[rr * WSTR + c8 * 8] = rw[j];
        }
    };

    f32x16 acc[MT][MC];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MC; ++j) acc[i][j] = zero16();
    u32x4 ra[NR][NA], rw[NR][NWL];
#pragma unroll
    for (int u = 0; u < NR; ++u) load_stage(u, ra[u], rw[u]);
    store_stage(0, ra[0], rw[0]);
    load_stage(NR, ra[0], rw[0]);
    __syncthreads();
    for (int s0 = 0; s0 < NS; s0 += NR) {
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int s = s0 + u;
            const uint16_t *wl = st + (u & 1) * (G::LW + G::LA);
            const uint16_t *al = wl + G::LW;
            if (s < NS) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    Tr<bf16_t>::K32 af[MT];
#pragma unroll
                    for (int i = 0; i < MT; ++i) {
                        const int r = (wt * MT + i) * 32 + n;
#pragma unroll
                        for (int q = 0; q < 2; ++q)  // chunks 4t + h and 4t + 2 + h of the row
                            af[i].v[q] = *(const bf16x8 *)&al[r * KC + 8 * ((4 * t + 2 * q + h) ^ akey(r))];
                    }
#pragma unroll
                    for (int j = 0; j < MC; ++j) {
                        const Tr<bf16_t>::K32 bf = load_k32_tr(&wl[(wc * MC + j) * 32], WSTR, 32 * t, 32, lane);
#pragma unroll
                        for (int i = 0; i < MT; ++i) Tr<bf16_t>::mma_k32(acc[i][j], af[i], bf);
                    }
                }
            }
            // stage s+1 (loaded NR stages ago) into the other buffer; its
            // register stage then takes stage s+1+NR
            const int un = (u + 1) % NR;
            store_stage((u + 1) & 1, ra[un], rw[un]);
            load_stage(s + 1 + NR, ra[un], rw[un]);
            __syncthreads();
        }
    }

    if constexpr (!LN) {
        // dY is the result: each wave's tiles as bf16 through an LDS tile of its
        // own (16-byte stores; the stages' last reads are behind the barrier above)
        constexpr int TSTR = 40;
        uint16_t *const tl = st + wave * 32 * TSTR;
        const rsrc_t ro = make_buf((char *)a.dx + row0 * C * 2, (uint32_t)nrows * C * 2u);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < MC; ++j) {
#pragma unroll
                for (int e = 0; e < 16; ++e) tl[(8 * (e / 4) + 4 * h + (e % 4)) * TSTR + sig(n)] = f2bf(acc[i][j][e]);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int t = q * 16 + (lane >> 2), c4 = lane & 3;
                    const u32x4 v = *(const u32x4 *)&tl[t * TSTR + c4 * 8];
                    bstore16(v, ro, (uint32_t)(((wt * MT + i) * 32 + t) * C + (wc * MC + j) * 32 + c4 * 8) * 2u);
                }
                __builtin_amdgcn_wave_barrier();
            }
        return;
    }
    // ---- epilogue: D[token rho(i,h)][channel ct*32 + sig(n)] as fp32 rows in
    // LDS (the stages' last reads are behind the barrier above), then whole
    // rows: LPR lanes per row, 8 channels a lane, RPW rows per wave and pass
    constexpr int LPR = C / 8, RPW = 64 / LPR, NP = TM / (8 * RPW);
    float *const ot = (float *)lds;
    const int li = lane % LPR, rs = lane / LPR;
    const rsrc_t rx = make_buf((const char *)a.x + row0 * C * 2, (uint32_t)nrows * C * 2u);
    u32x4 xv[NP];
    float mv[NP], rv[NP];
    {
        const rsrc_t rm = make_buf(a.mean + row0, (uint32_t)nrows * 4u), rr = make_buf(a.rstd + row0, (uint32_t)nrows * 4u);
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int r = (p * 8 + wave) * RPW + rs;
            xv[p] = bload16(rx, (uint32_t)(r * C + 8 * li) * 2u);
            mv[p] = __uint_as_float(bload4(rm, (uint32_t)r * 4u));
            rv[p] = __uint_as_float(bload4(rr, (uint32_t)r * 4u));
        }
    }
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MC; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int t = (wt * MT + i) * 32 + 8 * (e / 4) + 4 * h + (e % 4);
                ot[t * G::OSTR + (wc * MC + j) * 32 + sig(n)] = acc[i][j][e];
            }
    float wv[8], pw[8], pb[8];
    {
        const rsrc_t rlw = make_buf(a.lnw, C * 4);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f32x4 w4 = __builtin_bit_cast(f32x4, bload16(rlw, (uint32_t)(8 * li + 4 * q) * 4u));
#pragma unroll
            for (int e = 0; e < 4; ++e) wv[4 * q + e] = w4[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) pw[e] = pb[e] = 0.0f;
    }
    __syncthreads();
    const rsrc_t rd = make_buf((char *)a.dx + row0 * C * 2, (uint32_t)nrows * C * 2u);
    constexpr float inv_c = 1.0f / (float)C;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
        const int r = (p * 8 + wave) * RPW + rs;
        bf16x8 o;
        {
            const f32x4 d0 = *(const f32x4 *)&ot[r * G::OSTR + 8 * li], d1 = *(const f32x4 *)&ot[r * G::OSTR + 8 * li + 4];
            const float dy[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
            const uint32_t xw[4] = {xv[p].x, xv[p].y, xv[p].z, xv[p].w};
            float xh[8], g[8], sg = 0.0f, sgx = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = __builtin_bit_cast(float, (e & 1) ? (xw[e / 2] & 0xffff0000u) : (xw[e / 2] << 16));
                xh[e] = (x - mv[p]) * rv[p];
                g[e] = dy[e] * wv[e];
                sg += g[e];
                sgx = __builtin_fmaf(g[e], xh[e], sgx);
                pw[e] = __builtin_fmaf(dy[e], xh[e], pw[e]);
                pb[e] += dy[e];
            }
            const float ma = row_sum<LPR>(sg) * inv_c, mc = row_sum<LPR>(sgx) * inv_c;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)(rv[p] * (g[e] - ma - xh[e] * mc));
        }
        bstore16(__builtin_bit_cast(u32x4, o), rd, (uint32_t)(r * C + 8 * li) * 2u);
    }
    {
        // column sums: the row slots of a wave, then the waves in order
        float *const red = ot + TM * G::OSTR;
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int m = LPR; m < 64; m <<= 1) {
                pw[e] += __shfl_xor(pw[e], m, 64);
                pb[e] += __shfl_xor(pb[e], m, 64);
            }
        if (rs == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                red[wave * 2 * C + 8 * li + e] = pw[e];
                red[wave * 2 * C + C + 8 * li + e] = pb[e];
            }
        }
        __syncthreads();
        if (tid < 2 * C) {
            float t = red[tid];
#pragma unroll
            for (int k = 1; k < 8; ++k) t += red[k * 2 * C + tid];
            part_ln[(int64_t)blockIdx.x * 2 * C + tid] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// Partial dW (FB features x C channels) and dbias over one chunk of tokens.
// Tokens go through LDS 32 at a time (dout [32][FB] and y [32][C] rows,
// double-buffered); their global loads run through a ring of four register
// stages, issued four sub-blocks before the sub-block is staged.  The block
// has 16 waves when its (FB/32) x (C/32) tile grid has 16 tiles or more, else
// 8; wave w owns TPW consecutive tiles, all in one feature tile, so its dout
// fragment serves all of them.  One wave per feature tile (spread over the
// SIMDs) also sums dbias through an all-ones operand.  A feature block may
// span projections (FB > HD): its dout columns are loaded per projection
// segment, each segment by whole waves.  With `xcd_map`, the feature blocks
// of one token chunk are placed on one XCD (workgroups are dealt to the eight
// XCDs in turn), so that chunk's y rows are fetched into that XCD's L2 once.
template <int C, int FB>
struct DwCfg {
    static constexpr int NTILE = (FB / 32) * (C / 32);
    static constexpr int NW = NTILE >= 16 ? 16 : 8;
    static constexpr int NT = 64 * NW;
};

template <int C, int FB>
__global__ __launch_bounds__((DwCfg<C, FB>::NT)) void dw_kernel(PjBwdArgs a, int64_t chunk_tokens, int nfb,
                                                            int xcd_map, float *__restrict__ part_w,
                                                            float *__restrict__ part_b) {
    constexpr int NW = DwCfg<C, FB>::NW, NT = DwCfg<C, FB>::NT;
    constexpr int NFT = FB / 32, NCT = C / 32, NTILE = NFT * NCT;
    constexpr int TPW = NTILE / NW > 0 ? NTILE / NW : 1;
    constexpr int WPF = NCT / TPW;            // waves per feature tile
    constexpr int NR = 4;
    constexpr int DSTR = FB + kLdsPad, YSTR = C + kLdsPad;
    constexpr int ND = (32 * FB / 8 + NT - 1) / NT;
    constexpr int NY = (32 * C / 8 + NT - 1) / NT;
    __shared__ __attribute__((aligned(16))) uint16_t dl[2][32 * DSTR];
    __shared__ __attribute__((aligned(16))) uint16_t yl[2][32 * YSTR];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int F = a.P * a.HD;
    const int L = blockIdx.x;
    int fb, chunk_i;
    if (xcd_map) {
        const int j = L >> 3;
        fb = j % nfb;
        chunk_i = (L & 7) + 8 * (j / nfb);
    } else {
        fb = L % nfb;
        chunk_i = L / nfb;
    }
    const int64_t chunk = chunk_i;
    const int64_t t_begin = chunk * chunk_tokens;
    int64_t t_end = t_begin + chunk_tokens;
    t_end = t_end < a.R ? t_end : a.R;
    const int f0 = fb * FB;
    const int ft = wave / WPF, ct0 = (wave % WPF) * TPW;
    const bool active = ft < NFT;
    const bool bias_owner = active && (wave % WPF) == ft % WPF;

    // dout chunk j of this thread: segment (projection) seg of the block,
    // token row r, 16-byte column c; segments are `segw` features wide and
    // 4 segw chunks long, a multiple of 64, so each wave loads one projection
    const int segw = FB <= a.HD ? FB : a.HD;
    const char *d_base[ND];
    int d_off[ND], d_lds[ND];
#pragma unroll
    for (int j = 0; j < ND; ++j) {
        const int idx = tid + j * NT;
        const int per = 4 * segw;           // chunks per segment: 32 rows x segw / 8
        const int seg = idx / per, rem = idx % per;
        const int r = rem / (segw / 8), c = rem % (segw / 8);
        const int f = f0 + seg * segw;      // first feature of the segment
        const int pj = __builtin_amdgcn_readfirstlane(f / a.HD);
        d_base[j] = uniform_ptr((const char *)dout_ptr(a, pj < a.P ? pj : 0));
        const bool ok = idx < 32 * FB / 8;
        d_off[j] = ok ? (r * a.HD + f % a.HD + 8 * c) * 2 : -1;
        d_lds[j] = r * DSTR + seg * segw + 8 * c;
    }

    auto load_sub = [&](int64_t t0, u32x4 (&dr)[ND], u32x4 (&yr)[NY]) {
        // dout rows t0..t0+31 of this block's features, y rows t0..t0+31
        const int64_t nt = t_end - t0 < 32 ? t_end - t0 : 32;
        const uint32_t dbytes = nt > 0 ? (uint32_t)nt * a.HD * 2u : 0u;
#pragma unroll
        for (int j = 0; j < ND; ++j) {
            const rsrc_t rd_ = make_buf(d_base[j] + t0 * a.HD * 2, dbytes);
            dr[j] = bload16(rd_, d_off[j] >= 0 ? (uint32_t)d_off[j] : kOOB);
        }
        const rsrc_t ry_ = make_buf((const char *)a.y + t0 * C * 2, nt > 0 ? (uint32_t)nt * C * 2u : 0u);
#pragma unroll
        for (int j = 0; j < NY; ++j) {
            const int idx = tid + j * NT;
            const int r = idx / (C / 8), c8 = idx % (C / 8);
            yr[j] = bload16(ry_, idx < 32 * C / 8 ? (uint32_t)(r * C + c8 * 8) * 2u : kOOB);
        }
    };
    auto store_sub = [&](int buf, const u32x4 (&dr)[ND], const u32x4 (&yr)[NY]) {
#pragma unroll
        for (int j = 0; j < ND; ++j)
            if (d_off[j] >= 0) *(u32x4 *)&dl[buf][d_lds[j]] = dr[j];
#pragma unroll
        for (int j = 0; j < NY; ++j) {
            const int idx = tid + j * NT;
            if (idx < 32 * C / 8) {
                const int r = idx / (C / 8), c8 = idx % (C / 8);
                *(u32x4 *)&yl[buf][r * YSTR + c8 * 8] = yr[j];
            }
        }
    };

    // all-ones B operand: D[f][n] += sum over the tokens of dout[t][f]
    Tr<bf16_t>::K32 ones;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < 8; ++s) ones.v[t][s] = (__bf16)1.0f;
    f32x16 acc[TPW], accb = zero16();
#pragma unroll
    for (int j = 0; j < TPW; ++j) acc[j] = zero16();

    const int64_t nsub = (t_end - t_begin + 31) / 32;
    u32x4 dr[NR][ND], yr[NR][NY];
#pragma unroll
    for (int u = 0; u < NR; ++u) load_sub(t_begin + u * 32, dr[u], yr[u]);
    store_sub(0, dr[0], yr[0]);
    load_sub(t_begin + NR * 32, dr[0], yr[0]);
    __syncthreads();
    for (int64_t s0 = 0; s0 < nsub; s0 += NR) {
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            const int64_t sb = s0 + u;
            const int buf = u & 1;
            if (sb < nsub && active) {
                const Tr<bf16_t>::K32 af = load_k32_tr(&dl[buf][ft * 32], DSTR, 0, 32, lane);
#pragma unroll
                for (int j = 0; j < TPW; ++j) {
                    const Tr<bf16_t>::K32 bf = load_k32_tr(&yl[buf][(ct0 + j) * 32], YSTR, 0, 32, lane);
                    Tr<bf16_t>::mma_k32(acc[j], af, bf);
                }
                if (bias_owner) Tr<bf16_t>::mma_k32(accb, af, ones);
            }
            // sub-block sb+1 (loaded NR sub-blocks ago) into the other buffer; its
            // register stage then takes sub-block sb+1+NR
            const int un = (u + 1) % NR;
            store_sub(buf ^ 1, dr[un], yr[un]);
            load_sub(t_begin + (sb + 1 + NR) * 32, dr[un], yr[un]);
            __syncthreads();
        }
    }

    // partial tiles: D[feature ft*32 + sig(rho(i,h))][channel ct*32 + sig(n)]
    if (!active) return;
    const rsrc_t rpw = make_buf(part_w + chunk * (int64_t)F * C, (uint32_t)F * C * 4u);
#pragma unroll
    for (int j = 0; j < TPW; ++j) {
        const int ct = ct0 + j;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int f = f0 + ft * 32 + sig(8 * (i / 4) + 4 * h + (i % 4));
            bstore4(__float_as_uint(acc[j][i]), rpw, (uint32_t)(f * C + ct * 32 + sig(n)) * 4u);
        }
    }
    if (part_b && bias_owner) {
        const rsrc_t rpb = make_buf(part_b + chunk * (int64_t)F, (uint32_t)F * 4u);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int f = f0 + ft * 32 + sig(8 * (i / 4) + 4 * h + (i % 4));
            bstore4(__float_as_uint(accb[i]), rpb, n == 0 ? (uint32_t)f * 4u : kOOB);
        }
    }
}

// Sums over the partial rows of up to three arrays in one launch:
//   dW [n_part][width], dbias [n_part][width2]: a 256-thread block takes 256 / KS
//   groups of four columns and splits the rows into KS interleaved slices (thread
//   slice ks sums k = ks, ks + KS, ... in order); the slice sums are then added
//   in slice order, so the result does not depend on timing;
//   dln_w | dln_b [n_ln][2C] likewise with 64 slices of four groups (many
//   rows, few columns).
struct ColsumArgs {
    const float *part, *part2, *part_ln;
    float *out, *out2, *dlnw, *dlnb;
    int64_t width, width2, n_part, n_ln;
    int C;
};

template <int KS>
__device__ __forceinline__ f32x4 slice_sum(const float *part, int64_t width, int64_t n_part, int64_t x4, int ks,
                                           f32x4 *red, int qb, int QB) {
    if (x4 >= width) n_part = 0;
    const float *p = part + x4;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    int64_t k = ks;
    for (; k + 3 * KS < n_part; k += 4 * KS) {
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = *(const f32x4 *)(p + (k + u * KS) * width);
#pragma unroll
        for (int u = 0; u < 4; ++u) s += v[u];
    }
    for (; k < n_part; k += KS) s += *(const f32x4 *)(p + k * width);
    if constexpr (KS > 1) {
        red[ks * QB + qb] = s;
        __syncthreads();
        s = red[qb];
#pragma unroll 4
        for (int j = 1; j < KS; ++j) s += red[j * QB + qb];
    }
    return s;
}

template <int KS>
__global__ __launch_bounds__(256) void colsum_kernel(ColsumArgs c) {
    constexpr int QB = 256 / KS;              // four-column groups per block
    constexpr int KL = 64, QL = 256 / KL;
    __shared__ f32x4 red[256];
    int64_t blk = blockIdx.x;
    const int64_t nb1 = (c.width / 4 + QB - 1) / QB, nb2 = (c.width2 / 4 + QB - 1) / QB;
    if (blk < nb1 + nb2) {
        const bool second = blk >= nb1;
        if (second) blk -= nb1;
        const int ks = threadIdx.x / QB, qb = threadIdx.x % QB;
        const int64_t width = second ? c.width2 : c.width, x4 = (blk * QB + qb) * 4;
        const f32x4 s = slice_sum<KS>(second ? c.part2 : c.part, width, c.n_part, x4, ks, red, qb, QB);
        if (ks != 0 || x4 >= width) return;
        bstore16(__builtin_bit_cast(u32x4, s), make_buf(second ? c.out2 : c.out, (uint32_t)(width * 4)),
                 (uint32_t)x4 * 4u);
        return;
    }
    blk -= nb1 + nb2;
    const int ks = threadIdx.x / QL, qb = threadIdx.x % QL;
    const int64_t x4 = (blk * QL + qb) * 4;
    const f32x4 s = slice_sum<KL>(c.part_ln, 2 * c.C, c.n_ln, x4, ks, red, qb, QL);
    if (ks != 0 || x4 >= 2 * c.C) return;
    const bool hi = x4 >= c.C;
    bstore16(__builtin_bit_cast(u32x4, s), make_buf(hi ? c.dlnb : c.dlnw, (uint32_t)c.C * 4u),
             (uint32_t)(hi ? x4 - c.C : x4) * 4u);
}

template <int C, int TM>
hipError_t launch_dy_t(const PjBwdArgs &a, float *part_ln, hipStream_t s) {
    const unsigned nt = (unsigned)((a.R + TM - 1) / TM);
    // one or two stages (a narrow plain layer): a ring of two, the rest would
    // only load zeros
    if (a.lnw)
        hipLaunchKernelGGL((dy_kernel<C, TM, true, 4>), dim3(nt), dim3(512), 0, s, a, part_ln);
    else if (a.P * a.HD > 128)
        hipLaunchKernelGGL((dy_kernel<C, TM, false, 4>), dim3(nt), dim3(512), 0, s, a, part_ln);
    else
        hipLaunchKernelGGL((dy_kernel<C, TM, false, 2>), dim3(nt), dim3(512), 0, s, a, part_ln);
    return hipGetLastError();
}

template <int C, int FB>
void launch_dw(dim3 grid, hipStream_t s, const PjBwdArgs &a, int64_t ct, int nfb, int xm, float *pw, float *pb) {
    hipLaunchKernelGGL((dw_kernel<C, FB>), grid, dim3(DwCfg<C, FB>::NT), 0, s, a, ct, nfb, xm, pw, pb);
}

template <int C>
hipError_t launch_c(const PjBwdArgs &a, void *ws, const PjBwdPlan &plan, hipStream_t s) {
    char *w = (char *)ws;
    // without a LayerNorm (a plain linear layer) dY is the input gradient itself
    const bool ln = a.lnw != nullptr;
    float *pl = (float *)(w + plan.off_ln);
    const int tm = dy_block_tokens(a.R, C);
    hipError_t e;
    if constexpr (C == 256) {
        e = tm == 32 ? launch_dy_t<C, 32>(a, pl, s) : tm == 64 ? launch_dy_t<C, 64>(a, pl, s) : launch_dy_t<C, 128>(a, pl, s);
    } else {
        e = launch_dy_t<C, C == 128 ? 64 : 128>(a, pl, s);
    }
    if (e != hipSuccess) return e;
    const int F = a.P * a.HD;
    float *pw = (float *)(w + plan.off_dw);
    float *pb = a.dbias ? (float *)(w + plan.off_db) : nullptr;
    const int fb = proj_bwd_fb(C, a.HD, a.P);
    const int nfb = F / fb;
    const int xcd_map = plan.n_chunks % 8 == 0;
    const dim3 grid((unsigned)(nfb * plan.n_chunks));
    if (fb == 128) {
        launch_dw<C, 128>(grid, s, a, plan.chunk_tokens, nfb, xcd_map, pw, pb);
    } else if (fb == 64) {
        launch_dw<C, 64>(grid, s, a, plan.chunk_tokens, nfb, xcd_map, pw, pb);
    } else {
        launch_dw<C, 32>(grid, s, a, plan.chunk_tokens, nfb, xcd_map, pw, pb);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // dW, dbias and dln partial sums in one launch (the dbias part empty without
    // a bias, the dln part without a LayerNorm); the chunk range is split over more threads when there are few
    // columns, so that the launch still has about 256 blocks
    const int64_t q = (int64_t)F * C / 4;
    ColsumArgs c{pw, pb, pl, a.dW, a.dbias, a.dlnw, a.dlnb, (int64_t)F * C, a.dbias ? F : 0, plan.n_chunks,
                 ln ? (a.R + tm - 1) / tm : 0, C};
    const unsigned nln = ln ? (unsigned)((2 * C / 4 + 3) / 4) : 0u;
    auto blocks = [&](int qb) {
        return dim3((unsigned)((q + qb - 1) / qb + (c.width2 / 4 + qb - 1) / qb) + nln);
    };
    if (q >= 65536) hipLaunchKernelGGL((colsum_kernel<1>), blocks(256), dim3(256), 0, s, c);
    else if (q >= 16384) hipLaunchKernelGGL((colsum_kernel<4>), blocks(64), dim3(256), 0, s, c);
    else hipLaunchKernelGGL((colsum_kernel<16>), blocks(16), dim3(256), 0, s, c);
    return hipGetLastError();
}

}  // namespace

PjBwdPlan plan_proj_bwd(int64_t R, int C, int HD, int P, bool ln) {
    PjBwdPlan pl{};
    const int F = P * HD;
    const int FB = proj_bwd_fb(C, HD, P);
    const int64_t nfb = F / FB > 0 ? F / FB : 1;
    // about one (feature block, token chunk) workgroup per CU: fewer chunks
    // mean fewer partial sums to write and add up; chunks of whole 32-token
    // sub-blocks
    int64_t nch = (proj_bwd_dw_wgs() + nfb - 1) / nfb;
    // chunks of at least 256 tokens: at few tokens the partial sums would
    // otherwise cost more traffic than the inputs (at 4096 tokens x 256
    // channels, 256-token chunks measured 11.2 us, 512-token chunks 12.8)
    const int64_t nmax = R / 256 > 0 ? R / 256 : 1;
    if (nch > nmax) nch = nmax;
    const int64_t cap = ((int64_t)1 << 30) / ((int64_t)F * C * 4);  // partials below 1 GiB
    if (nch > cap) nch = cap > 0 ? cap : 1;
    const int64_t nsub = (R + 31) / 32;
    if (nch > nsub) nch = nsub > 0 ? nsub : 1;
    int64_t subs = (nsub + nch - 1) / nch;
    pl.chunk_tokens = subs * 32;
    pl.n_chunks = R > 0 ? (R + pl.chunk_tokens - 1) / pl.chunk_tokens : 1;
    size_t off = 0;
    const int tm = dy_block_tokens(R, C);
    pl.off_ln = off;
    if (ln) off += align256((size_t)((R + tm - 1) / tm) * 2 * C * 4);
    pl.off_dw = off;
    off += align256((size_t)pl.n_chunks * F * C * 4);
    pl.off_db = off;
    off += align256((size_t)pl.n_chunks * F * 4);
    pl.total = off;
    return pl;
}

hipError_t launch_ln_proj_bwd(const PjBwdArgs &a, void *ws, const PjBwdPlan &plan, hipStream_t s) {
    switch (a.C) {
        case 64: return launch_c<64>(a, ws, plan, s);
        case 128: return launch_c<128>(a, ws, plan, s);
        case 256: return launch_c<256>(a, ws, plan, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace evo
