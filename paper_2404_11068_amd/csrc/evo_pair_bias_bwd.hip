// evo_pair_bias_bwd.hip -- backward of the pair-bias projection, gfx950.
//
// The forward (evo_pair_bias.hip) maps each layer-normalised pair entry
// y = LN(z[b, i, j, :]) to one logit bias per head, v[h] = sum_c y[c] W[h, c]
// (ScaleFold Section 3.3, the pair-bias term of the attention).  Given the
// attention backward's dL/dbias g[b, h, i, j] (fp32, in the forward's output
// layout), this computes
//
//   dY[c]   = sum_h g[h] W[h, c]                      per entry
//   dz      = LayerNorm backward of dY                 per entry, bf16
//   dW[h,c] = sum over entries of g[h] y[c]
//   dln_w   = sum over entries of dY * xhat,   dln_b = sum over entries of dY
//
// With xhat the normalised entry (y = xhat lnw + lnb) every parameter gradient
// follows from two sums over the entries,
//   A[h, c] = sum g[h] xhat[c],   G[h] = sum g[h]:
//   dW[h, c] = lnw[c] A[h, c] + lnb[c] G[h],
//   dln_w[c] = sum_h W[h, c] A[h, c],   dln_b[c] = sum_h W[h, c] G[h],
// and the first row mean of the LayerNorm backward, of lnw dY, is
// sum_h g[h] U[h] / C with U[h] = sum_c lnw[c] W[h, c]: so an entry costs two
// multiply-adds per head and channel, and one row sum besides the statistics.
//
// Workgroups of 4 waves take tiles of 4 rows i x TJ columns j (in turn, when
// there are more tiles than workgroups).  The tile's g values (H x 4 x TJ
// floats) are staged in LDS from 16-byte loads in either layout; each wave then
// takes one row, an entry read by C/8 lanes (16 bytes each), recomputes the
// LayerNorm statistics as the forward does, and writes dz with 16-byte stores.
// A and G accumulate in registers over all of the workgroup's entries and are
// summed in a fixed order (lanes, by the row and half-wave swaps that add two
// registers into one, then waves), and leave as the workgroup's share of the
// gradients, one partial row per workgroup; a second kernel adds the rows in
// workgroup order.  No atomics, so repeated calls give identical bits.
//
// What bounds it: at 256 x 256 entries every workgroup has one tile, so launch,
// one round of loads, the tile's arithmetic and the final sums follow each other.
// Up to four heads the registers leave four waves per SIMD, and tiles are half
// as wide (1024 workgroups).  256 x 256 x 128 (event-timed, kernel + reduction):
// H 4 19.1 -> 17.3 us, H 8 22.6 -> 19.1; 384 x 384: H 4 30.6 -> 24.1, H 8 35.1 -> 30.6.
#include "evo_frag.h"
#include "evo_kernels.h"

namespace evo {
namespace {

constexpr int kPbbWaves = 4;   // rows i per tile, one per wave

// entries per lane group and tile (all loaded before the arithmetic)
__host__ __device__ constexpr int pbb_sl(int H) { return H <= 4 ? 4 : 8; }
// persistent grid: four or two workgroups per CU
__host__ __device__ constexpr int pbb_max_wg(int H) { return H <= 4 ? 1024 : 512; }
// columns j per tile: wave slots of 64 / (C / 8) entries
__host__ __device__ constexpr int pbb_tj(int C, int H) { return pbb_sl(H) * (64 / (C / 8)); }
// floats of a partial row: dW [H][C], dln_w, dln_b
__host__ __device__ constexpr int pbb_row(int C, int H) { return H * C + 2 * C; }

// sum over an LPR-lane group (DPP within 16-lane rows, a swizzle across them)
template <int LPR>
__device__ __forceinline__ float pbb_row_sum(float v) {
    if constexpr (LPR >= 2) v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, false));
    if constexpr (LPR >= 4) v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, false));
    if constexpr (LPR >= 8) v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, false));
    if constexpr (LPR >= 16) v += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xF, 0xF, false));
    if constexpr (LPR >= 32) v += __shfl_xor(v, 16, 64);
    return v;
}

// Sums over the lanes that hold the same channels (lane bits >= log2(LPR)), in
// a fixed order.  Step 32: for registers k and k + N/2 the half-wave swap leaves
// both halves of k in the one and both of k + N/2 in the other's lanes, so one
// add sums the two at once: lanes 0..31 go on with k, the rest with k + N/2.
// Step 16 likewise with the rows of 16 lanes; step 8 (eight-lane groups) adds
// the other half of the row.  Afterwards v[0 .. COUNT) of a lane are the sums of
// registers first .. first + COUNT - 1.
template <int LPR, int N>
struct PbbScatter {
    static constexpr int S16 = LPR <= 16 ? 2 : 1;
    static constexpr int COUNT = N / 2 / S16;
    __device__ __forceinline__ static void run(float (&v)[N], int lane, int *first) {
#pragma unroll
        for (int k = 0; k < N / 2; ++k) {
            const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[k]), __float_as_uint(v[k + N / 2]), false, false);
            v[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        }
        *first = lane >= 32 ? N / 2 : 0;
        if constexpr (LPR <= 16) {
#pragma unroll
            for (int k = 0; k < N / 4; ++k) {
                const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[k]), __float_as_uint(v[k + N / 4]), false, false);
                v[k] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
            }
            *first += (lane & 16) ? N / 4 : 0;
        }
        if constexpr (LPR == 8) {
#pragma unroll
            for (int k = 0; k < COUNT; ++k)
                v[k] += __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v[k]), 0x128, 0xF, 0xF, false));
        }
    }
};

template <int C, int H>
__global__ __launch_bounds__(64 * kPbbWaves) __attribute__((amdgpu_waves_per_eu(H <= 4 ? 4 : 2))) void
pair_bias_bwd_kernel(PbBwdArgs a, int n_tiles, float *__restrict__ part) {
    constexpr int LPR = C / 8;          // lanes per pair entry
    constexpr int PPS = 64 / LPR;       // entries per wave slot
    constexpr int SL = pbb_sl(H);       // slots per wave
    constexpr int TJ = pbb_tj(C, H);    // columns per tile
    constexpr int NX = pbb_row(C, H);
    __shared__ __attribute__((aligned(16))) float gst[H][kPbbWaves][TJ];
    __shared__ __attribute__((aligned(16))) float red[kPbbWaves][H * C + H];  // the waves' A and G
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane % LPR, rs = lane / LPR;
    const int Li = a.Li, Lj = a.Lj;
    const int ntj = (Lj + TJ - 1) / TJ, nti = Li / kPbbWaves;
    constexpr float inv_c = 1.0f / (float)C;

    // ---- loads of a tile: g (in this thread's registers, then LDS) and z
    constexpr int NG = (H * kPbbWaves * TJ / 4 + 64 * kPbbWaves - 1) / (64 * kPbbWaves);
    u32x4 graw[NG], raw[SL];
    int b_t = 0, i0 = 0, j0 = 0;
    auto load_tile = [&](int t) {
        const int jt = t % ntj, rest = t / ntj;
        i0 = rest % nti * kPbbWaves;
        j0 = jt * TJ;
        b_t = rest / nti;
        const rsrc_t rg = make_buf(a.dbias + b_t * (int64_t)H * Li * Lj, (uint32_t)(H * Li * Lj) * 4u);
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            const int idx = tid + q * 64 * kPbbWaves;
            uint32_t off = kOOB;
            if (!a.transpose) {  // rows (h, i) of TJ columns: pieces of 4 columns
                constexpr int NPC = TJ / 4;
                const int h = idx / (kPbbWaves * NPC), w = (idx / NPC) % kPbbWaves, jj = j0 + 4 * (idx % NPC);
                if (h < H && jj < Lj) off = (uint32_t)((h * Li + i0 + w) * Lj + jj) * 4u;
            } else {             // rows (h, j): the tile's 4 rows i are 16 contiguous bytes
                const int h = idx / TJ, jj = j0 + idx % TJ;
                if (h < H && jj < Lj) off = (uint32_t)((h * Lj + jj) * Li + i0) * 4u;
            }
            graw[q] = bload16(rg, off);
        }
        // this wave's row of z (entries past Lj read as zeros and are not
        // written; Li is a multiple of 8, so rows i0..i0+3 exist)
        const rsrc_t rz = make_buf((const char *)a.z + ((int64_t)b_t * Li + i0 + wave) * Lj * C * 2, (uint32_t)Lj * C * 2u);
#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const int j = j0 + s * PPS + rs;
            raw[s] = bload16(rz, j < Lj ? (uint32_t)(j * C + li * 8) * 2u : kOOB);
        }
    };

    // this lane's 8 channels: lnw times every head's weight, and its sums U
    float ww[H][8], U[H];
    {
        const rsrc_t rw = make_buf(a.lnw, C * 4), rW = make_buf(a.W, H * C * 2);
        float wv[8];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f32x4 w4 = __builtin_bit_cast(f32x4, bload16(rw, (uint32_t)(li * 8 + 4 * q) * 4u));
#pragma unroll
            for (int e = 0; e < 4; ++e) wv[4 * q + e] = w4[e];
        }
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const u32x4 w = bload16(rW, (uint32_t)(h * C + li * 8) * 2u);
            const uint32_t wp[4] = {w.x, w.y, w.z, w.w};
            float u = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                ww[h][e] = wv[e] * __uint_as_float((e & 1) ? (wp[e / 2] & 0xffff0000u) : (wp[e / 2] << 16));
                u += ww[h][e];
            }
            U[h] = pbb_row_sum<LPR>(u) * inv_c;
        }
    }

    float acc[H * 8], G[H];
#pragma unroll
    for (int k = 0; k < H * 8; ++k) acc[k] = 0.f;
#pragma unroll
    for (int h = 0; h < H; ++h) G[h] = 0.f;

    for (int t = blockIdx.x; t < n_tiles; t += gridDim.x) {
        load_tile(t);
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            const int idx = tid + q * 64 * kPbbWaves;
            if (!a.transpose) {
                constexpr int NPC = TJ / 4;
                const int h = idx / (kPbbWaves * NPC), w = (idx / NPC) % kPbbWaves, ch = idx % NPC;
                if (h < H) *(u32x4 *)&gst[h][w][4 * ch] = graw[q];
            } else {
                const int h = idx / TJ, c = idx % TJ;
                const f32x4 v = __builtin_bit_cast(f32x4, graw[q]);
                if (h < H) {
#pragma unroll
                    for (int w = 0; w < kPbbWaves; ++w) gst[h][w][c] = v[w];
                }
            }
        }
        const rsrc_t rdz = make_buf((char *)a.dz + ((int64_t)b_t * Li + i0 + wave) * Lj * C * 2, (uint32_t)Lj * C * 2u);
        __syncthreads();

#pragma unroll
        for (int s = 0; s < SL; ++s) {
            const uint32_t xw[4] = {raw[s].x, raw[s].y, raw[s].z, raw[s].w};
            float f[8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                f[2 * q] = __uint_as_float(xw[q] << 16);
                f[2 * q + 1] = __uint_as_float(xw[q] & 0xffff0000u);
            }
            // statistics as in the forward: shift by the entry's first value,
            // mean, then the variance of the centred values
            const float k0 = __shfl(f[0], lane & ~(LPR - 1), 64);
            float sum = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                f[e] -= k0;
                sum += f[e];
            }
            const float mus = pbb_row_sum<LPR>(sum) * inv_c;
            float ss = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                f[e] -= mus;
                ss = fmaf(f[e], f[e], ss);
            }
            const float rstd = rsqrtf(pbb_row_sum<LPR>(ss) * inv_c + a.eps);
            const int p = s * PPS + rs;
            float wd[8], m1 = 0.f;  // lnw dY of the entry, and its mean
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                f[e] *= rstd;
                wd[e] = 0.f;
            }
#pragma unroll
            for (int h = 0; h < H; ++h) {
                const float g = gst[h][wave][p];
                m1 = fmaf(g, U[h], m1);
                G[h] += g;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    wd[e] = fmaf(g, ww[h][e], wd[e]);
                    acc[h * 8 + e] = fmaf(g, f[e], acc[h * 8 + e]);
                }
            }
            float s2 = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) s2 = fmaf(wd[e], f[e], s2);
            const float m2 = pbb_row_sum<LPR>(s2) * inv_c;
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (__bf16)(rstd * (wd[e] - fmaf(f[e], m2, m1)));
            const int j = j0 + p;
            bstore16(__builtin_bit_cast(u32x4, o), rdz, j < Lj ? (uint32_t)(j * C + li * 8) * 2u : kOOB);
            __builtin_amdgcn_sched_barrier(0);  // (slots interleaved would not fit the registers)
        }
        __syncthreads();  // the next tile overwrites gst
    }

    // partial row of this workgroup: lanes holding the same channels, then
    // the four waves, each in a fixed order
    int first = 0;
    using SC = PbbScatter<LPR, H * 8>;
    SC::run(acc, lane, &first);
    if (LPR > 8 || (lane & 8) == 0) {
#pragma unroll
        for (int k = 0; k < SC::COUNT; ++k) {
            const int x = first + k;  // register h * 8 + e
            red[wave][(x >> 3) * C + li * 8 + (x & 7)] = acc[k];
        }
    }
    // G: the entries of a lane group's lanes are the same; the groups in order
#pragma unroll
    for (int h = 0; h < H; ++h) {
        float v = G[h];
#pragma unroll
        for (int m = LPR; m < 64; m *= 2) v += __shfl_xor(v, m, 64);
        if (lane == 0) red[wave][H * C + h] = v;
    }
    __syncthreads();
    for (int x = tid; x < H * C + H; x += 64 * kPbbWaves) {
        float v = red[0][x];
#pragma unroll
        for (int w = 1; w < kPbbWaves; ++w) v += red[w][x];
        red[0][x] = v;
    }
    __syncthreads();
    const rsrc_t rp = make_buf(part + (int64_t)blockIdx.x * NX, NX * 4);
    for (int c = tid; c < C; c += 64 * kPbbWaves) {  // this channel of every head
        const float lw = a.lnw[c], lb = a.lnb[c];
        float dw = 0.f, db = 0.f;
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const float A = red[0][h * C + c], g = red[0][H * C + h];
            const float Wv = bf2f(((const uint16_t *)a.W)[h * C + c]);
            dw = fmaf(Wv, A, dw);
            db = fmaf(Wv, g, db);
            bstore4(__float_as_uint(fmaf(lw, A, lb * g)), rp, (uint32_t)(h * C + c) * 4u);
        }
        bstore4(__float_as_uint(dw), rp, (uint32_t)(H * C + c) * 4u);
        bstore4(__float_as_uint(db), rp, (uint32_t)(H * C + C + c) * 4u);
    }
}

// out = sum over workgroups of the partial rows, in a fixed order: a block
// takes 4 groups of four columns and splits the rows into 64 interleaved
// slices, whose sums are then added in slice order (80 blocks at C = 128,
// H = 8: 16 groups per block left the partial rows to 20 CUs, 4.8 us against
// 4.0 us)
__global__ __launch_bounds__(256) void pb_param_reduce_kernel(const float *__restrict__ part, int n_part, int HC,
                                                             int C, float *__restrict__ dW, float *__restrict__ dlw,
                                                             float *__restrict__ dlb) {
    constexpr int KS = 64, QB = 4;
    __shared__ f32x4 sred[KS][QB];
    const int ks = threadIdx.x / QB, qb = threadIdx.x % QB;
    const int NX = HC + 2 * C;
    const int x4 = (blockIdx.x * QB + qb) * 4;
    const bool ok = x4 < NX;
    const rsrc_t rp = make_buf(part, (uint32_t)n_part * NX * 4u);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    int k = ks;
    for (; k + 3 * KS < n_part; k += 4 * KS) {  // four loads in flight, added in k order
        f32x4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            v[u] = __builtin_bit_cast(f32x4, bload16(rp, ok ? (uint32_t)((k + u * KS) * NX + x4) * 4u : kOOB));
#pragma unroll
        for (int u = 0; u < 4; ++u) s += v[u];
    }
    for (; k < n_part; k += KS) s += __builtin_bit_cast(f32x4, bload16(rp, ok ? (uint32_t)(k * NX + x4) * 4u : kOOB));
    sred[ks][qb] = s;
    __syncthreads();
    if (ks != 0 || !ok) return;
    s = sred[0][qb];
#pragma unroll
    for (int j = 1; j < KS; ++j) s += sred[j][qb];
    float *dst = x4 < HC ? dW + x4 : x4 < HC + C ? dlw + (x4 - HC) : dlb + (x4 - HC - C);
    *(f32x4 *)dst = s;
}

template <int C, int H>
hipError_t launch_ch(const PbBwdArgs &a, void *ws, hipStream_t s) {
    const int64_t n_tiles = a.B * (a.Li / kPbbWaves) * ((a.Lj + pbb_tj(C, H) - 1) / pbb_tj(C, H));
    if (n_tiles > 0x7fffffff) return hipErrorInvalidValue;
    const int64_t nwg = pair_bias_bwd_workgroups(a.B, a.Li, a.Lj, C, H);
    float *part = (float *)ws;
    hipLaunchKernelGGL((pair_bias_bwd_kernel<C, H>), dim3((unsigned)nwg), dim3(64 * kPbbWaves), 0, s, a, (int)n_tiles,
                       part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int nx4 = (H * C + 2 * C) / 4;
    hipLaunchKernelGGL(pb_param_reduce_kernel, dim3((unsigned)((nx4 + 3) / 4)), dim3(256), 0, s, part, (int)nwg,
                       H * C, C, a.dW, a.dlnw, a.dlnb);
    return hipGetLastError();
}

template <int C>
hipError_t launch_c(const PbBwdArgs &a, void *ws, hipStream_t s) {
    switch (a.H) {
        case 1: return launch_ch<C, 1>(a, ws, s);
        case 2: return launch_ch<C, 2>(a, ws, s);
        case 4: return launch_ch<C, 4>(a, ws, s);
        case 8: return launch_ch<C, 8>(a, ws, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace

bool pair_bias_bwd_supported(int C, int H) {
    return (C == 64 || C == 128 || C == 256) && (H == 1 || H == 2 || H == 4 || H == 8);
}

int64_t pair_bias_bwd_workgroups(int64_t B, int Li, int Lj, int C, int H) {
    const int tj = pbb_tj(C, H), most = pbb_max_wg(H);
    const int64_t n_tiles = B * (Li / kPbbWaves) * ((Lj + tj - 1) / tj);
    return n_tiles < most ? (n_tiles > 0 ? n_tiles : 1) : most;
}

size_t pair_bias_bwd_workspace(int64_t B, int Li, int Lj, int C, int H) {
    return (size_t)pair_bias_bwd_workgroups(B, Li, Lj, C, H) * (size_t)pbb_row(C, H) * 4;
}

hipError_t launch_pair_bias_bwd(const PbBwdArgs &a, void *ws, hipStream_t s) {
    switch (a.C) {
        case 64: return launch_c<64>(a, ws, s);
        case 128: return launch_c<128>(a, ws, s);
        case 256: return launch_c<256>(a, ws, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace evo
