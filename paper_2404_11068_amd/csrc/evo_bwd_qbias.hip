// evo_bwd_qbias.hip -- second pass of the two-pass attention backward (dQ and
// dBias) for bf16 at head_dim 8 / 16 / 32, gfx950, where plan_bwd does not find
// qbias_kernel (evo_bwd.hip) cheaper.
//
// One workgroup of eight waves per (bias plane, head, 32-query tile, chunk of
// rows).  The waves take rows of their own (KS = 1) or share a row between
// them, each a part of its key tiles (KS = 2, 4): a wave recomputes
// S^T = K Q^T + sqrt(d) bias^T and dP^T = V dA^T over its key tiles (lane =
// query, registers = keys), keeps dQ of the row in registers, and adds
// dS = P (dP - Dsum) to dBias accumulators it holds over all its rows (16
// registers per key tile).  The pair-bias tiles, the same for every row, sit in
// LDS in fp32 in the logit tiles' register order and are the starting values
// of the S products.  K and V go from memory to LDS without registers, into
// two tile buffers of the wave's own, two key tiles ahead.  With KS = 1 nothing
// in the row loop waits for another wave; otherwise the key parts' shares of dQ
// meet in LDS, one barrier per row.  After the rows the accumulators are added
// in wave order through LDS and leave as one partial dBias tile per chunk (or,
// with one chunk, as dBias).
//
// Why: qbias_kernel gives each of a workgroup's waves one key tile of one row,
// stages K and V of the row through registers, and sums dQ over all waves
// behind two barriers per row, which pays only where a workgroup has few rows.
// Measured (event-timed, MI355X, bf16, d 32, H 4, a bias shared by all rows):
//   256 rows x 160 keys   39.6 -> 24.7 us     384 x 384   280 -> 132-139 us
//   256 x 224             56.4 -> 36 us       317 x 317   206 -> 75 us
//   256 x 256             48 -> 41 us         256 x 512   162 -> 156 us
// What bounds it now: 0.6 ns per 32 x 32 tile on the chip against about 0.3 of
// issue (VALU busy a third of the time, matrix unit a ninth, waves waiting 0.38
// of theirs).  Without the
// loads of K and V a 384-key call still takes two thirds of its time, without
// the exponentials or the dQ product all of it: two waves per SIMD, all that
// the accumulators leave room for, do not cover the LDS and matrix-unit
// latencies of a tile.  Loading the fragments straight from memory (every lane
// of a load in another cache line) was slower, 154 us at 384 keys; taking the
// rows in another order per query tile, so that not all of them ask for the
// same row at once, was slower too (142 us).
#include <math.h>

#include "evo_frag.h"
#include "evo_kernels.h"

namespace evo {

namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kRqWaves = 8;

struct RqArgs {
    const void *q, *k, *v, *bias;
    const uint8_t *mask;
    const float *lse;
    const void *da;     // workspace [N][H][L][D]
    const float *dsum;  // workspace [N][H][L]
    void *dq;
    float *dst;         // dBias sums: [plane][head][chunk] planes of L rows, `pitch` floats each, or null
    int64_t L, rpb, srow, stok, chunks, rows_per_chunk, n_units;
    int H, pitch;
    float scale;
};

// One wave's K or V tile in LDS: 32 rows of D channels as the memory-to-LDS
// loads leave them (lane l of load j writes its 16 bytes at 1024 j + 16 l).
// At head_dim 32 the lanes pick their chunks so that the tile comes out
// swizzled (sw32).  At head_dim 8 only lanes 0..31 carry the tile; the rest
// repeat it behind it.
template <int D> constexpr int kRqLoads = D == 32 ? 2 : 1;
template <int D> constexpr int kRqTile = kRqLoads<D> * 512;  // elements
typedef __attribute__((address_space(3))) void lds_void;

template <int D, int NKT, int KS>
__global__ void __launch_bounds__(kRqWaves * 64) __attribute__((amdgpu_waves_per_eu(2))) rows_qbias_kernel(RqArgs a) {
    using E = uint16_t;
    using K32 = Tr<bf16_t>::K32;
    using QF = ChFrag<bf16_t, D>;
    constexpr int NW = kRqWaves;
    constexpr int NR = NW / KS;                // rows in flight
    constexpr int NMB = (NKT * 32 + 63) / 64;  // mask bytes per lane
    constexpr int TILE = kRqTile<D>;
    // accumulator tiles per wave and step of the final sum: one in the bias area,
    // at head_dim 32 one in each K/V buffer too
    constexpr int TPS = D == 32 ? 3 : 1;
    // key tiles per step: two where the accumulators leave the registers for
    // it, so that one tile's exponentials run beside the other's products
    constexpr int NP = NKT <= 4 && KS <= 2 ? 2 : 1;
    constexpr int XB = KS <= 2 ? 2 : 1;        // buffers of the dQ shares (two save a barrier per row)
    constexpr int AREA = (KS * NKT > NW ? KS * NKT : NW) * 1024;
    // the bias tiles during the row loop, the accumulators of the final sum after it
    __shared__ __attribute__((aligned(16))) float area[AREA];
    // two K/V tile buffers per wave, each an array of its own so that the
    // compiler's load counters tell a read of one from the loads into the other
    __shared__ __attribute__((aligned(16))) E kv0_lds[NW * 2 * TILE];
    __shared__ __attribute__((aligned(16))) E kv1_lds[NW * 2 * TILE];
    __shared__ __attribute__((aligned(16))) float dqx[KS > 1 ? XB * (KS - 1) * NR * 32 * D : 4];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h2 = lane >> 5, n = lane & 31;
    const int L = (int)a.L;
    const int nqt = (L + 31) / 32;
    // unit -> (plane, chunk, query tile, head), head fastest: the query tiles
    // and heads of one chunk run on one XCD and share its rows' K and V
    const uint32_t unit = xcd_unit32(blockIdx.x, gridDim.x);
    if (unit >= (uint32_t)a.n_units) return;
    const int hh = (int)(unit % (uint32_t)a.H);
    uint32_t rest = unit / (uint32_t)a.H;
    const int qt = (int)(rest % (uint32_t)nqt);
    rest /= (uint32_t)nqt;
    const int64_t chunk = rest % (uint32_t)a.chunks, b = rest / (uint32_t)a.chunks;
    const int64_t r_begin = b * a.rpb + chunk * a.rows_per_chunk;
    int64_t r_end = r_begin + a.rows_per_chunk;
    if (r_end > (b + 1) * a.rpb) r_end = (b + 1) * a.rpb;

    const int ks = KS == 1 ? 0 : wave % KS;  // this wave's key part
    const int rw = wave / KS;                // and its row of the NR in flight
    const int key0 = ks * NKT * 32;
    const int qi = qt * 32 + n;              // this lane's query
    const bool qvalid = qi < L;
    const bool has_mask = a.mask != nullptr;
    const uint32_t stok_b = (uint32_t)(a.stok * 2);
    const uint32_t row_bytes = (uint32_t)(a.L * a.stok * 2);
    const uint32_t q_off = qvalid ? (uint32_t)qi * stok_b : kOOB;
    const rsrc_t none = make_buf(nullptr, 0u);
    const float c2 = a.scale * kLog2e;

    // ---- the bias tiles, once: sqrt(d) * bias in fp32, [tile][4-register group][lane][4]
    {
        const BiasBuf rb = make_bias_buf((const E *)a.bias + (a.bias ? (b * a.H + hh) * (int64_t)L * L : 0),
                                         a.bias ? (uint32_t)(L * L) : 0u);
        const uint32_t b_off = rb.off + (uint32_t)(qi * L + 8 * h2) * 2u;
        float sq_hi, sq_lo;
        sqrt_split(D, sq_hi, sq_lo);
        const float sqd = sq_hi + sq_lo;
        for (int t = wave; t < KS * NKT; t += NW) {
            BiasRaw<true> raw;  // (right for even lengths too: the shift is then 0)
            raw.load(rb.r, qvalid ? b_off + 64u * t : kOOB);
            const K32 f = raw.get(b_off, t * 32 + 32 <= L, L - t * 32 - 8 * h2);
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                f32x4 x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = sqd * (float)f.v[g4 >> 1][4 * (g4 & 1) + e];
                *reinterpret_cast<f32x4 *>(&area[(t * 4 + g4) * 256 + lane * 4]) = x;
            }
        }
    }
    __syncthreads();

    // ---- a row's K and V tiles: memory -> LDS, each token's 16-byte chunks by
    // consecutive lanes (a load in fragment order touches one cache line per
    // lane and ran four times as long in the address unit).  Tokens past the
    // row's end read its last token: their keys are masked.
    constexpr int CPT = D / 8;  // 16-byte chunks per token
    const int lt = (lane / CPT) & 31, lc = D == 32 ? (lane & 3) ^ ((lane >> 4) & 3) : lane % CPT;
    const uint32_t kv_off = (uint32_t)(key0 + lt) * stok_b + (uint32_t)(lc * 16);
    const uint32_t kv_max = (uint32_t)(L - 1) * stok_b + (uint32_t)(lc * 16);
    // (more: false after the chunk's last row, whose prefetches then touch no memory)
    auto load_kv = [&](int64_t r, int kt, E *buf, bool more) {
        const int64_t tb = r * a.srow + (int64_t)hh * D;
        const uint32_t bytes = more ? row_bytes : 0u;
        const rsrc_t rk = make_buf((const E *)a.k + tb, bytes), rv = make_buf((const E *)a.v + tb, bytes);
        E *const dst = buf + wave * 2 * TILE;
#pragma unroll
        for (int j = 0; j < kRqLoads<D>; ++j) {
            const uint32_t o = kv_off + (uint32_t)(32 * kt + 16 * j) * stok_b;
            const uint32_t off = o < kv_max ? o : kv_max;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (lds_void *)(dst + 512 * j), 16, off, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (lds_void *)(dst + TILE + 512 * j), 16, off, 0, 0, 0);
        }
    };
    QF qn, dan;
    float lr = 0.0f, dr = 0.0f;
    uint32_t mr[NMB];
    auto load_row = [&](int64_t r, bool more) {
        const int64_t tb = r * a.srow + (int64_t)hh * D, rh = r * a.H + hh;
        qn.load(make_buf((const E *)a.q + tb, more ? row_bytes : 0u), q_off, h2);
        dan.load(make_buf((const E *)a.da + rh * (int64_t)L * D, more ? (uint32_t)(L * D * 2) : 0u),
                 qvalid ? (uint32_t)(qi * D * 2) : kOOB, h2);
        const uint32_t qo = qvalid && more ? (uint32_t)qi * 4u : kOOB;
        lr = __builtin_bit_cast(float, bload4(make_buf(a.lse + rh * L, (uint32_t)L * 4u), qo));
        dr = __builtin_bit_cast(float, bload4(make_buf(a.dsum + rh * L, (uint32_t)L * 4u), qo));
        const rsrc_t rm = has_mask && more ? make_buf(a.mask + r * L, (uint32_t)L) : none;
#pragma unroll
        for (int j = 0; j < NMB; ++j) mr[j] = bload1(rm, (uint32_t)(key0 + 64 * j + lane));
    };

    const float *const btile = &area[ks * NKT * 1024 + lane * 4];
    const int64_t iters = (r_end - r_begin + NR - 1) / NR;
    int64_t r = r_begin + rw;
    // a wave without a row (left) repeats the chunk's last one and drops the results
    auto row_at = [&](int64_t x) { return x < r_end ? x : r_end - 1; };
    load_row(row_at(r), true);
    load_kv(row_at(r), 0, kv0_lds, true);
    if (NKT > 1) load_kv(row_at(r), 1, kv1_lds, true);
    f32x16 acc[NKT];
#pragma unroll
    for (int t = 0; t < NKT; ++t) acc[t] = zero16();
    for (int64_t it = 0; it < iters; ++it, r += NR) {
        const bool rok = r < r_end;
        if (KS == 1 && !rok) break;
        const int64_t rc = row_at(r), rn = row_at(r + NR);
        const bool more = it + 1 < iters;
        // padded or fully masked queries (and rows past the chunk): P = 0
        const float l2 = qvalid && rok && lr != -INFINITY ? lr * kLog2e : INFINITY;
        const QF qb = qn, dab = dan;
        uint32_t kbs[NMB * 2];
#pragma unroll
        for (int j = 0; j < NMB; ++j) {
            const int key = key0 + 64 * j + lane;
            const uint64_t bal = __ballot((!has_mask || mr[j] != 0) && key < L);
            kbs[2 * j] = (uint32_t)bal;
            kbs[2 * j + 1] = (uint32_t)(bal >> 32);
        }
        // -Dsum: the starting value of the dP tiles where there are registers
        // for it (one subtraction per logit less)
        const float ds = dr;
        f32x16 nds = zero16();
        if constexpr (NP == 2) {
#pragma unroll
            for (int i = 0; i < 16; ++i) nds[i] = -ds;
        }
        f32x16 dq = zero16();
#pragma unroll
        for (int kp = 0; kp < NKT; kp += NP) {
            const int np = NP == 2 && kp + 1 < NKT ? 2 : 1;
            QF ka[NP], va[NP];
            K32 kT[NP];
            f32x16 S[NP], dP[NP];
#pragma unroll
            for (int u = 0; u < np; ++u) {
                const E *const ktile = ((kp + u) & 1 ? kv1_lds : kv0_lds) + wave * 2 * TILE, *const vtile = ktile + TILE;
                if constexpr (D == 32) {
                    load_sw32(ka[u], ktile, sig(n), h2);
                    load_sw32(va[u], vtile, sig(n), h2);
                    kT[u] = load_k32_tr_sw32(ktile, 0, lane);
                } else {
                    ka[u].load(&ktile[sig(n) * D], h2);
                    va[u].load(&vtile[sig(n) * D], h2);
                    kT[u] = load_k32_tr(ktile, D, 0, D, lane, false, false);
                }
            }
            // the tiles are in registers: their buffers take the tiles two
            // further (at the row's end, the next row's first two)
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const int kn = kp + u + 2;
                if (kn < NKT) load_kv(rc, kn, kn & 1 ? kv1_lds : kv0_lds, true);
                else if (NP == 2 && kp + 2 < NKT) continue;
                else load_kv(rn, kn & 1, kn & 1 ? kv1_lds : kv0_lds, more);
            }
            if (NP == 2 ? kp + 2 >= NKT : kp == (NKT > 2 ? NKT - 3 : 0)) load_row(rn, more);
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t kb0 = kbs[kp], kb1 = np > 1 ? kbs[kp + 1] : kb0;
            if ((kb0 | kb1) == 0) continue;
            // S^T = sqrt(d) bias^T + K Q^T, dP^T = V dA^T: lane = query, reg i = key krow(i, h2)
#pragma unroll
            for (int u = 0; u < np; ++u) {
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const f32x4 x = *reinterpret_cast<const f32x4 *>(&btile[((kp + u) * 4 + g4) * 256]);
                    S[u][4 * g4] = x.x; S[u][4 * g4 + 1] = x.y; S[u][4 * g4 + 2] = x.z; S[u][4 * g4 + 3] = x.w;
                }
                QF::mma(S[u], ka[u], qb);
            }
            if ((kb0 & kb1) != 0xffffffffu) {  // masked keys: -2^64 on their rows (row n is key sig(n))
#pragma unroll
                for (int u = 0; u < np; ++u) {
                    // (the lane half from an opaque copy: the term's constant
                    // operand is formed here instead of held over the rows)
                    const short mv = (((u ? kb1 : kb0) >> sig(n)) & 1u) ? (short)0 : kBf16MaskNeg;
                    mma_rank1(S[u], mv, kBf16One, (int)(opaque_u32((uint32_t)lane) >> 5));
                }
            }
#pragma unroll
            for (int u = 0; u < np; ++u) {
                dP[u] = nds;
                QF::mma(dP[u], va[u], dab);
            }
#pragma unroll
            for (int u = 0; u < np; ++u) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(S[u][i], c2, -l2));
                    const float v = p * (NP == 2 ? dP[u][i] : dP[u][i] - ds);
                    acc[kp + u][i] += v;
                    dP[u][i] = v;
                }
                // dQ^T (channels x queries) += K^T dS^T
                Tr<bf16_t>::mma_k32(dq, kT[u], Tr<bf16_t>::pack(dP[u]));
            }
        }
        if constexpr (KS > 1) {
            // the other key parts' shares of dQ, added in part order
            float *const xb = &dqx[((XB > 1 ? (it & 1) : 0) * NR + rw) * (KS - 1) * 32 * D];
            constexpr int GS = D == 8 ? 128 : 256;  // floats per 4-register group
            if (XB == 1) __syncthreads();           // the previous row's shares have been read
            if (ks > 0) {
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {  // [part][4-register group][lane], the groups that hold channels
                    if (16 * (g4 >> 1) >= D) continue;
                    if (D == 8 && h2 == 1) continue;
                    const f32x4 x = {dq[4 * g4], dq[4 * g4 + 1], dq[4 * g4 + 2], dq[4 * g4 + 3]};
                    *reinterpret_cast<f32x4 *>(&xb[(ks - 1) * 32 * D + g4 * GS + lane * 4]) = x;
                }
            }
            __syncthreads();
            if (ks == 0) {
#pragma unroll
                for (int part = 0; part < KS - 1; ++part)
#pragma unroll
                    for (int g4 = 0; g4 < 4; ++g4) {
                        if (16 * (g4 >> 1) >= D) continue;
                        if (D == 8 && h2 == 1) continue;
                        const f32x4 x = *reinterpret_cast<const f32x4 *>(&xb[part * 32 * D + g4 * GS + lane * 4]);
                        dq[4 * g4] += x.x; dq[4 * g4 + 1] += x.y; dq[4 * g4 + 2] += x.z; dq[4 * g4 + 3] += x.w;
                    }
            }
        }
        // ---- dQ of the row's query tile (lane = query, registers 8t .. 8t+7 = channels 16t + 8 h2 ..)
        const rsrc_t rdq = make_buf((E *)a.dq + (rok ? r * a.srow + (int64_t)hh * D : 0), rok ? row_bytes : 0u);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (16 * t >= D) continue;
            const int c0 = 16 * t + 8 * h2;
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                w[e] = (uint32_t)f2bf(dq[8 * t + 2 * e] * a.scale) | ((uint32_t)f2bf(dq[8 * t + 2 * e + 1] * a.scale) << 16);
            bstore16(u32x4{w[0], w[1], w[2], w[3]}, rdq, (c0 < D && ks == 0) ? q_off + (uint32_t)(c0 * 2) : kOOB);
        }
    }
    // (the last row's prefetches write this workgroup's LDS: none may be in
    // flight when it ends)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (a.dst == nullptr) return;

    // ---- dBias of the chunk: the row waves' accumulators added in wave order
    // through LDS, TPS tiles of each wave at a time
    const rsrc_t rp = make_buf(a.dst + ((b * a.H + hh) * a.chunks + chunk) * (int64_t)L * a.pitch,
                               (uint32_t)L * (uint32_t)a.pitch * 4u);
    const bool vec = a.pitch % 4 == 0;
    auto red = [&](int j) { return j == 0 ? area : reinterpret_cast<float *>(j == 1 ? kv0_lds : kv1_lds); };
    static_assert(TPS == 1 || NW * 2 * TILE * 2 >= NW * 1024 * 4, "a K/V buffer holds a tile of every wave");
#pragma unroll
    for (int t0 = 0; t0 < NKT; t0 += TPS) {
        __syncthreads();  // the reads of the bias and K/V tiles, or of the previous step
#pragma unroll
        for (int j = 0; j < TPS; ++j) {
            if (t0 + j >= NKT) continue;
            float *const rj = red(j);
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                const f32x16 &c = acc[t0 + j < NKT ? t0 + j : 0];
                const f32x4 x = {c[4 * g4], c[4 * g4 + 1], c[4 * g4 + 2], c[4 * g4 + 3]};
                *reinterpret_cast<f32x4 *>(&rj[(wave * 4 + g4) * 256 + lane * 4]) = x;
            }
        }
        __syncthreads();
        // four consecutive keys per thread and step: (tile of the step), key
        // part, query, 4-key group
#pragma unroll
        for (int j = 0; j < TPS; ++j) {
            if (t0 + j >= NKT) continue;
            const float *const rj = red(j);
#pragma unroll
            for (int i = 0; i < (KS * 256 + NW * 64 - 1) / (NW * 64); ++i) {
                const int idx = tid + i * NW * 64;
                if (idx >= KS * 256) continue;
                const int c = idx & 7, q = (idx >> 3) & 31, part = idx >> 8;
                // keys 4c .. 4c+3 of the tile are registers 4 g4 .. of lane half hs
                const int g4 = 2 * (c >> 2) + (c & 1), hs = (c >> 1) & 1;
                f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int w = 0; w < NR; ++w)
                    sum += *reinterpret_cast<const f32x4 *>(&rj[((w * KS + part) * 4 + g4) * 256 + (hs * 32 + q) * 4]);
                const int key = (part * NKT + t0 + j) * 32 + 4 * c, qq = qt * 32 + q;
                const bool ok = qq < L && key < L;
                const uint32_t off = ok ? (uint32_t)(qq * a.pitch + key) * 4u : kOOB;
                if (vec) {
                    bstore16(__builtin_bit_cast(u32x4, sum), rp, off);
                } else {
                    const float v[4] = {sum.x, sum.y, sum.z, sum.w};
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        bstore4(__builtin_bit_cast(uint32_t, v[e]), rp, ok && key + e < L ? off + 4u * e : kOOB);
                }
            }
        }
    }
}

// dbias[p][q][k] = sum over chunks c of part[p][c][q][k] in chunk order; the
// partial planes' rows are padded to a multiple of four floats.  Four
// consecutive keys per thread, four chunks' loads in flight.
__global__ void __launch_bounds__(256) qbias_reduce_kernel(const float *__restrict__ part, float *__restrict__ dbias,
                                                     int64_t planes, int64_t chunks, int L, int pitch) {
    // (quads of one plane fit 32 bits: L <= 512)
    const uint32_t quads = (uint32_t)L * (uint32_t)(pitch / 4);
    const int64_t plane = (int64_t)L * pitch;
    // blockIdx.y strides over the planes, blockIdx.x covers one plane's quads
    const uint32_t x4 = blockIdx.x * 256u + threadIdx.x;
    if (x4 >= quads) return;
    const int64_t x = (int64_t)x4 * 4;
    const uint32_t q = x4 / (uint32_t)(pitch / 4);
    const int k = (int)(x4 % (uint32_t)(pitch / 4)) * 4;
    for (int64_t p = blockIdx.y; p < planes; p += gridDim.y) {
        const float *src = part + p * chunks * plane + x;
        f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
        int64_t c = 0;
        for (; c + 4 <= chunks; c += 4) {
            f32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = *reinterpret_cast<const f32x4 *>(src + (c + u) * plane);
#pragma unroll
            for (int u = 0; u < 4; ++u) acc += v[u];
        }
        for (; c < chunks; ++c) acc += *reinterpret_cast<const f32x4 *>(src + c * plane);
        float *dst = dbias + (p * L + q) * L + k;
        if (L % 4 == 0) {
            *reinterpret_cast<f32x4 *>(dst) = acc;
        } else {
            for (int i = 0; i < 4 && k + i < L; ++i) dst[i] = acc[i];
        }
    }
}

template <int D, int NKT, int KS>
hipError_t launch_rq_t(const RqArgs &a, hipStream_t s) {
    const unsigned grid = (unsigned)((a.n_units + 7) / 8 * 8);  // XCD-aware order; surplus workgroups exit
    hipLaunchKernelGGL((rows_qbias_kernel<D, NKT, KS>), dim3(grid), dim3(kRqWaves * 64), 0, s, a);
    return hipGetLastError();
}

template <int D>
hipError_t launch_rq_d(const RqArgs &a, int ks, hipStream_t s) {
    const int nkt = (int)((a.L + 31) / 32);
    // (up to 128 keys: the single-pass backward)
    switch (ks) {
        case 1:
            if (nkt <= 5) return launch_rq_t<D, 5, 1>(a, s);
            if (nkt <= 6) return launch_rq_t<D, 6, 1>(a, s);
            if (nkt <= 7) return launch_rq_t<D, 7, 1>(a, s);
            if constexpr (D < 32) return launch_rq_t<D, 8, 1>(a, s);
            return hipErrorInvalidValue;
        case 2:
            if (nkt <= 6) return launch_rq_t<D, 3, 2>(a, s);
            if (nkt <= 8) return launch_rq_t<D, 4, 2>(a, s);
            if (nkt <= 10) return launch_rq_t<D, 5, 2>(a, s);
            if (nkt <= 12) return launch_rq_t<D, 6, 2>(a, s);
            if constexpr (D < 32) return nkt <= 14 ? launch_rq_t<D, 7, 2>(a, s) : launch_rq_t<D, 8, 2>(a, s);
            return hipErrorInvalidValue;
        default:
            if constexpr (D == 32) return launch_rq_t<D, 4, 4>(a, s);
            return hipErrorInvalidValue;
    }
}

}  // namespace

bool rows_qbias_supported(const Problem &p) { return p.dtype == 1 && p.D <= 32 && p.L <= 512; }

int rows_qbias_pitch(const Problem &p) { return (int)((p.L + 3) / 4 * 4); }

int64_t rows_qbias_chunks(const Problem &p, bool has_bias, int64_t waves, int64_t *chunks, int *ks) {
    const int64_t planes = has_bias ? p.N / p.rpb : 1, rpb = has_bias ? p.rpb : p.N;
    const int64_t nqt = (p.L + 31) / 32;
    const int64_t base = planes * p.H * nqt;  // workgroups per row chunk
    // Waves per row: as few as the accumulator registers allow (head_dim 32:
    // 7, 12 and 16 key tiles with 1, 2 and 4; below it 8 and 16 with 1 and 2),
    // or two for up to 8 tiles where that costs less.  Cost of a call: rounds
    // of 256 workgroups (one per CU), each its rows' tile steps plus the
    // prologue and the final sum, worth about six.
    const int k0 = p.D == 32 ? (nqt <= 7 ? 1 : nqt <= 12 ? 2 : 4) : (nqt <= 8 ? 1 : 2);
    int64_t best = -1, bc = 1;
    int bk = k0;
    // (waves: the row chunks that bring the grid to as many, at least one row each)
    int64_t c0 = 1, c1 = rpb < 64 ? rpb : 64;
    if (waves > 0) {
        const int64_t c = (waves + base * kRqWaves - 1) / (base * kRqWaves);
        c0 = c1 = c < rpb ? c : rpb;
    }
    for (int k = k0; k <= (nqt <= 8 ? 2 : k0); k *= 2) {
        for (int64_t c = c0; c <= c1; ++c) {
            const int64_t g = (rpb + c - 1) / c;
            const int64_t rounds = (base * c + 255) / 256, per = (g + kRqWaves / k - 1) / (kRqWaves / k);
            if (best >= 0 && rounds * ((nqt + k - 1) / k + 6) >= best) break;  // (nor can more chunks be cheaper)
            const int64_t cost = rounds * (per * ((nqt + k - 1) / k) + 6);
            if (best < 0 || cost < best) { best = cost; bc = c; bk = k; }
        }
    }
    const int64_t g = (rpb + bc - 1) / bc;
    *chunks = (rpb + g - 1) / g;
    *ks = bk;
    return best;
}

hipError_t launch_rows_qbias(const Problem &p, const BwdPtrs &x, const void *da, const float *dsum, float *part,
                          int64_t chunks, int64_t rows_per_chunk, int ks, hipStream_t s, Tracer &tr) {
    RqArgs a;
    a.q = x.q; a.k = x.k; a.v = x.v; a.bias = x.bias; a.mask = x.mask; a.lse = x.lse;
    a.da = da; a.dsum = dsum; a.dq = x.dq;
    a.dst = !x.bias ? nullptr : chunks > 1 ? part : x.dbias;
    a.L = p.L; a.rpb = x.bias ? p.rpb : p.N; a.srow = p.srow; a.stok = p.stok;
    a.chunks = chunks; a.rows_per_chunk = rows_per_chunk;
    a.H = p.H; a.scale = 1.0f / sqrtf((float)p.D);
    a.pitch = chunks > 1 ? rows_qbias_pitch(p) : (int)p.L;
    const int64_t planes = x.bias ? p.N / p.rpb : 1;
    a.n_units = planes * chunks * ((p.L + 31) / 32) * p.H;
    hipError_t e;
    switch (p.D) {
        case 8: e = launch_rq_d<8>(a, ks, s); break;
        case 16: e = launch_rq_d<16>(a, ks, s); break;
        default: e = launch_rq_d<32>(a, ks, s); break;
    }
    if (e != hipSuccess) return e;
    tr.mark(s);
    if (!x.bias || chunks <= 1) return hipSuccess;
    const unsigned bx = (unsigned)((p.L * (a.pitch / 4) + 255) / 256);
    const int64_t np = planes * p.H;
    hipLaunchKernelGGL(qbias_reduce_kernel, dim3(bx, (unsigned)(np < 8192 ? np : 8192)), dim3(256), 0, s,
                       (const float *)part, x.dbias, np, chunks, (int)p.L, a.pitch);
    e = hipGetLastError();
    if (e == hipSuccess) tr.mark(s);
    return e;
}

}  // namespace evo
