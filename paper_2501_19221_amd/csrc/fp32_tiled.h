// FP32 product on the matrix cores, shared by the SBM step, the PA FP32 dense step and the
// relaxed-dynamics adjoint:  G = J Q  with J [n][dense_ld(n)] symmetric (row k of J is column
// k; rows padded to 16 bytes) and Q [n][Rp] (replica fastest, Rp a multiple of 32),
// followed by an element-wise epilogue.
//
// Every sum must be the sequential chain of fused multiply-adds in ascending k (the
// definition of the FP32 fields).  v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32 give
// exactly that chain: each of their k terms is one fused multiply-add, ascending, denormals
// and signed zeros kept (checked against fmaf on 5e4 sums of 256 terms).  So a product may
// be cut into output tiles freely, but never along k.
//
// What bounds it: the FP32 matrix rate (157 TFLOP/s nominal, 147 measured with 32 x 32
// tiles in registers; the vector units reach 78.6 without packed FP32) for large n and R,
// and the chain itself (8 cycles per k and wave) where there are few outputs.  At n = 4096,
// R = 1024 a step takes 254 us (135 TFLOP/s) against 637 us for the product on the vector
// units (8 x 8 sums per thread); at n = 512, R = 256 6.8 us against 87 us, where
// the vector product's 128 x 128 tiles left 248 of 256 compute units idle.  About 4 us of
// a small step are the launch, the first chunk's latency and the state.
//
// A workgroup owns a tile of BI variables x BR replicas; wave (wi, wr) owns FI x FR
// matrix tiles of MT x MT.  A = J (rows: variables), B = Q (columns: replicas), so that a
// wave's loads and stores of [n][Rp] state are contiguous in replicas.  Chunks of KC
// reduction indices of J and Q go to LDS by direct global->LDS loads (rows stay
// contiguous, fragment reads of 16 or 32 consecutive floats are free of bank conflicts),
// NST stages, NST - 1 chunks ahead, one fence-free barrier per chunk.  Rows past n
// repeat row n - 1, columns past the edge repeat the last ones; the products of the rows
// are replaced by -0.0 * +0.0 = -0.0, the identity of the sum, and the columns' sums are
// never stored.
#pragma once

#include "qpa_internal.h"

#include <type_traits>

namespace qpa {
namespace {

typedef float ft_f16 __attribute__((ext_vector_type(16)));
typedef float ft_f4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void ft_lds_void;

template <int BI_, int BR_, int MT_, int FI_, int FR_, int KC_, int NST_, int GS_> struct FpTile {
    static constexpr int BI = BI_, BR = BR_, MT = MT_, FI = FI_, FR = FR_, KC = KC_, NST = NST_;
    static constexpr int GS = GS_;
    static constexpr int WI = BI / (MT * FI), WR = BR / (MT * FR), WAVES = WI * WR;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int KS = 64 / MT;             // reduction indices per instruction
    static constexpr int NV = MT * MT / 64;        // sums per lane and matrix tile
    static constexpr int STG = KC * (BI + BR);     // floats per stage
    static_assert(KC * BI % (256 * WAVES) == 0 && KC * BR % (256 * WAVES) == 0, "even loads");
    static_assert(NST * STG * 4 <= 160 * 1024, "LDS of one workgroup");
};

// The tiles, largest first.  One CU does 256 multiply-adds per cycle and four matrix
// instructions at a time, so a tile costs BI * BR / 128 cycles per k when it is alone on its CU and
// tiles of a CU add up.
typedef FpTile<128, 128, 32, 2, 1, 32, 4, 4> FpTileL;    // 8 waves
typedef FpTile<64, 64, 32, 1, 1, 32, 4, 4> FpTileM;      // 4 waves
typedef FpTile<64, 32, 16, 2, 1, 32, 6, 4> FpTileN;      // 4 waves
typedef FpTile<32, 32, 16, 1, 1, 64, 5, 4> FpTileS;      // 4 waves

// Workgroup barrier without a memory fence, after this wave's loads of all but the N
// youngest have landed and its LDS reads are done.
template <int N> __device__ __forceinline__ void ft_wait_barrier() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

template <int MT> struct FtAcc;
template <> struct FtAcc<32> { typedef ft_f16 type; };
template <> struct FtAcc<16> { typedef ft_f4 type; };

__device__ __forceinline__ ft_f16 ft_mfma(float a, float b, ft_f16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ ft_f4 ft_mfma(float a, float b, ft_f4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Epi: typedef Pre and
//   float bias(i)                            b_i
//   void begin()                             uniform values, read while the first chunks load
//   Pre load(r, idx)                         the element's own state, loaded before the loop
//   void point(acc, bias, r, idx, Pre)       its update from the sum
//   void finish()                            once per thread, after its elements
template <class TL, class Epi>
__global__ void __launch_bounds__(TL::THREADS) k_fp32_mfma_step(int64_t n, int64_t Rp,
                                                                const float *__restrict__ J,
                                                                const float *__restrict__ qi,
                                                                Epi epi) {
    constexpr int BI = TL::BI, BR = TL::BR, MT = TL::MT, FI = TL::FI, FR = TL::FR, KC = TL::KC;
    constexpr int NST = TL::NST, KS = TL::KS, NV = TL::NV;
    constexpr int LJ = KC * BI / (256 * TL::WAVES);                   // loads per wave and chunk
    constexpr int LQ = KC * BR / (256 * TL::WAVES);
    static_assert((NST - 2) * (LJ + LQ) < 64, "vmcnt range");
    __shared__ __attribute__((aligned(16))) float lds[NST * TL::STG];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i0 = (int64_t)blockIdx.x * BI, r0 = (int64_t)blockIdx.y * BR;

    // load u of this wave covers floats 256 (u WAVES + wave) .. of the stage's J (or Q)
    // rows: row jr + u * JSTEP of the chunk at column jc
    const int jr = (256 * wave + 4 * lane) / BI, jc = (4 * lane) % BI;
    const int qr = (256 * wave + 4 * lane) / BR, qc = (4 * lane) % BR;
    constexpr int JSTEP = 256 * TL::WAVES / BI, QSTEP = 256 * TL::WAVES / BR;
    static_assert(256 * TL::WAVES % BI == 0 && 256 * TL::WAVES % BR == 0, "whole rows");
    // the MT-column blocks of row k sit at block ^ (row of k within an instruction), as far
    // as there are blocks, so that the KS rows of a fragment read fall on distinct banks
    // (the steps between a lane's loads are whole instructions, so its block is fixed)
    static_assert(JSTEP % KS == 0 && QSTEP % KS == 0, "a lane's rows share their swizzle");
    constexpr int SWJ = (BI / MT < KS ? BI / MT : KS) - 1, SWQ = (BR / MT < KS ? BR / MT : KS) - 1;
    auto swz = [](int k, int mask) { return ((KS / (mask + 1) > 1 ? k / (KS / (mask + 1)) : k) & mask) * MT; };
    const int64_t ldj = dense_ld(n);
    const uint32_t jcol = (uint32_t)min(i0 + (jc ^ swz(jr % KS, SWJ)), ldj - 4);
    const uint32_t ldj32 = (uint32_t)ldj;
    const int64_t qcol = min(r0 + (qc ^ swz(qr % KS, SWQ)), Rp - 4);
    const int nch = (int)((n + KC - 1) / KC);
    // load u of a chunk (u < LJ: J, then Q); the last chunk's rows past n repeat row n - 1,
    // and past the end the last chunk is loaded again, unused
    uint32_t oj[2][LJ];
    int64_t oq[2][LQ];
    const int lim = (int)(n - 1 - (int64_t)(nch - 1) * KC);
#pragma unroll
    for (int u = 0; u < LJ; ++u) {
        oj[0][u] = (uint32_t)(jr + u * JSTEP) * ldj32 + jcol;
        oj[1][u] = (uint32_t)min(jr + u * JSTEP, lim) * ldj32 + jcol;
    }
#pragma unroll
    for (int u = 0; u < LQ; ++u) {
        oq[0][u] = (qr + u * QSTEP) * Rp + qcol;
        oq[1][u] = min(qr + u * QSTEP, lim) * Rp + qcol;
    }
    auto load = [&](int c, int st, int u) {
        float *dst = lds + st * TL::STG;
        const bool last = c >= nch - 1;                            // uniform
        const int64_t k0 = (int64_t)(last ? nch - 1 : c) * KC;
        if (u < LJ) {
            const uint32_t o = last ? oj[1][u] : oj[0][u];
            __builtin_amdgcn_global_load_lds(
                J + k0 * ldj + o, (ft_lds_void *)(dst + 256 * (u * TL::WAVES + wave)), 16, 0, 0);
        } else {
            u -= LJ;
            const int64_t o = last ? oq[1][u] : oq[0][u];
            __builtin_amdgcn_global_load_lds(
                qi + k0 * Rp + o, (ft_lds_void *)(dst + KC * BI + 256 * (u * TL::WAVES + wave)),
                16, 0, 0);
        }
    };

    // element v of matrix tile (f, g): variable ib + MT f + vrow(v), replica rb + MT g
    const int lk = lane / MT, lm = lane % MT;
    const int wi = wave % TL::WI, wr = wave / TL::WI;
    const int64_t ib = i0 + wi * (MT * FI) + 4 * lk, rb = r0 + wr * (MT * FR) + lm;
    auto vrow = [](int v) { return MT == 32 ? 8 * (v >> 2) + (v & 3) : v; };
    const bool full = i0 + BI <= n && r0 + BR <= Rp;           // uniform
    typename FtAcc<MT>::type acc[FI][FR];
    typename Epi::Pre pre[FI][FR][NV];
    float bi[FI][NV];
    auto load_bias = [&]() {
#pragma unroll
        for (int f = 0; f < FI; ++f)
#pragma unroll
            for (int v = 0; v < NV; ++v) bi[f][v] = epi.bias(min(ib + MT * f + vrow(v), n - 1));
    };
    constexpr bool EARLY = FI * NV <= 16;                      // registers to hold the bias
    if (EARLY) load_bias();
#pragma unroll
    for (int f = 0; f < FI; ++f)
#pragma unroll
        for (int g = 0; g < FR; ++g)
#pragma unroll
            for (int v = 0; v < NV; ++v) acc[f][g][v] = 0.0f;
    if (full) {
        const int64_t base = ib * Rp + rb;
#pragma unroll
        for (int f = 0; f < FI; ++f)
#pragma unroll
            for (int g = 0; g < FR; ++g)
#pragma unroll
                for (int v = 0; v < NV; ++v)
                    pre[f][g][v] = epi.load(rb + MT * g, base + (MT * f + vrow(v)) * Rp + MT * g);
    } else {
#pragma unroll
        for (int f = 0; f < FI; ++f)
#pragma unroll
            for (int g = 0; g < FR; ++g)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int64_t i = min(ib + MT * f + vrow(v), n - 1);
                    const int64_t r = min(rb + MT * g, Rp - 1);
                    pre[f][g][v] = epi.load(r, i * Rp + r);
                }
    }
#pragma unroll
    for (int s = 0; s < NST - 1; ++s)
#pragma unroll
        for (int u = 0; u < LJ + LQ; ++u) load(s, s, u);
    epi.begin();

    // Fragments are read a group ahead of their products (GS reduction steps of one
    // instruction each), across chunk borders, right after the first products of the group
    // before: the compiler waits for every outstanding read at a group's first product, so
    // the next group's come after it.  The order is fixed by scheduling barriers; left
    // alone, the compiler reads each fragment right before its use.
    constexpr int GS = TL::GS, NG = KC / (KS * GS);
    static_assert(NG * KS * GS == KC && NG % 2 == 0, "fragment sets alternate");
    float fa[2][GS][FI], fb[2][GS][FR];
    int aofs[FI], bofs[FR];
#pragma unroll
    for (int f = 0; f < FI; ++f) aofs[f] = (MT * (wi * FI + f)) ^ swz(lk, SWJ);
#pragma unroll
    for (int h = 0; h < FR; ++h) bofs[h] = (MT * (wr * FR + h)) ^ swz(lk, SWQ);
    auto read = [&](int st, int g, int e0, int e1, float (&ra)[GS][FI], float (&rb_)[GS][FR]) {
        const float *As = lds + st * TL::STG + lm + lk * BI;
        const float *Bs = lds + st * TL::STG + KC * BI + lm + lk * BR;
#pragma unroll
        for (int e = e0; e < e1; ++e) {
            const int kk = (g * GS + e) * KS;
#pragma unroll
            for (int f = 0; f < FI; ++f) ra[e][f] = As[kk * BI + aofs[f]];
#pragma unroll
            for (int h = 0; h < FR; ++h) rb_[e][h] = Bs[kk * BR + bofs[h]];
        }
    };
    // the products of a chunk; after them the reads of the next group, then (not in the
    // last chunk) the loads of chunk cl into its stage, a few after each product
    constexpr int SLOTS = NG * (GS / 2), LPS = (LJ + LQ + SLOTS - 1) / SLOTS;
    auto multiply = [&](int st, int st_next, auto tail, int kend, int cl, int stl) {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
#pragma unroll
            for (int e = 0; e < GS; ++e) {
                float(&a)[FI] = fa[g & 1][e];
                float(&b)[FR] = fb[g & 1][e];
                if constexpr (decltype(tail)::value) {
                    const bool in = (g * GS + e) * KS + lk < kend;
#pragma unroll
                    for (int f = 0; f < FI; ++f) a[f] = in ? a[f] : -0.0f;
#pragma unroll
                    for (int h = 0; h < FR; ++h) b[h] = in ? b[h] : 0.0f;
                }
#pragma unroll
                for (int f = 0; f < FI; ++f)
#pragma unroll
                    for (int h = 0; h < FR; ++h) acc[f][h] = ft_mfma(a[f], b[h], acc[f][h]);
                if (2 * e < GS) {
                    __builtin_amdgcn_sched_barrier(0);
                    if (g + 1 < NG)
                        read(st, g + 1, 2 * e, 2 * e + 2, fa[(g + 1) & 1], fb[(g + 1) & 1]);
                    else if constexpr (!decltype(tail)::value)
                        read(st_next, 0, 2 * e, 2 * e + 2, fa[0], fb[0]);
                    __builtin_amdgcn_sched_barrier(0);
                } else if constexpr (!decltype(tail)::value) {
#pragma unroll
                    for (int q = 0; q < LPS; ++q) {
                        const int u = (g * (GS / 2) + e - GS / 2) * LPS + q;
                        if (u < LJ + LQ) load(cl, stl, u);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // chunk 0 has landed in every wave; its first fragments
    ft_wait_barrier<(NST - 2) * (LJ + LQ)>();
    read(0, 0, 0, GS, fa[0], fb[0]);
    int st = 0, nx = NST - 1;                      // stages of chunk c and of chunk c + NST - 1
    for (int c = 0; c < nch - 1; ++c) {
        // this wave's loads of chunk c + 1 have landed (younger chunks' may not have); after
        // the barrier every wave's have, and every wave is done with the stage refilled next
        ft_wait_barrier<(NST - 3) * (LJ + LQ)>();
        const int sn = st + 1 == NST ? 0 : st + 1;
        multiply(st, sn, std::false_type{}, KC, c + NST - 1, nx);
        st = sn;
        nx = nx + 1 == NST ? 0 : nx + 1;
    }
    ft_wait_barrier<0>();              // no load is left in flight when the LDS is given back
    multiply(st, st, std::true_type{}, (int)(n - (int64_t)(nch - 1) * KC), 0, 0);
    if (!EARLY) load_bias();
    if (full) {
        const int64_t base = ib * Rp + rb;
#pragma unroll
        for (int f = 0; f < FI; ++f)
#pragma unroll
            for (int g = 0; g < FR; ++g)
#pragma unroll
                for (int v = 0; v < NV; ++v)
                    epi.point(acc[f][g][v], bi[f][v], rb + MT * g,
                              base + (MT * f + vrow(v)) * Rp + MT * g, pre[f][g][v]);
    } else {
#pragma unroll
        for (int f = 0; f < FI; ++f)
#pragma unroll
            for (int g = 0; g < FR; ++g)
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int64_t i = ib + MT * f + vrow(v), r = rb + MT * g;
                    if (i < n && r < Rp) epi.point(acc[f][g][v], bi[f][v], r, i * Rp + r, pre[f][g][v]);
                }
    }
    epi.finish();
}

enum Fp32Tile : int { FP32_TILE_L, FP32_TILE_M, FP32_TILE_N, FP32_TILE_S };

// The tile for an n x Rp product: the one whose workgroups, spread over the compute
// units, finish first; among equals the largest (least traffic).  An element of the smaller
// tiles takes longer where they fill the chip: n = 4096, R = 4096 1014, 1078, 1242 and
// 1298 us a step.  Counted alike, the smallest was taken for n = 209, R = 65536 (143 us, 109
// with the largest) and n = 1500, R = 8192 (461 and 311).
inline Fp32Tile fp32_tile_of(int64_t n, int64_t Rp) {
    auto cost = [&](int64_t bi, int64_t br, double element) {
        const int64_t tiles = ((n + bi - 1) / bi) * ((Rp + br - 1) / br);
        return (double)((tiles + 255) / 256 * (bi * br)) * element;
    };
    if (Rp > 32 * 65535) return FP32_TILE_L;        // grid y
    const double l = cost(128, 128, 1.0), m = cost(64, 64, 1.06), nn = cost(64, 32, 1.22),
                 s = cost(32, 32, 1.28);
    if (l <= m && l <= nn && l <= s) return FP32_TILE_L;
    if (m <= nn && m <= s) return FP32_TILE_M;
    return nn <= s ? FP32_TILE_N : FP32_TILE_S;
}

inline dim3 fp32_tile_grid(Fp32Tile t, int64_t n, int64_t Rp) {
    const int64_t bi = t == FP32_TILE_L ? 128 : t == FP32_TILE_S ? 32 : 64;
    const int64_t br = t == FP32_TILE_L ? 128 : t == FP32_TILE_M ? 64 : 32;
    return dim3((unsigned)((n + bi - 1) / bi), (unsigned)((Rp + br - 1) / br));
}

template <class Epi>
hipError_t launch_fp32_product(int64_t n, int64_t Rp, const float *J, const float *q,
                               const Epi &epi, hipStream_t st) {
    if (Rp % 32 || Rp < 32 || n < 1) return hipErrorInvalidValue;
    const Fp32Tile t = fp32_tile_of(n, Rp);
    const dim3 grid = fp32_tile_grid(t, n, Rp);
    if (grid.y > 65535u) return hipErrorInvalidValue;
#define QPA_FP32_TILE(T, TL)                                                               \
    if (t == T) k_fp32_mfma_step<TL, Epi><<<grid, TL::THREADS, 0, st>>>(n, Rp, J, q, epi);
    QPA_FP32_TILE(FP32_TILE_L, FpTileL)
    QPA_FP32_TILE(FP32_TILE_M, FpTileM)
    QPA_FP32_TILE(FP32_TILE_N, FpTileN)
    QPA_FP32_TILE(FP32_TILE_S, FpTileS)
#undef QPA_FP32_TILE
    return hipGetLastError();
}

}  // namespace
}  // namespace qpa
