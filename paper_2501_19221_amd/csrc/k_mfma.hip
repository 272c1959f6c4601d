// Dense PA step on the CDNA4 matrix cores with BF16 couplings (App. B field J s + b,
// couplings stored as bf16(J / 2^e), FP32 accumulation, result scaled back by 2^e).
//
// One launch advances every replica by one step.  A workgroup owns an output tile of
// 256 replicas x 64 variables (128 x 128 where the replicas are no multiple of 256, and
// for batch instances) and has 16 waves, four per SIMD:
//   * 8 matrix waves: 64 x 64 sub-tiles, each worked on by two waves that split every
//     chunk's eight k steps between them (steps 0..3 and 4..7),
//     so that every SIMD runs two matrix waves whose instruction streams interleave (one
//     wave alone cannot issue its operand expansion while its matrix ops run); each wave
//     keeps 2 x 2 accumulators of 32 x 32 and the two halves are summed in LDS at the end;
//   * 8 state waves: they load the tile's x and m into registers while the reduction
//     runs, then wait for the field and run the PA update and write x, m and the spins.
// No single resource bounds it.  Counters at n = 4096: a workgroup takes 63.6 thousand clock
// cycles with 256 of them (R = 1024) and 62.5 with 128 (R = 512), so nothing that they share
// slows them; the matrix cores are busy for 32.8 thousand, the rest is the expansion, LDS
// reads and loads that the eight matrix waves do not fully overlap (leaving any one of them
// out saves 6 us of 38.9, the products 17.7).  That a step takes 38.7 us with every compute
// unit busy and 32.2 with half of them is the clock: 11 % fewer cycles a microsecond.
// Fewer bytes per reduction index still pay: spins travel as sign bits (1 bit per variable
// and replica; as pre-expanded words of 4 bits each before), which makes replicas nearly
// free, and a tile of 256 x 64 then needs 160 bytes against 272 for 128 x 128.  sk4096 (n =
// 4096, R = 1024): 38.5 us per step against 42.7 with 4-bit words and 128 x 128 tiles (320
// bytes).
// Chunks are staged through LDS with direct global->LDS loads issued by the matrix waves
// only (NST stages, NST-1 chunks in flight): per chunk the BN x 128 bf16 block of J
// (loads of 16 bytes per lane, each filling 4 rows of 256 bytes) and the sign bits
// of the tile's replicas for those 128 variables (16 bytes per replica, the first BM / 64
// waves one load each).
// Inside a J row the sixteen 16-byte pieces sit at position piece ^ (row % 16), so that the
// fragment reads of 16 consecutive rows fall on distinct banks.  One barrier per
// chunk publishes a stage and frees the one that is loaded next; the state waves take
// part in every barrier and issue no loads in between, so that the matrix waves' waits
// count their own loads only.  After the loop the raw sums go to the state waves
// through LDS, one FP32 buffer per k half (rows padded by 8 floats so that the two
// halves of a wave's stores use different banks), added by the state waves.
//
// Spin bits, chunk-major: for replica r and chunk kc (variables 128 kc .. 128 kc + 127)
// there are 4 u32 words at (kc * Rp + r) * 4; bit j of word w is set where variable
// 128 kc + 32 w + j has spin -1.  The bf16 operand is made from them in registers, two
// full-rate operations per pair of spins (expand_spins).
//
// Matrix instruction: v_mfma_f32_32x32x16_bf16.  Operand layout (64 lanes):
//   A (32 x 16, rows = replicas): lane l holds row l%32, k = 8*(l/32) .. +7
//   B (16 x 32, cols = variables): lane l holds col l%32, k = 8*(l/32) .. +7
//   D (32 x 32): register v of lane l holds row 8*(v/4) + 4*(l/32) + v%4, col l%32.
#include "qpa_internal.h"

#include <algorithm>
#include <type_traits>

namespace qpa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int KC = 128;                      // reduction chunk (variables)
// A BF16 tile shape: replicas, variables and stages.
template <int BM_, int BN_, int NST_> struct BfTile {
    static constexpr int BM = BM_, BN = BN_, NST = NST_;
    static constexpr int JSTG = BN * KC * 2;         // J block of a stage: rows of 256 bytes
    static constexpr int STG = JSTG + BM * 16;       // and 16 bytes of sign bits per replica
    static constexpr int HS = BN + 8;                // row stride of the field handoff (floats)
    static constexpr int LDS = NST * STG > 2 * BM * HS * 4 ? NST * STG : 2 * BM * HS * 4;
    static constexpr int WC = BN / 64;               // 64-column sub-tiles
    static constexpr int JL = BN / 32;               // J loads per matrix wave and chunk
    static constexpr int SL = BM / 64;               // matrix waves that load spins
    static constexpr int RS = 512 / BN;              // row step of a state thread
    static_assert(BM * BN == 128 * 128, "8 matrix waves of 64 x 64, 32 elements per state thread");
    static_assert(LDS <= 160 * 1024, "LDS of one workgroup");
};
typedef BfTile<256, 64, 7> BfWide;
typedef BfTile<128, 128, 4> BfSquare;
// Integer couplings with |J| <= 127 (exact in int8) run on tiles of 64 replicas x 128
// variables (see the int8 section below): J rows of 128 bytes per chunk, spins one byte per
// (replica, variable) (+1 = 0x01, -1 = 0xFF), chunk-major (128 bytes per replica and
// chunk), v_mfma_i32_32x32x32_i8 with exact int32 sums.
constexpr int BM8 = MF_BM8, BN8 = MF_BN8;    // 64 replicas x 128 variables
constexpr int JSTG8 = BN8 * KC;              // 128 rows x 128 bytes
constexpr int SSTG8 = BM8 * KC;              // 64 replicas x 128 bytes
constexpr int STG8 = JSTG8 + SSTG8;
constexpr int NST8 = 3;
constexpr int HS8 = BN8 + 8;                 // row stride of the int8 handoff (int32)
constexpr int SR8 = BM8 / 8;                 // rows of four columns per state thread
constexpr int LDS8_BYTES = NST8 * STG8;
constexpr int MW8 = 4, THREADS8 = 512;       // 4 matrix waves + 4 state waves
static_assert(LDS8_BYTES <= 80 * 1024, "LDS of two workgroups per compute unit");
static_assert(2 * BM8 * HS8 * 4 <= LDS8_BYTES, "the int8 handoff's two partial-sum buffers");
static_assert(BN8 == KC && BN8 / 16 == 2 * MW8, "two row groups of 16 per state wave");
constexpr int THREADS = 1024;                // 8 matrix waves + 8 state waves
constexpr int MW = 8;                        // matrix waves
constexpr int SR = 32;                       // rows per state thread
static_assert(MF_NPAD % KC == 0, "np must be a multiple of the chunk");

__device__ __forceinline__ void pa_update(float h, float lam, float eta, float alpha, float &x,
                                          float &m) {
    float g = __fadd_rn(__fmul_rn(lam, x), h);
    float mn = __fsub_rn(__fmul_rn(alpha, m), __fmul_rn(eta, g));
    float y = __fadd_rn(x, mn);
    y = fminf(1.0f, fmaxf(-1.0f, y));
    m = mn;
    x = y;
}

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// Eight sign bits (the low byte of the low or high half of w) -> eight bf16 +-1 values:
// dword q holds elements 2q (low half) and 2q+1 (high half); a set bit sets the half's
// sign bit on top of 0x3F80 (= 1.0).  One packed 16-bit shift of the same half by 15 - 2q
// and 14 - 2q brings the two bits to the tops of the halves (whatever lies above the byte
// is shifted out); a mask keeps the two sign positions.  Two full-rate operations per dword.
template <int HI>
__device__ __forceinline__ bf16x8 expand_spins(uint32_t w, uint32_t sign_mask) {
    const u16x2 src = __builtin_bit_cast(u16x2, w);
    u32x4 d;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const u16x2 v = (u16x2){src[HI], src[HI]} << (u16x2){(uint16_t)(15 - 2 * q),
                                                             (uint16_t)(14 - 2 * q)};
        // one v_and_or_b32: the mask comes in a VGPR because a VOP3 instruction can read only
        // one scalar operand here.  (Not as inline assembly: the compiler would not see a
        // vector result on its way into a matrix instruction and leave out the wait states
        // between them.)
        const uint32_t r = (__builtin_bit_cast(uint32_t, v) & sign_mask) | 0x3F803F80u;
        d[q] = r;
    }
    return __builtin_bit_cast(bf16x8, d);
}

typedef __attribute__((address_space(3))) void lds_void;

// Workgroup barrier without the memory fence of __syncthreads (which would also wait for
// every load in flight, including the chunks loaded ahead): the callers order their LDS
// traffic with the explicit waits below.
__device__ __forceinline__ void barrier() { asm volatile("s_barrier" ::: "memory"); }

// This wave's loads of all but the N youngest are done and its LDS accesses are complete,
// then the workgroup barrier.
template <int N> __device__ __forceinline__ void wait_barrier() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The tile of a workgroup: replicas from R0 (rows at or past `rlive` are padding:
// their state is neither read nor written and they report +1 spins), variables
// from I0 of an instance with np padded variables and Rp padded replicas.
struct Tile {
    int64_t np, Rp, I0, R0, rlive;
    const uint16_t *Jb;
    const float *b;
    float scale;
    float *x, *m;
    const uint32_t *E = nullptr;     // sparse int8 tiles: entries and block offsets
    const int32_t *O = nullptr;
};

// ---- matrix waves: the reduction of one step, left in LDS as raw sums --------------
// Executes nchunk + 3 workgroup barriers (the state waves execute as many).
template <class TL> struct MatrixStep {
    static __device__ __forceinline__ void run(uint8_t *lds, const Tile &tl, int nchunk,
                                               const uint32_t *__restrict__ s_cur, int wave,
                                               int lane);
};
template <class TL>
__device__ __forceinline__ void MatrixStep<TL>::run(uint8_t *lds, const Tile &tl, int nchunk,
                                                    const uint32_t *__restrict__ s_cur,
                                                    int wave, int lane) {
    constexpr int BM = TL::BM, NST = TL::NST, JL = TL::JL, HS = TL::HS;
    const int64_t np = tl.np, I0 = tl.I0, R0 = tl.R0;
    const uint16_t *__restrict__ Jb = tl.Jb;
    float *hs = reinterpret_cast<float *>(lds);
    const int kh = wave >> 2;                      // k steps 4 kh .. 4 kh + 3 of a chunk
    const int wr = (wave & 3) / TL::WC, wc = (wave & 3) % TL::WC;
    const int half = lane >> 5, l32 = lane & 31;
    // J: load u of wave w fills LDS rows 4 JL w + 4u + lane/16 at position lane % 16,
    // which holds piece (lane % 16) ^ (row % 16) of that row.  Addresses are a
    // wave-uniform base plus 32-bit lane offsets (fewer registers than 64-bit pointers).
    const uint16_t *Jw = Jb + (I0 + 4 * JL * wave) * np;
    uint32_t oJ[JL];
#pragma unroll
    for (int u = 0; u < JL; ++u) {
        const int r = 4 * u + (lane >> 4);         // row - 4 JL w
        oJ[u] = (uint32_t)r * (uint32_t)np +
                8u * (uint32_t)((lane & 15) ^ ((4 * JL * wave + r) & 15));
    }
    // spins: the load of wave w < SL fills the 16 bytes of replicas 64 w + lane (replicas
    // past the padded ones repeat the last)
    const bool loads_s = wave < TL::SL;
    const uint32_t *Sw = s_cur + min(R0 + 64 * wave + lane, tl.Rp - 1) * 4;
    const int64_t sstride = tl.Rp * 4;             // u32 words between consecutive chunks
    auto stage = [&](int kc, int st) {
        kc = kc < nchunk ? kc : nchunk - 1;        // past the end: reload the last chunk
        uint8_t *dst = lds + st * TL::STG;
        const uint16_t *jc = Jw + (int64_t)kc * KC;
#pragma unroll
        for (int u = 0; u < JL; ++u)
            __builtin_amdgcn_global_load_lds(jc + oJ[u],
                                             (lds_void *)(dst + (JL * wave + u) * 1024), 16, 0, 0);
        if (loads_s)
            __builtin_amdgcn_global_load_lds(Sw + (int64_t)kc * sstride,
                                             (lds_void *)(dst + TL::JSTG + 1024 * wave), 16, 0, 0);
    };

    uint32_t sign_mask = 0x80008000u;
    asm volatile("" : "+v"(sign_mask));        // a VGPR whose value the compiler does not know
    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    // J fragments of one k step and this lane's 64 sign bits of a chunk per replica
    // fragment, moved so that the byte of its half is the low byte of each 16 bits
    auto read_j = [&](u32x4 (&bq)[2], int st, int qq) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = 64 * wc + 32 * j + l32;
            const int pos = (2 * (4 * kh + qq) + half) ^ (row & 15);
            bq[j] = *reinterpret_cast<const u32x4 *>(lds + st * TL::STG + row * 256 + pos * 16);
        }
    };
    auto read_s = [&](u32x2 (&sw)[2], int st) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            sw[i] = *reinterpret_cast<const u32x2 *>(lds + st * TL::STG + TL::JSTG +
                                                     16 * (64 * wr + 32 * i + l32) + 8 * kh);
    };
    // The products of a chunk.  The next k step's fragments (the next chunk's first ones and
    // its signs in the last step) are read right after a step's first product, in an order
    // fixed by scheduling barriers: the compiler would read them before their use and wait.
    u32x4 bq[2][2];
    u32x2 sw[2][2];
    auto multiply = [&](int st, int st_next, u32x2 (&s_now)[2], u32x2 (&s_next)[2]) {
        u32x2 w[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) w[i] = s_now[i] >> (u32x2){8u * half, 8u * half};
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const bf16x8 a = qq & 1 ? expand_spins<1>(w[i][qq >> 1], sign_mask)
                                        : expand_spins<0>(w[i][qq >> 1], sign_mask);
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        a, __builtin_bit_cast(bf16x8, bq[qq & 1][j]), acc[i][j], 0, 0, 0);
                    if (i == 0 && j == 0) {
                        __builtin_amdgcn_sched_barrier(0);
                        if (qq < 3) {
                            read_j(bq[(qq + 1) & 1], st, qq + 1);
                        } else {
                            read_j(bq[0], st_next, 0);
                            read_s(s_next, st_next);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
    };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) stage(s, s);
    // chunk 0 has landed in every wave; its first fragments
    if (loads_s) wait_barrier<(NST - 2) * (JL + 1)>();
    else wait_barrier<(NST - 2) * JL>();
    read_j(bq[0], 0, 0);
    read_s(sw[0], 0);
    int st = 0, nx = NST - 1;                      // stages of chunk c and of chunk c + NST - 1
    auto chunk = [&](int c, u32x2 (&s_now)[2], u32x2 (&s_next)[2]) {
        // this wave's loads of chunk c + 1 have landed (the NST-3 younger chunks may not);
        // after the barrier every wave's have, and every wave is done with the stage of
        // chunk c-1, which is refilled next
        if (loads_s) wait_barrier<(NST - 3) * (JL + 1)>();
        else wait_barrier<(NST - 3) * JL>();
        stage(c + NST - 1, nx);
        const int sn = st + 1 == NST ? 0 : st + 1;
        multiply(st, sn, s_now, s_next);
        st = sn;
        nx = nx + 1 == NST ? 0 : nx + 1;
    };
    int c = 0;
    for (; c + 2 <= nchunk; c += 2) {
        chunk(c, sw[0], sw[1]);
        chunk(c + 1, sw[1], sw[0]);
    }
    if (c < nchunk) chunk(c, sw[0], sw[1]);
    wait_barrier<0>();     // the trailing (redundant) loads have landed in every wave and
                           // every stage read is done: the stages can take the sums
    // each k half stores its sums into its own buffer (the state waves add the two, first
    // half + second half), in one pass
    float *hp0 = hs + kh * (BM * HS);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 64 * wr + 32 * i + 8 * (v >> 2) + 4 * half + (v & 3);
                const int col = 64 * wc + 32 * j + l32;
                hp0[row * HS + col] = acc[i][j][v];
            }
    wait_barrier<0>();      // partial sums stored
}

// ---- state waves: thread t (0..511) owns column t % BN of rows RS e + t / BN -----------
// Addresses are the tile's uniform base plus one 32-bit lane offset that steps by rows
// (256 rows of np <= 2^18 floats stay below 2^32 bytes).  Row pointers held in scalar
// registers spilled: 22 scalar operations per row and 3 us more per step.
template <typename P> __device__ __forceinline__ P *next_rows(P *p, int64_t stride) {
    P *q = p + stride;
    asm volatile("" : "+s"(q));
    return q;
}

struct StateRegs {
    float xv[SR], mv[SR];
    float bi;
};

// Loads the tile's x, m and b, spread over the matrix waves' nchunk chunk barriers (a
// few elements before each), so that this traffic shares the memory system with the
// chunk loads instead of delaying the first chunks.  Rows past rlive are padding: they
// are not read and take zeros.  Executes nchunk barriers.  NTL: non-temporal loads
// (the grouped batch step).
template <class TL, bool NTL>
__device__ __forceinline__ void state_load(StateRegs &st, const Tile &tl, int nchunk, int t) {
    constexpr int RS = TL::RS;
    const int col = t & (TL::BN - 1);
    const int rsub = __builtin_amdgcn_readfirstlane(t / TL::BN);
    const int per = (SR + nchunk - 1) / nchunk;
    const char *xb = reinterpret_cast<const char *>(tl.x + tl.R0 * tl.np + tl.I0);
    const char *mb = reinterpret_cast<const char *>(tl.m + tl.R0 * tl.np + tl.I0);
    uint32_t o = 4u * ((uint32_t)rsub * (uint32_t)tl.np + (uint32_t)col);
    const uint32_t step = 4u * RS * (uint32_t)tl.np;
    auto get = [](const char *b, uint32_t off) {
        const float *p = reinterpret_cast<const float *>(b + off);
        return NTL ? __builtin_nontemporal_load(p) : *p;
    };
    int passed = 0, left = per;
    auto rows = [&](auto full) {
#pragma unroll
        for (int e = 0; e < SR; ++e) {
            if (left == 0 && passed < nchunk) {
                barrier();
                ++passed;
                left = per;
            }
            --left;
            // padding rows (uniform per wave) are not read: they start from zero each step
            if (decltype(full)::value || tl.R0 + RS * e + rsub < tl.rlive) {
                st.xv[e] = get(xb, o);
                st.mv[e] = get(mb, o);
            } else {
                st.xv[e] = 0.0f;
                st.mv[e] = 0.0f;
            }
            o += step;
        }
    };
    if (tl.R0 + TL::BM <= tl.rlive) rows(std::true_type{});
    else rows(std::false_type{});
    st.bi = tl.b[tl.I0 + col];
    for (; passed < nchunk; ++passed) barrier();   // the remaining chunks
}

// Waits for the loads of state_load, once, so that later stores wait for nothing.
__device__ __forceinline__ void state_collect(StateRegs &st) {
#pragma unroll
    for (int e = 0; e < SR; ++e) asm volatile("" ::"v"(st.xv[e]), "v"(st.mv[e]));
    asm volatile("" ::"v"(st.bi));
}

// The PA update of the tile from the field sums in LDS, then the new spins as sign bits.
// Rows are taken in groups of 8 with no branch inside the loop (the field reads of a group
// are issued together); lane e keeps the ballot of the wave's row e (64 variables: half a
// chunk), and after the loop lanes 0..31 store them.  With h_last the fields are stored by a
// second pass.  Executes no barrier.
template <class TL>
__device__ __forceinline__ void state_update(StateRegs &st, const Tile &tl, const float *hs,
                                             uint32_t *__restrict__ s_nxt,
                                             float *__restrict__ h_last, int t, int lane,
                                             float lt, float eta, float alpha) {
    constexpr int RS = TL::RS, HS = TL::HS, BM = TL::BM;
    const int col = t & (TL::BN - 1);
    const int rsub = __builtin_amdgcn_readfirstlane(t / TL::BN);
    const int u_mine = lane & 7, g_mine = lane >> 3;
    uint64_t mine = 0;
#pragma unroll
    for (int g = 0; g < SR / 8; ++g) {
        float hv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int k = (RS * (8 * g + u) + rsub) * HS + col;
            hv[u] = hs[k] + hs[BM * HS + k];          // first k half + second k half
        }
        uint64_t bal[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = 8 * g + u;
            const bool live = tl.R0 + RS * e + rsub < tl.rlive;      // uniform per wave
            const float h = __fadd_rn(__fmul_rn(hv[u], tl.scale), st.bi);
            pa_update(h, lt, eta, alpha, st.xv[e], st.mv[e]);
            bal[u] = __ballot(live && st.xv[e] < 0.0f);
        }
        uint64_t mg = bal[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) mg = u_mine == k ? bal[k] : mg;
        mine = g_mine == g ? mg : mine;
    }
    // this wave covers variables v0 .. v0 + 63 (half a chunk: two of its four words)
    const int64_t v0 = tl.I0 + 64 * __builtin_amdgcn_readfirstlane((t & (TL::BN - 1)) >> 6);
    const int64_t r = tl.R0 + RS * lane + rsub;
    if (lane < SR && r < tl.Rp)
        *reinterpret_cast<u32x2 *>(s_nxt + ((v0 / KC) * tl.Rp + r) * 4 + (v0 % KC) / 32) =
            (u32x2){(uint32_t)mine, (uint32_t)(mine >> 32)};
    if (h_last) {
        float *hr = h_last + (tl.R0 + rsub) * tl.np + tl.I0;
#pragma unroll
        for (int e = 0; e < SR; ++e) {
            if (tl.R0 + RS * e + rsub < tl.rlive) {
                const int k = (RS * e + rsub) * HS + col;
                hr[col] = __fadd_rn(__fmul_rn(hs[k] + hs[BM * HS + k], tl.scale), st.bi);
            }
            hr = next_rows(hr, RS * tl.np);
        }
    }
}

// NT: non-temporal stores.  Measured: 1.6 % faster for the single-instance step; for the
// grouped batch step (a batch's state, couplings and spins are more than the caches hold
// between steps) non-temporal stores and loads (NTL in state_load) together 6 % faster.
template <class TL, bool NT>
__device__ __forceinline__ void state_store(const StateRegs &st, const Tile &tl, int t) {
    constexpr int RS = TL::RS;
    const int col = t & (TL::BN - 1);
    const int rsub = __builtin_amdgcn_readfirstlane(t / TL::BN);
    char *xb = reinterpret_cast<char *>(tl.x + tl.R0 * tl.np + tl.I0);
    char *mb = reinterpret_cast<char *>(tl.m + tl.R0 * tl.np + tl.I0);
    uint32_t o = 4u * ((uint32_t)rsub * (uint32_t)tl.np + (uint32_t)col);
    const uint32_t step = 4u * RS * (uint32_t)tl.np;
    auto put = [](char *b, uint32_t off, float v) {
        float *p = reinterpret_cast<float *>(b + off);
        if (NT) __builtin_nontemporal_store(v, p);
        else *p = v;
    };
    auto rows = [&](auto full) {
#pragma unroll
        for (int e = 0; e < SR; ++e) {
            if (decltype(full)::value || tl.R0 + RS * e + rsub < tl.rlive) {
                put(xb, o, st.xv[e]);
                put(mb, o, st.mv[e]);
            }
            o += step;
        }
    };
    if (tl.R0 + TL::BM <= tl.rlive) rows(std::true_type{});
    else rows(std::false_type{});
}

// One PA step of one BF16 tile: matrix and state waves side by side.
template <class TL, bool NT, bool NTL = false>
__device__ __forceinline__ void mfma_tile_step(uint8_t *lds, const Tile &tl,
                                               const uint32_t *__restrict__ s_cur,
                                               uint32_t *__restrict__ s_nxt,
                                               float *__restrict__ h_last, float lt, float eta,
                                               float alpha) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nchunk = (int)(tl.np / KC);
    if (wave >= MW) {
        const int t = tid - MW * 64;
        StateRegs st;
        barrier();                                     // chunk 0 landed
        state_load<TL, NTL>(st, tl, nchunk, t);
        barrier();                                     // stages drained
        barrier();                                     // partial sums stored
        state_collect(st);
        state_update<TL>(st, tl, reinterpret_cast<const float *>(lds), s_nxt, h_last, t, lane, lt,
                         eta, alpha);
        state_store<TL, NT>(st, tl, t);
        return;
    }
    MatrixStep<TL>::run(lds, tl, nchunk, s_cur, wave, lane);
}

// Workgroup k of a launch runs on compute die k mod 8; the tiles go to the dies in
// consecutive runs with the replicas fastest, so that the replica tiles of one block of
// variables, which read the same rows of J, share a die's L2 whatever their number
// (n = 3968, 31 blocks of 128: 37.4 us per step against 51.7 with one block after the other
// round the dies).  False: no tile.
__device__ __forceinline__ bool die_tile(int64_t gx, int64_t gy, int64_t &ix, int64_t &iy) {
    const int64_t pos = (blockIdx.x & 7) * (int64_t)(gridDim.x >> 3) + (blockIdx.x >> 3);
    ix = pos / gy;
    iy = pos - ix * gy;
    return ix < gx;
}
unsigned die_grid(int64_t gx, int64_t gy) { return (unsigned)((gx * gy + 7) / 8 * 8); }

template <class TL>
__global__ void __launch_bounds__(THREADS, 1) k_mfma_step(
    int64_t Rp, int64_t np, int64_t rlive, const uint16_t *__restrict__ Jb,
    const float *__restrict__ b, const CanonScalars *__restrict__ sc,
    const uint32_t *__restrict__ s_cur, uint32_t *__restrict__ s_nxt, float *__restrict__ x,
    float *__restrict__ m, float *__restrict__ h_last, int t, const float *__restrict__ lam,
    float eta, float alpha) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[TL::LDS];
    int64_t ix, iy;
    if (!die_tile(np / TL::BN, (rlive + TL::BM - 1) / TL::BM, ix, iy)) return;
    const Tile tl{np, Rp, ix * TL::BN, iy * TL::BM, rlive, Jb, b, sc->scale, x, m};
    mfma_tile_step<TL, true>(lds, tl, s_cur, s_nxt, h_last, lam[t], eta, alpha);
}

// ---- small tiles: 32 variables x 32 FR replicas -------------------------------------------
// The 128 x 128 tiles leave most compute units idle for smaller instances (n = 1001, R =
// 200: 16 workgroups).  Here a workgroup is two waves, the two k halves of the big tile
// (chunk steps 0..3 and 4..7), each with FR accumulators of 32 x 32 over the whole
// reduction, so that every sum is formed in the big tile's order and its bits are the
// same.  What bounds such a step is the latency of its loads, not their volume: J and
// the sign bits go from global memory straight to registers (a lane's 64 bytes of a J row
// and 8 of its replica's 16 bytes of signs per chunk), D chunks ahead, with no LDS and no
// barrier in the loop.  At the end each wave hands half of its rows' sums to the other and
// updates the other half of the rows.
template <int FR, int D>
__global__ void __launch_bounds__(128, 1) k_mfma_small(
    int64_t Rp, int64_t np, int64_t rlive, const uint16_t *__restrict__ Jb,
    const float *__restrict__ b, const CanonScalars *__restrict__ sc,
    const uint32_t *__restrict__ s_cur, uint32_t *__restrict__ s_nxt, float *__restrict__ x,
    float *__restrict__ m, float *__restrict__ h_last, int t, const float *__restrict__ lam,
    float eta, float alpha) {
    __shared__ float ex[FR][2][8][64];
    const int lane = threadIdx.x & 63, half = lane >> 5, l32 = lane & 31;
    const int kh = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t ix, iy;
    if (!die_tile(np / 32, (rlive + 32 * FR - 1) / (32 * FR), ix, iy)) return;
    const int64_t I0 = ix * 32, R0 = iy * (32 * FR);
    const int nchunk = (int)(np / KC);
    const uint16_t *Jr = Jb + (I0 + l32) * np + 64 * kh + 8 * half;
    const uint32_t *Sr = s_cur + (R0 + l32) * 4 + 2 * kh;
    // rows updated by this wave: sums 8 kh .. 8 kh + 7 of each lane
    auto row = [&](int v) { return 8 * ((8 * kh + v) >> 2) + 4 * half + (v & 3); };
    float xv[FR][8], mv[FR][8];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            const int64_t k = min(R0 + 32 * f + row(v), rlive - 1) * np + I0 + l32;
            xv[f][v] = x[k];
            mv[f][v] = m[k];
        }
    const float bi = b[I0 + l32], lt = lam[t], scale = sc->scale;
    u32x4 jq[D][4];
    u32x2 sq[D][FR];
    auto load = [&](int d, int c) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            jq[d][q] = *reinterpret_cast<const u32x4 *>(Jr + (int64_t)c * KC + 16 * q);
#pragma unroll
        for (int f = 0; f < FR; ++f)
            sq[d][f] = *reinterpret_cast<const u32x2 *>(Sr + ((int64_t)c * Rp + 32 * f) * 4);
    };
    uint32_t sign_mask = 0x80008000u;
    asm volatile("" : "+v"(sign_mask));        // a VGPR whose value the compiler does not know
    f32x16 acc[FR];
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[f][v] = 0.0f;
    auto multiply = [&](int d) {
        u32x2 w[FR];
#pragma unroll
        for (int f = 0; f < FR; ++f) w[f] = sq[d][f] >> (u32x2){8u * half, 8u * half};
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int f = 0; f < FR; ++f)
                acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    q & 1 ? expand_spins<1>(w[f][q >> 1], sign_mask)
                          : expand_spins<0>(w[f][q >> 1], sign_mask),
                    __builtin_bit_cast(bf16x8, jq[d][q]), acc[f], 0, 0, 0);
    };
#pragma unroll
    for (int d = 0; d < D; ++d) load(d, min(d, nchunk - 1));
    int c = 0;
    for (; c + 2 * D <= nchunk; c += D)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            multiply(d);
            load(d, c + D + d);
        }
    // the last D .. 2 D - 1 chunks (all of them where there are fewer)
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (c + d < nchunk) {
            multiply(d);
            if (c + D + d < nchunk) load(d, c + D + d);
        }
    c += D;
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
        if (c + d < nchunk) multiply(d);
#pragma unroll
    for (int f = 0; f < FR; ++f)
#pragma unroll
        for (int v = 0; v < 8; ++v) ex[f][1 - kh][v][lane] = kh ? acc[f][v] : acc[f][8 + v];
    __syncthreads();
#pragma unroll
    for (int f = 0; f < FR; ++f) {
        uint32_t mine = 0;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            // first k half + second k half
            const float own = kh ? acc[f][8 + v] : acc[f][v], other = ex[f][kh][v][lane];
            const int64_t r = R0 + 32 * f + row(v), k = r * np + I0 + l32;
            const bool live = r < rlive;
            const float h = __fadd_rn(__fmul_rn(own + other, scale), bi);
            pa_update(h, lt, eta, alpha, xv[f][v], mv[f][v]);
            if (live) {
                x[k] = xv[f][v];
                m[k] = mv[f][v];
                if (h_last) h_last[k] = h;
            }
            const uint64_t bal = __ballot(live && xv[f][v] < 0.0f);
            mine = lane == v ? (uint32_t)bal : lane == 8 + v ? (uint32_t)(bal >> 32) : mine;
        }
        // lane q < 16: the 32 sign bits of the row of sum q % 8 in lane half q / 8
        if (lane < 16) {
            const int vv = 8 * kh + (lane & 7);
            const int64_t r = R0 + 32 * f + 8 * (vv >> 2) + 4 * (lane >> 3) + (vv & 3);
            s_nxt[((I0 / KC) * Rp + r) * 4 + (I0 % KC) / 32] = mine;
        }
    }
}

// Many instances in one launch: block k runs tile k of the table.  Each tile points at
// its instance's couplings, bias, state and the two spin buffers (picked by step parity).
__global__ void __launch_bounds__(THREADS, 1) k_mfma_grouped(const MfmaTile *__restrict__ tiles,
                                                             int t, const float *__restrict__ lam,
                                                             float eta, float alpha) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[BfSquare::LDS];
    const MfmaTile mt = tiles[blockIdx.x];
    if (mt.np == 0) return;      // filler entry of the compute-die-ordered table
    const uint32_t *cur = (t & 1) ? mt.s1 : mt.s0;
    uint32_t *nxt = (t & 1) ? mt.s0 : mt.s1;
    const Tile tl{mt.np, mt.Rp, mt.I0, mt.R0, mt.rlive, mt.Jb, mt.b, mt.sc->scale, mt.x, mt.m};
    mfma_tile_step<BfSquare, true, true>(lds, tl, cur, nxt, nullptr, lam[t], eta, alpha);
}

// ---- int8 tiles of a batch: 64 replicas x 128 variables ---------------------------------
// For integer couplings with |J| <= 127 a workgroup of 8 waves owns 64 replicas (R0 ..
// R0 + 63) and 128 variables (I0 .. I0 + 127) of an instance; every tile row is a replica
// (with 64 replicas per instance, as in the batch workload, no row is padding).  Two
// workgroups share a compute unit, so that one's state (128 KiB read and written) moves
// while the other multiplies.  Per chunk of 128 reduction variables a stage holds the 128 x
// 128 int8 block of J (rows of 128 bytes, the 16-byte piece p of row r at position
// p ^ (r % 8)) and the 64 x 128 byte spins of the tile's replicas (same layout); NST8 = 3
// stages, 72 KiB.
//   * matrix waves: wave w takes columns 64 (w % 2) .. + 63 and k steps 2 (w / 2),
//     2 (w / 2) + 1 of every chunk (32 each), 2 x 2 accumulators of 32 x 32
//     (v_mfma_i32_32x32x32_i8); they load the spins of every stage (two 1 KiB direct
//     loads each: rows 16w .. 16w + 15) and, for dense rows, the couplings (four: rows
//     32w .. 32w + 31);
//   * state waves: thread t owns columns 4 (t % 32) .. + 3 of rows 8e + t / 32 (8 rows); for
//     entry-list tiles, state wave g also writes the couplings of row groups 2g and 2g + 1
//     (16 rows each) of every stage: it clears their 2 KiB and stores each entry's weight
//     byte at its position (entries of chunk c placed after the barrier of chunk c - 1
//     into the stage of chunk c - 3, loaded three chunks ahead into three register sets
//     used in turn; lanes past a block's end repeat its last entry, the same byte with the
//     same value, so that no load or store sits behind a per-lane branch and each wait
//     for a register set covers that set only).
// After the reduction the two k halves' exact int32 partial sums go through two LDS
// buffers (rows padded to 136 words), added by the state waves, which then run the PA
// update and store x, m and the byte spins of their live rows.  Barriers per tile:
// nchunk + 2 in both roles.
// What bounds it: a tile takes about 11 us for its state and 1.1 us per chunk with two on
// a compute unit; the chunks are mostly LDS time (byte writes of the entries, reads of the
// products).  512 ER QUBOs of 100 to 2000 variables (p = 0.1), 64 replicas: 205 us a step
// against 240 with one workgroup of 64 x 256 (padding to 256) and single-word state
// accesses; 1024 of 508 variables: 127 against 159.
// The table's pointers are generic; these views make the offsets scalar loads (uniform,
// read-only during the launch) and the entries global loads, which count on the
// vector-memory counter only (generic loads also count on the counter that the LDS
// barriers wait for).
typedef __attribute__((address_space(4))) const int32_t c_i32;
typedef __attribute__((address_space(1))) const uint32_t g_u32;
typedef __attribute__((address_space(1))) const float g_f32;
typedef __attribute__((address_space(1))) float g_f32w;
typedef __attribute__((address_space(1))) uint8_t g_u8w;

// The LDS stores of this wave are complete, then the workgroup barrier.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <bool SPARSE>
__device__ __forceinline__ void matrix_tile8(uint8_t *lds, const Tile &tl, int nchunk,
                                             const uint8_t *__restrict__ s_cur, int wave,
                                             int lane) {
    const int64_t np = tl.np;
    const int kh = wave >> 1, wc = wave & 1;
    const int half = lane >> 5, l32 = lane & 31;
    // wave-uniform bases plus 32-bit lane offsets (fewer registers than 64-bit pointers):
    // load u of the couplings fills rows 32w + 8u + lane / 8, that of the spins rows
    // 16w + 8u + lane / 8, each at position lane % 8 (piece (lane % 8) ^ (row % 8))
    const uint8_t *Jw = reinterpret_cast<const uint8_t *>(tl.Jb) + (tl.I0 + 32 * wave) * np;
    const uint8_t *Sw = s_cur + (tl.R0 + 16 * wave) * KC;
    const int r8 = lane >> 3;
    const uint32_t piece = (uint32_t)((lane & 7) ^ r8);
    uint32_t oJ[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) oJ[u] = (uint32_t)(8 * u + r8) * (uint32_t)np + 16u * piece;
    const uint32_t oS = (uint32_t)r8 * (uint32_t)KC + 16u * piece;
    const int64_t sstride = tl.Rp * KC;            // bytes between consecutive spin chunks
    auto stage = [&](int kc, int st) {
        kc = kc < nchunk ? kc : nchunk - 1;        // past the end: reload the last chunk
        uint8_t *dst = lds + st * STG8;
        if (!SPARSE) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
                __builtin_amdgcn_global_load_lds(Jw + (int64_t)kc * KC + oJ[u],
                                                 (lds_void *)(dst + (4 * wave + u) * 1024), 16, 0,
                                                 0);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            __builtin_amdgcn_global_load_lds(Sw + (int64_t)kc * sstride + 8 * u * KC + oS,
                                             (lds_void *)(dst + JSTG8 + (2 * wave + u) * 1024),
                                             16, 0, 0);
    };
    constexpr int LOADS = SPARSE ? 2 : 6;          // per chunk and wave
    i32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0;
#pragma unroll
    for (int s = 0; s < NST8 - 1; ++s) stage(s, s);
    for (int c = 0; c < nchunk; ++c) {
        // this wave's loads of chunk c have landed (NST8 - 2 younger chunks may not)
        wait_barrier<(NST8 - 2) * LOADS>();
        stage(c + NST8 - 1, (c + NST8 - 1) % NST8);
        const uint8_t *src = lds + (c % NST8) * STG8;
#pragma unroll
        for (int qq = 0; qq < 2; ++qq) {
            const int pc = 2 * (2 * kh + qq) + half;
            i32x4 a[2], bq[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int row = 32 * i + l32;
                a[i] = *reinterpret_cast<const i32x4 *>(src + JSTG8 + row * KC +
                                                        16 * (pc ^ (row & 7)));
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int row = 64 * wc + 32 * j + l32;
                bq[j] = *reinterpret_cast<const i32x4 *>(src + row * KC + 16 * (pc ^ (row & 7)));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], bq[j], acc[i][j], 0,
                                                                      0, 0);
        }
    }
    wait_barrier<0>();     // every load has landed and every stage read is done
    // the two k halves' exact int32 partial sums, one buffer each
    int32_t *hp = reinterpret_cast<int32_t *>(lds) + kh * (BM8 * HS8);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 32 * i + 8 * (v >> 2) + 4 * half + (v & 3);
                const int col = 64 * wc + 32 * j + l32;
                hp[row * HS8 + col] = acc[i][j][v];
            }
    wait_barrier<0>();     // partial sums stored
}

// Entries of one 16 x 128 block (I8S_EPL per lane).
struct EntryRegs {
    uint32_t e[I8S_EPL];
    int32_t cnt;
};

// Row group gg (0..7) of the tile, chunk kc (past the last chunk: the last again).  The
// block belongs to the 128-row tile I0 / 128 of the entry-list layout.
__device__ __forceinline__ void entries_load(EntryRegs &er, const Tile &tl, int kc, int nchunk,
                                             int gg, int lane) {
    kc = kc < nchunk ? kc : nchunk - 1;
    const int64_t blk = (tl.I0 / KC * (tl.np / KC) + kc) * 8 + gg;
    const c_i32 *O = (const c_i32 *)tl.O;
    const int32_t beg = O[blk];
    er.cnt = O[blk + 1] - beg;
    // an empty block reads the word at its start, which lies inside the coupling buffer
    // (the entries end at least a quarter of the buffer before its end); it is not placed
    // (ordinary loads: the cache holds part of the lists from one step to the next, as the
    // state, far more than it holds, goes past it)
    const g_u32 *src = (const g_u32 *)tl.E + beg;
    const int32_t last = max(er.cnt - 1, 0);
#pragma unroll
    for (int j = 0; j < I8S_EPL; ++j)
        er.e[j] = src[min(lane + 64 * j, last)];
}

// Clears row group gg's 2 KiB of the stage and writes its entries there.  An entry's
// position within its 16 rows is its low 11 bits (the rows of its block); the words an
// empty block loaded write zeros into cleared bytes of the same rows.
__device__ __forceinline__ void entries_place(const EntryRegs &er, uint8_t *stage, int gg,
                                              int lane) {
    uint8_t *rg = stage + 2048 * gg;
    *reinterpret_cast<u32x4 *>(rg + 16 * lane) = (u32x4){0u, 0u, 0u, 0u};
    *reinterpret_cast<u32x4 *>(rg + 1024 + 16 * lane) = (u32x4){0u, 0u, 0u, 0u};
    const uint32_t keep = er.cnt > 0 ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int j = 0; j < I8S_EPL; ++j)
        rg[er.e[j] & 0x7FFu] = (uint8_t)((er.e[j] & keep) >> 16);
}

// The two row groups (2g, 2g + 1) of a state wave.
struct EntryPair {
    EntryRegs a, b;
};

__device__ __forceinline__ void pair_load(EntryPair &p, const Tile &tl, int kc, int nchunk,
                                          int g, int lane) {
    entries_load(p.a, tl, kc, nchunk, 2 * g, lane);
    entries_load(p.b, tl, kc, nchunk, 2 * g + 1, lane);
}

__device__ __forceinline__ void pair_place(const EntryPair &p, uint8_t *stage, int g, int lane) {
    entries_place(p.a, stage, 2 * g, lane);
    entries_place(p.b, stage, 2 * g + 1, lane);
}

typedef float st4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) const st4 g_st4;
typedef __attribute__((address_space(1))) st4 g_st4w;
typedef __attribute__((address_space(1))) uint32_t g_u32w;

// State thread t: columns 4 (t % 32) .. + 3 of rows 8e + t / 32.
struct StateRegs8 {
    st4 xv[SR8], mv[SR8];
    st4 bi;
};

// x, m of rows 8e + t / 32, E0 <= e < E1, of this thread (eight rows at or past rlive are
// not read; others past it read the last live row again, unused).  The state of a batch
// step (all instances', with the couplings and spins far more than the caches hold between
// steps) is read and written non-temporally.
template <int E0, int E1>
__device__ __forceinline__ void xm_load8(StateRegs8 &st, const Tile &tl, int t) {
    const int col = 4 * (t & 31), rsub = t >> 5;
    const int64_t left = tl.rlive - tl.R0;             // live rows from the tile's first on
#pragma unroll
    for (int e = E0; e < E1; ++e) {
        st.xv[e] = st.mv[e] = 0.0f;
        if (8 * e < left) {
            const int row = 8 * e + rsub < left ? 8 * e + rsub : (int)left - 1;
            const int64_t o = (tl.R0 + row) * tl.np + tl.I0 + col;
            st.xv[e] = __builtin_nontemporal_load((const g_st4 *)((const g_f32 *)tl.x + o));
            st.mv[e] = __builtin_nontemporal_load((const g_st4 *)((const g_f32 *)tl.m + o));
        }
    }
}

// One chunk barrier of a placing state wave: then the entries held in p (chunk c + 1) go
// into the stage of chunk c - 2 (free since the barrier of chunk c - 1) and p is reloaded
// with the chunk three further on.  Past the last chunk the reloaded last chunk is placed
// again, into a stage that no later chunk of the loop uses (they take those of c at
// most); the barrier after the loop waits for these stores.  No branch, so that the waits
// for one register set cover that set only.
__device__ __forceinline__ void place_step(EntryPair &p, const Tile &tl, int c, int nchunk,
                                           uint8_t *lds, int g, int lane) {
    lds_barrier();
    const int kc = c + NST8 - 2;
    pair_place(p, lds + (kc % NST8) * STG8, g, lane);
    pair_load(p, tl, kc + 3, nchunk, g, lane);
}

// State waves of an int8 tile, up to the partial sums: x, m and b loaded, and for
// entry-list tiles the couplings of every chunk placed.  Executes nchunk barriers.
template <bool SPARSE>
__device__ __forceinline__ void state_load8(StateRegs8 &st, const Tile &tl, int nchunk, int t,
                                            uint8_t *lds, int g, int lane) {
    static_assert(SR8 == 8 && NST8 == 3, "the load pattern below");
    const g_st4 *bias = (const g_st4 *)((const g_f32 *)tl.b + tl.I0 + 4 * (t & 31));
    if (!SPARSE) {
        xm_load8<0, SR8>(st, tl, t);
        st.bi = *bias;
        for (int c = 0; c < nchunk; ++c) barrier();
        return;
    }
    // the prologue's chunk, and the next three chunks' entries; x and m follow in three
    // groups after the first three chunks' entry loads, since loads complete in issue order
    // and a wait for entries would otherwise wait for them
    EntryPair p0, p1, p2;
    pair_load(p2, tl, 0, nchunk, g, lane);
    pair_load(p0, tl, 1, nchunk, g, lane);
    pair_load(p1, tl, 2, nchunk, g, lane);
    pair_place(p2, lds, g, lane);
    pair_load(p2, tl, 3, nchunk, g, lane);
    if (nchunk > 0) place_step(p0, tl, 0, nchunk, lds, g, lane);
    xm_load8<0, 3>(st, tl, t);
    if (nchunk > 1) place_step(p1, tl, 1, nchunk, lds, g, lane);
    xm_load8<3, 6>(st, tl, t);
    if (nchunk > 2) place_step(p2, tl, 2, nchunk, lds, g, lane);
    xm_load8<6, 8>(st, tl, t);
    st.bi = *bias;
    int c = 3;
    for (; c + 3 <= nchunk; c += 3) {
        place_step(p0, tl, c, nchunk, lds, g, lane);
        place_step(p1, tl, c + 1, nchunk, lds, g, lane);
        place_step(p2, tl, c + 2, nchunk, lds, g, lane);
    }
    if (c < nchunk) place_step(p0, tl, c, nchunk, lds, g, lane);
    if (c + 1 < nchunk) place_step(p1, tl, c + 1, nchunk, lds, g, lane);
}

// One PA step of one int8 tile.
template <bool SPARSE>
__device__ __forceinline__ void tile8_step(uint8_t *lds, const Tile &tl,
                                           const uint8_t *__restrict__ s_cur,
                                           uint8_t *__restrict__ s_nxt, float lt, float eta,
                                           float alpha) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nchunk = (int)(tl.np / KC);
    if (wave < MW8) {
        matrix_tile8<SPARSE>(lds, tl, nchunk, s_cur, wave, lane);
        return;
    }
    const int t = tid - MW8 * 64;
    const int col = 4 * (t & 31), rsub = t >> 5;
    StateRegs8 st;
    state_load8<SPARSE>(st, tl, nchunk, t, lds, wave - MW8, lane);
    lds_barrier();                                     // stages drained (and written)
    barrier();                                         // partial sums stored
#pragma unroll
    for (int e = 0; e < SR8; ++e) asm volatile("" ::"v"(st.xv[e]), "v"(st.mv[e]));
    asm volatile("" ::"v"(st.bi));
    // field = sum of the two k halves' int32 partials (exact), unscaled; rows at or past
    // rlive are not updated and their spins not written
    const int32_t *h0 = reinterpret_cast<const int32_t *>(lds), *h1 = h0 + BM8 * HS8;
    const int64_t left = tl.rlive - tl.R0;
    // spins as bytes: row r of chunk I0 / 128 at (chunk * Rp + r) * 128 + col
    g_u8w *srow = (g_u8w *)s_nxt + (tl.I0 / KC * tl.Rp + tl.R0) * KC + col;
#pragma unroll
    for (int e = 0; e < SR8; ++e) {
        const int row = 8 * e + rsub;
        if (8 * e >= left) break;
        const int k = row * HS8 + col;
        const i32x4 ha = *reinterpret_cast<const i32x4 *>(h0 + k);
        const i32x4 hb = *reinterpret_cast<const i32x4 *>(h1 + k);
        uint32_t spins = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float h = __fadd_rn((float)(ha[u] + hb[u]), st.bi[u]);
            float xk = st.xv[e][u], mk = st.mv[e][u];
            pa_update(h, lt, eta, alpha, xk, mk);
            st.xv[e][u] = xk;
            st.mv[e][u] = mk;
            spins |= (xk < 0.0f ? 0xFFu : 0x01u) << (8 * u);
        }
        if (row < left) {
            const int64_t o = (tl.R0 + row) * tl.np + tl.I0 + col;
            __builtin_nontemporal_store(st.xv[e], (g_st4w *)((g_f32w *)tl.x + o));
            __builtin_nontemporal_store(st.mv[e], (g_st4w *)((g_f32w *)tl.m + o));
            *(g_u32w *)(srow + row * KC) = spins;
        }
    }
}

// Many int8 instances in one launch (tiles as above).
template <bool SPARSE>
__global__ void __launch_bounds__(THREADS8) __attribute__((amdgpu_waves_per_eu(4)))
    k_mfma_grouped8(const MfmaTile *__restrict__ tiles, int t, const float *__restrict__ lam,
                    float eta, float alpha) {
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS8_BYTES];
    const MfmaTile mt = tiles[blockIdx.x];
    if (mt.np == 0) return;      // filler entry of the compute-die-ordered table
    const uint8_t *cur = reinterpret_cast<const uint8_t *>((t & 1) ? mt.s1 : mt.s0);
    uint8_t *nxt = reinterpret_cast<uint8_t *>((t & 1) ? mt.s0 : mt.s1);
    const Tile tl{mt.np, mt.Rp, mt.I0, mt.R0, mt.rlive, mt.Jb, mt.b, 1.0f, mt.x, mt.m,
                  mt.E, mt.O};
    tile8_step<SPARSE>(lds, tl, cur, nxt, lam[t], eta, alpha);
}

// Byte spins of the signs of x (chunk-major, 128 bytes per replica and chunk).
__global__ void __launch_bounds__(256) k_mfma_pack_i8(int64_t Rp, int64_t np,
                                                      const float *__restrict__ x,
                                                      uint8_t *__restrict__ s8) {
    const int64_t total = Rp * np;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t kc = k / (Rp * KC), rem = k - kc * Rp * KC;
        const int64_t r = rem / KC, j = rem - r * KC;
        s8[k] = x[r * np + KC * kc + j] < 0.0f ? (uint8_t)0xFF : (uint8_t)0x01;
    }
}

// Sign bits of x (layout above): one thread per word.
__global__ void __launch_bounds__(256) k_mfma_pack(int64_t Rp, int64_t np,
                                                   const float *__restrict__ x,
                                                   uint32_t *__restrict__ sw) {
    const int64_t total = Rp * (np / 32);
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < total;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int64_t kc = k / (Rp * 4), rem = k - kc * Rp * 4;
        const int64_t r = rem / 4, wd = rem - r * 4;
        const float4 *xr = reinterpret_cast<const float4 *>(x + r * np + KC * kc + 32 * wd);
        uint32_t bits = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float4 v = xr[j];
            bits |= (v.x < 0.0f ? 1u : 0u) << (4 * j) | (v.y < 0.0f ? 2u : 0u) << (4 * j) |
                    (v.z < 0.0f ? 4u : 0u) << (4 * j) | (v.w < 0.0f ? 8u : 0u) << (4 * j);
        }
        sw[k] = bits;
    }
}

// ---- sparse int8 tiles: entry lists of the 16 x 128 blocks of J8 ------------------------
// One wave per block: lane l covers row 16 g + l / 4 of the row tile, columns
// 32 (l % 4) .. 32 (l % 4) + 31 of the chunk.
__device__ __forceinline__ void i8s_block(const I8sTask &tk, int64_t blk, int lane,
                                          const int8_t *&src, int &row, int &k0) {
    const int64_t nch = tk.np / KC;
    const int64_t ib = blk / (nch * 8), kc = (blk / 8) % nch, g = blk % 8;
    row = 16 * (int)g + (lane >> 2);
    k0 = 32 * (lane & 3);
    src = tk.J8 + (ib * KC + row) * tk.np + kc * KC + k0;
}

__device__ __forceinline__ int nonzero_bytes(uint32_t v) {
    int c = 0;
#pragma unroll
    for (int b = 0; b < 4; ++b) c += ((v >> (8 * b)) & 0xFFu) != 0u;
    return c;
}

__global__ void __launch_bounds__(256) k_i8s_count(const I8sTask *__restrict__ tasks) {
    const I8sTask tk = tasks[blockIdx.y];
    const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (blk >= i8s_blocks(tk.np)) return;                 // whole waves leave together
    const int8_t *src;
    int row, k0;
    i8s_block(tk, blk, lane, src, row, k0);
    const u32x4 v0 = *reinterpret_cast<const u32x4 *>(src);
    const u32x4 v1 = *reinterpret_cast<const u32x4 *>(src + 16);
    int c = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) c += nonzero_bytes(v0[q]) + nonzero_bytes(v1[q]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
    if (lane == 0) tk.cnt[blk] = c;
}

// Counts -> exclusive offsets in place (nblk + 1 values, the last the total), and the
// largest block and the total into stats.  One workgroup per task.
__global__ void __launch_bounds__(1024) k_i8s_scan(const I8sTask *__restrict__ tasks) {
    __shared__ int32_t part[1024], mx[1024];
    const I8sTask tk = tasks[blockIdx.x];
    const int64_t nblk = i8s_blocks(tk.np);
    const int t = threadIdx.x;
    const int64_t per = (nblk + 1023) / 1024;
    const int64_t a = std::min<int64_t>(nblk, t * per), b = std::min<int64_t>(nblk, a + per);
    int32_t s = 0, m = 0;
    for (int64_t i = a; i < b; ++i) {
        s += tk.cnt[i];
        m = max(m, tk.cnt[i]);
    }
    part[t] = s;
    mx[t] = m;
    __syncthreads();
    if (t == 0) {                 // 1024 partial sums in order: exact and deterministic
        int32_t run = 0, mm = 0;
        for (int i = 0; i < 1024; ++i) {
            const int32_t v = part[i];
            part[i] = run;
            run += v;
            mm = max(mm, mx[i]);
        }
        tk.stats[0] = mm;
        tk.stats[1] = run;
        tk.cnt[nblk] = run;
    }
    __syncthreads();
    int32_t run = part[t];
    for (int64_t i = a; i < b; ++i) {
        const int32_t v = tk.cnt[i];
        tk.cnt[i] = run;
        run += v;
    }
}

// The entries of every block (tasks whose largest block exceeds I8S_BLOCK_MAX keep their
// dense rows and are skipped).  Within a block the entries follow (row, column) order.
__global__ void __launch_bounds__(256) k_i8s_fill(const I8sTask *__restrict__ tasks) {
    const I8sTask tk = tasks[blockIdx.y];
    const int64_t blk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (blk >= i8s_blocks(tk.np) || tk.stats[0] > I8S_BLOCK_MAX) return;
    const int8_t *src;
    int row, k0;
    i8s_block(tk, blk, lane, src, row, k0);
    const u32x4 v0 = *reinterpret_cast<const u32x4 *>(src);
    const u32x4 v1 = *reinterpret_cast<const u32x4 *>(src + 16);
    int c = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) c += nonzero_bytes(v0[q]) + nonzero_bytes(v1[q]);
    int incl = c;                                     // inclusive prefix over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    uint32_t *dst = tk.E + tk.cnt[blk] + (incl - c);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const uint32_t v = q < 4 ? v0[q] : v1[q - 4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const uint32_t w = (v >> (8 * b)) & 0xFFu;
            if (w != 0u) {
                const int k = k0 + 4 * q + b;
                const uint32_t pos = (uint32_t)(row * KC + 16 * ((k >> 4) ^ (row & 7)) + (k & 15));
                *dst++ = (w << 16) | pos;
            }
        }
    }
}

}  // namespace

hipError_t launch_i8s_count(const I8sTask *tasks, int32_t ntask, int64_t max_np,
                            hipStream_t st) {
    if (ntask <= 0) return hipSuccess;
    const int64_t bx = (i8s_blocks(max_np) + 3) / 4;
    if (bx <= 0 || bx > INT32_MAX || ntask > 65535) return hipErrorInvalidValue;
    k_i8s_count<<<dim3((unsigned)bx, (unsigned)ntask), 256, 0, st>>>(tasks);
    return hipGetLastError();
}

hipError_t launch_i8s_scan(const I8sTask *tasks, int32_t ntask, hipStream_t st) {
    if (ntask <= 0) return hipSuccess;
    k_i8s_scan<<<(unsigned)ntask, 1024, 0, st>>>(tasks);
    return hipGetLastError();
}

hipError_t launch_i8s_fill(const I8sTask *tasks, int32_t ntask, int64_t max_np,
                           hipStream_t st) {
    if (ntask <= 0) return hipSuccess;
    const int64_t bx = (i8s_blocks(max_np) + 3) / 4;
    if (bx <= 0 || bx > INT32_MAX || ntask > 65535) return hipErrorInvalidValue;
    k_i8s_fill<<<dim3((unsigned)bx, (unsigned)ntask), 256, 0, st>>>(tasks);
    return hipGetLastError();
}

hipError_t launch_mfma_pack_spins(int64_t Rp, int64_t np, const float *x, uint32_t *sbits,
                                  hipStream_t st) {
    int64_t total = Rp * (np / 32);
    int64_t g = (total + 255) / 256;
    if (g > 65536) g = 65536;
    k_mfma_pack<<<(unsigned)g, 256, 0, st>>>(Rp, np, x, sbits);
    return hipGetLastError();
}

namespace {
template <class TL> unsigned wide_grid(int64_t np, int64_t rlive) {
    return die_grid(np / TL::BN, (rlive + TL::BM - 1) / TL::BM);
}

// Replicas (in 32s) of the small tiles an instance runs on, 0: the 16384-element tiles.  The
// tile with the least estimated step: a fixed part plus, per chunk of 128 variables, the
// time of the workgroups that share a compute unit, plus the state of those past the second,
// which no longer overlaps.  The estimates are off by up to 30 % (the 16384-element tiles at
// n = 4096, R = 1024: 28.6 for 38.5 us), all to the same side where it is close: over 276 sizes
// (n = 100 to 6000, R = 1 to 16384) the tile taken is within 9 % of the fastest, 0.2 % on
// average.  Without the last part it was up to 2.1 times the fastest where there are many
// more replicas than variables.  Measured, us per step:
//   n     R     32 x 32   32 x 64   32 x 128   16384-element
//   256   256     5.6       7.1       9.2         8.3
//   1001  200     6.1       8.4      11.7        12.8
//   1001  1024   12.7      11.4      12.9        13.5
//   2048  256    12.4      10.7      15.3        18.3
//   2048  1024   38.8      27.9      20.7        20.1
//   4096  128    20.5      15.5      21.1        31.0
//   4096  256    35.3      23.7      22.3        28.4
//   4096  512    69.7      45.0      30.8        29.5
//   300   4096   21.1      18.6      13.0        11.1
//   768   2048   20.3      19.9      14.5        13.2
int small_tile_replicas(int64_t np, int64_t Rp, int64_t rlive) {
    const double nc = (double)(np / KC);
    auto rounds = [](int64_t tiles) { return (double)((tiles + 255) / 256); };
    double best = 7.5 + 0.66 * nc *
                  rounds(Rp % 256 == 0 ? (np / 64) * (Rp / 256) : (np / 128) * (Rp / 128));
    int fr = 0;
    const double fixed[3] = {4.2, 5.7, 9.0}, chunk[3] = {0.26, 0.30, 0.40};
    const double state[3] = {2.0, 4.0, 2.0};
    for (int k = 0; k < 3; ++k) {
        const int64_t br = 32 << k;
        const double r = rounds((np / 32) * ((rlive + br - 1) / br));
        const double t = fixed[k] + chunk[k] * nc * r + state[k] * std::max(0.0, r - 2.0);
        if (t < best) {
            best = t;
            fr = 1 << k;
        }
    }
    return fr;
}
}  // namespace

hipError_t launch_mfma_step(int64_t Rp, int64_t np, int64_t rlive, const uint16_t *Jb,
                            const float *b, const CanonScalars *sc, const uint32_t *s_cur,
                            uint32_t *s_nxt, float *x, float *m, float *h_last, int32_t t,
                            const float *lam, float eta, float alpha, hipStream_t st) {
    if (Rp % MF_BM || np % MF_NPAD || np <= 0 || rlive < 1 || rlive > Rp)
        return hipErrorInvalidValue;
    const int fr = small_tile_replicas(np, Rp, rlive);
    const unsigned gs = die_grid(np / 32, (rlive + 32 * fr - 1) / (32 * std::max(fr, 1)));
#define QPA_BF(KERNEL, GRID, N)                                                             \
    KERNEL<<<GRID, N, 0, st>>>(Rp, np, rlive, Jb, b, sc, s_cur, s_nxt, x, m, h_last, t, lam, \
                               eta, alpha)
    if (fr == 1) QPA_BF((k_mfma_small<1, 8>), gs, 128);
    else if (fr == 2) QPA_BF((k_mfma_small<2, 8>), gs, 128);
    else if (fr == 4) QPA_BF((k_mfma_small<4, 6>), gs, 128);
    else if (Rp % 256 == 0) QPA_BF(k_mfma_step<BfWide>, wide_grid<BfWide>(np, rlive), THREADS);
    else QPA_BF(k_mfma_step<BfSquare>, wide_grid<BfSquare>(np, rlive), THREADS);
#undef QPA_BF
    return hipGetLastError();
}

hipError_t launch_mfma_grouped(const MfmaTile *tiles, int32_t ntiles, int32_t t,
                               const float *lam, float eta, float alpha, GroupKind kind,
                               hipStream_t st) {
    if (ntiles <= 0) return hipSuccess;
    if (kind == GK_I8_SPARSE)
        k_mfma_grouped8<true><<<(unsigned)ntiles, THREADS8, 0, st>>>(tiles, t, lam, eta, alpha);
    else if (kind == GK_I8)
        k_mfma_grouped8<false><<<(unsigned)ntiles, THREADS8, 0, st>>>(tiles, t, lam, eta, alpha);
    else
        k_mfma_grouped<<<(unsigned)ntiles, THREADS, 0, st>>>(tiles, t, lam, eta, alpha);
    return hipGetLastError();
}

hipError_t launch_mfma_pack_spins_i8(int64_t Rp, int64_t np, const float *x, uint8_t *s8,
                                     hipStream_t st) {
    int64_t g = (Rp * np + 255) / 256;
    if (g > 65536) g = 65536;
    k_mfma_pack_i8<<<(unsigned)g, 256, 0, st>>>(Rp, np, x, s8);
    return hipGetLastError();
}

// Dense int8 copy of a CSR instance (integer weights with |w| <= 127, checked by the
// caller): J8[i][j] = w_ij for the stored off-diagonal entries, zero elsewhere (the caller
// clears J8 first).  One wave per row.
template <typename TW, typename TI>
__global__ void __launch_bounds__(256) k_csr_to_i8(int64_t n, int64_t np,
                                                   const int32_t *__restrict__ rp,
                                                   const TI *__restrict__ col,
                                                   const TW *__restrict__ w,
                                                   int8_t *__restrict__ J8) {
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    for (int64_t k = rp[i] + lane; k < rp[i + 1]; k += 64) {
        const int64_t j = (int64_t)col[k];
        if (j == i) continue;
        J8[i * np + j] = (int8_t)w[k];
    }
}

// The same matrix written whole, one workgroup per row (rows n .. np-1 zero): the row is
// cleared and its entries placed in LDS, then stored in 16-byte pieces, so that the
// matrix needs no separate clear.  np is a multiple of 128 and at most ROWS8_MAX_NP.
constexpr int64_t ROWS8_MAX_NP = 65536;

template <typename TW, typename TI>
__device__ __forceinline__ void csr_to_i8_row(int64_t i, int64_t n, int64_t np,
                                              const int32_t *__restrict__ rp,
                                              const TI *__restrict__ col,
                                              const TW *__restrict__ w,
                                              int8_t *__restrict__ J8) {
    extern __shared__ uint4 row16[];              // np bytes
    int8_t *row = reinterpret_cast<int8_t *>(row16);
    const int64_t np16 = np / 16;
    for (int64_t q = threadIdx.x; q < np16; q += blockDim.x) row16[q] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (i < n) {
        for (int64_t k = rp[i] + threadIdx.x; k < rp[i + 1]; k += blockDim.x) {
            const int64_t j = (int64_t)col[k];
            if (j != i) row[j] = (int8_t)w[k];
        }
    }
    __syncthreads();
    uint4 *dst = reinterpret_cast<uint4 *>(J8 + i * np);
    for (int64_t q = threadIdx.x; q < np16; q += blockDim.x) dst[q] = row16[q];
}

template <typename TW, typename TI>
__global__ void __launch_bounds__(256) k_csr_to_i8_rows(int64_t n, int64_t np,
                                                        const int32_t *__restrict__ rp,
                                                        const TI *__restrict__ col,
                                                        const TW *__restrict__ w,
                                                        int8_t *__restrict__ J8) {
    csr_to_i8_row<TW, TI>(blockIdx.x, n, np, rp, col, w, J8);
}

// Batched: row blockIdx.x of instance blockIdx.y (rows past the instance's np return).
template <typename TW, typename TI>
__global__ void __launch_bounds__(256) k_csr_to_i8_rows_batch(const SlotInitTask *__restrict__ tasks) {
    const SlotInitTask &t = tasks[blockIdx.y];
    if ((int64_t)blockIdx.x >= t.np) return;
    csr_to_i8_row<TW, TI>(blockIdx.x, t.n, t.np, t.rp, static_cast<const TI *>(t.col),
                          static_cast<const TW *>(t.w), t.J8);
}

hipError_t launch_csr_to_i8_batch(const SlotInitTask *tasks, int32_t ntask, qpa_dtype coupling,
                                  qpa_dtype index, int64_t max_np, hipStream_t st) {
    if (max_np < MF_NPAD || max_np % MF_NPAD || max_np > ROWS8_MAX_NP)
        return hipErrorInvalidValue;
    auto run = [&](auto wtag, auto itag) {
        using TW = decltype(wtag);
        using TI = decltype(itag);
        for (int32_t c0 = 0; c0 < ntask; c0 += 65535) {
            const dim3 g((unsigned)max_np, (unsigned)std::min(65535, ntask - c0));
            k_csr_to_i8_rows_batch<TW, TI><<<g, 256, (size_t)max_np, st>>>(tasks + c0);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    };
    auto byw = [&](auto itag) -> hipError_t {
        switch (coupling) {
            case QPA_I8: return run((int8_t)0, itag);
            case QPA_I16: return run((int16_t)0, itag);
            case QPA_I32: return run((int32_t)0, itag);
            default: return hipErrorInvalidValue;
        }
    };
    return index == QPA_I16 ? byw((int16_t)0) : byw((int32_t)0);
}

hipError_t launch_csr_to_i8(const qpa_problem &p, int64_t np, int8_t *J8, hipStream_t st) {
    const bool rows = np % 128 == 0 && np >= p.n && np <= ROWS8_MAX_NP;
    if (!rows) {
        const hipError_t e = hipMemsetAsync(J8, 0, (size_t)(np * np), st);
        if (e != hipSuccess) return e;
    }
    const int64_t g = (p.n + 3) / 4;
    auto run = [&](auto wtag, auto itag) {
        using TW = decltype(wtag);
        using TI = decltype(itag);
        if (rows)
            k_csr_to_i8_rows<TW, TI><<<(unsigned)np, 256, (size_t)np, st>>>(
                p.n, np, p.row_ptr, static_cast<const TI *>(p.col),
                static_cast<const TW *>(p.weights), J8);
        else
            k_csr_to_i8<TW, TI><<<(unsigned)g, 256, 0, st>>>(
                p.n, np, p.row_ptr, static_cast<const TI *>(p.col),
                static_cast<const TW *>(p.weights), J8);
        return hipGetLastError();
    };
    auto byw = [&](auto itag) -> hipError_t {
        switch (p.coupling_dtype) {
            case QPA_I8: return run((int8_t)0, itag);
            case QPA_I16: return run((int16_t)0, itag);
            case QPA_I32: return run((int32_t)0, itag);
            default: return hipErrorInvalidValue;
        }
    };
    return p.index_dtype == QPA_I16 ? byw((int16_t)0) : byw((int32_t)0);
}


// Dense BF16 copy of a CSR instance: Jb[i][j] = bf16(w_ij * 2^-e) for the stored
// off-diagonal entries (zero elsewhere; the caller clears Jb first).  One wave per row,
// the row's entries split over the lanes.
template <typename TW, typename TI>
__global__ void __launch_bounds__(256) k_csr_to_bf16(int64_t n, int64_t np,
                                                     const int32_t *__restrict__ rp,
                                                     const TI *__restrict__ col,
                                                     const TW *__restrict__ w,
                                                     const CanonScalars *__restrict__ sc,
                                                     uint16_t *__restrict__ Jb) {
    const float inv = sc->inv_scale;
    const int lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    for (int64_t k = rp[i] + lane; k < rp[i + 1]; k += 64) {
        const int64_t j = (int64_t)col[k];
        if (j == i) continue;
        uint32_t u = __float_as_uint(__fmul_rn((float)w[k], inv));
        u += 0x7fffu + ((u >> 16) & 1u);
        Jb[i * np + j] = (uint16_t)(u >> 16);
    }
}

hipError_t launch_csr_to_bf16(const qpa_problem &p, int64_t np, const CanonScalars *sc,
                              uint16_t *Jb, hipStream_t st) {
    hipError_t e = hipMemsetAsync(Jb, 0, sizeof(uint16_t) * (size_t)(np * np), st);
    if (e != hipSuccess) return e;
    const int64_t g = (p.n + 3) / 4;
    auto run = [&](auto wtag, auto itag) {
        using TW = decltype(wtag);
        using TI = decltype(itag);
        k_csr_to_bf16<TW, TI><<<(unsigned)g, 256, 0, st>>>(
            p.n, np, p.row_ptr, static_cast<const TI *>(p.col),
            static_cast<const TW *>(p.weights), sc, Jb);
        return hipGetLastError();
    };
    auto byw = [&](auto itag) -> hipError_t {
        switch (p.coupling_dtype) {
            case QPA_I8: return run((int8_t)0, itag);
            case QPA_I16: return run((int16_t)0, itag);
            case QPA_I32: return run((int32_t)0, itag);
            default: return run(0.0f, itag);
        }
    };
    return p.index_dtype == QPA_I16 ? byw((int16_t)0) : byw((int32_t)0);
}

}  // namespace qpa
