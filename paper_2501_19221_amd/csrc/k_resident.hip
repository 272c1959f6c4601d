// Sparse PA steps (App. B) with the whole state on chip: one launch runs every step.
//
// A workgroup owns G replicas (G in {1, 2, 4, 8}) and every variable of the instance.
// Thread t owns variables t, t + 1024, ... (VPT of them) for its workgroup's G replicas,
// and keeps their x and m in registers for all steps.  The instance's CSR structure is
// copied once into LDS (row pointers int32, columns uint16, weights int32 or FP32), next
// to two byte arrays of spins: byte j holds in bit g the sign of variable j in replica g
// of the workgroup (bit set <=> spin -1).  A step is, for every owned variable, a walk of
// its row -- one spin byte serves all G replicas -- followed by the fused update and one
// byte store; a workgroup barrier separates the steps.  The first CACHE off-diagonal
// entries of each owned row (CACHE = min(8, 16 / VPT)) are held in registers, so that a
// step issues their spin-byte reads together; longer rows continue from LDS in order.  Nothing is written to
// memory until the last step, when x and m go back to the workspace state ([n][Rp],
// replica fastest) and, if asked, the last field.
// The field sums follow the entry order of the row: int32 (exact; rows are validated
// below 2^24) for integer couplings, FP32 for float couplings, as in the streamed kernel.
// Integer rows whose sum of |w| stays below 2^16 (SW) take a packed form instead: with
// b' = b XOR [w < 0] a term is w (1 - 2b) = |w| (1 - 2b'), so the field is
// sum |w| - 2 A with A = sum |w| b' < 2^16.  The A of two replicas share one 32-bit word
// (16-bit lanes), summed modulo 2^32 as a row constant sum_{w<0} |w| (1 + 2^16) plus, per
// entry, w times the spread spin bits (bit of the first replica at 0, second at 16, from
// a 256-entry LDS table indexed by the spin byte): one signed 24-bit multiply-add per
// entry and replica pair.  The total is A_0 + 2^16 A_1 exactly, whatever the signs of the
// partial sums.  The cached entries are padded with zero weights, so the integer walk has
// no per-entry branch.
// This form, with one bit per spin, needs the least LDS and the fewest registers.  Rows whose
// sum of |w| stays below 2^8 (such as +-1 graphs) can take k_csr_resident8, four replicas a
// word, and all can take k_csr_residentf, spins as floats: the rule stands at res_form.
#include "qpa_internal.h"

#include <type_traits>

namespace qpa {
namespace {

constexpr int RT = 1024;                 // threads per workgroup

__device__ __forceinline__ void pa_update(float h, float lam, float eta, float alpha, float &x,
                                          float &m) {
    float g = __fadd_rn(__fmul_rn(lam, x), h);
    float mn = __fsub_rn(__fmul_rn(alpha, m), __fmul_rn(eta, g));
    float y = __fadd_rn(x, mn);
    y = fminf(1.0f, fmaxf(-1.0f, y));
    m = mn;
    x = y;
}

template <typename T> __device__ __forceinline__ T ld_as(const void *p, int32_t dt, int64_t k) {
    switch (dt) {
        case QPA_I8: return (T) static_cast<const int8_t *>(p)[k];
        case QPA_I16: return (T) static_cast<const int16_t *>(p)[k];
        case QPA_I32: return (T) static_cast<const int32_t *>(p)[k];
        default: return (T) static_cast<const float *>(p)[k];
    }
}

// Spread words of spin byte b (NP of them) from the LDS table.
template <int NP>
__device__ __forceinline__ void lut_read(const uint32_t *lut, uint32_t b, uint32_t (&sp)[NP]) {
    if constexpr (NP == 4) {
        const uint4 v = reinterpret_cast<const uint4 *>(lut)[b];
        sp[0] = v.x; sp[1] = v.y; sp[2] = v.z; sp[3] = v.w;
    } else if constexpr (NP == 2) {
        const uint2 v = reinterpret_cast<const uint2 *>(lut)[b];
        sp[0] = v.x; sp[1] = v.y;
    } else {
        sp[0] = lut[b];
    }
}

constexpr size_t RES_LUT_BYTES = 256 * 4 * sizeof(uint32_t);

// LDS: spread table [256][4] uint32 | rp [n+1] int32 | w [nnz] int32 or float |
//      col [nnz] uint16 | spins [2][n] bytes
template <int G, int VPT, bool INT, bool SW>
__global__ void __launch_bounds__(RT) k_csr_resident(
    int32_t n, int32_t nnz, int64_t R, int64_t Rp, const int32_t *__restrict__ rp_g,
    const void *__restrict__ col_g, int32_t col_dt, const void *__restrict__ w_g, int32_t w_dt,
    int32_t skip_diag, const float *__restrict__ b, float *__restrict__ x,
    float *__restrict__ m, float *__restrict__ h_last, int32_t t0, int32_t t1,
    const float *__restrict__ lam, float eta, float alpha) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint32_t *lut = reinterpret_cast<uint32_t *>(lds);
    int32_t *rp = reinterpret_cast<int32_t *>(lds + RES_LUT_BYTES);
    int32_t *wi = rp + (n + 1);
    float *wf = reinterpret_cast<float *>(wi);
    uint16_t *col = reinterpret_cast<uint16_t *>(wi + nnz);
    uint8_t *sp0 = reinterpret_cast<uint8_t *>(col + nnz);
    uint8_t *sp1 = sp0 + n;
    const int tid = threadIdx.x;
    const int64_t r0 = (int64_t)blockIdx.x * G;

    constexpr int NP = (G + 1) / 2;     // replica pairs, one 32-bit word each (SW)
    if (SW)
        for (int e = tid; e < 256 * NP; e += RT) {
            const uint32_t byte = (uint32_t)(e / NP), p = (uint32_t)(e % NP);
            lut[e] = ((byte >> (2 * p)) & 1u) | (((byte >> (2 * p + 1)) & 1u) << 16);
        }
    for (int32_t k = tid; k <= n; k += RT) rp[k] = rp_g[k];
    for (int32_t k = tid; k < nnz; k += RT) {
        col[k] = (uint16_t)(col_dt == QPA_I16 ? (int32_t) static_cast<const int16_t *>(col_g)[k]
                                              : static_cast<const int32_t *>(col_g)[k]);
        if (INT) wi[k] = ld_as<int32_t>(w_g, w_dt, k);
        else wf[k] = ld_as<float>(w_g, w_dt, k);
    }

    constexpr int CACHE = (16 / VPT) < 8 ? (16 / VPT) : 8;
    // cached entries of each owned row (diagonal entries of a QUBO left out), then the
    // LDS position where the rest of the row continues
    int32_t cj[VPT][CACHE];
    int32_t cwi[VPT][CACHE];
    float cwf[VPT][CACHE];
    int32_t ccount[VPT], crest[VPT];
    int32_t wabs[VPT];            // SW: sum of |w| over the row (diagonal excluded)
    uint32_t cneg[VPT];           // SW: sum over w < 0 of |w| (1 + 2^16), modulo 2^32
    float xs[VPT][G], ms[VPT][G], bi[VPT];
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * RT;
        uint32_t byte = 0;
        bi[u] = 0.0f;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            xs[u][g] = 0.0f;
            ms[u][g] = 0.0f;
        }
        if (i < n) {
            bi[u] = b[i];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (r0 + g < R) {
                    xs[u][g] = x[(int64_t)i * Rp + r0 + g];
                    ms[u][g] = m[(int64_t)i * Rp + r0 + g];
                }
                byte |= (xs[u][g] < 0.0f ? 1u : 0u) << g;
            }
            sp0[i] = (uint8_t)byte;
        }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * RT;
        int32_t cnt = 0, k = 0, k1 = 0;
        if (i < n) {
            k = rp[i];
            k1 = rp[i + 1];
        }
#pragma unroll
        for (int c = 0; c < CACHE; ++c) {
            cj[u][c] = 0;
            cwi[u][c] = 0;
            cwf[u][c] = 0.0f;
        }
        wabs[u] = 0;
        cneg[u] = 0u;
        if (SW)
            for (int32_t kk = k; kk < k1; ++kk)
                if (!(skip_diag && col[kk] == i)) {
                    const int32_t a = wi[kk] < 0 ? -wi[kk] : wi[kk];
                    wabs[u] += a;
                    if (wi[kk] < 0) cneg[u] += (uint32_t)a * 0x10001u;
                }
        // take entries in row order until CACHE of them are held
        for (; k < k1 && cnt < CACHE; ++k) {
            const int32_t j = col[k];
            if (skip_diag && j == i) continue;
#pragma unroll
            for (int c = 0; c < CACHE; ++c)
                if (c == cnt) {
                    cj[u][c] = j;
                    if (INT) {
                        cwi[u][c] = wi[k];
                    } else {
                        cwf[u][c] = wf[k];
                    }
                }
            ++cnt;
        }
        ccount[u] = cnt;
        crest[u] = k;
    }

    uint8_t *cur = sp0, *nxt = sp1;
    for (int32_t t = t0; t < t1; ++t) {
        const float lt = lam[t];
        const bool last = (t == t1 - 1);
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int32_t i = tid + u * RT;
            if (i >= n) continue;
            int32_t ai[G];
            float af[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                ai[g] = 0;
                af[g] = 0.0f;
            }
            if (SW) {
                uint32_t acc[NP];
#pragma unroll
                for (int p = 0; p < NP; ++p) acc[p] = cneg[u];
                uint32_t cb[CACHE];
#pragma unroll
                for (int c = 0; c < CACHE; ++c) cb[c] = cur[cj[u][c]];
#pragma unroll
                for (int c = 0; c < CACHE; ++c) {
                    uint32_t sp[NP];
                    lut_read<NP>(lut, cb[c], sp);
#pragma unroll
                    for (int p = 0; p < NP; ++p)
                        acc[p] += (uint32_t)__mul24(cwi[u][c], (int32_t)sp[p]);
                }
                const int32_t k1 = rp[i + 1];
                for (int32_t k = crest[u]; k < k1; ++k) {
                    const int32_t j = col[k];
                    if (skip_diag && j == i) continue;
                    uint32_t sp[NP];
                    lut_read<NP>(lut, cur[j], sp);
#pragma unroll
                    for (int p = 0; p < NP; ++p) acc[p] += (uint32_t)__mul24(wi[k], (int32_t)sp[p]);
                }
#pragma unroll
                for (int g = 0; g < G; ++g)
                    ai[g] = wabs[u] - 2 * (int32_t)((acc[g >> 1] >> (16 * (g & 1))) & 0xffffu);
            } else {
            // cached entries: their spin bytes are read together, then summed in order
            uint32_t cb[CACHE];
#pragma unroll
            for (int c = 0; c < CACHE; ++c) cb[c] = c < ccount[u] ? cur[cj[u][c]] : 0u;
#pragma unroll
            for (int c = 0; c < CACHE; ++c) {
                if (c < ccount[u]) {
                    if (INT) {
                        const int32_t wk = cwi[u][c];
#pragma unroll
                        for (int g = 0; g < G; ++g) ai[g] += ((cb[c] >> g) & 1u) ? -wk : wk;
                    } else {
                        const float wk = cwf[u][c];
#pragma unroll
                        for (int g = 0; g < G; ++g)
                            af[g] = __fadd_rn(af[g], ((cb[c] >> g) & 1u) ? -wk : wk);
                    }
                }
            }
            const int32_t k1 = rp[i + 1];
            for (int32_t k = crest[u]; k < k1; ++k) {
                const int32_t j = col[k];
                if (skip_diag && j == i) continue;
                const uint32_t byte = cur[j];
                if (INT) {
                    const int32_t wk = wi[k];
#pragma unroll
                    for (int g = 0; g < G; ++g) ai[g] += ((byte >> g) & 1u) ? -wk : wk;
                } else {
                    const float wk = wf[k];
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        af[g] = __fadd_rn(af[g], ((byte >> g) & 1u) ? -wk : wk);
                }
            }
            }
            uint32_t byte = 0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float h = INT ? __fadd_rn((float)ai[g], bi[u]) : __fadd_rn(af[g], bi[u]);
                pa_update(h, lt, eta, alpha, xs[u][g], ms[u][g]);
                byte |= (xs[u][g] < 0.0f ? 1u : 0u) << g;
                if (last && h_last && r0 + g < R) h_last[(int64_t)i * Rp + r0 + g] = h;
            }
            nxt[i] = (uint8_t)byte;
        }
        __syncthreads();
        uint8_t *tmp = cur;
        cur = nxt;
        nxt = tmp;
    }

#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * RT;
        if (i >= n) continue;
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (r0 + g < R) {
                x[(int64_t)i * Rp + r0 + g] = xs[u][g];
                m[(int64_t)i * Rp + r0 + g] = ms[u][g];
            }
    }
}

// ---- rows with sum of |w| below 2^8: four replicas per 32-bit word ---------------------------
// The kernel above is bound by its vector instructions (about 25 per update at n = 2048,
// G = 4, 6 entries a row).  Here a variable's spins are one word with a 0 / 1 byte per
// replica, read as it is (no table), and with A as above (now below 2^8) one packed
// v_pk_mad_u16 by the weight in both halves adds an entry for four replicas: each half
// holds A_0 + 2^8 A_1 modulo 2^16, exact at the end whatever the partial sums.  Then per
// update: v_cvt_f32_ubyte and one fused multiply-add for the field (sum |w| + b - 2 A, all
// exact integers below 2^24), the seven operations of the definition, and 1.25 to gather the
// four signs (byte permutes of the sign bytes; a -0.0 would count as negative there, so
// the state's -0.0 are loaded as +0.0, and x + m' never makes one).  CACHE entries of each
// row are in registers; workgroups whose rows hold at most 6 skip the rest.
// The second spin buffer lies at a constant offset, so that both copies of the step share
// their address registers; the schedule is loaded 64 steps at a time and broadcast.  n = 2048,
// R = 1024, 6 entries a row: 0.845 us a step against 1.66 for the kernel above; n = 512:
// 0.33 against 0.59; n = 4000, 3 entries a row: 1.43 against 2.23.  With several variables and
// replicas a thread the registers do not hold all of this (spilled: 28 with 2 variables in
// groups of 8, 3 and 33 with 4 in groups of 2 and 4, 49 and 116 with 8 in groups of 1 and
// 2; none elsewhere), which the rule at res_form takes into account.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_mad(uint32_t w2, uint32_t s, uint32_t acc) {
    const u16x2 r = __builtin_bit_cast(u16x2, w2) * __builtin_bit_cast(u16x2, s) +
                    __builtin_bit_cast(u16x2, acc);
    return __builtin_bit_cast(uint32_t, r);
}

// bit 0 of byte g <- sign bit of x[g]
__device__ __forceinline__ uint32_t sign_bytes(const float *x, int count) {
    auto u = [&](int g) { return g < count ? __float_as_uint(x[g]) : 0u; };
    // byte 3 of two words each, then the two pairs
    const uint32_t a = __builtin_amdgcn_perm(u(1), u(0), 0x0C0C0703u);
    if (count <= 2) return (a >> 7) & 0x0101u;
    const uint32_t b = __builtin_amdgcn_perm(u(3), u(2), 0x07030C0Cu);
    return ((a | b) >> 7) & 0x01010101u;
}

// The state of the G replicas r0 .. of variable i, zeros where there is none.  Every load is
// made (of the last variable or replica again where there is none): a load behind a condition
// is waited for there, one after the other (Chimera C16, R = 1024: a call of one step 105 us
// with them, 71 so).
template <int G>
__device__ __forceinline__ void res_state(int32_t i, int32_t n, int64_t r0, int64_t R, int64_t Rp,
                                          const float *x, const float *m, float (&xs)[G],
                                          float (&ms)[G]) {
    const int64_t o = (int64_t)(i < n ? i : n - 1) * Rp + r0;
    const int last = (int)(R - r0 < G ? R - r0 : G) - 1;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        xs[g] = x[o + (g < last ? g : last)];
        ms[g] = m[o + (g < last ? g : last)];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const bool in = i < n && g <= last;
        xs[g] = in ? xs[g] : 0.0f;
        ms[g] = in ? ms[g] : 0.0f;
    }
}

// the second spin buffer's LDS address: a constant, so that both are offsets of one address
constexpr int RES8_BUF = 32 * 1024;
constexpr size_t res8_lds(int64_t n, int64_t nnz, int G) {
    return RES8_BUF + (size_t)n * 4 * (size_t)((G + 3) / 4) + sizeof(int32_t) * (size_t)(n + 1) +
           6 * (size_t)nnz + 16;
}
constexpr bool res8_fits(int64_t n, int64_t nnz, int G) {
    return n * 4 * ((G + 3) / 4) <= RES8_BUF && res8_lds(n, nnz, G) <= RES_MAX_LDS;
}

// LDS: spins [n][NW] uint32 | at RES8_BUF the second spins | rp [n+1] int32 | w [nnz] int32 |
//      col [nnz] uint16 | flag
template <int G, int VPT>
__global__ void __launch_bounds__(RT) k_csr_resident8(
    int32_t n, int32_t nnz, int64_t R, int64_t Rp, const int32_t *__restrict__ rp_g,
    const void *__restrict__ col_g, int32_t col_dt, const void *__restrict__ w_g, int32_t w_dt,
    int32_t skip_diag, const float *__restrict__ b, float *__restrict__ x,
    float *__restrict__ m, float *__restrict__ h_last, int32_t t0, int32_t t1,
    const float *__restrict__ lam, float eta, float alpha) {
    constexpr int NW = (G + 3) / 4;          // spin words per variable
    constexpr int GW = G < 4 ? G : 4;        // replicas per word
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint32_t *sp = reinterpret_cast<uint32_t *>(lds);
    int32_t *rp = reinterpret_cast<int32_t *>(sp + RES8_BUF / 4 + (size_t)n * NW);
    int32_t *wi = rp + (n + 1);
    uint16_t *col = reinterpret_cast<uint16_t *>(wi + nnz);
    int32_t *many = wi + nnz + (nnz + 1) / 2;       // past the columns, in the 16 spare bytes
    const int tid = threadIdx.x, lane = tid & 63, nt = blockDim.x;   // VPT * nt >= n
    const int64_t r0 = (int64_t)blockIdx.x * G;

    if (tid == 0) *many = 0;
    for (int32_t k = tid; k <= n; k += nt) rp[k] = rp_g[k];
    for (int32_t k = tid; k < nnz; k += nt) {
        col[k] = (uint16_t)(col_dt == QPA_I16 ? (int32_t) static_cast<const int16_t *>(col_g)[k]
                                              : static_cast<const int32_t *>(col_g)[k]);
        wi[k] = ld_as<int32_t>(w_g, w_dt, k);
    }

    constexpr int CACHE = (16 / VPT) < 8 ? (16 / VPT) : 8;
    int32_t cj[VPT][CACHE];      // LDS word of a cached entry's spins
    uint32_t cw[VPT][CACHE];     // its weight in both halves
    int32_t crest[VPT], cend[VPT];
    uint32_t cneg[VPT];          // sum over w < 0 of |w|, in each byte lane's place
    float hb[VPT];               // sum of |w| plus the field
    float xs[VPT][G], ms[VPT][G];
    int most = 0;
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * nt;
        res_state<G>(i, n, r0, R, Rp, x, m, xs[u], ms[u]);
    }
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * nt;
#pragma unroll
        for (int g = 0; g < G; ++g) xs[u][g] = __fadd_rn(xs[u][g], 0.0f);
        if (i < n)
#pragma unroll
            for (int p = 0; p < NW; ++p) {
                uint32_t word = 0;
#pragma unroll
                for (int g = 0; g < GW; ++g) word |= (xs[u][4 * p + g] < 0.0f ? 1u : 0u) << (8 * g);
                sp[(size_t)i * NW + p] = word;
            }
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * nt;
        int32_t cnt = 0, k = 0, k1 = 0, sum = 0;
        if (i < n) {
            k = rp[i];
            k1 = rp[i + 1];
        }
#pragma unroll
        for (int c = 0; c < CACHE; ++c) {
            cj[u][c] = 0;
            cw[u][c] = 0u;
        }
        cneg[u] = 0u;
        for (int32_t kk = k; kk < k1; ++kk) {
            if (skip_diag && col[kk] == i) continue;
            const int32_t a = wi[kk] < 0 ? -wi[kk] : wi[kk];
            sum += a;
            if (wi[kk] < 0) cneg[u] += (uint32_t)a * 0x01010101u;
        }
        hb[u] = i < n ? __fadd_rn((float)sum, b[i]) : 0.0f;
        for (; k < k1 && cnt < CACHE; ++k) {
            const int32_t j = col[k];
            if (skip_diag && j == i) continue;
#pragma unroll
            for (int c = 0; c < CACHE; ++c)
                if (c == cnt) {
                    cj[u][c] = j * NW;
                    cw[u][c] = ((uint32_t)wi[k] & 0xFFFFu) * 0x10001u;
                }
            ++cnt;
        }
        crest[u] = k;
        cend[u] = k1;
        most = max(most, cnt);
    }
    bool longer = false;
#pragma unroll
    for (int u = 0; u < VPT; ++u) longer = longer || crest[u] < cend[u];
    const bool rest = __ballot(longer) != 0;       // per wave
    // of the whole workgroup: the two step loops hold a barrier each, and all waves have to
    // wait at the same one
    if (most > 6) *many = 1;
    __syncthreads();
    const bool few = __builtin_amdgcn_readfirstlane(*many) == 0;

    // one step from buffer CUR into the other; NC entries of each row from the registers, the
    // others from LDS.  With one variable a thread, where a step waits for its longest row, they
    // are read four at a time (n = 200, 20 entries a row, R = 64: 1.3 us a step against 2.65);
    // with more, the code's registers cost the other rows as much.
    constexpr int BATCH = 4;
    auto step = [&](auto nc, auto cur, auto keep, float lt) {
        constexpr int NC = decltype(nc)::value, CUR = decltype(cur)::value;
        const uint32_t *s_now = sp + CUR * (RES8_BUF / 4);
        uint32_t *s_nxt = sp + (CUR ^ 1) * (RES8_BUF / 4);
        uint32_t acc[VPT][NW], s[VPT][NC][NW];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int u = 0; u < VPT; ++u)
#pragma unroll
                for (int p = 0; p < NW; ++p) s[u][c][p] = s_now[cj[u][c] + p];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int u = 0; u < VPT; ++u)
#pragma unroll
                for (int p = 0; p < NW; ++p)
                    acc[u][p] = pk_mad(cw[u][c], s[u][c][p], c == 0 ? cneg[u] : acc[u][p]);
        if (rest) {
#pragma unroll
            for (int u = 0; u < VPT; ++u) {
                const int32_t i = tid + u * nt;
                if constexpr (VPT == 1) {
                    // BATCH entries' reads together; one past the row or on the diagonal
                    // adds nothing
                    for (int32_t k = crest[u]; k < cend[u]; k += BATCH) {
                        int32_t j[BATCH];
                        uint32_t w2[BATCH], sv[BATCH][NW];
#pragma unroll
                        for (int d = 0; d < BATCH; ++d) {
                            const int32_t kk = min(k + d, cend[u] - 1);
                            j[d] = col[kk];
                            w2[d] = ((uint32_t)wi[kk] & 0xFFFFu) * 0x10001u;
                        }
#pragma unroll
                        for (int d = 0; d < BATCH; ++d) {
                            const bool out = (k + d >= cend[u]) | (skip_diag & (j[d] == i));
                            w2[d] &= (uint32_t)out - 1u;
#pragma unroll
                            for (int p = 0; p < NW; ++p) sv[d][p] = s_now[j[d] * NW + p];
                        }
#pragma unroll
                        for (int d = 0; d < BATCH; ++d)
#pragma unroll
                            for (int p = 0; p < NW; ++p)
                                acc[u][p] = pk_mad(w2[d], sv[d][p], acc[u][p]);
                    }
                } else {
                    for (int32_t k = crest[u]; k < cend[u]; ++k) {
                        const int32_t j = col[k];
                        if (skip_diag && j == i) continue;
                        const uint32_t w2 = ((uint32_t)wi[k] & 0xFFFFu) * 0x10001u;
#pragma unroll
                        for (int p = 0; p < NW; ++p)
                            acc[u][p] = pk_mad(w2, s_now[j * NW + p], acc[u][p]);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int32_t i = tid + u * nt;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float a = (float)((acc[u][g >> 2] >> (8 * (g & 3))) & 0xFFu);
                const float h = __fmaf_rn(-2.0f, a, hb[u]);
                const float gr = __fadd_rn(__fmul_rn(lt, xs[u][g]), h);
                const float mn = __fsub_rn(__fmul_rn(alpha, ms[u][g]), __fmul_rn(eta, gr));
                ms[u][g] = mn;
                // fmin(1, fmax(-1, y)), also for a NaN (-1)
                xs[u][g] = __builtin_amdgcn_fmed3f(__fadd_rn(xs[u][g], mn), -1.0f, 1.0f);
                if (decltype(keep)::value && i < n && r0 + g < R)
                    h_last[(int64_t)i * Rp + r0 + g] = h;
            }
            if (i < n)
#pragma unroll
                for (int p = 0; p < NW; ++p)
                    s_nxt[(size_t)i * NW + p] = sign_bytes(&xs[u][4 * p], GW);
        }
        __syncthreads();
    };
    auto run = [&](auto nc) {
        std::integral_constant<int, 0> b0;
        std::integral_constant<int, 1> b1;
        const int32_t te = h_last ? t1 - 1 : t1;      // steps that keep no field
        int32_t t = t0;
        for (; t < te; t += 64) {                     // the schedule 64 steps at a time
            const float lv = t + lane < t1 ? lam[t + lane] : 0.0f;
            auto l = [&](int k) {
                return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lv), k));
            };
            const int cnt = min(64, te - t);
            int k = 0;
            // the loop's place among the 64-byte lines of the instruction cache is worth up to 6 %
            // (Chimera C16, R = 1024: 0.755 to 0.802 us a step at four offsets); this fixes it
            asm volatile(".p2align 6" ::: "memory");
            for (; k + 2 <= cnt; k += 2) {
                step(nc, b0, std::false_type{}, l(k));
                step(nc, b1, std::false_type{}, l(k + 1));
            }
            if (k < cnt) step(nc, b0, std::false_type{}, l(k));    // only the last 64 steps
        }
        if (h_last) {
            if ((te - t0) & 1) step(nc, b1, std::true_type{}, lam[te]);
            else step(nc, b0, std::true_type{}, lam[te]);
        }
    };
    if (few) run(std::integral_constant<int, CACHE < 6 ? CACHE : 6>{});
    else run(std::integral_constant<int, CACHE>{});
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * nt;
        if (i >= n) continue;
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (r0 + g < R) {
                x[(int64_t)i * Rp + r0 + g] = xs[u][g];
                m[(int64_t)i * Rp + r0 + g] = ms[u][g];
            }
    }
}

template <int G, int VPT>
hipError_t launch_res8(const CsrView &c, int64_t R, int64_t Rp, const float *b, float *x, float *m,
                       float *h_last, int32_t t0, int32_t t1, const float *lam, float eta,
                       float alpha, hipStream_t st) {
    const size_t lds = res8_lds(c.n, c.nnz, G);
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_csr_resident8<G, VPT>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
    // no more waves than the variables need: a second block then fits beside a small one
    const unsigned nt = 64u * (unsigned)((c.n + 64 * VPT - 1) / (64 * VPT));
    k_csr_resident8<G, VPT><<<(unsigned)((R + G - 1) / G), nt, lds, st>>>(
        (int32_t)c.n, (int32_t)c.nnz, R, Rp, c.rp, c.col, c.col_dt, c.w, c.w_dt,
        c.skip_diag ? 1 : 0, b, x, m, h_last, t0, t1, lam, eta, alpha);
    return hipGetLastError();
}

// ---- other rows: spins as floats ----------------------------------------------------------
// The kernels with spin bits pick a bit and a weight's sign for every entry and replica or
// pair of replicas.
// Here a variable's spins are G floats +-1 in LDS: one read and one multiply-add per entry
// and replica (w s is exact, so the sum is the definition's chain; an unused slot's
// weight 0 changes no sum, which starts at +0.0 and so is never -0.0).  Two buffers, one
// barrier a step; the state's -0.0 are loaded as +0.0 (a spin is x's sign bit) as above.
// n = 2048, 6 entries a row, R = 1024: 1.14 us a step, float couplings 1.99 with spin bits,
// integer ones (row sums from 2^8 to 2^16) 1.66; n = 512, R = 256: 0.26, 0.56 and 0.43.
constexpr size_t resf_lds(int64_t n, int64_t nnz, int G) {
    return 2 * (size_t)n * G * 4 + sizeof(int32_t) * (size_t)(n + 1) + 6 * (size_t)nnz + 16;
}

template <int G> __device__ __forceinline__ void resf_read(const float *p, float (&s)[G]) {
    if constexpr (G % 4 == 0) {
#pragma unroll
        for (int g = 0; g < G; g += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(p + g);
            s[g] = v.x, s[g + 1] = v.y, s[g + 2] = v.z, s[g + 3] = v.w;
        }
    } else if constexpr (G == 2) {
        const float2 v = *reinterpret_cast<const float2 *>(p);
        s[0] = v.x, s[1] = v.y;
    } else {
        s[0] = *p;
    }
}

// LDS: spins [2][n][G] float | rp [n+1] int32 | w [nnz] float | col [nnz] uint16
template <int G, int VPT>
__global__ void __launch_bounds__(RT) k_csr_residentf(
    int32_t n, int32_t nnz, int64_t R, int64_t Rp, const int32_t *__restrict__ rp_g,
    const void *__restrict__ col_g, int32_t col_dt, const void *__restrict__ w_g, int32_t w_dt,
    int32_t skip_diag, const float *__restrict__ b, float *__restrict__ x,
    float *__restrict__ m, float *__restrict__ h_last, int32_t t0, int32_t t1,
    const float *__restrict__ lam, float eta, float alpha) {
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float *sp = reinterpret_cast<float *>(lds);
    int32_t *rp = reinterpret_cast<int32_t *>(sp + 2 * (size_t)n * G);
    float *wf = reinterpret_cast<float *>(rp + (n + 1));
    uint16_t *col = reinterpret_cast<uint16_t *>(wf + nnz);
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t r0 = (int64_t)blockIdx.x * G;
    for (int32_t k = tid; k <= n; k += RT) rp[k] = rp_g[k];
    for (int32_t k = tid; k < nnz; k += RT) {
        col[k] = (uint16_t)(col_dt == QPA_I16 ? (int32_t) static_cast<const int16_t *>(col_g)[k]
                                              : static_cast<const int32_t *>(col_g)[k]);
        wf[k] = ld_as<float>(w_g, w_dt, k);
    }
    // cached entries (at most 32 spins read together)
    constexpr int CA = (16 / VPT) < 8 ? (16 / VPT) : 8;
    constexpr int CACHE = CA * G > 32 ? 32 / G : CA;
    int32_t cj[VPT][CACHE], crest[VPT], cend[VPT];
    float cw[VPT][CACHE], bi[VPT], xs[VPT][G], ms[VPT][G];
    auto sign = [](float v) {
        return __uint_as_float((__float_as_uint(v) & 0x80000000u) | 0x3F800000u);
    };
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * RT;
        bi[u] = i < n ? b[i] : 0.0f;
        res_state<G>(i, n, r0, R, Rp, x, m, xs[u], ms[u]);
    }
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * RT;
#pragma unroll
        for (int g = 0; g < G; ++g) {
            xs[u][g] = __fadd_rn(xs[u][g], 0.0f);
            if (i < n) sp[i * G + g] = xs[u][g] < 0.0f ? -1.0f : 1.0f;
        }
    }
    __syncthreads();
    bool longer = false;
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * RT;
        int32_t k = 0, k1 = 0, cnt = 0;
        if (i < n) {
            k = rp[i];
            k1 = rp[i + 1];
        }
#pragma unroll
        for (int c = 0; c < CACHE; ++c) {
            cj[u][c] = 0;
            cw[u][c] = 0.0f;
        }
        for (; k < k1 && cnt < CACHE; ++k) {
            const int32_t j = col[k];
            if (skip_diag && j == i) continue;
#pragma unroll
            for (int c = 0; c < CACHE; ++c)
                if (c == cnt) {
                    cj[u][c] = j * G;
                    cw[u][c] = wf[k];
                }
            ++cnt;
        }
        crest[u] = k;
        cend[u] = k1;
        longer = longer || k < k1;
    }
    const bool rest = __ballot(longer) != 0;       // per wave
    int cur = 0;
    auto step = [&](auto keep, float lt) {
        const float *now = sp + (size_t)cur * n * G;
        float *nxt = sp + (size_t)(cur ^ 1) * n * G;
#pragma unroll
        for (int u = 0; u < VPT; ++u) {
            const int32_t i = tid + u * RT;
            if (i >= n) continue;
            float sv[CACHE][G], acc[G];
#pragma unroll
            for (int c = 0; c < CACHE; ++c) resf_read<G>(now + cj[u][c], sv[c]);
#pragma unroll
            for (int g = 0; g < G; ++g) acc[g] = 0.0f;
#pragma unroll
            for (int c = 0; c < CACHE; ++c)
#pragma unroll
                for (int g = 0; g < G; ++g) acc[g] = __fmaf_rn(cw[u][c], sv[c][g], acc[g]);
            if (rest) {
                if constexpr (VPT == 1 && G <= 4) {
                    // four entries' reads together, as in the byte form; one past the row or on
                    // the diagonal has weight 0, which changes no sum
                    for (int32_t k = crest[u]; k < cend[u]; k += 4) {
                        int32_t j[4];
                        float wk[4], s[4][G];
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const int32_t kk = min(k + d, cend[u] - 1);
                            j[d] = col[kk];
                            wk[d] = wf[kk];
                        }
#pragma unroll
                        for (int d = 0; d < 4; ++d) {
                            const bool out = (k + d >= cend[u]) | (skip_diag & (j[d] == i));
                            wk[d] = __uint_as_float(__float_as_uint(wk[d]) & ((uint32_t)out - 1u));
                            resf_read<G>(now + j[d] * G, s[d]);
                        }
#pragma unroll
                        for (int d = 0; d < 4; ++d)
#pragma unroll
                            for (int g = 0; g < G; ++g) acc[g] = __fmaf_rn(wk[d], s[d][g], acc[g]);
                    }
                } else {
                    for (int32_t k = crest[u]; k < cend[u]; ++k) {
                        const int32_t j = col[k];
                        if (skip_diag && j == i) continue;
                        float s[G];
                        resf_read<G>(now + j * G, s);
#pragma unroll
                        for (int g = 0; g < G; ++g) acc[g] = __fmaf_rn(wf[k], s[g], acc[g]);
                    }
                }
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const float h = __fadd_rn(acc[g], bi[u]);
                const float gr = __fadd_rn(__fmul_rn(lt, xs[u][g]), h);
                const float mn = __fsub_rn(__fmul_rn(alpha, ms[u][g]), __fmul_rn(eta, gr));
                ms[u][g] = mn;
                // fmin(1, fmax(-1, y)), also for a NaN (-1)
                xs[u][g] = __builtin_amdgcn_fmed3f(__fadd_rn(xs[u][g], mn), -1.0f, 1.0f);
                if (decltype(keep)::value && r0 + g < R) h_last[(int64_t)i * Rp + r0 + g] = h;
            }
#pragma unroll
            for (int g = 0; g < G; ++g) nxt[i * G + g] = sign(xs[u][g]);
        }
        __syncthreads();
        cur ^= 1;
    };
    const int32_t te = h_last ? t1 - 1 : t1;       // steps that keep no field
    for (int32_t t = t0; t < te; t += 64) {        // the schedule 64 steps at a time
        const float lv = t + lane < t1 ? lam[t + lane] : 0.0f;
        const int cnt = min(64, te - t);
        for (int k = 0; k < cnt; ++k)
            step(std::false_type{},
                 __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lv), k)));
    }
    if (h_last) step(std::true_type{}, lam[te]);
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
        const int32_t i = tid + u * RT;
        if (i >= n) continue;
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (r0 + g < R) {
                x[(int64_t)i * Rp + r0 + g] = xs[u][g];
                m[(int64_t)i * Rp + r0 + g] = ms[u][g];
            }
    }
}

template <int G, int VPT>
hipError_t launch_resf(const CsrView &c, int64_t R, int64_t Rp, const float *b, float *x, float *m,
                       float *h_last, int32_t t0, int32_t t1, const float *lam, float eta,
                       float alpha, hipStream_t st) {
    const size_t lds = resf_lds(c.n, c.nnz, G);
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_csr_residentf<G, VPT>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
    k_csr_residentf<G, VPT><<<(unsigned)((R + G - 1) / G), RT, lds, st>>>(
        (int32_t)c.n, (int32_t)c.nnz, R, Rp, c.rp, c.col, c.col_dt, c.w, c.w_dt,
        c.skip_diag ? 1 : 0, b, x, m, h_last, t0, t1, lam, eta, alpha);
    return hipGetLastError();
}

template <int G, int VPT, bool INT, bool SW>
hipError_t launch_one(const CsrView &c, int64_t R, int64_t Rp, const float *b, float *x,
                      float *m, float *h_last, int32_t t0, int32_t t1, const float *lam,
                      float eta, float alpha, size_t lds, hipStream_t st) {
    const unsigned blocks = (unsigned)((R + G - 1) / G);
    // allow more than the default dynamic LDS; a runtime without the attribute leaves the
    // launch to report a real limit
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&k_csr_resident<G, VPT, INT, SW>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)hipGetLastError();
    k_csr_resident<G, VPT, INT, SW><<<blocks, RT, lds, st>>>(
        (int32_t)c.n, (int32_t)c.nnz, R, Rp, c.rp, c.col, c.col_dt, c.w, c.w_dt,
        c.skip_diag ? 1 : 0, b, x, m, h_last, t0, t1, lam, eta, alpha);
    return hipGetLastError();
}

// The form of an instance.  All give the same bits (integer rows sum to less than 2^24).  What is
// fastest depends on how the columns spread over the LDS banks too; the lines below are
// drawn so that random graphs (n variables, d entries a row) and Chimera graphs are no
// slower than with spin bits, the form that always fits.  us a step:
//   * groups of at most 4 replicas have about one workgroup per compute unit: bytes or float
//     spins where they fit, 0.6x to 0.9x the time of bits.  With four or more variables a
//     thread the byte form spills registers, and float spins are faster (random, n = 3000,
//     d = 3, R = 1024: bits 4.08, bytes 4.28, floats 3.57).
//   * groups of 8, other rows than byte sums: two workgroups of 1024 threads share a compute
//     unit if they use bits, one if they use float spins (registers).  Integer rows below
//     2^16 take bits (random, n = 500, d = 6, R = 4096: 2.36 against 4.00; Chimera n = 512:
//     1.48 and 1.99).  Float rows take bits where one variable a thread and more than one
//     workgroup per compute unit meet (random 3.24 against 3.94, Chimera 1.86 and 2.00) and
//     floats elsewhere (R = 2048: random 2.44 and 2.05, Chimera 1.30 and 1.05; n = 1152,
//     R = 4096: Chimera 4.57 and 4.08).  Integer rows of 2^16 or more take floats (random,
//     n = 1000, d = 8, R = 4096: 8.14 against 8.98).
//   * groups of 8 in bytes: faster (n = 500, d = 6, R = 4096: 2.15) unless only bits leave room
//     in LDS for a second workgroup and there is one (random, n = 1000, d = 6, R = 4096: 4.37
//     against 4.75), or two variables a thread, whose byte form spills, hold very few
//     entries (random, n = 1500, d = 3, R = 2048: 2.42 against 2.69; at d = 6 both 4.0;
//     Chimera, n = 1152: 1.86 against 1.70).
enum class ResForm { Bytes, Floats, Bits };

template <int G, int VPT>
ResForm res_form(const CsrView &c, int64_t R, bool is_int, double max_row, size_t lds, int cus) {
    const bool queue = (R + G - 1) / G > cus;       // more workgroups than compute units
    const bool floats = resf_lds(c.n, c.nnz, G) <= RES_MAX_LDS;
    auto two = [](size_t bytes) { return 2 * bytes <= RES_MAX_LDS; };
    if (is_int && max_row < 256.0 && res8_fits(c.n, c.nnz, G) && !(VPT >= 4 && floats)) {
        const bool bits = G == 8 && (VPT == 2 ? c.nnz < 4 * c.n
                                              : queue && two(lds) && !two(res8_lds(c.n, c.nnz, G)));
        return bits ? ResForm::Bits : ResForm::Bytes;
    }
    if (!floats) return ResForm::Bits;
    if (G < 8 || (is_int && max_row >= 65536.0)) return ResForm::Floats;
    return is_int || (VPT == 1 && queue) ? ResForm::Bits : ResForm::Floats;
}

template <int G, int VPT>
hipError_t launch_g_v(const CsrView &c, int64_t R, int64_t Rp, bool is_int, double max_row,
                      int cus, const float *b, float *x, float *m, float *h_last, int32_t t0,
                      int32_t t1, const float *lam, float eta, float alpha, size_t lds,
                      hipStream_t st) {
    switch (res_form<G, VPT>(c, R, is_int, max_row, lds, cus)) {
        case ResForm::Bytes:
            return launch_res8<G, VPT>(c, R, Rp, b, x, m, h_last, t0, t1, lam, eta, alpha, st);
        case ResForm::Floats:
            return launch_resf<G, VPT>(c, R, Rp, b, x, m, h_last, t0, t1, lam, eta, alpha, st);
        case ResForm::Bits: break;
    }
    if (is_int && max_row < 65536.0)
        return launch_one<G, VPT, true, true>(c, R, Rp, b, x, m, h_last, t0, t1, lam, eta,
                                              alpha, lds, st);
    if (is_int)
        return launch_one<G, VPT, true, false>(c, R, Rp, b, x, m, h_last, t0, t1, lam, eta,
                                               alpha, lds, st);
    return launch_one<G, VPT, false, false>(c, R, Rp, b, x, m, h_last, t0, t1, lam, eta, alpha,
                                            lds, st);
}

}  // namespace

size_t csr_resident_lds(int64_t n, int64_t nnz) {
    return RES_LUT_BYTES + sizeof(int32_t) * (size_t)(n + 1) +
           (sizeof(int32_t) + sizeof(uint16_t)) * (size_t)nnz + 2 * (size_t)n + 16;
}

namespace {
// variables per thread as instantiated: 1, 2, 4 or 8
int64_t resident_vpt(int64_t n) {
    const int64_t v = (n + RT - 1) / RT;
    return v <= 1 ? 1 : v <= 2 ? 2 : v <= 4 ? 4 : 8;
}
}  // namespace

int csr_resident_group(int64_t n, int64_t R, int cus) {
    if (n < 1 || n > RES_MAX_N) return 0;
    const int64_t v = resident_vpt(n);
    // the largest group that still gives every compute unit a workgroup, with at most
    // 16 (variable, replica) pairs per thread
    int G = 8;
    while (G > 1 && ((R + G - 1) / G < cus || v * G > 16)) G >>= 1;
    return v * G <= 16 ? G : 0;
}

hipError_t launch_csr_resident(const CsrView &c, int G, int64_t R, int64_t Rp, bool is_int,
                               double max_row, int cus, const float *b, float *x, float *m,
                               float *h_last, int32_t t0, int32_t t1, const float *lam, float eta,
                               float alpha, hipStream_t st) {
    if (t1 <= t0) return hipSuccess;
    const size_t lds = csr_resident_lds(c.n, c.nnz);
    if (lds > RES_MAX_LDS || c.n > RES_MAX_N || c.nnz > INT32_MAX) return hipErrorInvalidValue;
    const int v = (int)resident_vpt(c.n);
    if (v * G > 16) return hipErrorInvalidValue;
#define QPA_RES_CASE(GG, VV)                                                                   \
    if (G == GG && v == VV)                                                                    \
        return launch_g_v<GG, VV>(c, R, Rp, is_int, max_row, cus, b, x, m, h_last, t0, t1, lam, \
                                  eta, alpha, lds, st);
    QPA_RES_CASE(8, 1)
    QPA_RES_CASE(8, 2)
    QPA_RES_CASE(4, 1)
    QPA_RES_CASE(4, 2)
    QPA_RES_CASE(4, 4)
    QPA_RES_CASE(2, 1)
    QPA_RES_CASE(2, 2)
    QPA_RES_CASE(2, 4)
    QPA_RES_CASE(2, 8)
    QPA_RES_CASE(1, 1)
    QPA_RES_CASE(1, 2)
    QPA_RES_CASE(1, 4)
    QPA_RES_CASE(1, 8)
#undef QPA_RES_CASE
    return hipErrorInvalidValue;
}

}  // namespace qpa
