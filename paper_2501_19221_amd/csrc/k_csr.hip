// Sparse (CSR) PA step (App. B): h_i = sum_k w_k s_{col_k} + b_i, then the fused update.
//
// Replicas are packed into groups of G lanes (G a power of two, G <= 64).  A wave handles
// V = 64/G consecutive variables x G replicas of one group, so every lane owns one
// (variable, replica) pair; the lanes of a variable read the same CSR entries (broadcast)
// and each picks its own replica's spin bit out of a shared 64-bit word (G < 64; groups of 64
// have a kernel of their own below).
// Layouts:
//   x, m   [np][Rp] FP32, replica fastest (Rp = groups * G)
//   spins  words[g][w], 64 bits each: variable i, replica r = g*G + rl sits in word
//          w = i / V at bit (i % V) * G + rl; bit set <=> spin -1.
// Integer couplings are summed in int32 (exact: rows are validated below 2^24) and the
// total converted once; float couplings are summed in FP32 in row order.  Both match the
// definition's ascending-entry order.
#include "qpa_internal.h"

#include <type_traits>

namespace qpa {
namespace {

__device__ __forceinline__ void pa_update(float h, float lam, float eta, float alpha, float &x,
                                          float &m) {
    float g = __fadd_rn(__fmul_rn(lam, x), h);
    float mn = __fsub_rn(__fmul_rn(alpha, m), __fmul_rn(eta, g));
    float y = __fadd_rn(x, mn);
    y = fminf(1.0f, fmaxf(-1.0f, y));
    m = mn;
    x = y;
}

constexpr int CSR_BATCH = 4;   // row entries whose loads are issued together

template <typename TW, typename TI, bool INT>
__global__ void __launch_bounds__(256) k_csr_step(
    int64_t n, int64_t Rp, int G, int shiftG, int64_t nwords, const int32_t *__restrict__ rp,
    const TI *__restrict__ col, const TW *__restrict__ wts, int skip_diag,
    const float *__restrict__ b, const uint64_t *__restrict__ s_cur,
    uint64_t *__restrict__ s_nxt, float *__restrict__ x, float *__restrict__ m,
    float *__restrict__ h_last, int t, const float *__restrict__ lam, float eta, float alpha) {
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t g = blockIdx.y;
    const int V = 64 >> shiftG;
    const int vsub = lane >> shiftG, rl = lane & (G - 1);
    const int64_t i = w * V + vsub;
    const int64_t r = g * G + rl;
    const uint64_t *sg = s_cur + g * nwords;
    const int wsh = 6 - shiftG;
    bool neg = false;
    if (w < nwords && i < n) {
        // every load that does not depend on a gathered value is issued up front; the
        // entries of the row follow in batches of CSR_BATCH (column and weight loads, then
        // all spin-word gathers, then the sums in entry order), so a wave waits for three
        // memory round trips per batch instead of two per entry
        const int64_t gi = i * Rp + r;
        const int64_t k0 = rp[i], k1 = rp[i + 1];
        float xv = x[gi], mv = m[gi];
        const float bi = b[i];
        int32_t ai = 0;
        float af = 0.0f;
        auto batch = [&](int64_t kb) {
            int64_t j[CSR_BATCH];
            TW wk[CSR_BATCH];
            uint64_t word[CSR_BATCH];
#pragma unroll
            for (int d = 0; d < CSR_BATCH; ++d) {
                const int64_t k = kb + d < k1 ? kb + d : k1 - 1;   // in bounds: kb < k1
                j[d] = (int64_t)col[k];
                wk[d] = wts[k];
            }
#pragma unroll
            for (int d = 0; d < CSR_BATCH; ++d) {
                word[d] = 0;
                if (kb + d < k1) word[d] = sg[j[d] >> wsh];
            }
#pragma unroll
            for (int d = 0; d < CSR_BATCH; ++d) {
                if (kb + d >= k1 || (skip_diag && j[d] == i)) continue;
                const int bit = (int)((word[d] >> (((j[d] & (V - 1)) << shiftG) + rl)) & 1u);
                if (INT) {
                    const int32_t v = (int32_t)wk[d];
                    ai += bit ? -v : v;
                } else {
                    const float v = (float)wk[d];
                    af = __fadd_rn(af, bit ? -v : v);
                }
            }
        };
        if (k0 < k1) batch(k0);   // the first batch outside the loop: most rows end in it
        for (int64_t kb = k0 + CSR_BATCH; kb < k1; kb += CSR_BATCH) batch(kb);
        const float h = INT ? __fadd_rn((float)ai, bi) : __fadd_rn(af, bi);
        pa_update(h, lam[t], eta, alpha, xv, mv);
        x[gi] = xv;
        m[gi] = mv;
        if (h_last) h_last[gi] = h;
        neg = xv < 0.0f;
    }
    const uint64_t bal = __ballot(neg);
    if (lane == 0 && w < nwords) s_nxt[g * nwords + w] = bal;
}

// ---- groups of 64 replicas: U variables per wave -------------------------------------------
// With one variable and 64 replicas a wave (the kernel above) the step is bound by latency:
// three dependent memory trips for 512 bytes of state.  Here a wave takes U consecutive
// variables: their state is loaded up front (2 U rows of 256 bytes in flight), and 64 / U
// entries of each row, one per lane, whose spin words the lanes gather.  An entry's word
// then comes from its lane as a scalar that is the select mask of the 64 replicas, its
// weight as a scalar operand, in row order.  Unused slots hold zero weights; four slots of
// all rows are left out together where no row reaches them.
// The sums are +-1 x weight FP32 multiply-adds: one rounding per term, as in the definition,
// and exact for integer rows (validated below 2^24).
// n = 90000, 4 entries a row, R = 256: 108 us a step with one variable a wave, 58.5 now
// (6.3 TB/s of state, the rate of a large copy; non-temporal state accesses cost 10 %,
// state loads ahead of the entries' change nothing); n = 9216, R = 64: 5.8 and 4.8.
template <typename TW, typename TI, int U>
__global__ void __launch_bounds__(256) k_csr_step64(
    int64_t n, int64_t Rp, const int32_t *__restrict__ rp, const TI *__restrict__ col,
    const TW *__restrict__ wts, int skip_diag, const float *__restrict__ b,
    const uint64_t *__restrict__ s_cur, uint64_t *__restrict__ s_nxt, float *__restrict__ x,
    float *__restrict__ m, float *__restrict__ h_last, int t, const float *__restrict__ lam,
    float eta, float alpha) {
    constexpr int D = 64 / U;              // slots of a row per pass
    const int lane = threadIdx.x & 63;
    const int64_t i0 =
        ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * U;
    if (i0 >= n) return;
    const int64_t g = blockIdx.y;
    const int cnt = (int)(n - i0 < U ? n - i0 : U);
    const uint64_t *sg = s_cur + g * n;
    const int ul = lane / D;               // the row of this lane's slots
    const int32_t il = (int32_t)i0 + (ul < cnt ? ul : cnt - 1);
    int32_t k = rp[il];
    const int32_t k1 = ul < cnt ? rp[il + 1] : k;
    const int32_t left = k1 - k;           // entries of the row
    int32_t slot = lane % D;
    const float bl = b[i0 + (lane < cnt ? lane : cnt - 1)];
    const float lt = lam[t];
    float xv[U], mv[U];
    auto at = [&](int u) { return (i0 + (u < cnt ? u : cnt - 1)) * Rp + g * 64; };

    // the entry of this lane's slot; a diagonal one adds a zero, which changes no sum
    auto load = [&](int32_t &j, float &w) {
        j = 0;
        w = 0.0f;
        if (slot < left) {
            j = (int32_t)col[k + slot];
            w = (float)wts[k + slot];
            if (skip_diag && j == il) w = 0.0f;
        }
    };
    int32_t j;
    float w;
    load(j, w);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        xv[u] = x[at(u) + lane];
        mv[u] = m[at(u) + lane];
    }
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.0f;
    uint64_t used = __ballot(slot < left);
    while (used) {
        const uint64_t word = sg[j];
        const int32_t lo = (int32_t)word, hi = (int32_t)(word >> 32);
        const float wc = w;
        slot += D;
        const uint64_t next = __ballot(slot < left);
        if (next) load(j, w);
#pragma unroll
        for (int d0 = 0; d0 < D; d0 += 4) {
            uint64_t quads = 0;            // the lanes of slots d0 .. d0 + 3 of all rows
#pragma unroll
            for (int u = 0; u < U; ++u) quads |= (uint64_t)0xF << (u * D + d0);
            if (!(used & quads)) break;    // no row has a later slot either
#pragma unroll
            for (int d = d0; d < d0 + 4; ++d)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = u * D + d;
                    const uint64_t mask =
                        (uint64_t)(uint32_t)__builtin_amdgcn_readlane(lo, e) |
                        (uint64_t)(uint32_t)__builtin_amdgcn_readlane(hi, e) << 32;
                    const float we = __int_as_float(
                        __builtin_amdgcn_readlane(__float_as_int(wc), e));
                    const float s = __builtin_amdgcn_inverse_ballot_w64(mask) ? -1.0f : 1.0f;
                    acc[u] = __fmaf_rn(s, we, acc[u]);
                }
        }
        used = next;
    }
    uint64_t words = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const float bi = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bl), u));
        const float h = __fadd_rn(acc[u], bi);
        pa_update(h, lt, eta, alpha, xv[u], mv[u]);
        const uint64_t bal = __ballot(xv[u] < 0.0f);
        words = lane == u ? bal : words;
        if (u < cnt) {
            x[at(u) + lane] = xv[u];
            m[at(u) + lane] = mv[u];
            if (h_last) h_last[at(u) + lane] = h;
        }
    }
    if (lane < cnt) s_nxt[g * n + i0 + lane] = words;
}

__global__ void __launch_bounds__(256) k_csr_pack(int64_t n, int64_t Rp, int G, int shiftG,
                                                  int64_t nwords, const float *__restrict__ x,
                                                  uint64_t *__restrict__ sbits) {
    const int lane = threadIdx.x & 63;
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t g = blockIdx.y;
    const int V = 64 >> shiftG;
    const int64_t i = w * V + (lane >> shiftG);
    const int64_t r = g * G + (lane & (G - 1));
    bool neg = false;
    if (w < nwords && i < n) neg = x[i * Rp + r] < 0.0f;
    const uint64_t bal = __ballot(neg);
    if (lane == 0 && w < nwords) sbits[g * nwords + w] = bal;
}

int log2i(int v) {
    int s = 0;
    while ((1 << s) < v) ++s;
    return s;
}

}  // namespace

int csr_group_size(int64_t R) {
    int G = 1;
    while (G < R && G < 64) G <<= 1;
    return G;
}

int64_t csr_words_per_group(int64_t n, int G) {
    const int V = 64 / G;
    return (n + V - 1) / V;
}

hipError_t launch_csr_pack_spins(int64_t n, int64_t Rp, int G, const float *x, uint64_t *sbits,
                                 hipStream_t st) {
    const int64_t nwords = csr_words_per_group(n, G);
    dim3 grid((unsigned)((nwords + 3) / 4), (unsigned)(Rp / G));
    k_csr_pack<<<grid, 256, 0, st>>>(n, Rp, G, log2i(G), nwords, x, sbits);
    return hipGetLastError();
}

hipError_t launch_csr_step(const CsrView &c, int64_t Rp, int G, const float *b_f32,
                           const uint64_t *s_cur, uint64_t *s_nxt, float *x, float *m,
                           float *h_last, int32_t t, const float *lam, float eta, float alpha,
                           bool is_int, hipStream_t st) {
    const int64_t nwords = csr_words_per_group(c.n, G);
    dim3 grid((unsigned)((nwords + 3) / 4), (unsigned)(Rp / G));
    const int sh = log2i(G);
    auto run64 = [&](auto wtag, auto itag, auto utag) {
        using TW = decltype(wtag);
        using TI = decltype(itag);
        constexpr int U = decltype(utag)::value;
        const dim3 gr((unsigned)((c.n + 4 * U - 1) / (4 * U)), (unsigned)(Rp / 64));
        k_csr_step64<TW, TI, U><<<gr, 256, 0, st>>>(
            c.n, Rp, c.rp, static_cast<const TI *>(c.col), static_cast<const TW *>(c.w),
            c.skip_diag, b_f32, s_cur, s_nxt, x, m, h_last, t, lam, eta, alpha);
        return hipGetLastError();
    };
    auto run = [&](auto wtag, auto itag) {
        using TW = decltype(wtag);
        using TI = decltype(itag);
        if (G == 64) {
            // 8 variables a wave where that still makes 4096 waves, else 4: n = 9216, R = 64
            // 4.8 us a step with 4, 5.5 with 8; n = 40000, R = 256 31.6 and 28.2
            return c.n * (Rp / 64) < 32768 ? run64(wtag, itag, std::integral_constant<int, 4>{})
                                           : run64(wtag, itag, std::integral_constant<int, 8>{});
        }
        const TW *w = static_cast<const TW *>(c.w);
        const TI *cl = static_cast<const TI *>(c.col);
        if (is_int)
            k_csr_step<TW, TI, true><<<grid, 256, 0, st>>>(c.n, Rp, G, sh, nwords, c.rp, cl, w,
                                                           c.skip_diag, b_f32, s_cur, s_nxt, x,
                                                           m, h_last, t, lam, eta, alpha);
        else
            k_csr_step<TW, TI, false><<<grid, 256, 0, st>>>(c.n, Rp, G, sh, nwords, c.rp, cl, w,
                                                            c.skip_diag, b_f32, s_cur, s_nxt, x,
                                                            m, h_last, t, lam, eta, alpha);
        return hipGetLastError();
    };
    auto byw = [&](auto itag) -> hipError_t {
        switch (c.w_dt) {
            case QPA_I8: return run((int8_t)0, itag);
            case QPA_I16: return run((int16_t)0, itag);
            case QPA_I32: return run((int32_t)0, itag);
            case QPA_F32: return run(0.0f, itag);
            default: return hipErrorInvalidValue;
        }
    };
    if (c.col_dt == QPA_I16) return byw((int16_t)0);
    return byw((int32_t)0);
}

}  // namespace qpa
