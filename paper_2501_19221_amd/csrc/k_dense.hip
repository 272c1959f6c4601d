// Dense PA steps in FP32 (App. B).  Every kernel accumulates each local field
// sum_j J_ij s_j in ascending j from zero and then adds b_i: with s = +-1 every product is
// exact, so the result is the same FP32 sum whatever the tiling, and trajectories are
// reproducible bit for bit.  For the same reason a fused multiply-add s_j J_ij + acc,
// rounded once, equals the separately rounded product and sum, in one instruction.
//
// The update after the field is, each operation rounded separately:
//   g = lambda_t * x + h;  m' = alpha * m - eta * g;  x' = clip(x + m', -1, 1).
#include "qpa_internal.h"

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

__device__ __forceinline__ float spin_of(float x) { return x >= 0.0f ? 1.0f : -1.0f; }

// ------------------------------------------------- all steps in one launch (small n)
// A workgroup owns one replica, lane i of its ceil(n / 64) waves variable i: row i of J in
// registers (16 NC >= n of them) with x_i, m_i, for every step in [t0, t1).  A step is a
// serial chain of n fused multiply-adds per lane (the sums must ascend in j), so what
// bounds it is the instructions per term and the exchange of the spins.  The spins of 16
// variables sit in one register, the same in each row of 16 lanes, and the DPP operand
// row_newbcast:j hands spin j of the row to every lane: one vector instruction per
// term and nothing on the scalar unit.  The registers come from
//   * n <= 64: the wave's own spins, the rows of lanes that hold any copied across by
//     v_permlane32_swap / v_permlane16_swap -- no LDS, no barrier (with more waves than the
//     chip holds these count: n = 12, R = 65536 3.25 us a step, 3.75 with all rows copied);
//   * larger n: the replica's spins in LDS (two buffers), one barrier per step.
// Terms j >= n are +0.0 (zero couplings, +1 spins): a sum that starts at +0.0 never becomes
// -0.0 under round-to-nearest, so adding them changes no bit.  The schedule is read 64
// steps at a time, one value per lane.
// Measured: n = 20, R = 256, 2000 steps 244 us (signs from a ballot, a bit extraction
// and a sign flip per term: 448 us); n = 100, R = 150, 1000 steps 378 us (J and the
// spins of several replicas in LDS, one LDS read of each per term: 3.98 ms); 5 cycles per
// term.  Past 208 columns the registers run out.  Up to there no number of replicas makes the
// per-step product the faster form: us a step at n = 208 here and at n = 209 there, R = 256 0.74
// and 5.1, R = 4096 7.2 and 10.5, R = 16384 27.6 and 28.4, R = 65536 109.5 and 108.2.
constexpr int DR_MAXC = 13;              // columns in groups of 16: n <= 208 (registers)

// acc += s_j J_j for the 16 columns of a group, ascending.  The leading nop separates a
// vector write of the spins from their use as a DPP operand.
__device__ __forceinline__ void dr_fma16(float &acc, float s, const float (&J)[16]) {
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %12 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %13 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %15 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %16 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf"
        : "+v"(acc)
        : "v"(s), "v"(J[0]), "v"(J[1]), "v"(J[2]), "v"(J[3]), "v"(J[4]), "v"(J[5]), "v"(J[6]),
          "v"(J[7]), "v"(J[8]), "v"(J[9]), "v"(J[10]), "v"(J[11]), "v"(J[12]), "v"(J[13]),
          "v"(J[14]), "v"(J[15]));
}

// The first 4 columns of a group only (n just past a multiple of 16).
__device__ __forceinline__ void dr_fma4(float &acc, float s, const float (&J)[16]) {
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf"
        : "+v"(acc)
        : "v"(s), "v"(J[0]), "v"(J[1]), "v"(J[2]), "v"(J[3]));
}

// Rows of 16 lanes of v, each copied to all four rows: r[c] holds row c.
__device__ __forceinline__ void dr_rows(float v, float (&r)[4]) {
    const unsigned u = __float_as_uint(v);
    const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // rows 0 1 0 1, 2 3 2 3
    const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
    r[0] = __uint_as_float(lo[0]);
    r[1] = __uint_as_float(lo[1]);
    r[2] = __uint_as_float(hi[0]);
    r[3] = __uint_as_float(hi[1]);
}

template <int NC, bool LAST4>
__global__ void __launch_bounds__(NC <= 4 ? 64 : NC <= 8 ? 128 : 256, 1) k_dense_resident(
    int n, const float *__restrict__ J, const float *__restrict__ b, float *__restrict__ x,
    float *__restrict__ m, float *__restrict__ h_last, int t0, int t1,
    const float *__restrict__ lam, float eta, float alpha) {
    constexpr bool ONE = NC <= 4;                    // one wave: no exchange through LDS
    __shared__ float sp[ONE ? 1 : 2][ONE ? 1 : 16 * NC];
    const int i = threadIdx.x, lane = i & 63;
    const bool act = i < n;
    const int64_t g = (int64_t)blockIdx.x * n + i, ldj = dense_ld(n);
    float Jr[NC][16];                                // J is symmetric: column i, coalesced
#pragma unroll
    for (int j = 0; j < 16 * NC; ++j) Jr[j / 16][j % 16] = (act && j < n) ? J[j * ldj + i] : 0.0f;
    float xi = 0.0f, mi = 0.0f, bi = 0.0f, hi = 0.0f;
    if (act) {
        xi = x[g];
        mi = m[g];
        bi = b[i];
    }
    float s = act ? spin_of(xi) : 1.0f;
    int cur = 0;
    if (!ONE) {
        if (i < 16 * NC) sp[0][i] = s;
        __syncthreads();
    }
    for (int tb = t0; tb < t1; tb += 64) {
        const float lv = tb + lane < t1 ? lam[tb + lane] : 0.0f;
        const int te = t1 - tb < 64 ? t1 - tb : 64;
        for (int k = 0; k < te; ++k) {
            const float lt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lv), k));
            float sv[ONE ? 4 : NC];
            if constexpr (NC == 1) {
                sv[0] = s;                           // the variables' own row
            } else if constexpr (NC == 2) {
                const auto h = __builtin_amdgcn_permlane16_swap(
                    __float_as_uint(s), __float_as_uint(s), false, false);   // rows 0 0, 1 1
                sv[0] = __uint_as_float(h[0]);
                sv[1] = __uint_as_float(h[1]);
            } else if constexpr (ONE) {
                dr_rows(s, sv);
            } else {
#pragma unroll
                for (int c = 0; c < NC; ++c) sv[c] = sp[cur][16 * c + (lane & 15)];
            }
            float acc = 0.0f;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (LAST4 && c == NC - 1) dr_fma4(acc, sv[c], Jr[c]);
                else dr_fma16(acc, sv[c], Jr[c]);
            }
            hi = __fadd_rn(acc, bi);
            pa_update(hi, lt, eta, alpha, xi, mi);
            s = act ? spin_of(xi) : 1.0f;
            if (!ONE) {
                cur ^= 1;
                if (i < 16 * NC) sp[cur][i] = s;
                __syncthreads();
            }
        }
    }
    if (act) {
        x[g] = xi;
        m[g] = mi;
        if (h_last && t1 > t0) h_last[g] = hi;
    }
}

__global__ void __launch_bounds__(256) k_sign_f32(int64_t count, const float *__restrict__ x,
                                                  float *__restrict__ s) {
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < count;
         k += (int64_t)gridDim.x * blockDim.x)
        s[k] = spin_of(x[k]);
}

}  // namespace

bool dense_resident_fits(int64_t n) { return n >= 1 && n <= 16 * DR_MAXC; }

hipError_t launch_dense_resident(int64_t n, int64_t R, const float *J, const float *b,
                                 float *x, float *m, float *h_last, int32_t t0, int32_t t1,
                                 const float *lam, float eta, float alpha, hipStream_t st) {
    if (!dense_resident_fits(n)) return hipErrorInvalidValue;
    const int nc = (int)((n + 15) / 16);
    const bool last4 = n - 16 * (nc - 1) <= 4;
    const unsigned threads = (unsigned)((n + 63) / 64 * 64);
    constexpr int64_t PART = (int64_t)1 << 23;      // replicas a launch: a grid has < 2^32 threads
    for (int64_t r0 = 0; r0 < R; r0 += PART) {
        const unsigned grid = (unsigned)(R - r0 < PART ? R - r0 : PART);
        float *xr = x + r0 * n, *mr = m + r0 * n, *hr = h_last ? h_last + r0 * n : nullptr;
        switch (nc) {
#define QPA_DR(C)                                                                          \
    case C:                                                                                \
        if (last4)                                                                         \
            k_dense_resident<C, true><<<grid, threads, 0, st>>>((int)n, J, b, xr, mr, hr, t0, \
                                                                t1, lam, eta, alpha);      \
        else                                                                               \
            k_dense_resident<C, false><<<grid, threads, 0, st>>>((int)n, J, b, xr, mr, hr, t0, \
                                                                 t1, lam, eta, alpha);     \
        break;
            QPA_DR(1) QPA_DR(2) QPA_DR(3) QPA_DR(4) QPA_DR(5) QPA_DR(6) QPA_DR(7)
            QPA_DR(8) QPA_DR(9) QPA_DR(10) QPA_DR(11) QPA_DR(12) QPA_DR(13)
#undef QPA_DR
        }
    }
    return hipGetLastError();
}

hipError_t launch_sign_f32(int64_t count, const float *x, float *s, hipStream_t st) {
    if (count == 0) return hipSuccess;
    int64_t g = (count + 255) / 256;
    if (g > 65536) g = 65536;
    k_sign_f32<<<(unsigned)g, 256, 0, st>>>(count, x, s);
    return hipGetLastError();
}

}  // namespace qpa
