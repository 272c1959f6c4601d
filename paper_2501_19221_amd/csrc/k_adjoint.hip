// Relaxed PA (analog spins in the target part, s := x) and its reverse-mode adjoint, for
// one instance or a batch of instances sharing the dynamics parameters.
//
// Forward step t of one element (FP32, each operation rounded separately):
//   f = (J x_t)_i;  h = f + b_i;  g = lambda_t x + h;  m' = alpha m - eta g;
//   y = x + m';  x' = clip(y, -1, 1).
// Loss: L = scale * sum over instances and replicas of [ (1/2) x_T^T J x_T + b^T x_T ].
// Reverse, with mu_{T+1} = 0 and xbar_T = scale (J x_T + b):
//   A(t):  ybar = xbar_{t+1} * [|y_{t+1}| <= 1];  mu_{t+1} = ybar + alpha mu_{t+2};
//          dL/deta += <mu, -g_t>,  dL/dalpha += <mu, m_t>,  dL/dlambda_t = <mu, -eta x_t>
//   B(t):  xbar_t = ybar - eta (lambda_t mu_{t+1} + J mu_{t+1})
// A needs only the element's own values; B needs J mu, a product over neighbours.  A step
// of the reverse pass is one launch that runs B(t) and then A(t-1) on each element ("BA"),
// with mu double-buffered since neighbours read it; a segment's first step runs A alone
// and its last B alone, because the state of the step before a segment is recomputed
// only with the next segment.
//
// State: every vector is [rows][Rp] FP32 (replica fastest); instance k of a batch owns the
// global rows [row0_k, row0_k + n_k).  Replicas r >= R are padding: held at zero and left
// out of every sum.
// Products with J: CSR couplings through row launches over blocks of 64 rows, the input
// vector staged through LDS (a wave = four rows and 64 replicas, sixteen lanes a row, four
// replicas a lane, each row's entries walked in order); dense FP32 couplings through the matrix-core
// product shared with the SBM step, with the element work in its epilogue.  Both add one fused multiply-add
// per term in ascending column order.
// Inner products are accumulated in FP64 per thread, reduced per workgroup in a fixed
// order and written to a table of partial sums, whose rows (a step each) further launches
// add up in a fixed order: results do not depend on timing.  The steps at the ends of the
// checkpoint segments form their sums in the element-wise pass, the others in the product
// launches.  Both group them alike where all instances are sparse and of one (coupling,
// index) type: their results do not depend on the checkpoint interval either.  With dense
// instances or several types the gradients of two intervals agree to the rounding of the
// FP64 sums (the loss, which no interval changes, bit for bit).
#include "fp32_tiled.h"
#include <type_traits>

namespace qpa {
namespace {

constexpr int REL_FWD = REL_MODE_FWD, REL_LOSS = REL_MODE_LOSS, REL_A = REL_MODE_A,
              REL_B = REL_MODE_B, REL_BA = REL_MODE_BA;

__device__ __forceinline__ void rel_fwd_point(float f, float bi, float lt, float eta,
                                              float alpha, float &x, float &m) {
    const float h = __fadd_rn(f, bi);
    const float g = __fadd_rn(__fmul_rn(lt, x), h);
    const float mn = __fsub_rn(__fmul_rn(alpha, m), __fmul_rn(eta, g));
    x = fminf(1.0f, fmaxf(-1.0f, __fadd_rn(x, mn)));
    m = mn;
}

// A(t) on one element from its stored state (x_t, m_t, f_t): the same FP32 operations as
// the forward step rebuild g_t and y_{t+1}.
__device__ __forceinline__ void rel_a_point(float x, float m, float f, float bi, float lt,
                                            float eta, float alpha, float xbar_next,
                                            float mu_next2, float &mu, float &yb, double &se,
                                            double &sa, double &sl) {
    const float h = __fadd_rn(f, bi);
    const float g = __fadd_rn(__fmul_rn(lt, x), h);
    const float mn = __fsub_rn(__fmul_rn(alpha, m), __fmul_rn(eta, g));
    const float y = __fadd_rn(x, mn);
    yb = fabsf(y) <= 1.0f ? xbar_next : 0.0f;
    mu = __fadd_rn(yb, __fmul_rn(alpha, mu_next2));
    se += (double)mu * (double)(-g);
    sa += (double)mu * (double)m;
    sl += (double)mu * (-(double)eta * (double)x);
}

__device__ __forceinline__ float rel_b_point(float yb, float mu, float jmu, float lt, float eta) {
    return __fsub_rn(yb, __fmul_rn(eta, __fadd_rn(__fmul_rn(lt, mu), jmu)));
}

__device__ __forceinline__ double rel_wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Fixed-order sum over the workgroup's waves (nw of them), result in thread 0.
__device__ __forceinline__ double rel_group_sum(double v, double *sh, int nw) {
    v = rel_wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < nw; ++k) s += sh[k];
    return s;
}

// N consecutive floats as one access (N = 1 or 4, 4-float aligned).
template <int N> struct RelVec {
    float v[N];
    __device__ __forceinline__ void load(const float *p) {
        if constexpr (N == 4) {
            const float4 q = *reinterpret_cast<const float4 *>(p);
            v[0] = q.x, v[1] = q.y, v[2] = q.z, v[3] = q.w;
        } else {
            v[0] = *p;
        }
    }
    __device__ __forceinline__ void store(float *p) const {
        if constexpr (N == 4) *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
        else *p = v[0];
    }
};

// Element work of one launch on N consecutive replicas, the first `live` of them real;
// `acc` is the product (J v)_i when the mode has one.
template <int MODE, int N>
__device__ __forceinline__ void rel_element(const RelArgs &a, int64_t idx, int live,
                                            const float (&acc)[N], float bi, double &s0,
                                            double &s1, double &s2) {
    auto in = [&](const float *p) {
        RelVec<N> v{};
        if (live > 0) v.load(p + idx);
        return v;
    };
    if constexpr (MODE == REL_FWD) {
        RelVec<N> x = in(a.xi), m = in(a.mi), f;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            f.v[k] = k < live ? acc[k] : 0.0f;
            rel_fwd_point(acc[k], bi, a.lam[a.t_f], a.eta, a.alpha, x.v[k], m.v[k]);
            if (k >= live) x.v[k] = m.v[k] = 0.0f;
        }
        x.store(a.xo + idx);
        m.store(a.mo + idx);
        if (a.fo) f.store(a.fo + idx);
    } else if constexpr (MODE == REL_LOSS) {
        const RelVec<N> xi = in(a.xi);
        RelVec<N> xb;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            xb.v[k] = 0.0f;
            if (k < live) {
                const double x = xi.v[k], f = acc[k], b = bi;
                s0 += 0.5 * x * f + b * x;
                xb.v[k] = (float)(a.scale * (f + b));
            }
        }
        xb.store(a.xbar + idx);
    } else {
        RelVec<N> xn{}, mu_in = in(a.mu_in);
        if constexpr (MODE == REL_A) {
            xn.load(a.xbar + idx);
        } else {
            // B of the previous launch's step: xbar_t from ybar, mu_{t+1} and J mu_{t+1}
            const RelVec<N> yb = in(a.yb);
#pragma unroll
            for (int k = 0; k < N; ++k)
                xn.v[k] = k < live ? rel_b_point(yb.v[k], mu_in.v[k], acc[k], a.lam[a.t_f], a.eta)
                                   : 0.0f;
            if constexpr (MODE == REL_B) {
                xn.store(a.xbar + idx);
                return;
            }
        }
        const RelVec<N> sx = in(a.sx), sm = in(a.sm), sf = in(a.sf);
        RelVec<N> mu{}, yb{};
#pragma unroll
        for (int k = 0; k < N; ++k)
            if (k < live)
                rel_a_point(sx.v[k], sm.v[k], sf.v[k], bi, a.lam[a.t_a], a.eta, a.alpha,
                            xn.v[k], mu_in.v[k], mu.v[k], yb.v[k], s0, s1, s2);
        mu.store(a.mu_out + idx);
        yb.store(a.yb + idx);
    }
}

// Writes this workgroup's partial sums (thread 0 holds the group sums).
template <int MODE>
__device__ __forceinline__ void rel_write_partials(const RelArgs &a, int64_t wg, double s0,
                                                   double s1, double s2, double *sh, int nw) {
    if (MODE == REL_FWD || MODE == REL_B) return;
    const double g0 = rel_group_sum(s0, sh, nw);
    if (MODE == REL_LOSS) {
        if (threadIdx.x == 0) a.part[a.slot0 + wg] = g0 * a.scale;
        return;
    }
    const double g1 = rel_group_sum(s1, sh, nw);
    const double g2 = rel_group_sum(s2, sh, nw);
    if (threadIdx.x == 0) {
        a.part[a.slot0 + wg] = g0;
        a.part[a.nblk + a.slot0 + wg] = g1;
        a.part[2 * a.nblk + a.slot0 + wg] = g2;
    }
}

// Row launches: the CSR product with its input staged through LDS (the gather modes), and
// the element-wise pass (REL_A) over every instance's rows with the same work items, so
// that for sparse instances of one type a step's partial sums are grouped alike whichever
// launch computes them.  Work item
// = (block of 64 consecutive rows of one instance, 64-replica chunk c); a workgroup of 16
// waves takes its items in the order below.  Sixteen lanes own a row, four replicas each,
// so a wave owns four rows; the input vector (x or mu of the instance, the chunk's 64
// replicas) goes through LDS 256 columns at a time (one buffer of 64 KiB: a range is
// staged, then walked; the other workgroup on the compute unit walks while this one
// stages), and each row walks its entries whose column falls in the staged range, in
// ascending order, one fused multiply-add per term (the order of the definition), while
// each staged value serves all 64 rows of the block instead of one gather per entry.
// A row's entries come in windows of 64, 16 of them in a register across its lanes.  A step
// of the walk broadcasts one entry's LDS offset and weight within the row's lanes as DPP
// operands of the address addition and of a move, so a step serves an entry of each of the
// wave's rows with one 16-byte read and six vector instructions (four multiply-adds).
// Lanes whose row has no further entry in the range read a column of zeros with weight 0
// (which changes no sum).  The windows past the range's entries are loaded before the walk;
// with FEW entries per row and range most ranges hold none of a wave's, and it keeps its
// windows then (n = 20000, 8 entries a row, R = 16, 60 steps: 33.0 ms loading them again,
// 29.1 so; where nearly every range has some, the check costs 1 %).
// 96 ER QUBOs of 100 to 2000 variables (p = 0.1, 13.4 million entries), 64 replicas: 95 us
// a launch, against 230 with one row's entry per step (an address, a weight and a product
// for every entry) and items in the given order.  The 3.4 GB of staged values read at 128
// bytes a clock take 46 us, the padded entries and the staging bring that to 67, and the
// vector instructions alone take about 65.  (Eight waves a SIMD leave 64 registers: none are
// spilled for int16 couplings and columns, 2 to 4 for most other types.)
typedef __attribute__((address_space(3))) void lds_void;
constexpr int GR_THREADS = 1024, GR_WAVES = GR_THREADS / 64, GR_RPW = 4;
constexpr int GR_ROWS = GR_WAVES * GR_RPW;       // 64 rows per block
constexpr int GR_CW = 256;                       // staged columns per range
constexpr int GR_WIN = 4;                        // registers of 16 entries per row
static_assert(GR_ROWS == 64, "blocks of 64 rows");

typedef const __attribute__((address_space(1))) int32_t *gr_i32;

// A row's window as prepared for a range: LDS byte offsets and weights.
struct GrWalk {
    int32_t off[GR_WIN];
    float w[GR_WIN];

    // entry K of register Q of every row: lane K of each 16 broadcast within them
    template <int K> static __device__ __forceinline__ int32_t bcast(int32_t v) {
        return __builtin_amdgcn_mov_dpp(v, 0x150 + K, 0xf, 0xf, true);
    }
    template <int K>
    __device__ __forceinline__ void four(int q, const char *src, float (&acc)[4]) const {
        const float4 v0 = *reinterpret_cast<const float4 *>(src + bcast<K>(off[q]));
        const float4 v1 = *reinterpret_cast<const float4 *>(src + bcast<K + 1>(off[q]));
        const float4 v2 = *reinterpret_cast<const float4 *>(src + bcast<K + 2>(off[q]));
        const float4 v3 = *reinterpret_cast<const float4 *>(src + bcast<K + 3>(off[q]));
        add<K>(q, v0, acc);
        add<K + 1>(q, v1, acc);
        add<K + 2>(q, v2, acc);
        add<K + 3>(q, v3, acc);
    }
    template <int K>
    __device__ __forceinline__ void add(int q, const float4 &v, float (&acc)[4]) const {
        const float wk = __int_as_float(bcast<K>(__float_as_int(w[q])));
        acc[0] = __fmaf_rn(wk, v.x, acc[0]);
        acc[1] = __fmaf_rn(wk, v.y, acc[1]);
        acc[2] = __fmaf_rn(wk, v.z, acc[2]);
        acc[3] = __fmaf_rn(wk, v.w, acc[3]);
    }
};

// Two workgroups per CU (64 KiB of LDS each, 8 waves per SIMD): the walks are bound by
// the latency of their LDS reads, which the second workgroup's waves hide, as they hide
// each range's staging.
template <int MODE, typename TW, typename TI, bool FEW>
__global__ void __launch_bounds__(GR_THREADS)
    __attribute__((amdgpu_waves_per_eu(8))) k_rel_gather(const RelInst *__restrict__ insts,
                                                           int32_t ninst, int64_t blocks,
                                                           int32_t C, const RelArgs a) {
    constexpr bool GATHER = MODE != REL_A;
    typedef const __attribute__((address_space(1))) TW *gw_t;
    typedef const __attribute__((address_space(1))) TI *gi_t;
    // the staged columns and one of zeros
    __shared__ __attribute__((aligned(16))) float vs[GATHER ? (GR_CW + 1) * 64 : 1];
    __shared__ double sh[GR_WAVES];
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rl = lane >> 4, ln = lane & 15;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    const int64_t total = blocks * C;
    if (GATHER && threadIdx.x < 64) vs[GR_CW * 64 + threadIdx.x] = 0.0f;
    // items in chunks of P = (workgroups / 8) consecutive ones, eight chunks a round, one
    // per compute die (workgroup b runs on die b mod 8): the items a die runs at a time are
    // neighbouring blocks, mostly of one instance, whose input vector its L2 then holds
    // for all of them instead of every die fetching every instance's.  The table's items
    // come longest first, and every other round runs through them backwards, which evens
    // out the workgroups' shares (96 ER QUBOs, n = 100 to 2000: 115 us a launch with the
    // instances as given, 95 so).
    const int64_t P = gridDim.x >> 3;
    const int64_t me = (blockIdx.x & 7) * P + (blockIdx.x >> 3);
    for (int64_t round = 0; round * gridDim.x < total; ++round) {
        const int64_t it = round * gridDim.x + (round & 1 ? gridDim.x - 1 - me : me);
        if (it >= total) continue;
        const int64_t blk = it / C;
        const int c = (int)(it - blk * C);
        int lo = 0, hi = ninst - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (insts[mid].blk0 <= blk) lo = mid;
            else hi = mid - 1;
        }
        // the instance's fields, read once (a staging load may write memory as far as the
        // compiler knows, which would otherwise make it read them again)
        const RelInst &I = insts[lo];
        const int64_t n = I.n;
        const int64_t i = (blk - I.blk0) * GR_ROWS + GR_RPW * wv + rl;
        float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (GATHER) {
            const gr_i32 rp = (gr_i32)I.rp;
            const int32_t rp0 = rp[0];
            // (an instance without stored entries has nothing to gather: uniform per item)
            if (rp[n] > rp0) {
                const float *v = ((MODE == REL_FWD || MODE == REL_LOSS) ? a.xi : a.mu_in) +
                                 I.row0 * a.Rp + (int64_t)c * 64;
                const gi_t col = (gi_t)I.col;
                const gw_t w = (gw_t)I.w;
                const bool skip = I.skip_diag != 0;
                // staging of columns GR_CW q .. GR_CW q + GR_CW - 1 (past n: column n - 1
                // again, unused): thread t moves GR_CW / 64 pieces of 16 bytes, element
                // e = 1024 u + t = column e / 16 of the range, floats 4 (e % 16) .. + 3; a
                // wave's destinations are contiguous.  Addresses are the range's uniform
                // base plus 32-bit offsets.
                const uint32_t rp4 = (uint32_t)a.Rp;
                auto stage = [&](int q) {
                    const float *vq = v + (int64_t)q * GR_CW * a.Rp;
                    const uint32_t lim =
                        (uint32_t)min((int64_t)GR_CW - 1, n - 1 - (int64_t)q * GR_CW);
#pragma unroll
                    for (int u = 0; u < GR_CW / 64; ++u) {
                        const uint32_t e = 1024u * u + threadIdx.x;
                        const uint32_t o = __umul24(min(e >> 4, lim), rp4) + 4u * (e & 15u);
                        __builtin_amdgcn_global_load_lds(
                            vq + o, (lds_void *)(vs + 4 * (1024 * u + 64 * wv)), 16, 0, 0);
                    }
                };
                // the row's cursor and end, and its window as loaded (lanes past the row's
                // end hold some stored entry of the instance)
                int32_t kc = i < n ? rp[i] : rp0;
                const int32_t ke = i < n ? rp[i + 1] : rp0;
                const int32_t klast = max(ke - 1, rp0);
                TI wj[GR_WIN];
                TW ww[GR_WIN];
                auto load = [&]() {
#pragma unroll
                    for (int q = 0; q < GR_WIN; ++q) {
                        const int32_t kk = min(kc + 16 * q + ln, klast);
                        wj[q] = col[kk];
                        ww[q] = w[kk];
                    }
                };
                load();
                const char *src = reinterpret_cast<const char *>(vs) + 16 * ln;
                const int nq = (int)((n + GR_CW - 1) / GR_CW);
                for (int q = 0; q < nq; ++q) {
                    // every wave is done with range q - 1, then the buffer takes range q
                    // and every wave's part has landed
                    if (q > 0) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    stage(q);
                    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                    const int32_t base = q * GR_CW, bound = base + GR_CW;
                    bool more;
                    do {
                        GrWalk W;
                        int steps[GR_WIN];       // of the longest of the four rows
                        int cnt = 0;
#pragma unroll
                        for (int r = 0; r < GR_WIN; ++r) {
                            const int32_t j = (int32_t)wj[r];
                            const bool in = kc + 16 * r + ln < ke && j < bound;
                            const uint64_t bal = __ballot(in);
                            const uint32_t l = (uint32_t)bal, h = (uint32_t)(bal >> 32);
                            cnt += __popc(((rl & 2 ? h : l) >> (16 * (rl & 1))) & 0xFFFFu);
                            steps[r] = __popc(((l | h) | ((l | h) >> 16)) & 0xFFFFu);
                            W.off[r] = (in ? j - base : GR_CW) << 8;
                            // (a stored QUBO diagonal is folded into b: weight 0)
                            W.w[r] = in && !(skip && j == (int32_t)i) ? (float)ww[r] : 0.0f;
                        }
                        kc += cnt;
                        more = __ballot(cnt == 16 * GR_WIN) != 0;
                        if (FEW && steps[0] == 0) break;     // no entry: the windows stay
                        load();
#pragma unroll
                        for (int r = 0; r < GR_WIN; ++r) {
                            if (steps[r] == 0) break;
                            W.four<0>(r, src, acc);
                            if (steps[r] > 4) W.four<4>(r, src, acc);
                            if (steps[r] > 8) W.four<8>(r, src, acc);
                            if (steps[r] > 12) W.four<12>(r, src, acc);
                        }
                    } while (more);              // a row's window may end within the range
                }
                // every wave is done with the staging buffers before the next item loads
                // them
                __syncthreads();
            }
        }
        const int r0 = c * 64 + 4 * ln;
        if (i < n)
            rel_element<MODE, 4>(a, (I.row0 + i) * a.Rp + r0, min(max(a.R - r0, 0), 4), acc,
                                 I.b[i], s0, s1, s2);
    }
    rel_write_partials<MODE>(a, blockIdx.x, s0, s1, s2, sh, GR_WAVES);
}

// Epilogue of the dense product for every mode (b, and the state pointers in `a`,
// already offset to the instance's rows).
template <int MODE>
struct RelTileEpilogue {
    RelArgs a;
    const float *b;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    __device__ __forceinline__ void begin() const {}
    struct Pre {};
    __device__ __forceinline__ float bias(int64_t i) const { return b[i]; }
    __device__ __forceinline__ Pre load(int64_t, int64_t) const { return Pre{}; }
    __device__ __forceinline__ void point(float acc, float bi, int64_t r, int64_t idx,
                                          const Pre &) {
        const float v[1] = {acc};
        rel_element<MODE, 1>(a, idx, r < a.R ? 1 : 0, v, bi, s0, s1, s2);
    }
    __device__ __forceinline__ void finish() const {
        __shared__ double sh[8];
        rel_write_partials<MODE>(a, (int64_t)blockIdx.y * gridDim.x + blockIdx.x, s0, s1, s2,
                                 sh, (int)(blockDim.x >> 6));
    }
};

__global__ void __launch_bounds__(256) k_rel_fill(double *__restrict__ p, int64_t count) {
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < count;
         q += (int64_t)gridDim.x * blockDim.x)
        p[q] = 0.0;
}

// p[0] + p[1] + ... + p[n - 1], one after the other, in every lane of a wave; 64 are loaded
// together.  f(k) for each k that this lane loaded.
template <typename F>
__device__ __forceinline__ double rel_ordered_sum(const double *p, int32_t n, F &&f) {
    const int32_t lane = threadIdx.x & 63;
    auto load = [&](int32_t k) { return k + lane < n ? p[k + lane] : 0.0; };
    double sum = 0.0, next = load(0);
    for (int32_t k = 0; k < n; k += 64) {
        const double v = next;
        next = load(k + 64);
        if (k + lane < n) f(k + lane);
#pragma unroll
        for (int i = 0; i < 64; ++i)
            sum += __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), i),
                                    __builtin_amdgcn_readlane(__double2loint(v), i));
    }
    return sum;
}

// Sums of partial rows: wave (kind, row) adds its nblk slots and clears them.  Kind 0: d_eta
// terms, 1: d_alpha, 2: d_lambda.
__global__ void __launch_bounds__(64) k_rel_steps(int32_t t_first, int32_t nblk, double *part,
                                                  double *__restrict__ steps, int32_t T,
                                                  double *__restrict__ d_lam) {
    const int32_t kind = blockIdx.x, t = t_first - (int32_t)blockIdx.y;
    double *p = part + ((int64_t)blockIdx.y * 3 + kind) * nblk;
    const double sum = rel_ordered_sum(p, nblk, [&](int32_t k) { p[k] = 0.0; });
    if (threadIdx.x != 0) return;
    if (kind < 2) steps[(int64_t)kind * T + t] = sum;
    else if (d_lam) d_lam[t] = sum;
}

// Final sums, a wave each: the loss partials and the steps' terms.
__global__ void __launch_bounds__(64) k_rel_finish(int32_t T, int32_t nblk,
                                                   const double *__restrict__ steps,
                                                   const double *__restrict__ part_loss,
                                                   double *__restrict__ loss,
                                                   double *__restrict__ d_eta,
                                                   double *__restrict__ d_alpha) {
    const int32_t kind = blockIdx.x;
    double *out = kind == 0 ? loss : kind == 1 ? d_eta : d_alpha;
    if (!out) return;
    const double *p = kind == 0 ? part_loss : steps + (int64_t)(kind - 1) * T;
    const double sum = rel_ordered_sum(p, kind == 0 ? nblk : T, [](int32_t) {});
    if (threadIdx.x == 0) *out = sum;
}

template <typename F>
hipError_t rel_by_dtypes(int32_t wdt, int32_t idt, F &&f) {
    auto byw = [&](auto itag) -> hipError_t {
        switch (wdt) {
            case QPA_I8: return f((int8_t)0, itag);
            case QPA_I16: return f((int16_t)0, itag);
            case QPA_I32: return f((int32_t)0, itag);
            default: return f(0.0f, itag);
        }
    };
    return idt == QPA_I16 ? byw((int16_t)0) : byw((int32_t)0);
}

template <int MODE>
hipError_t rel_gather_launch(const RelInst *insts, int32_t ninst, int64_t blocks, int32_t C,
                             int32_t wdt, int32_t idt, bool few, const RelArgs &a, hipStream_t st) {
    const unsigned g = (unsigned)rel_gather_blocks(blocks, C);
    if (g % 8) return hipErrorInvalidValue;       // the item order assumes whole dies
    if (MODE == REL_A) {
        k_rel_gather<REL_A, float, int32_t, false><<<g, GR_THREADS, 0, st>>>(insts, ninst, blocks, C, a);
        return hipGetLastError();
    }
    return rel_by_dtypes(wdt, idt, [&](auto wtag, auto itag) {
        using TW = decltype(wtag);
        using TI = decltype(itag);
        if (few) k_rel_gather<MODE, TW, TI, true><<<g, GR_THREADS, 0, st>>>(insts, ninst, blocks, C, a);
        else k_rel_gather<MODE, TW, TI, false><<<g, GR_THREADS, 0, st>>>(insts, ninst, blocks, C, a);
        return hipGetLastError();
    });
}

template <int MODE>
hipError_t rel_tile_launch(int64_t n, const float *J, const float *b, const RelArgs &a,
                           hipStream_t st) {
    const RelTileEpilogue<MODE> epi{a, b};
    const float *q = (MODE == REL_FWD || MODE == REL_LOSS) ? a.xi : a.mu_in;
    return launch_fp32_product(n, a.Rp, J, q, epi, st);
}

}  // namespace

int64_t rel_gather_blocks(int64_t blocks, int32_t C) {
    int64_t g = (blocks * (int64_t)C + 7) / 8 * 8;          // a multiple of the 8 dies
    if (g > REL_GATHER_BLOCKS_MAX) g = REL_GATHER_BLOCKS_MAX;
    return g < 8 ? 8 : g;
}

hipError_t launch_rel_gather(int32_t mode, const RelInst *insts, int32_t ninst, int64_t blocks,
                             int32_t C, int32_t wdt, int32_t idt, bool few,
                             const RelArgs &a, hipStream_t st) {
    switch (mode) {
        case REL_FWD: return rel_gather_launch<REL_FWD>(insts, ninst, blocks, C, wdt, idt, few, a, st);
        case REL_LOSS: return rel_gather_launch<REL_LOSS>(insts, ninst, blocks, C, wdt, idt, few, a, st);
        case REL_A: return rel_gather_launch<REL_A>(insts, ninst, blocks, C, wdt, idt, few, a, st);
        case REL_B: return rel_gather_launch<REL_B>(insts, ninst, blocks, C, wdt, idt, few, a, st);
        case REL_BA: return rel_gather_launch<REL_BA>(insts, ninst, blocks, C, wdt, idt, few, a, st);
    }
    return hipErrorInvalidValue;
}

int64_t rel_tile_blocks(int64_t n, int64_t Rp) {
    const dim3 g = fp32_tile_grid(fp32_tile_of(n, Rp), n, Rp);
    return (int64_t)g.x * g.y;
}

hipError_t launch_rel_tiles(int32_t mode, int64_t n, const float *J, const float *b,
                            const RelArgs &a, hipStream_t st) {
    switch (mode) {
        case REL_FWD: return rel_tile_launch<REL_FWD>(n, J, b, a, st);
        case REL_LOSS: return rel_tile_launch<REL_LOSS>(n, J, b, a, st);
        case REL_B: return rel_tile_launch<REL_B>(n, J, b, a, st);
        case REL_BA: return rel_tile_launch<REL_BA>(n, J, b, a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_rel_fill(double *p, int64_t count, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    int64_t g = (count + 255) / 256;
    if (g > 1024) g = 1024;
    k_rel_fill<<<(unsigned)g, 256, 0, st>>>(p, count);
    return hipGetLastError();
}

hipError_t launch_rel_steps(int32_t t_first, int32_t rows, int32_t nblk, double *part,
                            double *steps, int32_t T, double *d_lam, hipStream_t st) {
    k_rel_steps<<<dim3(3, (unsigned)rows), 64, 0, st>>>(t_first, nblk, part, steps, T, d_lam);
    return hipGetLastError();
}

hipError_t launch_rel_finish(int32_t T, int32_t nblk, const double *steps,
                             const double *part_loss, double *loss, double *d_eta,
                             double *d_alpha, hipStream_t st) {
    k_rel_finish<<<3, 64, 0, st>>>(T, nblk, steps, part_loss, loss, d_eta, d_alpha);
    return hipGetLastError();
}

}  // namespace qpa
