// Binned sparse PA step (App. B field h = J s + b and the fused update) for CSR instances
// with integer couplings and at most 8 replicas.
//
// When the spin words of a large graph far exceed the L2 cache, the per-row gather of the
// streamed kernel pulls one cache line per coupling, about 16x the bytes of the CSR entry
// it serves.  Here the gather is split into two streaming passes over an entry order
// fixed once per run (propagation blocking):
//   source chunks: C = 2^20 / G variables, whose spin words (128 KiB) fit in LDS;
//   destination bins: B = 2^14 L / G rows, whose field sums fit in 2^14 words of LDS,
//     L = 4, 2 or 1 sums per word (8-, 16- or 32-bit lanes, chosen from the row bound);
//   entries (diagonal excluded for QUBO) ordered by (chunk, bin), any order inside a block.
//   pass 1, k_bin_gather: a workgroup loads the spin words of one chunk into LDS and, for
//     a contiguous share of the chunk's entries, writes the G spin bits of each entry's
//     column to bits[p];
//   pass 2, k_bin_update: a workgroup clears its sums in LDS and adds, for every entry of
//     its bin, |w| b' per replica with b' = b XOR [w < 0] (one LDS atomic per word of L
//     lanes); the field is then h = c - 2 A with A the replica's sum and c = sum |w| + b
//     per row (built once per call), since a term w (1 - 2b) equals |w| (1 - 2b').  Then
//     the fused update of its rows (x, m, spin words), the arithmetic of the streamed
//     kernel.  A lane of W bits never carries into the next: A <= sum |w| < 2^W.
// Integer sums are exact, so the order of the entries inside a block does not change a
// bit of the result, and (float)(c - 2A) equals the streamed kernel's (float)sum + b.
// Entries carry the column's offset in its chunk (uint32) and the row's offset in its bin
// with the weight (low / high 16 bits of a uint32).
#include "qpa_internal.h"

#include <type_traits>

namespace qpa {
namespace {

constexpr int BT = 1024;                 // threads per workgroup of every kernel here
constexpr int CHUNK_WORDS = 1 << 14;     // spin words (uint64) of one source chunk
constexpr int BIN_WORDS = 1 << 14;       // LDS words of field sums of one bin
constexpr int SCAN_TILE = 4 * BT;        // elements per workgroup of the offset scan

__device__ __forceinline__ void pa_update(float h, float lam, float eta, float alpha, float &x,
                                          float &m) {
    float g = __fadd_rn(__fmul_rn(lam, x), h);
    float mn = __fsub_rn(__fmul_rn(alpha, m), __fmul_rn(eta, g));
    float y = __fadd_rn(x, mn);
    y = fminf(1.0f, fmaxf(-1.0f, y));
    m = mn;
    x = y;
}

// Exclusive prefix sums of PER values per thread over a 1024-thread workgroup, in thread
// order; returns the workgroup total.  `wsum` holds 16 ints of LDS.
template <int PER>
__device__ int32_t block_scan_excl(int32_t (&v)[PER], int32_t *wsum) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t own = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int32_t t = v[u];
        v[u] = own;
        own += t;
    }
    int32_t inc = own;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(inc, d, 64);
        if (lane >= d) inc += y;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < BT / 64; ++w) {
        const int32_t s = wsum[w];
        before += w < wave ? s : 0;
        total += s;
    }
    __syncthreads();
    const int32_t base = before + inc - own;
#pragma unroll
    for (int u = 0; u < PER; ++u) v[u] += base;
    return total;
}

// The entries of a row in batches: their columns and weights are loaded together, then given
// to f in order (the diagonal left out where skip_diag).
template <typename TI, typename TW, typename F>
__device__ __forceinline__ void bin_row(int64_t i, const int32_t *__restrict__ rp,
                                        const TI *__restrict__ col, const TW *__restrict__ w,
                                        int skip_diag, F &&f) {
    constexpr int D = 4;
    const int64_t k1 = rp[i + 1];
    for (int64_t k = rp[i]; k < k1; k += D) {
        int64_t j[D];
        int32_t v[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int64_t kk = k + d < k1 ? k + d : k1 - 1;
            j[d] = (int64_t)col[kk];
            v[d] = w ? (int32_t)w[kk] : 0;
        }
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (k + d < k1 && !(skip_diag && j[d] == i)) f(j[d], v[d]);
    }
}

// Entries per (chunk, bin) block: one workgroup per bin, thread per row, the bin's Nc counts
// in LDS (dynamic).  Columns were validated in range.  n = 24 million, 72 million entries:
// 0.14 ms; 5.5 with an atomic on the block's count in memory for every entry.
template <typename TI>
__global__ void __launch_bounds__(BT) k_bin_count(int64_t n, const int32_t *__restrict__ rp,
                                                  const TI *__restrict__ col, int skip_diag,
                                                  int cshift, int bshift, int64_t Nc, int64_t Nb,
                                                  int32_t *__restrict__ cnt) {
    extern __shared__ int32_t own[];
    const int64_t bin = blockIdx.x;
    for (int64_t c = threadIdx.x; c < Nc; c += BT) own[c] = 0;
    __syncthreads();
    const int64_t end = (bin + 1) << bshift < n ? (bin + 1) << bshift : n;
    for (int64_t i = (bin << bshift) + threadIdx.x; i < end; i += BT)
        bin_row<TI, int8_t>(i, rp, col, nullptr, skip_diag,
                            [&](int64_t j, int32_t) { atomicAdd(&own[j >> cshift], 1); });
    __syncthreads();
    for (int64_t c = threadIdx.x; c < Nc; c += BT) cnt[c * Nb + bin] = own[c];
}

// Offset scan, step 1: the total of every SCAN_TILE-element tile.
__global__ void __launch_bounds__(BT) k_bin_tile_sums(const int32_t *__restrict__ cnt, int64_t M,
                                                      int32_t *__restrict__ tsum) {
    __shared__ int32_t wsum[BT / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * 4;
    int32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = base + u < M ? cnt[base + u] : 0;
    const int32_t tot = block_scan_excl<4>(v, wsum);
    if (threadIdx.x == 0) tsum[blockIdx.x] = tot;
}

// Step 2 (one workgroup): exclusive scan of the tile totals in place; off[M] = total.
__global__ void __launch_bounds__(BT) k_bin_scan_tiles(int32_t *__restrict__ tsum, int64_t nt,
                                                       int32_t *__restrict__ off, int64_t M) {
    __shared__ int32_t wsum[BT / 64];
    int32_t carry = 0;
    for (int64_t b0 = 0; b0 < nt; b0 += SCAN_TILE) {
        const int64_t base = b0 + (int64_t)threadIdx.x * 4;
        int32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = base + u < nt ? tsum[base + u] : 0;
        const int32_t tot = block_scan_excl<4>(v, wsum);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (base + u < nt) tsum[base + u] = v[u] + carry;
        carry += tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) off[M] = carry;
}

// Step 3: exclusive offsets of every block.
__global__ void __launch_bounds__(BT) k_bin_offsets(const int32_t *__restrict__ cnt, int64_t M,
                                                    const int32_t *__restrict__ tsum,
                                                    int32_t *__restrict__ off) {
    __shared__ int32_t wsum[BT / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * 4;
    int32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = base + u < M ? cnt[base + u] : 0;
    (void)block_scan_excl<4>(v, wsum);
    const int32_t t0 = tsum[blockIdx.x];
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (base + u < M) off[base + u] = v[u] + t0;
}

// Entries into their blocks (column offset in its chunk; row offset in its bin | weight) and
// the row constants c_i = sum over off-diagonal entries of |w| + b_i (exact integers).  One
// workgroup per bin, which alone writes the bin's blocks: their Nc cursors in LDS (dynamic).
// n = 24 million, 72 million entries: 0.91 ms; 7.3 with a cursor in memory for every block.
template <typename TI, typename TW>
__global__ void __launch_bounds__(BT) k_bin_scatter(int64_t n, const int32_t *__restrict__ rp,
                                                    const TI *__restrict__ col,
                                                    const TW *__restrict__ w, int skip_diag,
                                                    int cshift, int bshift, int64_t Nc,
                                                    int64_t Nb, const int32_t *__restrict__ off,
                                                    const int64_t *__restrict__ b_i64,
                                                    uint32_t *__restrict__ src,
                                                    uint32_t *__restrict__ drec,
                                                    int32_t *__restrict__ crow) {
    extern __shared__ int32_t cur[];
    const int64_t bin = blockIdx.x;
    for (int64_t c = threadIdx.x; c < Nc; c += BT) cur[c] = off[c * Nb + bin];
    __syncthreads();
    const uint32_t cmask = (uint32_t)((1ll << cshift) - 1);
    const int64_t i0 = bin << bshift, end = (bin + 1) << bshift < n ? (bin + 1) << bshift : n;
    for (int64_t i = i0 + threadIdx.x; i < end; i += BT) {
        int64_t c = b_i64[i];
        bin_row<TI, TW>(i, rp, col, w, skip_diag, [&](int64_t j, int32_t v) {
            const int32_t pos = atomicAdd(&cur[j >> cshift], 1);
            src[pos] = (uint32_t)j & cmask;
            drec[pos] = (uint32_t)(i - i0) | ((uint32_t)(uint16_t)(int16_t)v << 16);
            c += v < 0 ? -v : v;
        });
        crow[i] = (int32_t)c;
    }
}

// Four consecutive entry records or spin bytes, in one access from any entry.
typedef uint32_t rec4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t byte4 __attribute__((aligned(1)));

// Pass 1.  Grid (Nc, S): chunk c, share s of its entries, four consecutive ones per lane.
// An access that starts on one of the share's entries may run up to three entries past
// them: reads stay within the workspace (other arrays follow), writes are exact.
// n = 24 million, 72 million entries, G = 4: 81 us (99 with one entry per access).
__global__ void __launch_bounds__(BT) k_bin_gather(int shiftG, int64_t nwords, int64_t Nb,
                                                   const int32_t *__restrict__ off,
                                                   const uint32_t *__restrict__ src,
                                                   const uint64_t *__restrict__ s_cur,
                                                   uint8_t *__restrict__ bits) {
    __shared__ uint64_t words[CHUNK_WORDS];
    const int64_t c = blockIdx.x;
    const int64_t w0 = c * CHUNK_WORDS;
    const int64_t wn = nwords - w0 < CHUNK_WORDS ? nwords - w0 : CHUNK_WORDS;
#pragma unroll
    for (int u = 0; u < CHUNK_WORDS / BT; ++u) {
        const int64_t q = threadIdx.x + u * BT;
        if (q < wn) words[q] = s_cur[w0 + q];
    }
    const int64_t p0 = off[c * Nb], p1 = off[(c + 1) * Nb];
    const int64_t len = p1 - p0, S = gridDim.y;
    const int64_t a = p0 + len * (int64_t)blockIdx.y / S;
    const int64_t e = p0 + len * ((int64_t)blockIdx.y + 1) / S;
    __syncthreads();
    const int vsh = 6 - shiftG;
    const uint32_t vmask = (1u << vsh) - 1, gmask = (1u << (1 << shiftG)) - 1;
    constexpr int U = 4;
    for (int64_t p = a + 4 * threadIdx.x; p < e; p += (int64_t)4 * U * BT) {
        rec4 r[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = p + (int64_t)4 * u * BT;
            r[u] = 0u;
            if (q < e) r[u] = __builtin_nontemporal_load(reinterpret_cast<const rec4 *>(src + q));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = p + (int64_t)4 * u * BT;
            uint32_t out = 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                // an entry past the share may belong to a chunk of any size
                const uint32_t o = r[u][k] & ((uint32_t)CHUNK_WORDS << vsh) - 1u;
                const uint64_t word = words[o >> vsh];
                out |= ((uint32_t)(word >> ((o & vmask) << shiftG)) & gmask) << (8 * k);
            }
            if (q + 3 < e) {
                *reinterpret_cast<byte4 *>(bits + q) = out;
            } else {
                for (int k = 0; k < 4; ++k)
                    if (q + k < e) bits[q + k] = (uint8_t)(out >> (8 * k));
            }
        }
    }
}

// The L lanes of a word, from L bits: all ones in the lane of each set bit.
template <int L> __device__ __forceinline__ uint32_t lane_masks(uint32_t b) {
    if (L == 4) {
        const uint32_t s = __umul24(b, 0x00204081u) & 0x01010101u;
        return (s << 8) - s;
    }
    const uint32_t s = (b | (b << 15)) & 0x00010001u;
    return (s << 16) - s;
}

// Pass 2.  One workgroup per bin of B = BIN_WORDS L / G rows; dynamic LDS holds the run
// starts and lengths of the bin's Nc runs (2 (Nc + 1) int32), so that two workgroups share
// a compute unit and one's loads overlap the other's arithmetic.  A wave takes pieces of
// up to 256 consecutive entries of one run, four per lane, and finds a piece's run by
// comparing 64 runs' piece counts at once (one LDS read; its pieces only grow).  The
// update takes four consecutive (row, replica) pairs per lane.
// n = 24 million, 3 entries a row, G = 4: 360 us (439 with one entry and one pair per access
// and a search of the run per entry), of which the 1.6 GB of the update alone are 311 and
// the entries alone 94: the two workgroups of a compute unit overlap little, as they run
// the same phases at the same time.  Non-temporal entry loads (here and in pass 1) leave
// the last-level cache to the spin bytes: 446 us a step against 473.
template <int L>
__global__ void __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(8))) k_bin_update(
    int64_t n, int shiftG, int64_t Nb, int64_t Nc, int64_t nwords,
    const int32_t *__restrict__ off, const uint8_t *__restrict__ bits,
    const uint32_t *__restrict__ drec, const int32_t *__restrict__ crow,
    uint64_t *__restrict__ s_nxt, float *__restrict__ x, float *__restrict__ m,
    float *__restrict__ h_last, int t, const float *__restrict__ lam, float eta, float alpha) {
    constexpr int LW = 32 / L;                          // lane width in bits
    constexpr int SUMS = BIN_WORDS * L;                 // (row, replica) sums of a bin
    __shared__ __attribute__((aligned(16))) uint32_t acc[BIN_WORDS];
    __shared__ int32_t wsum[BT / 64];
    extern __shared__ int32_t runs[];
    int32_t *st = runs;               // start of the run of chunk c
    // pieces of the bin before chunk c's run, times 256, plus the run's length - 1 mod 256
    // (at most 2^23 + Nc pieces)
    uint32_t *pre = reinterpret_cast<uint32_t *>(runs + Nc + 1);
    const int64_t bin = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int G = 1 << shiftG;
    const int WPE = G / L;            // words of one entry (L <= G)
    const uint32_t gmask = (1u << G) - 1;
    // run of chunk c in this bin: [off[c*Nb + bin], off[c*Nb + bin + 1])
    int32_t v[2], last[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int64_t c = 2 * tid + u;
        v[u] = last[u] = 0;
        if (c < Nc) {
            const int32_t a0 = off[c * Nb + bin];
            st[c] = a0;
            const int32_t len = off[c * Nb + bin + 1] - a0;
            v[u] = (len + 255) >> 8;
            last[u] = (len + 255) & 255;
        }
    }
    for (int q = 4 * tid; q < BIN_WORDS; q += 4 * BT)
        *reinterpret_cast<uint4 *>(acc + q) = make_uint4(0u, 0u, 0u, 0u);
    const int32_t total = block_scan_excl<2>(v, wsum);
#pragma unroll
    for (int u = 0; u < 2; ++u)
        if (2 * tid + u < Nc) pre[2 * tid + u] = ((uint32_t)v[u] << 8) | (uint32_t)last[u];
    if (tid == 0) pre[Nc] = (uint32_t)total << 8;
    __syncthreads();
    auto add = [&](uint32_t rec, uint32_t b) {
        const int32_t wv = (int32_t)rec >> 16;
        const uint32_t aw = (uint32_t)(wv < 0 ? -wv : wv);
        const uint32_t fb = b ^ (wv < 0 ? gmask : 0u);            // b' of each replica
        uint32_t *a = acc + ((rec & 0xffffu) << shiftG) / L;
        if (L == 1) {
            for (int r = 0; r < G; ++r)
                if ((fb >> r) & 1u) atomicAdd(a + r, aw);
        } else {
            // |w| in every lane (below 2^LW, as the row's sum is)
            const uint32_t rep = L == 4 ? __umul24(aw, 0x00010101u) | aw << 24 : aw | aw << 16;
            for (int k = 0; k < WPE; ++k)
                atomicAdd(a + k, rep & lane_masks<L>((fb >> (k * L)) & ((1u << L) - 1)));
        }
    };
    int32_t c0 = 0;                   // a chunk whose run does not begin after the piece
    constexpr int U = 2;
    for (int32_t k0 = wave; k0 < total; k0 += U * (BT / 64)) {
        rec4 rec[U];
        uint32_t bv[U];
        int nv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t k = k0 + u * (BT / 64);
            nv[u] = 0;
            rec[u] = 0u;
            bv[u] = 0u;
            if (k >= total) continue;
            // the run of piece k: the last chunk c with pre[c] <= k (pre[Nc] = total > k)
            uint32_t pl;
            int adv;
            for (;;) {
                const int32_t c = c0 + lane;
                pl = c <= (int32_t)Nc ? pre[c] : UINT32_MAX;
                adv = __popcll(__ballot((pl >> 8) <= (uint32_t)k)) - 1;
                if (adv < 63) break;
                c0 += 63;
            }
            const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int32_t)pl, adv);
            const uint32_t next = (uint32_t)__builtin_amdgcn_readlane((int32_t)pl, adv + 1);
            c0 += adv;
            const int32_t cnt = (uint32_t)k + 1u == next >> 8 ? (int32_t)(first & 255u) + 1 : 256;
            nv[u] = cnt - 4 * lane;
            if (nv[u] > 0) {
                const int64_t p = (int64_t)st[c0] + 256 * (int64_t)((uint32_t)k - (first >> 8)) + 4 * lane;
                rec[u] = __builtin_nontemporal_load(reinterpret_cast<const rec4 *>(drec + p));
                bv[u] = *reinterpret_cast<const byte4 *>(bits + p);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k < nv[u]) add(rec[u][k], (bv[u] >> (8 * k)) & 0xffu);
    }
    __syncthreads();
    // fused update of the bin's (row, replica) pairs; state index = row * G + replica, four
    // consecutive ones per lane, UQ times per round: every load of a round is issued before
    // its stores.  x and m stream through once per step (gigabytes, far beyond the caches):
    // their loads and stores are non-temporal, leaving the caches to the entry records.
    constexpr int UQ = 2;
    static_assert(SUMS % (4 * BT * UQ) == 0, "rounds must cover the bin exactly");
    typedef float f4 __attribute__((ext_vector_type(4)));
    const int64_t q0 = bin * SUMS, pairs = n << shiftG;
    const float lt = lam[t];
    uint32_t *s32 = reinterpret_cast<uint32_t *>(s_nxt);
    for (int qb = 4 * tid; qb < SUMS; qb += 4 * UQ * BT) {
        f4 xv[UQ], mv[UQ];
        int32_t cr[UQ][4];
#pragma unroll
        for (int u = 0; u < UQ; ++u) {
            const int64_t gi = q0 + qb + 4 * u * BT;
            xv[u] = mv[u] = 0.0f;
            if (gi + 3 < pairs) {
                xv[u] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(x + gi));
                mv[u] = __builtin_nontemporal_load(reinterpret_cast<const f4 *>(m + gi));
                if (shiftG >= 2) {
                    cr[u][0] = cr[u][1] = cr[u][2] = cr[u][3] = crow[gi >> shiftG];
                } else if (shiftG == 1) {
                    cr[u][0] = cr[u][1] = crow[gi >> 1];
                    cr[u][2] = cr[u][3] = crow[(gi >> 1) + 1];
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k) cr[u][k] = crow[gi + k];
                }
            } else {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    cr[u][k] = 0;
                    if (gi + k < pairs) {
                        xv[u][k] = x[gi + k];
                        mv[u][k] = m[gi + k];
                        cr[u][k] = crow[(gi + k) >> shiftG];
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < UQ; ++u) {
            const int q = qb + 4 * u * BT;
            const int64_t gi = q0 + q;
            uint32_t neg = 0u;
            f4 hv;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t wd = acc[(q + k) / L];
                const int32_t A = (int32_t)(
                    L == 1 ? wd : (wd >> (LW * (k % L))) & ((1u << (LW % 32)) - 1u));
                hv[k] = (float)(cr[u][k] - 2 * A);
                float xk = xv[u][k], mk = mv[u][k];
                pa_update(hv[k], lt, eta, alpha, xk, mk);
                xv[u][k] = xk;
                mv[u][k] = mk;
                neg |= (xk < 0.0f && gi + k < pairs ? 1u : 0u) << k;
            }
            if (gi + 3 < pairs) {
                __builtin_nontemporal_store(xv[u], reinterpret_cast<f4 *>(x + gi));
                __builtin_nontemporal_store(mv[u], reinterpret_cast<f4 *>(m + gi));
                if (h_last) *reinterpret_cast<f4 *>(h_last + gi) = hv;
            } else {
                for (int k = 0; k < 4; ++k)
                    if (gi + k < pairs) {
                        x[gi + k] = xv[u][k];
                        m[gi + k] = mv[u][k];
                        if (h_last) h_last[gi + k] = hv[k];
                    }
            }
            // the bits of eight lanes (32 pairs) in the first of them
            auto from = [](uint32_t w, auto ctrl) {
                return (uint32_t)__builtin_amdgcn_mov_dpp((int)w, decltype(ctrl)::value, 0xf, 0xf,
                                                          true);
            };
            neg |= from(neg, std::integral_constant<int, 0x101>{}) << 4;      // lane + 1
            neg |= from(neg, std::integral_constant<int, 0x102>{}) << 8;      // lane + 2
            neg |= from(neg, std::integral_constant<int, 0x104>{}) << 16;     // lane + 4
            if ((lane & 7) == 0 && (gi >> 6) < nwords) s32[gi >> 5] = neg;
        }
    }
}

int ilog2(int64_t v) {
    int s = 0;
    while (((int64_t)1 << s) < v) ++s;
    return s;
}

}  // namespace

bool bin_geometry(int64_t n, int G, int lanes, BinGeom &g) {
    if (G < 1 || G > 8 || (G & (G - 1)) != 0 || n < 1) return false;
    if (lanes != 1 && lanes != 2 && lanes != 4) return false;
    if (lanes > G) return false;
    g.G = G;
    g.lanes = lanes;
    g.shiftG = ilog2(G);
    g.cshift = 20 - g.shiftG;                    // C * G / 64 = CHUNK_WORDS
    g.bshift = 14 + ilog2(lanes) - g.shiftG;     // B * G = BIN_WORDS * lanes
    g.Nc = (n + ((int64_t)1 << g.cshift) - 1) >> g.cshift;
    g.Nb = (n + ((int64_t)1 << g.bshift) - 1) >> g.bshift;
    g.M = g.Nc * g.Nb;
    return g.Nc <= BIN_MAX_CHUNKS && g.M < ((int64_t)1 << 31) - SCAN_TILE;
}

int64_t bin_scan_tiles(const BinGeom &g) { return (g.M + SCAN_TILE - 1) / SCAN_TILE; }

hipError_t launch_bin_build(const CsrView &c, const BinGeom &g, const int64_t *b_i64,
                            int32_t *off, int32_t *cnt, int32_t *tsum, uint32_t *src,
                            uint32_t *drec, int32_t *crow, hipStream_t st) {
    const unsigned nb = (unsigned)g.Nb;
    const size_t lds = sizeof(int32_t) * (size_t)g.Nc;
    auto byi = [&](auto itag) -> hipError_t {
        using TI = decltype(itag);
        const TI *col = static_cast<const TI *>(c.col);
        k_bin_count<TI><<<nb, BT, lds, st>>>(c.n, c.rp, col, c.skip_diag, g.cshift, g.bshift,
                                             g.Nc, g.Nb, cnt);
        hipError_t e2 = hipGetLastError();
        if (e2 != hipSuccess) return e2;
        const int64_t nt = bin_scan_tiles(g);
        k_bin_tile_sums<<<(unsigned)nt, BT, 0, st>>>(cnt, g.M, tsum);
        k_bin_scan_tiles<<<1, BT, 0, st>>>(tsum, nt, off, g.M);
        k_bin_offsets<<<(unsigned)nt, BT, 0, st>>>(cnt, g.M, tsum, off);
        e2 = hipGetLastError();
        if (e2 != hipSuccess) return e2;
        auto scatter = [&](auto wtag) {
            using TW = decltype(wtag);
            k_bin_scatter<TI, TW><<<nb, BT, lds, st>>>(c.n, c.rp, col,
                                                       static_cast<const TW *>(c.w), c.skip_diag,
                                                       g.cshift, g.bshift, g.Nc, g.Nb, off,
                                                       b_i64, src, drec, crow);
        };
        if (c.w_dt == QPA_I8) scatter((int8_t)0);
        else scatter((int16_t)0);
        return hipGetLastError();
    };
    if (c.w_dt != QPA_I8 && c.w_dt != QPA_I16) return hipErrorInvalidValue;
    return c.col_dt == QPA_I16 ? byi((int16_t)0) : byi((int32_t)0);
}

hipError_t launch_bin_step(const BinGeom &g, int64_t n, int64_t nnz, int64_t nwords,
                           const int32_t *off,
                           const uint32_t *src, const uint32_t *drec, uint8_t *bits,
                           const int32_t *crow, const uint64_t *s_cur, uint64_t *s_nxt, float *x,
                           float *m, float *h_last, int32_t t, const float *lam, float eta,
                           float alpha, int cus, hipStream_t st) {
    // shares of a chunk's entries: the count with the least work per compute unit, one
    // workgroup each at a time, where every share also loads the chunk's 128 KiB of words
    // (an entry moves 5 bytes)
    const double fixed = 131072.0 * (double)g.Nc / (5.0 * (double)(nnz > 0 ? nnz : 1));
    int64_t S = 1;
    double best = 0.0;
    for (int64_t q = 1; q <= 64; ++q) {
        const double work = (double)((g.Nc * q + cus - 1) / cus) * (1.0 / (double)q + fixed);
        if (q == 1 || work < best) {
            best = work;
            S = q;
        }
    }
    k_bin_gather<<<dim3((unsigned)g.Nc, (unsigned)S), BT, 0, st>>>(g.shiftG, nwords, g.Nb, off,
                                                                   src, s_cur, bits);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = sizeof(int32_t) * 2 * (size_t)(g.Nc + 1);
    const unsigned nb = (unsigned)g.Nb;
    if (g.lanes == 4)
        k_bin_update<4><<<nb, BT, lds, st>>>(n, g.shiftG, g.Nb, g.Nc, nwords, off, bits, drec,
                                             crow, s_nxt, x, m, h_last, t, lam, eta, alpha);
    else if (g.lanes == 2)
        k_bin_update<2><<<nb, BT, lds, st>>>(n, g.shiftG, g.Nb, g.Nc, nwords, off, bits, drec,
                                             crow, s_nxt, x, m, h_last, t, lam, eta, alpha);
    else
        k_bin_update<1><<<nb, BT, lds, st>>>(n, g.shiftG, g.Nb, g.Nc, nwords, off, bits, drec,
                                             crow, s_nxt, x, m, h_last, t, lam, eta, alpha);
    return hipGetLastError();
}

}  // namespace qpa
