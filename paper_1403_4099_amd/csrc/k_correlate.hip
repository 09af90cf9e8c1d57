// Correlation (Eq. 7 of Section 2.2.3) and the BF16 hi + lo split of C.
//
//   row stats : mean_i and s_i = sum_t (R_it - mean_i)^2 (two passes, FP64)
//   corr      : C_ij = sum_t x_it x_jt / sqrt(s_i s_j): FP64 MFMA Gram on 128 x 128
//               output tiles of the upper triangle (t split into slices), x =
//               R - mean staged through LDS; the slices added in order, C_ii =
//               1, clamp to [-1, 1], zero-variance stocks get 0 off the
//               diagonal, mirrored store, and the split of the values written
//   small     : the same in one launch, a workgroup per 16 x 16 output tile
//   split     : hi = bf16(C), lo = bf16(C - hi), round to nearest even from
//               FP64, zero padding up to the 32-aligned leading dimension
//   ewma      : online exponentially weighted correlation with the market
//               mode removed (pre-processing step before the path)
#include "pga_internal.hpp"

#include <math.h>

#include <type_traits>

namespace pga {

// Sum over a workgroup of 256 threads, the same bits in every thread; red: 4 doubles.
__device__ __forceinline__ double block_sum256(double v, double *red) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const double r = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return r;
}

// Bound by the read of R. The first CACHE samples of a thread stay in registers between the two passes (all of a row
// up to T = 256 CACHE), so R is read once; the slots that a short row leaves empty cost their instructions, so it
// has few (T = 40: N = 2048 6.3 us with 16 of them, 5.0 with one; N = 4096 9.5 and 7.2). The mean is taken
// of the differences to the row's first sample, so a constant row has variance exactly 0.
template <int CACHE>
__global__ __launch_bounds__(256) void k_row_stats(const double *R, int T, int64_t ld, double *mu,
                                                   double *ss, int32_t *status) {
    __shared__ double red[4];
    const int i = blockIdx.x;
    const double *__restrict__ row = R + (size_t)i * ld;
    const double x0 = row[0];
    double x[CACHE];
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < CACHE; ++u) {
        const int t = threadIdx.x + 256 * u;
        x[u] = t < T ? row[t] : x0;
    }
#pragma unroll
    for (int u = 0; u < CACHE; ++u) s += x[u] - x0;
    for (int t = threadIdx.x + 256 * CACHE; t < T; t += 256) s += row[t] - x0;
    const double m = x0 + block_sum256(s, red) / (double)T;
    double q = 0.0;
#pragma unroll
    for (int u = 0; u < CACHE; ++u) {
        const double d = threadIdx.x + 256 * u < T ? x[u] - m : 0.0;
        q = fma(d, d, q);
    }
    for (int t = threadIdx.x + 256 * CACHE; t < T; t += 256) {
        const double d = row[t] - m;
        q = fma(d, d, q);
    }
    q = block_sum256(q, red);
    if (threadIdx.x == 0) {
        mu[i] = m;
        ss[i] = q;
        if (q == 0.0 && status) atomicAdd(&status[PGA_ST_ZEROVAR], 1);
    }
}

// Round an FP64 value to the nearest bfloat16 value (ties to even) in one
// step, by integer arithmetic on the FP64 bit pattern: keep the top 7 of
// the 52 stored mantissa bits with round-half-even on the 45 dropped bits.
// Below 2^-126 bfloat16 is subnormal with spacing 2^-133: there the value is
// scaled by 2^133, rounded to an integer (rint is half-even) and scaled back.
__device__ __forceinline__ double bf16_round(double x) {
    if (x == 0.0 || !isfinite(x)) return x;
    unsigned long long u = (unsigned long long)__double_as_longlong(x);
    const int bexp = (int)((u >> 52) & 0x7FF);
    if (bexp >= 1023 - 126) {
        const unsigned long long lsb = (u >> 45) & 1ull;
        u += (1ull << 44) - 1ull + lsb;
        u &= ~((1ull << 45) - 1ull);
        return __longlong_as_double((long long)u);
    }
    return rint(x * 0x1p133) * 0x1p-133;
}

__device__ __forceinline__ uint16_t bf16_bits(double r) {
    return (uint16_t)(__float_as_uint((float)r) >> 16);
}

// Where C goes: C itself and, with hi, its BF16 split (ld x ld, zero past N).
struct CorrOut {
    double *C;
    uint16_t *hi, *lo;
    int N, ld;               // ld: split_ld(N) with hi, else N
};
__device__ __forceinline__ void corr_store(const CorrOut &o, int i, int j, double v) {
    if (i < o.N && j < o.N) o.C[(size_t)i * o.N + j] = v;
    if (o.hi && i < o.ld && j < o.ld) {
        const double h = bf16_round(v);
        o.hi[(size_t)i * o.ld + j] = bf16_bits(h);
        o.lo[(size_t)i * o.ld + j] = bf16_bits(bf16_round(v - h));
    }
}
CorrOut corr_out(double *C, int N, uint16_t *hi, uint16_t *lo) {
    return CorrOut{C, hi, lo, N, hi ? split_ld(N) : N};
}

// ---- Gram matrix on FP64 MFMA ----------------------------------------------------
// G_ij = sum_t x_it x_jt over the upper triangle of 128 x 128 output tiles,
// each tile's t range split into S slices (gram_split: at most one workgroup
// per CU), one workgroup per (tile, slice):
//   * the workgroup stages x of its 128 + 128 rows, 32 samples at a time, in
//     LDS (two buffers: the next chunk's global loads are in flight while the
//     current one is multiplied, 128 MFMAs per SIMD and chunk, enough to cover a
//     memory latency); x = R - mean of the row for the correlation, the
//     weighted sw_t (R - m_t) for the EWMA covariance;
//   * wave w of eight owns the 32 x 64 part (w / 2, w % 2) of the tile: eight
//     16 x 16 blocks, each accumulated by v_mfma_f64_16x16x4_f64 (lane l
//     supplies A[l % 16][l / 16] and B[l / 16][l % 16]: row l % 16 of A and
//     column l % 16 of B at the samples t0 + 8 h + 2 (l / 16) + v, h = 0..3,
//     v = 0, 1, one (h, v) per MFMA, so both operands see the same t, and a
//     slice's last chunk stops after the last h that holds a sample);
//   * the slice's 128 x 128 partial Gram goes to the workspace; a finish kernel
//     (one workgroup per 32 x 32 block of a tile) adds the S slices in slice
//     order (a fixed order: the result does not depend on timing), applies the
//     normalisation and writes the block and its mirror image through LDS,
//     both coalesced.
// A 128 x 128 tile moves half the bytes per flop of a 64 x 64 one: at N = 1024,
// T = 4096 the rows of R are read from the shared caches about 9 times in all.
typedef double gram_d4 __attribute__((ext_vector_type(4)));
typedef double gram_d2 __attribute__((ext_vector_type(2)));

constexpr int kGT = 128;                // output tile edge
constexpr int kGThreads = 512;          // eight waves, two per SIMD
constexpr int kGR = 32, kGC = 64;       // rows and columns of one wave's part
constexpr int kGK = 32;                 // samples per staged chunk
constexpr int kGS = kGK / 2;            // staging threads per row, two samples each
constexpr int kGPad = kGK + 2;          // LDS row stride (doubles): 16-byte aligned rows, spread banks
constexpr int kGMaxSplit = 16;

int gram_tiles(int N) {
    const int nt = (N + kGT - 1) / kGT;
    return nt * (nt + 1) / 2;
}

// Slices per tile for a given N (upper bound) and, with T known, the slices used: as many as keep all workgroups
// resident at once (one per CU: the LDS of one leaves no room for a second), at most kGMaxSplit, and at least 64
// samples per slice. One slice more and a few workgroups start a second round, as long as the first: a correlation
// call at N = 1307 (66 tiles), T = 2000 takes 151 us with 3 slices, 205 with 4; at T = 295, where slices also
// end at a quarter of a chunk instead of a whole one, the Gram takes 26 us against 42. Above 128 tiles the
// rule gives one slice whatever the rounds, which is not the best: their number over the slices sets the time there.
// N = 2048 (136 tiles), T = 4096: 624 us with one slice, 626 / 437 / 488 with two / three / four; N = 2900 (276
// tiles): 1238, 947 / 861 / 822. At T = 300 a slice's partial tiles cost what it gains: N = 2048 77, 82 / 70 / 81.
int gram_split_max(int N) {
    const int S = 256 / gram_tiles(N);
    return S < 1 ? 1 : (S > kGMaxSplit ? kGMaxSplit : S);
}

int gram_split(int N, int T) {
    int S = gram_split_max(N);
    const int by_t = T / 64 > 1 ? T / 64 : 1;
    return S < by_t ? S : by_t;
}

size_t gram_ws_doubles(int N) { return (size_t)gram_tiles(N) * gram_split_max(N) * kGT * kGT; }

// Tile u of the upper triangle, row-major: (ti, tj) with ti <= tj.
__device__ __forceinline__ void gram_tile_ij(int u, int nt, int &ti, int &tj) {
    ti = 0;
    while (u >= nt - ti) {
        u -= nt - ti;
        ++ti;
    }
    tj = ti + u;
}

template <bool EWMA>
__global__ __launch_bounds__(kGThreads) void k_gram_mfma(const double *X, int N, int T, int64_t ld, const double *mu,
                                                         const double *sw, int nt, int tiles, int S, double *part) {
    __shared__ __align__(16) double sA[2][kGT * kGPad];
    __shared__ __align__(16) double sB[2][kGT * kGPad];
    const int total = tiles * S;
    const int unit = xcd_tile(blockIdx.x, total);           // each XCD: a contiguous range of units
    const int slice = unit / tiles, tile = unit - slice * tiles;
    int ti, tj;
    gram_tile_ij(tile, nt, ti, tj);
    const int i0 = ti * kGT, j0 = tj * kGT;
    const int per = ((T + S - 1) / S + 7) / 8 * 8;          // samples per slice, whole quarters of a chunk
    const int ts = slice * per;
    const int te = min(T, ts + per);

    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    // staging: thread t takes samples 2 (t % 16), +1 of rows t / 16 + 32 e (e = 0..3) of each
    // panel, so 16 threads read a row's 32-sample segment and a load instruction of a wave
    // covers four rows
    const int srow = tid / kGS, scol = 2 * (tid % kGS);
    // Loads take clamped (always valid) addresses and the value is zeroed afterwards where the row is
    // past N or the sample past the slice (a clamped address repeats an element of the same row or
    // of row N - 1, whose entries are discarded), so every load is issued unconditionally and
    // together with the others.
    constexpr int kE = kGT * kGS / kGThreads;                  // rows of each panel per thread
    double muA[kE], muB[kE];
    int rowA[kE], rowB[kE];
    uint32_t valid = 0;                                      // bit e: row e of A; bit 4 + e: of B
#pragma unroll
    for (int e = 0; e < kE; ++e) {
        const int ra = i0 + kGThreads / kGS * e + srow, rb = j0 + kGThreads / kGS * e + srow;
        rowA[e] = min(ra, N - 1);
        rowB[e] = min(rb, N - 1);
        muA[e] = EWMA ? 0.0 : mu[rowA[e]];
        muB[e] = EWMA ? 0.0 : mu[rowB[e]];
        valid |= (ra < N ? 1u : 0u) << e;
        valid |= (rb < N ? 1u : 0u) << (4 + e);
    }
    // The raw values are loaded first and only used when they are stored into LDS, after the
    // current chunk's MFMAs have been issued, so the loads' latency is hidden behind them.
    double va[kE][2], vb[kE][2];
    double mt[2], wt[2];                                     // EWMA: the samples' market means and weight roots
    bool tin0 = false, tin1 = false;
    auto load = [&](int t0) {
        const int t = t0 + scol;
        tin0 = t < te;
        tin1 = t + 1 < te;
        const int tc0 = min(t, te - 1), tc1 = min(t + 1, te - 1);
        if constexpr (EWMA) {
            mt[0] = mu[tc0];
            mt[1] = mu[tc1];
            wt[0] = sw[tc0];
            wt[1] = sw[tc1];
        }
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            va[e][0] = X[(size_t)rowA[e] * ld + tc0];
            va[e][1] = X[(size_t)rowA[e] * ld + tc1];
            vb[e][0] = X[(size_t)rowB[e] * ld + tc0];
            vb[e][1] = X[(size_t)rowB[e] * ld + tc1];
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int e = 0; e < kE; ++e) {
            const bool a = (valid >> e) & 1u, b = (valid >> (4 + e)) & 1u;
            double *pa = &sA[buf][(kGThreads / kGS * e + srow) * kGPad + scol];
            double *pb = &sB[buf][(kGThreads / kGS * e + srow) * kGPad + scol];
            auto x = [&](double v, double mean, int h) { return EWMA ? wt[h] * (v - mt[h]) : v - mean; };
            pa[0] = (tin0 && a) ? x(va[e][0], muA[e], 0) : 0.0;
            pa[1] = (tin1 && a) ? x(va[e][1], muA[e], 1) : 0.0;
            pb[0] = (tin0 && b) ? x(vb[e][0], muB[e], 0) : 0.0;
            pb[1] = (tin1 && b) ? x(vb[e][1], muB[e], 1) : 0.0;
        }
    };

    const int qr = wave >> 1, qc = wave & 1;
    const int m = lane & 15, kq = lane >> 4;
    gram_d4 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = gram_d4{0.0, 0.0, 0.0, 0.0};

    // Two buffers of 32 samples, one barrier per chunk: the next chunk's loads are issued first, its
    // store comes before the last quarter of the MFMAs, so that the store's vector work of one
    // wave of a SIMD runs beside the MFMAs of the other. Each quarter's operands are read during
    // the quarter before. (N = 1024, T = 4096: 104 us, against 114 with four waves and 16-sample
    // chunks; 63 us of it are the MFMAs at their rate, without store and loads it runs 96. Three
    // buffers of 16 samples with the operands read across the barrier: 105.)
    constexpr int kQ = kGK / 8;                              // sample pairs per lane and chunk
    gram_d2 xa[2][2], xb[2][4];
    auto read = [&](int h, int buf) {                        // this lane's two of the eight samples 8h..8h + 7
#pragma unroll
        for (int a = 0; a < 2; ++a)
            xa[h & 1][a] = *(const gram_d2 *)&sA[buf][(kGR * qr + 16 * a + m) * kGPad + 8 * h + 2 * kq];
#pragma unroll
        for (int b = 0; b < 4; ++b)
            xb[h & 1][b] = *(const gram_d2 *)&sB[buf][(kGC * qc + 16 * b + m) * kGPad + 8 * h + 2 * kq];
    };
    auto mul = [&](int h) {
#pragma unroll
        for (int v = 0; v < 2; ++v)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[h & 1][a][v], xb[h & 1][b][v], acc[a][b], 0, 0, 0);
    };
    if (ts < te) {
        load(ts);
        store(0);
    }
    __syncthreads();
    int buf = 0, t0 = ts;
    for (; t0 + kGK < te; t0 += kGK) {
        load(t0 + kGK);
        read(0, buf);
#pragma unroll
        for (int h = 0; h < kQ; ++h) {
            if (h + 1 < kQ) read(h + 1, buf);
            if (h + 1 == kQ) store(buf ^ 1);
            mul(h);
        }
        __syncthreads();
        buf ^= 1;
    }
    read(0, buf);                                            // the last chunk: its quarters that hold samples
#pragma unroll
    for (int h = 0; h < kQ; ++h) {
        if (t0 + 8 * h >= te) break;
        if (h + 1 < kQ) read(h + 1, buf);
        mul(h);
    }
    // Where each accumulator register sits in its 16 x 16 block is read off the hardware: one
    // MFMA with A[i][0] = i, B[0][j] = 1 (zero for k > 0) gives every register its row i, one with
    // A[i][0] = 1, B[0][j] = j its column j (small integers, exact in FP64). On this GPU register r
    // of lane l holds D[l / 16 + 4 r][l % 16].
    const double idx = kq == 0 ? (double)m : 0.0, one = kq == 0 ? 1.0 : 0.0;
    const gram_d4 zero = {0.0, 0.0, 0.0, 0.0};
    const gram_d4 rowv = __builtin_amdgcn_mfma_f64_16x16x4f64(idx, one, zero, 0, 0, 0);
    const gram_d4 colv = __builtin_amdgcn_mfma_f64_16x16x4f64(one, idx, zero, 0, 0, 0);
    double *out = part + ((size_t)slice * tiles + tile) * (kGT * kGT);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int ri = (int)rowv[r], ci = (int)colv[r];
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b)
                out[(kGR * qr + 16 * a + ri) * kGT + kGC * qc + 16 * b + ci] = acc[a][b][r];
    }
}

// One workgroup per 32 x 32 block of a tile (blockIdx.x = 16 tile + block): stores value
// f(i, j, g) of every element of the block at (i, j) and, off the diagonal, at (j, i), both
// row-wise through an LDS transpose. g is the sum of the element's S slice partials in slice
// order; a thread issues the partial loads of its 4 elements together (one memory latency for
// all). Only i <= j is stored directly and i < j mirrored, so the blocks below the diagonal of
// a diagonal tile store nothing. Elements past N are 0 (store decides what to do with them).
constexpr int kGE = 32;
template <class F, class St>
__device__ __forceinline__ void gram_emit(const double *part, int N, int nt, int tiles, int S, F f, St store) {
    __shared__ double tr[kGE][kGE + 1];
    const int tile = blockIdx.x >> 4, blk = blockIdx.x & 15;
    int ti, tj;
    gram_tile_ij(tile, nt, ti, tj);
    const int r0 = kGE * (blk >> 2), c0 = kGE * (blk & 3);   // within the tile
    if (ti == tj && r0 > c0) return;                          // uniform: every element has i > j
    const int i0 = ti * kGT + r0, j0 = tj * kGT + c0;
    const size_t sstride = (size_t)tiles * (kGT * kGT);
    const double *base = part + (size_t)tile * (kGT * kGT);
    double g[4][kGMaxSplit];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u, r = e / kGE, c = e % kGE;
        const double *p = base + (size_t)(r0 + r) * kGT + c0 + c;
#pragma unroll
        for (int s = 0; s < kGMaxSplit; ++s) g[u][s] = s < S ? p[(size_t)s * sstride] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u, r = e / kGE, c = e % kGE;
        const int i = i0 + r, j = j0 + c;
        double sum = 0.0;
#pragma unroll
        for (int s = 0; s < kGMaxSplit; ++s)
            if (s < S) sum += g[u][s];
        double v = 0.0;
        if (i <= j) {
            if (i < N && j < N) v = f(i, j, sum);
            store(i, j, v);
        }
        tr[c][r] = v;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = threadIdx.x + 256 * u, r = e / kGE, c = e % kGE;   // destination row j0 + r, column i0 + c
        const int j = j0 + r, i = i0 + c;
        if (i < j) store(j, i, tr[r][c]);
    }
}

// C_ij from the Gram entry g and the rows' sums of squares (or variances) a, b.
__device__ __forceinline__ double corr_value(int i, int j, double g, double a, double b) {
    if (i == j) return 1.0;
    if (a == 0.0 || b == 0.0) return 0.0;
    return fmin(1.0, fmax(-1.0, g / sqrt(a * b)));
}

__global__ __launch_bounds__(256) void k_corr_finish(const double *part, int N, int nt, int tiles, int S,
                                                     const double *ss, CorrOut o) {
    gram_emit(
        part, N, nt, tiles, S, [&](int i, int j, double g) { return corr_value(i, j, g, ss[i], ss[j]); },
        [&](int i, int j, double v) { corr_store(o, i, j, v); });
}

// ---- small windows: one launch -------------------------------------------------
// A workgroup of eight waves per 16 x 16 output tile of the upper triangle, each wave an eighth
// of the samples (whole steps of 16). A wave reads a step of both panels row-wise, eight lanes to
// a row's 128 bytes, and passes the centred (or weighted) samples to the MFMA's operand order
// through 4 KB of LDS of its own. (Loads in operand order, where neighbouring lanes hold
// different rows, cost one address per lane: 58 us at N = 18, T = 4096, now 32.) The first
// kSmAhead steps of a wave stay in registers between the means and the products, so up to
// T = 256 R is read once, and twice above (EWMA: always once); the sums of squares are accumulated in the
// same order in every tile. The eight partial tiles meet in LDS and are added in wave order.
//   EWMA: x_it = sw_t (R_it - m_t) with m and sw from k_ewma_mean; S is updated in place, and its
//   old diagonal is read from the copy that k_ewma_mean made (another tile updates it here).
// What bounds it: the chain of a few dependent memory reads and the L2 reads of 32 rows per tile
// against 4 MFMAs per 16 samples; the large path reads each row for 128 columns at a time.
constexpr int kSmThreads = 512;

constexpr int kSmAhead = 2;              // steps of 16 samples whose loads are in flight together
constexpr int kSmWaves = kSmThreads / 64;
constexpr int kSmTile = 16;
typedef double sm_d2 __attribute__((ext_vector_type(2), aligned(8)));   // rows need not be 16-byte aligned

struct EwmaArgs {
    const double *m, *sw;    // T: market mean, weight root
    const double *diag0;     // N: S_ii before this call
    double *S;
    double decay;
    int reset;
};

template <bool EWMA>
__global__ __launch_bounds__(kSmThreads) void k_corr_small(const double *R, int N, int T, int64_t ld, int nt,
                                                           CorrOut o, EwmaArgs w, int32_t *status) {
    // a wave's step buffer, and after its last step its partial tile (the first half)
    __shared__ __align__(16) double stage[kSmWaves][2 * kSmTile * 16];
    __shared__ double rowred[kSmWaves][2 * kSmTile];
    __shared__ double tv[kSmTile * kSmTile], tg[EWMA ? kSmTile * kSmTile : 1];
    int ti, tj;
    gram_tile_ij(blockIdx.x, nt, ti, tj);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int m = lane & 15, kq = lane >> 4;
    const int i0 = kSmTile * ti, j0 = kSmTile * tj;
    // this lane loads samples 2 (lane % 8), +1 of a step of rows lane / 8 and lane / 8 + 8 of both panels
    const int lr = lane >> 3, ls = lane & 7;
    const double *row[4];                                     // A, A + 8, B, B + 8; past N: row N - 1, results unused
#pragma unroll
    for (int v = 0; v < 4; ++v) row[v] = R + (size_t)min((v < 2 ? i0 : j0) + lr + 8 * (v & 1), N - 1) * ld + 2 * ls;
    const int steps = (T + 15) / 16, per = (steps + kSmWaves - 1) / kSmWaves;
    const int t0 = 16 * per * wave, t1 = min(T, t0 + 16 * per);
    const int groups = t0 < t1 ? (t1 - t0 + 16 * kSmAhead - 1) / (16 * kSmAhead) : 0;
    sm_d2 x[kSmAhead][4], mw[kSmAhead][EWMA ? 2 : 1];         // one group of steps; EWMA: means and weights
    auto pair = [&](const double *r, int tb, bool whole) {    // samples tb + 2 ls, +1; 0 past T
        if (whole) return *(const PGA_GLOBAL sm_d2 *)(r + tb);
        sm_d2 v = {0.0, 0.0};
        if (tb + 2 * ls < T) v.x = gld(r + tb);
        if (tb + 2 * ls + 1 < T) v.y = gld(r + tb + 1);
        return v;
    };
    auto load = [&](int g) {
#pragma unroll
        for (int u = 0; u < kSmAhead; ++u) {
            const int tb = t0 + 16 * (kSmAhead * g + u);
            if (tb >= t1) break;                              // uniform
            const bool whole = tb + 16 <= T;
#pragma unroll
            for (int v = 0; v < 4; ++v) x[u][v] = pair(row[v], tb, whole);
            if constexpr (EWMA) {
                mw[u][0] = pair(w.m + 2 * ls, tb, whole);
                mw[u][1] = pair(w.sw + 2 * ls, tb, whole);
            }
        }
    };
    // Sums over the workgroup of a value per row: the 8 lanes of a row, then the waves in order.
    auto row_total = [&](double (&a)[4]) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
#pragma unroll
            for (int k = 1; k < 8; k <<= 1) a[v] += __shfl_xor(a[v], k, 64);
            if (ls == 0) rowred[wave][8 * v + lr] = a[v];
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            a[v] = 0.0;
#pragma unroll
            for (int q = 0; q < kSmWaves; ++q) a[v] += rowred[q][8 * v + lr];
        }
        __syncthreads();
    };
    double mean[4] = {0.0, 0.0, 0.0, 0.0};
    if (groups > 0) load(0);
    if constexpr (!EWMA) {                                    // as k_row_stats: differences to the first sample
        double first[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) first[v] = gld(row[v] - 2 * ls);
        for (int g = 0; g < groups; ++g) {
            if (g > 0) load(g);
#pragma unroll
            for (int u = 0; u < kSmAhead; ++u)
                if (t0 + 16 * (kSmAhead * g + u) < t1)        // uniform
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int t = t0 + 16 * (kSmAhead * g + u) + 2 * ls;
                        mean[v] += (t < T ? x[u][v].x - first[v] : 0.0) + (t + 1 < T ? x[u][v].y - first[v] : 0.0);
                    }
        }
        row_total(mean);
#pragma unroll
        for (int v = 0; v < 4; ++v) mean[v] = first[v] + mean[v] / (double)T;
        if (groups > 1) load(0);
    }
    // Step buffer: row r's eight sample pairs at slots p ^ (r % 8), which spreads the operand reads
    // over the banks. A wave's LDS operations complete in order, so the next step may overwrite it.
    sm_d2 *const sb = (sm_d2 *)stage[wave];
    gram_d4 acc = {0.0, 0.0, 0.0, 0.0};
    double q[4] = {0.0, 0.0, 0.0, 0.0};
    for (int g = 0; g < groups; ++g) {
        if (g > 0) load(g);
#pragma unroll
        for (int u = 0; u < kSmAhead; ++u) {
            const int tb = t0 + 16 * (kSmAhead * g + u);
            if (tb >= t1) break;                              // uniform
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                sm_d2 y;
                if constexpr (EWMA) {
                    y.x = mw[u][1].x * (x[u][v].x - mw[u][0].x);   // a weight past T is 0
                    y.y = mw[u][1].y * (x[u][v].y - mw[u][0].y);
                } else {
                    y.x = tb + 2 * ls < T ? x[u][v].x - mean[v] : 0.0;
                    y.y = tb + 2 * ls + 1 < T ? x[u][v].y - mean[v] : 0.0;
                }
                q[v] = fma(y.x, y.x, q[v]);
                q[v] = fma(y.y, y.y, q[v]);
                sb[8 * (8 * v + lr) + (ls ^ lr)] = y;          // row 8v + lr: panel A, then B
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const sm_d2 a0 = sb[8 * m + ((2 * kq) ^ (m & 7))], a1 = sb[8 * m + ((2 * kq + 1) ^ (m & 7))];
            const sm_d2 b0 = sb[8 * (16 + m) + ((2 * kq) ^ (m & 7))], b1 = sb[8 * (16 + m) + ((2 * kq + 1) ^ (m & 7))];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a0.x, b0.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a0.y, b0.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a1.x, b1.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a1.y, b1.y, acc, 0, 0, 0);
        }
    }
    // register r of lane l holds D[l / 16 + 4 r][l % 16] (see k_gram_mfma)
#pragma unroll
    for (int r = 0; r < 4; ++r) stage[wave][(kq + 4 * r) * kSmTile + m] = acc[r];
    row_total(q);                                             // its barriers also close the writes to stage
    if (wave == 0 && ls == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = (v < 2 ? i0 : j0) + lr + 8 * (v & 1);
            if constexpr (EWMA)
                if (!w.reset) q[v] = fma(w.decay, w.diag0[min(i, N - 1)], q[v]);
            rowred[0][8 * v + lr] = q[v];
            if (ti == tj && v < 2 && i < N && q[v] == 0.0 && status) atomicAdd(&status[PGA_ST_ZEROVAR], 1);
        }
    }
    __syncthreads();
    // Threads 0..255 make element (r, c) of the tile, i <= j, and store it; threads 256..511 store
    // its mirror image row-wise from LDS.
    const int e = tid & 255, r = e >> 4, c = e & 15;
    if (tid < 256) {
        const int i = i0 + r, j = j0 + c;
        double g = 0.0;
#pragma unroll
        for (int v = 0; v < kSmWaves; ++v) g += stage[v][e];
        double v = 0.0;
        if (i <= j && i < N && j < N) {
            if constexpr (EWMA) {
                g = w.reset ? g : fma(w.decay, w.S[(size_t)i * N + j], g);
                w.S[(size_t)i * N + j] = g;
            }
            v = corr_value(i, j, g, rowred[0][r], rowred[0][kSmTile + c]);
        }
        if (i <= j) corr_store(o, i, j, v);
        tv[e] = v;
        if constexpr (EWMA) tg[e] = g;
    }
    __syncthreads();
    if (tid >= 256) {
        const int i = i0 + c, j = j0 + r, x = c * kSmTile + r;     // stored at (j, i): row r, column c
        if (i < j) {
            if constexpr (EWMA)
                if (i < N && j < N) w.S[(size_t)j * N + i] = tg[x];
            corr_store(o, j, i, tv[x]);
        }
    }
}

// Where the small path ends (back-to-back calls, us small / large path). Its workgroups are as many as the 16 x 16 tiles of the
// upper triangle (with the split, whose padding counts, so that C is the same bits without it); their time is that of the
// rounds of one per CU, which read every row twice (the means first) from T = 257.
// One round (N <= 352): ahead wherever measured (300 x 390 13 / 26, 300 x 4096 40 / 56, 300 x 8192 73 / 97);
// the rule ends at T = 4096, the longest window of its first measurements. Two (448 x 1024 25 / 31, x 2048 45 / 40):
// to T = 1024. Three (576 x 768 31 / 32, x 1024 38 / 35; 512 x 1024 37 / 31): to T = 768. Four (704 x 256 25 / 28,
// x 390 33 / 32, x 1024 51 / 38): to T = 256. Five and more lose from 100 samples on (896 x 64 34 / 26).
bool corr_small(int N, int T) {
    const int nt = split_ld(N) / kSmTile, rounds = (nt * (nt + 1) / 2 + 255) / 256;
    return rounds <= 1 ? T <= 4096 : rounds == 2 ? T <= 1024 : rounds == 3 ? T <= 768 : rounds == 4 && T <= 256;
}
// The EWMA's small path reads each row once and its large path has a launch more: N = 704, T = 1024 34 / 46 with the split
// (608 x 390 21 / 37, 352 x 1024 20 / 37). Its limits are those of the first measurements.
bool ewma_small(int N, int T) { return N <= 352 ? T <= 4096 : N <= 704 && T <= 1024; }

hipError_t launch_corr(const double *R, int N, int T, int64_t ld, double *mu, double *ss, double *C, uint16_t *hi,
                       uint16_t *lo, double *part, int32_t *status, hipStream_t s) {
    const CorrOut o = corr_out(C, N, hi, lo);
    if (corr_small(N, T)) {
        const int nt = (o.ld + kSmTile - 1) / kSmTile;
        hipLaunchKernelGGL(k_corr_small<false>, dim3(nt * (nt + 1) / 2), dim3(kSmThreads), 0, s, R, N, T, ld, nt, o,
                           EwmaArgs{}, status);
        return hipGetLastError();
    }
    const int nt = (N + kGT - 1) / kGT, tiles = gram_tiles(N), S = gram_split(N, T);
    hipLaunchKernelGGL(T <= 256 ? k_row_stats<1> : T <= 1024 ? k_row_stats<4> : k_row_stats<16>, dim3(N), dim3(256), 0, s, R,
                       T, ld, mu, ss, status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gram_mfma<false>, dim3(tiles * S), dim3(kGThreads), 0, s, R, N, T, ld, mu, nullptr, nt, tiles,
                       S, part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_corr_finish, dim3(16 * tiles), dim3(256), 0, s, part, N, nt, tiles, S, ss, o);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_split(const double *C, int N, int ld, uint16_t *hi, uint16_t *lo) {
    const size_t total = (size_t)ld * ld;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (size_t)gridDim.x * 256) {
        const int i = (int)(e / ld), j = (int)(e % ld);
        const double v = (i < N && j < N) ? C[(size_t)i * N + j] : 0.0;
        const double h = bf16_round(v);
        const double l = bf16_round(v - h);
        hi[e] = bf16_bits(h);
        lo[e] = bf16_bits(l);
    }
}

hipError_t launch_split(const double *C, int N, uint16_t *hi, uint16_t *lo, hipStream_t s) {
    const int ld = split_ld(N);
    const size_t total = (size_t)ld * ld;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_split, dim3(blocks), dim3(256), 0, s, C, N, ld, hi, lo);
    return hipGetLastError();
}

// ---- online EWMA correlation (Section 4.2.5 pre-processing) ------------------
// The recursion S <- lambda S + (1 - lambda) x_t x_t^T over t = 0 .. T-1 is
// S <- lambda^T S + sum_t w_t x_t x_t^T with w_t = (1 - lambda) lambda^(T-1-t):
//   mean : m_t = the equal-weight market return (or 0) and sw_t = sqrt(w_t);
//   gram : S_ij <- lambda^T S_ij + sum_t y_it y_jt, y_it = sw_t (R_it - m_t), on the tiles of
//          the upper triangle (the MFMA Gram of the correlation), mirrored;
//   norm : C_ij = S_ij / sqrt(S_ii S_jj), clamp, C_ii = 1, zero variance -> 0.
// The mean kernel also copies the old diagonal of S, so that the tiles, which update S in
// place, can normalise at once. A workgroup takes 8 samples: 32 rows of 64 bytes at a time (one
// thread per sample over all N rows, as the sum had been, took 73 us at N = 300, T = 390).
constexpr int kEwmaCols = 8;
__global__ __launch_bounds__(256) void k_ewma_mean(const double *R, int N, int T, int64_t ld, double lam, int market,
                                                   const double *S, double *m, double *sw, double *diag0) {
    __shared__ double red[256 / kEwmaCols][kEwmaCols];
    const int tt = threadIdx.x % kEwmaCols, rg = threadIdx.x / kEwmaCols;
    const int t = blockIdx.x * kEwmaCols + tt;
    double v = 0.0;
    if (market && t < T) {
#pragma unroll 4
        for (int i = rg; i < N; i += 256 / kEwmaCols) v += R[(size_t)i * ld + t];
    }
    red[rg][tt] = v;
    if (S)
        for (int j = blockIdx.x * 256 + threadIdx.x; j < N; j += gridDim.x * 256) diag0[j] = S[(size_t)j * N + j];
    __syncthreads();
    if (threadIdx.x < kEwmaCols && t < T) {
        double sum = 0.0;
#pragma unroll
        for (int g = 0; g < 256 / kEwmaCols; ++g) sum += red[g][tt];
        m[t] = market ? sum / (double)N : 0.0;
        sw[t] = sqrt((1.0 - lam) * pow(lam, (double)(T - 1 - t)));
    }
}

// The finish of the large path: the new S, and C from it. The diagonal entries a block needs are
// summed as the diagonal tiles sum them.
__global__ __launch_bounds__(256) void k_ewma_finish(const double *part, int N, int nt, int tiles, int S,
                                                     EwmaArgs w, CorrOut o, int32_t *status) {
    __shared__ double dd[2][kGE];                            // new S_ii of the block's rows, of its columns
    {
        const int tile = blockIdx.x >> 4, blk = blockIdx.x & 15;
        int ti, tj;
        gram_tile_ij(tile, nt, ti, tj);
        if (threadIdx.x < 2 * kGE) {
            const int side = threadIdx.x / kGE, x = threadIdx.x % kGE;
            const int tb = side ? tj : ti, lx = kGE * (side ? blk & 3 : blk >> 2) + x, i = tb * kGT + lx;
            double g = 0.0;
            if (i < N) {
                const int dt = tb * nt - tb * (tb - 1) / 2;  // the diagonal tile of row block tb
                const double *p = part + (size_t)dt * (kGT * kGT) + (size_t)lx * kGT + lx;
                for (int v = 0; v < S; ++v) g += p[(size_t)v * tiles * (kGT * kGT)];
                if (!w.reset) g = fma(w.decay, w.diag0[i], g);
                if (ti == tj && side == 0 && (blk >> 2) == (blk & 3) && g == 0.0 && status)
                    atomicAdd(&status[PGA_ST_ZEROVAR], 1);
            }
            dd[side][x] = g;
        }
    }
    __syncthreads();
    gram_emit(
        part, N, nt, tiles, S,
        [&](int i, int j, double g) {
            g = w.reset ? g : fma(w.decay, w.S[(size_t)i * N + j], g);
            return g;
        },
        [&](int i, int j, double g) {
            const bool in = i < N && j < N;
            if (in) w.S[(size_t)i * N + j] = g;
            // (i, j) of the direct store has i among the block's rows, the mirror image's among its columns
            const int a = i <= j ? i : j, b = i <= j ? j : i;
            corr_store(o, i, j, in ? corr_value(a, b, g, dd[0][a % kGE], dd[1][b % kGE]) : 0.0);
        });
}

size_t ewma_ws_doubles(int N, int T) { return 2 * (size_t)T + (size_t)N; }

hipError_t launch_ewma(const double *R, int N, int T, int64_t ld, double lam, int reset, int market, double *S,
                       double *C, uint16_t *hi, uint16_t *lo, double *ws, double *part, int32_t *status,
                       hipStream_t s) {
    const CorrOut o = corr_out(C, N, hi, lo);
    double *m = ws, *sw = ws + T, *diag0 = ws + 2 * (size_t)T;
    const EwmaArgs w{m, sw, diag0, S, pow(lam, (double)T), reset};
    hipLaunchKernelGGL(k_ewma_mean, dim3((T + kEwmaCols - 1) / kEwmaCols), dim3(256), 0, s, R, N, T, ld, lam, market,
                       reset ? nullptr : S, m, sw, diag0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ewma_small(N, T)) {
        const int nt = (o.ld + kSmTile - 1) / kSmTile;
        hipLaunchKernelGGL(k_corr_small<true>, dim3(nt * (nt + 1) / 2), dim3(kSmThreads), 0, s, R, N, T, ld, nt, o, w,
                           status);
        return hipGetLastError();
    }
    const int nt = (N + kGT - 1) / kGT, tiles = gram_tiles(N), Sp = gram_split(N, T);
    hipLaunchKernelGGL(k_gram_mfma<true>, dim3(tiles * Sp), dim3(kGThreads), 0, s, R, N, T, ld, m, sw, nt, tiles, Sp,
                       part);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_ewma_finish, dim3(16 * tiles), dim3(256), 0, s, part, N, nt, tiles, Sp, w, o, status);
    return hipGetLastError();
}

}  // namespace pga
