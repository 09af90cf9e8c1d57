// Fitness kernels: the Giada-Marsili likelihood L_c (Eq. 8) of a population,
// from n_s (Eq. 5) and c_s (Eq. 6).
//
// Split into two launches:
//   pair-sum  v_pj = C_jj + 2 sum_{i<j} [s_pi = s_pj] C_ij for every
//             individual p and stock j (the O(N^2) part; FP64 VALU form here,
//             BF16x2 MFMA form in k_mfma.hip);
//   finish    per individual: n_s by an LDS histogram, c_s = sum_{j in s} v_pj
//             grouped exactly in 64-bit fixed point, then the FP64 log terms
//             and a fixed-order wave reduction.
// Nothing here uses floating-point atomics, so every result is a pure
// function of (C, labels): reruns and batching cannot change a bit.
#include "pga_internal.hpp"

#include <math.h>

#include <type_traits>

namespace pga {

// ---------------------------------------------------------------------------
// Descriptor upload alone (the tuner's next variant).
__global__ __launch_bounds__(256) void k_write_desc(DescBlob b, InstDesc *dst, int32_t *prefix) { write_desc(b, dst, prefix); }

hipError_t launch_write_desc(const InstDesc &d, int32_t tiles, InstDesc *dst, int32_t *prefix, hipStream_t s) {
    hipLaunchKernelGGL(k_write_desc, dim3(1), dim3(256), 0, s, DescBlob::of(d, tiles), dst, prefix);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FP64 pair-sum. One workgroup = 64 consecutive stocks j (one per lane) x 4B
// individuals (B = 8 or 16 per wave); the four waves are independent (no
// workgroup barrier). Each lane keeps its B labels s_pj and B FP64 accumulators in
// registers and walks the rows i < j of its column in chunks of 64 rows:
//   - C_ij is loaded once per (wave, row), coalesced across the wave, and
//     reused by B individuals; loads run one group of 4 rows ahead, in two sets of
//     registers that change roles (copied from one to the other, a copy waited for
//     loads that had just gone out);
//   - the row labels s_pi of the wave's B individuals are staged per chunk in
//     a wave-private LDS buffer (transposed, so one 16-byte broadcast read
//     serves 4 individuals), double-buffered: the next chunk's labels are
//     fetched into registers while the current chunk is processed. An add block's labels
//     are read into registers before the block above it.
// Per (pair, individual): compare, masked FP64 add. Rows i >= j and rows
// past N contribute C = 0, so every chunk runs all 64 rows without branches.
// Bound by vector issue: 17.3 vector instructions per row of 8 individuals, 72 cycles of a SIMD at
// their own rate with many waves; planted partitions at N = 1024, P = 4096 (4 waves per SIMD), 217 us
// with the reads next to their uses and 8 masks, 173 us now. Tried without gain: row labels by scalar
// loads (a line per individual: 312 us two rows at a time, 214 us 16 rows at a time, against 217),
// a select of the value's high word instead of EXEC (275 us).
// acc[b] += c on the lanes where the row label of individual b equals lj[b], for two rows of 8
// individuals (row 0 first) or one row of 16: 16 compares under the full EXEC write 16 lane
// masks to SGPR pairs (0 on inactive lanes), then each FP64 add runs with its mask as EXEC, which
// is restored before the block ends. Two vector instructions per (pair, individual); the scalar ones
// issue alongside other waves' vector work. 16 masks, because a switch between the two runs costs
// most where few waves share a SIMD: cycles per 8 pairs with 4 / 8 waves, 95 / 79 with 8 masks,
// 78 / 72 with 16 (64 of them the 16 vector instructions).
__device__ __forceinline__ void add_if_equal8(double *acc, const int *r0, const int *r1, const int *lj, double c0, double c1) {
    uint64_t m[16], sv;
    asm volatile(
        "s_mov_b64 %[sv], exec\n\t"
        "v_cmp_eq_u32_e64 %[m0], %[r0], %[l0]\n\t"
        "v_cmp_eq_u32_e64 %[m1], %[r1], %[l1]\n\t"
        "v_cmp_eq_u32_e64 %[m2], %[r2], %[l2]\n\t"
        "v_cmp_eq_u32_e64 %[m3], %[r3], %[l3]\n\t"
        "v_cmp_eq_u32_e64 %[m4], %[r4], %[l4]\n\t"
        "v_cmp_eq_u32_e64 %[m5], %[r5], %[l5]\n\t"
        "v_cmp_eq_u32_e64 %[m6], %[r6], %[l6]\n\t"
        "v_cmp_eq_u32_e64 %[m7], %[r7], %[l7]\n\t"
        "v_cmp_eq_u32_e64 %[m8], %[r8], %[l0]\n\t"
        "v_cmp_eq_u32_e64 %[m9], %[r9], %[l1]\n\t"
        "v_cmp_eq_u32_e64 %[m10], %[r10], %[l2]\n\t"
        "v_cmp_eq_u32_e64 %[m11], %[r11], %[l3]\n\t"
        "v_cmp_eq_u32_e64 %[m12], %[r12], %[l4]\n\t"
        "v_cmp_eq_u32_e64 %[m13], %[r13], %[l5]\n\t"
        "v_cmp_eq_u32_e64 %[m14], %[r14], %[l6]\n\t"
        "v_cmp_eq_u32_e64 %[m15], %[r15], %[l7]\n\t"
        "s_mov_b64 exec, %[m0]\n\t"
        "v_add_f64 %[a0], %[a0], %[c0]\n\t"
        "s_mov_b64 exec, %[m1]\n\t"
        "v_add_f64 %[a1], %[a1], %[c0]\n\t"
        "s_mov_b64 exec, %[m2]\n\t"
        "v_add_f64 %[a2], %[a2], %[c0]\n\t"
        "s_mov_b64 exec, %[m3]\n\t"
        "v_add_f64 %[a3], %[a3], %[c0]\n\t"
        "s_mov_b64 exec, %[m4]\n\t"
        "v_add_f64 %[a4], %[a4], %[c0]\n\t"
        "s_mov_b64 exec, %[m5]\n\t"
        "v_add_f64 %[a5], %[a5], %[c0]\n\t"
        "s_mov_b64 exec, %[m6]\n\t"
        "v_add_f64 %[a6], %[a6], %[c0]\n\t"
        "s_mov_b64 exec, %[m7]\n\t"
        "v_add_f64 %[a7], %[a7], %[c0]\n\t"
        "s_mov_b64 exec, %[m8]\n\t"
        "v_add_f64 %[a0], %[a0], %[c1]\n\t"
        "s_mov_b64 exec, %[m9]\n\t"
        "v_add_f64 %[a1], %[a1], %[c1]\n\t"
        "s_mov_b64 exec, %[m10]\n\t"
        "v_add_f64 %[a2], %[a2], %[c1]\n\t"
        "s_mov_b64 exec, %[m11]\n\t"
        "v_add_f64 %[a3], %[a3], %[c1]\n\t"
        "s_mov_b64 exec, %[m12]\n\t"
        "v_add_f64 %[a4], %[a4], %[c1]\n\t"
        "s_mov_b64 exec, %[m13]\n\t"
        "v_add_f64 %[a5], %[a5], %[c1]\n\t"
        "s_mov_b64 exec, %[m14]\n\t"
        "v_add_f64 %[a6], %[a6], %[c1]\n\t"
        "s_mov_b64 exec, %[m15]\n\t"
        "v_add_f64 %[a7], %[a7], %[c1]\n\t"
        "s_mov_b64 exec, %[sv]"
        : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3]), [a4] "+v"(acc[4]), [a5] "+v"(acc[5]), [a6] "+v"(acc[6]), [a7] "+v"(acc[7]),
          [m0] "=&s"(m[0]), [m1] "=&s"(m[1]), [m2] "=&s"(m[2]), [m3] "=&s"(m[3]), [m4] "=&s"(m[4]), [m5] "=&s"(m[5]), [m6] "=&s"(m[6]), [m7] "=&s"(m[7]), [m8] "=&s"(m[8]), [m9] "=&s"(m[9]), [m10] "=&s"(m[10]), [m11] "=&s"(m[11]), [m12] "=&s"(m[12]), [m13] "=&s"(m[13]), [m14] "=&s"(m[14]), [m15] "=&s"(m[15]), [sv] "=&s"(sv)
        : [r0] "v"(r0[0]), [r1] "v"(r0[1]), [r2] "v"(r0[2]), [r3] "v"(r0[3]), [r4] "v"(r0[4]), [r5] "v"(r0[5]), [r6] "v"(r0[6]), [r7] "v"(r0[7]), [r8] "v"(r1[0]), [r9] "v"(r1[1]), [r10] "v"(r1[2]), [r11] "v"(r1[3]), [r12] "v"(r1[4]), [r13] "v"(r1[5]), [r14] "v"(r1[6]), [r15] "v"(r1[7]),
          [l0] "v"(lj[0]), [l1] "v"(lj[1]), [l2] "v"(lj[2]), [l3] "v"(lj[3]), [l4] "v"(lj[4]), [l5] "v"(lj[5]), [l6] "v"(lj[6]), [l7] "v"(lj[7]), [c0] "v"(c0), [c1] "v"(c1));
}

__device__ __forceinline__ void add_if_equal16(double *acc, const int *r, const int *lj, double c) {
    uint64_t m[16], sv;
    asm volatile(
        "s_mov_b64 %[sv], exec\n\t"
        "v_cmp_eq_u32_e64 %[m0], %[r0], %[l0]\n\t"
        "v_cmp_eq_u32_e64 %[m1], %[r1], %[l1]\n\t"
        "v_cmp_eq_u32_e64 %[m2], %[r2], %[l2]\n\t"
        "v_cmp_eq_u32_e64 %[m3], %[r3], %[l3]\n\t"
        "v_cmp_eq_u32_e64 %[m4], %[r4], %[l4]\n\t"
        "v_cmp_eq_u32_e64 %[m5], %[r5], %[l5]\n\t"
        "v_cmp_eq_u32_e64 %[m6], %[r6], %[l6]\n\t"
        "v_cmp_eq_u32_e64 %[m7], %[r7], %[l7]\n\t"
        "v_cmp_eq_u32_e64 %[m8], %[r8], %[l8]\n\t"
        "v_cmp_eq_u32_e64 %[m9], %[r9], %[l9]\n\t"
        "v_cmp_eq_u32_e64 %[m10], %[r10], %[l10]\n\t"
        "v_cmp_eq_u32_e64 %[m11], %[r11], %[l11]\n\t"
        "v_cmp_eq_u32_e64 %[m12], %[r12], %[l12]\n\t"
        "v_cmp_eq_u32_e64 %[m13], %[r13], %[l13]\n\t"
        "v_cmp_eq_u32_e64 %[m14], %[r14], %[l14]\n\t"
        "v_cmp_eq_u32_e64 %[m15], %[r15], %[l15]\n\t"
        "s_mov_b64 exec, %[m0]\n\t"
        "v_add_f64 %[a0], %[a0], %[c0]\n\t"
        "s_mov_b64 exec, %[m1]\n\t"
        "v_add_f64 %[a1], %[a1], %[c0]\n\t"
        "s_mov_b64 exec, %[m2]\n\t"
        "v_add_f64 %[a2], %[a2], %[c0]\n\t"
        "s_mov_b64 exec, %[m3]\n\t"
        "v_add_f64 %[a3], %[a3], %[c0]\n\t"
        "s_mov_b64 exec, %[m4]\n\t"
        "v_add_f64 %[a4], %[a4], %[c0]\n\t"
        "s_mov_b64 exec, %[m5]\n\t"
        "v_add_f64 %[a5], %[a5], %[c0]\n\t"
        "s_mov_b64 exec, %[m6]\n\t"
        "v_add_f64 %[a6], %[a6], %[c0]\n\t"
        "s_mov_b64 exec, %[m7]\n\t"
        "v_add_f64 %[a7], %[a7], %[c0]\n\t"
        "s_mov_b64 exec, %[m8]\n\t"
        "v_add_f64 %[a8], %[a8], %[c0]\n\t"
        "s_mov_b64 exec, %[m9]\n\t"
        "v_add_f64 %[a9], %[a9], %[c0]\n\t"
        "s_mov_b64 exec, %[m10]\n\t"
        "v_add_f64 %[a10], %[a10], %[c0]\n\t"
        "s_mov_b64 exec, %[m11]\n\t"
        "v_add_f64 %[a11], %[a11], %[c0]\n\t"
        "s_mov_b64 exec, %[m12]\n\t"
        "v_add_f64 %[a12], %[a12], %[c0]\n\t"
        "s_mov_b64 exec, %[m13]\n\t"
        "v_add_f64 %[a13], %[a13], %[c0]\n\t"
        "s_mov_b64 exec, %[m14]\n\t"
        "v_add_f64 %[a14], %[a14], %[c0]\n\t"
        "s_mov_b64 exec, %[m15]\n\t"
        "v_add_f64 %[a15], %[a15], %[c0]\n\t"
        "s_mov_b64 exec, %[sv]"
        : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3]), [a4] "+v"(acc[4]), [a5] "+v"(acc[5]), [a6] "+v"(acc[6]), [a7] "+v"(acc[7]), [a8] "+v"(acc[8]), [a9] "+v"(acc[9]), [a10] "+v"(acc[10]), [a11] "+v"(acc[11]), [a12] "+v"(acc[12]), [a13] "+v"(acc[13]), [a14] "+v"(acc[14]), [a15] "+v"(acc[15]),
          [m0] "=&s"(m[0]), [m1] "=&s"(m[1]), [m2] "=&s"(m[2]), [m3] "=&s"(m[3]), [m4] "=&s"(m[4]), [m5] "=&s"(m[5]), [m6] "=&s"(m[6]), [m7] "=&s"(m[7]), [m8] "=&s"(m[8]), [m9] "=&s"(m[9]), [m10] "=&s"(m[10]), [m11] "=&s"(m[11]), [m12] "=&s"(m[12]), [m13] "=&s"(m[13]), [m14] "=&s"(m[14]), [m15] "=&s"(m[15]), [sv] "=&s"(sv)
        : [r0] "v"(r[0]), [r1] "v"(r[1]), [r2] "v"(r[2]), [r3] "v"(r[3]), [r4] "v"(r[4]), [r5] "v"(r[5]), [r6] "v"(r[6]), [r7] "v"(r[7]), [r8] "v"(r[8]), [r9] "v"(r[9]), [r10] "v"(r[10]), [r11] "v"(r[11]), [r12] "v"(r[12]), [r13] "v"(r[13]), [r14] "v"(r[14]), [r15] "v"(r[15]),
          [l0] "v"(lj[0]), [l1] "v"(lj[1]), [l2] "v"(lj[2]), [l3] "v"(lj[3]), [l4] "v"(lj[4]), [l5] "v"(lj[5]), [l6] "v"(lj[6]), [l7] "v"(lj[7]), [l8] "v"(lj[8]), [l9] "v"(lj[9]), [l10] "v"(lj[10]), [l11] "v"(lj[11]), [l12] "v"(lj[12]), [l13] "v"(lj[13]), [l14] "v"(lj[14]), [l15] "v"(lj[15]), [c0] "v"(c));
}

template <int B, bool LISTED>
__global__ __launch_bounds__(256) void k_pairsum_fp64(Tables t, int parity, int order) {
    __shared__ int4 lab_s[kFp64Waves][2][64][B / 4];

    const int total = const_at(t.tiles, t.n_inst);       // the grid may exceed it (capacity-sized graph)
    const bool none = none_dense(t, parity), past = (int)blockIdx.x >= total;   // one wait for both loads
    if (none | past) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform, kept scalar
    const int lane = threadIdx.x & 63;
    auto work = [&](const InstDesc &d, int local) {        // the waves share no barrier
        const int N = d.N, P = d.P;
        const int n_jb = (N + kFp64Cols - 1) / kFp64Cols;
        const int n_pairs = (n_jb + 1) / 2;
        const TilePos tp = tile_pos(local, n_pairs, (P + kFp64Waves * B - 1) / (kFp64Waves * B), order);
        const int jp = tp.jp, pb = tp.pb;
        const int pbase = pb * (kFp64Waves * B) + wave * B;
        if (pbase >= P) return;
        if (d.route) {
            int any = 0;                                 // the loads together: no test between them
#pragma unroll
            for (int b = 0; b < B; ++b) any |= gld(d.route + min(pbase + b, P - 1));
            if (!any) return;
        }
        const int32_t *__restrict__ labels = d.pop[parity];
        const double *__restrict__ C = d.C;
        const __amdgpu_buffer_rsrc_t c_r = __builtin_amdgcn_make_buffer_rsrc((void *)C, (short)0, 8 * N * N, kBufWord3);   // N <= 4096

        auto fetch_labels = [&](int i0, int *v) {
            const int ir = i0 + lane;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int p = pbase + b;
                v[b] = (ir < N && p < P) ? gld(labels + (size_t)p * N + ir) : (int)0x80000001;
            }
        };
        auto store_labels = [&](int buf, const int *v) {
#pragma unroll
            for (int q = 0; q < B / 4; ++q)
                lab_s[wave][buf][lane][q] = make_int4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
        };

        // The four waves of a SIMD have equal work but, left to themselves, the oldest issues first and
        // the youngest ends alone, at half the rate (they lived 74% of the launch on average): the
        // highest priority goes round by wave slot, a chunk each (86%; 188.7 -> 176.6 us at N = 1024, P = 4096).
        // Not where the launch has more than one round of workgroups and the upper triangle of C (4 N^2 bytes) is larger
        // than the L2s (N > 2896): the waves that turns keep out of step share fewer C rows there, and a young wave's end is
        // covered by the next round. N = 4096, P = 4096: 2758 us with turns, 2286 without; N = 3584, P = 4672: 2199 / 1999;
        // N = 3072, P = 4096: 1345 / 1317. Below, with more rounds, they win or lose up to 4% (N = 2560, P = 2464:
        // 649 / 671; P = 4928: 1196 / 1185); within one round they win at every N (3584, P = 864: 414 / 460).
        const bool turns = total <= kFp64Round || 4ll * N * N <= kL2Bytes;
        const int slot = __builtin_amdgcn_s_getreg((3 << 11) | 4);   // HW_ID.WAVE_ID
        // The triangle is folded: column blocks n_jb-1-jp (jp + 1 ... n_jb chunks of rows) and
        // jp are done by the same workgroup, so every workgroup has n_jb + 1 chunks of work.
        for (int half = 0; half < 2; ++half) {
            const int jb = half == 0 ? n_jb - 1 - jp : jp;
            if (half == 1 && jb == n_jb - 1 - jp) break;       // middle block of an odd count: once
            const int j = jb * kFp64Cols + lane;
            const bool jok = j < N;

            int lj[B];
            double acc[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int p = pbase + b;
                lj[b] = (jok && p < P) ? gld(labels + (size_t)p * N + j) : (int)0x80000000;
                acc[b] = 0.0;
            }

            const int nchunks = jb + 1;                      // rows 0 .. 64 (jb + 1) - 1
            int nxt[B];
            fetch_labels(0, nxt);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();                 // previous block's reads of buffer 0 are done
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            store_labels(0, nxt);
            // C loads go through a buffer descriptor over C: the lane's column offset stays in one
            // register and the row offset is a scalar, so a load costs no vector address arithmetic.
            // Rows past N read row N - 1 (the range check of a buffer leaves the scalar offset out) and
            // lanes past N column N - 1; the former are >= j, the latter never stored. Chunks before the
            // last hold rows i < 64 jb <= j only, so their values need no test.
            const int jc = jok ? j : N - 1;
            const uint32_t jc_off = 8u * (uint32_t)jc;
            // (The clamp only where rows may be past N: in every load it cost 3%.)
            auto load_c = [&](auto clamped, double *c, int i) {
#pragma unroll
                for (int q = 0; q < kFp64Ahead; ++q) {
                    const int row = fp64_row(i + q, N, decltype(clamped)::value);
                    c[q] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(c_r, jc_off, 8u * (uint32_t)row * (uint32_t)N, 0));
                }
            };
            double ca[kFp64Ahead], cb[kFp64Ahead];
            load_c(std::true_type{}, ca, 0);
            auto chunk = [&](auto checked_tag, int ch) {
                constexpr bool checked = decltype(checked_tag)::value;
                if (turns) {
                    switch ((ch + slot) & 3) {
                    case 0: __builtin_amdgcn_s_setprio(0); break;
                    case 1: __builtin_amdgcn_s_setprio(1); break;
                    case 2: __builtin_amdgcn_s_setprio(2); break;
                    default: __builtin_amdgcn_s_setprio(3); break;
                    }
                }
                const int i0 = ch * 64;
                const int buf = ch & 1;
                if (ch + 1 < nchunks) fetch_labels(i0 + 64, nxt);   // in flight during this chunk
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

                constexpr int kRows = 16 / B;                    // of one add block
                int ra[kRows][B], rb[kRows][B];
                auto labels_of = [&](int *rl, int r) {
#pragma unroll
                    for (int u = 0; u < B / 4; ++u) {
                        const int4 v = lab_s[wave][buf][r & 63][u];
                        rl[4 * u + 0] = v.x;
                        rl[4 * u + 1] = v.y;
                        rl[4 * u + 2] = v.z;
                        rl[4 * u + 3] = v.w;
                    }
                };
                // rows r .. r + kFp64Ahead - 1 with values c, the labels of the first kRows in rl; the
                // C loads of the next rows go out before them, the label reads of a block's rows before
                // the block above it (the barriers keep the compiler from moving a read next to its use)
                auto rows = [&](auto clamped, int r, double *c, double *cn) {
                    load_c(clamped, cn, i0 + r + kFp64Ahead);
#pragma unroll
                    for (int q = 0; q < kFp64Ahead; q += kRows) {
                        int(*cur)[B] = q / kRows & 1 ? rb : ra, (*next)[B] = q / kRows & 1 ? ra : rb;
#pragma unroll
                        for (int u = 0; u < kRows; ++u) labels_of(next[u], r + q + kRows + u);
                        __builtin_amdgcn_sched_barrier(0);
                        double cq[kRows];
#pragma unroll
                        for (int u = 0; u < kRows; ++u) {
                            cq[u] = c[q + u];
                            if constexpr (checked) cq[u] = i0 + r + q + u < j ? cq[u] : 0.0;
                        }
                        if constexpr (B == 16) add_if_equal16(acc, cur[0], lj, cq[0]);
                        else add_if_equal8(acc, cur[0], cur[1], lj, cq[0], cq[1]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                };
#pragma unroll
                for (int u = 0; u < kRows; ++u) labels_of(ra[u], u);
                constexpr std::bool_constant<fp64_clamps(checked, 64 - 2 * kFp64Ahead)> within{};   // groups 0 .. 64 - 2 kFp64Ahead
                constexpr std::bool_constant<fp64_clamps(checked, 64 - kFp64Ahead)> next{};         // the last: rows of the next chunk
                for (int r = 0; r < 64 - 2 * kFp64Ahead; r += 2 * kFp64Ahead) {
                    rows(within, r, ca, cb);
                    rows(within, r + kFp64Ahead, cb, ca);
                }
                rows(within, 64 - 2 * kFp64Ahead, ca, cb);
                rows(next, 64 - kFp64Ahead, cb, ca);
                if (ch + 1 < nchunks) store_labels(buf ^ 1, nxt);
            };
            for (int ch = 0; ch + 1 < nchunks; ++ch) chunk(std::false_type{}, ch);
            chunk(std::true_type{}, nchunks - 1);
            if (jok) {
                const double cjj = gld(C + (size_t)j * N + j);
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const int p = pbase + b;
                    if (p < P) gst(d.wsum + (size_t)p * N + j, fma(2.0, acc[b], cjj));
                }
            }
        }
    };
    if constexpr (LISTED) {
        each_listed_tile(t, parity, total, [&](int tile) {
            const int k = find_inst(t.tiles, t.n_inst, tile);
            work(const_at(t.desc, k), tile - const_at(t.tiles, k));
        });
    } else {
        const int tile = order ? xcd_tile(blockIdx.x, total) : blockIdx.x;
        const int k = find_inst(t.tiles, t.n_inst, tile);
        const InstDesc &d = const_at(t.desc, k);
        if (inst_stopped(d)) return;
        work(d, tile - const_at(t.tiles, k));
    }
}

// The tiles with an individual of the pair-sum's, listed by XCD in tile order: a thread per tile, an append per wave.
__global__ __launch_bounds__(256) void k_tiles(Tables t, int parity, int order, int per) {
    if (none_dense(t, parity)) return;
    const int total = const_at(t.tiles, t.n_inst), cap = tile_list_cap(total), span = (cap + 63) & ~63;
    const int g = blockIdx.x * 256 + threadIdx.x, x = __builtin_amdgcn_readfirstlane(g / span), b = (g % span) * kXcds + x;
    if (x >= kXcds) return;
    bool active = false;
    const int tile = order ? xcd_tile(min(b, total - 1), total) : b;
    if (b < total) {
        const int k = find_inst(t.tiles, t.n_inst, tile);
        const InstDesc &d = const_at(t.desc, k);
        if (!inst_stopped(d)) {
            const int local = tile - const_at(t.tiles, k), n_pairs = ((d.N + 63) / 64 + 1) / 2;
            const int p0 = tile_pos(local, n_pairs, (d.P + per - 1) / per, order).pb * per;
            int any = 0;
            for (int p = p0; p < p0 + per; p += 4)
#pragma unroll
                for (int q = 0; q < 4; ++q) any |= gld(d.route + min(p + q, d.P - 1));
            active = any != 0;
        }
    }
    const uint64_t m = __builtin_amdgcn_ballot_w64(active);
    if (!m) return;
    const int lane = threadIdx.x & 63;
    int at = 0;
    if (lane == 0) at = atomicAdd(tile_count(t, parity, x), __popcll(m));
    at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & (((uint64_t)1 << lane) - 1));
    if (active) gst(t.tile_list + (size_t)x * cap + at, tile);
}

hipError_t launch_tiles(Tables t, int total_tiles, int parity, int order, int per, hipStream_t s) {
    const int span = (total_tiles / kXcds + 1 + 63) & ~63;   // of the capacity: no less than the kernel's
    hipLaunchKernelGGL(k_tiles, dim3((kXcds * span + 255) / 256), dim3(256), 0, s, t, parity, order, per);
    return hipGetLastError();
}

hipError_t launch_pairsum_fp64(Tables t, int total_tiles, int parity, int listed, const Variant &v, hipStream_t s) {
    if (total_tiles <= 0) return hipSuccess;
    if (v.ipg != 16 && v.ipg != 8) return hipErrorInvalidValue;
    if (listed) {
        const hipError_t e = launch_tiles(t, total_tiles, parity, v.order, kFp64Waves * v.ipg, s);
        if (e != hipSuccess) return e;
    }
    auto kernel = listed ? (v.ipg == 16 ? k_pairsum_fp64<16, true> : k_pairsum_fp64<8, true>)
                         : (v.ipg == 16 ? k_pairsum_fp64<16, false> : k_pairsum_fp64<8, false>);
    hipLaunchKernelGGL(kernel, dim3(listed ? kTileListGrid : total_tiles), dim3(256), 0, s, t, parity, v.order);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Finish: one 256-thread workgroup per individual.
//   1. validity of labels and of v_j; max |v_j| (order-free);
//   2. n_s and sum_{j in s} v_j by integer LDS atomics, v_j scaled by 2^sc and
//      rounded to int64 (sc chosen per individual so N max|v| 2^sc < 2^62:
//      the integer sums are exact and order-free, error <= n_s 2^-(sc+1));
//   3. per label s with n_s > 1: c_s, domain check, the two FP64 log terms
//      of Eq. 8 in literal form. Wave w lists the labels of the w-th quarter
//      of [0, N) with n_s > 1 in ascending order (ballot + prefix); thread t
//      takes entries t, t + 256, ... of the four lists in wave order and sums
//      their terms in that order, each wave adds its lanes by a butterfly, and
//      the four wave sums are added in wave order (a fixed order).
__device__ __forceinline__ double wave_sum(double v) { return group_sum<64>(v); }

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v = fmax(v, __shfl_xor(v, m, 64));
    return v;
}

constexpr int kFinWaves = 4;
constexpr int kFinThreads = 64 * kFinWaves;
constexpr int kFinCache = 8;                       // stocks per thread kept in registers (N <= 2048)

// LDS of the finish workgroup: csum (int64) [N], cnt (int32) [N], the label
// lists (uint16, a quarter of N per wave), then per-wave reduction slots.
// Arrays are padded to 16 bytes (64-bit LDS atomics need aligned addresses).
__host__ __device__ constexpr size_t finish_csum_bytes(int max_n) {
    return ((size_t)max_n * sizeof(long long) + 15) / 16 * 16;
}
__host__ __device__ constexpr size_t finish_cnt_bytes(int max_n) {
    return ((size_t)max_n * sizeof(int) + 15) / 16 * 16;
}
__host__ __device__ constexpr int finish_quarter(int max_n) {
    return (max_n + kFinWaves - 1) / kFinWaves;
}
__host__ __device__ constexpr size_t finish_lst_bytes(int max_n) {
    return ((size_t)kFinWaves * finish_quarter(max_n) * sizeof(uint16_t) + 15) / 16 * 16;
}
__host__ __device__ constexpr size_t finish_lds_bytes(int max_n) {
    // 14.1 KB at N = 1024 (eight workgroups per CU), 57 KB at N = 4096
    return finish_csum_bytes(max_n) + finish_cnt_bytes(max_n) + finish_lst_bytes(max_n) +
           2 * kFinWaves * sizeof(double) + kFinWaves * sizeof(int);
}
// Every region of the layout starts 16-byte aligned for every N the library takes (a 64-bit LDS
// atomic at a misaligned address through a generic pointer faults), and the whole fits in LDS.
constexpr bool finish_layout_ok() {
    for (int n = 1; n <= PGA_N_MAX; ++n) {
        if (finish_csum_bytes(n) % 16 || finish_cnt_bytes(n) % 16 || finish_lst_bytes(n) % 16) return false;
        if (finish_lds_bytes(n) > (size_t)kMaxLdsBytes) return false;
    }
    return true;
}
static_assert(finish_layout_ok(), "finish LDS layout: aligned regions within the LDS limit");

// Per-label outputs and the log terms of Eq. 8 from n_s (cnt) and c_s held in
// 64-bit fixed point (csum, scale 2^sc); thread 0 writes fitness[p]. Called by
// all threads of a kFinThreads workgroup after the barrier that closed the
// writes to cnt and csum. lst holds kFinWaves lists of lst_stride labels;
// nlw holds kFinWaves ints.
__device__ __forceinline__ void finish_terms(const InstDesc &d, int p, int N, const int *cnt,
                                             const long long *csum, int sc, uint16_t *lst, int lst_stride,
                                             double *red, int *nlw, int32_t *status) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, tid = threadIdx.x;
    // Pass A (wave w, labels [w Q, (w + 1) Q)): per-label outputs, and the labels
    // with n_s > 1 compacted in ascending order; the four lists, in wave order,
    // list every such label of the individual in ascending order.
    const int QN = finish_quarter(N);                // this instance's quarter; storage is sized by max_n
    const int s_lo = wave * QN, s_hi = min(N, s_lo + QN);
    uint16_t *wl = lst + (size_t)wave * lst_stride;
    int nlist = 0;
    for (int s0 = s_lo; s0 < s_hi; s0 += 64) {
        const int s = s0 + lane;
        const int n = s < s_hi ? cnt[s] : 0;
        if (s < s_hi) {
            if (d.n_s_out) gst(d.n_s_out + (size_t)p * N + s, n);
            if (d.c_s_out) gst(d.c_s_out + (size_t)p * N + s, ldexp((double)csum[s], -sc));
        }
        const uint64_t m = __ballot(n > 1);
        if (n > 1) wl[nlist + __popcll(m & ((1ull << lane) - 1ull))] = (uint16_t)s;
        nlist += __popcll(m);
    }
    if (lane == 0) nlw[wave] = nlist;
    __syncthreads();

    // Pass B: the two FP64 log terms of Eq. 8 for each listed cluster; entry m of
    // the concatenated lists goes to thread m mod 256, so the (FP64, costly) terms
    // are spread over the whole workgroup rather than over one wave per quarter.
    int pre[kFinWaves + 1];
    pre[0] = 0;
#pragma unroll
    for (int w = 0; w < kFinWaves; ++w) pre[w + 1] = pre[w] + nlw[w];
    double L = 0.0;
    int nbad = 0;
    for (int m = tid; m < pre[kFinWaves]; m += kFinThreads) {
        int w = 0;
#pragma unroll
        for (int v = 1; v < kFinWaves; ++v) w += m >= pre[v] ? 1 : 0;
        const int s = lst[(size_t)w * lst_stride + (m - pre[w])];
        const double nd = (double)cnt[s];
        const double c = ldexp((double)csum[s], -sc);
        const double n2 = nd * nd;
        if (!(c > 0.0 && c < n2)) {
            nbad += 1;
        } else {
            L += log(nd / c) + (nd - 1.0) * log((n2 - nd) / (n2 - c));
        }
    }
    {
        const double wl_sum = wave_sum(L);
        const double wb_sum = wave_sum((double)nbad);
        if (lane == 0) {
            red[wave] = wl_sum;                      // every read of red above precedes the
            red[kFinWaves + wave] = wb_sum;          // barrier that closed the atomics
        }
    }
    __syncthreads();
    if (tid == 0) {
        double Ltot = 0.0, badtot = 0.0;
        for (int w = 0; w < kFinWaves; ++w) {
            Ltot += red[w];
            badtot += red[kFinWaves + w];
        }
        if (badtot > 0.0) {
            d.fitness[p] = -INFINITY;
            if (status) {
                atomicAdd(&status[PGA_ST_DOMAIN], (int)badtot);
                atomicAdd(&status[PGA_ST_NONFINITE], 1);
            }
        } else {
            d.fitness[p] = 0.5 * Ltot;
        }
    }
}

// The finish of individual p of instance k by one kFinThreads workgroup (every
// thread; the early returns are uniform over the workgroup).
__device__ __forceinline__ void finish_one(const Tables &t, int k, int p, int max_n, int parity, int32_t *status,
                                           unsigned char *smem) {
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, tid = threadIdx.x;
    const InstDesc &d = const_at(t.desc, k);
    if (inst_stopped(d)) return;                     // uniform over the workgroup
    const int N = d.N;
    if (d.route && gld(d.route + p) == 0) return;    // evaluated by the cluster-pair kernel
    const int32_t *__restrict__ lab = d.pop[parity] + (size_t)p * N;
    const double *__restrict__ v = d.wsum + (size_t)p * N;
    long long *csum = (long long *)smem;
    int *cnt = (int *)(smem + finish_csum_bytes(max_n));
    uint16_t *lst = (uint16_t *)(smem + finish_csum_bytes(max_n) + finish_cnt_bytes(max_n));
    double *red = (double *)(smem + finish_csum_bytes(max_n) + finish_cnt_bytes(max_n) + finish_lst_bytes(max_n));

    // Stocks j = tid + 256 u; the first kFinCache per thread stay in registers (all
    // loads issued together), later ones are read again in the accumulation pass.
    // ucache: cached slots in use, uniform over the workgroup, so the slots past N
    // cost nothing (not even masked-off instructions).
    const int ucache = min(kFinCache, (N + kFinThreads - 1) / kFinThreads);
    int lr[kFinCache];
    double vr[kFinCache];
#pragma unroll
    for (int u = 0; u < kFinCache; ++u) {
        if (u >= ucache) break;
        const int j = tid + kFinThreads * u;
        lr[u] = j < N ? gld(lab + j) : 0;
        vr[u] = j < N ? gld(v + j) : 0.0;
    }
    int bad = 0;
    double mx = 0.0;
#pragma unroll
    for (int u = 0; u < kFinCache; ++u) {
        if (u >= ucache) break;
        if (lr[u] < 0 || lr[u] >= N) bad |= 1;
        if (!isfinite(vr[u])) bad |= 2;
        else mx = fmax(mx, fabs(vr[u]));
    }
    for (int j = tid + kFinThreads * kFinCache; j < N; j += kFinThreads) {
        const int l = gld(lab + j);
        if (l < 0 || l >= N) bad |= 1;
        const double x = gld(v + j);
        if (!isfinite(x)) bad |= 2;
        else mx = fmax(mx, fabs(x));
    }
    for (int s = tid; s < N; s += kFinThreads) {
        csum[s] = 0;
        cnt[s] = 0;
    }
    {
        const double wmx = wave_max(mx);
        const double wbad = (double)((__any(bad & 1) ? 1 : 0) | (__any(bad & 2) ? 2 : 0));
        if (lane == 0) {
            red[wave] = wmx;
            red[kFinWaves + wave] = wbad;
        }
    }
    __syncthreads();
    int any_bad = 0;
#pragma unroll
    for (int w = 0; w < kFinWaves; ++w) {
        mx = fmax(mx, red[w]);
        any_bad |= (int)red[kFinWaves + w];
    }
    if (any_bad) {
        if (tid == 0) {
            d.fitness[p] = -INFINITY;
            if (status) {
                if (any_bad & 1) atomicAdd(&status[PGA_ST_LABEL], 1);
                atomicAdd(&status[PGA_ST_NONFINITE], 1);
            }
        }
        if (d.n_s_out)
            for (int s = tid; s < N; s += kFinThreads) d.n_s_out[(size_t)p * N + s] = 0;
        if (d.c_s_out)
            for (int s = tid; s < N; s += kFinThreads) d.c_s_out[(size_t)p * N + s] = 0.0;
        return;                                      // uniform: any_bad is the same for every thread
    }
    int sc = 0;
    if (mx > 0.0) {
        int e;
        frexp(mx * (double)N, &e);                   // N max|v| < 2^e
        sc = 61 - e;
    }
#pragma unroll
    for (int u = 0; u < kFinCache; ++u) {
        if (u >= ucache) break;
        if (tid + kFinThreads * u < N) {
            atomicAdd(&cnt[lr[u]], 1);
            atomicAdd((unsigned long long *)&csum[lr[u]], (unsigned long long)llrint(ldexp(vr[u], sc)));
        }
    }
    for (int j = tid + kFinThreads * kFinCache; j < N; j += kFinThreads) {
        const int l = gld(lab + j);
        const long long q = llrint(ldexp(gld(v + j), sc));
        atomicAdd(&cnt[l], 1);
        atomicAdd((unsigned long long *)&csum[l], (unsigned long long)q);
    }
    __syncthreads();

    finish_terms(d, p, N, cnt, csum, sc, lst, finish_quarter(max_n), red, (int *)(red + 2 * kFinWaves), status);
}

// Workgroup g takes individual g.
__global__ __launch_bounds__(kFinThreads) void k_finish(Tables t, int max_n, int parity, int32_t *status) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int g = blockIdx.x;
    const bool none = none_dense(t, parity), past = g >= const_at(t.inds, t.n_inst);   // the grid may exceed the total
    if (none | past) return;                         // (capacity-sized graph); one wait for both loads
    const int k = find_inst(t.inds, t.n_inst, g);
    finish_one(t, k, g - const_at(t.inds, k), max_n, parity, status, smem);
}

// Listed (cluster-pair route on, large launches): per slice of this parity's
// dense list, `per` workgroups (gridDim.x = slices * per) take its entries at,
// at + per, ... below the slice's length, so a list that is nearly empty costs a
// small launch rather than a workgroup per possible entry. (A kernel of its own:
// the loop needs more registers than the one-individual form.)
__global__ __launch_bounds__(kFinThreads) void k_finish_listed(Tables t, int max_n, int parity, int slices, int cap,
                                                               int32_t *status) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int slice = (int)blockIdx.x % slices, per = (int)gridDim.x / slices;
    const int n = __builtin_amdgcn_readfirstlane(gld(list_count(t, parity, slice)));
    for (int at = (int)blockIdx.x / slices; at < n; at += per) {
        const int32_t *e = list_entry(t, slice, cap, at);
        const int p = __builtin_amdgcn_readfirstlane(gld(e));
        const int k = __builtin_amdgcn_readfirstlane(gld(e + 1));
        finish_one(t, k, p, max_n, parity, status, smem);
        __syncthreads();                             // the next entry reuses the LDS
    }
}

// Workgroups per dense-list slice in a listed finish (at most the slice capacity).
constexpr int kFinListPerSlice = 8;

hipError_t launch_finish(Tables t, int total_inds, int max_n, int parity, int listed, int32_t *status,
                         hipStream_t s) {
    if (total_inds <= 0) return hipSuccess;
    const int n_wg = (total_inds + 3) / 4, slices = list_slices(n_wg), cap = list_slice_cap(n_wg);
    const int per = cap < kFinListPerSlice ? cap : kFinListPerSlice;
    if (listed)
        hipLaunchKernelGGL(k_finish_listed, dim3(slices * per), dim3(kFinThreads), finish_lds_bytes(max_n), s, t, max_n,
                           parity, slices, cap, status);
    else
        hipLaunchKernelGGL(k_finish, dim3(total_inds), dim3(kFinThreads), finish_lds_bytes(max_n), s, t, max_n, parity,
                           status);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Cluster-pair fitness (exact FP64 route). c_s of Eq. 6 only involves the pairs
// inside cluster s, so an individual with few such pairs is evaluated from
// them directly instead of by the O(N^2) pair-sum, by a group of GL lanes: 16
// (N <= 32), 32 (N <= 64), a wave (N <= 512) or a workgroup (N <= 2048), so that
// a 256-thread workgroup holds 16, 8, 4 or 1 individuals of one instance:
//   1. labels into registers; n_s by LDS atomics, whose old values add up to
//      the pair count sum_s n_s (n_s - 1) / 2 and give max n_s; a second atomic
//      exchanges the label's last stock for this one, which chains the stocks
//      of a cluster: prev[j] is the stock of j's cluster before it (N: none), so
//      the pairs of a cluster are j with every stock on j's chain, once each;
//   2. pairs above the limit: route[p] = 1 (the pair-sum and finish evaluate it,
//      through the dense list in large launches) and stop; the pair count of an
//      individual with N <= 64 is within the limit whatever its labels;
//   3. the labels with n_s > 1 compacted in ascending order (their n_s, and
//      csum, which starts with the sum of the diagonal), then the stocks with
//      a predecessor as items, so that the lanes of step 4 are busy whatever the
//      labels;
//   4. per item, its chain: the entries C_ij (upper triangle, as the FP64 pair-sum
//      reads it), four at a time in flight, summed in 64-bit fixed point: with
//      |C| <= 1 every partial sum is bounded by max n_s^2, and the scale 2^sc
//      keeps max n_s^2 2^sc <= 2^61, so the integer sums are exact and no result
//      depends on the order of the chain or of the atomics;
//   5. an entry with |C| > 1 or not finite sends the individual to the dense
//      route (step 2's flag), which treats it exactly as without this route; for
//      N <= 64 the wave evaluates it so itself (dense_small), and the launches of
//      a batch of small instances need no pair-sum and no finish. Otherwise the
//      log terms follow, added in the finish's order, so an individual has the
//      same bits whatever GL evaluates it.
// A chain needs no sort and no scan over the labels: the counting sort, the pair
// prefix and the search and square root per pair run that it replaces were half of
// the instructions at N = 272. What bounds it: vector instructions (log terms,
// fixed point) and the latency of LDS and C reads, about evenly.
constexpr int kSparseMaxN = 2048;                  // larger instances always take the dense route
constexpr int kSmallMaxN = kRouteAllPairsMaxN;     // evaluated here even when a C entry is out of range

__host__ __device__ constexpr size_t pad16(size_t b) { return (b + 15) / 16 * 16; }
__host__ __device__ constexpr int eval_lanes(int N) { return N <= 32 ? 16 : N <= 64 ? 32 : N <= 512 ? 64 : 256; }
// LDS of one individual: n_s, then the items, uint32[n] | a cluster's last stock, then its
// list index, uint32[n], then (N > 512: beside it) csum int64[n / 2 + 1] | prev uint16[n + 1] |
// list uint32[n / 2 + 1]. 12 n bytes: at N = 512 six workgroups per CU; 16 n above.
__host__ __device__ constexpr size_t eval_csum_off(int n) {
    return pad16(4 * (size_t)n) + (eval_lanes(n) == 256 ? pad16(4 * (size_t)n) : 0);
}
__host__ __device__ constexpr size_t eval_bytes(int n) {
    return eval_csum_off(n) + pad16(8 * ((size_t)n / 2 + 1)) + pad16(2 * ((size_t)n + 1)) +
           pad16(4 * ((size_t)n / 2 + 1));
}
constexpr uint32_t kNoCluster = 0xFFFFu;           // list index of a label with n_s <= 1
constexpr size_t kSmallScratch = 64 * (8 + 4 + 4);  // dense_small, per wave
__host__ __device__ constexpr size_t eval_lds_bytes(int N) {
    const int g = 256 / eval_lanes(N);
    return (size_t)g * eval_bytes(N) + (N <= kSmallMaxN ? 4 * kSmallScratch : 0) + (g == 1 ? 256 : 0);
}
constexpr bool eval_layout_ok() {
    for (int n = 1; n <= kSparseMaxN; ++n)
        if (eval_bytes(n) % 16 || eval_lds_bytes(n) > (size_t)kMaxLdsBytes) return false;
    return true;
}
static_assert(eval_layout_ok(), "cluster-pair LDS layout: aligned regions within the LDS limit");

int eval_blocks(int N, int P) { return N > kSparseMaxN ? (P + 255) / 256 : ceil_div(P, 256 / eval_lanes(N)); }
size_t eval_lds(int N) { return N > kSparseMaxN ? 0 : eval_lds_bytes(N); }

// Orders the LDS accesses of the wave's lanes (one wave: no barrier needed).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ unsigned long long fixed_pt(double c, int sc) {
    return (unsigned long long)llrint(ldexp(c, sc));
}

// An individual that goes to the pair-sum route joins the dense list (one
// thread). listed = 0: no lists in use (the finish reads every individual's route).
__device__ __forceinline__ void to_dense(const Tables &t, const InstDesc &d, int k, int p, int parity, int listed,
                                         int slices, int cap) {
    gst(d.route + p, 1);
    gst(any_dense(t, parity), 1);
    if (!listed) return;
    const int slice = ((const_at(t.inds, k) + p) >> 2) % slices;
    int32_t *e = list_entry(t, slice, cap, atomicAdd(list_count(t, parity, slice), 1));
    gst(e, p);
    gst(e + 1, k);
}

// The log terms of Eq. 8 of one cluster of n stocks; false if c is outside (0, n^2).
__device__ __forceinline__ bool cluster_term(int n, long long csum, int sc, double &term) {
    const double nd = (double)n;
    const double c = ldexp((double)csum, -sc);
    const double n2 = nd * nd;
    if (!(c > 0.0 && c < n2)) return false;
    term = log(nd / c) + (nd - 1.0) * log((n2 - nd) / (n2 - c));
    return true;
}

__device__ __forceinline__ void store_fitness(const InstDesc &d, int p, double Ltot, int nbad, int32_t *status) {
    if (nbad > 0) {
        d.fitness[p] = -INFINITY;
        if (status) {
            atomicAdd(&status[PGA_ST_DOMAIN], nbad);
            atomicAdd(&status[PGA_ST_NONFINITE], 1);
        }
    } else {
        d.fitness[p] = 0.5 * Ltot;
    }
}

// Individual p (N <= 64, valid labels, all 64 lanes of a wave) as the pair-sum and the finish evaluate
// it: lane j holds stock j. scratch: kSmallScratch bytes of LDS.
typedef __bf16 fit_bf16x8 __attribute__((ext_vector_type(8)));
typedef float fit_floatx4 __attribute__((ext_vector_type(4)));
__device__ __attribute__((noinline)) void dense_small(const InstDesc &d, int p, int parity, int form, int32_t *status,
                                                      unsigned char *scratch) {
    const int lane = threadIdx.x & 63, N = d.N;
    long long *csum = (long long *)scratch;
    int *cnt = (int *)(scratch + 64 * 8), *lst = cnt + 64;
    const bool in = lane < N;
    const int j = min(lane, N - 1);
    const int l = gld(d.pop[parity] + (size_t)p * N + j);
    double acc = 0.0;
    if (form == PGA_FORM_FP64) {
        for (int i = 0; i + 1 < N; ++i) {
            const int li = __builtin_amdgcn_readlane(l, i);
            if (i < j && li == l) acc += gld(d.C + (size_t)i * N + j);
        }
    } else {
        // the column kernel's MFMAs: 16 stocks at a time (lane: row and column n, rows 8 g ..), the
        // scaled split parts from their tile-major copies, the one-hot 2^-125 where i < j share a label
        const int n = lane & 15, g = lane >> 4, nti = d.ld_h >> 5;
        for (int jt = 0; 16 * jt < N; ++jt) {
            const int jj = 16 * jt + n, lj = __shfl(l, min(jj, N - 1), 64);
            fit_floatx4 a4 = {0.f, 0.f, 0.f, 0.f};
            for (int i0 = 0; i0 < min(16 * jt + 16, N); i0 += 32) {
                const size_t off = ((size_t)jt * nti + (i0 >> 5)) * 512 + (size_t)lane * 8;
                const fit_bf16x8 Ah = __builtin_bit_cast(fit_bf16x8, gld_u4(d.hs + off));
                const fit_bf16x8 Al = __builtin_bit_cast(fit_bf16x8, gld_u4(d.ls + off));
                uint32_t b[4] = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int i = i0 + 8 * g + e;
                    const int li = __shfl(l, min(i, N - 1), 64);
                    if (i < jj && li == lj) b[e >> 1] |= 0x0100u << (16 * (e & 1));
                }
                const fit_bf16x8 B = __builtin_bit_cast(fit_bf16x8, make_uint4(b[0], b[1], b[2], b[3]));
                a4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ah, B, a4, 0, 0, 0);
                a4 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Al, B, a4, 0, 0, 0);
            }
            // D[n][n] is register n % 4 of the lane of column n whose row group holds row n
            const int r = n & 3;
            const float v = r == 0 ? a4[0] : r == 1 ? a4[1] : r == 2 ? a4[2] : a4[3];
            const float s = __shfl(v, 16 * ((lane & 15) >> 2) + (lane & 15), 64);
            if ((lane >> 4) == jt) acc += (double)s;
        }
    }
    const double v = in ? fma(2.0, acc, gld(d.C + (size_t)j * N + j)) : 0.0;
    const bool nonfinite = __any(!isfinite(v));
    const double mx = wave_max(isfinite(v) ? fabs(v) : 0.0);
    cnt[lane] = 0;
    csum[lane] = 0;
    wave_lds_sync();
    if (nonfinite) {
        if (lane == 0) {
            d.fitness[p] = -INFINITY;
            if (status) atomicAdd(&status[PGA_ST_NONFINITE], 1);
        }
        if (in && d.n_s_out) gst(d.n_s_out + (size_t)p * N + lane, 0);
        if (in && d.c_s_out) gst(d.c_s_out + (size_t)p * N + lane, 0.0);
        return;
    }
    int sc = 0;
    if (mx > 0.0) {
        int e;
        frexp(mx * (double)N, &e);
        sc = 61 - e;
    }
    if (in) {
        atomicAdd(&cnt[l], 1);
        atomicAdd((unsigned long long *)&csum[l], (unsigned long long)llrint(ldexp(v, sc)));
    }
    wave_lds_sync();
    const int ns = in ? cnt[lane] : 0;
    if (in && d.n_s_out) gst(d.n_s_out + (size_t)p * N + lane, ns);
    if (in && d.c_s_out) gst(d.c_s_out + (size_t)p * N + lane, ldexp((double)csum[lane], -sc));
    const uint64_t m = __ballot(ns > 1);
    if (ns > 1) lst[__popcll(m & ((1ull << lane) - 1ull))] = lane;
    wave_lds_sync();
    double term = 0.0;
    bool bad = false;
    if (lane < __popcll(m)) {
        const int s = lst[lane];
        bad = !cluster_term(cnt[s], csum[s], sc, term);
        if (bad) term = 0.0;
    }
    const double Ltot = group_sum<64>(term);
    const int nbad = __popcll(__ballot(bad));
    if (lane == 0) store_fitness(d, p, Ltot, nbad, status);
    wave_lds_sync();                                 // the next individual reuses the scratch
}

// The evaluation of individuals local * (256 / GL) + (group) of instance k by the groups of a
// 256-thread workgroup (see above). SL: stocks per lane.
template <int GL, int SL>
__device__ __forceinline__ void eval_pairs(const Tables &t, const InstDesc &d, int k, int local, int parity,
                                           double frac, int listed, int slices, int cap, int form, int32_t *status,
                                           unsigned char *smem, int32_t stopped) {
    constexpr bool kBlock = GL == 256;
    constexpr int WL = kBlock ? 64 : GL;             // lanes that vote together
    constexpr int NW = kBlock ? 4 : 1;               // such sets per individual
    const int tid = threadIdx.x, lane = tid & 63, gl = tid & (GL - 1), grp = tid / GL;
    const int wv = kBlock ? __builtin_amdgcn_readfirstlane(tid >> 6) : 0;
    const int N = d.N, P = d.P;
    int p = local * (256 / GL) + grp;
    if constexpr (GL == 64) p = __builtin_amdgcn_readfirstlane(p);
    const bool live = p < P;                         // GL < 64: a group past P works on P - 1 and stores nothing
    if (GL >= 64 && !live) return;
    const int pc = min(p, P - 1);
    unsigned char *b = smem + (size_t)grp * eval_bytes(N);
    uint32_t *cnt = (uint32_t *)b;
    uint32_t *last = (uint32_t *)(b + pad16(4 * (size_t)N));
    b += eval_csum_off(N);
    unsigned long long *csum = (unsigned long long *)b;   b += pad16(8 * ((size_t)N / 2 + 1));
    uint16_t *prev = (uint16_t *)b;         b += pad16(2 * ((size_t)N + 1));
    uint32_t *lst = (uint32_t *)b;
    // kBlock: per wave T | max n_s | lists per label quarter (two words) | items, flags; then 4 doubles
    uint32_t *ired = (uint32_t *)(smem + eval_bytes(N));
    double *red = (double *)(ired + 20);
    auto sync = [&]() {
        if constexpr (kBlock) __syncthreads();
        else wave_lds_sync();
    };
    // votes of a set of WL lanes; bit i: its lane i
    auto vote = [&](bool x) -> uint64_t {
        const uint64_t m = __ballot(x);
        if constexpr (WL == 64) return m;
        else return (m >> (lane & ~(WL - 1))) & ((1ull << WL) - 1ull);
    };
    const int wl = lane & (WL - 1);
    const uint64_t below = (1ull << wl) - 1ull;

    const int32_t *__restrict__ lab = d.pop[parity] + (size_t)pc * N;
    const double *__restrict__ C = d.C;
    const int nu = (N + GL - 1) / GL;                // slots in use, uniform
    uint32_t lr[SL];
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        if (u >= nu) break;
        const int j = gl + GL * u;
        lr[u] = j < N ? (uint32_t)gld(lab + j) : 0u;
    }
    const bool ones = gld(d.diag + N) == 1.0;        // every C_jj is 1 (uniform)
    if (flag_stops(d, stopped)) return;              // uniform over the workgroup
    bool badl = false;
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        if (u >= nu) break;
        const int j = gl + GL * u;
        if (j < N) {
            cnt[j] = 0;
            last[j] = (uint32_t)N;
            if (lr[u] >= (uint32_t)N) {
                badl = true;
                lr[u] = 0;
            }
        }
    }
    if (gl == 0) {
        prev[N] = (uint16_t)N;
        if constexpr (kBlock) ired[16] = ired[17] = ired[18] = 0;   // items, a label out of range, an entry out of range
    }
    sync();
    bool bad_label = false;
    if constexpr (kBlock) {
        if (badl) ired[17] = 1;                      // read after the next barrier
    } else {
        bad_label = vote(badl) != 0;
    }
    auto invalid = [&]() {                           // as the finish: labels outside [0, N)
        if (gl == 0) {
            gst(d.route + p, 0);
            d.fitness[p] = -INFINITY;
            if (status) {
                atomicAdd(&status[PGA_ST_LABEL], 1);
                atomicAdd(&status[PGA_ST_NONFINITE], 1);
            }
        }
        for (int s = gl; s < N; s += GL) {
            if (d.n_s_out) gst(d.n_s_out + (size_t)p * N + s, 0);
            if (d.c_s_out) gst(d.c_s_out + (size_t)p * N + s, 0.0);
        }
    };
    if constexpr (!kBlock) {
        if (bad_label && live) invalid();
        if (GL >= 64 && bad_label) return;
    }
    const bool good = live && !bad_label;

    // ---- n_s, pair count, chains
    uint32_t T = 0, nmax = 0;
    uint32_t has = 0;                                // bit u: the slot's stock has a predecessor
    const int QN = (N + NW - 1) / NW;                // labels per wave of a workgroup
    uint32_t ql = 0, qh = 0;                         // kBlock: labels that reach two stocks here, by quarter (16 bits each)
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        if (u >= nu) break;
        const int j = gl + GL * u;
        if (j < N) {
            const uint32_t old = atomicAdd(&cnt[lr[u]], 1u);
            const uint32_t pv = atomicExch(&last[lr[u]], (uint32_t)j);
            T += old;
            nmax = max(nmax, old + 1);
            if constexpr (kBlock) {
                if (old == 1) {
                    const uint32_t l = lr[u];
                    const uint32_t one = l >= (uint32_t)(2 * QN) ? (l >= (uint32_t)(3 * QN) ? 0x10000u : 1u)
                                                                 : (l >= (uint32_t)QN ? 0x10000u : 1u);
                    if (l >= (uint32_t)(2 * QN)) qh += one;
                    else ql += one;
                }
            }
            prev[j] = (uint16_t)pv;
            has |= (pv < (uint32_t)N ? 1u : 0u) << u;
        }
    }
    nmax = group_reduce<WL>(nmax, [](uint32_t a, uint32_t c) { return max(a, c); });
    if constexpr (GL >= 64) T = group_reduce<WL>(T, [](uint32_t a, uint32_t c) { return a + c; });
    int nl = 0, base = 0;                            // list entries, and this wave's first
    if constexpr (kBlock) {
        const auto add = [](uint32_t a, uint32_t c) { return a + c; };
        ql = group_reduce<64>(ql, add);
        qh = group_reduce<64>(qh, add);
        if (wl == 0) {
            ired[wv] = T;
            ired[4 + wv] = nmax;
            ired[8 + wv] = ql;
            ired[12 + wv] = qh;
        }
    }
    sync();
    if constexpr (kBlock) {
        if (ired[17]) {
            invalid();
            return;                                  // uniform
        }
        T = ired[0] + ired[1] + ired[2] + ired[3];
        nmax = max(max(ired[4], ired[5]), max(ired[6], ired[7]));
        ql = ired[8] + ired[9] + ired[10] + ired[11];
        qh = ired[12] + ired[13] + ired[14] + ired[15];
        const int q0 = (int)(ql & 0xFFFFu), q1 = (int)(ql >> 16), q2 = (int)(qh & 0xFFFFu), q3 = (int)(qh >> 16);
        base = wv == 0 ? 0 : wv == 1 ? q0 : wv == 2 ? q0 + q1 : q0 + q1 + q2;
        nl = q0 + q1 + q2 + q3;
    }
    if (GL >= 64 && (double)T > route_limit(N, frac)) {
        if (gl == 0) to_dense(t, d, k, p, parity, listed, slices, cap);
        return;                                      // uniform over the individual's lanes
    }
    const int sc = 61 - (32 - __builtin_clz(nmax * nmax));   // max n_s^2 < 2^(61 - sc)

    // ---- clusters with n_s > 1, ascending (wave w of a workgroup: the w-th quarter of the labels)
    const int s_lo = wv * QN, s_hi = min(N, s_lo + QN);
    bool badc = false;
    for (int s0 = s_lo; s0 < s_hi; s0 += WL) {
        const int s = s0 + wl;
        const uint32_t n = s < s_hi ? cnt[s] : 0;
        if (good && s < s_hi) {
            if (d.n_s_out) gst(d.n_s_out + (size_t)p * N + s, (int32_t)n);
            if (d.c_s_out && n <= 1)                 // an unused label, or a singleton's diagonal entry
                gst(d.c_s_out + (size_t)p * N + s,
                    n == 0 ? 0.0 : ones ? 1.0 : ldexp((double)(long long)fixed_pt(gld(d.diag + last[s]), sc), -sc));
        }
        const uint64_t m = vote(n > 1);
        const int at = base + __popcll(m & below);
        if (n > 1) {
            lst[at] = n | ((uint32_t)s << 16);
            if constexpr (kBlock) csum[at] = ones ? (unsigned long long)n << sc : 0ull;
        }
        if (s < s_hi) last[s] = n > 1 ? (uint32_t)at : kNoCluster;   // the chains are complete: now the list index
        base += __popcll(m);
    }
    if constexpr (!kBlock) nl = base;
    sync();
    // ---- items: stocks with a predecessor, with their cluster (in the place of n_s)
    int ni = 0;
    if constexpr (kBlock) {
        int own = 0;
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            if (u >= nu) break;
            own += __popcll(__ballot((has >> u) & 1u));
        }
        int at = 0;
        if (wl == 0) at = (int)atomicAdd(&ired[16], (uint32_t)own);
        ni = __builtin_amdgcn_readfirstlane(at);
    }
#pragma unroll
    for (int u = 0; u < SL; ++u) {
        if (u >= nu) break;
        const bool h = (has >> u) & 1u;
        const uint64_t m = vote(h);
        lr[u] = last[lr[u]];                         // the list index from here on
        if (h) cnt[ni + __popcll(m & below)] = (uint32_t)(gl + GL * u) | (lr[u] << 16);
        ni += __popcll(m);
    }
    sync();
    if constexpr (kBlock) {
        ni = (int)ired[16];
    } else {                                         // csum takes the place of last: the sum of the diagonal to start with
        for (int m = gl; m < nl; m += GL) csum[m] = ones ? (unsigned long long)(lst[m] & 0xFFFFu) << sc : 0ull;
        sync();
    }
    if (!ones) {
#pragma unroll
        for (int u = 0; u < SL; ++u) {
            if (u >= nu) break;
            const int j = gl + GL * u;
            if (j < N) {
                const double dg = gld(d.diag + j);
                if (!(fabs(dg) <= 1.0)) badc = true;
                else if (lr[u] != kNoCluster) atomicAdd(&csum[lr[u]], fixed_pt(dg, sc));
            }
        }
        sync();
    }

    // ---- pairs
    const double S = ldexp(2.0, sc);                 // rint(c S) = the fixed point of 2 c (exact scaling)
    for (int x = gl; x < ni; x += GL) {
        const uint32_t it = cnt[x];
        const int j = (int)(it & 0xFFFFu);
        double hi = 0.0, lo = 0.0;                   // the integer sum as hi 2^32 + lo, both exact
        auto entry = [&](int i) { return gld(C + (uint32_t)(__mul24(min(i, j), N) + max(i, j))); };
        auto take = [&](double c) {
            badc |= !(fabs(c) <= 1.0);
            const double q = rint(c * S);
            const double h = floor(q * 0x1p-32);
            hi += h;
            lo += fma(h, -0x1p32, q);
        };
        int i = prev[j];
        do {
            const int i1 = prev[i], i2 = prev[i1], i3 = prev[i2];
            // Past the end of its chain a lane loads nothing (an unused load still costs its line: with
            // the diagonal entry in its place half of the L2 reads at N = 1024 were such loads).
            const bool v1 = i1 < N, v2 = i2 < N, v3 = i3 < N;
            const double c0 = entry(i);
            double c1 = 0.0, c2 = 0.0, c3 = 0.0;
            if (v1) c1 = entry(i1);
            if (v2) c2 = entry(i2);
            if (v3) c3 = entry(i3);
            if (__any(v2)) {
                take(c2);
                take(c3);
            }
            if (__any(v1)) take(c1);
            take(c0);
            i = prev[i3];
        } while (i < N);
        const double h2 = floor(lo * 0x1p-32);
        const unsigned long long v = ((unsigned long long)(uint32_t)((int)hi + (int)h2) << 32) +
                                     (uint32_t)fma(h2, -0x1p32, lo);
        atomicAdd(&csum[it >> 16], v);
    }
    bool handed = false;
    if constexpr (kBlock) {
        if (badc) ired[18] = 1;
        __syncthreads();
        handed = ired[18] != 0;
    } else {
        handed = vote(badc) != 0;
        sync();
    }
    if constexpr (GL >= 64) {
        if (handed) {
            if (gl == 0) to_dense(t, d, k, p, parity, listed, slices, cap);
            return;
        }
    }

    // ---- log terms, in the finish's order: entry m of the list to virtual thread m mod 256, the
    // virtual waves' butterflies, then the four in order
    if (d.c_s_out && good && !handed)
        for (int m = gl; m < nl; m += GL)
            gst(d.c_s_out + (size_t)p * N + (lst[m] >> 16), ldexp((double)(long long)csum[m], -sc));
    double Ltot = 0.0;
    int nbad = 0;
    if constexpr (kBlock) {
        double L = 0.0;
        for (int m = tid; m < nl; m += 256) {
            double term;
            if (cluster_term((int)(lst[m] & 0xFFFFu), (long long)csum[m], sc, term)) L += term;
            else ++nbad;
        }
        L = group_sum<64>(L);
        nbad = (int)group_reduce<64>((uint32_t)nbad, [](uint32_t a, uint32_t c) { return a + c; });
        if (wl == 0) {
            red[wv] = L;
            ired[wv] = (uint32_t)nbad;
        }
        __syncthreads();
        for (int w = 0; w < 4; ++w) Ltot += red[w];
        nbad = (int)(ired[0] + ired[1] + ired[2] + ired[3]);
    } else {
        // The two logs of a term go to neighbouring lanes (half the vector work when the list is
        // short, and in a converged population it is: 128 x 1000 individuals of N = 18, 42 to 39 us;
        // a workgroup with four waves for one list gains nothing); the term replaces its cluster's csum.
        double *terms = (double *)csum;
        for (int x0 = 0; x0 < 2 * nl; x0 += GL) {
            const int x = x0 + gl, m = x >> 1;
            const bool in = x < 2 * nl;
            const int n = in ? (int)(lst[m] & 0xFFFFu) : 2;
            const double nd = (double)n, n2 = nd * nd;
            const double c = in ? ldexp((double)(long long)csum[m], -sc) : 1.0;
            const bool ok = c > 0.0 && c < n2;
            const double l = log((x & 1 ? n2 - nd : nd) / (x & 1 ? n2 - c : c));
            const double term = fma(nd - 1.0, dpp_val<kQuad1>(l), l);   // even lanes: log(n / c) + (n - 1) log(..)
            if (in && !(x & 1)) {
                terms[m] = ok ? term : 0.0;
                nbad += ok ? 0 : 1;
            }
        }
        nbad = (int)group_reduce<GL>((uint32_t)nbad, [](uint32_t a, uint32_t c) { return a + c; });
        sync();
        for (int m0 = 0; m0 < nl; m0 += GL)          // GL < 64: one round, nl <= N / 2 <= GL
            Ltot += group_sum<GL>(0.0 + (m0 + gl < nl ? terms[m0 + gl] : 0.0));
    }
    if (gl == 0 && good && !handed) {
        gst(d.route + p, 0);
        store_fitness(d, p, Ltot, nbad, status);
    }
    if constexpr (GL < 64) {
        // individuals with an entry out of range, one after another by the whole wave
        uint64_t todo = __ballot(gl == 0 && good && handed);
        while (todo) {
            const int src = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int q = __builtin_amdgcn_readlane(p, src);
            if (lane == 0) gst(d.route + q, 0);
            dense_small(d, q, parity, form, status,
                        smem + (size_t)(256 / GL) * eval_bytes(N) + (size_t)(tid >> 6) * kSmallScratch);
        }
    }
}

constexpr int kEvalRun = 128;

// Workgroup b takes the next individuals of the instance that t.evals gives it. In large launches
// (listed) workgroup 0 also empties the dense list of the other parity, which the evaluation
// before this one used. Instances above kSparseMaxN: a thread per individual sends it to the
// dense route.
__global__ __launch_bounds__(256, 8) void k_eval(Tables t, int parity, double frac, int listed, int slices, int cap,
                                                 int form, int32_t *status) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int b = blockIdx.x;
    if (listed && b == 0)
        for (int i = threadIdx.x; i < kListSlices; i += 256) gst(list_count(t, parity ^ 1, i), 0);
    if (b == 0 && threadIdx.x < kXcds) {             // the next evaluation's tile lists
        gst(tile_count(t, parity ^ 1, threadIdx.x), 0);
        gst(tile_next(t, parity ^ 1, threadIdx.x), 0);
        if (threadIdx.x == 0) gst(any_dense(t, parity ^ 1), 0);
    }
    if (b >= const_at(t.evals, t.n_inst)) return;              // the grid may exceed the total (capacity-sized graph)
    // Workgroups go to the XCDs in turn; runs of kEvalRun consecutive ones are given to one XCD, so
    // that it reads the C of few instances at a time (256 instances, N ~ U{32..512}: 334 us without,
    // 290 with runs of 128 to 512; a run of an eighth of the launch is less even).
    const int total = const_at(t.evals, t.n_inst), run8 = b / (kXcds * kEvalRun), in8 = b % (kXcds * kEvalRun);
    const int bb = (run8 + 1) * kXcds * kEvalRun > total
                       ? b
                       : run8 * kXcds * kEvalRun + in8 % kXcds * kEvalRun + in8 / kXcds;
    const int k = find_inst(t.evals, t.n_inst, bb);
    const InstDesc &d = const_at(t.desc, k);
    const int32_t stopped = stop_flag(d, t);         // tested behind the label loads
    const int N = d.N, local = bb - const_at(t.evals, k);
    if (N <= 32) eval_pairs<16, 2>(t, d, k, local, parity, frac, listed, slices, cap, form, status, smem, stopped);
    else if (N <= 64) eval_pairs<32, 2>(t, d, k, local, parity, frac, listed, slices, cap, form, status, smem, stopped);
    else if (N <= 512) eval_pairs<64, 8>(t, d, k, local, parity, frac, listed, slices, cap, form, status, smem, stopped);
    else if (N <= kSparseMaxN)
        eval_pairs<256, 8>(t, d, k, local, parity, frac, listed, slices, cap, form, status, smem, stopped);
    else {
        const int p = 256 * local + threadIdx.x;
        if (p < d.P && !flag_stops(d, stopped)) to_dense(t, d, k, p, parity, listed, slices, cap);
    }
}

hipError_t launch_eval(Tables t, int total_inds, int blocks, size_t lds, int parity, double frac, int listed, int form,
                       int32_t *status, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    const int n_wg = (total_inds + 3) / 4, slices = list_slices(n_wg), cap = list_slice_cap(n_wg);
    hipLaunchKernelGGL(k_eval, dim3(blocks), dim3(256), lds, s, t, parity, frac, listed, slices, cap, form, status);
    return hipGetLastError();
}

}  // namespace pga
