// Internal declarations shared by the libpga translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pga.h"

namespace pga {

// Device-side descriptor of one GA instance (or of one pga_fitness call).
// Written into the workspace before the kernels run; every kernel finds its
// instance through it, so the same kernels serve one instance or a ragged
// batch, and a captured HIP graph stays valid when pointers change.
struct InstDesc {
    int32_t N, P, E, ld_h;
    const double *C;
    const uint16_t *hi, *lo;    // BF16 split parts (ld_h x ld_h)
    uint16_t *hs, *ls;          // split parts times 2^125, tile-major (workspace; BF16x2 form only)
    int32_t *pop[2];            // ping-pong population buffers
    double *fitness;            // P
    double *stats;              // (G + 1) x 4 or null
    double *wsum;               // P x N: v_pj = C_jj + 2 sum_{i<j} [s_pi = s_pj] C_ij
    int32_t *elite;             // PGA_E_MAX
    int32_t *n_s_out;           // P x N or null
    double *c_s_out;            // P x N or null
    uint32_t p_cross, p_mut;
    uint64_t seed;
    uint32_t inst_id, gen0;
    pga_term_state *term;       // termination state or null
    int32_t stall_gens;         // 0: no termination test
    int32_t ind0;               // first global individual index
    double tol;
    int32_t selection;          // PGA_SELECT_*
    int32_t pad_;
    int32_t *sus_rank;          // P: 1-based rank (SUS only; workspace)
    uint64_t *sus_cum;          // P: inclusive prefix of the SUS weights (workspace)
    int32_t *route;             // P: 1 = evaluated by pair-sum + finish, 0 = by the cluster-pair
                                // kernel (workspace); null: every individual takes the pair-sum
    double *diag;               // N + 1: C_jj, contiguous, then 1 if every C_jj is 1 (workspace; with route)
    uint32_t *ns2;              // P x ceil(N / 32): bit l set when label l has n_s >= 2 (workspace; BF16x2 form)
};

// Prefix tables: for n instances, arrays of n + 1 exclusive prefix sums.
struct Tables {
    const InstDesc *desc;
    const int32_t *tiles;       // prefix of pair-sum tiles (of the kernel variant in use)
    const int32_t *inds;        // prefix of individuals
    const int32_t *evals;       // prefix of cluster-pair workgroups (eval_blocks)
    const int32_t *breeds;      // prefix of breed workgroups (of the launch's BreedShape)
    int32_t *sq;                // dense list counters (see list_count)
    int32_t *sq_list;           // dense list entries (see list_entry)
    int32_t *tile_list;         // pair-sum tiles to do (see tile_count); null in a workspace without room for them
    int32_t n_inst;
    int32_t routed;             // the cluster-pair kernel has run: any_dense and the routes hold
};

// Workgroups of one launch are handed to the eight XCDs in turn (workgroup i
// to XCD i mod 8), each XCD with its own L2.

// Dense list. With the cluster-pair route on, a large launch's cluster-pair
// kernel lists the individuals that it leaves to the pair-sum and the finish, so
// that the finish has work for the listed ones only. The list is cut into
// kListSlices slices with a counter each, so that its appends do not all meet on
// one address; an entry is the pair (index in the instance, instance). The
// evaluation of parity q fills the list of q and empties that of 1 - q, which the
// evaluation before it used.
constexpr int kListSlices = 1024;
constexpr int kListCounters = 2 * kListSlices;     // [parity][slice]
// Tile lists, one per XCD: counters [parity][XCD], a line each for the entries and for the next to take,
// behind the dense list's.
constexpr int kXcds = 8;
constexpr int kTileCounterStride = 32;
constexpr int kTileCounters = 2 * kXcds * 2 * kTileCounterStride;
// Slices in use for a launch of n_wg groups of four individuals (group i's go to
// slice i mod slices; one slice per group up to kListSlices, so the list launches
// of a small population are no larger than a workgroup per individual), and
// entries per slice.
__host__ __device__ constexpr int list_slices(int n_wg) {
    return n_wg < 1 ? 1 : (n_wg < kListSlices ? n_wg : kListSlices);
}
__host__ __device__ constexpr int list_slice_cap(int n_wg) {
    return 4 * ((n_wg + list_slices(n_wg) - 1) / list_slices(n_wg));
}
// int32 words of the entries
__host__ __device__ constexpr size_t list_words(int n_wg) {
    return (size_t)2 * kListSlices * (size_t)list_slice_cap(n_wg);
}

// ---- geometry of the pair-sum kernels --------------------------------------
constexpr int kFp64Waves = 4;                      // waves per workgroup, one column (stock) per lane
constexpr int kFp64Cols = 64;                      // columns per workgroup
constexpr int kFp64Ahead = 4;                      // rows whose C loads go out together: two or four add blocks
constexpr int kFp64Round = 1024;                   // workgroups resident at once: four a CU (registers)
constexpr int64_t kL2Bytes = 8ll << 22;            // the eight XCDs' L2s, 4 MiB each
// The FP64 pair-sum walks a column block's rows in chunks of 64, kFp64Ahead at a time: with rows r .. of a chunk go out the
// loads of the kFp64Ahead rows behind them. They may be past N, where row N - 1 is loaded instead, in the
// last chunk of a block and where they belong to the next chunk.
__host__ __device__ constexpr bool fp64_clamps(bool last_chunk, int r) { return last_chunk || r + 2 * kFp64Ahead > 64; }
__host__ __device__ constexpr int fp64_row(int i, int N, bool clamped) { return clamped && i > N - 1 ? N - 1 : i; }
constexpr int kMfmaWaves = 4;                      // waves per workgroup, 16 columns each
constexpr int kMfmaCols = 16 * kMfmaWaves;         // columns per workgroup
constexpr int kMfmaRowCodes = 8192;                // row codes staged in LDS per workgroup (column kernel)
constexpr int kMfmaFlushRows = 512;                // FP32 accumulators are flushed to FP64 every 512 rows
constexpr int kMaxLdsBytes = 65536;                // LDS a workgroup may allocate
// Fourth word of a raw buffer descriptor (no swizzle, no stride, 32-bit data
// format): byte addressing from the base, loads past num_records return zero.
constexpr int kBufWord3 = 0x00020000;

inline int32_t ceil_div(int64_t a, int64_t b) { return (int32_t)((a + b - 1) / b); }
// Pair-sum tiles fold the triangle: column blocks jb and n_jb - 1 - jb share a workgroup.
inline int32_t fold_pairs(int32_t N, int32_t cols) { return (ceil_div(N, cols) + 1) / 2; }
inline int32_t split_ld(int32_t N) { return (int32_t)(((int64_t)N + 31) / 32 * 32); }

// A pair-sum kernel variant (what the autotuner chooses between):
//   ipg    individuals per group: per wave in the FP64 kernel (the workgroup
//          holds 4 x ipg), per workgroup in the MFMA kernel;
//   order  tile order: 0 workgroup b runs tile b, column pairs fastest;
//          1 tiles renumbered so each XCD gets a contiguous range, column
//          pairs fastest (an XCD sees few individual batches, all columns);
//          2 as 1 with individual batches fastest (an XCD sees few column
//          pairs, so their C rows stay in its L2);
//   kind   MFMA form only: how the B operand (the one-hot) is made and how
//          many columns there are:
//          kKindCols   one column per stock, one-hot built in registers from
//                      row codes (a DPP broadcast, an xor and a saturating
//                      subtract per two elements);
//          kKindPacked compacted columns (one per label with n_s >= 2, packed
//                      over the workgroup's individuals), one-hot built in
//                      registers from each lane's own row codes;
//          kKindLut    one column per stock, one-hot read from LDS: an 8-bit
//                      row mask per (individual, label code, row group) indexes
//                      a 256-entry table of bf16 one-hot octets.
// Every variant performs the same arithmetic in the same order per
// individual, so all of them give bitwise identical results.
constexpr int32_t kKindCols = 0, kKindPacked = 1, kKindLut = 2;
struct Variant {
    int32_t form, ipg, order, kind;
};
int n_variants(int form);
Variant variant_at(int form, int idx);
inline int32_t pair_tiles(int32_t N, int32_t P, const Variant &v) {
    const int per = v.form == PGA_FORM_FP64 ? kFp64Waves * v.ipg : v.ipg;
    return fold_pairs(N, 64) * ceil_div(P, per);
}
inline size_t mfma_code_stride(int max_n) { return ((size_t)max_n + 15) / 16 * 16; }
constexpr int kMfmaASlots = 2;                     // A ring slots per wave (2 KB each) in the packed kernel
// Rows of row codes staged per pass and individual by the packed kernel (a
// multiple of 512), and the per-individual stride of its staged codes in 16-bit
// words (16 bytes of padding).
__host__ __device__ constexpr int mfma_rows(int ipg) { return 4096 / ipg > 512 ? 4096 / ipg : 512; }
__host__ __device__ constexpr int mfma_row_stride(int ipg) { return mfma_rows(ipg) + 8; }
// LDS of the MFMA kernels.
// Column and packed kernels: row codes (the column kernel: kMfmaRowCodes words
// for all individuals; the packed kernel: [ipg][stride]), label -> code tables,
// and for the packed kernel A rings and 1 KB per wave of scratch.
// LUT kernel, at fixed offsets: the one-hot table (256 x 16 bytes), two
// buffers of row masks (16 KB each: [chunk][ipg][64 codes][4 row groups]
// 16-bit words of lut_rows(ipg) rows, one pass), then the label -> code tables.
__host__ __device__ constexpr size_t mfma_align256(size_t x) { return (x + 255) / 256 * 256; }
constexpr size_t kLutTableBytes = 256 * 16;
constexpr size_t kLutMaskOff = kLutTableBytes;
constexpr size_t kLutMaskBytes = 16384;             // one buffer
constexpr size_t kLutCodeOff = kLutMaskOff + 2 * kLutMaskBytes;
__host__ __device__ constexpr int lut_rows(int ipg) { return (int)(kLutMaskBytes / 512) * 32 / ipg; }
__host__ __device__ constexpr size_t mfma_lds_code_off(int ipg, int kind) {
    return kind == kKindLut      ? kLutCodeOff
           : kind == kKindPacked ? mfma_align256(sizeof(uint16_t) * (size_t)ipg * mfma_row_stride(ipg))
                                 : sizeof(uint16_t) * (size_t)kMfmaRowCodes;
}
__host__ __device__ constexpr size_t mfma_lds_ring_off(int ipg, int cstride, int kind) {
    return mfma_lds_code_off(ipg, kind) + mfma_align256((size_t)ipg * cstride);
}
__host__ __device__ constexpr size_t mfma_lds_scratch_off(int ipg, int cstride, int kind) {
    return mfma_lds_ring_off(ipg, cstride, kind) + (size_t)kMfmaWaves * kMfmaASlots * 2048;
}
inline size_t mfma_lds_bytes(int ipg, int max_n, int kind) {
    const int cstride = (int)mfma_code_stride(max_n);
    if (kind == kKindLut) return kLutCodeOff + (size_t)ipg * cstride;
    return kind == kKindPacked ? mfma_lds_scratch_off(ipg, cstride, kind) + (size_t)kMfmaWaves * 1024
                               : mfma_lds_ring_off(ipg, cstride, kind);
}
static_assert(mfma_lds_code_off(4, kKindPacked) % 256 == 0 && mfma_lds_code_off(8, kKindPacked) % 256 == 0 &&
                  mfma_lds_code_off(16, kKindPacked) % 256 == 0 && mfma_lds_code_off(8, kKindCols) % 256 == 0 &&
                  kLutMaskOff % 256 == 0 && kLutCodeOff % 256 == 0,
              "MFMA LDS regions are 256-byte aligned");
static_assert(lut_rows(4) % 32 == 0 && lut_rows(8) % 32 == 0 && lut_rows(16) % 32 == 0 &&
                  lut_rows(8) * 8 / 32 * 512 == (int)kLutMaskBytes,
              "a LUT pass is whole 32-row chunks and its row masks fill the mask region");
inline bool variant_ok(const Variant &v, int max_n) {
    return v.form != PGA_FORM_BF16X2 ||
           (mfma_lds_bytes(v.ipg, max_n, v.kind) <= (size_t)kMaxLdsBytes && (v.kind != kKindLut || v.ipg <= 8));
}

struct TilePos {
    int jp, pb;
};
// (column pair, individual batch) of tile `local` of an instance.
__device__ __forceinline__ TilePos tile_pos(int local, int n_pairs, int n_pb, int order) {
    if (order == 2) return TilePos{local / n_pb, local % n_pb};
    return TilePos{local % n_pairs, local / n_pairs};
}

// Workgroup b of T runs tile xcd_tile(b, T): the hardware deals workgroups to
// the 8 XCDs round-robin (b mod 8), so XCD x receives the contiguous tiles
// [start_x, start_x + count_x) and shares their labels in its own L2.
__device__ __forceinline__ int xcd_tile(int b, int T) {
    const int q = T >> 3, r = T & 7, x = b & 7, i = b >> 3;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + i;
}

// ---- Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11) ---------------------
enum : uint32_t { kTagInit = 0, kTagSel = 1, kTagXov = 2, kTagMut = 3, kTagSus = 4, kTagShuf = 5 };

struct U4 { uint32_t x, y, z, w; };

__device__ __forceinline__ U4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                            uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t a = (uint64_t)0xD2511F53u * (uint64_t)c0;
        const uint64_t b = (uint64_t)0xCD9E8D57u * (uint64_t)c2;
        const uint32_t n0 = (uint32_t)(b >> 32) ^ c1 ^ k0;
        const uint32_t n2 = (uint32_t)(a >> 32) ^ c3 ^ k1;
        c1 = (uint32_t)b;
        c3 = (uint32_t)a;
        c0 = n0;
        c2 = n2;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return U4{c0, c1, c2, c3};
}

__device__ __forceinline__ U4 draw(uint32_t blk, uint32_t who, uint32_t gen, uint32_t tag,
                                   uint32_t inst, uint64_t seed) {
    return philox4x32_10(blk, who, gen, tag | (inst << 4), (uint32_t)seed, (uint32_t)(seed >> 32));
}

// floor(w * m / 2^32)
__device__ __forceinline__ uint32_t scale_u32(uint32_t w, uint32_t m) { return __umulhi(w, m); }

// ---- lane groups ------------------------------------------------------------
// Cross-lane steps without LDS: rotations within rows of 16 lanes (DPP), and the swaps of
// neighbouring rows and of the wave's halves.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
constexpr int kRor8 = 0x128, kRor4 = 0x124, kRor2 = 0x122, kRor1 = 0x121;   // row_ror:n
constexpr int kQuad2 = 0x4E, kQuad1 = 0xB1;                                  // quad_perm [2,3,0,1], [1,0,3,2]

template <int GL, class Op>                       // over GL <= 64 lanes; op commutative and associative
__device__ __forceinline__ uint32_t group_reduce(uint32_t v, Op op) {
    v = op(v, dpp<kRor8>(v));
    v = op(v, dpp<kRor4>(v));
    v = op(v, dpp<kRor2>(v));
    v = op(v, dpp<kRor1>(v));
    if constexpr (GL >= 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        v = op(r[0], r[1]);
    }
    if constexpr (GL >= 64) {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        v = op(r[0], r[1]);
    }
    return v;
}

template <int CTRL>
__device__ __forceinline__ double dpp_val(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(double, ((uint64_t)dpp<CTRL>((uint32_t)(b >> 32)) << 32) | dpp<CTRL>((uint32_t)b));
}
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    return v + dpp_val<CTRL>(v);
}
// The butterfly sum over a wave (lane l with l ^ 32, 16, 8, 4, 2, 1), in every lane: a step's sum is commutative,
// and once the values repeat with period 8 (4) in a row, the row's rotation by 4 (2) pairs the same
// values as the exchange. GL = 32 and 16: the sum of the group's values followed by zeros.
template <int GL>
__device__ __forceinline__ double group_sum(double v) {
    auto halves = [](double x, auto swap) {
        const uint64_t b = __builtin_bit_cast(uint64_t, x);
        const auto l = swap((uint32_t)b), h = swap((uint32_t)(b >> 32));
        return __builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]) +
               __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]);
    };
    if constexpr (GL >= 64)
        v = halves(v, [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); });
    if constexpr (GL >= 32)
        v = halves(v, [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); });
    v = dpp_add<kRor8>(v);
    v = dpp_add<kRor4>(v);
    v = dpp_add<kQuad2>(v);
    return dpp_add<kQuad1>(v);
}

// ---- explicit global-memory access ------------------------------------------
// Pointers read from a descriptor are generic; the compiler then emits flat
// loads, which count on the same wait counter as LDS operations, so a wait for
// an LDS result would also wait for every in-flight prefetch. These helpers
// access global memory through address-space-1 pointers (global loads/stores).
#define PGA_GLOBAL __attribute__((address_space(1)))
typedef uint32_t pga_u32x4 __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ T gld(const T *p) { return *(const PGA_GLOBAL T *)p; }
template <class T>
__device__ __forceinline__ void gst(T *p, T v) { *(PGA_GLOBAL T *)p = v; }
__device__ __forceinline__ uint4 gld_u4(const void *p) {
    const pga_u32x4 v = *(const PGA_GLOBAL pga_u32x4 *)p;
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Descriptors and prefixes do not change during a launch. Through the constant address space their loads are
// scalar also behind a store (of which the compiler cannot tell that it leaves them alone): as vector loads the
// lookup of a workgroup's instance and descriptor was a chain of up to a dozen memory latencies in
// the cluster-pair kernel, and put the pair-sums' addresses into vector registers.
#define PGA_CONST __attribute__((address_space(4)))
template <typename T>
__device__ __forceinline__ const T &const_at(const T *p, int i) {
    return *(const T *)(const PGA_CONST T *)(uintptr_t)(p + i);
}

// Instance lookup: largest k with prefix[k] <= t (prefix is exclusive, n + 1 entries).
__device__ __forceinline__ int find_inst(const int32_t *prefix, int n, int t) {
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (const_at(prefix, mid) <= t) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// A stopped instance (termination test fired) is skipped by every kernel.
__device__ __forceinline__ bool inst_stopped(const InstDesc &d) {
    return d.term != nullptr && gld(&d.term->stopped) != 0;
}

// Tile lists of launches with more than kTileListMin pair-sum tiles: k_tiles lists the tiles that hold an
// individual of the pair-sum's, and kTileListGrid workgroups take them one by one, each from its XCD's list
// first (the tiles that share C and labels stay on one XCD). Where the cluster-pair kernel has most
// individuals, a workgroup per tile only to find that out took 83 us for the 79 000 tiles of 256 instances of N ~
// U{32..512}, P = 512; the two launches take 29 us there. (Without a list, 8 tiles a workgroup: 47 us, but
// 5 to 12% slower where every tile is to do.) Where every tile is to do the list costs 2% (15 000 tiles of N ~ 700),
// so smaller launches, which have less to gain, keep a workgroup per tile.
__device__ __forceinline__ int32_t *tile_count(const Tables &t, int parity, int xcd) {
    return t.sq + kListCounters + (parity * kXcds + xcd) * 2 * kTileCounterStride;
}
__device__ __forceinline__ int32_t *tile_next(const Tables &t, int parity, int xcd) {
    return tile_count(t, parity, xcd) + kTileCounterStride;
}
// One word per parity: does the evaluation leave any individual to the pair-sum and the finish? Their workgroups
// look at it before anything else. (Where there is nothing to do each workgroup looked up its instance and its
// individuals' routes first: pair-sum and finish 6.1 and 4.7 us at N = 1024, P = 4096, now 4.7 and 4.6 in the
// trace, and 20 generations 1170 -> 1092 us.)
__device__ __forceinline__ int32_t *any_dense(const Tables &t, int parity) { return tile_count(t, parity, 0) + 1; }
__device__ __forceinline__ bool none_dense(const Tables &t, int parity) {
    return (t.routed != 0) & (const_at(any_dense(t, parity), 0) == 0);   // one wait with the caller's other first loads
}
__device__ __forceinline__ int tile_list_cap(int total) { return total / kXcds + 1; }

// work(tile) for every listed tile, by the whole workgroup. Only thread 0 looks at what changes during the
// launch (the next tile to take) and hands its tile to the others. While more than two tiles a workgroup are left
// it takes one ahead, so that the two latencies of a tile pass behind the work (48 instances of N ~ 145, every
// tile to do: 7.4 ms for 10 generations against 8.4); near the end a tile taken ahead would wait for a busy
// workgroup (256 instances, few tiles: 34 us a launch against 23).
template <typename F>
__device__ __forceinline__ void each_listed_tile(const Tables &t, int parity, int total, F &&work) {
    __shared__ int taken[2];
    const int cap = tile_list_cap(total);
    for (int o = 0; o < kXcds; ++o) {
        const int x = ((int)blockIdx.x + o) % kXcds;
        const int n = __builtin_amdgcn_readfirstlane(gld(tile_count(t, parity, x)));   // the same in every wave
        if (n == 0) continue;
        const int32_t *list = t.tile_list + (size_t)x * cap;
        int32_t *next = tile_next(t, parity, x);
        __syncthreads();                                   // taken is free
        const int margin = 2 * (int)gridDim.x / kXcds;
        auto take = [&] { return gld(next) >= n ? n : atomicAdd(next, 1); };   // (an old value of next: the sum is >= n)
        auto take_ahead = [&](int i) { return i + margin < n ? atomicAdd(next, 1) : -1; };   // -1: not yet
        auto tile_of = [&](int i) { return i < n ? gld(list + i) : -1; };
        int ahead = -1;                                    // thread 0's
        if (threadIdx.x == 0) {
            const int i = take();
            taken[0] = tile_of(i);
            ahead = take_ahead(i);
        }
        for (int k = 0;; ++k) {
            __syncthreads();                               // taken[k & 1] is there, the other one and the work's LDS free
            const int tile = __builtin_amdgcn_readfirstlane(taken[k & 1]);
            if (tile < 0) break;
            int after = -1;
            const bool have = ahead >= 0;
            if (threadIdx.x == 0 && have) {
                after = tile_of(ahead);
                ahead = take_ahead(ahead);
            }
            work(tile);
            if (threadIdx.x == 0) taken[(k + 1) & 1] = have ? after : tile_of(take());
        }
    }
}

// The same, to be tested later: the load goes out here, and the test waits for it (by readfirstlane; a load
// from an address that the compiler knows to be uniform is waited for at once). A memory latency less at
// the start of every workgroup.
__device__ __forceinline__ int32_t stop_flag(const InstDesc &d, const Tables &t) {
    int z = 0;
    asm("" : "+v"(z));
    return gld((d.term ? &d.term->stopped : (const int32_t *)t.desc) + z);   // (without a state: any word)
}
__device__ __forceinline__ bool flag_stops(const InstDesc &d, int32_t flag) {
    return d.term && __builtin_amdgcn_readfirstlane(flag) != 0;
}

// Total order used for ranking, elites and tournaments: higher fitness first,
// then lower index. -inf compares equal to -inf, so ties among invalid
// individuals also go to the lower index.
__device__ __forceinline__ bool ranks_before(double fa, int a, double fb, int b) {
    return fa > fb || (fa == fb && a < b);
}

// Cluster-pair route limit of an instance of N stocks: frac N (N - 1) / 2 pairs,
// and every pair when N <= 64 (a 64-stock block is the pair-sum's smallest unit
// of work per individual, and its finish a workgroup per individual, while the
// cluster-pair evaluation is bounded by the N (N - 1) / 2 <= 2016 pairs).
constexpr int kRouteAllPairsMaxN = 64;
__host__ __device__ __forceinline__ double route_limit(int N, double frac) {
    const double all = 0.5 * (double)N * (double)(N - 1);
    return N <= kRouteAllPairsMaxN ? all : floor(frac * all);
}

__device__ __forceinline__ int32_t *list_count(const Tables &t, int parity, int slice) {
    return t.sq + parity * kListSlices + slice;
}
__device__ __forceinline__ int32_t *list_entry(const Tables &t, int slice, int cap, int at) {
    return t.sq_list + 2 * ((size_t)slice * cap + at);
}

// ---- launchers (defined in the kernel translation units) ---------------------
hipError_t launch_corr(const double *R, int N, int T, int64_t ld, double *mu, double *ss, double *C, uint16_t *hi,
                       uint16_t *lo, double *part, int32_t *status, hipStream_t s);
size_t gram_ws_doubles(int N);      // partial Gram tiles of the FP64 MFMA Gram (correlation, EWMA)
hipError_t launch_split(const double *C, int N, uint16_t *hi, uint16_t *lo, hipStream_t s);
size_t ewma_ws_doubles(int N, int T);   // market means, weight roots and the old diagonal
hipError_t launch_ewma(const double *R, int N, int T, int64_t ld, double lam, int reset, int market, double *S,
                       double *C, uint16_t *hi, uint16_t *lo, double *ws, double *part, int32_t *status, hipStream_t s);

hipError_t launch_write_desc(const InstDesc &d, int32_t tiles, InstDesc *dst, int32_t *prefix2, hipStream_t s);
hipError_t launch_pairsum_fp64(Tables t, int total_tiles, int parity, int listed, const Variant &v, hipStream_t s);
hipError_t launch_pairsum_mfma(Tables t, int total_tiles, int parity, int listed, const Variant &v, int max_n,
                               hipStream_t s);
hipError_t launch_nsmask(Tables t, int total_inds, int max_n, int parity, hipStream_t s);
// listed: evaluate the dense list of this parity (cluster-pair route on), else every individual.
hipError_t launch_finish(Tables t, int total_inds, int max_n, int parity, int listed, int32_t *status, hipStream_t s);
// Cluster-pair workgroups of an instance, and the LDS of one of them.
int eval_blocks(int N, int P);
// The tables of a single-instance call, as a kernel argument.
struct DescBlob {
    InstDesc d;
    int32_t prefix[8];   // {0, tiles}, {0, P}, {0, evaluation blocks}, {0, 0}; the list counters follow, zeroed
    static DescBlob of(const InstDesc &d, int32_t tiles) {
        DescBlob b{};
        b.d = d;
        b.prefix[1] = tiles;
        b.prefix[3] = d.P;
        b.prefix[5] = eval_blocks(d.N, d.P);
        return b;
    }
};
__device__ __forceinline__ void write_desc(const DescBlob &b, InstDesc *dst, int32_t *prefix) {   // one workgroup
    if (threadIdx.x == 0) *dst = b.d;
    if (threadIdx.x < 8) prefix[threadIdx.x] = b.prefix[threadIdx.x];
    for (int i = threadIdx.x; i < kListCounters + kTileCounters; i += blockDim.x) prefix[8 + i] = 0;
}
// Split parts (max_ld > 0), diagonals and, single != null, the tables of a call.
hipError_t launch_prep(const Tables &t, const InstDesc *single, int32_t tiles, int max_ld, hipStream_t s);
size_t eval_lds(int N);
// listed: fill the dense list (kManyInds individuals or more).
hipError_t launch_eval(Tables t, int total_inds, int blocks, size_t lds, int parity, double frac, int listed, int form,
                       int32_t *status, hipStream_t s);


hipError_t launch_rank(Tables t, int gen_off, int final, hipStream_t s);
// Shape of a breed launch: the most passes of a slot's lanes over its gene pairs (few in small
// launches, whose time is a slot's chain of passes; many in large ones, where few lanes per
// slot keep all of them busy), and at least this many slots per workgroup of an instance of at most kBreedSmallN stocks.
struct BreedShape {
    int passes, min_small;
};
constexpr int kBreedSmallN = 128;
constexpr int kBreedRun = 16;    // workgroups of a run on one XCD (8: within 2% everywhere)
struct BreedSplit {
    int gl, chr;             // lanes per slot, slots per workgroup: powers of two, gl chr >= 256
};
__host__ __device__ constexpr BreedSplit breed_split(int N, const BreedShape &b) {
    const int npair = (N + 1) / 2;
    int gl = 16;
    while (gl < 256 && gl * b.passes < npair) gl *= 2;
    const int chr = N <= kBreedSmallN && 256 / gl < b.min_small ? b.min_small : 256 / gl;
    return BreedSplit{gl, chr};
}
// LDS of a breed workgroup of an instance of N stocks: per slot its two parents, whether it crosses, and four
// crossover words per 128 genes.
__host__ __device__ constexpr size_t breed_bytes(int N, const BreedShape &b) {
    return sizeof(uint32_t) * (size_t)breed_split(N, b).chr * (3 + 4 * (size_t)((N + 127) / 128));
}
// The most over N = 1 .. max_n. The words rise with N and the slots fall: the largest is at the last N of one of the slot
// counts, kBreedSmallN or 2 gl passes, or at max_n.
constexpr size_t breed_lds_bytes(int max_n, const BreedShape &b) {
    size_t most = breed_bytes(max_n, b);
    auto at = [&](int n) {
        const size_t x = n < max_n ? breed_bytes(n, b) : 0;
        most = x > most ? x : most;
    };
    at(kBreedSmallN);
    for (int gl = 16; gl < 256; gl *= 2) at(2 * gl * b.passes);
    return most;
}
// Why the lines lie there (us of a breed launch in the trace). 4096 slots: 2 / 8 passes 6.5 / 9.7 at 1 x 1000 slots of N =
// 500 and 9.1 / 10.4 at 3 x 1000 of N <= 900, but 15.2 / 13.2 at 4096 slots of N = 1024 and 22 / 17 at 16 000 of N ~
// U{32..512}. 65 536 slots: 8 / 16 passes 25.4 / 26.7 at 32 768 slots of N ~ U{32..512}, 39.6 / 36.4 at 65 536 and
// 97.6 / 97.6 at 131 072; 16 / 64 slots a workgroup 14.9 / 11.5 at 66 000 and 26 / 17.6 at 131 000 slots of N <= 32,
// 36.4 / 32.9 at 131 000 of N = 96, 42.4 / 40.5 at N = 128; past it they lose: 64 / 75 at N = 200, 112 / 129 at
// N = 300, 161 / 216 at 66 000 of N = 1024, 611 / 1279 of N = 4096. Below 65 536, 16 / 64 slots 6.5 / 8 at 20 000 of
// N = 18.
constexpr BreedShape breed_shape(int inds) {
    return BreedShape{inds >= 65536 ? 16 : inds >= 4096 ? 8 : 2, inds >= 65536 ? 64 : 1};
}
inline int breed_blocks(int N, int P, const BreedShape &b) { return ceil_div(P, breed_split(N, b).chr); }
hipError_t launch_init(Tables t, int blocks, const BreedShape &b, hipStream_t s);
constexpr int kTileListMin = 16384, kTileListGrid = 1024;   // grid: four workgroups a CU, what their registers allow
// (a value of bucket(), so that launches of one captured shape agree on it)
// Lists the tiles of the launch; per = individuals of a tile.
hipError_t launch_tiles(Tables t, int total_tiles, int parity, int order, int per, hipStream_t s);
// An MFMA pair-sum launch of at most kSplitTiles tiles (two workgroups a CU) gives each of a tile's two column blocks
// a workgroup, the long ones first: N = 333, P = 777 (294 tiles) 15 -> 12 us, the call 33.0 -> 29.4; N = P = 500
// 47.8 -> 45.9. (The FP64 kernel gained 2 to 3% with few tiles and lost 3% near 512; a launch argument
// instead of a kernel of its own cost the large launches 0.8%.)
constexpr int kSplitTiles = 512;
hipError_t launch_breed(Tables t, int blocks, const BreedShape &b, int parity, int gen_off, int fold, int sus_listed, int max_n,
                        hipStream_t s);
// Launches of at least kManyInds individuals (more than the chip holds at a
// workgroup each) run the finish over the dense list; smaller ones a workgroup
// per individual.
constexpr int kManyInds = 8192;
constexpr int kSusSortMax = 4096;                  // largest P of a launch whose rank kernel does the SUS: its LDS and registers
hipError_t launch_rank_sus(Tables t, int max_p, int gen_off, hipStream_t s);
hipError_t launch_sus(Tables t, int max_p, hipStream_t s);
hipError_t launch_copy_back(Tables t, int blocks, const BreedShape &b, int G, hipStream_t s);
// Records a hipError_t for pga_last_hip_error() on this thread.
void note_hip_error(int e);

// pga_fitness with a choice of whether launches may be event-timed (the
// allocation-free entry point passes false).
int fitness_call(const double *C, const uint16_t *C_hi, const uint16_t *C_lo, int32_t N, const int32_t *labels,
                 int32_t P, int32_t form, double *fitness, int32_t *n_s, double *c_s, int32_t *status, void *ws,
                 size_t ws_bytes, hipStream_t s, bool timing_allowed);

hipError_t launch_best(const double *fitness, const int32_t *labels, int P, int N, int32_t *out,
                       double *out_f, hipStream_t s);

}  // namespace pga
