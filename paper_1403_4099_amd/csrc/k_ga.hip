// Genetic-algorithm kernels (Algorithm 1 of Section 4.2.3; operators of
// Section 3.1): initial population, ranking and statistics, the fused
// breed step (elitism + tournament selection + uniform crossover +
// mutation + replacement into the other ping-pong buffer), and the
// report of the fittest labeling in canonical form.
//
// Random numbers: Philox4x32-10, counter (block, individual or child,
// generation, tag | instance << 4), key = seed. A draw is keyed by the
// absolute generation and the instance id, never by launch layout, so a run
// gives the same bits alone or inside a batch and across resumes.
#include "pga_internal.hpp"

#include <type_traits>

#include <math.h>

namespace pga {

typedef int32_t gene2 __attribute__((ext_vector_type(2), aligned(4)));   // rows need not be aligned
typedef int32_t gene4 __attribute__((ext_vector_type(4), aligned(4)));

// ---------------------------------------------------------------------------
// Initial population: gene i of individual p is scale_u32(word i%4 of draw
// (i/4, p, gen0, INIT), N). The breed launch's split: a workgroup makes the slots [c0, c0 + chr)
// of one instance, gl lanes each (a workgroup per individual took 113 us for 128 000 of N = 18,
// five of its lanes at work; 14.6 us).
__global__ __launch_bounds__(256) void k_init(Tables t, BreedShape shape) {
    const int wg = blockIdx.x;
    if (wg >= const_at(t.breeds, t.n_inst)) return;                  // the grid may exceed the total (capacity-sized graph)
    const int k = find_inst(t.breeds, t.n_inst, wg);
    const InstDesc &d = const_at(t.desc, k);
    const int N = d.N, tid = threadIdx.x;
    const BreedSplit split = breed_split(N, shape);
    const int c0 = (wg - const_at(t.breeds, k)) * split.chr, gl = tid & (split.gl - 1);
    if (c0 == 0 && tid == 0 && d.term) {
        pga_term_state z;
        z.ref = -INFINITY;
        z.stall = z.stopped = z.gens = z.call_gens = 0;
        *d.term = z;
    }
    const int nq = (N + 3) >> 2;
    for (int ci = tid / split.gl; ci < split.chr; ci += 256 / split.gl) {
        const int p = c0 + ci;
        if (p >= d.P) break;
        int32_t *__restrict__ row = d.pop[0] + (size_t)p * N;
        for (int q = gl; q < nq; q += split.gl) {
            const U4 w = draw((uint32_t)q, (uint32_t)p, d.gen0, kTagInit, d.inst_id, d.seed);
            const gene4 v = {(int32_t)scale_u32(w.x, (uint32_t)N), (int32_t)scale_u32(w.y, (uint32_t)N),
                             (int32_t)scale_u32(w.z, (uint32_t)N), (int32_t)scale_u32(w.w, (uint32_t)N)};
            const int i = 4 * q;
            if (i + 4 <= N) {
                *(PGA_GLOBAL gene4 *)(row + i) = v;
            } else {
                gst(row + i, v.x);
                if (i + 1 < N) gst(row + i + 1, v.y);
                if (i + 2 < N) gst(row + i + 2, v.z);
            }
        }
    }
}

hipError_t launch_init(Tables t, int blocks, const BreedShape &b, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_init, dim3(blocks), dim3(256), 0, s, t, b);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Ranking and statistics: one workgroup per instance. Elite r is the best
// individual ranked after elite r-1 in the total order (fitness desc, index
// asc), found by a block arg-best reduction; the order is total, so the
// result does not depend on the reduction's shape. Statistics row gen_off:
// {best, mean of finite fitnesses (-inf if none), #-inf, argbest}.
struct Cand {
    double f;
    int i;
};

__device__ Cand block_best(Cand c, double *rf, int *ri) {
    rf[threadIdx.x] = c.f;
    ri[threadIdx.x] = c.i;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) {
            const double fo = rf[threadIdx.x + w];
            const int io = ri[threadIdx.x + w];
            const int im = ri[threadIdx.x];
            if (io >= 0 && (im < 0 || ranks_before(fo, io, rf[threadIdx.x], im))) {
                rf[threadIdx.x] = fo;
                ri[threadIdx.x] = io;
            }
        }
        __syncthreads();
    }
    Cand r{rf[0], ri[0]};
    __syncthreads();
    return r;
}

// Best of a wave (i < 0: no candidate), in every lane: the largest fitness, then the lowest index
// among the lanes that hold it, by row rotations and row and half swaps without LDS. (Exchanges
// of whole candidates with a comparison each are four times the instructions, in one chain.)
__device__ __forceinline__ Cand wave_best(Cand c) {
    const auto swap16 = [](uint32_t x) { return __builtin_amdgcn_permlane16_swap(x, x, false, false); };
    const auto swap32 = [](uint32_t x) { return __builtin_amdgcn_permlane32_swap(x, x, false, false); };
    auto halves = [](double x, auto swap) {
        const uint64_t b = __builtin_bit_cast(uint64_t, x);
        const auto l = swap((uint32_t)b), h = swap((uint32_t)(b >> 32));
        return fmax(__builtin_bit_cast(double, ((uint64_t)h[0] << 32) | l[0]),
                    __builtin_bit_cast(double, ((uint64_t)h[1] << 32) | l[1]));
    };
    const double own = c.i >= 0 ? c.f : -INFINITY;
    double f = own;
    f = fmax(f, dpp_val<kRor8>(f));
    f = fmax(f, dpp_val<kRor4>(f));
    f = fmax(f, dpp_val<kRor2>(f));
    f = fmax(f, dpp_val<kRor1>(f));
    f = halves(f, swap16);
    f = halves(f, swap32);
    const uint32_t i = group_reduce<64>(own == f ? (uint32_t)c.i : 0xFFFFFFFFu,   // -1 is the largest
                                        [](uint32_t a, uint32_t b) { return min(a, b); });
    return Cand{f, (int)i};
}

// Elite selection, termination state and statistics of one instance by one
// workgroup of kRankThreads threads: the rank kernel, and, when the breed
// kernel does the ranking itself (no SUS, no early stop), a breed workgroup per
// instance. Both use this code with the same thread count, so their
// statistics agree bit for bit. Each thread keeps up to CACHE of its fitness
// values in registers (all loads issued at once) and re-reads the rest; every
// thread visits its values in the same order whatever CACHE is, so CACHE
// changes no result.
constexpr int kRankThreads = 256;
constexpr int kRankWaves = kRankThreads / 64;
constexpr int kRankCache = 16;

struct RankLds {
    double wf[kRankWaves];
    int wi[kRankWaves];
    double lf[kRankWaves * PGA_E_MAX];                     // each wave's best, in rank order
    int li[kRankWaves * PGA_E_MAX];
    int ord[PGA_E_MAX];                                    // the ranking
    double best;
};

__device__ __forceinline__ void stats_row(const InstDesc &d, int gen_off, Cand best, int P, double total, double inv) {
    double *row = d.stats + 4 * (size_t)gen_off;
    const double nfin = (double)P - inv;
    row[0] = best.f;
    row[1] = nfin > 0.0 ? total / nfin : -INFINITY;
    row[2] = inv;
    row[3] = (double)best.i;
}

template <int CACHE>
struct RankBlock {
    const double *__restrict__ f;
    int P;
    RankLds &sh;
    double fr[CACHE];

    __device__ void load() {
#pragma unroll
        for (int v = 0; v < CACHE; ++v) {
            const int p = threadIdx.x + v * kRankThreads;
            fr[v] = p < P ? gld(f + p) : -INFINITY;
        }
    }
    // Best candidate of this thread ranked after prev (prev.i < 0: no bound).
    __device__ Cand thread_best(Cand prev) const {
        Cand c{0.0, -1};
#pragma unroll
        for (int v = 0; v < CACHE; ++v) {
            const int p = threadIdx.x + v * kRankThreads;
            if (p >= P) break;
            if (prev.i >= 0 && !ranks_before(prev.f, prev.i, fr[v], p)) continue;
            if (c.i < 0 || ranks_before(fr[v], p, c.f, c.i)) c = Cand{fr[v], p};
        }
        for (int p0 = threadIdx.x + CACHE * kRankThreads; p0 < P; p0 += 4 * kRankThreads) {
            double fq[4];                                  // four loads in flight, then the compares
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * kRankThreads;
                fq[u] = p < P ? gld(f + p) : -INFINITY;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * kRankThreads;
                if (p >= P) break;
                if (prev.i >= 0 && !ranks_before(prev.f, prev.i, fq[u], p)) continue;
                if (c.i < 0 || ranks_before(fq[u], p, c.f, c.i)) c = Cand{fq[u], p};
            }
        }
        return c;
    }
    // Sums of a and b over the workgroup, for thread 0.
    __device__ void block_sum2(double &a, double &b) {
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        a = group_sum<64>(a);
        b = group_sum<64>(b);
        if (lane == 0) {
            sh.wf[wave] = a;
            sh.wi[wave] = (int)b;
        }
        __syncthreads();
        a = b = 0.0;
        for (int w = 0; w < kRankWaves; ++w) {
            a += sh.wf[w];
            b += (double)sh.wi[w];
        }
    }
    // Ranks 0 .. rounds-1 from one read of the values: each thread keeps its kTop
    // best in rank order, and round r of a wave takes the best of its threads' heads. A
    // thread whose kTop are all taken looks for its next best again (thread_best),
    // so any number of ranks is exact; up to P = kTop kRankThreads no thread has more
    // values than it keeps. The same read accumulates the statistics partials.
    static constexpr int kTop = 4;
    __device__ void ranked_once(int rounds, double &sum, double &ninv) {
        Cand top[kTop];
#pragma unroll
        for (int k = 0; k < kTop; ++k) top[k] = Cand{0.0, -1};
        sum = 0.0;
        ninv = 0.0;
        auto take = [&](double fp, int p) {
            if (isfinite(fp)) sum += fp;
            else ninv += 1.0;
            Cand x{fp, p};
#pragma unroll
            for (int k = 0; k < kTop; ++k)
                if (x.i >= 0 && (top[k].i < 0 || ranks_before(x.f, x.i, top[k].f, top[k].i))) {
                    const Cand y = top[k];
                    top[k] = x;
                    x = y;
                }
        };
#pragma unroll
        for (int v = 0; v < CACHE; ++v) {
            const int p = threadIdx.x + v * kRankThreads;
            if (p >= P) break;
            take(fr[v], p);
        }
        for (int p0 = threadIdx.x + CACHE * kRankThreads; p0 < P; p0 += 4 * kRankThreads) {
            double fq[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * kRankThreads;
                fq[u] = p < P ? gld(f + p) : -INFINITY;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int p = p0 + u * kRankThreads;
                if (p >= P) break;
                take(fq[u], p);
            }
        }
        // Each wave lists its own `rounds` best (no barrier between the rounds), then every listed
        // candidate counts those that rank before it.
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        for (int r = 0; r < rounds; ++r) {
            const Cand b = wave_best(top[0]);
            if (lane == 0) {
                sh.lf[wave * rounds + r] = b.f;
                sh.li[wave * rounds + r] = b.i;            // -1: the wave has no more
            }
            if (b.i >= 0 && b.i == top[0].i) {                 // this thread's head was taken
#pragma unroll
                for (int k = 0; k + 1 < kTop; ++k) top[k] = top[k + 1];
                top[kTop - 1] = Cand{0.0, -1};
                if (top[0].i < 0 && r + 1 < rounds && (int)threadIdx.x + kTop * kRankThreads < P) top[0] = thread_best(b);
            }
        }
        __syncthreads();
        const int n = kRankWaves * rounds;                     // at most kRankThreads
        if ((int)threadIdx.x < n) {
            const double f = sh.lf[threadIdx.x];
            const int i = sh.li[threadIdx.x];
            int before = 0;
#pragma unroll 8
            for (int q = 0; q < n; ++q) {
                const int iq = sh.li[q];
                before += iq >= 0 && ranks_before(sh.lf[q], iq, f, i) ? 1 : 0;
            }
            if (i >= 0 && before < rounds) {
                sh.ord[before] = i;
                if (before == 0) sh.best = f;
            }
        }
        __syncthreads();
    }
    // Ranks 0 .. rounds-1 (rounds <= min(P, PGA_E_MAX)) into sh.ord and, with stats set,
    // the statistics row gen_off: {best, mean of finite fitnesses (-inf if none),
    // #-inf, argbest}; returns the best. ranked(): called once the ranks are known,
    // before the statistics.
    template <typename F>
    __device__ Cand rank_and_stats(const InstDesc &d, int rounds, int gen_off, bool stats, F &&ranked) {
        double sum, ninv;
        ranked_once(rounds, sum, ninv);
        ranked();
        const Cand best{sh.best, sh.ord[0]};
        if (stats) store_stats(d, gen_off, best, sum, ninv);
        return best;
    }
    __device__ void store_stats(const InstDesc &d, int gen_off, Cand best, double total, double inv) {
        block_sum2(total, inv);
        if (threadIdx.x == 0) stats_row(d, gen_off, best, P, total, inv);
    }
};

// Termination state after this generation's best b (thread 0 of the ranking
// workgroup): improvement, stall count, stop flag; the generation about to be
// bred is counted unless this is the final evaluation or the run stopped.
// Algorithm 1 tests each generation once: the first evaluation of a call
// (first != 0) re-evaluates the population a previous call tested last when
// the state has already tested a generation (ref finite or stall > 0), and
// then does not enter the test again, so a run split into several calls is
// the same run as one call.
__device__ void term_update(const InstDesc &d, pga_term_state st, double b, int final, int first) {
    const bool retest = first && (isfinite(st.ref) || st.stall != 0);
    if (!retest) {
        const bool improved = isfinite(st.ref) ? (b > st.ref + d.tol * fmax(1.0, fabs(st.ref))) : isfinite(b);
        if (improved) {
            st.ref = b;
            st.stall = 0;
        } else {
            st.stall += 1;
        }
        if (d.stall_gens > 0 && st.stall >= d.stall_gens) st.stopped = 1;
    }
    if (!final && !st.stopped) {
        st.gens += 1;
        st.call_gens += 1;
    }
    *d.term = st;
}

__global__ __launch_bounds__(kRankThreads) void k_rank(Tables t, int gen_off, int final) {
    __shared__ RankLds sh;
    const InstDesc &d = const_at(t.desc, blockIdx.x);
    if (d.P == 0) return;                                  // a padding slot of a capacity-sized launch
    const int P = d.P, E = d.E;
    // The fitness values, the stop flag and (thread 0) the termination state are
    // all requested before any of them is used.
    RankBlock<kRankCache> rb{d.fitness, P, sh};
    rb.load();
    pga_term_state st{};
    if (d.term) {
        const bool stopped = inst_stopped(d);
        if (threadIdx.x == 0) st = *d.term;
        __syncthreads();                                   // every thread has read the flag
        if (gen_off == 0 && threadIdx.x == 0) {
            gst(&d.term->call_gens, 0);
            st.call_gens = 0;
        }
        if (stopped) return;
    }
    if (d.selection == PGA_SELECT_SUS)                     // the SUS rank kernel adds into these
        for (int p = threadIdx.x; p < P; p += kRankThreads) gst(d.sus_rank + p, 1);
    const Cand best = rb.rank_and_stats(d, E > 1 ? E : 1, gen_off, d.stats != nullptr, [&] {
        if ((int)threadIdx.x < E) gst(d.elite + threadIdx.x, sh.ord[threadIdx.x]);
    });
    if (d.term && threadIdx.x == 0) term_update(d, st, best.f, final, gen_off == 0);
}

hipError_t launch_rank(Tables t, int gen_off, int final, hipStream_t s) {
    hipLaunchKernelGGL(k_rank, dim3(t.n_inst), dim3(kRankThreads), 0, s, t, gen_off, final);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Breed: slot c of the next population.
//   c < E : copy elite c unchanged (elitism).
//   c >= E: parents A, B = winners of two tournaments of two on draw
//           (0, c, g, SELECT); crossover iff word 0 of (0, c, g, CROSSOVER)
//           < p_cross, and then gene j from B iff bit j%32 of word (j%128)/32
//           of (1 + j/128, c, g, CROSSOVER); mutation of gene j iff word
//           2(j%2) of (j/2, c, g, MUTATION) < p_mut, new label from the
//           next word.
// A thread takes gene pairs (j, j+1) so one mutation draw covers two genes.
__device__ __forceinline__ int tournament2(const double *f, int a, int b) {
    const double fa = f[a], fb = f[b];
    return ranks_before(fa, a, fb, b) ? a : b;
}

// ---------------------------------------------------------------------------
// Stochastic universal sampling after rank scaling (PGA_SELECT_SUS).
// P <= 4096: the rank kernel of the launch does it all (k_rank_sus below). Larger:
//   k_sus_rank:   rank_p = 1 + #{q : q ranks before p}; workgroup (x, y, inst)
//                 compares individuals [256x, 256x + 256) with [256y, 256y + 256)
//                 and adds its integer counts atomically (exact, order-free);
//   k_sus_prefix: weight floor(sqrt(floor(2^48 / rank))) (0 for -inf, 1 for all
//                 when every fitness is -inf) and the inclusive prefix over the
//                 individuals in index order, in 64-bit integers;
//   k_breed:      pointer k at floor((u + k W) / n) picks the individual whose
//                 segment holds it; child E + j uses pointers pi(2j), pi(2j+1).
__global__ __launch_bounds__(256) void k_sus_rank(Tables t) {
    __shared__ double fq[256];
    const InstDesc &d = const_at(t.desc, blockIdx.z);
    if (d.P == 0 || d.selection != PGA_SELECT_SUS || inst_stopped(d)) return;
    const int P = d.P;
    const int p0 = blockIdx.x * 256, q0 = blockIdx.y * 256;
    if (p0 >= P || q0 >= P) return;                          // uniform over the workgroup
    const int p = p0 + threadIdx.x, q = q0 + threadIdx.x;
    fq[threadIdx.x] = q < P ? gld(d.fitness + q) : 0.0;
    __syncthreads();
    if (p >= P) return;
    const double fp = gld(d.fitness + p);
    const int nq = min(256, P - q0);
    int cnt = 0;
    for (int r = 0; r < nq; ++r) cnt += ranks_before(fq[r], q0 + r, fp, p) ? 1 : 0;
    if (cnt) atomicAdd(d.sus_rank + p, cnt);
}

// The permutation of [0, n) that pairs SUS parents: a Feistel network on two halves of h bits, walked
// until the image is below n. f(R, round): its round function, before the mask to h bits.
__device__ __forceinline__ int shuffle_bits(uint32_t n) {
    int h = 1;
    while (((uint64_t)1 << (2 * h)) < (uint64_t)n) ++h;
    return h;
}
template <typename F>
__device__ __forceinline__ uint32_t feistel(uint32_t x, int h, F &&f) {
    const uint32_t mask = (1u << h) - 1u;
    uint32_t L = x >> h, R = x & mask;
    for (uint32_t round = 0; round < 4; ++round) {
        const uint32_t t = R;
        R = L ^ (f(R, round) & mask);
        L = t;
    }
    return (L << h) | R;
}

// u = floor(w0 W / 2^32) of the pointers floor((u + k W) / n).
__device__ __forceinline__ uint64_t sus_offset(const InstDesc &d, uint32_t gen, uint64_t W) {
    const uint32_t w0 = draw(0u, 0xFFFFFFFFu, gen, kTagSus, d.inst_id, d.seed).x;
    return __umul64hi((uint64_t)w0 << 32, W);
}
// The parents, two per child, where the rank kernel lists them: in the prefix's place (2 (P - E) words of 2 P).
__device__ __forceinline__ int32_t *sus_parents(const InstDesc &d) { return (int32_t *)d.sus_cum; }

__device__ __forceinline__ uint64_t isqrt_u48(uint64_t x) {
    uint64_t y = (uint64_t)sqrt((double)x);                 // within one of the exact root
    while (y * y > x) --y;
    while ((y + 1) * (y + 1) <= x) ++y;
    return y;
}

__global__ __launch_bounds__(1024) void k_sus_prefix(Tables t) {
    __shared__ uint64_t wsum[16];
    __shared__ uint64_t carry_s;
    const InstDesc &d = const_at(t.desc, blockIdx.x);
    if (d.P == 0 || d.selection != PGA_SELECT_SUS || inst_stopped(d)) return;
    const int P = d.P;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int pass = 0; pass < 2; ++pass) {                   // pass 1 only if every weight was 0
        uint64_t carry = 0;
        for (int base = 0; base < P; base += 1024) {
            const int p = base + threadIdx.x;
            uint64_t w = 0;
            if (p < P) {
                if (pass == 1) w = 1;
                else if (isfinite(gld(d.fitness + p)))
                    w = isqrt_u48(((uint64_t)1 << 48) / (uint64_t)gld(d.sus_rank + p));
            }
            uint64_t x = w;                                  // inclusive scan over the wave
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint64_t y = __shfl_up(x, o, 64);
                if (lane >= o) x += y;
            }
            if (lane == 63) wsum[wave] = x;
            __syncthreads();
            uint64_t before = carry;
            for (int v = 0; v < wave; ++v) before += wsum[v];
            if (p < P) gst(d.sus_cum + p, before + x);
            if (threadIdx.x == 1023) carry_s = before + x;
            __syncthreads();
            carry = carry_s;
            __syncthreads();
        }
        if (carry != 0) break;
    }
}

// ---- ranking and SUS of one instance by one workgroup -------------------------------------------
// A fitness as a key that sorts ascending where ranks_before sorts (higher fitness first, +0 and -0 equal).
__device__ __forceinline__ uint64_t rank_key(double f) {
    const uint64_t b = __builtin_bit_cast(uint64_t, f + 0.0);
    return ~(b >> 63 ? ~b : b ^ (uint64_t)1 << 63);
}
__device__ __forceinline__ bool key_finite(uint64_t key) {
    const uint64_t u = ~key;
    return isfinite(__builtin_bit_cast(double, u >> 63 ? u ^ (uint64_t)1 << 63 : ~u));
}
// isqrt_u48(2^48 / r): the FP64 quotient's floor is exact (2^48 / r is a whole number, or at least 1 / r
// below the next one, and half a unit in its last place is at most 2^-5 / r).
__device__ __forceinline__ uint64_t sus_weight(int r) { return isqrt_u48((uint64_t)(0x1p48 / (double)r)); }

// Rank kernel of the launches that select by SUS with P <= 1024 V: what k_rank, k_sus_rank and
// k_sus_prefix do together, and the pointers' individuals with it. A bitonic sort of (key, index)
// by 1024 threads, V elements each (element e in register e % V of thread e / V): partners up to 32
// lanes away come by DPP and lane swaps, farther ones through LDS (10 of 55 steps at P = 1024).
// Then, by sorted position, the elites and the weights (into LDS by individual); the inclusive prefix
// cum of the weights in index order; for each individual p the number of pointers before the end of its
// segment, ks(p): pointer k lies at floor((u + k W) / n), and cum(p) > floor(x) for a whole cum(p) is
// cum(p) > x, so ks(p) = ceil((n cum(p) - u) / W) (n cum < 2^13 2^36); and each child's parents, the first
// individuals p with ks(p) > k by a search in LDS, k the shuffled pointer. The shuffle's round function has 4 2^h
// values (h <= 7): one draw per thread here, against 8 draws and more per parent in the breed kernel. The
// statistics are those of RankBlock: 256 threads, the same order of additions.
// 128 instances of P = 1000: three launches of 45 us (29 of them to count all pairs) and 36 us of breeding,
// which drew the shuffle and searched the prefix in memory, against one of 20 us and 19 us (with 512
// or 256 threads of 2 or 4 elements the whole run took 1.03 or 1.13 times as long). By phase, in cycles of 43 000: the sort 16 400, the
// parents 8 400, the shuffle 5 400, loads and weights 5 000.
constexpr int kSusHalfBits = 7;                              // of the pairing's halves, n <= 2 kSusSortMax
static_assert((1 << 2 * kSusHalfBits) >= 2 * kSusSortMax && kSusHalfBits <= 8, "a byte per value");

struct SusElem {
    uint64_t key;
    uint32_t idx;
};

// Lanes where (a.key, a.idx) < (b.key, b.idx): the borrow of their difference. (Written as compares it is
// five, and four scalar instructions.)
__device__ __forceinline__ uint64_t sus_less(const SusElem &a, const SusElem &b) {
    uint64_t m;
    uint32_t t;
    asm("v_sub_co_u32_e32 %[t], vcc, %[ai], %[bi]\n\t"
        "v_subb_co_u32_e32 %[t], vcc, %[al], %[bl], vcc\n\t"
        "v_subb_co_u32_e32 %[t], vcc, %[ah], %[bh], vcc\n\t"
        "s_mov_b64 %[m], vcc"
        : [m] "=s"(m), [t] "=&v"(t)
        : [ai] "v"(a.idx), [bi] "v"(b.idx), [al] "v"((uint32_t)a.key), [bl] "v"((uint32_t)b.key),
          [ah] "v"((uint32_t)(a.key >> 32)), [bh] "v"((uint32_t)(b.key >> 32))
        : "vcc");
    return m;
}
__device__ __forceinline__ SusElem sus_select(uint64_t lanes, const SusElem &a, const SusElem &b) {   // a on `lanes`
    const bool s = __builtin_amdgcn_inverse_ballot_w64(lanes);
    return SusElem{s ? a.key : b.key, s ? a.idx : b.idx};
}
template <typename F>
__device__ __forceinline__ SusElem sus_each(const SusElem &x, F &&f) {
    return SusElem{(uint64_t)f((uint32_t)(x.key >> 32)) << 32 | f((uint32_t)x.key), f(x.idx)};
}

// One step with lane l ^ J; up: lanes whose run ascends.
template <int J, int V>
__device__ __forceinline__ void sus_step(SusElem (&x)[V], uint64_t up) {
    constexpr uint64_t kUpper = J == 1    ? 0xAAAAAAAAAAAAAAAA
                                : J == 2  ? 0xCCCCCCCCCCCCCCCC
                                : J == 4  ? 0xF0F0F0F0F0F0F0F0
                                : J == 8  ? 0xFF00FF00FF00FF00
                                : J == 16 ? 0xFFFF0000FFFF0000
                                          : 0xFFFFFFFF00000000;      // the upper lane of each pair
#pragma unroll
    for (int v = 0; v < V; ++v) {
        if constexpr (J >= 16) {
            // a swap of x with itself: the lower lane's element and the upper lane's, in both
            uint32_t lo[3], hi[3];
            const uint32_t w[3] = {(uint32_t)x[v].key, (uint32_t)(x[v].key >> 32), x[v].idx};
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const auto r = J == 16 ? __builtin_amdgcn_permlane16_swap(w[q], w[q], false, false)
                                       : __builtin_amdgcn_permlane32_swap(w[q], w[q], false, false);
                lo[q] = r[0];
                hi[q] = r[1];
            }
            const SusElem L{(uint64_t)lo[1] << 32 | lo[0], lo[2]}, U{(uint64_t)hi[1] << 32 | hi[0], hi[2]};
            x[v] = sus_select(~(sus_less(U, L) ^ up) ^ kUpper, U, L);
        } else {
            const SusElem y = sus_each(x[v], [](uint32_t z) {
                auto mov = [](uint32_t q, auto ctrl) {
                    return (uint32_t)__builtin_amdgcn_mov_dpp((int)q, decltype(ctrl)::value, 0xF, 0xF, true);
                };
                if constexpr (J == 1) return mov(z, std::integral_constant<int, kQuad1>{});
                else if constexpr (J == 2) return mov(z, std::integral_constant<int, kQuad2>{});
                else if constexpr (J == 4)                   // half mirror: l ^ 7, quads reversed: l ^ 3
                    return mov(mov(z, std::integral_constant<int, 0x141>{}), std::integral_constant<int, 0x1B>{});
                else return mov(z, std::integral_constant<int, kRor8>{});
            });
            x[v] = sus_select(~(sus_less(y, x[v]) ^ up ^ kUpper), y, x[v]);
        }
    }
}

template <int T, int V>
__global__ __launch_bounds__(T) void k_rank_sus(Tables t, int gen_off) {
    __shared__ uint64_t key_s[T * V];                        // sort; then the weights by individual; then the shuffle
    __shared__ uint32_t idx_s[T * V];                        // sort; then ks by individual
    __shared__ uint64_t wsum[T / 64];
    __shared__ double wf[kRankWaves];
    __shared__ int wi[kRankWaves];
    __shared__ uint8_t round_s[4 << kSusHalfBits];           // the pairing's round function: [round][right half]
    __shared__ int first;
    const InstDesc &d = const_at(t.desc, blockIdx.x);
    if (d.P == 0) return;                                    // a padding slot of a capacity-sized launch
    const int P = d.P, E = d.E, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const double *__restrict__ f = d.fitness;
    SusElem x[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int p = V * tid + v;
        x[v] = SusElem{p < P ? rank_key(gld(f + p)) : ~(uint64_t)0, (uint32_t)p};
    }
    const bool sus = d.selection == PGA_SELECT_SUS;
    const uint32_t n = 2u * (uint32_t)(P - E), gen = d.gen0 + (uint32_t)gen_off;
    const int h = shuffle_bits(n);
    if (sus)
        for (int e = tid; e < 4 << h; e += T)
            round_s[e] = (uint8_t)draw((uint32_t)e & ((1u << h) - 1u), (uint32_t)e >> h, gen, kTagShuf, d.inst_id, d.seed).x;
    pga_term_state st{};
    if (d.term) {
        const bool stopped = inst_stopped(d);
        if (tid == 0) st = *d.term;
        __syncthreads();                                     // every thread has read the flag
        if (gen_off == 0 && tid == 0) {
            gst(&d.term->call_gens, 0);
            st.call_gens = 0;
        }
        if (stopped) return;
    }
    if (d.stats && tid < kRankThreads) {                     // whole waves
        double sum = 0.0, ninv = 0.0;
        for (int p = tid; p < P; p += kRankThreads) {
            const double fp = gld(f + p);
            if (isfinite(fp)) sum += fp;
            else ninv += 1.0;
        }
        sum = group_sum<64>(sum);
        ninv = group_sum<64>(ninv);
        if (lane == 0) {
            wf[wave] = sum;
            wi[wave] = (int)ninv;
        }
    }

    int n2 = 64 * V;
    while (n2 < P) n2 *= 2;
    const bool busy = (tid & ~63) * V < n2;                  // per wave
    for (int k = 2; k <= n2; k *= 2) {
        const uint64_t up = __builtin_amdgcn_ballot_w64(((V * tid) & k) == 0);   // (k < V: by register, below)
        for (int j = k / 2; j >= 64 * V; j /= 2) {           // uniform over the workgroup
#pragma unroll
            for (int v = 0; v < V; ++v) {
                key_s[v * T + tid] = x[v].key;
                idx_s[v * T + tid] = x[v].idx;
            }
            __syncthreads();
            const int q = tid ^ (j / V);
            const uint64_t upper = tid & (j / V) ? ~(uint64_t)0 : 0;      // per wave
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const SusElem y{key_s[v * T + q], idx_s[v * T + q]};
                x[v] = sus_select(~(sus_less(y, x[v]) ^ up ^ upper), y, x[v]);
            }
            __syncthreads();
        }
        if (!busy) continue;
        if (k > 32 * V) sus_step<32>(x, up);
        if (k > 16 * V) sus_step<16>(x, up);
        if (k > 8 * V) sus_step<8>(x, up);
        if (k > 4 * V) sus_step<4>(x, up);
        if (k > 2 * V) sus_step<2>(x, up);
        if (k > V) sus_step<1>(x, up);
#pragma unroll
        for (int j = V / 2; j > 0; j /= 2) {
            if (k <= j) continue;
#pragma unroll
            for (int v = 0; v < V; ++v) {
                if (v & j) continue;
                const uint64_t up_v = k < V ? (v & k) == 0 ? ~(uint64_t)0 : 0 : up;
                const SusElem a = x[v], b = x[v ^ j];
                const uint64_t swap = ~(sus_less(b, a) ^ up_v);
                x[v] = sus_select(swap, b, a);
                x[v ^ j] = sus_select(swap, a, b);
            }
        }
    }
    __syncthreads();                                         // (n2 <= 64 V: no barrier above)
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int r = V * tid + v;                           // its rank - 1
        const int i = (int)x[v].idx;
        if (r >= P) continue;
        if (r < E) gst(d.elite + r, i);
        if (r == 0) first = i;
        if (sus) key_s[i] = key_finite(x[v].key) ? sus_weight(r + 1) : 0;
    }
    __syncthreads();
    if (tid == 0) {
        const double best = gld(f + first);
        if (d.stats) {
            double total = 0.0, inv = 0.0;
            for (int w = 0; w < kRankWaves; ++w) {
                total += wf[w];
                inv += (double)wi[w];
            }
            stats_row(d, gen_off, Cand{best, first}, P, total, inv);
        }
        if (d.term) term_update(d, st, best, 0, gen_off == 0);
    }
    if (!sus) return;

    uint64_t cum[V];
    uint64_t w = 0;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int p = V * tid + v;
        if (p < P) w += key_s[p];
        cum[v] = w;
    }
    uint64_t inc = w;                                        // inclusive scan over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint64_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint64_t before = inc - w, W = 0;
#pragma unroll
    for (int v = 0; v < T / 64; ++v) {
        if (v < wave) before += wsum[v];
        W += wsum[v];
    }
    const bool uniform = W == 0;                             // every fitness is -inf: every weight 1
    if (uniform) W = (uint64_t)P;
    const uint64_t u = sus_offset(d, gen, W);
    const double per = 1.0 / (double)W;
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int p = V * tid + v;
        if (p >= P) continue;
        const uint64_t a = (uint64_t)n * (uniform ? (uint64_t)p + 1 : before + cum[v]);
        // floor((a - u) / W) by FP64 within one, then exactly; then the ceiling
        const uint64_t num = a <= u ? 0 : a - u;
        uint32_t q = (uint32_t)((double)num * per);
        int64_t r = (int64_t)(num - q * W);
        if (r < 0) {
            --q;
            r += (int64_t)W;
        } else if (r >= (int64_t)W) {
            ++q;
            r -= (int64_t)W;
        }
        idx_s[p] = q + (r > 0 ? 1u : 0u);
    }
    // The Feistel network's image of every number of 2h bits (the weights have been read): 4 rounds here,
    // one read per turn of the cycle walk.
    uint16_t *const shuffle_s = (uint16_t *)key_s;
    static_assert(sizeof(key_s) >= sizeof(uint16_t) << (V * T > 2048 ? 14 : 12), "2h = 12 bits up to n = 4096");
#pragma unroll 4
    for (int e = tid; e < 1 << 2 * h; e += T)
        shuffle_s[e] = (uint16_t)feistel((uint32_t)e, h, [&](uint32_t R, uint32_t round) { return (uint32_t)round_s[round << h | R]; });
    __syncthreads();
    int32_t *__restrict__ parents = sus_parents(d);
    for (uint32_t i0 = tid; i0 < n; i0 += 2 * T) {           // two at a time: chains of LDS reads
        uint32_t x[2] = {i0, i0 + T < n ? i0 + T : i0};
        x[0] = shuffle_s[x[0]];
        x[1] = shuffle_s[x[1]];
        while (x[0] >= n || x[1] >= n) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (x[q] >= n) x[q] = shuffle_s[x[q]];
        }
        int at[2] = {0, 0};
        for (int s = n2 / 2; s > 0; s /= 2) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (at[q] + s <= P && idx_s[at[q] + s - 1] <= x[q]) at[q] += s;
        }
        gst(parents + i0, at[0]);
        if (i0 + T < n) gst(parents + i0 + T, at[1]);
    }
}

hipError_t launch_rank_sus(Tables t, int max_p, int gen_off, hipStream_t s) {
    if (max_p <= 1024)
        hipLaunchKernelGGL((k_rank_sus<1024, 1>), dim3(t.n_inst), dim3(1024), 0, s, t, gen_off);
    else if (max_p <= 2048)
        hipLaunchKernelGGL((k_rank_sus<1024, 2>), dim3(t.n_inst), dim3(1024), 0, s, t, gen_off);
    else if (max_p <= kSusSortMax)
        hipLaunchKernelGGL((k_rank_sus<1024, 4>), dim3(t.n_inst), dim3(1024), 0, s, t, gen_off);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_sus(Tables t, int max_p, hipStream_t s) {
    if (t.n_inst <= 0 || max_p <= 0) return hipSuccess;
    const int nb = (max_p + 255) / 256;
    hipLaunchKernelGGL(k_sus_rank, dim3(nb, nb, t.n_inst), dim3(256), 0, s, t);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sus_prefix, dim3(t.n_inst), dim3(1024), 0, s, t);
    return hipGetLastError();
}

// Individual whose SUS segment holds pointer k (smallest p with cum[p] > pos).
__device__ int sus_pick(const InstDesc &d, uint32_t k, uint32_t n, uint64_t u, uint64_t W) {
    const uint64_t pos = (u + (uint64_t)k * W) / (uint64_t)n;
    int lo = 0, hi = d.P - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (gld(d.sus_cum + mid) > pos) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// Parent pair of child c (c >= E): two tournaments of two on draw (0, c, g,
// SELECT), or, with SUS, the individuals under shuffled pointers 2(c - E) and
// 2(c - E) + 1 (which = 0, 1).
__device__ int sus_parent(const InstDesc &d, int c, uint32_t gen, int which, int listed) {
    const int P = d.P, E = d.E;
    const uint32_t n = 2u * (uint32_t)(P - E);
    const uint32_t x = 2u * (uint32_t)(c - E) + (uint32_t)which;
    if (listed) return gld(sus_parents(d) + x);
    const int h = shuffle_bits(n);
    uint32_t k = x;
    do {                                                     // until the image is one of [0, n)
        k = feistel(k, h, [&](uint32_t R, uint32_t round) { return draw(R, round, gen, kTagShuf, d.inst_id, d.seed).x; });
    } while (k >= n);
    const uint64_t W = gld(d.sus_cum + (P - 1));
    return sus_pick(d, k, n, sus_offset(d, gen, W), W);
}

// Ranking by the breed launch ("fold": no instance selects by SUS or can stop
// early): workgroup k < n_inst ranks instance k (the RankBlock code and thread
// count of the rank kernel, so the statistics are the same bits), copies its
// elites and keeps its termination state and statistics row, beside the
// workgroups that make the children, which need only the fitness values
// (tournaments): no rank launch between fitness and breeding.
__device__ __forceinline__ void fold_rank(const Tables &t, int k, int parity, int gen_off) {
    __shared__ RankLds sh;
    const InstDesc &d = const_at(t.desc, k);
    const int P = d.P, E = d.E, N = d.N;
    if (P == 0 || (E == 0 && !d.term && !d.stats)) return;   // a padding slot, or nothing to rank
    if (inst_stopped(d)) {                                 // by an earlier call: it stays as it is
        if (gen_off == 0 && threadIdx.x == 0) gst(&d.term->call_gens, 0);
        return;
    }
    // This workgroup's chain of reductions is the longest path of the launch:
    // its waves issue ahead of the slot waves that share their SIMDs.
    __builtin_amdgcn_s_setprio(3);
    RankBlock<4> rb{d.fitness, P, sh};                     // the slot waves share the register budget
    rb.load();
    pga_term_state st{};
    if (d.term && threadIdx.x == 0) st = *d.term;
    const int32_t *__restrict__ src = d.pop[parity];
    int32_t *__restrict__ dst = d.pop[parity ^ 1];
    const Cand best = rb.rank_and_stats(d, E > 1 ? E : 1, gen_off, d.stats != nullptr, [&] {
        // Wave w copies the elites w, w + 4, ..: four genes a lane, the loads of a whole row (N <=
        // 1024) in flight together. (One gene a thread and four rows at a time: ten rows of 768
        // genes were nine memory latencies, 9 us.)
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        constexpr int kV = 4;
        for (int r = wave; r < E; r += kRankWaves) {
            const int32_t *__restrict__ e = src + (size_t)sh.ord[r] * N;
            int32_t *__restrict__ o = dst + (size_t)r * N;
            for (int j0 = 4 * lane; j0 < N; j0 += 4 * 64 * kV) {
                gene4 v[kV];
#pragma unroll
                for (int q = 0; q < kV; ++q) {
                    const int j = j0 + 256 * q;
                    if (j + 4 <= N) v[q] = *(const PGA_GLOBAL gene4 *)(e + j);
                    else if (j < N) v[q] = gene4{gld(e + j), gld(e + min(j + 1, N - 1)), gld(e + min(j + 2, N - 1)), 0};
                }
#pragma unroll
                for (int q = 0; q < kV; ++q) {
                    const int j = j0 + 256 * q;
                    if (j + 4 <= N) *(PGA_GLOBAL gene4 *)(o + j) = v[q];
                    else {
                        if (j < N) gst(o + j, v[q].x);
                        if (j + 1 < N) gst(o + j + 1, v[q].y);
                        if (j + 2 < N) gst(o + j + 2, v[q].z);
                    }
                }
            }
        }
    });
    if (d.term && threadIdx.x == 0) {
        if (gen_off == 0) st.call_gens = 0;
        term_update(d, st, best.f, 0, gen_off == 0);
    }
}

// A workgroup makes the slots [c0, c0 + chr) of one instance (chr a power of
// two), gl lanes per slot and 256 / gl slots at a time (breed_split). No draw is
// made twice:
//   1. the draws that all genes of a child share (its parents, whether it
//      crosses, a 128-bit crossover word per 128 genes), one per thread over the
//      children of the workgroup, into LDS (made by every lane of a child's
//      wave they were five of its eight draws at N = 272);
//   2. per gene pair the mutation draw and the two parents' genes; with 16
//      lanes per slot a pass of a wave serves four slots, and the last pass of a
//      slot leaves few lanes idle (136 pairs: 9 passes of 16, against 3 of 64).
// Every draw is keyed by child and gene pair, so a child is the same bits
// whatever gl and chr are. Large launches are near the memory: 256 instances of
// N ~ U{32..512} read two parents per child and write it, 430 MB in 95 us (4.5
// TB/s; 133 us with 64 slots a workgroup, 198 with a wave per slot and all draws in it). (Loading the next
// pass's genes before the draw: 139 us, and no gain in small launches.)
__global__ __launch_bounds__(256) void k_breed(Tables t, int parity, int gen_off, int fold, int sus_listed, BreedShape shape) {
    extern __shared__ __align__(16) uint32_t blds[];       // [parent A, B | crosses][chr], words [4 nq][chr]
    int wg = blockIdx.x;
    if (fold) {
        if (wg < t.n_inst) {
            fold_rank(t, wg, parity, gen_off);
            return;
        }
        wg -= t.n_inst;
    }
    const int total = const_at(t.breeds, t.n_inst);
    if (wg >= total) return;                               // the grid may exceed the total (capacity-sized graph)
    // runs of workgroups on one XCD: its L2 holds their instance's parents
    const int run = kBreedRun, run8 = wg / (kXcds * run), in8 = wg % (kXcds * run);
    if ((run8 + 1) * kXcds * run <= total) wg = run8 * kXcds * run + in8 % kXcds * run + in8 / kXcds;
    const int k = find_inst(t.breeds, t.n_inst, wg);
    const InstDesc &d = const_at(t.desc, k);
    const int32_t stopped = stop_flag(d, t);               // set by this generation's rank; tested before the genes
    const int N = d.N, P = d.P, E = d.E, tid = threadIdx.x;
    const BreedSplit split = breed_split(N, shape);
    const int chr = split.chr, gl_n = split.gl, c0 = (wg - const_at(t.breeds, k)) * chr;
    const int32_t *__restrict__ src = d.pop[parity];
    const uint32_t gen = d.gen0 + (uint32_t)gen_off;
    const bool sus = d.selection == PGA_SELECT_SUS;
    const int nq = (N + 127) >> 7;
    int32_t *par = (int32_t *)blds;
    uint32_t *crosses = blds + 2 * chr, *words = blds + 3 * chr;

    {
        const int ci = tid & (chr - 1), c = c0 + ci;
        const int kinds = (sus ? 3 : 2) + nq;              // parents (one thread, or one each with SUS), cross, words
        for (int x = tid / chr; x < kinds; x += 256 / chr) {
            if (c >= P || c < E) continue;
            if (sus && x < 2) {
                par[x * chr + ci] = sus_parent(d, c, gen, x, sus_listed);
                continue;
            }
            const int y = sus ? x - 1 : x;                 // 0 parents, 1 cross, 2 + q: word q
            const U4 w = draw(y < 2 ? 0u : (uint32_t)(y - 1), (uint32_t)c, gen, y == 0 ? kTagSel : kTagXov, d.inst_id,
                              d.seed);
            if (y == 0) {
                const double *__restrict__ f = d.fitness;
                par[ci] = tournament2(f, (int)scale_u32(w.x, (uint32_t)P), (int)scale_u32(w.y, (uint32_t)P));
                par[chr + ci] = tournament2(f, (int)scale_u32(w.z, (uint32_t)P), (int)scale_u32(w.w, (uint32_t)P));
            } else if (y == 1) {
                crosses[ci] = w.x < d.p_cross ? 1u : 0u;
            } else {
                uint32_t *o = words + (size_t)(4 * (y - 2)) * chr + ci;
                o[0] = w.x;
                o[chr] = w.y;
                o[2 * chr] = w.z;
                o[3 * chr] = w.w;
            }
        }
    }
    if (flag_stops(d, stopped)) return;                    // uniform over the workgroup
    __syncthreads();

    const int gl = tid & (gl_n - 1), npair = (N + 1) >> 1;
    const uint32_t pm = d.p_mut;
    for (int ci = tid / gl_n; ci < chr; ci += 256 / gl_n) {
        const int c = c0 + ci;
        if (c >= P) break;
        int32_t *__restrict__ out = d.pop[parity ^ 1] + (size_t)c * N;
        if (c < E) {
            if (fold) continue;                            // copied by the instance's ranking workgroup
            const int32_t *__restrict__ e = src + (size_t)d.elite[c] * N;
            for (int j = gl; j < N; j += gl_n) out[j] = e[j];
            continue;
        }
        const int32_t *__restrict__ ra = src + (size_t)par[ci] * N;
        const int32_t *__restrict__ rb = src + (size_t)par[chr + ci] * N;
        const bool cross = crosses[ci] != 0;
        for (int jp = gl; jp < npair; jp += gl_n) {
            const int j = 2 * jp;
            const bool has1 = j + 1 < N;
            // genes j, j + 1 (the last pair of an odd N: gene j twice)
            auto pair = [&](const int32_t *r) -> gene2 {
                if (has1) return *(const PGA_GLOBAL gene2 *)(r + j);
                const int32_t g = gld(r + j);
                return gene2{g, g};
            };
            gene2 g = pair(ra);
            if (cross) {
                const gene2 h = pair(rb);
                const uint32_t w = words[(size_t)(j >> 5) * chr + ci] >> (j & 31);
                if (w & 1u) g.x = h.x;
                if (w & 2u) g.y = h.y;
            }
            const U4 m = draw((uint32_t)jp, (uint32_t)c, gen, kTagMut, d.inst_id, d.seed);
            if (m.x < pm) g.x = (int32_t)scale_u32(m.y, (uint32_t)N);
            if (m.z < pm) g.y = (int32_t)scale_u32(m.w, (uint32_t)N);
            if (has1) *(PGA_GLOBAL gene2 *)(out + j) = g;
            else gst(out + j, g.x);
        }
    }
}

// The draws of every launch size, beside the ranking's, fit in LDS for every N the library takes.
constexpr bool breed_layout_ok() {
    for (int inds : {1, 4096, 65536})
        if (breed_lds_bytes(PGA_N_MAX, breed_shape(inds)) + sizeof(RankLds) + 16 > (size_t)kMaxLdsBytes) return false;
    return true;
}
static_assert(breed_layout_ok(), "breed LDS within the LDS limit");

hipError_t launch_breed(Tables t, int blocks, const BreedShape &b, int parity, int gen_off, int fold, int sus_listed, int max_n,
                        hipStream_t s) {
    const int grid = (fold ? t.n_inst : 0) + blocks;
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_breed, dim3(grid), dim3(256), breed_lds_bytes(max_n, b), s, t, parity, gen_off, fold, sus_listed, b);
    return hipGetLastError();
}

// After an odd number of bred generations the population sits in pop[1]; copy
// it back so the caller always finds the result in the buffer it passed as
// pop. Without a termination test every call breeds G generations.
// A workgroup copies the rows of the slots that it would breed: one run of memory (a workgroup per row: 90 us
// for 128 000 of N = 18 without a row to copy; 3.9 us).
__global__ __launch_bounds__(256) void k_copy_back(Tables t, int G, BreedShape shape) {
    const int wg = blockIdx.x;
    if (wg >= const_at(t.breeds, t.n_inst)) return;                  // the grid may exceed the total (capacity-sized graph)
    const int k = find_inst(t.breeds, t.n_inst, wg);
    const InstDesc &d = const_at(t.desc, k);
    const int bred = d.term ? gld(&d.term->call_gens) : G;
    if ((bred & 1) == 0) return;
    const int N = d.N, chr = breed_split(N, shape).chr, c0 = (wg - const_at(t.breeds, k)) * chr;
    const int len = min(chr, d.P - c0) * N;
    const int32_t *__restrict__ a = d.pop[1] + (size_t)c0 * N;
    int32_t *__restrict__ b = d.pop[0] + (size_t)c0 * N;
    for (int j = 4 * threadIdx.x; j < len; j += 4 * 256) {
        if (j + 4 <= len) {
            *(PGA_GLOBAL gene4 *)(b + j) = *(const PGA_GLOBAL gene4 *)(a + j);
        } else {
            gst(b + j, gld(a + j));
            if (j + 1 < len) gst(b + j + 1, gld(a + j + 1));
            if (j + 2 < len) gst(b + j + 2, gld(a + j + 2));
        }
    }
}

hipError_t launch_copy_back(Tables t, int blocks, const BreedShape &b, int G, hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy_back, dim3(blocks), dim3(256), 0, s, t, G, b);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Best: arg-best over P (lowest index among ties), then relabel that row in
// first-occurrence order. first[s] = smallest stock index carrying label s
// (integer atomicMin, order-free); stock i opens a new cluster iff
// first[s_i] == i; the new label of s is the number of clusters opened
// before first[s] (exclusive scan). Out-of-range labels are copied through.
// out[0..N) = labels, out[N] = index; out_f = fitness.
__global__ __launch_bounds__(256) void k_best(const double *f, const int32_t *labels, int P, int N,
                                               int32_t *out, double *out_f) {
    __shared__ double rf[256];
    __shared__ int ri[256];
    __shared__ int first[PGA_N_MAX];
    __shared__ int open[PGA_N_MAX];
    __shared__ int part[256];

    Cand c{0.0, -1};
    for (int p = threadIdx.x; p < P; p += 256)
        if (c.i < 0 || ranks_before(f[p], p, c.f, c.i)) c = Cand{f[p], p};
    const Cand b = block_best(c, rf, ri);
    const int32_t *__restrict__ row = labels + (size_t)b.i * N;

    for (int s = threadIdx.x; s < N; s += 256) first[s] = 0x7fffffff;
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += 256) {
        const int l = row[i];
        if (l >= 0 && l < N) atomicMin(&first[l], i);
    }
    __syncthreads();
    // contiguous chunk per thread, then an exclusive scan of chunk totals
    const int chunk = (N + 255) / 256;
    const int i0 = threadIdx.x * chunk, i1 = min(N, i0 + chunk);
    int local = 0;
    for (int i = i0; i < i1; ++i) {
        const int l = row[i];
        const int o = (l >= 0 && l < N && first[l] == i) ? 1 : 0;
        open[i] = local;
        local += o;
    }
    part[threadIdx.x] = local;
    __syncthreads();
    if (threadIdx.x == 0) {
        int run = 0;
        for (int q = 0; q < 256; ++q) {
            const int v = part[q];
            part[q] = run;
            run += v;
        }
    }
    __syncthreads();
    for (int i = i0; i < i1; ++i) open[i] += part[threadIdx.x];
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += 256) {
        const int l = row[i];
        out[i] = (l >= 0 && l < N) ? open[first[l]] : l;
    }
    if (threadIdx.x == 0) {
        out[N] = b.i;
        *out_f = b.f;
    }
}

hipError_t launch_best(const double *fitness, const int32_t *labels, int P, int N, int32_t *out,
                       double *out_f, hipStream_t s) {
    hipLaunchKernelGGL(k_best, dim3(1), dim3(256), 0, s, fitness, labels, P, N, out, out_f);
    return hipGetLastError();
}

}  // namespace pga
