// Ranking of the blocks of a layer by a per-block score and the split into pools (step 2 of the
// per-layer pair search): the score tau of the block of rank n_top (ranks count from the best score)
// is found exactly, every block at least as good as tau stays in the first pool, the others form the
// fitting pool of the second codebook.  Several thresholds at once (the sweep over the partition parameter) give
// nested pools: a level per block, the number of thresholds that it ranks strictly worse than; several score planes go through
// the same launches (blockIdx.y).
//
// The score is mapped to a 32-bit key whose unsigned order is the ranking order (+0 and -0 share a
// key; for "lower is better" the key is complemented, so the best score always has the largest key).
// Counting passes over the keys fix the thresholds' keys from the top.
//   One threshold of one plane (up to SOP_K_SEL_ONE_MAX scores): three passes, of 11, 11 and 10 bits.  A pass counts, in a 2048-bin histogram, the digit of every key that
//   agrees with the digits fixed so far; the next kernel finds, from that histogram, the digit in which the wanted rank falls.  A last kernel writes the
//   pool mask, tau and the size of the first pool.
//   Several: cosines and their squares crowd below 1, so the first pass counts the keys of [7/8, 1) 256 to a bin and all others 2^21 to a
//   bin; a threshold in there is known after a second pass over the eight bits left, any other after two (11 and 10 bits).  The third pass is launched with the
//   others, and its workgroups leave at once where no threshold needs it.  The workgroup that finishes a pass last finds the digits and hands them on.  What bounds
//   a pass is the read of the scores and, for few of them, five round trips to memory one after the other (state, scores, sums, ticket, totals).  Three passes of 11, 11 and
//   10 bits whatever the scores, with a kernel after each that found the digits, against these, 2.8 M scores, four thresholds: six planes 109 us -> 66, one plane 51 -> 31 (scores spread
//   over many binades, where the third pass counts: 56.6 -> 47.6); 98 304 scores 31.8 -> 20.9; 14.7 M 134 -> 69.
// Counts are integers added with atomics, so every result is exact and reproducible.  Every call leaves the counts that the next one adds to at zero itself, so a captured call can
// be replayed: each is cleared by a kernel of the call in which no workgroup reads it any more, or none yet.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sop_kparams.h"

namespace sopk {

__device__ __forceinline__ uint32_t rank_key(float v, bool higher)
{
    uint32_t u = __float_as_uint(v);
    if (u == 0x80000000u) u = 0u;                                  // -0 ranks with +0
    const uint32_t k = (u & 0x80000000u) ? ~u : (u | 0x80000000u); // ascending with the value
    return higher ? k : ~k;
}
__device__ __forceinline__ float key_score(uint32_t k, bool higher)
{
    if (!higher) k = ~k;
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return __uint_as_float(u);
}

// ---- one threshold, one plane ----
struct Digit { int digit; unsigned int rank_in, above; };

// The workgroup (at least 256 threads) walks a 2048-bin histogram from its top bin down and finds the bin in
// which the key of rank `rank` (1-based from the top) falls: `above` keys lie in higher bins and the
// wanted key has rank `rank_in` inside the bin.  Thread t holds the eight bins 2047-8t .. 2040-8t in
// registers; a scan over the threads' sums names the one thread whose bins contain the rank.
__device__ Digit find_digit(const unsigned int* hist, unsigned int rank, Digit* s_found, unsigned int* s_wave)
{
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const bool on = t < SOP_K_SEL_BINS / 8;                         // the first 256 threads hold the bins
    const int base = on ? SOP_K_SEL_BINS - 8 * (t + 1) : 0;
    uint4 lo = make_uint4(0, 0, 0, 0), hi = lo;
    if (on) { lo = *reinterpret_cast<const uint4*>(hist + base); hi = *reinterpret_cast<const uint4*>(hist + base + 4); }
    const unsigned int h[8] = {hi.w, hi.z, hi.y, hi.x, lo.w, lo.z, lo.y, lo.x};     // from the top bin down
    const unsigned int sum = ((h[0] + h[1]) + (h[2] + h[3])) + ((h[4] + h[5]) + (h[6] + h[7]));
    unsigned int inc = sum;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
        const unsigned int v = __shfl_up(inc, st, 64);
        if (lane >= st) inc += v;
    }
    if (t == 0) { s_found->digit = 0; s_found->rank_in = 1; s_found->above = 0; }   // histogram shorter than rank: stay in bounds
    if (on && lane == 63) s_wave[wv] = inc;
    __syncthreads();
    if (on) {
        for (int i = 0; i < wv; ++i) inc += s_wave[i];
        const unsigned int exc = inc - sum;
        if (exc < rank && rank <= inc) {                            // exactly one thread
            unsigned int c = exc;
            int d = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {                           // ci: keys above bin i of this thread
                const unsigned int ci = exc + (i > 0 ? h[0] : 0u) + (i > 1 ? h[1] : 0u) + (i > 2 ? h[2] : 0u) + (i > 3 ? h[3] : 0u)
                                      + (i > 4 ? h[4] : 0u) + (i > 5 ? h[5] : 0u) + (i > 6 ? h[6] : 0u);
                if (ci < rank && rank <= ci + h[i]) { d = i; c = ci; }
            }
            s_found->digit = base + 7 - d; s_found->rank_in = rank - c; s_found->above = c;
        }
    }
    __syncthreads();
    const Digit f = *s_found;
    __syncthreads();
    return f;
}

// one count into an LDS histogram for every active lane; lanes that share the first active lane's
// digit are counted with one atomic (block cosines crowd into very few digits in the first pass)
__device__ __forceinline__ void count_digit(unsigned int* s_hist, bool active, int digit)
{
    const unsigned long long act = __builtin_amdgcn_ballot_w64(active);
    if (act == 0ull) return;
    const int first = __builtin_ctzll(act);
    const int lead = __builtin_amdgcn_readlane(digit, first);
    const bool same = active && digit == lead;
    const unsigned long long m = __builtin_amdgcn_ballot_w64(same);
    if ((int)(threadIdx.x & 63) == first) atomicAdd(&s_hist[lead], (unsigned int)__builtin_popcountll(m));
    if (active && !same) atomicAdd(&s_hist[digit], 1u);
}

// digits of a key: pass 0 bits 31..21, pass 1 bits 20..10, pass 2 bits 9..0
__device__ __forceinline__ int digit_of(uint32_t k, int pass) { return pass == 0 ? (int)(k >> 21) : pass == 1 ? (int)((k >> 10) & 0x7FFu) : (int)(k & 0x3FFu); }

template <int PASS>
__global__ __launch_bounds__(SOP_K_CNT_THREADS) void rank_count_kernel(const SelParams p)
{
    __shared__ unsigned int s_hist[SOP_K_SEL_BINS];
    __shared__ Digit s_found;
    __shared__ unsigned int s_wave[SOP_K_SEL_BINS / 8 / 64];
    for (int i = threadIdx.x; i < SOP_K_SEL_BINS; i += SOP_K_CNT_THREADS) s_hist[i] = 0u;
    // the digits fixed by the earlier passes
    uint32_t prefix = 0, pmask = 0;
    if (PASS >= 1) {
        const Digit f0 = find_digit(p.hist, (unsigned int)p.n_top, &s_found, s_wave);
        prefix = (uint32_t)f0.digit << 21; pmask = 0xFFE00000u;
        if (PASS >= 2) {
            const Digit f1 = find_digit(p.hist + SOP_K_SEL_BINS, f0.rank_in, &s_found, s_wave);
            prefix |= (uint32_t)f1.digit << 10; pmask = 0xFFFFFC00u;
            // (what the split kernel goes on from: it reads the first two histograms no more, and clears them)
            if (blockIdx.x == 0 && threadIdx.x == 0) { p.found[0] = prefix; p.found[1] = f1.rank_in; p.found[2] = f0.above + f1.above; }
        }
    }
    if (PASS == 0)                                                  // the last pass's counts of the call before, which nothing reads any more
        for (int i = (int)(blockIdx.x * SOP_K_CNT_THREADS + threadIdx.x); i < SOP_K_SEL_BINS; i += (int)gridDim.x * SOP_K_CNT_THREADS) p.hist[2 * SOP_K_SEL_BINS + i] = 0u;
    __syncthreads();
    const bool higher = p.higher != 0;
    const long long n4 = p.n >> 2;
    const float4* s4 = reinterpret_cast<const float4*>(p.score);
    for (long long i = (long long)blockIdx.x * SOP_K_CNT_THREADS + threadIdx.x; i < n4; i += (long long)gridDim.x * SOP_K_CNT_THREADS) {
        const float4 v = s4[i];
        const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t k = rank_key(e[j], higher);
            count_digit(s_hist, (k & pmask) == prefix, digit_of(k, PASS));
        }
    }
    if (blockIdx.x == 0 && (long long)threadIdx.x < (p.n & 3)) {     // ragged tail
        const uint32_t k = rank_key(p.score[(n4 << 2) + threadIdx.x], higher);
        if ((k & pmask) == prefix) atomicAdd(&s_hist[digit_of(k, PASS)], 1u);
    }
    __syncthreads();
    unsigned int* out = p.hist + PASS * SOP_K_SEL_BINS;
    for (int i = threadIdx.x; i < SOP_K_SEL_BINS; i += SOP_K_CNT_THREADS) {
        const unsigned int v = s_hist[i];
        if (v) atomicAdd(out + i, v);
    }
}

__global__ __launch_bounds__(SOP_K_SEL_THREADS) void rank_split_kernel(const SelParams p)
{
    __shared__ Digit s_found;
    __shared__ unsigned int s_wave[SOP_K_SEL_THREADS / 64];
    const bool higher = p.higher != 0;
    uint32_t tkey = 0xFFFFFFFFu;
    unsigned int n_a = 0;
    float tau = higher ? __uint_as_float(0x7F800000u) : __uint_as_float(0xFF800000u);
    if (!p.all_b) {
        const Digit f2 = find_digit(p.hist + 2 * SOP_K_SEL_BINS, p.found[1], &s_found, s_wave);
        tkey = p.found[0] | (uint32_t)f2.digit;
        tau = key_score(tkey, higher);
        // keys above tau's, plus every key equal to it
        n_a = p.found[2] + f2.above + p.hist[2 * SOP_K_SEL_BINS + f2.digit];
    }
    const long long n4 = p.n >> 2;
    const float4* s4 = reinterpret_cast<const float4*>(p.score);
    uint32_t* m4 = reinterpret_cast<uint32_t*>(p.pool_b);
    for (long long i = (long long)blockIdx.x * SOP_K_SEL_THREADS + threadIdx.x; i < n4; i += (long long)gridDim.x * SOP_K_SEL_THREADS) {
        uint32_t w = 0x01010101u;
        if (!p.all_b) {
            const float4 v = s4[i];
            const float e[4] = {v.x, v.y, v.z, v.w};
            w = 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) w |= (rank_key(e[j], higher) < tkey ? 1u : 0u) << (8 * j);
        }
        m4[i] = w;
    }
    if (blockIdx.x == 0 && (long long)threadIdx.x < (p.n & 3)) {
        const long long i = (n4 << 2) + threadIdx.x;
        p.pool_b[i] = p.all_b ? 1 : (rank_key(p.score[i], higher) < tkey ? 1 : 0);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) { *p.tau = tau; *p.n_a = (long long)n_a; }
    // the first two histograms are zero for the next call (the last one is cleared by its first kernel: every workgroup of this one reads it)
    for (long long gi = (long long)blockIdx.x * SOP_K_SEL_THREADS + threadIdx.x; !p.all_b && gi < 2 * SOP_K_SEL_BINS; gi += (long long)gridDim.x * SOP_K_SEL_THREADS)
        p.hist[gi] = 0u;
}

// ---- several thresholds at once (the sweep over the partition parameter: nested pools), several planes ----
// Bins of the first pass, in the keys' order: 2^21 keys each, but for the scores in [7/8, 1) (2^21 keys from `fine0`), which have SOP_K_SEL_FINE bins of
// 256 keys in the place of one
__device__ __forceinline__ uint32_t fine_from(bool higher) { return higher ? 0xBF600000u : ~0xBF7FFFFFu; }
__device__ __forceinline__ int first_bin(uint32_t k, uint32_t fine0)
{
    const uint32_t in = k - fine0;
    const int c = (int)(k >> 21), f = (int)((fine0 >> 21) + (in >> 8));
    return in < (1u << 21) ? f : k < fine0 ? c : c + (SOP_K_SEL_FINE - 1);
}

struct Found { int bin; unsigned int rank_in, above, count; };

// NT threads look into the NT * PER bins of a histogram in LDS: thread t of them holds the PER bins below (NT - t) PER.  For every rank (1-based from the top) of thresholds
// j0 .. j1-1, the one thread whose bins contain it writes what it finds: `above` keys lie in higher bins, the wanted key has rank `rank_in` among the bin's
// `count`.  NT is a multiple of 64; s_wave holds a word for every wavefront of the workgroup.  All threads of the workgroup come here (j0 = j1: with nothing to look for).
template <int NT, int PER, class R>
__device__ __forceinline__ void find_ranks(const unsigned int* hist, int j0, int j1, R rank_of, Found* out, unsigned int* s_wave)
{
    const int t = (int)threadIdx.x % NT, lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6, w0 = (int)threadIdx.x / NT * (NT / 64);
    const unsigned int base = (unsigned int)((NT - 1 - t) * PER);
    unsigned int h[PER], sum = 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) h[i] = j0 < j1 ? hist[base + i] : 0u;
#pragma unroll
    for (int i = 0; i < PER; ++i) sum += h[i];
    unsigned int inc = sum;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
        const unsigned int v = __shfl_up(inc, st, 64);
        if (lane >= st) inc += v;
    }
    if (lane == 63) s_wave[wv] = inc;
    if (t == 0) for (int j = j0; j < j1; ++j) out[j] = Found{0, 1u, 0u, 0u};          // (fewer keys than the rank: stay in bounds)
    __syncthreads();
    for (int i = w0; i < wv; ++i) inc += s_wave[i];
    for (int j = j0; j < j1; ++j) {
        const unsigned int rank = rank_of(j);
        unsigned int c = inc - sum;
        if (c < rank && rank <= inc) {                              // exactly one thread
            Found f = {0, 1u, 0u, 0u};
#pragma unroll
            for (int i = PER - 1; i >= 0; --i) {
                if (c < rank && rank <= c + h[i]) { f.bin = (int)base + i; f.rank_in = rank - c; f.above = c; f.count = h[i]; }
                c += h[i];
            }
            out[j] = f;
        }
    }
    __syncthreads();
}

// One count into an LDS histogram for every active lane.  Adds to one word are served one after the other, so the lanes that share the first one's bin are counted with a single
// add where they are many (a plane of equal scores, or half of one); few of them cost less as adds of their own.  (Merged only where all lanes agree: 14.7 M scores of which half
// are equal 153 us, 92 so; 2.8 M, four thresholds, 59.5 and 47.7.  From 8 lanes on or from 24: the same.  With a look at the first lane that holds another
// bin, 104 and 50.7, and 10 % longer for scores of any kind.)
#define SOP_K_SEL_MERGE 24
__device__ __forceinline__ void count_bin(unsigned int* s_hist, int bin)
{
    const int lead = __builtin_amdgcn_readfirstlane(bin);
    const unsigned long long same = __builtin_amdgcn_ballot_w64(bin == lead);
    if (__builtin_popcountll(same) >= SOP_K_SEL_MERGE) {
        if ((int)(threadIdx.x & 63) == __builtin_ctzll(same)) atomicAdd(&s_hist[lead], (unsigned int)__builtin_popcountll(same));
        else if (bin != lead) atomicAdd(&s_hist[bin], 1u);
    } else atomicAdd(&s_hist[bin], 1u);
}

// the parameters of one plane of a launch over several score planes
__device__ __forceinline__ SelMParams plane_of(SelMParams p, unsigned int q)
{
    p.score += (size_t)q * (size_t)p.n;
    p.hist += (size_t)q * SOP_K_SELM_WORDS;
    p.level += (size_t)q * (size_t)p.n;
    p.tau += q * SOP_K_SEL_MAXLEV;
    p.n_a += q * SOP_K_SEL_MAXLEV;
    p.state += q;
    return p;
}

// threshold j's rank (below 2^31; by selects: an index into the launch parameters would put them in scratch memory)
__device__ __forceinline__ unsigned int top_of(const SelMParams& p, int j)
{
    unsigned int r = 0u;
    _Pragma("unroll") for (int t = 0; t < SOP_K_SEL_MAXLEV; ++t) r = t == j ? (unsigned int)p.n_top[t] : r;
    return r;
}

// This workgroup's counts join the plane's, and the workgroup whose ticket is the last returns true: all counts have arrived then (every add's
// returned value has been waited for before the ticket is taken).
// It holds the totals in s_hist then, in place of its own counts (read from memory lane by lane; each thread reading the run of bins that it looks into took 10 us more).
template <int AT_ONCE>
__device__ __forceinline__ bool join_counts(unsigned int* s_hist, unsigned int words, unsigned int* out, unsigned int* done, unsigned int* s_last)
{
    __syncthreads();
    for (unsigned int i0 = threadIdx.x; i0 < words; i0 += AT_ONCE * SOP_K_CNT_THREADS) {      // (a round trip to memory for AT_ONCE words)
        unsigned int before[AT_ONCE];
#pragma unroll
        for (int j = 0; j < AT_ONCE; ++j) {
            const unsigned int i = i0 + j * SOP_K_CNT_THREADS, v = i < words ? s_hist[i] : 0u;
            before[j] = 0u;
            if (v) before[j] = atomicAdd(out + i, v);
        }
#pragma unroll
        for (int j = 0; j < AT_ONCE; ++j) asm volatile("" :: "v"(before[j]) : "memory");
    }
    __syncthreads();
    if (threadIdx.x == 0) *s_last = atomicAdd(done, 1u) == gridDim.x - 1 ? 1u : 0u;
    __syncthreads();
    if (*s_last == 0u) return false;
    for (unsigned int i0 = threadIdx.x; i0 < words; i0 += AT_ONCE * SOP_K_CNT_THREADS) {
        unsigned int v[AT_ONCE];
#pragma unroll
        for (int j = 0; j < AT_ONCE; ++j) v[j] = __hip_atomic_load(out + min(i0 + j * SOP_K_CNT_THREADS, words - 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < AT_ONCE; ++j) if (i0 + j * SOP_K_CNT_THREADS < words) s_hist[i0 + j * SOP_K_CNT_THREADS] = v[j];
    }
    __syncthreads();
    return true;
}

// What a pass hands on: lane j of a wavefront comes with threshold j's digits.  Thresholds that look into the same bin share the histogram of
// the first of them.
struct Digits { unsigned int prefix, mask, rank_in, above; unsigned long long tkey; };
__device__ __forceinline__ void hand_on(const SelMParams& p, const Digits& d)
{
    const int j = (int)threadIdx.x & 63;
    int alias = j;
#pragma unroll
    for (int i = SOP_K_SEL_MAXLEV - 1; i >= 0; --i) {
        const unsigned int pi = (unsigned int)__builtin_amdgcn_readlane((int)d.prefix, i), mi = (unsigned int)__builtin_amdgcn_readlane((int)d.mask, i);
        if (i < j && mi == d.mask && pi == d.prefix) alias = i;
    }
    const unsigned int open = (unsigned int)__builtin_amdgcn_ballot_w64(j < SOP_K_SEL_MAXLEV && d.mask != 0xFFFFFFFFu && alias == j);
    if (j < SOP_K_SEL_MAXLEV) {
        SelMState& st = *p.state;
        st.prefix[j] = d.prefix; st.mask[j] = d.mask; st.rank_in[j] = d.rank_in; st.above[j] = d.above; st.alias[j] = alias; st.tkey[j] = d.tkey;
        if (j == 0) st.open = open;
    }
}

// the keys of the plane's scores, four at a time, the next four asked for before the ones at hand are used; f(keys, how many)
template <class F>
__device__ __forceinline__ void every_key(const SelMParams& p, F f)
{
    const bool higher = p.higher != 0;
    const long long n4 = p.n >> 2, step = (long long)gridDim.x * SOP_K_CNT_THREADS;
    const float4* s4 = reinterpret_cast<const float4*>(p.score);
    long long i = (long long)blockIdx.x * SOP_K_CNT_THREADS + threadIdx.x;
    float4 nv = i < n4 ? s4[i] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (; i < n4; i += step) {
        const float4 v = nv;
        if (i + step < n4) nv = s4[i + step];
        const uint32_t k[4] = {rank_key(v.x, higher), rank_key(v.y, higher), rank_key(v.z, higher), rank_key(v.w, higher)};
        f(k, 4);
    }
    if (blockIdx.x == 0 && (long long)threadIdx.x < (p.n & 3)) {     // ragged tail
        const uint32_t k[4] = {rank_key(p.score[(n4 << 2) + threadIdx.x], higher), 0u, 0u, 0u};
        f(k, 1);
    }
}

__global__ __launch_bounds__(SOP_K_CNT_THREADS) void rank_first_kernel(const SelMParams pp)
{
    const SelMParams p = plane_of(pp, blockIdx.y);
    __shared__ unsigned int s_hist[SOP_K_SEL_BINS1_PAD];
    __shared__ unsigned int s_wave[SOP_K_CNT_THREADS / 64], s_last;
    __shared__ Found s_found[SOP_K_SEL_MAXLEV];
    for (int i = threadIdx.x; i < SOP_K_SEL_BINS1_PAD; i += SOP_K_CNT_THREADS) s_hist[i] = 0u;
    __syncthreads();
    const uint32_t fine0 = fine_from(p.higher != 0);
    every_key(p, [&](const uint32_t (&k)[4], int n) {
#pragma unroll
        for (int j = 0; j < 4; ++j) if (j < n) count_bin(s_hist, first_bin(k[j], fine0));
    });
    if (!join_counts<5>(s_hist, SOP_K_SEL_BINS1_PAD, p.hist, p.hist + SOP_K_SEL_DONE, &s_last)) return;
    find_ranks<SOP_K_CNT_THREADS, SOP_K_SEL_BINS1_PAD / SOP_K_CNT_THREADS>(s_hist, 0, p.n_levels, [&](int j) { return top_of(p, j); }, s_found, s_wave);
    if (threadIdx.x < 64) {
        const int j = (int)threadIdx.x, f0 = (int)(fine0 >> 21);
        Digits d = {0u, 0xFFFFFFFFu, 1u, 0u, 1ull << 32};
        if (j < p.n_levels && top_of(p, j) == 0u) {                    // every block goes to the second pool
            p.tau[j] = p.higher ? __uint_as_float(0x7F800000u) : __uint_as_float(0xFF800000u);
            p.n_a[j] = 0;
        } else if (j < p.n_levels) {
            const Found f = s_found[j];
            const bool fine = f.bin >= f0 && f.bin < f0 + SOP_K_SEL_FINE;
            d.mask = fine ? 0xFFFFFF00u : 0xFFE00000u;
            d.prefix = fine ? fine0 + ((uint32_t)(f.bin - f0) << 8) : (uint32_t)(f.bin < f0 ? f.bin : f.bin - (SOP_K_SEL_FINE - 1)) << 21;
            d.rank_in = f.rank_in; d.above = f.above;
        }
        hand_on(p, d);
    }
}

// Second and third pass: every open bin's keys by their next digit, 11 bits below a coarse bin of the first pass, else all that is left (eight bits or ten)
template <int PASS>
__global__ __launch_bounds__(SOP_K_CNT_THREADS) __attribute__((amdgpu_waves_per_eu(8))) void rank_next_kernel(const SelMParams pp)
{
    const SelMParams p = plane_of(pp, blockIdx.y);
    extern __shared__ unsigned int s_mh[];                          // [n_levels][SOP_K_SEL_BINS]
    __shared__ unsigned int s_wave[SOP_K_CNT_THREADS / 64], s_last;
    __shared__ Found s_found[SOP_K_SEL_MAXLEV];
    // (what the pass before handed on, the same in every lane: scalar reads)
    typedef const __attribute__((address_space(4))) SelMState ConstState;
    ConstState& cs = *(ConstState*)(uintptr_t)p.state;
    const uint32_t open = cs.open;
    if (open == 0u) return;
    const int L = p.n_levels;
    for (int i = threadIdx.x; i < L * SOP_K_SEL_BINS; i += SOP_K_CNT_THREADS) s_mh[i] = 0u;
    __syncthreads();
    every_key(p, [&](const uint32_t (&k)[4], int n) {
        for (uint32_t left = open; left != 0u; left &= left - 1u) {
            const int t = __builtin_ctz(left);
            const uint32_t pre = cs.prefix[t], msk = cs.mask[t];
            const bool in[4] = {(k[0] & msk) == pre, n > 1 && (k[1] & msk) == pre, n > 1 && (k[2] & msk) == pre, n > 1 && (k[3] & msk) == pre};
            if (__builtin_amdgcn_ballot_w64(in[0] | in[1] | in[2] | in[3]) == 0ull) continue;     // (most often: a bin holds a thousandth of the keys)
            const uint32_t shift = msk == 0xFFE00000u ? 10u : 0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) if (in[j]) count_bin(s_mh + t * SOP_K_SEL_BINS, (int)((k[j] & ~msk) >> shift));
        }
    });
    const int my = ((int)threadIdx.x / 128) & (SOP_K_SEL_MAXLEV - 1), me = (int)threadIdx.x & (SOP_K_SEL_MAXLEV - 1);
    const bool on = my < L && p.state->mask[my] != 0xFFFFFFFFu;
    const unsigned int rank = p.state->rank_in[my];
    const int alias = p.state->alias[my];
    Digits d = {p.state->prefix[me], p.state->mask[me], p.state->rank_in[me], p.state->above[me], p.state->tkey[me]};
    unsigned int* const hist = p.hist + SOP_K_SEL_BINS1_PAD + (PASS == 1 ? 0 : SOP_K_SEL_MAXLEV * SOP_K_SEL_BINS);
    if (!join_counts<4>(s_mh, (unsigned int)(L * SOP_K_SEL_BINS), hist, p.hist + SOP_K_SEL_DONE + PASS * 32, &s_last)) return;
    static_assert(SOP_K_CNT_THREADS == 128 * SOP_K_SEL_MAXLEV, "two wavefronts a threshold");
    find_ranks<128, SOP_K_SEL_BINS / 128>(s_mh + (on ? alias : 0) * SOP_K_SEL_BINS, my, on ? my + 1 : my, [&](int) { return rank; }, s_found, s_wave);
    if (threadIdx.x < 64) {
        const int j = (int)threadIdx.x;
        if (j >= SOP_K_SEL_MAXLEV) d.mask = 0xFFFFFFFFu;
        if (j < L && d.mask != 0xFFFFFFFFu) {
            const Found f = s_found[j];
            if (d.mask == 0xFFE00000u) {
                d.prefix |= (uint32_t)f.bin << 10; d.mask = 0xFFFFFC00u;
                d.rank_in = f.rank_in; d.above += f.above;
            } else {                                                // the key is known: the first pool holds the keys above it and all those equal to it
                const uint32_t key = d.prefix | (uint32_t)f.bin;
                d.mask = 0xFFFFFFFFu; d.tkey = key;
                p.tau[j] = key_score(key, p.higher != 0);
                p.n_a[j] = (long long)(d.above + f.above + f.count);
            }
        }
        hand_on(p, d);
    }
}

__global__ __launch_bounds__(SOP_K_SEL_THREADS) void rank_level_kernel(const SelMParams pp)
{
    const SelMParams p = plane_of(pp, blockIdx.y);
    const bool higher = p.higher != 0;
    // the thresholds' keys (the same in every lane: scalar registers); those that every block ranks worse than are counted in `base`
    uint32_t tkey[SOP_K_SEL_MAXLEV], base = 0u;
    const int L = p.n_levels;
    _Pragma("unroll") for (int j = 0; j < SOP_K_SEL_MAXLEV; ++j) {
        tkey[j] = 0u;
        if (j >= L) continue;
        const unsigned long long t = p.state->tkey[j];
        tkey[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)t);
        base += (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(t >> 32));
    }
    auto level_of = [&](float v) {
        const uint32_t k = rank_key(v, higher);
        uint32_t lv = base;
        _Pragma("unroll") for (int t = 0; t < SOP_K_SEL_MAXLEV; ++t) lv += k < tkey[t] ? 1u : 0u;      // (beyond the last threshold: no key ranks worse)
        return lv;
    };
    const long long n4 = p.n >> 2;
    const float4* s4 = reinterpret_cast<const float4*>(p.score);
    uint32_t* m4 = reinterpret_cast<uint32_t*>(p.level);
    for (long long i = (long long)blockIdx.x * SOP_K_SEL_THREADS + threadIdx.x; i < n4; i += (long long)gridDim.x * SOP_K_SEL_THREADS) {
        const float4 v = s4[i];
        m4[i] = level_of(v.x) | level_of(v.y) << 8 | level_of(v.z) << 16 | level_of(v.w) << 24;
    }
    if (blockIdx.x == 0 && (long long)threadIdx.x < (p.n & 3)) {
        const long long i = (n4 << 2) + threadIdx.x;
        p.level[i] = (unsigned char)level_of(p.score[i]);
    }
    // counts and tickets, which nothing reads any more (the thresholds are in the state), are zero again for the next call or the next replay of this one
    for (long long gi = (long long)blockIdx.x * SOP_K_SEL_THREADS + threadIdx.x; gi < SOP_K_SELM_WORDS; gi += (long long)gridDim.x * SOP_K_SEL_THREADS)
        p.hist[gi] = 0u;
}

// no first pool wanted of any threshold: the defaults (every block ranks worse)
__global__ void rank_none_kernel(const SelMParams pp)
{
    const SelMParams p = plane_of(pp, blockIdx.x);
    const int j = (int)threadIdx.x;
    if (j < p.n_levels) {
        p.tau[j] = p.higher ? __uint_as_float(0x7F800000u) : __uint_as_float(0xFF800000u);
        p.n_a[j] = 0;
    }
    if (j < SOP_K_SEL_MAXLEV) p.state->tkey[j] = 1ull << 32;
}

}  // namespace sopk

extern "C" hipError_t sopk_selm_launch(const SelMParams* pp, int n_wg_count, int n_wg_next, int n_wg, void* stream)
{
    const SelMParams p = *pp;
    hipStream_t st = (hipStream_t)stream;
    const unsigned planes = (unsigned)(p.n_planes > 0 ? p.n_planes : 1);
    const dim3 grid((unsigned)n_wg, planes), block(SOP_K_SEL_THREADS), cgrid((unsigned)n_wg_count, planes), ngrid((unsigned)n_wg_next, planes), cblock(SOP_K_CNT_THREADS);
    bool any = false;
    for (int j = 0; j < p.n_levels; ++j) any = any || p.n_top[j] != 0;
    if (any) {
        const size_t lds = (size_t)p.n_levels * SOP_K_SEL_BINS * sizeof(unsigned int);
        if (lds > 48 * 1024) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sopk::rank_next_kernel<1>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sopk::rank_next_kernel<2>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(sopk::rank_first_kernel, cgrid, cblock, 0, st, p);
        hipLaunchKernelGGL((sopk::rank_next_kernel<1>), ngrid, cblock, lds, st, p);
        hipLaunchKernelGGL((sopk::rank_next_kernel<2>), ngrid, cblock, lds, st, p);
    } else hipLaunchKernelGGL(sopk::rank_none_kernel, dim3(planes), dim3(64), 0, st, p);
    hipLaunchKernelGGL(sopk::rank_level_kernel, grid, block, 0, st, p);
    return hipGetLastError();
}

extern "C" hipError_t sopk_sel_launch(const SelParams* pp, int n_wg_count, int n_wg, void* stream)
{
    const SelParams p = *pp;
    hipStream_t st = (hipStream_t)stream;
    const dim3 grid((unsigned)n_wg), block(SOP_K_SEL_THREADS);
    if (!p.all_b) {
        // few, large workgroups: every workgroup adds its whole histogram to the layer's with
        // same-address atomics, which serialise
        const dim3 cgrid((unsigned)n_wg_count), cblock(SOP_K_CNT_THREADS);
        hipLaunchKernelGGL((sopk::rank_count_kernel<0>), cgrid, cblock, 0, st, p);
        hipLaunchKernelGGL((sopk::rank_count_kernel<1>), cgrid, cblock, 0, st, p);
        hipLaunchKernelGGL((sopk::rank_count_kernel<2>), cgrid, cblock, 0, st, p);
    }
    hipLaunchKernelGGL(sopk::rank_split_kernel, grid, block, 0, st, p);
    return hipGetLastError();
}
