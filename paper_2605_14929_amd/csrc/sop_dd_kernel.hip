// Statistics pass of the data-derived codebook (DD atom): a channel-norm-weighted histogram of the
// block-normalised weights of one layer, in exact integer arithmetic.
//
// Definition (every operation one IEEE binary32 rounding unless it is exact):
//   cmax   = max_k c_k                       cs = fl(2^20 / cmax)          (c == NULL: c_k = 1)
//   block  a = max_i |w_i|; blocks with a == 0 contribute nothing;  r = fl(1 / a)
//   weight x = fl(w_i * r)   in [-1, 1]      mass = rint(fl(c_i * cs))   (units of 2^-20 cmax, half to even)
//          bin    = clamp(floor(fl(fl(x * H/2) + H/2)), 0, H-1)         H bins over [-1, 1]
//   hist[bin] += mass                                                   (64-bit integers)
// Integer sums do not depend on the order of addition, so the histogram is reproducible bit for bit.
// Only rows 0, row_step, 2*row_step, ... enter (row_step = 1: the whole layer), and, when a block
// mask is given, only blocks whose mask byte is non-zero.  With levels (the sweep over the partition
// parameter of the per-layer search: nested fitting pools) the mask byte names one of L histograms, and
// the result holds the L pool histograms: one pass over the weights serves every pool of the sweep.  With several
// level planes (one per codebook of the search: each ranks the blocks its own way) the same pass fills every
// plane's histograms: the weights are read, normalised and binned once.
//
// Work mapping as in the search kernel: a lane owns min(g,16) consecutive elements of a row, a
// wavefront walks down the rows of a 64-lane strip, the next row requested a step ahead.  Each workgroup (16 wavefronts,
// one per compute unit) finds cmax itself, accumulates in LDS and adds its histogram to one of the layer's rows of running sums (kept in
// the context, zero between calls; dd_rows()) with 64-bit global atomics; the workgroup that finishes last moves the result to
// the caller's buffer and leaves zeros behind.  One kernel per call.
//
// What does not depend on the layer's size is most of a layer below 100 MB: launch, norms, first row, and then 256 workgroups that add to
// the same words and take tickets.  First row, norms and the clearing of LDS overlap, the workgroups are divided among four rows of
// sums, and each begins at a place of its own in its row (all in one order, they queued up on one line after the other).
// bf16, 1024 bins: 2048 x 4096 15.1 us -> 11.3, 4096 x 4096 18.5 -> 14.6, 4096 x 11008 26.3 -> 23.2; 8192 words: 27.5 -> 23.8, 30 -> 26.9,
// 39.8 -> 37; 28672 x 8192 88 before and after.
//
// In LDS a weight costs one 32-bit add.  The pass is bound by those adds (a wavefront's 64 lanes fall on random bins: bank
// conflicts) beside the read of the layer, and a 64-bit add takes twice the bank cycles.  The 32-bit counts sit in p.n_repl
// replicas, each shared by 16 / n_repl wavefronts, and never wrap: a step adds at most S = the sum of the masses of the
// strip's columns to any one word, and a wavefront that has added as much as its share of 2^32 - 1 since it last emptied its
// replica empties it (exchange with zero, word by word) into the 64-bit histogram first.  Heavy-tailed channel norms have S near
// 2^25 and are hardly ever emptied before the end.  With norms near their maximum (S up to 2^30) many words and shared
// replicas would be emptied at every other step, at several times the cost of the step's own adds: a wavefront whose strip's S
// is above p.dear_mass (dd_dear_mass()) and which cannot get through its steps without emptying adds to the 64-bit sums.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sop_kparams.h"

namespace sopk {

// floor of a non-negative value as an unsigned integer; values below zero and NaN give 0, values past 2^32 the largest integer
// (the hardware's conversion saturates; the language leaves such conversions undefined)
__device__ __forceinline__ unsigned int cvt_floor(float v)
{
    unsigned int r;
    asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// REPL: 32-bit counts in replicas; else every weight adds to the 64-bit sums (dd_replicas()).  AHEAD: the next row is requested a
// step ahead; without it for layers that give no wavefront a second step (a smaller kernel: 256 x 1024, 1024 bins, 6.0 us -> 5.8)
template <bool BF16, int EPL, int LPB, bool REPL, bool AHEAD>
__global__ __launch_bounds__(SOP_K_DD_THREADS) void dd_hist_kernel(const DdParams p)
{
    extern __shared__ __align__(16) unsigned long long s_hist[];      // [H] 64-bit sums, then n_repl x [H] 32-bit counts
    __shared__ float s_max[SOP_K_DD_THREADS / 64];
    __shared__ unsigned int s_flag;
    constexpr int NW = SOP_K_DD_THREADS / 64, NV = BF16 ? EPL / 8 : EPL / 4;
    constexpr int PRE = 4;                                            // level planes whose bytes are requested a step ahead
    const int HB = p.n_bins;                                          // bins of one histogram
    const int NP = p.n_levels > 0 ? p.n_planes : 1;                   // level planes
    const int H = p.n_bins * (p.n_levels > 0 ? p.n_levels : 1) * NP;  // words of all the histograms of the call
    unsigned int* s_cnt = reinterpret_cast<unsigned int*>(s_hist + H);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // this wavefront's steps: floor(T b / G) = (T / G) b + (T % G) b / G with the first two from the host, all of it in 32 bits but
    // for a product (64-bit divisions took a few tenths of a microsecond of a small layer's six)
    const unsigned int wave = blockIdx.x * NW + (unsigned int)wv, n_waves = (unsigned int)p.n_waves;
    const unsigned int r0 = p.units_r * wave / n_waves, r1 = p.units_r * (wave + 1u) / n_waves;       // (G below 2^16)
    const long long u0 = p.units_q * wave + r0;
    const int n_steps = __builtin_amdgcn_readfirstlane((int)p.units_q + (int)(r1 - r0));
    const float half = 0.5f * (float)HB;
    unsigned int* const cnt = s_cnt + (REPL ? (wv & (p.n_repl - 1)) * H : 0);                         // this wavefront's replica
    const unsigned int budget = REPL ? 0xFFFFFFFFu / (unsigned int)(NW / p.n_repl) : 0u;
    unsigned int spent = 0u, per_step = 0u;                       // added to any one word since the last emptying, at most; by one step, at most

    // request side: band, strip and row of the next step, kept on the scalar unit.  Steps run down the BAND rows of a strip, then
    // through the strips of the band, then through the bands: the wavefronts of a workgroup stay
    // within a few megabytes of the layer, where a walk down whole strips spreads them over all of it, a row's stride between any
    // two reads (28672 x 8192: 108 us, 92 in bands of 32 or 128 rows; 4096 x 11008, a third of a band a workgroup: 30.1 us, 30.7).
    constexpr unsigned int BAND = 128;
    const unsigned int strips = (unsigned int)p.strips;
    auto rows_of = [&](long long b) -> unsigned int { return (unsigned int)min((long long)BAND, p.Ms - b); };
    long long rb = 0, rm = 0;                     // first row of the band; row of the step: indices among the sampled rows
    unsigned int rh = 0u, rs = 0u;                // rows of the band; strip
    if (n_steps > 0) {
        if (p.total_units < (1ll << 31) && strips <= (1u << 24)) {
            const unsigned int u = (unsigned int)__builtin_amdgcn_readfirstlane((int)u0), band = u / (BAND * strips);
            rb = (long long)__builtin_amdgcn_readfirstlane((int)(band * BAND));
            rh = rows_of(rb);
            const unsigned int rem = u - band * (BAND * strips);
            rs = (unsigned int)__builtin_amdgcn_readfirstlane((int)(rem / rh));
            rm = rb + (rem - rs * rh);
        } else {
            const long long per_band = (long long)BAND * p.strips, band = u0 / per_band, rem = u0 - band * per_band;
            rb = band * BAND;
            rh = rows_of(rb);
            rs = (unsigned int)(rem / rh);
            rm = rb + (rem - (long long)rs * rh);
        }
    }
    uint4 raw[NV];
    int lvl[PRE];
    auto request = [&]() __attribute__((always_inline)) {
        const long long c0 = (long long)rs * (64 * EPL), room = p.K - c0;
        const bool valid = (long long)lane * EPL < room;
        const char* src = reinterpret_cast<const char*>(p.W) + (rm * p.row_step * p.ldw + c0 + lane * EPL) * (BF16 ? 2 : 4);
#pragma unroll
        for (int i = 0; i < NV; ++i) raw[i] = valid ? reinterpret_cast<const uint4*>(src)[i] : make_uint4(0u, 0u, 0u, 0u);
        if (p.block_mask) {
            const long long blk = rm * p.row_step * p.Bk + ((long long)rs * 64 + lane) / LPB;
#pragma unroll
            for (int pl = 0; pl < PRE; ++pl) lvl[pl] = pl < NP && valid ? p.block_mask[(long long)pl * p.plane_stride + blk] : 0;
        }
    };
    // channel norms of the lane's columns in strip st
    float4 cv[EPL / 4];
    auto load_norms = [&](unsigned int st) __attribute__((always_inline)) {
        const long long col0 = ((long long)st * 64 + lane) * EPL;
#pragma unroll
        for (int i = 0; i < EPL / 4; ++i) {
            cv[i] = make_float4(1.f, 1.f, 1.f, 1.f);
            if (p.c) cv[i] = col0 < p.K ? reinterpret_cast<const float4*>(p.c + col0)[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    // The first row and the first strip's norms are asked for ahead of everything that does not need them: the largest norm,
    // the clearing of the sums and the barrier take as long as they travel.
    if (n_steps > 0) {
        if (AHEAD) request();
        load_norms(rs);
    }
    {
        uint4* z = reinterpret_cast<uint4*>(s_hist);                  // (H is a multiple of 64)
        const int n16 = (H / 4) * (REPL ? 2 + p.n_repl : 2);
        for (int i = threadIdx.x; i < n16; i += SOP_K_DD_THREADS) z[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    // cmax = max_k c_k (order-independent), found by every workgroup for itself
    float cmax = 1.0f;
    if (p.c) {
        // 16 bytes per lane and four loads in flight (a loop of single dependent loads would spend a round
        // trip to L2 per element); K is a multiple of 8 and c is 16-byte aligned
        float v = 0.0f;
        const long long k4 = p.K >> 2;
        const float4* c4 = reinterpret_cast<const float4*>(p.c);
        for (long long k0 = threadIdx.x; k0 < k4; k0 += 4 * SOP_K_DD_THREADS) {
            float4 t[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) t[j] = k0 + j * SOP_K_DD_THREADS < k4 ? c4[k0 + j * SOP_K_DD_THREADS] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int j = 0; j < 4; ++j) v = fmaxf(fmaxf(fmaxf(v, t[j].x), fmaxf(t[j].y, t[j].z)), t[j].w);
        }
#pragma unroll
        for (int st = 1; st < 64; st <<= 1) v = fmaxf(v, __shfl_xor(v, st, 64));
        if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (p.c) {
        cmax = s_max[0];
#pragma unroll
        for (int i = 1; i < NW; ++i) cmax = fmaxf(cmax, s_max[i]);
    }

    const float cs = cmax > 0.0f ? 1048576.0f / cmax : 0.0f;      // all-zero channel norms: an empty histogram
    // cs overflows for norms below 2^20 / FLT_MAX: the conversion below then gives 2^31 - 1 for every non-zero norm, and a step's
    // additions to one word do not fit 32 bits
    const bool huge = !(cs < INFINITY);
    unsigned int cur_strip = 0xFFFFFFFFu;
    bool wide = !REPL;                            // this strip's steps add to the 64-bit sums
    unsigned int mass[EPL]; // rint(fl(c*cs)) of the owned columns
#pragma unroll
    for (int i = 0; i < EPL; ++i) mass[i] = 0u;

    for (int u = 0; u < n_steps; ++u) {
        const unsigned int strip = rs;
        const long long m = rm;
        const long long col0 = ((long long)strip * 64 + lane) * EPL;
        const bool valid = col0 < p.K;
        if (strip != cur_strip) {
            cur_strip = strip;
            if (u > 0) load_norms(strip);
            unsigned int sum = 0u;                                // at most 16 * 2^20 a lane
#pragma unroll
            for (int i = 0; i < EPL; i += 4) {
                const float t[4] = {cv[i / 4].x, cv[i / 4].y, cv[i / 4].z, cv[i / 4].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    mass[i + j] = (unsigned int)__float2int_rn(t[j] * cs);
                    sum += mass[i + j];
                }
            }
            if constexpr (REPL) {
#pragma unroll
                for (int st = 1; st < 64; st <<= 1) sum += (unsigned int)__shfl_xor((int)sum, st, 64);
                per_step = (unsigned int)__builtin_amdgcn_readfirstlane((int)sum);       // at most 2^30 (not used where `huge`)
                // (a step that alone exceeds the wavefront's share, as in a shared replica under near-equal norms, goes there too)
                wide = huge || per_step > budget ||
                       (per_step > p.dear_mass && (unsigned long long)per_step * (unsigned int)(n_steps - u) > budget - spent);
            }
        }
        if (REPL && !wide) {
            if (per_step > budget - spent) {
                for (int i = lane; i < H; i += 64) {
                    const unsigned int v = atomicExch(&cnt[i], 0u);
                    if (v) atomicAdd(&s_hist[i], (unsigned long long)v);
                }
                spent = 0u;
            }
            spent += per_step;
        }
        if (!AHEAD) request();
        float w[EPL];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const uint32_t v[4] = {raw[i].x, raw[i].y, raw[i].z, raw[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (BF16) { w[8 * i + 2 * j] = __uint_as_float(v[j] << 16); w[(8 * i + 2 * j + 1) % EPL] = __uint_as_float(v[j] & 0xFFFF0000u); }
                else w[4 * i + j] = __uint_as_float(v[j]);
            }
        }
        int lv_now[PRE];
#pragma unroll
        for (int pl = 0; pl < PRE; ++pl) lv_now[pl] = lvl[pl];
        if (++rm == rb + rh) {
            if (++rs == strips) { rs = 0u; rb += BAND; rh = rows_of(rb); }
            rm = rb;
        }
        if (AHEAD && u + 1 < n_steps) request();
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < EPL; ++i) a = fmaxf(a, fabsf(w[i]));
        if (LPB >= 2) a = fmaxf(a, __shfl_xor(a, 1, 64));
        if (LPB >= 4) a = fmaxf(a, __shfl_xor(a, 2, 64));
        if (valid && a > 0.0f) {
            const float r = 1.0f / a;
            unsigned int bin[EPL];
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
                const float x = w[i] * r;
                // x*half is exact: the fma rounds the sum once; the conversion truncates, takes what is below zero to 0 and NaN to 0
                bin[i] = min(cvt_floor(__fmaf_rn(x, half, half)), (unsigned int)(HB - 1));
            }
            auto add = [&](int hb) __attribute__((always_inline)) {
                if (REPL && !wide) {
#pragma unroll
                    for (int i = 0; i < EPL; ++i) atomicAdd(&cnt[hb + bin[i]], mass[i]);
                } else {
#pragma unroll
                    for (int i = 0; i < EPL; ++i) atomicAdd(&s_hist[hb + bin[i]], (unsigned long long)mass[i]);
                }
            };
            if (!p.block_mask) add(0);
            else {
                for (int pl = 0; pl < NP; ++pl) {                 // several level planes: the bins are found once
                    int lv = pl == 0 ? lv_now[0] : pl == 1 ? lv_now[1] : pl == 2 ? lv_now[2] : lv_now[3];
                    if (pl >= PRE) lv = p.block_mask[(long long)pl * p.plane_stride + m * p.row_step * p.Bk + ((long long)strip * 64 + lane) / LPB];
                    if (lv != 0) add(p.n_levels > 0 ? (pl * p.n_levels + min(lv, p.n_levels) - 1) * HB : 0);
                }
            }
        }
    }
    __syncthreads();
    // the workgroup's histogram joins the layer's through 64-bit integer atomics; their returned
    // values are consumed so that they have completed before the workgroup takes its ticket
    // (all of a thread's atomics are issued before the first returned value is looked at: one round trip)
    const unsigned int R = p.n_rows, row = blockIdx.x & (R - 1u);
    {
        // (each workgroup begins elsewhere in the row: 2048 x 4096, 8192 words, 35 us -> 23.8)
        const int turn = (int)((blockIdx.x / R * 64u) % (unsigned int)H);
        unsigned long long before[SOP_K_DD_MAXBINS / SOP_K_DD_THREADS];
#pragma unroll
        for (int j = 0; j < SOP_K_DD_MAXBINS / SOP_K_DD_THREADS; ++j) {
            int i = threadIdx.x + j * SOP_K_DD_THREADS;
            before[j] = 0ull;
            if (i < H) {
                i += turn;
                if (i >= H) i -= H;
                unsigned long long v = s_hist[i];
                if (REPL)
                    for (int r = 0; r < p.n_repl; ++r) v += s_cnt[r * H + i];
                if (v) before[j] = atomicAdd(p.acc + row * (unsigned int)H + i, v);
            }
        }
#pragma unroll
        for (int j = 0; j < SOP_K_DD_MAXBINS / SOP_K_DD_THREADS; ++j) asm volatile("" :: "v"(before[j]) : "memory");
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // the last of a row's workgroups takes the row's ticket, the last row's finishes the call
        unsigned int* const mine = p.done + (1u + row) * SOP_K_DD_DONE_STRIDE;
        unsigned int last = 0u;
        if (R == 1u) last = atomicAdd(p.done, 1u) == gridDim.x - 1u;
        else if (atomicAdd(mine, 1u) == (gridDim.x - row + R - 1u) / R - 1u) { atomicExch(mine, 0u); last = atomicAdd(p.done, 1u) == R - 1u; }
        s_flag = last;
    }
    __syncthreads();
    if (s_flag) {
        constexpr int PER = SOP_K_DD_MAXBINS / SOP_K_DD_THREADS;
        unsigned long long got[PER];
#pragma unroll
        for (int j = 0; j < PER; ++j) got[j] = 0ull;
        if (R > 1u) {
            // (several rows: at most a word a thread, the rows' words asked for together)
            unsigned long long part[SOP_K_DD_ROWS];
            if ((int)threadIdx.x < H) {
#pragma unroll
                for (int r = 0; r < SOP_K_DD_ROWS; ++r) part[r] = atomicExch(p.acc + r * H + threadIdx.x, 0ull);
#pragma unroll
                for (int r = 0; r < SOP_K_DD_ROWS; ++r) got[0] += part[r];
            }
        } else {
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const int i = threadIdx.x + j * SOP_K_DD_THREADS;
                if (i < H) got[j] = atomicExch(p.acc + i, 0ull);
            }
        }
        if (p.n_levels > 1 || NP > 1) {
            // nested pools: histogram j of the result is the sum of the level histograms j .. L-1
            __syncthreads();
#pragma unroll
            for (int j = 0; j < SOP_K_DD_MAXBINS / SOP_K_DD_THREADS; ++j) {
                const int i = threadIdx.x + j * SOP_K_DD_THREADS;
                if (i < H) s_hist[i] = got[j];
            }
            __syncthreads();
            for (int b = threadIdx.x; b < HB * NP; b += SOP_K_DD_THREADS) {
                const int pl = b / HB, bb = b - pl * HB;
                const int base = pl * p.n_levels * HB + bb;
                unsigned long long run = 0ull;
                for (int l = p.n_levels - 1; l >= 0; --l) { run += s_hist[base + l * HB]; p.hist[base + l * HB] = (long long)run; }
            }
        } else {
#pragma unroll
            for (int j = 0; j < SOP_K_DD_MAXBINS / SOP_K_DD_THREADS; ++j) {
                const int i = threadIdx.x + j * SOP_K_DD_THREADS;
                if (i < H) p.hist[i] = (long long)got[j];
            }
        }
        if (threadIdx.x == 0) atomicExch(p.done, 0u);
    }
}

// Weighted Lloyd fit of a codebook on a histogram, a workgroup each: the rounds of sop_dd_fit, to the same bits (integer prefix sums of mass and first
// moment; a cell is the run of bins whose centres lie above one midpoint and not above the next; binary64 midpoints, centres and divisions as on the
// host).  Bound by a round's chain (midpoint, bin, two prefix sums, two divisions), not by data: one wavefront, a lane an entry.  Twenty-four fits of 1024 bins and 20
// rounds take 18 us at once, where the host took 5 us for each while the GPU waited.
__global__ __launch_bounds__(SOP_K_FIT_THREADS) void dd_fit_kernel(const FitParams p)
{
    typedef unsigned long long u64;
    extern __shared__ __align__(16) u64 s_pre[];                      // [n_bins + 1] mass, then [n_bins + 1] first moment in units of 1 / n_bins
    __shared__ u64 s_part[2][SOP_K_FIT_THREADS / 64];
    const int H = p.n_bins, n = p.n_entries, tid = (int)threadIdx.x, lane = tid & 63, wv = tid >> 6;
    u64* const pm = s_pre;
    u64* const pf = s_pre + H + 1;
    const long long* const hist = p.hist + (size_t)blockIdx.x * H;
    // The largest first moment is below 2 H times the total mass, so the sums are exact in 64 bits where the total is at most `most`.  No bin may exceed it either (a negative
    // one does), or the total itself could wrap to something small: a weight's mass is up to 2^31 - 1, and 2^33 of those, 16 GiB of bf16, fit this GPU
    const u64 most = (0x7FFFFFFFFFFFFFFFull >> 1) / (u64)H;
    int beyond = 0;
    for (int b = tid; b < H; b += SOP_K_FIT_THREADS) { const u64 v = (u64)hist[b]; pm[b] = v; beyond |= v > most ? 1 : 0; }
    beyond = __syncthreads_or(beyond);
    // prefix sums: a run of bins a thread
    const int per = (H + SOP_K_FIT_THREADS - 1) / SOP_K_FIT_THREADS, b0 = min(tid * per, H), b1 = min(b0 + per, H);
    u64 m = 0ull, f = 0ull;
    for (int b = b0; b < b1; ++b) { const u64 v = pm[b]; m += v; f += v * (unsigned)(2 * b + 1); }
    u64 im = m, jf = f;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
        const u64 a = (u64)__shfl_up((long long)im, st, 64), c = (u64)__shfl_up((long long)jf, st, 64);
        if (lane >= st) { im += a; jf += c; }
    }
    if (lane == 63) { s_part[0][wv] = im; s_part[1][wv] = jf; }
    __syncthreads();
    for (int i = 0; i < wv; ++i) { im += s_part[0][i]; jf += s_part[1][i]; }
    u64 am = im - m, af = jf - f;
    for (int b = b0; b < b1; ++b) {
        const u64 v = pm[b];
        pm[b] = am; pf[b] = af;
        am += v; af += v * (unsigned)(2 * b + 1);
    }
    if (tid == SOP_K_FIT_THREADS - 1) { pm[H] = im; pf[H] = jf; }
    __syncthreads();
    if (wv != 0) return;
    const u64 total = pm[H];
    int status = beyond || total > most ? SOP_K_FIT_HOST : total == 0ull ? SOP_K_FIT_EMPTY : SOP_K_FIT_OK;
    const bool on = lane < n;
    double cent = on ? (double)p.init[min(lane, SOP_K_FIT_MAXENT - 1)] : 0.0;
    const double inv = 1.0 / (double)H, halfH = 0.5 * (double)H;
    auto centre = [inv](int b) { return -1.0 + (2.0 * (double)b + 1.0) * inv; };
    if (status == SOP_K_FIT_OK) {
        for (int it = 0; it < p.iters; ++it) {
            const double next = __shfl_down(cent, 1, 64), before = cent;
            int end = H;                                              // one past the last bin of the lane's cell
            if (lane + 1 < n) {
                const double mid = 0.5 * (cent + next), g = (mid + 1.0) * halfH;
                int b = g > 0.0 ? (g < (double)H ? (int)g : H) : 0;
                while (b > 0 && mid < centre(b - 1)) --b;
                while (b < H && !(mid < centre(b))) ++b;
                end = b;
            }
            int lo = __shfl_up(end, 1, 64);
            if (lane == 0) lo = 0;
            if (on) {
                const u64 mass = pm[end] - pm[lo], first = pf[end] - pf[lo];
                if (mass > 0ull) cent = ((double)first / (double)mass) * inv - 1.0;      // (H is a power of two: the division by it, exactly)
            }
            const double below = __shfl_up(cent, 1, 64);
            if (__builtin_amdgcn_ballot_w64(on && lane > 0 && !(below <= cent)) != 0ull) { status = SOP_K_FIT_HOST; break; }
            if (__builtin_amdgcn_ballot_w64(on && cent != before) == 0ull) break;      // a round that moves no entry is the last one that could
        }
        const float o = (float)cent, prev = __shfl_up(o, 1, 64);
        const bool bad = (on && lane > 0 && !(prev < o)) || (lane == 0 && !(o < 0.0f)) || (lane == n - 1 && !(o > 0.0f));
        if (status == SOP_K_FIT_OK && __builtin_amdgcn_ballot_w64(bad) != 0ull) status = SOP_K_FIT_NONE;
        if (on) p.out[(size_t)blockIdx.x * SOP_K_FIT_MAXENT + lane] = o;
    }
    if (lane == 0) p.status[blockIdx.x] = status;
}

}  // namespace sopk

// one workgroup a histogram
extern "C" hipError_t sopk_fit_launch(const FitParams* pp, int n_hist, void* stream)
{
    const FitParams p = *pp;
    const size_t lds = (size_t)(p.n_bins + 1) * 16;
    if (lds > 48 * 1024) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sopk::dd_fit_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(sopk::dd_fit_kernel, dim3((unsigned)n_hist), dim3(SOP_K_FIT_THREADS), lds, (hipStream_t)stream, p);
    return hipGetLastError();
}

extern "C" hipError_t sopk_dd_launch(const DdParams* pp, int is_bf16, int g, void* stream)
{
    DdParams p = *pp;
    hipStream_t st = (hipStream_t)stream;
    const unsigned int words = (unsigned int)p.n_bins * (unsigned int)(p.n_levels > 0 ? p.n_levels * p.n_planes : 1);
    const unsigned int wpl = (unsigned int)(g < 16 ? g : 16);
    p.n_repl = (int)dd_replicas(words, wpl, p.n_levels > 0, p.c == nullptr, p.total_units, p.n_waves);
    p.dear_mass = p.n_repl ? dd_dear_mass(words, wpl, (unsigned int)p.n_repl) : 0u;
    p.n_rows = dd_rows(words, (unsigned int)(p.n_waves / (SOP_K_DD_THREADS / 64)));
    p.units_q = p.total_units / p.n_waves;
    p.units_r = (unsigned int)(p.total_units % p.n_waves);
    const size_t lds = (size_t)words * (sizeof(unsigned long long) + (size_t)p.n_repl * 4);
    const dim3 grid((unsigned)(p.n_waves / (SOP_K_DD_THREADS / 64))), block(SOP_K_DD_THREADS);
#define SOPK_DDR(B, E, L, R, N) do { \
        if (lds > 48 * 1024) { const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&sopk::dd_hist_kernel<B, E, L, R, N>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds); if (e != hipSuccess) return e; } \
        hipLaunchKernelGGL((sopk::dd_hist_kernel<B, E, L, R, N>), grid, block, lds, st, p); } while (0)
#define SOPK_DD(B, E, L) do { \
        if (p.n_repl) SOPK_DDR(B, E, L, true, true); \
        else if (p.total_units > p.n_waves) SOPK_DDR(B, E, L, false, true); \
        else SOPK_DDR(B, E, L, false, false); } while (0)
    if (is_bf16) {
        if (g == 8) SOPK_DD(true, 8, 1); else if (g == 16) SOPK_DD(true, 16, 1); else if (g == 32) SOPK_DD(true, 16, 2); else SOPK_DD(true, 16, 4);
    } else {
        if (g == 8) SOPK_DD(false, 8, 1); else if (g == 16) SOPK_DD(false, 16, 1); else if (g == 32) SOPK_DD(false, 16, 2); else SOPK_DD(false, 16, 4);
    }
#undef SOPK_DD
#undef SOPK_DDR
    return hipGetLastError();
}
