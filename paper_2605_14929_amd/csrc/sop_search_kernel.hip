// Pair-search kernel for gfx950 (MI355X).  This file is compiled once per (weight dtype, metric)
// part; SOPK_PART_BF16 and SOPK_PART_METRIC select which instantiations the object holds.
//
// Work mapping.  A lane owns EPL = min(g,16) consecutive elements of one row (one block when
// g <= 16, a half or a quarter of a block when g = 32 / 64: LPB = g/EPL lanes cooperate through
// cross-lane exchanges).  A wavefront covers a "strip" of 64*EPL consecutive columns of one row
// per step and walks down the rows of that strip, so the channel norms of the strip stay in
// registers.  The (strip,row) steps of the whole layer are cut into equal contiguous ranges, one
// per resident wavefront, so every SIMD gets the same amount of work whatever the shape.  The
// weights of the next step are requested before the current step is evaluated.
//
// Every block is read from HBM exactly once.  LDS holds a table over uniform bins of the scaled
// weight x: for every atom each bin contains at most one code boundary, so the nearest entry is a
// table read and one compare.  A bin is a record (BinRec) of half the lower and half the upper value of each of the 8 atoms; the boundary
// is their sum.  For scale words of
// up to 11 magnitude bits LDS also holds (twice the scale, the scale's reciprocal) of every scale code.
//
// Atoms with equal endpoints form a scale group: they share the ideal scale, the scale code and the
// scaled weights, which are computed once per group.
//
// Arithmetic contract (what makes the integer outputs reproducible on any implementation):
//   scale      s* = max(pmax/t+, nmax/-t-)  (IEEE division), times 2^k, rounded to the scale word
//              (nearest, ties to the lower code, saturating), s = value(q) * 2^-k, r = 1/s (IEEE)
//   element    x = fl(w*r); code = number of midpoints strictly below x
//   error      d = fma(-s, L[code], w) (evaluated as fma(-2s, L[code]/2, w): the same product, both factors exact);
//              err = sum fma(fl(c*d), d, .) over chunks of 8 consecutive
//              elements, chunk partials added in a balanced tree in index order
//   cosine     (metric COS only) w^ = fl(s*L[code]); num = sum fma(fl(c*w), w^, .),
//              den = sum fma(fl(c*w^), w^, .), same chunks and tree
//   selection  metrics WSE / MSE: strictly smaller err wins (second atom of a pair, negative scale
//              sign); metric COS: b beats a when fl(q_b*den_a) > fl(q_a*den_b), q = fl(num*|num|),
//              a zero reconstruction counting as q = 0, den = 1
// The cosine values are not decisions; they are evaluated in fp32 and accumulated per lane as the
// deficit 1 - cos; workgroup sums enter the layer sums as 64-bit fixed-point integers.  A lane whose
// block has zero weighted norm adds exactly 1 to every column and 1 to a count column that is
// subtracted at the end.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "sop_kparams.h"

#ifndef SOPK_PART_BF16
#error "compile with -DSOPK_PART_BF16=0|1 -DSOPK_PART_METRIC=0|1|2"
#endif

namespace sopk {

// value of the lane's partner under lane ^ MASK (1 or 2): a data-parallel-primitive move inside quads of lanes, on the vector
// ALU (a general exchange goes through LDS, which the element passes keep busy).  Used where all 64 lanes are active.
template <int MASK> __device__ __forceinline__ float xor_lanes(float v)
{
    static_assert(MASK == 1 || MASK == 2, "exchange inside a quad");
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), MASK == 1 ? 0xB1 : 0x4E, 0xF, 0xF, false));   // quad_perm [1,0,3,2] / [2,3,0,1]
}

template <int LPB> __device__ __forceinline__ float group_max(float v)
{
    if (LPB >= 2) v = fmaxf(v, xor_lanes<1>(v));
    if (LPB >= 4) v = fmaxf(v, xor_lanes<2>(v));
    return v;
}
// balanced tree over the lanes of a block, in lane (= index) order; both partners compute the
// same rounded sum because addition commutes
template <int LPB> __device__ __forceinline__ float group_sum(float v)
{
    if (LPB >= 2) v = v + xor_lanes<1>(v);
    if (LPB >= 4) v = v + xor_lanes<2>(v);
    return v;
}

// wave-uniform switches of the row loop
struct Switches {
    int A;
    uint32_t pair_mask, flip_mask, gid, unit_tpos, unit_tneg, wide, mirror, selfsym, second;
};

// round a non-negative fp32 to the scale word: nearest, ties to the lower code, saturating
__device__ __forceinline__ int encode_scale(float sp, const KParams& p)
{
    const uint32_t u = __float_as_uint(sp);
    const int E = (int)(u >> 23);
    const int y = p.man_bits;
    // normal range of the target: rebias the exponent, round the 23-bit mantissa to y bits
    const uint32_t ut = u - ((uint32_t)(127 - p.bias) << 23);
    uint32_t q = (ut + ((1u << (22 - y)) - 1u)) >> (23 - y);
    const bool sub = E < 128 - p.bias;
    if (__any(sub)) {
        // subnormal range of the target (or zero): quantum 2^(1-bias-y)
        const int Ee = max(E, 1);
        const uint32_t m = (u & 0x7FFFFFu) | ((uint32_t)min(E, 1) << 23);
        int S = 151 - p.bias - y - Ee;
        S = S > 31 ? 31 : S;
        const uint32_t qs = S > 0 ? ((m + ((1u << (S - 1)) - 1u)) >> S) : 0u;
        q = sub ? qs : q;
    }
    return (int)(q > (uint32_t)p.max_code ? (uint32_t)p.max_code : q);
}

// TWICE value(q) * 2^-k (exact; the element passes multiply it with the halved codebook values of the table) and the
// IEEE reciprocal of value(q) * 2^-k (0 for the zero scale); the tabulated pair holds the doubled scale already
__device__ __forceinline__ void decode_scale(int q, const KParams& p, const float2* __restrict__ s_tab, float& s2, float& rinv)
{
    if (p.n_tab_codes) {
        const float2 t = s_tab[q];
        s2 = t.x;
        rinv = t.y;
    } else {
        const int y = p.man_bits;
        const int e = q >> y, f = q & ((1 << y) - 1);
        const float nrm = __uint_as_float(((uint32_t)(e - p.bias - p.k + 127) << 23) | ((uint32_t)f << (23 - y)));
        const float sub = (float)f * p.sub_quantum;
        const float s = e > 0 ? nrm : sub;
        s2 = s + s;
        rinv = s > 0.0f ? 1.0f / s : 0.0f;
    }
}

// ideal scale of a block against endpoints (tp, -tn); a unit endpoint needs no division
__device__ __forceinline__ float ideal_scale(float pmax, float nmax, float tp, float tn, bool unit_p, bool unit_n)
{
    float s1 = pmax, s2 = nmax;
    // the flags are wave-uniform; the empty asm statements keep these real branches (a division is a
    // dozen instructions, and the common codebooks have unit endpoints)
    if (!unit_p) { asm volatile(""); s1 = pmax / tp; }
    if (!unit_n) { asm volatile(""); s2 = nmax / tn; }
    return fmaxf(s1, s2);
}

// Scale of one (group, sign): code q, twice the signed scale in ss, scaled weights x and their bin offsets.
// boff receives the LDS byte address of each element's bin record (lds_neg = table address minus the
// product the 24-bit multiply adds for the constant's exponent bits).
// ARGMAX: the scale maps the block's largest-magnitude element onto the endpoint of larger magnitude
// and its sign follows from the two signs (per lane, returned in neg_out); otherwise the absmax rule
// for the sign given in `negative`.
// Scale of one (group, sign) without the scaled weights: code q, TWICE the signed scale in ss (the table holds half of
// every codebook value, see read_rec: 2s * L/2 is the product s * L), signed reciprocal rr, and whether the scaled
// weights may leave the bin table (see prepare_sign).
struct ScalePrep { int q; float ss, rr; bool nonzero, beyond; };
__device__ __forceinline__ ScalePrep prepare_scale(float pmax, float nmax, bool negative, int a, const KParams& p, const Switches& sw,
                                                   const float2* __restrict__ s_tab, const float4* __restrict__ s_gpar)
{
    const float4 gp = s_gpar[2 * a];                   // (t+, -t-, bin scale, bin offset): same address in every lane
    const float tp = gp.x, tn = gp.y;
    const bool unit_p = (sw.unit_tpos >> a) & 1u, unit_n = (sw.unit_tneg >> a) & 1u;
    const float sstar = negative ? ideal_scale(pmax, nmax, tn, tp, unit_n, unit_p) : ideal_scale(pmax, nmax, tp, tn, unit_p, unit_n);
    ScalePrep r;
    r.q = encode_scale(sstar * p.pow2k, p);
    float s2, rinv;
    decode_scale(r.q, p, s_tab, s2, rinv);
    r.ss = negative ? -s2 : s2;
    r.nonzero = s2 > 0.0f;
    r.rr = negative ? -rinv : rinv;
    r.beyond = !(sstar * rinv <= SOP_K_BIN_SAFE);
    return r;
}

template <int EPL, bool ARGMAX>
__device__ __forceinline__ void prepare_sign(const float (&w)[EPL], float pmax, float nmax, bool negative, int a,
                                             const KParams& p, const Switches& sw, const float2* __restrict__ s_tab,
                                             const float4* __restrict__ s_gpar, uint32_t lds_neg, uint32_t rec,
                                             int& q, float& ss, bool& nonzero, float (&x)[EPL], uint32_t (&boff)[EPL], bool& neg_out)
{
    const float4 gp = s_gpar[2 * a];                   // (t+, -t-, bin scale, bin offset): same address in every lane
    const float tp = gp.x, tn = gp.y;
    const bool unit_p = (sw.unit_tpos >> a) & 1u, unit_n = (sw.unit_tneg >> a) & 1u;
    float sstar;
    if constexpr (ARGMAX) {
        const bool x_pos = pmax >= nmax, t_pos = tp >= tn;          // ties: the positive element, the positive endpoint
        sstar = (x_pos ? pmax : nmax) / (t_pos ? tp : tn);
        negative = x_pos != t_pos;
    } else {
        sstar = negative ? ideal_scale(pmax, nmax, tn, tp, unit_n, unit_p) : ideal_scale(pmax, nmax, tp, tn, unit_p, unit_n);
    }
    neg_out = negative;
    q = encode_scale(sstar * p.pow2k, p);
    float s2, rinv;
    decode_scale(q, p, s_tab, s2, rinv);             // (twice the scale: the element passes multiply it with half of the codebook value)
    ss = negative ? -s2 : s2;
    nonzero = s2 > 0.0f;
    const float rr = negative ? -rinv : rinv;
    const float sc = gp.z, off = gp.w;
    // the table covers a scale rounded down by up to the factor SOP_K_BIN_SAFE; beyond it (the scale
    // word saturated) the whole wavefront clamps its scaled weights into the table's range
    // (the argmax rule lets elements pass the smaller endpoint by any factor: always clamp)
    const bool beyond = ARGMAX || !(sstar * rinv <= SOP_K_BIN_SAFE);
    if (__builtin_expect(ARGMAX || __any(beyond) != 0, ARGMAX ? 1 : 0)) {
        const float4 g2 = s_gpar[2 * a + 1];           // (table range low, high, -, -)
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            x[i] = w[i] * rr;
            const float xc = __builtin_amdgcn_fmed3f(x[i], g2.x, g2.y);
            boff[i] = __umul24(__float_as_uint(__fmaf_rn(xc, sc, off)), rec) + lds_neg;
        }
    } else {
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            x[i] = w[i] * rr;
            // off carries 1.5*2^23, so the low mantissa bits of the sum are the bin number; one 24-bit
            // multiply-add turns them into the byte offset of the bin record
            boff[i] = __umul24(__float_as_uint(__fmaf_rn(x[i], sc, off)), rec) + lds_neg;
        }
    }
}

// Where an element pass takes a scaled weight and the LDS address of its bin record from: arrays filled by
// prepare_sign (a scale group's atoms share them), or formed on the spot from the weight and the scale's reciprocal
// (signed scale words: the arrays of two signs would cost a wavefront per SIMD in registers, and with every atom
// evaluated under two scales there is little left to share).  Same arithmetic either way.
// WIDE: the records are those of kernels that write planes (SOP_K_WIDE_BIN_BYTES).
template <int EPL, bool WIDE_>
struct ArrSrc {
    static constexpr bool WIDE = WIDE_;
    const float (&x)[EPL];
    const uint32_t (&boff)[EPL];
    __device__ __forceinline__ void get(int i, float& xo, uint32_t& bo) const { xo = x[i]; bo = boff[i]; }
};
template <int EPL, bool CLAMP, bool WIDE_>
struct FlySrc {
    static constexpr bool WIDE = WIDE_;
    const float (&w)[EPL];
    float rr, sc, off, lo, hi;
    uint32_t lds_neg, rec;
    __device__ __forceinline__ void get(int i, float& xo, uint32_t& bo) const
    {
        xo = w[i] * rr;
        const float xc = CLAMP ? __builtin_amdgcn_fmed3f(xo, lo, hi) : xo;
        bo = __umul24(__float_as_uint(__fmaf_rn(xc, sc, off)), rec) + lds_neg;
    }
};

// Sums of one (atom, sign) candidate over the lane's elements, before the cross-lane tree.
struct Sums {
    float err;    // decision score of metrics WSE / MSE (and the blk_err output)
    float wd;     // RESIDUAL form: <w,d>_c;  DIRECT form: numerator sum
    float ew;     // RESIDUAL form with metric MSE: c-weighted ||d||^2;  DIRECT form: denominator sum
    float rn = 0.0f, rd = 0.0f; // RESIDUAL form with RANK: numerator and denominator sums of the ranking score (the DIRECT form's)
};

// One element's share of the ranking score's sums (chunks of 8 and the tree, as the DIRECT form)
template <int EPL>
struct RankSums {
    float n0 = 0.0f, n1 = 0.0f, d0 = 0.0f, d1 = 0.0f;
    __device__ __forceinline__ void add(int i, float w, float c, float ss, float yv)
    {
        const float what = ss * yv;
        const float cw = c * w, cwh = c * what;
        if (i < 8) { n0 = __fmaf_rn(cw, what, n0); d0 = __fmaf_rn(cwh, what, d0); }
        else       { n1 = __fmaf_rn(cw, what, n1); d1 = __fmaf_rn(cwh, what, d1); }
    }
    __device__ __forceinline__ float num() const { return EPL == 16 ? n0 + n1 : n0; }
    __device__ __forceinline__ float den() const { return EPL == 16 ? d0 + d1 : d0; }
};

// What an element pass reads of a bin record (BinRec): the halved values below and above the boundary, and the code below it when codes are wanted.
// `addr` is the LDS byte address of the record and A the atom's slot in it: all reads are register + immediate offset.
// The table holds HALF of each codebook value (exact: the host refuses entries whose half is not), and every
// element pass multiplies by twice the block scale, which is the same product.  What that buys: the boundary
// between two neighbouring entries, the binary64 mean rounded once to binary32, equals the binary32 sum of their
// halves (one rounding of the same real number; the host checks it entry by entry), so it is formed with one addition
// instead of being read.  In a bin without a boundary the upper value, and with it the sum, is +infinity: no scaled weight lies above it or on it.
// What bounds a pass is issue: a SIMD's four wavefronts get one instruction of any kind into about 2.4 cycles, and an LDS instruction takes
// as much as one to two vector ones whatever it reads (64 vector instructions 150 cycles, with eight 4-, 8- or 16-byte reads among them 175 to 187).  LDS itself
// serves two 4-byte reads (ds_read2_b32) of 64 lanes at random bins in 5.1 cycles, an 8-byte read in 2.9, a 16-byte one in 6.9.  So two atoms of one
// group are read together with 16 bytes, and one alone with 8 (4-byte fields at 132-byte records before: 96 look-ups a step of six atoms, now 64).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const f32x2 lds_f32x2;
typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;
// Kernels that write planes hold for every atom of a bin its two values, their sum and the code below: a pass that forms codes takes all four
// with one instruction.
struct Rec { float thr, ylo, yhi; int clo; };
template <bool WIDE> __device__ __forceinline__ f32x2 read_pair(uint32_t addr, int a) { return ((lds_f32x2*)(size_t)addr)[WIDE ? 2 * a : a]; }
// (lower, upper) of slots a and a + 1, a even
template <bool WIDE> __device__ __forceinline__ f32x4 read_two(uint32_t addr, int a)
{
    if constexpr (!WIDE) return ((lds_f32x4*)(size_t)addr)[a / 2];
    else { const f32x2 u = read_pair<WIDE>(addr, a), v = read_pair<WIDE>(addr, a + 1); return {u[0], u[1], v[0], v[1]}; }
}
template <bool WIDE, bool CODES>
__device__ __forceinline__ Rec read_rec(uint32_t addr, int a)
{
    static_assert(!CODES || WIDE, "codes are formed where planes are written");
    if constexpr (CODES) {
        const f32x4 v = ((lds_f32x4*)(size_t)addr)[a];
        return {v[2], v[0], v[1], __float_as_int(v[3])};
    } else {
        const f32x2 v = read_pair<WIDE>(addr, a);
        return {v[0] + v[1], v[0], v[1], 0};
    }
}

template <int EPL, bool CODES>
__device__ __forceinline__ void put_code(uint32_t (&codes)[EPL / 4], int i, uint32_t code, bool wide_codes)
{
    if (CODES) {
        if (wide_codes) codes[i / 4] |= code << (8 * (i % 4));
        else codes[i / 8] |= code << (4 * (i % 8));
    }
}

// Element pass, RESIDUAL form (metrics WSE and MSE): the cosine inputs come from the residual sums
//   <w,w^> = ||w||^2 - <w,d>,   ||w^||^2 = ||w||^2 - 2<w,d> + ||d||^2      (all c-weighted),
// which shares c*d with the error sum.  The form cancels when the reconstruction is much smaller
// than the block (saturated or vanished scale); the caller checks that and falls back to
// direct_cosine_sums() for the wavefront.
// TIES: `tie` collects, as a lane mask, the lanes that hold a scaled weight exactly on a code boundary (the one place
// where a codebook under the negative scale sign and its sign-negated copy under the positive sign part ways).  The
// comparison writes a scalar lane mask and the masks are joined on the scalar unit: one vector instruction per
// element.  (-0 and +0 compare equal, so a boundary at zero is seen from either side.)
template <int EPL, int METRIC, bool CODES, bool TIES = false, bool RANK = false, class SRC>
__device__ __forceinline__ Sums eval_residual(const float (&w)[EPL], const float (&cb)[EPL], const SRC& src, float ss, int a,
                                              bool wide_codes, uint32_t (&codes)[EPL / 4], unsigned long long* tie = nullptr)
{
    float e0 = 0.0f, e1 = 0.0f, wd = 0.0f, ew = 0.0f;
    RankSums<EPL> rk;
    if (CODES) {
#pragma unroll
        for (int j = 0; j < EPL / 4; ++j) codes[j] = 0;
    }
    // (look-ups in flight: two where the variant of 8-element lanes with most sums has no registers for four)
    constexpr int CH = EPL == 8 && CODES && RANK && METRIC == 2 ? 2 : 4;
#pragma unroll
    for (int i0 = 0; i0 < EPL; i0 += CH) {
        Rec r[CH];
        float xe[CH];
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            uint32_t bo;
            src.get(i0 + j, xe[j], bo);
            r[j] = read_rec<SRC::WIDE, CODES>(bo, a);
        }
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int i = i0 + j;
            const bool up = xe[j] > r[j].thr;
            if constexpr (TIES) *tie |= __builtin_amdgcn_ballot_w64(xe[j] == r[j].thr);
            const float yv = up ? r[j].yhi : r[j].ylo;
            const float d = __fmaf_rn(-ss, yv, w[i]);
            const float cd = cb[i] * d;
            const float dd = METRIC == 2 ? d : cd;
            if (i < 8) e0 = __fmaf_rn(dd, d, e0); else e1 = __fmaf_rn(dd, d, e1);
            wd = __fmaf_rn(cd, w[i], wd);
            if (METRIC == 2) ew = __fmaf_rn(cd, d, ew);
            if constexpr (RANK) rk.add(i, w[i], cb[i], ss, yv);
            put_code<EPL, CODES>(codes, i, (uint32_t)r[j].clo + (up ? 1u : 0u), wide_codes);
        }
        // (one chunk's look-ups in flight at a time where the pass keeps many sums: a register budget, not an order.  With codes beside the tie test as well: the
        // elements' lane masks would otherwise push a hundred constants of the row loop out of the scalar registers, 33 with the barrier)
        if constexpr (RANK) {
            asm volatile("" : "+v"(e0), "+v"(e1), "+v"(wd), "+v"(rk.n0), "+v"(rk.n1), "+v"(rk.d0), "+v"(rk.d1));
            if constexpr (METRIC == 2) asm volatile("" : "+v"(ew));
        }
        if constexpr (RANK || (CODES && TIES && EPL == 16)) __builtin_amdgcn_sched_barrier(0);
    }
    Sums s;
    s.err = EPL == 16 ? e0 + e1 : e0;
    s.wd = wd;
    s.ew = ew;
    if constexpr (RANK) { s.rn = rk.num(); s.rd = rk.den(); }
    return s;
}

// Element pass of N atoms of one scale group at once (slots a .. a+N-1): the scaled weight and its
// table address are formed once per element, used for every atom and dropped, so no array of either is ever held.  Same
// arithmetic, in the same order, as eval_residual (metrics WSE and MSE) or eval_direct (metric COS; ERR: with the error sum).  CODES: one
// atom (N = 1).
template <int EPL, int METRIC, int N, bool CODES, bool RANK, int KEEPCW, bool ERR, class SRC>
__device__ __forceinline__ void eval_residual_group(const float (&w)[EPL], const float (&cb)[EPL], const SRC& src, float ss, int a, Sums (&out)[N],
                                                    bool wide_codes, uint32_t (&codes)[EPL / 4])
{
    static_assert(N == 1 || !CODES, "codes are formed atom by atom");
    // Elements whose look-ups are in flight.  Atoms evaluated together ask for the next elements' look-ups before the ones at hand are used, at half as many
    // elements a set (same registers; 28672 x 8192, seven atoms 8 % of a search, a model's layers 2 %).  One atom alone does not: five atoms of fitted codebooks, 4096 x 11008,
    // 73.2 us against 75.1.
    constexpr bool AHEAD = METRIC != 1 && !SRC::WIDE && N > 1;
    constexpr int CH = AHEAD ? (N > 2 ? 1 : 2) : N > 2 || (N > 1 && RANK) ? 2 : 4;
    float e0[N], e1[N], wd[N], ew[N];
    RankSums<EPL> rk[N];
#pragma unroll
    for (int n = 0; n < N; ++n) e0[n] = e1[n] = wd[n] = ew[n] = 0.0f;
    if (CODES) {
#pragma unroll
        for (int j = 0; j < EPL / 4; ++j) codes[j] = 0;
    }
    f32x4 r4[AHEAD ? 2 : 1][(N + 1) / 2][CH];
    Rec r[N][CH];
    float xe[AHEAD ? 2 : 1][CH];
    auto ask = [&](int i0, int b) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            uint32_t bo;
            src.get(i0 + j, xe[b][j], bo);
            if constexpr (CODES) r[0][j] = read_rec<SRC::WIDE, true>(bo, a);
            else if constexpr (N == 1) { const f32x2 v = read_pair<SRC::WIDE>(bo, a); r4[b][0][j] = {v[0], v[1], 0.0f, 0.0f}; }
            else {
#pragma unroll
                for (int n = 0; n < N; n += 2) r4[b][n / 2][j] = read_two<SRC::WIDE>(bo, a + n);
            }
        }
    };
    if constexpr (AHEAD) ask(0, 0);
#pragma unroll
    for (int i0 = 0; i0 < EPL; i0 += CH) {
        const int b = AHEAD ? (i0 / CH) & 1 : 0;
        if constexpr (AHEAD) {
            if (i0 + CH < EPL) ask(i0 + CH, b ^ 1);
            __builtin_amdgcn_sched_barrier(0);
        } else ask(i0, 0);
        if constexpr (!CODES) {
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int j = 0; j < CH; ++j) {
                    const float lo = r4[b][n / 2][j][n % 2 * 2], hi = r4[b][n / 2][j][n % 2 * 2 + 1];
                    r[n][j] = {lo + hi, lo, hi, 0};
                }
        }
#pragma unroll
        for (int n = 0; n < N; ++n) {
#pragma unroll
            for (int j = 0; j < CH; ++j) {
                const int i = i0 + j;
                const bool up = xe[b][j] > r[n][j].thr;
                const float yv = up ? r[n][j].yhi : r[n][j].ylo;
                if constexpr (ERR) {
                    const float d = __fmaf_rn(-ss, yv, w[i]);
                    const float cd = cb[i] * d;
                    const float dd = METRIC == 2 ? d : cd;
                    if (i < 8) e0[n] = __fmaf_rn(dd, d, e0[n]); else e1[n] = __fmaf_rn(dd, d, e1[n]);
                    if (METRIC != 1) wd[n] = __fmaf_rn(cd, w[i], wd[n]);
                    if (METRIC == 2) ew[n] = __fmaf_rn(cd, d, ew[n]);
                }
                if constexpr (RANK || METRIC == 1) {
                    float wi = w[i];
                    if (i >= KEEPCW) asm volatile("" : "+v"(wi));             // (c w is formed again for every atom rather than kept: a register an element)
                    rk[n].add(i, wi, cb[i], ss, yv);
                }
                put_code<EPL, CODES>(codes, i, (uint32_t)r[n][j].clo + (up ? 1u : 0u), wide_codes);
            }
        }
        // one chunk's look-ups in flight at a time: four wavefronts per SIMD hide them, and more in flight would cost the fourth
#pragma unroll
        for (int n = 0; n < N; ++n) {
            if constexpr (ERR) asm volatile("" : "+v"(e0[n]), "+v"(e1[n]));
            if constexpr (METRIC != 1) asm volatile("" : "+v"(wd[n]));
            if constexpr (METRIC == 2) asm volatile("" : "+v"(ew[n]));
            if constexpr (RANK || METRIC == 1) asm volatile("" : "+v"(rk[n].n0), "+v"(rk[n].n1), "+v"(rk[n].d0), "+v"(rk[n].d1));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int n = 0; n < N; ++n) {
        if constexpr (METRIC == 1) { wd[n] = rk[n].num(); ew[n] = rk[n].den(); }
        out[n].err = EPL == 16 ? e0[n] + e1[n] : e0[n]; out[n].wd = wd[n]; out[n].ew = ew[n];
        if constexpr (RANK) { out[n].rn = rk[n].num(); out[n].rd = rk[n].den(); }
    }
}

// Element pass, DIRECT form with the decision sums of metric COS:
//   w^ = fl(ss*y), num = sum fma(fl(c*w), w^), den = sum fma(fl(c*w^), w^), chunks of 8 and the tree;
// err is formed as well when WANT_ERR (the blk_err output).
template <int EPL, bool CODES, bool WANT_ERR, bool TIES = false, class SRC>
__device__ __forceinline__ Sums eval_direct(const float (&w)[EPL], const float (&cb)[EPL], const SRC& src, float ss, int a,
                                            bool wide_codes, uint32_t (&codes)[EPL / 4], unsigned long long* tie = nullptr)
{
    float e0 = 0.0f, e1 = 0.0f, n0 = 0.0f, n1 = 0.0f, d0 = 0.0f, d1 = 0.0f;
    if (CODES) {
#pragma unroll
        for (int j = 0; j < EPL / 4; ++j) codes[j] = 0;
    }
#pragma unroll
    for (int i0 = 0; i0 < EPL; i0 += 4) {
        Rec r[4];
        float xe[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint32_t bo;
            src.get(i0 + j, xe[j], bo);
            r[j] = read_rec<SRC::WIDE, CODES>(bo, a);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = i0 + j;
            const bool up = xe[j] > r[j].thr;
            if constexpr (TIES) *tie |= __builtin_amdgcn_ballot_w64(xe[j] == r[j].thr);
            const float yv = up ? r[j].yhi : r[j].ylo;
            const float what = ss * yv;
            const float cw = cb[i] * w[i];
            const float cwh = cb[i] * what;
            if (i < 8) { n0 = __fmaf_rn(cw, what, n0); d0 = __fmaf_rn(cwh, what, d0); }
            else       { n1 = __fmaf_rn(cw, what, n1); d1 = __fmaf_rn(cwh, what, d1); }
            if (WANT_ERR) {
                const float d = __fmaf_rn(-ss, yv, w[i]);
                const float cd = cb[i] * d;
                if (i < 8) e0 = __fmaf_rn(cd, d, e0); else e1 = __fmaf_rn(cd, d, e1);
            }
            put_code<EPL, CODES>(codes, i, (uint32_t)r[j].clo + (up ? 1u : 0u), wide_codes);
        }
        // (a register budget, not an order: with the chunks apart the signed six-atom search keeps 139 registers, without 168 and up to 60 spilled;
        // every plane of eight atoms of 8-element lanes 162 to 167, without 168 and up to 12 spilled)
        if constexpr ((TIES && !CODES && EPL == 16) || (CODES && (EPL == 8 || !TIES))) asm volatile("" : "+v"(n0), "+v"(n1), "+v"(d0), "+v"(d1));
    }
    Sums s;
    s.err = EPL == 16 ? e0 + e1 : e0;
    s.wd = EPL == 16 ? n0 + n1 : n0;
    s.ew = EPL == 16 ? d0 + d1 : d0;
    return s;
}

// Cosine inputs straight from the codebook values in the scaled domain, where the block scale
// cancels: cos = sign(s) <w,y>_c / sqrt(||w||_c^2 ||y||_c^2).  Used when the residual form would cancel.
// (y is read as the table holds it, halved: the ratio does not change.)
// LEAN: the products c w of the block statistics are formed again rather than kept for it in registers, and four look-ups are in
// flight at a time.
template <int EPL, int LPB, bool LEAN, class SRC>
__device__ __forceinline__ void direct_cosine_sums(const float (&cb)[EPL], const float (&w)[EPL], const SRC& src, bool nonzero, bool negative,
                                                   int a, float& ny_out, float& dy_out)
{
    float ny = 0.0f, dy = 0.0f;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        float xe;
        uint32_t bo;
        src.get(i, xe, bo);
        const Rec r = read_rec<SRC::WIDE, false>(bo, a);
        const float yv = xe > r.thr ? r.yhi : r.ylo;
        float wi = w[i];
        if constexpr (LEAN) asm volatile("" : "+v"(wi));
        ny = __fmaf_rn(cb[i] * wi, yv, ny);
        dy = __fmaf_rn(cb[i], yv * yv, dy);
        if constexpr (LEAN) {
            if (i % 4 == 3) { asm volatile("" : "+v"(ny), "+v"(dy)); __builtin_amdgcn_sched_barrier(0); }
        }
    }
    const float nsum = group_sum<LPB>(negative ? -ny : ny), dsum = group_sum<LPB>(dy);
    ny_out = nonzero ? nsum : 0.0f;                    // a zero scale reconstructs nothing
    dy_out = nonzero ? dsum : 0.0f;
}

// Candidate after the cross-lane tree
struct Cand {
    float err;    // decision score of WSE / MSE; the weighted error in COS mode when wanted
    float ny;     // cosine numerator   (cos = ny / sqrt(||w||^2 dy))
    float dy;     // cosine denominator part
    bool weak;    // residual form not trustworthy for this block
};

// The cosine is a ratio of sums that all scale with the square of the block's magnitude; formed of the raw
// sums, the product ||w||^2 ||w^||^2 would leave binary32's range for blocks of very small or very large
// weights.  The value path therefore works on sums multiplied by a power of two, sc = 2^-e with
// ||w||_c^2 = m 2^e (exact, and the same bits as before wherever nothing over- or underflowed):
// wns = sc ||w||^2 lies in [1, 2), and the residual form yields sc <w,w^> and sc ||w^||^2 directly.
struct NormScale { float wns, qwns, sc, sc2; };      // sc ||w||^2, a quarter of it, sc, 2 sc

template <int LPB, int METRIC>
__device__ __forceinline__ Cand finish_residual(const Sums& s, const NormScale& n)
{
    Cand c;
    c.err = group_sum<LPB>(s.err);
    const float wd = group_sum<LPB>(s.wd);
    const float errw = METRIC == 2 ? group_sum<LPB>(s.ew) : c.err;
    c.ny = __fmaf_rn(-wd, n.sc, n.wns);
    c.dy = __fmaf_rn(errw, n.sc, __fmaf_rn(-n.sc2, wd, n.wns));
    c.weak = !(c.dy >= n.qwns);
    return c;
}

template <int LPB>
__device__ __forceinline__ Cand finish_direct(const Sums& s)
{
    Cand c;
    c.err = group_sum<LPB>(s.err);
    c.ny = group_sum<LPB>(s.wd);
    c.dy = group_sum<LPB>(s.ew);
    c.weak = false;
    return c;
}

// first / second atom of the pair with lexicographic position pi among all pairs of SOP_K_MAXA atoms
struct PairTab { int first[SOP_K_MAXP], second[SOP_K_MAXP]; };
constexpr PairTab make_pair_tab()
{
    PairTab t{};
    int pi = 0;
    for (int i = 0; i < SOP_K_MAXA; ++i)
        for (int j = i + 1; j < SOP_K_MAXA; ++j) { t.first[pi] = i; t.second[pi] = j; ++pi; }
    return t;
}
constexpr PairTab kPairTab = make_pair_tab();
template <int PI> struct PairOf { static constexpr int i = kPairTab.first[PI], j = kPairTab.second[PI]; };
template <int V> struct ic { constexpr operator int() const { return V; } };      // a compile-time integer as an argument

// Running sums of 1 - cos in units of 2^-22 (integers: exact, so their order does not matter): atoms, pairs, and the number of steps in which
// the lane's block had zero norm.
// IN_LDS: not in the lane's registers but in LDS (lane_sums_in_lds()), where the wavefronts that share a SIMD's steps add to one set of 64 words a column, each lane to the word of
// its number.  An add is one instruction either way.  Every wavefront empties its set after SOP_K_FLUSH_STEPS steps of its own, so a word never holds
// more than that many steps of each of four wavefronts: 240 of at most 2^23.
typedef __attribute__((address_space(3))) int lds_int;
template <bool IN_LDS, int NA>
struct LaneSums {
    static constexpr bool in_lds = IN_LDS;
    int a[IN_LDS ? 1 : SOP_K_MAXA], p[IN_LDS ? 1 : SOP_K_MAXP], z;
    uint32_t at;                                   // LDS byte address of the lane's word of column 0
    static __device__ __forceinline__ constexpr int pair_col(int pi) { return NA + kPairTab.first[pi] * (2 * NA - kPairTab.first[pi] - 1) / 2 + kPairTab.second[pi] - kPairTab.first[pi] - 1; }
    __device__ __forceinline__ void clear()
    {
        z = 0;
        if constexpr (!IN_LDS) {
#pragma unroll
            for (int i = 0; i < SOP_K_MAXA; ++i) a[i] = 0;
#pragma unroll
            for (int i = 0; i < SOP_K_MAXP; ++i) p[i] = 0;
        }
    }
    __device__ __forceinline__ lds_int* word(int col) const { return (lds_int*)(size_t)at + 64 * col; }
    __device__ __forceinline__ void add(int col, int v) const { __hip_atomic_fetch_add(word(col), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); }
    __device__ __forceinline__ void atom(int i, int v) { if constexpr (IN_LDS) add(i, v); else a[i] += v; }
    __device__ __forceinline__ void pair(int pi, int v) { if constexpr (IN_LDS) add(pair_col(pi), v); else p[pi] += v; }
};

// The pairs of a block by their errors' bit patterns, which order as the errors do where none is below zero or a NaN (else see numbered_pairs).  The selector is "b strictly
// better than a" for the caller's pair (a, b), and the internal order may have swapped the two, in which case internal j keeps the block on a tie:
// pick_j = error[j] < error[i] + swapped, the borrow of a subtraction with a carry.  A pair adds the chosen atom's deficit to its running sum and
// shifts its bit into `chain` by the carry of an addition; pair (i, j) ends at bit chain_bit(i, j).  Five instructions a pair and no test of
// whether it is requested, where the general form takes eleven (scalar instructions and branches cost about as much issue time as vector ones).  Pairs that are
// not requested are formed as well and go nowhere.  That costs a list of one pair (4096 x 4096, six atoms: unsigned 30.2 us either way, signed word 40.8 pair by pair
// and 43.1 in the chain, all fifteen 43.7 and 43.1), but a second form beside the chain for short lists made the chain's own step 1 % slower and gained one
// pair 1 to 2 %, and tests that leave out columns without a requested pair cost every other list 0.5 to 1 %.
// Up to three pairs (i, J) at once: a lane mask that a vector instruction writes may be read by another two instructions later at the earliest, which
// three subtractions in a row are.  (The compiler makes more of either carry.)   SOPK_FIELD: offset and width of the pair's bit in `flips`.
#define SOPK_FIELD(i, j) (pair_index(i, j) | 1 << 16)
template <int J, int I, class SUMS>
__device__ __forceinline__ void pairs_1(unsigned long long flips, const float (&score)[SOP_K_MAXA], const int (&dlt)[SOP_K_MAXA], SUMS& sums, uint32_t& chain)
{
    unsigned long long m0;
    int t0;
    asm("s_bfe_i64 %[m0], %[fl], %[f0]\n"
        "v_subb_co_u32 %[t0], %[m0], %[ej], %[e0], %[m0]\n s_nop 1\n"
        "v_cndmask_b32 %[t0], %[d0], %[dj], %[m0]\n"
        "v_addc_co_u32 %[ch], %[m0], %[ch], %[ch], %[m0]"
        : [m0] "=&s"(m0), [t0] "=&v"(t0), [ch] "+v"(chain)
        : [fl] "s"(flips), [ej] "v"(score[J]), [dj] "v"(dlt[J]), [e0] "v"(score[I]), [d0] "v"(dlt[I]), [f0] "n"(SOPK_FIELD(I, J)) : "scc");
    sums.pair(pair_index(I, J), t0);
}
// pairs (I, J) and (I - 1, J)
template <int J, int I, class SUMS>
__device__ __forceinline__ void pairs_2(unsigned long long flips, const float (&score)[SOP_K_MAXA], const int (&dlt)[SOP_K_MAXA], SUMS& sums, uint32_t& chain)
{
    unsigned long long m0, m1;
    int t0, t1;
    asm("s_bfe_i64 %[m0], %[fl], %[f0]\n s_bfe_i64 %[m1], %[fl], %[f1]\n"
        "v_subb_co_u32 %[t0], %[m0], %[ej], %[e0], %[m0]\n v_subb_co_u32 %[t1], %[m1], %[ej], %[e1], %[m1]\n s_nop 0\n"
        "v_cndmask_b32 %[t0], %[d0], %[dj], %[m0]\n v_cndmask_b32 %[t1], %[d1], %[dj], %[m1]\n"
        "v_addc_co_u32 %[ch], %[m0], %[ch], %[ch], %[m0]\n v_addc_co_u32 %[ch], %[m1], %[ch], %[ch], %[m1]"
        : [m0] "=&s"(m0), [m1] "=&s"(m1), [t0] "=&v"(t0), [t1] "=&v"(t1), [ch] "+v"(chain)
        : [fl] "s"(flips), [ej] "v"(score[J]), [dj] "v"(dlt[J]), [e0] "v"(score[I]), [e1] "v"(score[I - 1]), [d0] "v"(dlt[I]), [d1] "v"(dlt[I - 1]),
          [f0] "n"(SOPK_FIELD(I, J)), [f1] "n"(SOPK_FIELD(I - 1, J)) : "scc");
    sums.pair(pair_index(I, J), t0);
    sums.pair(pair_index(I - 1, J), t1);
}
// pairs (I, J), (I - 1, J) and (I - 2, J)
template <int J, int I, class SUMS>
__device__ __forceinline__ void pairs_3(unsigned long long flips, const float (&score)[SOP_K_MAXA], const int (&dlt)[SOP_K_MAXA], SUMS& sums, uint32_t& chain)
{
    unsigned long long m0, m1, m2;
    int t0, t1, t2;
    asm("s_bfe_i64 %[m0], %[fl], %[f0]\n s_bfe_i64 %[m1], %[fl], %[f1]\n s_bfe_i64 %[m2], %[fl], %[f2]\n"
        "v_subb_co_u32 %[t0], %[m0], %[ej], %[e0], %[m0]\n v_subb_co_u32 %[t1], %[m1], %[ej], %[e1], %[m1]\n v_subb_co_u32 %[t2], %[m2], %[ej], %[e2], %[m2]\n"
        "v_cndmask_b32 %[t0], %[d0], %[dj], %[m0]\n v_cndmask_b32 %[t1], %[d1], %[dj], %[m1]\n v_cndmask_b32 %[t2], %[d2], %[dj], %[m2]\n"
        "v_addc_co_u32 %[ch], %[m0], %[ch], %[ch], %[m0]\n v_addc_co_u32 %[ch], %[m1], %[ch], %[ch], %[m1]\n v_addc_co_u32 %[ch], %[m2], %[ch], %[ch], %[m2]"
        : [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [t0] "=&v"(t0), [t1] "=&v"(t1), [t2] "=&v"(t2), [ch] "+v"(chain)
        : [fl] "s"(flips), [ej] "v"(score[J]), [dj] "v"(dlt[J]), [e0] "v"(score[I]), [e1] "v"(score[I - 1]), [e2] "v"(score[I - 2]),
          [d0] "v"(dlt[I]), [d1] "v"(dlt[I - 1]), [d2] "v"(dlt[I - 2]), [f0] "n"(SOPK_FIELD(I, J)), [f1] "n"(SOPK_FIELD(I - 1, J)), [f2] "n"(SOPK_FIELD(I - 2, J)) : "scc");
    sums.pair(pair_index(I, J), t0);
    sums.pair(pair_index(I - 1, J), t1);
    sums.pair(pair_index(I - 2, J), t2);
}
#undef SOPK_FIELD
// pairs (N - 1, J) .. (0, J) in this order
template <int J, int N, class SUMS>
__device__ __forceinline__ void pair_column(unsigned long long flips, const float (&score)[SOP_K_MAXA], const int (&dlt)[SOP_K_MAXA], SUMS& sums, uint32_t& chain)
{
    constexpr int done = N == 1 ? 1 : (N == 2 || N == 4) ? 2 : 3;
    if constexpr (done == 1) pairs_1<J, N - 1>(flips, score, dlt, sums, chain);
    else if constexpr (done == 2) pairs_2<J, N - 1>(flips, score, dlt, sums, chain);
    else pairs_3<J, N - 1>(flips, score, dlt, sums, chain);
    if constexpr (N > done) pair_column<J, N - done>(flips, score, dlt, sums, chain);
}
template <int J, int NA, class SUMS>
__device__ __forceinline__ void ordered_pairs(int A, unsigned long long flips, const float (&score)[SOP_K_MAXA], const int (&dlt)[SOP_K_MAXA], SUMS& sums, uint32_t& chain)
{
    // (a variant unrolled for six serves three atoms or more, one for eight seven or more)
    if (J < (NA == 8 ? 7 : 3) || J < A) pair_column<J, J>(flips, score, dlt, sums, chain);
    if constexpr (J > 1) ordered_pairs<J - 1, NA>(A, flips, score, dlt, sums, chain);
}

// Pair PI and the following ones by the errors as numbers: what the chain took another way is put right.  (Errors below zero, which bit patterns order
// the other way round; a NaN is not less than anything nor anything less than it, and internal i keeps the block.)
template <int PI, int NA, class SUMS>
__device__ __forceinline__ void numbered_pairs(unsigned long long flips, const float (&score)[SOP_K_MAXA], const int (&dlt)[SOP_K_MAXA], SUMS& sums, uint32_t& chain)
{
    constexpr int i = PairOf<PI>::i, j = PairOf<PI>::j, c = chain_bit(i, j);
    if constexpr (j < NA) {
        const bool took_j = (chain >> c) & 1u, pick_j = score[j] < score[i] || (((flips >> PI) & 1u) && score[j] == score[i]);
        if (took_j != pick_j) {
            sums.pair(PI, pick_j ? dlt[j] - dlt[i] : dlt[i] - dlt[j]);
            chain ^= 1u << c;
        }
    }
    if constexpr (PI + 1 < SOP_K_MAXP) numbered_pairs<PI + 1, NA>(flips, score, dlt, sums, chain);
}

// Selector of pair PI and of all following pairs (i < j in internal order), for every metric and alphabet: bit `slot` of the
// block's selector word, and the chosen atom's deficit into the pair's running sum.
template <int PI, int NA, int METRIC, class SUMS>
__device__ __forceinline__ void all_pairs(const KParams& p, const Switches& sw, const float (&score)[SOP_K_MAXA],
                                          const float (&den)[SOP_K_MAXA], const int (&dlt)[SOP_K_MAXA],
                                          SUMS& sums, uint32_t& bits)
{
    constexpr int i = PairOf<PI>::i, j = PairOf<PI>::j;
    static_assert(pair_index(i, j) == PI, "pair enumeration");
    if constexpr (j < NA) {
        if (__builtin_expect((sw.pair_mask >> PI) & 1u, 1)) {
            // caller's pair (a,b): selector = "b strictly better than a" (ties keep a).  The internal
            // order may have swapped the two (b is internal i): then internal j keeps the block on a tie.
            const float si = score[i], sj = score[j], ni = den[i], nj = den[j];
            const int di = dlt[i], dj = dlt[j];
            const bool flip = (sw.flip_mask >> PI) & 1u;
            // both comparisons are formed as lane masks; the wave-uniform flag picks one of them in
            // scalar registers (no branch, no per-lane select of booleans)
            const float lhs = METRIC == 1 ? sj * ni : sj, rhs = METRIC == 1 ? si * nj : si;
            const unsigned long long lt = __builtin_amdgcn_ballot_w64(METRIC == 1 ? lhs > rhs : lhs < rhs);
            const unsigned long long le = __builtin_amdgcn_ballot_w64(METRIC == 1 ? lhs >= rhs : lhs <= rhs);
            const bool pick_j = __builtin_amdgcn_inverse_ballot_w64(flip ? le : lt);
            const int chosen = pick_j ? dj : di;
            sums.pair(PI, chosen);
            // bit = "internal j taken"; for swapped pairs the caller's selector is its complement, put
            // right by one xor with the mask of swapped pairs after the last pair
            const int slot = (p.pair_slot_w[PI / 4] >> (8 * (PI % 4))) & 0xFF;
            bits |= (pick_j ? 1u : 0u) << slot;
        }
    }
    if constexpr (PI + 1 < SOP_K_MAXP) all_pairs<PI + 1, NA, METRIC>(p, sw, score, den, dlt, sums, bits);
}

// The weights one lane reads per step, as they come from memory
template <bool BF16, int EPL> struct RawBlk { uint4 v[BF16 ? EPL / 8 : EPL / 4]; };

// Strip and row are the same in every lane: the address is a scalar base plus the lane's own 32-bit offset.  `lanes`: lanes
// of the strip that hold weights (64 but for the last strip of a row); the others lie past the end the load is given and read zeros.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
template <bool BF16, int EPL>
__device__ __forceinline__ RawBlk<BF16, EPL> load_raw(const void* W, long long ldw, unsigned int strip, unsigned int m, unsigned int lanes, unsigned int lane)
{
    RawBlk<BF16, EPL> r;
    constexpr int NV = BF16 ? EPL / 8 : EPL / 4;
    constexpr unsigned int esz = BF16 ? 2u : 4u;
    const char* row = reinterpret_cast<const char*>(W) + ((long long)m * ldw + (long long)strip * (64 * EPL)) * esz;
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(row), 0, (int)(lanes * (EPL * esz)), 0x00027000);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(rs, lane * (EPL * esz) + 16u * i, 0, 0);
        r.v[i] = make_uint4(t.x, t.y, t.z, t.w);
    }
    return r;
}

template <bool BF16, int EPL>
__device__ __forceinline__ void widen(const RawBlk<BF16, EPL>& r, float (&w)[EPL])
{
    if (BF16) {
#pragma unroll
        for (int i = 0; i < EPL / 8; ++i) {
            const uint32_t v[4] = {r.v[i].x, r.v[i].y, r.v[i].z, r.v[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w[8 * i + 2 * j] = __uint_as_float(v[j] << 16);
                w[8 * i + 2 * j + 1] = __uint_as_float(v[j] & 0xFFFF0000u);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < EPL / 4; ++i) {
            w[4 * i] = __uint_as_float(r.v[i].x); w[4 * i + 1] = __uint_as_float(r.v[i].y);
            w[4 * i + 2] = __uint_as_float(r.v[i].z); w[4 * i + 3] = __uint_as_float(r.v[i].w);
        }
    }
}

// Ranking score of step 2 of the per-layer search: a decision quantity, formed in binary32 from the block's tree sums
// num = <w,w^>_c, den = ||w^||_c^2 (chunks of 8, balanced tree) and wn = ||w||_c^2:
// fl(fl(num / wn) * fl(|num| / den)), 1 for a block without weighted norm, 0 for a zero reconstruction
__device__ __forceinline__ float rank_score(float num, float dn, float wn)
{
    return wn > 0.0f ? (dn > 0.0f ? (num / wn) * (fabsf(num) / dn) : 0.0f) : 1.0f;
}

// the codes of the lane's elements into the atom's plane (two codes per byte, or one for atoms of more than 16 entries)
template <int EPL>
__device__ __forceinline__ void store_codes(const KParams& p, const Switches& sw, int a, long long row, long long col0, const uint32_t (&codes)[EPL / 4])
{
    if (!((sw.wide >> a) & 1u)) {
        uint8_t* dst = p.codes + p.code_off[a] + (row * p.K + col0) / 2;
#pragma unroll
        for (int j = 0; j < EPL / 8; ++j) reinterpret_cast<uint32_t*>(dst)[j] = codes[j];
    } else {
        uint8_t* dst = p.codes + p.code_off[a] + row * p.K + col0;
#pragma unroll
        for (int j = 0; j < EPL / 4; ++j) reinterpret_cast<uint32_t*>(dst)[j] = codes[j];
    }
}

// NA: atoms the kernel is unrolled for (2, 6 or 8).  OCC: wavefronts per SIMD the register budget is set
// for; a workgroup is 4*OCC wavefronts and fills one compute unit on its own (one copy of the tables in
// LDS per compute unit, one addition per output and compute unit in the layer reduction).
// MULTI: one launch works through a list of layers (model-wide call).  The workgroups stay, the tables are
// loaded once, and every share's steps of all the layers form one sequence with one counter: a wavefront
// passes from a layer to the next without waiting for anyone, adding what it holds to the finished layer's
// sums in LDS on the way (one set of sums per layer of the launch); a ticket and the conversion to ACos happen
// once, at the end of the launch, for all its layers.
// SIGNMODE 0: the scale is positive; 1: both signs of the scale are tried and the better one kept
// (signed scale word, absmax rule); 2: argmax rule, the rule fixes the sign.
template <bool BF16, int EPL, int LPB, int SIGNMODE, int METRIC, bool EMIT, int NA, int OCC, bool MULTI>
__global__ __launch_bounds__(256 * OCC, 1) void search_kernel(const KParams p)
{
    static_assert(!MULTI || !EMIT, "the model-wide kernel searches only");
    constexpr bool SIGNED = SIGNMODE == 1, ARGMAX = SIGNMODE == 2;
    // atoms of a scale group are evaluated four or two at a time.  (Not for the planes of more than two atoms under the cosine metric, whose sums
    // leave two wavefronts either way: 4096 x 11008, six atoms, every plane, 182 us atom by atom, 217 in groups)
    constexpr bool GROUPED = SIGNMODE == 0 && EPL == 16 && (METRIC != 1 || !EMIT || NA == 2);
    // the direct cosine sums outside the grouped passes: in the form that keeps registers low for the variants that are short of them
    // (the others have some left, and the form's scheduling fences cost the signed eight-atom search a sixth: 4096 x 4096, 77 us
    // -> 92; the signed one-atom search with every plane, g = 32, takes 33.4 us with it and 35.0 without)
    constexpr bool LSUM = lane_sums_in_lds(BF16, EPL, SIGNMODE, METRIC, EMIT, NA, MULTI);
    constexpr bool LEAN = NA == 6 || (NA == 2 && EMIT);
    // ranking sums in a pass of their own where eight atoms of 8-element lanes leave no registers for them in the one element pass (up to
    // 17 spilled; argmax rule, metric MSE, fp32, 4096 x 4096, every plane: 157 us in one pass, 127 in two)
    constexpr bool SPLIT_RANK = EMIT && EPL == 8 && NA == 8;
    constexpr bool TOP_TEST = EMIT || (NA == 2 && SIGNMODE == 0 && EPL == 16);       // the row loop's test at its top (see there)
    // wavefronts per SIMD, threads of the workgroup (a launch of short shares may have one wavefront less than the variant is built for, see search_waves())
    const int waves = !MULTI && OCC == 4 && p.deal ? (int)p.deal : OCC, NT = 256 * waves;
    extern __shared__ __align__(16) char s_mem[];
    // LDS: selector bits | bin table | (scale, reciprocal) table | group parameters | reduction scratch
    constexpr int NPERM = search_perm_tables(NA, METRIC == 1);                      // (a comparison of cosines is one of products: no chain)
    constexpr bool ORDERED = NPERM != 0;
    uint32_t* const s_perm = reinterpret_cast<uint32_t*>(s_mem);                  // [NPERM][256] selector bits of eight bits of a chain of pairs
    char* const s_bins = s_mem + NPERM * 1024;                                    // [n_bins] records
    const uint32_t rec = EMIT ? SOP_K_WIDE_BIN_BYTES(NA) : p.rec_bytes;
    const size_t bins_bytes = (size_t)p.n_bins * rec;
    float2* s_tab = reinterpret_cast<float2*>(s_bins + bins_bytes);
    float4* s_gpar = reinterpret_cast<float4*>(s_bins + bins_bytes + (((size_t)p.n_tab_codes * sizeof(float2) + 15) & ~(size_t)15));
    // reduction scratch: flag word (MULTI), list of outputs (not MULTI), the workgroup's own totals (64-bit integers)
    unsigned long long* s_red = reinterpret_cast<unsigned long long*>(s_gpar + 2 * SOP_K_MAXA);
    unsigned int* s_out = reinterpret_cast<unsigned int*>(s_red + 1);             // (not MULTI) output: its sum column, and from bit 8 its place in the table
    constexpr int NLIVE = search_cols(NA), NSLOT = search_slots(NA);              // sum columns of this variant: atoms, pairs, count column
    unsigned long long* s_acc = s_red + 1 + SOP_K_OUT_WORDS;                     // [NSLOT] this workgroup's sums (MULTI: per layer)
    const int n_acc = MULTI ? p.n_layers * NSLOT : NSLOT;
    __shared__ unsigned int s_next[4];                                            // next step of each SIMD's share
    const uint32_t lds_neg = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)s_bins + SOP_K_BIN_NEGC(rec);

    const int lane = threadIdx.x & 63;
    // the wavefront's number is the same in all its lanes: saying so keeps the row loop's counters
    // and tests in scalar registers
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // The workgroup's range of steps is cut into four equal shares, one per SIMD.  The hardware deals the
    // wavefronts of a workgroup out to the four SIMDs in turn, so wavefronts w, w+4, w+8, ... share a SIMD
    // (as measured on this GPU) and work on share w mod 4; were they dealt out
    // otherwise, only the balance would suffer: every share has wavefronts of its own.  The wavefronts of
    // a share take its steps one at a time from a counter in LDS: the hardware favours the oldest
    // wavefront of a SIMD, and with fixed parts the younger ones would run on alone, at a fraction of the
    // SIMD's rate, for a fifth of the kernel.  Which wavefront takes which step does not change any
    // result: all sums are integers.
    const int simd = wv & 3;
    // the share's range of the steps of a layer of uq * gridDim.x + ur (rest ur below gridDim.x, which is below 2^10)
    auto share_of = [&](unsigned int uq, unsigned int ur, unsigned int& first, unsigned int& count) {
        const unsigned int b = blockIdx.x, g0 = uq * b + __umulhi(ur * b, p.grid_magic), g1 = uq * (b + 1u) + __umulhi(ur * (b + 1u), p.grid_magic);
        first = g0 + (g1 - g0) * (unsigned int)simd / 4u;
        count = g0 + (g1 - g0) * (unsigned int)(simd + 1) / 4u - first;
    };
    // Request side (the row loads run one step ahead of the arithmetic): the layer the next requested step
    // lies in.  One layer: sb, cnt are the share's range.  MULTI: the shares of all layers follow one another
    // in one sequence of step numbers; rq_base is the number of the first step of layer rq_l in it.
    unsigned int sb, cnt;
    int rq_l = 0;
    unsigned int rq_base = 0u, rq_M32 = 0u, rq_magic = 0u;
    const void* rq_W = nullptr;
    long long rq_ldw = 0, rq_K = 0;
    // (everything here is the same in all lanes; saying so keeps it in scalar registers)
    auto uni = [](unsigned int x) { return (unsigned int)__builtin_amdgcn_readfirstlane((int)x); };
    auto uni64 = [&](unsigned long long x) { return ((unsigned long long)uni((unsigned int)(x >> 32)) << 32) | uni((unsigned int)x); };
    auto rq_enter = [&](int l) {
        const LayerDesc& d = p.layers[l];
        share_of(uni(d.units_q), uni(d.units_r), sb, cnt);
        rq_W = reinterpret_cast<const void*>(uni64((unsigned long long)reinterpret_cast<uintptr_t>(d.W)));
        rq_ldw = (long long)uni64((unsigned long long)d.ldw);
        rq_K = (long long)uni((unsigned int)d.K);
        rq_M32 = uni(d.M32); rq_magic = uni(d.m_magic);
    };
    if constexpr (MULTI) rq_enter(0);
    else share_of(p.units_q, p.units_r, sb, cnt);   // (the layer's own values are read from the kernel arguments where used)
    // is step v of the sequence there?  (MULTI: moves the request side on to its layer; v never decreases)
    auto seek = [&](unsigned int v) -> bool {
        if constexpr (!MULTI) return v < cnt;
        else {
            if (rq_l >= p.n_layers) return false;
            while (v - rq_base >= cnt) {
                rq_base += cnt;
                if (++rq_l >= p.n_layers) return false;
                rq_enter(rq_l);
            }
            return true;
        }
    };
    auto grab = [&]() -> unsigned int {
        unsigned int v = 0u;
        if (lane == 0) v = atomicAdd(&s_next[simd], 1u);
        return (unsigned int)__builtin_amdgcn_readfirstlane((int)v);
    };
    // lanes of a strip that hold weights (row length K, below 2^31 * 64 * EPL as there are fewer than 2^31 strip rows)
    auto lanes_of = [&](unsigned int st, long long K) -> unsigned int {
        const unsigned int full = (unsigned int)((unsigned long long)K / (64u * EPL));
        return st < full ? 64u : (unsigned int)((unsigned long long)K % (64u * EPL)) / EPL;
    };
    // step number -> (strip, row): steps run down the rows of a strip; division by multiplication with
    // floor(2^32 / M), one correction (scalar arithmetic)
    auto locate = [&](unsigned int u, unsigned int& st, unsigned int& row) {
        const unsigned int magic = MULTI ? rq_magic : p.m_magic, rows = MULTI ? rq_M32 : p.M32;
        unsigned int q = __umulhi(u, magic);
        unsigned int r = u - q * rows;
        if (r >= rows) { ++q; r -= rows; }
        st = q; row = r;
    };

    LaneSums<LSUM, NA> sums;
    sums.clear();
    if constexpr (LSUM) sums.at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(char*)(s_acc + NSLOT + 1) + (uint32_t)((simd * NSLOT * 64 + lane) * 4);
    // Lane sums of every column, exact.  Four columns at a time: exchanges of half and quarter wavefronts (gfx950's lane swaps)
    // leave one column's sums over four lanes in each row of 16 lanes, the row is added up with data-parallel-primitive moves
    // (quads, half rows, rows: every lane of the row then holds the column's sum), and the first lane of each row adds it to
    // the workgroup's 64-bit sum in LDS: one add of four lanes to four different words for four columns.  (Rows summed for every
    // column on its own, four lanes to one word: 88 moves and 22 adds for six atoms against 66 and 6, and the adds of four lanes to
    // one word are served one after the other, with every wavefront's.)
    // Range: a step adds at most 2^23 to a lane, so SOP_K_FLUSH_STEPS = 60 steps of four lanes stay below 2^31; the sum is split
    // at bit 15 and both halves are added over the row (below 2^19 and 2^20), then joined in 64 bits.  A lane's sum can be a few units below
    // zero: all of it is signed.
    // (This translation unit is compiled with the compiler's atomic optimizer off: it would turn each of these adds into a
    // loop over the active lanes.)
    auto row_sum = [](int x) -> int {
        x += __builtin_amdgcn_update_dpp(0, x, 0xB1, 0xF, 0xF, false);      // quad_perm [1,0,3,2]
        x += __builtin_amdgcn_update_dpp(0, x, 0x4E, 0xF, 0xF, false);      // quad_perm [2,3,0,1]
        x += __builtin_amdgcn_update_dpp(0, x, 0x141, 0xF, 0xF, false);     // row_half_mirror
        x += __builtin_amdgcn_update_dpp(0, x, 0x140, 0xF, 0xF, false);     // row_mirror
        return x;
    };
    // a's sums of lanes l and l + 32 in the lower half, b's in the upper half; the same with rows 0, 1 and 2, 3
    auto fold_halves = [](int a, int b) -> int { const auto t = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false); return (int)(t[0] + t[1]); };
    auto fold_rows = [](int a, int b) -> int { const auto t = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false); return (int)(t[0] + t[1]); };
    int cl = MULTI ? -1 : 0;                       // the layer the arithmetic is in
    // (LSUM: four columns' words, of any size, cut at bit 15 before the folds: below 2^18 for four words each)
    auto join = [&](const int (&lo)[4], const int (&hi)[4], unsigned long long* dst, int fl) {
        const int rl = row_sum(fold_rows(fold_halves(lo[0], lo[2]), fold_halves(lo[1], lo[3])));
        const int rh = row_sum(fold_rows(fold_halves(hi[0], hi[2]), fold_halves(hi[1], hi[3])));
        if ((fl & 15) == 0) atomicAdd(dst, (unsigned long long)(((long long)rh << 15) + (long long)rl));
    };
    auto flush = [&](int layer) {
        int fl = lane;
        asm volatile("" : "+v"(fl));                 // (the address is formed here, not kept in a register through the row loop)
        unsigned long long* dst = s_acc + (MULTI ? layer * NSLOT : 0) + (fl >> 4);
        int val[NSLOT], n = 0;                       // the live columns of this variant (compile-time list)
        if constexpr (LSUM) {
            // (what the other wavefronts of the SIMD added goes along)
            sums.add(NLIVE - 1, sums.z << 22); sums.z = 0;
#pragma unroll
            for (int j = 0; j < NSLOT; j += 4) {
                int lo[4], hi[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) { hi[i] = __hip_atomic_exchange(sums.word(j + i), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); lo[i] = hi[i] & 0x7FFF; hi[i] >>= 15; }
                join(lo, hi, dst + j, fl);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < NA; ++i) { val[n++] = sums.a[i]; sums.a[i] = 0; }
#pragma unroll
        for (int i = 0; i < SOP_K_MAXP; ++i)
            if (kPairTab.second[i] < NA) { val[n++] = sums.p[i]; sums.p[i] = 0; }
        val[n++] = sums.z << 22; sums.z = 0;
#pragma unroll
        for (int i = NLIVE; i < NSLOT; ++i) val[i] = 0;
#pragma unroll
        for (int j = 0; j < NSLOT; j += 4) {
            // (row r of the result holds column j + r)
            const int t = fold_rows(fold_halves(val[j], val[j + 2]), fold_halves(val[j + 1], val[j + 3]));
            const int rl = row_sum(t & 0x7FFF), rh = row_sum(t >> 15);
            if ((fl & 15) == 0) atomicAdd(dst + j, (unsigned long long)(((long long)rh << 15) + (long long)rl));
        }
    };
    // what the arithmetic needs of its layer
    const float* lc_c = nullptr;
    void* lc_sel = nullptr;
    long long lc_K = 0, lc_Bk = 0;
    unsigned int lc_Kc = 1u;

    unsigned int strip = 0u, m = 0u;
    unsigned int cur_strip = 0xFFFFFFFFu;
    float cb[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) cb[i] = 0.0f;
    // channel norms of the lane's columns (rows may have been folded, see KParams::Kc: the channel of a column is its index modulo the true
    // row length; hidden from the compiler, which would keep the division's reciprocal in a vector register through the loop)
    auto load_norms = [&](const float* c, unsigned int kc, unsigned int col0, bool valid) {
        asm volatile("" : "+s"(kc));
        const unsigned int ch0 = col0 % kc;
#pragma unroll
        for (int i = 0; i < EPL; i += 4) {
            const float4 t = valid ? *reinterpret_cast<const float4*>(c + ch0 + i) : make_float4(0.f, 0.f, 0.f, 0.f);
            cb[i] = t.x; cb[i + 1] = t.y; cb[i + 2] = t.z; cb[i + 3] = t.w;
        }
    };
    // metric WSE: a norm below zero, which the interface rules out, may take errors below zero
    unsigned int norms_below = 0u;                 // wave-uniform
    auto look_at_norms = [&]() {
        if constexpr (METRIC == 0 && ORDERED) {
            float least = 0.0f;
#pragma unroll
            for (int i = 0; i < EPL; ++i) least = fminf(least, cb[i]);
            norms_below = uni(__any(least < 0.0f) != 0);
        }
    };
    // (norms are waited for where they are asked for, not at their first use, which lies behind the request of the next row)
    auto norms_here = [&]() {
#pragma unroll
        for (int i = 0; i < EPL; ++i) asm volatile("" : "+v"(cb[i]));
    };
    // Where they are dealt out, the first step of each wavefront is its own and the others come from the counter (all from the counter, the first
    // two steps of a share went to its first wavefront, one after the other, while the others had none: six atoms, 1536 steps, 16.4 us
    // -> 13.6), and its row and channel norms are asked for ahead of everything else.  For which launches: search_deal().  The model-wide kernel takes every step
    // from the counter: wavefronts that start in step stay in step, and use the units by turns less well (six model layers of 2048 x 2048: 57 us ->
    // 59 with the first steps dealt out).
    const bool dealt = !MULTI && p.deal;
    unsigned int i_cur = 0u;
    RawBlk<BF16, EPL> nxt;
    bool ok_cur = false;
    auto first_row = [&]() {
        ok_cur = seek(i_cur);
        if (ok_cur) { locate(sb + (i_cur - rq_base), strip, m); nxt = load_raw<BF16, EPL>(MULTI ? rq_W : p.W, MULTI ? rq_ldw : p.ldw, strip, m, lanes_of(strip, MULTI ? rq_K : p.K), (unsigned int)lane); }
    };
    if (dealt) {
        i_cur = (unsigned int)wv >> 2;
        first_row();
        if (ok_cur) {
            cur_strip = strip;
            load_norms(p.c, (unsigned int)p.Kc, (strip * 64u + (unsigned int)lane) * EPL, (unsigned int)lane < lanes_of(strip, p.K));
        }
    }
    // Tables into LDS: the first words of the bin table, of the scale table and the group parameters are all asked for before the first of them is waited
    // for; a loop of one load, wait, one write would spend a round trip to L2 per word.  (A table has an even number of bins: whole 16-byte words.)
    {
        const int n16 = EMIT ? 0 : p.n_bins * (int)p.rec_bytes / 16, nt = p.n_tab_codes, tid = (int)threadIdx.x;
        const uint4* src = reinterpret_cast<const uint4*>(p.bins);
        uint4* dst = reinterpret_cast<uint4*>(s_bins);
        constexpr int NB = MULTI ? 1 : 2, NS = NB;      // words of the bin table and of the scale table in the first round
        uint4 t[NB];
        float2 u[NS];
        float4 gp = make_float4(0.f, 0.f, 0.f, 0.f);
        // planes: two atoms of a bin a thread, of the atoms that the variant is unrolled for; their values, the sums and the codes
        const int n_two = EMIT ? p.n_bins * (NA / 2) : 0;
        f32x4 two_v = {0.0f, 0.0f, 0.0f, 0.0f};
        uint32_t two_c = 0u;
        auto ask_two = [&](int i, f32x4& v, uint32_t& cd) {
            const int q = i % (NA / 2);
            const BinRec& r = *reinterpret_cast<const BinRec*>(p.bins + (size_t)(i / (NA / 2)) * p.rec_bytes);
            const float2 v0 = *reinterpret_cast<const float2*>(r.val[2 * q]), v1 = *reinterpret_cast<const float2*>(r.val[2 * q + 1]);
            v = {v0.x, v0.y, v1.x, v1.y};
            cd = *reinterpret_cast<const uint16_t*>(&r.code_lo[2 * q]);
        };
        auto put_two = [&](int i, const f32x4& v, uint32_t cd) {
            f32x4* const to = reinterpret_cast<f32x4*>(s_bins + (i / (NA / 2)) * rec) + 2 * (i % (NA / 2));
            to[0] = f32x4{v[0], v[1], v[0] + v[1], __int_as_float((int)(cd & 0xFFu))};
            to[1] = f32x4{v[2], v[3], v[2] + v[3], __int_as_float((int)(cd >> 8))};
        };
        if constexpr (EMIT) ask_two(min(tid, n_two - 1), two_v, two_c);
        // (a uniform test skips what is not there; indices past the end read the last word again)
#pragma unroll
        for (int j = 0; j < NB; ++j) { t[j] = make_uint4(0, 0, 0, 0); if (j * NT < n16) t[j] = src[min(tid + j * NT, n16 - 1)]; }
#pragma unroll
        for (int j = 0; j < NS; ++j) { u[j] = make_float2(0.f, 0.f); if (j * NT < nt) u[j] = p.stab[min(tid + j * NT, nt - 1)]; }
        if (tid < 2 * SOP_K_MAXA) gp = reinterpret_cast<const float4*>(p.gpar)[tid];
        if (!MULTI && tid < p.A + p.P) s_out[tid] = tid < p.A ? (unsigned)tid | (unsigned)p.uidx[tid] << 8 : (unsigned)p.pair_col[tid - p.A] | (unsigned)(tid - p.A) << 8;
        // (256 threads a table; a word of selector bits for every bit of the chain comes from the host, and an entry takes those of its set bits: two instructions a
        // bit.  With the words formed here, pair by pair, by the first 256 threads, this was 0.3 us of every launch of six atoms and 1.0 us of eight.)
        if constexpr (ORDERED) {
            if (MULTI || p.sel_words) {
                for (int k = wv >> 2; k < NPERM; k += waves) {
                    uint32_t v = 0u;
#pragma unroll
                    for (int i = 0; i < 8; ++i) v |= (uint32_t)__builtin_amdgcn_sbfe(tid, i, 1) & p.chain_sel[8 * k + i];
                    s_perm[256 * k + (tid & 255)] = k == 0 ? v ^ p.flip_slots : v;
                }
            }
        }
        if (tid < 4) s_next[tid] = dealt ? (unsigned int)waves : 0u;
        for (int i = tid; i < n_acc; i += NT) s_acc[i] = 0ull;
        if constexpr (LSUM) {
            static_assert((2 + SOP_K_OUT_WORDS + NSLOT) % 2 == 0, "16-byte words");
            for (int i = tid; i < 4 * NSLOT * 16; i += NT) reinterpret_cast<uint4*>(s_acc + NSLOT + 1)[i] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) if (tid + j * NT < n16) dst[tid + j * NT] = t[j];
#pragma unroll
        for (int j = 0; j < NS; ++j) if (tid + j * NT < nt) s_tab[tid + j * NT] = u[j];
        if (tid < 2 * SOP_K_MAXA) s_gpar[tid] = gp;
        if constexpr (EMIT) {
            if (tid < n_two) put_two(tid, two_v, two_c);
            for (int i0 = tid + NT; i0 < n_two; i0 += 4 * NT) {
                f32x4 v[4];
                uint32_t cd[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) ask_two(min(i0 + j * NT, n_two - 1), v[j], cd[j]);
#pragma unroll
                for (int j = 0; j < 4; ++j) if (i0 + j * NT < n_two) put_two(i0 + j * NT, v[j], cd[j]);
            }
        }
        for (int i0 = tid + NB * NT; i0 < n16; i0 += 4 * NT) {
            uint4 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = src[min(i0 + j * NT, n16 - 1)];
#pragma unroll
            for (int j = 0; j < 4; ++j) if (i0 + j * NT < n16) dst[i0 + j * NT] = v[j];
        }
        for (int i0 = tid + NS * NT; i0 < nt; i0 += 2 * NT) {
            float2 v[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) v[j] = p.stab[min(i0 + j * NT, nt - 1)];
#pragma unroll
            for (int j = 0; j < 2; ++j) if (i0 + j * NT < nt) s_tab[i0 + j * NT] = v[j];
        }
    }
    __syncthreads();
    if (!dealt) { i_cur = grab(); }
    unsigned int i_nxt = grab();
    if (!dealt) first_row();
    int l_nxt = rq_l;                              // layer of the row in nxt
    int since_flush = 0;
    if constexpr (TOP_TEST) look_at_norms();
    // The first row is waited for here: at the top of the loop the wait is then that of a step, whose row is older than its stores, which stay in
    // flight.  The loop stands in the same branch: a way round the wait into the loop, which nothing ever takes, would make every step's wait one for the
    // stores of the step before as well (two atoms under the argmax rule, lanes of eight bf16 weights: 1 to 3 %).  Where that way is joined with the loop's own
    // test at its top by itself, and with planes, whose stores have branches of their own, the test stays there: positive scale, 2048 x 5504, one atom 11.9 us
    // against 12.2, planes of two atoms under a signed word 2 to 4 %.
    if (TOP_TEST || ok_cur) {
    if (!TOP_TEST || ok_cur) {
#pragma unroll
        for (int i = 0; i < (int)(sizeof(nxt.v) / sizeof(nxt.v[0])); ++i) asm volatile("" : "+v"(nxt.v[i].x), "+v"(nxt.v[i].y), "+v"(nxt.v[i].z), "+v"(nxt.v[i].w));
        norms_here();
    }
    if constexpr (!TOP_TEST) look_at_norms();
    while (!TOP_TEST || ok_cur) {
        if constexpr (MULTI) {
            if (l_nxt != cl) {
                // the arithmetic enters another layer: its channel norms are requested first, and while they
                // travel the sums the lanes hold, which belong to the layer left, join that layer's
                const int left = cl;
                cl = l_nxt;
                const LayerDesc& d = p.layers[cl];
                lc_c = reinterpret_cast<const float*>(uni64((unsigned long long)reinterpret_cast<uintptr_t>(d.c)));
                lc_sel = reinterpret_cast<void*>(uni64((unsigned long long)reinterpret_cast<uintptr_t>(d.sel_words)));
                lc_K = (long long)uni((unsigned int)d.K); lc_Bk = (long long)uni((unsigned int)d.Bk);
                lc_Kc = uni((unsigned int)d.Kc);
                cur_strip = strip;
                load_norms(lc_c, lc_Kc, (strip * 64u + (unsigned int)lane) * EPL, (unsigned int)lane < lanes_of(strip, lc_K));
                if (left >= 0) flush(left);
                norms_here();
                look_at_norms();
                since_flush = 0;
            }
        }
        // The uniform switches below are re-read every row.  Left loop-invariant, each test would be
        // hoisted out of the loop as a 64-bit lane mask and the hundred-odd masks would spill.
        Switches sw = {p.A, p.pair_mask, p.flip_mask, p.gid_w, p.unit_tpos, p.unit_tneg, p.wide_mask, p.mirror_mask, p.selfsym_mask, p.second_mask};
        asm volatile("" : "+s"(sw.A), "+s"(sw.pair_mask), "+s"(sw.flip_mask), "+s"(sw.gid), "+s"(sw.unit_tpos), "+s"(sw.unit_tneg), "+s"(sw.wide));
        if constexpr (SIGNED) asm volatile("" : "+s"(sw.mirror), "+s"(sw.selfsym));
        if constexpr (GROUPED) asm volatile("" : "+s"(sw.second));
        unsigned long long flips = p.flip_mask;
        if constexpr (ORDERED) asm volatile("" : "+s"(flips));
        const unsigned int cm32 = m, cs = strip;
        const long long cm = cm32;
        const unsigned int lanes_here = lanes_of(cs, MULTI ? lc_K : p.K);
        const bool valid = (unsigned int)lane < lanes_here;
        if (cs != cur_strip) {
            cur_strip = cs;
            load_norms(MULTI ? lc_c : p.c, MULTI ? lc_Kc : (unsigned int)p.Kc, (cs * 64u + (unsigned int)lane) * EPL, valid);
            norms_here();
            look_at_norms();
        }
        // ---- the block: one read from HBM, requested one step ahead ----
        float w[EPL];
        widen<BF16, EPL>(nxt, w);
        // (widened before the next row is asked for: its registers take that row)
#pragma unroll
        for (int i = 0; i < EPL; ++i) asm volatile("" : "+v"(w[i]));
        const bool ok_nxt = seek(i_nxt);
        l_nxt = rq_l;
        // (after the last step the first row of the layer the request side is in is read and not used: a load on every path
        // leaves the rows in place, where a conditional one costs a copy of them per step.  That layer can be a later one, with
        // fewer rows than the one at hand, when the share has no steps in it: the position at hand may lie outside it.)
        if (ok_nxt) locate(sb + (i_nxt - rq_base), strip, m);
        else { strip = 0u; m = 0u; }
        nxt = load_raw<BF16, EPL>(MULTI ? rq_W : p.W, MULTI ? rq_ldw : p.ldw, strip, m, lanes_of(strip, MULTI ? rq_K : p.K), (unsigned int)lane);
        // the next step opens another layer: its channel norms are asked for now (one word per lane brings
        // every cache line of the strip's norms in), so that the loads at the top of that step find them
        // near; the value is only held until the end of this step
        float c_touch = 0.0f;
        if constexpr (MULTI) {
            if (ok_nxt && l_nxt != cl) {
                const float* cn = reinterpret_cast<const float*>(uni64((unsigned long long)reinterpret_cast<uintptr_t>(p.layers[l_nxt].c)));
                if ((unsigned int)lane < lanes_of(strip, rq_K)) c_touch = cn[(strip * 64u + (unsigned int)lane) * EPL % uni((unsigned int)p.layers[l_nxt].Kc)];
            }
        }
        const unsigned int i_nn = grab();              // the step after the next one; used at the end of this step

        // ---- block statistics ----
        float pmax = 0.0f, nmin = 0.0f, wn0 = 0.0f, wn1 = 0.0f;
#pragma unroll
        for (int i = 0; i < EPL; i += 2) {
            pmax = fmaxf(fmaxf(pmax, w[i]), w[i + 1]);
            nmin = fminf(fminf(nmin, w[i]), w[i + 1]);
        }
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const float cw = cb[i] * w[i];
            if (i < 8) wn0 = __fmaf_rn(cw, w[i], wn0); else wn1 = __fmaf_rn(cw, w[i], wn1);
        }
        pmax = group_max<LPB>(pmax);
        float nmax = group_max<LPB>(-nmin);
        // Lanes past the end of a row hold zero weights.  Their scale would be zero, which sends the whole
        // wavefront through the scale word's subnormal branch on every row of the last strip; a unit
        // maximum keeps them on the common path.  Nothing of theirs is written, and with zero weights they
        // still add exactly 1 to every sum and to the count column, as a zero block does.
        pmax = valid ? pmax : 1.0f;
        nmax = valid ? nmax : 1.0f;
        const float wn = group_sum<LPB>(EPL == 16 ? wn0 + wn1 : wn0);
        sums.z += wn > 0.0f ? 0 : 1;
        // power of two that brings ||w||^2 into [1, 2) (exponent fields 1 .. 253: norms within 2^-126 .. 2^126)
        NormScale nsc;
        {
            const uint32_t eb = min(max(__float_as_uint(wn) >> 23, 1u), 253u);
            nsc.sc = __uint_as_float((254u - eb) << 23);
            nsc.sc2 = nsc.sc + nsc.sc;
            nsc.wns = wn * nsc.sc;
            nsc.qwns = 0.25f * nsc.wns;
        }

        const long long blk0 = cm * (MULTI ? lc_Bk : p.Bk) + (long long)cs * (64 / LPB), blk = blk0 + (unsigned int)lane / LPB;    // (the step's first block; the lane's)
        const bool leader = valid && lane % LPB == 0;

        // per-block results of every atom that the pair stage needs: score = err (WSE / MSE) or
        // q = num*|num| (COS, 0 for a zero reconstruction), den (COS only, 1 for a zero reconstruction), 1 - cos
        float score[SOP_K_MAXA], den[SOP_K_MAXA];
        int dlt[SOP_K_MAXA];
        // state of the current scale group: scale code, scale, scaled weights and the addresses of their bin records.
        // A signed scale word keeps the scale of both signs instead and forms scaled weights and addresses inside the
        // element pass (FlySrc): the arrays of two signs would cost 64 registers and with them a wavefront per SIMD.
        // wave-uniform: an error may be below zero (then so is a norm) or a NaN (then no lane trusts the residual form of its atom)
        unsigned int odd = norms_below;
        int gq = 0;
        float gss = 0.0f;                              // twice the scale (the table holds halved codebook values)
        bool gnz = false, gneg = false;
        constexpr bool FLY = GROUPED || (SIGNED && EPL == 16);       // (a lane of 8 elements has the registers for both signs' arrays)
        float gx[FLY ? 1 : EPL], gx2[(SIGNED && !FLY) ? EPL : 1];
        uint32_t gboff[FLY ? 1 : EPL], gboff2[(SIGNED && !FLY) ? EPL : 1];
        ScalePrep spP = {0, 0.0f, 0.0f, false, false}, spM = {0, 0.0f, 0.0f, false, false};
        int cur_gid = -1;                              // scale group the state above belongs to (wave-uniform)
        // Signed scale word: the two candidates of the atom before (0: positive scale sign, 1: negative), kept for an
        // atom that is its sign-negated copy.  Codebook -a under the positive sign reconstructs what a does under the
        // negative sign, and the other way round (same scale code, same residuals bit for bit, codes k <-> N-1-k),
        // unless a scaled weight lies exactly on a code boundary: there the two resolve the tie differently.  So
        // the copy takes over the kept candidates with their roles exchanged (the wave-uniform flag f0neg: candidate
        // 0 is the negative sign), unless some lane of the wavefront saw such a tie, in which case the copy is
        // evaluated like any other atom.
        // (plain scalars: copying candidate structs would drag their padding bytes through scratch memory)
        float pv_err0 = 0.0f, pv_ny0 = 0.0f, pv_dy0 = 0.0f, pv_err1 = 0.0f, pv_ny1 = 0.0f, pv_dy1 = 0.0f;
        float pv_rn0 = 0.0f, pv_rd0 = 0.0f, pv_rn1 = 0.0f, pv_rd1 = 0.0f;   // sums of the ranking score (emit mode)
        int pv_q0 = 0, pv_q1 = 0;
        uint32_t pv_codes0[EPL / 4], pv_codes1[EPL / 4];
        bool pv_f0neg = false;                         // wave-uniform: the kept candidate 0 is the negative sign (it was kept by a copy)
        bool pv_tie = true;                            // wave-uniform: the kept candidates may not be taken over
        bool pv_raw0 = false, pv_raw1 = false;         // wave-uniform: the kept cosine sums are the direct ones (not scaled)

        if constexpr (GROUPED) {
            uint32_t weak_atoms = 0u;                  // wave-uniform: atoms whose residual form some lane does not trust
            ScalePrep sp = {0, 0.0f, 0.0f, false, false};
            uint32_t codes[EPL / 4];
            const bool want_rank = EMIT && p.blk_rank, want_codes = EMIT && p.codes;      // wave-uniform
            // the atom's share of the outputs: decision score, deficit 1 - cos in units of 2^-22 (see below), planes
            auto settle = [&](int a, const Sums& s, bool have_codes) __attribute__((always_inline)) {
                Cand t;
                float ny_raw = 0.0f, dy_raw = 0.0f;
                if constexpr (METRIC == 1) {
                    t = finish_direct<LPB>(s);
                    score[a] = t.dy > 0.0f ? t.ny * fabsf(t.ny) : 0.0f;
                    den[a] = t.dy > 0.0f ? t.dy : 1.0f;
                    ny_raw = t.ny; dy_raw = t.dy;
                    t.ny *= nsc.sc; t.dy *= nsc.sc;    // (the decision sums are raw: brought to the scaled norm's units)
                } else {
                    t = finish_residual<LPB, METRIC>(s, nsc);
                    score[a] = t.err; den[a] = 1.0f;
                }
                const float rs = __frsqrt_rn(__fmaf_rn(nsc.wns, t.dy, 1.0e-37f));
                dlt[a] = (int)__float_as_uint(__fmaf_rn(-t.ny, rs, 3.0f)) - 0x40000000;
                sums.atom(a, dlt[a]);
                if (__builtin_expect(__any(t.weak) != 0, 0)) weak_atoms |= 1u << a;
                if constexpr (EMIT) {
                    const long long ua = p.uidx[a];
                    if (have_codes && valid) store_codes<EPL>(p, sw, a, cm, (long long)(cs * 64u + (unsigned int)lane) * EPL, codes);
                    if (want_rank) {
                        const float r = METRIC == 1 ? rank_score(ny_raw, dy_raw, wn) : rank_score(group_sum<LPB>(s.rn), group_sum<LPB>(s.rd), wn);
                        if (leader) p.blk_rank[ua * p.Nb + blk] = r;
                    }
                    if (p.scale_code && leader) p.scale_code[ua * p.Nb + blk] = (uint16_t)sp.q;
                    if (p.blk_cos && leader) p.blk_cos[ua * p.Nb + blk] = wn > 0.0f ? 1.0f - __fmaf_rn(-t.ny, rs, 1.0f) : 1.0f;
                    if (p.blk_err && leader) p.blk_err[ua * p.Nb + blk] = t.err;
                }
            };
            auto scale_of = [&](int a) __attribute__((always_inline)) {
                const int gid = (int)((sw.gid >> (4 * a)) & 15u);
                if (gid != cur_gid) { cur_gid = gid; sp = prepare_scale(pmax, nmax, false, a, p, sw, s_tab, s_gpar); }
            };
            // N atoms of the current scale group (CL: scaled weights clamped into the table's range, CD: codes, RK: ranking sums)
            auto pass = [&](auto n_, auto cl_, auto cd_, auto rk_, int a) __attribute__((always_inline)) {
                constexpr int N = n_;
                constexpr bool CL = cl_, CD = cd_, RK = rk_;
                // (planes of six atoms: the forms of a pass stay apart; with their equal beginnings joined, as the compiler does, registers are spilled.  Planes of two
                // have the registers and are faster joined, 4096 x 11008 67 us against 76)
                if constexpr (EMIT && NA == 6) asm volatile("; %0" :: "n"(8 * N + 4 * CL + 2 * CD + RK));
                const float4 gpar = s_gpar[2 * a];
                float lo = 0.0f, hi = 0.0f;
                if (CL) { const float4 g2 = s_gpar[2 * a + 1]; lo = g2.x; hi = g2.y; }
                // Products c w of the statistics kept for the passes with ranking or direct cosine sums: all of them where two atoms leave registers for them; fp32
                // planes of two atoms have room for ten, with metric MSE for eight (up to five registers spilled with more; formed again for every atom, with none
                // kept: 4096 x 11008, every plane, 83.5 us, with ten 78.5; bf16 65.6 with all).
                constexpr int keep_cw = NA != 2 ? 0 : BF16 || !EMIT || METRIC == 1 ? EPL : METRIC == 2 ? 8 : 10;
                Sums sn[N];
                eval_residual_group<EPL, METRIC, N, CD, RK && METRIC != 1, keep_cw, METRIC != 1 || EMIT>(w, cb, FlySrc<EPL, CL, EMIT>{w, sp.rr, gpar.z, gpar.w, lo, hi, lds_neg, rec}, sp.ss, a, sn, EMIT && ((sw.wide >> a) & 1u), codes);
#pragma unroll
                for (int n = 0; n < N; ++n) settle(a + n, sn[n], CD && want_codes);
            };
            // one atom on its own
            auto one = [&](int a) __attribute__((always_inline)) {
                scale_of(a);
                // the table covers a scale rounded down by up to the factor SOP_K_BIN_SAFE; beyond it (the scale word
                // saturated) the whole wavefront clamps its scaled weights into the table's range
                if (__builtin_expect(__any(sp.beyond) != 0, 0)) pass(ic<1>(), ic<1>(), ic<EMIT>(), ic<EMIT>(), a);
                else if constexpr (!EMIT) pass(ic<1>(), ic<0>(), ic<0>(), ic<0>(), a);
                else if (want_codes) { if (want_rank) pass(ic<1>(), ic<0>(), ic<1>(), ic<1>(), a); else pass(ic<1>(), ic<0>(), ic<1>(), ic<0>(), a); }
                else if (want_rank) pass(ic<1>(), ic<0>(), ic<0>(), ic<1>(), a);
                else pass(ic<1>(), ic<0>(), ic<0>(), ic<0>(), a);
            };
            // two atoms: together when they are of one group (and no codes are wanted), else one after the other
            auto two = [&](auto a_) __attribute__((always_inline)) {
                constexpr int a = a_;
                score[a] = score[a + 1] = 0.0f; den[a] = den[a + 1] = 1.0f; dlt[a] = dlt[a + 1] = 0;
                if (__builtin_expect(a < sw.A, 1)) {
                    bool joint = ((sw.second >> (a + 1)) & 1u) && !want_codes;
                    if (joint) {
                        scale_of(a);
                        joint = __any(sp.beyond) == 0;
                    }
                    if (joint) {
                        if constexpr (!EMIT) pass(ic<2>(), ic<0>(), ic<0>(), ic<0>(), a);
                        else if (want_rank) pass(ic<2>(), ic<0>(), ic<0>(), ic<1>(), a);
                        else pass(ic<2>(), ic<0>(), ic<0>(), ic<0>(), a);
                    } else {
                        one(a);
                        if (a + 1 < sw.A) one(a + 1);
                    }
                }
            };
            // four atoms: together when they are of one group (the bit of the third one) and no planes are wanted
            auto four = [&](auto a_) __attribute__((always_inline)) {
                constexpr int a = a_;
                bool joint = !EMIT && ((sw.second >> (a + 2)) & 1u);
                if (joint) {
                    scale_of(a);
                    joint = __any(sp.beyond) == 0;
                }
                if (joint) pass(ic<4>(), ic<0>(), ic<0>(), ic<0>(), a);
                else { two(ic<a>()); two(ic<a + 2>()); }
            };
            if constexpr (NA == 2) two(ic<0>());
            else {
                four(ic<0>());
                if constexpr (NA == 6) two(ic<4>()); else four(ic<4>());
            }
            // the residual form is accurate while the reconstruction carries a fair share of the block's norm; otherwise
            // the whole wavefront recomputes the atom's cosine directly
            odd |= weak_atoms;
            while (__builtin_expect(weak_atoms != 0u, 0)) {
                const int wa = __builtin_ctz(weak_atoms);
                weak_atoms &= weak_atoms - 1u;
                const ScalePrep sq = prepare_scale(pmax, nmax, false, wa, p, sw, s_tab, s_gpar);
                const float4 gpar = s_gpar[2 * wa], g2 = s_gpar[2 * wa + 1];
                float ny1, dy1;
                direct_cosine_sums<EPL, LPB, true>(cb, w, FlySrc<EPL, true, EMIT>{w, sq.rr, gpar.z, gpar.w, g2.x, g2.y, lds_neg, rec}, sq.nonzero, false, wa, ny1, dy1);
                // (direct sums go with the raw norm, which is the scaled one times the inverse power of two, exactly)
                float sc = nsc.sc;
                asm volatile("" : "+v"(sc));               // (else the exponent that it was formed of is kept in a register for this)
                const float wnr = nsc.wns * __uint_as_float((254u << 23) - __float_as_uint(sc));
                const float rs = __frsqrt_rn(__fmaf_rn(wnr, dy1, 1.0e-37f));
                const int ia = (int)__float_as_uint(__fmaf_rn(-ny1, rs, 3.0f)) - 0x40000000;
#pragma unroll
                for (int a = 0; a < NA; ++a)
                    if (a == wa) { sums.atom(a, ia - dlt[a]); dlt[a] = ia; }
                if constexpr (EMIT) {
                    if (p.blk_cos && leader) p.blk_cos[(long long)p.uidx[wa] * p.Nb + blk] = wnr > 0.0f ? 1.0f - __fmaf_rn(-ny1, rs, 1.0f) : 1.0f;
                }
            }
        } else {
#pragma unroll
        for (int a = 0; a < NA; ++a) {
            score[a] = 0.0f; den[a] = 1.0f; dlt[a] = 0;
            if (__builtin_expect(a < sw.A, 1)) {
                bool derived = false;
                if constexpr (SIGNED) derived = ((sw.mirror >> a) & 1u) && !pv_tie;
                const int gid = (int)((sw.gid >> (4 * a)) & 15u);
                if (!derived && gid != cur_gid) {
                    cur_gid = gid;
                    if constexpr (FLY) {
                        spP = prepare_scale(pmax, nmax, false, a, p, sw, s_tab, s_gpar);
                        spM = prepare_scale(pmax, nmax, true, a, p, sw, s_tab, s_gpar);
                    } else if constexpr (SIGNED) {
                        bool unused;
                        prepare_sign<EPL, false>(w, pmax, nmax, false, a, p, sw, s_tab, s_gpar, lds_neg, rec, spP.q, spP.ss, spP.nonzero, gx, gboff, unused);
                        prepare_sign<EPL, false>(w, pmax, nmax, true, a, p, sw, s_tab, s_gpar, lds_neg, rec, spM.q, spM.ss, spM.nonzero, gx2, gboff2, unused);
                    } else {
                        prepare_sign<EPL, ARGMAX>(w, pmax, nmax, false, a, p, sw, s_tab, s_gpar, lds_neg, rec, gq, gss, gnz, gx, gboff, gneg);
                    }
                }
                const bool wide = EMIT && ((sw.wide >> a) & 1u);
                uint32_t codes[EPL / 4];
                Cand best;
                int q = gq;
                bool neg = ARGMAX ? gneg : false;
                bool raw = false;                      // best.ny, best.dy are raw sums (else multiplied by nsc.sc); per lane for signed words
                float rk_num = 0.0f, rk_dn = 0.0f;     // sums of the ranking score of the chosen sign (signed words, emit mode)
                if constexpr (SIGNED) {
                    // ---- both signs of the scale: candidate 0 (the positive sign; the negative one when f0neg) and candidate 1 ----
                    float err0, ny0, dy0, err1, ny1, dy1, rn0 = 0.0f, rd0 = 0.0f, rn1 = 0.0f, rd1 = 0.0f;
                    int q0, q1;
                    bool raw0, raw1, f0neg;
                    uint32_t codes0[EPL / 4], codes1[EPL / 4];
                    // codes of the mirrored codebook: N-1-k in every field (no borrows: every field holds at most N-1)
                    const uint32_t cmask = (uint32_t)(p.nent[a] - 1) * (wide ? 0x01010101u : 0x11111111u);
                    if (derived) {
                        err0 = pv_err0; ny0 = pv_ny0; dy0 = pv_dy0; err1 = pv_err1; ny1 = pv_ny1; dy1 = pv_dy1;
                        rn0 = pv_rn0; rd0 = pv_rd0; rn1 = pv_rn1; rd1 = pv_rd1;
                        q0 = pv_q0; q1 = pv_q1; raw0 = pv_raw0; raw1 = pv_raw1;
                        f0neg = !pv_f0neg;                 // what was the original's negative sign is the copy's positive one
                        if (EMIT) {
#pragma unroll
                            for (int j = 0; j < EPL / 4; ++j) { codes0[j] = cmask - pv_codes0[j]; codes1[j] = cmask - pv_codes1[j]; }
                        }
                    } else {
                        unsigned long long tie = 0ull;          // lanes that saw a scaled weight exactly on a code boundary
                        f0neg = false;
                        // one sign of the scale: the atom's element pass with scaled weights formed on the spot
                        const float4 gpar = s_gpar[2 * a];             // (t+, -t-, bin scale, bin offset): same address in every lane
                        auto eval_sign = [&](const ScalePrep& sp, const bool sgn, const auto& xarr, const auto& barr,
                                             float& err, float& ny, float& dy, int& qq, bool& rawf,
                                             uint32_t (&cds)[EPL / 4], float& rn, float& rd) {
                            qq = sp.q;
                            auto run = [&](const auto& src) {
                                Cand t;
                                if constexpr (METRIC == 1) t = finish_direct<LPB>(eval_direct<EPL, EMIT, EMIT, true>(w, cb, src, sp.ss, a, wide, cds, &tie));
                                else {
                                    // (the ranking score's sums, where wanted, are formed in the same pass)
                                    Sums s;
                                    if (EMIT && p.blk_rank) {
                                        s = eval_residual<EPL, METRIC, EMIT, true, EMIT>(w, cb, src, sp.ss, a, wide, cds, &tie);
                                        rn = group_sum<LPB>(s.rn); rd = group_sum<LPB>(s.rd);
                                    } else s = eval_residual<EPL, METRIC, EMIT, true>(w, cb, src, sp.ss, a, wide, cds, &tie);
                                    t = finish_residual<LPB, METRIC>(s, nsc);
                                }
                                err = t.err; ny = t.ny; dy = t.dy;
                                rawf = METRIC == 1;
                                if constexpr (METRIC != 1) {
                                    // the residual form is accurate while the reconstruction carries a fair share of the block's
                                    // norm; otherwise the whole wavefront recomputes this candidate's cosine sums directly
                                    if (__builtin_expect(__any(t.weak) != 0, 0)) {
                                        direct_cosine_sums<EPL, LPB, LEAN>(cb, w, src, sp.nonzero, sgn, a, ny, dy);
                                        rawf = true;
                                        odd = 1u;
                                    }
                                }
                                if constexpr (EMIT && METRIC == 1) { rn = t.ny; rd = t.dy; }
                            };
                            // the table covers a scale rounded down by up to the factor SOP_K_BIN_SAFE; beyond it (the scale word
                            // saturated) the whole wavefront clamps its scaled weights into the table's range
                            if constexpr (!FLY) {
                                run(ArrSrc<EPL, EMIT>{xarr, barr});
                            } else if (__builtin_expect(__any(sp.beyond) != 0, 0)) {
                                const float4 g2 = s_gpar[2 * a + 1];       // (table range low, high, -, -)
                                run(FlySrc<EPL, true, EMIT>{w, sp.rr, gpar.z, gpar.w, g2.x, g2.y, lds_neg, rec});
                            } else {
                                run(FlySrc<EPL, false, EMIT>{w, sp.rr, gpar.z, gpar.w, 0.0f, 0.0f, lds_neg, rec});
                            }
                        };
                        eval_sign(spP, false, gx, gboff, err0, ny0, dy0, q0, raw0, codes0, rn0, rd0);
                        // a codebook that is its own sign-negated copy reconstructs the same under both signs (away
                        // from ties), and an equal candidate never replaces the positive sign
                        if (((sw.selfsym >> a) & 1u) && (tie & __builtin_amdgcn_ballot_w64(valid)) == 0ull) {
                            err1 = err0; ny1 = ny0; dy1 = dy0; q1 = spM.q; raw1 = raw0; rn1 = rn0; rd1 = rd0;
                            if (EMIT) {
#pragma unroll
                                for (int j = 0; j < EPL / 4; ++j) codes1[j] = cmask - codes0[j];
                            }
                        } else {
                            eval_sign(spM, true, gx2, gboff2, err1, ny1, dy1, q1, raw1, codes1, rn1, rd1);
                        }
                        pv_tie = (tie & __builtin_amdgcn_ballot_w64(valid)) != 0ull;
                    }
                    pv_err0 = err0; pv_ny0 = ny0; pv_dy0 = dy0; pv_err1 = err1; pv_ny1 = ny1; pv_dy1 = dy1;
                    pv_q0 = q0; pv_q1 = q1; pv_raw0 = raw0; pv_raw1 = raw1; pv_f0neg = f0neg;
                    if (EMIT) {
                        pv_rn0 = rn0; pv_rd0 = rd0; pv_rn1 = rn1; pv_rd1 = rd1;
#pragma unroll
                        for (int j = 0; j < EPL / 4; ++j) { pv_codes0[j] = codes0[j]; pv_codes1[j] = codes1[j]; }
                    }
                    // the negative sign only when strictly better: candidate 1 is taken when it is strictly better, or, if it
                    // is the positive sign (f0neg), when it is at least as good.  Both comparisons are formed as lane masks
                    // and the wave-uniform flag picks one of them in scalar registers.
                    bool pick1;
                    if constexpr (METRIC == 1) {
                        const float bq0 = dy0 > 0.0f ? ny0 * fabsf(ny0) : 0.0f, bd0 = dy0 > 0.0f ? dy0 : 1.0f;
                        const float bq1 = dy1 > 0.0f ? ny1 * fabsf(ny1) : 0.0f, bd1 = dy1 > 0.0f ? dy1 : 1.0f;
                        const unsigned long long gt = __builtin_amdgcn_ballot_w64(bq1 * bd0 > bq0 * bd1);
                        const unsigned long long ge = __builtin_amdgcn_ballot_w64(!(bq0 * bd1 > bq1 * bd0));
                        pick1 = __builtin_amdgcn_inverse_ballot_w64(f0neg ? ge : gt);
                        score[a] = pick1 ? bq1 : bq0;
                        den[a] = pick1 ? bd1 : bd0;
                    } else {
                        const unsigned long long lt = __builtin_amdgcn_ballot_w64(err1 < err0);
                        const unsigned long long le = __builtin_amdgcn_ballot_w64(!(err0 < err1));
                        pick1 = __builtin_amdgcn_inverse_ballot_w64(f0neg ? le : lt);
                        score[a] = pick1 ? err1 : err0;
                    }
                    neg = pick1 != f0neg;
                    best.err = pick1 ? err1 : err0;
                    best.ny = pick1 ? ny1 : ny0;
                    best.dy = pick1 ? dy1 : dy0;
                    best.weak = false;
                    raw = pick1 ? raw1 : raw0;
                    q = pick1 ? q1 : q0;
                    if (EMIT) {
                        rk_num = pick1 ? rn1 : rn0; rk_dn = pick1 ? rd1 : rd0;
#pragma unroll
                        for (int j = 0; j < EPL / 4; ++j) codes[j] = pick1 ? codes1[j] : codes0[j];
                    }
                } else if constexpr (METRIC == 1) {
                    // (emit mode without a code plane, as when only the ranking scores are wanted: the pass that forms no codes)
                    if (!EMIT || p.codes) best = finish_direct<LPB>(eval_direct<EPL, EMIT, EMIT>(w, cb, ArrSrc<EPL, EMIT>{gx, gboff}, gss, a, wide, codes));
                    else best = finish_direct<LPB>(eval_direct<EPL, false, EMIT>(w, cb, ArrSrc<EPL, EMIT>{gx, gboff}, gss, a, wide, codes));
                    score[a] = best.dy > 0.0f ? best.ny * fabsf(best.ny) : 0.0f;
                    den[a] = best.dy > 0.0f ? best.dy : 1.0f;
                    raw = true;
                } else {
                    // (emit mode without a code plane, as when only the ranking scores are wanted: the pass that forms no codes; the ranking score's sums are formed in the same pass)
                    const ArrSrc<EPL, EMIT> src{gx, gboff};
                    Sums s;
                    if constexpr (!EMIT) s = eval_residual<EPL, METRIC, false>(w, cb, src, gss, a, wide, codes);
                    else if constexpr (SPLIT_RANK) {
                        if (p.codes) s = eval_residual<EPL, METRIC, true>(w, cb, src, gss, a, wide, codes);
                        else s = eval_residual<EPL, METRIC, false>(w, cb, src, gss, a, wide, codes);
                    }
                    else if (p.codes) s = p.blk_rank ? eval_residual<EPL, METRIC, true, false, true>(w, cb, src, gss, a, wide, codes) : eval_residual<EPL, METRIC, true>(w, cb, src, gss, a, wide, codes);
                    else s = p.blk_rank ? eval_residual<EPL, METRIC, false, false, true>(w, cb, src, gss, a, wide, codes) : eval_residual<EPL, METRIC, false>(w, cb, src, gss, a, wide, codes);
                    best = finish_residual<LPB, METRIC>(s, nsc);
                    if constexpr (SPLIT_RANK) {
                        if (p.blk_rank) {
                            uint32_t nocodes[EPL / 4];
                            const Cand c1 = finish_direct<LPB>(eval_direct<EPL, false, false>(w, cb, src, gss, a, false, nocodes));
                            rk_num = c1.ny; rk_dn = c1.dy;
                        }
                    } else if (EMIT) { rk_num = group_sum<LPB>(s.rn); rk_dn = group_sum<LPB>(s.rd); }
                    // the residual form is accurate while the reconstruction carries a fair share of
                    // the block's norm; otherwise the whole wavefront recomputes this atom directly
                    if (__builtin_expect(__any(best.weak) != 0, 0)) {
                        float ny1, dy1;
                        direct_cosine_sums<EPL, LPB, LEAN>(cb, w, ArrSrc<EPL, EMIT>{gx, gboff}, gnz, ARGMAX ? gneg : false, a, ny1, dy1);
                        best.ny = ny1;
                        best.dy = dy1;
                        raw = true;
                        odd = 1u;
                    }
                    score[a] = best.err;
                }
                // cosine value; a vanishing reconstruction has ny = 0 and gives cos 0; a zero-norm block
                // gives exactly 1 - 0 here and is corrected through the count column
                // 3 - cos lies in [2, 4], where binary32 values are 2^-22 apart and their bit patterns count
                // those steps: the fma's own rounding (nearest, ties to even) rounds 1 - cos to the unit of
                // the integer sums, and pattern minus pattern of 2.0 is that integer (no conversion)
                // (direct sums come with the codebook's own magnitude: paired with the raw norm, as they were formed;
                // the COS metric's decision sums are raw sums of w^ and are brought to the scaled norm's units)
                const float ny_raw = best.ny, dy_raw = best.dy;
                if constexpr (METRIC == 1) { best.ny *= nsc.sc; best.dy *= nsc.sc; }
                const float rs = __frsqrt_rn(__fmaf_rn((raw && METRIC != 1) ? wn : nsc.wns, best.dy, 1.0e-37f));
                const int ia = (int)__float_as_uint(__fmaf_rn(-best.ny, rs, 3.0f)) - 0x40000000;
                dlt[a] = ia;
                sums.atom(a, ia);
                if (EMIT) {
                    const long long ua = p.uidx[a];
                    if (p.codes && valid) store_codes<EPL>(p, sw, a, cm, (long long)(cs * 64u + (unsigned int)lane) * EPL, codes);
                    if (p.blk_rank) {
                        const float rank = METRIC == 1 && !SIGNED ? rank_score(ny_raw, dy_raw, wn) : rank_score(rk_num, rk_dn, wn);
                        if (leader) p.blk_rank[ua * p.Nb + blk] = rank;
                    }
                    if (p.scale_code && leader) p.scale_code[ua * p.Nb + blk] = (uint16_t)(q | (neg ? 0x8000 : 0));
                    if (p.blk_cos && leader) p.blk_cos[ua * p.Nb + blk] = wn > 0.0f ? 1.0f - __fmaf_rn(-best.ny, rs, 1.0f) : 1.0f;
                    if (p.blk_err && leader) p.blk_err[ua * p.Nb + blk] = best.err;
                }
            }
        }
        }
        // ---- selector of every requested pair: one word per block ----
        uint32_t bits = 0;
        if constexpr (ORDERED) {
            uint32_t chain = 0u;
            ordered_pairs<NA - 1, NA>(sw.A, flips, score, dlt, sums, chain);
            if (__builtin_expect(odd != 0u, 0)) {
                bool some = false;
#pragma unroll
                for (int a = 0; a < NA; ++a) some = some || !(score[a] >= 0.0f);
                if (__any(some) != 0) numbered_pairs<0, NA>(flips, score, dlt, sums, chain);
            }
            // from the chain's order to the selector's, eight bits at a time (the table holds the swapped pairs' complement too)
            if (MULTI ? lc_sel != nullptr : p.sel_words != nullptr) {
#pragma unroll
                for (int k = 0; k < NPERM; ++k) bits ^= s_perm[256 * k + ((chain >> (8 * k)) & 0xFFu)];
            }
        } else {
            all_pairs<0, NA, METRIC>(p, sw, score, den, dlt, sums, bits);
            bits ^= p.flip_slots;
        }
        void* const sel_words = MULTI ? lc_sel : p.sel_words;
        // One store without a branch ends every path of a step: lanes without a word to store, or all of them, lie past the end the store is given
        // and are dropped by the hardware.  Behind a branch it may or may not be the last access, the compiler waits for every access in
        // flight, and a step began with a wait for memory's answer to the words of the one before (4096 x 11008, six atoms, rows from HBM:
        // 71.5 us -> 70.1, rows in cache 68.4 -> 68.1; fp32, 1531 x 5024, cosine metric, 20.8 -> 20.1).  (The planes of emit mode keep their branches: a range to set up for each costs
        // more than it saves, 4096 x 11008, two atoms, 67.8 us -> 72.7.)  32-bit words belong to more than sixteen pairs: of the two stores of eight atoms one
        // has nothing to store.
        unsigned int at = (unsigned int)lane;
        asm volatile("" : "+v"(at));                   // (the offset is formed here rather than kept in a register)
        at = at % LPB == 0u ? at / LPB : 0x20000000u;      // (past every end, counted in 16-bit words as in 32-bit ones)
        const unsigned int n_here = lanes_here / LPB;
        char* const sel_at = reinterpret_cast<char*>(sel_words);
        const bool w32 = NA == 8 && p.sel_u32;
        __builtin_amdgcn_raw_buffer_store_b16((uint16_t)bits, __builtin_amdgcn_make_buffer_rsrc(sel_at + blk0 * 2, 0, sel_words && !w32 ? (int)(n_here * 2u) : 0, 0x00027000), at * 2u, 0, 0);
        if constexpr (NA == 8)
            __builtin_amdgcn_raw_buffer_store_b32(bits, __builtin_amdgcn_make_buffer_rsrc(sel_at + blk0 * 4, 0, sel_words && w32 ? (int)(n_here * 4u) : 0, 0x00027000), at * 4u, 0, 0);
        if constexpr (MULTI) asm volatile("" :: "v"(c_touch));
        i_cur = i_nxt;
        ok_cur = ok_nxt;
        i_nxt = i_nn;
        if (++since_flush == SOP_K_FLUSH_STEPS) { flush(cl); since_flush = 0; }
        if (!TOP_TEST && !ok_cur) break;
    }
    }

    // ---- per-workgroup sums: what the lanes still hold joins the workgroup's integer sums in LDS ----
    if constexpr (LSUM) {
        sums.add(NLIVE - 1, sums.z << 22);
        __syncthreads();
        static_assert(NSLOT / 4 <= (OCC == 4 ? 12 : 4 * OCC), "a wavefront for every four columns");
        if (wv < NSLOT / 4) {                                    // (four columns of all four SIMDs' words)
            const lds_int* const from = (lds_int*)(size_t)(sums.at - (uint32_t)(simd * NSLOT * 256)) + wv * 256;
            int v[4][4], lo[4] = {0, 0, 0, 0}, hi[4] = {0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[q][i] = from[q * NSLOT * 64 + 64 * i];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int i = 0; i < 4; ++i) { lo[i] += v[q][i] & 0x7FFF; hi[i] += v[q][i] >> 15; }
            join(lo, hi, s_acc + wv * 4 + (lane >> 4), lane);
        }
    } else if (!MULTI || cl >= 0) flush(cl);
    __syncthreads();
    const int tid = wv * 64 + lane;                // (not kept through the row loop)
    if constexpr (!MULTI) {
        // ---- layer reduction, one thread per output ----
        // A word of the layer's sums counts in its top bits the workgroups that have added to it, so the one that adds last knows by the value it
        // gets back that it holds the total: no ticket is taken and nothing is read afterwards.  Atomics to one address are served
        // one after the other (about 20 ns each), so a workgroup adds to one of seven words, chosen by its number, and the last of each adds
        // that total to the eighth: two round trips to memory on the last workgroup's path (sums, a ticket and the reading of the sums were
        // three, with up to 256 tickets on one address; six atoms: 256 x 1024 10.1 us -> 9.4, 1024 x 4096 16.1 -> 13.4, 4096 x 11008
        // 70.1 -> 68.4).  All adds are of integers: their order does not matter.
        // (Range of the sums beside their counts: SOP_K_SUM_MIN and sum_max().)
        // Lanes whose block had zero weighted norm (and lanes past the end of a row) added exactly 1 to every column; the count column
        // takes them out again.
        const int o = tid;
        if (o < p.A + p.P) {
            const unsigned int oc = s_out[o], G = gridDim.x;
            double* const to = o < p.A ? p.acos_atom : p.acos_pair;
            if (to) {
                constexpr unsigned int R = SOP_K_REPL - 1;
                const unsigned int r = blockIdx.x % R, members = sum_members(G, r), used = sum_rows_used(G);
                unsigned long long* const w1 = p.sums + r * SOP_K_NCOL + o;
                unsigned long long* const w2 = p.sums + R * SOP_K_NCOL + o;
                const unsigned long long add1 = sum_add1((long long)(s_acc[oc & 0xFFu] - s_acc[NLIVE - 1]), p.sum_max);
                const unsigned long long s1 = atomicAdd(w1, add1) + add1;
                if ((s1 >> 56) == members) {
                    __hip_atomic_store(w1, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);       // (zero for the next call)
                    const unsigned long long add2 = sum_add2(s1, members);
                    const unsigned long long s2 = atomicAdd(w2, add2) + add2;
                    if ((s2 >> 60) == used) {
                        __hip_atomic_store(w2, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        to[oc >> 8] = 1.0 - ((double)(long long)(s2 - used * kSumOne2) * (1.0 / 4194304.0)) / ((double)p.Nb * (double)p.lpb);
                    }
                }
            }
        }
        return;
    }
    if constexpr (MULTI) {
        // every layer's sums of this workgroup join the layer's replica; eight adds of a thread are in
        // flight before their returned values are consumed (see below for why they are consumed)
        for (int base = 0; base < n_acc; base += 8 * NT) {
            unsigned long long before[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int idx = base + j * NT + tid;
                before[j] = 0ull;
                if (idx < n_acc) {
                    const unsigned long long v = s_acc[idx];
                    const int layer = idx / NSLOT, col = idx - layer * NSLOT;
                    if (v != 0ull) before[j] = atomicAdd(p.sums + ((size_t)layer * SOP_K_REPL + blockIdx.x % SOP_K_REPL) * SOP_K_NCOL + col, v);
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) asm volatile("" :: "v"(before[j]) : "memory");
        }
    }
    // every workgroup takes a ticket; the one that takes the last finishes the layers of the launch
    __syncthreads();
    unsigned int* s_flag = reinterpret_cast<unsigned int*>(s_red);
    if (tid == 0) {
        unsigned int last = 0u;
        if (atomicAdd(p.done, 1u) == gridDim.x - 1) { atomicExch(p.done, 0u); last = 1u; }
        *s_flag = last;
    }
    __syncthreads();
    if constexpr (MULTI) {
        if (*s_flag) {
            // totals of every (layer, column) over the replicas into LDS, in place of the workgroup's own sums
            // (the exchanges leave zeros for the next call), then one ACos per (layer, atom or pair)
            __syncthreads();
            for (int idx = tid; idx < n_acc; idx += NT) {
                const int layer = idx / NSLOT, col = idx - layer * NSLOT;
                if (col >= NLIVE) continue;
                unsigned long long* src = p.sums + (size_t)layer * SOP_K_REPL * SOP_K_NCOL + col;
                unsigned long long part[SOP_K_REPL];
#pragma unroll
                for (int r = 0; r < SOP_K_REPL; ++r) part[r] = atomicExch(src + r * SOP_K_NCOL, 0ull);
                unsigned long long tot = 0ull;
#pragma unroll
                for (int r = 0; r < SOP_K_REPL; ++r) tot += part[r];
                s_acc[idx] = tot;
            }
            __syncthreads();
            const int per = p.A + p.P;
            for (int o = tid; o < p.n_layers * per; o += NT) {
                const int layer = o / per, q = o - layer * per;
                int col;
                double* dst;
                const size_t row = (size_t)p.layers[layer].out_row;
                if (q < p.A) { col = q; dst = p.acos_atom ? p.acos_atom + row * p.A + p.uidx[q] : nullptr; }
                else { col = p.pair_col[q - p.A]; dst = p.acos_pair ? p.acos_pair + row * p.P + (q - p.A) : nullptr; }
                const long long z = (long long)s_acc[layer * NSLOT + NLIVE - 1];
                const long long t = (long long)s_acc[layer * NSLOT + col];
                if (dst) *dst = 1.0 - ((double)(t - z) * (1.0 / 4194304.0)) / ((double)p.layers[layer].Nb * (double)p.lpb);
            }
        }
    }
}

}  // namespace sopk

// ---- kernel table of this part ----
namespace {
// Wavefronts per SIMD each variant is built for (512 / occ registers a lane): as many as its registers allow without spilling (the
// signed cosine search, with its chunks of look-ups kept apart, at three: 4096 x 4096, six atoms, g = 16, bf16, 47.8 us against 51.6
// with 18 to 61 registers spilled, fp32 52.8 at three against 59.5 at two, eight atoms 67.6 against 76.8).  The passes that
// evaluate a scale group's atoms together (16 elements a lane, positive scale) hold neither scaled weights
// nor table addresses and fit one wavefront more than the others: the headline layer (4096 x 11008, six atoms) takes 75.7 us at
// four against 78.4 with the arrays at three, a 28672 x 8192 layer with seven atoms 530 us at three against 640 at two.  fp32
// weights keep 8 more registers of requested rows: one wavefront less where that is the difference.  Metric COS, from the arrays of one
// atom at a time at two wavefronts: 4096 x 11008, bf16, 2 / 4 / 6 / 7 atoms 40.2 / 76.3 / 96.6 / 112 us -> 37.6 / 59.6 / 83 / 104.5, two atoms with every
// plane 84 -> 72.7, fp32 4096 x 4096, six atoms 43.2 -> 37.4; the model-wide search of six atoms (bf16) spills a register at four wavefronts.
constexpr int occ_for(bool bf16, int epl, int sign_mode, bool emit, int na, int metric, bool multi)
{
    if (lane_sums_in_lds(bf16, epl, sign_mode, metric, emit, na, multi)) return (na == 8 && sign_mode != 0) || (sign_mode == 2 && metric == 1) ? 3 : 4;      // (109 to 128 registers; 126 to 168)
    if (epl == 8) {
        if (na == 2) return (sign_mode == 1 && emit) ? 3 : 4;
        if (sign_mode == 1) return emit ? 2 : 3;
        return (emit || na == 8) ? 3 : 4;
    }
    if (sign_mode == 0) {
        if (!emit) return na == 8 || (na == 6 && metric == 1 && multi) ? 3 : (na == 2 || bf16) ? 4 : 3;
        return na == 2 || (na == 6 && bf16 && metric != 1) ? 3 : 2;
    }
    if (na == 2) return emit ? (sign_mode == 1 && metric != 1 && bf16 ? 3 : 2) : 3;
    if (sign_mode == 1) return emit ? (na == 8 ? 1 : 2) : (na == 8 && metric != 1) ? 2 : 3;
    if (emit) return 2;
    return (na == 8 || metric == 1) ? 2 : 3;        // (argmax rule) the cosine metric keeps two more sums per candidate alive
}

// one variant: *occ = wavefronts per SIMD its registers allow (a workgroup has 4 * occ wavefronts).  mode 0: one
// layer; 2: a list of layers, which exists for the searches of more than two atoms that write no per-block
// planes; *mode_out tells which mode was given.
template <bool BF16, int EPL, int LPB, int S, bool E, int NA>
const void* variant(int mode, int* occ, int* mode_out)
{
    constexpr int MT = SOPK_PART_METRIC;
    constexpr int O = occ_for(BF16, EPL, S, E, NA, MT, false);
    *occ = O;
    *mode_out = 0;
    if constexpr (!E && NA != 2) {
        if (mode == 2) {
            constexpr int OM = occ_for(BF16, EPL, S, E, NA, MT, true);
            *occ = OM;
            *mode_out = 2;
            return reinterpret_cast<const void*>(&sopk::search_kernel<BF16, EPL, LPB, S, MT, E, NA, OM, true>);
        }
    }
    return reinterpret_cast<const void*>(&sopk::search_kernel<BF16, EPL, LPB, S, MT, E, NA, O, false>);
}

// na_class: 0 = at most two atoms, 1 = at most six, 2 = up to eight
template <bool BF16, int EPL, int LPB>
const void* pick_geom(int sign_mode, bool emit, int na_class, int mode, int* occ, int* mode_out)
{
#define SOPK_FN(S, E, NA) variant<BF16, EPL, LPB, S, E, NA>(mode, occ, mode_out)
#define SOPK_BY_SIGN(E, NA) (sign_mode == 1 ? SOPK_FN(1, E, NA) : sign_mode == 2 ? SOPK_FN(2, E, NA) : SOPK_FN(0, E, NA))
    if (emit) return na_class == 0 ? SOPK_BY_SIGN(true, 2) : na_class == 1 ? SOPK_BY_SIGN(true, 6) : SOPK_BY_SIGN(true, 8);
    if (na_class == 0) return SOPK_BY_SIGN(false, 2);
    if (na_class == 1) return SOPK_BY_SIGN(false, 6);
    return SOPK_BY_SIGN(false, 8);
#undef SOPK_BY_SIGN
#undef SOPK_FN
}
}  // namespace

#define SOPK_CAT2(a, b, c) a##b##_##c
#define SOPK_CAT(a, b, c) SOPK_CAT2(a, b, c)

// g: block size; na_class: 0 / 1 / 2 for alphabets of at most 2 / 6 / 8 atoms; mode: 0 one layer, 2 a list of layers
// (*mode_out: the mode of the kernel returned, 0 where the one asked for does not exist).  *occ receives the
// wavefronts per SIMD the variant is built for (its workgroup has 256 * occ threads)
extern "C" const void* SOPK_CAT(sopk_part_, SOPK_PART_BF16, SOPK_PART_METRIC)(int g, int sign_mode, int emit, int na_class, int mode, int* occ, int* mode_out)
{
    constexpr bool B = SOPK_PART_BF16 != 0;
    switch (g) {
        case 8:  return pick_geom<B, 8, 1>(sign_mode, emit, na_class, mode, occ, mode_out);
        case 16: return pick_geom<B, 16, 1>(sign_mode, emit, na_class, mode, occ, mode_out);
        case 32: return pick_geom<B, 16, 2>(sign_mode, emit, na_class, mode, occ, mode_out);
        default: return pick_geom<B, 16, 4>(sign_mode, emit, na_class, mode, occ, mode_out);
    }
}
