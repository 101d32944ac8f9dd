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
template <int EPL, bool CODES, bool WANT_ERR, bool TIES = false, bool APART = false, class SRC>
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
        // (APART: eight atoms under the argmax rule, which spill 4 registers of three wavefronts' otherwise)
        // (a register budget, not an order: with the chunks apart the signed six-atom search keeps 139 registers, without 168 and up to 60 spilled;
        // every plane of eight atoms of 8-element lanes 162 to 167, without 168 and up to 12 spilled)
        if constexpr (APART || (TIES && !CODES && EPL == 16) || (CODES && (EPL == 8 || !TIES))) asm volatile("" : "+v"(n0), "+v"(n1), "+v"(d0), "+v"(d1));
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
// PLANES: the per-block planes the kernel can write: none, any of them, or one and no other (SOP_K_PLANES_*), which is then there.
// SIGNMODE 0: the scale is positive; 1: both signs of the scale are tried and the better one kept
// (signed scale word, absmax rule); 2: argmax rule, the rule fixes the sign.
template <bool BF16, int EPL, int LPB, int SIGNMODE, int METRIC, bool EMIT_, int NA, int OCC, bool MULTI>
__global__ __launch_bounds__(256 * OCC, 1) void search_kernel(const KParams p)
{
    constexpr int PLANES = EMIT_ ? SOP_K_PLANES_ALL : SOP_K_PLANES_NONE;
#include "sop_search_body.inc"
}

// a search that writes one plane (see one_plane_variants())
template <bool BF16, int EPL, int LPB, int SIGNMODE, int METRIC, int PLANES, int NA, int OCC>
__global__ __launch_bounds__(256 * OCC, 1) void plane_kernel(const KParams p)
{
    constexpr bool MULTI = false;
#include "sop_search_body.inc"
}

}  // namespace sopk

// ---- kernel table of this part ----
namespace {
// Wavefronts per SIMD each variant is built for (512 / occ registers a lane): as many as its registers allow without spilling.  (With the lanes' sums in registers: the
// signed cosine search, its chunks of look-ups kept apart, 4096 x 4096, six atoms, g = 16, bf16, three wavefronts 47.8 us against 51.6
// with 18 to 61 registers spilled, fp32 52.8 at three against 59.5 at two, eight atoms 67.6 against 76.8; in LDS, see lane_sums_in_lds(), they fit one more.)  The passes that
// evaluate a scale group's atoms together (16 elements a lane, positive scale) hold neither scaled weights
// nor table addresses and fit one wavefront more than the others: the headline layer (4096 x 11008, six atoms) takes 75.7 us at
// four against 78.4 with the arrays at three, a 28672 x 8192 layer with seven atoms 530 us at three against 640 at two (425 at four, sums in LDS).  fp32
// weights keep 8 more registers of requested rows: one wavefront less where that is the difference.  Metric COS, from the arrays of one
// atom at a time at two wavefronts: 4096 x 11008, bf16, 2 / 4 / 6 / 7 atoms 40.2 / 76.3 / 96.6 / 112 us -> 37.6 / 59.6 / 83 / 104.5, two atoms with every
// plane 84 -> 72.7, fp32 4096 x 4096, six atoms 43.2 -> 37.4; the model-wide search of six atoms (bf16) spills a register at four wavefronts.
constexpr int occ_for(bool bf16, int epl, int sign_mode, int planes, int na, int metric, bool multi)
{
    const bool emit = planes == SOP_K_PLANES_ALL;
    if (planes == SOP_K_PLANES_ERR) return 4;
    if (planes == SOP_K_PLANES_RANK) return sign_mode == 0 || epl == 8 ? 4 : bf16 || na == 2 ? 3 : 2;
    if (lane_sums_in_lds(bf16, epl, sign_mode, metric, planes, na, multi)) return epl == 16 && ((na == 8 && sign_mode != 0) || (sign_mode == 2 && metric == 1)) ? 3 : 4;      // (109 to 128 registers; 126 to 168)
    if (epl == 8) {
        if (na == 2) return (sign_mode == 1 && emit) ? 3 : 4;
        if (sign_mode == 1) return emit ? 2 : multi && na == 6 && metric == 0 ? 4 : 3;      // (model-wide, g = 8, at three wavefronts and at four: eight layers of 4096 x 4096, six atoms, bf16 380 us and 328, fp32 387 and 337)
        return (emit || na == 8) ? 3 : 4;
    }
    if (sign_mode == 0) {
        if (!emit) return na == 8 || (na == 6 && metric == 1 && multi) ? 3 : (na == 2 || bf16) ? 4 : 3;
        return na == 2 || (na == 6 && bf16 && metric != 1) ? 3 : 2;
    }
    if (na == 2) return emit ? (sign_mode == 1 && metric != 1 && bf16 ? 3 : 2) : sign_mode == 1 && metric != 2 ? 4 : 3;      // (signed: 104 to 128 registers, MSE a few more; 4096 x 11008, two atoms, 61.7 us at three wavefronts, 56.9 at four, one 38.0 and 34.6)
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
    if constexpr (E && NA != 8 && one_plane_variants(EPL, S, MT, NA, SOP_K_PLANES_RANK)) {
        if (mode == SOP_K_PLANES_RANK) {
            constexpr int OP = occ_for(BF16, EPL, S, SOP_K_PLANES_RANK, NA, MT, false);
            *occ = OP; *mode_out = mode;
            return reinterpret_cast<const void*>(&sopk::plane_kernel<BF16, EPL, LPB, S, MT, SOP_K_PLANES_RANK, NA, OP>);
        }
    }
    if constexpr (E && NA != 8 && one_plane_variants(EPL, S, MT, NA, SOP_K_PLANES_ERR)) {
        if (mode == SOP_K_PLANES_ERR) {
            constexpr int OP = occ_for(BF16, EPL, S, SOP_K_PLANES_ERR, NA, MT, false);
            *occ = OP; *mode_out = mode;
            return reinterpret_cast<const void*>(&sopk::plane_kernel<BF16, EPL, LPB, S, MT, SOP_K_PLANES_ERR, NA, OP>);
        }
    }
    constexpr int PL = E ? SOP_K_PLANES_ALL : SOP_K_PLANES_NONE;
    constexpr int O = occ_for(BF16, EPL, S, PL, NA, MT, false);
    *occ = O;
    *mode_out = 0;
    if constexpr (!E && NA != 2) {
        if (mode == 2) {
            constexpr int OM = occ_for(BF16, EPL, S, PL, NA, MT, true);
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
