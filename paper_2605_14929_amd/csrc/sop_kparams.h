// Launch parameters shared by the host side of the library and its kernels (passed by value).
#ifndef SOP_KPARAMS_H
#define SOP_KPARAMS_H
#include <stddef.h>
#include <stdint.h>

#define SOP_K_MAXA 8                 /* atoms                                        */
#define SOP_K_MAXP 28                /* pairs i < j among SOP_K_MAXA atoms           */
#define SOP_K_NCOL (SOP_K_MAXA + SOP_K_MAXP + 1)   /* sum columns: atoms, pairs, zero-norm lane count */
#define SOP_K_OUT_WORDS ((SOP_K_MAXA + SOP_K_MAXP + 1) / 2)   /* 64-bit words of a list of the outputs, 32 bits each */
#define SOP_K_FLUSH_STEPS 60         /* steps a lane's running sums are kept before they join the workgroup's (4 * 60 * 2^23 < 2^31) */
#define SOP_K_REPL 8                 /* rows of layer sums (spread same-address atomics): replicas, the last one of a single layer's the totals of the others */
#define SOP_K_MAXBINS 1024           /* bins of the element-search table                        */
#define SOP_K_MAXTABCODES 2048       /* scale codes whose (scale, reciprocal) pair is tabulated */
#define SOP_K_BIN_BYTES (8 * (SOP_K_MAXA + 1))          /* a bin record (see BinRec) */
#define SOP_K_PAIR_BIN_BYTES (8 * (SOP_K_MAXA + 2))     /* the same where atoms are evaluated two or four at a time */
#define SOP_K_WIDE_BIN_BYTES(na) (16 * ((na) + 1))       /* the same in the LDS of kernels that write planes (unrolled for na atoms): values, their sum and the code of every atom */
#define SOP_K_BIN_MAGIC 12582912.0f  /* 1.5 * 2^23: one unit in the last place is 1               */
/* bits(MAGIC + v) = 0x4B400000 + v; the 24-bit multiply sees 0x400000 + v: subtract its product */
#define SOP_K_BIN_NEGC(bytes) (0u - 0x400000u * (unsigned)(bytes))
/* The bin table covers scaled weights from BIN_EXT * L[0] to BIN_EXT * L[N-1]: a block scale that
 * was rounded down (by at most a factor 1.5, in the subnormal range of the scale word) leaves every
 * scaled weight inside the table without a clamp.  Blocks whose scale saturated take a clamped path,
 * selected when ideal scale / rounded scale exceeds BIN_SAFE. */
#define SOP_K_BIN_EXT 1.5625f
#define SOP_K_BIN_SAFE 1.55f

#if defined(__HIPCC__) || defined(__HIP__)
#define SOP_K_HD __host__ __device__
#else
#define SOP_K_HD
struct float2 { float x, y; };       /* (host-only translation units see the launch parameters' layout without a HIP header) */
#endif

/* position of (i,j), i < j, in the lexicographic list of all pairs of SOP_K_MAXA atoms */
SOP_K_HD constexpr int pair_index(int i, int j) { return i * (2 * SOP_K_MAXA - i - 1) / 2 + (j - i - 1); }
/* bit of pair (i,j), i < j, in the chain in which a search of more than two atoms forms the pairs (metrics WSE and MSE) */
SOP_K_HD constexpr int chain_bit(int i, int j) { return j * (j - 1) / 2 + i; }

/* Tables of 256 selector words that take the pairs from the order of a chain to the order requested (metrics WSE and MSE, more than two atoms) */
SOP_K_HD constexpr int search_perm_tables(int na, bool cosine) { return na == 2 || cosine ? 0 : (na * (na - 1) / 2 + 7) / 8; }

/* Sum columns of a variant unrolled for na atoms: atoms, pairs i < j of them (lexicographic), count of zero-norm lanes; and the same
 * rounded up to the four columns that a wavefront adds up together */
SOP_K_HD constexpr int search_cols(int na) { return na + na * (na - 1) / 2 + 1; }
SOP_K_HD constexpr int search_slots(int na) { return (search_cols(na) + 3) / 4 * 4; }

/* Per-block planes that a variant of the search can write: none; any of them; the ranking scores or the block errors and no other.
 * The variants of one plane are those of the searches that a program makes for a plane alone (metric WSE): the ranking scores of up to six atoms, the first pass of the
 * per-layer procedure, and the errors of one or two under a positive scale, the comparison of weight formats.  They form no codes, need no 16-byte records and keep no
 * pointers of planes that are not there, which is a wavefront more per SIMD, and store without a branch.  4096 x 11008, bf16, ranking scores of six atoms 130 us (any plane) -> 113,
 * of two 49.8 -> 44.4, under a signed word (whose codes were formed to no end) 272 -> 165 and 105 -> 86 (g = 64); fp32 174 -> 121; 28672 x 8192, errors of one atom 149 -> 121;
 * lanes of eight weights, ranking scores of six atoms 161 -> 126, under a signed word 286 -> 157.
 * Other planes alone (and the ranking scores of a procedure with seven or more atoms, of the argmax rule or the other metrics) come from the kernel of any plane.  By their registers they would gain
 * as well (bf16, g = 16: ranking scores of eight atoms 154, three wavefronts where any plane leaves two; errors of six 126, four and not three): they are left out for the library's size
 * and build time, of which every such kind takes a kernel more per block size and weight type (these 38 take 1.3 MB). */
#define SOP_K_PLANES_NONE 0
#define SOP_K_PLANES_ALL 1
#define SOP_K_PLANES_RANK 3
#define SOP_K_PLANES_ERR 4
SOP_K_HD constexpr bool one_plane_variants(int epl, int sign_mode, int metric, int na, int planes)
{
    return metric == 0 && na != 8 && (planes == SOP_K_PLANES_RANK ? sign_mode != 2 : epl == 16 && na == 2 && sign_mode == 0);
}

/* Searches of one layer that keep their lanes' running sums in LDS rather than in registers: 22 registers less for six atoms, 37 for eight, where that is
 * a wavefront more per SIMD (see occ_for(); an add is one instruction either way, and the adds of a wavefront meet no other lane's word).  Measured, registers -> LDS,
 * 4096 x 4096 and 4096 x 11008, bf16, g = 16: six atoms under a signed word 43.1 us -> 38.4 and 95.3 -> 89.1 (145 registers, now 126: three wavefronts, now four), by
 * the cosine 43.6 -> 37.7 and 99.6 -> 90.8; seven 39.4 -> 35.4 and 88.7 -> 83.1, eight 45.2 -> 40.8 and 101.9 -> 96.2 (143 -> 109), under a signed word 72.6 -> 61.8 and
 * 175 -> 143.8 (two wavefronts, now three); argmax rule 33.1 -> 30.2 and 74.0 -> 70.9; fp32, six atoms 35.5 -> 33.4 and 77.8 -> 74.0; 28672 x 8192, seven 475 -> 425.
 * Lanes of 8 elements, six under a signed word and all of eight, three wavefronts, now four: 4096 x 11008, g = 8, 120 -> 105 and 130 -> 116.
 * Where the sums are not what holds a wavefront back they stay in registers: six atoms of bf16 weights (four wavefronts as it is), most of one or two, planes, MSE of 16-element lanes under a
 * signed word or the argmax rule (six spill up to 113 registers at four wavefronts), and the model-wide kernel, whose wavefronts of a SIMD are in different layers at a time. */
SOP_K_HD constexpr bool lane_sums_in_lds(bool bf16, int epl, int sign_mode, int metric, int planes, int na, bool multi)
{
    if (planes == SOP_K_PLANES_RANK) return na == 6 && (epl == 16 || sign_mode == 1);
    if (epl == 8) return !multi && planes == SOP_K_PLANES_NONE && (na == 8 || (na == 6 && sign_mode == 1));
    if (na == 2) return planes == SOP_K_PLANES_NONE && sign_mode == 1 && !bf16 && metric == 0;      // (one register short of four wavefronts)
    return !multi && planes == SOP_K_PLANES_NONE && epl == 16 && !(sign_mode == 0 && na == 6 && bf16) && !(sign_mode != 0 && na == 6 && metric == 2);
}
/* LDS of these sums: four sets (one a SIMD) of 64 words a column, on a 16-byte boundary */
SOP_K_HD constexpr size_t lane_sums_bytes(int na) { return (size_t)4 * search_slots(na) * 64 * 4 + 8; }

/* One bin of the element-search table.  For every atom the bin holds at most one code boundary.
 * The two values are stored HALVED (exactly; the element passes multiply by twice the block scale): the boundary
 * between two neighbouring entries then equals the binary32 sum of the two stored values, and the passes form it with
 * one addition instead of reading it.  In a bin without a boundary the upper value is +infinity, and so is the sum: nothing
 * lies above it or on it.
 * One atom's values come with an 8-byte read of LDS, those of an even slot and the next with a 16-byte one.  An alphabet whose atoms are all evaluated one by one
 * has its records 72 bytes apart, an odd number of 8-byte words: 32 neighbouring bins have an atom's values in 32 different pairs of LDS's 64 banks.  16-byte
 * reads want records on 16-byte boundaries; an odd number of those, 80 bytes, puts 16 neighbouring bins into 16 different quadruples of banks.
 * (72 bytes and ds_read2_b64 for two atoms: 4096 x 11008, six atoms, 1 to 2 % slower; 80 bytes for atoms one by one: five atoms of fitted codebooks 1 % slower.) */
struct BinRec {
    float val[SOP_K_MAXA][2];            // half of the codebook value at and below the boundary, half of the one above it
    unsigned char code_lo[SOP_K_MAXA];   // code at and below the boundary
};
static_assert(sizeof(BinRec) == SOP_K_BIN_BYTES && SOP_K_BIN_BYTES % 16 == 8 && SOP_K_PAIR_BIN_BYTES % 32 == 16 && SOP_K_WIDE_BIN_BYTES(2) % 32 == 16 && SOP_K_MAXA % 2 == 0, "odd numbers of words");

/* Atoms are handled in an internal order in which atoms with equal endpoints (one "scale group":
 * same ideal scale, same scale code, same scaled weights) are adjacent, and an atom that is the
 * sign-negated copy of another follows it directly where the grouping allows. */
struct KParams {
    // inputs
    const void*   W;
    const float*  c;
    const char*   bins;              // [n_bins] records (BinRec) rec_bytes apart, atoms in internal order
    const float2* stab;              // [n_tab_codes] (twice the scale value(q) * 2^-k, the scale's reciprocal), or null
    long long M, K, ldw;             // as the kernel walks the layer: rows may be folded (see Kc)
    long long Kc;                    // true row length.  When the rows lie back to back (ldw == K) and 64 lanes do not divide a
                                     // row's lanes, the host folds f rows into one of f*K columns (M/f rows): the last strip of
                                     // every row then wastes fewer lanes (none when 64 divides f*K/EPL).  Block and element
                                     // indices are unchanged by this; only the channel of a column becomes its index modulo Kc.
    long long Bk;                    // blocks per row
    long long Nb;                    // blocks in the layer
    long long strips;                // 64-lane strips per row
    long long total_units;           // strips * M
    unsigned int units_q, units_r;   // total_units = units_q * workgroups + units_r
    unsigned int grid_magic;         // ceil(2^32 / workgroups) (2^32 - 1 for one): a product of two numbers up to the workgroups, divided by them
    unsigned int M32, m_magic;       // M, and floor(2^32 / M) (2^32 - 1 for M = 1): step number -> (strip, row)
    int A, P, lpb;
    int n_bins;
    unsigned int rec_bytes;          // SOP_K_BIN_BYTES or SOP_K_PAIR_BIN_BYTES
    int n_tab_codes;                 // 0: scale and reciprocal are computed arithmetically
    // scale word
    int man_bits, bias, max_code, k;
    float pow2k;                     // 2^k
    float sub_quantum;               // 2^(1-bias-man_bits-k)
    // atoms, internal order
    alignas(16) float gpar[SOP_K_MAXA][8];         // t+, -t-, bin scale and offset (bin = bits(fma(x, sc, off)) - bits(magic)), range of x the table covers
                                                   // (clamped path, low and high), 0, 0: two 16-byte words an atom, copied to LDS as they are
    unsigned int gid_w;                            // 4 bits per atom: its scale group (atoms of a group are adjacent)
    unsigned int second_mask;                      // odd bit a: atoms a-1 and a are of one scale group (evaluated together, also where planes but no codes
                                                   // are written); bits 2 and 6: atoms 0..3 and 4..7 are (evaluated together in search mode)
    unsigned int deal;                             // (one layer) not 0: the wavefronts' first steps are dealt out (search_deal()), and this is the launch's wavefronts per SIMD, which the
                                                   // kernel takes its number of threads from: never 0 where search_waves() gives fewer than the variant is built for
    unsigned int mirror_mask;                      // bit a: atom a is the sign-negated copy of atom a-1 (signed scale words take its candidates over)
    unsigned int selfsym_mask;                     // bit a: atom a is its own sign-negated copy
    alignas(8) unsigned char nent[SOP_K_MAXA];     // entries of the atom
    unsigned int unit_tpos, unit_tneg;             // bit a: the endpoint is exactly 1 (no division needed)
    unsigned int wide_mask;                        // bit a: more than 16 entries (one byte per code)
    alignas(8) unsigned char uidx[SOP_K_MAXA];     // caller's index of the atom
    long long code_off[SOP_K_MAXA];                // byte offset of the atom's code plane
    unsigned int pair_mask;                           // bit pair_index(i,j): the pair is requested
    unsigned int flip_mask;                           // bit pair_index(i,j): the caller's first atom is internal j
    unsigned int flip_slots;                          // bit q: output pair q is such a swapped pair
    // (byte arrays sit on 8-byte boundaries so that the kernels fetch them with scalar loads)
    unsigned int pair_slot_w[SOP_K_MAXP / 4];          // byte pi%4 of word pi/4: output index of pair pi = pair_index(i,j)
    alignas(8) unsigned char pair_col[SOP_K_MAXP + 4]; // sum column of output pair o (in the variant's own numbering, see search_cols)
    // outputs
    // layer sums of 1-cos in fixed point (2^-22 units): every workgroup adds its share with integer
    // atomics (order-independent, so the result is reproducible); the workgroup that finishes last
    // turns them into the ACos outputs and leaves the sums (and the model-wide kernel's counter) at zero for the next call
    unsigned long long* sums;        // [SOP_K_REPL][SOP_K_NCOL]
    unsigned int* done;              // (model-wide kernel) workgroups finished (zero between calls)
    long long sum_max;               // (single search) the largest sum that a workgroup adds, sum_max(workgroups)
    double*   acos_pair;
    double*   acos_atom;
    void*     sel_words;             // [Nb] selector word of every block
    int       sel_u32;               // 1: 32-bit selector words, 0: 16-bit
    uint16_t* scale_code;
    uint8_t*  codes;
    float*    blk_cos;
    float*    blk_err;
    float*    blk_rank;              // [A][Nb] ranking score of step 2 (signed squared block cosine, binary32 decision quantity)
    // model-wide kernel: the layers of one launch (W, c, M, K, ldw, Nb, sel_words above are then unused); sums is
    // [n_layers][SOP_K_REPL][SOP_K_NCOL], acos_pair / acos_atom are tables with rows of P / A values (a layer names its row)
    const struct LayerDesc* layers;
    int n_layers;
    unsigned int chain_sel[(SOP_K_MAXP + 7) / 8 * 8];  // (last: only the searches that chain their pairs read it) bit of the selector word that bit chain_bit(i,j) of a chain of pairs becomes, 0: not requested
};

/* One layer of a model-wide launch (72 bytes, read with scalar loads) */
struct LayerDesc {
    const void*  W;
    const float* c;
    void*        sel_words;          // or NULL
    long long    ldw;
    long long    Nb;
    int          Bk;
    int          out_row;            // row of the ACos tables this layer's results go to
    unsigned int M32, m_magic;       // rows, floor(2^32 / rows)
    int          K;
    unsigned int units_q, units_r;   // strips * rows = units_q * workgroups + units_r
    int          Kc;                 // true row length (rows may be folded as in KParams)
};

/* Workgroups of a search, one per compute unit at most, from whole steps per SIMD.  A step more on every SIMD costs about
 * 0.3 us + 0.1 us per evaluation (evaluations: codebooks times signs tried, twice that where planes are written), a workgroup
 * more about 10/3 ns in the layer reduction.  Beyond SOP_K_SHORT_SHARE steps a SIMD every compute unit has a workgroup.
 * Measured at 64 to 8000 steps over 31 kinds of call, captured in a graph, against every number of workgroups that changes the steps per
 * SIMD: 0.3 % above the best on average, 5.6 % at worst (one atom with every plane, 8000 steps: 14.3 us with 250 workgroups,
 * 13.6 with 256; one atom, 771: 5.3 with 193, 5.6 with 97; 1024: 5.6 with 128, 5.4 with 256; six atoms, 1536: 9.8 with 192 or 256, 11.2 with 128;
 * every plane of six signed ones, 1536: 21.5 with 192, 31.9 with 128). */
#define SOP_K_SHORT_SHARE 8
inline long long search_workgroups(long long steps, int n_cu, int evaluations)
{
    const long long least = (steps + 4ll * n_cu - 1) / (4ll * n_cu);
    if (least > SOP_K_SHORT_SHARE) return n_cu;
    long long best = 0, best_cost = 0;
    for (long long s = least; s <= SOP_K_SHORT_SHARE; ++s) {
        const long long wg = (steps + 4 * s - 1) / (4 * s), cost = s * (900 + 300 * evaluations) + 10 * wg;       // (in thirds of a nanosecond)
        if (best == 0 || cost < best_cost) { best = wg; best_cost = cost; }
    }
    return best;
}

/* Wavefronts per SIMD of such a launch, of a variant built for occ.  A share of eight steps, two for each of four wavefronts, takes longer than with three wavefronts, which
 * end one after the other (7.03 to 8 steps a SIMD in layers of 1024, 2048, 4096, 5024, 5632, 8192, 11008 and 16384 columns, four wavefronts -> three: six atoms 18.7 - 19.5 us -> 17.8 - 18.6, of
 * fp32 weights 18.3 - 20.7 -> 17.6 - 19.4, by the cosine of fp32 weights 18.0 - 20.7 -> 17.0 - 19.0, seven 21.2 - 21.9 -> 20.7 - 21.3, one 8.8 - 9.8 -> 8.5 - 9.4, two 10.9 - 11.9 -> 10.4 - 11.4; six under a
 * signed word 23.6 - 24.5 -> 23.4 - 24.0).  Other shares do not (7 steps and a few more than 8, six, seven and six signed atoms: 2 to 10 % slower with three wavefronts, one and two atoms within 4 % either way;
 * 5024 columns, 5 and 6 steps: 4 to 10 %, 9 to 17: 1 to 5 %). */
inline int search_waves(int occ, long long steps, long long wg)
{
    const long long most = ((steps + wg - 1) / wg + 3) / 4;          /* steps of the longest share */
    return occ == 4 && most == 8 ? occ - 1 : occ;
}

/* Are the wavefronts' first steps dealt out, and their rows asked for ahead of the tables?  In short shares, always (see search_kernel).  In longer ones
 * searches of more than two atoms gain 0.3 to 0.7 us a call by it (2048 x 5120, six under a signed word 27.2 us -> 26.5, eight 28.0 -> 27.3, fp32 26.8 -> 25.8; 4096 x 11008, seven 80.8 ->
 * 80.2), one or two atoms and the searches that write planes lose 0.1 to 0.4. */
inline bool search_deal(int na, bool emit, long long steps, int n_cu) { return steps <= 4ll * SOP_K_SHORT_SHARE * n_cu || (na > 2 && !emit); }

/* LDS of a search unrolled for na atoms, beside the kernel's own variables (below 1 KiB): selector tables, bin records, scale table, group parameters, outputs and sums */
inline size_t search_lds(int na, bool cosine, int n_bins, int rec_bytes, int n_codes)
{
    return (size_t)search_perm_tables(na, cosine) * 1024 + (size_t)n_bins * rec_bytes + (((size_t)n_codes * 8 + 15) & ~(size_t)15) + 2 * SOP_K_MAXA * 16 + (1 + SOP_K_OUT_WORDS + search_slots(na)) * 8;
}
/* Scale codes tabulated: all of them, or none where the table does not fit beside the bins and the kernel computes the scales instead, to the same bits: planes of seven
 * or eight atoms with 1024 bins beside more than about 1300 codes (seven atoms, 4096 x 11008, 2048 codes: 267 us; such planes of three atoms, which fit, 106.) */
inline int search_tab_codes(int na, bool cosine, int n_bins, int rec_bytes, int n_codes, size_t lds_max) { return search_lds(na, cosine, n_bins, rec_bytes, n_codes) + 1024 > lds_max ? 0 : n_codes; }

/* Layer sums of a single search.  A word of them counts in its top bits the workgroups that have added to it (units of 2^56 in the first
 * SOP_K_REPL - 1 rows, of 2^60 in the last one, which takes those rows' totals).  A sum must never reach into its count or borrow from it,
 * whatever the weights held: a word that misses its count is not cleared, and spoils the calls that follow.  A bias beside every one of a
 * count keeps a word's sum above zero, and a workgroup's sum is cut to SOP_K_SUM_MIN .. sum_max() before it is added.
 * That changes none of a valid layer: a lane step reads 16 bytes or more, so 288 GB hold fewer than 2^35 of at most 2^23 each, below 2^58 for the
 * layer, and a large layer is spread evenly over all compute units (26 or more: sum_max(g) >= 2^58 / g); a lane's sum can be a few units below
 * zero.  Where a block's own sums leave binary32's range the lanes' 32-bit sums wrap: a NaN deficit counts 2^30 - 2^22, four of them -2^24. */
#define SOP_K_SEARCH_MAXWG 256       /* workgroups of a single search (one per compute unit) */
#define SOP_K_SUM_MIN (-(1ll << 48))
constexpr unsigned long long kSumOne1 = (1ull << 56) + (1ull << 49), kSumOne2 = (1ull << 60) + (1ull << 54);
/* workgroups that add to first-row word r of a launch of g, and first-row words that g workgroups add to */
SOP_K_HD constexpr unsigned int sum_members(unsigned int g, unsigned int r) { return (g - r + SOP_K_REPL - 2u) / (SOP_K_REPL - 1u); }
SOP_K_HD constexpr unsigned int sum_rows_used(unsigned int g) { return g < SOP_K_REPL - 1u ? g : SOP_K_REPL - 1u; }
/* largest sum that a workgroup of a launch of g adds */
SOP_K_HD constexpr long long sum_max(unsigned int g) { return (45ll << 50) / sum_members(g, 0u); }
/* what workgroup sum v adds to its first-row word; what a complete first-row word s (of m workgroups) adds to the last row's */
SOP_K_HD constexpr unsigned long long sum_add1(long long v, long long max) { return kSumOne1 + (unsigned long long)(v < SOP_K_SUM_MIN ? SOP_K_SUM_MIN : v > max ? max : v); }
SOP_K_HD constexpr unsigned long long sum_add2(unsigned long long s, unsigned int m) { return kSumOne2 + (s - m * kSumOne1); }
constexpr long long kSumMostMembers = sum_members(SOP_K_SEARCH_MAXWG, 0u);
static_assert((45ll << 50) + kSumMostMembers * (1ll << 49) < (1ll << 56) && SOP_K_SUM_MIN + (1ll << 49) > 0, "a first-row sum stays within its 56 bits");
static_assert((SOP_K_REPL - 1) * ((45ll << 50) + (1ll << 54)) < (1ll << 60) && kSumMostMembers * SOP_K_SUM_MIN + (1ll << 54) > 0, "a last-row sum stays within its 60 bits");

/* Statistics pass of the data-derived codebook */
#define SOP_K_DD_THREADS 1024
#define SOP_K_DD_MAXBINS 8192
#define SOP_K_DD_ROWS 4              /* rows of running sums among which a launch's workgroups are divided (dd_rows()) */
#define SOP_K_DD_DONE_STRIDE 32      /* words between ticket counters: a 128-byte line each */
struct DdParams {
    const void*  W;
    const float* c;                  // null: uniform weights
    const unsigned char* block_mask; // null: every block; else [M*K/g], non-zero = the block enters
    int n_levels;                    // 0: plain mask.  L >= 1: the mask byte is a level 0..L; a block of level l >= 1 enters
                                     // histogram l-1 of L (n_bins bins each), and the result holds, for every j, the sum of
                                     // the histograms j .. L-1 (the pool of every block of level > j)
    int n_planes;                    // levels only: P >= 1 level planes, plane_stride bytes apart (one per codebook whose pools are
    long long plane_stride;          // wanted): one pass over the weights fills P * L histograms, laid out [plane][level][bin]
    long long M, K, ldw, Bk;
    long long row_step, Ms;          // every row_step-th row is used: Ms = ceil(M / row_step) rows
    long long strips, total_units, n_waves;  // total_units = strips * Ms; n_waves below 2^16
    long long units_q;               // total_units = units_q * n_waves + units_r
    unsigned int units_r;
    int n_bins;
    int n_repl;                      // copies of the 32-bit counts in a workgroup's LDS (set by the launch: 0, 1, 2, 4, 8 or 16)
    unsigned int dear_mass;          // a strip whose columns' masses sum to more is not worth emptying replicas for (dd_dear_mass)
    unsigned int n_rows;             // rows of running sums (set by the launch, dd_rows())
    unsigned long long* acc;         // [n_rows][words] running histograms of the layer (zero between calls)
    unsigned int* done;              // counters of finished rows and, a line apart, of each row's finished workgroups (zero between calls)
    long long* hist;                 // [n_bins] output
};

/* Largest sum of a strip's column masses for which 32-bit counts that have to be emptied on the way pay.  A wavefront empties its
 * replica (one of n_repl, shared by the others of the workgroup's wavefronts) every budget / sum steps: words / 64 exchanges a
 * lane, each followed by a 64-bit add, against weights_per_lane adds a step, of which each saves about a quarter of the cost
 * of such a pair.  Measured at 4096 x 11008, bf16, 16 weights a lane, 64-bit adds -> 32-bit: 1024 words 31 us -> 27 where
 * nothing is emptied, 31 where every third step is; 4096 words 34 -> 40 at every fifth step, 80 at every second. */
inline unsigned int dd_dear_mass(unsigned int words, unsigned int weights_per_lane, unsigned int n_repl)
{
    const unsigned int waves_per_repl = SOP_K_DD_THREADS / 64 / n_repl;
    const unsigned long long budget = 0xFFFFFFFFull / waves_per_repl;
    const unsigned long long m = budget * weights_per_lane * 64u / (4ull * words);
    return m < 0xFFFFFFFFull ? (unsigned int)m : 0xFFFFFFFFu;
}

/* Replicas of the 32-bit counts: one per wavefront where they take at most 64 KiB, else as many as fit; none (every weight adds to the
 * 64-bit sums) where they do not pay:
 *  - fewer than eight steps a wavefront: clearing and joining the replicas costs more than the cheaper adds save (64-bit -> 32-bit:
 *    768 x 2048, a step a wavefront, 8.8 us -> 10.4; 4096 x 4096, four steps, 18.9 -> 18.9; 8192 x 4096, eight, 25.1 -> 23.6);
 *  - level planes: part of the blocks add, to as many times the words (4 x 1024, 4096 x 11008: 31.6 -> 33.6);
 *  - no norms: every strip's mass is the largest there is, above dd_dear_mass() for all but a few bins. */
inline unsigned int dd_replicas(unsigned int words, unsigned int weights_per_lane, bool levels, bool no_norms, long long total_units, long long n_waves)
{
    if (levels || total_units < 8 * n_waves) return 0u;
    unsigned int n = SOP_K_DD_THREADS / 64;
    while (n > 1u && words * n * 4u > (64u << 10)) n /= 2u;
    if (no_norms && (64u * weights_per_lane << 20) > dd_dear_mass(words, weights_per_lane, n)) return 0u;
    return n;
}

/* Rows of running sums.  Atomics to one 128-byte line are served one after the other, about 20 ns each: 256 workgroups that end together
 * wait 5 us for their sums in one row and as long for their tickets on one counter.  Four rows take a second ticket (one more round
 * trip to memory) and the reading of four words for one, by a single workgroup at about half a nanosecond each, which many words do
 * not repay: one row -> four and eight, bf16, 2048 x 4096, 256 words 14.5 us -> 11.2, 10.7; 1024 words 15.1 -> 11.1, 11.9; 4096 words 20.4 -> 24, 27. */
inline unsigned int dd_rows(unsigned int words, unsigned int workgroups)
{
    return words <= SOP_K_DD_THREADS && workgroups >= 64u ? SOP_K_DD_ROWS : 1u;
}

/* Fits of data-derived codebooks, one histogram a workgroup (the weighted Lloyd rounds of sop_dd_fit) */
#define SOP_K_FIT_THREADS 256
#define SOP_K_FIT_MAXENT 64          /* entries of a codebook: a lane each */
#define SOP_K_FIT_OK 0
#define SOP_K_FIT_NONE 1             /* not strictly ascending in binary32, or one-sided: no codebook (SOP_EATOM) */
#define SOP_K_FIT_EMPTY 2            /* an empty histogram */
#define SOP_K_FIT_HOST 3             /* moments that 64 bits may not hold, a negative bin, or entries out of order on the way: left to the host */
struct FitParams {
    const long long* hist;           // [histograms][n_bins]
    int n_bins, n_entries, iters;
    float init[SOP_K_FIT_MAXENT];    // start grid, strictly ascending
    float* out;                      // [histograms][SOP_K_FIT_MAXENT]
    int* status;                     // [histograms]
};

/* Statistics pass of the per-layer scale shift */
#define SOP_K_FL_THREADS 1024
#define SOP_K_FL_BINS 320            /* binary exponents -160 .. 159 of sc = m * 2^e, 1/2 <= m < 1 */
struct FlParams {
    const void* W;
    long long M, K, ldw;
    long long strips, total_units, n_waves;
    int units_per_wg, units_rem;     // total_units = workgroups * units_per_wg + units_rem
    float t_pos, t_neg;              // endpoints t+ and -t- of the codebook
    float m_top;                     // m of the scale format's largest value
    unsigned long long* acc;         // [2 * SOP_K_FL_BINS] running counts (zero between calls)
    unsigned int* done;
    long long* hist;                 // [2][SOP_K_FL_BINS] output
};

/* Read-rate calibration kernel: workgroups (of 256 threads) of one launch */
#define SOP_K_PROBE_WG 2048

/* Layer-scope weight formats and the binary64 sum */
#define SOP_K_LS_MAXWG 2048
#define SOP_K_LS_MAXREP 64           /* copies of the running layer maxima */
#define SOP_K_LS_DONE_STRIDE 32      /* words between ticket counters: a 128-byte line each */
struct LsParams {
    const void*  W;                  // weights (or the binary32 array of the sum kernel)
    const float* c;                  // null: c = 1
    long long M, K, ldw;
    long long strips, total_units, n_waves;   // sum kernel: total_units = number of elements
    long long max_waves;             // wavefronts of the maxima pass
    int w_man, w_bias, w_max_code;   // weight grid ExMy
    int s_man, s_bias, s_max_code;   // scale word
    int k;
    float pow2k;
    unsigned int* maxbits;           // [SOP_K_LS_MAXREP][32], two words used: bit patterns of the largest positive / negative weight (zero between calls)
    unsigned long long* part;        // [SOP_K_LS_MAXWG][3] workgroup partials (bit patterns of doubles)
    unsigned int* done;              // [17] tickets, SOP_K_LS_DONE_STRIDE words apart: over the groups, then per group of workgroups
    double* out;                     // [4] weighted error, plain error, ||W||_c^2, scale code   (sum kernel: [1])
    uint16_t* codes;                 // optional [M*K] index into the ascending signed grid
};

/* Ranking of the blocks by a per-block score (exact selection of the scores of given ranks: nested pools) */
#define SOP_K_SEL_THREADS 256         /* pool-mask and level kernels */
#define SOP_K_CNT_THREADS 1024        /* counting kernels */
#define SOP_K_SEL_MAXLEV 8
#define SOP_K_SEL_FINE 8192          /* bins of 256 keys for the scores in [7/8, 1) in the first pass */
#define SOP_K_SEL_BINS1 (2048 - 1 + SOP_K_SEL_FINE)     /* bins of the first pass */
#define SOP_K_SEL_BINS1_PAD ((SOP_K_SEL_BINS1 + SOP_K_CNT_THREADS - 1) / SOP_K_CNT_THREADS * SOP_K_CNT_THREADS)
#define SOP_K_SEL_BINS 2048          /* one threshold: bins of a pass (11 + 11 + 10 bits of the 32-bit key); several: bins of a threshold in the second and third pass */
#define SOP_K_SEL_DONE (SOP_K_SEL_BINS1_PAD + 2 * SOP_K_SEL_MAXLEV * SOP_K_SEL_BINS)      /* tickets of the passes, a 128-byte line each */
#define SOP_K_SELM_WORDS (SOP_K_SEL_DONE + 3 * 32)      /* one set of counts and tickets of a plane */
/* One threshold of one plane of at most SOP_K_SEL_ONE_MAX scores goes through three passes of 11, 11 and 10 bits, whose digits every workgroup of the next finds for
 * itself: no pass ends in a ticket.  Against the passes of several thresholds, 2.8 M scores: cosines 27.3 us and 28.1, errors (spread over many binades) 27.0 and
 * 39.9, cosines that crowd in [3/4, 7/8) 27.1 and 38.8; 0.7 M 18.6 and 22.1, 18.4 and 30.1, 18.6 and 30.0; 8.4 M 55.0 and 42.8, 53.9 and 58.5, 54.6 and 58.7; 14.7 M 93 and 61, 90 and 80,
 * 92 and 83 (the three passes with a split that looked for three digits: 1 to 2 us more). */
#define SOP_K_SEL_ONE_MAX (8 << 20)
/* Scores of which the smaller is the better are errors and no cosines: the line lies where both ways take them as long (8.4 M 54.1 us and 59.1, 9.4 M 63.2 and 63.1, 10.4 M
 * 68.2 and 66.5; spread over the whole range of binary32, 50.2 and 57.1, 59.3 and 61.4, 63.5 and 65.1). */
#define SOP_K_SEL_ONE_ERR_MAX (9 << 20)
/* The same asked for as levels: cosines of up to 3 M scores are as fast this way (8.4 M 55 us and 43), all others faster. */
#define SOP_K_SEL_ONE_LEVELS_MAX (3 << 20)
/* Does a ranking of one threshold go through these three passes?  With no first pool wanted there is nothing to count, and its split kernel writes the whole mask without a look at the
 * scores (14.7 M 10.2 us; 17.9 by the level kernel, which reads them). */
inline bool sel_three_passes(long long n, bool levels, bool higher, bool none) { return none || n <= (levels ? SOP_K_SEL_ONE_LEVELS_MAX : higher ? SOP_K_SEL_ONE_MAX : SOP_K_SEL_ONE_ERR_MAX); }
struct SelParams {
    const float* score;              // [n]
    long long n, n_top;              // 1 <= n_top <= n (n_top == 0: all_b)
    int higher;                      // 1: a larger score ranks better
    int all_b;                       // 1: every block goes to the second pool
    unsigned int* hist;              // [3][SOP_K_SEL_BINS] digit counts of the passes (the first two are zero between calls, the last one is cleared by the first pass)
    unsigned int* found;             // [3] what the last pass hands to the split: digits of the first two passes in place, rank wanted among the keys with them, keys above them
    unsigned char* pool_b;           // [n] 1 = ranked strictly worse than the threshold
    float* tau;                      // [1] the threshold score
    long long* n_a;                  // [1] blocks that stay in the first pool
};

/* what the passes hand on, per score plane (written by the last workgroup of a pass) */
struct SelMState {
    unsigned int prefix[SOP_K_SEL_MAXLEV];       // digits of every threshold's key fixed so far
    unsigned int mask[SOP_K_SEL_MAXLEV];         // their bits; all: the key is known, or every block ranks worse
    unsigned int rank_in[SOP_K_SEL_MAXLEV];      // rank wanted among the keys with those digits
    unsigned int above[SOP_K_SEL_MAXLEV];        // keys above those digits
    int alias[SOP_K_SEL_MAXLEV];                 // first threshold with the same digits so far (its histogram is the one used)
    unsigned int open;                           // bit t: threshold t has a histogram of its own in the next pass
    unsigned long long tkey[SOP_K_SEL_MAXLEV];   // the threshold's key (2^32: every block ranks worse)
};
struct SelMParams {
    const float* score;              // [n]
    long long n;
    int higher;                      // 1: a larger score ranks better
    int n_levels;                    // thresholds, 1 .. SOP_K_SEL_MAXLEV
    long long n_top[SOP_K_SEL_MAXLEV];   // non-decreasing sizes of the first pool (0: every block goes to the second pool)
    unsigned int* hist;              // first pass [SOP_K_SEL_BINS1_PAD], second and third [MAXLEV][BINS], tickets (zero when the call starts; its last kernel clears them)
    unsigned char* level;            // [n] number of thresholds the block ranks strictly worse than
    float* tau;                      // [n_levels] threshold scores
    long long* n_a;                  // [n_levels] blocks at least as good as the threshold
    SelMState* state;                // [n_planes]
    // several score planes in one launch (blockIdx.y names the plane): plane q reads score + q * n, counts into
    // hist + q * SOP_K_SELM_WORDS and writes level + q * n, tau / n_a + q * SOP_K_SEL_MAXLEV
    int n_planes;
};

/* Packing of scale words and code payloads */
struct PackParams {
    long long Nb, Bk;                // blocks, blocks per row
    long long M, K;
    int g, n_bits;
    int wide_a, wide_b;              // 1: the atom's plane holds one byte per code (else two codes per byte)
    const uint16_t* scale_a; const uint16_t* scale_b;   // [Nb] bit 15 = sign, low bits = magnitude code
    const unsigned char* codes_a; const unsigned char* codes_b;
    const void* sel_words;           // null: single codebook
    int sel_u32, pair_q;
    int sign_pos, mag_shift, sel_pos;   // bit positions inside the container (-1: absent)
    uint16_t* words;                 // [Nb]
    unsigned char* payload;          // [Nb][g*n_bits/8]
};
#endif
