// The pruned search (Sec. VI-B) of many problems on few shapes, as a sweep over accelerators asks for it.
//
// For a fixed tiling, recomputation choice r and stationary combination every key is a monotone function of a
// candidate's DRAM traffic: DRAM energy and DRAM time grow with it, every rounded sum, product and maximum they
// pass through keeps the order, and the capacity test does not look at the combination.  Of the rows that fit,
// the one with the least traffic therefore has the least cost under every combination and every key, bit for bit
// the value that costing row by row gives.  (Rounding may give rows with more traffic the same cost: positions
// are recovered by comparing costs, not traffic.)  So the search is, per tiling,
//   1. the least traffic of each (r, f) class under the buffer capacity -- a matter of the workload's shape
//      and the capacity alone, shared by every accelerator that is searched on that shape;
//   2. the nine combinations on top of it, per accelerator.
//
// k_search_batch (batch.h) does both per problem and is bound by step 1: eight table values per row and tiling
// from LDS, 270 rows, 32 LDS cycles each.  Here step 1 is done once per shape and distinct capacity, over the rows that
// the least traffic needs (rows.h: 181 suffice), each of them under all of a round's capacities: three operations per capacity.
//
// A work item is (shape, chunk of 64 tilings), lane = tiling, one block.  The block decodes the chunk, its waves take
// an eighth of the rows each (step 1), then the accelerators one wave each (step 2).  Positions: each
// wave publishes its values, takes the launch-wide lowest ones back, and only a value that nothing published beats is
// followed up, by the block's waves in turn: the lowest class (f, combination, r), then the first row, then the first tiling that
// reach it.  Each item leaves one record per problem and key for k_pruned_finish.
//
// 64 accelerators x 8 attention shapes x 2 keys: 1.63 ms in k_search_batch, 0.20 ms here.  Of a block's 125 000 cycles (1088
// blocks, two per CU) step 1 takes 24 000, step 2 49 000 (6000 per problem and wave, four waves on a SIMD), the
// positions 23 000 (some 29 a block: ties with the optimum, not late news), the meetings of the waves the rest.  Before, 0.29 ms:
// 38 000 cycles more for the capacities of 64 problems read one after the other, rows as straight-line code on six of the
// eight waves, tile costs mode by mode and once per key, positions left to the wave whose problem it was.
// What k_search_batch keeps (keep_shared): calls whose problems share little, where this kernel's step 1 would be
// done for one accelerator at a time, and small ones, where a block's chain of problems is long against the
// chip's other blocks, and two launches of more code count (a single 1764-tiling problem: 17 us against 11).
//
// Included once by mmee.hip.
#pragma once
#include "boundary.h"

namespace mmee {

constexpr int PRUNED_THREADS = 512;          // two blocks per CU, four waves per SIMD
constexpr int PRUNED_WAVES = PRUNED_THREADS / 64;
constexpr int PRUNED_MEMBERS = 64;           // problems of one group at most
constexpr int PRUNED_ROUND = 16;             // capacities per round of a shared chunk
constexpr int PRUNED_INLINE = 3000;          // bytes of problem descriptions that ride in the kernel arguments

// A group: problems with one shape and tiling mode.  Offsets are bytes from the start of the descriptions.
struct PrunedGroup {
    uint32_t first_item, n_items;            // its work items, one block each
    uint32_t member0, n_members;             // its problems, by ascending capacity
    uint32_t n_caps, caps_off;               // the distinct capacities, words, ascending (fp64)
    uint32_t T, list_off;                    // tilings; the four divisor lists one after the other
    uint64_t key0;                           // its records in PrunedArgs::keys: [n_items][n_members][N_OBJ]
    uint32_t X[4], ndiv[4];                  // extents and divisor counts of i, k, l, j
    DigitConst dg;
    double extent[4], size[5];               // the extents, and the words of A, B, D, E, C: as fp64 they reach the kernel
                                             // in scalar registers, where converting the integers would take vector ones
};

struct PrunedMember {
    ModelConst mc;
    // MACs (times three: RF accesses) and MACs with their softmax elements, both times B*H, of the producer (repeated per j
    // tile by recomputation) and the consumer; their energies without recomputation, which no tiling changes
    double rf_words[2], mac_ops[2], e_rf0, e_mac0;
    uint32_t exact_k;                        // the DRAM time is one exact product (ModelConst::dram_k)
    uint32_t pad_;
    uint32_t slot;                           // where its N_OBJ final records and hints are
    uint32_t cap;                            // number of its capacity in the group's list
    uint32_t mask;                           // keys asked for
    uint32_t group;
};

struct PrunedArgs {
    const unsigned char *desc;               // descriptions in device memory; null: in `inl`
    uint32_t n_groups, n_items;
    uint32_t members_off;
    const uint4 *enc;                        // every encoded row (for the winner's record)
    Key *keys;                               // the items' records, group after group
    unsigned long long *hints;               // [slot][N_OBJ] lowest value published so far (bit pattern); +inf between launches
    FinalRecord *final_out;                  // [slot][N_OBJ]
    alignas(16) unsigned char inl[PRUNED_INLINE];
};

__device__ __forceinline__ ConstBytes pruned_desc(const PrunedArgs &a)
{
    if (a.desc) return as_constant(a.desc);
    return (ConstBytes)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(PrunedArgs, inl);
}

// ---- step 1: the least traffic of a class ------------------------------------------------------

// no row fits: larger than any traffic (below 2^53), still finite whatever its low word holds
__device__ __forceinline__ double nothing_fits() { return __hiloint2double(0x7fe00000, 0); }
constexpr double FITS_BELOW = 1e300;

__device__ const LeastOffsets least_dev = LEAST_OFF;

// The least traffic of a wave's piece of the rows, for this lane's tiling, under K capacities: Eq. (1), (2), (4), the mask,
// Eq. (7), the running minima.  tab: the staged compact table; all its words are whole numbers (unscaled), so the
// association is free.  As straight-line code on registers (options formed once, sums shared between rows: 4 + 3 K operations a row where
// this has 14 + 3 K) the same took a block three times as long, 60 000 cycles for nine capacities: 24 KiB of
// instructions that eight waves run once each are bound by their fetch, also where they hit the instruction cache.
template <int K>
__device__ __forceinline__ void least_traffic(const double *tab, uint32_t wave, const double (&cap)[K], double (&least)[K])
{
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
    ConstPtr<u32x8> offs = (ConstPtr<u32x8>)&least_dev.off[0][0];
    const uint32_t lo = as_constant(least_dev.lo)[wave], hi = as_constant(least_dev.hi)[wave];
    const char *col = reinterpret_cast<const char *>(tab) + (threadIdx.x & 63) * 8;
#pragma unroll
    for (int k = 0; k < K; ++k) least[k] = nothing_fits();
    u32x8 next = offs[lo];
#pragma unroll 4
    for (uint32_t i = lo; i < hi; ++i) {
        const u32x8 off = next;
        next = offs[min(i + 1, hi - 1)];
        double w[NSEL];
#pragma unroll
        for (int q = 0; q < NSEL; ++q) w[q] = *reinterpret_cast<const double *>(col + off[q]);
        const double bs = fmax(w[0] + w[2] + w[1], w[3] + w[2] + w[4]), da = w[5] + w[6] + w[7];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool fits = bs <= cap[k];
            least[k] = fmin(least[k], __hiloint2double(fits ? __double2hiint(da) : 0x7fe00000, __double2loint(da)));
        }
    }
}

// ---- step 2: an accelerator's costs on top of it -----------------------------------------------

// What the two operators contribute per stationary mode, words and cycles over all their tile stages, without
// recomputation (which multiplies the first operator's by D_J): tile_cost_f64 times the number of tiles, with the
// products taken apart.  A tile's extent times its count is the matrix's, so what is left of a mode is the operands' sizes
// times one factor per dimension -- D * ceil(G / width), nine in all instead of eighteen quotients -- and sums of two
// or three such terms, some of them common to modes.  All of them are whole numbers below 2^53: the values are the same whatever
// the association, and fused operations are exact.  58 operations instead of about 130.
struct StageTerms { double br1[3], cy1[3], br2[3], cy2[3]; };

__device__ __forceinline__ StageTerms stage_terms(const TilingF &v, const double (&X)[4], const double (&size)[5], const ModelConst &mc)
{
    // D * ceil(G / b); the rounded quotient of G - 1/2 is never a whole number (cdiv_f64)
    auto folds = [&](int q, double rcp_b) { return v.D[q] * __builtin_ceil((v.G[q] - 0.5) * rcp_b); };
    const double row_i = folds(DI, mc.rcp_rows), row_k = folds(DK, mc.rcp_rows), row_l = folds(DL, mc.rcp_rows);
    const double col_k = folds(DK, mc.rcp_cols), col_l = folds(DL, mc.rcp_cols), col_j = folds(DJ, mc.rcp_cols);
    const double wide_k = folds(DK, mc.rcp_cols_g), wide_l = folds(DL, mc.rcp_cols_g), wide_j = folds(DJ, mc.rcp_cols_g);
    const double A = size[0], B = size[1], D = size[2], E = size[3], C = size[4];
    const double a_wide = A * wide_l, b_row = B * row_i, c_wide = C * wide_j, d_row = D * row_i, row_col = row_i * col_l;
    StageTerms t;
    // m x r x n = I x K x L: weight, input, output stationary
    t.br1[0] = __builtin_fma(B, v.D[DI], __builtin_fma(C, row_k, a_wide));  t.cy1[0] = X[DI] * (row_k * col_l);
    t.br1[1] = __builtin_fma(A, v.D[DL], __builtin_fma(C, wide_k, b_row));  t.cy1[1] = X[DL] * (row_i * col_k);
    t.br1[2] = __builtin_fma(C, v.D[DK], a_wide + b_row);                   t.cy1[2] = X[DK] * row_col;
    // I x L x J
    t.br2[0] = __builtin_fma(D, v.D[DI], __builtin_fma(E, row_l, c_wide));  t.cy2[0] = X[DI] * (row_l * col_j);
    t.br2[1] = __builtin_fma(C, v.D[DJ], __builtin_fma(E, wide_l, d_row));  t.cy2[1] = X[DJ] * row_col;
    t.br2[2] = __builtin_fma(E, v.D[DL], c_wide + d_row);                   t.cy2[2] = X[DL] * (row_i * col_j);
    return t;
}

// max(compute cycles, buffer<->RF time) of combination s1 + 3 s2, without the factor c_lat: a minimum of such times times
// c_lat is the minimum of the products, bit for bit.  POW2: the buffer bandwidth is a power of two, gb1 and gb2 are the
// two operators' shares of the time (br1, br2 times one exact constant).  r: the first operator's share once per j tile.
template <bool POW2>
__device__ __forceinline__ double combo_time(const StageTerms &t, const double (&gb1)[3], const double (&gb2)[3], const ModelConst &mc, double dj, int r, int c)
{
    auto both = [&](double one, double two) { return r ? __builtin_fma(dj, one, two) : one + two; };
    const double cyc = both(t.cy1[c % 3], t.cy2[c / 3]);
    if constexpr (POW2) return fmax(cyc, both(gb1[c % 3], gb2[c / 3]));
    else return fmax(cyc, buffer_time_general(mc, both(t.br1[c % 3], t.br2[c / 3])));
}

// the row side of a candidate's costs, from its traffic; +inf both when no row fits
struct RowSide { double words, e_part, time; };
__device__ __forceinline__ RowSide row_side(const ModelConst &mc, double least, bool exact_k = false)
{
    RowSide rs;
    const bool fits = least < FITS_BELOW;
    const double d = fits ? least : 0.0, over = fits ? 0.0 : pos_inf();
    rs.words = mc.BH * d;
    rs.e_part = fmax(mc.e_dram * rs.words, over);
    rs.time = fmax(exact_k ? rs.words * mc.dram_k : dram_time_general(mc, d), over);
    return rs;
}
__device__ __forceinline__ double energy_of(const ModelConst &mc, const RowSide &rs, double br, double e_rf, double e_mac)
{
    double en = rs.e_part + mc.e_gb * __builtin_fma(mc.BH, br, rs.words);     // (whole numbers: exact)
    en = en + e_rf;
    return en + e_mac;
}

// energy and latency of combination c under every class, from the classes' row sides.  Class numbers go up with the
// index: f, then the combination, then r (f = 0: the combination; f = 1: 9 + 2 * combination + r).  One combination
// per call, in loops that are not unrolled: nine of them side by side do not fit the registers.
template <class Use>
__device__ __forceinline__ void each_class(const TilingF &v, const double (&X)[4], const ModelConst &mc, const RowSide (&rs)[LEAST_CLASSES],
                                           uint32_t c, Use &&use)
{
    double br1, cy1, br2, cy2;
    tile_cost_f64(v.G[DI], v.G[DK], v.G[DL], c % 3, mc, br1, cy1);
    tile_cost_f64(v.G[DI], v.G[DL], v.G[DJ], c / 3, mc, br2, cy2);
#pragma unroll
    for (uint32_t r = 0; r < 2; ++r) {
        const ComboTerms ct = combo_terms_from(v, X, mc, r, br1, cy1, br2, cy2);
#pragma unroll
        for (uint32_t g = r ? 2 : 0; g < (r ? 3u : 2u); ++g)
            use(g == 0 ? c : 9u + 2u * c + r, energy_of(mc, rs[g], ct.br, ct.e_rf_part, ct.e_mac_part), fmax(rs[g].time, ct.lat_part));
    }
}

// key o of a candidate as a (primary, secondary) pair; the secondary is 0 for the scalar keys
__device__ __forceinline__ void key_values(uint32_t o, double en, double lat, double &kp, double &ks)
{
    kp = o == MMEE_OBJ_ENERGY ? en : (o == MMEE_OBJ_EDP ? en * lat : lat);
    ks = o == MMEE_OBJ_LATENCY_THEN_ENERGY ? en : 0.0;
}

// a wave's best of one key: value, lowest class that reaches it, and the tilings (lanes) that do in that class
struct ClassBest {
    double p, s;
    uint32_t code;                            // 0xFFFFFFFF: nothing feasible
    unsigned long long lanes;
};

__device__ __forceinline__ void class_of_code(uint32_t code, uint32_t &cls, uint32_t &combo)
{
    cls = code < 9 ? 0u : 1u + ((code - 9) & 1);
    combo = code < 9 ? code : (code - 9) / 2;
}

// The first row (index order) of class b.code in which one of the tilings `b.lanes` reaches (b.p, b.s), at its lowest
// such tiling: together the lowest index that does.  Rows are costed with the staged table.  The row's place in the
// class list and the tiling's lane; row 0xFFFFFFFF: none.
struct Found { uint32_t row, lane; };
__device__ __forceinline__ Found first_row(const double *tab, const ComboTerms &ct, const ModelConst &mc, uint32_t nt, uint32_t o,
                                           const ClassBest &b, uint32_t row_lo, uint32_t n_rows)
{
    const uint4 *offs = reinterpret_cast<const uint4 *>(&kept_dev.off[0][0]);
    typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
    const uint32_t lane = threadIdx.x & 63;
    Found f = {0xFFFFFFFFu, 0};
    unsigned long long cands = b.lanes;
    // does the row with these offsets reach the value for the tiling in column `col`?
    auto reaches = [&](const char *col, const uint32_t (&off)[NSEL], double cap, double br, double time, double rf, double mac) {
        double w[NSEL];
#pragma unroll
        for (int k = 0; k < NSEL; ++k) w[k] = *reinterpret_cast<const double *>(col + off[k]);
        const bool ok = fmax(w[0] + w[2] + w[1], w[3] + w[2] + w[4]) <= cap;      // Eq. (1), (2), (4)
        const RowSide rr = row_side(mc, ok ? w[5] + w[6] + w[7] : nothing_fits());  // Eq. (7)
        double kp, ks;
        key_values(o, energy_of(mc, rr, br, rf, mac), fmax(rr.time, time), kp, ks);
        return kp == b.p && ks == b.s;
    };
    if (2u * (uint32_t)__popcll(cands) <= n_rows) {
        // few tilings: one by one with lane = row, 64 rows of the class at a time
        while (cands && f.row != 0) {
            const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)__ffsll((long long)cands) - 1u);
            cands &= cands - 1;
            const char *col = reinterpret_cast<const char *>(tab) + l * 8;
            const double br_l = lane_value_f64(ct.br, l), time_l = lane_value_f64(ct.lat_part, l);
            const double rf_l = lane_value_f64(ct.e_rf_part, l), mac_l = lane_value_f64(ct.e_mac_part, l);
#pragma unroll 1
            for (uint32_t i0 = 0; i0 < n_rows && i0 < f.row; i0 += 64) {
                const uint32_t i = row_lo + min(i0 + lane, n_rows - 1);
                const uint4 oa = offs[2 * i], ob = offs[2 * i + 1];
                const uint32_t off[NSEL] = {oa.x, oa.y, oa.z, oa.w, ob.x, ob.y, ob.z, ob.w};
                const unsigned long long hits = __ballot(reaches(col, off, mc.cap_words, br_l, time_l, rf_l, mac_l) && i0 + lane < n_rows);
                if (!hits) continue;
                const uint32_t at = i0 + (uint32_t)__ffsll((long long)hits) - 1u;
                if (at < f.row) { f.row = at; f.lane = l; }  // ascending tilings: the lower one stays on equal rows
                break;
            }
        }
    } else {
        // many: all at once, row by row; the first rows reach it where the cost hangs on something else than traffic
        const double cap = lane < nt ? mc.cap_words : -1.0;
        const char *col = reinterpret_cast<const char *>(tab) + lane * 8;
        ConstPtr<u32x8> list = (ConstPtr<u32x8>)(&kept_dev.off[row_lo][0]);
        u32x8 next = list[0];
#pragma unroll 1
        for (uint32_t i = 0; i < n_rows; ++i) {
            const uint32_t off[NSEL] = {next[0], next[1], next[2], next[3], next[4], next[5], next[6], next[7]};
            next = list[min(i + 1, n_rows - 1)];
            const unsigned long long hits = __ballot(reaches(col, off, cap, ct.br, ct.lat_part, ct.e_rf_part, ct.e_mac_part));
            if (!hits) continue;
            f.row = i;
            f.lane = (uint32_t)__ffsll((long long)hits) - 1u;
            break;
        }
    }
    return f;
}

// where a class's rows are in the lists
__device__ __forceinline__ void rows_of_class(uint32_t cls, uint32_t &first, uint32_t &n)
{
    first = cls == 0 ? KEPT.first[0] : (cls == 1 ? KEPT.first[1] : KEPT.first[2]);
    n = cls == 0 ? KEPT.rows[0] : (cls == 1 ? KEPT.rows[1] : KEPT.rows[2]);
}

// ---- many problems: chunks of a shape, shared by its accelerators -------------------------------
// Capacities are taken PRUNED_ROUND at a time, all of a round by every wave on its eighth of the rows (least_traffic).
__global__ __launch_bounds__(PRUNED_THREADS, 4) void k_search_pruned(PrunedArgs a)
{
    __shared__ double tab[KEPT_LINES * PRUNED_TC];           // recovery: entry-major, lane = tiling: conflict-free as it is
    __shared__ double gd[8 * PRUNED_TC];                     // the chunk's boundary vectors: G[0..3], D[0..3] per tiling
    __shared__ double least[PRUNED_ROUND * LEAST_CLASSES][PRUNED_TC];
    __shared__ uint32_t div_lds[4 * MAXDIV];                 // the group's divisor lists
    // per problem of the group and key: the value, its class and tilings
    __shared__ Key best[PRUNED_MEMBERS][N_OBJ];
    __shared__ unsigned long long lanes_of[PRUNED_MEMBERS][N_OBJ];
    __shared__ uint32_t code_of[PRUNED_MEMBERS][N_OBJ];
    __shared__ unsigned char follow_list[PRUNED_MEMBERS * N_OBJ];     // problems and keys whose position is wanted
    __shared__ uint32_t n_follow;

    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t item = blockIdx.x;
    ConstBytes desc = pruned_desc(a);
    // the item's group: the last one whose first item is not beyond it
    uint32_t gi;
    {
        uint32_t lo = 0, hi = a.n_groups;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (((ConstPtr<uint32_t>)(desc + mid * sizeof(PrunedGroup)))[0] <= item) lo = mid; else hi = mid;
        }
        gi = lo;
    }
    const PrunedGroup G = read_const<PrunedGroup>(desc + gi * sizeof(PrunedGroup));
    ConstBytes members = desc + a.members_off + G.member0 * sizeof(PrunedMember);
    ConstF64 caps = (ConstF64)(desc + G.caps_off);
    {
        ConstPtr<uint32_t> lists = (ConstPtr<uint32_t>)(desc + G.list_off);
        for (uint32_t k = threadIdx.x; k < G.ndiv[0] + G.ndiv[1] + G.ndiv[2] + G.ndiv[3]; k += PRUNED_THREADS) div_lds[k] = lists[k];
    }
    const double (&X)[4] = G.extent;
    __syncthreads();

    const uint32_t t0 = (item - G.first_item) * PRUNED_TC, nt = min((uint32_t)PRUNED_TC, G.T - t0);
    // ---- decode: dimension q of every tiling of the chunk by wave q (beyond the chunk: its last
    // tiling once more, masked out below)
    if (wave < 4) {
        // (by scalar loads at wave's own offset: indexed as an array the description would move to scratch memory)
        ConstBytes Gp = desc + gi * sizeof(PrunedGroup);
        auto f64_at = [&](size_t off) { return ((ConstF64)(Gp + off))[wave]; };
        const double extent = f64_at(offsetof(PrunedGroup, extent));
        const uint32_t list0 = (wave > 0 ? G.ndiv[0] : 0u) + (wave > 1 ? G.ndiv[1] : 0u) + (wave > 2 ? G.ndiv[2] : 0u);
        const uint32_t digit = digit_of(t0 + min(lane, nt - 1), f64_at(offsetof(PrunedGroup, dg) + offsetof(DigitConst, rcp_radix)),
                                        f64_at(offsetof(PrunedGroup, dg) + offsetof(DigitConst, rcp_n)),
                                        ((ConstPtr<uint32_t>)(Gp + offsetof(PrunedGroup, ndiv)))[wave]);
        const double g = (double)div_lds[list0 + digit];
        gd[wave * PRUNED_TC + lane] = g;
        gd[(4 + wave) * PRUNED_TC + lane] = whole_quotient(extent, g);
    }
    __syncthreads();
    // Read again by every part, and by every problem of step 2: kept in registers, the tiling and the products that
    // problems share would spill what a problem needs (2.5 GB of scratch traffic per sweep, 0.47 ms; 0.3 GB as it is).
    auto this_tiling = [&]() {
        TilingF v;
        uint32_t l = lane;
        asm volatile("" : "+v"(l));
#pragma unroll
        for (int q = 0; q < 4; ++q) { v.G[q] = gd[q * PRUNED_TC + l]; v.D[q] = gd[(4 + q) * PRUNED_TC + l]; }
        return v;
    };
    // ---- the table that the recovery of positions reads
    stage_kept(tab + lane, wave, this_tiling(), G.size, 1.0);

    // members are sorted by capacity: a round's members follow those of the round before
    uint32_t m_lo = 0;
    // lane m: the capacity of problem m (read one after the other, 64 of them took a quarter of the kernel)
    static_assert(PRUNED_MEMBERS <= 64, "a lane per problem");
    const uint32_t cap_of_member =
        *reinterpret_cast<const uint32_t *>((const char *)(members + min(lane, G.n_members - 1) * sizeof(PrunedMember) + offsetof(PrunedMember, cap)));
    if (threadIdx.x == 0) n_follow = 0;
#pragma unroll 1
    for (uint32_t cap0 = 0; cap0 < G.n_caps; cap0 += PRUNED_ROUND) {
        // ---- step 1.  Every wave takes an eighth of the rows, all of one class, under all of the round's capacities; the waves
        // of a class meet in the LDS minima (no row's traffic: nothing_fits, and bit patterns order like the values)
        const uint32_t n_caps = min(G.n_caps - cap0, (uint32_t)PRUNED_ROUND);
        for (uint32_t k = threadIdx.x; k < n_caps * LEAST_CLASSES * PRUNED_TC; k += PRUNED_THREADS) (&least[0][0])[k] = nothing_fits();
        __syncthreads();                                     // (the staged table is there, too)
        auto step1 = [&](auto most) {
            constexpr int K = decltype(most)::value;
            double cap[K], l[K];
#pragma unroll
            for (uint32_t k = 0; k < K; ++k) cap[k] = caps[cap0 + min(k, n_caps - 1)];
            least_traffic<K>(tab, wave, cap, l);
            const uint32_t cls = as_constant(least_dev.cls)[wave];
#pragma unroll
            for (uint32_t k = 0; k < K; ++k)
                if (k < n_caps)
                    (void)__hip_atomic_fetch_min(reinterpret_cast<unsigned long long *>(&least[k * LEAST_CLASSES + cls][lane]),
                                                 (unsigned long long)__double_as_longlong(l[k]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        };
        if (n_caps <= 2) step1(std::integral_constant<int, 2>{});
        else if (n_caps <= 6) step1(std::integral_constant<int, 6>{});
        else if (n_caps <= 10) step1(std::integral_constant<int, 10>{});
        else step1(std::integral_constant<int, PRUNED_ROUND>{});
        __syncthreads();
        const uint32_t m_hi = (uint32_t)__popcll(__ballot(lane < G.n_members && cap_of_member < cap0 + PRUNED_ROUND));

        // ---- step 2.  This wave's problems: wave, wave + 8, ..., at most eight.  Lane 4 m + o looks after key o of the
        // m-th: it holds what has been published of it when the step begins; a value above that needs no class.
        const uint32_t m_first = m_lo + wave;
        const uint32_t my_j = m_first + (lane / N_OBJ) * PRUNED_WAVES;
        const bool my_key = lane < (PRUNED_MEMBERS / PRUNED_WAVES) * N_OBJ && my_j < m_hi;
        unsigned long long *my_hint = a.hints;
        double seen = inf;
        if (my_key) {
            my_hint += (uint64_t)((ConstPtr<uint32_t>)(members + my_j * sizeof(PrunedMember) + offsetof(PrunedMember, slot)))[0] * N_OBJ + lane % N_OBJ;
            seen = __longlong_as_double((long long)__hip_atomic_load(my_hint, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
#pragma unroll 1
        for (uint32_t j = m_first, m = 0; j < m_hi; j += PRUNED_WAVES, ++m) {
            const PrunedMember mb = read_const<PrunedMember>(members + j * sizeof(PrunedMember));
            const ModelConst &mc = mb.mc;
            RowSide rs[LEAST_CLASSES];
            auto row_sides = [&](bool exact_k) {
#pragma unroll
                for (uint32_t g = 0; g < LEAST_CLASSES; ++g) {
                    const double d = least[(mb.cap - cap0) * LEAST_CLASSES + g][lane];
                    rs[g] = row_side(mc, lane < nt ? d : nothing_fits(), exact_k);
                }
            };
            if (mb.exact_k) row_sides(true);
            else row_sides(false);
            auto keep = [&](uint32_t o, double p, double s, uint32_t code, bool reached) {
                const uint32_t low = __builtin_amdgcn_readfirstlane(wave_min_u32(reached ? code : 0xFFFFFFFFu));
                const unsigned long long who = __ballot(reached && code == low);
                if (lane == 0) {
                    best[j][o].p = p; best[j][o].s = s; best[j][o].idx = ~0ull;
                    lanes_of[j][o] = who;
                    code_of[j][o] = low;
                }
            };
            auto beaten = [&](uint32_t o, double p) {
                const double s = lane_value_f64(seen, m * N_OBJ + o);
                if (p < inf && !(p > s)) return false;
                if (lane == 0) { best[j][o].p = inf; best[j][o].s = 0.0; best[j][o].idx = ~0ull; }
                return true;
            };
            if (mb.mask & 3) {
              const TilingF tiling = this_tiling();
              const StageTerms t = stage_terms(tiling, X, G.size, mc);
              const double dj = tiling.D[DJ];
              if (mb.mask & 1) {
                // the energy grows with the buffer<->RF words: the least of them decides
                const double br1 = fmin(fmin(t.br1[0], t.br1[1]), t.br1[2]), br2 = fmin(fmin(t.br2[0], t.br2[1]), t.br2[2]);
                const double e_rf1 = mc.e_rf * __builtin_fma(dj, mb.rf_words[0], mb.rf_words[1]);
                const double e_mac1 = mc.e_mac * __builtin_fma(dj, mb.mac_ops[0], mb.mac_ops[1]);
                const double val = fmin(fmin(energy_of(mc, rs[0], br1 + br2, mb.e_rf0, mb.e_mac0), energy_of(mc, rs[1], br1 + br2, mb.e_rf0, mb.e_mac0)),
                                        energy_of(mc, rs[2], __builtin_fma(dj, br1, br2), e_rf1, e_mac1));
                const double p = uniform_f64(wave_min_f64(val));
                // (its class is looked for below, where it matters: rarely)
                if (!beaten(0, p) && lane == 0) { best[j][0].p = p; best[j][0].s = 0.0; best[j][0].idx = ~0ull; }
              }
              if (mb.mask & 2) {
                auto latency = [&](auto pow2) {
                    constexpr bool POW2 = decltype(pow2)::value;
                    double gb1[3], gb2[3], fastest[2] = {inf, inf};
#pragma unroll
                    for (int s = 0; s < 3; ++s) { gb1[s] = t.br1[s] * mc.gb_k; gb2[s] = t.br2[s] * mc.gb_k; }
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
#pragma unroll
                        for (int c = 0; c < 9; ++c) fastest[r] = fmin(fastest[r], combo_time<POW2>(t, gb1, gb2, mc, dj, r, c));
                        fastest[r] = mc.c_lat * fastest[r];
                    }
                    const double val = fmin(fmin(fmax(rs[0].time, fastest[0]), fmax(rs[1].time, fastest[0])), fmax(rs[2].time, fastest[1]));
                    const double p = uniform_f64(wave_min_f64(val));
                    if (!beaten(1, p)) {
                        // no candidate is below p: one has it if neither of its two parts exceeds it
                        // (descending codes: the last one met is the lowest)
                        uint32_t low[2] = {9, 9};
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int c = 8; c >= 0; --c) low[r] = mc.c_lat * combo_time<POW2>(t, gb1, gb2, mc, dj, r, c) <= p ? (uint32_t)c : low[r];
                        uint32_t code = rs[2].time <= p && low[1] < 9 ? 10u + 2u * low[1] : 0xFFFFFFFFu;
                        code = rs[1].time <= p && low[0] < 9 ? min(code, 9u + 2u * low[0]) : code;
                        code = rs[0].time <= p && low[0] < 9 ? low[0] : code;
                        keep(1, p, 0.0, code, val == p);
                    }
                };
                if (mc.gb_pow2) latency(std::true_type{});
                else latency(std::false_type{});
              }
            }
            // the other two keys: candidate by candidate, one key at a time
#pragma unroll 1
            for (uint32_t o = 2; o < N_OBJ; ++o) {
                if (!((mb.mask >> o) & 1)) continue;
                const TilingF v = this_tiling();
                double mine_p = inf, mine_s = inf;
                uint32_t code = 0xFFFFFFFFu;
#pragma unroll 1
                for (uint32_t c = 0; c < 9; ++c)
                    each_class(v, X, mc, rs, c, [&](uint32_t cls_code, double en, double lat) {
                        double kp, ks;
                        key_values(o, en, lat, kp, ks);
                        const bool same = kp == mine_p && ks == mine_s, lower = kp < mine_p || (kp == mine_p && ks < mine_s);
                        mine_p = lower ? kp : mine_p;
                        mine_s = lower ? ks : mine_s;
                        code = lower || (same && cls_code < code) ? cls_code : code;
                    });
                const double p = uniform_f64(wave_min_f64(mine_p));
                if (beaten(o, p)) continue;
                const double sec = o == MMEE_OBJ_LATENCY_THEN_ENERGY ? uniform_f64(wave_min_f64(mine_p == p ? mine_s : inf)) : 0.0;
                keep(o, p, sec, code, mine_p == p && mine_s == sec);
            }
            if (lane < N_OBJ && !((mb.mask >> lane) & 1)) { best[j][lane].p = inf; best[j][lane].s = 0.0; best[j][lane].idx = ~0ull; }
        }
        // ---- publish, all of the wave's values at once; what something lower was published for is dropped here
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        bool up = false;
        if (my_key && best[my_j][lane % N_OBJ].p < inf) {
            const unsigned long long bits = (unsigned long long)__double_as_longlong(best[my_j][lane % N_OBJ].p);
            up = bits <= __hip_atomic_fetch_min(my_hint, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!up) best[my_j][lane % N_OBJ].p = inf;
        }
        // ---- positions of the others, dealt out to the waves: those of a wave's own problems can be many
        // (a wave then worked ten times as long as the rest)
        {
            const unsigned long long follow = __ballot(up);
            uint32_t at = 0;
            if (lane == 0 && follow) at = __hip_atomic_fetch_add(&n_follow, (uint32_t)__popcll(follow), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            at = __builtin_amdgcn_readfirstlane(at) + (uint32_t)__popcll(follow & ((1ull << lane) - 1));
            if (up) follow_list[at] = (unsigned char)(my_j * N_OBJ + lane % N_OBJ);
        }
        __syncthreads();
        const uint32_t follows = __builtin_amdgcn_readfirstlane(n_follow);
        for (uint32_t at = wave; at < follows; at += PRUNED_WAVES) {
            const uint32_t which = __builtin_amdgcn_readfirstlane((uint32_t)follow_list[at]);
            const uint32_t j = which / N_OBJ, o = which % N_OBJ;
            const PrunedMember mb = read_const<PrunedMember>(members + j * sizeof(PrunedMember));
            ClassBest b;
            b.p = uniform_f64(best[j][o].p); b.s = uniform_f64(best[j][o].s);
            b.code = __builtin_amdgcn_readfirstlane(code_of[j][o]);
            b.lanes = uniform_u64(lanes_of[j][o]);
            if (o == MMEE_OBJ_ENERGY) {
                // the lowest class in which one of these tilings has it
                RowSide rs[LEAST_CLASSES];
#pragma unroll
                for (uint32_t g = 0; g < LEAST_CLASSES; ++g) {
                    const double d = least[(mb.cap - cap0) * LEAST_CLASSES + g][lane];
                    rs[g] = row_side(mb.mc, lane < nt ? d : nothing_fits());
                }
                const TilingF v = this_tiling();
                const StageTerms t = stage_terms(v, X, G.size, mb.mc);
                const double dj = v.D[DJ];
                const double e_rf1 = mb.mc.e_rf * __builtin_fma(dj, mb.rf_words[0], mb.rf_words[1]);
                const double e_mac1 = mb.mc.e_mac * __builtin_fma(dj, mb.mac_ops[0], mb.mac_ops[1]);
                uint32_t low[LEAST_CLASSES] = {9, 9, 9};     // (descending combinations: the last one met is the lowest)
#pragma unroll
                for (int c = 8; c >= 0; --c) {
                    const double br = t.br1[c % 3] + t.br2[c / 3];
                    low[0] = energy_of(mb.mc, rs[0], br, mb.e_rf0, mb.e_mac0) == b.p ? (uint32_t)c : low[0];
                    low[1] = energy_of(mb.mc, rs[1], br, mb.e_rf0, mb.e_mac0) == b.p ? (uint32_t)c : low[1];
                    low[2] = energy_of(mb.mc, rs[2], __builtin_fma(dj, t.br1[c % 3], t.br2[c / 3]), e_rf1, e_mac1) == b.p ? (uint32_t)c : low[2];
                }
                uint32_t code = low[2] < 9 ? 10u + 2u * low[2] : 0xFFFFFFFFu;
                code = low[1] < 9 ? min(code, 9u + 2u * low[1]) : code;
                code = low[0] < 9 ? low[0] : code;
                b.code = __builtin_amdgcn_readfirstlane(wave_min_u32(code));
                b.lanes = __ballot(code == b.code);
            }
            uint32_t cls, combo, row_lo, n_rows;
            class_of_code(b.code, cls, combo);
            rows_of_class(cls, row_lo, n_rows);
            const ComboTerms ct = combo_terms(this_tiling(), X, mb.mc, cls == 2u, combo % 3, combo / 3);
            const Found f = first_row(tab, ct, mb.mc, nt, o, b, row_lo, n_rows);
            if (lane == 0) {
                if (f.row == 0xFFFFFFFFu) best[j][o].p = inf;        // cannot happen: the value came from here
                else {
                    const uint32_t row = index_row_base(kept_dev.number[row_lo + f.row]) + 30000u * (combo % 3) + 90000u * (combo / 3);
                    best[j][o].idx = (uint64_t)t0 + f.lane + (uint64_t)G.T * row;
                }
            }
        }
        m_lo = m_hi;
        __syncthreads();                                      // the round's minima and its list are free again
        if (threadIdx.x == 0) n_follow = 0;
    }
    // ---- the item's records
    for (uint32_t k = threadIdx.x; k < G.n_members * N_OBJ; k += PRUNED_THREADS)
        a.keys[G.key0 + (uint64_t)(item - G.first_item) * (G.n_members * N_OBJ) + k] = best[k / N_OBJ][k % N_OBJ];
}

// After the search: one block per problem reduces the problem's records, one per item of its group, and writes the
// winner's full cost record and mapping.
__global__ __launch_bounds__(256) void k_pruned_finish(PrunedArgs a)
{
    __shared__ Key wave_best[N_OBJ][4];
    __shared__ DivTable dv_s;
    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    ConstBytes desc = pruned_desc(a);
    const PrunedMember mb = read_const<PrunedMember>(desc + a.members_off + blockIdx.x * sizeof(PrunedMember));
    const PrunedGroup G = read_const<PrunedGroup>(desc + mb.group * sizeof(PrunedGroup));
    {
        // the packed lists back into the table form the decoding helpers take
        ConstPtr<uint32_t> list = (ConstPtr<uint32_t>)(desc + G.list_off);
        uint32_t first = 0;
        for (int q = 0; q < 4; ++q) {
            for (uint32_t k = threadIdx.x; k < G.ndiv[q]; k += 256) dv_s.div[q][k] = list[first + k];
            first += G.ndiv[q];
        }
        if (threadIdx.x < 4) { dv_s.X[threadIdx.x] = G.X[threadIdx.x]; dv_s.ndiv[threadIdx.x] = G.ndiv[threadIdx.x]; }
    }
    const uint32_t member = blockIdx.x - G.member0;
#pragma unroll
    for (int o = 0; o < N_OBJ; ++o) {
        if (!((mb.mask >> o) & 1)) continue;
        Key k; k.p = inf; k.s = 0.0; k.idx = ~0ull;
        for (uint32_t b = threadIdx.x; b < G.n_items; b += 256) {
            const Key c = a.keys[G.key0 + ((uint64_t)b * G.n_members + member) * N_OBJ + o];
            if (key_less(c, k)) k = c;
        }
        k = wave_min(k);
        if (lane == 0) wave_best[o][wave] = k;
    }
    __syncthreads();
    if (threadIdx.x < N_OBJ) a.hints[(uint64_t)mb.slot * N_OBJ + threadIdx.x] = INF_BITS;     // for the next launch
    if (threadIdx.x < N_OBJ && ((mb.mask >> threadIdx.x) & 1)) {
        const int o = threadIdx.x;
        Key k = wave_best[o][0];
        for (int wv = 1; wv < 4; ++wv)
            if (key_less(wave_best[o][wv], k)) k = wave_best[o][wv];
        mmee_result res;
        winner_record(a.enc, dv_s, mb.mc, k, res);
        write_record(a.final_out + (uint64_t)mb.slot * N_OBJ + o, k, res);
    }
}

}  // namespace mmee
