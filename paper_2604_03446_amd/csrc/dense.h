// Exhaustive search over the full row set, one or two keys a pass: k_search_dense, one launch per pass.
//
// The rows of one (order, r, f) class are the 5^4 buffering levels, and their terms split by operand: what A's level p_A
// adds to a footprint and to the traffic does not depend on the other levels (rows.h).  So a lane is a tiling, a
// wave takes the 125 rows of a (class, p_E) task, everything about a row is wave-uniform, and a row is an (A, B) part
// next to a (D, E) part and C's.  All of these sums are exact integers below 2^53 (the host refuses workloads where
// they are not), so their association is free, and a row needs no footprint of its own: it fits if what A and B take does
// not exceed what the (D, E) part and C leave of the capacity.
//
// Which rows fit.  An operand's footprint never shrinks with its level (levels_ascend below, checked by the compiler), so the
// rows of a task that fit a tiling are a staircase: where (p_A, p_B) does not fit beside p_D = 0 for any tiling of the wave, no
// larger p_A does, and where p_A = 0 does not, no larger p_B; and p_D ends at the first row that fits none.  A step (p_A, p_B)
// whose five rows all fit every tiling -- two comparisons -- takes them as straight-line code without a mask.  A row over
// capacity costs +inf, whatever the combination: its lanes are masked out of the nine combinations, a wave none of
// whose tilings it fits passes over it.
//
// Lanes.  A chunk is 64 neighbours in an order of the tilings of its own: k's divisors fastest, then j's, l's, i's.  In attention
// and in feed-forward layers i and l are the long extents, so the footprints of neighbours differ least, and a row fits all
// of a wave or nothing of it more often than in index order (counted over the whole space: 12544 tilings of 8192 x 128, buffer 8 MiB,
// 62.7 % of the wave-rows run, 92 % of these full, against 72.1 and 48 % in index order; 10692 tilings of 2048 x 768 x 3072 x 768,
// 1 MiB, 10.9 %, 40 % of these full, against 12.1 and 10 %).
//
// Tables.  Single operands' terms are 41 values a tiling, the nine combinations' constants 40: a block forms them for its
// chunk straight from the divisor lists, in LDS, and nothing per tiling is in memory.  (Sums of pairs, 123 values,
// were built by a launch of their own and staged per eight tasks: 10 to 15 us ahead of the search and 62 KB per item.)
//
// A block's item is a chunk and a range of its tasks; the waves take them one by one (a task's work varies with what fits: in
// rounds of eight the waves wait for the slowest).  Persistent blocks, items from a global counter, the last ones small.
//
// What it measured, us a call, before (rows tested one by one, tables from memory, eight tasks an item) and now: 12544 tilings (8192 x
// 128, all divisors, 8 MiB), energy 338 and 239; 4900 tilings (512 x 64, 256 KiB), energy and latency 295 and 246;
// 10692 tilings (2048 x 768 x 3072 x 768, 1 MiB), energy 218 and 86.  Vector issue bounds it where most rows fit (84 % of the
// first one's cycles); small buffers are bound by what a task costs before its first row.
//
// Argmin: lazy.  Only minima are kept; a position is recovered where the optimum can be, by costing the task's rows again.
//
// Included once by mmee.hip.
#pragma once
#include "boundary.h"

namespace mmee {

constexpr int DENSE_THREADS = 512;           // eight waves, two blocks per CU
constexpr int DENSE_BLOCKS_PER_CU = 2;
constexpr int DENSE_WAVES = DENSE_THREADS / 64;
// The last tasks of an item are handed out in fifths (one p_B each; two keys: one p_D): a whole one takes a wave up to 19 us, which the
// others would wait for.  Eight of them (fifths cost 7 to 16 % more) / four / two: 258 / 251 / 249 us (12544 tilings, energy), 265 / 259 / 261
// (4900 tilings, energy and latency), 69 / 69 / 73 (1225 tilings).
constexpr uint32_t DENSE_FIFTHS = 4;
constexpr uint32_t DENSE_DIVS = 560;         // divisors of a problem: 240 + 240 + 72 + 1 at most (T <= 2^22)

// the lines of the per-tiling table, 64 tilings each: per operand the footprint's and the traffic's four options (layout.h)
constexpr uint32_t DENSE_BS = 0, DENSE_DA = 20, DENSE_ZERO = 40, DENSE_LINES = 41;     // BS: A, B, D, E, C; DA: A, B, D, E, C
constexpr uint32_t DENSE_LINE = 64 * 8;      // bytes of a line

// the constants of a tiling and recomputation choice r: the buffer<->RF words (B*H-scaled; regrouped: their energy, the second
// operator's with all that no combination changes) per operator and stationary mode, a combination's being the sum of its two; the
// register-file and MAC energies; the combinations' shares of the time
constexpr uint32_t DENSE_RF = 6, DENSE_LAT = 8, DENSE_NCS = 17;

// A class's rows: per operand and level the lines of its footprint and its traffic, as byte offsets (low and high 16 bits);
// C's; C's traffic is the zero line where the class is fused.
struct alignas(32) DenseClass {
    uint32_t a[5], b[5], d[5], e[5], c, pad_[3];
};
struct DenseClasses {
    DenseClass cls[96];                      // order + 24 * (r + 2 f)
    bool ascend;                             // every operand's footprint options and retention go up with its level
};
constexpr DenseClasses dense_classes()
{
    DenseClasses out{};
    out.ascend = true;
    for (uint32_t g = 0; g < N_GROUPS; ++g)
        for (uint32_t rank = 0; rank < 24; ++rank) {
            DenseClass &c = out.cls[rank + 24 * g];
            RowTerms last{};
            for (int p = 0; p < 5; ++p) {
                const int lvl[4] = {p, p, p, p};
                const RowTerms t = row_terms(rank, g & 1, g >> 1, lvl);
                uint32_t w[4] = {};
                for (uint32_t y = 0; y < 4; ++y) {
                    w[y] = (DENSE_BS + 4 * y + t.bs[y]) * DENSE_LINE | (DENSE_DA + 4 * y + t.da[y]) * DENSE_LINE << 16;
                    if (p && (last.bs[y] & ~t.bs[y])) out.ascend = false;
                    if (((t.tau >> y) & 1) != (uint32_t)(p >= 1)) out.ascend = false;
                }
                c.a[p] = w[0]; c.b[p] = w[1]; c.d[p] = w[2]; c.e[p] = w[3];
                c.c = (DENSE_BS + 16 + t.c) * DENSE_LINE | (t.dac >= 4 ? DENSE_ZERO : DENSE_DA + 16 + t.dac) * DENSE_LINE << 16;
                last = t;
            }
        }
    return out;
}
constexpr DenseClasses DENSE_CLASSES = dense_classes();
static_assert(DENSE_CLASSES.ascend, "the rows that fit are a staircase");
// ... and one operand's terms do not depend on the other levels: a row's terms are those of the equal-level rows
constexpr bool levels_separate()
{
    for (uint32_t g = 0; g < N_GROUPS; ++g)
        for (uint32_t rank = 0; rank < 24; ++rank)
            for (int y = 0; y < 4; ++y)
                for (int p = 0; p < 5; ++p)
                    for (int o = 0; o < 5; o += 4) {
                        const int same[4] = {p, p, p, p}, mixed[4] = {y == 0 ? p : o, y == 1 ? p : o, y == 2 ? p : o, y == 3 ? p : o};
                        const RowTerms a = row_terms(rank, g & 1, g >> 1, same), b = row_terms(rank, g & 1, g >> 1, mixed);
                        if (a.bs[y] != b.bs[y] || a.da[y] != b.da[y] || a.c != b.c || a.dac != b.dac) return false;
                    }
    return true;
}
static_assert(levels_separate(), "an operand's terms are a matter of its own level");
__device__ const DenseClasses dense_dev = DENSE_CLASSES;

struct DenseArgs {
    ModelConst mc;
    DigitConst dg;                           // of the chunks' order: k fastest, then j, l, i
    double extent[4], size[5];
    uint32_t X[4], ndiv[4];
    const uint4 *enc;                        // every encoded row (for the winner's record)
    const uint32_t *cls;                     // the (order, r, f) classes that denote dataflows (order + 24 * (r + 2 f))
    uint32_t n_cls;
    // Items: chunk by chunk, smaller ones towards the end.  From chunk `chunk` on, `groups` items to a chunk; `item` is the first.
    struct Phase { uint32_t item, chunk, groups, pad_; } phase[3];
    uint32_t n_items;
    Key *partials;                           // [gridDim.x][N_OBJ]
    uint32_t *ticket, *work_counter;
    FinalRecord *final_out;                  // [N_OBJ]
    Key *final_key_dev;                      // [N_OBJ] the winning keys once more, in device memory, for a pass that follows
    const Key *lat_cap;                      // LATCAP only: candidates with a latency above lat_cap->p are left out
    double e_limit;                          // LIMIT only: candidates with energy >= e_limit are left out
    // per key the lowest value any wave of the launch has recorded so far, as the bit pattern of the (non-negative)
    // double; +inf between launches
    unsigned long long *hints;
    Done *done;                              // [N_OBJ] not null: the host looks here for the launch's records
    uint64_t number, *begin;                 // the call's number; when the search began (device memory)
    uint32_t first_launch, pad_;             // of the call: it says when
    uint32_t list[DENSE_DIVS];               // the four divisor lists one after the other
};

// best = min(best, x) in best's own register: the paths of the row loop meet with their minima where they were, and not in copies.
__device__ __forceinline__ void min_in_place(double &best, double x) { asm("v_min_f64 %0, %0, %1" : "+v"(best) : "v"(x)); }

// SUM: how a candidate's energy is added up (ModelConst::regroup and gb_product_exact decide).  SUM_ORDERED forms it term by term,
// 6 operations per candidate with the minimum; SUM_FUSED forms the first sum with one fused multiply-add whose
// product is exact, i.e. with the bits of the two separate roundings; SUM_REGROUPED adds a row and a tiling part.
// The energy key alone leaves the two addends that all candidates of a (tiling, r) share, the register-file
// and MAC parts, to the nine minima: adding a constant and rounding keeps the order, so the minimum of the
// finished sums is the finished sum of the minimum, bit for bit (OUTSIDE).  Per candidate that is addition,
// multiplication, addition, minimum (4), with SUM_FUSED 3, with SUM_REGROUPED 2.
//
// FAST: the DRAM time is one exact multiply of the B*H-scaled traffic (ModelConst::dram_k).  Otherwise the table
// holds the traffic per instance and the time is dram_time_general; a true division here cost
// 1.2 to 5 times the whole rest of the loop.
//
// Registers decide the shape of the row loop.  One key: the 18 per-tiling constants, the (D, E) parts of all
// five p_D values and nine minima fit 128 registers (four waves per SIMD), and a step (p_A, p_B) serves five rows.  Two keys
// hold 18 minima: there one p_D value at a time is kept and a step serves one row.
template <int MASK, bool FAST, bool LIMIT = false, int SUM = SUM_ORDERED, bool LATCAP = false>
__global__ __launch_bounds__(DENSE_THREADS, 4) void k_search_dense(DenseArgs a)
{
    static_assert(!LATCAP || (MASK == 1 && !LIMIT), "the latency cap goes with the energy key alone");
    constexpr bool REGROUP = SUM == SUM_REGROUPED;
    static_assert(!(MASK & 4) && popcount4(MASK) <= 2, "one or two of the scalar keys");
    constexpr bool OUTSIDE = !REGROUP && (MASK & 1) && !(MASK & 8) && !LIMIT;
    constexpr bool ENERGY = MASK != (1 << MMEE_OBJ_LATENCY) || LIMIT, TIME = MASK != (1 << MMEE_OBJ_ENERGY) || LATCAP;
    // What a row's costs need of its traffic.  The energy alone, or the time alone: the operands' shares of it, whole numbers times
    // one exact constant, are in the table instead of the words.  Both: the words, weighed per row.
    constexpr bool E_SUMS = ENERGY && !TIME && REGROUP, L_SUMS = TIME && !ENERGY && FAST, WORDS = !E_SUMS && !L_SUMS;
    static_assert(!E_SUMS || FAST, "the energy's shares are of the scaled words");
    constexpr uint32_t ROWS_PER_STEP = popcount4(MASK) == 2 ? 1u : 5u;       // p_D values held in registers

    __shared__ double tab[DENSE_LINES * PRUNED_TC];           // entry-major, lane = tiling: conflict-free as it is
    __shared__ double cst[2 * DENSE_NCS * PRUNED_TC];         // [r][constant][tiling]
    __shared__ double gd[8 * PRUNED_TC];                      // the chunk's boundary vectors: G[0..3], D[0..3] per tiling
    __shared__ double tc[TIME ? 6 * 2 * PRUNED_TC : 1];       // the operators' costs: [op * 3 + mode][words, cycles][tiling]
    __shared__ uint32_t digits[4 * PRUNED_TC];
    __shared__ DivTable dv_s;
    __shared__ Key wave_best[N_OBJ][DENSE_WAVES];
    __shared__ uint32_t is_last;
    __shared__ uint32_t s_item;
    __shared__ uint32_t tickets[PRUNED_TC];                   // [0]: tasks of the item handed out so far
    // The lowest value any wave of this block has recorded (bit pattern; the keys are
    // non-negative, so the patterns order like the values), refreshed once per item from the launch-wide
    // one.  A wave whose values all lie strictly above it cannot hold the optimum and recovers no position.
    __shared__ unsigned long long hint_bits[N_OBJ];

    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ModelConst &mc = a.mc;
    ConstBytes args = (ConstBytes)__builtin_amdgcn_kernarg_segment_ptr();
    if (wave == DENSE_WAVES - 1) ask_for_arguments<DenseArgs>(lane);
    if (a.done && a.first_launch && blockIdx.x == 0 && threadIdx.x == 0)
        __hip_atomic_store(a.begin, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x < N_OBJ) hint_bits[threadIdx.x] = INF_BITS;
    if (threadIdx.x < PRUNED_TC) tab[DENSE_ZERO * PRUNED_TC + lane] = 0.0;
    {
        // the packed lists into the table form the decoding helpers take
        ConstPtr<uint32_t> list = (ConstPtr<uint32_t>)(args + offsetof(DenseArgs, list));
        uint32_t first = 0;
        for (int q = 0; q < 4; ++q) {
            for (uint32_t k = threadIdx.x; k < a.ndiv[q]; k += DENSE_THREADS) dv_s.div[q][k] = list[first + k];
            first += a.ndiv[q];
        }
        if (threadIdx.x < 4) {
            dv_s.X[threadIdx.x] = ((ConstPtr<uint32_t>)(args + offsetof(DenseArgs, X)))[threadIdx.x];
            dv_s.ndiv[threadIdx.x] = ((ConstPtr<uint32_t>)(args + offsetof(DenseArgs, ndiv)))[threadIdx.x];
        }
    }
    double run_p[N_OBJ];
    uint64_t run_idx[N_OBJ];
#pragma unroll
    for (int o = 0; o < N_OBJ; ++o) { run_p[o] = inf; run_idx[o] = ~0ull; }
    ConstPtr<uint32_t> cls_list = as_constant(a.cls);
    // the class's table, read at wave-uniform places: scalar loads
    ConstBytes classes = (ConstBytes)&dense_dev.cls[0];
    auto words_energy = [&](double words) { return FAST ? mc.e_sum * words : mc.e_sum * (words * mc.BH); };
    auto ballot = [](bool x) { return __builtin_amdgcn_ballot_w64(x); };
    struct DePart { double room_bs, room_ret, d; };
    // LATCAP: the second pass of the (latency, energy) key over the full row set.  The first pass found
    // the lowest latency; a candidate's latency max(l_dram, constant) stays within it exactly when both
    // parts do, so the cap masks rows and combinations separately and the pass costs what an
    // energy-only pass costs.
    const double lat_cap = LATCAP ? uniform_f64(a.lat_cap->p) : inf;

    if (threadIdx.x == 0) s_item = blockIdx.x;
    uint32_t built = 0xFFFFFFFFu;
    while (true) {
        __syncthreads();                          // also: the previous item's LDS readers are done
        const uint32_t item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= a.n_items) break;
        // Thread 0 asks for the next item and for the launch-wide values; the replies come while the tables are formed (kept
        // until the next item they would cost every lane registers).
        uint32_t upcoming = 0;
        unsigned long long seen[N_OBJ];
        if (threadIdx.x == 0) {
            tickets[0] = 0;
            // (an address that the compiler takes for the lane's own: one that it knows to be the wave's it reduces over the lanes
            // first, and waits for the reply here)
            uint32_t none = threadIdx.x;
            asm volatile("" : "+v"(none));
            upcoming = __hip_atomic_fetch_add(a.work_counter + none, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int o = 0; o < N_OBJ; ++o)
                if ((MASK >> o) & 1) seen[o] = __hip_atomic_load(a.hints + o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const uint32_t ph = (item >= a.phase[1].item) + (item >= a.phase[2].item);
        ConstPtr<uint32_t> phase = (ConstPtr<uint32_t>)(args + offsetof(DenseArgs, phase) + ph * sizeof(DenseArgs::Phase));
        const uint32_t j = item - phase[0], groups = phase[2], n_tasks = a.n_cls * 5u;
        const uint32_t chunk = phase[1] + j / groups, group = j % groups;
        const uint32_t task_lo = n_tasks * group / groups, task_n = n_tasks * (group + 1) / groups - task_lo;
        const uint32_t whole = task_n - min(task_n, DENSE_FIFTHS), turns = whole + 5u * (task_n - whole);
        const uint32_t t0 = chunk * PRUNED_TC, nt = min((uint32_t)PRUNED_TC, mc.T - t0);
        if (chunk != built) {
            built = chunk;
            // (problem and lane anew for every chunk: what is formed of them here alone would be kept in registers through the row loops)
            uint32_t own_lane = lane;
            asm volatile("" : "+v"(own_lane));
            ConstBytes problem = args;
            asm volatile("" : "+s"(problem));
            const ModelConst mc = read_const<ModelConst>(problem + offsetof(DenseArgs, mc));
            double extent[4], size[5];
#pragma unroll
            for (int q = 0; q < 4; ++q) extent[q] = ((ConstF64)(problem + offsetof(DenseArgs, extent)))[q];
#pragma unroll
            for (int q = 0; q < 5; ++q) size[q] = ((ConstF64)(problem + offsetof(DenseArgs, size)))[q];
            // ---- decode: a dimension per wave (beyond the chunk: its last tiling once more, as a candidate like any other)
            if (wave < 4) {
                auto f64_at = [&](size_t off) { return ((ConstF64)(problem + off))[wave]; };
                const uint32_t digit = digit_of(t0 + min(own_lane, nt - 1), f64_at(offsetof(DenseArgs, dg) + offsetof(DigitConst, rcp_radix)),
                                                f64_at(offsetof(DenseArgs, dg) + offsetof(DigitConst, rcp_n)),
                                                ((ConstPtr<uint32_t>)(problem + offsetof(DenseArgs, ndiv)))[wave]);
                const double g = (double)dv_s.div[wave][digit];
                digits[wave * PRUNED_TC + own_lane] = digit;
                gd[wave * PRUNED_TC + own_lane] = g;
                gd[(4 + wave) * PRUNED_TC + own_lane] = whole_quotient(f64_at(offsetof(DenseArgs, extent)), g);
            }
            __syncthreads();
            TilingF v;
#pragma unroll
            for (int q = 0; q < 4; ++q) { v.G[q] = gd[q * PRUNED_TC + own_lane]; v.D[q] = gd[(4 + q) * PRUNED_TC + own_lane]; }
            // ---- the two operators' costs per stationary mode over all their tile stages, and the operands' terms
            if (wave < 6) {
                double words, cycles;
                if (wave < 3) tile_cost_f64(v.G[DI], v.G[DK], v.G[DL], wave, mc, words, cycles);
                else tile_cost_f64(v.G[DI], v.G[DL], v.G[DJ], wave - 3, mc, words, cycles);
                // (whole numbers: the association is free)
                const double stages = v.D[DI] * v.D[DL] * (wave < 3 ? v.D[DK] : v.D[DJ]);
                words = words * stages;
                cycles = cycles * stages;
#pragma unroll
                for (uint32_t rr = 0; rr < 2; ++rr) {
                    // the first operator runs once per j tile where it recomputes; the addends that all combinations share ride
                    // on the second's
                    const double rho = rr ? v.D[DJ] : 1.0;
                    double share = mc.BH * (wave < 3 ? rho * words : words);
                    if constexpr (REGROUP) share = mc.e_gb * share;
                    if (wave >= 3) {
                        const double m1 = rho * (extent[DI] * extent[DK] * extent[DL]), m2 = extent[DI] * extent[DL] * extent[DJ];
                        const double e_rf_part = mc.e_rf * (mc.BH * 3.0 * (m1 + m2));
                        const double e_mac_part = mc.e_mac * (mc.BH * ((m1 + m2) + (double)mc.c_softmax * (rho * (extent[DI] * extent[DL]))));
                        if constexpr (REGROUP) share = (share + e_rf_part) + e_mac_part;
                        else if (wave == 3) {
                            cst[(rr * DENSE_NCS + DENSE_RF) * PRUNED_TC + own_lane] = e_rf_part;
                            cst[(rr * DENSE_NCS + DENSE_RF + 1) * PRUNED_TC + own_lane] = e_mac_part;
                        }
                    }
                    if constexpr (ENERGY) cst[(rr * DENSE_NCS + wave) * PRUNED_TC + own_lane] = share;
                }
                if constexpr (TIME) {
                    tc[(wave * 2) * PRUNED_TC + own_lane] = words;
                    tc[(wave * 2 + 1) * PRUNED_TC + own_lane] = cycles;
                }
            }
            auto line = [&](uint32_t n) -> double & { return tab[n * PRUNED_TC + own_lane]; };
            // the DRAM terms as the row loop wants them: words (B*H-scaled with FAST), or their energy or time
            auto weigh = [&](double words) {
                if constexpr (FAST) words = mc.BH * words;
                if constexpr (E_SUMS) words = words_energy(words);
                if constexpr (L_SUMS) words = words * mc.dram_k;
                return words;
            };
            auto operand = [&](uint32_t y, double tile, double d0, double d1, double whole, double n0, double n1) {
                double o[5];
                footprints(o, tile, d0, d1);
#pragma unroll
                for (int k = 0; k < 4; ++k) line(DENSE_BS + 4 * y + k) = o[k];
                footprints(o, whole, n0, n1);
#pragma unroll
                for (int k = 0; k < 4; ++k) line(DENSE_DA + 4 * y + k) = weigh(o[k]);
            };
            if (wave == 6) {
                operand(0, v.G[DI] * v.G[DK], v.D[DI], v.D[DK], size[0], v.D[DL], v.D[DJ]);
                operand(1, v.G[DK] * v.G[DL], v.D[DK], v.D[DL], size[1], v.D[DI], v.D[DJ]);
            }
            if (wave == 7) {
                operand(2, v.G[DL] * v.G[DJ], v.D[DL], v.D[DJ], size[2], v.D[DI], v.D[DK]);
                operand(3, v.G[DI] * v.G[DJ], v.D[DI], v.D[DJ], size[3], v.D[DK], v.D[DL]);
            }
            if (wave == 0) {
                double o[5];
                footprints(o, v.G[DI] * v.G[DL], v.D[DI], v.D[DL]);
#pragma unroll
                for (int k = 0; k < 4; ++k) line(DENSE_BS + 16 + k) = o[k];
            }
            if (wave == 3) {
                // unfused C: spilled by Op1, fetched by Op2, one softmax pass over S and P
#pragma unroll
                for (int k = 0; k < 4; ++k) line(DENSE_DA + 16 + k) = weigh(size[4] * (((k & 1) ? v.D[DK] : 1.0) + ((k & 2) ? v.D[DJ] : 1.0) + 2.0));
            }
            if constexpr (TIME) {
                __syncthreads();
                // ---- the combinations' shares of the time, 18 (recomputation, combination) pairs shared out over the waves, two at a time
                auto time_of = [&](uint32_t job) {
                    const uint32_t rr = job / 9, c9 = job % 9, s1 = c9 % 3, s2 = c9 / 3;
                    const double rho = rr ? v.D[DJ] : 1.0;
                    const double br = rho * tc[(s1 * 2) * PRUNED_TC + own_lane] + tc[((3 + s2) * 2) * PRUNED_TC + own_lane];
                    const double cyc = rho * tc[(s1 * 2 + 1) * PRUNED_TC + own_lane] + tc[((3 + s2) * 2 + 1) * PRUNED_TC + own_lane];
                    return mc.c_lat * fmax(cyc, buffer_time_general(mc, br));
                };
                auto place = [&](uint32_t job) -> double & { return cst[(job / 9 * DENSE_NCS + DENSE_LAT + job % 9) * PRUNED_TC + own_lane]; };
                const double one = time_of(wave), two = time_of(wave + DENSE_WAVES);
                place(wave) = one;
                place(wave + DENSE_WAVES) = two;
                if (wave < 18 - 2 * DENSE_WAVES) place(wave + 2 * DENSE_WAVES) = time_of(wave + 2 * DENSE_WAVES);
            }
        }
        __syncthreads();                          // the tables are there, and every wave has read the item
        if (threadIdx.x == 0) {
            s_item = gridDim.x + upcoming;
            // take what is lower there, hand over what is lower here (no reply awaited)
#pragma unroll
            for (int o = 0; o < N_OBJ; ++o) {
                if (!((MASK >> o) & 1)) continue;
                const unsigned long long here = hint_bits[o];
                if (seen[o] < here) atomicMin(&hint_bits[o], seen[o]);
                else if (here < seen[o]) (void)__hip_atomic_fetch_min(a.hints + o, here, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }

        for (;;) {
            // (every lane asks, each at a word of its own: a branch on lane 0 could be joined with one at the turn's end)
            const uint32_t at =
                __builtin_amdgcn_readfirstlane(__hip_atomic_fetch_add(tickets + lane, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
            if (at >= turns) break;
            const bool fine = at >= whole;
            const uint32_t task = task_lo + (fine ? whole + (at - whole) / 5u : at), pE = task % 5u;
            const uint32_t cls = cls_list[task / 5u];
            const uint32_t rank = cls % 24, g = cls / 24, r = g & 1;
            const uint32_t lo = fine ? (at - whole) % 5u : 0u, hi = fine ? lo + 1 : 5u;        // p_B's, two keys: p_D's
            const uint32_t row0 = 625u * rank + ROWS_PER_GROUP * g + 125u * pE;   // the task's row (p_A, p_B, p_D) = 0
            ConstPtr<uint32_t> words = (ConstPtr<uint32_t>)(classes + cls * sizeof(DenseClass));
            ConstPtr<uint32_t> words_a = words, words_b = words + 5, words_d = words + 10, words_e = words + 15;

            const char *col = reinterpret_cast<const char *>(tab + lane);
            auto at_lo = [&](uint32_t w) { return *reinterpret_cast<const double *>(col + (w & 0xFFFFu)); };
            auto at_hi = [&](uint32_t w) { return *reinterpret_cast<const double *>(col + (w >> 16)); };
            const double cap = mc.cap_words;
            const uint32_t w_c = words[20], w_e = words_e[pE];
            const double c_bs = at_lo(w_c), e_bs = at_lo(w_e), e_ret = pE ? e_bs : 0.0;
            {
                // the task's least row first: where it fits no tiling, none of the others does (small buffers: most tasks)
                const uint32_t lo_d = words_d[ROWS_PER_STEP == 5 ? 0u : lo], lo_b = words_b[ROWS_PER_STEP == 5 ? lo : 0u];
                const bool d_kept = ROWS_PER_STEP != 5 && lo, b_kept = ROWS_PER_STEP == 5 && lo;
                const double d_bs = at_lo(lo_d), b_bs = at_lo(lo_b), a_bs = at_lo(words_a[0]);
                const double bs1 = (a_bs + b_bs) + (c_bs + ((d_kept ? d_bs : 0.0) + e_ret)), bs2 = (c_bs + (d_bs + e_bs)) + (b_kept ? b_bs : 0.0);
                if (!(ballot(bs1 <= cap) & ballot(bs2 <= cap))) continue;
            }
            const double c_d = at_hi(w_c), e_d = at_hi(w_e);
            // the (D, E) part and C beside p_D = q: what they leave of the capacity for A and B beside operator 1's and operator 2's
            // operands, and their traffic
            auto de_part = [&](uint32_t w_d, bool retained) {
                DePart y;
                const double d_bs = at_lo(w_d);
                y.room_bs = cap - (c_bs + ((retained ? d_bs : 0.0) + e_ret));
                y.room_ret = cap - (c_bs + (d_bs + e_bs));
                y.d = c_d + (at_hi(w_d) + e_d);
                return y;
            };

            const double *cs = cst + r * DENSE_NCS * PRUNED_TC + lane;
            double gb[9], latc[9];
            {
                double one[3], two[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) { one[k] = ENERGY ? cs[k * PRUNED_TC] : 0.0; two[k] = ENERGY ? cs[(3 + k) * PRUNED_TC] : 0.0; }
#pragma unroll
                for (int c = 0; c < 9; ++c) { gb[c] = one[c % 3] + two[c / 3]; latc[c] = TIME ? cs[(DENSE_LAT + c) * PRUNED_TC] : 0.0; }
            }
            const double e_rf_part = REGROUP || OUTSIDE ? 0.0 : cs[DENSE_RF * PRUNED_TC], e_mac_part = REGROUP || OUTSIDE ? 0.0 : cs[(DENSE_RF + 1) * PRUNED_TC];
            double bestE[9], bestL[9], bestP[9];
#pragma unroll
            for (int c9 = 0; c9 < 9; ++c9) bestE[c9] = bestL[c9] = bestP[c9] = inf;

            // One row of this lane's tiling, from its traffic (E_SUMS, L_SUMS: its energy, its time): the nine combinations.  A tiling
            // it does not fit: +inf for the parts that are the row's, under a branch that the whole wave takes or passes.
            auto cost_row = [&](double traffic, bool fits, unsigned long long who) {
                double e_part = traffic, l_dram = traffic, dram_words = 0.0;
                if constexpr (WORDS) {
                    if constexpr (ENERGY && REGROUP) e_part = words_energy(traffic);
                    else if constexpr (ENERGY) {
                        dram_words = FAST ? traffic : traffic * mc.BH;
                        e_part = mc.e_dram * dram_words;
                    }
                    if constexpr (TIME) l_dram = FAST ? traffic * mc.dram_k : dram_time_general(mc, traffic);
                }
                if constexpr (LATCAP) {
                    fits = fits & (l_dram <= lat_cap);
                    who = ballot(fits);
                }
                if (who != ~0ull) {
                    asm volatile("");                             // (not a select for every wave)
                    e_part = fits ? e_part : inf;
                    l_dram = fits ? l_dram : inf;
                }
#pragma unroll
                for (int c9 = 0; c9 < 9; ++c9) {
                    double en = 0.0;
                    if constexpr (ENERGY && REGROUP) {
                        en = e_part + gb[c9];
                    } else if constexpr (ENERGY) {
                        double gb_words = dram_words + gb[c9];
                        if constexpr (SUM == SUM_FUSED) en = __builtin_fma(mc.e_gb, gb_words, e_part);
                        else en = e_part + mc.e_gb * gb_words;
                        if constexpr (!OUTSIDE) {
                            en = en + e_rf_part;
                            en = en + e_mac_part;
                        }
                    }
                    double lat = fmax(l_dram, latc[c9]);
                    if constexpr (LIMIT) {
                        bool out_of_range = !(en < a.e_limit);
                        en = out_of_range ? inf : en;
                        lat = out_of_range ? inf : lat;
                    }
                    if constexpr (MASK & 8) min_in_place(bestP[c9], en * lat);
                    if constexpr (MASK & 1) min_in_place(bestE[c9], en);
                    if constexpr (MASK & 2) min_in_place(bestL[c9], lat);
                }
            };

            if constexpr (ROWS_PER_STEP == 5) {
                DePart y[5];
#pragma unroll
                for (uint32_t q = 0; q < 5; ++q) y[q] = de_part(words_d[q], q != 0);
                uint32_t w_b = words_b[lo], w_a[5];
#pragma unroll
                for (int p = 0; p < 5; ++p) w_a[p] = words_a[p];
                // A's and B's terms are read one step ahead, where the registers allow it
                constexpr bool AHEAD = !((ENERGY && TIME) && !OUTSIDE);
                double b_bs = at_lo(w_b), b_d = at_hi(w_b), a_bs = at_lo(w_a[0]), a_d = at_hi(w_a[0]);
                bool more = true;                                 // (wave-uniform)
#pragma unroll 1
                for (uint32_t pB = lo; more && pB < hi; ++pB) {
                    if constexpr (!AHEAD) { w_b = words_b[pB]; b_bs = at_lo(w_b); b_d = at_hi(w_b); }
                    const double x_b = b_bs, d_b = b_d, ret_b = pB ? b_bs : 0.0;
                    if constexpr (AHEAD) w_b = words_b[min(pB + 1, 4u)];
                    // A's levels one after the other, as long as a tiling has room (nested, so that no path leaves in the middle: the
                    // compiler keeps the minima in one place)
                    auto steps = [&](auto &self, auto level) {
                        constexpr int pA = decltype(level)::value;
                        if constexpr (!AHEAD) { a_bs = at_lo(w_a[pA]); a_d = at_hi(w_a[pA]); }
                        const double x_bs = a_bs + x_b, x_ret = (pA ? a_bs : 0.0) + ret_b, x_d = a_d + d_b;
                        if constexpr (AHEAD) {
                            a_bs = at_lo(w_a[(pA + 1) % 5]); a_d = at_hi(w_a[(pA + 1) % 5]);
                            if constexpr (pA == 0) { b_bs = at_lo(w_b); b_d = at_hi(w_b); }
                        }
                        const bool bs0 = x_bs <= y[0].room_bs, ret0 = x_ret <= y[0].room_ret;
                        const unsigned long long some = ballot(bs0) & ballot(ret0);   // (of each: a comparison's mask as it is)
                        if constexpr (pA == 0) more = some != 0;
                        if (some) {
                            unsigned long long all = ballot(x_bs <= y[4].room_bs) & ballot(x_ret <= y[4].room_ret);
                            if (all != ~0ull) {
                                cost_row(x_d + y[0].d, bs0 & ret0, some);
                                auto rows = [&](auto &next, auto which) {
                                    constexpr int q = decltype(which)::value;
                                    const bool bs = x_bs <= y[q].room_bs, ret = x_ret <= y[q].room_ret;
                                    const unsigned long long who = ballot(bs) & ballot(ret);
                                    if (who) {
                                        cost_row(x_d + y[q].d, bs & ret, who);
                                        if constexpr (q < 4) next(next, std::integral_constant<int, q + 1>{});
                                    }
                                };
                                rows(rows, std::integral_constant<int, 1>{});
                            }
                            asm volatile("" : "+s"(all));       // (two branches: as one with two sides it keeps the minima twice)
                            if (all == ~0ull) {
#pragma unroll
                                for (int q = 0; q < 5; ++q) cost_row(x_d + y[q].d, true, ~0ull);
                            }
                            if constexpr (pA < 4) self(self, std::integral_constant<int, pA + 1>{});
                        }
                    };
                    steps(steps, std::integral_constant<int, 0>{});
                    if constexpr (AHEAD) { a_bs = at_lo(w_a[0]); a_d = at_hi(w_a[0]); }
                }
            } else {
                uint32_t w_a[5];
#pragma unroll
                for (int p = 0; p < 5; ++p) w_a[p] = words_a[p];
                bool some_q = true;                               // (wave-uniform)
#pragma unroll 1
                for (uint32_t q = lo; some_q && q < hi; ++q) {
                    const DePart y = de_part(words_d[q], q != 0);
                    bool more = true;
                    some_q = false;
#pragma unroll 1
                    for (uint32_t pB = 0; more && pB < 5; ++pB) {
                        const uint32_t w_b = words_b[pB];
                        const double b_bs = at_lo(w_b), room_bs = y.room_bs - b_bs, room_ret = y.room_ret - (pB ? b_bs : 0.0), d = y.d + at_hi(w_b);
                        auto steps = [&](auto &self, auto level) {
                            constexpr int pA = decltype(level)::value;
                            const double a_bs = at_lo(w_a[pA]);
                            const bool bs = a_bs <= room_bs, ret = (pA ? a_bs : 0.0) <= room_ret;
                            const unsigned long long who = ballot(bs) & ballot(ret);
                            if constexpr (pA == 0) { more = who != 0; some_q = some_q | more; }
                            if (who) {
                                cost_row(at_hi(w_a[pA]) + d, bs & ret, who);
                                if constexpr (pA < 4) self(self, std::integral_constant<int, pA + 1>{});
                            }
                        };
                        steps(steps, std::integral_constant<int, 0>{});
                    }
                }
            }

            // (read again below, by a lane number that the compiler does not know: from here on, and not through the row loops)
            uint32_t late_lane = lane;
            asm volatile("" : "+v"(late_lane));
            const double *late = cst + r * DENSE_NCS * PRUNED_TC + late_lane;
            const double rf_late = REGROUP || !ENERGY ? 0.0 : late[DENSE_RF * PRUNED_TC], mac_late = REGROUP || !ENERGY ? 0.0 : late[(DENSE_RF + 1) * PRUNED_TC];
            if constexpr (OUTSIDE) {
#pragma unroll
                for (int c9 = 0; c9 < 9; ++c9) bestE[c9] = (bestE[c9] + rf_late) + mac_late;
            }
            if constexpr (LATCAP) {
                // combinations beyond the cap, whatever the row (no cap found: nothing qualifies)
#pragma unroll
                for (int c9 = 0; c9 < 9; ++c9) bestE[c9] = late[(DENSE_LAT + c9) * PRUNED_TC] <= lat_cap && lat_cap < inf ? bestE[c9] : inf;
            }
#pragma unroll
            for (int o = 0; o < N_OBJ; ++o) {
                if (!((MASK >> o) & 1)) continue;
                const double *best = o == 0 ? bestE : (o == 1 ? bestL : bestP);
                double mine_v = best[0];
#pragma unroll
                for (int c9 = 1; c9 < 9; ++c9) mine_v = fmin(mine_v, best[c9]);
                const double hint = __longlong_as_double((long long)hint_bits[o]);
                if (!__ballot(mine_v <= run_p[o] && mine_v < inf && mine_v <= hint)) continue;   // the usual case: nothing new here
                const double wave_v = uniform_f64(wave_min_f64(mine_v));
                // the lowest combination in which some tiling reaches the minimum: its candidates
                // precede those of every higher combination
                uint32_t cstar = 9;
#pragma unroll
                for (int c9 = 8; c9 >= 0; --c9) cstar = best[c9] == wave_v ? (uint32_t)c9 : cstar;
                const uint32_t c_u = __builtin_amdgcn_readfirstlane(wave_min_u32(cstar));
                // index row (Sec. VI-A numbering) of the task's first row under that combination
                const uint32_t first_row = index_row_base(row0) + 30000u * (c_u % 3) + 90000u * (c_u / 3);
                if (!(wave_v < run_p[o] || (uint64_t)mc.T * first_row < run_idx[o])) continue;
                // Make the value known before its position is: of the waves of a block that reach this point
                // together, only those holding the lowest value go on (the holder of the lowest value always
                // passes its own mark, so what the others leave out is recorded by it).
                if (lane == 0) atomicMin(&hint_bits[o], (unsigned long long)__double_as_longlong(wave_v));
                if (wave_v > __longlong_as_double((long long)hint_bits[o])) continue;
                // Recover the row: the first of the 125 rows of (class, p_E) (index order) in which a tiling reaches the
                // minimum under combination c_u, at its tiling of the lowest number.  Rows are costed again with the very
                // operations of the loop above.  (A fifth of a task looks at all 125 rows: what another fifth's row has is a candidate, too.)
                double best_u = best[0];
#pragma unroll
                for (int c9 = 1; c9 < 9; ++c9) best_u = c_u == (uint32_t)c9 ? best[c9] : best_u;
                const double gb_u = ENERGY ? late[c_u % 3 * PRUNED_TC] + late[(3 + c_u / 3) * PRUNED_TC] : 0.0, latc_u = TIME ? late[(DENSE_LAT + c_u) * PRUNED_TC] : 0.0;
                // row `code` of one tiling (its column of the table, its constants)
                auto recost = [&](const char *column, uint32_t code, uint32_t wa, uint32_t wb, uint32_t wd, double gb_t, double latc_t, double rf_t,
                                  double mac_t) {
                    auto lo = [&](uint32_t w) { return *reinterpret_cast<const double *>(column + (w & 0xFFFFu)); };
                    auto hi = [&](uint32_t w) { return *reinterpret_cast<const double *>(column + (w >> 16)); };
                    const uint32_t wc = words[20];
                    const double a2 = lo(wa), b2 = lo(wb), d2 = lo(wd), e2 = lo(w_e), c2 = lo(wc);
                    const double bs1 = (a2 + b2) + (c2 + ((code / 25u ? d2 : 0.0) + (pE ? e2 : 0.0)));
                    const double bs2 = (c2 + (d2 + e2)) + ((code % 5u ? a2 : 0.0) + (code / 5u % 5u ? b2 : 0.0));
                    // The very sum of the loop, also where a total taken on trust is not exact (E_SUMS).  With one p_D value a step the loop
                    // adds the same words in another order, which is the same sum as long as they are whole.
                    static_assert(WORDS || ROWS_PER_STEP == 5, "shares that are not exact are summed as in the loop");
                    const double ab = hi(wa) + hi(wb), de = hi(wc) + (hi(wd) + hi(w_e)), traffic2 = ab + de;
                    bool ok2 = fmax(bs1, bs2) <= cap;
                    double dram2 = 0.0, en2 = traffic2, l2 = traffic2;
                    if constexpr (WORDS) {
                        dram2 = FAST ? traffic2 : traffic2 * mc.BH;
                        en2 = REGROUP ? words_energy(traffic2) : mc.e_dram * dram2;
                        if constexpr (TIME) l2 = FAST ? traffic2 * mc.dram_k : dram_time_general(mc, traffic2);
                    }
                    if constexpr (LATCAP) ok2 = ok2 & (l2 <= lat_cap) & (latc_t <= lat_cap);
                    const double over2 = __hiloint2double(ok2 ? 0 : 0x7ff00000, 0);
                    en2 = fmax(en2, over2);
                    l2 = fmax(l2, over2);
                    pin(en2);
                    pin(l2);
                    if constexpr (REGROUP) {
                        en2 = en2 + gb_t;
                    } else {
                        double gb2 = dram2 + gb_t;
                        en2 = en2 + mc.e_gb * gb2;
                        en2 = en2 + rf_t;
                        en2 = en2 + mac_t;
                    }
                    double lat2 = fmax(l2, latc_t);
                    if constexpr (LIMIT) {
                        const bool out_of_range = !(en2 < a.e_limit);
                        en2 = out_of_range ? inf : en2;
                        lat2 = out_of_range ? inf : lat2;
                    }
                    return o == 0 ? en2 : (o == 1 ? lat2 : en2 * lat2);
                };
                constexpr uint32_t N_CODES = 125;
                // this lane's tiling: digits of a mixed radix, i's least significant
                const uint32_t *dig = digits + late_lane;
                const uint32_t tiling = dig[0] + a.ndiv[0] * (dig[PRUNED_TC] + a.ndiv[1] * (dig[2 * PRUNED_TC] + a.ndiv[2] * dig[3 * PRUNED_TC]));
                uint32_t found_code = 0xFFFFFFFFu, found_t = 0xFFFFFFFFu;
                // only a tiling whose own minimum under c_u is the wave's can hold it
                unsigned long long cands = __ballot(best_u == wave_v && lane < nt);
                if (__popcll(cands) <= 4) {
                    // few such tilings: one at a time with lane = row (64 rows of the task per step)
                    while (cands) {
                        const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)__ffsll((long long)cands) - 1u);
                        cands &= cands - 1;
                        const double gb_l = lane_value_f64(gb_u, l), latc_l = lane_value_f64(latc_u, l);
                        const double rf_l = lane_value_f64(rf_late, l), mac_l = lane_value_f64(mac_late, l);
                        const uint32_t t_l = __builtin_amdgcn_readlane(tiling, l);
                        for (uint32_t code0 = 0; code0 < N_CODES && code0 <= found_code; code0 += 64) {
                            const uint32_t code = min(code0 + late_lane, N_CODES - 1);
                            const uint32_t *own = &dense_dev.cls[cls].a[0];
                            const double val2 = recost(reinterpret_cast<const char *>(tab + l), code, own[code % 5u], own[5u + code / 5u % 5u],
                                                       own[10u + code / 25u], gb_l, latc_l, rf_l, mac_l);
                            const unsigned long long hits = __ballot(code0 + late_lane < N_CODES && val2 == wave_v);
                            if (!hits) continue;
                            const uint32_t c_hit = code0 + (uint32_t)__ffsll((long long)hits) - 1u;
                            if (c_hit < found_code || (c_hit == found_code && t_l < found_t)) { found_code = c_hit; found_t = t_l; }
                            break;
                        }
                    }
                } else {
                    for (uint32_t code = 0; code < N_CODES; ++code) {
                        const double val2 = recost(col, code, words_a[code % 5u], words_b[code / 5u % 5u], words_d[code / 25u], gb_u, latc_u,
                                                   rf_late, mac_late);
                        if (!__ballot(val2 == wave_v)) continue;
                        found_code = code;
                        found_t = __builtin_amdgcn_readfirstlane(wave_min_u32(val2 == wave_v ? tiling : 0xFFFFFFFFu));
                        break;
                    }
                }
                if (found_code != 0xFFFFFFFFu) {
                    const uint64_t idx = (uint64_t)found_t + (uint64_t)mc.T * (first_row + found_code);
                    if (wave_v < run_p[o] || idx < run_idx[o]) {
                        run_p[o] = wave_v;
                        run_idx[o] = uniform_u64(idx);
                    }
                }
            }
        }
    }

    if (lane == 0) {
#pragma unroll
        for (int o = 0; o < N_OBJ; ++o) {
            if (!((MASK >> o) & 1)) continue;
            wave_best[o][wave].p = run_p[o]; wave_best[o][wave].s = 0.0; wave_best[o][wave].idx = run_idx[o];
        }
    }
    // ---- the waves' bests -> one record per block -> ticket; the last block to arrive reduces them and writes the winner
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int o = 0; o < N_OBJ; ++o) {
            if (!((MASK >> o) & 1)) continue;
            Key k = wave_best[o][0];
            for (int wv = 1; wv < DENSE_WAVES; ++wv)
                if (key_less(wave_best[o][wv], k)) k = wave_best[o][wv];
            Key *dst = a.partials + (uint64_t)blockIdx.x * N_OBJ + o;
            __hip_atomic_store(&dst->idx, k.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(reinterpret_cast<uint64_t *>(&dst->p), (uint64_t)__double_as_longlong(k.p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // records and ticket meet where all XCDs see them; the wait keeps the ticket behind the records, and nothing else has to be
        // written back
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        is_last = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    }
    __syncthreads();
    if (!is_last) return;
#pragma unroll
    for (int o = 0; o < N_OBJ; ++o) {
        if (!((MASK >> o) & 1)) continue;
        Key k; k.p = inf; k.s = 0.0; k.idx = ~0ull;
        for (uint32_t b = threadIdx.x; b < gridDim.x; b += DENSE_THREADS) {
            Key *src = a.partials + (uint64_t)b * N_OBJ + o;
            Key c;
            c.s = 0.0;
            c.idx = __hip_atomic_load(&src->idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            c.p = __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<uint64_t *>(&src->p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            if (key_less(c, k)) k = c;
        }
        k = wave_min(k);
        if (lane == 0) wave_best[o][wave] = k;
    }
    __syncthreads();
    if (threadIdx.x < N_OBJ) a.hints[threadIdx.x] = INF_BITS;
    if (threadIdx.x == 0) { *a.ticket = 0; *a.work_counter = 0; }   // ready for the next launch on this stream
    if (threadIdx.x < N_OBJ && ((MASK >> threadIdx.x) & 1)) {
        const int o = threadIdx.x;
        Key k = wave_best[o][0];
        for (int wv = 1; wv < DENSE_WAVES; ++wv)
            if (key_less(wave_best[o][wv], k)) k = wave_best[o][wv];
        if (a.final_key_dev) a.final_key_dev[o] = k;
        mmee_result res;
        winner_record(a.enc, dv_s, mc, k, res);
        write_record(a.final_out + o, k, res);
        if (a.done) say_done(a.done + o, a.number, __hip_atomic_load(a.begin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
}

}  // namespace mmee
