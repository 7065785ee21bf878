// Batched search over short row lists (the pruned rows of Sec. VI-B): many problems in one launch.
//
// The online stage of Sec. VI-A costs a few hundred surviving rows against a few thousand tilings
// per problem -- microseconds of arithmetic -- so a sweep over hardware designs and sequence lengths
// (Sec. VII-H, VII-I) is bound by launches and table traffic unless the problems share a launch.
// Here one work item is (problem, chunk of 64 tilings) and a block builds the chunk's slice of the
// boundary-side tables straight into LDS, from the problem's divisor lists: nothing per tiling ever
// touches HBM.  Lane = tiling, wave = a contiguous piece of one group's row list, so a row's table
// offsets are wave-uniform and the per-tiling constants of the nine stationary combinations sit in
// registers for the whole item.  Only the table entries that the rows refer to are staged (77 of 123
// for the pruned rows), which lets two 512-thread blocks share a CU; the entries' places in the staged
// table are known at compile time (rows.h): immediate offsets of straight-line rows, or scalar loads.  A block takes a contiguous range
// of items, waves carry their best (value, index) across the items of a problem, and each (block,
// problem) stretch leaves one record per key.  Where the launch has one problem, its last block reduces the records and writes the
// winner's full cost record and mapping; where it has many, k_batch_finish, launched behind the search, does.
//
// Included once by mmee.hip.
#pragma once
#include "boundary.h"

namespace mmee {

constexpr int BATCH_THREADS = 512;           // two blocks per CU, four waves per SIMD
constexpr int BATCH_WAVES = BATCH_THREADS / 64;

constexpr int BATCH_INLINE_DIVS = 448;       // divisors (all four lists together) of a problem that rides in the kernel arguments

struct BatchProblemHead {
    ModelConst mc;
    uint32_t first_item;                     // its first work item in the launch
    uint32_t n_work;                         // its work items: chunks of 64 tilings x row shares
    uint32_t slot;                           // where its N_OBJ final records go
    uint32_t pad_;
    uint32_t X[4], ndiv[4];                  // extents and divisor counts of i, k, l, j
};

struct BatchProblem {                        // one problem, in device memory
    BatchProblemHead h;
    uint32_t list[4 * MAXDIV];               // the four divisor lists one after the other, ndiv[q] entries each
};

// A launch of one problem carries it inside the kernel arguments: no descriptor copy has to reach the
// device before the kernel may start.  Same layout as the front of a BatchProblem, then the launch's
// two-entry first-item table.
struct BatchInline {
    BatchProblemHead h;
    uint32_t list[BATCH_INLINE_DIVS];
    uint32_t firsts[2];
    uint32_t on, pad_;
};

struct BatchArgs {
    const BatchProblem *prob;
    const uint32_t *first_items;             // [n_prob + 1] ascending, for the item -> problem search
    uint32_t n_prob, n_items;
    const uint4 *enc;                        // every encoded row (for the winner's record)
    // A chunk's rows are shared out over `split` work items (1 in a large launch; more when the launch
    // would otherwise leave most of the chip idle), and inside a work item over the waves of the block.
    uint32_t split;                              // 1 or 2
    uint32_t task_lo[PIECE_SPLITS * BATCH_WAVES];        // per (share, wave): its first row in the lists,
    uint32_t task_cnt[PIECE_SPLITS * BATCH_WAVES];       //                    how many rows it takes,
    uint32_t task_g[PIECE_SPLITS * BATCH_WAVES];         //                    and the group g = r + 2 f they belong to
    Key *item_keys;                          // [n_items][N_OBJ]; written at the first item of every (block, problem) stretch
    uint32_t per_block, extra;               // items per block of the search launch: the first `extra` blocks take one more
    FinalRecord *final_out;                  // [result slot][N_OBJ]
    mmee_result *packed;                     // not null: the launch's one key of its one problem goes here, as a result record
    uint64_t space, evaluated;               // ... with these
    uint32_t *ticket;                        // inl.on: blocks that have left their records, modulo the launch's blocks; 0 between launches
    Done *done;                              // [N_OBJ] not null: the host looks here for the launch's one problem
    uint64_t number, *begin;                 // the call's number; when the search began (device memory)
    BatchInline inl;                         // inl.on: the launch's only problem is here, prob and first_items are unused
};

// The first item of block b (b = the launch's blocks: the number of items), and the block that item x is in.
__device__ __forceinline__ uint32_t first_item_of(const BatchArgs &a, uint32_t b) { return b * a.per_block + min(b, a.extra); }
__device__ __forceinline__ uint32_t block_of(const BatchArgs &a, uint32_t x)
{
    const uint32_t longer = a.extra * (a.per_block + 1);
    return x < longer ? x / (a.per_block + 1) : a.extra + (x - longer) / a.per_block;
}

// Where a launch's problems and first-item table are: in device memory, or inside the kernel
// arguments themselves (which are ordinary read-only memory to the kernel).
__device__ __forceinline__ void batch_tables(const BatchArgs &a, const BatchProblem *&probs, ConstPtr<uint32_t> &firsts)
{
    probs = a.prob;
    firsts = as_constant(a.first_items);
    if (a.inl.on) {
        ConstPtr<char> args = (ConstPtr<char>)__builtin_amdgcn_kernarg_segment_ptr();
        probs = (const BatchProblem *)(args + offsetof(BatchArgs, inl));
        firsts = (ConstPtr<uint32_t>)(args + offsetof(BatchArgs, inl) + offsetof(BatchInline, firsts));
    }
}

// The least traffic (B*H * Eq. (7)) of piece PIECE's rows that fit, for the tiling whose table column is `col`; +inf: none does.
// Straight-line code: the entries' places are immediate offsets of the LDS reads.  In a loop every row waited for its
// offsets (a scalar load) and then for its entries, 330 cycles a row, more than half of a chunk's time, whatever the
// number of reads (1050 instead of 2160 per tiling in a loop gained 2 %).  Kernels, us, loop -> this, with the fold of then: 1600 chunks, energy
// 48 -> 35, energy and latency 71 -> 59 (with the fold as it is 27 and 47); 20736 chunks 356 -> 239 and 452 -> 331.  Rows come in runs with common entries of D, E and C (rows.h); a row compares its entries of A and B with what
// the run leaves of the capacity: Eq. (1), (2), (4), whole numbers, so exact in any order.
template <uint32_t SPLIT, int RUN, int ROW, int... I>
__device__ __forceinline__ void run_least(const char *col, double cap, double &least, std::integer_sequence<int, I...>)
{
    auto at = [&](uint32_t off) { return *reinterpret_cast<const double *>(col + off); };
    constexpr const uint32_t (&run)[8] = pieces<SPLIT>().run[RUN];
    const double c = at(run[1]), room_bs = cap - (c + at(run[0])), room_ret = cap - (at(run[2]) + c), da = at(run[3]) + at(run[4]);
    auto row = [&](auto n) {
        constexpr const uint32_t (&off)[4] = pieces<SPLIT>().row[ROW + decltype(n)::value];
        const bool bs_fits = at(off[0]) <= room_bs, ret_fits = at(off[1]) <= room_ret;
        least = fmin(least, (bs_fits & ret_fits) ? at(off[2]) + da : pos_inf());
    };
    (row(std::integral_constant<int, I>{}), ...);
}
template <uint32_t SPLIT, int RUN, int ROW, int END>
__device__ __forceinline__ void runs_least(const char *col, double cap, double &least)
{
    if constexpr (RUN < END) {
        constexpr int N = (int)pieces<SPLIT>().run[RUN][5];
        run_least<SPLIT, RUN, ROW>(col, cap, least, std::make_integer_sequence<int, N>{});
        if constexpr (RUN % 3 == 2) __builtin_amdgcn_sched_barrier(0);       // (all reads at once would not fit the registers)
        runs_least<SPLIT, RUN + 1, ROW + N, END>(col, cap, least);
    }
}
template <uint32_t SPLIT, int PIECE>
__device__ __forceinline__ double piece_least(const char *col, double cap)
{
    double least = pos_inf();
    runs_least<SPLIT, (int)pieces<SPLIT>().first_run[PIECE], (int)pieces<SPLIT>().first_row[PIECE], (int)pieces<SPLIT>().first_run[PIECE + 1]>(col, cap, least);
    pin(least);                                              // (or the compiler moves what the pieces' ends have in common behind all of them)
    return least;
}
template <uint32_t SPLIT, int SHARE>
__device__ __forceinline__ double share_least(uint32_t wave, const char *col, double cap)
{
    switch (wave) {
    case 0: return piece_least<SPLIT, 8 * SHARE>(col, cap);
    case 1: return piece_least<SPLIT, 8 * SHARE + 1>(col, cap);
    case 2: return piece_least<SPLIT, 8 * SHARE + 2>(col, cap);
    case 3: return piece_least<SPLIT, 8 * SHARE + 3>(col, cap);
    case 4: return piece_least<SPLIT, 8 * SHARE + 4>(col, cap);
    case 5: return piece_least<SPLIT, 8 * SHARE + 5>(col, cap);
    case 6: return piece_least<SPLIT, 8 * SHARE + 6>(col, cap);
    default: return piece_least<SPLIT, 8 * SHARE + 7>(col, cap);
    }
}

// MASK, FAST, REGROUP as in k_search.  Every block takes a contiguous range of the work items, so
// that it stays with one problem for many items: a wave keeps its running best (value, index) per key
// across the items of a problem and recovers a position only where it can matter; one record per
// (block, problem) leaves the block, at the slot of the first item of that stretch.
template <int MASK, bool FAST, bool REGROUP>
__global__ __launch_bounds__(BATCH_THREADS, 4) void k_search_batch(BatchArgs a)
{
    __shared__ double tab[KEPT_LINES * PRUNED_TC];        // entry-major, lane = tiling: conflict-free as it is
    __shared__ double gd[8 * PRUNED_TC];                      // the chunk's boundary vectors: G[0..3], D[0..3] per tiling
    __shared__ double tc[6 * 2 * PRUNED_TC];                  // the operators' costs: [op * 3 + mode][words, cycles][tiling]
    __shared__ uint32_t div_lds[4 * MAXDIV];                 // the current problem's divisor lists
    __shared__ Key wave_best[N_OBJ][BATCH_WAVES];
    __shared__ uint4 rows_lds[KEPT_ALL];                      // the kept rows: their eight entries' byte offsets, 16 bits each,
    __shared__ uint32_t number_lds[KEPT_ALL];                 // and their numbers
    // per key the lowest value the block has met on the stretch (bit pattern: they are not negative); on the item, of those that have
    // it, the lowest secondary value and the lowest class
    __shared__ unsigned long long low_p[N_OBJ], low_s;
    __shared__ uint32_t low_code[N_OBJ];

    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // the arguments' lines and the rows that a position may be recovered from, all asked for at the start (0.8 us of a one-chunk block's 7)
    if (wave == BATCH_WAVES - 1) ask_for_arguments<BatchArgs>(lane);
    static_assert(KEPT_ALL <= BATCH_THREADS, "a thread per row");
    if (threadIdx.x < KEPT_ALL) {
        rows_lds[threadIdx.x] = *reinterpret_cast<const uint4 *>(kept_dev.packed[threadIdx.x]);
        number_lds[threadIdx.x] = kept_dev.number[threadIdx.x];
    }

    const uint32_t item_lo = first_item_of(a, blockIdx.x), item_hi = first_item_of(a, blockIdx.x + 1);
    if (a.done && blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(a.begin, (uint64_t)wall_clock64(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // the first item's problem: the last p with first_items[p] <= item; later items move p on
    const BatchProblem *probs;
    ConstPtr<uint32_t> firsts;
    batch_tables(a, probs, firsts);
    uint32_t p;
    {
        uint32_t lo = 0, hi = a.n_prob;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (firsts[mid] <= item_lo) lo = mid; else hi = mid;
        }
        p = lo;
    }
    const char *tab_bytes = reinterpret_cast<const char *>(tab) + lane * 8;

    // the wave's running best over the items of the current problem
    double run_p[N_OBJ], run_s[N_OBJ];                       // (primary, secondary) as in Key; secondary 0 for scalar keys
    uint64_t run_idx[N_OBJ];
    uint32_t run_c[N_OBJ], run_i[N_OBJ], run_t0[N_OBJ];      // its combination, its row (place in the row lists), its chunk
    auto reset_running = [&]() {
#pragma unroll
        for (int o = 0; o < N_OBJ; ++o) { run_p[o] = inf; run_s[o] = 0.0; run_idx[o] = ~0ull; run_c[o] = run_i[o] = run_t0[o] = 0; }
    };
    reset_running();
    uint32_t staged_p = 0xFFFFFFFFu;

    // one stretch = the block's items of one problem
    for (uint32_t seg_first = item_lo; seg_first < item_hi;) {
      while (firsts[p + 1] <= seg_first) ++p;
      const uint32_t seg_end = min(item_hi, firsts[p + 1]), seg_len = seg_end - seg_first;
      // The items of a stretch are visited with a stride of about 0.618 of its length (coprime to it):
      // costs tend to move steadily along the tiling index, and in such an order the running minimum
      // improves a logarithmic number of times instead of at every item, so positions are rarely recovered.
      uint32_t stride = max(1u, (uint32_t)(((uint64_t)seg_len * 40503u) >> 16));
      {
          auto gcd = [](uint32_t x, uint32_t y) { while (y) { const uint32_t z = x % y; x = y; y = z; } return x; };
          while (stride < seg_len && gcd(stride, seg_len) != 1) ++stride;
          if (stride >= seg_len) stride = 1;
      }
      uint32_t place = 0;                                    // (visit * stride) mod seg_len, kept by addition
      for (uint32_t visit = 0; visit < seg_len; ++visit, place = place + stride >= seg_len ? place + stride - seg_len : place + stride) {
        const uint32_t item = seg_first + place;
        const BatchProblem *pr = probs + p;
        // the descriptors are read-only while the kernel runs: wave-uniform fields through scalar loads
        ModelConst mc;
        {
            ConstPtr<uint32_t> words = as_constant(reinterpret_cast<const uint32_t *>(&pr->h.mc));
            uint32_t buf[sizeof(ModelConst) / 4];
#pragma unroll
            for (uint32_t k = 0; k < sizeof(ModelConst) / 4; ++k) buf[k] = words[k];
            __builtin_memcpy(&mc, buf, sizeof(ModelConst));
        }
        ConstPtr<uint32_t> tail = as_constant(&pr->h.first_item);
        const uint32_t work = item - tail[0];
        const uint32_t t0 = (a.split == 1 ? work : work >> 1) * PRUNED_TC;
        // this wave's piece of one group's rows, within the work item's share of the chunk's rows
        const uint32_t task = (work & (a.split - 1)) * BATCH_WAVES + wave;
        const uint32_t n_rows = a.task_cnt[task], row_lo = a.task_lo[task], r = a.task_g[task] & 1;
        const uint32_t T = mc.T;
        const uint32_t nt = min((uint32_t)PRUNED_TC, T - t0);
        ConstPtr<uint32_t> dvw = as_constant(pr->h.X);       // X[4], ndiv[4]
        const uint32_t nd0 = dvw[4], nd1 = dvw[5], nd2 = dvw[6], nd3 = dvw[7];
        if (staged_p != p) {
            // a new problem: its divisor lists into LDS (the previous item's barriers have passed)
            const uint32_t n_list = nd0 + nd1 + nd2 + nd3;
            for (uint32_t k = threadIdx.x; k < n_list; k += BATCH_THREADS) div_lds[k] = pr->list[k];
            staged_p = p;
            __syncthreads();
        }

        if (threadIdx.x < N_OBJ) {
            if (visit == 0) low_p[threadIdx.x] = INF_BITS;
            low_s = INF_BITS;
            low_code[threadIdx.x] = 0xFFFFFFFFu;
        }
        // ---- decode: dimension q of every tiling of the chunk by wave q (beyond the chunk: its last
        // tiling once more, masked out below)
        if (wave < 4) {
            const uint32_t t = t0 + min(lane, nt - 1);
            const uint32_t radix = wave == 0 ? 1u : (wave == 1 ? nd0 : (wave == 2 ? nd0 * nd1 : nd0 * nd1 * nd2));
            const uint32_t nq = wave == 0 ? nd0 : (wave == 1 ? nd1 : (wave == 2 ? nd2 : nd3));
            const uint32_t list0 = wave == 0 ? 0u : (wave == 1 ? nd0 : (wave == 2 ? nd0 + nd1 : nd0 + nd1 + nd2));
            const uint32_t g = div_lds[list0 + (t / radix) % nq];
            gd[wave * PRUNED_TC + lane] = (double)g;
            gd[(4 + wave) * PRUNED_TC + lane] = (double)(dvw[wave] / g);
        }
        __syncthreads();

        // ---- the two operators' costs per stationary mode over all their tile stages (one per wave), and the table entries the rows refer to
        TilingF v;
#pragma unroll
        for (int q = 0; q < 4; ++q) { v.G[q] = gd[q * PRUNED_TC + lane]; v.D[q] = gd[(4 + q) * PRUNED_TC + lane]; }
        const double X[4] = {(double)dvw[0], (double)dvw[1], (double)dvw[2], (double)dvw[3]};
        const double size[5] = {X[DI] * X[DK], X[DK] * X[DL], X[DL] * X[DJ], X[DI] * X[DJ], X[DI] * X[DL]};   // A, B, D, E, C
        if (wave < 6) {
            double words, cycles;
            if (wave < 3) tile_cost_f64(v.G[DI], v.G[DK], v.G[DL], wave, mc, words, cycles);
            else tile_cost_f64(v.G[DI], v.G[DL], v.G[DJ], wave - 3, mc, words, cycles);
            const double stages = v.D[DI] * v.D[DL] * (wave < 3 ? v.D[DK] : v.D[DJ]);
            tc[(wave * 2) * PRUNED_TC + lane] = words * stages;
            tc[(wave * 2 + 1) * PRUNED_TC + lane] = cycles * stages;
        }
        // one kind of table entry per wave (layout.h); the two waves without a tile cost take the 25-entry kinds
        stage_kept(tab + lane, wave, v, size, mc.BH);
        __syncthreads();
        // ---- cost: this wave's rows against the chunk
        const double cap = lane < nt ? mc.cap_words : -1.0;  // a lane beyond the chunk never passes the capacity test

        // Every key is a monotone function of a candidate's DRAM traffic once tiling, recomputation choice
        // and stationary combination are fixed: DRAM energy and DRAM time grow with it, every rounded sum,
        // product and maximum they pass through keeps the order, and the capacity test does not look at the
        // combination.  All rows of a wave's piece share the recomputation choice.  Among the rows that fit,
        // the one with the least traffic therefore has the least cost under every combination and every key
        // -- bit for bit the value a row-by-row minimum gives -- and the loop over the rows only has to keep
        // that least traffic per tiling.  (Rounding may give rows with more traffic the same cost: positions
        // are recovered below by comparing costs, not traffic.)
        // row i of the lists, for the tiling whose table column is `col`
        auto row_words = [&](const char *col, uint32_t i, double room) -> double {
            const uint4 p = rows_lds[i];
            const uint32_t two[4] = {p.x, p.y, p.z, p.w};
            double w[NSEL];
#pragma unroll
            for (int k = 0; k < NSEL; ++k) w[k] = *reinterpret_cast<const double *>(col + (k & 1 ? two[k / 2] >> 16 : two[k / 2] & 0xFFFFu));
            const bool ok = fmax(w[0] + w[2] + w[1], w[3] + w[2] + w[4]) <= room;    // Eq. (1), (2), (4)
            const double dram_words = w[5] + w[6] + w[7];                            // B*H * Eq. (7)
            return ok ? dram_words : inf;
        };
        // the row side of a candidate's costs, from its traffic: DRAM energy (regrouped: DRAM and buffer
        // energy of the DRAM words) and DRAM time, +inf both when no row fits; the words themselves (0 then)
        struct RowSide { double d, e_part, l_dram; };
        auto row_side = [&](double dram_words) {
            RowSide rs;
            const bool feasible = dram_words < inf;
            rs.d = feasible ? dram_words : 0.0;
            const double over = feasible ? 0.0 : inf;
            rs.e_part = fmax((REGROUP ? mc.e_sum : mc.e_dram) * rs.d, over);
            double l_dram;
            if constexpr (FAST) l_dram = rs.d * mc.dram_k;
            else l_dram = mc.dram_bw > 0.0 ? mc.c_lat * (((rs.d / mc.BH) * mc.word) / mc.dram_bw) : 0.0;
            rs.l_dram = fmax(l_dram, over);
            return rs;
        };
        // ... joined with a combination's constants: energy and latency of the candidate
        auto costs_with = [&](const RowSide &rs, double gb_c, double latc_c, double rf_part, double mac_part, double &en, double &lat) {
            if constexpr (REGROUP) {
                en = rs.e_part + gb_c;
            } else {
                const double gb_words = rs.d + gb_c;
                en = rs.e_part + mc.e_gb * gb_words;
                en = en + rf_part;
                en = en + mac_part;
            }
            lat = fmax(rs.l_dram, latc_c);
        };
        // key o of a candidate as a (primary, secondary) pair; the secondary is 0 for the scalar keys
        auto key_of = [&](int o, double en, double lat, double &kp, double &ks) {
            kp = o == 0 ? en : (o == 3 ? en * lat : lat);
            ks = o == 2 ? en : 0.0;
        };

        double min_d;
        if (a.split == 1) min_d = share_least<1, 0>(wave, tab_bytes, cap);
        else if (work & 1) min_d = share_least<2, 1>(wave, tab_bytes, cap);
        else min_d = share_least<2, 0>(wave, tab_bytes, cap);

        // ---- the nine combinations' constants, from the operators' costs (whole numbers: the association is free).  By every wave for
        // itself, and not before it has its rows: as a phase of their own, shared out and exchanged, they took 1400 of a short call's 17 000
        // cycles a block, and their registers through the rows.
        double gb[9], latc[9];
        double e_rf_part = 0.0, e_mac_part = 0.0;
        {
            uint32_t l = lane;
            asm volatile("" : "+v"(l));
            const double rho = r ? gd[(4 + DJ) * PRUNED_TC + l] : 1.0;       // producer repeated per j tile (Sec. V-D)
            const double mac = rho * (X[DI] * X[DK] * X[DL]) + X[DI] * X[DL] * X[DJ], sm = rho * (X[DI] * X[DL]);
            const double e_rf = mc.e_rf * (mc.BH * 3.0 * mac), e_mac = mc.e_mac * (mc.BH * (mac + (double)mc.c_softmax * sm));
            if constexpr (!REGROUP) { e_rf_part = e_rf; e_mac_part = e_mac; }
            double words[6], cycles[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                words[k] = tc[2 * k * PRUNED_TC + l]; cycles[k] = tc[(2 * k + 1) * PRUNED_TC + l];
                if (k < 3) { words[k] = rho * words[k]; cycles[k] = rho * cycles[k]; }
            }
#pragma unroll
            for (int c = 0; c < 9; ++c) {
                const double br = words[c % 3] + words[3 + c / 3];
                gb[c] = REGROUP ? (mc.e_gb * (mc.BH * br) + e_rf) + e_mac : mc.BH * br;
                latc[c] = mc.c_lat * fmax(cycles[c % 3] + cycles[3 + c / 3], buffer_time_general(mc, br));
            }
        }
        auto costs_of = [&](const RowSide &rs, double gb_c, double latc_c, double &en, double &lat) {
            costs_with(rs, gb_c, latc_c, e_rf_part, e_mac_part, en, lat);
        };
        // ---- fold the item into the wave's running best
        {
            double en9[9], lat9[9];
            const RowSide best_row = row_side(min_d);
#pragma unroll
            for (int c9 = 0; c9 < 9; ++c9) costs_of(best_row, gb[c9], latc[c9], en9[c9], lat9[c9]);
            // Only minima were kept; the position is recovered where it can matter, which is long: by the waves that hold the lowest value
            // the block has met so far in the lowest class of candidates -- they meet for it, once for the value and once for the class
            // (1600 chunks, two keys: 57 us from the first block to the last record, now 45).
            // What only a recovered position reads, the nine combinations' constants, the compiler stores to scratch once an item where two keys,
            // the pair or the product are held: 25, 20 and 10 registers at most.  Formed again instead, for the one combination or for
            // all nine at either meeting, it costs more than it saves wherever a block has several items (us a call as it is / one / nine:
            // 40 shapes, 5568 chunks, energy and latency 158 / 164 / 168, energy, where nothing is stored, 124 / 130 / 132; 1600 chunks, energy and
            // latency 53.2 / 54.1 / 55.3) and saves up to 5 % where it has one (484 chunks 31.2 / 30.9 / 29.5).
            double own_p[N_OBJ], own_s[N_OBJ];
            uint32_t own_c[N_OBJ], own_code[N_OBJ];
#pragma unroll
            for (int o = 0; o < N_OBJ; ++o) {
                if (!((MASK >> o) & 1)) continue;
                double mine_p = inf;
#pragma unroll
                for (int c9 = 0; c9 < 9; ++c9) {
                    double kp, ks;
                    key_of(o, en9[c9], lat9[c9], kp, ks);
                    mine_p = fmin(mine_p, kp);
                }
                own_p[o] = uniform_f64(wave_min_f64(mine_p));
                own_p[o] += 0.0;                              // (no -0: bit patterns are compared)
                if (lane == 0)
                    (void)__hip_atomic_fetch_min(&low_p[o], (unsigned long long)__double_as_longlong(own_p[o]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();
#pragma unroll
            for (int o = 0; o < N_OBJ; ++o) {
                if (!((MASK >> o) & 1)) continue;
                own_s[o] = 0.0;
                if (uniform_u64(low_p[o]) != (unsigned long long)__double_as_longlong(own_p[o])) own_p[o] = inf;
                if constexpr (MASK == 4) {
                    double mine_s = inf;
#pragma unroll
                    for (int c9 = 0; c9 < 9; ++c9) mine_s = fmin(mine_s, lat9[c9] == own_p[o] ? en9[c9] : inf);
                    own_s[o] = uniform_f64(wave_min_f64(mine_s)) + 0.0;
                    if (lane == 0 && own_p[o] < inf)
                        (void)__hip_atomic_fetch_min(&low_s, (unsigned long long)__double_as_longlong(own_s[o]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    __syncthreads();
                    if (uniform_u64(low_s) != (unsigned long long)__double_as_longlong(own_s[o])) own_p[o] = inf;
                }
                // the lowest combination in which some tiling reaches the minimum, and its class: index order is (f, combination, r, row, tiling)
                uint32_t cstar = 9;
#pragma unroll
                for (int c9 = 8; c9 >= 0; --c9) {
                    double kp, ks;
                    key_of(o, en9[c9], lat9[c9], kp, ks);
                    cstar = ((kp == own_p[o]) & (ks == own_s[o])) ? (uint32_t)c9 : cstar;
                }
                own_c[o] = __builtin_amdgcn_readfirstlane(wave_min_u32(cstar));
                own_code[o] = (a.task_g[task] >> 1 ? 9u + 2u * own_c[o] : own_c[o]) + r;
                if (lane == 0 && own_p[o] < inf) (void)__hip_atomic_fetch_min(&low_code[o], own_code[o], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            __syncthreads();
#pragma unroll
            for (int o = 0; o < N_OBJ; ++o) {
                if (!((MASK >> o) & 1)) continue;
                const double wave_p = own_p[o], wave_s = own_s[o];
                // nothing feasible, or another wave of the block has it, or this wave already holds a lower value
                if (!(wave_p < inf) || own_code[o] != (uint32_t)__builtin_amdgcn_readfirstlane(low_code[o])) continue;
                if (wave_p > run_p[o] || (wave_p == run_p[o] && wave_s > run_s[o])) continue;
                const uint32_t c_u = own_c[o];
                const uint32_t combo_rows = 30000u * (c_u % 3) + 90000u * (c_u / 3);
                // Index order is (combination, row, tiling).  An equal value only matters where it can sit at a
                // lower index than the running best: in a lower combination; or in the same one in an earlier
                // row, or in the same row if this chunk comes before the running best's.
                // (A wave's pieces all lie in one group's list, whatever the share: list places compare like indices.)
                uint32_t scan = n_rows;
                if (wave_p == run_p[o] && wave_s == run_s[o]) {
                    if (c_u > run_c[o]) continue;
                    if (c_u == run_c[o]) {
                        const uint32_t upto = t0 < run_t0[o] ? run_i[o] + 1 : run_i[o];    // list places below this one matter
                        scan = upto > row_lo ? min(upto - row_lo, n_rows) : 0u;
                    }
                }
                double gb_u = gb[0], latc_u = latc[0];
#pragma unroll
                for (int c9 = 1; c9 < 9; ++c9) {
                    gb_u = c_u == (uint32_t)c9 ? gb[c9] : gb_u;
                    latc_u = c_u == (uint32_t)c9 ? latc[c9] : latc_u;
                }
                // The first row (index order) in which a tiling reaches it, at its lowest such tiling.  Only a
                // tiling whose least-traffic row reaches the value can hold it at all.
                uint32_t found_i = 0xFFFFFFFFu, found_lane = 0;
                double en_u, lat_u, kp_u, ks_u;
                costs_of(best_row, gb_u, latc_u, en_u, lat_u);
                key_of(o, en_u, lat_u, kp_u, ks_u);
                unsigned long long cands = __ballot((kp_u == wave_p) & (ks_u == wave_s));
                if (n_rows <= 64 && 2u * (uint32_t)__popcll(cands) <= scan) {
                    // Few such tilings: take them one by one with lane = row, all rows of the piece at once.
                    while (cands) {
                        const uint32_t l = __builtin_amdgcn_readfirstlane((uint32_t)__ffsll((long long)cands) - 1u);
                        cands &= cands - 1;
                        // (a tiling beyond the chunk's end is never among them: plain capacity)
                        const double words = row_words(reinterpret_cast<const char *>(tab) + l * 8, row_lo + min(lane, n_rows - 1), mc.cap_words);
                        double en, lat, kp, ks;
                        costs_with(row_side(words), lane_value_f64(gb_u, l), lane_value_f64(latc_u, l), lane_value_f64(e_rf_part, l),
                                   lane_value_f64(e_mac_part, l), en, lat);
                        key_of(o, en, lat, kp, ks);
                        const unsigned long long hits = __ballot((lane < scan) & (kp == wave_p) & (ks == wave_s));
                        if (!hits) continue;
                        const uint32_t i = (uint32_t)__ffsll((long long)hits) - 1u;
                        if (i < found_i) { found_i = i; found_lane = l; }     // ascending tilings: the lower one stays on equal rows
                        if (found_i == 0) break;
                    }
                } else {
                    for (uint32_t i = 0; i < scan; ++i) {
                        double en, lat, kp, ks;
                        costs_of(row_side(row_words(tab_bytes, row_lo + i, cap)), gb_u, latc_u, en, lat);
                        key_of(o, en, lat, kp, ks);
                        const unsigned long long hits = __ballot((kp == wave_p) & (ks == wave_s));
                        if (!hits) continue;
                        found_i = i;
                        found_lane = (uint32_t)__ffsll((long long)hits) - 1u;
                        break;
                    }
                }
                if (found_i != 0xFFFFFFFFu) {
                    const uint64_t idx = (uint64_t)t0 + found_lane + (uint64_t)T * (index_row_base(__builtin_amdgcn_readfirstlane(number_lds[row_lo + found_i])) + combo_rows);
                    if (wave_p < run_p[o] || wave_s < run_s[o] || idx < run_idx[o]) {
                        run_p[o] = wave_p; run_s[o] = wave_s; run_idx[o] = idx; run_c[o] = c_u; run_i[o] = row_lo + found_i; run_t0[o] = t0;
                    }
                }
            }
        }

        // ---- after the stretch's last item its record leaves the block
        const bool flush = visit + 1 == seg_len;
        if (!flush) {
            __syncthreads();                                 // every wave is done with the staged tables
            continue;
        }
        if (lane == 0) {
#pragma unroll
            for (int o = 0; o < N_OBJ; ++o) {
                if (!((MASK >> o) & 1)) continue;
                Key k;
                k.p = run_p[o]; k.s = run_s[o]; k.idx = run_idx[o];
                wave_best[o][wave] = k;
            }
        }
        reset_running();
        __syncthreads();
        if (threadIdx.x < N_OBJ && ((MASK >> threadIdx.x) & 1)) {
            const uint32_t o = threadIdx.x;
            Key k = wave_best[o][0];
            for (int wv = 1; wv < BATCH_WAVES; ++wv)
                if (key_less(wave_best[o][wv], k)) k = wave_best[o][wv];
            Key *dst = a.item_keys + (uint64_t)seg_first * N_OBJ + o;
            if (!a.inl.on) *dst = k;                         // read by the finish kernel, after this one
            else {                                           // read by the launch's last block
                __hip_atomic_store(reinterpret_cast<uint64_t *>(&dst->p), (uint64_t)__double_as_longlong(k.p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(reinterpret_cast<uint64_t *>(&dst->s), (uint64_t)__double_as_longlong(k.s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&dst->idx, k.idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (a.inl.on) break;                                 // (one problem: its only stretch)
        __syncthreads();                                     // wave_best and the staged tables are free again
      }
      seg_first = seg_end;
    }
    if (!a.inl.on || wave > 0) return;

    // A launch of one problem: the last block to arrive reduces the blocks' records, its first wave alone.  Records and ticket are
    // agent-scope atomics, which meet where all XCDs see them; the wait keeps the ticket behind the records, so nothing else needs to
    // be written back.  (A second launch for this took 6.5 us from the last record to the result, this 4.)  The last arrival turns the
    // ticket to 0 in the same operation: launches that overlap lose no count, and whole launches leave it at 0.
    const uint32_t n_blocks = gridDim.x;
    uint32_t arrived = 0;
    if (lane == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        arrived = atomicInc(a.ticket, n_blocks - 1);
    }
    if ((uint32_t)__builtin_amdgcn_readfirstlane(arrived) != n_blocks - 1) return;
    uint64_t began = 0;
    if (a.done) began = __hip_atomic_load(a.begin, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    Key best;
    best.p = inf; best.s = 0.0; best.idx = ~0ull;
#pragma unroll
    for (int o = 0; o < N_OBJ; ++o) {
        if (!((MASK >> o) & 1)) continue;
        Key k; k.p = inf; k.s = 0.0; k.idx = ~0ull;
        constexpr int AHEAD = 4;                              // records a lane has under way
        for (uint32_t b0 = lane; b0 < n_blocks; b0 += 64 * AHEAD) {
            uint64_t p[AHEAD], q[AHEAD], idx[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {                 // (beyond the last: it once more)
                Key *src = a.item_keys + (uint64_t)first_item_of(a, min(b0 + 64u * i, n_blocks - 1)) * N_OBJ + o;
                p[i] = __hip_atomic_load(reinterpret_cast<uint64_t *>(&src->p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                q[i] = MASK == 4 ? __hip_atomic_load(reinterpret_cast<uint64_t *>(&src->s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
                idx[i] = __hip_atomic_load(&src->idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                Key c;
                c.p = __longlong_as_double((long long)p[i]); c.s = __longlong_as_double((long long)q[i]); c.idx = idx[i];
                if (key_less(c, k)) k = c;
            }
        }
        k = wave_min(k);
        if (lane == (uint32_t)o) best = k;
    }
    const BatchProblem *pr = probs;
    uint32_t X[4], ndiv[4], before[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        X[q] = as_constant(pr->h.X)[q]; ndiv[q] = as_constant(pr->h.ndiv)[q];
        before[q] = q ? before[q - 1] + ndiv[q - 1] : 0u;
    }
    if (lane < N_OBJ && ((MASK >> lane) & 1)) {
        mmee_result res;
        winner_record_with(a.enc, X, ndiv, [&](int q, uint32_t digit) { return div_lds[before[q] + digit]; }, read_const<ModelConst>((ConstBytes)&pr->h.mc), best, res);
        if (a.packed) {
            res.space = a.space; res.evaluated = a.evaluated;
            *a.packed = res;
        } else
            write_record(a.final_out + (uint64_t)pr->h.slot * N_OBJ + lane, best, res);
        if (a.done) say_done(a.done + lane, a.number, began);
    }
}

// After the search of many problems: one block per problem reduces the problem's records -- one per (block, problem)
// stretch of the search launch, at the problem's first item and at every block boundary inside the
// problem -- and writes the winner's full cost record and mapping.
template <int MASK>
__global__ __launch_bounds__(256) void k_batch_finish(BatchArgs a)
{
    __shared__ Key wave_best[N_OBJ][4];
    __shared__ BatchProblemHead head_s;                      // the problem's description, fetched while the records arrive
    __shared__ DivTable dv_s;
    const double inf = pos_inf();
    const uint32_t p = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const BatchProblem *pr = a.prob + p;
    {
        const uint32_t *src = reinterpret_cast<const uint32_t *>(&pr->h);
        uint32_t *dst = reinterpret_cast<uint32_t *>(&head_s);
        for (uint32_t k = threadIdx.x; k < sizeof(BatchProblemHead) / 4; k += 256) dst[k] = src[k];
        // the packed lists back into the table form the decoding helpers take
        uint32_t first = 0;
        for (int q = 0; q < 4; ++q) {
            const uint32_t n = pr->h.ndiv[q];
            for (uint32_t k = threadIdx.x; k < n; k += 256) dv_s.div[q][k] = pr->list[first + k];
            first += n;
        }
        if (threadIdx.x < 4) { dv_s.X[threadIdx.x] = pr->h.X[threadIdx.x]; dv_s.ndiv[threadIdx.x] = pr->h.ndiv[threadIdx.x]; }
    }
    const uint32_t item0 = pr->h.first_item, n_work = pr->h.n_work;
    const uint32_t inner0 = block_of(a, item0) + 1;          // the block behind the one with the problem's first item
#pragma unroll
    for (int o = 0; o < N_OBJ; ++o) {
        if (!((MASK >> o) & 1)) continue;
        Key k; k.p = inf; k.s = 0.0; k.idx = ~0ull;
        for (uint32_t b = threadIdx.x;; b += 256) {
            const uint64_t at = b == 0 ? item0 : first_item_of(a, inner0 + b - 1);
            if (at >= (uint64_t)item0 + n_work) break;
            const Key c = a.item_keys[at * N_OBJ + o];
            if (key_less(c, k)) k = c;
        }
        k = wave_min(k);
        if (lane == 0) wave_best[o][wave] = k;
    }
    __syncthreads();
    if (threadIdx.x < N_OBJ && ((MASK >> threadIdx.x) & 1)) {
        const int o = threadIdx.x;
        Key k = wave_best[o][0];
        for (int wv = 1; wv < 4; ++wv)
            if (key_less(wave_best[o][wv], k)) k = wave_best[o][wv];
        mmee_result res;
        winner_record(a.enc, dv_s, head_s.mc, k, res);
        write_record(a.final_out + (uint64_t)head_s.slot * N_OBJ + o, k, res);
    }
}

}  // namespace mmee
