// The boundary side of the pruned searches: one tiling's table entries, the two operators' tile costs, the terms of a
// stationary combination, and a winner's full record, each straight from the problem's divisor lists.  Used by
// k_search_batch (batch.h) and k_search_pruned (pruned.h).
#pragma once
#include <utility>
#include "kernels.h"

namespace mmee {

constexpr int PRUNED_TC = 64;                // tilings per work item = lanes of a wave

// ---- the boundary side, one value at a time ---------------------------------------------------
// Every count of the model is an integer below 2^53 (the host refuses workloads where it is not),
// so products and sums of them are exact in fp64 whatever their order.

struct TilingF {                             // boundary vector of one tiling (Eq. (10)), as fp64
    double G[4], D[4];
};

// tile_X * {1, d0, d1, d0 d1}; option 4 = the operand takes no space
__device__ __forceinline__ double footprint(double tile, double d0, double d1, uint32_t opt)
{
    const double v = tile * ((opt & 1) ? d0 : 1.0) * ((opt & 2) ? d1 : 1.0);
    return opt >= 4 ? 0.0 : v;
}

// ceil(a / b) for a whole number 1 <= a < 2^32 held in fp64, given 1 / b rounded once (ModelConst)
__device__ __forceinline__ double cdiv_f64(double a, double rcp_b) { return __builtin_floor((a - 0.5) * rcp_b) + 1.0; }

// words crossing buffer<->RF and cycles of one tile matmul m x r x n; mode 0 WS, 1 IS, 2 OS
__device__ __forceinline__ void tile_cost_f64(double m, double r, double n, uint32_t mode, const ModelConst &mc,
                                              double &words, double &cycles)
{
    const double rd = mode == 0 ? r : m;                     // spread over PE rows
    const double cd = mode == 1 ? r : n;                     // spread over PE columns
    const double time_dim = mode == 0 ? m : (mode == 1 ? n : r);
    const double row_folds = cdiv_f64(rd, mc.rcp_rows);
    words = rd * cd + time_dim * rd * cdiv_f64(cd, mc.rcp_cols_g) + time_dim * cd * row_folds;
    cycles = row_folds * cdiv_f64(cd, mc.rcp_cols) * time_dim;
}

// fl(fl(words * word) / gb_bw), as dram_time_general; scaled back by a power of two, which is exact
__device__ __forceinline__ double buffer_time_general(const ModelConst &mc, double words)
{
    const double x = words * mc.word;
    double q = x * mc.gb_y;
    q = __builtin_fma(__builtin_fma(-mc.gb_b, q, x), mc.gb_y, q);
    q = __builtin_fma(__builtin_fma(-mc.gb_b, q, x), mc.gb_y, q);
    return q * mc.gb_scale;
}

// what one stationary combination (s1, s2) and recomputation choice r contribute for one tiling
struct ComboTerms {
    double br, cyc, mac, sm;                 // buffer<->RF words, cycles, MACs, softmax elements (per instance)
    double lat_part;                         // c_lat * max(cycles, buffer<->RF time)
    double e_rf_part, e_mac_part;
};

// ... from the two operators' tile costs (words and cycles of one tile matmul each)
__device__ __forceinline__ ComboTerms combo_terms_from(const TilingF &v, const double X[4], const ModelConst &mc, uint32_t r,
                                                       double br1, double cy1, double br2, double cy2)
{
    ComboTerms o;
    const double rho = r ? v.D[DJ] : 1.0;                    // producer repeated per j tile (Sec. V-D)
    const double st1 = rho * v.D[DI] * v.D[DK] * v.D[DL], st2 = v.D[DI] * v.D[DL] * v.D[DJ];
    o.br = st1 * br1 + st2 * br2;
    o.cyc = st1 * cy1 + st2 * cy2;
    o.mac = rho * X[DI] * X[DK] * X[DL] + X[DI] * X[DL] * X[DJ];
    o.sm = rho * X[DI] * X[DL];
    const double t_gb = buffer_time_general(mc, o.br);
    o.lat_part = mc.c_lat * fmax(o.cyc, t_gb);
    o.e_rf_part = mc.e_rf * (mc.BH * 3.0 * o.mac);
    o.e_mac_part = mc.e_mac * (mc.BH * (o.mac + (double)mc.c_softmax * o.sm));
    return o;
}

__device__ __forceinline__ ComboTerms combo_terms(const TilingF &v, const double X[4], const ModelConst &mc, uint32_t r,
                                                  uint32_t s1, uint32_t s2)
{
    double br1, cy1, br2, cy2;
    tile_cost_f64(v.G[DI], v.G[DK], v.G[DL], s1, mc, br1, cy1);
    tile_cost_f64(v.G[DI], v.G[DL], v.G[DJ], s2, mc, br2, cy2);
    return combo_terms_from(v, X, mc, r, br1, cy1, br2, cy2);
}

// The cost record of one decoded candidate (Sec. V-D's order of the energy terms, as eval_candidate).  Each selector names an
// entry of a known kind, so an entry is two footprints and a sum: a switch over all kinds per selector, and the
// tiling's digits once for the cost and once for the mapping, were three times the instructions, which a winner's lone thread
// waits for one cache line after the other.
__device__ __forceinline__ void eval_candidate_direct(const uint4 *enc, const uint32_t (&extent)[4], const ModelConst &mc, const mmee_mapping &m,
                                                      mmee_cost &c)
{
    uint32_t row, t;
    split_index(m.idx, mc.T, row, t);
    const uint32_t r = m.recompute, s1 = m.stat1, s2 = m.stat2, f = m.fused;
    const uint4 e = enc[row % ROWS_PER_GROUP + ROWS_PER_GROUP * (r + 2 * f)];
    if (!(sel_of(e, ROW_FLAGS) & 1)) {
        c.bs_words = c.da_words = c.br_words = c.mac_total = c.comp_cycles = 0;
        c.energy_pj = pos_inf(); c.latency_cycles = pos_inf();
        c.valid = 0; c.reason = 1;
        return;
    }
    TilingF v;
#pragma unroll
    for (int q = 0; q < 4; ++q) { v.G[q] = (double)m.xG[q]; v.D[q] = (double)m.xD[q]; }
    const double X[4] = {(double)extent[0], (double)extent[1], (double)extent[2], (double)extent[3]};
    // layout.h: the pairs' options are packed by fours, those of the retained ones by fives (4: not retained)
    auto bs_of = [&](int one, int two, uint32_t opt) { return footprint(v.G[one] * v.G[two], v.D[one], v.D[two], opt); };
    auto da_of = [&](int own0, int own1, int n0, int n1, uint32_t opt) { return footprint(X[own0] * X[own1], v.D[n0], v.D[n1], opt); };
    const uint32_t ab = sel_of(e, 0) - ENT_BS_AB, ret_de = sel_of(e, 1) - ENT_RET_DE, bs_c = sel_of(e, 2) - ENT_BS_C, de = sel_of(e, 3) - ENT_BS_DE,
                   ret_ab = sel_of(e, 4) - ENT_RET_AB, da_ab = sel_of(e, 5) - ENT_DA_AB, da_de = sel_of(e, 6) - ENT_DA_DE, da_c = sel_of(e, 7) - ENT_DA_C;
    const double w_c = bs_of(DI, DL, bs_c);
    const double bs1 = bs_of(DI, DK, ab & 3) + bs_of(DK, DL, ab >> 2) + w_c + (bs_of(DL, DJ, ret_de % 5) + bs_of(DI, DJ, ret_de / 5));
    const double bs2 = bs_of(DL, DJ, de & 3) + bs_of(DI, DJ, de >> 2) + w_c + (bs_of(DI, DK, ret_ab % 5) + bs_of(DK, DL, ret_ab / 5));
    const double through = da_c >= 4 ? 0.0 : X[DI] * X[DL] * (((da_c & 1) ? v.D[DK] : 1.0) + ((da_c & 2) ? v.D[DJ] : 1.0) + 2.0);
    const double bs = fmax(bs1, bs2);                                    // Eq. (1), (2), (4)
    const double da = da_of(DI, DK, DL, DJ, da_ab & 3) + da_of(DK, DL, DI, DJ, da_ab >> 2) +
                      (da_of(DL, DJ, DI, DK, da_de & 3) + da_of(DI, DJ, DK, DL, da_de >> 2)) + through;      // Eq. (7)
    const ComboTerms ct = combo_terms(v, X, mc, r, s1, s2);
    c.bs_words = (uint64_t)bs; c.da_words = (uint64_t)da; c.br_words = (uint64_t)ct.br;
    c.mac_total = (uint64_t)ct.mac; c.comp_cycles = (uint64_t)ct.cyc;
    if (bs > mc.cap_words) {
        c.energy_pj = pos_inf(); c.latency_cycles = pos_inf();
        c.valid = 0; c.reason = 2;
        return;
    }
    double en = mc.e_dram * (mc.BH * da);
    en = en + mc.e_gb * (mc.BH * (da + ct.br));
    en = en + ct.e_rf_part;
    en = en + ct.e_mac_part;
    double l_dram;
    if (mc.bw_pow2) l_dram = da * mc.eval_k;
    else l_dram = (da * mc.word) / mc.dram_bw;
    c.energy_pj = en;
    c.latency_cycles = fmax(mc.c_lat * l_dram, ct.lat_part);
    c.valid = 1; c.reason = 0;
}

// footprints of one operand under its five options (4 = takes no space)
__device__ __forceinline__ void footprints(double (&o)[5], double tile, double d0, double d1)
{
    o[0] = tile; o[1] = tile * d0; o[2] = tile * d1; o[3] = tile * d0 * d1; o[4] = 0.0;
}

// The kept rows (rows.h) in device memory, and the number of lines of the compact table.
__device__ const KeptRows kept_dev = KEPT;
constexpr int KEPT_LINES = (int)KEPT.used;

// The table entries of one kind, for this lane's tiling, into the staged table: x[a] + y[b] for every
// option pair (NA x NB of them, entry number FIRST + a + NA * b) that a kept row refers to.
template <int FIRST, int NA, int A, int B>
__device__ __forceinline__ void stage_pair_sum(double *tab_lane, const double (&x)[5], const double (&y)[5])
{
    constexpr uint32_t AT = KEPT.place[FIRST + A + NA * B];
    if constexpr (AT != (uint32_t)NENT) tab_lane[AT * PRUNED_TC] = x[A] + y[B];
}
template <int FIRST, int NA, int... I>
__device__ __forceinline__ void stage_pair_sums(double *tab_lane, const double (&x)[5], const double (&y)[5], std::integer_sequence<int, I...>)
{
    (stage_pair_sum<FIRST, NA, I % NA, I / NA>(tab_lane, x, y), ...);
}
template <int... C>
__device__ __forceinline__ void stage_c(double *tab_lane, const double (&bs)[5], const double (&da)[5], std::integer_sequence<int, C...>)
{
    auto one = [&](auto c) {
        constexpr int K = decltype(c)::value;
        if constexpr (K < 4 && KEPT.place[ENT_BS_C + (K & 3)] != (uint32_t)NENT) tab_lane[KEPT.place[ENT_BS_C + (K & 3)] * PRUNED_TC] = bs[K];
        if constexpr (KEPT.place[ENT_DA_C + K] != (uint32_t)NENT) tab_lane[KEPT.place[ENT_DA_C + K] * PRUNED_TC] = da[K];
    };
    (one(std::integral_constant<int, C>{}), ...);
}

// Stage the compact table of the chunk, one kind of entry per wave; bh = B*H for scaled DRAM terms, 1 for the raw ones.
__device__ __forceinline__ void stage_kept(double *tab_lane, uint32_t wave, const TilingF &v, const double (&size)[5], double bh)
{
    using Sq4 = std::make_integer_sequence<int, 16>;
    using Sq5 = std::make_integer_sequence<int, 25>;
    double x[5], y[5];
    switch (wave) {
    case 0:                                                   // BS_A[a] + BS_B[b]
        footprints(x, v.G[DI] * v.G[DK], v.D[DI], v.D[DK]);
        footprints(y, v.G[DK] * v.G[DL], v.D[DK], v.D[DL]);
        stage_pair_sums<ENT_BS_AB, 4>(tab_lane, x, y, Sq4{});
        break;
    case 1:                                                   // BS_D[a] + BS_E[b]
        footprints(x, v.G[DL] * v.G[DJ], v.D[DL], v.D[DJ]);
        footprints(y, v.G[DI] * v.G[DJ], v.D[DI], v.D[DJ]);
        stage_pair_sums<ENT_BS_DE, 4>(tab_lane, x, y, Sq4{});
        break;
    case 6:                                                   // tau_D BS_D[a] + tau_E BS_E[b]
        footprints(x, v.G[DL] * v.G[DJ], v.D[DL], v.D[DJ]);
        footprints(y, v.G[DI] * v.G[DJ], v.D[DI], v.D[DJ]);
        stage_pair_sums<ENT_RET_DE, 5>(tab_lane, x, y, Sq5{});
        break;
    case 7:                                                   // tau_A BS_A[a] + tau_B BS_B[b]
        footprints(x, v.G[DI] * v.G[DK], v.D[DI], v.D[DK]);
        footprints(y, v.G[DK] * v.G[DL], v.D[DK], v.D[DL]);
        stage_pair_sums<ENT_RET_AB, 5>(tab_lane, x, y, Sq5{});
        break;
    case 2:                                                   // BS_C[c]; DA_C[c]
        footprints(x, v.G[DI] * v.G[DL], v.D[DI], v.D[DL]);
        // unfused C: spilled by Op1, fetched by Op2, one softmax pass over S and P; option 4: fused
        y[0] = bh * size[4] * 4.0; y[1] = bh * size[4] * (v.D[DK] + 3.0); y[2] = bh * size[4] * (v.D[DJ] + 3.0);
        y[3] = bh * size[4] * (v.D[DK] + v.D[DJ] + 2.0); y[4] = 0.0;
        stage_c(tab_lane, x, y, std::make_integer_sequence<int, 5>{});
        break;
    case 3:                                                   // |A| {1, l_D, j_D, l_D j_D} + |B| {1, i_D, j_D, i_D j_D}
        footprints(x, bh * size[0], v.D[DL], v.D[DJ]);
        footprints(y, bh * size[1], v.D[DI], v.D[DJ]);
        stage_pair_sums<ENT_DA_AB, 4>(tab_lane, x, y, Sq4{});
        break;
    case 4:                                                   // |D| {1, i_D, k_D, i_D k_D} + |E| {1, k_D, l_D, k_D l_D}
        footprints(x, bh * size[2], v.D[DI], v.D[DK]);
        footprints(y, bh * size[3], v.D[DK], v.D[DL]);
        stage_pair_sums<ENT_DA_DE, 4>(tab_lane, x, y, Sq4{});
        break;
    default: break;
    }
}

// X / g for a divisor g of X < 2^32: the reciprocal to about fifty bits, and rounding to the whole number there is
__device__ __forceinline__ double whole_quotient(double X, double g) { return __builtin_rint(X * reciprocal(g)); }

// Digit q of a tiling number.  Quotients by reciprocals (t < 2^22, radix <= 2^22: t + 0.5
// over a whole number stays 2^-23 away from whole numbers, the rounding errors are far below that).
struct DigitConst { double rcp_radix[4], rcp_n[4]; };
__device__ __forceinline__ uint32_t digit_of(uint32_t t, double rcp_radix, double rcp_n, uint32_t n)
{
    const double above = __builtin_floor(((double)t + 0.5) * rcp_radix);
    const double higher = __builtin_floor((above + 0.5) * rcp_n);
    return (uint32_t)(above - higher * (double)n);
}

// a winner's record
template <class Div>
__device__ __forceinline__ void winner_record_with(const uint4 *enc, const uint32_t (&X)[4], const uint32_t (&ndiv)[4], Div &&div, const ModelConst &mc,
                                                   const Key &k, mmee_result &res)
{
    __builtin_memset(&res, 0, sizeof(res));
    if (k.p < pos_inf()) {
        decode_candidate_with(X, ndiv, div, mc.T, k.idx, res.best);
        eval_candidate_direct(enc, X, mc, res.best, res.cost);
    } else {
        res.cost.energy_pj = pos_inf(); res.cost.latency_cycles = pos_inf();
        res.best.idx = ~0ull;
    }
}
__device__ __forceinline__ void winner_record(const uint4 *enc, const DivTable &dv, const ModelConst &mc, const Key &k, mmee_result &res)
{
    winner_record_with(enc, dv.X, dv.ndiv, [&](int q, uint32_t digit) { return dv.div[q][digit]; }, mc, k, res);
}
// Behind a record's last store, by the thread that made it (or one that has met all that did, each past a system-wide fence).
__device__ __forceinline__ void say_done(Done *done, uint64_t number, uint64_t began)
{
    done->ticks = wall_clock64() - began;
    __hip_atomic_store(&done->number, number, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}
__device__ __forceinline__ void write_record(FinalRecord *fr, const Key &k, const mmee_result &res)
{
    fr->key = k;
    __builtin_memcpy(fr->cost, &res.cost, sizeof(mmee_cost));
    __builtin_memcpy(fr->map, &res.best, sizeof(mmee_mapping));
}

}  // namespace mmee
