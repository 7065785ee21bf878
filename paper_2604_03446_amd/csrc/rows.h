// What a row of the query side -- loop order, buffering levels, recomputation choice r, fusion f -- stands for,
// and the rows that can hold the least DRAM traffic.
//
// row_terms is the single statement of the row side of the model: k_build_rows encodes every row with it at run
// time, and least_rows lists at compile time, per (r, f), the rows that are needed to know the least DRAM traffic
// of a tiling under a buffer capacity.  Both use only symbols (which inter-tile loops multiply which term).
#pragma once
#include <stdint.h>
#include "layout.h"

namespace mmee {

// the 24 inter-tile loop orders, outer -> inner, in lexicographic order over i<k<l<j;
// 2 bits per slot, slot 0 = outermost
constexpr uint32_t order_of_rank(uint32_t rank)
{
    uint32_t avail = 0xE4;            // nibble list 3,2,1,0 packed 2 bits each: entry e at bits 2e
    uint32_t packed = 0;
    uint32_t f = 6, left = 4;
    for (uint32_t slot = 0; slot < 4; ++slot) {
        const uint32_t pick = rank / f;
        rank -= pick * f;
        const uint32_t sym = (avail >> (2 * pick)) & 3;
        packed |= sym << (2 * slot);
        // delete entry `pick` from the list
        const uint32_t low = avail & ((1u << (2 * pick)) - 1);
        const uint32_t high = (avail >> (2 * pick + 2)) << (2 * pick);
        avail = low | high;
        --left;
        if (left) f /= left;
    }
    return packed;
}

// selector of a DRAM term: which of the two loops an operand does not own multiply its
// matrix size.  nest_mask: loops of the operand's operator nest; own0/own1: its own dims;
// n0/n1: the other two dims in table order.
constexpr uint32_t dram_selector(const int (&pos)[4], uint32_t nest_mask, uint32_t prefix_mask, int own0, int own1, int n0, int n1,
                                 int level)
{
    // blocker: innermost own loop outside the buffering level (Sec. V-A)
    int bpos = 99, bdim = -1;
    if (pos[own0] >= level) { bpos = pos[own0]; bdim = own0; }
    if (pos[own1] >= level && pos[own1] < bpos) { bpos = pos[own1]; bdim = own1; }
    if (bdim < 0) return 0;                                   // whole matrix resident: fetched once
    uint32_t counted = 0;
    if (level == 0 && ((prefix_mask >> bdim) & 1)) {
        counted = prefix_mask;                                // evicted at every operator switch
    } else {
        for (int q = 0; q < 4; ++q)                           // Scenario 1: blocker and all loops above it
            if (((nest_mask >> q) & 1) && pos[q] >= bpos) counted |= 1u << q;
    }
    return ((counted >> n0) & 1) | (((counted >> n1) & 1) << 1);
}

// The optional factors of every term, as option numbers (layout.h).  Operands in the order A, B, D, E.
struct RowTerms {
    uint32_t bs[4];              // buffer size options
    uint32_t tau;                // bit per operand: retained across operator switches
    uint32_t c;                  // buffer size option of C
    uint32_t da[4];              // DRAM options
    uint32_t dac;                // DRAM option of C, 4 = fused: none
    bool valid;                  // denotes a dataflow
};

constexpr RowTerms row_terms(uint32_t rank, uint32_t r, uint32_t f, const int (&lvl)[4])
{
    RowTerms t{};
    const uint32_t ord = order_of_rank(rank);
    int pos[4] = {0, 0, 0, 0};
    for (int slot = 0; slot < 4; ++slot) pos[(ord >> (2 * slot)) & 3] = 3 - slot;
    // loops iterated by both operators lead the nest (Sec. IV-B); the rest splits per operator
    const uint32_t shared_mask = (1u << DI) | (1u << DL) | (r ? (1u << DJ) : 0u);
    uint32_t prefix_mask = 0;
    for (int slot = 0; slot < 4; ++slot) {
        const uint32_t q = (ord >> (2 * slot)) & 3;
        if (!((shared_mask >> q) & 1)) break;
        prefix_mask |= 1u << q;
    }
    const uint32_t nest1 = prefix_mask | (1u << DI) | (1u << DK) | (1u << DL);
    const uint32_t nest2 = prefix_mask | (1u << DI) | (1u << DL) | (1u << DJ);
    const int own[4][2] = {{DI, DK}, {DK, DL}, {DL, DJ}, {DI, DJ}}, other[4][2] = {{DL, DJ}, {DI, DJ}, {DI, DK}, {DK, DL}};
    for (int y = 0; y < 4; ++y) {
        t.bs[y] = (uint32_t)(pos[own[y][0]] < lvl[y]) | ((uint32_t)(pos[own[y][1]] < lvl[y]) << 1);
        // retained operands (buffered at an inter-tile loop) also occupy the other operator's buffer
        t.tau |= (uint32_t)(lvl[y] >= 1) << y;
        t.da[y] = dram_selector(pos, y < 2 ? nest1 : nest2, prefix_mask, own[y][0], own[y][1], other[y][0], other[y][1], lvl[y]);
    }
    // C holds every tile the producer finishes before the consumer starts (fused), else one tile
    t.c = f ? ((uint32_t)!((prefix_mask >> DI) & 1) | ((uint32_t)!((prefix_mask >> DL) & 1) << 1)) : 0u;
    t.dac = 4;                                                // fused: DA_C = 0 (Sec. V-C)
    if (!f) {
        const uint32_t out_k = dram_selector(pos, nest1, prefix_mask, DI, DL, DK, DJ, 0) & 1;
        const uint32_t in_j = (dram_selector(pos, nest2, prefix_mask, DI, DL, DK, DJ, 0) >> 1) & 1;
        t.dac = out_k | (in_j << 1);
    }
    // recomputation must revisit C tiles (j outside k) and needs an on-chip C
    t.valid = !(r && (!f || pos[DK] > pos[DJ]));
    return t;
}

// symbolic signature: one bit per optional factor of every term; a row whose bits are a
// subset of another's is no larger in any term, for every tiling (all factors are >= 1)
constexpr uint32_t row_signature(const RowTerms &t)
{
    uint32_t s = t.bs[0] | (t.bs[1] << 2) | (t.c << 4) | (t.bs[2] << 6) | (t.bs[3] << 8) | (t.tau << 10);
    for (int y = 0; y < 4; ++y) s |= t.da[y] << (14 + 2 * y);
    return s | ((t.dac & 3u) << 22);
}

// ---- the rows that the least traffic needs -----------------------------------------------------
// Within one (r, f) a row that another one does not exceed in any term never has less traffic, nor fits where
// the other does not.  Unlike the offline stage's list, which must keep the lowest index among equals, the order
// of the rows plays no part here: 65, 39 and 77 rows remain of the 86, 74 and 110 that stage keeps.
constexpr int LEAST_CLASSES = 3;                              // (r, f) = (0, 0), (0, 1), (1, 1), in index order
constexpr int LEAST_MAX = 80;
struct LeastRows {
    int n;
    RowTerms row[LEAST_MAX];
};

constexpr LeastRows least_rows(uint32_t r, uint32_t f)
{
    LeastRows out{};
    uint32_t sig[LEAST_MAX] = {};
    for (uint32_t rank = 0; rank < 24; ++rank) {
        int lvl[4] = {0, 0, 0, 0};
        if (!row_terms(rank, r, f, lvl).valid) continue;
        // per operand, the levels whose options differ from the level below
        int list[4][5] = {}, count[4] = {0, 0, 0, 0};
        for (int y = 0; y < 4; ++y) {
            RowTerms last{};
            for (int p = 0; p < 5; ++p) {
                int l[4] = {0, 0, 0, 0};
                l[y] = p;
                const RowTerms t = row_terms(rank, r, f, l);
                if (p == 0 || t.bs[y] != last.bs[y] || t.da[y] != last.da[y] || t.tau != last.tau) list[y][count[y]++] = p;
                last = t;
            }
        }
        for (int e = 0; e < count[3]; ++e)
            for (int d = 0; d < count[2]; ++d)
                for (int b = 0; b < count[1]; ++b)
                    for (int a = 0; a < count[0]; ++a) {
                        const int l[4] = {list[0][a], list[1][b], list[2][d], list[3][e]};
                        const RowTerms t = row_terms(rank, r, f, l);
                        const uint32_t s = row_signature(t);
                        bool covered = false;
                        for (int k = 0; k < out.n && !covered; ++k) covered = (sig[k] & ~s) == 0;
                        if (covered) continue;
                        int n = 0;                            // drop what the new row covers
                        for (int k = 0; k < out.n; ++k)
                            if ((s & ~sig[k]) != 0) { sig[n] = sig[k]; out.row[n] = out.row[k]; ++n; }
                        sig[n] = s;
                        out.row[n] = t;
                        out.n = n + 1;
                    }
    }
    return out;
}

// ---- the rows that the offline stage keeps, at compile time ---------------------------------------
// Eq. (12) as k_prune_rows applies it: a row goes if a row of its class with a lower number covers it.  A level
// whose options are those of the level below is always covered by it, and covering is transitive, so only
// the distinct levels are walked, in index order, against the rows kept so far.  The library compares the list with
// the device's when it starts.
constexpr int KEPT_MAX = 112;
struct KeptClass {
    int n;
    RowTerms row[KEPT_MAX];
    uint16_t number[KEPT_MAX];               // within its group: levels/order
};

constexpr KeptClass kept_class(uint32_t r, uint32_t f)
{
    KeptClass out{};
    uint32_t sig[KEPT_MAX] = {};
    for (uint32_t rank = 0; rank < 24; ++rank) {
        int lvl[4] = {0, 0, 0, 0};
        if (!row_terms(rank, r, f, lvl).valid) continue;
        int list[4][5] = {}, count[4] = {0, 0, 0, 0};
        for (int y = 0; y < 4; ++y) {
            RowTerms last{};
            for (int p = 0; p < 5; ++p) {
                int l[4] = {0, 0, 0, 0};
                l[y] = p;
                const RowTerms t = row_terms(rank, r, f, l);
                if (p == 0 || t.bs[y] != last.bs[y] || t.da[y] != last.da[y] || t.tau != last.tau) list[y][count[y]++] = p;
                last = t;
            }
        }
        for (int e = 0; e < count[3]; ++e)
            for (int d = 0; d < count[2]; ++d)
                for (int b = 0; b < count[1]; ++b)
                    for (int a = 0; a < count[0]; ++a) {
                        const int l[4] = {list[0][a], list[1][b], list[2][d], list[3][e]};
                        const RowTerms t = row_terms(rank, r, f, l);
                        const uint32_t s = row_signature(t);
                        bool covered = false;
                        for (int k = 0; k < out.n && !covered; ++k) covered = (sig[k] & ~s) == 0;
                        if (covered) continue;
                        sig[out.n] = s;
                        out.row[out.n] = t;
                        out.number[out.n] = (uint16_t)(l[0] + 5 * l[1] + 25 * l[2] + 125 * l[3] + 625 * rank);
                        ++out.n;
                    }
    }
    return out;
}

// the eight table entries of a row (layout.h)
constexpr uint32_t row_entry(const RowTerms &t, int k)
{
    uint32_t ret[4] = {0, 0, 0, 0};
    for (int y = 0; y < 4; ++y) ret[y] = (t.tau >> y) & 1 ? t.bs[y] : 4u;
    const uint32_t e[NSEL] = {ENT_BS_AB + t.bs[0] + 4 * t.bs[1], ENT_RET_DE + ret[2] + 5 * ret[3], ENT_BS_C + t.c,
                              ENT_BS_DE + t.bs[2] + 4 * t.bs[3], ENT_RET_AB + ret[0] + 5 * ret[1], ENT_DA_AB + t.da[0] + 4 * t.da[1],
                              ENT_DA_DE + t.da[2] + 4 * t.da[3], ENT_DA_C + t.dac};
    return e[k];
}

// All kept rows, class after class, and the compact table they refer to: 77 of the 123 entries, one line of
// KEPT_LINE bytes (64 tilings) each.
constexpr int KEPT_ALL = 270, KEPT_LINE = 64 * 8;
struct alignas(32) KeptRows {
    uint32_t off[KEPT_ALL][NSEL];            // a row's entries, as byte offsets of their lines
    uint32_t packed[KEPT_ALL][NSEL / 2];     // ... two to a word
    uint32_t first[LEAST_CLASSES], rows[LEAST_CLASSES];
    uint32_t n, used;
    uint32_t number[KEPT_ALL];               // levels/order + 15000 * (r + 2 f)
    uint32_t place[NENT];                    // table entry -> its line in the compact table, NENT: no row refers to it
};
constexpr KeptClass KEPT_CLASS[LEAST_CLASSES] = {kept_class(0, 0), kept_class(0, 1), kept_class(1, 1)};
constexpr KeptRows kept_rows()
{
    KeptRows k{};
    for (int e = 0; e < NENT; ++e) k.place[e] = NENT;
    for (int c = 0; c < LEAST_CLASSES; ++c) {
        const KeptClass &cls = KEPT_CLASS[c];
        k.first[c] = k.n;
        k.rows[c] = (uint32_t)cls.n;
        for (int i = 0; i < cls.n; ++i, ++k.n) {
            k.number[k.n] = cls.number[i] + ROWS_PER_GROUP * (c == 0 ? 0u : (c == 1 ? 2u : 3u));
            for (int q = 0; q < NSEL; ++q) {
                k.off[k.n][q] = row_entry(cls.row[i], q);
                k.place[k.off[k.n][q]] = 0;
            }
        }
    }
    for (int e = 0; e < NENT; ++e)
        if (k.place[e] == 0) k.place[e] = k.used++;
    for (uint32_t i = 0; i < k.n; ++i)
        for (int q = 0; q < NSEL; ++q) {
            k.off[i][q] = k.place[k.off[i][q]] * KEPT_LINE;
            k.packed[i][q / 2] |= k.off[i][q] << (16 * (q & 1));
        }
    return k;
}
constexpr KeptRows KEPT = kept_rows();
static_assert(KEPT.n == KEPT_ALL && KEPT.used * KEPT_LINE <= 1 << 16, "the arrays are sized for the kept rows, 16 bits hold an offset");

// ---- the kept rows of k_search_batch's waves, in runs --------------------------------------------
// A block's eight waves take a contiguous piece of one class's kept rows each; with two blocks to a chunk (`split`) each of these
// is cut once more.
constexpr int PIECE_WAVES = 8;
constexpr uint32_t PIECE_SPLITS = 2;
constexpr uint32_t WAVES_OF_CLASS[LEAST_CLASSES] = {3, 2, 3};
struct PieceRange { uint32_t cls, lo, n; };                   // within the class's list
constexpr PieceRange piece_range(uint32_t split, uint32_t share, uint32_t wave)
{
    uint32_t c = 0, k = wave;
    while (k >= WAVES_OF_CLASS[c]) k -= WAVES_OF_CLASS[c++];
    const uint32_t n = (uint32_t)KEPT_CLASS[c].n, lo = n * k / WAVES_OF_CLASS[c], cnt = n * (k + 1) / WAVES_OF_CLASS[c] - lo;
    return {c, lo + cnt * share / split, cnt * (share + 1) / split - cnt * share / split};
}

// What the least traffic of a piece needs: the rows that no other row of the piece covers, those with equal (D, E) and
// C entries side by side: a run reads these five entries once, a row its three of A and B.  One block to a chunk: 220 rows in 78 runs,
// 1050 reads per tiling instead of 2160.  Piece: share * 8 + wave.
constexpr int RUNS_MAX = 144;
template <uint32_t SPLIT>
struct PieceRuns {
    uint32_t run[RUNS_MAX][8];               // byte offsets: ret D E, bs C, bs D E, da D E, da C; number of rows
    uint32_t row[KEPT_ALL][4];               // byte offsets: bs A B, ret A B, da A B
    uint32_t first_run[SPLIT * PIECE_WAVES + 1], first_row[SPLIT * PIECE_WAVES];
};
template <uint32_t SPLIT>
constexpr PieceRuns<SPLIT> piece_runs()
{
    PieceRuns<SPLIT> out{};
    uint32_t runs = 0, rows = 0;
    for (uint32_t wave = 0; wave < SPLIT * PIECE_WAVES; ++wave) {
        const PieceRange p = piece_range(SPLIT, wave / PIECE_WAVES, wave % PIECE_WAVES);
        const KeptClass &cls = KEPT_CLASS[p.cls];
        out.first_run[wave] = runs;
        out.first_row[wave] = rows;
        bool gone[KEPT_MAX] = {};
        uint32_t sig[KEPT_MAX] = {};
        for (uint32_t i = 0; i < p.n; ++i) sig[i] = row_signature(cls.row[p.lo + i]);
        for (uint32_t i = 0; i < p.n; ++i)
            for (uint32_t j = 0; j < p.n && !gone[i]; ++j)
                gone[i] = j != i && (sig[j] & ~sig[i]) == 0 && (sig[j] != sig[i] || j < i);
        for (uint32_t i = 0; i < p.n; ++i) {
            if (gone[i]) continue;
            const int of_run[5] = {1, 2, 3, 6, 7}, of_row[3] = {0, 4, 5};
            uint32_t (&run)[8] = out.run[runs++];
            for (int q = 0; q < 5; ++q) run[q] = row_entry(cls.row[p.lo + i], of_run[q]);
            for (uint32_t j = i; j < p.n; ++j) {
                bool same = !gone[j];
                for (int q = 0; q < 5; ++q) same = same && row_entry(cls.row[p.lo + j], of_run[q]) == run[q];
                if (!same) continue;
                gone[j] = true;
                ++run[5];
                for (int q = 0; q < 3; ++q) out.row[rows][q] = KEPT.place[row_entry(cls.row[p.lo + j], of_row[q])] * KEPT_LINE;
                ++rows;
            }
            for (int q = 0; q < 5; ++q) run[q] = KEPT.place[run[q]] * KEPT_LINE;
        }
    }
    out.first_run[SPLIT * PIECE_WAVES] = runs;
    return out;
}
constexpr PieceRuns<1> PIECE_RUNS_1 = piece_runs<1>();        // (no variable template: the device compiler reads one from memory)
constexpr PieceRuns<2> PIECE_RUNS_2 = piece_runs<2>();
static_assert(PIECE_RUNS_1.first_run[PIECE_WAVES] <= RUNS_MAX && PIECE_RUNS_2.first_run[2 * PIECE_WAVES] <= RUNS_MAX, "the arrays hold them");
template <uint32_t SPLIT>
constexpr const PieceRuns<SPLIT> &pieces()
{
    if constexpr (SPLIT == 1) return PIECE_RUNS_1;
    else return PIECE_RUNS_2;
}

constexpr LeastRows LEAST[LEAST_CLASSES] = {least_rows(0, 0), least_rows(0, 1), least_rows(1, 1)};

// The same rows as places in the compact table (every one of them is among the kept rows, up to equal terms), class after
// class, and how eight waves share them, each a piece of one class.
constexpr int LEAST_ALL = LEAST[0].n + LEAST[1].n + LEAST[2].n, LEAST_WAVES = 8;
struct alignas(32) LeastOffsets {
    uint32_t off[LEAST_ALL][NSEL];           // byte offsets of the entries' lines
    uint32_t lo[LEAST_WAVES], hi[LEAST_WAVES], cls[LEAST_WAVES];
};
constexpr LeastOffsets least_offsets()
{
    LeastOffsets o{};
    const int pieces[LEAST_CLASSES] = {3, 2, 3};
    uint32_t first = 0;
    int wave = 0;
    for (int c = 0; c < LEAST_CLASSES; ++c) {
        const uint32_t n = (uint32_t)LEAST[c].n;
        for (uint32_t i = 0; i < n; ++i)
            for (int q = 0; q < NSEL; ++q) o.off[first + i][q] = KEPT.place[row_entry(LEAST[c].row[i], q)] * KEPT_LINE;
        for (int k = 0; k < pieces[c]; ++k, ++wave) {
            o.lo[wave] = first + n * k / pieces[c];
            o.hi[wave] = first + n * (k + 1) / pieces[c];
            o.cls[wave] = (uint32_t)c;
        }
        first += n;
    }
    return o;
}
constexpr LeastOffsets LEAST_OFF = least_offsets();
constexpr bool least_is_staged()
{
    for (int i = 0; i < LEAST_ALL; ++i)
        for (int q = 0; q < NSEL; ++q)
            if (LEAST_OFF.off[i][q] >= KEPT.used * KEPT_LINE) return false;
    return true;
}
static_assert(least_is_staged(), "the compact table has all their entries");

}  // namespace mmee
