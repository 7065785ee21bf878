// Both fronts over the kept rows in three launches.
//
// Walking a front point by point (a pass over every candidate, a synchronisation, the next bound) costs a pass and a
// host round trip per point: 23 passes of 26 us and as much again on the host for the 22 points of a 4900-tiling
// problem.  Here k_front_points takes every candidate once: a block per chunk of 64 tilings, lane = tiling, each
// wave with its share of the rows (buffer size / DRAM access) or of the combinations on top of the least
// traffic per class (energy / latency: only those can lie on the front, see pruned.h).  A wave walks its own front
// in registers, the block sorts its waves' points and drops what another one covers; k_front_merge does the same
// for FRONT_FAN blocks' points, and once more for what these leave, and writes the points' full records.
// Short chains decide (a few dozen chunks, one wave per SIMD): a single merge of all chunks' points (some two
// thousand) took 65 us, in two levels it takes 54; with FRONT_FAN blocks or fewer the second merge has nothing to add
// and is left out (one tiling: 61 us, 49 without it).  22 points of a 4900-tiling problem: a call of 0.89 ms walked,
// 0.14 here; energy and latency of 17424 tilings 0.38 ms walked, 0.09 here.
//
// Room.  How many points a wave or a block has is a matter of the extents' divisors: over 600 shapes of attention layers
// and GEMM chains at most 91 in a wave, 431 in the waves of a block, 118 in its front, 2917 in all lists (counted
// on the CPU); over 4200 chains of highly composite extents 339, 1213, 355 and 29481.  So the waves of a block
// share one pool, a block whose waves do not fit it merges them one by one, and a merge takes its lists in as many
// turns as it has room for.  Problems of more than FRONT_CHUNKS chunks are walked, and what outgrows FRONT_BLOCK or
// FRONT_POINTS all the same.
//
// Included once by mmee.hip.
#pragma once
#include "pruned.h"

namespace mmee {

constexpr uint32_t FRONT_CHUNKS = 512;       // chunks of 64 tilings a problem may have
constexpr uint32_t FRONT_SPLIT = 2;          // blocks that share a chunk's rows (buffer size / DRAM access): a wave's 17 rows
                                             // fit its registers, 34 spilled (110 us instead of 68)
constexpr uint32_t FRONT_BLOCKS = FRONT_CHUNKS * FRONT_SPLIT;
constexpr uint32_t FRONT_POOL_BS_DA = 1024, FRONT_POOL_EL = 512;     // points the waves of a block may have together
constexpr uint32_t FRONT_BLOCK = 512;        // points the front of a block may have
constexpr uint32_t FRONT_FAN = 16;           // blocks whose points one block merges
constexpr uint32_t FRONT_LISTS = FRONT_BLOCKS / FRONT_FAN;
constexpr uint32_t FRONT_POINTS = 4096;      // points a merge sorts at a time in LDS, and the most a list or the front may have
constexpr uint32_t FRONT_DIVS = 512;         // divisors of a problem of FRONT_CHUNKS chunks: 240 + 136 + 1 + 1 at most
constexpr uint32_t TOO_MANY = 0xFFFFFFFFu;
constexpr int FRONT_ROWS = (KEPT_ALL + FRONT_SPLIT * PRUNED_WAVES - 1) / (FRONT_SPLIT * PRUNED_WAVES);     // rows per wave

struct FrontArgs {
    ModelConst mc;
    DigitConst dg;
    double extent[4], size[5];
    uint32_t X[4], ndiv[4];
    uint32_t capacity;                       // records the caller has room for
    uint32_t one_merge;                      // not 0: there are at most FRONT_FAN blocks, the last merge takes their points as they are
    uint32_t n_blocks, n_lists;
    Key *points;                             // [FRONT_BLOCKS][FRONT_BLOCK] the blocks' fronts
    Key *lists;                              // [FRONT_LISTS][FRONT_POINTS] those of FRONT_FAN blocks each
    uint32_t *counts;                        // [FRONT_BLOCKS], then [FRONT_LISTS]: their points; TOO_MANY: outgrew its room
    const uint4 *enc;
    FinalRecord *out;                        // [capacity], ascending
    uint32_t *n_out;                         // points of the front; TOO_MANY: walk it
    uint32_t list[FRONT_DIVS];
};

__device__ __forceinline__ Key no_point()
{
    Key k;
    k.p = pos_inf(); k.s = 0.0; k.idx = ~0ull;
    return k;
}

// The front of a wave's candidates into the block's pool: per lane K pairs (P, S) with wave-uniform ids that go up with
// the index.  By ascending P, each point with an S below all before; equal pairs: the lowest id, and all lanes that
// have it.  keep(place, p, s, id, lanes), called by lane 0, stores a point; places come from the counter `filled`, which
// ends above `room` if the pool was too small.  The place asked for in vain at the end holds no point.
template <int K, class Keep>
__device__ __forceinline__ void wave_front(const double (&P)[K], const double (&S)[K], const uint32_t (&id)[K], Key *pool, uint32_t *filled,
                                           uint32_t room, Keep &&keep)
{
    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    double limit = inf;
    for (;;) {
        // (asked for ahead of the reductions: the answer is there when they are)
        uint32_t place = 0;
        if (lane == 0) place = __hip_atomic_fetch_add(filled, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        double bp = inf, bs = inf;
        uint32_t bi = 0xFFFFFFFFu;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const bool better = (S[k] < limit) & ((P[k] < bp) | ((P[k] == bp) & (S[k] < bs)));
            bp = better ? P[k] : bp;
            bs = better ? S[k] : bs;
            bi = better ? id[k] : bi;                        // ids ascend: the first of equals stays
        }
        const double p = uniform_f64(wave_min_f64(bp));
        place = __builtin_amdgcn_readfirstlane(place);
        if (place >= room) return;
        if (!(p < inf)) {
            if (lane == 0) pool[place] = no_point();
            return;
        }
        const double s = uniform_f64(wave_min_f64(bp == p ? bs : inf));
        const uint32_t low = __builtin_amdgcn_readfirstlane(wave_min_u32(bp == p && bs == s ? bi : 0xFFFFFFFFu));
        const unsigned long long who = __ballot(bp == p && bs == s && bi == low);
        if (lane == 0) keep(place, p, s, low, who);
        limit = s;
    }
}

// Bitonic sort of N keys in LDS by the block's THREADS threads (N a power of two), ascending.
template <int THREADS>
__device__ __forceinline__ void block_sort(Key *keys, uint32_t N)
{
    for (uint32_t k = 2; k <= N; k <<= 1)
        for (uint32_t j = k >> 1; j; j >>= 1) {
            __syncthreads();
            for (uint32_t i = threadIdx.x; i < N / 2; i += THREADS) {
                const uint32_t a = 2 * i - (i & (j - 1)), b = a + j;
                const Key ka = keys[a], kb = keys[b];
                if (key_less(kb, ka) == ((a & k) == 0)) { keys[a] = kb; keys[b] = ka; }
            }
        }
    __syncthreads();
}

// Of sorted keys, the number of the front's points up to and including each: keep[i] counts those among keys[0 .. i].  A
// point is on the front if its s is below the s of all before it.  low, keep: N entries each.
template <int THREADS, uint32_t ROOM>
__device__ __forceinline__ uint32_t block_front(const Key *keys, double *low, uint32_t *keep, uint32_t N)
{
    constexpr uint32_t MAX_PER = ROOM / THREADS;
    for (uint32_t i = threadIdx.x; i < N; i += THREADS) low[i] = keys[i].p < pos_inf() ? keys[i].s : pos_inf();
    for (uint32_t d = 1; d < N; d <<= 1) {                   // running minimum, in place: read, meet, write
        double v[MAX_PER];
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < MAX_PER; ++q) {
            const uint32_t i = threadIdx.x + q * THREADS;
            v[q] = i < N && i >= d ? low[i - d] : pos_inf();
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < MAX_PER; ++q) {
            const uint32_t i = threadIdx.x + q * THREADS;
            if (i < N) low[i] = fmin(low[i], v[q]);
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < N; i += THREADS)
        keep[i] = keys[i].p < pos_inf() && (i == 0 || keys[i].s < low[i - 1]) ? 1u : 0u;
    for (uint32_t d = 1; d < N; d <<= 1) {
        uint32_t v[MAX_PER];
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < MAX_PER; ++q) {
            const uint32_t i = threadIdx.x + q * THREADS;
            v[q] = i < N && i >= d ? keep[i - d] : 0u;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t q = 0; q < MAX_PER; ++q) {
            const uint32_t i = threadIdx.x + q * THREADS;
            if (i < N) keep[i] += v[q];
        }
    }
    __syncthreads();
    return keep[N - 1];
}

// points[0 .. n) sorted and the front's among them counted in keep; their number.  N: entries sorted.
template <int THREADS, uint32_t ROOM>
__device__ __forceinline__ uint32_t front_of(Key *points, double *low, uint32_t *keep, uint32_t n, uint32_t &N)
{
    N = 64;
    while (N < n) N <<= 1;
    for (uint32_t i = n + threadIdx.x; i < N; i += THREADS) points[i] = no_point();
    block_sort<THREADS>(points, N);
    return block_front<THREADS, ROOM>(points, low, keep, N);
}

// the points that keep counts to the front of the array
template <int THREADS, uint32_t ROOM>
__device__ __forceinline__ void close_up(Key *points, const uint32_t *keep, uint32_t N)
{
    constexpr uint32_t MAX_PER = ROOM / THREADS;
    double p[MAX_PER], s[MAX_PER];           // (one array per field: an array of keys would live in scratch memory)
    uint64_t idx[MAX_PER];
    uint32_t to[MAX_PER];
#pragma unroll
    for (uint32_t q = 0; q < MAX_PER; ++q) {
        const uint32_t i = min(threadIdx.x + q * THREADS, N - 1);
        to[q] = threadIdx.x + q * THREADS < N && keep[i] != (i ? keep[i - 1] : 0u) ? keep[i] : 0u;
        p[q] = points[i].p; s[q] = points[i].s; idx[q] = points[i].idx;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < MAX_PER; ++q)
        if (to[q]) {
            Key &k = points[to[q] - 1];
            k.p = p[q]; k.s = s[q]; k.idx = idx[q];
        }
    __syncthreads();
}

// Keys: (buffer size, DRAM words, index) with BS_DA, (latency, energy, index) without.
template <bool BS_DA>
__global__ __launch_bounds__(PRUNED_THREADS, BS_DA ? 2 : 4) void k_front_points(FrontArgs a)
{
    constexpr uint32_t POOL = BS_DA ? FRONT_POOL_BS_DA : FRONT_POOL_EL;
    __shared__ double tab[KEPT_LINES * PRUNED_TC];           // entry-major, lane = tiling: conflict-free as it is
    __shared__ double gd[8 * PRUNED_TC];                     // the chunk's boundary vectors: G[0..3], D[0..3] per tiling
    __shared__ double least[BS_DA ? 1 : PRUNED_WAVES][PRUNED_TC];
    __shared__ uint32_t div_lds[FRONT_DIVS];
    __shared__ Key points[POOL];
    __shared__ unsigned long long lanes[BS_DA ? 1 : POOL];
    __shared__ double low_own[BS_DA ? 1 : POOL];
    __shared__ uint32_t keep_own[BS_DA ? 1 : POOL];
    __shared__ uint32_t filled;
    __shared__ double end_s[PRUNED_WAVES], end_p[PRUNED_WAVES];
    // (buffer size / DRAM access: the table has been read when the points are sorted, and two blocks fit a CU)
    static_assert(POOL + POOL / 2 <= KEPT_LINES * PRUNED_TC, "the scans fit the table's room");
    double *low = BS_DA ? tab : low_own;
    uint32_t *keep = BS_DA ? reinterpret_cast<uint32_t *>(tab + POOL) : keep_own;

    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ModelConst &mc = a.mc;
    ConstBytes args = (ConstBytes)__builtin_amdgcn_kernarg_segment_ptr();
    div_lds[threadIdx.x] = ((ConstPtr<uint32_t>)(args + offsetof(FrontArgs, list)))[threadIdx.x];
    if (threadIdx.x == 0) filled = 0;
    __syncthreads();
    const uint32_t t0 = blockIdx.x / (BS_DA ? FRONT_SPLIT : 1) * PRUNED_TC, nt = min((uint32_t)PRUNED_TC, mc.T - t0);
    // dimension q of every tiling of the chunk by wave q (beyond the chunk: its last tiling once more, left out below)
    if (wave < 4) {
        auto f64_at = [&](size_t off) { return ((ConstF64)(args + off))[wave]; };
        const uint32_t list0 = (wave > 0 ? a.ndiv[0] : 0u) + (wave > 1 ? a.ndiv[1] : 0u) + (wave > 2 ? a.ndiv[2] : 0u);
        const uint32_t digit = digit_of(t0 + min(lane, nt - 1), f64_at(offsetof(FrontArgs, dg) + offsetof(DigitConst, rcp_radix)),
                                        f64_at(offsetof(FrontArgs, dg) + offsetof(DigitConst, rcp_n)),
                                        ((ConstPtr<uint32_t>)(args + offsetof(FrontArgs, ndiv)))[wave]);
        const double g = (double)div_lds[list0 + digit];
        gd[wave * PRUNED_TC + lane] = g;
        gd[(4 + wave) * PRUNED_TC + lane] = whole_quotient(f64_at(offsetof(FrontArgs, extent)), g);
    }
    __syncthreads();
    TilingF v;
#pragma unroll
    for (int q = 0; q < 4; ++q) { v.G[q] = gd[q * PRUNED_TC + lane]; v.D[q] = gd[(4 + q) * PRUNED_TC + lane]; }
    stage_kept(tab + lane, wave, v, a.size, 1.0);

    uint32_t m, N;                                           // points of the block's front, entries they are found among
    if constexpr (BS_DA) {
        __syncthreads();
        // every dataflow, the capacity plays no part; neither metric depends on the stationary modes
        typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
        ConstPtr<u32x8> offs = (ConstPtr<u32x8>)&kept_dev.off[0][0];
        double P[FRONT_ROWS], S[FRONT_ROWS];
        uint32_t id[FRONT_ROWS];
        const char *col = reinterpret_cast<const char *>(tab) + lane * 8;
#pragma unroll
        for (int k = 0; k < FRONT_ROWS; ++k) {
            const uint32_t i = (blockIdx.x % FRONT_SPLIT * PRUNED_WAVES + wave) * FRONT_ROWS + k;
            const u32x8 off = offs[min(i, (uint32_t)KEPT_ALL - 1)];
            double w[NSEL];
#pragma unroll
            for (int q = 0; q < NSEL; ++q) w[q] = *reinterpret_cast<const double *>(col + off[q]);
            P[k] = fmax(w[0] + w[2] + w[1], w[3] + w[2] + w[4]);                     // Eq. (1), (2), (4)
            S[k] = i < (uint32_t)KEPT_ALL && lane < nt ? w[5] + w[6] + w[7] : inf;   // Eq. (7)
            id[k] = i;                                       // list places go up with the index
            if (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // (all rows' reads at once would not fit the registers)
        }
        // What the candidate with the least traffic in the block covers goes before the walk: with one or two long
        // extents that is nearly everything (a block of the 240 tilings of a 720720 x 1 x 1 x 1 chain: 67 points in one
        // of its waves, 2 in its front; the call 133 us, 91 us walked point by point, 54 us with this).
        {
            double es = inf, ep = inf;
#pragma unroll
            for (int k = 0; k < FRONT_ROWS; ++k) {
                const bool better = (S[k] < es) | ((S[k] == es) & (P[k] < ep));
                es = better ? S[k] : es;
                ep = better ? P[k] : ep;
            }
            const double s = wave_min_f64(es), p = wave_min_f64(es == s ? ep : inf);
            if (lane == 0) { end_s[wave] = s; end_p[wave] = p; }
            __syncthreads();
            es = end_s[0]; ep = end_p[0];
#pragma unroll
            for (int w = 1; w < PRUNED_WAVES; ++w) {
                const bool better = (end_s[w] < es) | ((end_s[w] == es) & (end_p[w] < ep));
                es = better ? end_s[w] : es;
                ep = better ? end_p[w] : ep;
            }
#pragma unroll
            for (int k = 0; k < FRONT_ROWS; ++k) S[k] = (P[k] >= ep) & (S[k] > es) ? inf : S[k];
        }
        // index so far: the row's place, then its lowest tiling
        auto mine = [&]() {
            wave_front(P, S, id, points, &filled, POOL, [&](uint32_t place, double p, double s, uint32_t row, unsigned long long who) {
                points[place].p = p; points[place].s = s;
                points[place].idx = ((uint64_t)row << 32) | ((uint32_t)__ffsll((long long)who) - 1u);
            });
        };
        mine();
        __syncthreads();
        if (filled <= POOL) {
            m = front_of<PRUNED_THREADS, POOL>(points, low, keep, filled, N);
        } else {
            // more than the pool holds (two long extents with hundreds of divisors): one wave after the other, each
            // beside the front of those before it
            m = 0;
            for (uint32_t turn = 0;; ++turn) {
                __syncthreads();
                if (threadIdx.x == 0) filled = m;
                __syncthreads();
                if (wave == turn) mine();
                __syncthreads();
                const uint32_t n = filled;
                if (n > POOL) { m = TOO_MANY; break; }
                m = front_of<PRUNED_THREADS, POOL>(points, low, keep, n, N);
                if (turn == PRUNED_WAVES - 1) break;
                close_up<PRUNED_THREADS, POOL>(points, keep, N);
            }
        }
    } else {
        {
            const double cap[1] = {mc.cap_words};
            double l[1];
            switch (wave) {
            case 0: least_traffic<0, 0, 3>(v, a.size, cap, l); break;
            case 1: least_traffic<0, 1, 3>(v, a.size, cap, l); break;
            case 2: least_traffic<0, 2, 3>(v, a.size, cap, l); break;
            case 3: least_traffic<1, 0, 2>(v, a.size, cap, l); break;
            case 4: least_traffic<1, 1, 2>(v, a.size, cap, l); break;
            case 5: least_traffic<2, 0, 3>(v, a.size, cap, l); break;
            case 6: least_traffic<2, 1, 3>(v, a.size, cap, l); break;
            default: least_traffic<2, 2, 3>(v, a.size, cap, l); break;
            }
            least[wave][lane] = l[0];
        }
        __syncthreads();
        double d[LEAST_CLASSES];
        d[0] = fmin(fmin(least[0][lane], least[1][lane]), least[2][lane]);
        d[1] = fmin(least[3][lane], least[4][lane]);
        d[2] = fmin(fmin(least[5][lane], least[6][lane]), least[7][lane]);
        RowSide rs[LEAST_CLASSES];
#pragma unroll
        for (int g = 0; g < LEAST_CLASSES; ++g) rs[g] = row_side(mc, lane < nt ? d[g] : nothing_fits());
        // the 18 pairs (combination, r), at most three per wave: two classes with r = 0, one with r = 1; class numbers
        // (each_class) ascending within the wave
        constexpr int PAIRS = (18 + PRUNED_WAVES - 1) / PRUNED_WAVES;
        double P[2 * PAIRS], S[2 * PAIRS];
        uint32_t id[2 * PAIRS];
#pragma unroll
        for (int k = 0; k < PAIRS; ++k) {
            const uint32_t p = wave + PRUNED_WAVES * k, c = p < 9 ? p : p - 9;
            const bool on = p < 18, r = p >= 9;
            const ComboTerms ct = combo_terms(v, a.extent, mc, r, c % 3, c / 3 % 3);
            const RowSide &one = r ? rs[2] : rs[1];
            P[k] = fmax(rs[0].time, ct.lat_part);
            S[k] = on && !r ? energy_of(mc, rs[0], ct.br, ct.e_rf_part, ct.e_mac_part) : inf;
            id[k] = c;
            P[PAIRS + k] = fmax(one.time, ct.lat_part);
            S[PAIRS + k] = on ? energy_of(mc, one, ct.br, ct.e_rf_part, ct.e_mac_part) : inf;
            id[PAIRS + k] = 9u + 2u * c + r;
        }
        // (ids of equal pairs are compared across lanes only after the first of equals per lane: put them in order)
#pragma unroll
        for (int i = 1; i < 2 * PAIRS; ++i)
#pragma unroll
            for (int k = i; k > 0; --k) {
                const bool swap = id[k] < id[k - 1];
                const double p = P[k], s = S[k];
                const uint32_t x = id[k];
                P[k] = swap ? P[k - 1] : p; S[k] = swap ? S[k - 1] : s; id[k] = swap ? id[k - 1] : x;
                P[k - 1] = swap ? p : P[k - 1]; S[k - 1] = swap ? s : S[k - 1]; id[k - 1] = swap ? x : id[k - 1];
            }
        // index so far: the class, then where the lanes are
        wave_front(P, S, id, points, &filled, POOL, [&](uint32_t place, double p, double s, uint32_t code, unsigned long long who) {
            points[place].p = p; points[place].s = s; points[place].idx = ((uint64_t)code << 32) | place;
            lanes[place] = who;
        });
        __syncthreads();
        m = filled <= POOL ? front_of<PRUNED_THREADS, POOL>(points, low, keep, filled, N) : TOO_MANY;
    }
    const bool fits = m <= FRONT_BLOCK;
    if (threadIdx.x == 0) a.counts[blockIdx.x] = fits ? m : TOO_MANY;
    if (!fits) return;
    Key *out = a.points + (uint64_t)blockIdx.x * FRONT_BLOCK;
    if constexpr (BS_DA) {
        for (uint32_t i = threadIdx.x; i < N; i += PRUNED_THREADS) {
            const uint32_t place = keep[i];
            if (place == (i ? keep[i - 1] : 0u)) continue;
            Key k = points[i];
            k.idx = (uint64_t)t0 + (uint32_t)k.idx + (uint64_t)mc.T * index_row_base(kept_dev.number[k.idx >> 32]);
            out[place - 1] = k;
        }
    } else {
        for (uint32_t i = wave; i < N; i += PRUNED_WAVES) {
            const uint32_t place = __builtin_amdgcn_readfirstlane(keep[i]);
            if (place == (i ? __builtin_amdgcn_readfirstlane(keep[i - 1]) : 0u)) {
                if (place == m) break;                       // no more points behind this one
                continue;
            }
            Key k = points[i];
            const uint32_t slot = __builtin_amdgcn_readfirstlane((uint32_t)k.idx);
            const unsigned long long who = lanes[slot];
            ClassBest b;
            b.p = uniform_f64(k.p); b.s = uniform_f64(k.s);
            b.code = __builtin_amdgcn_readfirstlane((uint32_t)(k.idx >> 32));
            b.lanes = ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(who >> 32)) << 32) | __builtin_amdgcn_readfirstlane((uint32_t)who);
            uint32_t cls, combo, row_lo, n_rows;
            class_of_code(b.code, cls, combo);
            rows_of_class(cls, row_lo, n_rows);
            const ComboTerms ct = combo_terms(v, a.extent, mc, cls == 2u, combo % 3, combo / 3);
            const Found f = first_row(tab, ct, mc, nt, (uint32_t)MMEE_OBJ_LATENCY_THEN_ENERGY, b, row_lo, n_rows);
            const uint32_t row = index_row_base(as_constant(kept_dev.number)[row_lo + min(f.row, n_rows - 1)]) + 30000u * (combo % 3) + 90000u * (combo / 3);
            k.idx = (uint64_t)t0 + f.lane + (uint64_t)mc.T * row;
            if (lane == 0) out[place - 1] = k;
        }
    }
}

constexpr int MERGE_THREADS = 1024;

// LAST: the lists of all blocks of the launch before (or the blocks' points themselves, if they are few) into the front's
// records; else FRONT_FAN blocks' points into a list.
// As many lists as there is room for at a time, beside the front of those before.
template <bool LAST>
__global__ __launch_bounds__(MERGE_THREADS) void k_front_merge(FrontArgs a)
{
    __shared__ Key points[FRONT_POINTS];
    __shared__ double low[FRONT_POINTS];
    __shared__ uint32_t keep[FRONT_POINTS];
    __shared__ DivTable dv_s;
    const bool lists = LAST && !a.one_merge;
    const uint32_t source_room = lists ? FRONT_POINTS : FRONT_BLOCK, first = LAST ? 0u : blockIdx.x * FRONT_FAN;
    const uint32_t n_sources = lists ? a.n_lists : min(FRONT_FAN, a.n_blocks - first);
    const Key *from = lists ? a.lists : a.points + (uint64_t)first * FRONT_BLOCK;
    ConstPtr<uint32_t> counts = as_constant(a.counts + (lists ? FRONT_BLOCKS : first));
    uint32_t *n_out = LAST ? a.n_out : a.counts + FRONT_BLOCKS + blockIdx.x;
    if constexpr (LAST) {
        uint32_t at = 0;
        for (int q = 0; q < 4; ++q) {
            for (uint32_t k = threadIdx.x; k < a.ndiv[q]; k += MERGE_THREADS) dv_s.div[q][k] = a.list[at + k];
            at += a.ndiv[q];
        }
        if (threadIdx.x < 4) { dv_s.X[threadIdx.x] = a.X[threadIdx.x]; dv_s.ndiv[threadIdx.x] = a.ndiv[threadIdx.x]; }
    }
    uint32_t m, N, have = 0, q = 0;
    for (;;) {
        const uint32_t before = q;
        bool fits = true;
        for (; q < n_sources; ++q) {
            const uint32_t n = counts[q];                    // the same for all threads: so are the branches
            fits = n <= source_room;
            if (!fits || have + n > FRONT_POINTS) break;
            for (uint32_t i = threadIdx.x; i < n; i += MERGE_THREADS) points[have + i] = from[(uint64_t)q * source_room + i];
            have += n;
        }
        if (!fits || q == before) {
            if (threadIdx.x == 0) *n_out = TOO_MANY;
            return;
        }
        m = front_of<MERGE_THREADS, FRONT_POINTS>(points, low, keep, have, N);
        if (q == n_sources) break;
        close_up<MERGE_THREADS, FRONT_POINTS>(points, keep, N);
        have = m;
    }
    for (uint32_t i = threadIdx.x; i < N; i += MERGE_THREADS) {
        const uint32_t place = keep[i];
        if (place == (i ? keep[i - 1] : 0u)) continue;
        if constexpr (LAST) {
            if (place > a.capacity) continue;
            mmee_result res;
            winner_record(a.enc, dv_s, a.mc, points[i], res);
            write_record(a.out + place - 1, points[i], res);
        } else
            a.lists[(uint64_t)blockIdx.x * FRONT_POINTS + place - 1] = points[i];
    }
    if (threadIdx.x == 0) *n_out = m;
}

}  // namespace mmee
