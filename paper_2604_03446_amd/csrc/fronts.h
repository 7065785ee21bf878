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
// thousand) took 65 us, in two levels it takes 54.  22 points of a 4900-tiling problem: a call of 0.89 ms walked, 0.14 here; energy and
// latency of 17424 tilings 0.38 ms walked, 0.10 here.
//
// For problems of at most FRONT_CHUNKS chunks; larger ones, and lists that outgrow their room, are walked.
//
// Included once by mmee.hip.
#pragma once
#include "pruned.h"

namespace mmee {

constexpr uint32_t FRONT_CHUNKS = 512;       // chunks of 64 tilings a problem may have
constexpr uint32_t FRONT_SPLIT = 2;          // blocks that share a chunk's rows (buffer size / DRAM access): a wave's 17 rows
                                             // fit its registers, 34 spilled (110 us instead of 68)
constexpr uint32_t FRONT_BLOCKS = FRONT_CHUNKS * FRONT_SPLIT;
constexpr uint32_t FRONT_WAVE = 64;          // points the front of a wave, and that of a block, may have
constexpr uint32_t FRONT_FAN = 16;           // blocks whose points one block merges
constexpr uint32_t FRONT_LISTS = FRONT_BLOCKS / FRONT_FAN;
constexpr uint32_t FRONT_LIST = FRONT_FAN * FRONT_WAVE;      // points such a list may have
constexpr uint32_t FRONT_POINTS = 4096;      // points all of them may have together: what one block sorts in LDS
constexpr uint32_t FRONT_DIVS = 512;         // divisors of a problem of FRONT_CHUNKS chunks: 240 + 136 + 1 + 1 at most
constexpr uint32_t TOO_MANY = 0xFFFFFFFFu;
constexpr int FRONT_ROWS = (KEPT_ALL + FRONT_SPLIT * PRUNED_WAVES - 1) / (FRONT_SPLIT * PRUNED_WAVES);     // rows per wave

struct FrontArgs {
    ModelConst mc;
    DigitConst dg;
    double extent[4], size[5];
    uint32_t X[4], ndiv[4];
    uint32_t capacity, pad_;                 // records the caller has room for
    uint32_t n_blocks, n_lists;
    Key *points;                             // [FRONT_BLOCKS][FRONT_WAVE] the blocks' fronts
    Key *lists;                              // [FRONT_LISTS][FRONT_LIST] those of FRONT_FAN blocks each
    uint32_t *counts;                        // [FRONT_BLOCKS], then [FRONT_LISTS]: their points; TOO_MANY: outgrew its room
    const uint4 *enc;
    FinalRecord *out;                        // [capacity], ascending
    uint32_t *n_out;                         // points of the front; TOO_MANY: walk it
    uint32_t list[FRONT_DIVS];
};

// The front of a wave's candidates: per lane K pairs (P, S) with wave-uniform ids that go up with the index.  By
// ascending P, each point with an S below all before; equal pairs: the lowest id, and all lanes that have it.  Returns
// the number of points, FRONT_WAVE + 1 if there are more than fit.
template <int K>
__device__ __forceinline__ uint32_t wave_front(const double (&P)[K], const double (&S)[K], const uint32_t (&id)[K], Key *points,
                                               unsigned long long *lanes)
{
    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    double limit = inf;
    for (uint32_t n = 0;; ++n) {
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
        if (!(p < inf)) return n;
        if (n == FRONT_WAVE) return n + 1;
        const double s = uniform_f64(wave_min_f64(bp == p ? bs : inf));
        const uint32_t low = __builtin_amdgcn_readfirstlane(wave_min_u32(bp == p && bs == s ? bi : 0xFFFFFFFFu));
        const unsigned long long who = __ballot(bp == p && bs == s && bi == low);
        if (lane == 0) {
            points[n].p = p; points[n].s = s; points[n].idx = low;
            lanes[n] = who;
        }
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
template <int THREADS>
__device__ __forceinline__ uint32_t block_front(const Key *keys, double *low, uint32_t *keep, uint32_t N)
{
    constexpr uint32_t MAX_PER = FRONT_POINTS / THREADS > 0 ? FRONT_POINTS / THREADS : 1;
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

// Keys: (buffer size, DRAM words, index) with BS_DA, (latency, energy, index) without.
template <bool BS_DA>
__global__ __launch_bounds__(PRUNED_THREADS, BS_DA ? 2 : 4) void k_front_points(FrontArgs a)
{
    constexpr uint32_t N = PRUNED_WAVES * FRONT_WAVE;
    __shared__ double tab[KEPT_LINES * PRUNED_TC];           // entry-major, lane = tiling: conflict-free as it is
    __shared__ double gd[8 * PRUNED_TC];                     // the chunk's boundary vectors: G[0..3], D[0..3] per tiling
    __shared__ double least[PRUNED_WAVES][PRUNED_TC];
    __shared__ uint32_t div_lds[FRONT_DIVS];
    __shared__ Key points[N];
    __shared__ unsigned long long lanes[N];
    __shared__ double low[N];
    __shared__ uint32_t keep[N];
    __shared__ uint32_t outgrown;

    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ModelConst &mc = a.mc;
    ConstBytes args = (ConstBytes)__builtin_amdgcn_kernarg_segment_ptr();
    div_lds[threadIdx.x] = ((ConstPtr<uint32_t>)(args + offsetof(FrontArgs, list)))[threadIdx.x];
    points[threadIdx.x].p = inf; points[threadIdx.x].s = 0.0; points[threadIdx.x].idx = ~0ull;
    if (threadIdx.x == 0) outgrown = 0;
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

    uint32_t n_mine;
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
        n_mine = wave_front(P, S, id, points + wave * FRONT_WAVE, lanes + wave * FRONT_WAVE);
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
        n_mine = wave_front(P, S, id, points + wave * FRONT_WAVE, lanes + wave * FRONT_WAVE);
    }
    if (n_mine > FRONT_WAVE) {
        if (lane == 0) outgrown = 1;
    } else if (lane < n_mine) {
        // index so far: class or row first, then where the lanes are; a row's lowest tiling is known already
        Key &k = points[wave * FRONT_WAVE + lane];
        k.idx = (k.idx << 32) | (wave * FRONT_WAVE + lane);
    }

    block_sort<PRUNED_THREADS>(points, N);
    const uint32_t m = block_front<PRUNED_THREADS>(points, low, keep, N);
    const bool fits = !outgrown && m <= FRONT_WAVE;          // (the sort's barriers lie between)
    if (threadIdx.x == 0) a.counts[blockIdx.x] = fits ? m : TOO_MANY;
    if (!fits) return;
    for (uint32_t i = wave; i < N; i += PRUNED_WAVES) {
        const uint32_t place = __builtin_amdgcn_readfirstlane(keep[i]);
        if (place == (i ? __builtin_amdgcn_readfirstlane(keep[i - 1]) : 0u)) {
            if (place == m) break;                           // no more points behind this one
            continue;
        }
        Key k = points[i];
        const uint32_t id = __builtin_amdgcn_readfirstlane((uint32_t)(k.idx >> 32)), slot = __builtin_amdgcn_readfirstlane((uint32_t)k.idx);
        const unsigned long long who64 = lanes[slot];
        const unsigned long long who = ((unsigned long long)__builtin_amdgcn_readfirstlane((uint32_t)(who64 >> 32)) << 32) |
                                       __builtin_amdgcn_readfirstlane((uint32_t)who64);
        uint32_t row, l;
        if constexpr (BS_DA) {
            row = index_row_base(as_constant(kept_dev.number)[id]);
            l = (uint32_t)__ffsll((long long)who) - 1u;
        } else {
            ClassBest b;
            b.p = uniform_f64(k.p); b.s = uniform_f64(k.s); b.code = id; b.lanes = who;
            uint32_t cls, combo, row_lo, n_rows;
            class_of_code(id, cls, combo);
            rows_of_class(cls, row_lo, n_rows);
            const ComboTerms ct = combo_terms(v, a.extent, mc, cls == 2u, combo % 3, combo / 3);
            const uint4 *offs = reinterpret_cast<const uint4 *>(&kept_dev.off[0][0]);
            const Found f = first_row(tab, [&](uint32_t q) { return offs[q]; }, ct, mc, nt, (uint32_t)MMEE_OBJ_LATENCY_THEN_ENERGY, b, row_lo, n_rows);
            row = index_row_base(as_constant(kept_dev.number)[row_lo + min(f.row, n_rows - 1)]) + 30000u * (combo % 3) + 90000u * (combo / 3);
            l = f.lane;
        }
        k.idx = (uint64_t)t0 + l + (uint64_t)mc.T * row;
        if (lane == 0) a.points[blockIdx.x * FRONT_WAVE + place - 1] = k;
    }
}

constexpr int MERGE_THREADS = 1024;

// LAST: the lists of all blocks of the launch before into the front's records; else FRONT_FAN blocks' points into a list.
template <bool LAST>
__global__ __launch_bounds__(MERGE_THREADS) void k_front_merge(FrontArgs a)
{
    constexpr uint32_t ROOM = LAST ? FRONT_POINTS : FRONT_LIST, SOURCES = LAST ? FRONT_LISTS : FRONT_FAN;
    constexpr uint32_t SOURCE_ROOM = LAST ? FRONT_LIST : FRONT_WAVE;
    __shared__ Key points[ROOM];
    __shared__ double low[ROOM];
    __shared__ uint32_t keep[ROOM];
    __shared__ DivTable dv_s;
    const double inf = pos_inf();
    const uint32_t first = LAST ? 0u : blockIdx.x * FRONT_FAN, n_sources = min(SOURCES, (LAST ? a.n_lists : a.n_blocks) - first);
    const Key *from = LAST ? a.lists : a.points + (uint64_t)first * FRONT_WAVE;
    ConstPtr<uint32_t> counts = as_constant(a.counts + (LAST ? FRONT_BLOCKS : first));
    uint32_t total = 0;
    for (uint32_t q = 0; q < n_sources; ++q) {
        const uint32_t n = counts[q];                        // the same for all threads: so are the returns
        if (n > SOURCE_ROOM || total + n > ROOM) {
            if (threadIdx.x == 0) *(LAST ? a.n_out : a.counts + FRONT_BLOCKS + blockIdx.x) = TOO_MANY;
            return;
        }
        for (uint32_t i = threadIdx.x; i < n; i += MERGE_THREADS) points[total + i] = from[(uint64_t)q * SOURCE_ROOM + i];
        total += n;
    }
    uint32_t N = 64;
    while (N < total) N <<= 1;
    for (uint32_t i = total + threadIdx.x; i < N; i += MERGE_THREADS) {
        Key k;
        k.p = inf; k.s = 0.0; k.idx = ~0ull;
        points[i] = k;
    }
    if constexpr (LAST) {
        uint32_t at = 0;
        for (int q = 0; q < 4; ++q) {
            for (uint32_t k = threadIdx.x; k < a.ndiv[q]; k += MERGE_THREADS) dv_s.div[q][k] = a.list[at + k];
            at += a.ndiv[q];
        }
        if (threadIdx.x < 4) { dv_s.X[threadIdx.x] = a.X[threadIdx.x]; dv_s.ndiv[threadIdx.x] = a.ndiv[threadIdx.x]; }
    }
    block_sort<MERGE_THREADS>(points, N);
    const uint32_t m = block_front<MERGE_THREADS>(points, low, keep, N);
    for (uint32_t i = threadIdx.x; i < N; i += MERGE_THREADS) {
        const uint32_t place = keep[i];
        if (place == (i ? keep[i - 1] : 0u)) continue;
        if constexpr (LAST) {
            if (place > a.capacity) continue;
            mmee_result res;
            winner_record(a.enc, dv_s, a.mc, points[i], res);
            write_record(a.out + place - 1, points[i], res);
        } else
            a.lists[(uint64_t)blockIdx.x * FRONT_LIST + place - 1] = points[i];
    }
    if (threadIdx.x == 0) *(LAST ? a.n_out : a.counts + FRONT_BLOCKS + blockIdx.x) = m;
}

}  // namespace mmee
