// Both fronts over the kept rows in two launches.
//
// Walking a front point by point (a pass over every candidate, a synchronisation, the next bound) costs a pass and a
// host round trip per point: 23 passes of 26 us and as much again on the host for the 22 points of a 4900-tiling
// problem.  Here k_front_points takes every candidate once: a block per chunk of 64 tilings, lane = tiling, each
// wave with its share of the rows (buffer size / DRAM access) or of the combinations on top of the least
// traffic per class (energy / latency: only those can lie on the front, see pruned.h).
//
// Nearly all of them lie far behind the front, and a look at a coarse staircase shows it.  The first metric's range is cut
// into FRONT_STEPS steps; per step the least second metric of any candidate, first of the block, then of the whole
// launch (atomic minima in memory that every block publishes to and reads back).  A candidate whose second metric is no lower
// than the least of the steps below its own is covered, whoever has that least, and goes; which blocks have published
// by then changes only how much goes at once.  What is left of a wave, a handful, is walked in registers: a
// wave's own front; the block drops what another of its waves covers and appends the rest to one list.  k_front_merge,
// one block, looks at the staircase again, complete by now, settles what passes pair by pair, and writes the records.
//
// Short chains decide (a few dozen chunks, one wave per SIMD).  With walks of everything (30 to 60 points a wave, 1 us
// each), a bitonic sort per block and two levels of merges that sorted thousands of points, the 22 points of a
// 4900-tiling problem took 65 + 27 + 26 us in three launches (a call of 134 us; walked 890), energy and latency of 17424 tilings
// 34 + 16 + 22 (87 us; walked 380).  Now 30 + 12 us
// (call 58) and 31 + 10 (50).
//
// Room.  How many points a wave or a block has is a matter of the extents' divisors: without the staircase, over 600 shapes of
// attention layers and GEMM chains at most 91 in a wave, 431 in the waves of a block, 118 in its front, 2917 in all blocks' (counted
// on the CPU); over 4200 chains of highly composite extents 339, 1213, 355 and 29481.  So the waves of a block
// share one pool, a block whose waves do not fit it merges them one by one, and the merge takes the list in as many
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
constexpr uint32_t FRONT_POINTS = 4096;      // points the merge takes at a time in LDS, and the most the front may have
constexpr uint32_t FRONT_STEPS = 512;        // steps of the staircase: one per thread of a block
constexpr uint32_t FRONT_DIVS = 512;         // divisors of a problem of FRONT_CHUNKS chunks: 240 + 136 + 1 + 1 at most
constexpr uint32_t TOO_MANY = 0xFFFFFFFFu;
// Which way a front took (mmee_front_way): a block's front outgrew FRONT_BLOCK or its pool; a block's points were sorted, or
// merged wave by wave; the merge took the list in several turns, sorted what was left at the end, or before.
enum : uint32_t { WAY_OUTGROWN = 1, WAY_POOL_SORTED = 2, WAY_WAVE_BY_WAVE = 4, WAY_TURNS = 8, WAY_SORTED = 16, WAY_SORTED_EARLY = 32 };
constexpr int FRONT_ROWS = (KEPT_ALL + FRONT_SPLIT * PRUNED_WAVES - 1) / (FRONT_SPLIT * PRUNED_WAVES);     // rows per wave

struct FrontArgs {
    ModelConst mc;
    DigitConst dg;
    double extent[4], size[5];
    uint32_t X[4], ndiv[4];
    uint32_t capacity;                       // records the caller has room for
    uint32_t pool;                           // points the waves of a block may have together, at most POOL
    uint32_t step_shift;                     // a value's step: the upper word of its fp64, shifted, less step0, held to
    int32_t step0;                           // 0 .. FRONT_STEPS - 1 (goes up with the value, whatever these two are)
    Key *points;                             // [FRONT_BLOCKS * FRONT_BLOCK] the blocks' fronts, block after block as they end
    unsigned long long *stairs;              // [FRONT_STEPS] least second metric per step (bit patterns), +inf between calls
    uint32_t *counts;                        // [0] points in the list; [1] which way the blocks took; 0 between calls
    const uint4 *enc;
    FinalRecord *out;                        // [capacity], ascending
    uint32_t *n_out;                         // [0] points of the front; TOO_MANY: walk it.  [1] which way it took
    Done *done;                              // where the host looks for the call's end
    uint64_t number, *begin;                 // the call's number; when it began (device memory)
    uint32_t list[FRONT_DIVS];
};

__device__ __forceinline__ Key no_point()
{
    Key k;
    k.p = pos_inf(); k.s = 0.0; k.idx = ~0ull;
    return k;
}

// ---- the staircase

__device__ __forceinline__ uint32_t step_of(const FrontArgs &a, double p)
{
    const int b = (int)((uint32_t)__double2hiint(p) >> a.step_shift) - a.step0;
    return (uint32_t)min(max(b, 0), (int)FRONT_STEPS - 1);
}

// below[b] = the least of own over the steps below b; own: step threadIdx.x's, for the first FRONT_STEPS threads.  Ends with a
// barrier.
__device__ __forceinline__ void steps_below(double own, double *below, double (&wave_least)[FRONT_STEPS / 64])
{
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double least = own;                                      // of this step and those before it in the wave
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const double v = __shfl_up(least, d);
        least = lane >= (uint32_t)d ? fmin(least, v) : least;
    }
    if (wave < FRONT_STEPS / 64 && lane == 63) wave_least[wave] = least;
    __syncthreads();
    double before = __shfl_up(least, 1);
    before = lane ? before : pos_inf();
#pragma unroll
    for (uint32_t w = 0; w < FRONT_STEPS / 64; ++w) before = w < wave ? fmin(before, wave_least[w]) : before;
    if (threadIdx.x < FRONT_STEPS) below[threadIdx.x] = before;
    __syncthreads();
}

// The block's candidates against its own and the launch's staircase: the S of what is covered becomes +inf.
template <int K>
__device__ __forceinline__ void drop_covered(const FrontArgs &a, const double (&P)[K], double (&S)[K], unsigned long long *steps,
                                             double (&wave_least)[FRONT_STEPS / 64])
{
    static_assert(FRONT_STEPS == PRUNED_THREADS, "a step per thread");
    steps[threadIdx.x] = INF_BITS;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        // (a look first: most candidates lower nothing, and minima on one address take turns)
        unsigned long long *at = steps + step_of(a, P[k]);
        const unsigned long long bits = (unsigned long long)__double_as_longlong(S[k]);
        if (bits < __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
            (void)__hip_atomic_fetch_min(at, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
    const unsigned long long mine = steps[threadIdx.x];
    unsigned long long all = __hip_atomic_load(a.stairs + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (mine < all) {
        (void)__hip_atomic_fetch_min(a.stairs + threadIdx.x, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        all = mine;
    }
    double *below = reinterpret_cast<double *>(steps);       // (each thread has taken its entry)
    steps_below(__longlong_as_double((long long)all), below, wave_least);
#pragma unroll
    for (int k = 0; k < K; ++k) S[k] = S[k] < below[step_of(a, P[k])] ? S[k] : pos_inf();
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
        // (asked for ahead of the reductions: the answer is there when they are; the wave meets first, or the compiler may
        // join lane 0's branch at the end of a turn with this one and send the other lanes round without it)
        __builtin_amdgcn_wave_barrier();
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

// The front of points[0 .. n), n <= THREADS, to the front of the array, in any order; its size.  Pair by pair: a point goes if
// one before it (Key order) has no larger s.  Every point's comparisons are shared out over PARTS threads.
// 256 points and fewer in some 2 us where the sort and the two scans take 13: their barriers are one after the other.
template <int THREADS>
__device__ __forceinline__ uint32_t front_by_pairs(Key *points, uint32_t *gone, uint32_t *left, uint32_t n)
{
    __syncthreads();
    if (threadIdx.x < n) gone[threadIdx.x] = 0;
    if (threadIdx.x == 0) *left = 0;
    __syncthreads();
    uint32_t parts = 1;                                      // (uniform)
    while (parts < 16 && n * parts * 2 <= THREADS) parts *= 2;
    const uint32_t i = threadIdx.x / parts;
    if (i < n) {
        const Key me = points[i];
        bool covered = !(me.p < pos_inf());
        for (uint32_t j = threadIdx.x % parts; j < n; j += parts) {
            const Key k = points[j];
            covered |= k.s <= me.s && key_less(k, me);
        }
        if (covered) gone[i] = 1;
    }
    __syncthreads();
    Key me = no_point();
    const bool stays = threadIdx.x < n && !gone[threadIdx.x];
    if (stays) me = points[threadIdx.x];
    __syncthreads();
    if (stays) points[__hip_atomic_fetch_add(left, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] = me;
    __syncthreads();
    return *left;
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
    __shared__ uint32_t keep_own[BS_DA ? 1 : POOL];
    __shared__ unsigned long long steps[FRONT_STEPS];
    __shared__ double wave_least[FRONT_STEPS / 64];
    __shared__ uint32_t filled, n_left, list_at;
    // (buffer size / DRAM access: the table has been read when the points are sorted, and two blocks fit a CU)
    static_assert(POOL + POOL / 2 <= KEPT_LINES * PRUNED_TC, "the scans fit the table's room");
    [[maybe_unused]] double *low = tab;                      // (sorts: buffer size / DRAM access only)
    uint32_t *keep = BS_DA ? reinterpret_cast<uint32_t *>(tab + POOL) : keep_own;

    const double inf = pos_inf();
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const ModelConst &mc = a.mc;
    const uint32_t room = min(a.pool, POOL);
    // (here and in the merge: an energy-latency front of 1024 x 96 42.3 us a call without, 41.3 with)
    if (wave == PRUNED_WAVES - 1) ask_for_arguments<FrontArgs>(lane);
    if (blockIdx.x == 0 && threadIdx.x == 0) *a.begin = wall_clock64();
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

    uint32_t m, N, way = 0;                                  // points of the block's front, entries sorted, which way
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
        drop_covered(a, P, S, steps, wave_least);
        // index so far: the row's place, then its lowest tiling
        auto mine = [&]() {
            wave_front(P, S, id, points, &filled, room, [&](uint32_t place, double p, double s, uint32_t row, unsigned long long who) {
                points[place].p = p; points[place].s = s;
                points[place].idx = ((uint64_t)row << 32) | ((uint32_t)__ffsll((long long)who) - 1u);
            });
        };
        mine();
        __syncthreads();
        if (filled <= min(room, (uint32_t)PRUNED_THREADS)) {
            m = front_by_pairs<PRUNED_THREADS>(points, keep, &n_left, filled);
        } else if (filled <= room) {
            way = WAY_POOL_SORTED;
            m = front_of<PRUNED_THREADS, POOL>(points, low, keep, filled, N);
            close_up<PRUNED_THREADS, POOL>(points, keep, N);
        } else {
            // more than the pool holds (two long extents with hundreds of divisors): one wave after the other, each
            // beside the front of those before it
            way = WAY_WAVE_BY_WAVE;
            m = 0;
            for (uint32_t turn = 0;; ++turn) {
                __syncthreads();
                if (threadIdx.x == 0) filled = m;
                __syncthreads();
                if (wave == turn) mine();
                __syncthreads();
                const uint32_t n = filled;
                if (n > room) { m = TOO_MANY; break; }
                m = front_of<PRUNED_THREADS, POOL>(points, low, keep, n, N);
                close_up<PRUNED_THREADS, POOL>(points, keep, N);
                if (turn == PRUNED_WAVES - 1) break;
            }
        }
    } else {
        __syncthreads();
        {
            const double cap[1] = {mc.cap_words};
            double l[1];
            least_traffic<1>(tab, wave, cap, l);
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
        drop_covered(a, P, S, steps, wave_least);
        // index so far: the class, then where the lanes are
        wave_front(P, S, id, points, &filled, room, [&](uint32_t place, double p, double s, uint32_t code, unsigned long long who) {
            points[place].p = p; points[place].s = s; points[place].idx = ((uint64_t)code << 32) | place;
            lanes[place] = who;
        });
        __syncthreads();
        static_assert(BS_DA || POOL <= (uint32_t)PRUNED_THREADS, "a point per thread");
        m = filled <= room ? front_by_pairs<PRUNED_THREADS>(points, keep, &n_left, filled) : TOO_MANY;
    }
    // the block's front, in any order, behind those of the blocks that ended before
    if (threadIdx.x == 0) {
        if (m <= FRONT_BLOCK) list_at = __hip_atomic_fetch_add(a.counts, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else way |= WAY_OUTGROWN;
        if (way) (void)__hip_atomic_fetch_or(a.counts + 1, way, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (m > FRONT_BLOCK) return;
    __syncthreads();
    Key *out = a.points + list_at;
    if constexpr (BS_DA) {
        for (uint32_t i = threadIdx.x; i < m; i += PRUNED_THREADS) {
            Key k = points[i];
            k.idx = (uint64_t)t0 + (uint32_t)k.idx + (uint64_t)mc.T * index_row_base(kept_dev.number[k.idx >> 32]);
            out[i] = k;
        }
    } else {
        for (uint32_t i = wave; i < m; i += PRUNED_WAVES) {
            Key k = points[i];
            const uint32_t slot = __builtin_amdgcn_readfirstlane((uint32_t)k.idx);
            ClassBest b;
            b.p = uniform_f64(k.p); b.s = uniform_f64(k.s);
            b.code = __builtin_amdgcn_readfirstlane((uint32_t)(k.idx >> 32));
            b.lanes = uniform_u64(lanes[slot]);
            uint32_t cls, combo, row_lo, n_rows;
            class_of_code(b.code, cls, combo);
            rows_of_class(cls, row_lo, n_rows);
            const ComboTerms ct = combo_terms(v, a.extent, mc, cls == 2u, combo % 3, combo / 3);
            const Found f = first_row(tab, ct, mc, nt, (uint32_t)MMEE_OBJ_LATENCY_THEN_ENERGY, b, row_lo, n_rows);
            const uint32_t row = index_row_base(as_constant(kept_dev.number)[row_lo + min(f.row, n_rows - 1)]) + 30000u * (combo % 3) + 90000u * (combo / 3);
            k.idx = (uint64_t)t0 + f.lane + (uint64_t)mc.T * row;
            if (lane == 0) out[i] = k;
        }
    }
}

constexpr int MERGE_THREADS = 1024;

// Of points[0 .. n) what a step's corner -- its least s, there the least p, there the least index -- covers goes, the rest
// to the front of the array, in any order; their number.  least: the s.  Steps are narrow: hardly anything but the
// front and what many candidates share is left (600 x 64: 27854 points of all blocks, 2292 behind no other step's, 115 after this).
__device__ __forceinline__ uint32_t drop_behind_corners(const FrontArgs &a, Key *points, uint32_t n, const double *least,
                                                        unsigned long long *corner_p, unsigned long long *corner_idx, uint32_t *filled)
{
    if (threadIdx.x < FRONT_STEPS) { corner_p[threadIdx.x] = INF_BITS; corner_idx[threadIdx.x] = ~0ull; }
    if (threadIdx.x == 0) *filled = 0;
    __syncthreads();
    constexpr uint32_t PER = FRONT_POINTS / MERGE_THREADS;
    Key k[PER];
    uint32_t step[PER];
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t i = q * MERGE_THREADS + threadIdx.x;
        k[q] = no_point();
        if (i < n) k[q] = points[i];
        step[q] = step_of(a, k[q].p);
        if (i < n && k[q].s == least[step[q]])
            (void)__hip_atomic_fetch_min(corner_p + step[q], (unsigned long long)__double_as_longlong(k[q].p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q)
        if (q * MERGE_THREADS + threadIdx.x < n && k[q].s == least[step[q]] && (unsigned long long)__double_as_longlong(k[q].p) == corner_p[step[q]])
            (void)__hip_atomic_fetch_min(corner_idx + step[q], (unsigned long long)k[q].idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        if (q * MERGE_THREADS + threadIdx.x >= n) continue;
        Key c;
        c.p = __longlong_as_double((long long)corner_p[step[q]]); c.s = least[step[q]]; c.idx = corner_idx[step[q]];
        if (!(c.s <= k[q].s && key_less(c, k[q])))
            points[__hip_atomic_fetch_add(filled, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)] = k[q];
    }
    __syncthreads();
    const uint32_t left = *filled;
    __syncthreads();
    return left;
}

// The blocks' points into the front's records.  Counters and staircase are left as the next call needs them.
__global__ __launch_bounds__(MERGE_THREADS) void k_front_merge(FrontArgs a)
{
    __shared__ Key points[FRONT_POINTS];
    __shared__ double low[FRONT_POINTS];
    __shared__ uint32_t keep[FRONT_POINTS];
    __shared__ DivTable dv_s;
    __shared__ double wave_least[FRONT_STEPS / 64];
    __shared__ uint32_t filled, n_left;
    // the staircase, until the first sort: the least below each step, in each step, and each step's corner
    static_assert(4 * FRONT_STEPS <= FRONT_POINTS, "they fit");
    double *below = low, *least = low + FRONT_STEPS;
    unsigned long long *corner_p = reinterpret_cast<unsigned long long *>(low + 2 * FRONT_STEPS), *corner_idx = corner_p + FRONT_STEPS;
    const uint32_t lane = threadIdx.x & 63;
    if (threadIdx.x >= MERGE_THREADS - 64) ask_for_arguments<FrontArgs>(lane);
    const uint32_t n_list = a.counts[0];
    uint32_t way = a.counts[1];
    bool fits = !(way & WAY_OUTGROWN);
    double own = pos_inf();
    if (threadIdx.x < FRONT_STEPS) own = __longlong_as_double((long long)a.stairs[threadIdx.x]);
    {
        uint32_t at = 0;
        for (int q = 0; q < 4; ++q) {
            for (uint32_t k = threadIdx.x; k < a.ndiv[q]; k += MERGE_THREADS) dv_s.div[q][k] = a.list[at + k];
            at += a.ndiv[q];
        }
        if (threadIdx.x < 4) { dv_s.X[threadIdx.x] = a.X[threadIdx.x]; dv_s.ndiv[threadIdx.x] = a.ndiv[threadIdx.x]; }
    }
    if (threadIdx.x == 0) filled = 0;
    if (threadIdx.x < FRONT_STEPS) least[threadIdx.x] = own;
    steps_below(own, below, wave_least);                     // (its barriers: everybody has read counters and staircase)
    if (threadIdx.x < FRONT_STEPS) a.stairs[threadIdx.x] = INF_BITS;
    if (threadIdx.x < 2) a.counts[threadIdx.x] = 0;

    uint32_t n = 0;                                          // points in LDS
    bool sorted = false;
    for (uint32_t at = 0; fits && at < n_list;) {
        if (at) way |= WAY_TURNS;
        const uint32_t upto = min(n_list, at + (FRONT_POINTS - n));
        constexpr uint32_t AHEAD = 4;                        // points a thread has under way
        for (uint32_t i0 = at; i0 < upto; i0 += AHEAD * MERGE_THREADS) {
            Key k[AHEAD];
#pragma unroll
            for (uint32_t q = 0; q < AHEAD; ++q) {
                const uint32_t i = i0 + q * MERGE_THREADS + threadIdx.x;
                k[q] = a.points[min(i, upto - 1)];
                if (i >= upto) k[q].p = pos_inf();
            }
#pragma unroll
            for (uint32_t q = 0; q < AHEAD; ++q) {
                // (once the room of the staircase has served a sort, the sort drops what it would have dropped)
                const bool stays = k[q].p < pos_inf() && (sorted || k[q].s < below[step_of(a, k[q].p)]);
                const unsigned long long who = __ballot(stays);
                if (!who) continue;
                uint32_t place = 0;
                if (lane == 0) place = __hip_atomic_fetch_add(&filled, (uint32_t)__popcll(who), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                place = __builtin_amdgcn_readfirstlane(place) + (uint32_t)__popcll(who & ((1ull << lane) - 1));
                if (stays) points[place] = k[q];
            }
        }
        at = upto;
        __syncthreads();
        n = filled;
        __syncthreads();                                     // (everybody has read it)
        if (at < n_list && n <= FRONT_POINTS / 2) continue;
        if (!sorted) n = drop_behind_corners(a, points, n, least, corner_p, corner_idx, &filled);
        if (n > (at < n_list ? FRONT_POINTS / 2 : (uint32_t)MERGE_THREADS)) {
            way |= at < n_list ? WAY_SORTED_EARLY : WAY_SORTED;
            uint32_t N;
            const uint32_t m = front_of<MERGE_THREADS, FRONT_POINTS>(points, low, keep, n, N);
            close_up<MERGE_THREADS, FRONT_POINTS>(points, keep, N);
            sorted = true;
            n = m;
            if (threadIdx.x == 0) filled = n;
            __syncthreads();
        }
        fits = at == n_list || n < FRONT_POINTS;
    }
    if (!fits) {
        if (threadIdx.x == 0) {
            a.n_out[0] = TOO_MANY;
            a.n_out[1] = way;
            say_done(a.done, a.number, *a.begin);
        }
        return;
    }
    if (n <= MERGE_THREADS) n = front_by_pairs<MERGE_THREADS>(points, keep, &n_left, n);
    for (uint32_t i = threadIdx.x; i < n; i += MERGE_THREADS) {
        const Key me = points[i];
        uint32_t place = 0;                                  // along the front p goes up
        if (n <= MERGE_THREADS)
            for (uint32_t j = 0; j < n; ++j) place += points[j].p < me.p;
        else place = i;
        if (place >= a.capacity) continue;
        mmee_result res;
        winner_record(a.enc, dv_s, a.mc, me, res);
        write_record(a.out + place, me, res);
    }
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) {
        a.n_out[0] = n;
        a.n_out[1] = way;
        say_done(a.done, a.number, *a.begin);
    }
}

}  // namespace mmee
