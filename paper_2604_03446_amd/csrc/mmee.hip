// libmmee: host side of the C ABI declared in include/mmee.h.
// Argument checking, integer factorisation of the loop extents (the online
// tiling enumeration of Sec. VI-A), launch plumbing and result unpacking.
// Every number the calls return is produced by the kernels in kernels.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <vector>

#include "kernels.h"
#include "batch.h"
#include "pruned.h"
#include "fronts.h"
#include "dense.h"
#include "pinned.h"

// ---- fixed scratch of the entry point that allocates nothing (mmee_search_noalloc) ------------
// One array per GPU, held from the moment the library is loaded until the process ends.  In host
// code the array's name is only a stand-in: its device address comes from hipGetSymbolAddress,
// once per device, and that pointer is what kernels, fills and copies are given.
namespace mmee {
namespace noalloc {
constexpr size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }
constexpr uint32_t MAX_TPAD = 16384;        // tilings a problem may have (rounded up to 64)
constexpr uint32_t MAX_BLOCKS = 1024;       // persistent blocks the partial records have room for
constexpr size_t OFF_ENC = 0;
constexpr size_t OFF_SIG = OFF_ENC + up256(sizeof(uint4) * N_DFROWS);
constexpr size_t OFF_FLAGS = OFF_SIG + up256(sizeof(uint32_t) * N_DFROWS);
constexpr size_t OFF_ROWS0 = OFF_FLAGS + up256(N_DFROWS);
constexpr size_t OFF_ROWS1 = OFF_ROWS0 + up256(sizeof(uint32_t) * N_DFROWS);
constexpr size_t OFF_RENC0 = OFF_ROWS1 + up256(sizeof(uint32_t) * N_DFROWS);
constexpr size_t OFF_RENC1 = OFF_RENC0 + up256(sizeof(uint4) * N_DFROWS);
constexpr size_t OFF_COUNTS = OFF_RENC1 + up256(sizeof(uint4) * N_DFROWS);
constexpr size_t OFF_TICKET = OFF_COUNTS + up256(sizeof(uint32_t) * 8);
// Behind the two words of the exhaustive search the tickets of k_search_batch, 0 from the load on but while a launch uses one.  A ticket
// serves launches of one number of blocks, which it counts modulo that number: calls that overlap, though they may not (two replays of a
// captured one, say), spoil each other but leave it at 0 once all have ended, and no later call goes on from a count of theirs.  Of the
// tickets for its number of blocks a call takes the next one.
constexpr uint32_t TICKETS = 16;
constexpr size_t OFF_KEYS = OFF_TICKET + up256(sizeof(uint32_t) * (2 + TICKETS * MAX_BLOCKS));
constexpr size_t OFF_PARTIALS = OFF_KEYS + up256(sizeof(Key) * N_OBJ);
constexpr size_t OFF_FINAL = OFF_PARTIALS + up256(sizeof(Key) * N_OBJ * MAX_BLOCKS);
constexpr size_t OFF_DV = OFF_FINAL + up256(sizeof(FinalRecord) * N_OBJ);
constexpr size_t OFF_BTAB = OFF_DV + up256(sizeof(DivTable));
constexpr size_t OFF_CTAB_S = OFF_BTAB + up256(sizeof(double) * NENT_ALL * MAX_TPAD);
constexpr size_t OFF_CTAB_E = OFF_CTAB_S + up256(sizeof(double) * 2 * NCS * MAX_TPAD);
constexpr size_t BYTES = OFF_CTAB_E + up256(sizeof(uint64_t) * 2 * NCE * MAX_TPAD);
static_assert(BYTES <= (40u << 20), "the fixed scratch is documented as at most 40 MiB");
}  // namespace noalloc
}  // namespace mmee

static __device__ __align__(256) unsigned char scratch[mmee::noalloc::BYTES];

namespace mmee {
namespace {

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t err_ = (expr);                                                            \
        if (err_ != hipSuccess) {                                                            \
            std::snprintf(g_last_error, sizeof(g_last_error), "%s: %s (%s:%d)", #expr,       \
                          hipGetErrorString(err_), __FILE__, __LINE__);                      \
            return MMEE_EDEVICE;                                                             \
        }                                                                                    \
    } while (0)

char g_last_error[512] = "";
std::mutex g_lock;
uint64_t g_front_walks = 0;         // fronts walked point by point so far
uint32_t g_front_way = 0;           // which way the last front in two launches took (fronts.h)

struct State {
    bool ready = false;
    hipStream_t stream = nullptr;
    // offline stage
    uint4 *enc = nullptr;
    uint32_t *sig = nullptr;
    uint8_t *flags = nullptr;
    uint32_t *rows[2] = {nullptr, nullptr};     // [0] every row that denotes a dataflow, [1] survivors
    uint4 *row_enc[2] = {nullptr, nullptr};     // the encoded rows in list order
    uint32_t *counts_dev = nullptr;
    uint32_t counts[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    Key *key_dev = nullptr;                     // [N_OBJ] winning keys of a pass, for the pass that follows it
    uint32_t *cls_dev = nullptr;                // (order, r, f) classes whose rows denote dataflows
    uint32_t n_cls = 0;
    // online scratch, grown on demand
    double *btab = nullptr, *ctab_s = nullptr;
    uint64_t *ctab_e = nullptr;
    size_t tiling_cap = 0;
    Key *partials = nullptr;
    size_t partials_cap = 0;
    uint32_t *ticket = nullptr;
    unsigned long long *hints = nullptr;
    // result records: pinned host memory that the search's last block writes directly
    FinalRecord *final_host = nullptr, *final_map = nullptr;     // host address / device address
    DivTable *dv_dev = nullptr;
    size_t slots = 0;
    std::vector<hipEvent_t> events;
    void *eval_dev = nullptr;
    size_t eval_cap = 0;
    // short index lists of mmee_decode and their mappings: pinned host memory the kernel reads and writes directly
    Pinned decode;
    uint32_t resident_blocks = 512;
    uint32_t front_pool = FRONT_POOL_BS_DA;
    // batched search over the pruned rows: problem descriptors (pinned staging + device copy), one record
    // per work item and objective
    unsigned char *batch_host = nullptr, *batch_dev = nullptr;
    size_t batch_blob_cap = 0;
    Key *item_keys = nullptr;
    size_t item_cap = 0;
    // pruned search of many problems on one shape: problem descriptions (pinned staging + device copy), the lowest
    // published values per result slot
    unsigned char *desc_host = nullptr, *desc_dev = nullptr;
    size_t desc_cap = 0;
    // fronts over the kept rows: the blocks' points, the staircase and the counters; FRONT_POINTS records of the front and their
    // number (pinned)
    Key *front_points = nullptr;
    unsigned long long *front_stairs = nullptr;
    uint32_t *front_counts = nullptr;
    bool front_clean = false;                   // staircase and counters are as a call must find them: a merge that was seen to end left them
    Pinned front;
    void *block_records = nullptr;              // what the blocks of a pruned search leave for the reduction
    size_t block_records_cap = 0;
    unsigned long long *pruned_hints = nullptr;
    // what a short call waits for instead of the stream (Done): one per key in pinned memory, the number of the last such call,
    // the device's clock when its kernels began, and that clock's rate
    Pinned done;
    uint64_t call_number = 0, *call_begin = nullptr;
    double clock_hz = 1e8;
} S;

// The device buffers one search pass works in.  The allocating entry points fill this from the
// cached State; the entry point that allocates nothing fills it from the static scratch array.
struct Bufs {
    const uint4 *enc = nullptr;
    const uint32_t *rows[2] = {nullptr, nullptr};
    const uint4 *row_enc[2] = {nullptr, nullptr};
    uint32_t counts[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    const uint32_t *cls_dev = nullptr;          // null: no class list, the dense kernel is not used
    uint32_t n_cls = 0;
    double *btab = nullptr, *ctab_s = nullptr;
    uint64_t *ctab_e = nullptr;
    Key *partials = nullptr;
    size_t partials_cap = 0;                    // blocks the partial records have room for
    uint32_t *ticket = nullptr;                 // [0] finish ticket, [1] work counter
    unsigned long long *hints = nullptr;        // [N_OBJ] launch-wide lowest values of the dense kernel, there where cls_dev is
    Key *key_dev = nullptr;
    FinalRecord *final_dev = nullptr;           // device address of this pass's N_OBJ records
    DivTable *dv_dev = nullptr;                 // this pass's copy of the divisor lists
    hipEvent_t ev_begin = nullptr, ev_end = nullptr;   // null: the pass is not timed
    bool *signalled = nullptr;                  // not null: the pass is the call's only one and may be waited for with wait_signalled; set if so
    uint32_t resident_blocks = 512;
};

// ---- argument checking and the per-call plan ---------------------------------

struct Plan {
    DivTable dv;
    ModelConst mc;
    uint64_t T;
    uint64_t space;
    bool exact_k;
    bool can_regroup;   // every term of the energy is an exact integer below 2^53
    bool whole_energies; // the four energies per access are whole numbers (their size aside)
};

bool finite_nonneg(double v) { return std::isfinite(v) && v >= 0.0; }

int list_divisors_uncached(uint32_t X, uint32_t mode, uint32_t *out);

// the last few factorisations are kept: a sweep asks for the same extents over and over
int list_divisors(uint32_t X, uint32_t mode, uint32_t *out)
{
    struct Entry { uint32_t X = 0, mode = 0; int n = 0; std::vector<uint32_t> div; };
    static thread_local Entry cache[8];
    static thread_local unsigned next = 0;
    for (const Entry &e : cache)
        if (e.X == X && e.mode == mode && e.n > 0) {
            std::memcpy(out, e.div.data(), sizeof(uint32_t) * std::min(e.n, (int)MAXDIV));
            return e.n;
        }
    Entry &e = cache[next++ % 8];
    e.div.assign(MAXDIV, 0);
    e.n = list_divisors_uncached(X, mode, e.div.data());
    e.X = X; e.mode = mode;
    std::memcpy(out, e.div.data(), sizeof(uint32_t) * std::min(std::max(e.n, 0), (int)MAXDIV));
    return e.n;
}

int list_divisors_uncached(uint32_t X, uint32_t mode, uint32_t *out)
{
    // trial division up to sqrt(X); ascending order
    std::vector<uint32_t> lo, hi;
    for (uint64_t a = 1; a * a <= X; ++a) {
        if (X % a) continue;
        lo.push_back((uint32_t)a);
        if (a * a != X) hi.push_back((uint32_t)(X / a));
    }
    int n = 0;
    auto keep = [&](uint32_t v) {
        if (mode == 0 && (v & (v - 1))) return;
        if (n < MAXDIV) out[n] = v;
        ++n;
    };
    for (uint32_t v : lo) keep(v);
    for (auto it = hi.rbegin(); it != hi.rend(); ++it) keep(*it);
    return n;
}

// attention as a chain (Sec. III-A): A = Q, B = K^T, D = V, E = O, one instance per head
int chain_of(const mmee_workload *w, mmee_chain &c)
{
    if (!w) return MMEE_EINVAL;
    if (w->reserved || (uint64_t)w->B * w->H > 0xffffffffull) return MMEE_EINVAL;
    c.batch = w->B * w->H;
    c.I = w->N; c.K = w->d; c.L = w->N; c.J = w->d;
    c.word_bytes = w->word_bytes; c.tiling_mode = w->tiling_mode; c.c_softmax = w->c_softmax;
    return MMEE_OK;
}

int make_plan(const mmee_chain *w, const mmee_hw *hw, Plan &p)
{
    if (!w || !hw) return MMEE_EINVAL;
    if (!w->batch || !w->I || !w->K || !w->L || !w->J || !w->word_bytes || w->tiling_mode > 1) return MMEE_EINVAL;
    if (!hw->pe_rows || !hw->pe_cols || !hw->n_arrays) return MMEE_EINVAL;
    if ((uint64_t)hw->rf_bytes < 3ull * w->word_bytes) return MMEE_EINVAL;
    if (!finite_nonneg(hw->e_dram) || !finite_nonneg(hw->e_gb) || !finite_nonneg(hw->e_rf) ||
        !finite_nonneg(hw->e_mac) || !finite_nonneg(hw->dram_bw) || !finite_nonneg(hw->gb_bw))
        return MMEE_EINVAL;
    std::memset(&p, 0, sizeof(p));
    p.dv.X[DI] = w->I; p.dv.X[DK] = w->K; p.dv.X[DL] = w->L; p.dv.X[DJ] = w->J;
    p.T = 1;
    for (int q = 0; q < 4; ++q) {
        int n = list_divisors(p.dv.X[q], w->tiling_mode, p.dv.div[q]);
        if (n <= 0 || n > MAXDIV) return MMEE_EINVAL;
        p.dv.ndiv[q] = (uint32_t)n;
        p.T *= (uint64_t)n;
    }
    if (p.T > (1ull << 22)) return MMEE_EINVAL;
    p.space = p.T * ROWS_PER_TILING;
    // every count of the model must stay an exact integer in fp64
    long double bound = (long double)w->batch * (long double)w->I * w->K * (long double)w->L * w->J *
                        (16.0L + (long double)w->c_softmax) * (long double)w->word_bytes;
    if (bound >= 9007199254740992.0L) return MMEE_EINVAL;
    ModelConst &mc = p.mc;
    mc.BH = (double)w->batch;
    mc.c_lat = mc.BH / (double)hw->n_arrays;
    uint64_t cap = hw->gb_bytes / w->word_bytes;
    mc.cap_words = cap >= (1ull << 53) ? 9007199254740992.0 : (double)cap;
    mc.word = (double)w->word_bytes;
    mc.e_dram = hw->e_dram; mc.e_gb = hw->e_gb; mc.e_rf = hw->e_rf; mc.e_mac = hw->e_mac;
    mc.e_sum = hw->e_dram + hw->e_gb;
    {
        // Per instance, with P = I*K*L*J: DRAM words <= 8 P (four operands at most P each, the
        // unfused intermediate at most I*L*(K+J+2) <= 4 P), buffer<->RF words <= 6 P (three terms
        // per tile matmul, each at most its MAC count; MACs <= 2 P with recomputation), RF accesses
        // 3 * MACs <= 6 P, softmax elements <= P.  The total energy bounds every partial sum.
        auto whole = [](double v) { return v == std::floor(v); };
        const long double P = (long double)w->batch * (long double)w->I * w->K * (long double)w->L * w->J;
        const long double worst = P * (8.0L * hw->e_dram + 14.0L * hw->e_gb + 6.0L * hw->e_rf +
                                       (2.0L + (long double)w->c_softmax) * hw->e_mac);
        p.whole_energies = whole(hw->e_dram) && whole(hw->e_gb) && whole(hw->e_rf) && whole(hw->e_mac);
        p.can_regroup = p.whole_energies && worst < 9007199254740992.0L;
        // buffer words of a candidate: DRAM words + buffer<->RF words <= 14 P
        mc.gb_product_exact = whole(hw->e_gb) && 14.0L * P * hw->e_gb < 9007199254740992.0L ? 1u : 0u;
    }
    mc.dram_bw = hw->dram_bw; mc.gb_bw = hw->gb_bw;
    // with a power-of-two bandwidth and array count, (B*H/n) * (words*word/bw) is the B*H-scaled
    // table value times one exactly representable constant
    int ex = 0;
    const bool bw_pow2 = hw->dram_bw == 0.0 || std::frexp(hw->dram_bw, &ex) == 0.5;
    const bool n_pow2 = (hw->n_arrays & (hw->n_arrays - 1)) == 0;
    p.exact_k = bw_pow2 && n_pow2;
    mc.dram_k = hw->dram_bw > 0.0 ? mc.word / hw->dram_bw / (double)hw->n_arrays : 0.0;
    mc.eval_k = hw->dram_bw > 0.0 ? mc.word / hw->dram_bw : 0.0;
    mc.bw_pow2 = bw_pow2 ? 1u : 0u;
    mc.dram_b = mc.dram_y = 1.0;
    if (hw->dram_bw > 0.0) {
        mc.dram_b = 2.0 * std::frexp(hw->dram_bw, &ex);
        mc.dram_y = 1.0 / mc.dram_b;
        mc.dram_c = std::ldexp(mc.c_lat, 1 - ex);
    }
    mc.pe_rows = hw->pe_rows; mc.pe_cols = hw->pe_cols;
    mc.g_words = hw->rf_bytes / w->word_bytes / 2;
    mc.gb_pow2 = hw->gb_bw > 0.0 && std::frexp(hw->gb_bw, &ex) == 0.5 ? 1u : 0u;
    mc.gb_k = mc.gb_pow2 ? mc.word / hw->gb_bw : 0.0;
    mc.gb_b = mc.gb_y = 1.0;
    if (hw->gb_bw > 0.0) {
        mc.gb_b = 2.0 * std::frexp(hw->gb_bw, &ex);
        mc.gb_y = 1.0 / mc.gb_b;
        mc.gb_scale = std::ldexp(1.0, 1 - ex);
    }
    mc.rcp_rows = 1.0 / (double)mc.pe_rows;
    mc.rcp_cols = 1.0 / (double)mc.pe_cols;
    mc.rcp_cols_g = 1.0 / ((double)mc.pe_cols * (double)mc.g_words);
    mc.c_softmax = w->c_softmax;
    mc.T = (uint32_t)p.T;
    mc.tpad = (uint32_t)((p.T + 63) & ~63ull);
    return MMEE_OK;
}

// ---- device state ------------------------------------------------------------

// What the device's offline stage found, back to the host: on the library's stream, with one synchronisation.  The pruned
// searches have the kept rows compiled in (rows.h); they must be the ones found.
int read_offline(const uint32_t *counts_dev, const uint32_t *kept, uint32_t (&counts)[2][4])
{
    const uint32_t group_of[LEAST_CLASSES] = {0, 2, 3};      // class (r, f) -> g = r + 2 f
    uint32_t h[8], rows[KEPT_ALL];
    HIP_TRY(hipMemcpyAsync(h, counts_dev, sizeof(h), hipMemcpyDeviceToHost, S.stream));
    for (int c = 0; c < LEAST_CLASSES; ++c)
        HIP_TRY(hipMemcpyAsync(rows + KEPT.first[c], kept + (size_t)group_of[c] * ROWS_PER_GROUP, sizeof(uint32_t) * KEPT.rows[c],
                               hipMemcpyDeviceToHost, S.stream));
    HIP_TRY(hipStreamSynchronize(S.stream));
    for (int g = 0; g < 4; ++g) { counts[0][g] = h[g]; counts[1][g] = h[4 + g]; }
    bool same = counts[1][1] == 0;
    for (int c = 0; c < LEAST_CLASSES; ++c)
        same = same && counts[1][group_of[c]] == KEPT.rows[c] && std::memcmp(rows + KEPT.first[c], KEPT.number + KEPT.first[c], sizeof(uint32_t) * KEPT.rows[c]) == 0;
    if (same) return MMEE_OK;
    std::snprintf(g_last_error, sizeof(g_last_error), "the offline stage's rows are not the compiled ones");
    return MMEE_EDEVICE;
}

int ensure_ready()
{
    if (S.ready) return MMEE_OK;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) {
        std::snprintf(g_last_error, sizeof(g_last_error), "no HIP device");
        return MMEE_EDEVICE;
    }
    {
        int dev = 0, cus = 0;
        HIP_TRY(hipGetDevice(&dev));
        HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        S.resident_blocks = (uint32_t)std::max(cus, 1) * BLOCKS_PER_CU;
        int khz = 0;
        HIP_TRY(hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev));
        if (khz > 0) S.clock_hz = 1e3 * khz;
        // MMEE_RESIDENT_BLOCKS (read once, an even number from 2 up to what the chip holds): fewer persistent
        // blocks, i.e. another split of the work over blocks and another order of the reduction.  Results do
        // not depend on it; it exists so that a test can show that.
        if (const char *env = std::getenv("MMEE_RESIDENT_BLOCKS")) {
            const long v = std::atol(env);
            if (v >= 2 && v % 2 == 0 && (uint64_t)v <= S.resident_blocks) S.resident_blocks = (uint32_t)v;
        }
        // MMEE_FRONT_POOL (read once, up to what the kernel holds): less room for the points of a front's blocks, i.e. other
        // ways to the same front; for tests of the ways that hardly any problem takes.
        if (const char *env = std::getenv("MMEE_FRONT_POOL")) {
            const long v = std::atol(env);
            if (v >= 1 && v <= (long)FRONT_POOL_BS_DA) S.front_pool = (uint32_t)v;
        }
    }
    HIP_TRY(hipMalloc(&S.enc, sizeof(uint4) * N_DFROWS));
    HIP_TRY(hipMalloc(&S.sig, sizeof(uint32_t) * N_DFROWS));
    HIP_TRY(hipMalloc(&S.flags, N_DFROWS));
    HIP_TRY(hipMalloc(&S.rows[0], sizeof(uint32_t) * N_DFROWS));
    HIP_TRY(hipMalloc(&S.rows[1], sizeof(uint32_t) * N_DFROWS));
    HIP_TRY(hipMalloc(&S.counts_dev, sizeof(uint32_t) * 8));
    HIP_TRY(hipMalloc(&S.key_dev, sizeof(Key) * N_OBJ));
    HIP_TRY(hipMalloc(&S.ticket, 3 * sizeof(uint32_t)));        // [0] finish ticket, [1] work counter, [2] k_search_batch's ticket
    HIP_TRY(hipMalloc(&S.hints, N_OBJ * sizeof(unsigned long long)));
    {
        // +inf until a launch lowers them; the last block of every launch puts +inf back
        static const unsigned long long inf_bits[N_OBJ] = {INF_BITS, INF_BITS, INF_BITS, INF_BITS};
        HIP_TRY(hipMemcpyAsync(S.hints, inf_bits, sizeof(inf_bits), hipMemcpyHostToDevice, S.stream));
    }
    // on the library's stream, like the kernels that follow: a caller's non-blocking stream is not
    // ordered against the null stream
    HIP_TRY(hipMemsetAsync(S.ticket, 0, 3 * sizeof(uint32_t), S.stream));
    HIP_TRY(hipMemsetAsync(S.rows[0], 0, sizeof(uint32_t) * N_DFROWS, S.stream));
    HIP_TRY(hipMemsetAsync(S.rows[1], 0, sizeof(uint32_t) * N_DFROWS, S.stream));
    for (int w = 0; w < 2; ++w) {
        HIP_TRY(hipMalloc(&S.row_enc[w], sizeof(uint4) * N_DFROWS));
        HIP_TRY(hipMemsetAsync(S.row_enc[w], 0, sizeof(uint4) * N_DFROWS, S.stream));
    }
    // offline stage: encode every (order, levels, r, f) row, prune, compact
    hipLaunchKernelGGL(k_build_rows, dim3((N_DFROWS + 255) / 256), dim3(256), 0, S.stream, S.enc, S.sig);
    hipLaunchKernelGGL(k_prune_rows, dim3((ROWS_PER_GROUP + 255) / 256, N_GROUPS), dim3(256), 0, S.stream, S.sig,
                       S.flags);
    hipLaunchKernelGGL(k_compact_rows, dim3(8), dim3(1024), 0, S.stream, S.flags, S.enc, S.rows[0], S.rows[1],
                       S.row_enc[0], S.row_enc[1],
                       S.counts_dev);
    HIP_TRY(hipGetLastError());
    {
        const int rc = read_offline(S.counts_dev, S.rows[1], S.counts);
        if (rc) return rc;
    }
    {
        // whether a row denotes a dataflow depends on (order, r, f) only: list those classes
        std::vector<uint8_t> flags(N_DFROWS);
        HIP_TRY(hipMemcpy(flags.data(), S.flags, N_DFROWS, hipMemcpyDeviceToHost));
        std::vector<uint32_t> cls;
        for (uint32_t g = 0; g < N_GROUPS; ++g)
            for (uint32_t rank = 0; rank < 24; ++rank) {
                uint32_t on = 0;
                for (uint32_t q = 0; q < 625; ++q) on += flags[g * ROWS_PER_GROUP + rank * 625 + q] & 1u;
                if (on != 0 && on != 625) {
                    std::snprintf(g_last_error, sizeof(g_last_error), "row validity is not uniform within a class");
                    return MMEE_EDEVICE;
                }
                if (on) cls.push_back(rank + 24 * g);
            }
        uint64_t rows = 0;
        for (int g = 0; g < 4; ++g) rows += S.counts[0][g];
        if (cls.empty() || cls.size() * 625ull != rows) {
            std::snprintf(g_last_error, sizeof(g_last_error), "class list does not match the row list");
            return MMEE_EDEVICE;
        }
        HIP_TRY(hipMalloc(&S.cls_dev, sizeof(uint32_t) * 96));
        HIP_TRY(hipMemcpy(S.cls_dev, cls.data(), sizeof(uint32_t) * cls.size(), hipMemcpyHostToDevice));
        S.n_cls = (uint32_t)cls.size();
    }
    S.ready = true;
    return MMEE_OK;
}

struct HipPinned {
    hipError_t success = hipSuccess;
    hipError_t alloc(unsigned char **host, size_t bytes) const
    {
        return hipHostMalloc(reinterpret_cast<void **>(host), bytes, hipHostMallocMapped);
    }
    hipError_t address(unsigned char **map, unsigned char *host) const
    {
        return hipHostGetDevicePointer(reinterpret_cast<void **>(map), host, 0);
    }
    hipError_t release(unsigned char *host) const { return hipHostFree(host); }
};

int ensure_tilings(uint64_t tpad)
{
    if (tpad <= S.tiling_cap) return MMEE_OK;
    if (S.btab) { HIP_TRY(hipStreamSynchronize(S.stream)); (void)hipFree(S.btab); (void)hipFree(S.ctab_s); (void)hipFree(S.ctab_e); }
    S.btab = nullptr; S.ctab_s = nullptr; S.ctab_e = nullptr; S.tiling_cap = 0;
    HIP_TRY(hipMalloc(&S.btab, sizeof(double) * NENT_ALL * tpad));
    HIP_TRY(hipMalloc(&S.ctab_s, sizeof(double) * 2 * NCS * tpad));
    HIP_TRY(hipMalloc(&S.ctab_e, sizeof(uint64_t) * 2 * NCE * tpad));
    S.tiling_cap = tpad;
    return MMEE_OK;
}

int ensure_partials(size_t nblocks)
{
    if (nblocks <= S.partials_cap) return MMEE_OK;
    if (S.partials) { HIP_TRY(hipStreamSynchronize(S.stream)); (void)hipFree(S.partials); }
    S.partials = nullptr; S.partials_cap = 0;
    HIP_TRY(hipMalloc(&S.partials, sizeof(Key) * N_OBJ * nblocks));
    S.partials_cap = nblocks;
    return MMEE_OK;
}

int ensure_slots(size_t n)
{
    if (n <= S.slots) return MMEE_OK;
    if (S.dv_dev) {
        HIP_TRY(hipStreamSynchronize(S.stream));
        (void)hipFree(S.dv_dev); (void)hipFree(S.pruned_hints);
        if (S.final_host) (void)hipHostFree(S.final_host);
    }
    S.slots = 0; S.final_host = nullptr; S.final_map = nullptr; S.dv_dev = nullptr; S.pruned_hints = nullptr;
    HIP_TRY(hipMalloc(&S.dv_dev, sizeof(DivTable) * n));
    // +inf until a launch lowers them; the launch's finish puts +inf back
    HIP_TRY(hipMalloc(&S.pruned_hints, sizeof(unsigned long long) * N_OBJ * n));
    hipLaunchKernelGGL(k_fill_words64, dim3((uint32_t)((N_OBJ * n + 255) / 256)), dim3(256), 0, S.stream, S.pruned_hints, N_OBJ * (uint64_t)n,
                       INF_BITS);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipHostMalloc(&S.final_host, sizeof(FinalRecord) * N_OBJ * n, hipHostMallocMapped));
    HIP_TRY(hipHostGetDevicePointer(reinterpret_cast<void **>(&S.final_map), S.final_host, 0));
    while (S.events.size() < 2 * n) {
        hipEvent_t e;
        HIP_TRY(hipEventCreate(&e));
        S.events.push_back(e);
    }
    S.slots = n;
    return MMEE_OK;
}

// the model constants of one pass: whether the energy is regrouped is settled here, for the tables
// and for the kernel alike
//
// Beyond the size bound the sum may still be regrouped for the scalar keys other than the
// energy-delay product, subject to a check of the outcome (`*unproven` is set): all terms are
// non-negative whole numbers, so a candidate whose true total is below 2^53 is exact in either
// order, and any other candidate computes to more than 2^52 in either order.  An optimum below
// 2^52 pJ therefore is the optimum of the term-by-term sum too, ties included; otherwise the
// caller repeats the pass with MMEE_SEARCH_ORDERED_SUM.
constexpr int MASK_ENERGY = 1 << MMEE_OBJ_ENERGY;
constexpr double REGROUP_PROOF_LIMIT = 4503599627370496.0;   // 2^52
ModelConst pass_constants(const Plan &p, uint32_t flags, int mask = 8, bool *unproven = nullptr, bool any_time = false)
{
    ModelConst mc = p.mc;
    // (any_time: the kernel regroups whatever the DRAM time needs; the others take the DRAM time as one exact
    // product where they regroup, and only the energy alone has no DRAM time: 2048 x 768 x 3072 x 768 chain,
    // 60 B/cycle, exhaustive, a buffer that everything fits: 0.418 ms summed in order, 0.327 ms regrouped)
    const bool allowed = (p.exact_k || any_time || mask == MASK_ENERGY) && !(flags & MMEE_SEARCH_ORDERED_SUM);
    const bool on_trust = allowed && !p.can_regroup && p.whole_energies && !(mask & 8) && unproven;
    mc.regroup = ((allowed && p.can_regroup) || on_trust) ? 1u : 0u;
    if (unproven) *unproven = on_trust;
    return mc;
}

// the tables of one problem into b's table buffers (which must hold mc.tpad tilings)
int launch_tilings(const Plan &p, const ModelConst &mc, const Bufs &b, DivTable *dv_copy = nullptr)
{
    hipLaunchKernelGGL(k_build_tilings, dim3(mc.tpad / 64), dim3(64 * BUILD_PARTS), 0, S.stream, p.dv, mc, b.btab,
                       b.ctab_s, b.ctab_e, dv_copy);
    HIP_TRY(hipGetLastError());
    return MMEE_OK;
}

// the cached, growing buffers of the allocating entry points, for the pass in result slot `slot`; `tables`: the per-tiling ones too (2
// KiB a tiling, which the dense kernel has no use for)
int state_bufs(const Plan &p, size_t slot, bool tables, Bufs &b)
{
    if (slot >= S.slots) return MMEE_EINVAL;
    int rc = tables ? ensure_tilings(p.mc.tpad) : MMEE_OK;
    if (rc) return rc;
    // persistent blocks: never more than the chip holds at once
    rc = ensure_partials(S.resident_blocks);
    if (rc) return rc;
    b.enc = S.enc;
    for (int w = 0; w < 2; ++w) {
        b.rows[w] = S.rows[w]; b.row_enc[w] = S.row_enc[w];
        for (int g = 0; g < 4; ++g) b.counts[w][g] = S.counts[w][g];
    }
    b.cls_dev = S.cls_dev; b.n_cls = S.n_cls;
    b.btab = S.btab; b.ctab_s = S.ctab_s; b.ctab_e = S.ctab_e;
    b.partials = S.partials; b.partials_cap = S.partials_cap;
    b.ticket = S.ticket; b.hints = S.hints; b.key_dev = S.key_dev;
    b.final_dev = S.final_map + N_OBJ * slot;
    b.dv_dev = S.dv_dev + slot;
    b.ev_begin = S.events[2 * slot]; b.ev_end = S.events[2 * slot + 1];
    b.resident_blocks = S.resident_blocks;
    return MMEE_OK;
}

template <int MASK>
void launch_search_mask(bool exact_k, dim3 grid, const SearchArgs &a)
{
    if (a.mc.regroup) hipLaunchKernelGGL((k_search<MASK, true, false, true>), grid, dim3(SEARCH_THREADS), 0, S.stream, a);
    else if (exact_k) hipLaunchKernelGGL((k_search<MASK, true>), grid, dim3(SEARCH_THREADS), 0, S.stream, a);
    else hipLaunchKernelGGL((k_search<MASK, false>), grid, dim3(SEARCH_THREADS), 0, S.stream, a);
}

// one step of the Pareto walk: latency-then-energy among candidates with energy below a.e_limit
void launch_search_limited(bool exact_k, dim3 grid, const SearchArgs &a)
{
    if (a.mc.regroup) hipLaunchKernelGGL((k_search<4, true, true, true>), grid, dim3(SEARCH_THREADS), 0, S.stream, a);
    else if (exact_k) hipLaunchKernelGGL((k_search<4, true, true>), grid, dim3(SEARCH_THREADS), 0, S.stream, a);
    else hipLaunchKernelGGL((k_search<4, false, true>), grid, dim3(SEARCH_THREADS), 0, S.stream, a);
}

// One pass of the dense kernel.  MASK: energy, latency, both or the energy-delay product.  LIMIT: only
// candidates with energy below a.e_limit (first pass of a step of the Pareto walk).  LATCAP: only those with a
// latency within a.lat_cap (second pass of the (latency, energy) key).
template <int MASK, bool LIMIT = false, bool LATCAP = false>
void launch_dense(bool exact_k, dim3 grid, const DenseArgs &a)
{
    // keys that do not look at the energy or at the DRAM time need one variant only
    constexpr bool ENERGY = MASK != (1 << MMEE_OBJ_LATENCY) || LIMIT, TIME = MASK != MASK_ENERGY || LATCAP;
    auto with = [&](auto fast, auto sum) {
        hipLaunchKernelGGL((k_search_dense<MASK, decltype(fast)::value, LIMIT, decltype(sum)::value, LATCAP>), grid, dim3(DENSE_THREADS), 0,
                           S.stream, a);
    };
    auto with_sum = [&](auto sum) {
        if (!TIME || exact_k) with(std::true_type{}, sum);
        else with(std::integral_constant<bool, !TIME>{}, sum);
    };
    if (!ENERGY || a.mc.regroup) with_sum(std::integral_constant<int, SUM_REGROUPED>{});
    else if (a.mc.gb_product_exact) with_sum(std::integral_constant<int, ENERGY ? SUM_FUSED : SUM_REGROUPED>{});
    else with_sum(std::integral_constant<int, ENERGY ? SUM_ORDERED : SUM_REGROUPED>{});
}

void shape_constants(const DivTable &dv, double (&extent)[4], double (&size)[5]);

// The fewest tilings at which the dense kernel takes these keys over the full row set.  One or two scalar keys are one pass and always
// go there; the (latency, energy) key is one more, and so is a third scalar key.  k_search takes all keys in one pass, with the
// lanes on rows: it divides once per candidate where the DRAM time is not one exact product, keeps a code beside every
// minimum, and tries the rows that do not fit as well, which the dense kernel passes over.  So k_search is left where a pass costs more
// than that saves: few tilings, and three scalar keys or four keys with a buffer that holds most of what there is.  us per
// call, k_search / dense, buffer for everything | for a sixteenth of it, 14 shapes of 1 to 11664 tilings:
//   energy and latency      regrouped    T = 1: 38 / 34      500: 1.09 | 1.89 times     4900: 354 / 301 | 4.0 times
//   product and latency     in order     T = 1: 1.02 times   500: 1.01 | 2.38           4900: 1.03 | 4.4
//   two kinds of latency    regrouped    T = 1: 1.00 times   36: 1.27 | 1.61            4900: 2.67 | 7.2
//   energy and both         in order     T = 1: 0.86 times   36: 1.18 | 1.64            4900: 2.07 | 7.8
//   three scalar keys       regrouped    T = 36: 0.91 | 1.21   500: 0.84 | 1.46         4900: 519 / 547 | 3.2 times
//                           bandwidth 60 T = 36: 1.26 | 1.70   500: 1.40 | 2.63         4900: 2.12 | 7.5
//   all four                in order     T = 36: 0.89 | 1.25   225: 0.92 | 1.89         500: 0.98 | 2.18     4900: 1.44 | 5.6
// Buffers of a half to a quarter of everything lie between; the line is drawn where no shape loses.
uint32_t dense_from(const Plan &p, int mask)
{
    constexpr uint32_t NEVER = 0xFFFFFFFFu, HALF_A_CHUNK = PRUNED_TC / 2, FEW = 7 * PRUNED_TC;
    if (popcount4(mask) == 1 || (!(mask & 4) && mask != 11)) return 0;
    double extent[4], size[5];
    shape_constants(p.dv, extent, size);
    const bool roomy = 4.0 * p.mc.cap_words > size[0] + size[1] + size[2] + size[3] + size[4];
    if (!roomy || !p.exact_k) return HALF_A_CHUNK;
    return mask == 11 ? NEVER : (mask == 13 || mask == 15 ? FEW : HALF_A_CHUNK);
}

// whether these keys' pass goes through the dense kernel
bool goes_dense(const Plan &p, int mask, uint32_t flags, bool bs_da_step)
{
    return (flags & MMEE_SEARCH_EXHAUSTIVE) && !bs_da_step && p.T >= dense_from(p, mask);
}

uint32_t list_length(const DivTable &dv);
void pack_lists(const DivTable &dv, uint32_t *list);

int begin_signalled(Done *&done, uint64_t &number, uint64_t *&begin);

// One pass of these keys over the full row set in k_search_dense, or two or three (the launches share the arguments).
int enqueue_dense(const Bufs &B, const Plan &p, const ModelConst &mc, int mask, const double *e_limit)
{
    if (list_length(p.dv) > DENSE_DIVS) return MMEE_EINVAL;
    DenseArgs a;
    std::memset(&a, 0, sizeof(a));
    a.mc = mc;
    // a chunk's tilings: k's divisors fastest, then j's, l's, i's
    const int radix_order[4] = {DK, DJ, DL, DI};
    double radix = 1.0;
    for (int q : radix_order) {
        a.dg.rcp_radix[q] = 1.0 / radix;
        a.dg.rcp_n[q] = 1.0 / (double)p.dv.ndiv[q];
        radix *= (double)p.dv.ndiv[q];
    }
    shape_constants(p.dv, a.extent, a.size);
    for (int q = 0; q < 4; ++q) { a.X[q] = p.dv.X[q]; a.ndiv[q] = p.dv.ndiv[q]; }
    pack_lists(p.dv, a.list);
    a.enc = B.enc; a.cls = B.cls_dev; a.n_cls = B.n_cls;
    const uint32_t n_chunks = (uint32_t)((p.T + PRUNED_TC - 1) / PRUNED_TC), blocks = B.resident_blocks / BLOCKS_PER_CU * DENSE_BLOCKS_PER_CU;
    // Items: three quarters of the chunks in items of a quarter of a block's share of the tasks, a fifth in items a third as large, the
    // rest in the smallest.  Every item costs a block some 2 us (its tables, and waves that wait for its last task), every task
    // too many at the end all blocks up to 19 us.  us a call, so / all items a quarter of a block's share / an eighth / a twentieth: 12544
    // tilings (8192 x 128), energy 251 / 273 / 272 / 305; 4900 tilings (512 x 64), energy and latency 259 / 275 / 277 / 302.
    const double per_block = (double)n_chunks * B.n_cls * 5.0 / blocks, share[3] = {0.75, 0.2, 1.0}, part[3] = {0.25, 0.08, 0.03};
    uint64_t n_items = 0;
    uint32_t chunk = 0;
    for (int k = 0; k < 3; ++k) {
        const double tasks = std::max(part[k] * per_block, 1.6);
        DenseArgs::Phase &ph = a.phase[k];
        ph.item = (uint32_t)n_items; ph.chunk = chunk;
        ph.groups = std::max(1u, (uint32_t)(B.n_cls * 5.0 / tasks));
        const uint32_t n = std::min(n_chunks - chunk, (uint32_t)(share[k] * n_chunks));
        chunk += n;
        n_items += (uint64_t)n * ph.groups;
    }
    if (n_items > 0x7fffffffull) return MMEE_EINVAL;
    a.n_items = (uint32_t)n_items;
    // persistent blocks: as many as the chip holds at once
    const dim3 grid((uint32_t)std::min<uint64_t>(n_items, blocks));
    if (grid.x > B.partials_cap) return MMEE_EINVAL;
    a.partials = B.partials; a.ticket = B.ticket; a.work_counter = B.ticket + 1; a.hints = B.hints;
    a.final_out = B.final_dev;
    if (B.signalled) {
        const int rc = begin_signalled(a.done, a.number, a.begin);
        if (rc) return rc;
        a.first_launch = 1;
    }
    // The (latency, energy) key over the full row set is two passes that each cost what a single scalar
    // key costs: the lowest latency first, then the lowest energy among the candidates that reach it (a
    // candidate's latency is a maximum of a row part and a combination part, so the cap applies to the
    // two separately).  The second pass's energy record lands in the slot of this key.  The first pass
    // serves the latency key as well.  Of the scalar keys two go together in one pass, a third takes a pass of its own.
    const bool lex = mask & 4;
    a.final_key_dev = B.key_dev;
    if (e_limit) {
        // two scalar passes, as for the unbounded key; the second needs no energy bound: the
        // lowest energy among the candidates within the latency found is below it
        if (mask != 4) return MMEE_EINVAL;
        a.e_limit = *e_limit;
        launch_dense<2, true>(p.exact_k, grid, a);
    } else
        switch ((mask & 11) | (lex ? 2 : 0)) {
        case 1: launch_dense<1>(p.exact_k, grid, a); break;
        case 2: launch_dense<2>(p.exact_k, grid, a); break;
        case 8: launch_dense<8>(p.exact_k, grid, a); break;
        case 9: launch_dense<9>(p.exact_k, grid, a); break;
        case 10: launch_dense<10>(p.exact_k, grid, a); break;
        default: launch_dense<3>(p.exact_k, grid, a); break;
        }
    a.final_key_dev = nullptr;
    a.first_launch = 0;
    if (lex) {
        DenseArgs second = a;
        second.lat_cap = B.key_dev + 1;
        second.final_out = a.final_out + 2;
        if (a.done) second.done = a.done + 2;
        launch_dense<1, false, true>(p.exact_k, grid, second);
    }
    if (!e_limit && ((mask & 11) | (lex ? 2 : 0)) == 11) launch_dense<8>(p.exact_k, grid, a);
    return MMEE_OK;
}

// enqueue one pass (tables + search; the final records land in b.final_dev) in the buffers b
int enqueue_search_in(const Bufs &B, const Plan &p, int mask, uint32_t flags, uint64_t *evaluated,
                      const double *e_limit = nullptr, bool build_tables = true, bool bs_da_step = false,
                      bool *unproven = nullptr)
{
    const int which = (flags & MMEE_SEARCH_EXHAUSTIVE) ? 0 : 1;
    // the full row set goes through the dense kernel (lane = tiling, wave = 125 rows of a class), several keys on few
    // tilings excepted
    const bool dense = B.cls_dev && goes_dense(p, mask, flags, bs_da_step);
    const ModelConst mc = pass_constants(p, flags, bs_da_step ? 8 : mask, unproven, dense);
    if (dense) {
        uint64_t nrows = 0;
        for (int g = 0; g < 4; ++g) nrows += B.counts[0][g];
        if (B.ev_begin && !B.signalled) HIP_TRY(hipEventRecord(B.ev_begin, S.stream));
        const int drc = enqueue_dense(B, p, mc, mask, e_limit);
        if (drc) return drc;
        HIP_TRY(hipGetLastError());
        if (B.signalled) *B.signalled = true;
        else if (B.ev_end) HIP_TRY(hipEventRecord(B.ev_end, S.stream));
        *evaluated = nrows * p.T * 9ull;
        return MMEE_OK;
    }
    int rc = build_tables ? launch_tilings(p, mc, B, B.dv_dev) : MMEE_OK;
    if (rc) return rc;
    SearchArgs a;
    std::memset(&a, 0, sizeof(a));
    a.enc = B.enc; a.rows = B.rows[which]; a.row_enc = B.row_enc[which];
    // rows: one slot numbering per recomputation class r, over the lists of (r, f=0) and (r, f=1)
    uint32_t rb = 0;
    uint64_t nrows = 0;
    for (uint32_t r = 0; r < 2; ++r) {
        uint32_t in_class = 0;
        for (uint32_t f = 0; f < 2; ++f) {
            const uint32_t g = r + 2 * f;
            a.cls_off[r][f] = g * ROWS_PER_GROUP;
            a.cls_cnt[r][f] = B.counts[which][g];
            in_class += B.counts[which][g];
        }
        if (r == 0) a.rb_split = (in_class + SEARCH_THREADS - 1) / SEARCH_THREADS;
        rb += (in_class + SEARCH_THREADS - 1) / SEARCH_THREADS;
        nrows += in_class;
        // a short list fills few waves: let them come several times, each with a share of the tilings
        const uint32_t waves_for_rows = (in_class + 63) / 64;
        a.wave_split[r] = (!bs_da_step && waves_for_rows >= 1 && waves_for_rows <= 4) ? (SEARCH_THREADS / 64) / waves_for_rows : 1u;
    }
    const bool short_lists = a.wave_split[0] > 1 || a.wave_split[1] > 1;
    if (rb == 0) return MMEE_EINVAL;
    a.n_rb = rb;
    // tilings: chunks of TC, then chunks of TC_FINE worth about four fine items per resident block
    // (a coarse item's time), at least the ragged end
    {
        // (short lists split an item's tilings over the waves instead: short chunks only while one
        // round of blocks takes them all)
        const uint64_t all_fine = (p.T + TC_FINE - 1) / TC_FINE;
        const uint64_t fine_chunks_wanted = short_lists ? (rb * all_fine <= B.resident_blocks ? all_fine : 0)
                                                        : (4ull * B.resident_blocks + rb - 1) / rb;
        const uint64_t fine_tilings = std::min<uint64_t>(p.T, fine_chunks_wanted * TC_FINE);
        a.n_cc = (uint32_t)((p.T - fine_tilings) / TC);
        a.n_fc = (uint32_t)((p.T - (uint64_t)a.n_cc * TC + TC_FINE - 1) / TC_FINE);
    }
    a.btab = B.btab; a.ctab_s = B.ctab_s; a.ctab_e = B.ctab_e;
    a.mc = mc;
    const uint64_t n_items = (uint64_t)rb * ((uint64_t)a.n_cc + a.n_fc);
    a.n_coarse_items = rb * a.n_cc;
    if (n_items == 0 || n_items > 0x7fffffffull) return MMEE_EINVAL;
    a.n_items = (uint32_t)n_items;
    // persistent blocks: as many as the chip holds at once (LDS allows two per CU)
    const uint64_t nblocks = std::min<uint64_t>(n_items, (uint64_t)B.resident_blocks);
    if (nblocks > B.partials_cap) return MMEE_EINVAL;
    a.partials = B.partials; a.ticket = B.ticket; a.work_counter = B.ticket + 1;
    a.final_out = B.final_dev;
    a.dv = B.dv_dev;
    if (B.ev_begin) HIP_TRY(hipEventRecord(B.ev_begin, S.stream));
    dim3 grid((uint32_t)nblocks);
    if (bs_da_step) {
        if (!e_limit) return MMEE_EINVAL;
        a.e_limit = *e_limit;
        hipLaunchKernelGGL(k_front_step, grid, dim3(SEARCH_THREADS), 0, S.stream, a);
    } else if (e_limit) {
        if (mask != 4) return MMEE_EINVAL;
        a.e_limit = *e_limit;
        launch_search_limited(p.exact_k, grid, a);
    } else
    switch (mask) {
    case 1: launch_search_mask<1>(p.exact_k, grid, a); break;
    case 2: launch_search_mask<2>(p.exact_k, grid, a); break;
    case 3: launch_search_mask<3>(p.exact_k, grid, a); break;
    case 4: launch_search_mask<4>(p.exact_k, grid, a); break;
    case 5: launch_search_mask<5>(p.exact_k, grid, a); break;
    case 6: launch_search_mask<6>(p.exact_k, grid, a); break;
    case 7: launch_search_mask<7>(p.exact_k, grid, a); break;
    case 8: launch_search_mask<8>(p.exact_k, grid, a); break;
    case 9: launch_search_mask<9>(p.exact_k, grid, a); break;
    case 10: launch_search_mask<10>(p.exact_k, grid, a); break;
    case 11: launch_search_mask<11>(p.exact_k, grid, a); break;
    case 12: launch_search_mask<12>(p.exact_k, grid, a); break;
    case 13: launch_search_mask<13>(p.exact_k, grid, a); break;
    case 14: launch_search_mask<14>(p.exact_k, grid, a); break;
    case 15: launch_search_mask<15>(p.exact_k, grid, a); break;
    default: return MMEE_EINVAL;
    }
    HIP_TRY(hipGetLastError());
    if (B.ev_end) HIP_TRY(hipEventRecord(B.ev_end, S.stream));
    *evaluated = nrows * p.T * (bs_da_step ? 1ull : 9ull);
    return MMEE_OK;
}

// the same in the cached buffers of the allocating entry points, result slot `slot`
int enqueue_search(const Plan &p, int mask, uint32_t flags, size_t slot, uint64_t *evaluated,
                   const double *e_limit = nullptr, bool build_tables = true, bool bs_da_step = false,
                   bool *unproven = nullptr, bool *signalled = nullptr)
{
    Bufs b;
    int rc = state_bufs(p, slot, !goes_dense(p, mask, flags, bs_da_step), b);
    if (rc) return rc;
    b.signalled = signalled;
    return enqueue_search_in(b, p, mask, flags, evaluated, e_limit, build_tables, bs_da_step, unproven);
}

uint32_t list_length(const DivTable &dv) { return dv.ndiv[0] + dv.ndiv[1] + dv.ndiv[2] + dv.ndiv[3]; }
void pack_lists(const DivTable &dv, uint32_t *list)
{
    for (int q = 0; q < 4; ++q) {
        std::memcpy(list, dv.div[q], sizeof(uint32_t) * dv.ndiv[q]);
        list += dv.ndiv[q];
    }
}

static_assert(sizeof(BatchArgs) <= 4096, "kernel arguments are limited to 4 KiB");

// ---- batched search over the pruned rows -----------------------------------------------------

// The next call that ends by saying so: its place, its number.
int begin_signalled(Done *&done, uint64_t &number, uint64_t *&begin)
{
    const bool first = !S.done.host;
    HIP_TRY(ensure_pinned(HipPinned{}, S.done, sizeof(Done) * N_OBJ));
    if (first) std::memset(S.done.host, 0, sizeof(Done) * N_OBJ);
    if (!S.call_begin) HIP_TRY(hipMalloc(&S.call_begin, sizeof(uint64_t)));
    done = reinterpret_cast<Done *>(S.done.map);
    number = ++S.call_number;
    begin = S.call_begin;
    return MMEE_OK;
}

// what a core does between two looks at a word in memory
inline void between_looks()
{
#if defined(__x86_64__)
    __builtin_ia32_pause();
#elif defined(__aarch64__)
    asm volatile("yield");
#endif
}

// Until the records of the last signalled call are there (its keys: mask), and how long its kernels ran.  What does not come
// within 20 ms (a long search, work ahead of it on the caller's stream, an error) is waited for as any other command is.
int wait_signalled(int mask, double &seconds)
{
    const Done *done = reinterpret_cast<const Done *>(S.done.host);
    const auto give_up = std::chrono::steady_clock::now() + std::chrono::milliseconds(20);
    seconds = 0.0;
    bool synchronised = false;
    for (int o = 0; o < N_OBJ; ++o) {
        if (!((mask >> o) & 1)) continue;
        for (uint32_t look = 0; __atomic_load_n(&done[o].number, __ATOMIC_ACQUIRE) != S.call_number; ++look) {
            if (synchronised) {
                std::snprintf(g_last_error, sizeof(g_last_error), "a search ended without its records");
                return MMEE_EDEVICE;
            }
            if (look % 256 == 255 && std::chrono::steady_clock::now() > give_up) {
                HIP_TRY(hipStreamSynchronize(S.stream));
                synchronised = true;
            }
            between_looks();
        }
        seconds = std::max(seconds, (double)done[o].ticks / S.clock_hz);
    }
    return MMEE_OK;
}

// masks the batched kernel is built for; other key sets take the per-problem kernels
bool batch_mask(int mask) { return mask == 1 || mask == 2 || mask == 3 || mask == 4 || mask == 8; }

template <int MASK>
void launch_batch_mask(bool fast, bool regroup, dim3 grid, const BatchArgs &a)
{
    if (regroup) hipLaunchKernelGGL((k_search_batch<MASK, true, true>), grid, dim3(BATCH_THREADS), 0, S.stream, a);
    else if (fast) hipLaunchKernelGGL((k_search_batch<MASK, true, false>), grid, dim3(BATCH_THREADS), 0, S.stream, a);
    else hipLaunchKernelGGL((k_search_batch<MASK, false, false>), grid, dim3(BATCH_THREADS), 0, S.stream, a);
    // the problems' records are complete when the search kernel has ended: one block per problem finishes (a lone problem the search's own)
    if (!a.inl.on) hipLaunchKernelGGL((k_batch_finish<MASK>), dim3(a.n_prob), dim3(256), 0, S.stream, a);
}

// The kept rows shared out over the waves of a block and the row shares (rows.h: the kernel has the pieces' runs compiled in).
void set_batch_tasks(BatchArgs &a, uint32_t split)
{
    static_assert(PIECE_WAVES == BATCH_WAVES, "the pieces are those of the blocks");
    const uint32_t group_of[LEAST_CLASSES] = {0, 2, 3};      // class (r, f) -> g = r + 2 f
    a.split = split;
    for (uint32_t sh = 0; sh < split; ++sh)
        for (uint32_t wv = 0; wv < BATCH_WAVES; ++wv) {
            const PieceRange p = piece_range(split, sh, wv);
            a.task_lo[sh * BATCH_WAVES + wv] = KEPT.first[p.cls] + p.lo;
            a.task_cnt[sh * BATCH_WAVES + wv] = p.n;
            a.task_g[sh * BATCH_WAVES + wv] = group_of[p.cls];
        }
}

// Blocks that share a chunk's rows: two while both have a CU to themselves, which is as long as no CU has to take a second block.
// (Call, us, 1 block / 2: 1 chunk 20.6 / 19.4, 12 chunks 21.5 / 20.7, 46 chunks 21.7 / 21.0, 77 chunks 15.9 / 15.9 without the
// host's wait, 144 chunks 26.1 / 29.1.)
uint32_t batch_split(uint64_t chunks, uint32_t resident_blocks) { return chunks * 4 <= resident_blocks ? 2 : 1; }

void fill_batch_head(BatchProblemHead &h, uint32_t *list, const Plan &p, const ModelConst &mc, uint32_t slot, uint32_t first_item, uint32_t split)
{
    h.mc = mc;
    h.first_item = first_item;
    h.n_work = (uint32_t)((p.T + PRUNED_TC - 1) / PRUNED_TC) * split;
    h.slot = slot;
    h.pad_ = 0;
    for (int q = 0; q < 4; ++q) { h.X[q] = p.dv.X[q]; h.ndiv[q] = p.dv.ndiv[q]; }
    pack_lists(p.dv, list);
}

int launch_batch(int mask, bool fast, bool regroup, dim3 grid, const BatchArgs &a)
{
    switch (mask) {
    case 1: launch_batch_mask<1>(fast, regroup, grid, a); break;
    case 2: launch_batch_mask<2>(fast, regroup, grid, a); break;
    case 3: launch_batch_mask<3>(fast, regroup, grid, a); break;
    case 4: launch_batch_mask<4>(fast, regroup, grid, a); break;
    case 8: launch_batch_mask<8>(fast, regroup, grid, a); break;
    default: return MMEE_EINVAL;
    }
    HIP_TRY(hipGetLastError());
    return MMEE_OK;
}

int ensure_batch(size_t blob_bytes, size_t n_items)
{
    if (blob_bytes > S.batch_blob_cap) {
        if (S.batch_host) { HIP_TRY(hipStreamSynchronize(S.stream)); (void)hipHostFree(S.batch_host); (void)hipFree(S.batch_dev); }
        S.batch_host = nullptr; S.batch_dev = nullptr; S.batch_blob_cap = 0;
        const size_t cap = std::max<size_t>(blob_bytes * 2, 1 << 16);
        HIP_TRY(hipHostMalloc(&S.batch_host, cap, hipHostMallocDefault));
        HIP_TRY(hipMalloc(&S.batch_dev, cap));
        S.batch_blob_cap = cap;
    }
    if (n_items > S.item_cap) {
        if (S.item_keys) { HIP_TRY(hipStreamSynchronize(S.stream)); (void)hipFree(S.item_keys); }
        S.item_keys = nullptr; S.item_cap = 0;
        const size_t cap = std::max<size_t>(n_items * 2, 4096);
        HIP_TRY(hipMalloc(&S.item_keys, sizeof(Key) * N_OBJ * cap));
        S.item_cap = cap;
    }
    return MMEE_OK;
}

// One problem of a batched launch, as the host sees it.
struct BatchEntry {
    const Plan *plan;
    int mask;
    size_t slot;            // result slot: its N_OBJ final records
    ModelConst mc;          // with the regrouping decision taken
    bool unproven;          // regrouped on trust (pass_constants)
    uint64_t evaluated;
};

// Enqueue the entries (all pruned searches) as few launches as their kernel variants allow: one per
// (key set, exact DRAM constant, regrouped) combination present.  Events of slot `ev_slot` bracket it all, but for a lone
// problem that rides in the arguments: `signalled`, it is waited for with wait_signalled.
int enqueue_batches(std::vector<BatchEntry> &entries, uint32_t flags, size_t ev_slot, bool &signalled)
{
    signalled = false;
    if (entries.empty()) return MMEE_OK;
    struct Variant { int mask; bool fast, regroup; std::vector<size_t> members; uint64_t items = 0; uint32_t split = 1; };
    std::vector<Variant> variants;
    uint64_t kept_rows = 0;
    for (int g = 0; g < 4; ++g) kept_rows += S.counts[1][g];
    uint64_t total_items = 0;
    for (size_t k = 0; k < entries.size(); ++k) {
        BatchEntry &e = entries[k];
        e.mc = pass_constants(*e.plan, flags, e.mask, &e.unproven);
        e.evaluated = kept_rows * e.plan->T * 9ull;
        const bool fast = e.plan->exact_k, regroup = e.mc.regroup != 0;
        Variant *v = nullptr;
        for (Variant &c : variants)
            if (c.mask == e.mask && c.fast == fast && c.regroup == regroup) v = &c;
        if (!v) { variants.push_back(Variant{e.mask, fast, regroup, {}, 0, 1}); v = &variants.back(); }
        v->members.push_back(k);
        v->items += (e.plan->T + PRUNED_TC - 1) / PRUNED_TC;
    }
    for (Variant &v : variants) {
        v.split = batch_split(v.items, S.resident_blocks);
        v.items *= v.split;
        total_items += v.items;
    }
    if (total_items > 0x7fffffffull) return MMEE_EINVAL;
    auto fill_head = [&](BatchProblemHead &h, uint32_t *list, const BatchEntry &e, uint32_t first_item, uint32_t split) {
        fill_batch_head(h, list, *e.plan, e.mc, (uint32_t)e.slot, first_item, split);
    };
    // A variant with one problem whose divisor lists fit carries it in the kernel arguments; the others'
    // descriptors go through one blob: per variant its problem descriptors, then its first-item table.
    auto rides_in_arguments = [&](const Variant &v) {
        return v.members.size() == 1 && list_length(entries[v.members[0]].plan->dv) <= (uint32_t)BATCH_INLINE_DIVS;
    };
    size_t blob = 0;
    for (const Variant &v : variants)
        if (!rides_in_arguments(v))
            blob += sizeof(BatchProblem) * v.members.size() + sizeof(uint32_t) * ((v.members.size() + 1 + 3) & ~(size_t)3);
    int rc = ensure_batch(blob, total_items);
    if (rc) return rc;
    size_t off = 0;
    uint64_t item0 = 0;
    struct Launch { size_t desc_off, firsts_off, n_prob; uint64_t item0, n_items; bool in_args; };
    std::vector<Launch> launches;
    for (const Variant &v : variants) {
        Launch L;
        L.desc_off = L.firsts_off = 0;
        L.n_prob = v.members.size(); L.item0 = item0; L.n_items = v.items; L.in_args = rides_in_arguments(v);
        item0 += v.items;
        if (!L.in_args) {
            L.desc_off = off;
            BatchProblem *bp = reinterpret_cast<BatchProblem *>(S.batch_host + off);
            off += sizeof(BatchProblem) * v.members.size();
            L.firsts_off = off;
            uint32_t *firsts = reinterpret_cast<uint32_t *>(S.batch_host + off);
            off += sizeof(uint32_t) * ((v.members.size() + 1 + 3) & ~(size_t)3);
            uint32_t item = 0;
            for (size_t k = 0; k < v.members.size(); ++k) {
                fill_head(bp[k].h, bp[k].list, entries[v.members[k]], item, v.split);
                firsts[k] = item;
                item += bp[k].h.n_work;
            }
            firsts[v.members.size()] = item;
        }
        launches.push_back(L);
    }
    Done *done = nullptr;
    uint64_t number = 0, *begin = nullptr;
    signalled = entries.size() == 1 && launches[0].in_args;
    if (signalled) {
        rc = begin_signalled(done, number, begin);
        if (rc) return rc;
    } else
        HIP_TRY(hipEventRecord(S.events[2 * ev_slot], S.stream));
    if (off) HIP_TRY(hipMemcpyAsync(S.batch_dev, S.batch_host, off, hipMemcpyHostToDevice, S.stream));
    for (size_t k = 0; k < variants.size(); ++k) {
        const Variant &v = variants[k];
        const Launch &L = launches[k];
        BatchArgs a;
        std::memset(&a, 0, sizeof(a));
        if (L.in_args) {
            fill_head(a.inl.h, a.inl.list, entries[v.members[0]], 0, v.split);
            a.inl.firsts[0] = 0; a.inl.firsts[1] = a.inl.h.n_work;
            a.inl.on = 1;
        } else {
            a.prob = reinterpret_cast<const BatchProblem *>(S.batch_dev + L.desc_off);
            a.first_items = reinterpret_cast<const uint32_t *>(S.batch_dev + L.firsts_off);
        }
        a.n_prob = (uint32_t)L.n_prob; a.n_items = (uint32_t)L.n_items;
        a.enc = S.enc;
        set_batch_tasks(a, v.split);
        a.item_keys = S.item_keys + N_OBJ * L.item0;
        a.final_out = S.final_map;
        a.done = done; a.number = number; a.begin = begin;
        a.ticket = S.ticket + 2;
        // persistent blocks, two per CU, each with a contiguous range of the items
        dim3 grid((uint32_t)std::min<uint64_t>(L.n_items, (uint64_t)S.resident_blocks));
        a.per_block = a.n_items / grid.x; a.extra = a.n_items % grid.x;
        rc = launch_batch(v.mask, v.fast, v.regroup, grid, a);
        if (rc) return rc;
    }
    if (!signalled) HIP_TRY(hipEventRecord(S.events[2 * ev_slot + 1], S.stream));
    return MMEE_OK;
}

// ---- pruned search ---------------------------------------------------------------------------

static_assert(sizeof(PrunedArgs) <= 4096, "kernel arguments are limited to 4 KiB");

// One problem of a pruned search, as the host sees it.
struct PrunedEntry {
    const Plan *plan;
    int mask;
    uint32_t slot;          // result slot: its N_OBJ final records
};

DigitConst digit_constants(const DivTable &dv)
{
    DigitConst d;
    double radix = 1.0;
    for (int q = 0; q < 4; ++q) {
        d.rcp_radix[q] = 1.0 / radix;
        d.rcp_n[q] = 1.0 / (double)dv.ndiv[q];
        radix *= (double)dv.ndiv[q];
    }
    return d;
}

// extents and operand sizes (A, B, D, E, C) as fp64; exact: all counts of a problem are below 2^53
void shape_constants(const DivTable &dv, double (&extent)[4], double (&size)[5])
{
    for (int q = 0; q < 4; ++q) extent[q] = (double)dv.X[q];
    size[0] = extent[DI] * extent[DK]; size[1] = extent[DK] * extent[DL]; size[2] = extent[DL] * extent[DJ];
    size[3] = extent[DI] * extent[DJ]; size[4] = extent[DI] * extent[DL];
}

// Groups of problems with one shape, laid out as the kernel reads them.
struct PrunedLayout {
    unsigned char *desc = nullptr;          // room for `bytes`
    size_t bytes = 0;
    uint32_t n_groups = 0, n_members = 0, members_off = 0, n_items = 0;
    uint64_t n_keys = 0;    // records of all its items
};

// entries[order[k]], k in [lo, hi): the groups of one launch
struct PrunedSlice { uint32_t lo, hi, n_caps; };

bool same_shape(const Plan &a, const Plan &b)
{
    // (extents and divisor counts settle the divisor lists: two modes with equal counts list the same divisors)
    return std::memcmp(a.dv.X, b.dv.X, sizeof(a.dv.X)) == 0 && std::memcmp(a.dv.ndiv, b.dv.ndiv, sizeof(a.dv.ndiv)) == 0;
}

// Problems of one shape become groups of at most PRUNED_MEMBERS, by ascending capacity.
void pruned_slices(const std::vector<PrunedEntry> &entries, std::vector<uint32_t> &order, std::vector<PrunedSlice> &slices)
{
    // shapes in order of first appearance, through a small open-addressed table
    std::vector<uint32_t> head, shape_of(entries.size()), count;
    size_t cap = 16;
    while (cap < 2 * entries.size()) cap *= 2;
    std::vector<uint32_t> table(cap, 0xFFFFFFFFu);
    for (uint32_t k = 0; k < entries.size(); ++k) {
        const DivTable &dv = entries[k].plan->dv;
        uint64_t h = 0x9E3779B97F4A7C15ull;
        for (int q = 0; q < 4; ++q) h = (h ^ (dv.X[q] + ((uint64_t)dv.ndiv[q] << 32))) * 0xBF58476D1CE4E5B9ull;
        size_t at = (h >> 32) & (cap - 1);
        while (table[at] != 0xFFFFFFFFu && !same_shape(*entries[head[table[at]]].plan, *entries[k].plan)) at = (at + 1) & (cap - 1);
        if (table[at] == 0xFFFFFFFFu) { table[at] = (uint32_t)head.size(); head.push_back(k); count.push_back(0); }
        shape_of[k] = table[at];
        ++count[shape_of[k]];
    }
    std::vector<uint32_t> at(head.size() + 1, 0);
    for (size_t g = 0; g < head.size(); ++g) at[g + 1] = at[g] + count[g];
    order.resize(entries.size());
    std::vector<uint32_t> next(at.begin(), at.end() - 1);
    for (uint32_t k = 0; k < entries.size(); ++k) order[next[shape_of[k]]++] = k;
    auto cap_of = [&](uint32_t k) { return entries[order[k]].plan->mc.cap_words; };
    slices.clear();
    for (size_t g = 0; g < head.size(); ++g) {
        std::sort(order.begin() + at[g], order.begin() + at[g + 1], [&](uint32_t a, uint32_t b) {
            const double ca = entries[a].plan->mc.cap_words, cb = entries[b].plan->mc.cap_words;
            return ca != cb ? ca < cb : a < b;
        });
        for (uint32_t lo = at[g]; lo < at[g + 1]; lo += PRUNED_MEMBERS) {
            PrunedSlice sl{lo, std::min<uint32_t>(lo + PRUNED_MEMBERS, at[g + 1]), 1};
            for (uint32_t k = lo + 1; k < sl.hi; ++k) sl.n_caps += cap_of(k) != cap_of(k - 1);
            slices.push_back(sl);
        }
    }
}

// Of a call's groups, those that k_search_pruned takes; the others stay with k_search_batch, or, with a key set that it
// is not built for, get a pass of their own.
//
// A block of k_search_batch takes a chunk of one problem, 512 at a time on the chip; a block of k_search_pruned takes
// a chunk of all problems of a group, its waves an eighth of them each, one after the other: with few
// chunks that chain is longer than what the row side costs per problem.  So the ways are estimated, in microseconds per
// call apart from what the host does per problem either way (0.44): all in batches; groups of four problems or more
// shared and the rest in batches (two sets of copies and launches that wait for each other: 110); all shared.
// Fitted to 3200 calls of 1 to 640 problems on 1 to 40 shapes of 1 to 324 chunks with 1 to 64 capacities, one key set a
// call: the choice costs 1 % over the better way on average; 10 % or more over k_search_batch in 15 calls (64 problems
// on each of two shapes of 28 chunks, 16 capacities, latency: 180 us in batches, 274 shared), 10 % or more over sharing from
// four problems a group on in 16 (64 of 77 chunks with 64 capacities, energy: 146 us shared, 178 in batches).
// Sharing from four problems a group on whatever their size cost up to 208 % (64 problems of one chunk, energy: 118
// us, 68 in batches), never sharing up to 270 % (64 problems of 324 chunks, energy: 475 us, 126 shared).  A pass of its
// own costs 33 us a problem of one chunk and 105 us at 324 chunks (energy, latency and energy-delay product).
// These figures and the constants are of the kernels of the fit.  Both ways of 600 calls with the kernels as they are (2 to 640 problems on 1 to
// 16 shapes of 1 to 324 chunks): with a group of four problems or more the choice costs 1.6 % over the better way on average and 10 %
// or more in 19 of 413 calls (32 problems on one shape of 105 chunks, 16 capacities, latency: 103 us in batches, 146 shared).  Of the 187 calls
// without such a group, which stay in batches whatever the estimates say (none_large), 74 would be 10 % or more faster shared (three
// problems on each of eight shapes of 28 to 100 chunks, energy and latency: 82 us, 58 shared).
void keep_shared(const std::vector<PrunedEntry> &entries, const std::vector<uint32_t> &order, std::vector<PrunedSlice> &slices)
{
    struct Batches {                         // chunks, and kinds of kernel: each is a launch of its own
        double items = 0.0;
        uint64_t kinds = 0;
        void add(const PrunedEntry &e, double chunks)
        {
            items += chunks;
            kinds |= 1ull << (e.mask * 4 + (e.plan->exact_k ? 2 : 0) + (e.plan->can_regroup ? 1 : 0));
        }
        double us() const
        {
            const double rounds = items / 512.0;
            return items == 0.0 ? 0.0 : 21.0 + 20.0 * __builtin_popcountll(kinds) + 15.0 * std::min(1.0, rounds) + 10.5 * std::max(0.0, rounds - 1.0);
        }
    };
    struct Shared {                          // bytes of descriptions, the longest block, all blocks 512 at a time
        size_t bytes = 0;
        double longest = 0.0, work = 0.0;
        // wait_us: what the block's waves wait for memory and for each other, hidden where other blocks follow
        void add(size_t members, double chunks, double block_us, double wait_us)
        {
            bytes += sizeof(PrunedGroup) + members * sizeof(PrunedMember);
            longest = std::max(longest, block_us + wait_us);
            work += 1.2 / 512.0 * chunks * block_us;
        }
        // (descriptions beyond the kernel arguments are copied)
        double us() const { return 10.0 + (bytes > (size_t)PRUNED_INLINE ? 10.0 : 0.0) + std::max(longest, work); }
    };
    // one problem after the other: per problem, and what it waits
    auto key_us = [](int mask) {
        return ((mask & 3) == 3 ? 7.6 : ((mask & 1) ? 6.4 : ((mask & 2) ? 4.6 : 0.0))) + ((mask & 4) ? 15.3 : 0.0) + ((mask & 8) ? 6.6 : 0.0);
    };
    auto key_wait_us = [](int mask) { return ((mask & 2) ? 2.9 : ((mask & 1) ? 1.0 : 0.0)) + ((mask & 4) ? 3.4 : 0.0) + ((mask & 8) ? 0.7 : 0.0); };
    Batches all, rest;
    Shared large, every;
    double alone_us = 0.0, rest_alone_us = 0.0;
    auto is_large = [](const PrunedSlice &sl) { return sl.hi - sl.lo >= 4; };
    for (const PrunedSlice &sl : slices) {
        const double chunks = std::ceil((double)entries[order[sl.lo]].plan->T / PRUNED_TC);
        const uint32_t members = sl.hi - sl.lo;
        double keys = 0.0, waits = 0.0;
        for (uint32_t k = sl.lo; k < sl.hi; ++k) {
            const PrunedEntry &e = entries[order[k]];
            keys += key_us(e.mask);
            waits += key_wait_us(e.mask);
            if (!batch_mask(e.mask)) {
                alone_us += 33.0 + 0.22 * chunks;
                if (!is_large(sl)) rest_alone_us += 33.0 + 0.22 * chunks;
                continue;
            }
            all.add(e, chunks);
            if (!is_large(sl)) rest.add(e, chunks);
        }
        // (another round of capacities: the rows once more)
        const double turns = std::ceil(members / 8.0) / members;
        const double block_us = 20.0 + 16.0 * ((sl.n_caps - 1) / PRUNED_ROUND) + keys * turns;
        every.add(members, chunks, block_us, waits * turns);
        if (is_large(sl)) large.add(members, chunks, block_us, waits * turns);
    }
    // (85: the 110, less what the synchronisation adds to either part; 1.15: a lone problem's blocks are short of waves in step 2)
    const double batched_us = all.us() + alone_us, every_us = every.us() * (rest.items > 0.0 ? 1.15 : 1.0);
    const double mixed_us = large.bytes && rest.items > 0.0 ? large.us() + rest.us() + rest_alone_us + 85.0 : INFINITY;
    const bool none_large = !large.bytes && alone_us == 0.0;
    if (none_large || batched_us <= std::min(every_us, mixed_us)) slices.clear();
    else if (mixed_us < every_us) slices.erase(std::remove_if(slices.begin(), slices.end(), [&](const PrunedSlice &sl) { return !is_large(sl); }), slices.end());
}

size_t up16(size_t x) { return (x + 15) & ~(size_t)15; }

// bytes of the descriptions, and where their parts begin
size_t pruned_bytes(const std::vector<PrunedEntry> &entries, const std::vector<uint32_t> &order, const std::vector<PrunedSlice> &slices,
                    size_t &members_off, size_t &caps_off, size_t &list_off)
{
    size_t n_members = 0, n_caps = 0, n_list = 0;
    for (const PrunedSlice &sl : slices) {
        n_members += sl.hi - sl.lo;
        n_caps += sl.n_caps;
        n_list += list_length(entries[order[sl.lo]].plan->dv);
    }
    members_off = up16(sizeof(PrunedGroup) * slices.size());
    caps_off = up16(members_off + sizeof(PrunedMember) * n_members);
    list_off = up16(caps_off + sizeof(double) * n_caps);
    return up16(list_off + sizeof(uint32_t) * n_list);
}

// ... written to out.desc
void pruned_layout(const std::vector<PrunedEntry> &entries, const std::vector<uint32_t> &order, const std::vector<PrunedSlice> &slices,
                   PrunedLayout &out)
{
    size_t members_off, caps_off, list_off, n_members = 0;
    (void)pruned_bytes(entries, order, slices, members_off, caps_off, list_off);
    for (const PrunedSlice &sl : slices) n_members += sl.hi - sl.lo;
    out.n_groups = (uint32_t)slices.size();
    out.n_members = (uint32_t)n_members;
    out.members_off = (uint32_t)members_off;
    unsigned char *base = out.desc;
    PrunedGroup *groups = reinterpret_cast<PrunedGroup *>(base);
    PrunedMember *members = reinterpret_cast<PrunedMember *>(base + members_off);
    uint32_t item = 0, member = 0;
    for (size_t g = 0; g < slices.size(); ++g) {
        const PrunedSlice &sl = slices[g];
        const Plan &p = *entries[order[sl.lo]].plan;
        PrunedGroup G;
        std::memset(&G, 0, sizeof(G));
        G.first_item = item;
        G.n_items = (uint32_t)((p.T + PRUNED_TC - 1) / PRUNED_TC);
        G.member0 = member;
        G.n_members = sl.hi - sl.lo;
        G.n_caps = sl.n_caps;
        G.caps_off = (uint32_t)caps_off;
        G.T = (uint32_t)p.T;
        G.key0 = out.n_keys;
        out.n_keys += (uint64_t)G.n_items * G.n_members * N_OBJ;
        G.list_off = (uint32_t)list_off;
        double *caps = reinterpret_cast<double *>(base + caps_off);
        uint32_t cap = 0;
        for (uint32_t k = sl.lo; k < sl.hi; ++k) {
            const PrunedEntry &e = entries[order[k]];
            if (k == sl.lo) caps[0] = e.plan->mc.cap_words;
            else if (e.plan->mc.cap_words != caps[cap]) caps[++cap] = e.plan->mc.cap_words;
            PrunedMember &m = members[member++];
            m.mc = e.plan->mc;
            m.slot = e.slot; m.cap = cap; m.mask = (uint32_t)e.mask; m.group = (uint32_t)g;
            const DivTable &dv = e.plan->dv;
            const double X[4] = {(double)dv.X[0], (double)dv.X[1], (double)dv.X[2], (double)dv.X[3]};
            const double m1 = X[DI] * X[DK] * X[DL], m2 = X[DI] * X[DL] * X[DJ], sm = (double)m.mc.c_softmax * (X[DI] * X[DL]);
            m.rf_words[0] = m.mc.BH * 3.0 * m1; m.rf_words[1] = m.mc.BH * 3.0 * m2;      // (whole numbers: exact)
            m.mac_ops[0] = m.mc.BH * (m1 + sm); m.mac_ops[1] = m.mc.BH * m2;
            m.e_rf0 = m.mc.e_rf * (m.rf_words[0] + m.rf_words[1]); m.e_mac0 = m.mc.e_mac * (m.mac_ops[0] + m.mac_ops[1]);
            m.exact_k = e.plan->exact_k; m.pad_ = 0;
        }
        uint32_t *list = reinterpret_cast<uint32_t *>(base + list_off);
        for (int q = 0; q < 4; ++q) {
            G.X[q] = p.dv.X[q];
            G.ndiv[q] = p.dv.ndiv[q];
        }
        G.dg = digit_constants(p.dv);
        shape_constants(p.dv, G.extent, G.size);
        pack_lists(p.dv, list);
        list += list_length(p.dv);
        caps_off += sizeof(double) * sl.n_caps;
        list_off = (size_t)(reinterpret_cast<unsigned char *>(list) - base);
        item += G.n_items;
        groups[g] = G;
    }
    out.n_items = item;
}

// Launch the search and its finish.  desc_dev: the layout's descriptions in device memory; null: they fit the
// kernel arguments.
int launch_pruned(const PrunedLayout &l, const unsigned char *desc_dev, Key *keys)
{
    static PrunedArgs a;                       // (callers hold g_lock)
    std::memset(&a, 0, offsetof(PrunedArgs, inl));
    a.desc = desc_dev;
    if (!desc_dev) {
        if (l.bytes > sizeof(a.inl)) return MMEE_EINVAL;
        std::memcpy(a.inl, l.desc, l.bytes);
    }
    a.n_groups = l.n_groups; a.n_items = l.n_items;
    a.members_off = l.members_off;
    a.enc = S.enc; a.keys = keys; a.hints = S.pruned_hints; a.final_out = S.final_map;
    hipLaunchKernelGGL(k_search_pruned, dim3(l.n_items), dim3(PRUNED_THREADS), 0, S.stream, a);
    hipLaunchKernelGGL(k_pruned_finish, dim3(l.n_members), dim3(256), 0, S.stream, a);
    HIP_TRY(hipGetLastError());
    return MMEE_OK;
}

int ensure_desc(size_t bytes)
{
    if (bytes <= S.desc_cap) return MMEE_OK;
    if (S.desc_host) { HIP_TRY(hipStreamSynchronize(S.stream)); (void)hipHostFree(S.desc_host); (void)hipFree(S.desc_dev); }
    S.desc_host = nullptr; S.desc_dev = nullptr; S.desc_cap = 0;
    const size_t cap = std::max<size_t>(bytes * 2, 1 << 16);
    HIP_TRY(hipHostMalloc(&S.desc_host, cap, hipHostMallocDefault));
    HIP_TRY(hipMalloc(&S.desc_dev, cap));
    S.desc_cap = cap;
    return MMEE_OK;
}

int ensure_block_records(size_t bytes)
{
    if (bytes <= S.block_records_cap) return MMEE_OK;
    if (S.block_records) { HIP_TRY(hipStreamSynchronize(S.stream)); (void)hipFree(S.block_records); }
    S.block_records = nullptr; S.block_records_cap = 0;
    const size_t cap = std::max<size_t>(bytes + bytes / 2, 1 << 20);
    HIP_TRY(hipMalloc(&S.block_records, cap));
    S.block_records_cap = cap;
    return MMEE_OK;
}

// Enqueue the pruned searches of these groups.  Events of slot `ev_slot` bracket it all.
int enqueue_pruned(const std::vector<PrunedEntry> &entries, const std::vector<uint32_t> &order, const std::vector<PrunedSlice> &slices,
                   size_t ev_slot)
{
    uint64_t items = 0;
    for (const PrunedSlice &sl : slices) items += (entries[order[sl.lo]].plan->T + PRUNED_TC - 1) / PRUNED_TC;
    if (items > 0x7fffffffull) return MMEE_EINVAL;
    PrunedLayout l;
    size_t members_off, caps_off, list_off;
    l.bytes = pruned_bytes(entries, order, slices, members_off, caps_off, list_off);
    const bool inside = l.bytes <= (size_t)PRUNED_INLINE;
    alignas(16) unsigned char small[PRUNED_INLINE];
    int rc = inside ? MMEE_OK : ensure_desc(l.bytes);
    if (rc) return rc;
    l.desc = inside ? small : S.desc_host;
    pruned_layout(entries, order, slices, l);
    rc = ensure_block_records((size_t)l.n_keys * sizeof(Key));
    if (rc) return rc;
    HIP_TRY(hipEventRecord(S.events[2 * ev_slot], S.stream));
    if (!inside) HIP_TRY(hipMemcpyAsync(S.desc_dev, S.desc_host, l.bytes, hipMemcpyHostToDevice, S.stream));
    rc = launch_pruned(l, inside ? nullptr : S.desc_dev, static_cast<Key *>(S.block_records));
    if (rc) return rc;
    HIP_TRY(hipEventRecord(S.events[2 * ev_slot + 1], S.stream));
    return MMEE_OK;
}

uint64_t kept_row_count() { return (uint64_t)S.counts[1][0] + S.counts[1][1] + S.counts[1][2] + S.counts[1][3]; }

int unpack_record(const Plan &p, const FinalRecord &fr, uint64_t evaluated, double seconds, double ksec, mmee_result *out)
{
    std::memset(out, 0, sizeof(*out));
    std::memcpy(&out->cost, fr.cost, sizeof(mmee_cost));
    std::memcpy(&out->best, fr.map, sizeof(mmee_mapping));
    out->space = p.space;
    out->evaluated = evaluated;
    out->seconds = seconds;
    out->kernel_seconds = ksec;
    if (!(fr.key.p < INFINITY)) { out->cost.valid = 0; return MMEE_ENOFEASIBLE; }
    return MMEE_OK;
}

int unpack_result(const Plan &p, size_t slot, int objective, uint64_t evaluated, double seconds, double ksec,
                  mmee_result *out)
{
    return unpack_record(p, S.final_host[N_OBJ * slot + objective], evaluated, seconds, ksec, out);
}

// ---- fronts over the kept rows ---------------------------------------------------------------

static_assert(sizeof(FrontArgs) <= 4096, "kernel arguments are limited to 4 KiB");

constexpr size_t FRONT_N_AT = sizeof(FinalRecord) * FRONT_POINTS;     // where S.front has the number of its records, and which way

// The front in two launches; its records and their number land in S.front (TOO_MANY: something outgrew its room,
// walk the front).  Waited for with wait_signalled, as key 0.
int enqueue_front(const Plan &p, bool bs_da, uint32_t capacity)
{
    if (!S.front_points) HIP_TRY(hipMalloc(&S.front_points, sizeof(Key) * FRONT_BLOCKS * FRONT_BLOCK));
    if (!S.front_stairs) HIP_TRY(hipMalloc(&S.front_stairs, sizeof(unsigned long long) * FRONT_STEPS));
    if (!S.front_counts) HIP_TRY(hipMalloc(&S.front_counts, sizeof(uint32_t) * 2));
    HIP_TRY(ensure_pinned(HipPinned{}, S.front, FRONT_N_AT + 2 * sizeof(uint32_t)));
    FrontArgs a;
    std::memset(&a, 0, sizeof(a));
    a.mc = p.mc;
    a.dg = digit_constants(p.dv);
    shape_constants(p.dv, a.extent, a.size);
    for (int q = 0; q < 4; ++q) { a.X[q] = p.dv.X[q]; a.ndiv[q] = p.dv.ndiv[q]; }
    if (list_length(p.dv) > FRONT_DIVS) return MMEE_EINVAL;
    pack_lists(p.dv, a.list);
    a.capacity = std::min<uint32_t>(capacity, FRONT_POINTS);
    a.pool = S.front_pool;
    a.points = S.front_points; a.stairs = S.front_stairs; a.counts = S.front_counts; a.enc = S.enc;
    a.out = reinterpret_cast<FinalRecord *>(S.front.map);
    a.n_out = reinterpret_cast<uint32_t *>(S.front.map + FRONT_N_AT);
    // The staircase's steps.  Values of equal upper bits share one: how fine it is decides what a look at it spares,
    // not what the front is.  Buffer sizes lie between 1 and twice all five matrices: as many steps to a factor of
    // two as there is room for.  Latencies worth having lie within a few factors of two above what arithmetic and DRAM ask for
    // at the least: 64 steps to each of eight.
    double lowest = 1.0;
    uint32_t fine = 6;
    if (bs_da) {
        const double most = 2.0 * (a.size[0] + a.size[1] + a.size[2] + a.size[3] + a.size[4]);
        for (fine = 9; fine && ((uint64_t)(std::ilogb(most) + 1) << fine) > FRONT_STEPS; --fine) {}
    } else {
        const double cycles = (a.extent[DI] * a.extent[DK] * a.extent[DL] + a.extent[DI] * a.extent[DL] * a.extent[DJ]) /
                              ((double)p.mc.pe_rows * (double)p.mc.pe_cols);
        const double fetch = p.mc.dram_bw > 0.0 ? (a.size[0] + a.size[1] + a.size[2] + a.size[3]) * p.mc.word / p.mc.dram_bw : 0.0;
        lowest = 0.999 * p.mc.c_lat * std::max(cycles, fetch);
    }
    a.step_shift = 20 - fine;
    {
        uint64_t bits;
        std::memcpy(&bits, &lowest, sizeof(bits));
        a.step0 = (int32_t)((uint32_t)(bits >> 32) >> a.step_shift);
    }
    const uint32_t n_blocks = (uint32_t)((p.T + PRUNED_TC - 1) / PRUNED_TC) * (bs_da ? FRONT_SPLIT : 1);
    {
        const int rc = begin_signalled(a.done, a.number, a.begin);
        if (rc) return rc;
    }
    if (!S.front_clean) {
        hipLaunchKernelGGL(k_fill_words64, dim3((FRONT_STEPS + 255) / 256), dim3(256), 0, S.stream, S.front_stairs, (uint64_t)FRONT_STEPS, INF_BITS);
        hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(64), 0, S.stream, S.front_counts, 2u);
    }
    // Until the merge, which cleans up, has been seen to end: launches into a stream under capture are in the stream and
    // never run, nor do the two fills then, and a list that begins at whatever the counters hold lies outside its array.
    S.front_clean = false;
    if (bs_da) hipLaunchKernelGGL(k_front_points<true>, dim3(n_blocks), dim3(PRUNED_THREADS), 0, S.stream, a);
    else hipLaunchKernelGGL(k_front_points<false>, dim3(n_blocks), dim3(PRUNED_THREADS), 0, S.stream, a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_front_merge, dim3(1), dim3(MERGE_THREADS), 0, S.stream, a);
    HIP_TRY(hipGetLastError());
    return MMEE_OK;
}

bool same_problem(const mmee_chain &a, const mmee_hw &b, const mmee_chain &c, const mmee_hw &d)
{
    return std::memcmp(&a, &c, sizeof(a)) == 0 && b.pe_rows == d.pe_rows && b.pe_cols == d.pe_cols &&
           b.n_arrays == d.n_arrays && b.rf_bytes == d.rf_bytes && b.gb_bytes == d.gb_bytes &&
           b.e_dram == d.e_dram && b.e_gb == d.e_gb && b.e_rf == d.e_rf && b.e_mac == d.e_mac &&
           b.dram_bw == d.dram_bw && b.gb_bw == d.gb_bw;
}

double now_seconds()
{
    return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

// ---- the entry point that allocates nothing: per-device set-up of the fixed scratch -----------

constexpr int NOALLOC_MAX_DEVICES = 64;
struct NoAllocDevice {
    unsigned char *ptr = nullptr;        // this device's copy of `scratch`
    bool built = false;                  // offline stage done in it
    uint32_t counts[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
    uint32_t resident_blocks = 0;
    uint32_t tickets = 0;                // handed out
} g_noalloc[NOALLOC_MAX_DEVICES];

// First call on a device: the address of that device's array, then the offline stage (row encoding,
// pruning, compaction) into it; its eight counts and the kept rows' numbers come back to the host.  Nothing is allocated.
int noalloc_setup(int dev, NoAllocDevice *&out)
{
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return MMEE_EINVAL;
    NoAllocDevice &d = g_noalloc[dev];
    out = &d;
    if (d.built) return MMEE_OK;
    if (!d.ptr) {
        unsigned char *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(scratch)));
        if (!ptr) {
            std::snprintf(g_last_error, sizeof(g_last_error), "hipGetSymbolAddress returned no address for the scratch array");
            return MMEE_EDEVICE;
        }
        d.ptr = ptr;
    }
    int cus = 0;
    HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    d.resident_blocks = std::min<uint32_t>((uint32_t)std::max(cus, 1) * BLOCKS_PER_CU, noalloc::MAX_BLOCKS);
    unsigned char *q = d.ptr;
    uint4 *enc = reinterpret_cast<uint4 *>(q + noalloc::OFF_ENC);
    uint32_t *sig = reinterpret_cast<uint32_t *>(q + noalloc::OFF_SIG);
    uint8_t *flags = q + noalloc::OFF_FLAGS;
    uint32_t *rows0 = reinterpret_cast<uint32_t *>(q + noalloc::OFF_ROWS0);
    uint32_t *rows1 = reinterpret_cast<uint32_t *>(q + noalloc::OFF_ROWS1);
    uint4 *renc0 = reinterpret_cast<uint4 *>(q + noalloc::OFF_RENC0);
    uint4 *renc1 = reinterpret_cast<uint4 *>(q + noalloc::OFF_RENC1);
    uint32_t *counts = reinterpret_cast<uint32_t *>(q + noalloc::OFF_COUNTS);
    // the row lists must read as zero beyond their ends (lanes without a row read entry 0 of a list)
    const uint32_t list_words = (uint32_t)((noalloc::OFF_COUNTS - noalloc::OFF_ROWS0) / 4);
    hipLaunchKernelGGL(k_clear_words, dim3((list_words + 255) / 256), dim3(256), 0, S.stream, rows0, list_words);
    hipLaunchKernelGGL(k_build_rows, dim3((N_DFROWS + 255) / 256), dim3(256), 0, S.stream, enc, sig);
    hipLaunchKernelGGL(k_prune_rows, dim3((ROWS_PER_GROUP + 255) / 256, N_GROUPS), dim3(256), 0, S.stream, sig, flags);
    hipLaunchKernelGGL(k_compact_rows, dim3(8), dim3(1024), 0, S.stream, flags, enc, rows0, rows1, renc0, renc1, counts);
    HIP_TRY(hipGetLastError());
    const int rc = read_offline(counts, rows1, d.counts);
    if (rc) return rc;
    d.built = true;
    return MMEE_OK;
}

}  // namespace
}  // namespace mmee

using namespace mmee;

extern "C" {

int mmee_chain_space_size(const mmee_chain *w, const mmee_hw *hw, uint64_t *out)
{
    if (!out) return MMEE_EINVAL;
    Plan p;
    int rc = make_plan(w, hw, p);
    if (rc) return rc;
    *out = p.space;
    return MMEE_OK;
}

int mmee_set_stream(void *hip_stream)
{
    std::lock_guard<std::mutex> guard(g_lock);
    if (S.ready) { HIP_TRY(hipStreamSynchronize(S.stream)); }
    S.stream = (hipStream_t)hip_stream;
    return MMEE_OK;
}

int mmee_offline_stats(mmee_row_stats *out)
{
    if (!out) return MMEE_EINVAL;
    std::lock_guard<std::mutex> guard(g_lock);
    int rc = ensure_ready();
    if (rc) return rc;
    for (int g = 0; g < 4; ++g) {
        out->rows_total[g] = ROWS_PER_GROUP;
        out->rows_valid[g] = S.counts[0][g];
        out->rows_kept[g] = S.counts[1][g];
    }
    return MMEE_OK;
}

int mmee_offline_rows(uint32_t group, uint32_t which, uint32_t *rows_out, uint32_t capacity, uint32_t *n_rows)
{
    if (group >= N_GROUPS || which > 1 || !n_rows || (capacity && !rows_out)) return MMEE_EINVAL;
    std::lock_guard<std::mutex> guard(g_lock);
    int rc = ensure_ready();
    if (rc) return rc;
    const uint32_t n = S.counts[which][group];
    *n_rows = n;
    const uint32_t take = std::min(n, capacity);
    if (take) {
        HIP_TRY(hipMemcpyAsync(rows_out, S.rows[which] + (size_t)group * ROWS_PER_GROUP, sizeof(uint32_t) * take,
                               hipMemcpyDeviceToHost, S.stream));
        HIP_TRY(hipStreamSynchronize(S.stream));
        for (uint32_t a = 0; a < take; ++a) rows_out[a] -= group * ROWS_PER_GROUP;   // number inside the group
    }
    return n > capacity ? MMEE_EOVERFLOW : MMEE_OK;
}

static constexpr uint64_t DECODE_SHORT = 4096;

int mmee_chain_decode(const mmee_chain *w, const mmee_hw *hw, const uint64_t *idx, uint64_t n, mmee_mapping *out)
{
    if (n && (!idx || !out)) return MMEE_EINVAL;
    Plan p;
    int rc = make_plan(w, hw, p);
    if (rc) return rc;
    for (uint64_t a = 0; a < n; ++a)
        if (idx[a] >= p.space) return MMEE_ERANGE;
    if (!n) return MMEE_OK;
    std::lock_guard<std::mutex> guard(g_lock);
    rc = ensure_ready();
    if (rc) return rc;
    if (n <= DECODE_SHORT) {
        // (two allocations, two copies and two frees were 17 us more per call of sixteen indices)
        HIP_TRY(ensure_pinned(HipPinned{}, S.decode, (sizeof(mmee_mapping) + sizeof(uint64_t)) * DECODE_SHORT));
        constexpr size_t OUT = sizeof(uint64_t) * DECODE_SHORT;
        std::memcpy(S.decode.host, idx, sizeof(uint64_t) * n);
        hipLaunchKernelGGL(k_decode, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, S.stream, p.dv, p.mc.T,
                           reinterpret_cast<const uint64_t *>(S.decode.map), n, reinterpret_cast<mmee_mapping *>(S.decode.map + OUT));
        HIP_TRY(hipGetLastError());
        HIP_TRY(hipStreamSynchronize(S.stream));
        std::memcpy(out, S.decode.host + OUT, sizeof(mmee_mapping) * n);
        return MMEE_OK;
    }
    uint64_t *d_idx = nullptr;
    mmee_mapping *d_out = nullptr;
    HIP_TRY(hipMalloc(&d_idx, sizeof(uint64_t) * n));
    if (hipMalloc(&d_out, sizeof(mmee_mapping) * n) != hipSuccess) { (void)hipFree(d_idx); return MMEE_EDEVICE; }
    hipError_t e = hipMemcpyAsync(d_idx, idx, sizeof(uint64_t) * n, hipMemcpyHostToDevice, S.stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_decode, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, S.stream, p.dv, p.mc.T, d_idx, n,
                           d_out);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, sizeof(mmee_mapping) * n, hipMemcpyDeviceToHost, S.stream);
    if (e == hipSuccess) e = hipStreamSynchronize(S.stream);
    (void)hipFree(d_idx); (void)hipFree(d_out);
    if (e != hipSuccess) {
        std::snprintf(g_last_error, sizeof(g_last_error), "mmee_decode: %s", hipGetErrorString(e));
        return MMEE_EDEVICE;
    }
    return MMEE_OK;
}

int mmee_chain_eval_batch(const mmee_chain *w, const mmee_hw *hw, uint64_t first_idx, uint64_t n,
                          mmee_cost *out_costs)
{
    Plan p;
    int rc = make_plan(w, hw, p);
    if (rc) return rc;
    if (first_idx > p.space || n > p.space - first_idx) return MMEE_ERANGE;
    if (!n) return MMEE_OK;
    if (!out_costs) return MMEE_EINVAL;
    std::lock_guard<std::mutex> guard(g_lock);
    rc = ensure_ready();
    if (rc) return rc;
    rc = ensure_tilings(p.mc.tpad);
    if (rc) return rc;
    Bufs tables;
    tables.btab = S.btab; tables.ctab_s = S.ctab_s; tables.ctab_e = S.ctab_e;
    rc = launch_tilings(p, p.mc, tables);
    if (rc) return rc;

    hipPointerAttribute_t attr;
    bool on_device = false;
    if (hipPointerGetAttributes(&attr, out_costs) == hipSuccess) on_device = attr.type == hipMemoryTypeDevice;
    else (void)hipGetLastError();

    EvalArgs ea;
    ea.enc = S.enc; ea.btab = S.btab; ea.ctab_e = S.ctab_e; ea.mc = p.mc;
    // records per launch: 1 GiB of staging for host output, one launch (grid limit) for device output;
    // whole 4 KiB pages of 64 records each
    const uint64_t CHUNK = on_device ? (1ull << 30) : (1ull << 24);
    if (!on_device) {
        size_t need = (size_t)std::min<uint64_t>(n, CHUNK) * sizeof(mmee_cost);
        if (need > S.eval_cap) {
            if (S.eval_dev) { HIP_TRY(hipStreamSynchronize(S.stream)); (void)hipFree(S.eval_dev); }
            S.eval_dev = nullptr; S.eval_cap = 0;
            HIP_TRY(hipMalloc(&S.eval_dev, need));
            S.eval_cap = need;
        }
    }
    for (uint64_t done = 0; done < n; done += CHUNK) {
        const uint64_t cnt = std::min<uint64_t>(CHUNK, n - done);
        const uint64_t n_pages = (cnt + 63) / 64;
        // blocks come in groups of eight that share 32 neighbouring pages
        const uint64_t nblocks = (n_pages + 31) / 32 * 8;
        if (nblocks > 0x7fffffffull) return MMEE_EINVAL;
        v4u *dst = on_device ? reinterpret_cast<v4u *>(out_costs + done) : reinterpret_cast<v4u *>(S.eval_dev);
        const uint64_t first = first_idx + done;
        hipLaunchKernelGGL(k_eval_batch, dim3((uint32_t)nblocks), dim3(256), 0, S.stream, ea, (uint32_t)(first / p.T),
                           (uint32_t)(first % p.T), (uint32_t)cnt, (uint32_t)n_pages, dst);
        HIP_TRY(hipGetLastError());
        if (!on_device) {
            HIP_TRY(hipMemcpyAsync(out_costs + done, S.eval_dev, cnt * sizeof(mmee_cost), hipMemcpyDeviceToHost,
                                   S.stream));
            HIP_TRY(hipStreamSynchronize(S.stream));
        }
    }
    HIP_TRY(hipStreamSynchronize(S.stream));
    return MMEE_OK;
}

int mmee_chain_search_many(const mmee_chain *w, const mmee_hw *hw, const int *objectives, uint32_t count,
                           uint32_t flags, mmee_result *out, int *rc_out)
{
    if (!count) return MMEE_OK;
    if (!w || !hw || !objectives || !out) return MMEE_EINVAL;
    if (flags & ~(uint32_t)(MMEE_SEARCH_EXHAUSTIVE | MMEE_SEARCH_ORDERED_SUM)) return MMEE_EINVAL;
    std::lock_guard<std::mutex> guard(g_lock);
    const double t_start = now_seconds();
    int rc = ensure_ready();
    if (rc) return rc;

    // group neighbouring entries that describe the same problem into one pass
    struct Stretch { uint32_t first, n; int mask; };
    struct Pass {
        uint32_t first, n; int mask; Plan plan; int rc; uint64_t evaluated; bool unproven;
        Pass(const Stretch &st) : first(st.first), n(st.n), mask(st.mask), evaluated(0), unproven(false) {}
    };
    std::vector<Stretch> stretches;
    std::vector<int> codes(count, MMEE_OK);
    for (uint32_t a = 0; a < count;) {
        Stretch st{a, 0, 0};
        uint32_t b = a;
        while (b < count && same_problem(w[a], hw[a], w[b], hw[b])) {
            int o = objectives[b];
            if (o < 0 || o >= N_OBJ) codes[b] = MMEE_EINVAL;     // this entry only; its neighbours still run
            else if (st.mask & (1 << o)) break;      // same objective twice: start a new pass
            else st.mask |= 1 << o;
            ++b; ++st.n;
        }
        if (st.n == 0) { st.n = 1; b = a + 1; }
        stretches.push_back(st);
        a = b;
    }
    // (a plan holds its divisor lists, 4 KiB: made in place, once their number is known)
    std::vector<Pass> passes;
    passes.reserve(stretches.size());
    for (const Stretch &st : stretches) {
        passes.emplace_back(st);
        Pass &ps = passes.back();
        ps.rc = make_plan(w + st.first, hw + st.first, ps.plan);
        if (ps.mask == 0 && !ps.rc) ps.rc = MMEE_EINVAL;         // no valid objective in the group
    }
    rc = ensure_slots(passes.size());
    if (rc) return rc;
    // per pass: whether it ran in the round under way, whose events bracket its launches, what they took (apart from the passes,
    // which lie 4 KiB from one another)
    struct PassTime { size_t ev_slot = 0; double device_seconds = 0.0; bool ran = false; };
    std::vector<PassTime> times(passes.size());
    // Pruned searches share launches: problems on few shapes the tables and the row side too (enqueue_pruned), others
    // the launch only (enqueue_batches), where the kernel is built for their key set.  Everything else goes
    // problem by problem.  `round_flags` adds MMEE_SEARCH_ORDERED_SUM on the second round, which repeats what the
    // first could not prove and leaves the other problems' device times alone: a round's times are taken at its end.
    auto run_round = [&](uint32_t round_flags, bool only_unproven) -> int {
        bool signalled = false;                              // the stream holds one search, of the pass below, and it says when it is done
        size_t signalled_pass = 0;
        bool others = false;                                 // anything beside the batched searches and that one in the stream
        std::vector<PrunedEntry> pruned;
        std::vector<uint32_t> order;
        std::vector<PrunedSlice> slices;                     // the groups that share more than launches
        std::vector<char> in_slice(passes.size(), 0);
        size_t slice_ev = 0;
        std::vector<BatchEntry> batch;
        std::vector<size_t> batch_pass;
        auto takes_part = [&](const Pass &ps) { return ps.rc == MMEE_OK && (!only_unproven || ps.unproven); };
        if (!(round_flags & MMEE_SEARCH_EXHAUSTIVE) && passes.size() > 1) {
            for (size_t s = 0; s < passes.size(); ++s)
                if (takes_part(passes[s])) pruned.push_back(PrunedEntry{&passes[s].plan, passes[s].mask, (uint32_t)s});
            pruned_slices(pruned, order, slices);
            keep_shared(pruned, order, slices);
            for (const PrunedSlice &sl : slices)
                for (uint32_t k = sl.lo; k < sl.hi; ++k) in_slice[pruned[order[k]].slot] = 1;
            if (!slices.empty()) slice_ev = pruned[order[slices[0].lo]].slot;
        }
        for (size_t s = 0; s < passes.size(); ++s) {
            Pass &ps = passes[s];
            times[s].ran = takes_part(ps);
            if (!times[s].ran) continue;
            times[s].ev_slot = s;
            if (in_slice[s]) {
                times[s].ev_slot = slice_ev;
                ps.evaluated = kept_row_count() * ps.plan.T * 9ull;
                ps.unproven = false;
            } else if (!(round_flags & MMEE_SEARCH_EXHAUSTIVE) && batch_mask(ps.mask)) {
                BatchEntry e;
                e.plan = &ps.plan; e.mask = ps.mask; e.slot = s; e.unproven = false; e.evaluated = 0;
                batch.push_back(e);
                batch_pass.push_back(s);
            } else {
                bool unproven = false;
                ps.rc = enqueue_search(ps.plan, ps.mask, round_flags, s, &ps.evaluated, nullptr, true, false,
                                       only_unproven ? nullptr : &unproven, passes.size() == 1 ? &signalled : nullptr);
                ps.unproven = unproven;
                signalled_pass = s;
                others = others || !signalled;
            }
        }
        if (!slices.empty()) {
            others = true;
            const int src = enqueue_pruned(pruned, order, slices, slice_ev);
            for (size_t s = 0; s < passes.size(); ++s)
                if (in_slice[s]) passes[s].rc = src;
        }
        if (!batch.empty()) {
            int brc = enqueue_batches(batch, round_flags, batch_pass[0], signalled);
            if (brc) signalled = false;
            signalled_pass = batch_pass[0];
            for (size_t k = 0; k < batch.size(); ++k) {
                Pass &ps = passes[batch_pass[k]];
                ps.rc = brc;
                ps.evaluated = batch[k].evaluated;
                ps.unproven = !only_unproven && batch[k].unproven;
                times[batch_pass[k]].ev_slot = batch_pass[0];
            }
        }
        double signalled_seconds = 0.0;
        if (!signalled || others) HIP_TRY(hipStreamSynchronize(S.stream));
        if (signalled) {
            const int wrc = wait_signalled(passes[signalled_pass].mask, signalled_seconds);
            if (wrc) return wrc;
        }
        size_t timed = (size_t)-1;
        double timed_seconds = 0.0;
        for (size_t s = 0; s < passes.size(); ++s) {
            PassTime &t = times[s];
            if (!t.ran) continue;
            if (signalled && s == signalled_pass) {          // (no events were recorded)
                t.device_seconds = signalled_seconds;
                continue;
            }
            if (t.ev_slot != timed) {                        // (asked for once, not for each of hundreds that shared them)
                if (passes[s].rc != MMEE_OK) continue;
                float ms = 0.f;
                (void)hipEventElapsedTime(&ms, S.events[2 * t.ev_slot], S.events[2 * t.ev_slot + 1]);
                timed = t.ev_slot;
                timed_seconds = ms * 1e-3;
            }
            t.device_seconds = timed_seconds;
        }
        return MMEE_OK;
    };
    rc = run_round(flags, false);
    if (rc) return rc;
    // a regrouped sum taken on trust (pass_constants) stands only if the energies found prove it
    {
        bool again = false;
        for (size_t s = 0; s < passes.size(); ++s) {
            Pass &ps = passes[s];
            if (ps.rc != MMEE_OK || !ps.unproven) continue;
            bool proven = true;
            for (int o : {MMEE_OBJ_ENERGY, MMEE_OBJ_LATENCY_THEN_ENERGY}) {
                if (!(ps.mask & (1 << o))) continue;
                const FinalRecord &fr = S.final_host[N_OBJ * s + o];
                double energy;
                std::memcpy(&energy, &fr.cost[5], sizeof(double));          // mmee_cost::energy_pj
                if (fr.key.p < INFINITY && !(energy < REGROUP_PROOF_LIMIT)) proven = false;
            }
            ps.unproven = !proven;
            again = again || !proven;
        }
        if (again) {
            rc = run_round(flags | MMEE_SEARCH_ORDERED_SUM, true);
            if (rc) return rc;
        }
    }
    const double seconds = now_seconds() - t_start;
    int first_bad = MMEE_OK;
    for (size_t s = 0; s < passes.size(); ++s) {
        Pass &ps = passes[s];
        for (uint32_t a = ps.first; a < ps.first + ps.n; ++a) {
            int code = codes[a] ? codes[a] : ps.rc;
            if (code == MMEE_OK)
                code = unpack_result(ps.plan, s, objectives[a], ps.evaluated, seconds, times[s].device_seconds, out + a);
            else
                std::memset(out + a, 0, sizeof(mmee_result));
            if (rc_out) rc_out[a] = code;
            if (code && !first_bad) first_bad = code;
        }
    }
    return first_bad;
}

int mmee_chain_search_multi(const mmee_chain *w, const mmee_hw *hw, const int *objectives, uint32_t n_obj,
                            uint32_t flags, mmee_result *out)
{
    if (!w || !hw || !objectives || !out || n_obj < 1 || n_obj > N_OBJ) return MMEE_EINVAL;
    int seen = 0;
    for (uint32_t a = 0; a < n_obj; ++a) {
        if (objectives[a] < 0 || objectives[a] >= N_OBJ || (seen & (1 << objectives[a]))) return MMEE_EINVAL;
        seen |= 1 << objectives[a];
    }
    mmee_chain ws[N_OBJ] = {*w, *w, *w, *w};
    mmee_hw hs[N_OBJ] = {*hw, *hw, *hw, *hw};
    return mmee_chain_search_many(ws, hs, objectives, n_obj, flags, out, nullptr);
}

// A front.  Over the kept rows of a problem that is not too large, in two launches (fronts.h); else a walk along it.
// Energy-latency (Sec. VII-E): by ascending latency, each step the
// latency-then-energy optimum among the candidates whose energy is strictly below the previous
// point's.  Buffer size / DRAM access (Sec. VII-C): by ascending buffer size, each step the
// (size, traffic)-smallest dataflow whose traffic is strictly below the previous point's.
static int walk_front(const mmee_chain *w, const mmee_hw *hw, bool bs_da, uint32_t flags, mmee_result *out,
               uint32_t capacity, uint32_t *n_points)
{
    if (!w || !hw || !out || !n_points || !capacity) return MMEE_EINVAL;
    if (flags & ~(uint32_t)(MMEE_SEARCH_EXHAUSTIVE | MMEE_SEARCH_ORDERED_SUM)) return MMEE_EINVAL;
    *n_points = 0;
    Plan p;
    int rc = make_plan(w, hw, p);
    if (rc) return rc;
    std::lock_guard<std::mutex> guard(g_lock);
    const double t_start = now_seconds();
    rc = ensure_ready();
    if (rc) return rc;
    rc = ensure_slots(1);
    if (rc) return rc;
    if (!(flags & MMEE_SEARCH_EXHAUSTIVE) && (p.T + PRUNED_TC - 1) / PRUNED_TC <= FRONT_CHUNKS) {
        rc = enqueue_front(p, bs_da, capacity);
        if (rc) return rc;
        double ksec = 0.0;
        rc = wait_signalled(1, ksec);
        if (rc) return rc;
        S.front_clean = true;
        const FinalRecord *records = reinterpret_cast<const FinalRecord *>(S.front.host);
        const uint32_t *out_n = reinterpret_cast<const uint32_t *>(S.front.host + FRONT_N_AT), n = out_n[0];
        g_front_way = out_n[1];
        if (n != TOO_MANY) {
            const bool fits = n <= capacity;
            // counted as the walk counts: one pass over the candidates per point, and the one that finds nothing more
            const uint64_t formed = fits ? kept_row_count() * p.T * (bs_da ? 1ull : 9ull) * ((uint64_t)n + 1) : 0;
            const double seconds = fits ? now_seconds() - t_start : 0.0;
            *n_points = std::min(n, capacity);
            for (uint32_t k = 0; k < *n_points; ++k) (void)unpack_record(p, records[k], formed, seconds, fits ? ksec : 0.0, out + k);
            return !fits ? MMEE_EOVERFLOW : (n ? MMEE_OK : MMEE_ENOFEASIBLE);
        }
    }
    ++g_front_walks;
    double limit = INFINITY, ksec = 0.0;
    uint64_t evaluated = 0;
    for (uint32_t k = 0;; ++k) {
        uint64_t ev = 0;
        bool unproven = false;
        rc = enqueue_search(p, bs_da ? 1 : 4, flags, 0, &ev, &limit, k == 0, bs_da, &unproven);
        if (rc) return rc;
        HIP_TRY(hipStreamSynchronize(S.stream));
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, S.events[0], S.events[1]);
        ksec += ms * 1e-3;
        evaluated += ev;
        mmee_result r;
        rc = unpack_result(p, 0, bs_da ? 0 : MMEE_OBJ_LATENCY_THEN_ENERGY, 0, 0.0, 0.0, &r);
        if (rc == MMEE_ENOFEASIBLE) break;          // nothing below the bound is left: the front is complete
        if (unproven && !(r.cost.energy_pj < REGROUP_PROOF_LIMIT)) {
            // the regrouped sum was taken on trust and this point does not prove it (energies fall
            // along the front, so only its first point can): start again, term by term
            flags |= MMEE_SEARCH_ORDERED_SUM;
            limit = INFINITY;
            *n_points = 0;
            k = (uint32_t)-1;
            continue;
        }
        if (k == capacity) return MMEE_EOVERFLOW;   // out holds the first `capacity` points
        out[k] = r;
        *n_points = k + 1;
        limit = bs_da ? p.mc.BH * (double)r.cost.da_words : r.cost.energy_pj;
    }
    const double seconds = now_seconds() - t_start;
    for (uint32_t k = 0; k < *n_points; ++k) {
        out[k].evaluated = evaluated; out[k].seconds = seconds; out[k].kernel_seconds = ksec;
    }
    return *n_points ? MMEE_OK : MMEE_ENOFEASIBLE;
}

// Not part of the interface: which way the fronts took, for tests.
uint64_t mmee_front_walks(void)
{
    std::lock_guard<std::mutex> guard(g_lock);
    return g_front_walks;
}
uint32_t mmee_front_way(void)
{
    std::lock_guard<std::mutex> guard(g_lock);
    return g_front_way;
}

int mmee_chain_pareto(const mmee_chain *w, const mmee_hw *hw, uint32_t flags, mmee_result *out, uint32_t capacity,
                      uint32_t *n_points)
{
    return walk_front(w, hw, false, flags, out, capacity, n_points);
}

int mmee_chain_front_bs_da(const mmee_chain *w, const mmee_hw *hw, uint32_t flags, mmee_result *out,
                           uint32_t capacity, uint32_t *n_points)
{
    return walk_front(w, hw, true, flags, out, capacity, n_points);
}

// ---- attention workloads: the chain I = L = N, K = J = d, batch = B*H --------------------------

int mmee_pareto(const mmee_workload *w, const mmee_hw *hw, uint32_t flags, mmee_result *out, uint32_t capacity,
                uint32_t *n_points)
{
    mmee_chain c;
    int rc = chain_of(w, c);
    return rc ? rc : mmee_chain_pareto(&c, hw, flags, out, capacity, n_points);
}

int mmee_front_bs_da(const mmee_workload *w, const mmee_hw *hw, uint32_t flags, mmee_result *out,
                     uint32_t capacity, uint32_t *n_points)
{
    mmee_chain c;
    int rc = chain_of(w, c);
    return rc ? rc : mmee_chain_front_bs_da(&c, hw, flags, out, capacity, n_points);
}

int mmee_chain_energy_regrouped(const mmee_chain *w, const mmee_hw *hw, uint32_t flags, int *out)
{
    if (!out || (flags & ~(uint32_t)(MMEE_SEARCH_EXHAUSTIVE | MMEE_SEARCH_ORDERED_SUM))) return MMEE_EINVAL;
    Plan p;
    int rc = make_plan(w, hw, p);
    if (rc) return rc;
    *out = (int)pass_constants(p, flags).regroup;
    return MMEE_OK;
}

int mmee_energy_regrouped(const mmee_workload *w, const mmee_hw *hw, uint32_t flags, int *out)
{
    mmee_chain c;
    int rc = chain_of(w, c);
    return rc ? rc : mmee_chain_energy_regrouped(&c, hw, flags, out);
}

int mmee_space_size(const mmee_workload *w, const mmee_hw *hw, uint64_t *out)
{
    mmee_chain c;
    int rc = chain_of(w, c);
    return rc ? rc : mmee_chain_space_size(&c, hw, out);
}

int mmee_decode(const mmee_workload *w, const mmee_hw *hw, const uint64_t *idx, uint64_t n, mmee_mapping *out)
{
    mmee_chain c;
    int rc = chain_of(w, c);
    return rc ? rc : mmee_chain_decode(&c, hw, idx, n, out);
}

int mmee_eval_batch(const mmee_workload *w, const mmee_hw *hw, uint64_t first_idx, uint64_t n, mmee_cost *out_costs)
{
    mmee_chain c;
    int rc = chain_of(w, c);
    return rc ? rc : mmee_chain_eval_batch(&c, hw, first_idx, n, out_costs);
}

int mmee_search_many(const mmee_workload *w, const mmee_hw *hw, const int *objectives, uint32_t count,
                     uint32_t flags, mmee_result *out, int *rc_out)
{
    if (!count) return MMEE_OK;
    if (!w || !hw || !objectives || !out) return MMEE_EINVAL;
    std::vector<mmee_chain> chains(count);
    for (uint32_t a = 0; a < count; ++a) {
        // a malformed workload becomes a malformed chain and is reported per entry
        if (chain_of(w + a, chains[a])) std::memset(&chains[a], 0, sizeof(mmee_chain));
    }
    return mmee_chain_search_many(chains.data(), hw, objectives, count, flags, out, rc_out);
}

int mmee_search_multi(const mmee_workload *w, const mmee_hw *hw, const int *objectives, uint32_t n_obj,
                      uint32_t flags, mmee_result *out)
{
    mmee_chain c;
    int rc = chain_of(w, c);
    return rc ? rc : mmee_chain_search_multi(&c, hw, objectives, n_obj, flags, out);
}

int mmee_search_ex(const mmee_workload *w, const mmee_hw *hw, int objective, uint32_t flags, mmee_result *out)
{
    return mmee_search_multi(w, hw, &objective, 1, flags, out);
}

int mmee_search(const mmee_workload *w, const mmee_hw *hw, int objective, mmee_result *out)
{
    return mmee_search_ex(w, hw, objective, MMEE_SEARCH_PRUNED, out);
}

int mmee_search_noalloc(const mmee_workload *w, const mmee_hw *hw, int objective, uint32_t flags,
                        mmee_result *out_dev)
{
    if (!out_dev || objective < 0 || objective >= N_OBJ) return MMEE_EINVAL;
    if (flags & ~(uint32_t)(MMEE_SEARCH_EXHAUSTIVE | MMEE_SEARCH_ORDERED_SUM)) return MMEE_EINVAL;
    mmee_chain c;
    int rc = chain_of(w, c);
    if (rc) return rc;
    Plan p;
    rc = make_plan(&c, hw, p);
    if (rc) return rc;
    if (p.mc.tpad > noalloc::MAX_TPAD) {
        std::snprintf(g_last_error, sizeof(g_last_error),
                      "mmee_search_noalloc: %llu tilings, the fixed scratch holds %u; use mmee_search_ex",
                      (unsigned long long)p.T, noalloc::MAX_TPAD);
        return MMEE_ETOOBIG;
    }
    std::lock_guard<std::mutex> guard(g_lock);
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        std::snprintf(g_last_error, sizeof(g_last_error), "no HIP device");
        return MMEE_EDEVICE;
    }
    NoAllocDevice *d = nullptr;
    rc = noalloc_setup(dev, d);
    if (rc) return rc;
    unsigned char *q = d->ptr;
    Bufs b;
    b.enc = reinterpret_cast<const uint4 *>(q + noalloc::OFF_ENC);
    b.rows[0] = reinterpret_cast<const uint32_t *>(q + noalloc::OFF_ROWS0);
    b.rows[1] = reinterpret_cast<const uint32_t *>(q + noalloc::OFF_ROWS1);
    b.row_enc[0] = reinterpret_cast<const uint4 *>(q + noalloc::OFF_RENC0);
    b.row_enc[1] = reinterpret_cast<const uint4 *>(q + noalloc::OFF_RENC1);
    for (int k = 0; k < 2; ++k)
        for (int g = 0; g < 4; ++g) b.counts[k][g] = d->counts[k][g];
    b.cls_dev = nullptr;                       // row-per-lane kernel for every key
    b.btab = reinterpret_cast<double *>(q + noalloc::OFF_BTAB);
    b.ctab_s = reinterpret_cast<double *>(q + noalloc::OFF_CTAB_S);
    b.ctab_e = reinterpret_cast<uint64_t *>(q + noalloc::OFF_CTAB_E);
    b.partials = reinterpret_cast<Key *>(q + noalloc::OFF_PARTIALS);
    b.partials_cap = noalloc::MAX_BLOCKS;
    b.ticket = reinterpret_cast<uint32_t *>(q + noalloc::OFF_TICKET);
    b.key_dev = reinterpret_cast<Key *>(q + noalloc::OFF_KEYS);
    b.final_dev = reinterpret_cast<FinalRecord *>(q + noalloc::OFF_FINAL);
    b.dv_dev = reinterpret_cast<DivTable *>(q + noalloc::OFF_DV);
    b.resident_blocks = d->resident_blocks;
    if (!(flags & MMEE_SEARCH_EXHAUSTIVE)) {
        // The kept rows: no tables, no counters to clear, the finish writes the result record; 16384 tilings have at most
        // 240 + 68 + 1 + 1 divisors and 512 items.
        BatchArgs a;
        std::memset(&a, 0, sizeof(a));
        const uint32_t chunks = (uint32_t)((p.T + PRUNED_TC - 1) / PRUNED_TC), split = batch_split(chunks, b.resident_blocks);
        if (list_length(p.dv) > (uint32_t)BATCH_INLINE_DIVS || chunks * split > noalloc::MAX_BLOCKS) return MMEE_ETOOBIG;
        // the regrouped energy sum only where it is provably exact: nothing is read back to check it
        const ModelConst mc = pass_constants(p, flags, 1 << objective);
        fill_batch_head(a.inl.h, a.inl.list, p, mc, 0, 0, split);
        a.inl.firsts[0] = 0; a.inl.firsts[1] = a.inl.h.n_work;
        a.inl.on = 1;
        a.n_prob = 1; a.n_items = a.inl.h.n_work;
        a.enc = b.enc;
        set_batch_tasks(a, split);
        a.item_keys = b.partials;
        a.packed = out_dev; a.space = p.space;
        a.evaluated = ((uint64_t)d->counts[1][0] + d->counts[1][1] + d->counts[1][2] + d->counts[1][3]) * p.T * 9ull;
        const dim3 grid(std::min(a.n_items, b.resident_blocks));
        a.ticket = b.ticket + 2 + noalloc::TICKETS * (grid.x - 1) + d->tickets++ % noalloc::TICKETS;
        a.per_block = a.n_items / grid.x; a.extra = a.n_items % grid.x;
        return launch_batch(1 << objective, p.exact_k, mc.regroup != 0, grid, a);
    }
    // the finish ticket and the work counter must start at zero whatever the last call left
    hipLaunchKernelGGL(k_clear_words, dim3(1), dim3(64), 0, S.stream, b.ticket, 2u);
    uint64_t evaluated = 0;
    // the regrouped energy sum only where it is provably exact: nothing is read back to check it
    rc = enqueue_search_in(b, p, 1 << objective, flags, &evaluated);
    if (rc) return rc;
    hipLaunchKernelGGL(k_pack_result, dim3(1), dim3(64), 0, S.stream, b.final_dev + objective, p.space, evaluated,
                       out_dev);
    HIP_TRY(hipGetLastError());
    return MMEE_OK;
}

void mmee_shutdown(void)
{
    std::lock_guard<std::mutex> guard(g_lock);
    if (S.ready || S.btab || S.partials) (void)hipStreamSynchronize(S.stream);
    (void)hipFree(S.enc); (void)hipFree(S.sig); (void)hipFree(S.flags); (void)hipFree(S.cls_dev); (void)hipFree(S.key_dev);
    (void)hipFree(S.rows[0]); (void)hipFree(S.rows[1]); (void)hipFree(S.counts_dev);
    (void)hipFree(S.row_enc[0]); (void)hipFree(S.row_enc[1]);
    (void)hipFree(S.btab); (void)hipFree(S.ctab_s); (void)hipFree(S.ctab_e);
    (void)hipFree(S.partials); (void)hipFree(S.ticket); (void)hipFree(S.hints);
    (void)hipFree(S.dv_dev); (void)hipFree(S.eval_dev);
    if (S.final_host) (void)hipHostFree(S.final_host);
    if (S.batch_host) (void)hipHostFree(S.batch_host);
    (void)hipFree(S.batch_dev); (void)hipFree(S.item_keys);
    if (S.desc_host) (void)hipHostFree(S.desc_host);
    if (S.decode.host) (void)hipHostFree(S.decode.host);
    (void)hipFree(S.front_points); (void)hipFree(S.front_stairs); (void)hipFree(S.front_counts);
    if (S.front.host) (void)hipHostFree(S.front.host);
    if (S.done.host) (void)hipHostFree(S.done.host);
    (void)hipFree(S.call_begin);
    (void)hipFree(S.desc_dev); (void)hipFree(S.block_records); (void)hipFree(S.pruned_hints);
    for (hipEvent_t e : S.events) (void)hipEventDestroy(e);
    hipStream_t keep = S.stream;
    S = State();
    S.stream = keep;
}

const char *mmee_strerror(int code)
{
    switch (code) {
    case MMEE_OK: return "ok";
    case MMEE_EINVAL: return "invalid argument";
    case MMEE_ERANGE: return "candidate index out of range";
    case MMEE_ENOFEASIBLE: return "no feasible candidate";
    case MMEE_EDEVICE: return g_last_error[0] ? g_last_error : "HIP device error";
    case MMEE_EOVERFLOW: return "the Pareto front has more points than the caller made room for";
    case MMEE_ETOOBIG: return g_last_error[0] ? g_last_error : "the problem exceeds the fixed scratch of mmee_search_noalloc";
    default: return "unknown error";
    }
}

}  // extern "C"
