// C-ABI boundary of the CodedReduce hot path: plan (host), workspace binding, and the three stages of one iteration.
#include "codedreduce.h"

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "gc_design.h"
#include "kernels.h"
#include "latency_model.h"
#include "testing.h"
#include "tree_plan.h"

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string &msg)
{
    g_last_error = msg;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    return fail(CR_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define CR_HIP(call)                                        \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return hip_fail(e_, #call);   \
    } while (0)

constexpr uint64_t kDefaultSeed = 190201981ull;
constexpr int kProgramSlots = 16;     // encode programs the workspace holds at once: one host-to-device copy serves that many steps
constexpr int kStagingHalves = 2;     // pinned staging is two such batches, so the host fills one while the other is being copied
constexpr size_t kMaxSamples = size_t(1) << 16;

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// The pages of the library's table pool that plans hold, per device.  A plan takes a run of them when it is first bound and gives it
// back when it is destroyed, after the last launch that reads it.
class TablePages {
    static constexpr int kPages = cr::kTablePoolBytes / cr::kTablePageBytes;
    std::mutex mutex_;
    bool held_[cr::kMaxDevices][kPages] = {};

public:
    int take(int device, int pages)                      // the first page of the run, or -1: none is free
    {
        const std::lock_guard<std::mutex> lock(mutex_);
        if (device < 0 || device >= cr::kMaxDevices) return -1;
        for (int run = 0, at = 0; at < kPages; ++at) {
            run = held_[device][at] ? 0 : run + 1;
            if (run < pages) continue;
            const int first = at - pages + 1;
            std::fill(&held_[device][first], &held_[device][first] + pages, true);
            return first;
        }
        return -1;
    }
    void give(int device, int first, int pages)
    {
        const std::lock_guard<std::mutex> lock(mutex_);
        std::fill(&held_[device][first], &held_[device][first] + pages, false);
    }
};
TablePages g_table_pages;

struct TimedLaunch {
    int kernel;
    hipEvent_t start, stop;
};

}  // namespace

struct cr_plan_s {
    // problem
    int L = 0, n = 0, s = 0, model = 0, x_dtype = 0;
    int64_t m = 0, d = 0;
    cr::Tree tree;
    cr::GcCode code;
    std::vector<cr::WeightedSet> own;
    std::vector<cr::Slab> slabs;
    std::vector<int32_t> node_slab_begin;          // N+1
    std::vector<double> slab_coef;
    cr::TreeShape shape = {};
    std::unique_ptr<cr::TreeArguments> tree_arguments;                     // trees that the tree kernels take
    int64_t row_visits = 0, min_rows = 0, max_rows = 0;
    int64_t max_holders = 1;                       // most workers that hold a row: (s+1)^L, capped at 64
    mutable std::unordered_map<uint64_t, std::vector<double>> row_cache;   // padded straggler bitmask -> decode row

    // stage-1 split
    bool rows_once = false;                            // every row once (`work`), or every holder's rows (`split`)
    const cr::OnceVariant *once = nullptr;             // the stage-1 kernel in use; null: the two-pass path of wide rows
    const cr::Stage1Variant *variant = nullptr;        // ... of every holder's rows; the same
    const cr::OnceVariant *once_variant = nullptr;     // what exists for (x_dtype, d)
    const cr::Stage1Variant *variant_regs = nullptr;
    int cell_holders = 0;            // holders a workgroup of the shared-cells split serves; 0: no such split for this type and width
    cr::OnceWork work;               // `rows_once`: the runs and sums behind the split
    const cr::OnceVariant *wide_variant = nullptr;     // wide rows in one pass; null: two passes, or
    std::unique_ptr<cr::CrewVariant> crew;             // one pass with several workgroups per row
    int patience = cr::kCrewPatience;                  // polls for what another workgroup of a crew has to say
    int units = 0;                   // compute units the wide-row launches are sized for
    bool streams = false;            // rows_once: X is read past the caches
    bool rows_as_buffers = false;    // every row starts on a 4-byte boundary and every piece has fewer than 2^31 bytes
    int split_kind = -1;                            // -1: choose from the device when the workspace is sized
    int64_t split_value = 0;
    int split_kind_used = -1;                       // what ensure_split settled on
    int64_t split_value_used = 0;
    int l2_domains = 0, unit_slots = 0;             // what the split was laid out for (0 until it is fixed)
    int l2_sharing = -1;                            // 1 / 0: workgroup ids congruent modulo l2_domains were seen (not) to share a die; -1: not checked
    cr::Split split;

    // device binding
    bool bound = false;
    hipStream_t stream = nullptr;
    char *ws = nullptr;
    size_t ws_bytes = 0;
    cr::DevPiece *d_pieces = nullptr;
    int32_t *d_team_piece_begin = nullptr;
    cr::DevRun *d_parts = nullptr, *d_runs = nullptr;
    cr::DevSum *d_sums = nullptr;
    int32_t *d_dst = nullptr;
    uint64_t *d_crew_slots = nullptr;              // `crew`: what its kernel exchanges in
    uint32_t *d_crew_state = nullptr;
    int num_sums = 0;
    int64_t rows_summed = 0;                       // by all of them
    uint32_t *d_placement = nullptr;               // kPlacementSlots words: where the workgroups of a probe launch ran
    char *d_program = nullptr;                     // kProgramSlots encode programs
    int32_t *d_node_begin = nullptr;               // slabs of every node, their coefficients: what the tree kernels read
    double *d_slab_coef = nullptr;
    bool slabs_here = false;                       // the slabs are those that stage 1 left in the workspace, beside the tables
    int pool_device = -1, pool_first = -1, pool_pages = 0;      // pages of the table pool where d_node_begin and d_slab_coef lie instead
    double *d_measures = nullptr;                  // kProgramSlots steps' sums for the convergence measures
    size_t measures_stride = 0;                    // doubles per step
    size_t program_bytes = 0;                      // size of one
    float *d_G = nullptr, *d_M = nullptr, *d_residuals = nullptr;   // d_G: the output table, slabs then partial rows; residuals: wide-row path only
    const float *G_src = nullptr;                  // slabs the encode reads: d_G or the caller's buffer
    char *h_staging = nullptr;                     // pinned, kStagingHalves * kProgramSlots * program_bytes, then a copy of the tree's tables
    hipEvent_t staging_done[kStagingHalves] = {};
    bool staging_used[kStagingHalves] = {};
    int staging_next = 0;
    cr::DecTerms dec = {};                         // what cr_decode_root does: of the last mask encoded
    // layout of the workspace (offsets in bytes)
    size_t at_pieces = 0, at_team_piece_begin = 0, at_parts = 0, at_runs = 0, at_sums = 0, at_dst = 0, at_crew_slots = 0, at_crew_state = 0, at_placement = 0, at_program = 0,
           at_node_begin = 0, at_slab_coef = 0, tables_bytes = 0, at_measures = 0, at_G = 0, at_residuals = 0, at_M = 0;
    // layout of a program block (offsets in bytes, fixed per plan)
    size_t off_slab = 0, off_level = 0, off_row = 0, off_coef = 0, off_acoef = 0, off_sub = 0, off_dec = 0;
    size_t max_terms = 0;

    std::vector<int32_t> last_send;                // N: the last step of the call at hand in which a node sends (see Stores)
    bool have_grads = false, have_messages = false;
    std::vector<char> static_program;              // host copy of the encode program of cr_aggregate_static (ordinary memory)

    // timing
    unsigned profiling = 0;                         // bit k: launches of kernel id k are bracketed by events
    std::vector<TimedLaunch> timed;
    std::vector<hipEvent_t> event_pool;
    double total_ms[CR_K_COUNT] = {};
    int64_t launches[CR_K_COUNT] = {}, bytes_sum[CR_K_COUNT] = {}, bytes_last[CR_K_COUNT] = {};
    std::vector<float> samples[CR_K_COUNT];         // duration of every timed launch since the totals were last cleared (bounded)
};

namespace {

int64_t elem_size(const cr_plan_t *p) { return p->x_dtype == CR_BF16 ? 2 : 4; }
// X is read past the caches (non-temporal hint) from the size of the last-level cache on.  Below it X may survive there from one
// iteration to the next if its lines are allowed to (200 MB read again and again: 31.0 us with plain loads, 32.6 with the hint);
// above it the hint wins either way (300 MB: 49.6 against 46.8 us, 800 MB: 136 against 118).
constexpr int64_t kStreamFromBytes = int64_t(256) << 20;
// The default splits of large data (see ensure_split)
constexpr int64_t kLargeBytes = int64_t(1) << 30;

// decode row for one group under rule "pad with the highest-index survivors"; returns CR_E_UNDECODABLE if more than s flags are set
int group_decode_row(const cr_plan_t *p, const uint8_t *flags, const double **row)
{
    uint64_t bits = 0;
    int cnt = 0;
    for (int j = 0; j < p->n; ++j)
        if (flags[j]) { bits |= 1ull << j; ++cnt; }
    if (cnt > p->s) return CR_E_UNDECODABLE;
    for (int j = p->n - 1; cnt < p->s; --j)
        if (!((bits >> j) & 1ull)) { bits |= 1ull << j; ++cnt; }
    auto it = p->row_cache.find(bits);
    if (it == p->row_cache.end()) {
        std::vector<double> a(p->n);
        if (!cr::decode_row(p->code, bits, a.data())) return fail(CR_E_INVAL, "decode row: survivor system is inconsistent");
        it = p->row_cache.emplace(bits, std::move(a)).first;
    }
    *row = it->second.data();
    return CR_OK;
}

// MI355X has 8 accelerator dies (XCDs), each with its own L2; workgroups are dealt to them round-robin by workgroup id.  The count
// is asked of the current device; without one (planning on a host without a GPU) MI355X's 8 is assumed.  Whether congruent workgroup
// ids really share a die is checked on the device when a workspace is bound (see check_l2_sharing).
constexpr int kDefaultL2Domains = 8, kDefaultUnits = 256;
constexpr int kPlacementSlots = 1024;

int query_l2_domains()
{
    int dev = 0, xccs = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&xccs, hipDeviceAttributeNumberOfXccs, dev) == hipSuccess && xccs >= 1 && xccs <= 64)
        return xccs;
    (void)hipGetLastError();
    return kDefaultL2Domains;
}

// Compute units of the current device (MI355X's 256 without one).
int query_units()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0) return cus;
    (void)hipGetLastError();
    return kDefaultUnits;
}

// Workgroup slots of the shared-cells split: one per compute unit of the current device (a multiple of the L2 domains), two for rows
// of at most 8 KB (MI355X's 256 without a device).
int unit_slots(int64_t row_bytes, int domains)
{
    int count = 0;
    const bool device = hipGetDeviceCount(&count) == hipSuccess && count > 0;
    (void)hipGetLastError();
    const int slots = std::max(query_units(), domains) / domains * domains;
    return device && row_bytes <= 8192 ? 2 * slots : slots;
}

// Shared cells group the holders of a row by workgroup: how many of the up to max_holders (s+1)^L holders one workgroup serves.
// fp32 rows of 257 to 3072 chunks; 0 where there is no such split.
int shared_cell_holders(int x_dtype, int64_t d, int64_t max_holders)
{
    const int64_t nq = (d + 3) / 4;
    if (x_dtype != CR_F32 || nq <= 256 || nq > 3072) return 0;
    if (nq > 1536 && nq <= 2558 && d % 4 == 0 && max_holders >= 3) {
        if ((max_holders == 5 || max_holders == 6) && nq <= 2557) return 6;
        return (max_holders + 3) / 4 < (max_holders + 2) / 3 ? 4 : 3;      // whichever takes fewer workgroups per row
    }
    if (max_holders >= 5 && nq <= 1024) return 8;
    return max_holders >= 3 && nq <= 1536 ? 4 : 2;
}

// Bytes of X that the first pass over wide rows leaves in the 256 MB last-level cache for the second (both passes over 400 MB, 4 000 x 50 008
// bf16, with 0, 64, 160 and 220 MB: 142.6, 136.8, 132.9 and 129.8 us; 200 and 240 MB take the same as 220).
constexpr int64_t kKeptBytes = int64_t(200) << 20;

int64_t longest_range(const cr_plan_t *p)
{
    int64_t longest = 0;
    for (const cr::Slab &sl : p->slabs) longest = std::max(longest, sl.row_end - sl.row_begin);
    return longest;
}

// Small problems: a workgroup per distinct slab range forms its gradient whole, which saves the launch that adds up partial rows.  The
// line is where the two take the same time, at about 48 Ki elements in the longest range (fp32, us whole / parts and sum; a (3,2) tree:
// 160 x 150 elements in the longest range 5.6 / 7.9, 320 x 150 7.4 / 8.0, 640 x 150 12.0 / 7.9; 54 x 900 6.1 / 8.1, 107 x 900 8.9 / 9.7;
// 19 x 2500 7.9 / 8.0, 38 x 2500 13.4 / 8.3).  Ranges that overlap without being equal are formed one by one; on the trees measured that
// costs less than the launch as long as about 25 MB are read in all (a (5,4) tree, where a row is in 4 ranges on average: 160 x 150
// 8.9 / 9.2, 320 x 150 with 47 MB 13.6 / 10.0, but 54 x 900 with 52 MB 13.6 / 18.0, where parts have runs of less than one step).
bool whole_ranges_pay(const cr_plan_t *p) { return p->once_variant && longest_range(p) * p->d <= 48 * 1024; }

// Rows one after the other along X, every row once, on every compute unit: the parts of the default split.
void make_rows_once(cr_plan_t *p, int64_t rows_per_run)
{
    const cr::OnceVariant *v = p->once = p->once_variant;
    // small problems: no fewer rows per part than a workgroup takes in a step, two where the whole workgroup shares a row (the
    // partial rows of shorter parts cost more than the extra workgroups bring)
    const int64_t least = v->threads_per_row <= 64 ? std::min(v->rows_per_step, 128) : 2;
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(static_cast<int64_t>(query_units()) * v->parts_per_unit, p->m / least));
    cr::once_equal_parts(p->slabs, p->m, parts, rows_per_run, p->work);
}

int64_t wide_one_pass_parts(const cr_plan_t *p) { return std::max<int64_t>(1, std::min<int64_t>(query_units(), p->m / 4)); }

// The parts of the second of two passes, each of which has one workgroup per block of columns; two workgroups per compute unit, no fewer
// rows per part than a workgroup has in flight (4 000 x 50 008 bf16 with one, two, four and eight: 123, 124, 130 and 138 us, 4 000 x 60 000
// fp32 290, 281, 287 and more; fewer partial rows to add up as well).
int64_t wide_two_pass_parts(const cr_plan_t *p)
{
    const int64_t vec = p->x_dtype == CR_BF16 ? 8 : 4, blocks = ((p->d + vec - 1) / vec + cr::kWideColumnChunks - 1) / cr::kWideColumnChunks;
    return std::max<int64_t>(1, std::min<int64_t>(2 * static_cast<int64_t>(query_units()) / blocks, p->m / 16));
}

// Rows of more than 24 576 columns whose weights fit LDS take one pass where X has more bytes than nine tenths of the rows that the part
// per compute unit puts away and adds up beyond those of two passes, and from 48 MB of X on (us with sums, one pass / two:
// 300 x 30 000 bf16 22.8 / 18.2, 600 x 30 000 bf16, 36 MB, 24.9 / 24.2, 1 200 x 26 000 bf16 28.3 / 31.7, 3 000 x 30 001 fp32 78 / 118,
// 6 000 x 32 768 fp32 141 / 249; (2,12), s = 1, 300 slabs: 712 x 36 864 bf16 62.2 / 46.1, 2 134 x 28 672 56 / 60; (3,6), s = 2, 774 slabs:
// 1 423 x 36 864 bf16 79.0 / 69.5, 4 369 x 30 001 fp32 125 / 209).  On 1 089 trees and sizes the rule is 0.4 % behind the faster of the two, and 16 % at
// worst.
constexpr int64_t kWideOnePassBytes = int64_t(48) << 20;

// Rows that a split into `parts` parts puts away, and adds up where slabs are sums of several.
int64_t rows_put_away(const cr_plan_t *p, int64_t parts)
{
    cr::OnceWork work;
    cr::once_equal_parts(p->slabs, p->m, parts, p->m, work);
    int64_t rows = static_cast<int64_t>(work.runs.size());
    for (const cr::RowSum &sum : work.sums) rows += sum.row_end - sum.row_begin;
    return rows;
}

bool one_pass_pays(const cr_plan_t *p)
{
    const int64_t bytes = p->m * p->d * elem_size(p);
    if (bytes < kWideOnePassBytes || !cr::select_once_wide(p->x_dtype, p->d)) return false;
    return bytes / 9 * 10 > (rows_put_away(p, wide_one_pass_parts(p)) - rows_put_away(p, wide_two_pass_parts(p))) * p->d * 4;
}

// One pass over wide rows: a part per compute unit, at least four rows; the most rows that a part has, or 0: two passes.
int64_t wide_one_pass_rows(const cr_plan_t *p)
{
    const int64_t parts = wide_one_pass_parts(p);
    return one_pass_pays(p) ? (p->m + parts - 1) / parts : 0;
}

// Slabs that a workgroup of the one pass writes a run's whole row to; a row of 100 to 147 KB takes it a microsecond each, one after the
// other.  To more of them the sums' launch hands it, a workgroup per 64 chunks.
constexpr size_t kWideCopies = 2;

// Crews: as many as the dies have workgroups for, and at least four rows for each (us with sums, parts of at least 1, 2, 4, 8 and 16 rows:
// (2,4), s = 1, 40 x 37 000 bf16 17.8, 15.1, 13.8, 16.4, 23.4; 80 x 60 000 fp32 23.1, 22.9, 22.5, 22.6, 27.2; the same from 160 rows on).
int64_t crew_parts(const cr_plan_t *p, const cr::CrewVariant &crew)
{
    const int64_t units = query_units(), crews = units >= 64 ? units / 8 / crew.members * 8 : units / crew.members;
    return std::max<int64_t>(1, std::min<int64_t>(crews, p->m / 4));
}

// Rows too wide for one workgroup, weights in LDS or not, are shared by crews in one pass, or take two.  Two passes have long parts and so
// fewer partial rows, which pays where X is small against the rows that crews put away and add up beyond those of two passes, and there
// are rows enough for five parts (us with sums, crews / two passes, by that share of X: (1,10), s = 4, 640 x 37 000 bf16 (0.04)
// 22.9 / 32.2; (3,6), s = 2, 640 x 37 000 bf16 (0.20) 54.3 / 68.7; (2,12), s = 2, 320 x 36 000 fp32 (0.23) 36.8 / 36.9; (1,10), s = 4, fp32
// 160 x 100 000 (0.24) 32.5 / 27.3, 160 x 36 000 (0.44) 19.4 / 13.7, 40 x 60 000 (0.25) 17.0 / 16.7, 20 x 60 000 (0.50) 17.0 / 22.2;
// (2,4), s = 1, 40 x 60 000 fp32 (0.57) 17.9 / 21.4, 160 x 60 000 fp32 (0.19) 24.0 / 23.0).  Large X: 400 MB 75 to 95 / 125 to 144.
bool crew_pays(const cr_plan_t *p, const cr::CrewVariant &crew)
{
    if (p->m < 80) return true;
    const int64_t more = rows_put_away(p, crew_parts(p, crew)) - rows_put_away(p, wide_two_pass_parts(p));
    return p->m * p->d * elem_size(p) / 17 * 4 > more * p->d * 4;
}

// The same for wide rows.  One workgroup per row where that pays and runs of no more rows are asked for than its parts have, which the default
// split does; longer runs take two passes, where parts are long, and so do wider rows where crews do not pay.
void make_wide_once(cr_plan_t *p, int64_t rows_per_run)
{
    if (rows_per_run <= wide_one_pass_rows(p)) {
        p->wide_variant = cr::select_once_wide(p->x_dtype, p->d);
        return cr::once_equal_parts(p->slabs, p->m, wide_one_pass_parts(p), rows_per_run, p->work, kWideCopies);
    }
    p->units = query_units();
    cr::CrewVariant crew;
    if (!cr::select_once_wide(p->x_dtype, p->d) && cr::select_crew(p->x_dtype, p->d, p->units, &crew) && crew_pays(p, crew)) {
        p->crew = std::make_unique<cr::CrewVariant>(crew);
        cr::once_equal_parts(p->slabs, p->m, crew_parts(p, crew), rows_per_run, p->work, kWideCopies);
        int64_t longest = 0;
        for (size_t b = 0; b + 1 < p->work.part_run_begin.size(); ++b)
            longest = std::max(longest, p->work.runs[p->work.part_run_begin[b + 1] - 1].row_end - p->work.runs[p->work.part_run_begin[b]].row_begin);
        p->crew->ring_steps = cr::crew_ring_steps(crew, longest);
        return;
    }
    cr::once_equal_parts(p->slabs, p->m, wide_two_pass_parts(p), rows_per_run, p->work);
}

int make_split(cr_plan_t *p)
{
    int kind = p->split_kind;
    int64_t value = p->split_value;
    p->variant = nullptr;
    p->once = nullptr;
    p->wide_variant = nullptr;
    p->crew.reset();
    p->rows_once = false;
    p->work = cr::OnceWork();
    const int domains = query_l2_domains();
    p->l2_domains = domains;
    p->unit_slots = 0;
    p->l2_sharing = -1;
    const bool large = p->m * p->d * elem_size(p) >= kLargeBytes;
    if (kind < 0 && large && p->s == 0 && p->once_variant) {
        // no row is held twice
        kind = CR_SPLIT_EQUAL_RANGES;
        value = static_cast<int64_t>(query_units()) * p->once_variant->parts_per_unit;
    }
    if (kind < 0 && large && p->cell_holders >= p->max_holders) {
        // All holders of a cell in one workgroup, cells between slab boundaries, one queue of cells per compute unit.  The launch
        // lasts as long as the longest queue: take the cell height, 16 to 1024 rows in steps of 8, that makes it shortest; ties go
        // to the taller cell (fewer partial rows).  Against contiguous parts (rows once), stage 1 in us: 252 000 x 4 096 589 / 590,
        // 100 000 x 10 000 on a (4,2) tree 578 / 578, with 20 workers in one layer 612 / 579, 366 000 x 2 048 464 / 428.
        kind = CR_SPLIT_SHARED_CELLS;
        const int slots = unit_slots(p->d * elem_size(p), domains);
        value = 512;
        if (p->row_visits / p->cell_holders / 64 <= (int64_t(1) << 16)) {       // with longer queues than that the last round no longer matters
            int64_t best = -1;
            cr::Split trial;
            for (int64_t c = 16; c <= 1024; c += 8) {
                cr::split_shared_queues(p->slabs, c, domains, p->cell_holders, slots / domains, trial);
                if (best < 0 || trial.makespan <= best) { best = trial.makespan; value = c; }
            }
        }
    }
    if (kind < 0) {
        kind = CR_SPLIT_ROWS_ONCE;
        const int64_t wide = p->once_variant ? 0 : wide_one_pass_rows(p);
        value = whole_ranges_pay(p) ? CR_ROWS_WHOLE_RANGES : wide ? wide : p->m;
    }
    p->split_kind_used = kind;
    p->split_value_used = value;
    // more rows than there are mean all of them; the products and sums below then stay far inside 64 bits
    const bool whole_ranges = kind == CR_SPLIT_ROWS_ONCE && value == CR_ROWS_WHOLE_RANGES && p->once_variant && longest_range(p) <= cr::kMaxRunRows;
    if (kind != CR_SPLIT_EQUAL_RANGES) value = std::min(value, p->m);
    if (kind == CR_SPLIT_ROWS_ONCE) {
        if (p->m / value + 2 * static_cast<int64_t>(p->slabs.size()) > (int64_t(1) << 26)) return fail(CR_E_INVAL, "too many partial rows");
        if (whole_ranges) {
            p->once = cr::select_once_whole(p->x_dtype, p->d);
            cr::once_whole_ranges(p->slabs, p->work);
        } else if (p->once_variant) make_rows_once(p, value);
        else make_wide_once(p, value);
        p->rows_once = true;
        cr::once_as_split(p->slabs, p->work, p->split);
    } else if (kind == CR_SPLIT_SHARED_CELLS) {
        if (!p->cell_holders) return fail(CR_E_INVAL, "no shared cells for rows of this width and type");
        if (p->row_visits / value + 2 * static_cast<int64_t>(p->slabs.size()) > (int64_t(1) << 26)) return fail(CR_E_INVAL, "too many row cells");
        p->unit_slots = unit_slots(p->d * elem_size(p), domains);
        cr::split_shared_queues(p->slabs, value, domains, p->cell_holders, p->unit_slots / domains, p->split);
        p->once = p->once_variant;
        p->rows_once = true;
        cr::once_of_queues(p->slabs, p->split, p->cell_holders, p->work);
    } else if (kind == CR_SPLIT_EQUAL_RANGES && p->s == 0 && p->once_variant) {
        // no row is held twice: every holder's arithmetic is every row once
        cr::split_equal_ranges(p->slabs, static_cast<int>(std::min<int64_t>(value, p->m)), p->split);
        p->once = p->once_variant;
        p->rows_once = true;
        cr::once_of_pieces(p->slabs, p->split, p->work);
    } else {
        p->variant = p->variant_regs;
        const int teams_per_block = p->variant ? p->variant->teams_per_block() : 1;     // wide rows: one workgroup per piece
        if (kind == CR_SPLIT_ROW_CELLS) {
            if (p->row_visits / value + static_cast<int64_t>(p->slabs.size()) > (int64_t(1) << 26)) return fail(CR_E_INVAL, "too many row cells");
            // the wide-row kernels index pieces directly: no empty teams
            cr::split_row_cells(p->slabs, value, p->variant ? domains : 1, teams_per_block, p->split);
        } else {
            cr::split_equal_ranges(p->slabs, static_cast<int>(std::min<int64_t>(value, std::max<int64_t>(1, p->row_visits))), p->split);
        }
    }
    // rows that several workgroups read are left in the caches for each other
    int64_t rows_read = 0;
    for (const cr::RowRun &run : p->work.runs) rows_read += run.row_end - run.row_begin;
    p->streams = p->m * p->d * elem_size(p) >= kStreamFromBytes && rows_read <= p->m;
    return CR_OK;
}

int ensure_split(cr_plan_t *p)
{
    if (!p->split.pieces.empty() || p->model == CR_AGGREGATE_ONLY) return CR_OK;
    try {
        return make_split(p);
    } catch (const std::bad_alloc &) {
        p->split = cr::Split();                          // half a split is none
        p->work = cr::OnceWork();
        return fail(CR_E_NOMEM, "out of host memory");
    }
}

void compute_layout(cr_plan_t *p, size_t *total)
{
    const size_t S = p->slabs.size(), N = p->tree.N, P = p->split.pieces.size();
    const size_t runs = p->work.runs.size(), parts = p->work.part_run_begin.empty() ? 0 : p->work.part_run_begin.size() - 1;
    const size_t sums = p->rows_once ? p->work.sums.size() : S, dst = p->rows_once ? p->work.dst.size() : S;
    // worst case: one term per slab plus one dummy per node, each sub-program padded to the unroll
    p->max_terms = align_up(S + N + static_cast<size_t>(p->n) * cr::kEncodeUnroll, cr::kEncodeUnroll);
    size_t off = 0;
    p->off_slab = off;  off = align_up(off + p->max_terms * sizeof(int32_t), 256);
    p->off_level = off; off = align_up(off + p->max_terms * sizeof(int32_t), 256);
    p->off_row = off;   off = align_up(off + p->max_terms * sizeof(int32_t), 256);
    p->off_coef = off;  off = align_up(off + p->max_terms * sizeof(double), 256);
    p->off_acoef = off; off = align_up(off + p->max_terms * sizeof(double), 256);
    p->off_sub = off;   off = align_up(off + 2 * static_cast<size_t>(p->n) * sizeof(int32_t), 256);   // begin and end of every sub-program
    p->off_dec = off;   off = align_up(off + p->n * sizeof(double), 256);
    p->program_bytes = off;

    size_t w = 0;
    auto take = [&](size_t bytes) { const size_t at = w; w = align_up(w + bytes, 256); return at; };
    p->at_pieces = take(p->rows_once ? 0 : P * sizeof(cr::DevPiece));
    p->at_team_piece_begin = take(p->rows_once ? 0 : (p->split.teams + 1) * sizeof(int32_t));
    p->at_parts = take(parts * sizeof(cr::DevRun));
    p->at_runs = take(runs * sizeof(cr::DevRun));
    p->at_sums = take(p->model == CR_AGGREGATE_ONLY ? 0 : sums * sizeof(cr::DevSum));
    p->at_dst = take(p->model == CR_AGGREGATE_ONLY ? 0 : dst * sizeof(int32_t));
    p->at_crew_slots = take(p->crew ? parts * cr::crew_exchange_words(*p->crew) * sizeof(uint64_t) : 0);
    p->at_crew_state = take(p->crew ? 2 * sizeof(uint32_t) : 0);
    p->at_node_begin = take((N + 1) * sizeof(int32_t));
    p->at_slab_coef = take(S * sizeof(double));
    p->tables_bytes = w;                                 // what the plan fills in at binding, in one copy
    p->at_placement = take(kPlacementSlots * sizeof(uint32_t));
    p->at_program = take(kProgramSlots * p->program_bytes);
    const int groups_together = cr::tree_and_decode_together(p->shape, p->d) ? cr::tree_decode_groups(p->n, p->L, p->d) : 0;
    p->measures_stride = p->model == CR_AGGREGATE_ONLY ? 0 : 4 * static_cast<size_t>(std::max(cr::decode_groups(p->d), groups_together));
    p->at_measures = take(kProgramSlots * p->measures_stride * sizeof(double));
    const size_t row = static_cast<size_t>(p->d) * sizeof(float);
    if (p->model != CR_AGGREGATE_ONLY) {
        p->at_G = take((S + (p->rows_once ? p->work.partials : P)) * row);
        p->at_residuals = take(p->once || p->wide_variant || p->crew || p->variant ? 0 : static_cast<size_t>(p->rows_once ? p->m : p->row_visits) * sizeof(float));
    }
    p->at_M = take(N * row);
    *total = w;
}

hipEvent_t take_event(cr_plan_t *p)
{
    if (!p->event_pool.empty()) {
        hipEvent_t e = p->event_pool.back();
        p->event_pool.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}

struct LaunchTimer {     // brackets one launch with events when profiling is on
    cr_plan_t *p;
    int kernel;
    hipEvent_t start = nullptr, stop = nullptr;
    LaunchTimer(cr_plan_t *plan, int k, int64_t bytes) : p(plan), kernel(k)
    {
        p->bytes_last[k] = bytes;
        if (!((p->profiling >> k) & 1)) return;
        start = take_event(p);
        stop = take_event(p);
        if (start && stop) (void)hipEventRecord(start, p->stream);
    }
    void done()
    {
        if (!start || !stop) return;
        (void)hipEventRecord(stop, p->stream);
        p->timed.push_back({kernel, start, stop});
        p->bytes_sum[kernel] += p->bytes_last[kernel];
    }
};

int fold_timings(cr_plan_t *p)
{
    for (const TimedLaunch &t : p->timed) {
        float ms = 0.f;
        CR_HIP(hipEventElapsedTime(&ms, t.start, t.stop));
        p->total_ms[t.kernel] += ms;
        p->launches[t.kernel] += 1;
        if (p->samples[t.kernel].size() < kMaxSamples) p->samples[t.kernel].push_back(ms);
        p->event_pool.push_back(t.start);
        p->event_pool.push_back(t.stop);
    }
    p->timed.clear();
    return CR_OK;
}

// The row-cell and shared-cell splits put the holders of a cell on workgroup ids that are congruent modulo the number of L2
// domains, trusting that the dispatcher deals workgroups to the dies round-robin.  This runs a launch of kPlacementSlots small
// workgroups that record the die they ran on and checks exactly that; the outcome is reported by cr_plan_info (l2_sharing).
// A device that places workgroups differently still computes the same results, only without the shared fetches.
int check_l2_sharing(cr_plan_t *p)
{
    std::vector<uint32_t> where(kPlacementSlots);
    CR_HIP(cr::launch_placement_probe(p->d_placement, kPlacementSlots, p->stream));
    CR_HIP(hipMemcpyAsync(where.data(), p->d_placement, kPlacementSlots * sizeof(uint32_t), hipMemcpyDeviceToHost, p->stream));
    CR_HIP(hipStreamSynchronize(p->stream));
    const int domains = p->l2_domains;
    std::vector<int> die_of(domains, -1);
    bool ok = true;
    for (int g = 0; g < kPlacementSlots && ok; ++g) {
        const int die = static_cast<int>(where[g] >> 16);
        int &seen = die_of[g % domains];
        if (seen < 0) seen = die;
        ok = seen == die;
    }
    for (int a = 0; a < domains && ok; ++a)                  // and distinct residues on distinct dies
        for (int b = a + 1; b < domains; ++b) ok = ok && die_of[a] != die_of[b];
    p->l2_sharing = ok ? 1 : 0;
    return CR_OK;
}

// An aggregation-only plan keeps nothing in the workspace between calls, which may serve other plans in the meantime: its tree's tables
// go to pages of the library's, as long as there are free ones (else they go with every call, see mask_tables).
hipError_t keep_tables(cr_plan_t *p, const char *tables)
{
    const size_t bytes = p->tables_bytes - p->at_node_begin;
    int device = 0;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return e;
    if (p->pool_first >= 0 && p->pool_device != device) {
        g_table_pages.give(p->pool_device, p->pool_first, p->pool_pages);
        p->pool_first = -1;
    }
    if (p->pool_first < 0) {
        p->pool_device = device;
        p->pool_pages = static_cast<int>((bytes + cr::kTablePageBytes - 1) / cr::kTablePageBytes);
        p->pool_first = g_table_pages.take(device, p->pool_pages);
    }
    if (p->pool_first < 0) return hipSuccess;
    char *pool = nullptr;
    e = cr::table_pool(&pool);
    if (e != hipSuccess) return e;
    char *at = pool + static_cast<size_t>(p->pool_first) * cr::kTablePageBytes;
    p->d_node_begin = reinterpret_cast<int32_t *>(at);
    p->d_slab_coef = reinterpret_cast<double *>(at + (p->at_slab_coef - p->at_node_begin));
    return hipMemcpy(at, tables, bytes, hipMemcpyHostToDevice);
}

}  // namespace

extern "C" {

const char *cr_last_error(void) { return g_last_error.c_str(); }

int cr_plan(int L, int n, int s, int64_t m, int64_t d, cr_plan_t **out)
{
    return cr_plan_ex(L, n, s, m, d, CR_LINEAR, CR_F32, kDefaultSeed, nullptr, out);
}

int cr_plan_ex(int L, int n, int s, int64_t m, int64_t d, int model, int x_dtype, uint64_t seed, const double *B_or_null, cr_plan_t **out)
{
    if (!out) return fail(CR_E_INVAL, "out is NULL");
    *out = nullptr;
    if (L < 1 || L > cr::kMaxLevels) return fail(CR_E_INVAL, "L must be in 1..8");
    if (n < 2 || n > 64) return fail(CR_E_INVAL, "n must be in 2..64");
    if (s < 0 || s >= n) return fail(CR_E_INVAL, "s must be in 0..n-1");
    if (d < 1) return fail(CR_E_INVAL, "d must be positive");
    if (d > (int64_t(1) << 28)) return fail(CR_E_INVAL, "d exceeds 2^28");     // every kernel indexes columns with 32-bit integers
    if (model < CR_LINEAR || model > CR_AGGREGATE_ONLY) return fail(CR_E_INVAL, "unknown model");
    if (x_dtype != CR_F32 && x_dtype != CR_BF16) return fail(CR_E_INVAL, "unknown x_dtype");
    if (cr::num_straggler_sets(n, s, int64_t(1) << 20) < 0) return fail(CR_E_INVAL, "C(n,s) exceeds 2^20 straggler patterns");
    cr_plan_t *p = new (std::nothrow) cr_plan_s();
    if (!p) return fail(CR_E_NOMEM, "out of host memory");
    try {
        if (!cr::make_tree(n, L, p->tree)) { delete p; return fail(CR_E_INVAL, "tree has more than 2^24 workers"); }
        if (m < p->tree.N) { delete p; return fail(CR_E_INVAL, "m must be at least the number of workers"); }
        if (m > (int64_t(1) << 40)) { delete p; return fail(CR_E_INVAL, "m exceeds 2^40"); }
        p->L = L; p->n = n; p->s = s; p->m = m; p->d = d; p->model = model; p->x_dtype = x_dtype;
        bool ok = B_or_null ? cr::adopt_code(n, s, B_or_null, p->code) : cr::design_code(n, s, L, seed, p->code);
        if (!ok) { delete p; return fail(CR_E_INVAL, B_or_null ? "supplied B must have s+1 non-zeros per row and per column and decode every straggler set" : "code search found no usable candidate"); }
        cr::allocate(p->tree, s, m, p->code.B.data(), p->own, p->slabs);
        p->node_slab_begin.assign(p->tree.N + 1, 0);
        for (const cr::Slab &sl : p->slabs) p->node_slab_begin[sl.node + 1] += 1;
        for (int32_t i = 0; i < p->tree.N; ++i) p->node_slab_begin[i + 1] += p->node_slab_begin[i];
        for (const cr::Slab &sl : p->slabs) p->slab_coef.push_back(sl.coef);
        p->last_send.assign(p->tree.N, -1);
        p->shape = {n, L, s, p->tree.N, static_cast<int64_t>(p->slabs.size())};
        if (cr::tree_side_by_side(p->shape, d, cr::Otherwise::kCopy) || cr::tree_side_by_side(p->shape, d, cr::Otherwise::kLaunches) ||
            cr::tree_side_by_side(p->shape, d, cr::Otherwise::kBatch)) {
            p->tree_arguments = std::make_unique<cr::TreeArguments>();
            cr::lay_out_tree(p->tree.N, static_cast<int>(p->slabs.size()), p->node_slab_begin.data(), p->slab_coef.data(), p->tree_arguments.get());
        }
        p->min_rows = INT64_MAX;
        for (int32_t node = 0; node < p->tree.N; ++node) {
            int64_t rows = 0;
            for (const cr::Segment &g : p->own[node]) rows += g.row_end - g.row_begin;
            p->row_visits += rows;
            p->min_rows = std::min(p->min_rows, rows);
            p->max_rows = std::max(p->max_rows, rows);
        }
        if (p->slabs.size() > (size_t(1) << 30)) { delete p; return fail(CR_E_INVAL, "too many slabs"); }
        if (model != CR_AGGREGATE_ONLY) {
            p->variant_regs = cr::select_stage1(x_dtype, d);          // nullptr: rows too wide for one team's registers, two-pass path
            p->once_variant = cr::select_once(x_dtype, d);
            for (int l = 0; l < L && p->max_holders < 64; ++l) p->max_holders *= s + 1;     // a leaf's rows sit in s+1 workers of every level above it
            p->cell_holders = s > 0 ? shared_cell_holders(x_dtype, d, p->max_holders) : 0;
        }
    } catch (const std::bad_alloc &) {
        delete p;
        return fail(CR_E_NOMEM, "out of host memory");
    }
    *out = p;
    return CR_OK;
}

void cr_plan_destroy(cr_plan_t *p)
{
    if (!p) return;
    const bool idle = !p->bound || hipStreamSynchronize(p->stream) == hipSuccess;
    if (p->pool_first >= 0 && idle) g_table_pages.give(p->pool_device, p->pool_first, p->pool_pages);
    for (const TimedLaunch &t : p->timed) { (void)hipEventDestroy(t.start); (void)hipEventDestroy(t.stop); }
    for (hipEvent_t e : p->event_pool) (void)hipEventDestroy(e);
    for (hipEvent_t e : p->staging_done)
        if (e) (void)hipEventDestroy(e);
    if (p->h_staging) (void)hipHostFree(p->h_staging);
    delete p;
}

int cr_plan_info(const cr_plan_t *p, cr_plan_info_t *info)
{
    if (!p || !info) return fail(CR_E_INVAL, "NULL argument");
    std::memset(info, 0, sizeof *info);
    info->L = p->L; info->n = p->n; info->s = p->s; info->model = p->model; info->x_dtype = p->x_dtype;
    info->num_workers = p->tree.N;
    info->num_groups = p->tree.N / p->n;
    info->num_slabs = static_cast<int32_t>(p->slabs.size());
    info->num_decode_rows = static_cast<int32_t>(cr::num_straggler_sets(p->n, p->s, int64_t(1) << 20));
    info->code_candidate = p->code.candidate;
    info->num_teams = p->split.teams;
    info->num_pieces = static_cast<int32_t>(p->split.pieces.size());
    const bool split_known = !p->split.pieces.empty();
    info->split_kind = split_known ? p->split_kind_used : -1;
    info->split_value = split_known ? p->split_value_used : 0;
    const bool cells = split_known && p->split_kind_used == CR_SPLIT_SHARED_CELLS;
    const cr::OnceVariant *once = p->once ? p->once : split_known ? nullptr : p->once_variant;
    info->stage1_team_size = once ? once->threads_per_row : p->variant ? p->variant->team_size : 0;
    info->stage1_teams_per_group = cells ? p->cell_holders : once ? once->block / once->threads_per_row : p->variant ? p->variant->teams_per_block() : 1;
    info->stage1_staged = cells ? 1 : 0;
    info->m = p->m; info->d = p->d;
    info->row_visits = p->row_visits;
    info->min_rows = p->min_rows; info->max_rows = p->max_rows;
    info->gamma = p->code.gamma;
    double q = static_cast<double>(p->n) / (p->s + 1), sum = 0.0, pw = 1.0;
    for (int l = 1; l <= p->L; ++l) { pw *= q; sum += pw; }
    info->r_cr = 1.0 / sum;
    info->l2_domains = p->l2_domains ? p->l2_domains : kDefaultL2Domains;
    info->unit_slots = split_known ? p->unit_slots : 0;
    info->l2_sharing = p->l2_sharing;
    info->code_warning = std::pow(p->code.gamma, p->L) * std::ldexp(1.0, -24) > 1e-5 ? 1 : 0;
    return CR_OK;
}

int cr_plan_get_B(const cr_plan_t *p, double *B)
{
    if (!p || !B) return fail(CR_E_INVAL, "NULL argument");
    std::copy(p->code.B.begin(), p->code.B.end(), B);
    return CR_OK;
}

int cr_plan_get_A(const cr_plan_t *p, double *A)
{
    if (!p || !A) return fail(CR_E_INVAL, "NULL argument");
    const int64_t F = cr::num_straggler_sets(p->n, p->s, int64_t(1) << 20);
    for (int64_t f = 0; f < F; ++f)
        if (!cr::decode_row(p->code, cr::straggler_set_by_rank(p->n, p->s, f), A + f * p->n))
            return fail(CR_E_INVAL, "decode row: survivor system is inconsistent");
    return CR_OK;
}

int cr_plan_get_segments(const cr_plan_t *p, int64_t *row_begin, int64_t *row_end, double *coef, int32_t *worker)
{
    if (!p) return fail(CR_E_INVAL, "NULL plan");
    for (size_t i = 0; i < p->slabs.size(); ++i) {
        if (worker) worker[i] = p->slabs[i].node;
        if (row_begin) row_begin[i] = p->slabs[i].row_begin;
        if (row_end) row_end[i] = p->slabs[i].row_end;
        if (coef) coef[i] = p->slabs[i].coef;
    }
    return CR_OK;
}

int cr_plan_decode_row(const cr_plan_t *p, const uint8_t *flags, double *a)
{
    if (!p || !flags || !a) return fail(CR_E_INVAL, "NULL argument");
    const double *row = nullptr;
    int rc = group_decode_row(p, flags, &row);
    if (rc == CR_E_UNDECODABLE) return fail(rc, "more than s stragglers in the group");
    if (rc != CR_OK) return rc;
    std::copy(row, row + p->n, a);
    return CR_OK;
}

int cr_plan_set_split(cr_plan_t *p, int kind, int64_t value)
{
    if (!p) return fail(CR_E_INVAL, "NULL plan");
    if (kind < CR_SPLIT_EQUAL_RANGES || kind > CR_SPLIT_ROWS_ONCE) return fail(CR_E_INVAL, "unknown split kind");
    if (value < 1) return fail(CR_E_INVAL, "split value must be >= 1");
    if (kind == CR_SPLIT_EQUAL_RANGES && value > (int64_t(1) << 24)) return fail(CR_E_INVAL, "too many teams");
    if (p->bound) return fail(CR_E_STATE, "the work split cannot change once a workspace is bound");
    if (p->model == CR_AGGREGATE_ONLY) return fail(CR_E_INVAL, "an aggregation-only plan has no stage-1 split");
    p->split_kind = kind;
    p->split_value = value;
    p->split = cr::Split();
    return ensure_split(p);
}

int cr_plan_get_pieces(const cr_plan_t *p, int32_t *slab, int64_t *row_begin, int64_t *row_end, int32_t *team)
{
    if (!p) return fail(CR_E_INVAL, "NULL plan");
    for (size_t i = 0; i < p->split.pieces.size(); ++i) {
        if (slab) slab[i] = p->split.pieces[i].slab;
        if (row_begin) row_begin[i] = p->split.pieces[i].row_begin;
        if (row_end) row_end[i] = p->split.pieces[i].row_end;
        if (team) team[i] = p->split.pieces[i].team;
    }
    return CR_OK;
}

int cr_simulate_iteration(const cr_plan_t *p, double a, double mu, double t_c, uint64_t seed, int64_t iteration, uint8_t *mask,
                          double *ready, double *total)
{
    if (!p) return fail(CR_E_INVAL, "NULL plan");
    if (!(a >= 0.0) || !(mu > 0.0) || !(t_c >= 0.0) || iteration < 0) return fail(CR_E_INVAL, "a >= 0, mu > 0, t_c >= 0, iteration >= 0 required");
    std::vector<int64_t> rows(p->tree.N, 0);
    for (const cr::Slab &sl : p->slabs) rows[sl.node] += sl.row_end - sl.row_begin;
    const double t = cr::simulate_iteration(p->tree, p->s, rows, {a, mu, t_c}, seed, iteration, mask, ready);
    if (total) *total = t;
    return CR_OK;
}

int cr_workspace_bytes(cr_plan_t *p, size_t *bytes)
{
    if (!p || !bytes) return fail(CR_E_INVAL, "NULL argument");
    int rc = ensure_split(p);
    if (rc != CR_OK) return rc;
    compute_layout(p, bytes);
    return CR_OK;
}

int cr_bind_workspace(cr_plan_t *p, void *dev_ptr, size_t bytes, void *hip_stream)
try {
    if (!p || !dev_ptr) return fail(CR_E_INVAL, "NULL argument");
    if (reinterpret_cast<uintptr_t>(dev_ptr) % 256 != 0) return fail(CR_E_INVAL, "workspace must be 256-byte aligned");
    int rc = ensure_split(p);
    if (rc != CR_OK) return rc;
    size_t need = 0;
    compute_layout(p, &need);
    if (bytes < need) return fail(CR_E_INVAL, "workspace too small");
    if (p->bound) CR_HIP(hipStreamSynchronize(p->stream));
    p->bound = false;                                    // until the new workspace has its tables
    p->stream = static_cast<hipStream_t>(hip_stream);
    p->ws = static_cast<char *>(dev_ptr);
    p->ws_bytes = bytes;

    const int32_t S = static_cast<int32_t>(p->slabs.size()), P = static_cast<int32_t>(p->split.pieces.size());
    p->d_pieces = reinterpret_cast<cr::DevPiece *>(p->ws + p->at_pieces);
    p->d_team_piece_begin = reinterpret_cast<int32_t *>(p->ws + p->at_team_piece_begin);
    p->d_parts = reinterpret_cast<cr::DevRun *>(p->ws + p->at_parts);
    p->d_runs = reinterpret_cast<cr::DevRun *>(p->ws + p->at_runs);
    p->d_sums = reinterpret_cast<cr::DevSum *>(p->ws + p->at_sums);
    p->d_dst = reinterpret_cast<int32_t *>(p->ws + p->at_dst);
    p->d_crew_slots = reinterpret_cast<uint64_t *>(p->ws + p->at_crew_slots);
    p->d_crew_state = reinterpret_cast<uint32_t *>(p->ws + p->at_crew_state);
    p->d_placement = reinterpret_cast<uint32_t *>(p->ws + p->at_placement);
    p->d_program = p->ws + p->at_program;
    p->d_node_begin = reinterpret_cast<int32_t *>(p->ws + p->at_node_begin);
    p->d_slab_coef = reinterpret_cast<double *>(p->ws + p->at_slab_coef);
    p->d_measures = reinterpret_cast<double *>(p->ws + p->at_measures);
    const bool stage1 = p->model != CR_AGGREGATE_ONLY;
    p->d_G = stage1 ? reinterpret_cast<float *>(p->ws + p->at_G) : nullptr;
    p->d_residuals = stage1 ? reinterpret_cast<float *>(p->ws + p->at_residuals) : nullptr;
    p->d_M = reinterpret_cast<float *>(p->ws + p->at_M);
    p->G_src = p->d_G;

    std::vector<char> tables(p->tables_bytes);
    auto put = [&](size_t at, const auto &table) { if (!table.empty()) std::memcpy(tables.data() + at, table.data(), table.size() * sizeof table[0]); };
    std::vector<cr::DevSum> sums;
    std::vector<int32_t> dst;
    if (p->rows_once) {
        std::vector<cr::DevRun> runs, parts;
        for (const cr::RowRun &r : p->work.runs) runs.push_back({r.row_begin, static_cast<int32_t>(r.row_end - r.row_begin), r.dst_begin, r.dst_end, 0, 0, 0});
        for (size_t b = 0; b + 1 < p->work.part_run_begin.size(); ++b) {
            cr::DevRun part = runs[p->work.part_run_begin[b]];           // the part's first run, so that one load starts a workgroup
            part.more_begin = p->work.part_run_begin[b] + 1;
            part.more_end = p->work.part_run_begin[b + 1];
            parts.push_back(part);
        }
        for (const cr::RowSum &sum : p->work.sums) sums.push_back({sum.row_begin, sum.row_end, sum.dst_begin, sum.dst_end});
        dst = p->work.dst;
        if (p->crew) put(p->at_crew_state, std::vector<uint32_t>{1, 0});
        put(p->at_parts, parts);
        put(p->at_runs, runs);
    } else if (stage1) {
        // every piece's partial row lies where its slab's sum reads it: slab by slab, in row order
        std::vector<int32_t> out_row(P);
        for (int32_t i = 0; i < P; ++i) out_row[p->split.slab_pieces[i]] = S + i;
        std::vector<cr::DevPiece> hp(P);
        int64_t visit = 0, longest = 0;
        for (int32_t i = 0; i < P; ++i) longest = std::max(longest, p->split.pieces[i].row_end - p->split.pieces[i].row_begin);
        p->rows_as_buffers = (p->d * elem_size(p)) % 4 == 0 && longest * p->d * elem_size(p) < (int64_t(1) << 31);
        // a row that several holders fetch is left in the caches for them; with no redundancy a large X streams past
        const int32_t shared = p->s > 0 || p->m * p->d * elem_size(p) < kStreamFromBytes ? 1 : 0;
        for (int32_t i = 0; i < P; ++i) {
            const int64_t rows = p->split.pieces[i].row_end - p->split.pieces[i].row_begin;
            hp[i] = {p->split.pieces[i].row_begin, visit, static_cast<int32_t>(rows), shared, out_row[i], 0};
            visit += rows;
        }
        for (int32_t q = 0; q < S; ++q) {
            sums.push_back({S + p->split.slab_piece_begin[q], S + p->split.slab_piece_begin[q + 1], q, q + 1});
            dst.push_back(q);
        }
        put(p->at_pieces, hp);
        put(p->at_team_piece_begin, p->split.team_piece_begin);
    }
    p->num_sums = static_cast<int>(sums.size());
    p->rows_summed = 0;
    for (const cr::DevSum &sum : sums) p->rows_summed += sum.row_end - sum.row_begin;
    put(p->at_sums, sums);
    put(p->at_dst, dst);
    put(p->at_node_begin, p->node_slab_begin);
    put(p->at_slab_coef, p->slab_coef);
    if (stage1) CR_HIP(hipMemcpy(p->ws, tables.data(), tables.size(), hipMemcpyHostToDevice));
    else if (p->tree_arguments) CR_HIP(keep_tables(p, tables.data() + p->at_node_begin));
    p->l2_sharing = -1;
    if (P > 0 && (p->split_kind_used == CR_SPLIT_ROW_CELLS || p->split_kind_used == CR_SPLIT_SHARED_CELLS)) {
        int rc = check_l2_sharing(p);
        if (rc != CR_OK) return rc;
    }
    if (!p->h_staging) {
        const size_t programs = p->program_bytes * kProgramSlots * kStagingHalves, tree_tables = p->tree_arguments ? p->tables_bytes - p->at_node_begin : 0;
        CR_HIP(hipHostMalloc(reinterpret_cast<void **>(&p->h_staging), programs + tree_tables, hipHostMallocDefault));
        std::memcpy(p->h_staging + programs, tables.data() + p->at_node_begin, tree_tables);
        for (int i = 0; i < kStagingHalves; ++i) CR_HIP(hipEventCreateWithFlags(&p->staging_done[i], hipEventDisableTiming));
    }
    p->bound = true;
    p->slabs_here = false;
    p->have_grads = false;
    p->have_messages = false;
    return CR_OK;
} catch (const std::bad_alloc &) {
    return fail(CR_E_NOMEM, "out of host memory");
}

int cr_partial_grads(cr_plan_t *p, const void *X, const float *y, const float *w)
{
    if (!p || !X || !y || !w) return fail(CR_E_INVAL, "NULL argument");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    if (p->model == CR_AGGREGATE_ONLY) return fail(CR_E_STATE, "aggregation-only plan: use cr_load_partial_grads");
    if (reinterpret_cast<uintptr_t>(X) % 16 != 0) return fail(CR_E_INVAL, "X must be 16-byte aligned");
    const int64_t S = static_cast<int64_t>(p->slabs.size()), P = static_cast<int64_t>(p->split.pieces.size());
    const int logistic = p->model == CR_LOGISTIC ? 1 : 0;
    {
        // what the method must move: every holder reads its rows and targets once, each slab gradient is written once
        const int64_t bytes = p->row_visits * p->d * elem_size(p) + p->row_visits * 4 + S * p->d * 4 + p->d * 4;
        LaunchTimer t(p, CR_K_PARTIAL_GRADS, bytes);
        const cr::OnceVariant *once = p->once ? p->once : p->wide_variant;
        if (once) {
            CR_HIP(cr::launch_rows_once(*once, X, y, w, p->d_parts, static_cast<int>(p->work.part_run_begin.size()) - 1, p->d_runs, p->d_dst,
                                        p->d_G, p->d, logistic, p->streams, p->stream));
        } else if (p->crew) {
            CR_HIP(cr::launch_rows_once_crew(*p->crew, X, y, w, p->d_parts, static_cast<int>(p->work.part_run_begin.size()) - 1, p->d_runs, p->d_dst,
                                             p->d_G, p->d, logistic, p->streams, p->d_crew_slots, p->d_crew_state, p->patience, p->stream));
        } else if (p->rows_once) {
            const int64_t cached_from = std::max<int64_t>(0, p->m - kKeptBytes / (p->d * elem_size(p)));
            CR_HIP(cr::launch_wide_once(p->x_dtype, X, y, w, p->d_residuals, p->m, p->d_parts, static_cast<int>(p->work.part_run_begin.size()) - 1,
                                        p->d_runs, p->d_dst, p->d_G, p->d, logistic, cached_from, p->units, p->stream));
        } else if (p->variant) {
            CR_HIP(cr::launch_partial_grads(*p->variant, X, y, w, p->d_pieces, p->d_team_piece_begin, p->split.teams, p->d_G, p->d, logistic,
                                            p->rows_as_buffers, p->stream));
        } else {
            CR_HIP(cr::launch_residuals(p->x_dtype, X, y, w, p->d_pieces, static_cast<int>(P), p->d_residuals, p->d, logistic, p->stream));
            CR_HIP(cr::launch_xt_residuals(p->x_dtype, X, p->d_pieces, static_cast<int>(P), p->d_residuals, p->d_G, p->d, p->stream));
        }
        t.done();
    }
    if (p->num_sums > 0) {
        LaunchTimer t(p, CR_K_REDUCE_PIECES, ((p->rows_once ? p->work.partials : P) + S) * p->d * 4);
        CR_HIP(cr::launch_sum_rows(p->d_G, p->d_sums, p->num_sums, p->rows_summed, p->d_dst, p->d, p->stream));
        t.done();
    }
    p->G_src = p->d_G;
    p->slabs_here = true;
    p->have_grads = true;
    p->have_messages = false;
    return CR_OK;
}

int cr_load_partial_grads(cr_plan_t *p, const float *G)
{
    if (!p || !G) return fail(CR_E_INVAL, "NULL argument");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    if (reinterpret_cast<uintptr_t>(G) % 16 != 0) return fail(CR_E_INVAL, "G must be 16-byte aligned");
    p->G_src = G;
    p->slabs_here = false;
    p->have_grads = true;
    p->have_messages = false;
    return CR_OK;
}

namespace {

struct ProgramCounts { int64_t active_slabs = 0, stored_msgs = 0; int terms = 0; cr::DecTerms dec; };

// Which messages a mask's launches write to memory.  Nobody can read the messages of one call of several masks before the call is done
// but its own decode: a node's message is then the one of the last mask under which it sends, and the earlier ones need not leave the
// chip.  15 to 22 % of an aggregation's bytes are messages.
struct Stores {
    enum { kAll = -1, kNone = -2 };
    int step = kAll;                                     // or the step of a call of several, whose last_send is filled in
    bool first_level = true;                             // the master's children's in any case: a launch of its own decodes
};
bool stored(const cr_plan_t *p, const Stores &stores, int32_t node)
{
    return stores.step == Stores::kAll || (stores.first_level && node < p->n) || (stores.step >= 0 && p->last_send[node] == stores.step);
}

void note_last_sends(cr_plan_t *p, const uint8_t *masks, int steps)
{
    const int32_t N = p->tree.N;
    for (int t = 0; t < steps; ++t)
        for (int32_t i = 0; i < N; ++i)
            if (!masks[static_cast<size_t>(t) * N + i]) p->last_send[i] = t;
}

void decode_terms(int n, const uint8_t *mask, const double *row, cr::DecTerms *dec)
{
    dec->count = dec->pad = 0;
    for (int j = 0; j < n; ++j)
        if (!mask[j] && row[j] != 0.0) {
            dec->row[dec->count] = j;
            dec->coef[dec->count++] = row[j];
        }
}

// Turns a straggler mask into the encode program of one iteration, written into the host block h (program_bytes long, laid out
// by compute_layout): the post-order term list of every level-1 sub-tree; the master's decode terms go into *counts.  Any group
// beyond tolerance fails the call before anything is written (CR_E_UNDECODABLE).
int build_program(cr_plan_t *p, const uint8_t *mask, const Stores &stores, char *h, ProgramCounts *counts)
{
    const int n = p->n, L = p->L;
    const int32_t N = p->tree.N, groups = N / n;
    // decode row of every sibling group
    std::vector<const double *> rows(groups);
    for (int32_t g = 0; g < groups; ++g) {
        int rc = group_decode_row(p, mask + static_cast<size_t>(g) * n, &rows[g]);
        if (rc == CR_E_UNDECODABLE) return fail(rc, "sibling group " + std::to_string(g) + " has more than s stragglers");
        if (rc != CR_OK) return rc;
    }
    int32_t *t_slab = reinterpret_cast<int32_t *>(h + p->off_slab);
    int32_t *t_level = reinterpret_cast<int32_t *>(h + p->off_level);
    int32_t *t_row = reinterpret_cast<int32_t *>(h + p->off_row);
    double *t_coef = reinterpret_cast<double *>(h + p->off_coef);
    double *t_acoef = reinterpret_cast<double *>(h + p->off_acoef);
    auto put = [&](size_t t, int32_t slab, double coef) { t_slab[t] = slab; t_level[t] = 0; t_row[t] = 0; t_coef[t] = coef; t_acoef[t] = 0.0; };
    int32_t *sub = reinterpret_cast<int32_t *>(h + p->off_sub);

    // Post-order program of every level-1 sub-tree.  The messages of a straggler's children are used by nobody, but the kernel folds
    // them into the sum of the straggler's level, times zero, which is not nothing where they are not finite.  What hangs below
    // stragglers therefore comes after all else, below stragglers of the first levels first: a level's sum is then used no more once
    // it has taken such a message.
    size_t nt = 0;
    struct Frame { int32_t node; int level; int next_child; };
    std::vector<Frame> stack;
    std::vector<int32_t> below[cr::kMaxLevels + 1];       // children of stragglers, by their own level
    auto walk = [&](int32_t root, int root_level) {
        stack.push_back({root, root_level, 0});
        while (!stack.empty()) {
            Frame &f = stack.back();
            if (f.level < L && f.next_child < n) {
                const int32_t child = p->tree.level_offset[f.level + 1] + (f.node - p->tree.level_offset[f.level]) * n + f.next_child;
                ++f.next_child;
                if (mask[f.node]) below[f.level + 1].push_back(child);
                else stack.push_back({child, f.level + 1, 0});
                continue;
            }
            const int32_t node = f.node;
            const int level = f.level;
            stack.pop_back();
            if (mask[node]) continue;                     // a straggler sends nothing
            double acoef = 0.0;
            if (level >= 2) {
                const int32_t parent = p->tree.level_offset[level - 1] + (node - p->tree.level_offset[level]) / n;
                if (!mask[parent]) acoef = rows[node / n][node % n];
            }
            const int32_t sb = p->node_slab_begin[node], se = p->node_slab_begin[node + 1];
            for (int32_t q = sb; q < se; ++q) put(nt++, q, p->slabs[q].coef);
            if (se == sb) put(nt++, 0, 0.0);              // a node without rows still sends its children's combination
            t_level[nt - 1] = level;                      // the node's last term finishes it
            const bool put_down = stored(p, stores, node);
            t_row[nt - 1] = put_down ? node : ~node;
            t_acoef[nt - 1] = acoef;
            counts->active_slabs += se - sb;
            counts->stored_msgs += put_down;
        }
    };
    for (int i = 0; i < n; ++i) {
        sub[i] = static_cast<int32_t>(nt);
        below[1].assign(1, i);
        for (int level = 1; level <= L; ++level) {
            for (size_t k = 0; k < below[level].size(); ++k) walk(below[level][k], level);
            below[level].clear();
        }
        const size_t real_terms = nt - static_cast<size_t>(sub[i]);
        while (nt % cr::kEncodeUnroll != 0) {             // pad with no-op terms on an already fetched slab
            put(nt, nt > 0 ? t_slab[nt - 1] : 0, 0.0);
            ++nt;
        }
        sub[n + i] = sub[i] + static_cast<int32_t>(real_terms);
    }
    decode_terms(n, mask, rows[0], &counts->dec);
    double *dec = reinterpret_cast<double *>(h + p->off_dec);
    for (int j = 0; j < n; ++j) dec[j] = mask[j] ? 0.0 : rows[0][j];
    counts->terms = static_cast<int>(nt);                // padding included
    return CR_OK;
}

// The same for the tree kernels: a coefficient per node, and whether its message is written.
int build_coefs(cr_plan_t *p, const uint8_t *mask, const Stores &stores, cr::NodeCoefs *coefs, cr::NodeBits *bits, ProgramCounts *counts)
{
    *bits = cr::NodeBits();
    const int n = p->n;
    double straggler;
    std::memcpy(&straggler, &cr::kStraggler, sizeof straggler);
    for (int32_t g = 0; g < p->tree.N / n; ++g) {
        const double *row = nullptr;
        int rc = group_decode_row(p, mask + static_cast<size_t>(g) * n, &row);
        if (rc == CR_E_UNDECODABLE) return fail(rc, "sibling group " + std::to_string(g) + " has more than s stragglers");
        if (rc != CR_OK) return rc;
        if (g == 0) decode_terms(n, mask, row, &counts->dec);
        for (int j = 0; j < n; ++j) {
            const int32_t node = g * n + j;
            coefs->a[node] = mask[node] ? straggler : row[j];
            if (mask[node]) continue;
            counts->active_slabs += p->node_slab_begin[node + 1] - p->node_slab_begin[node];
            if (!stored(p, stores, node)) continue;
            bits->word[node / 32] |= 1u << node % 32;
            counts->stored_msgs += 1;
        }
    }
    return CR_OK;
}

// the program's arrays in a program block, in host or device memory
cr::ProgramTables program_tables(const cr_plan_t *p, char *block)
{
    return {reinterpret_cast<int32_t *>(block + p->off_slab), reinterpret_cast<int32_t *>(block + p->off_level), reinterpret_cast<int32_t *>(block + p->off_row),
            reinterpret_cast<double *>(block + p->off_coef), reinterpret_cast<double *>(block + p->off_acoef), reinterpret_cast<int32_t *>(block + p->off_sub)};
}

// the program's arrays as the encode kernel takes them, for a program block at device address d_program
cr::EncProgram program_view(const cr_plan_t *p, const char *d_program)
{
    cr::EncProgram prog;
    prog.slab = reinterpret_cast<const int32_t *>(d_program + p->off_slab);
    prog.level = reinterpret_cast<const int32_t *>(d_program + p->off_level);
    prog.row = reinterpret_cast<const int32_t *>(d_program + p->off_row);
    prog.coef = reinterpret_cast<const double *>(d_program + p->off_coef);
    prog.acoef = reinterpret_cast<const double *>(d_program + p->off_acoef);
    prog.sub_begin = reinterpret_cast<const int32_t *>(d_program + p->off_sub);
    prog.sub_end = prog.sub_begin + p->n;
    prog.dec = reinterpret_cast<const double *>(d_program + p->off_dec);
    return prog;
}

}  // namespace

namespace {

// every group of every mask within tolerance?  (checked before anything is enqueued or any staging is touched)
int check_masks(const cr_plan_t *p, const uint8_t *masks, int steps)
{
    const int n = p->n;
    const int32_t N = p->tree.N;
    for (int t = 0; t < steps; ++t)
        for (int32_t grp = 0; grp < N / n; ++grp) {
            int cnt = 0;
            for (int j = 0; j < n; ++j) cnt += masks[static_cast<size_t>(t) * N + static_cast<size_t>(grp) * n + j] ? 1 : 0;
            if (cnt > p->s)
                return fail(CR_E_UNDECODABLE, (steps > 1 ? "step " + std::to_string(t) + ": " : std::string()) + "sibling group " + std::to_string(grp) +
                                                  " has more than s stragglers");
        }
    return CR_OK;
}

// Builds the encode programs of `count` <= kProgramSlots masks in pinned staging and sends them to program slots 0 .. count-1 with
// one copy on the plan's stream (which therefore follows every kernel that still reads the slots).  counts[i] describes program i.
int upload_programs(cr_plan_t *p, const uint8_t *masks, int count, Stores stores, ProgramCounts *counts)
{
    const int half = p->staging_next;
    if (p->staging_used[half]) CR_HIP(hipEventSynchronize(p->staging_done[half]));     // the copy that last read this half is done
    char *h = p->h_staging + static_cast<size_t>(half) * kProgramSlots * p->program_bytes;
    for (int i = 0; i < count; ++i) {
        counts[i] = ProgramCounts();
        int rc = build_program(p, masks + static_cast<size_t>(i) * p->tree.N, stores, h + static_cast<size_t>(i) * p->program_bytes, &counts[i]);
        if (rc != CR_OK) return rc;
        if (stores.step >= 0) ++stores.step;
    }
    p->staging_next = (half + 1) % kStagingHalves;
    CR_HIP(hipMemcpyAsync(p->d_program, h, static_cast<size_t>(count) * p->program_bytes, hipMemcpyHostToDevice, p->stream));
    CR_HIP(hipEventRecord(p->staging_done[half], p->stream));
    p->staging_used[half] = true;
    return CR_OK;
}

int encode_slot(cr_plan_t *p, int slot, const ProgramCounts &counts)
{
    LaunchTimer t(p, CR_K_ENCODE, (counts.active_slabs + counts.stored_msgs) * p->d * 4);
    CR_HIP(cr::launch_encode(p->G_src, p->d_M, program_view(p, p->d_program + static_cast<size_t>(slot) * p->program_bytes), p->n, p->L, p->d, p->stream));
    t.done();
    p->dec = counts.dec;
    p->have_messages = true;
    return CR_OK;
}

// vectors that a gradient step reads and writes besides g
int64_t step_rows(const cr::GradientStep &step) { return (step.w ? 2 : 0) + (step.measures && step.w_star ? 1 : 0); }

// What the tree kernels take of the tree and a mask.
struct MaskTables {
    bool as_arguments = false;
    cr::DeviceTables device;                             // the coefficients of the mask in any case
    cr::ArgumentTables arguments;
    cr::NodeBits stored;
};

// The tables in the workspace are those that were written there with stage 1's, and stand as long as its slabs do.  With slabs of the
// caller's nothing in the workspace is relied on: the tables are in the plan's pages, or travel as kernel arguments, or, where they do not fit, in a
// copy from pinned memory, once per call (*sent).
int mask_tables(cr_plan_t *p, const uint8_t *mask, const Stores &stores, bool slabs_here, MaskTables *t, ProgramCounts *counts, bool *sent)
{
    *counts = ProgramCounts();
    int rc = build_coefs(p, mask, stores, &t->device.coefs, &t->stored, counts);
    if (rc != CR_OK) return rc;
    t->device.node_begin = p->d_node_begin;
    t->device.slab_coef = p->d_slab_coef;
    const bool there = slabs_here || p->pool_first >= 0;
    t->as_arguments = !there && cr::argument_tables(*p->tree_arguments, t->device.coefs, &t->arguments);
    if (there || t->as_arguments || *sent) return CR_OK;
    CR_HIP(hipMemcpyAsync(p->ws + p->at_node_begin, p->h_staging + p->program_bytes * kProgramSlots * kStagingHalves, p->tables_bytes - p->at_node_begin,
                          hipMemcpyHostToDevice, p->stream));
    *sent = true;
    return CR_OK;
}

int encode_tree(cr_plan_t *p, const MaskTables &tables, const ProgramCounts &counts)
{
    LaunchTimer t(p, CR_K_ENCODE, (counts.active_slabs + counts.stored_msgs) * p->d * 4);
    CR_HIP(tables.as_arguments ? cr::launch_tree_encode(p->G_src, p->d_M, tables.arguments, tables.stored, p->n, p->L, p->d, p->stream)
                               : cr::launch_tree_encode(p->G_src, p->d_M, tables.device, tables.stored, p->n, p->L, p->d, p->stream));
    t.done();
    p->dec = counts.dec;
    p->have_messages = true;
    return CR_OK;
}

// the master's decode; with step.w the gradient step w <- w - lr g rides in the same launch
int decode_root(cr_plan_t *p, float *g, const cr::GradientStep &step)
{
    if (!p || !g) return fail(CR_E_INVAL, "NULL argument");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    if (!p->have_messages) return fail(CR_E_STATE, "no messages yet: call cr_encode_tree first");
    LaunchTimer t(p, CR_K_DECODE, (p->dec.count + 1 + step_rows(step)) * p->d * 4);
    CR_HIP(cr::launch_decode(p->d_M, g, p->dec, step, p->d, p->stream));
    t.done();
    return CR_OK;
}

// Does the decoded vector lie among the slabs?  Encode and decode are then launches of their own: in one, a workgroup would decode over
// slabs that another has yet to read.
bool overlap(const float *a, int64_t a_floats, const float *b, int64_t b_floats)
{
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + static_cast<uintptr_t>(b_floats) * sizeof(float) && y < x + static_cast<uintptr_t>(a_floats) * sizeof(float);
}

// encode, decode and gradient step in one launch, which counts as the encode's
int encode_decode(cr_plan_t *p, const MaskTables &tables, const ProgramCounts &counts, float *g, const cr::GradientStep &step)
{
    LaunchTimer t(p, CR_K_ENCODE, (counts.active_slabs + counts.stored_msgs + 1 + step_rows(step)) * p->d * 4);
    CR_HIP(tables.as_arguments ? cr::launch_tree_encode_decode(p->G_src, p->d_M, tables.arguments, tables.stored, p->n, p->L, g, step, p->d, p->stream)
                               : cr::launch_tree_encode_decode(p->G_src, p->d_M, tables.device, tables.stored, p->n, p->L, g, step, p->d, p->stream));
    t.done();
    p->dec = counts.dec;
    p->have_messages = true;
    return CR_OK;
}

}  // namespace

int cr_encode_tree(cr_plan_t *p, const uint8_t *mask)
{
    if (!p || !mask) return fail(CR_E_INVAL, "NULL argument");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    if (!p->have_grads) return fail(CR_E_STATE, "no partial gradients yet");
    ProgramCounts counts;
    if (cr::tree_side_by_side(p->shape, p->d, cr::Otherwise::kCopy)) {
        MaskTables tables;
        bool sent = false;
        int rc = mask_tables(p, mask, Stores(), p->slabs_here, &tables, &counts, &sent);
        if (rc != CR_OK) return rc;
        return encode_tree(p, tables, counts);
    }
    int rc = check_masks(p, mask, 1);
    if (rc != CR_OK) return rc;
    rc = upload_programs(p, mask, 1, Stores(), &counts);
    if (rc != CR_OK) return rc;
    return encode_slot(p, 0, counts);
}

int cr_decode_root(cr_plan_t *p, float *g) { return decode_root(p, g, cr::GradientStep()); }

int cr_gd_update(cr_plan_t *p, float *w, const float *g, float lr)
{
    if (!p || !w || !g) return fail(CR_E_INVAL, "NULL argument");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    LaunchTimer t(p, CR_K_UPDATE, 3 * p->d * 4);
    CR_HIP(cr::launch_update(w, g, lr, p->d, p->stream));
    t.done();
    return CR_OK;
}

int cr_gd_run(cr_plan_t *p, const void *X, const float *y, float *w, float *g, const uint8_t *masks, int steps, float lr,
              const float *w_star, float *metrics)
{
    if (!p || !X || !y || !w || !g || !masks) return fail(CR_E_INVAL, "NULL argument");
    if (steps < 0) return fail(CR_E_INVAL, "steps must be >= 0");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    if (p->model == CR_AGGREGATE_ONLY) return fail(CR_E_STATE, "aggregation-only plan has no gradient stage");
    int rc = check_masks(p, masks, steps);              // every mask is checked before anything is enqueued
    if (rc != CR_OK) return rc;
    const int32_t N = p->tree.N;
    const bool side_by_side = cr::tree_side_by_side(p->shape, p->d, cr::Otherwise::kBatch);
    // vectors of the caller's that lie among the messages: everything in its place and in launches of its own, as the separate calls leave it
    auto lies_there = [&](const void *x, int64_t floats) { return x && overlap(static_cast<const float *>(x), floats, p->d_M, N * p->d); };
    const bool among_messages = lies_there(g, p->d) || lies_there(w, p->d) || lies_there(w_star, p->d) || lies_there(y, p->m) ||
                                lies_there(X, (p->m * p->d * elem_size(p) + 3) / 4) || lies_there(metrics, 2 * static_cast<int64_t>(steps));
    const bool one_for_two = overlap(w, p->d, g, p->d) || (w_star && (overlap(w_star, p->d, w, p->d) || overlap(w_star, p->d, g, p->d)));
    const bool together = cr::tree_and_decode_together(p->shape, p->d) && !among_messages && !one_for_two &&
                          !overlap(g, p->d, p->d_G, static_cast<int64_t>(p->slabs.size()) * p->d);
    note_last_sends(p, masks, steps);
    ProgramCounts counts[kProgramSlots];
    MaskTables tables;
    bool sent = false;
    for (int t0 = 0; t0 < steps; t0 += kProgramSlots) {
        const int count = std::min(kProgramSlots, steps - t0);
        auto stores = [&](int i) { return Stores{among_messages ? Stores::kAll : t0 + i, !together}; };
        // where the tree's kernels take programs, those of the next kProgramSlots steps travel in one copy
        if (!side_by_side) {
            rc = upload_programs(p, masks + static_cast<size_t>(t0) * N, count, stores(0), counts);
            if (rc != CR_OK) return rc;
        }
        for (int i = 0; i < count; ++i) {
            cr::GradientStep step;
            step.w = w;
            step.lr = lr;
            step.w_star = w_star;
            step.measures = metrics ? p->d_measures + i * p->measures_stride : nullptr;
            if (side_by_side) rc = mask_tables(p, masks + static_cast<size_t>(t0 + i) * N, stores(i), true, &tables, &counts[i], &sent);
            if (rc == CR_OK) rc = cr_partial_grads(p, X, y, w);
            if (together) {
                if (rc == CR_OK) rc = encode_decode(p, tables, counts[i], g, step);
            } else {
                if (rc == CR_OK) rc = side_by_side ? encode_tree(p, tables, counts[i]) : encode_slot(p, i, counts[i]);
                if (rc == CR_OK) rc = decode_root(p, g, step);
            }
            if (rc != CR_OK) return rc;
        }
        if (metrics) {
            const int groups = together ? cr::tree_decode_groups(p->n, p->L, p->d) : cr::decode_groups(p->d);
            LaunchTimer tm(p, CR_K_UPDATE, static_cast<int64_t>(count) * groups * 32);
            CR_HIP(cr::launch_measures(p->d_measures, static_cast<int64_t>(p->measures_stride), groups, count, w_star != nullptr,
                                       metrics + 2 * static_cast<size_t>(t0), p->stream));
            tm.done();
        }
    }
    return CR_OK;
}

int cr_aggregate_run(cr_plan_t *p, const float *G, int64_t G_step_stride, const uint8_t *masks, int steps, float *g, int64_t g_step_stride)
{
    if (!p || !G || !masks || !g) return fail(CR_E_INVAL, "NULL argument");
    if (steps < 0 || G_step_stride < 0 || g_step_stride < 0) return fail(CR_E_INVAL, "steps and strides must be >= 0");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    if (reinterpret_cast<uintptr_t>(G) % 16 != 0 || (G_step_stride * sizeof(float)) % 16 != 0) return fail(CR_E_INVAL, "G and its step stride must be 16-byte aligned");
    int rc = check_masks(p, masks, steps);
    if (rc != CR_OK) return rc;
    const int32_t N = p->tree.N;
    if (steps > 0) p->slabs_here = false;
    const int64_t more = std::max(0, steps - 1);
    const bool in_place = overlap(g, p->d + more * g_step_stride, G, static_cast<int64_t>(p->slabs.size()) * p->d + more * G_step_stride);
    // vectors of the caller's that lie among the messages: everything in its place and in launches of its own, as the separate calls leave it
    const bool among_messages = overlap(g, p->d + more * g_step_stride, p->d_M, N * p->d) ||
                                overlap(G, static_cast<int64_t>(p->slabs.size()) * p->d + more * G_step_stride, p->d_M, N * p->d);
    // one launch for several masks leaves the order in which workgroups decode open: vectors that overlap in part need it
    const bool in_order = in_place || among_messages || (g_step_stride > 0 && g_step_stride < p->d);
    const bool together = cr::tree_and_decode_together(p->shape, p->d) && !in_place && !among_messages;
    note_last_sends(p, masks, steps);
    ProgramCounts counts[kProgramSlots];
    MaskTables tables;
    bool sent = false;
    for (int t0 = 0; t0 < steps; t0 += kProgramSlots) {
        const int count = std::min(kProgramSlots, steps - t0);
        // one mask: the nodes side by side need no copy of a program; beyond 81 920 columns one launch for everything makes up for it
        const bool alone = count == 1 && cr::tree_side_by_side(p->shape, p->d, cr::Otherwise::kCopy) &&
                           (p->d <= 81920 || in_order || !cr::encode_in_steps(p->shape, p->d, 1));
        const bool in_steps = !in_order && !alone && cr::encode_in_steps(p->shape, p->d, count);
        const bool side_by_side = alone || cr::tree_side_by_side(p->shape, p->d, cr::Otherwise::kBatch);
        auto stores = [&](int i) { return Stores{among_messages ? Stores::kAll : t0 + i, !in_steps && !together}; };
        if (in_steps || !side_by_side) {
            rc = upload_programs(p, masks + static_cast<size_t>(t0) * N, count, stores(0), counts);
            if (rc != CR_OK) return rc;
        }
        if (in_steps) {
            int64_t rows = 0;
            for (int i = 0; i < count; ++i) rows += counts[i].active_slabs + counts[i].stored_msgs + 1;
            p->G_src = G + static_cast<int64_t>(t0 + count - 1) * G_step_stride;
            p->have_grads = true;
            LaunchTimer t(p, CR_K_ENCODE, rows * p->d * 4);
            CR_HIP(cr::launch_encode_steps(G + static_cast<int64_t>(t0) * G_step_stride, G_step_stride, p->d_M, program_view(p, p->d_program),
                                           static_cast<int64_t>(p->program_bytes), count, p->n, p->L, g + static_cast<int64_t>(t0) * g_step_stride,
                                           g_step_stride, p->d, p->stream));
            t.done();
            p->dec = counts[count - 1].dec;
            p->have_messages = true;
            continue;
        }
        for (int i = 0; i < count; ++i) {
            float *out = g + static_cast<int64_t>(t0 + i) * g_step_stride;
            if (side_by_side) rc = mask_tables(p, masks + static_cast<size_t>(t0 + i) * N, stores(i), false, &tables, &counts[i], &sent);
            if (rc != CR_OK) return rc;
            p->G_src = G + static_cast<int64_t>(t0 + i) * G_step_stride;
            p->have_grads = true;
            if (together) rc = encode_decode(p, tables, counts[i], out, cr::GradientStep());
            else {
                rc = side_by_side ? encode_tree(p, tables, counts[i]) : encode_slot(p, i, counts[i]);
                if (rc == CR_OK) rc = decode_root(p, out, cr::GradientStep());
            }
            if (rc != CR_OK) return rc;
        }
    }
    return CR_OK;
}

int cr_aggregate_static(cr_plan_t *p, const float *G, const uint8_t *mask, float *g, void *hip_stream)
{
    static_assert(CR_STATIC_SCRATCH_BYTES == cr::kStaticScratchBytes, "the header states the size of the library's device array");
    if (!p || !G || !mask || !g) return fail(CR_E_INVAL, "NULL argument");
    if (reinterpret_cast<uintptr_t>(G) % 16 != 0) return fail(CR_E_INVAL, "G must be 16-byte aligned");
    if (p->program_bytes == 0) {                        // offsets of the program's arrays: host arithmetic only
        size_t unused = 0;
        compute_layout(p, &unused);
    }
    const size_t msg_bytes = static_cast<size_t>(p->tree.N) * static_cast<size_t>(p->d) * sizeof(float);
    if (p->program_bytes > cr::kStaticProgramBytes)
        return fail(CR_E_INVAL, "cr_aggregate_static: the encode program of this tree (" + std::to_string(p->program_bytes) + " bytes) exceeds 64 KiB");
    if (msg_bytes > cr::kStaticScratchBytes - cr::kStaticProgramBytes)
        return fail(CR_E_INVAL, "cr_aggregate_static: N * d * 4 = " + std::to_string(msg_bytes) + " bytes of messages exceed the library's device array (" +
                                    std::to_string(cr::kStaticScratchBytes - cr::kStaticProgramBytes) + " bytes)");
    ProgramCounts counts;
    char *base = nullptr;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (cr::tree_side_by_side(p->shape, p->d, cr::Otherwise::kLaunches) && p->tree_arguments->fits) {
        cr::NodeCoefs coefs;
        cr::NodeBits stored;
        cr::ArgumentTables tables;
        const bool together = cr::tree_and_decode_together(p->shape, p->d) && !overlap(g, p->d, G, static_cast<int64_t>(p->slabs.size()) * p->d);
        int rc = build_coefs(p, mask, {Stores::kNone, !together}, &coefs, &stored, &counts);
        if (rc != CR_OK) return rc;
        if (cr::argument_tables(*p->tree_arguments, coefs, &tables)) {
            CR_HIP(cr::static_scratch(&base));          // this device's copy of the array; never the array's name
            float *M = reinterpret_cast<float *>(base + cr::kStaticProgramBytes);
            if (together) {
                CR_HIP(cr::launch_tree_encode_decode(G, M, tables, stored, p->n, p->L, g, cr::GradientStep(), p->d, stream));
            } else {
                CR_HIP(cr::launch_tree_encode(G, M, tables, stored, p->n, p->L, p->d, stream));
                CR_HIP(cr::launch_decode(M, g, counts.dec, cr::GradientStep(), p->d, stream));
            }
            return CR_OK;
        }
        counts = ProgramCounts();
    }
    if (p->static_program.size() != p->program_bytes) p->static_program.assign(p->program_bytes, 0);
    int rc = build_program(p, mask, {Stores::kNone, true}, p->static_program.data(), &counts);
    if (rc != CR_OK) return rc;
    CR_HIP(cr::static_scratch(&base));
    float *M = reinterpret_cast<float *>(base + cr::kStaticProgramBytes);
    CR_HIP(cr::launch_program(program_tables(p, base), program_tables(p, p->static_program.data()), counts.terms, 2 * p->n, stream));
    CR_HIP(cr::launch_encode(G, M, program_view(p, base), p->n, p->L, p->d, stream));
    CR_HIP(cr::launch_decode(M, g, counts.dec, cr::GradientStep(), p->d, stream));
    return CR_OK;
}

int cr_get_slab_grads(const cr_plan_t *p, const float **G)
{
    if (!p || !G) return fail(CR_E_INVAL, "NULL argument");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    *G = p->G_src;
    return CR_OK;
}

int cr_get_messages(const cr_plan_t *p, const float **M)
{
    if (!p || !M) return fail(CR_E_INVAL, "NULL argument");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    *M = p->d_M;
    return CR_OK;
}

int cr_profile_enable(cr_plan_t *p, int kernels)
{
    if (!p) return fail(CR_E_INVAL, "NULL plan");
    if (p->bound) {
        CR_HIP(hipStreamSynchronize(p->stream));
        int rc = fold_timings(p);
        if (rc != CR_OK) return rc;
    }
    if (kernels < 0 || kernels > CR_PROFILE_ALL) return fail(CR_E_INVAL, "kernel mask out of range");
    if (kernels) {                                      // a new selection starts new totals
        for (int k = 0; k < CR_K_COUNT; ++k) { p->total_ms[k] = 0.0; p->launches[k] = 0; p->bytes_sum[k] = 0; p->samples[k].clear(); }
    }
    p->profiling = static_cast<unsigned>(kernels);
    return CR_OK;
}

int cr_profile_read(cr_plan_t *p, int kernel, double *total_ms, int64_t *launches, int64_t *algorithmic_bytes)
{
    if (!p || kernel < 0 || kernel >= CR_K_COUNT) return fail(CR_E_INVAL, "bad argument");
    if (p->bound) {
        CR_HIP(hipStreamSynchronize(p->stream));
        int rc = fold_timings(p);
        if (rc != CR_OK) return rc;
    }
    if (total_ms) *total_ms = p->total_ms[kernel];
    if (launches) *launches = p->launches[kernel];
    if (algorithmic_bytes) *algorithmic_bytes = p->bytes_sum[kernel];
    return CR_OK;
}

int cr_profile_samples(cr_plan_t *p, int kernel, float *ms, int64_t capacity, int64_t *count)
{
    if (!p || !count || kernel < 0 || kernel >= CR_K_COUNT || capacity < 0 || (capacity > 0 && !ms)) return fail(CR_E_INVAL, "bad argument");
    if (p->bound) {
        CR_HIP(hipStreamSynchronize(p->stream));
        int rc = fold_timings(p);
        if (rc != CR_OK) return rc;
    }
    const std::vector<float> &v = p->samples[kernel];
    const int64_t n = std::min<int64_t>(capacity, static_cast<int64_t>(v.size()));
    std::copy(v.begin(), v.begin() + n, ms);
    *count = static_cast<int64_t>(v.size());
    return CR_OK;
}

int cr_probe_read_bandwidth(const void *src, size_t bytes, float *sink, int launches, void *hip_stream, double *gbps)
{
    if (!src || !sink || !gbps) return fail(CR_E_INVAL, "NULL argument");
    if (bytes < (size_t(1) << 20) || bytes % 16 != 0 || reinterpret_cast<uintptr_t>(src) % 16 != 0)
        return fail(CR_E_INVAL, "src must be 16-byte aligned, bytes a multiple of 16 and at least 1 MiB");
    if (launches < 1 || launches > 1000) return fail(CR_E_INVAL, "launches must be 1..1000");
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    hipEvent_t start = nullptr, stop = nullptr;
    CR_HIP(hipEventCreate(&start));
    if (hipEventCreate(&stop) != hipSuccess) { (void)hipEventDestroy(start); return fail(CR_E_HIP, "hipEventCreate failed"); }
    hipError_t e = cr::launch_stream_read(src, bytes / 16, sink, stream);                 // warm-up
    if (e == hipSuccess) e = hipEventRecord(start, stream);
    for (int i = 0; i < launches && e == hipSuccess; ++i) e = cr::launch_stream_read(src, bytes / 16, sink, stream);
    if (e == hipSuccess) e = hipEventRecord(stop, stream);
    if (e == hipSuccess) e = hipEventSynchronize(stop);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, start, stop);
    (void)hipEventDestroy(start);
    (void)hipEventDestroy(stop);
    if (e != hipSuccess) return fail(CR_E_HIP, std::string("read-bandwidth probe: ") + hipGetErrorString(e));
    *gbps = static_cast<double>(bytes) * launches / (static_cast<double>(ms) * 1e-3) / 1e9;
    return CR_OK;
}

int cr_last_algorithmic_bytes(const cr_plan_t *p, int kernel, int64_t *bytes)
{
    if (!p || !bytes || kernel < 0 || kernel >= CR_K_COUNT) return fail(CR_E_INVAL, "bad argument");
    *bytes = p->bytes_last[kernel];
    return CR_OK;
}

int cr_synchronize(cr_plan_t *p)
{
    if (!p) return fail(CR_E_INVAL, "NULL plan");
    if (!p->bound) return fail(CR_E_INVAL, "no workspace bound");
    CR_HIP(hipStreamSynchronize(p->stream));
    return CR_OK;
}

int cr_testing_patience(cr_plan_t *p, int polls)
{
    if (!p || polls < 0) return CR_E_INVAL;
    p->patience = polls;
    return CR_OK;
}

}  // extern "C"
