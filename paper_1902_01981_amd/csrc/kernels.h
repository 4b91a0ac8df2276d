// Device-side tables and kernel launchers of the CodedReduce hot path (gfx950).  Host code sees only plain launch functions.
#pragma once
#include <hip/hip_runtime_api.h>

#include <cstdint>

namespace cr {

struct DevPiece {            // one stage-1 work item: rows [row_begin, row_begin + nrows) of X, partial row = index of the piece
    int64_t row_begin;
    int64_t visit_begin;     // index of the piece's first row among all row visits, piece-major (wide-row path: where its residuals live)
    int32_t nrows;
    int32_t shared;          // 1: other workgroups fetch these rows at the same time, so the fetch should leave them in the L2
    int32_t out_row;         // row of the output table that receives the piece's gradient
    int32_t pad;
};

// Output table of stage 1: rows of d floats, first the slab gradients G[0 .. S), then the partial rows.
struct DevRun {              // rows [row_begin, row_begin + nrows) of X, formed once; the result goes to rows dst[dst_begin .. dst_end)
    int64_t row_begin;
    int32_t nrows;
    int32_t dst_begin, dst_end;
    int32_t more_begin, more_end;   // in the part table: the part's further runs, runs[more_begin .. more_end)
    int32_t pad;
};

struct DevSum {              // rows dst[dst_begin .. dst_end) = sum of rows [row_begin, row_end)
    int32_t row_begin, row_end;
    int32_t dst_begin, dst_end;
};

// Encode program: a post-order list of terms, stored as parallel arrays so that a wavefront fetches kEncodeUnroll terms with a few
// wide scalar loads.  Term t:  own += coef[t] * G[slab[t]];  if level[t] > 0 the term is the last of a node at that level:
// message = own + pending[level], stored to M[row[t]], or not at all where row[t] is negative, and folded into pending[level-1] with
// acoef[t]; own = 0.
struct EncProgram {
    const int32_t *slab;
    const int32_t *level;
    const int32_t *row;
    const double *coef;
    const double *acoef;
    const int32_t *sub_begin;    // first term of each sub-program, a multiple of kEncodeUnroll
    const int32_t *sub_end;      // one past its last real term; no-op terms pad it up to the next multiple of kEncodeUnroll
    const double *dec;           // per level-1 node, what the master's decode takes of its message (0: nothing)
#ifdef __HIPCC__
    // the program that lies `bytes` further on
    __device__ __forceinline__ EncProgram at(int64_t bytes) const
    {
        auto move = [&](auto *p) { return reinterpret_cast<decltype(p)>(reinterpret_cast<const char *>(p) + bytes); };
        return {move(slab), move(level), move(row), move(coef), move(acoef), move(sub_begin), move(sub_end), move(dec)};
    }
#endif
};

struct DecTerms {            // the master's decode: g = sum of coef[j] * M[row[j]]; a kernel argument
    int32_t count, pad;
    int32_t row[64];         // a group has at most 64 members
    double coef[64];
};

// The encode of short vectors takes what the mask decides as a kernel argument: a[node] = the coefficient with which the node's parent
// folds its message in (level 1: the master), or kStraggler: the node sends none.
constexpr int64_t kStraggler = -1;                       // bits of a NaN that no coefficient is
struct NodeCoefs {
    static constexpr int kNodes = 448;                   // kernel arguments take at most 4 KB
    double a[kNodes];
};
// The tree's tables as a kernel argument.  On the device, with the mask's coefficients beside them: the slabs of every node
// (node_begin: one entry per node and one more) and their coefficients.
struct DeviceTables {
    static constexpr size_t kLdsBytes = 0;
    const int32_t *node_begin;
    const double *slab_coef;
    NodeCoefs coefs;
};
// The same for trees of few nodes: what is not sent need not be read either.  20 steps of cr_gd_run on 1 200 x 100 and 12 workers 223 us with 3.7 KB of
// arguments, 218 with half a kilobyte; cr_encode_tree on the host 5.8 and 5.5.
struct SmallDeviceTables {
    static constexpr size_t kLdsBytes = 0;
    static constexpr int kNodes = 48;
    const int32_t *node_begin;
    const double *slab_coef;
    struct { double a[kNodes]; } coefs;
};
// Or all of it in the argument: the distinct coefficients, then 16-bit tables of first slabs and of places among the coefficients.
struct ArgumentTables {
    static constexpr int kWords = 470;
    static constexpr size_t kLdsBytes = kWords * 8;
    int32_t at_begin, at_coef, at_slab, used;            // in 16-bit units; 64-bit words in use
    uint64_t word[kWords];
};
// The nodes whose messages are written to memory: a message that nobody can read before another of the same call replaces it, or that
// lies in the library's own array, is formed and folded in but not stored.
struct NodeBits {
    uint32_t word[NodeCoefs::kNodes / 32] = {};
};
struct SmallArgumentTables {
    static constexpr int kWords = 96;
    static constexpr size_t kLdsBytes = kWords * 8;
    int32_t at_begin, at_coef, at_slab, used;
    uint64_t word[kWords];
};
// What the tree itself puts into ArgumentTables, laid out once per plan; argument_tables completes it for a mask, or says that there
// is no room for the mask's coefficients.
struct TreeArguments {
    static constexpr int kSlots = 1024;                  // of the hash table; there is room for fewer than 470 distinct coefficients
    bool fits = false;                                   // the tree's own part does
    int nodes = 0, values = 0, halves = 0;
    uint16_t slot[kSlots];                               // place of a coefficient among the values by its hash, 0xffff: none
    uint64_t value[ArgumentTables::kWords];
    uint16_t half[4 * ArgumentTables::kWords];           // first slab of every node and one more, place of every node's coefficient, of every slab's
};
void lay_out_tree(int nodes, int slabs, const int32_t *node_begin, const double *slab_coef, TreeArguments *out);
bool argument_tables(const TreeArguments &tree, const NodeCoefs &coefs, ArgumentTables *out);
struct TreeShape {           // what the rules of the encode go by
    int n, L, s, nodes;
    int64_t slabs;
};
// The nodes that a workgroup of the tree kernels has, leaves first, then level by level up: the nodes of level l have the places from
// first[l - 1] on, and place t is node t + shift[l - 1] + sub * width[l - 1] in level-1 sub-tree `sub`.
struct TreeLevels {
    int32_t n, L, total, leaves, threads;        // threads of the workgroup, as an argument: its size is a fetch of its own
    int32_t first[8], shift[8], width[8];
};
// The gradient step that rides in the launch of a decode.
struct GradientStep {
    float *w = nullptr;              // w <- w - lr g, g as stored (rounded to fp32); nullptr: no step
    const float *w_star = nullptr;
    double *measures = nullptr;      // per workgroup |w_new - w|^2, |w|^2, |w_new - w*|^2, |w*|^2 over its columns; nullptr: not wanted
    float lr = 0.f;
};

constexpr int kEncodeUnroll = 8;   // encode sub-programs are padded to a multiple of this many terms
constexpr int kMaxLevels = 8;

// Stage-1 kernels that do every holder's work separately: team size, chunks per thread, rows per step, teams per workgroup.
struct Stage1Variant {
    int xd, vec, team_size, k, rows, tpb;
    const void *fn[2];               // phi = identity, phi = sigmoid
    const void *fn_buffers[2] = {nullptr, nullptr};   // the same kernel fetching rows with buffer loads (see launch_partial_grads)
    int block() const { return team_size * tpb; }
    int teams_per_block() const { return tpb; }
};
// Returns nullptr if (x_dtype, d) is outside what the single-pass register kernels cover.
const Stage1Variant *select_stage1(int x_dtype, int64_t d);

// Stage-1 kernels that form every row once.
struct OnceVariant {
    int xd, vec, threads_per_row, k;
    int rows_per_step;               // rows a workgroup takes per step
    int block;                       // threads per workgroup
    int parts_per_unit;              // contiguous parts of X per compute unit (see the kernels)
    const void *fn[2];               // plain loads, loads with the non-temporal hint
};
// For (x_dtype, d), or nullptr if the row is too wide for the registers of a workgroup.
const OnceVariant *select_once(int x_dtype, int64_t d);
// The same for rows one and a half times as wide as those of select_once, or nullptr: their weights are in LDS.
const OnceVariant *select_once_wide(int x_dtype, int64_t d);
// The same with as many wavefronts per workgroup as there are for rows this narrow, for launches of a few workgroups.
const OnceVariant *select_once_whole(int x_dtype, int64_t d);
// Workgroup b runs parts[b], then runs[parts[b].more_begin .. more_end).  rows: the output table.
hipError_t launch_rows_once(const OnceVariant &v, const void *X, const float *y, const float *w, const DevRun *parts, int num_parts,
                            const DevRun *runs, const int32_t *dst, float *rows, int64_t d, int logistic, bool stream_past_caches,
                            hipStream_t stream);

// The same with several workgroups per row, `members` of them, for rows too wide for one (see rows_once_crew_kernel).  A part needs
// crew_exchange_words 8-byte words to exchange in; they are zero, and the two words of state 1 and 0, before the first launch, and
// nobody else writes to either.
struct CrewVariant {
    int xd, vec, k, rows_per_step;
    int members;                     // workgroups per row
    int ring_steps;                  // steps of a part whose slots are kept: a power of two
    const void *fn[2];               // plain loads, loads with the non-temporal hint
};
constexpr int kCrewMembers = 16;     // at most
constexpr int kCrewThreads = 448;    // that hold a member's slice of a row
constexpr int kCrewPatience = 64;    // polls for the others' part of a dot product, some 0.7 us each, before it is worked out again (8 to 64: the same)
bool select_crew(int x_dtype, int64_t d, int units, CrewVariant *v);       // units: compute units of the device
int crew_ring_steps(const CrewVariant &v, int64_t longest_part);           // rows
int64_t crew_exchange_words(const CrewVariant &v);
hipError_t launch_rows_once_crew(const CrewVariant &v, const void *X, const float *y, const float *w, const DevRun *parts, int num_parts,
                                 const DevRun *runs, const int32_t *dst, float *rows, int64_t d, int logistic, bool stream_past_caches,
                                 uint64_t *slots, uint32_t *state, int patience, hipStream_t stream);

// rows_as_buffers: every row starts on a 4-byte boundary and every piece has fewer than 2^31 bytes; variants that have a
// buffer-load twin (bf16 rows, one wavefront per team) then run it
hipError_t launch_partial_grads(const Stage1Variant &v, const void *X, const float *y, const float *w, const DevPiece *pieces,
                                const int32_t *team_piece_begin, int num_teams, float *rows, int64_t d, int logistic,
                                bool rows_as_buffers, hipStream_t stream);
// Wide rows (a row does not fit the registers of one team), every holder separately: two passes.  launch_residuals writes phi(x.w) - y for every row visit,
// launch_xt_residuals forms X^T r per piece and block of 256*kWideChunks*vec columns.  X is read twice on this path.
constexpr int kWideChunks = 8;
hipError_t launch_residuals(int x_dtype, const void *X, const float *y, const float *w, const DevPiece *pieces, int num_pieces,
                            float *residuals, int64_t d, int logistic, hipStream_t stream);
hipError_t launch_xt_residuals(int x_dtype, const void *X, const DevPiece *pieces, int num_pieces, const float *residuals, float *rows,
                               int64_t d, hipStream_t stream);
// The same with every row once, both passes: residuals has one entry per row of X; parts, runs, dst and rows as for launch_rows_once.
// Rows from cached_from on are kept in the last-level cache between the passes.
constexpr int kWideColumnChunks = 256;
hipError_t launch_wide_once(int x_dtype, const void *X, const float *y, const float *w, float *residuals, int64_t m, const DevRun *parts, int num_parts,
                            const DevRun *runs, const int32_t *dst, float *rows, int64_t d, int logistic, int64_t cached_from, int units,
                            hipStream_t stream);
// summed: rows that the sums add up, all together
hipError_t launch_sum_rows(float *rows, const DevSum *sums, int num_sums, int64_t summed, const int32_t *dst, int64_t d, hipStream_t stream);
hipError_t launch_encode(const float *G, float *M, const EncProgram &prog, int num_sub, int L, int64_t d, hipStream_t stream);
// Encode and decode of `steps` masks, one after the other, in one launch (where encode_in_steps says so); the programs lie prog_stride
// bytes apart.
bool encode_in_steps(const TreeShape &tree, int64_t d, int steps);
hipError_t launch_encode_steps(const float *G, int64_t G_stride, float *M, const EncProgram &prog, int64_t prog_stride, int steps, int n, int L,
                               float *g, int64_t g_stride, int64_t d, hipStream_t stream);
// The encode of trees of at most NodeCoefs::kNodes nodes and vectors of at most kTreeColumns columns (tree_side_by_side): a workgroup
// per level-1 sub-tree and 16 or 64 chunks of columns.  The tables travel with the launch or are on the device.
constexpr int64_t kTreeColumns = 163840, kTreeNarrowColumns = 32768;
// What the encode would take instead: a copy of one program, a program written out by launches, a program of which 16 share a copy.
enum class Otherwise { kCopy, kLaunches, kBatch };
bool tree_side_by_side(const TreeShape &tree, int64_t d, Otherwise otherwise);
hipError_t launch_tree_encode(const float *G, float *M, const DeviceTables &tables, const NodeBits &stored, int n, int L, int64_t d, hipStream_t stream);
hipError_t launch_tree_encode(const float *G, float *M, const ArgumentTables &tables, const NodeBits &stored, int n, int L, int64_t d, hipStream_t stream);
// the master's decode and, with step.w, the gradient step; decode_groups: workgroups of the launch
hipError_t launch_decode(const float *M, float *g, const DecTerms &terms, const GradientStep &step, int64_t d, hipStream_t stream);
int decode_groups(int64_t d);
// Encode, decode and gradient step in one launch, where tree_and_decode_together says so: vectors of at most kTogetherColumns columns
// (4 or 8 chunks of columns per workgroup; beyond kTogetherNarrowColumns 16 where the whole tree's messages fit LDS for them).
constexpr int64_t kTogetherColumns = 32768, kTogetherNarrowColumns = 8192;
bool tree_and_decode_together(const TreeShape &tree, int64_t d);
hipError_t launch_tree_encode_decode(const float *G, float *M, const DeviceTables &tables, const NodeBits &stored, int n, int L, float *g,
                                     const GradientStep &step, int64_t d, hipStream_t stream);
hipError_t launch_tree_encode_decode(const float *G, float *M, const ArgumentTables &tables, const NodeBits &stored, int n, int L, float *g,
                                     const GradientStep &step, int64_t d, hipStream_t stream);
int tree_decode_groups(int n, int L, int64_t d);
// metrics[2t], metrics[2t + 1] of `steps` steps from the measures their launches of `groups` workgroups left at sums + t * step_stride
hipError_t launch_measures(const double *sums, int64_t step_stride, int groups, int steps, bool with_star, float *metrics, hipStream_t stream);
hipError_t launch_update(float *w, const float *g, float lr, int64_t d, hipStream_t stream);
// plain streaming read of n16 16-byte words; every workgroup writes its sum to sink[workgroup] (kStreamGroups workgroups)
constexpr int kStreamGroups = 256 * 8;
hipError_t launch_stream_read(const void *src, size_t n16, float *sink, hipStream_t stream);
// ---- the library's own device memory, for callers that cannot allocate -------------------------------------------------------
// A file-scope device array of kStaticScratchBytes (every GPU the library runs on holds its own copy until the process ends).
// static_scratch returns its address on the CURRENT device (looked up once per device, no allocation) in *ptr.
constexpr int kMaxDevices = 64;
constexpr size_t kStaticProgramBytes = size_t(64) << 10;                 // head of the array: one encode program
constexpr size_t kStaticScratchBytes = size_t(96) << 20;                 // the whole array; messages follow the program
hipError_t static_scratch(char **ptr);
// Another one, whose pages hold the trees' tables of bound plans that are given their slabs.
constexpr size_t kTablePoolBytes = size_t(1) << 20, kTablePageBytes = size_t(4) << 10;
hipError_t table_pool(char **ptr);
// An encode program's tables, in device or in host memory; launch_program sends `terms` terms (at most 4096, of slabs and rows below
// 4096) and `subs` (an even number) sub-program words of the host's through kernel arguments: launches only, no staging buffer, no
// memcpy node; the host tables are consumed before the call returns
struct ProgramTables {
    int32_t *slab, *level, *row;
    double *coef, *acoef;
    int32_t *sub;
};
hipError_t launch_program(const ProgramTables &out, const ProgramTables &host, int terms, int subs, hipStream_t stream);

// one wavefront per workgroup; out[workgroup id] = (die the workgroup ran on) << 16 | (shader engine and compute unit inside the die)
hipError_t launch_placement_probe(uint32_t *out, int groups, hipStream_t stream);

}  // namespace cr
