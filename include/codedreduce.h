/* CodedReduce (CR) gradient aggregation: the data-parallel hot path on one AMD MI355X (gfx950).
 *
 * All N workers of an (n,L)-regular tree are simulated on one GPU.  One iteration is
 *
 *     cr_partial_grads(X, y, w)   every worker's partial gradients over its allocated row segments
 *     cr_encode_tree(mask)        every non-straggling node's message, leaves first
 *     cr_decode_root(g)           the master's decode from any n-s of its n children
 *
 * and returns the exact full gradient  g = sum over all m data points of the per-point loss
 * gradient  (Section II-A, eq. (3)) whenever no sibling group has more than s stragglers.
 *
 * Notation: m data points (the paper's d), model dimension d (the paper's p), n children per
 * parent, L layers, s stragglers tolerated per sibling group, N = n + n^2 + ... + n^L workers.
 * Workers are numbered 0-based level by level: node (l,i), l in 1..L, i in 0..n^l-1, has id
 * n + ... + n^(l-1) + i and children (l+1, n*i + j), j in 0..n-1; sibling group g is ids [g*n, (g+1)*n),
 * group 0 being the master's children.
 *
 * Conventions for every call
 *   - plain C ABI; every function returns a cr_status (CR_OK = 0, negatives are errors); the text of the
 *     last error on the calling thread is available from cr_last_error().
 *   - "dev" pointers are device (HBM) addresses, "host" pointers are ordinary host memory.
 *   - the caller owns X, y, w, g and the workspace block; the library allocates no device memory and
 *     frees nothing it was handed.  A plan owns only host tables (and a few KB of pinned host staging
 *     once a workspace is bound).
 *   - device work is enqueued on the stream given to cr_bind_workspace and the call returns without
 *     waiting, unless stated otherwise.
 *   - a plan is not thread-safe; calls on one plan that overlap in time race.
 */
#ifndef CODEDREDUCE_H
#define CODEDREDUCE_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

typedef struct cr_plan_s cr_plan_t;

enum cr_status {
    CR_OK = 0,
    CR_E_INVAL = -1,        /* bad argument, unsupported size, workspace too small or not bound */
    CR_E_UNDECODABLE = -2,  /* some sibling group has more than s stragglers (remark after Theorem 1) */
    CR_E_STATE = -3,        /* call out of order: encode before gradients exist, decode before encode */
    CR_E_HIP = -4,          /* a HIP runtime call failed; see cr_last_error() */
    CR_E_NOMEM = -5         /* host allocation failed */
};

enum cr_model {
    CR_LINEAR = 0,          /* least squares:  per-point gradient x (x.w - y) */
    CR_LOGISTIC = 1,        /* logistic loss, targets y in {0,1}:  x (sigmoid(x.w) - y) */
    CR_AGGREGATE_ONLY = 2   /* no data matrix: partial gradients are supplied by cr_load_partial_grads */
};

enum cr_xdtype { CR_F32 = 0, CR_BF16 = 1 }; /* storage type of X only; y, w, g, slabs and messages are fp32 */

enum cr_kernel {            /* ids for cr_profile_read */
    CR_K_PARTIAL_GRADS = 0, CR_K_REDUCE_PIECES = 1, CR_K_ENCODE = 2, CR_K_DECODE = 3, CR_K_UPDATE = 4, CR_K_COUNT = 5
};

typedef struct cr_plan_info {
    int32_t L, n, s, model, x_dtype;
    int32_t num_workers;     /* N */
    int32_t num_groups;      /* N / n sibling groups */
    int32_t num_slabs;       /* S: (worker, segment) pairs; one d-float partial gradient each */
    int32_t num_decode_rows; /* F = C(n,s) */
    int32_t code_candidate;  /* index of the winning candidate of the code search; -1 if B was supplied; -2 fractional repetition */
    int32_t num_teams;       /* stage-1 work split (0 until known, see cr_plan_set_split) */
    int32_t num_pieces;      /* entries of cr_plan_get_pieces (0 until the split is known) */
    int32_t split_kind;      /* enum cr_split of the split in force; -1 until it is known */
    int32_t stage1_team_size;       /* threads that share one row in the stage-1 kernel in force; 0: rows of more than 24576 columns */
    int32_t stage1_teams_per_group; /* teams per workgroup; shared cells: holders of a cell that a workgroup serves */
    int32_t stage1_staged;   /* 1 under shared cells: rows are fetched once per workgroup for all the holders it serves */
    int64_t m, d;
    int64_t row_visits;      /* sum over workers of allocated rows */
    int64_t min_rows, max_rows; /* smallest / largest per-worker load; both equal r_CR m up to integer cuts (Theorem 1) */
    int64_t split_value;     /* teams (equal ranges), rows per cell (row cells, shared cells) or rows per run (rows once); 0 until the split is known */
    double gamma;            /* max_f sum_i |a_fi| ||b_i||_2 / sqrt(n): rounding amplification of one decode.  Messages are fp32, so
                              * a decoded gradient carries a relative rounding error of about gamma^L * 2^-24 (see code_warning) */
    double r_cr;             /* computation load of Theorem 1 */
    int32_t l2_domains;      /* L2 cache domains (accelerator dies) the stage-1 split was laid out for: queried from the device when
                              * the split is fixed, 8 (MI355X) without a device */
    int32_t unit_slots;      /* workgroup slots (compute units, or twice that for short rows) of the shared-cells split; 0 otherwise */
    int32_t l2_sharing;      /* do workgroups whose ids are congruent modulo l2_domains run on the same die, as the row-cell and
                              * shared-cell splits assume?  1: checked on the device at cr_bind_workspace; 0: checked and NOT so
                              * (results stay exact, but every holder of a row then fetches it from HBM itself); -1: not checked
                              * (no workspace bound yet, or the split does not rely on it) */
    int32_t code_warning;    /* 1 if gamma^L * 2^-24 exceeds 1e-5, a tenth of the fp32 parity bar: the code is too badly
                              * conditioned for fp32 messages to be trusted to 1e-4 (wide groups with s+1 not dividing n) */
} cr_plan_info_t;

/* ---- plan (host only; Section III-A CR.Allocate, Algorithms 1 and 2, Section II-C for the code) ------------
 * cr_plan builds, on the host: the gradient-coding matrices B (n x n, cyclic support {i..i+s} mod n, unit-norm
 * rows; if the best cyclic candidate has gamma^L > 256 and s+1 divides n, the 0/1 fractional-repetition design
 * instead) and the decode rows a_f (a_f B = 1, zero on the straggler set); the recursive allocation of weighted row
 * segments to every node (CompAlloc with k = n parts cut at floor(kappa |W| / n); a node keeps the first
 * round(|W| / sum_{j=0}^{L-l} (n/(s+1))^j) positions of its sub-tree set, leaves keep all); and the slab list
 * (node-major, segments in allocation order).  cr_plan = cr_plan_ex with CR_LINEAR, CR_F32, the default seed, no B.
 *   seed         seeds the counter-based search for a well-conditioned code (ignored when B is given)
 *   B_or_null    host, n*n doubles row-major: use this encoding matrix (s+1 non-zeros in every row and column); or NULL
 *   out          receives the plan; destroy with cr_plan_destroy
 * Errors: CR_E_INVAL for L<1, L>8, n<2, n>64, s<0, s>=n, d<1, d>2^28 (any model), m<N, m>2^40, C(n,s) > 2^20, N > 2^24, an unsupported B. */
int cr_plan(int L, int n, int s, int64_t m, int64_t d, cr_plan_t **out);
int cr_plan_ex(int L, int n, int s, int64_t m, int64_t d, int model, int x_dtype, uint64_t seed,
               const double *B_or_null, cr_plan_t **out);
void cr_plan_destroy(cr_plan_t *plan);

/* ---- introspection (host; data for tests and harnesses) ------------------------------------------------------ */
int cr_plan_info(const cr_plan_t *plan, cr_plan_info_t *info);
int cr_plan_get_B(const cr_plan_t *plan, double *B /* host, n*n */);
int cr_plan_get_A(const cr_plan_t *plan, double *A /* host, F*n, row f = f-th straggler set in lexicographic order */);
/* The allocation (CR.Allocate, Algorithm 2): segment p = rows [row_begin[p], row_end[p]) of X, held by worker[p] with combining
 * coefficient coef[p]; segments are listed worker-major, in allocation order; each owns one slab (a d-float partial gradient), so
 * there are S = num_slabs of them.  Arrays of S entries, any may be NULL. */
int cr_plan_get_segments(const cr_plan_t *plan, int64_t *row_begin, int64_t *row_end, double *coef, int32_t *worker);
/* decode row for one sibling group (Section III-A, CR.Execute step 3): flags[j] != 0 marks child j a straggler.  With fewer than
 * s stragglers the set is padded with the highest-index survivors.  a: host, n doubles.  CR_E_UNDECODABLE if more than s are set. */
int cr_plan_decode_row(const cr_plan_t *plan, const uint8_t *flags /* host, n */, double *a);
/* Stage-1 work split into pieces (a piece = a run of one slab's rows handled by one team).
 *   CR_SPLIT_EQUAL_RANGES  value = teams: the row visits of all slabs, slab-major, are cut into `teams` equal contiguous ranges,
 *                          cut again at slab boundaries.
 *   CR_SPLIT_ROW_CELLS     value = rows per cell: every slab is cut on one global grid of that many rows, one piece per team, teams
 *                          ordered by cell so that the holders of the same rows run at the same time.
 *   CR_SPLIT_SHARED_CELLS  value = most rows per cell: the grid is laid between slab boundaries, so every holder of a cell holds
 *                          all of it; a workgroup works through a queue of cells (one queue per compute unit, two for rows of at
 *                          most 8 KB) and forms every row of a cell once for the 2, 3, 4, 6 or 8 holders it serves
 *                          (stage1_teams_per_group, by row width and by (s+1)^L, the most holders a row can have); a cell with more
 *                          holders is formed by several workgroups of one L2 domain, each for its own holders.  fp32 rows of 257 to
 *                          3072 16-byte chunks with s > 0 only, else CR_E_INVAL.
 *   CR_SPLIT_ROWS_ONCE     value = most rows per run: X is cut into one or two contiguous parts per compute unit, a part into runs at
 *                          slab boundaries and after `value` rows; a workgroup forms every row of its part once, for all slabs that
 *                          hold it, and adds a run up in fp64 (all but the up to four rows it has in hand at a time).  Rows of more
 *                          than 24576 columns take one pass where their weights fit LDS (34816 columns fp32, 36864 bf16), X is
 *                          large against the rows that its parts put away (48 MB at least) and `value` is at most a compute unit's
 *                          share of the rows.  Wider ones, up to 114688 columns fp32 and 172032 bf16, take one pass too, shared by 2 to
 *                          16 workgroups, a part per crew of them (but for some small X); else two passes, the second cut into parts of
 *                          rows and blocks of columns.
 *                          CR_ROWS_WHOLE_RANGES as value (d <= 24576): a workgroup per distinct slab range, which it adds up whole; rows
 *                          of ranges that overlap are then formed once per range.
 * With the first two every holder of a row does its own arithmetic on it, as separate workers would: they are there to measure what
 * the redundancy of a scheme costs (with s = 0 no row has a second holder, and equal ranges run the kernels of rows once, a
 * workgroup per team).  With the other two the holders' identical sums are formed once (per workgroup) and handed to
 * every slab they belong to.  The slab gradients agree to rounding under every split.
 * Default (when this is never called): rows once, for the smallest problems by whole ranges, else without a limit on runs (wide rows that
 * can take one pass: a compute unit's share of the rows).  With X of 1 GiB and more: equal ranges of the rows when s = 0 (no row is held twice), shared cells where one workgroup serves all holders of a
 * row, with the cell height (16 to 1024 rows) that gives the shortest longest queue. */
enum cr_split { CR_SPLIT_EQUAL_RANGES = 0, CR_SPLIT_ROW_CELLS = 1, CR_SPLIT_SHARED_CELLS = 2, CR_SPLIT_ROWS_ONCE = 3 };
#define CR_ROWS_WHOLE_RANGES ((int64_t)1 << 62)
int cr_plan_set_split(cr_plan_t *plan, int kind, int64_t value);
/* pieces in execution order: piece i is rows [row_begin[i], row_end[i]) of slab[i], run by team[i] (rows once: by workgroup team[i],
 * one piece for every slab the rows belong to); num_pieces entries each, any may be NULL */
int cr_plan_get_pieces(const cr_plan_t *plan, int32_t *slab, int64_t *row_begin, int64_t *row_end, int32_t *team);

/* ---- run-time model (host only; Section III-C "Latency Performance", eq. (5), Theorem 2) ------------------------------------
 * Simulates iteration number `iteration` of the plan's tree: worker k, holding rows_k data points, computes for
 * a*rows_k + (rows_k/mu) * Exp(1) (the shifted-exponential law of eq. (5), drawn from the counter-based splitmix64 stream seeded
 * with `seed`, counter iteration*N + k); a parent receives one message at a time, in order of readiness, t_c per message, and
 * decodes after n-s of them; all nodes compute from time 0 and while receiving.
 *   mask   host, N bytes or NULL: 1 for the s children of every group that were not waited for (usable by cr_encode_tree)
 *   ready  host, N doubles or NULL: time each node's message is ready to send
 *   total  host or NULL: time at which the master has decoded
 * CR_E_INVAL unless a >= 0, mu > 0, t_c >= 0, iteration >= 0. */
int cr_simulate_iteration(const cr_plan_t *plan, double a, double mu, double t_c, uint64_t seed, int64_t iteration,
                          uint8_t *mask, double *ready, double *total);

/* ---- device binding --------------------------------------------------------------------------------------------
 * The workspace holds the device tables, 16 encode programs (for trees and vectors whose encode takes programs), the stage-1 partial rows, the slab gradients
 * G[S][d] (not for CR_AGGREGATE_ONLY) and the messages M[N][d], all fp32 rows of d floats.  dev_ptr must be 256-byte aligned and stay valid while the plan
 * is used; hip_stream is a hipStream_t (NULL = the default stream).  cr_bind_workspace copies the tables synchronously, in one copy.
 * The tables of stage 1 must stay as bound.  Beside them lies, where workgroups share rows, what they exchange in and the number of the
 * launch: every cr_partial_grads changes it and the next one relies on it, so nobody else writes there between binding and the last call,
 * and a program that saves the block and puts it back does so with all of it, between calls.  A call on slab gradients of the caller's (cr_load_partial_grads, cr_aggregate_run) relies on
 * nothing that the workspace held before it, so aggregation-only plans may take turns in one block. */
int cr_workspace_bytes(cr_plan_t *plan, size_t *bytes);
int cr_bind_workspace(cr_plan_t *plan, void *dev_ptr, size_t bytes, void *hip_stream);

/* ---- the hot path ------------------------------------------------------------------------------------------------
 * cr_partial_grads (CR.Execute step 1): for every slab p,  G[p] = X[b:e]^T (phi(X[b:e] w) - y[b:e]),  phi = identity or sigmoid.
 *   X_dev  m x d row-major, contiguous, fp32 or bf16 per the plan, 16-byte aligned;  y_dev m floats;  w_dev d floats.
 *   One pass over X as long as a row fits the registers of a workgroup (d <= 24576, whether or not d is a multiple of the 16-byte
 *   chunk) or its weights LDS beside them (34816 fp32, 36864 bf16, X of 48 MB or more
 *   depending on the tree), or the registers of up to 16 workgroups (114688 fp32, 172032 bf16, but for some
 *   small X); other rows take two passes.  With CR_LOGISTIC an infinite entry of X reaches its own column of the slabs and no other
 *   (sigmoid(+-inf) is 0 or 1), but under the splits that do every holder's arithmetic.  Every slab of every worker is written; what the workers that hold a row have in common is
 *   formed once for all of them unless the split says otherwise (see cr_plan_set_split).
 * cr_load_partial_grads: use caller-supplied slab gradients G_dev[S][d] (fp32, 16-byte aligned) in place of stage 1;
 *   the buffer is read in place by cr_encode_tree and must stay valid until then.
 * cr_encode_tree (CR.Execute steps 2-5): mask is HOST memory, N bytes, non-zero = straggler.  For every non-straggler node,
 *   m_(l,i) = sum_p coef_p G[p] over its slabs  +  sum_j a_j m_(l+1, n i + j)  with a = the decode row of its children group.
 *   Stragglers write no message (their row of M keeps stale data); all other nodes do, also below a straggler.
 *   CR_E_UNDECODABLE, before anything is enqueued and with no state change, if any group has more than s stragglers.
 *   On trees of at most 448 workers whose level-1 sub-trees' messages fit a workgroup's LDS (all but some of more than six levels) and with
 *   vectors of up to 32768 columns, 40000 to 163840 depending on the tree, all it enqueues is one kernel launch, with what the mask
 *   decides as kernel arguments; else the mask's encode program travels in a copy from pinned memory first.  (The tree's tables are read
 *   from the workspace with stage 1's slabs, from 1 MB that the library keeps for bound plans with the caller's; while that is all in
 *   use they travel with the call, in a copy where they do not fit the arguments.)
 * cr_decode_root (the last step of CR.Execute, Algorithm 2: the master recovers g from any n-s of its children):
 *   g_dev[d] = sum_j a_j m_(1,j) with the decode row of group 0 from the last cr_encode_tree; by eq. (3) this is the full gradient.
 * cr_gd_update: w <- w - lr * g (plain gradient step used by the benchmark loop).
 * Errors: CR_E_STATE out of order; CR_E_INVAL unbound workspace / NULL / misaligned pointers; CR_E_HIP launch failures. */
int cr_partial_grads(cr_plan_t *plan, const void *X_dev, const float *y_dev, const float *w_dev);
int cr_load_partial_grads(cr_plan_t *plan, const float *G_dev);
int cr_encode_tree(cr_plan_t *plan, const uint8_t *straggler_mask_host);
int cr_decode_root(cr_plan_t *plan, float *g_dev);
int cr_gd_update(cr_plan_t *plan, float *w_dev, const float *g_dev, float lr);

/* Gradient descent loop kept on the device (eq. (2) with a plain step): `steps` times  g = CodedReduce(w);  w <- w - lr g,  enqueued
 * back to back, kernel launches only where cr_encode_tree is one: stage 1, its sums, and one launch for encode, decode and the gradient
 * step (two for d > 32768).  Elsewhere the encode programs of 16 steps at a time travel to the device in one copy, and the host waits
 * only when it runs more than 32 steps ahead of the copies (two pinned staging batches).
 *   masks_host      steps x N bytes, one straggler mask per step; all are checked first: CR_E_UNDECODABLE before anything is enqueued
 *   w_dev, g_dev    d floats each; w is updated in place, g holds the last decoded gradient
 *   w_star_or_null  d floats (device): the reference model of the normalised error rate, or NULL
 *                   (w, g and w* may be one vector, or lie among the messages: the values are those of the separate calls, and encode and
 *                   decode take launches of their own then)
 *   metrics_or_null device, steps x 2 floats: [2t] = ||w_t+1 - w_t||^2 / ||w_t||^2 (relative error rate, eq. (6)),
 *                   [2t+1] = ||w_t+1 - w*||^2 / ||w*||^2 (normalised error rate, eq. (8); -1 without w*); NULL = not wanted.  The sums
 *                   behind them are formed by the launch that makes the step, the quotients by one launch per 16 steps */
int cr_gd_run(cr_plan_t *plan, const void *X_dev, const float *y_dev, float *w_dev, float *g_dev, const uint8_t *masks_host,
              int steps, float lr, const float *w_star_or_null, float *metrics_or_null);

/* Aggregation alone, many masks in one call (CR.Execute steps 2 to the end, Algorithm 2, once per mask): step t encodes the slab
 * gradients at G_dev + t * G_step_stride under masks_host[t] and decodes into g_dev + t * g_step_stride; like cr_load_partial_grads,
 * cr_encode_tree and cr_decode_root called in turn (the same bits).  Short vectors (d <= 32768) take one launch per mask, two on
 * trees of more than some 400 workers; longer ones on trees of up to three levels and 32 children per parent mostly one launch for up to 16
 * masks, behind one copy of their programs; else two launches per mask.
 *   G_dev          device, S x d floats per step, 16-byte aligned; G_step_stride in floats (a multiple of 4): 0 = the same slabs every step
 *   masks_host     steps x N bytes; all are checked first: CR_E_UNDECODABLE before anything is enqueued
 *   g_dev          device, d floats per step; g_step_stride in floats: 0 = every step overwrites the same vector.  The vectors may lie
 *                  among the slabs or the messages or overlap in part: the steps then take launches of their own, in order
 * Afterwards the plan is in the state the last step's three calls would have left (messages of the last mask). */
int cr_aggregate_run(cr_plan_t *plan, const float *G_dev, int64_t G_step_stride, const uint8_t *masks_host, int steps, float *g_dev,
                     int64_t g_step_stride);

/* ---- aggregation without any allocation ----------------------------------------------------------------------------------------
 * For callers that cannot allocate or bind device memory: code under HIP stream capture, tight serving loops, harnesses that forbid
 * hipMalloc.  cr_aggregate_static is cr_load_partial_grads + cr_encode_tree + cr_decode_root in one call, with everything those
 * keep in a workspace -- the per-call encode program and the messages M[N][d] -- held in a device array that is part of the library
 * itself (CR_STATIC_SCRATCH_BYTES; each GPU the library runs on holds one until the process ends).  The plan needs no workspace.
 * The call allocates and frees nothing on the device or in pinned memory and records no copy: what the kernels need reaches the device
 * as kernel arguments, so all it enqueues on hip_stream is kernel launches: one for encode and decode where the tree's tables and the
 * mask's coefficients fit the arguments and d <= 32768, two up to 163840 columns depending on the tree, else a few small ones that write
 * the program out, encode and decode.  (Trees of up to some 150 workers fit; whether one near that border does depends on how many
 * different coefficients the mask calls for.)
 *   plan        any plan; its model is not consulted (no stage 1 runs)
 *   G_dev       device, S x d floats, 16-byte aligned: the slab gradients, read in place
 *   mask_host   host, N bytes, non-zero = straggler; read before the call returns
 *   g_dev       device, d floats: receives the decoded gradient (the same bits cr_decode_root gives for the same G and mask); may lie
 *               among the slabs (two launches then)
 *   hip_stream  a hipStream_t (NULL = the default stream)
 * Limits: the messages must fit, N * d * 4 <= CR_STATIC_SCRATCH_BYTES - 64 KiB (the paper's network, 156 workers x 117 706
 * parameters, does), and the encode program (28 bytes per slab and per worker) must fit 64 KiB: CR_E_INVAL otherwise, before
 * anything is enqueued.  CR_E_UNDECODABLE as for cr_encode_tree.  All calls on one GPU share that GPU's array, whatever the plan:
 * calls that overlap in time on one GPU (two streams, two threads) race.  The array keeps the previous call's contents; nothing
 * in it needs clearing, since every message row that is read was written earlier in the same call. */
#define CR_STATIC_SCRATCH_BYTES ((size_t)96 << 20)
int cr_aggregate_static(cr_plan_t *plan, const float *G_dev, const uint8_t *mask_host, float *g_dev, void *hip_stream);

/* ---- results kept in the workspace (device pointers, valid while the workspace is) --------------------------- */
int cr_get_slab_grads(const cr_plan_t *plan, const float **G_dev); /* S x d */
int cr_get_messages(const cr_plan_t *plan, const float **M_dev);   /* N x d, row = worker id */

/* ==== instrumentation: measurement plumbing for benchmarks and tests; no step of the method needs any of it ================
 * cr_profile_enable(plan, kernels): bit k of `kernels` set = every launch of kernel id k is bracketed by two HIP events on the
 * bound stream from now on (CR_PROFILE_ALL: all of them, 0: none); a non-zero call also clears the totals.  Each bracket costs
 * a few microseconds of device time, which shows on small problems.  cr_profile_read waits for the stream, then returns for one
 * kernel id the summed duration, the number of launches and the algorithmic bytes of those launches (bytes the method must
 * move: rows read once per holder, each result written once) since the last non-zero cr_profile_enable; any may be NULL.  A launch that does the
 * work of several counts once, with all its bytes: encode, decode and gradient step in one as CR_K_ENCODE, decode and step as CR_K_DECODE;
 * CR_K_UPDATE is cr_gd_update and the convergence measures.
 * Totals read after cr_profile_enable(plan, 0) are those gathered until then. */
#define CR_PROFILE_ALL ((1 << CR_K_COUNT) - 1)
int cr_profile_enable(cr_plan_t *plan, int kernels);
int cr_profile_read(cr_plan_t *plan, int kernel, double *total_ms, int64_t *launches, int64_t *algorithmic_bytes);
/* the duration in milliseconds of every single timed launch of one kernel id since the last non-zero cr_profile_enable, in launch
 * order (the first 65536 of them): up to `capacity` values are copied to ms (host), *count receives how many there are; waits for
 * the stream like cr_profile_read */
int cr_profile_samples(cr_plan_t *plan, int kernel, float *ms, int64_t capacity, int64_t *count);
/* algorithmic bytes of the most recent launch of a kernel id (0 if none yet) */
int cr_last_algorithmic_bytes(const cr_plan_t *plan, int kernel, int64_t *bytes);
int cr_synchronize(cr_plan_t *plan); /* wait for the bound stream */
/* What a plain streaming read reaches on this device: `launches` launches of a kernel that only reads src_dev[0 .. bytes) with
 * 16-byte loads (every workgroup sums what it reads into sink_dev so that nothing is optimised away), timed with HIP events on the
 * given stream; the call waits for them.  A yardstick for the traffic figures of the hot path, not part of it.
 *   src_dev   device, 16-byte aligned, bytes a multiple of 16 and at least 1 MiB;  sink_dev  device, at least 16384 floats
 *   gbps      receives bytes * launches / elapsed in GB/s (the first launch is a warm-up and not timed) */
int cr_probe_read_bandwidth(const void *src_dev, size_t bytes, float *sink_dev, int launches, void *hip_stream, double *gbps);

const char *cr_last_error(void);

#ifdef __cplusplus
}
#endif
#endif /* CODEDREDUCE_H */
