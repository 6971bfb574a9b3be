// Internal declarations shared by the HIP translation units of libcpapr.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <memory>
#include <string>

#include "../../include/cpapr.h"

namespace cpapr {

constexpr int kBlock = 256;  // threads per workgroup (4 wave64s); the PDNR row kernels use one wave per row
constexpr int kXcds = 8;     // MI355X: 8 accelerator complex dies, each with its own L2

struct Error {
    int code;
    std::string msg;
};

// Slots of the KKT max-reduction: blocks spread their atomics over kViolSlots
// addresses, one per 128-byte line, because same-address device atomics
// serialise; consumers take the max over the slots.
constexpr int kViolSlots = 64;
constexpr int kViolStride = 16;  // u64 words per slot (128 bytes)

// MU inner loop row by row (rows.hip): iterations per chunk when a KKT stop may
// end it, violation slots per iteration, row classes, ints of a mode's class counts.
constexpr int kInnerChunk = 16;
constexpr int kInnerSlots = 64;
constexpr int kBatchInnerSlots = 8;  // per batch slot
// Iterations per chunk of an inner loop of lmax: equal shares of at most `most`.
inline int inner_step(int lmax, int most = kInnerChunk)
{
    const int chunks = (lmax + most - 1) / most;
    return chunks > 0 ? (lmax + chunks - 1) / chunks : 0;
}
constexpr int kRowClasses = 20;
constexpr int kLenBuckets = 128;  // row lengths: four buckets per octave
constexpr int kRowMeta = 64 + 2 * kLenBuckets;

// Results a call reads back, in one transfer.
struct DevResults {
    double last_viol[CPAPR_MAX_MODES];  // last KKT violation seen per mode
    int done;                           // inner loop of the current mode has stopped
    int updates;                        // MU updates in the current inner loop
    int sweep_updates;                  // MU updates in the current outer sweep
    int rerun;                          // iteration of the chunk the rows are run again to (-1: none)
    long long total_updates;            // MU updates since the last reset
    long long phi_evals;                // Phi computations since the last reset
    double ll;                          // log-likelihood result
    long long row_steps;                // row solves: steps summed over rows since the last reset
    long long trial_evals;              // row solves: line-search passes since the last reset
    int mode_updates[CPAPR_MAX_MODES];  // MU updates in the last inner loop of each mode (row by row)
};

// Device-side state block of one inner loop (lives in the plan workspace).
struct DevState : DevResults {
    int pq_all_done;                                        // row solves: no row of the current mode is active
    int pq_idle;                                            // row solves: no row is in a line search
    int halt;                                               // the chunk's heavy rows need no further iteration
    unsigned long long viol[2][kViolSlots * kViolStride];   // per-parity slots, ordered bits of doubles >= 0
    unsigned long long iv[kInnerSlots][kInnerChunk];        // KKT violation per iteration of a chunk (ordered bits)
};

// PQNR (projected quasi-Newton row solves): constants shared by every kernel.
constexpr int kPqnrMem = 3;          // curvature pairs kept per row
constexpr int kPqnrTrials = 4;       // backtracking trials before the MU step
constexpr double kPqnrSigma = 1e-4;  // sufficient-decrease constant
constexpr double kPqnrCurv = 1e-10;  // pair kept when s.y > kPqnrCurv |s| |y|

// PQNR state of the mode being solved (rows x R matrices, per-row scalars).
struct PqnrState {
    double* G;      // gradient 1 - Phi at the current b
    double* Gp;     // gradient before the last step
    double* Dd;     // search direction
    double* Dt;     // trial step (after a step: the step taken)
    double* T;      // line-search sums (column 0 of each row)
    double* S;      // kPqnrMem x (rows x R) steps of the kept pairs
    double* Y;      // kPqnrMem x (rows x R) gradient changes of the kept pairs
    double* alpha;  // per row: current trial length
    double* gdel;   // per row: g . trial step
    double* viol;   // per row: last KKT violation
    int32_t* status;  // per row: 0 active, 1 in a line search, 3 converged
    int32_t* trials;  // per row: rejected trials in this line search
    int32_t* steps;   // per row: steps taken
    int32_t* npairs;  // per row: kept pairs
    int32_t* head;    // per row: ring position of the next pair
    int64_t stride;   // rows of every matrix (largest mode)
};

// PDNR (projected damped Newton row solves): constants shared by every kernel.
constexpr int kPdnrMaxRank = 64;       // one wave per row: lane r holds row r of the Newton system
constexpr int kPdnrTrials = 4;         // backtracking trials before the MU step
constexpr double kPdnrSigma = 1e-4;    // sufficient-decrease constant
constexpr double kPdnrHeld = 1e-10;    // entries at or below this with g > 0 are held at the bound
constexpr double kPdnrMu0 = 1e-3;      // damping at the start of an inner loop (times trace(H_FF) / |F|)
constexpr double kPdnrMuMin = 1e-8;
constexpr double kPdnrMuMax = 1e8;
constexpr double kPdnrMuStep = 4.0;    // damping growth / shrink factor

// PDNR state of the mode being solved.
struct PdnrState {
    double* HP;         // rows x (R*R + R): Hessian (row-major) then the Phi row, accumulated per pass
    int64_t hp_stride;  // R*R + R
    double* G;          // gradient 1 - Phi at the current b
    double* Dd;         // search direction
    double* Dt;         // trial step (after a step: the step taken)
    double* T;          // line-search sums (column 0 of each row)
    double* mu;         // per row: damping
    double* alpha;      // per row: current trial length
    double* gdel;       // per row: g . trial step
    double* viol;       // per row: last KKT violation
    int32_t* status;    // per row: 0 active, 1 in a line search, 3 converged
    int32_t* trials;    // per row: rejected trials in this line search
    int32_t* steps;     // per row: steps taken
};

// Rows of one mode by class (rows.hip).
struct RowPlan {
    int32_t* row_ptr;      // [I + 1] first sorted position of each row
    int32_t* order;        // [I] rows by class
    int32_t* chunk_begin;  // [heavy rows + 1] first chunk of each heavy row
    int32_t* chunk_row;    // [chunks] heavy row of each chunk
    int32_t* team_begin;   // [team rows + 1] first member of each team
    int32_t* team_row;     // [members] team of each member
    int32_t count[kRowClasses];
    int32_t nmembers;           // members of the teams
    bool use_teams;             // teams take the long rows but the longest; else all of them are heavy
    double resident;            // share of the nonzeros in light rows and teams
    int32_t nlong, nchunks_all; // long rows and their chunks
    int32_t nchunks;            // chunks of the heavy rows
    int32_t rows_in[kLenBuckets];   // rows per length bucket
    int32_t nnz_in[kLenBuckets];    // their nonzeros
    // Long rows' nonzeros again, each row's split by whether a second mode's
    // coordinate is one of its hot rows (in order inside each part).
    int32_t lead, hot, third;       // other modes: ordered by / hot rows kept in LDS / remaining one (-1); hot < 0: no split
    bool split_made;                // the first inner loop of the mode makes the split
    int32_t bucket, nhot;           // this mode's own hot rows: its rows in length buckets >= bucket, their number
    bool hot_made;                  // and their places
    uint32_t* s_lead;               // [nnz] offsets into the lead mode's factor
    uint32_t* s_hot;                // [nnz] offsets into the hot mode's factor (cold part); in the hot part,
                                    // which comes first, 16-bit places among the hot rows from the row's start on
    uint32_t* s_third;              // [nnz] offsets (three other modes)
    uint32_t* s_val;                // [nnz] FP32 values where all are exact in it, else positions in the sorted copy
    int4* entry;                    // pieces {long row, first, end, hot: 1 + the row's start} of the parts
    int32_t* entry_begin;           // [long rows + 1] first piece of each long row
    int32_t* xlist;                 // [pieces] pieces by die
    int32_t* xbegin;                // [kXcds + 1] first of each die
    uint16_t* hot_id;               // [I] this mode's rows' places among its hot rows (kCold: none)
    int32_t* hot_rows;              // [kMaxHot] this mode's hot rows
};

// Work buffers of the row-by-row inner loop (shared by the modes).
struct RowState {
    double* partial;       // [chunks x R] partial Phi rows of the heavy rows' chunks
    double* team_part;     // [3 x members x R] partial rows of the teams' members
    unsigned int* ticket;  // [tickets] next member, teams' arrivals, heavy rows' arrived chunks; zero between launches
    int64_t tickets;
    int* split;            // temporaries of the hot / cold split: [chunks] + [long rows] + [modes]
    int cus;               // compute units of the device
    double* hot_tab;       // the hot rows of the current inner loop's factor, in their places
    // tol > 0: what a stop goes back to
    double* B0;            // [maxI x R] light rows at the chunk's start
    double* B1;            // [maxI x R] and before the chunk's last update
    double* hist;          // heavy rows' B and Phi of their last iteration, then the team rows' of every iteration
    int64_t hist_n;        // its doubles
    unsigned int* finished;  // heavy rows that are done with an iteration; zero between launches
};

// Who runs inner loops in a plan's row buffers (RowState): a batch from its first
// inner loop to its next commit or its end, a single inner loop or solve for its
// duration. They are given back only when the device has done with them. Whoever
// finds them taken runs the general launches, which share nothing: a plan may be
// in several batches, on several streams.
// The plan and its batches hold it jointly, so either may end first.
using RowOwner = std::atomic<const void*>;

struct RowClaim {
    RowOwner* owner;
    hipStream_t stream;
    bool ok, queued = true;  // queued: the stream was not waited for (the call failed half-way)
    RowClaim(RowOwner* o, hipStream_t s) : owner(o), stream(s)
    {
        const void* none = nullptr;
        ok = o->compare_exchange_strong(none, this);
    }
    ~RowClaim()
    {
        if (!ok) return;
        if (queued) hipStreamSynchronize(stream);
        owner->store(nullptr);
    }
    RowClaim(const RowClaim&) = delete;
    RowClaim& operator=(const RowClaim&) = delete;
};

struct PlanMode {
    int32_t* rows;  // [nnz] sorted mode-n coordinates
    uint32_t* cofs;  // [(N-1) * nnz] the other modes' factor row offsets (coordinate x R), ascending m
    double* vals;   // [nnz]
    // [nnz] the same nonzeros as 16-byte records {row, offset 0, offset 1 (0 for
    // N = 2), value as FP32}: one load per staged nonzero instead of N + 1.
    // Only for N <= 3 and when every value is exact in FP32 (counts up to
    // 2^24); nullptr otherwise.
    int4* pk;
    int64_t segments;
    RowPlan rp;
};

constexpr int kMaxOther = CPAPR_MAX_MODES - 1;

// Operands of one Phi launch over one sorted copy (kernel argument).
struct PhiArgs {
    const int32_t* rows;
    const uint32_t* cofs;
    const double* vals;
    const int4* pk;        // packed records of the same nonzeros (nullptr: read the arrays above)
    const void* fac[kMaxOther];
    const double* B;
    double* Phi;
    const int* done;
    const double* D;       // trial step matrix (line-search pass only)
    const int32_t* live;   // line-search pass: rows with live[row] == 1 are evaluated, the others skipped
    double* det_part;      // deterministic mode: [2 x tiles x R] partial rows of the tile ends (head, tail)
    int32_t* det_rows;     // deterministic mode: [tiles x 2] their row ids (-1: none)
    int64_t det_tiles;     // tiles the partial buffers hold
    int64_t nnz;
    int R;
    int NM1;
    int L;
    int o32;               // 1: every gathered factor is below 4 GiB (32-bit byte offsets)
    double eps;
};

// One work item of a batched launch: operands and its first tile in the
// class's tile space.
struct alignas(16) BatchSlot {
    PhiArgs args;
    int64_t tile_begin;
    int32_t slot;  // caller's slot id (index of its done flag)
    int32_t pad;
};

// One list entry of the batched fill / conversion kernel.
struct alignas(16) BatchCopy {
    const double* src;
    void* dst;
    int64_t n;
    int64_t begin;  // offset in the concatenated element space
    int32_t op;     // 0: zero FP64 dst; 1: dst (FP32) = src (FP64)
    int32_t slot;   // op 0: skipped while this slot's done flag is set; -1: never skipped
};

// One list entry of the batched KKT / MU update kernels (one per slot).
struct alignas(16) BatchMu {
    double* B;
    const double* Phi;
    int64_t n;      // elements (I_mode x R)
    int64_t begin;  // offset in the concatenated element space
    double tol;     // the slot plan's KKT tolerance
    int32_t slot;
    int32_t pad;
};

constexpr int kMuSpread = 8;  // per-slot KKT maxima are spread over this many cache lines

// Dynamic tile claiming of the persistent batched Phi kernel.
constexpr int kBatchSubs = 64;      // tile sub-ranges per shape class (8 per XCD)
constexpr int kBatchClaim = 4;      // tiles claimed per atomic
constexpr int kCounterStride = 32;  // u32 words between counters (one 128-byte line each)
constexpr int kBatchClassesMax = 64;
constexpr int kBatchCounters = kBatchClassesMax * kBatchSubs;

}  // namespace cpapr

struct cpapr_plan {
    int32_t N;
    int64_t nnz;
    int32_t R;
    int64_t dims[CPAPR_MAX_MODES];
    cpapr_params params;
    cpapr::PlanMode mode[CPAPR_MAX_MODES];
    float* f32[CPAPR_MAX_MODES];      // FP32 factor copies (mixed precision)
    double* B;                        // [maxI x R] solve work matrix
    double* phi_prev[CPAPR_MAX_MODES];  // [I_m x R] last Phi per mode (solve)
    double* partial;                  // [kPartials x R] column-sum / reduction partials
    double* llpart;                   // [loglik_partials(nnz)] log-likelihood partials, one per tile
    double* colsums;                  // [N x R]
    cpapr::DevState* state;
    char* ws;
    size_t ws_bytes;
    int group, chunk;                 // resolved launch shape of the Phi kernel
    bool shape_auto;                  // group and chunk both from the launch-policy model
    cpapr::PqnrState pq;              // PQNR row-solve state (method CPAPR_METHOD_PQNR only)
    cpapr::PdnrState pd;              // PDNR row-solve state (method CPAPR_METHOD_PDNR only)
    cpapr::RowState rs;               // row-by-row inner loop (rows_supported)
    bool by_rows;                     // its structures are there
    std::shared_ptr<cpapr::RowOwner> row_owner;
    bool exact32;                     // every value is exact in FP32
    int64_t team_wait;                // clock ticks (10 ns) a team member waits for its team to start
    int expect[CPAPR_MAX_MODES];      // iterations the last inner loop of each mode computed before its stop (0: none ran)
    double* det_part;                 // deterministic mode: tile-end partial rows (nullptr: atomics)
    int32_t* det_rows;                // deterministic mode: their row ids
    int64_t det_tiles;                // tiles the buffers hold (launches with more tiles are refused)
};

namespace cpapr {

constexpr int kPartials = 512;   // blocks of the two-level deterministic column sums

// ---- plan construction (sort.hip) ----
int64_t sort_scratch_bytes(int64_t nnz, int N, bool rows);
// Validates coordinates/values, then builds the sorted copies of every mode
// (only >= 0: of that mode alone).
Error build_sorted(cpapr_plan* P, const cpapr_coo* X, char* scratch, hipStream_t s, int only = -1);

// ---- Phi (phi.hip) ----
// Whether a Phi kernel exists for this lane group, rank block and mode count.
bool phi_shape_supported(int group, int rpl, int nmodes_other);
// Resolve the lane-group size for rank R (the `group` parameter, 0 = automatic).
int resolve_group(int R, int requested, int nm1);
int resolve_chunk(int group, int requested);
int model_group(const cpapr_plan* P);             // launch-policy model: lanes per nonzero
int model_chunk(const cpapr_plan* P, int group);  // launch-policy model: nonzeros per lane group per tile
// Shape of this plan's slots in a batched launch: the model's shape for a
// tensor large enough to fill the device when the plan's shape is the model's,
// else the plan's own shape.
void batch_shape(const cpapr_plan* P, int* group, int* chunk);
// Deterministic mode: tiles the partial buffers are sized for (tiles of >= 128 nonzeros).
inline int64_t det_tile_capacity(int64_t nnz) { return nnz / 128 + 2; }
// Rank columns per lane (1 to 4) for rank R on `group` lanes; -1 if R > 4 * group.
int rank_block(int R, int group);
// The columns per lane that the Phi and MTTKRP launches take (nm1 other modes).
int rank_columns(int R, int group, int nm1, bool mixed);
Error launch_phi(const cpapr_plan* P, int mode, const double* B, const void* const* fac, bool mixed,
                 double eps, double* Phi, const int* done, hipStream_t s);
Error launch_mttkrp(const cpapr_plan* P, int mode, const double* const* A, double* M, hipStream_t s);

// ---- batched inner loops row by row (rows.hip; host side in batch.hip) ----
constexpr int kRowShapes = 16;  // launch shapes by rank and precision
// Whether a batch slot of this plan can run row by row, and as which shape (-1: not).
int rows_batch_shape(const cpapr_plan* P, int mode);
size_t rows_batch_item_bytes();
// Iterations a chunk of such a slot may take (its team rows' history).
int rows_batch_chunk(const cpapr_plan* P, int mode);
// Device-side descriptor of one slot (written to `out`), its workgroups without
// and with the rows restored after a stop, and its team members.
void rows_batch_item(const cpapr_plan* P, int mode, const double* B, const void* const* fac, double* Phi, int slot,
                     const int32_t* done, int32_t* rerun, unsigned long long* iv, void* out, int* light, int* again,
                     int* members);
// One shape's slots of a batch (descriptors and the prefixes of their workgroups, on the device).
struct RowsBatch {
    const void* items;
    const int32_t *light, *again, *members;  // [n + 1] prefixes
    int n, nlight, nagain, nmembers;         // slots and totals
    unsigned int* ticket;                    // next team member; zero between launches
};
Error launch_rows_batch(int shape, const RowsBatch& b, int n_it, bool again, hipStream_t s);

// ---- batched Phi (phi.hip; host side in batch.hip) ----
int batch_class_count();
int batch_class_of(int G, int RPL, int NM1, bool mixed);  // -1: no batched kernel for this shape
// counters: [kBatchCounters * kCounterStride] u32 in device memory.
// grid_tiles > 0: launch one workgroup per tile (that many) instead of the
// persistent kernel.
Error launch_phi_batch(int cls, const BatchSlot* slots, const int32_t* tile_map, const int64_t* class_off,
                       const int64_t* class_ntiles, const int32_t* slot_done, unsigned int* counters,
                       int* grid_cache, int64_t grid_tiles, hipStream_t s);
Error launch_batch_elementwise(const BatchCopy* items, const int32_t* nitems_dev, const int64_t* total_dev,
                               const int32_t* slot_done, unsigned int* counters, int grid, hipStream_t s);
PhiArgs phi_args(const cpapr_plan* P, int mode, const double* B, const void* const* fac, double eps, double* Phi);
// Per-slot state of the batched inner loop, all [max_slots]: done flag, MU
// updates made, last KKT violation.
struct BatchState {
    int32_t* done;
    int32_t* updates;
    double* viol;
    int32_t* hold;  // 1: the slot sits out the run (its done flag starts set)
};
// viol_spread: [kMuSpread * max_slots] u64 (slot s, spread j at j * max_slots + s).
Error launch_batch_mu(const BatchMu* items, const int32_t* nitems_dev, const int64_t* total_dev, int max_slots,
                      unsigned long long* viol_spread, BatchState st, int grid, hipStream_t s);
Error launch_batch_reset(BatchState st, int max_slots, hipStream_t s);
// End of n iterations of a row-by-row batch (all its slots' descriptors): stops, counters, tickets.
Error launch_rows_batch_decide(const void* items, int n, BatchState st, int32_t* rerun, int n_it, unsigned int* tickets,
                               hipStream_t s);

// ---- MU inner loop row by row (rows.hip) ----
bool rows_supported(int R, int64_t nnz);
// Bytes of a mode's row classes / of the inner loop's buffers, bound to `base`
// unless r is nullptr (stops: tol > 0).
size_t rows_mode_bind(RowPlan* r, char* base, int64_t nnz, int64_t dim, int R);
size_t rows_state_bind(RowState* r, char* base, int64_t nnz, int64_t maxI, int R, bool stops);
// Device part of all modes' row classes (meta: kRowMeta zeroed device ints per
// mode), then the host part of one from its meta's host copy.
Error rows_build(const cpapr_plan* P, int* meta, hipStream_t s);
void rows_finish(cpapr_plan* P, int mode, const int* meta);
// Long rows' nonzeros split by a second mode's hot rows, where that pays. Bytes
// bound to `base` unless P is nullptr.
size_t rows_hot_bind(cpapr_plan* P, char* base, int N, int64_t nnz, const int64_t* dims, int R);
// The modes' choices (after every mode's rows_finish; host only).
Error rows_hot_choose(cpapr_plan* P);
// The (last) lmax iterations of an MU inner loop of `mode`, or to the KKT stop; B
// in/out, Phi receives the last Phi. State and counters as the Phi / KKT / update
// launches leave them.
Error enqueue_inner_rows(cpapr_plan* P, int mode, double* B, const void* const* fac, double* Phi, int lmax,
                         hipStream_t s);
// Whether the loop's first iteration runs by the Phi / KKT / update launches.
bool rows_first_alone(const cpapr_plan* P, int mode);
// Whether an inner loop of the mode is faster row by row than by those launches.
bool rows_pay(const cpapr_plan* P, int mode);
// Nonzeros per chunk of a long row.
int heavy_chunk(int64_t nnz);
// The four-trial line-search sums of launch_delta4, row by row (R >= 4, the
// plan's rows by class): column k of `out` for rows with live[row] == 1, other
// entries are left alone.
Error launch_delta4_rows(const cpapr_plan* P, int mode, const double* B, const double* D, const int32_t* live,
                         const void* const* fac, double eps, double* out, const int* skip, hipStream_t s);

// ---- elementwise and reduction kernels (mu.hip) ----
Error launch_fill(double* p, int64_t n, double v, const int* done, hipStream_t s);
// Per-row sums of the likelihood-term changes along the trial steps D (m = B pi,
// dm = D pi; see delta_term) into column 0 of `out` (the other columns get 0),
// for rows with live[row] == 1 only; skipped when *skip != 0.
Error launch_delta(const cpapr_plan* P, int mode, const double* B, const double* D, const int32_t* live,
                   const void* const* fac, double eps, double* out, const int* skip, hipStream_t s);
// The same for the four trial steps max(b + alpha d, 0) - b, alpha = 1, 1/2,
// 1/4, 1/8, along the directions D, in one pass: trial k's sum in column k of
// `out`, the other columns 0. Needs R >= 4.
Error launch_delta4(const cpapr_plan* P, int mode, const double* B, const double* D, const int32_t* live,
                    const void* const* fac, double eps, double* out, const int* skip, hipStream_t s);

// ---- PQNR row solves (pqnr.hip) ----
size_t pqnr_bytes(int64_t maxI, int R);
void pqnr_bind(PqnrState* q, char* base, int64_t maxI, int R);
// One PQNR inner loop (lmax iterations) for the rows of `mode`; B in/out.
// `phi` (I_mode x R) receives every Phi pass, so it ends with the last Phi
// computed. Leaves per-mode stats in the device state (updates = most steps of
// a row, row_steps, last_viol[mode]).
Error enqueue_pqnr_inner(cpapr_plan* P, int mode, double* B, const void* const* fac, double* phi, hipStream_t s);

// ---- PDNR row solves (pdnr.hip) ----
size_t pdnr_bytes(int64_t maxI, int R);
void pdnr_bind(PdnrState* d, char* base, int64_t maxI, int R);
// One PDNR inner loop (lmax iterations) for the rows of `mode`; B in/out,
// `phi` as for PQNR, the same per-mode stats in the device state.
Error enqueue_pdnr_inner(cpapr_plan* P, int mode, double* B, const void* const* fac, double* phi, hipStream_t s);
Error launch_to_f32(const double* src, float* dst, int64_t n, hipStream_t s);
Error launch_reset_state(DevState* st, bool new_sweep, bool all, hipStream_t s);
Error launch_kkt(const double* B, const double* Phi, int64_t n, DevState* st, int l, hipStream_t s);
// tol <= 0: the KKT violation and the update in one pass (the violation reaches
// last_viol one launch later; launch_kkt_fold after the last iteration).
Error launch_mu_fused(double* B, double* Phi, int64_t n, DevState* st, int l, int mode, bool zero_phi, hipStream_t s);
Error launch_kkt_fold(DevState* st, int l, int mode, hipStream_t s);
Error launch_mu_update(double* B, double* Phi, int64_t n, DevState* st, int l, int mode, double tol, bool zero_phi,
                       hipStream_t s);
Error launch_shift_scale(double* A, const double* phi_prev, const double* lam, double* B, int64_t I, int R,
                         double kappa, double kappa_tol, bool shift, hipStream_t s, DevState* st = nullptr,
                         bool new_sweep = false);  // st: also begins a row-by-row inner loop (launch_reset_state otherwise)
// lambda and the normalised factor of a small matrix in one launch.
bool colnorm_small(int64_t I, int R);
Error launch_colnorm_small(const double* B, double* lam, double* A, float* A32, int64_t I, int R, hipStream_t s);
Error launch_colsum(const double* M, int64_t I, int R, double* partial, double* out, hipStream_t s);
Error launch_normalize(const double* B, const double* lam, double* A, float* A32, int64_t I, int R,
                       hipStream_t s);
Error launch_loglik(const cpapr_plan* P, const double* lam, const double* const* A, double eps,
                    hipStream_t s);
// Sum of x_k log(max(m_k, eps)) over the nonzeros of the mode-0 copy into
// `partial` (one entry per tile; returns the number of tiles in *nparts), where
// m_k = B[i_0(k), :] . pi_k and B = A(0) diag(lambda).
Error launch_loglik_terms(const cpapr_plan* P, const double* B, const double* const* A, double eps, double* partial,
                          int* nparts, hipStream_t s);
int64_t loglik_partials(int64_t nnz);
// The whole log-likelihood (into the state) where loglik_fused_supported: the
// terms and every factor's column sums in one launch, then one reduction.
bool loglik_fused_supported(int R);
Error launch_loglik_fused(const cpapr_plan* P, const double* lam, const double* const* A, double eps, hipStream_t s);

// ---- transient Phi without a plan (api.hip) ----
// Workspace bytes of a transient Phi for N modes and nnz nonzeros.
size_t transient_bytes(int N, int64_t nnz);
// Validate X and `mode`, sort the mode into `ws`, run Phi; waits for the stream.
Error phi_transient(const cpapr_coo* X, int32_t mode, int32_t R, const double* B, const double* const* A,
                    double eps, double* Phi, char* ws, size_t ws_bytes, hipStream_t s);
// Argument checks of a transient Phi that touch no device memory.
Error check_transient(const cpapr_coo* X, int32_t mode, int32_t R, bool need_data);

// ---- error message of the last failing entry point (api.hip, thread-local) ----
void set_last_error(const std::string& msg);

// ---- profiling hooks (api.hip) ----
void prof_begin(int mode, hipStream_t s);
void prof_end(hipStream_t s);

}  // namespace cpapr

#define CPAPR_HIP(call)                                                                 \
    do {                                                                                \
        hipError_t e_ = (call);                                                         \
        if (e_ != hipSuccess)                                                           \
            return ::cpapr::Error{CPAPR_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)}; \
    } while (0)

#define CPAPR_LAUNCHED()                                                                \
    do {                                                                                \
        hipError_t e_ = hipGetLastError();                                              \
        if (e_ != hipSuccess)                                                           \
            return ::cpapr::Error{CPAPR_EHIP, std::string("kernel launch: ") + hipGetErrorString(e_)}; \
    } while (0)
