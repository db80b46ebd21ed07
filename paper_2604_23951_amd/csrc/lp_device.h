// Internal device-side types and kernel launchers of the restarted-PDHG solver.
// Everything here is private to the library; the public surface is include/lp.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace lpgpu {

constexpr int kBlock = 256;       // threads per workgroup (4 wave64)
// Row-tile shapes of the LDS-staged SpMV: shape h holds at most tile_nnz_of(h) nonzeros
// (1024, 2048, 4096) and a quarter as many rows; the shape of an LP comes from its options or
// the tuned table (lp_tile_table.h).
constexpr int kTileShapes = 3;
__host__ __device__ constexpr int tile_nnz_of(int shape) { return 1024 << shape; }
constexpr int kTileNnzMax = 4096;
constexpr int kMaxRedBlocks = 512;
constexpr int kNQ = 8;            // reduced quantities per candidate
constexpr int kNR = 8;            // reduced quantities of the two candidate rays (infeasibility), 4 each
constexpr int kNF = 6;             // sums of the residual restarts: ||dx||^2, <dy, A~dx>, ||dy||^2 (last iterate, anchor)
constexpr int kNT = 2 * kNQ + kNR + kNF;  // all reduced quantities of one evaluation
constexpr int kTraceW = 12;

constexpr int kRunning = -1;

// Largest nonzero count accepted. The kernels form entry offsets in 32-bit ints and clamp
// indices that run past the end of a row, tile or unit (by at most a few thousand entries:
// the panel producer's prefetch reaches 16 groups of 256 entries ahead); the margin keeps
// every such offset below 2^31.
constexpr long long kMaxEntries = 0x7fffffffLL - (1LL << 16);

// Device-resident scalar state of one solve. The iteration kernels read it; only the
// single-workgroup decision kernels write it.
struct Scalars {
    double tau, sigma, omega, eta, omega0;
    double eps_rel, c0, qnorm, cnorm, sigma_max, sigma_prev;  // sigma_prev: the power step before
    double kkt_anchor, kkt_prev;
    double eps_infeas, ray_scale;  // certificate tolerance (0: off); 1/D or 1/G of a certificate
    double anc_rps2, anc_rds2, anc_gap;
    double pid_int, pid_prev;  // PID rule of the primal weight: integral and previous error
    // statistics of the returned point
    double out_pobj, out_dobj, out_rel_p, out_rel_d, out_rel_gap, out_erel;
    long long k, t, max_iters, restarts, n_trace, trace_cap;
    long long done_clock;  // device wall clock (wall_clock64) when the solve stopped
    long long deadline;    // device wall clock at which an evaluation stops the solve with LP_TIME_LIMIT (0: none)
    int status;        // kRunning or an lp_termination value
    int out_avg;       // returned point: 1 = running average
    int last_restart;  // what the apply kernel must do: 0 nothing, 1 keep current, 2 take average
    int eval_every;
    int restarts_on;
    int term_mode;     // what must fall to eps_rel to stop: 0 E_rel, 1 rel. primal residual, 2 rel. dual residual
    int ray_src;       // candidate ray of a certificate: 1 displacement since the previous evaluation, 2 anchored average
};

// What an iteration streams up to which plain loads of the matrices, which may stay in the 256 MB
// Infinity Cache from one iteration to the next, beat non-temporal ones. us per iteration, plain /
// non-temporal:
// - two phases (entries of both matrices and the products): 144 MB 80 / 91, 154 MB 86 / 99, 230 MB
//   144 / 138, 240 MB 140 / 137, 384 MB 209 / 207;
// - FP64 row tiles of one LP (iteration_bytes): uniform columns 215 MB 71 / 79, 307 MB 123 / 125, 414 MB
//   198 / 189; power-law columns 335 MB 139 / 140, 402 MB 181 / 176, 670 MB 360 / 351; rows of 40
//   entries 235 MB 96 / 119; dense 237 MB 110 / 135, 358 MB 191 / 197;
// - block-diagonal launches (the same, of all their LPs in the FP64 form): 308 MB 86 / 94, 402 MB 117 /
//   119, 473 MB 139 / 136, dense rows 263 MB 112 / 126, 478 MB 209 / 202, 980 MB of both 406 / 398. In the
//   FP32 form they are faster with plain loads, or as fast, whatever they stream: 407 MB 129 / 133,
//   637 MB 226 / 230, 813 MB 256 / 252, 2526 MB 847 / 879, 4096 LPs to 1e-4 2.07 / 2.16 s.
constexpr long long kKeepTwoPhase = 192LL << 20, kKeepTiles = 370LL << 20, kKeepMulti = 430LL << 20;
// Entries of both matrices, and the vectors twice: most are read and written. value: bytes of one.
constexpr long long iteration_bytes(long long m, long long n, long long nnz, int value) {
    return 2 * nnz * (value + 4) + 2 * value * (9 * n + 8 * m);
}

// A row tile: rows [r0, r1), entries [p0, p1).
struct TileRec {
    int r0, r1, p0, p1;
};

// CSR matrix with its LDS tiling: tile b covers rows [tiles[b], tiles[b+1]), or, when
// rowlist is set, the single row rowlist[b]. The launches read a tile's bounds from recs in
// one load: offset by offset (tiles, then row pointers) they are two more links in the chain of
// loads that such a short-lived workgroup is bound by.
struct Csr {
    int rows;
    int ntiles;
    int nnz;
    int shape;  // row-tile shape (tile_nnz_of(shape) nonzeros per tile at most)
    const int* rp;
    const int* ci;
    const double* v;
    const int* tiles;
    const int* rowlist;
    const float* v32;  // FP32 copy of v (FP32 storage form only)
    int cols;          // length of the vector the products gather from
    int tree_len;      // rows longer than this are reduced by a whole workgroup (at most the tile's nonzeros)
    const TileRec* recs;
    int keep;  // row tiles of FP64 launches: plain loads of the matrix (kKeepTiles), else non-temporal ones
};

// Panel-packed layout (see lp_layout.h): unit u (one wave) owns rows
// [unit_row[u], unit_row[u+1]) and the entries [unit_seg[u*(panels+1)], unit_seg[u*(panels+1)+panels]),
// stored panel by panel. packed = (row inside the unit << col_bits) | column.
struct Panels {
    int units;
    int panels;
    int col_bits;
    int nnz;
    int max_rows;  // rows of the largest unit (sizes the LDS accumulators)
    const int* unit_row;
    const int* unit_seg;
    const unsigned* pk;
    const double* v;
    const unsigned char* is_long;  // nullptr when the matrix has no long rows
    const float* v32;              // FP32 copy of v (FP32 storage form only)
    int cols;                      // length of the gathered vector
};

// Panel layout: a matrix whose gathered vector fits one XCD's 4 MB L2 is swept as row tiles
// unless a panel width was asked for. The gathers hit the L2 in any order then, and the panel
// units (a few hundred entries per wave and step, a barrier after each, ~20 us however small
// the matrix) only cost latency. us per iteration, Halpern form, panels / row tiles: 32k
// entries 11.8 / 7.8, dense rows with 993k (FP64) 57 / 16, power-law columns with 1.2M 51 / 32
// (FP32 44 / 27), 2.4M 77 / 53 (66 / 47); beyond, x at 6.4 MB: 111 / 114, y at 6.4 MB: 190 / 219.
// The FP64 products of the FP32 storage form gather twice the bytes and keep the panels where
// those exceed it (y at 8 MB, 1.2e7 entries: panels 107, row tiles 159).
constexpr long long kFlatBytes = 4LL << 20;

// Two-phase layout of a matrix (lp_two_phase.h): blocks of 2^width_bits columns and tiles of
// rows with at most tile_nnz entries: first those of the rows that are not long (tile_row
// numbers the matrix's rows, trp their entries without the long rows'), from tiles_short on
// those of the long rows of at most tile_nnz entries (tile_row numbers the list longs, trp
// continues with its entries). Entries in block order, tile by tile
// inside a block (block b's start at block_start[b], a multiple of 4): lcol (column inside the
// block), v. Tile t's entries in block order are positions 64 tile_chunk[t] + k of pos (CSR
// position inside the tile); entry k's product is buf[k + delta[t * blocks + run]], run the
// number of the run of consecutive products it belongs to: first[chunk] runs begin before its
// chunk of 64 and the bits of mask[chunk] mark those beginning inside it.
struct TwoPhase {
    int tiles;  // 0: not built
    int tiles_short, tiles_padded, blocks, width_bits, tile_nnz, fp32, cols, slots;
    const int *block_start, *tile_row, *tile_chunk, *trp, *delta;
    const unsigned long long* mask;
    const int* first;
    const unsigned short *lcol, *pos;
    const double* v;   // FP64 form only
    const float* v32;  // FP32 storage form only
    int keep;                      // plain loads of the matrix (see kKeepTwoPhase), else non-temporal ones
    const unsigned char* is_long;  // as in Panels
    const int* longs;
    int nhuge;          // rows longer than a tile, each reduced by a workgroup from its gathers
    const int* huge;
    void* buf;  // products of one launch, in the precision of the iterations
};
constexpr int kTpMaxBlocks = 1024;
constexpr int kTpSplit = 2;  // workgroups that share a block's entries
constexpr int kTpXcds = 8;
constexpr int kTpLds = 64 * 1024;      // of the gathered slice at most
constexpr int kTpTileLds = 64 * 1024;  // of a tile's products at most (FP64)
constexpr int kTpTileLds32 = 39 * 1024;  // (FP32)

// Index checks of the checked build (compiled with LPGPU_CHECKED=1): a gathered column or
// an accumulator row outside its array sets a bit of a device word and is replaced by 0, so
// the kernel reads nothing outside its arrays; the host reports the word after a call.
// Bits: 1 panel gather, 2 panel accumulator row, 4 row-tile gather, 8 long-row gather.
#ifndef LPGPU_CHECKED
#define LPGPU_CHECKED 0
#endif
constexpr bool kChecked = LPGPU_CHECKED != 0;
// Reads and clears the check word of `device` (0 in a build without checks).
int read_check_word(int device, unsigned* word);

constexpr int kUnitRowCap = 2048;  // rows per wave unit at most
constexpr int kChunks = 4;         // 64-entry chunks a wave loads together (one group)
constexpr int kStreamDepth = 4;    // groups of matrix entries a wave keeps loaded or in flight

// One sparse operand: CSR (scaling, inspection, long rows, row tiles) and its panel layout.
struct Mat {
    Csr csr;
    Panels pan;
    int nlong;
    const int* longrows;
    int layout;  // 0 panels, 1 row tiles
    // Row tiles for the launches of one LP, per layout, reducing by a workgroup the rows that the
    // layout does (null recs: none, see flat_tiles).
    Csr flat[2];
    TwoPhase tp;  // panel layout, vectors beyond the L2: in place of the panels' sweep
};

// The matrix of a one-workgroup solve: slices of 64 rows, each as wide as its longest row; a
// slot holds two consecutive entries of one row (columns in the halves of a 32-bit word,
// values side by side), slot p of lane l of slice s is entry ptr[s] + 64 p + l and belongs to
// row row[64 s + l] (a permutation; lanes without a row hold the row count). Slots past a row's
// end hold zeros whose column is the length of the gathered vector.
struct Sell {
    int slices;  // 0: not built (see solo_admits)
    int slots;
    const int* ptr;  // [slices + 1]
    const int* row;  // [64 slices]
    const unsigned* col;
    const double* v;
    const float* v32;  // FP32 storage form only
};

struct DevLP {
    int m, n;
    long long nnz;
    int nred;          // blocks of the fixed-grid reductions
    Mat A, AT;
    Sell sA, sAT;
    // scaled problem data
    const double *c, *bl, *bu, *xl, *xu;
    const double *R, *C, *Ri, *Ci;
    // iterate state (scaled space)
    double *x, *y, *xa, *ya;          // current and running averages
    double *ax, *axa, *aty, *atya;    // A~x, A~x_avg, A~^T y, A~^T y_avg
    double *xan, *yan;                // anchor (start of the current restart cycle)
    double *xp, *yp, *axp, *atyp;     // point of the previous evaluation (candidate rays)
    double *axan, *atyan;             // A~x, A~^T y of the anchor
    // Residual restarts of the Halpern form (restart_metric 1): z - T(z) as (x, y, A~x) parts,
    // written by the iteration epilogues for the last iterate before an evaluation (fr_*) and
    // for the first iterate of a restart cycle, the anchor (fa_*).
    int restart_metric;
    double *fr_x, *fr_y, *fr_ax, *fa_x, *fa_y, *fa_ax;
    // iteration form of the current solve: 0 averaged PDHG, 1 reflected Halpern PDHG with
    // reflection rho. In the Halpern form (x, y, ax) is the Halpern iterate and (xa, ya, axa)
    // the PDHG output T(z), the only candidate of the evaluations.
    int method;
    double rho;
    int omega_steps;                  // square-root steps of the primal-weight update (>= 1)
    int pw_rule;                      // 1 smoothing (omega_steps), 2 PID controller
    double kp, ki, kd;                // gains of the PID rule
    double *partials;                 // nred * kNT
    Scalars* sc;
    double* trace;
    double *out_x, *out_y, *out_z;
    // FP32 storage form: the FP32 loop iterates on the correction (dx, dy) around the FP64
    // master point (xh, yh); d32 = c~ - A~^T yh, lo32/hi32 = x~ bounds - xh,
    // rl32/ru32 = b~ bounds - A~ xh and yh32 = yh, all computed in FP64 and rounded.
    int fp32;
    float *dx, *dxa, *dy, *dya, *adx;
    float *d32, *lo32, *hi32, *rl32, *ru32, *yh32;
    double *xh, *yh;
};

// One LP of a batched solve: its device problem and the solve-time options.
struct BatchJob {
    DevLP P;
    double eps_rel;
    double eps_infeas;
    long long max_iters;
    long long trace_cap;
    int eval_every;
    int restarts_on;
    const double* x0;
    const double* y0;
    long long limit_ticks;  // time limit in device wall-clock ticks (0: none)
    const long long* t0;    // device wall clock at the start of the call (null: the LP's reset)
    // pinned host memory of the result, when the LP has it: the scalar state, and x, y, z
    Scalars* host_sc;
    double* host;
    // one-workgroup solver: the SoloVariant, the reduction blocks whose order its evaluations
    // keep, and the slices (slots) of A and A^T staged in LDS
    int variant, eval_blocks;
    int a_slices, a_slots, at_slices, at_slots;
    int plain_stop;  // an evaluation past the time limit sums in plain index order (time_limit_passed)
};

// Block maps of a block-diagonal batch: entry b of a map is (LP index, tile or block of it).
struct MapTile {
    int job;
    TileRec tile;
};
struct MultiMaps {
    const BatchJob* jobs;
    int count;
    const MapTile* map_a;    // row tiles of every A
    int n_a;
    const MapTile* map_at;   // row tiles of every A^T
    int n_at;
    const int2* map_red;  // reduction blocks (nred per LP)
    int n_red;
    const int2* map_elem; // vector blocks (ceil(max(m, n) / kBlock) per LP)
    int n_elem;
    int* active;          // number of LPs still running (MULTI_ACTIVE) or each LP's status (MULTI_STATUS)
    // The tile maps are grouped by form v = 2 * fp32 + method (FP64 / FP32 storage, averaged /
    // Halpern) and row-tile shape h: the tiles of group g = 3 v + h are entries
    // [off_a[g], off_a[g] + cnt_a[g]) of map_a (and likewise of map_at), so every launch runs
    // one kernel specialised per form and shape present.
    int off_a[12], cnt_a[12], off_at[12], cnt_at[12];
    int keep;  // plain loads of the matrices (see kKeepMulti)
};

constexpr int kMapGroups = 4 * kTileShapes;

enum MultiLaunch {
    MULTI_PRIMAL = 0, MULTI_DUAL, MULTI_AX_ALL, MULTI_AX_FP32, MULTI_ATY, MULTI_AXA, MULTI_ATYA, MULTI_PARTIALS,
    MULTI_DECIDE, MULTI_INIT, MULTI_REBASE_INIT, MULTI_MATERIALIZE, MULTI_APPLY, MULTI_EXTRACT, MULTI_RESET,
    MULTI_ACTIVE, MULTI_STATUS
};

// ---- setup ------------------------------------------------------------------------
void launch_fill(double* p, long long n, double v, hipStream_t s);
void launch_scale_pass(const DevLP& P, int* A_rp, int* A_ci, double* A_v, const int* AT_rp, const int* perm,
                       double* R, double* C, double* rf, double* cf, int use_sum, hipStream_t s);
void launch_gather(const int* perm, const double* src, double* dst, long long nnz, hipStream_t s);
void launch_prepare(const DevLP& P, double* c, double* bl, double* bu, double* xl, double* xu, double* R, double* C,
                    double* Ri, double* Ci, double* x0, double* y0, hipStream_t s);
void launch_norms(const DevLP& P, hipStream_t s);
// Power iteration on A~^T A~: the start vector (normalised into v, sigma_max and sigma_prev
// cleared), then `iters` steps (u = A~ v, w = A~^T u, sigma_max = ||u||, v = w / ||w||).
void launch_power_start(const DevLP& P, unsigned long long seed, double* v, hipStream_t s);
void launch_power_steps(const DevLP& P, int iters, double* v, double* u, double* w, hipStream_t s);
void launch_finalize_setup(const DevLP& P, double eta_override, double omega_override, double c0, hipStream_t s);

// ---- solve ------------------------------------------------------------------------
// omega_override > 0 starts the solve at that primal weight instead of the set-up one.
void launch_reset(const DevLP& P, double eps_rel, double eps_infeas, long long max_iters, int eval_every, int restarts_on,
                  long long trace_cap, hipStream_t s, int term_mode = 0, double omega_override = 0.0);
// Statistics (products, reductions, decision in mode 2) of the point held in x = xa, y = ya.
void launch_evaluate_point(const DevLP& P, hipStream_t s);
// p[i] <- 0 where p[i] is finite (the recession cone of a bound vector).
void launch_zero_finite(double* p, long long n, hipStream_t s);
void launch_init_state(const DevLP& P, const double* x0, const double* y0, hipStream_t s);
void launch_spmv_store(const Mat& M, const double* xin, double* out, const Scalars* gate, hipStream_t s);
// reps pairs of products (A~ x, then A~^T y) in the given layout (0 panels, 1 row tiles) in the
// precision of the solve, stored to the A~x and A~^T y buffers: the trial of the layout tuner.
void launch_layout_trial(const DevLP& P, int layout, int reps, hipStream_t s);
void launch_primal(const DevLP& P, int it, hipStream_t s);
void launch_dual(const DevLP& P, int it, hipStream_t s);
void launch_evaluate(const DevLP& P, int mode, hipStream_t s);  // mode 0 regular, 1 init, 2 final
void launch_apply_restart(const DevLP& P, hipStream_t s);
void launch_stop(const DevLP& P, int status, hipStream_t s);
void launch_extract(const DevLP& P, hipStream_t s);
void launch_to_float(const double* src, float* dst, long long n, hipStream_t s);
void launch_materialize(const DevLP& P, hipStream_t s);
// Batched form: `grid` workgroups take LPs jobs[order[0]], jobs[order[1]], ... from the
// device counter (which must start at 0) and each solves one LP at a time, entirely on chip.
// lds_cap > 0: each workgroup holds lds_cap bytes of LDS (at most kSmallLpLdsMax) and solves an LP
// from LDS when small_lp_lds_bytes(LP) <= lds_cap (bit-identical result, lower latency).
constexpr int kSmallLpLdsMax = 112 * 1024;
void launch_batch(const BatchJob* jobs, const int* order, int count, int* counter, int grid, hipStream_t s,
                  int lds_cap = 0);
size_t small_lp_lds_bytes(const DevLP& P);

// One-workgroup solver over Sell matrices (lp_one_workgroup.h). Instances by threads and by
// the rows and columns a thread keeps in registers.
enum SoloVariant {
    SOLO_NONE = -1,
    SOLO_256 = 0,  // 256 threads, one row and one column each, matrices in LDS
    SOLO_512,      // 512 threads, one each, matrices in LDS
    SOLO_1024,     // 1024 threads, two columns and one row each
    SOLO_WIDE,     // 1024 threads, four columns and two rows each
    SOLO_WIDE32,   // 1024 threads, ten columns and five rows each (FP32 storage form)
    SOLO_GLOBAL    // 1024 threads, every operand in global memory, gathered vectors in LDS
};
// Rows and columns whose operands the registers of 1024 threads hold.
constexpr bool solo_register_dims(int m, int n, bool fp32) {
    return (n <= 4096 && m <= 2048) || (fp32 && n <= 10240 && m <= 5120);
}
constexpr bool solo_sorted(int m, int n) { return n <= 2048 && m <= 1024; }
constexpr int solo_threads(int variant) { return variant == SOLO_256 ? 256 : variant == SOLO_512 ? 512 : 1024; }
constexpr int kSoloMaxDim = 14000;          // rows and columns: the gathered FP64 vector stays within LDS
constexpr long long kSoloMaxNnz = 65536;
// Entries of a row, summed by one thread while the others wait. us per iteration of a batch's LP
// with one long row, one thread / row tiles: 200 x 400 (tiles in LDS) 136 entries 4.1 / 6.8, 168
// 5.0 / 7.2, 264 9.1 / 8.0, 400 13.4 / 9.3; 800 x 1600 (tiles in global memory) 136 entries 5.3 / 20.9,
// 408 14.3 / 23.8, 1600 50 / 37. The limit lies on the safe side of the first crossover.
constexpr int kSoloMaxRow = 128;
constexpr int kSoloLdsMax = 152 * 1024;     // dynamic LDS of a workgroup at most
// Set-up of a two-phase layout: entries per cell, then the entries placed (cell_base: a cell's
// first place in block order, [block * tiles + tile]; cell_k: in its tile, [tile * blocks + block]).
void launch_tp_count(const TwoPhase& M, const Csr& A, int* counts, hipStream_t s);
void launch_tp_fill(const TwoPhase& M, const Csr& A, const int* cell_base, const int* cell_k, unsigned short* lcol,
                    double* v, float* v32, unsigned short* pos, hipStream_t s);
void launch_fill_sell(const Csr& M, const Sell& S, unsigned* col, double* v, float* v32, hipStream_t s);
int solo_lds_bytes(int m, int n, int fp32, int a_slots, int at_slots);  // of one LP with that many staged slots
// The power iteration of launch_power_start / launch_power_steps (chunks of iters steps, the
// chunk test included) of an LP with Sell matrices in one launch; `G` are the slices of the two
// matrices staged in LDS and lds the bytes that takes.
constexpr long long kSoloPowerNnz = 45000;
struct SoloStage {
    int a_slices, a_slots, at_slices, at_slots;
};
void launch_solo_power(const DevLP& P, const SoloStage& G, int lds, unsigned long long seed, int iters, int chunks,
                       hipStream_t s);
void launch_solo(int threads, const BatchJob* jobs, const int* order, int count, int* counter, int grid, int lds,
                 hipStream_t s);

// Allocation-free batched form: the job table, LP order and work counter of at most
// kStaticBatchMax LPs live in a file-scope device array of the kernel source (one copy per
// device, kept until the process ends). static_batch_scratch returns its device address on
// `device`, which must be the current device; the address is looked up once per device.
constexpr int kStaticBatchMax = 4096;
constexpr int kBatchCounters = 8;  // work counters of a batched call (one per launch)
struct StaticBatchScratch {
    BatchJob* jobs;  // kStaticBatchMax entries
    int* order;      // kStaticBatchMax entries
    int* counter;    // kBatchCounters work counters
    long long* t0;   // device wall clock at the start of the call
};
hipError_t static_batch_scratch(int device, StaticBatchScratch* out);
size_t static_batch_scratch_bytes();
// launch_solo_start does the same and writes the job table of one LP (the job travels as a
// kernel argument: no copies and no wait for them).
// Clears kBatchCounters counters and sets *t0 to the device wall clock, with a kernel (no
// memset node if the caller captures the stream).
void launch_solo_start(const BatchJob& J, BatchJob* job, int* order, int* counters, long long* t0, hipStream_t s);
void launch_batch_start(int* counters, long long* t0, hipStream_t s);
// One launch of a block-diagonal batch; it_or_mode is the iteration inside the bundle for
// MULTI_PRIMAL / MULTI_DUAL and the evaluation mode for MULTI_PARTIALS / MULTI_DECIDE.
void launch_multi(const MultiMaps& M, int kind, int it_or_mode, hipStream_t s);

}  // namespace lpgpu
