// Internal definitions shared by the host runtime and the HIP kernels of
// libhweno (gfx950).  Nothing here is part of the public C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/hweno.h"

namespace hweno {

// Arithmetic modes (values match HWENO_F64 ... HWENO_F32_KAHAN).
enum Prec : int { P_F64 = 0, P_F32 = 1, P_ACC64 = 2, P_KAHAN = 3 };
enum FluxKind : int { F_ADV = 0, F_BURGERS = 1, F_EULER = 2 };
enum SmoothnessKind : int { BETA_MOMENT = 0, BETA_CLASSICAL = 1 };
enum BC : int { BC_PERIODIC = 0, BC_TRANSMISSIVE = 1, BC_REFLECTIVE = 2 };
enum WeightMode : int { W_PAPER = 0, W_BETA = 1, W_BETA2 = 2, W_LINEAR = 3 };

// What a stage launch computes.
//   MODE_RHS: L(U) and U-hat of the input set, written as doubles;
//   MODE_S1 : U1 = Uhat^n + dt L(U^n), saves the hats of U^n;
//   MODE_S2 : U2 = 3/4 Uhat^n + 1/4 (Uhat1 + dt L(U1));
//   MODE_S3 : U^{n+1} = 1/3 Uhat^n + 2/3 (Uhat2 + dt L(U2)), written over U^n.
enum Mode : int { MODE_RHS = 0, MODE_S1 = 1, MODE_S2 = 2, MODE_S3 = 3 };

// Per-problem table, resident in device memory.
struct ProbDev {
    int32_t nx, ny, bc_x, bc_y;
    int64_t off_u;  // element offset of the problem's K u-bar planes
    int64_t off_d;  // element offset of its K*D derivative planes
    double dx, dy, inv_dx, inv_dy;
    double dxe, dye;   // dx^e, dy^e of the time-step rule
    double t, t_end;
    double dt;         // step being taken (0 when inactive)
    double dt_in;      // requested step when the caller supplies one
    uint64_t ax_bits;  // max wave speeds of the current state, as the bits of
    uint64_t ay_bits;  // non-negative doubles
    int32_t active;    // 1 while the current step advances this problem
    int32_t last;      // the current step lands exactly on t_end
    int32_t err;       // non-admissible state seen: ERR_STATE_BAD (a stored state),
                       // ERR_STAGE_BAD (an intermediate stage input)
    int32_t alpha_valid;  // ax_bits/ay_bits hold the speeds of the current state
    int64_t bad_cell;  // smallest flat index of a non-admissible cell
    int32_t err_next;  // err of the state being written, current at the step's end
    int32_t cur;       // state set (0 or 1) that holds the problem's state
};

// How the last launch of a step ends it.  Its tiles bring their speed maxima
// and then arrive; the last one of a problem ends the problem's step, the last
// problem writes the step counters.  Atomics on one address take 11 ns each,
// one after the other, so problems of more than SLOTS tiles spread maxima and
// arrivals over SLOTS lines (8620 tiles, 1 million cells in 1D: 100 us a step
// with one address, 57 us with 64), and batches their ends likewise.  The
// lines are apart from the problem table, which every tile reads when it
// starts: an atomic takes its line out of the L2s of all XCDs (512 problems of
// 1D, 2.1 million cells: 142 us a step with the maxima in the table, 105 apart).
constexpr int SLOTS = 64;
struct alignas(128) Slot {
    uint64_t ax, ay;   // speed maxima (of a tile group)
    int32_t arrived;   // tiles of the group, groups of a problem, problems of a group
    int32_t run, steps;  // problems of the group still short of t_end; most steps taken
};
// Per problem: its tiles in the step list, the groups they arrive in (1 or
// SLOTS) and its first line: the groups', followed by the problem's if there
// are several.
struct ProbEnd {
    int32_t ntiles, groups, slot0, pad;
};
inline int groups_of(int ntiles) { return ntiles > SLOTS ? SLOTS : 1; }
__host__ __device__ inline int lines_of(int groups) { return groups > 1 ? groups + 1 : 1; }
// Global step control, resident in device memory.  Kernels get its address
// alone: what they need only at a tile's end is then loaded there instead of
// being held in scalar registers through the tile.
struct StepCtl {
    double cfl;
    int32_t nprob;
    int32_t dim;
    int32_t nactive;   // problems still short of t_end after the last step
    int32_t step_active;  // some problem advanced in the current step
    int64_t steps;     // steps in which some problem advanced
    ProbEnd* ends;     // per problem
    Slot* slots;
    Slot* groups;      // SLOTS groups of problems and their total (batches)
};

// How a launch takes and ends a step of its problems (flags).
enum StepFlags : int {
    STEP_DT_IN = 1,    // the caller's step lengths (ProbDev::dt_in)
    STEP_CHOOSE = 2,   // the kernels choose dt themselves; else a dt kernel ran
    STEP_FLIP = 4      // the new state is in the other state set
};

// 2D tile: a strip of 64 loaded columns (60 output columns starting at i0)
// marching through rows j0 .. j0+nrows-1; slot: its group of the problem's
// tiles (number of the tile within the problem mod SLOTS).
struct Tile2D {
    int32_t prob, i0, j0;
    int16_t nrows, slot;
};

// 1D tile: 254 output cells starting at c0.
struct Tile1D {
    int32_t prob, c0;
};

// Reduction chunk: cells [start, start+count) of one problem.
struct Chunk {
    int32_t prob, start, count, pad;
};

constexpr int STRIP_OUT = 60;      // output columns per 2D strip (64 lanes - 4 halo)
constexpr int TILE1D_OUT = 254;    // output cells per 1D tile (256 threads - 2)
constexpr int STEP1D_HALO = 12;    // halo cells of a wave of the 1D step kernel
constexpr int CHUNK_CELLS = 2048;  // cells per reduction chunk

// Scheme constants of one handle.
struct Scheme {
    double gam[5];     // linear weights gamma_0..gamma_M
    double eps;
    double gas_gamma;
    double adv[2];
    int32_t weights;   // WeightMode
    int32_t Q;         // Gauss points per edge (2D)
    int32_t charwise;  // Euler: reconstruct in local characteristic variables
    int32_t smoothness;   // SmoothnessKind of p0's indicator
};

// Buffers of one state set in the internal layout.
struct StateBuf {
    void* u;  // K u-bar planes per problem (double, float, or float2 for Kahan)
    void* d;  // K*D derivative planes per problem
};

struct StageArgs {
    StateBuf in;        // U^(k): stencil input
    StateBuf in1;       // 1D right-hand sides: input of problems whose state set is 1
    StateBuf out;       // U^(k+1)
    const void* un;     // u-bar of U^n (stages 2, 3)
    void* h;            // saved hats of U^n
    double* L_out;      // MODE_RHS outputs (boundary layout, double)
    double* Uh_out;
    ProbDev* probs;
    const void* tiles;
    int32_t ntiles;
    int32_t tile_offset;
    StepCtl* ctl;
    int32_t flags;      // StepFlags
    Scheme sch;
};

struct Step1Args {
    StateBuf s[2];      // the state sets a step reads and writes, by ProbDev::cur
    ProbDev* probs;
    const Tile1D* tiles;  // of step1d_cells * 64 - STEP1D_HALO cells
    int32_t ntiles;
    int32_t flags;      // StepFlags
    StepCtl* ctl;
    Scheme sch;
};

// Steps of problems that fit one workgroup each (run1d.h).
constexpr int RUN1D_WAVES = 8;
struct Run1Args {
    StateBuf s[2];
    ProbDev* probs;
    StepCtl* ctl;
    double cfl;
    int32_t nsteps;
    int32_t flags;      // StepFlags
    // one problem on the caller's arrays in the boundary layout instead
    const double* ext_in;
    double* ext_out;
    double* dt_out;
    int64_t* bad_out;
    ProbDev prob;
    Scheme sch;
};

// --- launchers (defined in the .hip files) ------------------------------
hipError_t launch_stage1d(int prec, int flux, int mode, const StageArgs& a, int grid,
                          hipStream_t s);
// variant: register variant of the Euler stage kernels (0 or 1), ignored where
// there is one (stage2d_two_variants).
hipError_t launch_stage2d(int prec, int flux, int Q, int mode, int variant, const StageArgs& a,
                          int grid, hipStream_t s);
// all_problems: zero the speeds of every problem (queries), or only of those
// whose speeds are not current (time stepping).
// Which problems a speed reset / reduction covers: every problem (after
// set_state), those whose speeds are not current (step start), or those
// active in the step (the per-stage speeds of stages 2 and 3).
enum SpeedSel : int { SEL_STALE = 0, SEL_ALL = 1, SEL_ACTIVE = 2 };
constexpr int ERR_STATE_BAD = 1, ERR_STAGE_BAD = 2;
hipError_t launch_reset(ProbDev* probs, StepCtl* ctl, int nprob, int sel, hipStream_t s);
// all_problems: 1 = every problem (rhs / alpha queries); 0 = only problems
// still short of t_end, without a pending error and whose speeds are not
// current (time stepping: stage 3 computes them for the next step).
// u0, u1: the averages of problems whose state set is 0 and 1.
hipError_t launch_alpha(int prec, int flux, int dim, const void* u0, const void* u1, ProbDev* probs,
                        const Chunk* chunks, int nchunks, const Scheme& sch, int sel,
                        int grid, hipStream_t s);
hipError_t launch_dt(ProbDev* probs, StepCtl* ctl, int nprob, int use_dt_in, int own_ctl,
                     hipStream_t s);
// One whole 1D step; cells: cells per lane (step1d_cells).
hipError_t launch_step1d(int prec, int flux, int cells, const Step1Args& a, int grid, hipStream_t s);
// Steps of nprob problems of at most `waves` waves each.
hipError_t launch_run1d(int prec, int flux, int waves, int nprob, const Run1Args& a, hipStream_t s);
// Workgroups of the 2D stage kernels that share a CU, by their registers and LDS.
// The one-wave workgroups of the scalar laws (8 in FP64 with three Gauss points,
// up to 20 in single precision) are taken as 12 throughout.
constexpr int stage2d_slots(int prec, bool euler, int Q, bool charwise) {
    return !euler ? 12
                  : charwise ? (prec == P_F64 ? 1 : Q == 3 ? 2 : 3)
                             : (prec == P_F64 ? 3 : 5) - (Q == 3 ? 1 : 0);
}
// Whether the stage kernel has a variant 1, for one workgroup more per CU: where
// LDS, which holds the faces, would allow it.
constexpr bool stage2d_two_variants(int prec, bool euler, int Q, bool charwise) {
    return euler && !charwise && prec != P_F64 && Q == 2;
}
// Waves that hold the largest of these 1D problems in one workgroup; 0 where
// it does not fit.
int run1d_waves(const hweno_problem* probs, int32_t nprob, const hweno_config& cfg);
// Most steps of so many problems that one launch of the run kernel takes.
int run1d_steps(int nprob);
// Cells per lane of the 1D step kernel for these problems.
int step1d_cells(const hweno_problem* probs, int32_t nprob);
// What the host asks of a problem's table entry.
struct ProbStatus {
    double t, ax, ay;
    int64_t bad_cell;
    int32_t err, nx;
};
// What a conversion does besides: make the entry that of a new state at time
// t; leave the status in pinned host memory.
struct PackOp {
    double t;
    int32_t set_t, pad;
    ProbStatus* status;
};
// Converts one problem's state between the boundary layout (double,
// ext[((var*K + c)*ny + j)*nx + i]) and the internal planes of b0 or b1, the
// one prob->cur names: from src if given, else to dst.
hipError_t launch_pack(int prec, const double* src, double* dst, StateBuf b0, StateBuf b1,
                       ProbDev* prob, int64_t off_u, int64_t off_d, int K, int nvar, int64_t ncell,
                       const PackOp& op, hipStream_t s);
hipError_t launch_status(const ProbDev* prob, ProbStatus* out, hipStream_t s);

// --- host helpers of the C ABI (api.cpp) --------------------------------
// Checks problems and configuration (ERR_ARG with the reason as the
// thread's last error).
int validate_problems(const hweno_problem* probs, int32_t nprob, const hweno_config* cfg);
// Sets the thread's last error (hweno_last_error(NULL)); returns code.
int thread_error(int code, const char* fmt, ...);
Scheme scheme_of(const hweno_problem& p0, const hweno_config& cfg);
// Segment height a handle starts with; as tile_rows, the library's to shorten.
constexpr int DEFAULT_ROWS = 32;
// Segment height of the 2D tiles of one launch over these problems: `cap` rows,
// fewer where that would leave the GPU idle.
int split_rows(const hweno_problem* probs, int32_t nprob, const hweno_config& cfg, int cap);
// Tiles of one problem at that height, and the first row of segment s.
int tiles_2d(int nx, int ny, int rows);
// Tiles of a 1D problem in the step kernel with that many cells per lane.
inline int tiles_1d(int nx, int cells) {
    const int out = 64 * cells - STEP1D_HALO;
    return (nx + out - 1) / out;
}
__host__ __device__ inline int segment_row(int s, int nseg, int ny) {
    return (int)((int64_t)s * ny / nseg);
}
// Tile lists are sized for max(tiles at 8 rows, min(tiles at 2 rows, this)).
constexpr int64_t SPLIT_TILES = 4096;
// Per-problem table entry (static fields; time 0, speeds unknown).
ProbDev probdev_of(const hweno_problem& pr, const hweno_config& cfg, int64_t off_u,
                   int64_t off_d);

}  // namespace hweno
