// iod_internal.h -- shared between the C-ABI host code and the gfx950 kernels
// of libiod. Not part of the public interface (see include/iod.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace iodk {

// One observation row of the device table, TAB_W doubles:
//   [0] whole RK4 steps before the observation (also in KArgs::ns as int32)
//   [1] partial step tau (0 when the observation is on the grid)
//   [2..4] chief position at the observation time
//   [5..8] sin(az_obs), cos(az_obs), sin(el_obs), cos(el_obs)
//   [9] observed range (0 when the problem has angles only)
constexpr int TAB_W = 10;
constexpr int TAB_NS = 0, TAB_TAU = 1, TAB_RC = 2, TAB_SA = 5, TAB_CA = 6, TAB_SB = 7, TAB_CB = 8;
constexpr int TAB_RANGE = 9;

// Rows staged in LDS at a time by every workgroup.
constexpr int OBS_CHUNK = 64;

// Threads per workgroup of the FP64 kernels that give a particle several
// lanes: four waves, one for each SIMD of a compute unit (workgroups of two
// waves were placed two to a unit on the same pair of SIMDs, and took 1.3
// times as long as one lane per particle).
constexpr int SPLIT_BS = 256;

// Global-best record and argmin slot: [key, index, state[6]].
constexpr int REC = 8;

// Chief data of the FP32 propagation, which integrates the deputy's offset
// from the chief: for each of the four stage inputs C of a chief RK4 step
// (FP64, the integrator's own order), CST_W floats
//   d2x = Cx - (1 - mu), Cy, Cz, 1/|d1|^2, 1/|d2|^2,
//   (1 - mu)/|d1|^5, mu/|d2|^5, 1 - (1 - mu)/|d1|^3 - mu/|d2|^3,
// with d_j the chief's offset from primary j (d1 = d2 + (1, 0, 0)).
constexpr int CST_W = 8;
constexpr int CST_STEP = 4 * CST_W;   // floats per RK4 step
// Steps of chief data staged in LDS at a time; the per-step table carries
// this many zero rows past its last step, so a chunk never reads past it.
constexpr int CST_CHUNK = 16;

// Dynamics, observation table and cost of one problem.
struct KArgs {
    const double *tab;  // device [K][TAB_W]
    const int32_t *ns;  // device [K] whole steps before each observation
    int32_t K;
    int32_t mode;       // 0 = sum e_k^2, 1 = sum e_k
    bool fast;          // in-range sqrt/reciprocal sequences allowed (false: IEEE path only)
    double mu, mu1;     // mu and 1 - mu
    double h, h2, h6;   // h, h/2, h/6
    double w;           // 1 / sigma^2
    double wr;          // 1 / sigma_range^2, 0 = angles only
    // chief data of the FP32 propagation (null until an FP32 call needs it)
    const float *cst;   // device [ns[K-1] + CST_CHUNK][CST_STEP]: every grid step
    const float *cpt;   // device [K][CST_STEP]: each observation's partial step (if any)
    const double *cobs; // device [K + 1][6]: the chief state at t = 0, then at each observation
};

// Swarm variants (bits of ProbDesc::flags; the values of iod.h's IOD_PSO_*).
constexpr uint32_t PSO_PER_DIM_R = 2u;

// One problem of a swarm launch (a single problem or one member of a batch).
struct ProbDesc {
    KArgs k;
    double omega, eta1, eta2;   // Algorithm 1 weights
    double kappa;               // constriction factor (1 when off)
    double tol;                 // Algorithm 2 tolerance, 0 = off
    int32_t tol_lag;            // Algorithm 2 lag
    uint32_t flags;             // PSO_PER_DIM_R
    int64_t grid_n[6];          // grid initialisation levels per dimension
    int64_t grid_g;             // grid points (particles below it sit on the grid), 0 = off
    double lo[6], hi[6];        // initialisation box
    double chief[6];            // chief state at t = 0
    uint64_t seed, problem;     // Philox key word 0, counter word 2
    double *hist;               // device [hist_len] global-best costs, or null
    int64_t hist_len;
    int64_t m;                  // particles
    int64_t off;                // first particle in the swarm arrays
    int64_t slot_off;           // first argmin slot
    int64_t nslots;             // ceil(m / block)
    int32_t block;              // particles per workgroup of the swarm kernels (and per argmin slot)
    int16_t lanes;              // adjacent lanes per particle of the FP64 propagations: 1, 2 or 4
    int16_t solo;               // FP64 swarm launches of a batch: one wave per SIMD at a time
};

// Swarm storage of one launch. desc/work are null for a single problem.
struct SwarmArrays {
    const ProbDesc *desc;       // device [nprob]
    const int32_t *work;        // device [grid][2] = (problem, tile)
    double *x, *v, *p, *jp, *cost;  // [6][ld] / [ld] structure of arrays
    double *slots;              // [2][total_slots][REC]
    double *recs;               // [2][nprob][REC]
    double *stop;               // [nprob] Algorithm 2: -1 running, else the last iteration run
    const int32_t *porder;      // [nprob] problems by RK4 steps, longest first (per-problem
                                // launches dispatch in this order), or null: index order
    int64_t ld, total_slots, nprob;
    const int32_t *active = nullptr;  // [nprob]: 0 = the problem's workgroups of an evaluation,
                                      // gradient or normal-equation launch exit at once; null: all run
};

// Packed placement of the gradient and normal-equation launches: one
// (problem, particle) pair per thread, [n][2]; null: one problem per workgroup.
struct Lanes {
    const int32_t *pairs = nullptr;
    int64_t n = 0;
    const int64_t *count = nullptr;  // device: the number of valid pairs (overrides n when set)
};

// Largest top-k of the mixed-precision ranking.
constexpr int TOPK_MAX = 256;

// Steps between adjoint checkpoints.
constexpr int ADJ_CKPT = 64;

// Pipelined sensitivities (k_sens_pipe): particles per workgroup, steps handed
// over at a time forward and back, and the most steps of an evaluation that
// they take: a segment of the reverse sweep and one block more have to fit a
// compute unit's LDS.
constexpr int PIPE_P = 16;
constexpr int PIPE_FWD = 8, PIPE_SUB = 8;
constexpr int32_t PIPE_MAX_STEPS = 4096, PIPE_MAX_SEG = 32;
// One step of stage data and the three hand-over states, in double2: going
// forward without the velocities, in three chunks (produced, made Jacobians,
// used).
constexpr int PIPE_STEP = 12 * PIPE_P + PIPE_P + PIPE_P / 2;
constexpr int PIPE_TSTEP = 12 * PIPE_P, PIPE_SLOTS = 3;
constexpr int PIPE_XEND = 3 * 6 * PIPE_P / 2;

// Steps between its checkpoints: as few as the adjoint's scratch rows (one per
// ADJ_CKPT steps and ADJ_CKPT more) can hold, in whole blocks; at most 32.
__host__ __device__ inline int32_t pipe_segment(int32_t steps)
{
    const int32_t rows = (steps + ADJ_CKPT - 1) / ADJ_CKPT + ADJ_CKPT;
    const int32_t n = (steps + rows - 1) / rows;
    return n <= PIPE_SUB ? PIPE_SUB : (n + PIPE_SUB - 1) / PIPE_SUB * PIPE_SUB;
}

// A launch's turn, decided by a number on the device: it runs only while
// above < *count <= upto. Two forms of a launch with complementary gates let
// the refinement switch between them as its problems retire, with no host
// round trip. A null count: always runs.
struct Gate {
    const int32_t *count = nullptr;
    int32_t above = 0, upto = 0x7fffffff;
};

// LDS of a workgroup whose longest segment has seg steps.
inline int64_t pipe_lds_bytes(int32_t seg, bool tan, bool adj)
{
    const int64_t fwd = tan ? PIPE_SLOTS * PIPE_FWD * PIPE_TSTEP : 0;
    const int64_t rev = adj ? (seg + PIPE_SUB) * PIPE_STEP : 0;
    return (PIPE_XEND + (fwd > rev ? fwd : rev)) * 16;
}

struct PipeArgs {
    int32_t sub = 1;                 // workgroups per work entry (a batch)
    int32_t seg = PIPE_SUB;          // steps between checkpoints
    int32_t mode = -1;               // >= 0 overrides the cost mode
    const int32_t *done = nullptr;   // [columns]: results not wanted, or null
    Gate gate;
    double *chi2 = nullptr, *jtj = nullptr, *jtr = nullptr, *jrows = nullptr;
    int64_t jstride = 0, jld = 0;
    double *grad = nullptr, *work = nullptr;
    int64_t wld = 0;
    // launch_sens_stored: [columns] whose checkpoints are the column's (< 0: skipped)
    const int32_t *stored = nullptr;
};

// The refinement's trials (launch_gn_trials).
struct TrialArgs {
    const ProbDesc *descs = nullptr;   // the candidates'
    const int32_t *work = nullptr;     // active problems, [*count][2]
    const int32_t *count = nullptr;
    int simds = 0;
    bool first = false;                // the candidates themselves: only chi2t and ckpt, and stored
    int32_t T = 1;
    int64_t ld = 0;
    const double *x = nullptr, *jtj = nullptr, *jtr = nullptr, *grad = nullptr, *lam = nullptr;
    const double *jrows = nullptr;
    int64_t jstride = 0, jld = 0;
    const int32_t *done = nullptr;
    double hd = 0.0, alpha = 0.0;
    double *xt = nullptr, *chi2t = nullptr;
    double *ckpt = nullptr;            // [rows][6][ld], every seg steps and after the last; or null
    int32_t seg = PIPE_SUB;            // a power of two
    int32_t *stored = nullptr;
};

}  // namespace iodk
