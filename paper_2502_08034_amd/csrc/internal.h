// Internal interface between the HIP kernels (kernels.hip) and the host runtime (api.cpp).
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <vector>

namespace socfv {

// Per-cell flag byte: bits 0..5 = face shared with a fibre voxel (x-, x+, y-, y+, z-, z+),
// bit 6 = pore cell.  Domain walls are not flagged (they are known from the position).
constexpr uint8_t FL_XM = 1, FL_XP = 2, FL_YM = 4, FL_YP = 8, FL_ZM = 16, FL_ZP = 32,
                  FL_FIBRE = 63, FL_PORE = 64;

// Reduction slots (double per block, NV values per block).
constexpr int NV = 4;

// One problem on the device.  Face velocities are stored per cell for the cell's lower
// x / y / z face (x = 0 face: inlet; y = 0 and z = 0 faces: walls, zero), plus the outlet
// plane wxo (ny * nz) for the x = nx faces; upper y / z wall faces are zero by contract.
template <typename T>
struct Faces {
  const T *wx, *wy, *wz, *wxo;
};

struct Grid {
  int nx, ny, nz;
  long long n;          // nx * ny * nz
};

// Arguments of one explicit sweep.
template <typename T>
struct SweepArgs {
  Grid g;
  const uint8_t *flags;
  Faces<T> w;
  const float *kappa;   // nullable: uniform activity 1
  const T *s;           // state (or correction) read
  T *s_new;             // state (or correction) written
  const float *r0;      // defect correction: frozen FP64 residual in FP32 (else null)
  T dt, s_in, s_eq, Da; // in the correction form s_in = s_eq = 0
  T gscale;             // transpose sweeps: g_P = gscale * w_out,P on outlet cells
  int pinned;
  double lo, hi;        // bound check on the written state (ignored for corrections)
  double *partial;      // nullable: per-block [sum R^2, violations, sum R, -]
  int zc;               // z cells per block
  const int *gate = nullptr;  // nullable: the launch returns at once unless *gate == 0
                              // (device-side stop of the solve loop)
};

// FP64 residual refresh for the defect correction:
//   t = s64 + delta;  s64_new = t;  r0 = R64(t) (stored FP32); partials of R64.
struct RefreshArgs {
  Grid g;
  const uint8_t *flags;
  Faces<double> w;
  const float *kappa;
  const double *s64;
  const float *delta;   // nullable: zero correction
  double *s64_new;
  float *r0;
  double s_in, s_eq, Da;
  int pinned;
  double lo, hi;
  double *partial;
  int zc;
};

// Adjoint sweep: psi_new = psi + dt (g - A^T psi) (reversed advection).
template <typename T>
struct AdjointArgs {
  Grid g;
  const uint8_t *flags;
  Faces<T> w;
  const float *kappa;
  const T *psi;
  T *psi_new;
  const float *r0;      // correction form: frozen FP64 adjoint residual (else null)
  T dt, Da, gscale;     // g_P = gscale * w_out,P on outlet cells (0 in correction form)
  int pinned;
  double *partial;
  int zc;
};

struct AdjRefreshArgs {
  Grid g;
  const uint8_t *flags;
  Faces<double> w;
  const float *kappa;
  const double *psi64;
  const float *delta;
  double *psi64_new;
  float *r0;
  double Da, gscale;
  int pinned;
  double *partial;
  int zc;
};

struct SolveCtl;

// One problem of a batched launch (device table entry).
struct BatchProb {
  int nx, ny, nz;
  int w, rx;            // two-sweep items: cells per lane, lanes per row segment
  const uint8_t *flags;
  const float *wx, *wy, *wz, *wxo;
  const float *kappa;
  float *s0, *s1;       // ping-pong buffers: parity 0 reads s0, writes s1
  const float *r0;      // correction form: frozen FP64 residual (else unused)
  float dt, Da, s_in, s_eq;
  double lo, hi;
  int pinned;
  int gx, gy, gz, zc;   // tile grid of this problem: 64 x ty lanes x zc planes, or for the
                        // two-sweep path tiles of shape (w, rx) (tile2_xy) x zc planes
  int tile0;            // index of its first tile in the work list
  int two;              // items of the two-sweep kernel (else of the single-sweep one)
  SolveCtl *ctl;        // device-side loop state of this problem
  const double *rpart;  // its refresh partials (rnblk blocks)
  int rnblk;
};

// work: tile numbers of the unfinished problems; *nwork (device) their count
void launch_batch_sweep(const BatchProb *probs, const int *tile_prob, const int *work,
                        const int *nwork, int nblocks, int ty, int parity, bool dc,
                        double *partial, hipStream_t st);
// two sweeps per launch over the work list's (problem, tile) items; correction form, no
// activity field.  grab: two device ints, zero before the first launch; each launch takes
// items from grab[0] and leaves both at zero when it ends
void launch_batch_sweep2(const BatchProb *probs, const int *tile_prob, const int *work,
                         const int *nwork, int *grab, int nblocks, int parity, double *partial,
                         hipStream_t st);
void launch_batch_reduce(const BatchProb *probs, int n, const double *partial, double *out,
                         hipStream_t st);

// Iterative upsampling (even nx, ny, nz): coarse mask (fibre iff all eight children are
// fibre), coarse staggered FP64 face velocities (half the sum of the four fine faces), and
// the prolongation of a coarse state to the fine pore cells.
void launch_coarse_mask(const Grid &g, const uint8_t *flags, uint8_t *solid_c, hipStream_t st);
void launch_restrict(const Grid &g, const Faces<double> &w, double *ux_c, double *uy_c,
                     double *uz_c, hipStream_t st);
void launch_prolong(const Grid &g, const uint8_t *flags, const double *s_c, double *s_f,
                    hipStream_t st);

// Launch shapes.
struct Tiles {
  int ty;   // threads (rows) along y per block; x is one 64-wide wave
  int zc;   // z cells marched per block
  int zc2;  // z cells per block of the two-sweep kernel
  int two;  // FP32 sweeps two per launch (shapes below 2^30 cells)
  int rx = 64;  // two-sweep tiles: lanes per row segment (64: one row per wave; 32: two)
};

// Two-sweep tiles: a block of 1024 lanes holds rows of rx lanes (rx = 64: 16 rows of one wave
// each; rx = 32: 32 rows, two per wave), w cells per lane, and writes its interior
// (rx - 2) w x (1024 / rx - 2) cells.  gx, gy: tiles along x and y.
inline void tile2_xy(int nx, int ny, int w, int rx, int &gx, int &gy) {
  const int ox = (rx - 2) * w, oy = 1024 / rx - 2;
  gx = (nx + ox - 1) / ox;
  gy = (ny + oy - 1) / oy;
}

// Relative cost per lane of 32-lane rows against 64-lane rows, measured on the 1024 x 512 x 256
// slab (10% longer per lane: a wave's loads span two rows).
constexpr double RX32_COST = 1.10;

// The row-segment width with the lower cost of the lanes it computes per plane (ties: 64).
inline int pick_rx(int nx, int ny, int w) {
  int ax, ay, bx, by;
  tile2_xy(nx, ny, w, 64, ax, ay);
  tile2_xy(nx, ny, w, 32, bx, by);
  return RX32_COST * bx * by < (double)ax * ay ? 32 : 64;
}

// Explicit Nernst model (FP64): transport step on every pore cell; electrode (reactive)
// cells take sigma(V - eta) with eta relaxed toward the overpotential balancing the
// transport step.  eta is updated in place (each cell touches only its own).
struct NernstArgs {
  Grid g;
  const uint8_t *flags;
  Faces<double> w;
  const float *kappa;   // nullable: uniform activity 1
  const double *s;
  double *s_new;
  double *eta;
  double s_in, dt, Da, omega, V, K;   // V = logit(s_eq), K = 1 / sqrt(s_eq (1 - s_eq))
  double *partial;      // nullable: per-block [sum ((s'-s)/dt)^2, non-finite, -, -]
  int zc;
};
void launch_nernst(const NernstArgs &a, const Tiles &t, hipStream_t st);

// ---- upstream flow step: steady Stokes flow by projection steps (flow.hip) ------------
// Face arrays in the staggered layout (x faces (nz, ny, nx+1), y faces (nz, ny+1, nx),
// z faces (nz+1, ny, nx)).  code[a][f]: bit 15 = open face; bits 2n..2n+1 = class of the
// neighbour face n (x-, x+, y-, y+, z-, z+) of the same orientation: 0 beyond the inlet /
// outlet plane (zero gradient), 1 open, 2 closed along the face normal, 3 wall across it.
constexpr uint16_t FC_OPEN = 0x8000;
// Scalar slots of the flow step (device doubles after the partials)
// (FS_DONE: nonzero once the step's CG has met its target; FS_CG_STEP its iterations; FS_ALPHA the
// last one's alpha; FS_STALL: a step ran out of launched CG iterations (1) or its whole CG was given
// up (2), and everything enqueued after it returns at once)
enum FlowSlot { FS_TARGET = 0, FS_DONE = 1, FS_CG_STEP = 2, FS_CG_TOTAL = 3, FS_STEPS = 4,
                FS_STALL = 5, FS_ALPHA = 6, FS_N = 7 };
struct FlowArgs {
  Grid g;
  const uint8_t *flags;
  uint16_t *code[3];
  uint8_t *ccode;        // per cell: open-neighbour mask | inlet (64) | outlet (128); 0 = fibre
  double *u[3];          // velocity (updated in place by the projection)
  double *us[3];         // predictor output u*
  double *p, *r, *q, *d[2];       // pressure and CG vectors (cells)
  double dt, p_in, theta2;        // theta2: (CG stop factor)^2
  int nbc, nbf;          // blocks of the cell kernels / per face array of the face kernels
  int *corder, *forder[3];        // logical block of each workgroup (flow_order)
  unsigned long long *words;      // exchange words of the whole CG (CGW_WORDS)
  int *lost;                      // raised when a wait of the whole CG ran into its limit (null:
                                  // separate kernels)
  unsigned long long limit;       // that limit, in ticks of the 100 MHz clock
  double *prz[2], *prr[2], *pdq;  // per-block CG partials (cell kernels), ping-pong by parity
  double *pdu;           // per-block [sum du^2, sum u^2] of the projection, (3 nbf) x 2
  double *pdiv;          // per-block [max |div u|, inlet flux] (cell kernels), nbc x 2
  double *pfl;           // per-block sum of b^2 + (diag p)^2 of the CG start (the floor)
  double *sc;            // FlowSlot scalars
};
int flow_cell_blocks(const Grid &g);
int flow_face_blocks(const Grid &g);
// plane: cells or faces of one z plane
void flow_order(long long plane, int nb, int *order);
void launch_flow_codes(const FlowArgs &a, hipStream_t st);
void launch_flow_predict(const FlowArgs &a, hipStream_t st);
void launch_flow_cg_init(const FlowArgs &a, hipStream_t st);
// both CG kernels of iteration j of at most cap
void launch_flow_cg_iter(const FlowArgs &a, int j, int cap, hipStream_t st);
// a step's CG (cg_init included) in one launch of up to m iterations, from the pressure p to the
// pressure q; 2 m + 2 tags from tag0
// Largest box, 208 workgroups.  Its sums go from every workgroup to every other one, so an
// iteration grows with their number; 100 steps, one launch against the separate kernels (later ones
// / from rest): 40x32x32 9.1 / 9.4 ms against 18.4 / 19.0, 56x38x38 13.6 / 15.6 against 19.6 / 21.6,
// 60x42x42 (207 workgroups) 22.9 / 20.1 against 25.0 / 22.6, 62x42x42 (214) 34.2 / 23.2 against
// 33.8 / 23.6, 118x32x31 (229) 80.9 / 36.3 against 70.3 / 33.3, 64x45x45 29.0 / 25.6 against
// 23.7 / 22.6.
constexpr long long CGW_CELLS = 208 * 512;
constexpr int CGW_BLOCKS = 512;                  // its logical blocks
constexpr int CGW_SUMS = 4;                      // r.z, r.r, the floor's, d.q
constexpr long long CGW_WORDS = 2 * CGW_CELLS + 2ll * CGW_SUMS * CGW_BLOCKS * (CGW_BLOCKS / 2);
int flow_cg_whole_blocks(const FlowArgs &a);
bool flow_cg_whole(const FlowArgs &a, int ncu);
void launch_flow_cg_whole(const FlowArgs &a, int m, unsigned tag0, hipStream_t st);
// cap: CG iterations after which a step goes on without having met its target
void launch_flow_project(const FlowArgs &a, int cap, hipStream_t st);
void launch_flow_check(const FlowArgs &a, hipStream_t st);   // fills pdiv


dim3 sweep_grid(const Grid &g, const Tiles &t);
// FP32 sweeps use four cells per lane when nx % 4 == 0 (grid: 256 x cells per block)
bool vec4_path(const Grid &g);
dim3 sweep_grid_v4(const Grid &g, const Tiles &t);
// two FP32 sweeps per launch (nx even): tiles of 124 x 14 output cells
bool two_path(const Grid &g);
int two_w(const Grid &g);   // cells per lane of the two-sweep kernel: 2 for even nx, 1 for odd
dim3 sweep2_grid(const Grid &g, const Tiles &t);
// adj: sweeps of the transpose system (correction form only)
void launch_sweep2(const SweepArgs<float> &a, const Tiles &t, hipStream_t st, bool adj = false);

// Arguments of every FP64 march kernel (the fields an operation does not use are unset).
struct March64Args {
  Grid g;
  const uint8_t *flags;
  Faces<double> w;
  const float *kappa;
  const double *s;      // state (refresh: base state s64)
  const float *delta;   // refresh: FP32 correction added to s (nullable)
  double *s_new;        // sweep: s + dt R; refresh: s + delta (held cells s_eq)
  float *r0;            // refresh: R(s + delta) in FP32
  double dt, s_in, s_eq, Da;
  int pinned;
  double lo, hi;        // bound check on the written state
  double *partial;      // per block: sweep / refresh NV values, outputs NV2 values
  int zc;
  const int *gate;      // nullable: run only if *gate == gate_val
  int gate_val;
  const int *sel;       // nullable: s = pair[*sel], s_new = pair[*sel ^ 1]
  double *pair[2];
};

// One problem's gated refresh in a launch over several: its march grid and first item
struct BatchR64 {
  March64Args a;
  int gx, gy, gz, blk0;
};
// the (gated) refreshes of several problems in one launch over nitems items, item i problem of[i]'s
void launch_batch_refresh(const BatchR64 *probs, const int *of, int nitems, hipStream_t st);

// ---- kernels (launch wrappers; all enqueue on `st`) ---------------------------------

void launch_flags(const Grid &g, const uint8_t *solid, uint8_t *flags, double *partial,
                  int nblk, hipStream_t st);
int flags_blocks(const Grid &g);

// Pore cells not face-connected to the inlet plane: parent holds n + 1 ints (n < 2^31 - 1), one
// partial (their count) per block of flags_blocks(g)
void launch_connect(const Grid &g, const uint8_t *flags, int *parent, double *partial, int nblk,
                    hipStream_t st);

// velocity ingest: writes FP32 and FP64 per-cell lower faces and the outlet plane.
// partial per block: [Q_in, max|div|, max|u|, bad-face count]
void launch_velocity(const Grid &g, const uint8_t *flags, const double *ux, const double *uy,
                     const double *uz, double q, float *w32[4], double *w64[4],
                     double *partial, int nblk, hipStream_t st);
int velocity_blocks(const Grid &g);

// max over updated cells of sum max(w,0) + sum G + lam (partial slot 0, max)
void launch_maxdiag(const Grid &g, const uint8_t *flags, Faces<double> w, const float *kappa,
                    double Da, int pinned, double *partial, int nblk, hipStream_t st);

template <typename T>
void launch_sweep(const SweepArgs<T> &a, const Tiles &t, hipStream_t st);
void launch_refresh(const RefreshArgs &a, const Tiles &t, hipStream_t st);
template <typename T>
void launch_adjoint(const AdjointArgs<T> &a, const Tiles &t, hipStream_t st);
void launch_adj_refresh(const AdjRefreshArgs &a, const Tiles &t, hipStream_t st);

// FP64 sweeps (any nx) by the FP64 plane march; partials as for launch_sweep
void launch_sweep64(const SweepArgs<double> &a, hipStream_t st);
int march64_blocks(const Grid &g);
// Batched FP64 sweeps (the polish of a batched solve): one entry per problem of a launch
struct BatchM64 {
  SweepArgs<double> a;   // geometry, faces, flags, activity, dt, s_in, s_eq, Da, bounds
  double *pair[2];       // the problem's two FP64 state buffers
  int c0;                // buffer read at parity 0
  int gx, gy, gz, zc;    // its march grid (march64_shape)
  int blk0;              // its first item
  int prob;              // its index in the batch (result slot)
};
void march64_shape(const Grid &g, int &gx, int &gy, int &gz, int &zc);
// one FP64 sweep of every problem in probs[0..nprob) over nitems items; with partial (NV
// doubles per item) also each problem's sums into out[NV prob]
void launch_batch_march64(const BatchM64 *probs, int nprob, const int *item_prob, int nitems,
                          int parity, double *partial, double *out, hipStream_t st);
   // blocks (partial slots) of any FP64 march launch

// outputs of a state: partial per block (NV2 = 8 slots):
// [sum_out w s, sum_out w, F_in, F_in_adv, reaction, sum_R, sum R^2, -]
constexpr int NV2 = 8;
void launch_outputs(const Grid &g, const uint8_t *flags, Faces<double> w, const float *kappa,
                    const double *s, double s_in, double s_eq, double Da, int pinned,
                    double *partial, int nblk, hipStream_t st);
int outputs_blocks(const Grid &g);

// gradients (flags_blocks(g) blocks): dU_dkappa and partial
// [sum psi Radv, -, -, -]
void launch_gradients(const Grid &g, const uint8_t *flags, Faces<double> w, const double *s,
                      const double *psi, double s_in, double s_eq, double Da, int pinned,
                      double *dU_dkappa, double *partial, int nblk, hipStream_t st);

// deterministic second pass: out[k] = sum (or max if bit k of maxmask) over blocks
void launch_reduce(const double *partial, int nblk, int nv, unsigned maxmask, double *out,
                   hipStream_t st);

// Device-side control of the FP32 correction solve: the stop rule and the refresh decision of
// every chunk of sweeps are taken on the device, so the host enqueues many chunks between two
// reads of the state.  Sweeps run while state == CTL_RUN; the refresh while CTL_REFRESH; the
// corrections are zeroed before a chunk while `fill` is set.
enum { CTL_RUN = 0, CTL_REFRESH = 1, CTL_DONE = 2, CTL_STOP = 3, CTL_DIVERGED = 4,
       CTL_LOST = 5 };      // a resident launch was given up: its chunk has not run
struct SolveCtl {
  int state;            // CTL_*
  int fill;             // zero the corrections before the next chunk
  int cur;              // s64 buffer holding the state
  int stall;            // chunks without a 0.1% residual decrease
  long long it;         // FP32 sweeps done
  long long max_iter;
  int cycles;           // refreshes after the first
  int lost;             // raised by a resident launch that ran into its time limit
  double tol, tau, npore, reduction;   // stop tolerance, time scale, pore cells, per-cycle drop
  double target, best, res, ri;        // cycle target, best correction residual, last FP64 /
                                       // correction residual
};
// after a chunk of k sweeps (its last launch wrote nblk x NV partials): the correction
// residual, the iteration count, the cycle's stop test (refresh when due)
void launch_ctl_chunk(SolveCtl *ctl, const double *partial, int nblk, int k, hipStream_t st);
// after the (gated) refresh: the FP64 residual, the stop rule of the solve, the next cycle
void launch_ctl_refresh(SolveCtl *ctl, const double *partial, int nblk, hipStream_t st);
// The batched loop on the device: BATCH_WORKLIST rebuilds the work lists from the problems'
// states; BATCH_FILL zeroes the corrections of the problems that start a cycle; BATCH_CHUNK
// takes every sweeping problem's decision from the reduced partials `out` of a chunk of k
// sweeps; BATCH_REFRESH applies the stop rule after the problems' gated refreshes.
enum { BATCH_WORKLIST = 0, BATCH_FILL = 1, BATCH_CHUNK = 2, BATCH_REFRESH = 3 };
void launch_batch_control(const BatchProb *probs, int n, int *work, int max_tiles, int *nwork,
                          int which, const double *out, int k, hipStream_t st);
// the refresh of the correction, gated on state == CTL_REFRESH, reading s64[ctl->cur] (+ delta)
// and writing s64[ctl->cur ^ 1]
void launch_refresh_gated(const RefreshArgs &a, double *s64_0, double *s64_1,
                          const SolveCtl *ctl, hipStream_t st);
// zero two FP32 buffers of n values when ctl->fill is set
void launch_fill_gated(float *a, float *b, long long n, const SolveCtl *ctl, hipStream_t st);

// Resident sweeps: K sweeps of the correction in one launch, the box split into sub-boxes of
// X x Y columns of C cells, one sub-box per workgroup (resident.hip).
constexpr int RESIDENT_LANES = 512;            // lanes (columns) per workgroup
constexpr int RESIDENT_LDS = 156 * 1024;       // most LDS a sub-box may take
constexpr int RESIDENT_LDS_ALONE = 84 * 1024;  // more than half a CU's: one workgroup per CU
// Fewest sweeps of a resident launch: it reads the coefficients and fills the chip's registers once,
// which takes as long as a few sweeps of the other launches.  Launches of k sweeps against those, in
// time: FP32 forward / transpose on 175x89x89 k = 2 0.92 / 0.82, 4 1.05 / 0.96, 6 1.16 / 1.09, on
// 256x120x118 (lean columns) 4 0.94 / 0.85, 6 1.09 / 1.01; FP64 transpose on 128x64x64 4 0.93, 6 1.02;
// Nernst there 6 0.96, 8 1.02.  (A box of 64x32x32 gains from 2 sweeps on in FP32.)
constexpr int RESIDENT_LEAST = 6, RESIDENT_LEAST_NERNST = 8;
struct ResidentPlan {
  int C;                // cells per lane along z; 0: the box does not fit
  int X, Y;             // columns of a sub-box
  int gx, gy, gz;       // sub-boxes along x, y, z
  int lds;              // bytes of LDS per workgroup
  long long block_words, slot_words;   // exchange words per workgroup, and per slot
  double us;            // modelled time per sweep, of which for exchanged words:
  double words_us;
  int blocks() const { return gx * gy * gz; }
};
// The fastest split of a box over at most ncu workgroups (C = 0: it does not fit), and the splits
// that are faster than every one with fewer workgroups; bytes: of a value (4 or 8)
ResidentPlan resident_plan(const Grid &g, int bytes, int ncu);
std::vector<ResidentPlan> resident_plans(const Grid &g, int bytes, int ncu);
// Most exchange words and bytes of diagonals of any workgroup, FP32 or FP64
constexpr long long RESIDENT_BLOCK_WORDS = 10ll * RESIDENT_LANES;
constexpr long long RESIDENT_BLOCK_DIAG = 32ll * RESIDENT_LANES * 4;
// bytes of ResidentArgs::diag (0: not used by this plan)
long long resident_diag_bytes(const ResidentPlan &pl, int bytes);
struct ResidentArgs {
  int X, Y, gx, gy, gz;
  int K;                // sweeps of the launch
  unsigned tag0;        // tag of the first sweep; K - 1 tags are used
  unsigned long long *inbox;     // exchange words: two slots, each a run per workgroup
  long long block_words, slot_words;
  void *diag;           // lean columns: the diagonals
  int *abort;           // raised when a wait ran into its limit; the launch's output is void
  unsigned long long limit;      // longest wait, in ticks of the 100 MHz wall clock
  const int *fill;      // nullable: nonzero = start from zero instead of a.s
  int adj;              // sweeps of the transpose system
  // the Nernst iteration (a.Da is 0: transport only): reaction number, 1 / sqrt(s_eq (1 - s_eq)),
  // relaxation, V = logit(s_eq), the overpotentials read and written (they must differ)
  double Da, K0, omega, V;
  const double *eta;
  double *eta_new;
};
// a.partial is written (one entry per workgroup); a.s and a.s_new must differ
template <typename T>
void launch_resident(const SweepArgs<T> &a, const ResidentPlan &pl, const ResidentArgs &args,
                     hipStream_t st);

// K Nernst iterations in one launch (partials as launch_nernst's)
ResidentPlan resident_plan_nernst(const Grid &g, int ncu);
void launch_resident_nernst(const SweepArgs<double> &a, const ResidentPlan &pl,
                            const ResidentArgs &args, hipStream_t st);

// One problem of a launch over several: its arguments (p without tag0 and K), first workgroup and
// column length
template <typename T>
struct ResidentProb {
  SweepArgs<T> a;
  ResidentArgs p;
  int blk0, C;
};
// workgroup g works for problem tab[of[g]]; lds: the most any of them needs; K: sweeps of every
// problem (0: each its own p.K)
template <typename T>
void launch_resident_batch(const ResidentProb<T> *tab, const int *of, int nblocks, int lds,
                           unsigned tag0, int K, hipStream_t st);

// Static scratch of the allocation-free entry point: SCRATCH_DOUBLES doubles of device memory
// per GPU.  scratch_address gives its device address on device dev (which must be current at
// the first call for that device; the address is looked up once and kept); returns 0 or a
// hipError_t.
constexpr long long SCRATCH_DOUBLES = 1ll << 19;      // 4 MiB
constexpr int SCRATCH_MAX_DEVICES = 64;
int scratch_address(int dev, double **out);

// helpers
void launch_fill_f32(float *p, long long n, float v, hipStream_t st);
void launch_fill_f64(double *p, long long n, double v, hipStream_t st);
void launch_init_state(const Grid &g, const uint8_t *flags, const double *s_init, double s_in,
                       double s_eq, int pinned, double *s64, hipStream_t st);
void launch_f64_to_f32(const double *a, float *b, long long n, hipStream_t st);
void launch_f32_to_f64(const float *a, double *b, long long n, hipStream_t st);
void launch_mask_held(const Grid &g, const uint8_t *flags, int pinned, double *p, hipStream_t st);

}  // namespace socfv
