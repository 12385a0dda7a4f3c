// HIP kernels (gfx950) of the upstream flow step: steady Stokes flow through the voxel pore
// space by the projection method (Eqs. (cp1)-(cp4), Algorithm "Flow Simulation" with explicit
// momentum diffusion), in the Stokes regime of Eq. (stokes-flow) (no momentum advection).
//
// Discretisation (nondimensional: h = rho = mu = 1): normal velocity on open faces (both
// cells pore, or the inlet / outlet face of a pore cell), pressure in pore cells, applied
// pressure p_in at the inlet face and 0 at the outlet face (half a cell from the first / last
// cell centre), no-slip on fibre voxel faces and the y / z walls, zero normal gradient of the
// velocity across the inlet and outlet planes.  One step:
//   predictor   u* = u + dt L u                       (Eq. (cp1) without advection)
//   pressure    (-D G) p = D gbc - D u* / dt           (Eq. (cp4)), Jacobi-preconditioned CG
//   projection  u' = u* - dt (G p + gbc)               (Eq. (cp2))
// The CG starts from the previous step's pressure and stops once dt ||r|| (the divergence
// the projection leaves) is below theta times the previous step's velocity change, or at the
// per-step cap.  A fixed point of the step satisfies the pressure equation exactly (a CG
// started at its solution does not move), so it is the discrete Stokes solution L u = G p,
// D u = 0 whatever the inner tolerance; the tolerance only sets how fast the steps get there.
//
// Everything is FP64 (the velocity is an FP64 input of the state-of-charge solve).  The step
// is bandwidth bound (a few flops per 8-byte value); kernels are grid-stride loops over
// faces or cells with coalesced rows.  The CG's scalars are never sent to the host: every
// block of the next kernel sums the previous kernel's per-block partials itself, in a fixed
// order, so all blocks take the same (deterministic) values and the same stop decision.
#include "device.h"

#include <algorithm>
#include <vector>

namespace socfv {

namespace {

constexpr int FB = 256;        // threads per block of every flow kernel
constexpr int FLOW_MAX_BLOCKS = 2048;

__device__ __forceinline__ double fwave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ double fwave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// Block-wide sum (or max) of v, returned to every thread; fixed order.  Every thread of the
// block must reach it.
__device__ __forceinline__ double block_total(double v, bool mx, double *sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  v = mx ? fwave_max(v) : fwave_sum(v);
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = sh[0];
#pragma unroll
  for (int k = 1; k < FB / 64; ++k) t = mx ? fmax(t, sh[k]) : t + sh[k];
  return t;
}

// Sum of a[k * stride] for k < n by the whole block (same value in every thread and block).
// Eight loads per thread are in flight at once (indices past n read a[0], selected away).
__device__ __forceinline__ double sum_partials(const double *a, int n, int stride, double *sh) {
  double v = 0.0;
  for (int k0 = 0; k0 < n; k0 += 8 * FB) {
    double t[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int k = k0 + j * FB + (int)threadIdx.x;
      t[j] = a[(long long)(k < n ? k : 0) * stride];
      t[j] = k < n ? t[j] : 0.0;
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) v += t[j];
  }
  return block_total(v, false, sh);
}

// N such sums together (stride 1): one pass of loads and one exchange, each sum in the order of
// sum_partials and block_total.  Their waits do not add up.
template <int N>
__device__ __forceinline__ void sum_partials_n(const double *const (&a)[N], int n,
                                               double (&sh)[N][FB / 64], double (&out)[N]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < N; ++i) out[i] = 0.0;
  constexpr int J = 4;                       // (eight would cost registers, and with them waves)
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += J * FB) {
    double t[N][J];
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int k = k0 + j * FB + (int)threadIdx.x;
        t[i][j] = a[i][k < n ? k : 0];
        t[i][j] = k < n ? t[i][j] : 0.0;
      }
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = 0; j < J; ++j) out[i] += t[i][j];
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    out[i] = fwave_sum(out[i]);
    if (lane == 0) sh[i][w] = out[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    out[i] = sh[i][0];
#pragma unroll
    for (int k = 1; k < FB / 64; ++k) out[i] += sh[i][k];
  }
}

// The logical block of a workgroup (flow_order), and the place of its partials: a block's own,
// so that every sum is taken in one order whichever workgroup does the work.
struct Logical {
  unsigned lb, slot;
};
__device__ __forceinline__ Logical logical(const int *__restrict__ order) {
  const unsigned o = (unsigned)order[blockIdx.x];
  return {o & 0xffffu, o >> 16};
}

__device__ __forceinline__ bool pore_at(const uint8_t *fl, const Grid &g, int x, int y, int z) {
  return (fl[x + (long long)g.nx * (y + (long long)g.ny * z)] & FL_PORE) != 0;
}

struct FaceDims {
  int fx, fy, fz;
  long long n;
};
__device__ __forceinline__ FaceDims face_dims(const Grid &g, int a) {
  FaceDims d{g.nx + (a == 0), g.ny + (a == 1), g.nz + (a == 2), 0};
  d.n = (long long)d.fx * d.fy * d.fz;
  return d;
}

// Is the face of orientation a at (x, y, z) of its face array open?
__device__ __forceinline__ bool face_open(const uint8_t *fl, const Grid &g, int a, int x, int y,
                                          int z) {
  if (a == 0) {
    if (x == 0) return pore_at(fl, g, 0, y, z);
    if (x == g.nx) return pore_at(fl, g, g.nx - 1, y, z);
    return pore_at(fl, g, x - 1, y, z) && pore_at(fl, g, x, y, z);
  }
  if (a == 1) {
    if (y == 0 || y == g.ny) return false;
    return pore_at(fl, g, x, y - 1, z) && pore_at(fl, g, x, y, z);
  }
  if (z == 0 || z == g.nz) return false;
  return pore_at(fl, g, x, y, z - 1) && pore_at(fl, g, x, y, z);
}

// Pressure-operator row of a pore cell: diagonal and the open-neighbour mask (bit n for
// neighbour n = x-, x+, y-, y+, z-, z+).  Inlet / outlet faces add 2 to the diagonal.
struct PRow {
  double diag;
  unsigned nb;
};
__device__ __forceinline__ PRow prow(uint8_t fl, const Grid &g, int x, int y, int z) {
  PRow r{0.0, 0u};
  if (x > 0) { if (!(fl & FL_XM)) { r.nb |= 1u; r.diag += 1.0; } } else r.diag += 2.0;
  if (x < g.nx - 1) { if (!(fl & FL_XP)) { r.nb |= 2u; r.diag += 1.0; } } else r.diag += 2.0;
  if (y > 0 && !(fl & FL_YM)) { r.nb |= 4u; r.diag += 1.0; }
  if (y < g.ny - 1 && !(fl & FL_YP)) { r.nb |= 8u; r.diag += 1.0; }
  if (z > 0 && !(fl & FL_ZM)) { r.nb |= 16u; r.diag += 1.0; }
  if (z < g.nz - 1 && !(fl & FL_ZP)) { r.nb |= 32u; r.diag += 1.0; }
  return r;
}

// Cell code byte (built once per call): bits 0..5 the open-neighbour mask, bit 6 the inlet
// face, bit 7 the outlet face; 0 for fibre cells (a pore cell always has an open face or the
// inlet: it is face-connected to the inlet).  The CG kernels need nothing else of the cell.
constexpr unsigned CC_INLET = 64u, CC_OUTLET = 128u;
__device__ __forceinline__ int diag_of(unsigned cc) {
  return __popc(cc & 63u) + 2 * (int)((cc >> 6) & 1u) + 2 * (int)((cc >> 7) & 1u);
}
__device__ __forceinline__ PRow prow_code(unsigned cc) {
  return PRow{(double)diag_of(cc), cc & 63u};
}

// Sum of v over the open neighbours of a cell.  Branch-free: a closed neighbour's index is
// replaced by the cell's own (always in bounds) and its value selected away, so all six loads
// are in flight together (a load under a branch makes the join wait for every load).
__device__ __forceinline__ double nb_sum(const double *__restrict__ v, long long c, unsigned nb,
                                         long long sy, long long sz) {
  const double a0 = v[(nb & 1u) ? c - 1 : c];
  const double a1 = v[(nb & 2u) ? c + 1 : c];
  const double a2 = v[(nb & 4u) ? c - sy : c];
  const double a3 = v[(nb & 8u) ? c + sy : c];
  const double a4 = v[(nb & 16u) ? c - sz : c];
  const double a5 = v[(nb & 32u) ? c + sz : c];
  return (((nb & 1u) ? a0 : 0.0) + ((nb & 2u) ? a1 : 0.0)) +
         (((nb & 4u) ? a2 : 0.0) + ((nb & 8u) ? a3 : 0.0)) +
         (((nb & 16u) ? a4 : 0.0) + ((nb & 32u) ? a5 : 0.0));
}

// z = r / diag.  The diagonals are the whole numbers 1 to 10, and r / n follows from RN(1 / n) by
// one correction, exactly as the division rounds it (Markstein's theorem: the first quotient is
// within one unit in the last place).  inv holds (1 / diag, diag) by cell code.
struct alignas(16) InvDiag {
  double y, n;
};
__device__ __forceinline__ void fill_inv(InvDiag *inv) {
  const int n = diag_of(threadIdx.x);
  inv[threadIdx.x] = InvDiag{n ? 1.0 / (double)n : 0.0, (double)n};
}
__device__ __forceinline__ double over_diag(double r, const InvDiag &v) {
  const double q = r * v.y;
  return fma(fma(-q, v.n, r), v.y, q);
}

// nb_sum of z = r / diag
__device__ __forceinline__ double nb_sum_z(const double *__restrict__ r,
                                           const uint8_t *__restrict__ code, long long c,
                                           unsigned nb, long long sy, long long sz,
                                           const InvDiag *inv) {
  const long long at[6] = {(nb & 1u) ? c - 1 : c,   (nb & 2u) ? c + 1 : c,
                           (nb & 4u) ? c - sy : c,  (nb & 8u) ? c + sy : c,
                           (nb & 16u) ? c - sz : c, (nb & 32u) ? c + sz : c};
  double v[6];
  unsigned cc[6];
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    v[k] = r[at[k]];
    cc[k] = code[at[k]];
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) v[k] = over_diag(v[k], inv[cc[k]]);
  return (((nb & 1u) ? v[0] : 0.0) + ((nb & 2u) ? v[1] : 0.0)) +
         (((nb & 4u) ? v[2] : 0.0) + ((nb & 8u) ? v[3] : 0.0)) +
         (((nb & 16u) ? v[4] : 0.0) + ((nb & 32u) ? v[5] : 0.0));
}

// ---- face classification ---------------------------------------------------------------
__global__ void __launch_bounds__(FB) k_flow_codes(FlowArgs a) {
  const Grid g = a.g;
  const Logical me = logical(a.forder[blockIdx.y]);
  const int o = blockIdx.y;
  const FaceDims d = face_dims(g, o);
  uint16_t *code = a.code[o];
  for (long long f = (long long)me.lb * FB + threadIdx.x; f < d.n;
       f += (long long)gridDim.x * FB) {
    const unsigned fu = (unsigned)f, t = fu / (unsigned)d.fx;
    const int x = (int)(fu - t * (unsigned)d.fx);
    const int y = (int)(t % (unsigned)d.fy), z = (int)(t / (unsigned)d.fy);
    uint16_t c = 0;
    if (face_open(a.flags, g, o, x, y, z)) {
      c = FC_OPEN;
      for (int n = 0; n < 6; ++n) {
        const int b = n >> 1, s = (n & 1) ? 1 : -1;
        const int xx = x + (b == 0 ? s : 0), yy = y + (b == 1 ? s : 0), zz = z + (b == 2 ? s : 0);
        const bool inside = xx >= 0 && xx < d.fx && yy >= 0 && yy < d.fy && zz >= 0 && zz < d.fz;
        unsigned cls;
        if (!inside) cls = (b == 0) ? 0u : 3u;      // open plane: zero gradient; y / z wall
        else if (face_open(a.flags, g, o, xx, yy, zz)) cls = 1u;
        else cls = (b == o) ? 2u : 3u;
        c |= (uint16_t)(cls << (2 * n));
      }
    }
    code[f] = c;
  }
}

__global__ void __launch_bounds__(FB) k_flow_cell_codes(FlowArgs a) {
  const Grid g = a.g;
  const Logical me = logical(a.corder);
  for (long long c = (long long)me.lb * FB + threadIdx.x; c < g.n;
       c += (long long)gridDim.x * FB) {
    const uint8_t fl = a.flags[c];
    unsigned cc = 0;
    if (fl & FL_PORE) {
      const unsigned cu = (unsigned)c, row = cu / (unsigned)g.nx;
      const int x = (int)(cu - row * (unsigned)g.nx);
      const int y = (int)(row % (unsigned)g.ny), z = (int)(row / (unsigned)g.ny);
      cc = prow(fl, g, x, y, z).nb | (x == 0 ? CC_INLET : 0u) | (x == g.nx - 1 ? CC_OUTLET : 0u);
    }
    a.ccode[c] = (uint8_t)cc;
  }
}

// ---- predictor: u* = u + dt L u ----------------------------------------------------------
__global__ void __launch_bounds__(FB) k_flow_predict(FlowArgs a) {
  if (a.sc[FS_STALL] != 0.0) return;
  const Grid g = a.g;
  const Logical me = logical(a.forder[blockIdx.y]);
  const int o = blockIdx.y;
  const FaceDims d = face_dims(g, o);
  const uint16_t *__restrict__ code = a.code[o];
  const double *__restrict__ u = a.u[o];
  double *__restrict__ us = a.us[o];
  const long long off[6] = {-1, 1, -(long long)d.fx, (long long)d.fx,
                            -(long long)d.fx * d.fy, (long long)d.fx * d.fy};
  for (long long f = (long long)me.lb * FB + threadIdx.x; f < d.n;
       f += (long long)gridDim.x * FB) {
    const unsigned c = code[f];
    double out = 0.0;
    if (c & FC_OPEN) {
      const double u0 = u[f];
      double nbv[6];
#pragma unroll
      for (int n = 0; n < 6; ++n)      // branch-free gather: closed neighbours read the face
        nbv[n] = u[((c >> (2 * n)) & 3u) == 1u ? f + off[n] : f];
      double acc = 0.0, diag = 0.0;
#pragma unroll
      for (int n = 0; n < 6; ++n) {
        const unsigned cls = (c >> (2 * n)) & 3u;
        acc += cls == 1u ? nbv[n] : 0.0;
        diag += cls == 3u ? 2.0 : (cls != 0u ? 1.0 : 0.0);
      }
      out = u0 + a.dt * (acc - diag * u0);
    }
    us[f] = out;
  }
}

// ---- pressure CG -------------------------------------------------------------------------
// init: r = b - A p with b = D gbc - D u* / dt; partials of r.z, r.r (z = r / diag) into
// parity 0.  Block 0 also sets the step's stop target from the last projection's partials.
__global__ void __launch_bounds__(FB) k_flow_cg_init(FlowArgs a) {
  __shared__ double sh[FB / 64];
  if (a.sc[FS_STALL] != 0.0) return;
  const Grid g = a.g;
  const Logical me = logical(a.corder);
  if (blockIdx.x == 0) {
    const double du2 = sum_partials(a.pdu, 3 * a.nbf, 2, sh);
    if (threadIdx.x == 0) {
      a.sc[FS_TARGET] = a.theta2 * du2 / (a.dt * a.dt);
      a.sc[FS_DONE] = 0.0;
      a.sc[FS_CG_STEP] = 0.0;
    }
  }
  const long long sy = g.nx, sz = (long long)g.nx * g.ny;
  double rz = 0.0, rr = 0.0, fl = 0.0;
  for (long long c = (long long)me.lb * FB + threadIdx.x; c < g.n;
       c += (long long)gridDim.x * FB) {
    const unsigned cc = a.ccode[c];
    double rv = 0.0;
    if (cc) {
      // x faces: index c + (y + ny z); y faces: c + nx z
      const unsigned row = (unsigned)c / (unsigned)g.nx, z = row / (unsigned)g.ny;
      const long long ix = c + row;
      const long long iy = c + (long long)g.nx * z;
      const double div = (a.us[0][ix + 1] - a.us[0][ix]) + (a.us[1][iy + g.nx] - a.us[1][iy]) +
                         (a.us[2][c + sz] - a.us[2][c]);
      const double b = ((cc & CC_INLET) ? 2.0 * a.p_in : 0.0) - div / a.dt;
      const PRow pr = prow_code(cc);
      const double ap = pr.diag * a.p[c] - nb_sum(a.p, c, pr.nb, sy, sz);
      rv = b - ap;
      const double zv = rv / pr.diag;
      rz += rv * zv;
      rr += rv * rv;
      const double dp = pr.diag * a.p[c];
      fl += b * b + dp * dp;
    }
    a.r[c] = rv;
  }
  rz = block_total(rz, false, sh);
  rr = block_total(rr, false, sh);
  fl = block_total(fl, false, sh);
  if (threadIdx.x == 0) {
    a.prz[0][me.slot] = rz;
    a.prr[0][me.slot] = rr;
    a.pfl[me.slot] = fl;
  }
}

// Floor of the CG stop target: about what the recursively updated residual reaches in FP64,
// (CG_FLOOR eps)^2 (||b||^2 + ||diag p||^2) at the step's start.  Near the steady state the
// target (theta times the last velocity change) falls with the change; the floor keeps a
// target below rounding level from running the CG to the per-step cap.  It binds only there
// (the step's fixed point does not depend on it).
constexpr double CG_FLOOR = 16.0;

// Both halves of an iteration are bound by memory.  So z is not stored but taken from r wherever
// it is needed, and p, which nothing reads before the step's end, is advanced by the first half of
// the next iteration, which reads d anyway: 74 bytes a cell and iteration against 90, and
// 51.5 + 21.4 us on 256 x 128 x 128 (34 MB a vector; 4.0 and 4.9 TB/s) against 43 + 41.  More
// waves per SIMD (6, 8) and the cell codes loaded a turn ahead changed nothing.  A step's last
// p update is made by the first half that finds the target met, or, in iteration cap - 1 (which
// no first half follows), by the second half itself.

// iteration j, first half: p += alpha d_old (of iteration j - 1); stop test; d = z + beta d_old;
// q = A d; partials of d.q.  (FS_DONE is j + 1 once a block of this launch has found the target
// met: the others still have to advance p.)
__global__ void __launch_bounds__(FB) k_flow_cg_a(FlowArgs a, int j) {
  __shared__ double sh[FB / 64], sh4[4][FB / 64];
  __shared__ InvDiag inv[256];
  const double done = a.sc[FS_DONE];
  if ((done != 0.0 && done != (double)(j + 1)) || a.sc[FS_STALL] != 0.0) return;
  const Grid g = a.g;
  const Logical me = logical(a.corder);
  const int par = j & 1;
  fill_inv(inv);
  const long long c0 = (long long)me.lb * FB + threadIdx.x, stride = (long long)gridDim.x * FB;
  double s[4];
  sum_partials_n<4>({a.prz[par], a.prr[par], a.pfl, a.prz[par ^ 1]}, a.nbc, sh4, s);
  const double rz = s[0], rr = s[1], alpha = a.sc[FS_ALPHA];
  const double floor2 = (CG_FLOOR * 2.220446049250313e-16) * (CG_FLOOR * 2.220446049250313e-16) *
                        s[2];
  const double *__restrict__ dold = a.d[par ^ 1];
  if (rr <= fmax(a.sc[FS_TARGET], floor2)) {
    if (j > 0)
      for (long long c = c0; c < g.n; c += stride)
        if (a.ccode[c]) a.p[c] += alpha * dold[c];
    if (blockIdx.x == 0 && threadIdx.x == 0) a.sc[FS_DONE] = (double)(j + 1);
    return;
  }
  const double beta = j == 0 ? 0.0 : rz / s[3];
  const double *__restrict__ r = a.r;
  const uint8_t *__restrict__ code = a.ccode;
  double *__restrict__ dn = a.d[par];
  const long long sy = g.nx, sz = (long long)g.nx * g.ny;
  double dq = 0.0;
  for (long long c = c0; c < g.n; c += stride) {
    const unsigned cc = code[c];
    double dv = 0.0, qv = 0.0;
    if (cc) {
      const unsigned nb = cc & 63u;
      const InvDiag own = inv[cc];
      double nbs;
      dv = over_diag(r[c], own);
      if (j == 0) {
        nbs = nb_sum_z(r, code, c, nb, sy, sz, inv);
      } else {
        const double dc = dold[c], pv = a.p[c];
        nbs = nb_sum_z(r, code, c, nb, sy, sz, inv) + beta * nb_sum(dold, c, nb, sy, sz);
        a.p[c] = pv + alpha * dc;
        dv = dv + beta * dc;
      }
      qv = own.n * dv - nbs;
      dq += dv * qv;
    }
    dn[c] = dv;
    a.q[c] = qv;
  }
  dq = block_total(dq, false, sh);
  if (threadIdx.x == 0) a.pdq[me.slot] = dq;
}

// iteration j, second half: alpha = r.z / d.q; r -= alpha q; partials of the new r.z, r.r
// (z = r / diag) into the other parity.  last: nothing follows, so p += alpha d here
__global__ void __launch_bounds__(FB) k_flow_cg_b(FlowArgs a, int j, bool last) {
  __shared__ double sh[FB / 64], sh2[2][FB / 64];
  __shared__ InvDiag inv[256];
  if (a.sc[FS_DONE] != 0.0 || a.sc[FS_STALL] != 0.0) return;
  const Grid g = a.g;
  const Logical me = logical(a.corder);
  const int par = j & 1;
  fill_inv(inv);
  const long long c0 = (long long)me.lb * FB + threadIdx.x, stride = (long long)gridDim.x * FB;
  double s[2];
  sum_partials_n<2>({a.prz[par], a.pdq}, a.nbc, sh2, s);
  const double alpha = s[0] / s[1];
  const double *__restrict__ dn = a.d[par];
  double rzn = 0.0, rrn = 0.0;
  for (long long c = c0; c < g.n; c += stride) {
    const unsigned cc = a.ccode[c];
    if (!cc) continue;
    if (last) a.p[c] += alpha * dn[c];
    const double rv = a.r[c] - alpha * a.q[c];
    const double zv = over_diag(rv, inv[cc]);
    a.r[c] = rv;
    rzn += rv * zv;
    rrn += rv * rv;
  }
  rzn = block_total(rzn, false, sh);
  rrn = block_total(rrn, false, sh);
  if (threadIdx.x == 0) {
    a.prz[par ^ 1][me.slot] = rzn;
    a.prr[par ^ 1][me.slot] = rrn;
    if (blockIdx.x == 0) {
      a.sc[FS_CG_STEP] = (double)(j + 1);
      a.sc[FS_ALPHA] = alpha;
    }
  }
}

// ---- the whole pressure CG of a step in one launch ---------------------------------------
// For boxes of at most CGW_CELLS cells (one cell per lane, two logical blocks per workgroup, at
// most one workgroup per CU): r, z, p, d and q stay in registers, and so do the neighbours' d,
// which a lane advances itself (d = z + beta d from the neighbour's z); what travels between
// workgroups is z, and the logical blocks' partials, as tagged words that every workgroup sums in
// the order of the separate kernels.  An iteration then costs its two exchanges instead of two
// launches and, per step, launches past the end (both sides measured at CGW_CELLS), with the same arithmetic cell by cell and sum by sum.  A word is written again only
// after a sum that its readers have contributed to since they read it, so one slot per word is
// enough: z and the residual's sums after d.q's, d.q's after the residual's (which therefore
// have words of their own).  Waits
// end at a time limit as in the resident sweeps.  A workgroup can give up in the very last sum, to
// which it has contributed, and the others then come to the end; so whether a launch counts is
// decided behind it, by the projection: the new pressure goes to q, and `lost` (raised by any
// workgroup that gave up) makes FS_STALL 2 and the host repeat the step from the old pressure with
// the separate kernels.
constexpr int CGW_GROUPS = 2, CGW_LANES = CGW_GROUPS * FB;

// Sum over a group of 256 lanes, as block_total over a block of them.
__device__ __forceinline__ double group_total(double v, double (*sh)[FB / 64]) {
  const int lane = threadIdx.x & 63, w = (threadIdx.x >> 6) & 3, grp = threadIdx.x / FB;
  v = fwave_sum(v);
  __syncthreads();
  if (lane == 0) sh[grp][w] = v;
  __syncthreads();
  double t = sh[grp][0];
#pragma unroll
  for (int k = 1; k < FB / 64; ++k) t += sh[grp][k];
  return t;
}

__global__ void __launch_bounds__(CGW_LANES) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_flow_cg_whole(FlowArgs a, int m, unsigned tag0) {
  __shared__ double sh[CGW_GROUPS][FB / 64];
  __shared__ double zl[CGW_LANES], part[3][CGW_GROUPS];
  __shared__ int slots[CGW_GROUPS];
  // a wait of a sum / of z's words ran into its limit: two flags, so that between a barrier and
  // the reading of one of them no wave that is ahead can raise it
  __shared__ int dead_sum, dead_z;
  if (a.sc[FS_STALL] != 0.0) return;
  const Grid g = a.g;
  const int grp = threadIdx.x / FB, t = threadIdx.x % FB;
  const int lb = blockIdx.x * CGW_GROUPS + grp;
  const long long c = (long long)lb * FB + t;
  const long long sy = g.nx, sz = (long long)g.nx * g.ny;
  // the place of the logical block's partials (flow_order)
  const int q8 = a.nbc / 8, r8 = a.nbc % 8, long8 = r8 * (q8 + 1);
  const int run = lb < long8 ? lb / (q8 + 1) : r8 + (lb - long8) / max(q8, 1);
  if (t == 0) slots[grp] = 8 * (lb < long8 ? lb % (q8 + 1) : (lb - long8) % max(q8, 1)) + run;
  const int nb = gridDim.x;
  if (threadIdx.x == 0) dead_sum = dead_z = 0;
  unsigned long long *const zw = a.words, *const pw = a.words + 2 * CGW_CELLS;

  // waits until every word this lane asks for is there (a limit below 0.1 ms is looked at on every
  // turn: 256 of them take longer)
  const unsigned turns = a.limit < 10000 ? 0u : 255u;
  auto wait = [&](int &dead, auto &&all) {
    unsigned spins = 0;
    Waited waited;
    while (!all()) {
      if ((++spins & turns) == 0) {
        if (waited.over((float)a.limit) ||
            __hip_atomic_load(a.lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
          dead = 1;
          __hip_atomic_store(a.lost, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
      }
    }
  };
  // sums of N partials per logical block, the same in every lane (the first group takes them, in
  // sum_partials' order); the tag says which, and `first` which words
  auto share = [&](auto &v, unsigned tag, int first) {
    constexpr int N = sizeof(v) / sizeof(double);
    if (t == 0)
#pragma unroll
      for (int k = 0; k < N; ++k) part[k][grp] = v[k];
    __syncthreads();
    // one copy per workgroup: words that all of them polled would be read a hundred times from
    // the same few lines of memory
    for (int i = threadIdx.x; i < nb * N * CGW_GROUPS; i += CGW_LANES) {
      const int to = i / (N * CGW_GROUPS), k = i / CGW_GROUPS % N, from = i % CGW_GROUPS;
      if (blockIdx.x * CGW_GROUPS + from < a.nbc)
        put_value<double>(pw + 2 * ((to * CGW_SUMS + first + k) * CGW_BLOCKS + slots[from]),
                          part[k][from], tag);
    }
    const unsigned long long *const mine =
        pw + 2 * ((blockIdx.x * CGW_SUMS + first) * CGW_BLOCKS);
    double sum[N] = {};
    if (grp == 0)
#pragma unroll 1
      for (int i = t; i < a.nbc; i += FB) {
        double x[N];
        wait(dead_sum, [&] {
          bool ok = true;
#pragma unroll
          for (int k = 0; k < N; ++k)
            ok &= get_value<double>(mine + 2 * (k * CGW_BLOCKS + i), tag, x[k]);
          return ok;
        });
#pragma unroll
        for (int k = 0; k < N; ++k) sum[k] += x[k];
      }
#pragma unroll
    for (int k = 0; k < N; ++k) {
      (void)group_total(sum[k], sh);
      double s = sh[0][0];
#pragma unroll
      for (int w = 1; w < FB / 64; ++w) s += sh[0][w];
      v[k] = s;
    }
  };

  // the step's stop target, and k_flow_cg_init's part of this cell
  double target;
  {
    double v = 0.0;
    for (int k0 = 0; k0 < 3 * a.nbf; k0 += 8 * FB) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = k0 + j * FB + t;
        const double x = a.pdu[2ll * (k < 3 * a.nbf ? k : 0)];
        v += k < 3 * a.nbf ? x : 0.0;
      }
    }
    target = a.theta2 * group_total(v, sh) / (a.dt * a.dt);
  }
  const unsigned cc = c < g.n ? a.ccode[c] : 0u;
  const PRow pr = prow_code(cc);
  double p = c < g.n ? a.p[c] : 0.0, r = 0.0, z = 0.0;
  double tot[3] = {0.0, 0.0, 0.0};           // r.z, r.r, the floor's sum
  if (cc) {
    const unsigned row = (unsigned)c / (unsigned)g.nx, zz = row / (unsigned)g.ny;
    const long long ix = c + row;
    const long long iy = c + (long long)g.nx * zz;
    const double div = (a.us[0][ix + 1] - a.us[0][ix]) + (a.us[1][iy + g.nx] - a.us[1][iy]) +
                       (a.us[2][c + sz] - a.us[2][c]);
    const double b = ((cc & CC_INLET) ? 2.0 * a.p_in : 0.0) - div / a.dt;
    const double ap = pr.diag * p - nb_sum(a.p, c, pr.nb, sy, sz);
    r = b - ap;
    z = r / pr.diag;
    tot[0] += r * z;
    tot[1] += r * r;
    const double dp = pr.diag * p;
    tot[2] += b * b + dp * dp;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) tot[k] = group_total(tot[k], sh);
  // neighbours: those of this workgroup's cells come from its LDS copy of z, the others as words
  const int off[6] = {-1, 1, -(int)sy, (int)sy, -(int)sz, (int)sz};
  unsigned far = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    const int at = (int)threadIdx.x + off[k];
    if ((pr.nb >> k & 1u) && (at < 0 || at >= CGW_LANES)) far |= 1u << k;
  }
  double dn[6], d = 0.0, rz_old = 0.0, floor2 = 0.0;
#pragma unroll
  for (int k = 0; k < 6; ++k) dn[k] = 0.0;
  int j = 0;
  bool gone = false;                         // (the same in every lane)
  for (;; ++j) {
    const unsigned tag = tag0 + 2u * (unsigned)j;
    // the cells' z and the sums of the residual
    if (cc) put_value<double>(zw + 2 * c, z, tag);
    zl[threadIdx.x] = z;
    if (j == 0) {
      share(tot, tag, 0);
      floor2 = (CG_FLOOR * 2.220446049250313e-16) * (CG_FLOOR * 2.220446049250313e-16) * tot[2];
    } else {
      double two[2] = {tot[0], tot[1]};
      share(two, tag, 0);
      tot[0] = two[0];
      tot[1] = two[1];
    }
    gone = dead_sum != 0;
    if (gone || j >= m || tot[1] <= fmax(target, floor2)) break;
    // d = z + beta d, q = A d (k_flow_cg_a)
    const double beta = j == 0 ? 0.0 : tot[0] / rz_old;
    double zn[6];
    if (far)
      wait(dead_z, [&] {
        // both z neighbours' words in flight at once (a near one reads this cell's); x and y
        // neighbours are far only at the ends of the workgroup's run of cells
        bool ok = true;
#pragma unroll
        for (int k = 4; k < 6; ++k)
          ok &= get_value<double>(zw + 2 * (c + ((far >> k & 1u) ? off[k] : 0)), tag, zn[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (far >> k & 1u) ok &= get_value<double>(zw + 2 * (c + off[k]), tag, zn[k]);
        return ok;
      });
#pragma unroll
    for (int k = 0; k < 6; ++k)
      if (!(far >> k & 1u)) zn[k] = zl[(pr.nb >> k & 1u) ? threadIdx.x + off[k] : threadIdx.x];
    double qv = 0.0;
    double dq[1] = {0.0};
    if (cc) {
      auto sum = [&](const double (&v)[6]) {
        return (((pr.nb & 1u) ? v[0] : 0.0) + ((pr.nb & 2u) ? v[1] : 0.0)) +
               (((pr.nb & 4u) ? v[2] : 0.0) + ((pr.nb & 8u) ? v[3] : 0.0)) +
               (((pr.nb & 16u) ? v[4] : 0.0) + ((pr.nb & 32u) ? v[5] : 0.0));
      };
      double nbs;
      if (j == 0) {
        d = z;
        nbs = sum(zn);
#pragma unroll
        for (int k = 0; k < 6; ++k) dn[k] = zn[k];
      } else {
        d = fma(beta, d, z);
        nbs = fma(beta, sum(dn), sum(zn));
#pragma unroll
        for (int k = 0; k < 6; ++k) dn[k] = fma(beta, dn[k], zn[k]);
      }
      qv = fma(pr.diag, d, -nbs);
      dq[0] += d * qv;
    }
    dq[0] = group_total(dq[0], sh);
    share(dq, tag + 1u, 3);
    gone = dead_sum != 0 || dead_z != 0;
    if (gone) break;
    // the update (k_flow_cg_b)
    const double alpha = tot[0] / dq[0];
    rz_old = tot[0];
    double rzn = 0.0, rrn = 0.0;
    if (cc) {
      p = fma(alpha, d, p);
      r = fma(-alpha, qv, r);
      z = r / pr.diag;
      rzn += r * z;
      rrn += r * r;
    }
    tot[0] = group_total(rzn, sh);
    tot[1] = group_total(rrn, sh);
  }
  if (gone) return;
  if (c < g.n) a.q[c] = p;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    a.sc[FS_CG_STEP] = (double)j;
    a.sc[FS_DONE] = 1.0;
  }
}

// ---- projection: u' = u* - dt (G p + gbc); partials [sum (u' - u)^2, sum u'^2] -----------
// A step whose CG has neither met its target nor reached the cap has run out of launched
// iterations: nothing is projected, and the launches behind this one return until the host has
// enqueued more (the decision is the same in every block: none writes what it reads).  The same
// where the whole CG was given up.
__global__ void __launch_bounds__(FB) k_flow_project(FlowArgs a, int cap) {
  __shared__ double sh[FB / 64];
  if (a.sc[FS_STALL] != 0.0) return;
  if (a.lost && *a.lost) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.sc[FS_STALL] = 2.0;
    return;
  }
  if (a.sc[FS_DONE] == 0.0 && a.sc[FS_CG_STEP] < (double)cap) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.sc[FS_STALL] = 1.0;
    return;
  }
  const Grid g = a.g;
  const Logical me = logical(a.forder[blockIdx.y]);
  const int o = blockIdx.y;
  const FaceDims d = face_dims(g, o);
  const uint16_t *__restrict__ code = a.code[o];
  const double *__restrict__ us = a.us[o];
  double *__restrict__ u = a.u[o];
  const double *__restrict__ p = a.p;
  double du2 = 0.0, u2 = 0.0;
  for (long long f = (long long)me.lb * FB + threadIdx.x; f < d.n;
       f += (long long)gridDim.x * FB) {
    double un = 0.0;
    if (code[f] & FC_OPEN) {
      const unsigned fu = (unsigned)f, t = fu / (unsigned)d.fx;
      const int x = (int)(fu - t * (unsigned)d.fx);
      const int y = (int)(t % (unsigned)d.fy), z = (int)(t / (unsigned)d.fy);
      double gp;
      if (o == 0) {
        const long long c = (long long)x + (long long)g.nx * (y + (long long)g.ny * z);
        if (x == 0) gp = 2.0 * (p[c] - a.p_in);
        else if (x == g.nx) gp = -2.0 * p[c - 1];
        else gp = p[c] - p[c - 1];
      } else if (o == 1) {
        const long long c = (long long)x + (long long)g.nx * (y + (long long)g.ny * z);
        gp = p[c] - p[c - g.nx];
      } else {
        const long long c = (long long)x + (long long)g.nx * (y + (long long)g.ny * z);
        gp = p[c] - p[c - (long long)g.nx * g.ny];
      }
      un = us[f] - a.dt * gp;
    }
    const double dv = un - u[f];
    du2 += dv * dv;
    u2 += un * un;
    u[f] = un;
  }
  du2 = block_total(du2, false, sh);
  u2 = block_total(u2, false, sh);
  if (threadIdx.x == 0) {
    const long long b = (long long)o * a.nbf + me.slot;
    a.pdu[2 * b] = du2;
    a.pdu[2 * b + 1] = u2;
    if (o == 0 && blockIdx.x == 0) {
      a.sc[FS_CG_TOTAL] += a.sc[FS_CG_STEP];
      a.sc[FS_STEPS] += 1.0;
    }
  }
}

// ---- outputs: per block [max |D u|, inlet flux, max |u| over cell faces, outlet flux] ----
__global__ void __launch_bounds__(FB) k_flow_check(FlowArgs a) {
  __shared__ double sh[FB / 64];
  const Grid g = a.g;
  const Logical me = logical(a.corder);
  const long long sz = (long long)g.nx * g.ny;
  double dmax = 0.0, qin = 0.0, umax = 0.0, qout = 0.0;
  for (long long c = (long long)me.lb * FB + threadIdx.x; c < g.n;
       c += (long long)gridDim.x * FB) {
    const unsigned cc = a.ccode[c];
    if (!cc) continue;
    const unsigned row = (unsigned)c / (unsigned)g.nx, z = row / (unsigned)g.ny;
    const long long ix = c + row;
    const long long iy = c + (long long)g.nx * z;
    const double v[6] = {a.u[0][ix], a.u[0][ix + 1], a.u[1][iy], a.u[1][iy + g.nx], a.u[2][c],
                         a.u[2][c + sz]};
    dmax = fmax(dmax, fabs((v[1] - v[0]) + (v[3] - v[2]) + (v[5] - v[4])));
    for (int k = 0; k < 6; ++k) umax = fmax(umax, fabs(v[k]));
    if (cc & CC_INLET) qin += v[0];
    if (cc & CC_OUTLET) qout += v[1];
  }
  dmax = block_total(dmax, true, sh);
  qin = block_total(qin, false, sh);
  umax = block_total(umax, true, sh);
  qout = block_total(qout, false, sh);
  if (threadIdx.x == 0) {
    double *o = a.pdiv + 4ll * me.slot;
    o[0] = dmax;
    o[1] = qin;
    o[2] = umax;
    o[3] = qout;
  }
}

}  // namespace

int flow_cell_blocks(const Grid &g) {
  const long long b = (g.n + FB - 1) / FB;
  return (int)(b < FLOW_MAX_BLOCKS ? b : FLOW_MAX_BLOCKS);
}

int flow_face_blocks(const Grid &g) {
  const long long nmax = (long long)(g.nx + 1) * (g.ny + 1) * (g.nz + 1);
  const long long b = (nmax + FB - 1) / FB;
  return (int)(b < FLOW_MAX_BLOCKS ? b : FLOW_MAX_BLOCKS);
}

// Order of the logical blocks.  Workgroup b runs on XCD b % 8, each XCD with its own L2, and the
// blocks' window (256 nb cells) moves through the box plane by plane.  A logical block's place in
// its plane decides its XCD: each gets a band of rows over all the window's planes, so that a
// cell's z neighbours are always in the L2 that reads it and only the rows at a band's edges are
// read by two.  With runs of consecutive blocks per XCD (two planes each on 256 x 128 x 128) every
// XCD read its neighbours' planes too: 47 us for the first half of a CG iteration against
// 43 here.  order[b]: workgroup b's logical block, and << 16 the place of its partials: the
// sums run over the blocks eight apart (0, nb / 8, ... the runs' first blocks, then their second
// ones), the order in which workgroups took consecutive runs.  Bijections on [0, nb).
void flow_order(long long plane, int nb, int *order) {
  std::vector<int> lb(nb), slot(nb);
  for (int k = 0; k < nb; ++k) lb[k] = k;
  for (int b = 0; b < nb; ++b) {
    const int x = b % 8, k = b / 8;
    slot[x * (nb / 8) + std::min(x, nb % 8) + k] = b;
  }
  const auto place = [&](int k) { return (long long)FB * k % plane; };
  std::stable_sort(lb.begin(), lb.end(), [&](int a, int b) { return place(a) < place(b); });
  int at = 0;
  for (int x = 0; x < 8; ++x) {
    const int n = nb / 8 + (x < nb % 8 ? 1 : 0);
    std::sort(lb.begin() + at, lb.begin() + at + n);
    for (int k = 0; k < n; ++k) order[8 * k + x] = lb[at + k] | slot[lb[at + k]] << 16;
    at += n;
  }
}

void launch_flow_codes(const FlowArgs &a, hipStream_t st) {
  k_flow_codes<<<dim3(a.nbf, 3), FB, 0, st>>>(a);
  k_flow_cell_codes<<<a.nbc, FB, 0, st>>>(a);
}
void launch_flow_predict(const FlowArgs &a, hipStream_t st) {
  k_flow_predict<<<dim3(a.nbf, 3), FB, 0, st>>>(a);
}
void launch_flow_cg_init(const FlowArgs &a, hipStream_t st) {
  k_flow_cg_init<<<a.nbc, FB, 0, st>>>(a);
}
void launch_flow_cg_iter(const FlowArgs &a, int j, int cap, hipStream_t st) {
  k_flow_cg_a<<<a.nbc, FB, 0, st>>>(a, j);
  k_flow_cg_b<<<a.nbc, FB, 0, st>>>(a, j, j == cap - 1);
}
int flow_cg_whole_blocks(const FlowArgs &a) { return (a.nbc + CGW_GROUPS - 1) / CGW_GROUPS; }
bool flow_cg_whole(const FlowArgs &a, int ncu) {
  return a.g.n <= CGW_CELLS && flow_cg_whole_blocks(a) <= ncu;
}
void launch_flow_cg_whole(const FlowArgs &a, int m, unsigned tag0, hipStream_t st) {
  k_flow_cg_whole<<<flow_cg_whole_blocks(a), CGW_LANES, 0, st>>>(a, m, tag0);
}
void launch_flow_project(const FlowArgs &a, int cap, hipStream_t st) {
  k_flow_project<<<dim3(a.nbf, 3), FB, 0, st>>>(a, cap);
}
void launch_flow_check(const FlowArgs &a, hipStream_t st) {
  k_flow_check<<<a.nbc, FB, 0, st>>>(a);
}

}  // namespace socfv
