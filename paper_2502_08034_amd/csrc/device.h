// Device code shared by the kernel files: reductions, block order, global-memory accesses and
// the resolved coefficients of the FP32 residual.
#pragma once

#include "internal.h"

namespace socfv {

// ------------------------------------------------------------------------------------
// Reductions
// ------------------------------------------------------------------------------------

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// Reduce K values over the block and store them at out[0..K-1] (thread 0).  Bit k of
// maxmask selects max instead of sum for value k.  Must be reached by every thread.
template <int K>
__device__ __forceinline__ void block_store(double (&v)[K], unsigned maxmask, double *out) {
  __shared__ double sh[16][K];
  const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
  const int nthreads = blockDim.x * blockDim.y * blockDim.z;
  const int lane = tid & 63, wid = tid >> 6, nw = (nthreads + 63) >> 6;
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = ((maxmask >> k) & 1u) ? wave_max(v[k]) : wave_sum(v[k]);
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) sh[wid][k] = v[k];
  }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      double acc = sh[0][k];
      for (int w = 1; w < nw; ++w) acc = ((maxmask >> k) & 1u) ? fmax(acc, sh[w][k]) : acc + sh[w][k];
      out[k] = acc;
    }
  }
}

__device__ __forceinline__ float gbit(unsigned closed, int k) {
  return (float)(((~closed) >> k) & 1u);
}

// Block order across the eight XCDs: hardware hands consecutive workgroups to the XCDs
// in turn, so logical tile L is given to workgroup b with L contiguous per XCD.  Tiles that
// are neighbours in y and z then run on the same XCD and share its L2.
__device__ __forceinline__ int xcd_tile(int b, int nb) {
  const int q = nb >> 3, r = nb & 7;
  const int x = b & 7, k = b >> 3;
  return x * q + min(x, r) + k;
}

template <int W>
struct VecW {
  float v[W];
};

// Device-memory accesses through global-address-space pointers.  Array pointers read from a
// table in memory (the batched kernels) would otherwise be generic, and the compiler would
// emit flat accesses, which also count against the LDS wait counter and so make every LDS
// wait of a step wait for the loads in flight as well.
#define GMEM __attribute__((address_space(1)))
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));

template <int W>
__device__ __forceinline__ VecW<W> ldw(const float *p) {
  VecW<W> r;
  if constexpr (W == 4) {
    const f4v t = *(GMEM const f4v *)p;
    r.v[0] = t.x; r.v[1] = t.y; r.v[2] = t.z; r.v[3] = t.w;
  } else if constexpr (W == 2) {
    const f2v t = *(GMEM const f2v *)p;
    r.v[0] = t.x; r.v[1] = t.y;
  } else {
    r.v[0] = *(GMEM const float *)p;
  }
  return r;
}

template <int W>
__device__ __forceinline__ void stw(float *p, const VecW<W> &r) {
  if constexpr (W == 4) {
    f4v t;
    t.x = r.v[0]; t.y = r.v[1]; t.z = r.v[2]; t.w = r.v[3];
    *(GMEM f4v *)p = t;
  } else if constexpr (W == 2) {
    f2v t;
    t.x = r.v[0]; t.y = r.v[1];
    *(GMEM f2v *)p = t;
  } else {
    *(GMEM float *)p = r.v[0];
  }
}

template <int W>
__device__ __forceinline__ unsigned ldflags(const uint8_t *p) {
  if constexpr (W == 4) return *(GMEM const unsigned *)p;
  else if constexpr (W == 2) return *(GMEM const unsigned short *)p;
  else return *(GMEM const uint8_t *)p;
}

template <int W>
__device__ __forceinline__ VecW<W> zerow() {
  VecW<W> r;
#pragma unroll
  for (int k = 0; k < W; ++k) r.v[k] = 0.f;
  return r;
}

template <int W>
struct CoefW {        // per-lane coefficients of one plane (W cells)
  VecW<W> wx, wym, wyp, wzl, wzu, r0;
  VecW<W> kap;        // per-cell activity (kernels instantiated for an activity field)
  float wxr;          // x face velocity after the lane's last cell
  unsigned fl;
};

// Resolved coefficients of W cells for the FP32 residual in the form
//   R_P = src_P - s_P e_P + sum_f a_f (s_nb(f) - s_P),
// a_f = max(inflow velocity through f, 0) + G_f (zero on closed faces and on the outlet
// face, whose advective flux s_P w is part of e), e_P = div_P + lam_P, and src_P = lam_P s_eq,
// or the frozen FP64 residual r0 for a correction (whose s_in and s_eq are 0).  Cells that
// are not updated (fibre, held) get zero coefficients, so R = 0 there and a sweep keeps their
// value, which the initial state sets (0 on fibre cells, s_eq or 0 on held cells).
template <int W>
struct ResW {
  VecW<W> axm, axp, aym, ayp, azm, azp, e, src;
};

// max(w, 0) + G with one rounding (h = 1/2): w + |w| is 2w or 0 exactly.  With h = 0 and
// G = 0 the coefficient is 0, which is how cells that are not updated get theirs without
// a branch.
__device__ __forceinline__ float inflow_coef(float h, float w, float G) {
  return fmaf(h, w + fabsf(w), G);
}

// ACT: the activity field is set and its values came with the plane's loads (a load here
// would make the step wait for every load in flight).  ADJ: coefficients of the transpose
// system A^T psi = g in the same form, r = src - psi e + sum_f b_f (psi_nb - psi): b_f takes
// the outflow velocity through f (max(w_out, 0) + G_f), the outlet face's flux w psi_P goes
// to the diagonal, e = lam + w_out at the outlet, and src = g_P = gscale w_out on outlet
// cells (plus r0 for a correction).  Behind the inlet psi_nb = 0, as s_in is 0.
template <bool DC, bool ACT, bool ADJ, int W>
__device__ __forceinline__ void resolvew(const SweepArgs<float> &a, const CoefW<W> &c, int x,
                                         int y, int z, bool up, ResW<W> &q) {
  const int nx = a.g.nx, ny = a.g.ny;
  // walls of this row / plane as closed-face bits (y, z)
  const unsigned wall = (y > 0 ? 0u : (unsigned)FL_YM) | (y < ny - 1 ? 0u : (unsigned)FL_YP) |
                        (z > 0 ? 0u : (unsigned)FL_ZM) | (up ? 0u : (unsigned)FL_ZP);
  const float sg = ADJ ? -1.f : 1.f;     // inflow (forward) or outflow (transpose) velocity
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const unsigned f = (c.fl >> (8 * k)) & 0xffu;
    const int xk = x + k;
    const bool outlet = xk == nx - 1;
    const int nf = __popc(f & FL_FIBRE);
    const bool upd = (f & FL_PORE) && !(a.pinned && nf > 0);
    // not updated: every face closed and no advective part
    const unsigned closed = upd ? (f | wall) : (unsigned)FL_FIBRE;
    const float h = upd ? 0.5f : 0.f;
    const float lam = a.Da * (ACT ? c.kap.v[k] : 1.f) * (float)nf;
    const float wxm = c.wx.v[k], wxp = k == W - 1 ? c.wxr : c.wx.v[k + 1];
    // inlet face: Dirichlet value on the face, G = 2 (closed bit 0 is never set there); the
    // outlet face's flux is all on the diagonal
    q.axm.v[k] = inflow_coef(h, sg * wxm, gbit(closed, 0) + (upd && xk == 0 ? 1.f : 0.f));
    q.axp.v[k] = inflow_coef(h, outlet ? 0.f : -sg * wxp, outlet ? 0.f : gbit(closed, 1));
    q.aym.v[k] = inflow_coef(h, sg * c.wym.v[k], gbit(closed, 2));
    q.ayp.v[k] = inflow_coef(h, -sg * c.wyp.v[k], gbit(closed, 3));
    q.azm.v[k] = inflow_coef(h, sg * c.wzl.v[k], gbit(closed, 4));
    q.azp.v[k] = inflow_coef(h, -sg * c.wzu.v[k], gbit(closed, 5));
    float e, src;
    if (ADJ) {
      e = lam + (outlet ? wxp : 0.f);
      src = (outlet ? a.gscale * wxp : 0.f) + (DC ? c.r0.v[k] : 0.f);
    } else {
      const float div = (wxp - wxm) + (c.wyp.v[k] - c.wym.v[k]) + (c.wzu.v[k] - c.wzl.v[k]);
      e = div + lam;
      src = DC ? c.r0.v[k] : lam * a.s_eq;
    }
    q.e.v[k] = upd ? e : 0.f;
    q.src.v[k] = upd ? src : 0.f;
  }
}

// One value <-> 64-bit words that carry a tag beside 32 bits of it: written and read with relaxed
// agent-scope atomics, a word with the awaited tag is data and signal in one (see resident.hip).
template <typename T>
struct Wire {
  static constexpr int N = sizeof(T) / 4;     // words per value
};

__device__ __forceinline__ void put_word(unsigned long long *p, unsigned bits, unsigned tag) {
  __hip_atomic_store(p, ((unsigned long long)tag << 32) | bits, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long get_word(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ void put_value(unsigned long long *p, T v, unsigned tag) {
  if constexpr (sizeof(T) == 4) {
    put_word(p, __builtin_bit_cast(unsigned, v), tag);
  } else {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    put_word(p, (unsigned)b, tag);
    put_word(p + 1, (unsigned)(b >> 32), tag);
  }
}

// Reads a value; false while a word still carries another tag.
template <typename T>
__device__ __forceinline__ bool get_value(const unsigned long long *p, unsigned tag, T &v) {
  if constexpr (sizeof(T) == 4) {
    const unsigned long long a = get_word(p);
    v = __builtin_bit_cast(float, (unsigned)a);
    return (unsigned)(a >> 32) == tag;
  } else {
    const unsigned long long a = get_word(p), b = get_word(p + 1);
    v = __builtin_bit_cast(double, (b << 32) | (unsigned)a);
    return ((unsigned)(a >> 32) == tag) & ((unsigned)(b >> 32) == tag);
  }
}

// Time that a wait has taken, in ticks of the 100 MHz clock, for its limit.  A step between two
// looks counts for at most 1 ms: one in which this process's work was off the chip is longer.
// (32 bits each: the kernels that wait have few registers left.)
struct Waited {
  unsigned last = 0;
  float sum = -1.f;             // below 0: not looked yet
  __device__ __forceinline__ bool over(float limit) {
    const unsigned now = (unsigned)wall_clock64();
    sum = sum < 0.f ? 0.f : sum + (float)min(now - last, 100000u);
    last = now;
    return sum >= limit;
  }
};

}  // namespace socfv
