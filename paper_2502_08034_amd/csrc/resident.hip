// Resident sweeps (gfx950): a whole chunk of explicit sweeps in one launch, for problems that
// fit the chip's registers.
//
// Every workgroup owns a sub-box of X x Y columns of C cells along z, one column per lane, and
// keeps its cells' values and resolved coefficients in registers for all K sweeps of the
// launch; a column's z neighbours are the lane's own registers, its x and y neighbours come
// from the block's copy of the sub-box in LDS.  After a sweep the blocks exchange the values on
// their sub-boxes' faces through device memory, and nothing else moves: a sweep costs its
// arithmetic plus one exchange, where a launch per pair of sweeps reads every array again and,
// on a small box, marches ten dependent planes on a handful of CUs.
//
// Exchange.  A face value travels as one 64-bit word, the value in the low half and the sweep's
// tag in the high half (an FP64 value as two such words), written and read with relaxed
// agent-scope atomics: a reader polls the word until the tag is the sweep's, so data and signal
// arrive together and no fence or flag is needed.  Tags grow from launch to launch, so
// words of an earlier launch never match.  Each face has two slots (by the tag's parity): a
// block overwrites a slot two sweeps later, which it reaches only after its neighbour's next
// sweep arrived, that is after the neighbour has read the slot.
//
// Waits.  All blocks must be resident together: the grid is at most one block per CU and every
// CU holds one.  Should blocks wait for CUs that other work holds, or never get them (two
// processes' launches can each hold a part of them), every wait ends by a time limit: the block
// raises the abort flag, every block leaves, no state is lost (the launch writes only its output
// buffer), and the host goes on with the other launches for a while.
#include "device.h"

#include <algorithm>
#include <iterator>
#include <type_traits>

namespace socfv {

namespace {

constexpr int RT = RESIDENT_LANES;

// Side words (one value of a halo column) a lane handles, for columns of C cells: room for
// 2 (X + Y) C words over the lanes at X + Y <= 48 and a little more.
constexpr int resident_side_words(int C) { return (3 * C + 15) / 16; }

// Columns too long for nine registers per cell are kept lean (see Coefs).
constexpr bool resident_lean(int bytes, int C) { return bytes * C > 80; }

// A wave's values from LDS, 16 bytes at a time.
template <typename T>
struct V16;
template <>
struct V16<float> {
  typedef f4v type;
  static constexpr int n = 4;
};
typedef double d2r __attribute__((ext_vector_type(2)));
template <>
struct V16<double> {
  typedef d2r type;
  [[maybe_unused]] static constexpr int n = 2;
};

// Values between two columns of the LDS copy: a multiple of 16 bytes whose count of 16-byte
// units is odd, so that eight lanes of adjacent columns read all 32 banks once.
template <typename T, int C>
constexpr int col_stride() {
  return (C / V16<T>::n) % 2 ? C : C + V16<T>::n;
}

// Resolved coefficients of one cell (the residual R = src - s e + sum_f a_f (s_nb - s)).
template <typename T>
struct Res1 {
  T axm, axp, aym, ayp, azm, azp, e, src;
  // z faces encoded, one number per face for the cells on both sides: 0 if closed, else
  // 1 + |w| (rounded as in the coefficients) with the sign of the (inflow) velocity w, so that
  // with g = min(|t|, 1) the upper cell's coefficient is max(t, g) and the lower's max(-t, g)
  T tzm, tzp;
  bool upd;             // the cell is updated (a pore cell that is not held)
};

// Pins v to this place: what is computed from it is not hoisted out of the loop (the decoded
// coefficients and lane masks of a whole column would take more registers than they were encoded
// to save), and v itself is computed before.
template <typename V>
__device__ __forceinline__ void keep_in_loop(V &v) {
  asm volatile("" : "+v"(v));
}

// min(|t|, 1) and max(t, g), as medians: fmin and fmax would first quiet both arguments, an
// instruction each.
__device__ __forceinline__ float open_of(float t) {
  return __builtin_amdgcn_fmed3f(fabsf(t), 0.f, 1.f);
}
__device__ __forceinline__ float coef_of(float t, float g) {
  return __builtin_amdgcn_fmed3f(t, g, 3.4e38f);
}
__device__ __forceinline__ double open_of(double t) { return fmin(fabs(t), 1.0); }
__device__ __forceinline__ double coef_of(double t, double g) { return fmax(t, g); }

// A column's coefficients in registers.
template <typename T, int C, bool LEAN>
struct CoefsOf {
  T axm[C], axp[C], aym[C], ayp[C], azm[C], azp[C], e[C], src[C];
};
template <typename T, int C>
struct CoefsOf<T, C, true> {
  T axm[C], axp[C], aym[C], ayp[C], tz[C + 1];
};
template <typename T, int C>
using Coefs = CoefsOf<T, C, resident_lean(sizeof(T), C)>;

// The coefficients of resolvew for one cell; with adj those of the transpose system.  r0 is the
// frozen residual of a correction (null: the state itself is swept).
template <typename T>
__device__ __forceinline__ Res1<T> resolve1(const SweepArgs<T> &a, bool adj, int x, int y, int z,
                                            long long i, long long pl) {
  const int nx = a.g.nx, ny = a.g.ny, nz = a.g.nz;
  const bool inlet = x == 0, outlet = x == nx - 1;
  const T wxm = a.w.wx[i], wxp = outlet ? a.w.wxo[y + (long long)ny * z] : a.w.wx[i + 1];
  const T wym = a.w.wy[i], wyp = y < ny - 1 ? a.w.wy[i + nx] : T(0);
  const T wzm = a.w.wz[i], wzp = z < nz - 1 ? a.w.wz[i + pl] : T(0);
  const unsigned f = a.flags[i];
  const T kap = a.kappa ? (T)a.kappa[i] : T(1), r0 = a.r0 ? (T)a.r0[i] : T(0);
  const unsigned wall = (y > 0 ? 0u : (unsigned)FL_YM) | (y < ny - 1 ? 0u : (unsigned)FL_YP) |
                        (z > 0 ? 0u : (unsigned)FL_ZM) | (z < nz - 1 ? 0u : (unsigned)FL_ZP);
  const int nf = __popc(f & FL_FIBRE);
  const bool upd = (f & FL_PORE) && !(a.pinned && nf > 0);
  const unsigned closed = upd ? (f | wall) : (unsigned)FL_FIBRE;
  const T h = upd ? T(0.5) : T(0), sg = adj ? T(-1) : T(1);
  auto g = [&](int k) { return (T)(((~closed) >> k) & 1u); };
  // max(w, 0) + G with one rounding, as inflow_coef
  auto coef = [&](T w, T G) { return fma(h, w + fabs(w), G); };
  const T lam = a.Da * kap * (T)nf;
  Res1<T> q;
  q.axm = coef(sg * wxm, g(0) + (upd && inlet ? T(1) : T(0)));
  q.axp = coef(outlet ? T(0) : -sg * wxp, outlet ? T(0) : g(1));
  q.aym = coef(sg * wym, g(2));
  q.ayp = coef(-sg * wyp, g(3));
  q.azm = coef(sg * wzm, g(4));
  q.azp = coef(-sg * wzp, g(5));
  const T div = (wxp - wxm) + (wyp - wym) + (wzp - wzm);
  const T e = fma(a.Da * kap, (T)nf, adj ? (outlet ? wxp : T(0)) : div);
  const T src = adj ? (outlet ? a.gscale * wxp : T(0)) + r0 : a.r0 ? r0 : lam * a.s_eq;
  q.e = upd ? e : T(0);
  q.src = upd ? src : T(0);
  const bool pore = f & FL_PORE;
  auto face = [&](T w, unsigned fibre, bool inside) {
    return pore && inside && !(f & fibre) ? copysign(fma(T(0.5), fabs(w) + fabs(w), T(1)), w + T(0))
                                          : T(0);
  };
  q.tzm = face(sg * wzm, FL_ZM, z > 0);
  q.tzp = face(sg * wzp, FL_ZP, z < nz - 1);
  q.upd = upd;
  return q;
}

// Side columns of a sub-box in exchange order: x-, x+ (Y columns each), y-, y+ (X each); the z
// faces follow with one value per lane.  Position q of a side column: its face and place.
struct Side {
  int face, at;
};
__device__ __forceinline__ Side side_of(int q, int X, int Y) {
  if (q < Y) return {0, q};
  if (q < 2 * Y) return {1, q - Y};
  q -= 2 * Y;
  return q < X ? Side{2, q} : Side{3, q - X};
}

// What a sweep does to a cell beyond s + dt R: nothing; keep held cells of lean columns (whose
// encoded z faces do not tell them from their neighbours); the Nernst model's electrode update.
enum { RK_PLAIN = 0, RK_HELD = 1, RK_NERNST = 2 };

// K sweeps of workgroup b of one problem.
template <typename T, int C, int KIND>
__device__ __forceinline__ void resident_block(const SweepArgs<T> &a, const ResidentArgs &p,
                                               const int b) {
  if (a.gate && *a.gate != CTL_RUN) return;
  constexpr int S = col_stride<T, C>(), NV16 = V16<T>::n, WN = Wire<T>::N;
  constexpr int NJ = resident_side_words(C), NONE = 0xffff;
  constexpr bool LEAN = resident_lean(sizeof(T), C);
  typedef typename V16<T>::type vec;
  extern __shared__ __align__(16) char lds_raw[];
  __shared__ int dead;
  T *lds = reinterpret_cast<T *>(lds_raw);
  const int nx = a.g.nx, ny = a.g.ny, nz = a.g.nz;
  const int X = p.X, Y = p.Y, tid = threadIdx.x;
  const int gxy = p.gx * p.gy;
  const int bx = b % p.gx, by = (b / p.gx) % p.gy, bz = b / gxy;
  const int xe = min(X, nx - bx * X), ye = min(Y, ny - by * Y), ze = min(C, nz - bz * C);
  const int ly = tid / X, lx = tid - ly * X;
  const bool act = lx < xe && ly < ye;
  const int x = min(bx * X + lx, nx - 1), y = min(by * Y + ly, ny - 1), z0 = bz * C;
  const long long pl = (long long)nx * ny;
  const long long i0 = x + (long long)nx * (y + (long long)ny * z0);
  const bool zero = p.fill && *p.fill;
  const int stride = (X + 2) * S;            // between rows of columns
  // lanes without a column read the first one's neighbours: finite values for coefficients 0
  const int col = act ? (lx + 1) * S + (ly + 1) * stride : S + stride;
  if (tid == 0) dead = 0;

  // the lane's cells; lean columns keep the z faces encoded, the sources in LDS behind the copy
  // and the diagonals in memory (read from L2), 16 bytes per lane
  T s[C];
  Coefs<T, C> q;
  const int copy = stride * (Y + 2);
  vec *const lsrc = reinterpret_cast<vec *>(lds + (LEAN ? (copy + 3) / 4 * 4 : 0));
  vec *const ge = reinterpret_cast<vec *>(p.diag) + (long long)b * (C / NV16) * RT;
  unsigned upd = 0, pore = 0;
  T eta[KIND == RK_NERNST ? C : 1], rate[KIND == RK_NERNST ? C : 1];   // electrode cells
#pragma unroll
  for (int k0 = 0; k0 < C; k0 += NV16) {
    vec ve, vsrc;
#pragma unroll
    for (int v = 0; v < NV16; ++v) {
      const int k = k0 + v, kc = min(k, ze - 1);
      const bool in = act && k < ze;
      const long long i = i0 + pl * kc;
      const Res1<T> r = resolve1<T>(a, p.adj, x, y, z0 + kc, i, pl);
      const T on = in ? T(1) : T(0);
      s[k] = in && !zero ? a.s[i] : T(0);
      if (in && (a.flags[i] & FL_PORE)) pore |= 1u << k;
      if constexpr (KIND == RK_NERNST) {
        const int nf = __popc(a.flags[i] & FL_FIBRE);
        rate[k] = in ? p.Da * (a.kappa ? (T)a.kappa[i] : T(1)) * (T)nf / p.K0 : T(0);
        eta[k] = in && nf > 0 ? p.eta[i] : T(0);
        if (in && nf > 0) upd |= 1u << k;
      }
      q.axm[k] = in ? r.axm : T(0);
      q.axp[k] = in ? r.axp : T(0);
      q.aym[k] = in ? r.aym : T(0);
      q.ayp[k] = in ? r.ayp : T(0);
      ve[v] = in ? r.e : T(0);
      vsrc[v] = in ? r.src : T(0);
      if constexpr (LEAN) {
        q.tz[k] = on * r.tzm;
        if (k == C - 1) q.tz[C] = on * r.tzp;
        if (in && r.upd) upd |= 1u << k;
      } else {
        q.azm[k] = on * r.azm;
        q.azp[k] = on * r.azp;
        q.e[k] = ve[v];
        q.src[k] = vsrc[v];
      }
    }
    if constexpr (LEAN) {
      ge[(k0 / NV16) * RT + tid] = ve;
      lsrc[(k0 / NV16) * RT + tid] = vsrc;
    }
    // one group's loads and masks at a time: all of them together would not fit the registers
    __builtin_amdgcn_sched_barrier(0);
  }
  // the LDS copy (two, by the sweep's parity, where they fit): zero outside the box, s_in behind
  // the inlet, then the halo from memory
  constexpr int NB = LEAN ? 1 : 2;
  for (int i = tid; i < copy; i += RT)
#pragma unroll
    for (int n = 0; n < NB; ++n) lds[n * copy + i] = bx == 0 && (i % stride) < S ? a.s_in : T(0);
  T zlo = T(0), zhi = T(0);
  const bool below = act && bz > 0, above = act && bz < p.gz - 1;
  if (below && !zero) zlo = a.s[i0 - pl];
  if (above && !zero) zhi = a.s[i0 + pl * C];
  __syncthreads();
  if (act) {
#pragma unroll
    for (int k = 0; k < C; ++k) lds[col + k] = s[k];
  }
  // The lane's share of the side words: word i of a workgroup's inbox holds value k = i % C of
  // its halo column i / C.  For a column: where its values leave the LDS copy (low half) and
  // where they enter it (high half), and their first word in the neighbour's inbox.  Lean
  // columns look their words' columns up in LDS on every sweep: held in registers, they would be
  // spilled, and a reload between the exchange's stores would wait for each of them.
  auto column = [&](int qc, int &dest) -> unsigned {
    const Side f = side_of(qc, X, Y);
    const bool xface = f.face < 2, upper = f.face & 1;
    const bool there = qc < 2 * (X + Y) && f.at < (xface ? ye : xe) &&
                       (xface ? (upper ? bx < p.gx - 1 : bx > 0)
                              : (upper ? by < p.gy - 1 : by > 0));
    const int hx = xface ? (upper ? X + 1 : 0) : f.at + 1, hy = xface ? f.at + 1 : (upper ? Y + 1 : 0);
    const int ox = xface ? (upper ? X : 1) : f.at + 1, oy = xface ? f.at + 1 : (upper ? Y : 1);
    const int other = xface ? (upper ? f.at : Y + f.at) : 2 * Y + (upper ? f.at : X + f.at);
    const int nb = b + (xface ? 1 : p.gx) * (upper ? 1 : -1);
    dest = (int)(nb * p.block_words) + other * C * WN;
    return there ? (unsigned)(ox * S + oy * stride) | (unsigned)(hx * S + hy * stride) << 16
                 : NONE | (unsigned)NONE << 16;
  };
  unsigned places[LEAN ? 1 : NJ];
  int dst[LEAN ? 1 : NJ];
  uint2 *const table = reinterpret_cast<uint2 *>(lds + (LEAN ? (copy + 3) / 4 * 4 + RT * C : 0));
  if constexpr (LEAN) {
    for (int qc = tid; qc < (NJ * RT + C - 1) / C; qc += RT) {
      int dest;
      const unsigned at = column(qc, dest);
      table[qc] = make_uint2(at, (unsigned)dest);
    }
    __syncthreads();
  }
  // a word's place in the LDS copy as it leaves | as it enters << 16, or NONE twice
  auto place = [&](int m, int t, int &dest) -> unsigned {
    const int i = t + m * RT, qc = i / C, k = i - qc * C;
    unsigned at;
    if constexpr (LEAN) {
      const uint2 c = table[qc];
      at = c.x;
      dest = (int)c.y;
    } else {
      at = column(qc, dest);
    }
    dest += k * WN;
    return k < ze && (at & NONE) != NONE ? at + ((unsigned)k | (unsigned)k << 16)
                                         : NONE | (unsigned)NONE << 16;
  };
#pragma unroll
  for (int m = 0; m < NJ; ++m) {
    int dest;
    const unsigned at = place(m, tid, dest);
    if constexpr (!LEAN) {
      places[m] = at;
      dst[m] = dest;
    }
    const int i = tid + m * RT, qc = i / C, k = i - qc * C;
    const Side f = side_of(qc, X, Y);
    const int hx = f.face < 2 ? (f.face ? X : -1) : f.at, hy = f.face < 2 ? f.at : (f.face == 3 ? Y : -1);
    if ((at & NONE) != NONE && !zero)
      lds[at >> 16] = a.s[bx * X + hx + (long long)nx * (by * Y + hy + (long long)ny * (z0 + k))];
  }
  __syncthreads();

  const bool bound = !a.r0 && !p.adj;        // the state itself is swept: check its bounds
  double acc[NV] = {0, 0, 0, 0};
  T *rd = lds, *wr = NB == 2 ? lds + copy : lds;
  vec e0;                                    // diagonals of the next group
  if constexpr (LEAN) e0 = ge[tid];
  // one sweep of the lane's column; the last one also sums its residuals
  auto sweep = [&](auto lastc, int t) {
    constexpr bool LAST = decltype(lastc)::value;
    if constexpr (LEAN) {
      if (KIND == RK_HELD) keep_in_loop(upd);
#pragma unroll
      for (int k = 0; k <= C; ++k) keep_in_loop(q.tz[k]);
    }
    if constexpr (!LEAN) {
#pragma unroll
      for (int m = 0; m < NJ; ++m) keep_in_loop(places[m]);
    }
    T dn = zlo, g = T(0);
    if constexpr (LEAN) g = open_of(q.tz[0]);
#pragma unroll
    for (int k0 = 0; k0 < C; k0 += NV16) {
      const vec xm = *reinterpret_cast<const vec *>(rd + col - S + k0);
      const vec xp = *reinterpret_cast<const vec *>(rd + col + S + k0);
      const vec ym = *reinterpret_cast<const vec *>(rd + col - stride + k0);
      const vec yp = *reinterpret_cast<const vec *>(rd + col + stride + k0);
      vec ve, vsrc;
      if constexpr (LEAN) {
        // a group ahead (the first one during the exchange): a group of two waves takes about
        // the latency of this load
        constexpr int NG = C / NV16;
        const int gi = k0 / NV16;
        ve = e0;
        e0 = ge[(gi + 1) % NG * RT + t];
        vsrc = lsrc[gi * RT + t];
      }
#pragma unroll
      for (int v = 0; v < NV16; ++v) {
        const int k = k0 + v;
        const T c0 = s[k], up = k == C - 1 ? zhi : s[k + 1 < C ? k + 1 : k];
        T r, azm, azp;
        if constexpr (LEAN) {
          const T gu = open_of(q.tz[k + 1]);
          azm = coef_of(q.tz[k], g);
          azp = coef_of(-q.tz[k + 1], gu);
          g = gu;
          r = fma(-c0, ve[v], vsrc[v]);
        } else {
          azm = q.azm[k];
          azp = q.azp[k];
          r = fma(-c0, q.e[k], q.src[k]);
        }
        r = fma(q.axm[k], xm[v] - c0, r);
        r = fma(q.axp[k], xp[v] - c0, r);
        r = fma(q.aym[k], ym[v] - c0, r);
        r = fma(q.ayp[k], yp[v] - c0, r);
        r = fma(azm, dn - c0, r);
        r = fma(azp, up - c0, r);
        if constexpr (LEAN && KIND == RK_HELD)   // held cells keep their value
          r = (int)(upd << (31 - k)) < 0 ? r : T(0);
        T next = fma(a.dt, r, c0);
        if constexpr (KIND == RK_NERNST) {
          if (upd >> k & 1u) {
            // the overpotential that balances the transport step, relaxed; the electrode's value
            const T ei = 2.0 * asinh(-r / (2.0 * rate[k] * sqrt(c0 * (1.0 - c0))));
            eta[k] = (1.0 - p.omega) * eta[k] + p.omega * ei;
            next = 1.0 / (1.0 + exp(eta[k] - p.V));
          }
        }
        s[k] = next;
        dn = c0;
        if constexpr (LAST && KIND == RK_NERNST) {
          const double d = pore >> k & 1u ? (next - c0) / a.dt : 0.0;
          acc[0] += d * d;
          if (!isfinite(d)) acc[1] += 1.0;
        } else if (LAST) {
          const double rr = (double)r;
          acc[0] += rr * rr;
          acc[2] += rr;
          if (!isfinite(rr) || (bound && (pore >> k & 1u) && !(s[k] >= a.lo && s[k] <= a.hi)))
            acc[1] += 1.0;
        }
      }
      // finish the group here: sunk to where the values are used next, the arithmetic would keep
      // every group's neighbour values in registers
#pragma unroll
      for (int v = 0; v < NV16; ++v) keep_in_loop(s[k0 + v]);
      if (sizeof(T) * C > 64) __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int j = 0; j < p.K - 1; ++j) {
    int t = tid;                             // addresses are cheaper made anew than kept
    keep_in_loop(t);
    sweep(std::false_type{}, t);
    const unsigned tag = p.tag0 + (unsigned)j;
    unsigned long long *const slot = p.inbox + (tag & 1) * p.slot_words;
    // the z faces leave from registers
    if (below)
      put_value<T>(slot + (b - gxy) * p.block_words + (NJ + 1) * RT * WN + t * WN, s[0], tag);
    if (above) put_value<T>(slot + (b + gxy) * p.block_words + NJ * RT * WN + t * WN, s[C - 1], tag);
    if (NB == 1) __syncthreads();            // every lane has read the old values
    if (act) {
#pragma unroll
      for (int k0 = 0; k0 < C; k0 += NV16) {
        vec v;
#pragma unroll
        for (int m = 0; m < NV16; ++m) v[m] = s[k0 + m];
        *reinterpret_cast<vec *>(wr + col + k0) = v;
      }
    }
    __syncthreads();
    // side columns to the neighbours
    unsigned at[NJ];
    int to[NJ];
#pragma unroll
    for (int m = 0; m < NJ; ++m) {
      if constexpr (LEAN) {
        at[m] = place(m, t, to[m]);
      } else {
        at[m] = places[m];
        to[m] = dst[m];
      }
    }
    T v[NJ], va, vb;
    if constexpr (LEAN) {
      // all reads, then all stores: six words in turn would wait for LDS six times
#pragma unroll
      for (int m = 0; m < NJ; ++m) v[m] = wr[(at[m] & NONE) != NONE ? at[m] & NONE : 0];
    }
#pragma unroll
    for (int m = 0; m < NJ; ++m)
      if ((at[m] & NONE) != NONE)
        put_value<T>(slot + to[m], LEAN ? v[m] : wr[at[m] & NONE], tag);
    // the neighbours' values: every load of a round in flight at once
    const unsigned long long *const mine = slot + b * p.block_words + t * WN;
    unsigned spins = 0;
    Waited waited;
    bool gone = false, ok;
    do {
      ok = true;
#pragma unroll
      for (int m = 0; m < NJ; ++m)
        ok &= get_value<T>(mine + m * RT * WN, tag, v[m]) | (at[m] >> 16 == NONE);
      ok &= get_value<T>(mine + NJ * RT * WN, tag, va) | !below;
      ok &= get_value<T>(mine + (NJ + 1) * RT * WN, tag, vb) | !above;
      if (!ok && (p.limit == 0 || (++spins & 255u) == 0)) {
        gone = waited.over((float)p.limit) ||
               __hip_atomic_load(p.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
      }
    } while (!ok && !gone);
    if (gone) {
      dead = 1;
      __hip_atomic_store(p.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
#pragma unroll
    for (int m = 0; m < NJ; ++m)
      if (at[m] >> 16 != NONE) wr[at[m] >> 16] = v[m];
    if (below) zlo = va;
    if (above) zhi = vb;
    __syncthreads();
    if (dead) return;
    T *const old = rd;
    rd = wr;
    wr = old;
  }
  int t = tid;
  keep_in_loop(t);
  sweep(std::true_type{}, t);
  if (act) {
    const int wy = t / X, wx = t - wy * X;
    const long long o = bx * X + wx + (long long)nx * (by * Y + wy + (long long)ny * z0);
#pragma unroll
    for (int k = 0; k < C; ++k)
      if (k < ze) {
        a.s_new[o + pl * k] = s[k];
        if constexpr (KIND == RK_NERNST)
          if (upd >> k & 1u) p.eta_new[o + pl * k] = eta[k];
      }
  }
  block_store<NV>(acc, 0u, a.partial + (long long)NV * b);
}

// Two waves per SIMD: 256 registers a lane.
#define RESIDENT_KERNEL \
  __global__ void __launch_bounds__(RT) __attribute__((amdgpu_waves_per_eu(2, 2)))

template <typename T, int C, int KIND>
RESIDENT_KERNEL k_resident(SweepArgs<T> a, ResidentArgs p) {
  resident_block<T, C, KIND>(a, p, xcd_tile(blockIdx.x, gridDim.x));
}

// Workgroups of several problems in one launch: workgroup g works for problem of[g] of the table.
// Each problem's columns have their own length.
template <typename T>
RESIDENT_KERNEL k_resident_batch(const ResidentProb<T> *__restrict__ tab,
                                 const int *__restrict__ of, unsigned tag0, int K) {
  const int g = xcd_tile(blockIdx.x, gridDim.x);
  const ResidentProb<T> &e = tab[of[g]];
  const SweepArgs<T> a = e.a;
  ResidentArgs p = e.p;
  p.tag0 = tag0;
  if (K) p.K = K;
  const int b = g - e.blk0;
  if constexpr (sizeof(T) == 4) {
    switch (e.C) {
      case 4: resident_block<T, 4, RK_PLAIN>(a, p, b); break;
      case 8: resident_block<T, 8, RK_PLAIN>(a, p, b); break;
      case 12: resident_block<T, 12, RK_PLAIN>(a, p, b); break;
      case 16: resident_block<T, 16, RK_PLAIN>(a, p, b); break;
      case 20: resident_block<T, 20, RK_PLAIN>(a, p, b); break;
      case 24: resident_block<T, 24, RK_HELD>(a, p, b); break;
      default: resident_block<T, 32, RK_HELD>(a, p, b); break;
    }
  } else {
    switch (e.C) {
      case 2: resident_block<T, 2, RK_PLAIN>(a, p, b); break;
      case 4: resident_block<T, 4, RK_PLAIN>(a, p, b); break;
      case 8: resident_block<T, 8, RK_PLAIN>(a, p, b); break;
      case 10: resident_block<T, 10, RK_PLAIN>(a, p, b); break;
      case 12: resident_block<T, 12, RK_HELD>(a, p, b); break;
      default: resident_block<T, 16, RK_HELD>(a, p, b); break;
    }
  }
}

}  // namespace

// Values between two columns of the LDS copy (col_stride), bytes of LDS, on the host.
static int lds_bytes(int bytes, int C, int X, int Y) {
  const int n = 16 / bytes, S = (C / n) % 2 ? C : C + n;
  const int copy = (X + 2) * (Y + 2) * S;
  if (!resident_lean(bytes, C)) return 2 * copy * bytes;
  const int columns = (resident_side_words(C) * RT + C - 1) / C;
  return ((copy + 3) / 4 * 4 + RT * C) * bytes + columns * (int)sizeof(uint2);
}

// Cells per lane that the kernels are built for.
constexpr int RES_C32[] = {4, 8, 12, 16, 20, 24, 32}, RES_C64[] = {2, 4, 8, 10, 12, 16};

// Every split of a box over at most ncu workgroups with its time per sweep.  The model, fitted
// to splits of 65 thousand to 4.2 million cells (within a tenth): 1 us for the exchange's latency
// and the barriers, 0.06 us per cell of a full block's columns (0.12 in FP64), 1.8 us per million
// exchanged words, and more for lean columns: 1.6 us in FP32 (256 x 128 x 128 and batches of
// C = 32 take 6 us; at 1.0 the batched solves chose them too often: twelve boxes of mixed sizes
// 136.5 ms against 132.0) and 1.0 in FP64 (at 1.6 their polish took 7.55 ms, not 7.25).
template <typename F>
static void resident_splits(const Grid &g, int bytes, int ncu, F &&take) {
  const int *const Cs = bytes == 4 ? RES_C32 : RES_C64;
  const int nC = bytes == 4 ? (int)std::size(RES_C32) : (int)std::size(RES_C64);
  for (int ic = 0; ic < nC; ++ic) {
    const int C = Cs[ic];
    const int gz = (g.nz + C - 1) / C;
    if (gz > ncu) continue;
    for (int gx = 1; gx * gz <= ncu && gx <= g.nx; ++gx) {
      const int X = (g.nx + gx - 1) / gx;
      if (X > RT || (g.nx + X - 1) / X != gx) continue;
      for (int gy = 1; gx * gy * gz <= ncu && gy <= g.ny; ++gy) {
        const int Y = (g.ny + gy - 1) / gy;
        if (X * Y > RT || (g.ny + Y - 1) / Y != gy) continue;
        const int lds = lds_bytes(bytes, C, X, Y), nj = resident_side_words(C);
        if (lds > RESIDENT_LDS || 2 * (X + Y) * C > nj * RT) continue;
        const int waves = (X * Y + 63) / 64;
        const double words = (2.0 * (X + Y) * C + 2.0 * X * Y) * gx * gy * gz * (bytes / 4);
        ResidentPlan p{C, X, Y, gx, gy, gz, lds, (nj + 2ll) * RT * (bytes / 4), 0, 0.0,
                       1.8e-6 * words};
        p.slot_words = p.block_words * gx * gy * gz;
        p.us = 1.0 + 0.0075 * bytes * C * ((waves + 3) / 4) + p.words_us +
               (resident_lean(bytes, C) ? (bytes == 4 ? 1.6 : 1.0) : 0.0);
        take(p);
      }
    }
  }
}

ResidentPlan resident_plan(const Grid &g, int bytes, int ncu) {
  ResidentPlan best{};
  resident_splits(g, bytes, ncu, [&](const ResidentPlan &p) {
    if (!best.C || p.us < best.us) best = p;
  });
  return best;
}

// The Nernst iteration: at most RES_NERNST cells a column (two more numbers each, and the
// functions' temporaries); an electrode cell costs some ten plain ones, and a column's step is
// as slow as its wave's slowest, so a cell counts six times the plain sweep's here.
constexpr int RES_NERNST = 8;
ResidentPlan resident_plan_nernst(const Grid &g, int ncu) {
  ResidentPlan best{};
  resident_splits(g, 8, ncu, [&](ResidentPlan p) {
    if (p.C > RES_NERNST) return;
    p.us += 5 * 0.06 * p.C * (((p.X * p.Y + 63) / 64 + 3) / 4);
    if (!best.C || p.us < best.us) best = p;
  });
  return best;
}

std::vector<ResidentPlan> resident_plans(const Grid &g, int bytes, int ncu) {
  std::vector<ResidentPlan> all, front;
  resident_splits(g, bytes, ncu, [&](const ResidentPlan &p) { all.push_back(p); });
  std::sort(all.begin(), all.end(), [](const ResidentPlan &p, const ResidentPlan &q) {
    return p.blocks() != q.blocks() ? p.blocks() < q.blocks() : p.us < q.us;
  });
  for (const ResidentPlan &p : all)
    if (front.empty() || p.us < 0.97 * front.back().us) front.push_back(p);
  return front;
}

long long resident_diag_bytes(const ResidentPlan &pl, int bytes) {
  return resident_lean(bytes, pl.C) ? (long long)pl.gx * pl.gy * pl.gz * RT * pl.C * bytes : 0;
}

template <typename T, int C>
static void go_resident(const SweepArgs<T> &a, const ResidentPlan &pl, const ResidentArgs &p,
                        hipStream_t st) {
  // LDS beyond half of a CU's keeps every workgroup on a CU of its own
  const int bytes = pl.lds > RESIDENT_LDS_ALONE ? pl.lds : RESIDENT_LDS_ALONE;
  const int nb = pl.gx * pl.gy * pl.gz;
  if constexpr (resident_lean(sizeof(T), C)) {
    if (a.pinned) {
      k_resident<T, C, RK_HELD><<<nb, RT, bytes, st>>>(a, p);
      return;
    }
  }
  k_resident<T, C, RK_PLAIN><<<nb, RT, bytes, st>>>(a, p);
}

void launch_resident_nernst(const SweepArgs<double> &a, const ResidentPlan &pl,
                            const ResidentArgs &args, hipStream_t st) {
  ResidentArgs p = args;
  p.X = pl.X; p.Y = pl.Y; p.gx = pl.gx; p.gy = pl.gy; p.gz = pl.gz;
  p.block_words = pl.block_words;
  p.slot_words = pl.slot_words;
  const int bytes = pl.lds > RESIDENT_LDS_ALONE ? pl.lds : RESIDENT_LDS_ALONE, nb = pl.blocks();
  switch (pl.C) {
    case 2: k_resident<double, 2, RK_NERNST><<<nb, RT, bytes, st>>>(a, p); break;
    case 4: k_resident<double, 4, RK_NERNST><<<nb, RT, bytes, st>>>(a, p); break;
    default: k_resident<double, 8, RK_NERNST><<<nb, RT, bytes, st>>>(a, p); break;
  }
}

template <typename T>
void launch_resident(const SweepArgs<T> &a, const ResidentPlan &pl, const ResidentArgs &args,
                     hipStream_t st) {
  ResidentArgs p = args;
  p.X = pl.X; p.Y = pl.Y; p.gx = pl.gx; p.gy = pl.gy; p.gz = pl.gz;
  p.block_words = pl.block_words;
  p.slot_words = pl.slot_words;
  if constexpr (sizeof(T) == 4) {
    switch (pl.C) {
      case 4: go_resident<T, 4>(a, pl, p, st); break;
      case 8: go_resident<T, 8>(a, pl, p, st); break;
      case 12: go_resident<T, 12>(a, pl, p, st); break;
      case 16: go_resident<T, 16>(a, pl, p, st); break;
      case 20: go_resident<T, 20>(a, pl, p, st); break;
      case 24: go_resident<T, 24>(a, pl, p, st); break;
      default: go_resident<T, 32>(a, pl, p, st); break;
    }
  } else {
    switch (pl.C) {
      case 2: go_resident<T, 2>(a, pl, p, st); break;
      case 4: go_resident<T, 4>(a, pl, p, st); break;
      case 8: go_resident<T, 8>(a, pl, p, st); break;
      case 10: go_resident<T, 10>(a, pl, p, st); break;
      case 12: go_resident<T, 12>(a, pl, p, st); break;
      default: go_resident<T, 16>(a, pl, p, st); break;
    }
  }
}
template <typename T>
void launch_resident_batch(const ResidentProb<T> *tab, const int *of, int nblocks, int lds,
                           unsigned tag0, int K, hipStream_t st) {
  const int bytes = lds > RESIDENT_LDS_ALONE ? lds : RESIDENT_LDS_ALONE;
  k_resident_batch<T><<<nblocks, RT, bytes, st>>>(tab, of, tag0, K);
}
template void launch_resident_batch<float>(const ResidentProb<float> *, const int *, int, int,
                                           unsigned, int, hipStream_t);
template void launch_resident_batch<double>(const ResidentProb<double> *, const int *, int, int,
                                            unsigned, int, hipStream_t);

template void launch_resident<float>(const SweepArgs<float> &, const ResidentPlan &,
                                     const ResidentArgs &, hipStream_t);
template void launch_resident<double>(const SweepArgs<double> &, const ResidentPlan &,
                                      const ResidentArgs &, hipStream_t);

}  // namespace socfv
