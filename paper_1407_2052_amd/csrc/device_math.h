// Device arithmetic shared by the forward stage kernel and the adjoint:
// state addressing, primitive recovery, physical flux, fast and whistler
// speeds, MP5 and LIM03, tile geometry and the XCD-aware tile schedule.
// Sharing one definition makes the adjoint's recompute of the forward pass
// bitwise identical to the forward pass (no automatic FMA contraction; every
// fused multiply-add is explicit).
#pragma once
#include "amrvac_internal.h"

#include <type_traits>
#include <utility>

namespace amrvac {

// Variables: hydro (rho, m_1..m_NDIM, E); MHD (rho, m_x, m_y, m_z, E, B_x,
// B_y, B_z); GLM as MHD, then psi.
template <int NDIM, bool MHD, bool GLM = false>
struct Eq {
  static_assert(MHD || !GLM, "GLM extends MHD");
  static constexpr int NV = GLM ? 9 : MHD ? 8 : 2 + NDIM;
  static constexpr int NC = MHD ? 3 : NDIM;
  static constexpr int IE = 1 + NC;
};

template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// ---------------------------------------------------------------------------
// Addressing of state buffers.
// ---------------------------------------------------------------------------
// A wave-uniform int the compiler must treat as unknown at this point: the
// stage update's buffer addresses derived from it are then rebuilt per tile
// (a few scalar operations) instead of being hoisted out of the tile loop and
// held, or spilled, across it.  The empty asm emits no instruction.
__device__ __forceinline__ int opaque_uniform(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

// The same value, hidden from common-subexpression elimination (no
// instruction): a recomputation from it is not merged with an earlier one,
// so the earlier results need not stay live in registers until then.
__device__ __forceinline__ double opaque_value(double x) {
  asm volatile("" : "+v"(x));
  return x;
}

// Pointers into global memory (address space 1).  Block states and scratch
// slots are reached through pointers read from the block table, which the
// compiler would otherwise treat as generic: generic accesses compile to
// flat instructions, whose completion the LDS counter waits for as well, so
// every LDS wait would also wait for the global loads in flight.
using gptr = __attribute__((address_space(1))) const double*;
using gptr_w = __attribute__((address_space(1))) double*;

__device__ __forceinline__ gptr cell_addr(const StateTable& st, const BlockDev& B, int buf, int i, int j, int k,
                                          long long& vstride) {
  if (buf == 0) {
    vstride = (long long)B.P[0] * B.P[1] * B.P[2];
    return (gptr)(B.u + (((long long)(k + B.g[2]) * B.P[1] + (j + B.g[1])) * B.P[0] + (i + B.g[0])));
  }
  vstride = B.cells;
  return (gptr)(st.scr + (long long)(buf - 1) * st.slot_stride + B.off + (((long long)k * B.n[1] + j) * B.n[0] + i));
}

__device__ __forceinline__ gptr_w cell_addr_w(const StateTable& st, const BlockDev& B, int buf, int i, int j, int k,
                                              long long& vstride) {
  return (gptr_w)cell_addr(st, B, buf, i, j, k, vstride);
}

template <class T>
using cptr = const __attribute__((address_space(4))) T*;

// The block table and tile list do not change during a launch: uniform
// accesses to them are scalar loads.
template <class T>
__device__ __forceinline__ cptr<T> constant_ptr(const T* p) {
  return (cptr<T>)(unsigned long long)p;
}

// A lane's number, to be treated as new here: what is derived from it is
// recomputed at its use (a few 32-bit operations) instead of being hoisted out
// of the tile loop and held, or spilled, across it.
__device__ __forceinline__ int fresh(int i) {
  asm volatile("" : "+v"(i));
  return i;
}

// A uniform value, kept in scalar registers from here on.
template <class T>
__device__ __forceinline__ T held(T x) {
  asm volatile("" : "+s"(x));
  return x;
}

// Load all NV variables of cell (i,j,k) of block blk, where only coordinate
// D may lie outside [0, n_D): then the value comes from the face neighbour's
// interior (same buffer), or from this block's fixed ghost layer (buffer 0).
template <int NV, int D>
__device__ __forceinline__ void load_cell(const StateTable& st, int blk, int buf, int i, int j, int k,
                                          double* u) {
  const BlockDev* B = &st.blocks[blk];
  int c[3] = {i, j, k};
  int bf = buf;
  if (c[D] < 0) {
    int nb = B->nbr[2 * D];
    if (nb >= 0) {
      B = &st.blocks[nb];
      c[D] += B->n[D];
    } else {
      bf = 0;
    }
  } else if (c[D] >= B->n[D]) {
    int nb = B->nbr[2 * D + 1];
    if (nb >= 0) {
      c[D] -= B->n[D];
      B = &st.blocks[nb];
    } else {
      bf = 0;
    }
  }
  long long vs;
  gptr p = cell_addr(st, *B, bf, c[0], c[1], c[2], vs);
#pragma unroll
  for (int v = 0; v < NV; ++v) u[v] = p[v * vs];
}

// Where the cells along direction D of one block lie: below it, in it, above
// it (the face neighbour's interior, or the block's own fixed ghost layers in
// buffer 0), each with coordinates counted from this block's first cell.  All
// uniform, so that a lane's loads need selections but no lookups of their own
// and can all be in flight together.
template <int D>
struct SideRows {
  gptr p[3];
  int n0[3], n1[3];   // cells per row, rows per plane
  long long vs[3];
  int n;              // cells of this block along D

  __device__ __forceinline__ SideRows(const StateTable& st, int blk, int buf) {
    const cptr<BlockDev> blocks = constant_ptr(st.blocks);
    const cptr<BlockDev> B = blocks + blk;
    n = B->n[D];
#pragma unroll
    for (int side = 0; side < 3; ++side) {
      const int nb = side == 1 ? blk : B->nbr[2 * D + side / 2];
      const bool fixed = nb < 0;
      const cptr<BlockDev> N = fixed ? B : blocks + nb;
      const int shift = side == 1 || fixed ? 0 : side == 0 ? N->n[D] : -n;
      if (buf == 0 || fixed) {
        n0[side] = N->P[0];
        n1[side] = N->P[1];
        vs[side] = (long long)N->P[0] * N->P[1] * N->P[2];
        p[side] = (gptr)N->u + (((long long)N->g[2] * N->P[1] + N->g[1]) * N->P[0] + N->g[0]);
      } else {
        n0[side] = N->n[0];
        n1[side] = N->n[1];
        vs[side] = N->cells;
        p[side] = (gptr)st.scr + ((long long)(buf - 1) * st.slot_stride + N->off);
      }
      p[side] += shift * (D == 0 ? 1ll : D == 1 ? (long long)n0[side] : (long long)n0[side] * n1[side]);
    }
  }

  // Variables V0 .. V0+VN-1 of cell (i,j,k), whose coordinate D may lie outside.
  template <int V0, int VN>
  __device__ __forceinline__ void load(int i, int j, int k, double* u) const {
    const int c = D == 0 ? i : D == 1 ? j : k;
    const bool lo = c < 0, hi = c >= n;
    // selections of values, not of elements (which would put the arrays in scratch)
    const auto pick = [&](auto below, auto inside, auto above) { return lo ? below : hi ? above : inside; };
    const gptr q = pick(p[0], p[1], p[2]);
    const int q0 = pick(n0[0], n0[1], n0[2]), q1 = pick(n1[0], n1[1], n1[2]);
    const long long w = pick(vs[0], vs[1], vs[2]);
    const gptr a = q + (((long long)k * q1 + j) * q0 + i);
#pragma unroll
    for (int v = 0; v < VN; ++v) u[v] = a[(V0 + v) * w];
  }
};

// The rows of every direction, so that the table loads of one direction do not
// wait for the cells of another.
template <int NDIM>
struct AllRows {
  SideRows<0> x;
  SideRows<NDIM >= 2 ? 1 : 0> y;
  SideRows<NDIM >= 3 ? 2 : 0> z;
  __device__ __forceinline__ AllRows(const StateTable& st, int blk, int buf)
      : x(st, blk, buf), y(st, blk, buf), z(st, blk, buf) {}
  template <int D>
  __device__ __forceinline__ const auto& along() const {
    if constexpr (D == 0) return x;
    else if constexpr (D == 1) return y;
    else return z;
  }
};

// The current of cell (i,j,k) of block blk (planes of stride `plane`, interior
// layout, block at coff), where only coordinate D may lie outside the block:
// then the face neighbour's cell (its face must exist).
template <int D>
__device__ __forceinline__ void load_current(const StateTable& st, const double* J, long long plane, int blk, int i,
                                             int j, int k, double* Jc) {
  const BlockDev* B = &st.blocks[blk];
  int c[3] = {i, j, k};
  if (c[D] < 0) {
    B = &st.blocks[B->nbr[2 * D]];
    c[D] += B->n[D];
  } else if (c[D] >= B->n[D]) {
    c[D] -= B->n[D];
    B = &st.blocks[B->nbr[2 * D + 1]];
  }
  gptr p = (gptr)J + (B->coff + ((long long)c[2] * B->n[1] + c[1]) * B->n[0] + c[0]);
#pragma unroll
  for (int v = 0; v < 3; ++v) Jc[v] = p[v * plane];
}

// ---------------------------------------------------------------------------
// Physics: primitive recovery, flux along D, fast speed.
// ---------------------------------------------------------------------------
struct PrimD {
  double rho, ri, v[3], p, B[3], b2;
};

template <int NDIM, bool MHD>
__device__ __forceinline__ bool prim(const double* u, double gamma, PrimD& w) {
  using E = Eq<NDIM, MHD>;
  w.rho = u[0];
  w.ri = 1.0 / w.rho;
  double mv = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    w.v[k] = (k < E::NC) ? u[1 + k] * w.ri : 0.0;
    w.B[k] = 0.0;
  }
#pragma unroll
  for (int k = 0; k < E::NC; ++k) mv = fma(u[1 + k], w.v[k], mv);
  double eint = fma(-0.5, mv, u[E::IE]);
  w.b2 = 0.0;
  if constexpr (MHD) {
#pragma unroll
    for (int k = 0; k < 3; ++k) w.B[k] = u[5 + k];
    w.b2 = fma(w.B[2], w.B[2], fma(w.B[1], w.B[1], w.B[0] * w.B[0]));
    eint = fma(-0.5, w.b2, eint);
  }
  w.p = (gamma - 1.0) * eint;
  return (w.rho > 0.0) && (w.p > 0.0) && (w.p < __builtin_huge_val()) &&
         (w.rho < __builtin_huge_val());
}

// The primitives of a state whose 1/rho and p were already recovered by prim
// (the same operations on the same inputs: the same bits, without the
// division).
template <int NDIM, bool MHD>
__device__ __forceinline__ void prim_from(const double* u, double ri, double p, PrimD& w) {
  using E = Eq<NDIM, MHD>;
  w.rho = u[0];
  w.ri = ri;
  w.p = p;
  w.b2 = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    w.v[k] = (k < E::NC) ? u[1 + k] * ri : 0.0;
    w.B[k] = 0.0;
  }
  if constexpr (MHD) {
#pragma unroll
    for (int k = 0; k < 3; ++k) w.B[k] = u[5 + k];
    w.b2 = fma(w.B[2], w.B[2], fma(w.B[1], w.B[1], w.B[0] * w.B[0]));
  }
}

// Physical flux along D (Sect. 3 eqs. masscons, momentum, total; Sect. 4.1
// eq. b1eq and Sect. 4.3 eqs. momentummhd, fractional with B0 = 0).
template <int NDIM, bool MHD, int D>
__device__ __forceinline__ void phys_flux(const double* u, const PrimD& w, double* F) {
  using E = Eq<NDIM, MHD>;
  const double vd = w.v[D];
  F[0] = u[1 + D];
  if constexpr (!MHD) {
#pragma unroll
    for (int k = 0; k < E::NC; ++k) F[1 + k] = u[1 + k] * vd;
    F[1 + D] += w.p;
    F[E::IE] = vd * (u[E::IE] + w.p);
  } else {
    const double ptot = fma(0.5, w.b2, w.p);
    const double Bd = w.B[D];
    const double bv = fma(w.B[2], w.v[2], fma(w.B[1], w.v[1], w.B[0] * w.v[0]));
#pragma unroll
    for (int k = 0; k < 3; ++k) F[1 + k] = fma(u[1 + k], vd, -(Bd * w.B[k]));
    F[1 + D] += ptot;
    F[4] = fma(vd, u[4] + ptot, -(Bd * bv));
#pragma unroll
    for (int k = 0; k < 3; ++k) F[5 + k] = (k == D) ? 0.0 : fma(vd, w.B[k], -(Bd * w.v[k]));
  }
}

// Hall MHD: the fast whistler speed eta_h |B| k_max / rho at k_max = pi
// max_d 1/dx_d of the block (Sect. 4.4).
__device__ __forceinline__ double whistler_speed(const PrimD& w, double eta_h, double kmax) {
  const double babs = sqrt(w.B[0] * w.B[0] + w.B[1] * w.B[1] + w.B[2] * w.B[2]);
  return eta_h * babs / w.rho * kmax;
}

// Fast magnetosonic speed along d (sound speed for hydro).
template <bool MHD>
__device__ __forceinline__ double fast_speed(const PrimD& w, int d, double gamma) {
  const double a2 = gamma * w.p * w.ri;
  if constexpr (!MHD) {
    return sqrt(a2);
  } else {
    const double b2 = w.b2 * w.ri;
    const double bd2 = w.B[d] * w.B[d] * w.ri;
    const double s = a2 + b2;
    double disc = fma(s, s, -4.0 * a2 * bd2);
    disc = disc < 0.0 ? 0.0 : disc;
    return sqrt(0.5 * (s + sqrt(disc)));
  }
}

// Whether |v_d| + fast_speed(w, d) may exceed r: false only where the value
// the expression rounds to is at most r.  With M = r - |v_d| the speed is
// below M when s + sqrt(disc) < 2 M^2 (fast_speed's s and disc), that is when
// 2 M^2 - s > 0 and disc < (2 M^2 - s)^2.  M is lowered by 1e-14 and must be
// at least r/8, which outweighs the few roundings of either side; NaN gives
// true.
template <bool MHD>
__device__ __forceinline__ bool speed_may_exceed(const PrimD& w, int d, double gamma, double r) {
  const double M = (r - fabs(w.v[d])) * (1.0 - 1e-14);
  const double a2 = gamma * w.p * w.ri;
  if constexpr (!MHD) {
    return !(M > 0.125 * r && a2 < M * M);
  } else {
    const double b2 = w.b2 * w.ri;
    const double bd2 = w.B[d] * w.B[d] * w.ri;
    const double s = a2 + b2;
    const double disc = fma(s, s, -4.0 * a2 * bd2);
    const double q = fma(2.0 * M, M, -s);
    return !(M > 0.125 * r && q > 0.0 && disc < q * q);
  }
}

// ---------------------------------------------------------------------------
// MP5 (Suresh & Huynh 1997), alpha = 4, eps = 0, median form, in differences.
// ---------------------------------------------------------------------------
// Every quantity is taken relative to the stencil centre c = f_j, from the
// cell differences D_j = f_{j+1} - f_j:
//   g   = fL - c  = (-2 D_{j-2} + 11 D_{j-1} + 24 D_j - 3 D_{j+1}) / 60,
//   fMD - c = D_j / 2 - m4_{j+1/2} / 2,    fUL - c = 4 D_{j-1},
//   fLC - c = D_{j-1} / 2 + 4/3 m4_{j-1/2},
//   value   = c + median(g, fmin - c, fmax - c).
// A difference is formed once and serves as D_j of one interface and D_{j-1}
// of the next, and so do min(D, 0), max(D, 0) and D / 2; the bounds need no
// comparison with c, which is 0 here.  Per interface of a long run this is
// 30 FP64 instructions against 37 for the same formulas on f itself (and the
// comparisons take computed values, for which the compiler adds no
// canonicalising v_max), and g, a sum of differences, is the more exact.
//
// d^M4_{j+1/2} = minmod(4x - y, 4y - x, x, y) of the curvatures x = d_j and
// y = d_{j+1}, from the smaller and the larger of the two: with lo <= hi,
// 4 hi - lo cannot be the smallest of four positive values nor 4 lo - hi the
// largest of four negative ones, so the minmod is the median of 0,
// min(lo, 4 lo - hi) and max(hi, 4 hi - lo).  It is exactly one of its
// arguments, or zero, and symmetric, so neighbouring interfaces of a pencil
// share one evaluation.
__device__ __forceinline__ double m4pair(double x, double y) {
  const double lo = fmin(x, y), hi = fmax(x, y);
  const double a = fmin(lo, fma(4.0, lo, -hi));
  const double b = fmax(hi, fma(4.0, hi, -lo));
  return fmax(a, fmin(b, 0.0));
}

// Bounds of one interface relative to c; the chain (0, D_j, fMD - c) and the
// chain (0, fUL - c, fLC - c) each give a bound below and one above zero.
struct Mp5Bounds {
  double fMD, fLC;   // relative to c
  double amn, amx;   // the first chain's bounds
  double fmn, fmx;
};
__device__ __forceinline__ double mp5_clamp(double g, double dn, double dp, double hj, double dn1, double dp1,
                                            double hj1, double m4p, double m4m, Mp5Bounds& q) {
  q.fMD = fma(-0.5, m4p, hj);
  q.fLC = fma(4.0 / 3.0, m4m, hj1);
  q.amn = fmin(dn, q.fMD);
  q.amx = fmax(dp, q.fMD);
  q.fmn = fmax(q.amn, fmin(4.0 * dn1, q.fLC));
  q.fmx = fmin(q.amx, fmax(4.0 * dp1, q.fLC));
  return fmin(fmax(g, q.fmn), q.fmx);
}

// g of the interface whose stencil differences are D[0..3] = D_{j-2} .. D_{j+1}.
__device__ __forceinline__ double mp5_fifth(const double* D) {
  return fma(0.4, D[2], fma(11.0 / 60.0, D[1], fma(-1.0 / 30.0, D[0], -0.05 * D[3])));
}

// Linear pieces of MP5.  With eps = 0, mp5 is continuous and piecewise
// linear in its five inputs; mp5_piece names the piece it evaluates (the
// adjoint multiplies by that piece's constant weights):
//   0 fL;  1 c;  2 d;  3 fUL;  4 + k fMD and 9 + k fLC, where k (0..4) is
//   the argument the curvature minmod returned, k = 0 for zero, with the
//   arguments ordered (4d_j - d_{j+1}, 4d_{j+1} - d_j, d_j, d_{j+1}) for fMD
//   at j+1/2 and (4d_j - d_{j-1}, 4d_{j-1} - d_j, d_j, d_{j-1}) for fLC at
//   j-1/2.  The piece is fL when fmin <= fL <= fmax; else the candidate that
//   realised the bound r the value was clamped to (fmin when fL < fmin, fmax
//   when fL > fmax).  The bound is the max (min) of two chains, (c, d, fMD)
//   and (c, fUL, fLC), and the first chain wins ties, so r comes from the
//   second chain exactly when it differs from the first chain's value; in
//   that chain the piece is the first candidate equal to r, which is the
//   earlier-wins tie rule of the min/max chains.  All of it relative to c.
__device__ __forceinline__ int mp5_piece(double g, double Dj, double Dj1, const Mp5Bounds& q, int kp, int km) {
  const bool lo = g < q.fmn, hi = g > q.fmx;
  const double r = lo ? q.fmn : q.fmx;
  const bool second = r != (lo ? q.amn : q.amx);
  const int k = r == 0.0 ? 1 : second ? (4.0 * Dj1 == r ? 3 : 9 + km) : (Dj == r ? 2 : 4 + kp);
  return (lo || hi) ? k : 0;
}

// MP5 (Suresh & Huynh 1997, alpha = 4, eps = 0, median form) of RUN
// consecutive interfaces of a pencil: interface kk reconstructs from the
// stencil f[kk .. kk+4] (f_{j-2} .. f_{j+2}).  Differences, curvatures and
// curvature limiters are evaluated once and shared by the interfaces that
// use them; every value is bitwise that of RUN separate evaluations.  With
// CODES the linear piece of every interface is returned as well.
template <int RUN, bool CODES>
__device__ __forceinline__ void mp5_run(const double* f, double* out, int* code) {
  // curvature limiters of the pairs of stencil positions (j + 1, j + 2)
  auto limiters = [](const double* D, double* m4) {
    double dc[RUN + 2];   // curvature at stencil position j + 1
#pragma unroll
    for (int j = 0; j < RUN + 2; ++j) dc[j] = D[j + 1] - D[j];
#pragma unroll
    for (int j = 0; j < RUN + 1; ++j) m4[j] = m4pair(dc[j], dc[j + 1]);
  };
  bool clamped = false;
  {
    double D[RUN + 3];
#pragma unroll
    for (int j = 0; j < RUN + 3; ++j) D[j] = f[j + 1] - f[j];
    double m4[RUN + 1];
    limiters(D, m4);
#pragma unroll
    for (int kk = 0; kk < RUN; ++kk) {
      const double g = mp5_fifth(D + kk);
      Mp5Bounds q;
      const double r = mp5_clamp(g, fmin(D[kk + 2], 0.0), fmax(D[kk + 2], 0.0), 0.5 * D[kk + 2], fmin(D[kk + 1], 0.0),
                                 fmax(D[kk + 1], 0.0), 0.5 * D[kk + 1], m4[kk + 1], m4[kk], q);
      out[kk] = f[kk + 2] + r;
      if constexpr (CODES) clamped = clamped || r != g;   // fL < fmin or fL > fmax
    }
  }
  if constexpr (CODES) {
    // every piece is fL (code 0) unless the value was clamped; a wave in
    // which no lane clamped any interface of its run skips the search
    if (__ballot(clamped) == 0) {
#pragma unroll
      for (int kk = 0; kk < RUN; ++kk) code[kk] = 0;
      return;
    }
    // Recomputed from the stencil values (passed through opaque_value, so
    // that nothing of the first pass stays live for this rare path): the
    // same operations on the same inputs give the same differences, limiters
    // and bounds.
    double D[RUN + 3];
    {
      double e[RUN + 4];
#pragma unroll
      for (int j = 0; j < RUN + 4; ++j) e[j] = opaque_value(f[j]);
#pragma unroll
      for (int j = 0; j < RUN + 3; ++j) D[j] = e[j + 1] - e[j];
    }
    // the argument each pair limiter returned, in the two orders its
    // interfaces number them: (4x - y, 4y - x, x, y) where it is the limiter
    // at j+1/2 (fMD of interface kk = pair - 1), and (4y - x, 4x - y, y, x)
    // where it is the limiter at j-1/2 (fLC of interface kk = pair)
    double gm[RUN + 1];
    int kpp[RUN + 1], kmp[RUN + 1];
    limiters(D, gm);
#pragma unroll
    for (int j = 0; j < RUN + 1; ++j) {
      const double x = D[j + 1] - D[j], y = D[j + 2] - D[j + 1], m = gm[j];
      const bool z = m == 0.0, e1 = fma(4.0, x, -y) == m, e2 = fma(4.0, y, -x) == m, e3 = x == m, e4 = y == m;
      kpp[j] = z ? 0 : e1 ? 1 : e2 ? 2 : e3 ? 3 : 4;
      kmp[j] = z ? 0 : e2 ? 1 : e1 ? 2 : e4 ? 3 : 4;
    }
#pragma unroll
    for (int kk = 0; kk < RUN; ++kk) {
      const double g = mp5_fifth(D + kk);
      Mp5Bounds q;
      (void)mp5_clamp(g, fmin(D[kk + 2], 0.0), fmax(D[kk + 2], 0.0), 0.5 * D[kk + 2], fmin(D[kk + 1], 0.0),
                      fmax(D[kk + 1], 0.0), 0.5 * D[kk + 1], gm[kk + 1], gm[kk], q);
      code[kk] = mp5_piece(g, D[kk + 2], D[kk + 1], q, kpp[kk + 1], kmp[kk]);
    }
  }
}

// The values of mp5_run<RUN, false>, one interface after the other with only
// what the next one needs held: for kernels whose registers are few.  The
// barriers keep the scheduler from opening several interfaces at once.
// Returns a bit per interface: its value was clamped (its piece is not fL).
template <int RUN>
__device__ __forceinline__ unsigned mp5_stream(const double* f, double* out) {
  unsigned clamped = 0;
  double D[4];   // differences of the interface's stencil
  D[0] = f[1] - f[0];
  D[1] = f[2] - f[1];
  D[2] = f[3] - f[2];
  double dc = D[2] - D[1];                  // curvature at the stencil centre
  double m4m = m4pair(D[1] - D[0], dc);     // limiter below it
  double dn1 = fmin(D[1], 0.0), dp1 = fmax(D[1], 0.0), h1 = 0.5 * D[1];
#pragma unroll
  for (int kk = 0; kk < RUN; ++kk) {
    D[3] = f[kk + 4] - f[kk + 3];
    const double dcp = D[3] - D[2];
    const double m4p = m4pair(dc, dcp);
    const double dn = fmin(D[2], 0.0), dp = fmax(D[2], 0.0), h = 0.5 * D[2];
    Mp5Bounds q;
    const double g = mp5_fifth(D);
    const double r = mp5_clamp(g, dn, dp, h, dn1, dp1, h1, m4p, m4m, q);
    out[kk] = f[kk + 2] + r;
    clamped |= (r != g ? 1u : 0u) << kk;
    D[0] = D[1];
    D[1] = D[2];
    D[2] = D[3];
    dc = dcp;
    m4m = m4p;
    dn1 = dn;
    dp1 = dp;
    h1 = h;
    __builtin_amdgcn_sched_barrier(0);
  }
  return clamped;
}

// The piece of one reconstruction from its stencil, as mp5_run<1, true> finds
// it.
__device__ __forceinline__ int mp5_code(double a, double b, double c, double d, double e) {
  const double D[4] = {b - a, c - b, d - c, e - d};
  const double dm = D[1] - D[0], d0 = D[2] - D[1], dp = D[3] - D[2];
  const double m4m = m4pair(dm, d0), m4p = m4pair(d0, dp);
  const int kp = m4p == 0.0 ? 0 : fma(4.0, d0, -dp) == m4p ? 1 : fma(4.0, dp, -d0) == m4p ? 2 : d0 == m4p ? 3 : 4;
  const int km = m4m == 0.0 ? 0 : fma(4.0, d0, -dm) == m4m ? 1 : fma(4.0, dm, -d0) == m4m ? 2 : d0 == m4m ? 3 : 4;
  const double g = mp5_fifth(D);
  Mp5Bounds q;
  (void)mp5_clamp(g, fmin(D[2], 0.0), fmax(D[2], 0.0), 0.5 * D[2], fmin(D[1], 0.0), fmax(D[1], 0.0), 0.5 * D[1], m4p,
                  m4m, q);
  return mp5_piece(g, D[2], D[1], q, kp, km);
}

__device__ __forceinline__ double mp5(double a, double b, double c, double d, double e) {
  const double f[5] = {a, b, c, d, e};
  double r;
  mp5_run<1, false>(f, &r, nullptr);
  return r;
}

// ---------------------------------------------------------------------------
// LIM03 (Cada & Torrilhon 2009): compact third-order reconstruction with the
// asymptotic-region switch.
// ---------------------------------------------------------------------------
// Interface value at j+1/2 from a = f_{j-1}, b = f_j, c = f_{j+1}; kr =
// 1 / (r dx)^2 for the cell width dx along the pencil.  With dm = b - a and
// dp = c - b the value is b + H/2, where
//   H = (2 dp + dm)/3                      if (dm^2 + dp^2) kr <= 1,
//   H = phi(dm/dp) dp                      otherwise,
//   phi(t) = max(0, min(phi3, max(-t/2, min(2t, phi3, 1.6)))), phi3 = (2+t)/3.
// The limited branch is evaluated without a division: with s = sign(dp)
// and p3 = (2 dp + dm)/3,
//   phi(dm/dp) dp = s max(0, min(s p3, max(-s dm/2, min(2 s dm, s p3, 1.6 |dp|)))),
// which is 0 for dp = 0 (the limit of both one-sided branches).
// The function is piecewise linear in (a, b, c); with CODES the piece is
// returned for the adjoint: 0 H = 0; 1 the third-order formula (either
// branch); 2 -theta/2; 3 2 theta; 4 the 1.6 cap.
template <bool CODES>
__device__ __forceinline__ double lim03_eval(double a, double b, double c, double kr, int& code) {
  const double dm = b - a, dp = c - b;
  const double p3 = fma(2.0, dp, dm) * (1.0 / 3.0);
  const double eta = fma(dm, dm, dp * dp) * kr;
  const double s = dp > 0.0 ? 1.0 : (dp < 0.0 ? -1.0 : 0.0);
  const double sp3 = s * p3, sdm = s * dm, adp = s * dp;
  const double q = -0.5 * sdm, t = 2.0 * sdm, g = 1.6 * adp;
  const double lo = fmin(sp3, fmax(q, fmin(fmin(t, sp3), g)));
  const bool asym = eta <= 1.0;
  const double h = asym ? p3 : s * fmax(0.0, lo);
  if constexpr (CODES) {
    code = asym ? 1 : (!(lo > 0.0) || s == 0.0) ? 0 : lo == sp3 ? 1 : lo == q ? 2 : lo == t ? 3 : 4;
  }
  return fma(0.5, h, b);
}

__device__ __forceinline__ double lim03(double a, double b, double c, double kr) {
  int unused;
  return lim03_eval<false>(a, b, c, kr, unused);
}

// ---------------------------------------------------------------------------
// Tile geometry helpers (compile time).
// ---------------------------------------------------------------------------
template <int TX, int TY, int TZ, int HG = NG>
struct TileShape {
  static constexpr int T(int d) { return d == 0 ? TX : d == 1 ? TY : TZ; }
  static constexpr int TC = TX * TY * TZ;
  // extended box along D (halo of HG cells on both sides: 3 for MP5, 2 for
  // LIM03)
  static constexpr int E(int D, int d) { return T(d) + (d == D ? 2 * HG : 0); }
  static constexpr int NEXT(int D) { return E(D, 0) * E(D, 1) * E(D, 2); }
  static constexpr int SD(int D) { return D == 0 ? 1 : D == 1 ? E(D, 0) : E(D, 0) * E(D, 1); }
  // interface box along D
  static constexpr int I(int D, int d) { return T(d) + (d == D ? 1 : 0); }
  static constexpr int NIFC(int D) { return I(D, 0) * I(D, 1) * I(D, 2); }
  static constexpr int SI(int D) { return D == 0 ? 1 : D == 1 ? I(D, 0) : I(D, 0) * I(D, 1); }
};

template <int A, int B>
struct cmax_i { static constexpr int v = A > B ? A : B; };

// XCD-aware persistent tile schedule.  Work-groups of a launch are
// dispatched round-robin over the 8 XCDs (work-group w on XCD w % 8), each
// XCD with its own L2.  The tile list (Morton-ordered, so contiguous ranges
// are compact in space) is cut into 8 contiguous chunks and chunk x is
// processed only by the work-groups of XCD x, so tiles whose halos overlap
// mostly share one L2.  Every tile is visited exactly once; with fewer than
// 8 work-groups the schedule is the plain grid stride.
struct TileSchedule {
  int t, end, step;
  __device__ __forceinline__ TileSchedule(int ntiles) {
    const int G = (int)gridDim.x, w = (int)blockIdx.x;
    if (G < 8) {
      t = w;
      end = ntiles;
      step = G;
    } else {
      const int x = w & 7, r = w >> 3;
      const int gx = (G - x + 7) >> 3;   // work-groups on XCD x
      t = (int)((long long)ntiles * x / 8) + r;
      end = (int)((long long)ntiles * (x + 1) / 8);
      step = gx;
    }
  }
};

// The value of another lane, for reductions over a wavefront without the LDS
// pipe and without per-lane addresses (which would be held in registers):
// steps 0..3 rotate the 16 lanes of a row by 8, 4, 2, 1, step 4 pairs the rows
// of a half, step 5 the halves.  Combining a value with its partner of every
// step gives each lane the reduction over all 64.
template <int STEP>
__device__ __forceinline__ unsigned long long partner_bits(unsigned long long x) {
  const unsigned lo = (unsigned)x, hi = (unsigned)(x >> 32);
  unsigned a, b;
  if constexpr (STEP < 4) {
    constexpr int CTRL = 0x120 + (8 >> STEP);   // row_ror
    a = (unsigned)__builtin_amdgcn_update_dpp(0, (int)lo, CTRL, 0xf, 0xf, false);
    b = (unsigned)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, 0xf, 0xf, false);
  } else {
    // a swap of x with itself leaves one partner's rows in each result: the
    // rows that were replaced hold the partner, the others x itself
    const bool upper = STEP == 4 ? (threadIdx.x & 16) != 0 : (threadIdx.x & 32) != 0;
    if constexpr (STEP == 4) {
      const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
      const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
      a = upper ? l[0] : l[1];
      b = upper ? h[0] : h[1];
    } else {
      const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
      const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
      a = upper ? l[0] : l[1];
      b = upper ? h[0] : h[1];
    }
  }
  return ((unsigned long long)b << 32) | a;
}

// x of the first lane, in scalar registers.
__device__ __forceinline__ double uniform(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)b);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// c_max of a slot, per direction (0 for inactive ones): the maximum over its
// parts, formed by every wavefront for itself (all lanes active).
template <int NDIM>
__device__ __forceinline__ void load_cmax(const Control* ctl, int slot, double* c) {
  const CmaxPart* p = &ctl->cm[slot][threadIdx.x & (CM_SUBS - 1)];
  unsigned long long x[3] = {0ull, 0ull, 0ull};
#pragma unroll
  for (int d = 0; d < NDIM; ++d) x[d] = p->v[d];
  static_assert(CM_SUBS == 32, "one part per lane of a half wavefront");
  static_for<0, 5>([&](auto Step) {
#pragma unroll
    for (int d = 0; d < NDIM; ++d) {
      const unsigned long long y = partner_bits<decltype(Step)::value>(x[d]);
      x[d] = y > x[d] ? y : x[d];
    }
  });
#pragma unroll
  for (int d = 0; d < 3; ++d) c[d] = uniform(__longlong_as_double((long long)x[d]));
}

// Folds a work-group's maximum along d into a slot.
__device__ __forceinline__ void fold_cmax(Control* ctl, int slot, int d, double m) {
  atomicMax(&ctl->cm[slot][blockIdx.x & (CM_SUBS - 1)].v[d], (unsigned long long)__double_as_longlong(m));
}

// Clears a slot (the first CM_SUBS threads of the calling work-group).
__device__ __forceinline__ void clear_cmax(Control* ctl, int slot) {
  if (threadIdx.x < CM_SUBS) {
#pragma unroll
    for (int d = 0; d < 3; ++d) ctl->cm[slot][threadIdx.x].v[d] = 0ull;
  }
}

__device__ __forceinline__ double wave_max(double x) {
  static_for<0, 6>([&](auto Step) {
    x = fmax(x, __longlong_as_double(
                    (long long)partner_bits<decltype(Step)::value>((unsigned long long)__double_as_longlong(x))));
  });
  return x;
}

// Sum over the 64 lanes of a wave in a fixed butterfly order (deterministic).
__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) x = x + __shfl_xor(x, m, 64);
  return x;
}

}  // namespace amrvac
