// Whole runs of time steps of a small 1D list in one launch (k_line): hydro
// and ideal MHD, MP5 and LIM03, all three schemes, bit for bit what the stage
// kernels compute.
//
// What bounded such lists: a 512-cell tube is 8 tiles of 64 cells, so a stage
// was a launch of 7 us (hydro) or 10 us (MHD) that is nearly all latency (the
// launch itself, c_max and table loads, state loads, stores), and a step one
// launch more.  Here one work-group keeps every cell's state in registers, one
// cell per thread, and the split fluxes and interface fluxes of the whole list
// in LDS; a stage is three barriers:
//   A) split fluxes of every cell to LDS, also to the halo of the neighbour
//      block that reads them (each block's line has 3 halo entries at both
//      ends; fixed ghost cells have threads of their own, with constant state);
//   B) one item per (sign, variable, run of interfaces), R(F+) and
//      R(F-) to LDS;
//   C) difference, stage update, speeds, and their maximum over the list.
// Measured on 512 cells: an RK3 step of hydro in one call 36 -> 11.9 us (2.9 us
// per stage and 3.4 us for the launch), 40 SSPRK(5,4) steps of MHD 2.18 -> 1.10
// ms (5.4 us per stage).  What bounds it now: one CU is all the arithmetic
// there is (an MHD stage's reconstructions alone take it 2.4 us) and the chain
// of three barriers, a division and the square roots of the speeds.  The limit
// is a thread per cell (and fixed ghost cell) and the fluxes in one CU's LDS: up
// to 1018 hydro or 598 MHD cells in one block with fixed faces, fewer in many
// blocks.
#include "device_math.h"

namespace amrvac {

namespace {

template <bool MHD, bool LIM, int RUN>
__global__ void __launch_bounds__(line_threads(MHD)) k_line(LineParams P) {
  using E = Eq<1, MHD>;
  constexpr int NV = E::NV;
  constexpr int HG = LIM ? 2 : NG;
  constexpr int NT = line_threads(MHD), NW = NT / 64;
  // F+ and F- of every variable per line entry, then R(F+) and R(F-) per
  // interface, then the wavefront maxima.  Entries are ES = 2 NV + 1 apart: a
  // thread's accesses differ by constants, and the odd stride keeps lanes on
  // neighbouring entries, or on runs of odd length, off each other's banks.
  extern __shared__ double lds[];
  constexpr int ES = line_stride(NV);
  double* const phi = lds;
  double* const rec = lds + ES * P.length;
  double* const red = rec + ES * P.nifc;

  const int tid = threadIdx.x;
  const bool cell = tid < P.ncells;
  const bool has = tid < P.ncells + P.nghost;
  const double gamma = P.gamma;
  const LineCell me = P.cells[has ? tid : 0];
  double u[NV], U0[NV], S[NV];
  {
    gptr p = (gptr)me.u;
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = p[v * me.vs];
  }
  bool ok_all = true;
  double ri = 1.0, pr = 1.0;   // 1/rho and p of u
  // c_max of the current state, the same in every thread
  auto all_cmax = [&]() {
    PrimD w;
    const bool ok = prim<1, MHD>(u, gamma, w);
    ri = w.ri;
    pr = w.p;
    ok_all = (ok || !has) && ok_all;
    const double m = wave_max(cell ? fabs(w.v[0]) + fast_speed<MHD>(w, 0, gamma) : 0.0);
    if ((tid & 63) == 0) red[tid >> 6] = m;
    __syncthreads();
    double r = red[0];
#pragma unroll
    for (int q = 1; q < NW; ++q) r = fmax(r, red[q]);
    return r;
  };
  double c = all_cmax();
  double t = P.first ? P.t0 : P.ctl->t;
  double dt = 0.0;

  for (int step = 0; step < P.nsteps; ++step) {
    // the largest of c_max / dx over the list is the one of the smallest dx
    dt = P.dt_fixed > 0.0 ? P.dt_fixed : P.cfl / fmax(0.0, c / P.dx_min);
    t += dt;
#pragma unroll
    for (int v = 0; v < NV; ++v) U0[v] = u[v];
    for (int stage = 0; stage < P.nstages; ++stage) {
      const LineStage& R = P.stage[stage];
      if (has) {
        PrimD w;
        prim_from<1, MHD>(u, ri, pr, w);
        double F[NV];
        phys_flux<1, MHD, 0>(u, w, F);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double fp = fma(c, u[v], F[v]), fm = fma(-c, u[v], F[v]);
          phi[me.pos * ES + v] = fp;
          phi[me.pos * ES + NV + v] = fm;
          if (me.dup[0] >= 0) {
            phi[me.dup[0] * ES + v] = fp;
            phi[me.dup[0] * ES + NV + v] = fm;
          }
          if (me.dup[1] >= 0) {
            phi[me.dup[1] * ES + v] = fp;
            phi[me.dup[1] * ES + NV + v] = fm;
          }
        }
      }
      __syncthreads();
      for (int item = tid; item < 2 * NV * P.nruns; item += NT) {
        const int run = item % P.nruns, k = item / P.nruns;   // k: variable, then sign
        const bool minus = k >= NV;
        const LineRun L = P.runs[run];
        // interface q of the run lies above line entry pos + q + 2; windows as
        // in k_stage: F+ upwards from entry pos, F- downwards from pos + W
        constexpr int W = RUN + 2 * HG - 2;
        const double* f = phi + (L.pos + (NG - HG) + (minus ? W : 0)) * ES + k;
        const int s = minus ? -ES : ES;
        double fw[W], r[RUN];
#pragma unroll
        for (int m = 0; m < W; ++m) fw[m] = f[m * s];
        if constexpr (LIM) {
          int unused;
#pragma unroll
          for (int q = 0; q < RUN; ++q) r[q] = lim03_eval<false>(fw[q], fw[q + 1], fw[q + 2], L.kr, unused);
        } else {
          mp5_stream<RUN>(fw, r);
        }
        double* o = rec + (L.ifc + (minus ? RUN - 1 : 0)) * ES + k;
#pragma unroll
        for (int q = 0; q < RUN; ++q) o[q * s] = r[q];
      }
      __syncthreads();
      if (cell) {
        const double dtb = dt * R.b, dtsb = dt * R.sb;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double* p = rec + me.ifc * ES + v;
          const double diff = (p[ES] + p[ES + NV]) - (p[0] + p[NV]);
          const double L = fma(-diff, me.hidx, 0.0);
          const double un =
              R.x == 0 ? fma(dtb, L, R.a1 * u[v]) : fma(dtb, L, fma(R.a1, u[v], R.a0 * (R.x == 1 ? U0[v] : S[v])));
          if (R.y != 0) S[v] = fma(dtsb, L, fma(R.sa1, u[v], R.sa0 * (R.y == 1 ? U0[v] : S[v])));
          u[v] = un;
        }
      }
      c = all_cmax();
    }
  }
  if (cell) {
    gptr_w p = (gptr_w)me.u;
#pragma unroll
    for (int v = 0; v < NV; ++v) p[v * me.vs] = u[v];
  }
  if (tid == 0) {
    P.ctl->t = t;
    P.ctl->dt = dt;
  }
  if (!ok_all) atomicOr(&P.ctl->err, 1);
}

// f(kernel) for the kernel of a physics, reconstruction and run length.
template <class F>
hipError_t with_kernel(bool mhd, bool lim, int run, F&& f) {
  hipError_t e = hipErrorInvalidValue;
  auto pick = [&](auto Q) {
    constexpr int RUN = LINE_RUNS[decltype(Q)::value];
    if (RUN != run) return;
    if (mhd) e = lim ? f(&k_line<true, true, RUN>) : f(&k_line<true, false, RUN>);
    else e = lim ? f(&k_line<false, true, RUN>) : f(&k_line<false, false, RUN>);
  };
  pick(std::integral_constant<int, 0>{});
  pick(std::integral_constant<int, 1>{});
  pick(std::integral_constant<int, 2>{});
  pick(std::integral_constant<int, 3>{});
  pick(std::integral_constant<int, 4>{});
  static_assert(sizeof(LINE_RUNS) / sizeof(LINE_RUNS[0]) == 5, "one line per run length");
  return e;
}

}  // namespace

hipError_t launch_line(bool mhd, bool lim, const LineParams& p, size_t lds, hipStream_t s) {
  return with_kernel(mhd, lim, p.run, [&](auto k) {
    hipLaunchKernelGGL(k, dim3(1), dim3(line_threads(mhd)), lds, s, p);
    return hipGetLastError();
  });
}

// The kernels use more dynamic LDS than the default limit of a launch.
hipError_t prepare_line(bool mhd, bool lim, int run) {
  return with_kernel(mhd, lim, run, [&](auto k) {
    return hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, LINE_LDS_BYTES);
  });
}

}  // namespace amrvac
