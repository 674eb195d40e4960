// The fused Shu-Osher stage (Sects. 2.1-2.3) on small tiles with many
// wavefronts: k_tile computes what k_stage (kernels.hip) computes, bit for
// bit, for MP5 and LIM03 in hydro and ideal MHD.
//
// What bounded k_stage: with 2 wavefronts per SIMD every phase waited for its
// own loads.  On the 256^3 MHD list a step took 13.4 ms of which the state
// loads, update and stores alone take 5.5 ms and MP5 alone 3.3 ms, one after
// the other.  k_tile therefore
//   * holds its registers at 128, so that 16 wavefronts (two work-groups of 8)
//     share a CU and one work-group's arithmetic covers the other's loads;
//   * splits a work-group by role: TC owner threads keep their cell's state
//     and L in registers, the other threads keep halo cells in the same
//     registers, so every cell of the extended box is converted by one pass
//     of one instruction stream;
//   * issues the halo loads of the next direction (after the last one, of the
//     next tile) before the reconstructions of this one, with addresses from
//     scalar loads of the block table, so that no load is waited for where it
//     is issued;
//   * gives a wavefront one variable and splits the two signs between its
//     halves: lanes 0-31 reconstruct F+, lanes 32-63 F- (stored mirrored along
//     the direction, so both walk their pencil upwards), and the sums are
//     formed across the halves.
// Measured per SSPRK(5,4) + MP5 step, the best k_stage form against this one:
// 256^3 MHD 13.4 -> 11.9 ms, uneven 4096-block list 20.4 -> 19.5 ms, 2D MHD
// 512^2 (4 steps) 0.77 -> 0.66 ms, 2D Euler 256^2 (20 steps) 1.56 -> 1.41 ms;
// RK3 + LIM03 on 1024 uneven blocks (2 steps) 5.03 -> 4.05 ms.  (With c_max in
// 32 parts, shuffle-free reductions and the x row stride below: 11.1, 18.5,
// 0.52, 0.89 and 3.92 ms.)  The VALU is then busy 60 % of the cycles (45 % before) with 2940 instructions per cell
// and stage; 8x8x8 tiles of 1024 threads, one work-group per CU, take 12.9 ms
// on the 256^3 list: fewer halo cells, but nothing runs during its barriers.
#pragma once
#include "device_math.h"

#include <cstddef>

namespace amrvac {

namespace {

// Address of a table entry's first cell in buffer `buf`.
__device__ __forceinline__ gptr side_addr(const StateTable& st, cptr<TileSide> s, int buf) {
  return s->rel ? (gptr)st.scr + ((long long)(buf - 1) * st.slot_stride + s->addr) : (gptr)(unsigned long long)s->addr;
}

// Uniform base, 32-bit lane offset (in cells).
__device__ __forceinline__ double load_at(gptr base, unsigned off) {
  return *(gptr)((__attribute__((address_space(1))) const char*)base + off * 8u);
}
__device__ __forceinline__ void store_at(gptr_w base, unsigned off, double x) {
  *(gptr_w)((__attribute__((address_space(1))) char*)base + off * 8u) = x;
}

// x of lanes 0-31 beside y of lanes 0-31 (result x), and x of lanes 32-63
// beside y of lanes 32-63 (result y).
__device__ __forceinline__ void swap_halves(double& x, double& y) {
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  unsigned long long xb = (unsigned long long)__double_as_longlong(x), yb = (unsigned long long)__double_as_longlong(y);
  const u2 lo = __builtin_amdgcn_permlane32_swap((unsigned)xb, (unsigned)yb, false, false);
  const u2 hi = __builtin_amdgcn_permlane32_swap((unsigned)(xb >> 32), (unsigned)(yb >> 32), false, false);
  x = __longlong_as_double((long long)(((unsigned long long)hi.x << 32) | lo.x));
  y = __longlong_as_double((long long)(((unsigned long long)hi.y << 32) | lo.y));
}

// Work split of the reconstructions along one direction: NP pencils of NIF
// interfaces, NW wavefronts, NV variables.
template <int NP, int NIF, int NW, int NV>
struct Split {
  static constexpr int WPV = NW / NV;                   // wavefronts per variable
  static_assert(WPV >= 1, "one wavefront per variable at least");
  static constexpr bool BOTH = NP >= 64 * WPV;          // a lane does both signs of its pencil
  static_assert(BOTH ? NP == 64 * WPV : NP >= 32 ? NP % 32 == 0 && WPV % (NP / 32) == 0 : 32 % NP == 0,
                "pencils fill the wavefronts");
  static constexpr int PG = NP >= 32 ? NP / 32 : 1;     // groups of pencils (one per wavefront)
  static constexpr int SEGL = NP >= 32 ? 1 : 32 / NP;   // segments of a pencil in one wavefront
  static constexpr int NSEG = BOTH ? 1 : SEGL * (WPV / PG);
  static constexpr int RUN = (NIF + NSEG - 1) / NSEG;
};

// What a launch does with L, fixed at compile time: the update's loads are
// then unconditional and its values live in one straight piece of code.
enum StageForm {
  ONE_SOURCE,    // dst = a in + dt b L
  TWO_SOURCES,   // dst = a0 X + a1 in + dt b L
  ACCUMULATOR,   // the same, and sdst = sa0 Y + sa1 in + dt sb L
  RHS            // L itself
};

}  // namespace

template <int FORM, int NDIM, bool MHD, bool LIM, bool EMIT, int TX, int TY, int TZ, int NT, int WPE>
__global__ void __launch_bounds__(NT, WPE) k_tile(StageParams P) {
  constexpr int HG = LIM ? 2 : NG;
  using E = Eq<NDIM, MHD>;
  using S = TileShape<TX, TY, TZ, HG>;
  constexpr int NV = E::NV;
  constexpr int TC = S::TC;
  constexpr int NW = NT / 64;
  constexpr int NHT = NT - TC;   // halo threads
  static_assert(TC % 64 == 0 && NHT >= 64, "roles are whole wavefronts");
  // LDS stride of the x rows: odd, or 2 modulo 4, keeps 16 lanes on 16 rows
  // off each other's banks
  constexpr int XP = (TX + 2 * HG) % 4 == 2 ? TX + 2 * HG : (TX + 2 * HG) | 1;
  // per interface: a flux of every variable and, for the code-emitting forms,
  // two words of codes (byte v for variable v: the F+ piece, the F- piece)
  constexpr int NR = NV + (EMIT ? 2 : 0);
  static_assert(!EMIT || NV <= 8, "8 code bytes per word");
  constexpr int EXT = cmax_i<cmax_i<XP * TY * TZ, NDIM >= 2 ? S::NEXT(1) : 0>::v, NDIM >= 3 ? S::NEXT(2) : 0>::v;
  constexpr int IFC = cmax_i<cmax_i<S::NIFC(0), NDIM >= 2 ? S::NIFC(1) : 0>::v, NDIM >= 3 ? S::NIFC(2) : 0>::v;
  // interface fluxes beside the split fluxes (at the top of the array) where
  // both fit in the LDS of WPE * 4 / NW work-groups per CU
  constexpr int LDS_LIMIT = 20480 / (WPE * 4 / NW);
  constexpr int side0 = 2 * NV * XP * TY * TZ + NR * S::NIFC(0);
  constexpr int side1 = NDIM >= 2 ? 2 * NV * S::NEXT(1) + NR * S::NIFC(1) : 0;
  constexpr int side2 = NDIM >= 3 ? 2 * NV * S::NEXT(2) + NR * S::NIFC(2) : 0;
  constexpr int PAD = cmax_i<cmax_i<side0 <= LDS_LIMIT ? side0 : 0, side1 <= LDS_LIMIT ? side1 : 0>::v,
                             side2 <= LDS_LIMIT ? side2 : 0>::v;
  constexpr int LDS_N = cmax_i<cmax_i<2 * NV * EXT, NR * IFC>::v, PAD>::v;
  static_assert(LDS_N <= LDS_LIMIT, "tile too large for the resident work-groups");
  __shared__ double lds[LDS_N];
  double (*red)[3] = reinterpret_cast<double (*)[3]>(lds);

  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const bool owner = wv < TC / 64;
  const StateTable& st = P.st;
  Control* ctl = P.ctl;
  const double gamma = P.gamma;

  double cin[3];
  load_cmax<NDIM>(ctl, P.cm_in, cin);
  const double dt = FORM == RHS ? 0.0 : constant_ptr(ctl)->dt;
  if (P.cm_reset >= 0 && blockIdx.x == 0) clear_cmax(ctl, P.cm_reset);
  if constexpr (EMIT) {
    if (P.cm_hist && blockIdx.x == 0 && tid == 0) {
#pragma unroll
      for (int d = 0; d < 3; ++d) P.cm_hist[d] = cin[d];
    }
  }
  double run[3] = {0.0, 0.0, 0.0};
  bool ok_all = true;

  const cptr<TileInfo> tiles = constant_ptr(P.info + P.tile_begin);
  const int pad_in = P.in == 0 ? 0 : 1;   // which addresses of the table serve buffer `in`

  // own cell of an owner thread
  auto own_pos = [&](int* a) {
    const int i = fresh(tid);
    a[0] = i % TX;
    a[1] = (i / TX) % TY;
    a[2] = i / (TX * TY);
  };
  // The own cell's values in buffer `buf`.  Lanes without a cell of their own
  // (partial tiles) load the nearest one: no load is conditional per lane, so
  // u is dead before it.
  auto load_cell_of = [&](cptr<TileInfo> T, int buf, double* u) {
    int a[3];
    own_pos(a);
#pragma unroll
    for (int d = 0; d < 3; ++d) a[d] = a[d] < T->e[d] ? a[d] : T->e[d] - 1;
    const cptr<TileSide> sd = &T->side[buf == 0 ? 0 : 1][6];
    const gptr q = side_addr(st, sd, buf);
    const unsigned off = (unsigned)(a[0] + a[1] * sd->s1 + a[2] * sd->s2);
#pragma unroll
    for (int v = 0; v < NV; ++v) u[v] = load_at(held(q + v * sd->vs), off);
  };

  // halo cell h of direction D (2 HG planes): extended-box position and
  // whether the tile has it
  auto halo_pos = [&](auto Dc, int h, const int* tend, int* a) {
    constexpr int D = decltype(Dc)::value;
    constexpr int H0 = D == 0 ? 2 * HG : TX, H1 = D == 1 ? 2 * HG : TY, H2 = D == 2 ? 2 * HG : TZ;
    a[0] = h % H0;
    a[1] = (h / H0) % H1;
    a[2] = h / (H0 * H1);
    bool valid = h < H0 * H1 * H2;
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (d != D) valid = valid && a[d] < tend[d];
    return valid;
  };
  auto load_halo = [&](auto Dc, cptr<TileInfo> T, int h, double* u) {
    constexpr int D = decltype(Dc)::value;
    const int tend[3] = {T->e[0], T->e[1], T->e[2]};
    int a[3];
    constexpr int NH = 2 * HG * (TC / S::T(D));
    halo_pos(Dc, h < NH ? h : NH - 1, tend, a);
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (d != D) a[d] = a[d] < tend[d] ? a[d] : tend[d] - 1;
    const cptr<TileSide> lo = &T->side[pad_in][2 * D], hi = &T->side[pad_in][2 * D + 1];
    // both sides' entries by scalar loads (held, so that the selection per
    // lane is not turned into vector loads from a selected address)
    const gptr plo = held(side_addr(st, lo, P.in)), phi = held(side_addr(st, hi, P.in));
    const int l1 = held(lo->s1), l2 = held(lo->s2), h1 = held(hi->s1), h2 = held(hi->s2);
    const long long lv = held(lo->vs), hv = held(hi->vs);
    const bool up = a[D] >= HG;
    if (up) a[D] -= HG;
    gptr p = up ? phi : plo;
    int s1 = up ? h1 : l1, s2 = up ? h2 : l2;
    long long vs = up ? hv : lv;
    if (hi->rem < HG && up && a[D] < hi->rem) {
      // the block ends inside the upper halo: its first rows are its own
      const cptr<TileSide> own = &T->side[pad_in][6];
      p = side_addr(st, own, P.in);
      s1 = own->s1;
      s2 = own->s2;
      vs = own->vs;
      a[D] += tend[D];
    }
    p += a[0] + a[1] * s1 + a[2] * s2;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      u[v] = *p;
      p += vs;
    }
  };

  const TileSchedule sched(P.ntiles);
  // The tile loop, compiled once per role: the roles meet at the same
  // barriers, and neither's registers hold the other's values.
  auto tile_loop = [&](auto Role) __attribute__((always_inline)) {
  constexpr bool OWNER = decltype(Role)::value;
  // owner: the own cell's state and L; halo thread: up to two halo cells' states
  double w[NV], x[NV];
  double ri_own = 1.0, p_own = 1.0;
  int t = sched.t;
  if (t < sched.end) {
    if constexpr (OWNER) load_cell_of(tiles + t, P.in, w);
    else if ((wv - TC / 64) * 64 < 2 * HG * (TC / S::T(0)))
      load_halo(std::integral_constant<int, 0>{}, tiles + t, fresh(tid) - TC, w);
  }
  for (; t < sched.end; t += sched.step) {
    const cptr<TileInfo> T = tiles + t;
    const int tend[3] = {T->e[0], T->e[1], T->e[2]};
    // the next tile's table entry on its way into the scalar cache: one word
    // of each 64-byte line this launch reads (the header's, the halos' and both
    // own cells'), consumed at the end of this tile
    constexpr int NTOUCH = 6;
    int touch[NTOUCH];
    {
      static_assert(sizeof(TileInfo) == 512 && offsetof(TileInfo, side) == 64, "lines of the tile table");
      const cptr<int> line = (cptr<int>)(t + sched.step < sched.end ? T + sched.step : T);
      const int first = pad_in ? 4 : 1;
      touch[0] = line[0];
#pragma unroll
      for (int q = 0; q < 4; ++q) touch[1 + q] = line[16 * (first + q)];
      touch[5] = line[16 * (pad_in ? 4 : 7)];
    }
    auto inside = [&](const int* a) { return a[0] < tend[0] && a[1] < tend[1] && a[2] < tend[2]; };
    if constexpr (OWNER) {
#pragma unroll
      for (int v = 0; v < NV; ++v) x[v] = 0.0;
    }

    double s0[NV], s1[NV];
    static_for<0, NDIM>([&](auto Dc) {
      constexpr int D = decltype(Dc)::value;
      constexpr int E0 = D == 0 ? XP : S::E(D, 0), E1 = S::E(D, 1);
      constexpr int NEXTP = E0 * E1 * S::E(D, 2);
      constexpr int SD = D == 0 ? 1 : D == 1 ? E0 : E0 * E1;
      constexpr int ROWS = S::T(D) + 2 * HG;
      constexpr int NH = 2 * HG * (TC / S::T(D));
      constexpr int NIFC_D = S::NIFC(D), I0 = S::I(D, 0), I1 = S::I(D, 1), SI = S::SI(D);
      constexpr int NIF = S::T(D) + 1, NP = TC / S::T(D);
      using SP = Split<NP, NIF, NW, NV>;
      constexpr int RUN = SP::RUN;
      constexpr bool DISJ = 2 * NV * NEXTP + NR * NIFC_D <= LDS_N;
      constexpr int RB = DISJ ? LDS_N - NR * NIFC_D : 0;
      constexpr int CB = RB + NV * NIFC_D;   // the code words
      constexpr int DN = D + 1 < NDIM ? D + 1 : 0;
      constexpr int NEXT_SPAN =
          cmax_i<2 * NV * (DN == 0 ? XP : S::E(DN, 0)) * S::E(DN, 1) * S::E(DN, 2), 3 * NW>::v;
      constexpr bool SKIP_C_BARRIER = DISJ && NEXT_SPAN <= RB;
      static_assert(NH <= 2 * NHT, "two halo cells per halo thread at most");
      const double c = cin[D];
      const double hidx_d = T->hidx[D];   // the split's factor 1/2 is applied here

      // A) split fluxes of the extended box (without their factor 1/2); the
      // F- box mirrored along D
      auto split_to_lds = [&](const double* u, const PrimD& pw, const int* a, bool in) {
        double F[NV];
        phys_flux<NDIM, MHD, D>(u, pw, F);
        const int el = a[0] + E0 * (a[1] + E1 * a[2]);
        const int em = el + (ROWS - 1 - 2 * a[D]) * SD;
        if (in) {
#pragma unroll
          for (int v = 0; v < NV; ++v) {
            lds[v * NEXTP + el] = fma(c, u[v], F[v]);
            lds[(NV + v) * NEXTP + em] = fma(-c, u[v], F[v]);
          }
        }
      };
      if constexpr (OWNER) {
        PrimD pw;
        if constexpr (D == 0) {
          ok_all = prim<NDIM, MHD>(w, gamma, pw) && ok_all;
          ri_own = pw.ri;
          p_own = pw.p;
        } else {
          prim_from<NDIM, MHD>(w, ri_own, p_own, pw);
        }
        int a[3];
        own_pos(a);
        const bool in = inside(a);
        a[D] += HG;
        split_to_lds(w, pw, a, in);
      } else {
        auto halo = [&](const double* u, int h) {
          int a[3];
          const bool in = halo_pos(Dc, h, tend, a);
          PrimD pw;
          ok_all = prim<NDIM, MHD>(u, gamma, pw) && ok_all;
          if (a[D] >= HG) a[D] += tend[D];
          split_to_lds(u, pw, a, in);
        };
        // whole wavefronts without a halo cell skip the conversion
        if ((wv - TC / 64) * 64 < NH) halo(w, fresh(tid) - TC);
        if constexpr (NH > NHT) {
          if ((wv - TC / 64) * 64 + NHT < NH) halo(x, fresh(tid) - TC + NHT);
        }
        // the next direction's halo (or the next tile's first), in flight
        // during the reconstructions
        if constexpr (D + 1 < NDIM) {
          constexpr int NHN = 2 * HG * (TC / S::T(D + 1));
          if ((wv - TC / 64) * 64 < NHN) load_halo(std::integral_constant<int, D + 1>{}, T, fresh(tid) - TC, w);
          if constexpr (NHN > NHT) {
            if ((wv - TC / 64) * 64 + NHT < NHN)
              load_halo(std::integral_constant<int, D + 1>{}, T, fresh(tid) - TC + NHT, x);
          }
        } else {
          static_assert(2 * HG * (TC / S::T(0)) <= NHT, "the first direction's halo in one pass");
          if (t + sched.step < sched.end && (wv - TC / 64) * 64 < 2 * HG * (TC / S::T(0)))
            load_halo(std::integral_constant<int, 0>{}, tiles + (t + sched.step), fresh(tid) - TC, w);
        }
      }
      __syncthreads();

      // B) interface fluxes R(F+) + R(F-): one variable per wavefront
      const double kr = lim03_scale(hidx_d);
      constexpr int W = RUN + 2 * HG - 2;
      // codes: 4 bits per interface of the run
      auto reconstruct = [&](const double* f, double* r, unsigned long long& codes) {
        double fw[W];
#pragma unroll
        for (int m = 0; m < W; ++m) fw[m] = f[m * SD];
        codes = 0;
        if constexpr (LIM) {
#pragma unroll
          for (int kk = 0; kk < RUN; ++kk) {
            int code;
            r[kk] = lim03_eval<EMIT>(fw[kk], fw[kk + 1], fw[kk + 2], kr, code);
            if constexpr (EMIT) codes |= (unsigned long long)code << (4 * kk);
          }
        } else if constexpr (!EMIT) {
          mp5_stream<RUN>(fw, r);
        } else {
          // the piece is fL (0) unless the value was clamped: each lane
          // searches its own clamped interfaces one after the other, from LDS,
          // so that the search holds few registers and a wavefront repeats it
          // as often as its worst lane needs, not once per interface that is
          // clamped in any lane (128^3 MHD: 404 -> 396 us a recompute stage)
          unsigned left = mp5_stream<RUN>(fw, r);
#pragma unroll 1
          while (__ballot(left != 0) != 0) {
            const int kk = left != 0 ? __builtin_ctz(left) : 0;
            const double* g = f + kk * SD;
            const unsigned code = (unsigned)mp5_code(g[0], g[SD], g[2 * SD], g[3 * SD], g[4 * SD]);
            codes |= (unsigned long long)(left != 0 ? code : 0u) << (4 * kk);
            left &= left - 1;
          }
        }
      };
      // the codes of a run to LDS: q(kk) the interface of its kk-th value
      auto put_codes = [&](unsigned long long codes, bool minus, int var, auto q) {
        unsigned char* lc = reinterpret_cast<unsigned char*>(lds + CB + (minus ? NIFC_D : 0)) + var;
#pragma unroll
        for (int kk = 0; kk < RUN; ++kk) lc[q(kk) * 8] = (unsigned char)((codes >> (4 * kk)) & 15);
      };
      const int var = wv / SP::WPV;
      if constexpr (SP::BOTH) {
        // lane = pencil, both signs one after the other
        double r[RUN];
        unsigned long long cp, cm;
        int q0 = 0;
        const bool active = var < NV;
        if (active) {
          const int pen = fresh(lane) + 64 * (wv % SP::WPV);
          int a[3];
          if constexpr (D == 0) { a[0] = 0; a[1] = pen % TY; a[2] = pen / TY; }
          if constexpr (D == 1) { a[0] = pen % TX; a[1] = 0; a[2] = pen / TX; }
          if constexpr (D == 2) { a[0] = pen % TX; a[1] = pen / TX; a[2] = 0; }
          const int eb = a[0] + E0 * (a[1] + E1 * a[2]);
          q0 = a[0] + I0 * (a[1] + I1 * a[2]);
          double m[RUN];
          reconstruct(&lds[var * NEXTP + eb], r, cp);
          reconstruct(&lds[(NV + var) * NEXTP + eb], m, cm);
#pragma unroll
          for (int kk = 0; kk < RUN; ++kk) r[kk] = r[kk] + m[RUN - 1 - kk];
        }
        if constexpr (!DISJ) __syncthreads();
        if (active) {
#pragma unroll
          for (int kk = 0; kk < RUN; ++kk) lds[RB + var * NIFC_D + q0 + kk * SI] = r[kk];
          if constexpr (EMIT) {
            put_codes(cp, false, var, [&](int kk) { return q0 + kk * SI; });
            put_codes(cm, true, var, [&](int kk) { return q0 + (RUN - 1 - kk) * SI; });
          }
        }
      } else {
        // lanes 0-31 F+, lanes 32-63 F- of the same pencils and segments
        double r[RUN + 1];
        unsigned long long codes;
        int q0 = 0;
        const bool active = var < NV;
        const bool minus = lane >= 32;
        if (active) {
          const int h = fresh(lane) & 31;
          const int part = wv % SP::WPV;
          const int pen = NP >= 32 ? h + 32 * (part % SP::PG) : h % NP;
          const int seg = (part / SP::PG) * SP::SEGL + (NP >= 32 ? 0 : h / NP);
          const int k0 = seg * RUN < NIF - RUN ? seg * RUN : NIF - RUN;
          int a[3];
          if constexpr (D == 0) { a[0] = 0; a[1] = pen % TY; a[2] = pen / TY; }
          if constexpr (D == 1) { a[0] = pen % TX; a[1] = 0; a[2] = pen / TX; }
          if constexpr (D == 2) { a[0] = pen % TX; a[1] = pen / TX; a[2] = 0; }
          const int eb = a[0] + E0 * (a[1] + E1 * a[2]);
          // F- of interfaces k0 .. k0 + RUN - 1 starts, mirrored, at row ROWS
          // - 1 - (k0 + W)
          const int row = minus ? ROWS - 1 - W - k0 : k0;
          q0 = a[0] + I0 * (a[1] + I1 * a[2]) + k0 * SI;
          reconstruct(&lds[(minus ? NV + var : var) * NEXTP + eb + row * SD], r, codes);
          // F- came out from the last interface to the first
#pragma unroll
          for (int kk = 0; kk < RUN / 2; ++kk) {
            const double f = r[kk], l = r[RUN - 1 - kk];
            r[kk] = minus ? l : f;
            r[RUN - 1 - kk] = minus ? f : l;
          }
          if constexpr (RUN % 2) r[RUN] = r[RUN - 1];
          // sums: lanes 0-31 hold the even interfaces, lanes 32-63 the odd ones
#pragma unroll
          for (int kk = 0; kk < RUN; kk += 2) {
            swap_halves(r[kk], r[kk + 1]);
            r[kk] = r[kk] + r[kk + 1];
          }
        }
        if constexpr (!DISJ) __syncthreads();
        if (active) {
          const int odd = minus ? 1 : 0;
#pragma unroll
          for (int kk = 0; kk < RUN; kk += 2)
            if (kk + 1 < RUN || !minus) lds[RB + var * NIFC_D + q0 + (kk + odd) * SI] = r[kk];
          if constexpr (EMIT)
            put_codes(codes, minus, var, [&](int kk) { return q0 + (minus ? RUN - 1 - kk : kk) * SI; });
        }
      }
      if constexpr (D == NDIM - 1) {
        // the stage update's other sources, in flight during C
        if constexpr (OWNER && (FORM == TWO_SOURCES || FORM == ACCUMULATOR)) load_cell_of(T, P.src[0], s0);
        if constexpr (OWNER && FORM == ACCUMULATOR) load_cell_of(T, P.ssrc[0], s1);
      }
      __syncthreads();

      // C) conservative difference into the owned cells
      if constexpr (OWNER) {
        int a[3];
        own_pos(a);
        const int il = a[0] + I0 * (a[1] + I1 * a[2]);
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          const double diff = lds[RB + v * NIFC_D + il + SI] - lds[RB + v * NIFC_D + il];
          x[v] = fma(-diff, hidx_d, x[v]);
        }
        if constexpr (EMIT) {
          // one word per owned cell, the codes of its lower face (low nibbles
          // F+, high nibbles F-; unused bytes of a hydro word unspecified), and
          // for the last cell below a fixed upper face that face's too.  The two
          // stores are conditions beside each other under uniform branches: of a
          // divergent condition nested in another, both ending at one place, the
          // compiler restores the lanes of both only after the copies that its
          // register allocation puts between the two ends, so that they reach
          // some lanes only (seen in the 2D MHD LIM03 forms: the lane number was
          // lost on lists with fixed faces).
          const unsigned long long* lc = reinterpret_cast<const unsigned long long*>(lds + CB);
          const cptr<BlockDev> B = constant_ptr(st.blocks) + T->block;
          const cptr<TileSide> sd = &T->side[1][6];
          using cw = __attribute__((address_space(1))) unsigned long long*;
          const cw plane = (cw)(P.codes + D * P.code_plane);
          const bool in = inside(a);
          if (in) plane[B->coff + T->org + (a[0] + a[1] * sd->s1 + a[2] * sd->s2)] = lc[il] | (lc[NIFC_D + il] << 4);
          if (B->fco[D] >= 0) {
            const cptr<Tile> tl = constant_ptr(P.tiles + P.tile_begin) + t;
            const int ac[3] = {tl->o[0] + a[0], tl->o[1] + a[1], tl->o[2] + a[2]};
            const long long tr = D == 0 ? (long long)ac[1] + (long long)B->n[1] * ac[2]
                               : D == 1 ? (long long)ac[0] + (long long)B->n[0] * ac[2]
                                        : (long long)ac[0] + (long long)B->n[0] * ac[1];
            const bool last = in & (ac[D] == B->n[D] - 1);
            if (last) plane[P.code_faces + B->fco[D] + tr] = lc[il + SI] | (lc[NIFC_D + il + SI] << 4);
          }
        }
      }
      if constexpr (!SKIP_C_BARRIER) __syncthreads();
    });

    // Stage update (or right-hand side output), then the next tile's own
    // cells, then the speeds of the new state.
    if constexpr (OWNER) {
      double un[NV];
      int a[3];
      own_pos(a);
      const bool mine = inside(a);
      const cptr<TileInfo> Tn = t + sched.step < sched.end ? T + sched.step : T;
      auto put = [&](gptr_w p, const cptr<TileSide> sd, const double* val) {
        const unsigned off = (unsigned)(a[0] + a[1] * sd->s1 + a[2] * sd->s2);
        if (mine) {
#pragma unroll
          for (int v = 0; v < NV; ++v) store_at(p + v * sd->vs, off, val[v]);
        }
      };
      auto put_buf = [&](int dst, const double* val) {
        const cptr<TileSide> sd = &T->side[dst == 0 ? 0 : 1][6];
        put((gptr_w)side_addr(st, sd, dst), sd, val);
      };
      // The input comes from registers; the next tile's own cells are loaded
      // ahead of the stores, whose completion a wait for later loads would
      // include.
      if constexpr (FORM == RHS) {
        load_cell_of(Tn, P.in, w);
        put((gptr_w)P.rhs_out[T->block] + T->org, &T->side[1][6], x);
      } else {
        const double dtb = dt * P.b;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          double acc;
          if constexpr (FORM == ONE_SOURCE) acc = P.a[0] * w[v];
          else acc = fma(P.a[1], w[v], P.a[0] * s0[v]);
          un[v] = fma(dtb, x[v], acc);
        }
        if constexpr (FORM == ACCUMULATOR) {
          const double dtsb = dt * P.sb;
#pragma unroll
          for (int v = 0; v < NV; ++v) s1[v] = fma(dtsb, x[v], fma(P.sa[1], w[v], P.sa[0] * s1[v]));
        }
        load_cell_of(Tn, P.in, w);
        if constexpr (FORM == ACCUMULATOR) put_buf(P.sdst, s1);
        put_buf(P.dst, un);
      }
      if constexpr (FORM != RHS) {
        // run[d]: the largest speed this wavefront has met.  A wavefront
        // none of whose cells can exceed it skips the square roots.
        PrimD pw;
        const bool ok = prim<NDIM, MHD>(un, gamma, pw);
        ok_all = (ok || !mine) && ok_all;
#pragma unroll
        for (int d = 0; d < NDIM; ++d) {
          const bool above = mine && speed_may_exceed<MHD>(pw, d, gamma, run[d]);
          if (__ballot(above) != 0)
            run[d] = fmax(run[d], wave_max(mine ? fabs(pw.v[d]) + fast_speed<MHD>(pw, d, gamma) : 0.0));
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < NTOUCH; ++q) asm volatile("" ::"s"(touch[q]));
  }
  };
  if (owner) tile_loop(std::true_type{});
  else tile_loop(std::false_type{});

  // Fold the work-group maxima into the next stage's c_max slot.
  if constexpr (FORM != RHS) {
    if (lane == 0) {
#pragma unroll
      for (int d = 0; d < 3; ++d) red[wv][d] = run[d];
    }
    __syncthreads();
    if (tid == 0) {
#pragma unroll
      for (int d = 0; d < NDIM; ++d) {
        double m = red[0][d];
        for (int q = 1; q < TC / 64; ++q) m = fmax(m, red[q][d]);
        fold_cmax(ctl, P.cm_out, d, m);
      }
    }
  }
  if (!ok_all) atomicOr(&ctl->err, 1);
}

// The stage recipes (runtime.cpp) update from the stage input alone, or from
// another buffer and then the input.
template <int NDIM, bool MHD, bool LIM, bool EMIT, int TX, int TY, int TZ, int NT, int WPE>
static void launch_tile(const StageParams& p, int grid, hipStream_t s) {
  auto go = [&](auto Form) {
    hipLaunchKernelGGL((k_tile<decltype(Form)::value, NDIM, MHD, LIM, EMIT, TX, TY, TZ, NT, WPE>), dim3(grid), dim3(NT), 0,
                       s, p);
  };
  if constexpr (!EMIT) {
    if (p.mode == 1) return go(std::integral_constant<int, RHS>{});
  }
  if (p.sdst >= 0) go(std::integral_constant<int, ACCUMULATOR>{});
  else if (p.nsrc == 2) go(std::integral_constant<int, TWO_SOURCES>{});
  else go(std::integral_constant<int, ONE_SOURCE>{});
}

}  // namespace amrvac
