// Internal data structures shared by the host runtime and the HIP kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace amrvac {

constexpr int NG = 3;          // ghost layers (MP5 stencils reach i-2..i+3)
constexpr int MAX_SLOTS = 8;   // c_max slots per step (stages + 1)

// Radius r of LIM03's asymptotic region, in units of the data per cell width.
constexpr double LIM03_RADIUS = 1.0;

// LIM03's scale 1 / (r dx)^2 for split fluxes held without their factor 1/2
// (doubled data), from 0.5 / dx.
__host__ __device__ inline double lim03_scale(double hidx) {
  return (hidx * (1.0 / LIM03_RADIUS)) * (hidx * (1.0 / LIM03_RADIUS));
}

// One block as the kernels see it.
struct BlockDev {
  double* u;            // caller's padded state (buffer id 0)
  long long off;        // offset (doubles) of this block inside one scratch slot
  long long coff;       // offset (cells) of this block in per-cell arrays (off / nvar)
  long long cells;      // interior cells n0*n1*n2
  int n[3];             // interior extents (1 for inactive directions)
  int P[3];             // padded extents
  int g[3];             // ghost depth per direction (3 or 0)
  int nbr[6];           // face neighbours, -1 = fixed ghosts in u
  double dx[3];
  double inv_dx[3];
  // Adjoint bookkeeping of fixed faces (-1 where the face has a neighbour):
  // fco[d]: index, in 8-byte code words after the interior cells of a code
  //   plane, of the words of the interfaces on the upper face of direction d
  //   (one per face cell, transverse coordinates in x, y, z order);
  // gho[f]: index, in ghost cells of the boundary-data adjoint, of the 3
  //   ghost layers of face f (-x, +x, -y, +y, -z, +z), layer-major from the
  //   face outwards, transverse coordinates in x, y, z order.
  long long fco[3];
  long long gho[6];
};

// One unit of work: a box of interior cells of one block.
struct Tile {
  int block;
  int o[3];             // origin (interior coordinates)
};

// Where the cells of one side of a tile start in a state buffer, and their
// strides.  addr: a byte address (rel = 0: a caller's array), or a cell offset
// inside a scratch slot (rel = 1).
struct TileSide {
  long long addr;
  long long vs;         // between variables
  int s1, s2;           // between rows and planes
  int rel;
  int rem;              // upper halo: rows before this one are the block's own
};

// What the role-split stage kernel needs of a tile, so that it follows no
// chain of table lookups: side[0] addresses the callers' arrays, side[1] the
// scratch slots (fixed ghost layers are in the callers' arrays either way);
// sides 0..5 are the halos (-x, +x, -y, +y, -z, +z), 6 the tile's own cells.
struct TileInfo {
  int block;
  int e[3];             // cells per direction
  double hidx[3];       // 0.5 / dx
  long long org;        // first cell in an interior-layout array of the block
  long long pad_[2];    // to 64 bytes
  TileSide side[2][7];
};

// c_max slots are spread over CM_SUBS partial maxima in cache lines of their
// own (work-group w adds to part w mod CM_SUBS), which every reader folds:
// atomics to one line are served one after the other, about 11 ns each, and a
// launch ends with up to three per work-group (2048 work-groups of the
// stand-alone reduction took 75 us for 0.5 M cells, 512 of a stage 17 us at
// its end).
constexpr int CM_SUBS = 32;
struct CmaxPart {
  unsigned long long v[3];
  unsigned long long pad_[5];
};

// Device-resident step control: c_max slots (uint64 bit patterns of
// non-negative doubles, so integer max == floating max), dt, t, error flag.
struct Control {
  CmaxPart cm[MAX_SLOTS][CM_SUBS];
  double dt;
  double t;
  double dt_fixed;      // > 0: fixed step
  double cfl;
  int err;              // sticky: 1 = non-physical state met
  int ndx;              // number of distinct dx tuples in dxtab
  int pad[2];
  // c_max maximiser per direction ((block << 32) | interior linear index),
  // filled by the adjoint's argmax reduction
  long long arg[3];
  // GLM: factor exp(-dt c_h / c_r) of this step's psi decay
  double psi_decay;
};

// GLM: c_r = c_p^2 / c_h of the operator-split psi decay.
constexpr double GLM_CR = 0.18;

// Buffers: id 0 = caller's padded u; id k >= 1 = scratch slot k-1 with the
// interior-only layout, at scr + (k-1)*slot_stride + block.off.
struct StateTable {
  const BlockDev* blocks;
  double* scr;
  long long slot_stride;
};

constexpr int MAX_SRC = 3;

// Parameters of one fused stage launch:
//   L     = L(buffer `in`)   (c_max from slot cm_in)
//   dst   = sum_j a[j] * buffer src[j] + (dt * b) * L          (mode 0)
//   sdst  = sum_j sa[j] * buffer ssrc[j] + (dt * sb) * L       (optional)
//   rhs_out[block] = L  (interior layout)                     (mode 1)
// Every WG keeps a running maximum of |v_d| + c_f,d of the new state and
// folds it into slot cm_out at exit (cm_out < 0: none).  cm_reset >= 0:
// one thread clears that slot.
struct StageParams {
  StateTable st;
  const Tile* tiles;
  const TileInfo* info;   // the same tiles, for the role-split forms
  int tile_begin;
  int ntiles;
  Control* ctl;
  double gamma;
  int in;
  int mode;
  int cm_in, cm_out, cm_reset;
  int nsrc;
  int src[MAX_SRC];
  double a[MAX_SRC];
  double b;
  int dst;
  int snsrc;
  int ssrc[MAX_SRC];
  double sa[MAX_SRC];
  double sb;
  int sdst;
  double* const* rhs_out;
  // GLM: multiply psi by the step's decay factor (last stage of a step)
  int decay_psi;
  // Hall MHD: eta_h and the cell-centred current of the input state, three
  // planes of interior cells (plane v at J + v * jplane, block at coff)
  double eta_h;
  const double* J;
  long long jplane;
  // Optional (only the code-emitting kernels write it): linear-piece codes
  // of the reconstructions (MP5 or LIM03) of L(in), one byte per
  // (direction, cell, variable) for the
  // interface on the cell's lower face, low nibble for the F+ stencil and
  // high nibble for the F- stencil, at
  //   codes + D * code_plane + (block.coff + cell) * 8 + v.
  unsigned char* codes;
  long long code_plane;
  // words of the upper fixed-face interfaces start at word code_faces of a
  // plane (the number of interior cells)
  long long code_faces;
  // Optional (the adjoint's recompute): the c_max of this stage's input
  // state (slot cm_in as read at launch) is copied to cm_hist[0..2]
  double* cm_hist;
};

struct LineParams;

// One compiled form of the fused stage kernel (a tile shape and its
// options): its table entry, shared by the kernel file that instantiates it
// and the runtime that selects it.
struct StageVariant {
  int ndim, mhd, rec, hall, tx, ty, tz, nt, ngrp, wpe;   // mhd: physics code; rec: 0 MP5, 1 LIM03
  int info;              // > 0: reads the TileInfo table, built for this halo width
  const void* fn;
  void (*launch)(const StageParams&, int grid, hipStream_t);
  const char* name;
  // info > 0: fills the table of a tile list
  void (*make_info)(const BlockDev* blocks, const Tile* tiles, TileInfo* table, int ntiles, int ndim, int hg, int tx,
                    int ty, int tz, hipStream_t s) = nullptr;
  // 1D, if set: this form runs whole steps of a small list in one launch
  // (launch and the tile shape then serve right-hand sides), and what comes
  // before the first such launch
  hipError_t (*line)(bool mhd, bool lim, const LineParams& p, size_t lds, hipStream_t s) = nullptr;
  hipError_t (*prepare_line)(bool mhd, bool lim, int run) = nullptr;
  int preferred = 0;   // among the general forms (info == 0) of its kind; 2: in the batched forms only
};

const StageVariant* tile_variants(int* count);   // stage_tile.hip
const StageVariant* tile_emit_variant(int ndim, int mhd, int rec);   // stage_emit.hip, or nullptr
void launch_tile_info(const BlockDev* blocks, const Tile* tiles, TileInfo* info, int ntiles, int ndim, int hg, int tx,
                      int ty, int tz, hipStream_t s);
hipError_t launch_line(bool mhd, bool lim, const LineParams& p, size_t lds, hipStream_t s);   // line.hip
hipError_t prepare_line(bool mhd, bool lim, int run);

struct CmaxParams {
  StateTable st;
  const Tile* tiles;
  int ntiles;
  int tx, ty, tz;       // tile extents used for the tile list
  Control* ctl;
  double gamma;
  int in;
  int slot;
  double eta_h;         // Hall MHD: the whistler speed enters c_max
};

// ---------------------------------------------------------------------------
// Runs of steps of a small 1D list in one launch (line.hip).
// ---------------------------------------------------------------------------
// Threads of the one work-group: hydro 16 wavefronts; MHD 10, whose three
// states of 8 variables need more registers than 16 wavefronts leave a thread.
constexpr int line_threads(bool mhd) { return mhd ? 640 : 1024; }
// Doubles per line entry in LDS.
constexpr int line_stride(int nvar) { return 2 * nvar + 1; }
// Interfaces per reconstruction item that the kernel is compiled for.
constexpr int LINE_RUNS[] = {4, 5, 7, 9, 13};
constexpr int LINE_LDS_BYTES = 160 * 1024;
constexpr int LINE_STEPS = 64;                // steps per launch

// A cell of the list (then the ghost cells of its fixed faces), one per
// thread: where its state is, its entry in the lines of split fluxes and up to
// two halo entries that repeat it, its lower interface, 0.5 / dx.
struct LineCell {
  double* u;
  long long vs;
  double hidx;
  int pos, dup[2], ifc;
};

// Consecutive interfaces of a block, the first above line entry pos + 2; kr: LIM03's scale for doubled data.
struct LineRun {
  int pos, ifc;
  double kr;
};

// One stage's update: dst = a0 X + a1 u + dt b L (x: 0 no X, 1 the step's
// initial state, 2 the accumulator) and, with y != 0, the accumulator
// S = sa0 Y + sa1 u + dt sb L.
struct LineStage {
  int x, y;
  double a0, a1, b, sa0, sa1, sb;
};

struct LineParams {
  const LineCell* cells;
  const LineRun* runs;
  Control* ctl;
  double gamma, dt_fixed, cfl, t0, dx_min;
  int ncells, nghost, nruns, length, nifc;
  int run;                      // interfaces per item
  int nsteps, nstages, first;   // first: the start time is t0, else ctl->t
  LineStage stage[5];
};

// One fixed face of a block list (the adjoint's boundary-data pass).
struct FixedFace {
  int block;
  int face;   // 2 d + side
};

// What the VJP needs of a tile: as TileInfo, for scratch slots, with the code
// words of each side.  side: the halos (3 rows from row -3, or from the first
// row above the tile), and the tile's own cells (6).
struct VjpSide {
  long long slot, code, vs;   // first cell in a slot and in a code plane, variable stride
  int s1, s2;
  int fixed;                  // no neighbour: no mu
  int pad_;
};
struct alignas(64) VjpInfo {
  int block;
  int e[3];                   // cells per direction
  int rem[3];                 // rows of the upper halo that are the block's own
  int n0, n1;                 // block extents
  int p1, p2;                 // padded strides
  int pad_;
  double idx[3];
  long long org;              // first cell's index in the block
  long long face[3];          // code word above the tile on a fixed upper face, or -1
  double* u;                  // first cell in the caller's array
  long long pvs;
  VjpSide side[7];
};

constexpr int MAX_TERMS = 6;

// Parameters of one vector-Jacobian product of L (adjoint of one stage
// state U = buffer `in`):
//   mu   = sum_q mu_a[q]  * buffer mu_src[q]                (on the fly)
//   dst  = sum_q lam_a[q] * buffer lam_src[q] + scale * J_L(U)^T mu
// for the local dependence of L on U; the MP5 linear pieces come from the
// codes the forward recompute of U's stage wrote (layout as in
// StageParams).  The c_max part (through the maximising cell) is added by a
// separate reduction from the per-tile sums written to cpart[tile*3+d].
struct VjpParams {
  StateTable st;
  const VjpInfo* info;
  int ntiles;
  Control* ctl;
  double gamma;
  int in;
  const unsigned char* codes;
  long long code_plane;
  long long code_faces;   // as in StageParams
  int recon;   // reconstruction the codes refer to: 0 MP5, 1 LIM03
  int nmu;
  int mu_src[MAX_TERMS];
  double mu_a[MAX_TERMS];
  int nlam;
  int lam_src[MAX_TERMS];
  double lam_a[MAX_TERMS];
  int dst;
  double scale;
  // c_max of the state `in` per direction, as its recompute recorded it; the
  // VJP marks the maximising cells (lowest (block, cell) key, atomicMin into
  // ctl->arg, which the c_max term then consumes and resets)
  const double* cm_in;
  double* cpart;    // per-work-group c_max adjoint partials, 3 per work-group
};

// A VJP kernel (tile shape as the code-emitting stage kernel of the same
// ndim and physics), its c_max-term kernel and its fixed-face ghost kernel.
struct VjpVariant {
  int ndim, mhd, tx, ty, tz, nt;
  const void* fn;
  void (*launch)(const VjpParams&, int grid, hipStream_t);
  // the c_max term: sum of the partials, applied at the maximising cell
  void (*cmax_term)(StateTable, int, const double*, int, Control*, double, int, int, double, hipStream_t);
  void (*ghost)(const VjpParams&, const FixedFace*, int, double*, long long, double*, int, hipStream_t);
};

// dst = sum_j a[j] * src[j] over the interiors (up to 6 terms).
struct CombineParams {
  StateTable st;
  const Tile* tiles;
  int ntiles, tx, ty, tz, nv;
  int n;
  int src[6];
  double a[6];
  int dst;
};

const VjpVariant* vjp_variant(int ndim, int mhd);
void launch_vjp_info(const BlockDev* blocks, const Tile* tiles, VjpInfo* info, int ntiles, int ndim, int tx, int ty,
                     int tz, hipStream_t s);
void launch_combine(const CombineParams& p, int grid, hipStream_t s);
void launch_lam_import(StateTable st, double* const* ptrs, int nv, int dst, int nblocks, hipStream_t s);
void launch_lam_export(StateTable st, double* const* ptrs, int nv, int src, int nblocks, const double* gadj,
                       long long gplane, hipStream_t s);

}  // namespace amrvac
