// The role-split stage kernel's forms (stage_tile.h) and the tile table they
// read.
#include "stage_tile.h"

namespace amrvac {

// Fills the tile table: per tile its extents, dx and, for the caller's
// arrays (first index 0) and for the scratch slots (1), where its own cells
// and the 6 halos start.  One thread per tile.
__global__ void __launch_bounds__(64) k_tile_info(const BlockDev* blocks, const Tile* tiles, TileInfo* info, int ntiles,
                                                int ndim, int hg, int tx, int ty, int tz) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t >= ntiles) return;
  const Tile tl = tiles[t];
  const BlockDev& B = blocks[tl.block];
  const int T[3] = {tx, ty, tz};
  TileInfo I;
  I.block = tl.block;
  for (int d = 0; d < 3; ++d) {
    const int rem = B.n[d] - tl.o[d];
    I.e[d] = rem < T[d] ? rem : T[d];
    I.hidx[d] = 0.5 * B.inv_dx[d];
  }
  I.org = ((long long)tl.o[2] * B.n[1] + tl.o[1]) * B.n[0] + tl.o[0];
  for (int slot = 0; slot < 2; ++slot) {
    auto set = [&](TileSide& s, const BlockDev& b, bool padded, const int* c) {
      if (padded) {
        s.s1 = b.P[0];
        s.s2 = b.P[0] * b.P[1];
        s.vs = (long long)b.P[0] * b.P[1] * b.P[2];
        s.rel = 0;
        s.addr = (long long)(unsigned long long)(b.u + ((long long)(c[2] + b.g[2]) * s.s2 +
                                                        (long long)(c[1] + b.g[1]) * s.s1 + (c[0] + b.g[0])));
      } else {
        s.s1 = b.n[0];
        s.s2 = b.n[0] * b.n[1];
        s.vs = b.cells;
        s.rel = 1;
        s.addr = b.off + ((long long)c[2] * s.s2 + (long long)c[1] * s.s1 + c[0]);
      }
    };
    for (int f = 0; f < 6; ++f) {
      TileSide& s = I.side[slot][f];
      const int d = f / 2;
      int c[3] = {tl.o[0], tl.o[1], tl.o[2]};
      s = TileSide{};
      s.rem = hg;
      if (d >= ndim) continue;
      if (f % 2 == 0) {   // rows o - hg .. o - 1
        c[d] -= hg;
        if (tl.o[d] > 0) {
          set(s, B, slot == 0, c);
        } else if (B.nbr[f] >= 0) {
          const BlockDev& N = blocks[B.nbr[f]];
          c[d] += N.n[d];
          set(s, N, slot == 0, c);
        } else {
          set(s, B, true, c);
        }
      } else {            // rows o + e .. o + e + hg - 1; the first `rem` in this block when it ends among them
        const int in_block = B.n[d] - (tl.o[d] + I.e[d]);
        c[d] += I.e[d];
        if (in_block >= hg) {
          set(s, B, slot == 0, c);
        } else {
          if (B.nbr[f] >= 0) {
            c[d] -= B.n[d];
            set(s, blocks[B.nbr[f]], slot == 0, c);
          } else {
            set(s, B, true, c);
          }
          if (in_block > 0) s.rem = in_block;
        }
      }
    }
    const int c[3] = {tl.o[0], tl.o[1], tl.o[2]};
    I.side[slot][6] = TileSide{};
    set(I.side[slot][6], B, slot == 0, c);
    I.side[slot][6].rem = hg;
  }
  info[t] = I;
}

void launch_tile_info(const BlockDev* blocks, const Tile* tiles, TileInfo* info, int ntiles, int ndim, int hg, int tx,
                      int ty, int tz, hipStream_t s) {
  hipLaunchKernelGGL(k_tile_info, dim3((ntiles + 63) / 64), dim3(64), 0, s, blocks, tiles, info, ntiles, ndim, hg, tx,
                     ty, tz);
}

#define AMRVAC_TILE_ENTRY(ND, M, LIM, TX, TY, TZ, NT, WPE, SUFFIX)                                           \
  {ND, M, LIM, 0, TX, TY, TZ, NT, 1, WPE, LIM ? 2 : NG,                                                   \
   (const void*)&k_tile<ACCUMULATOR, ND, M, LIM, false, TX, TY, TZ, NT, WPE>,                                    \
   &launch_tile<ND, M, LIM, false, TX, TY, TZ, NT, WPE>,                                                         \
   #ND "d-" #M "-roles" #TX "x" #TY "x" #TZ "-nt" #NT "-w" #WPE SUFFIX}
#define AMRVAC_TILE(ND, M, TX, TY, TZ, NT, WPE) AMRVAC_TILE_ENTRY(ND, M, 0, TX, TY, TZ, NT, WPE, "")
#define AMRVAC_TILE_L(ND, M, TX, TY, TZ, NT, WPE) AMRVAC_TILE_ENTRY(ND, M, 1, TX, TY, TZ, NT, WPE, "-lim03")

static const StageVariant g_tile[] = {
    AMRVAC_TILE(2, false, 16, 8, 1, 256, 4),
    AMRVAC_TILE(2, false, 16, 16, 1, 512, 4),
    AMRVAC_TILE(2, true, 16, 16, 1, 512, 4),
    AMRVAC_TILE(3, false, 8, 8, 4, 512, 4),
    AMRVAC_TILE(3, true, 8, 8, 4, 512, 4),
    AMRVAC_TILE_L(2, false, 16, 16, 1, 512, 4),
    AMRVAC_TILE_L(2, true, 16, 16, 1, 512, 4),
    AMRVAC_TILE_L(3, false, 8, 8, 4, 512, 4),
    AMRVAC_TILE_L(3, true, 8, 8, 4, 512, 4),
};

const StageVariant* tile_variants(int* count) {
  *count = (int)(sizeof(g_tile) / sizeof(g_tile[0]));
  return g_tile;
}

}  // namespace amrvac
