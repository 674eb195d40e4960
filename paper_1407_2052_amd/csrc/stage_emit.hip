// The code-emitting forms of the role-split stage kernel (stage_tile.h): the
// adjoint's forward recompute in 2D and 3D.
#include "stage_tile.h"

namespace amrvac {

#define AMRVAC_EMIT(ND, M, LIM, TX, TY, TZ, NT, WPE)                                                        \
  {ND, M, LIM, 0, TX, TY, TZ, NT, 1, WPE, LIM ? 2 : NG,                                                   \
   (const void*)&k_tile<ACCUMULATOR, ND, M, LIM, true, TX, TY, TZ, NT, WPE>,                              \
   &launch_tile<ND, M, LIM, true, TX, TY, TZ, NT, WPE>,                                                   \
   #ND "d-" #M "-roles" #TX "x" #TY "x" #TZ "-nt" #NT "-w" #WPE "-rec" #LIM "-emit"}

static const StageVariant g_tile_emit[] = {
    AMRVAC_EMIT(2, false, 0, 16, 16, 1, 512, 4),
    AMRVAC_EMIT(2, true, 0, 16, 16, 1, 512, 4),
    AMRVAC_EMIT(3, false, 0, 8, 8, 4, 512, 4),
    AMRVAC_EMIT(3, true, 0, 8, 8, 4, 512, 4),
    AMRVAC_EMIT(2, false, 1, 16, 16, 1, 512, 4),
    AMRVAC_EMIT(2, true, 1, 16, 16, 1, 512, 4),
    AMRVAC_EMIT(3, false, 1, 8, 8, 4, 512, 4),
    AMRVAC_EMIT(3, true, 1, 8, 8, 4, 512, 4),
};

const StageVariant* tile_emit_variant(int ndim, int mhd, int rec) {
  for (const StageVariant& v : g_tile_emit)
    if (v.ndim == ndim && v.mhd == mhd && v.rec == rec) return &v;
  return nullptr;
}

}  // namespace amrvac
