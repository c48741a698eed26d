// Products whose operands lie beside the 16-byte grid, by plain addresses: the kernels of gemm_mfma.h a second time, in a code
// object of their own.
#include "gemm_mfma.h"

void launch_tile_off_grid(int epi, bool hd128, GemmArgs& a, int tile, hipStream_t s) {
  switch (epi) {
    case ME_STORE: launch_tile_of<ME_STORE, false, false>(a, tile, s); break;
    case ME_RESIDUAL: launch_tile_of<ME_RESIDUAL, false, false>(a, tile, s); break;
    case ME_SWIGLU: launch_tile_of<ME_SWIGLU, false, false>(a, tile, s); break;
    case ME_LMHEAD: launch_tile_of<ME_LMHEAD, false, false>(a, tile, s); break;
    case ME_QKV_ROPE:
      if (hd128) launch_tile_of<ME_QKV_ROPE, true, false>(a, tile, s);
      else launch_tile_of<ME_QKV_ROPE, false, false>(a, tile, s);
      break;
  }
}
