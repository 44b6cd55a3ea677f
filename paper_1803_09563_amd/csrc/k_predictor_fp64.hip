// Launches of the FP64 predictor.
#include "predictor_async.h"

namespace evp {

// Tiles: 32 x 8 cells (two blocks per CU by their LDS) or 16 x 8 (three).  The wide tile reads less
// halo per cell and is the faster one where both fill the chip alike (128^3 Saramito: 175 against
// 179 us; 512x256x256: 2550 against 2900 us); the narrow one wastes fewer columns of widths that are
// no multiple of 32 and gives small grids more blocks (48^3: 21 against 27 us; 32^3: 12 against 14).  A
// plane of the chip takes 1.3 times as long in wide tiles (512 x 256 cells against 768 x 128).  FENE-P
// stages its factor too, with which two wide tiles do not fit a CU's LDS: always narrow (512x256x256: 2710
// against 2965 us; 96x400x64: 230 against 260).
hipError_t launch_predictor_fp64(const Batch& b, int nx, int ny, int nz, bool freeze, hipStream_t s, int model, bool rk3, bool houc)
{
    const int fz = freeze ? 1 : 0;
    // the tile is chosen by the grid alone, the chunk by the batch
    const long long nw = (nx + 31) / 32 * ((ny + 7) / 8), nn = (nx + 15) / 16 * ((ny + 7) / 8);
    if (model != EVP_FENE_P && 1.3 * chunk_planes(nw, nz, 512, 1.0).cost <= chunk_planes(nn, nz, 768, 1.0).cost)
        return launch_tile<double, 2, 32, 8>(b, nx, ny, nz, chunk_planes(nw * b.count, nz, 512, 1.0).kc, fz, s, model, rk3, houc);
    return launch_tile<double, 2, 16, 8>(b, nx, ny, nz, chunk_planes(nn * b.count, nz, 768, 1.0).kc, fz, s, model, rk3, houc);
}

}  // namespace evp
