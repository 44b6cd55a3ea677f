// Launches of the predictor in the mixed form (FP32 stresses).
#include "predictor_async.h"

namespace evp {

// Tiles: 32 x 8 cells, three blocks per CU (FENE-P: two, by its registers), or 16 x 8, four.  The wide
// tile reads less halo per cell and is the faster one on a full chip (128^3 Saramito: 104 against 127 us;
// 512x256x256: 1462 against 1880; 256x128x128 FENE-P: 222 against 263; 64^3: 23.0 against 24.2); the narrow
// one has less work in its longest block and wastes fewer columns, which counts while the chip is not full
// (8^3: 10.7 against 12.2 us; 48^3: 16.4 against 20.3; 80^3: 36.7 against 41.8).  A plane of a full chip
// takes 1.12 times as long in wide tiles (768 x 256 cells against 1024 x 128), FENE-P 0.85 (512 x 256), and
// 0.5 and 0.42 of it where a CU is nearly empty (fitted to such sizes).  Rows of a number of cells that is
// no multiple of 4 are staged value by value, in narrow tiles.  Tile and chunk change no operation of a
// cell: a grid's numbers are the same alone and in any batch.
hipError_t launch_predictor_mixed(const Batch& b, int nx, int ny, int nz, bool freeze, hipStream_t s, int model, bool rk3, bool houc)
{
    const int fz = freeze ? 1 : 0;
    const long long nw = (long long)((nx + 31) / 32) * ((ny + 7) / 8) * b.count, nn = (long long)((nx + 15) / 16) * ((ny + 7) / 8) * b.count;
    const bool fene = model == EVP_FENE_P;
    const Chunk narrow = chunk_planes(nn, nz, 1024, 0.42), wide = chunk_planes(nw, nz, fene ? 512 : 768, 0.5);
    if (nx % 4 != 0) return launch_tile<float, 1, 16, 8>(b, nx, ny, nz, narrow.kc, fz, s, model, rk3, houc);
    if ((fene ? 0.85 : 1.12) * wide.cost <= narrow.cost) return launch_tile<float, 4, 32, 8>(b, nx, ny, nz, wide.kc, fz, s, model, rk3, houc);
    return launch_tile<float, 4, 16, 8>(b, nx, ny, nz, narrow.kc, fz, s, model, rk3, houc);
}

}  // namespace evp
