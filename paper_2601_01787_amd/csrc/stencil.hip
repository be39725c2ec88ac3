// stencil.hip -- standalone steepest-direction pass (pmsz_directions and the
// directions used by verification): one wave per tile (wave_tiles.hpp), writing
// one direction byte per vertex.
#include "launch.hpp"
#include "wave_tiles.hpp"

namespace pmsz {

template <class T, int DIM>
__global__ __launch_bounds__(256) void k_dirs(const T* h, TileGeo G, uint8_t* dirs,
                                              int32_t run) {
  __shared__ WaveLds<T, DIM, KIND_DIRS_ANY> sm[4];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int32_t tile = (int32_t)first_tile(blockIdx.x, run) + wave;
  if (tile >= (int32_t)tile_count(G)) return;
  wave_tile<T, KIND_DIRS_ANY, false, false, DIM>(sm[wave], nullptr, h, (const T*)nullptr, dirs,
                                             nullptr, T(0), G, tile, nullptr, (T*)nullptr);
}

// Longer marches than the correction engine's on small fields (no frontier to
// keep fine), while still giving the chip several waves per compute unit.
static int dirs_chunk(int ndim, int64_t nx, int64_t ny, int64_t nz) {
  const int64_t cols = ndim == 3 ? ((nx + TX - 1) / TX) * ((ny + TY - 1) / TY) : (nx + RX - 1) / RX;
  const int64_t depth = ndim == 3 ? nz : ny;
  int64_t c = depth * cols / 4096;
  if (c < 2) c = 2;
  const int most = ndim == 3 ? kMaxChunk : kMaxChunk / 2;
  if (c > most) c = most;
  return (int)c;
}

template <class T>
static void launch_dirs_t(const void* h, const TileGeo& G, uint8_t* dirs, hipStream_t s) {
  const dim3 grid((unsigned)tile_blocks(tile_count(G)));
  const int32_t run = xcd_run(tile_count(G));
  if (G.ndim == 3)
    hipLaunchKernelGGL((k_dirs<T, 3>), grid, dim3(256), 0, s, (const T*)h, G, dirs, run);
  else
    hipLaunchKernelGGL((k_dirs<T, 2>), grid, dim3(256), 0, s, (const T*)h, G, dirs, run);
}

hipError_t launch_dirs(int dtype, const void* h, const Geo& g, uint8_t* dirs, hipStream_t s) {
  const TileGeo G = make_tile_geo(g.ndim, g.nx, g.ny, g.nz, dirs_chunk(g.ndim, g.nx, g.ny, g.nz));
  if (dtype == PMSZ_F32)
    launch_dirs_t<float>(h, G, dirs, s);
  else
    launch_dirs_t<double>(h, G, dirs, s);
  return hipGetLastError();
}

}  // namespace pmsz
