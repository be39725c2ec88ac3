// blocks.hip -- copies and ghost-layer exchange of a decomposed domain.
//
// Sec. IV-B cuts the domain into non-overlapping blocks, each extended by a
// one-vertex ghost layer, corrects every block on its own and then
// reconciles the copies of shared vertices by taking their minimum.  On one
// GPU the blocks are fields of one batched engine launch (each compares only
// its core); these kernels move values between the global field and the
// block copies.
//
// Cuts: along an axis of n vertices split into b blocks, block k owns
// [floor(k n / b), floor((k+1) n / b)); its copy spans one more vertex on
// each side that has a neighbour block, so a coordinate is held by its owner,
// by the block before when it is the owner's first vertex and by the block
// after when it is the owner's last (the host tabulates this per axis).
#include "launch.hpp"

namespace pmsz {

// One launch moves every block: block row blockIdx.y (and every gridDim.y-th
// after it), a wave per grid row of the copy.  (A launch per block and array left
// the chip part empty and divided twice per vertex: 2 x 2 x 2 blocks of 384^3
// binary32 took 0.37 ms to gather in 16 launches and 0.18 ms to scatter.)
template <class T>
__global__ __launch_bounds__(256) void k_blocks_gather(const T* f, const T* g, int64_t nx,
                                                       int64_t sxy, const BlockCopy* tab,
                                                       int32_t blocks) {
  const gptr<const T> fs = as_global(f), gs = as_global(g);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  for (int32_t id = blockIdx.y; id < blocks; id += gridDim.y) {
    const BlockCopy b = tab[id];
    const gptr<T> fd = as_global((T*)b.f), gd = as_global((T*)b.g);
    const int64_t rows = (int64_t)b.lny * b.lnz;
    for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < rows; r += (int64_t)gridDim.x * 4) {
      const int32_t ly = (int32_t)(r % b.lny), lz = (int32_t)(r / b.lny);
      const int64_t from = b.ox + nx * (b.oy + ly) + sxy * (b.oz + lz), to = (int64_t)b.lnx * r;
      for (int32_t x = lane; x < b.lnx; x += 64) {
        fd[to + x] = fs[from + x];
        gd[to + x] = gs[from + x];
      }
    }
  }
}

// Owner copy-back: the cores of the block copies into the global field.
template <class T>
__global__ __launch_bounds__(256) void k_cores_scatter(T* g, int32_t nx, int32_t ny, int32_t nz,
                                                       const BlockCopy* tab, int32_t blocks) {
  const gptr<T> gd = as_global(g);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  for (int32_t id = blockIdx.y; id < blocks; id += gridDim.y) {
    const BlockCopy b = tab[id];
    const gptr<const T> gs = as_global((const T*)b.g);
    const int32_t cx0 = b.ox > 0, cy0 = b.oy > 0, cz0 = b.oz > 0;
    const int32_t cx1 = b.lnx - (b.ox + b.lnx < nx), cy1 = b.lny - (b.oy + b.lny < ny),
                  cz1 = b.lnz - (b.oz + b.lnz < nz);
    const int32_t ry = cy1 - cy0;
    const int64_t rows = (int64_t)ry * (cz1 - cz0);
    for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < rows; r += (int64_t)gridDim.x * 4) {
      const int32_t ly = cy0 + (int32_t)(r % ry), lz = cz0 + (int32_t)(r / ry);
      const int64_t from = (int64_t)b.lnx * (ly + (int64_t)b.lny * lz);
      const int64_t to = b.ox + (int64_t)nx * (b.oy + ly + (int64_t)ny * (b.oz + lz));
      for (int32_t x = cx0 + lane; x < cx1; x += 64) gd[to + x] = gs[from + x];
    }
  }
}

// Grid of the two: a wave per row of the largest block, at most 64 blocks per
// compute unit in all.
static dim3 rows_grid(int32_t blocks, int64_t max_rows) {
  const int32_t y = blocks < 65535 ? blocks : 65535;
  int64_t x = (max_rows + 3) / 4;
  const int64_t most = 16384 / y > 1 ? 16384 / y : 1;
  return dim3((unsigned)(x < 1 ? 1 : x < most ? x : most), (unsigned)y);
}

hipError_t blocks_gather(int dtype, const void* f, const void* g, const Geo& G,
                         const BlockCopy* tab, int32_t blocks, int64_t max_rows, hipStream_t s) {
  const dim3 grid = rows_grid(blocks, max_rows);
  if (dtype == PMSZ_F32)
    hipLaunchKernelGGL(k_blocks_gather<float>, grid, dim3(256), 0, s, (const float*)f,
                       (const float*)g, G.nx, G.sxy, tab, blocks);
  else
    hipLaunchKernelGGL(k_blocks_gather<double>, grid, dim3(256), 0, s, (const double*)f,
                       (const double*)g, G.nx, G.sxy, tab, blocks);
  return hipGetLastError();
}

hipError_t blocks_scatter_cores(int dtype, const BlockCopy* tab, int32_t blocks, int64_t max_rows,
                                void* g, const Geo& G, hipStream_t s) {
  const dim3 grid = rows_grid(blocks, max_rows);
  if (dtype == PMSZ_F32)
    hipLaunchKernelGGL(k_cores_scatter<float>, grid, dim3(256), 0, s, (float*)g, (int32_t)G.nx,
                       (int32_t)G.ny, (int32_t)G.nz, tab, blocks);
  else
    hipLaunchKernelGGL(k_cores_scatter<double>, grid, dim3(256), 0, s, (double*)g, (int32_t)G.nx,
                       (int32_t)G.ny, (int32_t)G.nz, tab, blocks);
  return hipGetLastError();
}

// Ghost-layer exchange of the shared vertices: every vertex held by more
// than one block copy lies on a boundary layer (the two vertices either side
// of a cut) of some axis.  planes lists those layers as (axis, coordinate);
// a vertex is handled in the plane of the first axis on which it is shared.
// It takes the smallest of its copies (the later block in block order among
// equal values), and every copy whose bits differ is overwritten; *lowered
// counts the copies that were larger.  (The global field receives the owners'
// cores once, after the last exchange.)
// hold: per axis and coordinate, the (up to three, ascending, -1 padded)
// blocks along that axis whose copies hold it, for x, then y, then z.
template <class T>
__global__ __launch_bounds__(256) void k_exchange(int32_t nx, int32_t ny, int32_t nz,
                                                  int32_t bx, int32_t by,
                                                  const BlockCopy* __restrict__ tab,
                                                  const int32_t* __restrict__ hold,
                                                  const int32_t* __restrict__ planes,
                                                  int32_t n_planes, unsigned long long* lowered) {
  const gptr<const BlockCopy> tb = as_global(tab);
  const gptr<const int32_t> hx = as_global(hold);
  const gptr<const int32_t> hy = hx + 3 * (int64_t)nx;
  const gptr<const int32_t> hz = hy + 3 * (int64_t)ny;
  const gptr<const int32_t> pl = as_global(planes);
  unsigned long long low = 0;
  const int32_t dims[3] = {nx, ny, nz};
  for (int32_t q = 0; q < n_planes; ++q) {
    const int32_t axis = pl[2 * q], coord = pl[2 * q + 1];
    // the plane's two other axes: u varies fastest
    const int32_t ua = axis == 0 ? 1 : 0, va = axis == 2 ? 1 : 2;
    const int64_t nu = dims[ua], nv = dims[va];
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < nu * nv;
         e += (int64_t)gridDim.x * 256) {
      int32_t xyz[3];
      xyz[axis] = coord;
      xyz[ua] = (int32_t)(e % nu);
      xyz[va] = (int32_t)(e / nu);
      const int32_t x = xyz[0], y = xyz[1], z = xyz[2];
      int32_t kx[3], ky[3], kz[3];
      for (int j = 0; j < 3; ++j) {
        kx[j] = hx[3 * (int64_t)x + j];
        ky[j] = hy[3 * (int64_t)y + j];
        kz[j] = hz[3 * (int64_t)z + j];
      }
      // shared on an earlier axis: that axis' plane handles it
      if (axis >= 1 && kx[1] >= 0) continue;
      if (axis == 2 && ky[1] >= 0) continue;
      T m = T(0);
      bool first = true;
      for (int c = 0; c < 3 && kz[c] >= 0; ++c)
        for (int b = 0; b < 3 && ky[b] >= 0; ++b)
          for (int a = 0; a < 3 && kx[a] >= 0; ++a) {
            const int32_t id = kx[a] + bx * (ky[b] + by * kz[c]);
            const int64_t li = (x - tb[id].ox) +
                               (int64_t)tb[id].lnx * ((y - tb[id].oy) + (int64_t)tb[id].lny * (z - tb[id].oz));
            const T cv = as_global((const T*)tb[id].g)[li];
            m = (first || !(m < cv)) ? cv : m;
            first = false;
          }
      for (int c = 0; c < 3 && kz[c] >= 0; ++c)
        for (int b = 0; b < 3 && ky[b] >= 0; ++b)
          for (int a = 0; a < 3 && kx[a] >= 0; ++a) {
            const int32_t id = kx[a] + bx * (ky[b] + by * kz[c]);
            const int64_t li = (x - tb[id].ox) +
                               (int64_t)tb[id].lnx * ((y - tb[id].oy) + (int64_t)tb[id].lny * (z - tb[id].oz));
            const gptr<T> p = as_global((T*)tb[id].g) + li;
            const T cv = *p;
            low += cv > m ? 1u : 0u;
            if (FP<T>::bits(cv) != FP<T>::bits(m)) *p = m;
          }
    }
  }
  const unsigned long long w = wave_sum(low);
  if ((threadIdx.x & 63) == 0 && w)
    __hip_atomic_fetch_add(as_global(lowered), w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

hipError_t blocks_exchange(int dtype, const Geo& G, const int32_t nb[3],
                           const BlockCopy* tab, const int32_t* hold, const int32_t* planes,
                           int32_t n_planes, int64_t max_plane, unsigned long long* lowered,
                           hipStream_t s) {
  if (n_planes == 0) return hipSuccess;
  int64_t grid = (max_plane + 255) / 256;
  if (grid > 4096) grid = 4096;
  if (grid < 1) grid = 1;
  if (dtype == PMSZ_F32)
    hipLaunchKernelGGL(k_exchange<float>, dim3((unsigned)grid), dim3(256), 0, s,
                       (int32_t)G.nx, (int32_t)G.ny, (int32_t)G.nz, nb[0], nb[1], tab, hold,
                       planes, n_planes, lowered);
  else
    hipLaunchKernelGGL(k_exchange<double>, dim3((unsigned)grid), dim3(256), 0, s,
                       (int32_t)G.nx, (int32_t)G.ny, (int32_t)G.nz, nb[0], nb[1], tab, hold,
                       planes, n_planes, lowered);
  return hipGetLastError();
}

}  // namespace pmsz
