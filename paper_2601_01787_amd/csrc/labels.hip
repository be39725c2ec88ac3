// labels.hip -- ascending / descending segmentation labels (Sec. III-A:
// integral lines follow the steepest direction to an extremum; a segmentation
// groups the vertices that reach the same one), and the check of
// caller-supplied direction bytes.
//
// The steepest-direction pointers form a forest whose roots are the extrema
// (each pointer strictly climbs the index-tie-broken order, so there are no
// cycles).  A block resolves the pointers of one tile in LDS (k_labels_tile);
// paths that leave the tile are followed on over the direction bytes, and the
// few that do not end within kWalkHops steps are finished by pointer jumping
// over the labels (k_labels_finish).  Grids too thin for tiles start with every
// vertex at its neighbour (k_labels_init) and are finished in the same way.
#include "launch.hpp"

namespace pmsz {

// 1 when `code` names the vertex itself or a Freudenthal neighbour of (x, y, z)
// inside the grid: no code 8, no z bit in 2D, no step out of the box.
__device__ __forceinline__ bool code_valid(int code, int64_t x, int64_t y, int64_t z,
                                           const Geo& G) {
  if (code == 0) return true;
  if (code == 8) return false;
  const int m = code & 7;
  if (G.ndim == 2 && (m & 4)) return false;
  const int s = (code & 8) ? -1 : 1;
  const int64_t X = x + s * (m & 1), Y = y + s * ((m >> 1) & 1), Z = z + s * ((m >> 2) & 1);
  return X >= 0 && X < G.nx && Y >= 0 && Y < G.ny && Z >= 0 && Z < G.nz;
}

// Counts the direction bytes holding a code that is not valid for their vertex
// (either nibble).
__global__ __launch_bounds__(256) void k_check_dirs(const uint8_t* __restrict__ dirs, Geo G,
                                                    unsigned long long* bad) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  unsigned long long nb = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < G.n; i += stride) {
    const int d = dirs[i];
    const int64_t x = i % G.nx, y = (i / G.nx) % G.ny, z = i / G.sxy;
    nb += !(code_valid(d & 15, x, y, z, G) && code_valid(d >> 4, x, y, z, G));
  }
  nb = wave_sum(nb);
  if ((threadIdx.x & 63) == 0 && nb) atomicAdd(bad, nb);
}

// Step of a direction code, as one increment per axis.
struct Step {
  int32_t x, y, z;
};
__device__ __forceinline__ Step step_of(int code) {
  const int s = (code & 8) ? -1 : 1;
  return Step{s * (code & 1), s * ((code >> 1) & 1), s * ((code >> 2) & 1)};
}

// Labels of one tile, for each nibble of the direction bytes that is asked for
// (n_max into lmax, n_min into lmin).
//
// The tile's 16384 vertices (64 x 16 x 16; 64 x 256 in 2D) hold local ids of
// 14 bits, so the whole pointer graph of a tile is 32 KiB of LDS.  A vertex
// whose pointer stays in the tile starts at its neighbour's id, the others (the
// extrema, and the vertices whose pointer leaves the tile) at their own: these
// are the ends of the paths inside the tile.  Every pass moves an id
// kTileHops steps further up; ids read while others update them are ancestors
// too, so a path of length L is done after log(L) passes at the latest, and a
// pass that moves nothing ends the loop.  The path ends that leave the tile
// (at most the vertices on its faces) are listed, followed over the direction
// bytes in memory, and their results kept in LDS; then every vertex looks up
// its end and writes its label once.
//
// The pass reads a byte and writes two words per vertex; all gathers but the
// walks out of the tile hit LDS.  What bounds it is the instruction count per
// vertex and the walks (a lane of a byte gather costs about a cycle of its
// compute unit, a step in LDS a fifth of that), so ids are held as byte offsets
// into the id array (a step is one LDS read), the codes that leave the grid or
// the tile are 16-bit masks fixed per lane and row, index arithmetic comes from
// a table per row, and the walks are bounded: at 8, 16 or 32 steps, what a
// longer walk costs the tile pass the shorter one costs k_labels_finish (512^3:
// 1.93, 1.92, 1.91 ms in all).  Labels of a 512^3 field, both nibbles: 8.7 ms
// when every vertex jumped over the labels in memory, 1.9 ms now (16384 tiles,
// 1430 of 16384 paths end on a tile's face).
//
// Labels that are not final are stored as ~(vertex reached), and flags[nibble]
// is set.  Invalid codes are counted in *bad (the vertex becomes its own end),
// and so are cycles inside a tile: after the passes an id that is not its own
// end's, or an end that is neither an extremum nor leaves the tile.  A cycle
// through several tiles never settles in k_labels_finish.
constexpr int kTileVerts = 1 << 14;
constexpr int kTileThreads = 1024;
constexpr int kTilePer = kTileVerts / kTileThreads;
constexpr int kTileRows = kTileVerts / 64;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kTileHops = 4;
constexpr int kTilePasses = 10;  // 4^10 steps: more than any path inside a tile
constexpr int kWalkHops = 16;
// vertices with a face on the tile's surface, the most that can leave it
constexpr int kMaxExits = kTileVerts - 62 * 14 * 14;  // 3D; 2D has fewer
constexpr uint32_t kExit = 0x8000u;
// direction codes with a step down / up along x, y, z
constexpr uint32_t kDownX = 0xAA00u, kUpX = 0x00AAu, kDownY = 0xCC00u, kUpY = 0x00CCu,
                   kDownZ = 0xF000u, kUpZ = 0x00F0u;

template <int DIM>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(8))) void
k_labels_tile(const uint8_t* __restrict__ dirs_in, Geo G, int32_t tiles_x, int32_t tiles_y,
              int32_t* lmax, int32_t* lmin, unsigned int* flags, unsigned long long* bad) {
  constexpr int LY = DIM == 3 ? 16 : 256, LZ = DIM == 3 ? 16 : 1;
  __shared__ uint16_t s_up[kTileVerts];  // byte offset of the id a vertex points at
  __shared__ uint32_t s_code[kTileVerts / 4];  // direction bytes (0 outside the grid)
  __shared__ int32_t s_lab[kMaxExits];   // listed ends: the vertex, then what it reaches
  __shared__ int32_t s_row[kTileRows];   // grid index of each row's lane 0
  __shared__ int32_t s_step[16];         // offset of each direction code in s_up
  __shared__ int s_n;
  const gptr<const uint8_t> dirs = as_global(dirs_in);
  const int32_t nx = (int32_t)G.nx, ny = (int32_t)G.ny, nz = (int32_t)G.nz, sxy = (int32_t)G.sxy;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int32_t b = (int32_t)blockIdx.x;
  const int32_t x0 = (b % tiles_x) * 64, y0 = (b / tiles_x % tiles_y) * LY,
                z0 = (b / (tiles_x * tiles_y)) * LZ;
  auto row_y = [&](int r) { return DIM == 3 ? r & 15 : r; };
  auto row_z = [&](int r) { return DIM == 3 ? r >> 4 : 0; };
  // the tile's bytes, 16 to a thread (a quarter of a row)
  {
    const int r = tid >> 2, c = 16 * (tid & 3);
    const int32_t y = y0 + row_y(r), z = z0 + row_z(r);
    uint32_t w[4] = {0, 0, 0, 0};
    if (y < ny && z < nz && x0 + c < nx) {
      const int32_t at = nx * y + sxy * z + x0 + c;
      const int32_t have = nx - (x0 + c);
      if (have >= 16) {
        __builtin_memcpy(w, dirs_in + at, 16);
      } else {
        for (int j = 0; j < have; ++j) w[j >> 2] |= (uint32_t)dirs[at + j] << (8 * (j & 3));
      }
    }
    if (c == 0) s_row[r] = x0 + nx * y + sxy * z;  // (read for rows in the grid only)
#pragma unroll
    for (int j = 0; j < 4; ++j) s_code[4 * tid + j] = w[j];
  }
  if (tid < 16) {
    const int m = tid & 7;
    const int o = 2 * ((m & 1) + 64 * ((m >> 1) & 1) + 64 * LY * ((m >> 2) & 1));
    s_step[tid] = tid & 8 ? -o : o;
  }
  const int32_t x = x0 + lane;
  // codes that leave the grid / the tile from this lane (x), rows added below;
  // code 8 and, in 2D, the codes with a z step are never valid
  const uint32_t grid_x = (x == 0 ? kDownX : 0u) | (x >= nx - 1 ? kUpX : 0u) | 0x0100u |
                          (DIM == 2 ? kDownZ | kUpZ : 0u);
  const uint32_t tile_x = (lane == 0 ? kDownX : 0u) | (lane == 63 ? kUpX : 0u);
  unsigned nb = 0;
  const char* up = (const char*)s_up;
  auto id_at = [&](uint32_t o) { return (uint32_t)*(const uint16_t*)(up + o); };
  for (int which = 0; which < 2; ++which) {
    const gptr<int32_t> lab = as_global(which ? lmin : lmax);
    if (!(which ? lmin : lmax)) continue;
    if (tid == 0) s_n = 0;
    __syncthreads();  // the bytes and tables are there; the last nibble is done
    // this thread's vertices: lane x of rows wave, wave + 16, ...
    uint32_t ends = 0, outs = 0;  // bit k: vertex k ends a path here; ... leaving the tile
#pragma unroll 4
    for (int k = 0; k < kTilePer; ++k) {
      const int r = wave + kTileWaves * k;
      const int ly = row_y(r), lz = row_z(r);
      const int32_t y = y0 + ly, z = z0 + lz;
      const uint32_t grid = grid_x | (y == 0 ? kDownY : 0u) | (y >= ny - 1 ? kUpY : 0u) |
                            (z == 0 ? kDownZ : 0u) | (z >= nz - 1 ? kUpZ : 0u);
      const uint32_t tile = tile_x | (ly == 0 ? kDownY : 0u) | (ly == LY - 1 ? kUpY : 0u) |
                            (lz == 0 ? kDownZ : 0u) | (lz == LZ - 1 ? kUpZ : 0u);
      const uint32_t v = 2u * (uint32_t)(lane + 64 * r);
      const uint32_t code = (((const uint8_t*)s_code)[lane + 64 * r] >> (4 * which)) & 15u;
      const uint32_t wrong = (grid >> code) & 1u;
      const uint32_t out = ((tile & ~grid) >> code) & 1u;
      const uint32_t end = ((tile | grid | 1u) >> code) & 1u;
      nb += wrong;
      ends |= end << k;
      outs |= out << k;
      s_up[v >> 1] = (uint16_t)(end ? v : v + (uint32_t)s_step[code]);
    }
    __syncthreads();
    uint32_t todo = ~ends & ((1u << kTilePer) - 1u);  // bit k: vertex k has not reached its end
    bool moving = true;
    for (int pass = 0; pass < kTilePasses && moving; ++pass) {
#pragma unroll 4
      for (int k = 0; k < kTilePer; ++k) {
        if (!((todo >> k) & 1)) continue;
        const int v = lane + 64 * (wave + kTileWaves * k);
        uint32_t u = s_up[v], w = u;
#pragma unroll
        for (int h = 0; h < kTileHops; ++h) {
          w = u;
          u = id_at(u);
        }
        s_up[v] = (uint16_t)u;
        if (u == w) todo &= ~(1u << k);  // an end: its id is its own
      }
      moving = __syncthreads_or(todo != 0);
    }
    // cycles: a path without an end, or an end that is none
    nb += __popc(todo);
#pragma unroll 4
    for (int k = 0; k < kTilePer; ++k) {
      const int v = lane + 64 * (wave + kTileWaves * k);
      nb += s_up[v] == 2 * v && !((ends >> k) & 1);
    }
    // list the ends that leave the tile; their entries then hold their numbers
    int slot = 0;
    {
      const int mine = __popc(outs);
      int incl = mine;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
      }
      int base = 0;
      if (lane == 63 && incl) base = atomicAdd(&s_n, incl);
      slot = __shfl(base, 63, 64) + incl - mine;
    }
    __syncthreads();
    for (uint32_t m = outs; m; m &= m - 1u) {
      const int v = lane + 64 * (wave + kTileWaves * (__ffs(m) - 1));
      s_lab[slot] = v;
      s_up[v] = (uint16_t)(kExit | (uint32_t)slot);
      ++slot;
    }
    __syncthreads();
    // follow them over the direction bytes (each code is checked before it is
    // used: the bytes of other tiles may be invalid too)
    int open = 0;
    for (int e = tid; e < s_n; e += kTileThreads) {
      const int v = s_lab[e];
      int32_t X = x0 + (v & 63), Y = y0 + row_y(v >> 6), Z = z0 + row_z(v >> 6);
      int32_t at = s_row[v >> 6] + (v & 63);
      bool done = false;
      for (int h = 0; h <= kWalkHops; ++h) {
        const int code = (dirs[at] >> (4 * which)) & 15;
        const Step st = step_of(code);
        X += st.x;
        Y += st.y;
        Z += st.z;
        // an invalid byte ends the walk too (its own tile counts it)
        done = code == 0 || code == 8 || X < 0 || X >= nx || Y < 0 || Y >= ny || Z < 0 || Z >= nz;
        if (done || h == kWalkHops) break;
        at += st.x + nx * st.y + sxy * st.z;
      }
      s_lab[e] = done ? at : ~at;
      open |= !done;
    }
    if (__syncthreads_or(open) && tid == 0) flags[which] = 1u;
#pragma unroll 4
    for (int k = 0; k < kTilePer; ++k) {
      const int r = wave + kTileWaves * k;
      const uint32_t u = s_up[lane + 64 * r];
      const uint32_t e = (u & kExit) ? u : id_at(u);
      const int32_t l = (e & kExit) ? s_lab[e & (kExit - 1)]
                                    : s_row[e >> 7] + (int32_t)((e >> 1) & 63);
      if (x < nx && y0 + row_y(r) < ny && z0 + row_z(r) < nz) lab[s_row[r] + lane] = l;
    }
  }
  const unsigned long long all_bad = wave_sum(nb);
  if (lane == 0 && all_bad) atomicAdd(bad, all_bad);
}

// First pass over a grid that fills little of its tiles (labels_by_tiles): every
// vertex labels itself (the extrema, and invalid codes, whose bytes are counted in
// *bad) or, not final, its neighbour; k_labels_finish does the rest.
__global__ __launch_bounds__(256) void k_labels_init(const uint8_t* __restrict__ dirs, Geo G,
                                                     int32_t* lmax, int32_t* lmin,
                                                     unsigned int* flags, unsigned long long* bad) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  unsigned long long nb = 0;
  int open = 0;  // bit k: a label of nibble k is not final
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < G.n; i += stride) {
    const int a = dirs[i] & 15, d = dirs[i] >> 4;
    const int64_t x = i % G.nx, y = (i / G.nx) % G.ny, z = i / G.sxy;
    const bool va = code_valid(a, x, y, z, G), vd = code_valid(d, x, y, z, G);
    nb += !(va && vd);
    const bool oa = va && a, od = vd && d;
    if (lmax) lmax[i] = (int32_t)(oa ? ~(i + code_delta(a, G.nx, G.sxy)) : i);
    if (lmin) lmin[i] = (int32_t)(od ? ~(i + code_delta(d, G.nx, G.sxy)) : i);
    open |= (int)oa | ((int)od << 1);
  }
  const bool any_a = __ballot(open & 1) != 0ull, any_d = __ballot(open & 2) != 0ull;
  if ((threadIdx.x & 63) == 0) {
    if (lmax && any_a) flags[0] = 1u;
    if (lmin && any_d) flags[1] = 1u;
  }
  nb = wave_sum(nb);
  if ((threadIdx.x & 63) == 0 && nb) atomicAdd(bad, nb);
}

// Pass `pass` (from 1) over the labels that are not final, ~(vertex reached):
// each follows up to kLabelHops of them, in place (whatever a thread reads is
// an ancestor).  Skipped when the pass before left none; flags[2 pass +
// nibble] is set when this one leaves some.
__global__ __launch_bounds__(256) void k_labels_finish(int32_t* lmax, int32_t* lmin, int nibbles,
                                                       int64_t n, unsigned int* flags, int pass) {
  const int which = nibbles == 3 ? (int)blockIdx.y : nibbles - 1;
  if (flags[2 * (pass - 1) + which] == 0u) return;
  const gptr<int32_t> lab = as_global(which ? lmin : lmax);
  const int64_t stride = (int64_t)gridDim.x * 256;
  int open = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += stride) {
    int32_t l = lab[i];
    if (l >= 0) continue;
#pragma unroll 1
    for (int hop = 0; hop < kLabelHops && l < 0; ++hop) l = lab[~l];
    lab[i] = l;
    open |= l < 0;
  }
  if (__ballot(open) != 0ull && (threadIdx.x & 63) == 0) atomicOr(flags + 2 * pass + which, 1u);
}

static unsigned grid_for(int64_t items, int64_t most = 16384) {
  int64_t b = (items + 255) / 256;
  if (b < 1) b = 1;
  if (b > most) b = most;
  return (unsigned)b;
}

hipError_t launch_check_dirs(const uint8_t* dirs, const Geo& G, unsigned long long* bad,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_check_dirs, dim3(grid_for(G.n)), dim3(256), 0, s, dirs, G, bad);
  return hipGetLastError();
}

// Tiles of a grid.
struct LabelTiles {
  int64_t x, y, z;
};
static LabelTiles label_tiles(const Geo& G) {
  const int ly = G.ndim == 3 ? 16 : 256, lz = G.ndim == 3 ? 16 : 1;
  return LabelTiles{(G.nx + 63) / 64, (G.ny + ly - 1) / ly, (G.nz + lz - 1) / lz};
}

// A tile costs k_labels_tile about the same however few of its vertices lie in the
// grid, so grids that fill less than a quarter of their tiles start from
// k_labels_init.  Both ways, us, white noise / smooth: 4096 vertices per tile
// (2048 x 2048 x 4) 294 / 319 by tiles, 261 / 441 from k_labels_init; 2048
// (2048 x 2048 x 2) 274 / 324 and 136 / 272; 1024 (4 x 4 M in 2D) 1114 / 1177 and 250 /
// 383; 64 (2 x 2 x 2 M) 6909 / 7166 and 142 / 188.  8192 and more: tiles (1024 x
// 2048 x 8: 187 / 207 and 256 / 431).  A grid within one tile is one launch by
// tiles and five the other way (3 x 3 x 3: 55 and 64).
constexpr int64_t kTileShare = kTileVerts / 4;
static_assert(((1ll << 31) / kTileShare + 1) * kTileThreads < (1ll << 32),
              "a launch holds fewer than 2^32 threads");
bool labels_by_tiles(const Geo& G) {
  const LabelTiles t = label_tiles(G);
  const int64_t tiles = t.x * t.y * t.z;
  return tiles == 1 || G.n >= kTileShare * tiles;
}

hipError_t launch_labels_init(const uint8_t* dirs, const Geo& G, int32_t* lmax, int32_t* lmin,
                              unsigned int* flags, unsigned long long* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_labels_init, dim3(grid_for(G.n, 2048)), dim3(256), 0, s, dirs, G, lmax, lmin,
                     flags, bad);
  return hipGetLastError();
}

hipError_t launch_labels_tile(const uint8_t* dirs, const Geo& G, int32_t* lmax, int32_t* lmin,
                              unsigned int* flags, unsigned long long* bad, hipStream_t s) {
  const LabelTiles t = label_tiles(G);
  const dim3 grid((unsigned)(t.x * t.y * t.z));
  if (G.ndim == 3)
    hipLaunchKernelGGL(k_labels_tile<3>, grid, dim3(kTileThreads), 0, s, dirs, G, (int32_t)t.x,
                       (int32_t)t.y, lmax, lmin, flags, bad);
  else
    hipLaunchKernelGGL(k_labels_tile<2>, grid, dim3(kTileThreads), 0, s, dirs, G, (int32_t)t.x,
                       (int32_t)t.y, lmax, lmin, flags, bad);
  return hipGetLastError();
}

hipError_t launch_labels_finish(int32_t* lmax, int32_t* lmin, int64_t n, unsigned int* flags,
                                int pass, hipStream_t s) {
  const int nibbles = (lmax ? 1 : 0) | (lmin ? 2 : 0);
  // (2048 blocks fill the chip; most launches of a batch return at once)
  hipLaunchKernelGGL(k_labels_finish, dim3(grid_for(n, 2048), nibbles == 3 ? 2 : 1), dim3(256), 0, s,
                     lmax, lmin, nibbles, n, flags, pass);
  return hipGetLastError();
}

}  // namespace pmsz
