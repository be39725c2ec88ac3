// wave_tiles.hpp -- the steepest-direction stencil with one tile per wave
// (internal): the plain kernels that compute directions and sweep tiles.
//
// The upper box of a vertex i, i + {0,1}^d, is the lower box of the vertex
// i + (1,..,1): both are the lattice box with its low corner at i.  A tile of
// tiles.hpp reduces the two separately; here every box is reduced once and
// serves both vertices, so a 3D vertex costs about five pair merges per
// direction instead of nine.  The passes are bound by the rate at which
// vector instructions issue, and this is what cuts them: directions of a 512^3
// binary32 field of white noise 64 -> 44 per vertex, 0.297 -> 0.224 ms; 8192 x 16384
// in 2D 0.161 -> 0.139 ms (4.8 TB/s).
//
// A wave marches a tile alone, without block barriers: its lanes are the
// tile's columns along x (64 x 4 rows in 3D, one column and four rows per lane;
// 256 wide in 2D, four columns per lane), the values of the lines it needs are in
// registers, and x neighbours and the boxes of the lane to the left come by
// DPP lane shifts.  What a lane shift cannot give (the values right of the
// tile, and the boxes whose corner is the column left of it) is gathered before the
// march into LDS, where every step reads it as the shift's fill value.
//
// Box positions.  A box's extremes carry the position of the winner in the box
// (x, y, z bits).  The bits of y and z hold the parity of the winner's line and
// plane instead of its place in the pair, so that a line's code is the same in
// both boxes that use it and no merge has to set a bit; one exclusive or per
// use turns parities into positions.  The minimum's x bit is inverted (the
// first merge, of two values, takes both extremes from one comparison).
//
// Absent neighbours: coordinates outside the grid are clamped, so that the
// box sees the boundary line twice.  Where both halves of a merge are the same
// the maximum takes the second and the minimum the first, and the bit of that axis
// is then forced to the half that exists; the code names the same vertex.
#pragma once

#include "tiles.hpp"

namespace pmsz {

// A constant as an argument.
template <int N>
struct Int {
  static constexpr int value = N;
};

// Value of the lane to the right (DPP wave_shl:1; lane 63 takes `fill`) or to
// the left (wave_shr:1; lane 0 takes `fill`).
template <int CTRL>
__device__ __forceinline__ uint32_t lane_shift(uint32_t v, uint32_t fill) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)fill, (int)v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v, float fill) {
  return __uint_as_float(lane_shift<CTRL>(__float_as_uint(v), __float_as_uint(fill)));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v, double fill) {
  const unsigned long long a = (unsigned long long)__double_as_longlong(v),
                           b = (unsigned long long)__double_as_longlong(fill);
  const uint32_t lo = lane_shift<CTRL>((uint32_t)a, (uint32_t)b);
  const uint32_t hi = lane_shift<CTRL>((uint32_t)(a >> 32), (uint32_t)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
constexpr int kFromRight = 0x130, kFromLeft = 0x138;

// The larger / smaller of two values, given the comparison that decided it: a
// select in binary32, the one-instruction maximum in binary64 (a select of
// two registers takes two).
__device__ __forceinline__ float higher(bool b, float B, float A) { return b ? B : A; }
__device__ __forceinline__ float lower(bool b, float B, float A) { return b ? B : A; }
__device__ __forceinline__ double higher(bool, double B, double A) { return __builtin_fmax(A, B); }
__device__ __forceinline__ double lower(bool, double B, double A) { return __builtin_fmin(A, B); }

// Pair of x neighbours (A left of B): the maximum's code, x bit set when B is
// taken; the minimum's is the same with the x bit inverted.
template <class T>
struct XPair {
  T hi, lo;
  uint32_t c;
};
template <class T>
__device__ __forceinline__ XPair<T> x_pair(T A, T B, uint32_t tag) {
  const bool b = B >= A;
  return XPair<T>{higher(b, B, A), lower(b, A, B), b ? (tag | 1u) : tag};
}
// Box extremes with raw position codes.
template <class T>
struct Box {
  T hi, lo;
  uint32_t ca, cd;
};
// Merge of disjoint halves, every vertex of B above every vertex of A in index.
template <class T>
__device__ __forceinline__ Box<T> box_merge(const Box<T>& A, const Box<T>& B) {
  const bool bh = B.hi >= A.hi, bl = B.lo < A.lo;
  return Box<T>{higher(bh, B.hi, A.hi), lower(bl, B.lo, A.lo), bh ? B.ca : A.ca,
                bl ? B.cd : A.cd};
}
template <class T>
__device__ __forceinline__ Box<T> box_of_pair(const XPair<T>& p) {
  return Box<T>{p.hi, p.lo, p.c, p.c};
}

// Code words hold the maximum's code in byte 0 and the minimum's in byte 1.
template <class T>
__device__ __forceinline__ uint32_t code_word(const Box<T>& b) {
  return b.ca | (b.cd << 8);  // minimum's x bit still inverted
}
// As the upper box of its corner: positions are the direction codes.  par: the
// parities of the corner's line and plane; keep: the bits of the axes along
// which the corner has a neighbour.
__device__ __forceinline__ uint32_t upper_codes(uint32_t w, uint32_t par, uint32_t keep) {
  return (w ^ (0x0100u | par | (par << 8))) & keep;
}
// As the lower box of the opposite corner: position m lies m ^ full steps back,
// code 8 | (m ^ full), or 0 for the corner itself; looked up by byte permute.
constexpr uint64_t lower_table(uint32_t par, uint32_t full) {
  uint64_t t = 0;
  for (uint32_t raw = 0; raw < 8; ++raw) {
    const uint32_t k = ((raw ^ par) & full) ^ full;
    t |= (uint64_t)(k ? (8u | k) : 0u) << (8 * raw);
  }
  return t;
}
template <uint32_t PAR, uint32_t FULL>
__device__ __forceinline__ uint32_t lower_codes(uint32_t w) {
  constexpr uint64_t t = lower_table(PAR, FULL);
  // bytes 2 and 3 of the selector: the constant zero
  return __builtin_amdgcn_perm((uint32_t)(t >> 32), (uint32_t)t, w ^ 0x0C0C0100u);
}
// Lower-box codes of a box whose position (no parities) is known: the axes in
// `gone` have no neighbour below.
__device__ __forceinline__ uint32_t lower_codes_at(uint32_t ca, uint32_t cd, uint32_t full,
                                                   uint32_t gone) {
  const uint32_t ka = (ca ^ full) & ~gone, kd = (cd ^ full) & ~gone;
  return (ka ? 8u | ka : 0u) | ((kd ? 8u | kd : 0u) << 8);
}

// What the lower box leaves for its vertex: extremes and codes.
template <class T>
struct Low {
  T hi, lo;
  uint32_t w;
};
// Direction byte of a vertex from its two boxes (every vertex of the lower box
// has an index at most, of the upper box at least, the vertex's own).
template <class T>
__device__ __forceinline__ uint32_t dir_byte(const Low<T>& L, const Box<T>& U, uint32_t wu) {
  const bool bh = U.hi >= L.hi, bl = U.lo < L.lo;
  const uint32_t a = bh ? wu : L.w, d = bl ? wu : L.w;
  return (a & 15u) | (d >> 4);
}

// LDS of one wave: the values right of the tile and the lower boxes whose
// corner is the column left of it, per plane (3D, four lines) or per row (2D).
template <class T>
struct alignas(16) Edge3 {
  T right[TY + 2];
  T hi[TY], lo[TY];
  uint32_t w[TY];
};
template <class T>
struct alignas(16) Edge2 {
  T right, hi, lo;
  uint32_t w;
};
template <class T, int DIM>
struct EdgeOf {
  using type = Edge3<T>;
};
template <class T>
struct EdgeOf<T, 2> {
  using type = Edge2<T>;
};
// 3D edges are gathered kEdgeGroup planes at a time, two planes ahead of their use,
// when the march (and its neighbours') load the same lines.
constexpr int kEdgeGroup = 4;
template <class T, int DIM, int KIND>
struct WaveLds {
  // of h and, where the directions of f are made too, of f
  // (2D: one more than a tile's rows, the march runs them in pairs)
  typename EdgeOf<T, DIM>::type
      edge[KIND == KIND_FIRST ? 2 : 1][DIM == 3 ? kEdgeGroup : kMaxChunk + 3];
  static constexpr bool FLAGS = KIND != KIND_DIRS && KIND != KIND_DIRS_ANY;
  uint32_t flags[FLAGS ? (DIM == 3 ? (kMaxChunk + 2) * (TY + 2) * kFlagW3
                                   : (kMaxChunk + 2) * kFlagW2)
                       : 1];
};

// Buffer accesses: a uniform 64-bit base per plane (the resource), a scalar
// byte offset per line and a 32-bit byte offset per lane, so a load costs no vector
// arithmetic.  A store at kNoStore, past the resource's end, is dropped, so
// that lanes outside the grid need no branch: a store in a branch makes the
// compiler's wait for older loads assume that it did not run, and the march
// would then wait for the planes ahead too.
using Rsrc = __amdgpu_buffer_rsrc_t;
constexpr uint32_t kNoStore = 0xFFFFFFFFu;
__device__ __forceinline__ Rsrc rsrc_at(gptr<const void> p, bool on = true) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, on ? 0xFFFFFFFEu : 0u, 0x00020000);
}
typedef uint32_t U32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t U32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void buf_load(Rsrc r, uint32_t lane_off, uint32_t line_off, float& v) {
  v = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, lane_off, line_off, 0));
}
__device__ __forceinline__ void buf_load(Rsrc r, uint32_t lane_off, uint32_t line_off, double& v) {
  const U32x2 x = __builtin_amdgcn_raw_buffer_load_b64(r, lane_off, line_off, 0);
  v = __longlong_as_double((long long)(((unsigned long long)x.y << 32) | x.x));
}
__device__ __forceinline__ void buf_load4(Rsrc r, uint32_t lane_off, float* v) {
  const U32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, 0, 0);
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = __uint_as_float(x[j]);
}
__device__ __forceinline__ void buf_load4(Rsrc r, uint32_t lane_off, double* v) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const U32x4 x = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off + 16u * h, 0, 0);
    v[2 * h] = __longlong_as_double((long long)(((unsigned long long)x.y << 32) | x.x));
    v[2 * h + 1] = __longlong_as_double((long long)(((unsigned long long)x.w << 32) | x.z));
  }
}

__device__ __forceinline__ void buf_store(Rsrc r, uint32_t lane_off, uint32_t line_off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, lane_off, line_off, 0);
}
__device__ __forceinline__ void buf_store(Rsrc r, uint32_t lane_off, uint32_t line_off, double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const U32x2 x = {(uint32_t)b, (uint32_t)(b >> 32)};
  __builtin_amdgcn_raw_buffer_store_b64(x, r, lane_off, line_off, 0);
}
__device__ __forceinline__ void buf_store4(Rsrc r, uint32_t lane_off, const float* v) {
  U32x4 x;
#pragma unroll
  for (int j = 0; j < 4; ++j) x[j] = __float_as_uint(v[j]);
  __builtin_amdgcn_raw_buffer_store_b128(x, r, lane_off, 0, 0);
}
__device__ __forceinline__ void buf_store4(Rsrc r, uint32_t lane_off, const double* v) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned long long a = (unsigned long long)__double_as_longlong(v[2 * h]),
                             b = (unsigned long long)__double_as_longlong(v[2 * h + 1]);
    const U32x4 x = {(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
    __builtin_amdgcn_raw_buffer_store_b128(x, r, lane_off + 16u * h, 0, 0);
  }
}

// LDS writes of the wave's lanes are visible to its other lanes (they execute
// in order; the compiler must keep that order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront", "local");
}

// flush_rows of one wave.
template <int W, class RowStart>
__device__ __forceinline__ void wave_flush_rows(uint32_t* flags, int32_t rows, RowStart row_start,
                                                gptr<uint32_t> bm) {
  for (int r = threadIdx.x & 63; r < rows; r += 64) {
    uint32_t L[W];
    uint32_t any = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      L[j] = flags[r * W + j];
      any |= L[j];
    }
    if (!any) continue;
#pragma unroll
    for (int j = 0; j < W; ++j) flags[r * W + j] = 0u;
    const int32_t gb0 = row_start(r);
    const int32_t w0 = gb0 >> 5;  // arithmetic shift: floor
    const uint32_t sh = (uint32_t)gb0 & 31u;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      uint32_t w = L[j] << sh;
      if (j > 0 && sh) w |= L[j - 1] >> (32u - sh);
      if (w)
        __hip_atomic_fetch_or(bm + (w0 + j), w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Order of the tiles: block b runs on XCD b mod 8, and runs of kXcdRun blocks'
// tiles go to one XCD, so that the lines that neighbouring tiles share are in its
// L2 (directions of 512^3 in binary32: 1.14 GB read from memory in launch order,
// 0.63 GB in this one).  Returns the first tile of virtual block vb, for blocks of
// four tiles; virtual blocks run to tile_blocks(tiles).
constexpr int32_t kXcds = 8, kXcdRun = 32;
__host__ __device__ inline int32_t xcd_run(int64_t tiles) {
  int32_t run = kXcdRun;
  while (run > 1 && (tiles + 3) / 4 < (int64_t)kXcds * run) run /= 2;
  return run;
}
__host__ __device__ inline int64_t tile_blocks(int64_t tiles) {
  const int64_t span = (int64_t)kXcds * xcd_run(tiles);
  return ((tiles + 3) / 4 + span - 1) / span * span;
}
__device__ __forceinline__ int64_t first_tile(int64_t vb, int32_t run) {
  const int64_t span = (int64_t)kXcds * run;  // a power of two
  const int64_t in = vb & (span - 1);
  return 4 * ((vb & ~(span - 1)) + (in & (kXcds - 1)) * run + (in >> 3));
}

// Part `part` of `parts` of a tile's planes or rows [at, at + chunk), which end at n.
struct Span {
  int32_t a, b;
};
__host__ __device__ inline Span part_of(int32_t at, int32_t chunk, int32_t n, int32_t part,
                                        int32_t parts) {
  const int32_t each = parts == 1 ? chunk : (chunk + parts - 1) / parts;
  const int32_t end = tile_end(at, chunk, n), off = part * each;
  if (off >= end - at) return Span{end, end};
  return Span{at + off, tile_end(at + off, each, end)};
}

// Counts of a tile, per lane.
struct LaneCounts {
  unsigned mism, nf, nb;
};

// Mismatches of one vertex: `o` its direction byte, `d` that of f; flags go to
// the wave's rows (flag_targets of tiles.hpp).
template <class T, bool PROP>
__device__ __forceinline__ unsigned flag_mismatch(uint32_t o, uint32_t d, int32_t bi, int32_t v,
                                                  const TileGeo& G, uint32_t* flags,
                                                  const int32_t* fdelta, void* prop,
                                                  gptr<const T> g, T lo) {
  return flag_targets<T>(bi, v, (int)(o & 15u), (int)(o >> 4), (int)(d & 15u), (int)(d >> 4), G,
                         flags, fdelta, PROP ? prop : nullptr, g, lo);
}

// Direction bytes of a wave's tile by the merges of tiles.hpp, each box reduced for
// its own vertex.  They define the bytes where values are NaN: such a vertex points to
// itself both ways, and every other one to itself, to a NaN or beyond its own value,
// so that the pointers stay a forest.  The marches below share a box between two
// vertices and keep neither, so a wave that meets a NaN there (an unordered pair costs
// one comparison) makes its tile again this way.  512^3 binary32: 208 us without NaN,
// 207 without the comparisons; 438 us with a NaN in every tile, 246 in the block
// march that reduced every box for its own vertex.
template <class T>
__device__ __forceinline__ T nan_of() {
  return T(__builtin_nan(""));
}
template <class T>
__device__ __forceinline__ void wave_dirs_any3(gptr<const T> h, gptr<uint8_t> dirs,
                                               const TileGeo& G, int32_t x0, int32_t y0,
                                               int32_t z0, int32_t z1) {
  constexpr int R = TY, V = TY + 2;
  const int lane = threadIdx.x & 63;
  const int32_t X = x0 + lane, xc = X < G.nx ? X : G.nx - 1;
  // lanes 0..5 hold the values left of the tile's lines, 8..13 those right of them
  const int er = lane & 7;
  const bool e_right = lane & 8;
  const bool e_in = lane < 16 && er < V && (er > 0 || y0 > 0) && er - 1 < G.ny - y0 &&
                    (e_right ? G.nx - x0 > TX : x0 > 0);
  const int64_t e_at = (int64_t)G.nx * clamp_step(y0, er - 1, G.ny) +
                       clamp_step(x0, e_right ? TX : -1, G.nx);
  struct Plane {
    T c[V], e;
  };
  // (one plane ahead; what lies outside the grid is read inside it and then absent)
  auto fetch = [&](int32_t q, Plane& S) {
    const gptr<const T> h_p = h + (int64_t)G.sxy * clamp_step(z0, q - 1, G.nz);
#pragma unroll
    for (int k = 0; k < V; ++k) S.c[k] = h_p[(int64_t)G.nx * clamp_step(y0, k - 1, G.ny) + xc];
    S.e = h_p[e_at];
  };
  Ext<T> up[R], dn[R], low[R];  // squares of the last plane; lower boxes of its vertices
  Plane now, next;
  fetch(0, next);
  for (int32_t q = 0; q < z1 - z0 + 2; ++q) {
    now = next;
    fetch(q + 1, next);
    const int32_t p = z0 - 1 + q;
    const bool plane = p >= 0 && p < G.nz;
    const T e = plane && e_in ? now.e : nan_of<T>();
    T c[V], l[V], r[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
      c[k] = plane && (k > 0 || y0 > 0) && k - 1 < G.ny - y0 && X < G.nx ? now.c[k] : nan_of<T>();
      l[k] = lane_shift<kFromLeft>(c[k], __shfl(e, k, 64));
      r[k] = lane_shift<kFromRight>(c[k], __shfl(e, 8 + k, 64));
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const Ext<T> u = merge_up(merge_up(ext_of(c[k + 1], 0), ext_of(r[k + 1], 1)),
                                merge_up(ext_of(c[k + 2], 2), ext_of(r[k + 2], 3)));
      const Ext<T> d = merge_dn(merge_dn(ext_of(l[k], 11), ext_of(c[k], 10)),
                                merge_dn(ext_of(l[k + 1], 9), ext_of(c[k + 1], 0)));
      if (q > 1 && X < G.nx && y0 + k < G.ny) {
        const Ext<T> b = merge_up(low[k], merge_up(up[k], with_bits(u, 4)));
        dirs[(int64_t)G.sxy * (p - 1) + (int64_t)G.nx * (y0 + k) + X] =
            (uint8_t)(b.ca | (b.cd << 4));
      }
      if (q > 0) low[k] = merge_dn(with_bits(dn[k], 12), d);
      up[k] = u;
      dn[k] = d;
    }
  }
}
// The same for a 2D tile.
template <class T>
__device__ __forceinline__ void wave_dirs_any2(gptr<const T> h, gptr<uint8_t> dirs,
                                               const TileGeo& G, int32_t x0, int32_t y0,
                                               int32_t y1) {
  constexpr int C = 4;
  const int32_t X = x0 + C * (int32_t)(threadIdx.x & 63);
  struct Row {
    T c[C], l, r;
  };
  auto fetch = [&](int32_t q, Row& S) {
    const gptr<const T> h_p = h + (int64_t)G.nx * clamp_step(y0, q - 1, G.ny);
#pragma unroll
    for (int j = 0; j < C; ++j) S.c[j] = h_p[X + j < G.nx ? X + j : G.nx - 1];
    S.l = h_p[x0 ? x0 - 1 : 0];
    S.r = h_p[clamp_step(x0, RX, G.nx)];
  };
  Ext<T> up[C], dn[C], low[C];  // pairs of the last row; lower boxes of its vertices
  Row now, next;
  fetch(0, next);
  for (int32_t q = 0; q < y1 - y0 + 2; ++q) {
    now = next;
    fetch(q + 1, next);
    const int32_t p = y0 - 1 + q;
    const bool row = p >= 0 && p < G.ny;
    T c[C + 2];  // from the column left of the lane's
#pragma unroll
    for (int j = 0; j < C; ++j) c[j + 1] = row && X + j < G.nx ? now.c[j] : nan_of<T>();
    c[0] = lane_shift<kFromLeft>(c[C], row && x0 > 0 ? now.l : nan_of<T>());
    c[C + 1] = lane_shift<kFromRight>(c[1], row && G.nx - x0 > RX ? now.r : nan_of<T>());
#pragma unroll
    for (int j = 0; j < C; ++j) {
      const Ext<T> u = merge_up(ext_of(c[j + 1], 0), ext_of(c[j + 2], 1));
      const Ext<T> d = merge_dn(ext_of(c[j], 9), ext_of(c[j + 1], 0));
      if (q > 1 && X + j < G.nx) {
        const Ext<T> b = merge_up(low[j], merge_up(up[j], with_bits(u, 2)));
        dirs[(int64_t)G.nx * (p - 1) + X + j] = (uint8_t)(b.ca | (b.cd << 4));
      }
      if (q > 0) low[j] = merge_dn(with_bits(dn[j], 10), d);
      up[j] = u;
      dn[j] = d;
    }
  }
}

// One 3D tile (tiles.hpp's 64 x 4 x chunk) on one wave.  Arguments as tile3;
// copy_to (COPY): the tile's values of h go there too (lanes and lines outside
// the grid repeat the last ones inside).
// The march visits the planes z0-1 .. z1; the step of plane p completes the
// boxes between planes p-1 and p, finishes the vertices of plane p-1 and leaves
// the boxes as lower boxes of plane p.  Loads run two planes ahead.
template <class T, int KIND, bool PROP, bool COPY, class LDS>
__device__ __forceinline__ LaneCounts wave_tile3(LDS& sm, const int32_t* fdelta, const T* h_in,
                                                 const T* f_in, uint8_t* dirs_in, uint32_t* bm_in,
                                                 T xi, const TileGeo& G_in, int32_t tile,
                                                 void* prop_in, T* copy_in, int32_t part,
                                                 int32_t parts) {
  const gptr<T> copy_to = as_global(uniform_ptr(copy_in));
  const TileGeo G = uniform_geo(G_in);
  void* const prop = PROP ? uniform_ptr(prop_in) : nullptr;
  const gptr<const T> h = as_global((const T*)uniform_ptr(h_in));
  const gptr<const T> f = as_global((const T*)uniform_ptr(f_in));
  const gptr<uint8_t> dirs = as_global(uniform_ptr(dirs_in));
  constexpr bool kAny = KIND == KIND_DIRS_ANY;
  constexpr bool kSweep = KIND != KIND_DIRS && !kAny, kMake = KIND == KIND_FIRST;
  constexpr bool kFirst = KIND == KIND_FIRST_GIVEN || kMake;
  constexpr int R = TY, V = TY + 2;  // lines out, lines in
  const int lane = threadIdx.x & 63;
  const int32_t bx = tile % G.tiles_x, by = (tile / G.tiles_x) % G.tiles_y,
                bz = tile / (G.tiles_x * G.tiles_y);
  const int32_t x0 = bx * TX, y0 = by * TY;
  const Span zs = part_of(bz * G.chunk, G.chunk, G.nz, part, parts);
  const int32_t z0 = zs.a, z1 = zs.b;
  if (z0 >= z1) return LaneCounts{0, 0, 0};
  const int32_t nq = z1 - z0 + 2;
  auto clamp_to = [](int32_t v, int32_t n) { return v < 0 ? 0 : v < n ? v : n - 1; };
  auto plane_at = [&](int32_t q) { return (int64_t)G.sxy * clamp_step(z0, q - 1, G.nz); };
  // a uniform base per plane, at the first line loaded and column x0; from there
  // the lines' offsets (below 6 nx sizeof(T), which the host keeps under 2^32) and
  // the lanes'
  const int32_t y_first = clamp_step(y0, -1, G.ny);
  const int64_t at0 = (int64_t)G.nx * y_first + x0;
  uint32_t row[V];
#pragma unroll
  for (int r = 0; r < V; ++r)
    row[r] = (uint32_t)G.nx * (uint32_t)(clamp_step(y0, r - 1, G.ny) - y_first);

  const int32_t X = x0 + lane;
  const bool in_x = X < G.nx;
  uint32_t core = 0;  // lines whose vertices are compared, a byte per line
#pragma unroll
  for (int r = 0; r < R; ++r)
    core |= in_x && X >= G.cx0 && X < G.cx1 && y0 + r >= G.cy0 && y0 + r < G.cy1 ? 0xffu << (8 * r)
                                                                              : 0u;
  const uint32_t xo = (uint32_t)(clamp_to(X, G.nx) - x0);
  const uint32_t xb = xo * (uint32_t)sizeof(T);
  uint32_t xs[R];  // where a line's direction bytes go
#pragma unroll
  for (int r = 0; r < R; ++r) xs[r] = in_x && y0 + r < G.ny ? xo : kNoStore;
  struct Plane {
    T v[V];
    uint32_t d[R];  // directions of f one plane lower
    T fv[kMake ? V : R];  // f in this plane (its lines out, or all)
  };
  constexpr int FO = kMake ? 1 : 0;  // first line out in fv
  auto fetch = [&](int32_t q, Plane& S) {
    const int64_t pl = plane_at(q) + at0;
    const Rsrc rh = rsrc_at(h + pl);
#pragma unroll
    for (int r = 0; r < V; ++r) buf_load(rh, xb, row[r] * (uint32_t)sizeof(T), S.v[r]);
    if (kFirst) {
      const Rsrc rf = rsrc_at(f + pl);
#pragma unroll
      for (int r = 0; r < (kMake ? V : R); ++r)
        buf_load(rf, xb, row[r + 1 - FO] * (uint32_t)sizeof(T), S.fv[r]);
    }
    if (kSweep && !kMake) {
      const Rsrc rd = rsrc_at(dirs + (plane_at(q - 1) + at0));
#pragma unroll
      for (int r = 0; r < R; ++r)
        S.d[r] = __builtin_amdgcn_raw_buffer_load_b8(rd, xo, row[r + 1], 0);
    }
  };
  Plane P0, P1;
  fetch(0, P0);
  fetch(1, P1);

  // ---- the tile's edges, for the planes q0 .. q0 + 3: lane 8 j + r has line r of
  // plane q0 + j (the upper lanes repeat them): the value right of the tile and
  // the two that the boxes to the left begin with.  The lines meet by a lane
  // shift, the planes by a shuffle over eight lanes, the first with the last
  // group's last.
  static_assert(R == 4 && V <= 8 && kEdgeGroup == 4, "lane layout of the edges");
  const int32_t ej = (lane >> 3) & 3, er = (lane & 7) < V ? lane & 7 : V - 1;
  const int32_t e_row = G.nx * clamp_step(y0, er - 1, G.ny);
  const uint32_t e_right = (uint32_t)(e_row + clamp_step(x0, TX, G.nx));
  const uint32_t e_left = (uint32_t)(e_row + (x0 ? x0 - 1 : 0));
  const uint32_t e_own = (uint32_t)(e_row + x0);
  struct Edges {
    T right, a, b;
  };
  // lanes 0..7: squares of plane q0 - 1
  Box<T> e_last[2] = {{T(0), T(0), 0u, 0u}, {T(0), T(0), 0u, 0u}};
  auto edges_load1 = [&](gptr<const T> from, int32_t q0, Edges& e) {
    const gptr<const T> p = from + plane_at(q0 + ej);
    e.right = p[e_right];
    e.a = p[e_left];
    e.b = p[e_own];
  };
  bool any_nan = false;  // (kAny)
  auto edges_store1 = [&](int which, int32_t q0, const Edges& e) {
    if (kAny) any_nan |= __builtin_isunordered(e.right, e.a);
    const XPair<T> xp = x_pair(e.a, e.b, 0u);
    const Box<T> ln{xp.hi, xp.lo, xp.c, xp.c ^ 1u};
    const Box<T> sq1 =
        box_merge(ln, Box<T>{lane_shift<kFromRight>(ln.hi, ln.hi),
                             lane_shift<kFromRight>(ln.lo, ln.lo),
                             lane_shift<kFromRight>(ln.ca, ln.ca) | 2u,
                             lane_shift<kFromRight>(ln.cd, ln.cd) | 2u});
    const int from = (lane - 8) & 31;
    Box<T> below{__shfl(sq1.hi, from, 64), __shfl(sq1.lo, from, 64),
                 (uint32_t)__shfl((int)sq1.ca, from, 64), (uint32_t)__shfl((int)sq1.cd, from, 64)};
    const Box<T> next = below;
    if (ej == 0) below = e_last[which];
    e_last[which] = next;
    const Box<T> b = box_merge(below, Box<T>{sq1.hi, sq1.lo, sq1.ca | 4u, sq1.cd | 4u});
    Edge3<T>& E = sm.edge[which][ej];
    E.right[er] = e.right;
    if ((lane & 7) < R) {
      E.hi[er] = b.hi;
      E.lo[er] = b.lo;
      E.w[er] = lower_codes_at(b.ca, b.cd, 7u,
                               (x0 == 0 ? 1u : 0u) | (y0 + er == 0 ? 2u : 0u) |
                                   (z0 + q0 + ej == 1 ? 4u : 0u));
    }
  };
  Edges edges[2];
  auto edges_load = [&](int32_t q0) {
    edges_load1(h, q0, edges[0]);
    if (kMake) edges_load1(f, q0, edges[1]);
  };
  auto edges_store = [&](int32_t q0) {
    edges_store1(0, q0, edges[0]);
    if (kMake) edges_store1(1, q0, edges[1]);
    wave_lds_fence();
  };
  edges_load(0);
  edges_store(0);

  const T xi_in = fast_margin<T>(xi);
  // axes along which the vertices have an upper neighbour, per line
  uint32_t keep[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    keep[r] = 0x0707u & ~((X >= G.nx - 1 ? 0x0101u : 0u) | (y0 + r >= G.ny - 1 ? 0x0202u : 0u));
  const uint32_t low_y = y0 == 0 ? 0x0202u : 0u;  // line 0's lower boxes: no neighbour below
  constexpr int32_t kPlaneBits3 = kRowBits3 * (TY + 2);
  const int32_t zc1 = G.cz1 < z1 ? G.cz1 : z1;  // end of the planes to compare
  LaneCounts n{0, 0, 0};
  struct March {
    Box<T> sq[R + 1];  // squares of the last plane
    Low<T> low[R];     // lower boxes of the last plane's vertices
  };
  March mh, mf;  // of h; of f, where its directions are made
  // The step of plane q (0 is z0 - 1) with parity PARITY: MODE 0 squares only, 1 boxes
  // only, 2 whole.
  auto pairs = [&](auto parity, const T* v, const Edge3<T>& E, XPair<T>* xp) {
    constexpr uint32_t ZT = 4u * (uint32_t)decltype(parity)::value;
#pragma unroll
    for (int r = 0; r < V; ++r)
      xp[r] = x_pair(v[r], lane_shift<kFromRight>(v[r], E.right[r]),
                     (uint32_t)(2 * (r & 1)) | ZT);
  };
  // emit(r, byte, lowest neighbour) for the vertices of the plane before
  auto boxes = [&](auto mode, auto parity, const XPair<T>* xp, const Edge3<T>& E, March& M,
                   auto emit) {
    constexpr int MODE = decltype(mode)::value;
    constexpr uint32_t ZP = 4u * (uint32_t)decltype(parity)::value ^ 4u;
    // from the last line down: line rr's new lower box replaces the one that
    // the vertex of line rr + 1 has used
#pragma unroll
    for (int rr = R; rr >= 0; --rr) {
      const Box<T> s = box_merge(box_of_pair(xp[rr]), box_of_pair(xp[rr + 1]));
      if (MODE != 0) {
        const Box<T> b = box_merge(M.sq[rr], s);
        const uint32_t w = code_word(b);
        const uint32_t par = (uint32_t)(2 * (rr & 1)) | ZP;
        if (MODE == 2 && rr > 0) {
          const int r = rr - 1;
          emit(r, dir_byte(M.low[r], b, upper_codes(w, par, keep[r])),
               PROP ? lower(b.lo < M.low[r].lo, b.lo, M.low[r].lo) : T(0));
        }
        if (rr < R) {
          uint32_t m = w;
          // no neighbour below line 0, and below plane 0 (the y and z bits of the
          // upper half: these boxes' line and plane parities are even)
          if (rr == 0) m |= low_y;
          if (MODE == 1 && z0 == 0) m |= 0x0404u;
          const uint32_t lw = (rr & 1) ? lower_codes<2u | ZP, 7u>(m) : lower_codes<ZP, 7u>(m);
          M.low[rr] = Low<T>{lane_shift<kFromLeft>(b.hi, E.hi[rr]),
                             lane_shift<kFromLeft>(b.lo, E.lo[rr]),
                             lane_shift<kFromLeft>(lw, E.w[rr])};
        }
      }
      M.sq[rr] = s;
    }
  };
  auto step = [&](auto mode, auto parity, int32_t q, Plane& S) {
    constexpr int MODE = decltype(mode)::value;
    const Edge3<T>& E = sm.edge[0][q & (kEdgeGroup - 1)];
    const Edge3<T>& Ef = sm.edge[kMake ? 1 : 0][q & (kEdgeGroup - 1)];
    const int32_t z = z0 + q - 2;  // plane of the vertices finished
    XPair<T> xp[V], xf[V];
    pairs(parity, S.v, E, xp);
    if (kAny) {
#pragma unroll
      for (int r = 0; r < V; r += 2) any_nan |= __builtin_isunordered(S.v[r], S.v[r + 1]);
    }
    if (kMake) pairs(parity, S.fv, Ef, xf);
    if (COPY && MODE != 0) {
      const Rsrc rc = rsrc_at(copy_to + (plane_at(q) + at0), q < nq - 1);
#pragma unroll
      for (int r = 0; r < R; ++r)
        buf_store(rc, xb, row[r + 1] * (uint32_t)sizeof(T), S.v[r + 1]);
    }
    if (kFirst && MODE != 0) {
      // validation of plane q (the last one is the next tile's or absent)
      // (bound_class's fast test for all lines, one branch for the rest)
      bool near = false;
#pragma unroll
      for (int r = 0; r < R; ++r)
        near |= !(__builtin_fabs(S.v[r + 1] - S.fv[r + FO]) < xi_in);
      if (near && in_x && q < nq - 1) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int bc = y0 + r < G.ny ? bound_class_exact<T>(S.fv[r + FO], S.v[r + 1], xi) : 0;
          n.nf += bc == 1;
          n.nb += bc == 2;
        }
      }
    }
    uint32_t os = 0, ds = 0;  // direction bytes of the lines, of g and of f
    T lows[R];                // their lowest neighbours (proposals)
    if (kSweep && !kMake && MODE == 2) {
#pragma unroll
      for (int r = 0; r < R; ++r) ds |= S.d[r] << (8 * r);
    }
    fetch(q + 2, S);
    const Rsrc rout = rsrc_at(dirs + ((int64_t)G.sxy * z + at0), z < z1);
    auto store = [&](int r, uint32_t o) {
      __builtin_amdgcn_raw_buffer_store_b8((uint8_t)o, rout, xs[r], row[r + 1], 0);
    };
    if (kMake)
      boxes(mode, parity, xf, Ef, mf, [&](int r, uint32_t o, T) {
        store(r, o);
        ds |= o << (8 * r);
      });
    boxes(mode, parity, xp, E, mh, [&](int r, uint32_t o, T lo) {
      if (kSweep) {
        os |= o << (8 * r);
        lows[r] = lo;
      } else {
        store(r, o);
      }
    });
    if (kSweep && MODE == 2) {
      // mismatches, a line at a time per lane (few lanes have more than one)
      uint32_t diff = (os ^ ds) & (z >= G.cz0 && z < zc1 ? core : 0u);
      while (__ballot(diff != 0u)) {
        if (diff != 0u) {
          const int r = __builtin_ctz(diff) >> 3;
          diff &= ~(0xffu << (8 * r));
          n.mism += flag_mismatch<T, PROP>(
              (os >> (8 * r)) & 0xffu, (ds >> (8 * r)) & 0xffu,
              (z - z0 + 1) * kPlaneBits3 + (r + 1) * kRowBits3 + lane + 1,
              X + G.nx * (y0 + r) + G.sxy * z, G, sm.flags, fdelta, prop, h,
              PROP ? (r == 0 ? lows[0] : r == 1 ? lows[1] : r == 2 ? lows[2] : lows[3]) : T(0));
        }
      }
    }
  };
  auto last_plane = [&](int32_t q) {
    if (q == nq - 1 && z1 == G.nz) {
#pragma unroll
      for (int r = 0; r < R; ++r) keep[r] &= ~0x0404u;
    }
  };
  step(Int<0>{}, Int<0>{}, 0, P0);
  step(Int<1>{}, Int<1>{}, 1, P1);
  // (an odd tile's last step finishes nothing: plane z1 is outside it)
  for (int32_t q = 2; q < nq; q += 4) {
    edges_load(q + 2);
    last_plane(q);
    step(Int<2>{}, Int<0>{}, q, P0);
    last_plane(q + 1);
    step(Int<2>{}, Int<1>{}, q + 1, P1);
    if (q + 2 >= nq) break;
    edges_store(q + 2);
    last_plane(q + 2);
    step(Int<2>{}, Int<0>{}, q + 2, P0);
    last_plane(q + 3);
    step(Int<2>{}, Int<1>{}, q + 3, P1);
  }
  if (kAny && __ballot(any_nan) != 0ull) {
    __builtin_amdgcn_s_waitcnt(0);  // the march's stores are done
    wave_dirs_any3<T>(h, dirs, G, x0, y0, z0, z1);
  }
  if (kSweep) {
    wave_lds_fence();
    wave_flush_rows<kFlagW3>(sm.flags, (z1 - z0 + 2) * (TY + 2), [&](int32_t r) {
      const int32_t lz = r / (TY + 2), ly = r - lz * (TY + 2);
      return G.nx * (y0 - 1 + ly) + G.sxy * (z0 - 1 + lz) + (x0 - 1);
    }, as_global(uniform_ptr(bm_in)));
    wave_lds_fence();
  }
  return n;
}

// One 2D tile (tiles.hpp's 256-wide strip) on one wave, four columns per lane,
// marched along y like wave_tile3 along z.  RAGGED: the strip ends inside the tile,
// and its columns are loaded one by one with clamped offsets.
template <class T, int KIND, bool PROP, bool COPY, bool RAGGED, class LDS>
__device__ __forceinline__ LaneCounts wave_tile2_t(LDS& sm, const int32_t* fdelta, const T* h_in,
                                                   const T* f_in, uint8_t* dirs_in,
                                                   uint32_t* bm_in, T xi, const TileGeo& G,
                                                   int32_t tile, void* prop_in, T* copy_in,
                                                   int32_t part, int32_t parts) {
  const gptr<T> copy_to = as_global(uniform_ptr(copy_in));
  void* const prop = PROP ? uniform_ptr(prop_in) : nullptr;
  const gptr<const T> h = as_global((const T*)uniform_ptr(h_in));
  const gptr<const T> f = as_global((const T*)uniform_ptr(f_in));
  const gptr<uint8_t> dirs = as_global(uniform_ptr(dirs_in));
  constexpr bool kAny = KIND == KIND_DIRS_ANY;
  constexpr bool kSweep = KIND != KIND_DIRS && !kAny, kMake = KIND == KIND_FIRST;
  constexpr bool kFirst = KIND == KIND_FIRST_GIVEN || kMake;
  constexpr int C = 4;
  const int lane = threadIdx.x & 63;
  const int32_t bx = tile % G.tiles_x, by = tile / G.tiles_x;
  const int32_t x0 = bx * RX;
  const Span ys = part_of(by * G.chunk, G.chunk, G.ny, part, parts);
  const int32_t y0 = ys.a, y1 = ys.b;
  if (y0 >= y1) return LaneCounts{0, 0, 0};
  const int32_t nq = y1 - y0 + 2;
  auto clamp_to = [](int32_t v, int32_t n) { return v < 0 ? 0 : v < n ? v : n - 1; };
  auto row_at = [&](int32_t q) { return (int64_t)G.nx * clamp_step(y0, q - 1, G.ny); };

  const int32_t X = x0 + C * lane;
  constexpr int NO = RAGGED ? C : 1;
  uint32_t off[NO], offb[NO];
#pragma unroll
  for (int j = 0; j < NO; ++j) {
    off[j] = (uint32_t)(clamp_to(X + j, G.nx) - x0);
    offb[j] = off[j] * (uint32_t)sizeof(T);
  }
  // columns inside the strip (bit j), and inside the detection box (byte j)
  uint32_t in_x = 0, core_x = 0;
  uint32_t keep[C];
#pragma unroll
  for (int j = 0; j < C; ++j) {
    in_x |= X + j < G.nx ? 1u << j : 0u;
    core_x |= X + j < G.nx && X + j >= G.cx0 && X + j < G.cx1 ? 0xffu << (8 * j) : 0u;
    keep[j] = 0x0303u & ~(X + j >= G.nx - 1 ? 0x0101u : 0u);
  }
  struct Row {
    T v[C];
    uint32_t d[RAGGED ? C : 1];  // directions of f one row lower
    T fv[C];                     // f in this row
  };
  auto load4 = [&](gptr<const T> p, T* out) {
    const Rsrc r = rsrc_at(p);
    if (RAGGED) {
#pragma unroll
      for (int j = 0; j < C; ++j) buf_load(r, offb[j % NO], 0, out[j]);
    } else {
      buf_load4(r, offb[0], out);
    }
  };
  auto fetch = [&](int32_t q, Row& S) {
    load4(h + (row_at(q) + x0), S.v);
    if (kFirst) load4(f + (row_at(q) + x0), S.fv);
    if (kSweep && !kMake) {
      const Rsrc r = rsrc_at(dirs + (row_at(q - 1) + x0));
      if (RAGGED) {
#pragma unroll
        for (int j = 0; j < C; ++j)
          S.d[j % NO] = __builtin_amdgcn_raw_buffer_load_b8(r, off[j % NO], 0, 0);
      } else {
        S.d[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off[0], 0, 0);
      }
    }
  };
  Row P0, P1;
  fetch(0, P0);
  fetch(1, P1);

  // ---- the tile's edges
  bool any_nan = false;  // (kAny)
  {
    const int32_t xr = clamp_step(x0, RX, G.nx);
    const uint32_t gone_x = x0 == 0 ? 1u : 0u;
    auto edges_of = [&](gptr<const T> from, int32_t q, Edge2<T>& E) {
      E.right = from[row_at(q) + xr];
      if (kAny) any_nan |= __builtin_isunordered(E.right, from[row_at(q) + (x0 ? x0 - 1 : x0)]);
      Box<T> ln[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const gptr<const T> p = from + (row_at(q - 1 + j) + x0);
        const T B = p[0], A = p[x0 ? -1 : 0];
        const XPair<T> xp = x_pair(A, B, (uint32_t)(2 * j));
        ln[j] = Box<T>{xp.hi, xp.lo, xp.c, xp.c ^ 1u};
      }
      const Box<T> b = box_merge(ln[0], ln[1]);
      E.hi = b.hi;
      E.lo = b.lo;
      E.w = lower_codes_at(b.ca, b.cd, 3u, gone_x | (y0 + q == 1 ? 2u : 0u));
    };
    for (int32_t q = lane; q < nq; q += 64) {
      edges_of(h, q, sm.edge[0][q]);
      if (kMake) edges_of(f, q, sm.edge[kMake ? 1 : 0][q]);
    }
    wave_lds_fence();
  }
  const T xi_in = fast_margin<T>(xi);
  const int32_t yc1 = G.cy1 < y1 ? G.cy1 : y1;  // end of the rows to compare
  LaneCounts n{0, 0, 0};
  struct March {
    XPair<T> pr[C];  // pairs of the last row
    Low<T> low[C];   // lower boxes of the last row's vertices
  };
  March mh, mf;  // of h; of f, where its directions are made
  auto pairs = [&](auto parity, const T* v, const Edge2<T>& E, XPair<T>* xp) {
    constexpr uint32_t YT = 2u * (uint32_t)decltype(parity)::value;
    const T right = lane_shift<kFromRight>(v[0], E.right);
#pragma unroll
    for (int j = 0; j < C; ++j) xp[j] = x_pair(v[j], j + 1 < C ? v[j + 1] : right, YT);
  };
  // The boxes of a row; returns the direction bytes of the row before, emit(j,
  // lowest neighbour) per column.
  auto boxes = [&](auto mode, auto parity, const XPair<T>* xp, const Edge2<T>& E, March& M,
                   auto emit) {
    constexpr int MODE = decltype(mode)::value;
    constexpr uint32_t YP = 2u * (uint32_t)decltype(parity)::value ^ 2u;
    uint32_t o = 0;
    if (MODE != 0) {
      Low<T> nl[C];
#pragma unroll
      for (int j = 0; j < C; ++j) {
        const Box<T> b = box_merge(box_of_pair(M.pr[j]), box_of_pair(xp[j]));
        uint32_t w = code_word(b);
        if (MODE == 2) {
          o |= dir_byte(M.low[j], b, upper_codes(w, YP, keep[j])) << (8 * j);
          emit(j, PROP ? lower(b.lo < M.low[j].lo, b.lo, M.low[j].lo) : T(0));
        }
        if (MODE == 1 && y0 == 0) w |= 0x0202u;  // no row below row 0
        nl[j] = Low<T>{b.hi, b.lo, lower_codes<YP, 3u>(w)};
      }
      M.low[0] = Low<T>{lane_shift<kFromLeft>(nl[C - 1].hi, E.hi),
                        lane_shift<kFromLeft>(nl[C - 1].lo, E.lo),
                        lane_shift<kFromLeft>(nl[C - 1].w, E.w)};
#pragma unroll
      for (int j = 1; j < C; ++j) M.low[j] = nl[j - 1];
    }
#pragma unroll
    for (int j = 0; j < C; ++j) M.pr[j] = xp[j];
    return o;
  };
  auto step = [&](auto mode, auto parity, int32_t q, Row& S) {
    constexpr int MODE = decltype(mode)::value;
    const Edge2<T>& E = sm.edge[0][q];
    const Edge2<T>& Ef = sm.edge[kMake ? 1 : 0][q];
    const int32_t y = y0 + q - 2;  // row of the vertices finished
    XPair<T> xp[C], xf[C];
    pairs(parity, S.v, E, xp);
    if (kAny) {
#pragma unroll
      for (int j = 0; j < C; j += 2) any_nan |= __builtin_isunordered(S.v[j], S.v[j + 1]);
    }
    if (kMake) pairs(parity, S.fv, Ef, xf);
    if (COPY && MODE != 0) {
      const Rsrc rc = rsrc_at(copy_to + (row_at(q) + x0), q < nq - 1);
      if (RAGGED) {
#pragma unroll
        for (int j = 0; j < C; ++j) buf_store(rc, offb[j % NO], 0, S.v[j]);
      } else {
        buf_store4(rc, offb[0], S.v);
      }
    }
    if (kFirst && MODE != 0) {
      bool near = false;
#pragma unroll
      for (int j = 0; j < C; ++j) near |= !(__builtin_fabs(S.v[j] - S.fv[j]) < xi_in);
      if (near && q < nq - 1) {
#pragma unroll
        for (int j = 0; j < C; ++j) {
          const int bc = (in_x >> j) & 1 ? bound_class_exact<T>(S.fv[j], S.v[j], xi) : 0;
          n.nf += bc == 1;
          n.nb += bc == 2;
        }
      }
    }
    uint32_t d = 0;
    if (kSweep && !kMake && MODE == 2) {
      d = S.d[0];
      if (RAGGED) {
#pragma unroll
        for (int j = 1; j < C; ++j) d |= S.d[j % NO] << (8 * j);
      }
    }
    fetch(q + 2, S);
    auto store = [&](uint32_t o) {
      const Rsrc r = rsrc_at(dirs + ((int64_t)G.nx * y + x0), y < y1);
      if (RAGGED) {
#pragma unroll
        for (int j = 0; j < C; ++j)
          __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(o >> (8 * j)), r,
                                               (in_x >> j) & 1 ? off[j % NO] : kNoStore, 0, 0);
      } else {
        __builtin_amdgcn_raw_buffer_store_b32(o, r, off[0], 0, 0);
      }
    };
    if (kMake) {
      d = boxes(mode, parity, xf, Ef, mf, [](int, T) {});
      if (MODE == 2) store(d);
    }
    T lows[C];
    const uint32_t o = boxes(mode, parity, xp, E, mh, [&](int j, T lo) { lows[j] = lo; });
    if (!kSweep && MODE == 2) store(o);
    if (kSweep && MODE == 2) {
      uint32_t diff = (o ^ d) & (y >= G.cy0 && y < yc1 ? core_x : 0u);
      while (__ballot(diff != 0u)) {
        if (diff != 0u) {
          const int j = __builtin_ctz(diff) >> 3;
          diff &= ~(0xffu << (8 * j));
          n.mism += flag_mismatch<T, PROP>(
              (o >> (8 * j)) & 0xffu, (d >> (8 * j)) & 0xffu,
              (y - y0 + 1) * kRowBits2 + C * lane + j + 1, X + j + G.nx * y, G, sm.flags, fdelta,
              prop, h, PROP ? (j == 0 ? lows[0] : j == 1 ? lows[1] : j == 2 ? lows[2] : lows[3]) : T(0));
        }
      }
    }
  };
  auto last_row = [&](int32_t q) {
    if (q == nq - 1 && y1 == G.ny) {
#pragma unroll
      for (int j = 0; j < C; ++j) keep[j] &= ~0x0202u;
    }
  };
  step(Int<0>{}, Int<0>{}, 0, P0);
  step(Int<1>{}, Int<1>{}, 1, P1);
  // (an odd tile's last step finishes nothing: row y1 is outside it)
  for (int32_t q = 2; q < nq; q += 2) {
    last_row(q);
    step(Int<2>{}, Int<0>{}, q, P0);
    last_row(q + 1);
    step(Int<2>{}, Int<1>{}, q + 1, P1);
  }
  if (kAny && __ballot(any_nan) != 0ull) {
    __builtin_amdgcn_s_waitcnt(0);  // the march's stores are done
    wave_dirs_any2<T>(h, dirs, G, x0, y0, y1);
  }
  if (kSweep) {
    wave_lds_fence();
    wave_flush_rows<kFlagW2>(sm.flags, y1 - y0 + 2,
                             [&](int32_t r) { return G.nx * (y0 - 1 + r) + (x0 - 1); },
                             as_global(uniform_ptr(bm_in)));
    wave_lds_fence();
  }
  return n;
}

// part, parts: march that part of the tile's planes (rows in 2D) alone.
template <class T, int KIND, bool PROP, bool COPY, int DIM, class LDS>
__device__ __forceinline__ LaneCounts wave_tile(LDS& sm, const int32_t* fdelta, const T* h,
                                                const T* f, uint8_t* dirs, uint32_t* bm, T xi,
                                                const TileGeo& G_in, int32_t tile, void* prop,
                                                T* copy_to, int32_t part = 0, int32_t parts = 1) {
  if constexpr (DIM == 3) {
    return wave_tile3<T, KIND, PROP, COPY>(sm, fdelta, h, f, dirs, bm, xi, G_in, tile, prop,
                                           copy_to, part, parts);
  } else {
    const TileGeo G = uniform_geo(G_in);
    if (G.nx - tile % G.tiles_x * RX < RX)
      return wave_tile2_t<T, KIND, PROP, COPY, true>(sm, fdelta, h, f, dirs, bm, xi, G, tile, prop,
                                                     copy_to, part, parts);
    return wave_tile2_t<T, KIND, PROP, COPY, false>(sm, fdelta, h, f, dirs, bm, xi, G, tile, prop,
                                                    copy_to, part, parts);
  }
}

}  // namespace pmsz
