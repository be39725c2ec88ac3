// edits.hip -- the edit stream: encoding of the corrections for storage.
//
// The correction changes a few values of the decompressed field; storing it
// means storing those changes (Sec. V-D reports this as the method's storage
// overhead; the paper fixes no format).  Stream layout (little-endian):
//   header   'PMSE', u8 version 1, u8 dtype, u16 0, u64 vertices, u64 edits,
//            u64 payload bytes, u32 chunk (entries per chunk), u32 chunks
//   table    per chunk: u64 payload offset of its first entry, u64 index of
//            the edited vertex before it (all ones when none)
//   payload  per vertex i whose bits changed, ascending: gap = i - previous
//            edited index - 1 and steps = key(fhat_i) - key(g_i), each as an
//            unsigned LEB128 varint; key() maps values to integers in value
//            order, so steps counts the representable values in (g_i, fhat_i].
// Encoding is a chain of data-parallel passes (count, scan, compact, sizes,
// scan, write); decoding runs one block per chunk of the table.
#include <string.h>

#include "launch.hpp"

namespace pmsz {

constexpr int kEditChunk = 4096;    // entries per chunk of the table
constexpr int kScanItems = 4096;    // items per block of the scans
constexpr int kCountItems = 4096;   // vertices per block of the count / compact

__device__ __forceinline__ unsigned long long order_key(float v) {
  const uint32_t b = __float_as_uint(v);
  return (b & 0x80000000u) ? (unsigned long long)(~b) : (unsigned long long)(b | 0x80000000u);
}
__device__ __forceinline__ unsigned long long order_key(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ void from_order_key(unsigned long long k, float* out) {
  const uint32_t kk = (uint32_t)k;
  *out = __uint_as_float((kk & 0x80000000u) ? (kk & 0x7fffffffu) : ~kk);
}
__device__ __forceinline__ void from_order_key(unsigned long long k, double* out) {
  *out = __longlong_as_double(
      (long long)((k & 0x8000000000000000ull) ? (k & 0x7fffffffffffffffull) : ~k));
}

template <class T>
__device__ __forceinline__ bool bits_differ(T a, T b);
template <>
__device__ __forceinline__ bool bits_differ<float>(float a, float b) {
  return __float_as_uint(a) != __float_as_uint(b);
}
template <>
__device__ __forceinline__ bool bits_differ<double>(double a, double b) {
  return __double_as_longlong(a) != __double_as_longlong(b);
}

__device__ __forceinline__ uint32_t leb_len(unsigned long long v) {
  uint32_t n = 1;
  while (v >= 0x80ull) {
    v >>= 7;
    ++n;
  }
  return n;
}

// Exclusive sum over the 256 threads of a block; *total (all threads).
__device__ __forceinline__ unsigned long long block_excl(unsigned long long v,
                                                         unsigned long long* sh,
                                                         unsigned long long* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  unsigned long long x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  unsigned long long before = 0, all = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < wave) before += sh[w];
    all += sh[w];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// ---- exclusive scan of n uint32 values into uint64 offsets -----------------
// Pass 1: sum of each block of kScanItems items.
__global__ __launch_bounds__(256) void k_scan_sums(const uint32_t* in, int64_t n,
                                                   unsigned long long* sums) {
  __shared__ unsigned long long sh[4];
  const int64_t b0 = (int64_t)blockIdx.x * kScanItems;
  unsigned long long v = 0;
  for (int k = 0; k < kScanItems / 256; ++k) {
    const int64_t i = b0 + threadIdx.x + 256 * k;
    if (i < n) v += in[i];
  }
  unsigned long long total;
  block_excl(v, sh, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}
// Pass 2: one block scans the block sums in place (exclusive); the grand
// total goes to *total.
__global__ __launch_bounds__(256) void k_scan_top(unsigned long long* sums, int64_t nb,
                                                  unsigned long long* total) {
  __shared__ unsigned long long sh[4];
  const int64_t per = (nb + 255) / 256;
  const int64_t b0 = threadIdx.x * per;
  unsigned long long v = 0;
  for (int64_t i = b0; i < b0 + per && i < nb; ++i) v += sums[i];
  unsigned long long all;
  unsigned long long run = block_excl(v, sh, &all);
  for (int64_t i = b0; i < b0 + per && i < nb; ++i) {
    const unsigned long long s = sums[i];
    sums[i] = run;
    run += s;
  }
  if (threadIdx.x == 0) *total = all;
}
// Pass 3: each block rescans its items from its offset.  A thread takes a
// contiguous run of kScanItems/256 items so the order is preserved.
__global__ __launch_bounds__(256) void k_scan_apply(const uint32_t* in, int64_t n,
                                                    const unsigned long long* sums,
                                                    unsigned long long* out) {
  __shared__ unsigned long long sh[4];
  constexpr int kPer = kScanItems / 256;
  const int64_t i0 = (int64_t)blockIdx.x * kScanItems + (int64_t)threadIdx.x * kPer;
  unsigned long long v = 0;
  for (int k = 0; k < kPer; ++k)
    if (i0 + k < n) v += in[i0 + k];
  unsigned long long total;
  unsigned long long run = sums[blockIdx.x] + block_excl(v, sh, &total);
  for (int k = 0; k < kPer; ++k)
    if (i0 + k < n) {
      out[i0 + k] = run;
      run += in[i0 + k];
    }
}

// ---- encoder passes ----------------------------------------------------------
template <class T>
__global__ __launch_bounds__(256) void k_edit_count(const T* fhat, const T* g, int64_t n,
                                                    uint32_t* counts) {
  __shared__ unsigned long long sh[4];
  constexpr int kPer = kCountItems / 256;
  const int64_t i0 = (int64_t)blockIdx.x * kCountItems + (int64_t)threadIdx.x * kPer;
  unsigned long long c = 0;
  for (int k = 0; k < kPer; ++k)
    if (i0 + k < n && bits_differ<T>(fhat[i0 + k], g[i0 + k])) ++c;
  unsigned long long total;
  block_excl(c, sh, &total);
  if (threadIdx.x == 0) counts[blockIdx.x] = (uint32_t)total;
}

// Index of every changed vertex, in ascending order, at its rank (block base
// from the scanned counts plus the rank inside the block); ranks at or past
// cap are not written.
template <class T>
__global__ __launch_bounds__(256) void k_edit_compact(const T* fhat, const T* g, int64_t n,
                                                      const unsigned long long* base,
                                                      uint32_t* idx, int64_t cap) {
  __shared__ unsigned long long sh[4];
  constexpr int kPer = kCountItems / 256;
  const int64_t i0 = (int64_t)blockIdx.x * kCountItems + (int64_t)threadIdx.x * kPer;
  unsigned long long c = 0;
  for (int k = 0; k < kPer; ++k)
    if (i0 + k < n && bits_differ<T>(fhat[i0 + k], g[i0 + k])) ++c;
  unsigned long long total;
  unsigned long long r = base[blockIdx.x] + block_excl(c, sh, &total);
  for (int k = 0; k < kPer; ++k)
    if (i0 + k < n && bits_differ<T>(fhat[i0 + k], g[i0 + k])) {
      if ((int64_t)r < cap) idx[r] = (uint32_t)(i0 + k);
      ++r;
    }
}

template <class T>
__device__ __forceinline__ void edit_entry(const T* fhat, const T* g, const uint32_t* idx,
                                           int64_t r, unsigned long long& gap,
                                           unsigned long long& steps) {
  const int64_t i = idx[r];
  const int64_t prev = r ? (int64_t)idx[r - 1] : -1;
  gap = (unsigned long long)(i - prev - 1);
  steps = order_key(fhat[i]) - order_key(g[i]);
}

template <class T>
__global__ __launch_bounds__(256) void k_edit_sizes(const T* fhat, const T* g,
                                                    const uint32_t* idx, int64_t ne,
                                                    uint32_t* len) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= ne) return;
  unsigned long long gap, steps;
  edit_entry<T>(fhat, g, idx, r, gap, steps);
  len[r] = leb_len(gap) + leb_len(steps);
}

__device__ __forceinline__ uint8_t* put_leb(uint8_t* p, unsigned long long v) {
  while (v >= 0x80ull) {
    *p++ = (uint8_t)(v | 0x80ull);
    v >>= 7;
  }
  *p++ = (uint8_t)v;
  return p;
}

template <class T>
__global__ __launch_bounds__(256) void k_edit_write(const T* fhat, const T* g,
                                                    const uint32_t* idx, int64_t ne,
                                                    const unsigned long long* off,
                                                    uint8_t* table, uint8_t* payload) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= ne) return;
  unsigned long long gap, steps;
  edit_entry<T>(fhat, g, idx, r, gap, steps);
  uint8_t* p = put_leb(payload + off[r], gap);
  put_leb(p, steps);
  if (r % kEditChunk == 0) {
    unsigned long long* t = (unsigned long long*)(table + 16 * (r / kEditChunk));
    t[0] = off[r];
    t[1] = r ? (unsigned long long)idx[r - 1] : ~0ull;
  }
}

// ---- decoder -------------------------------------------------------------------
// One block per chunk.  The payload is read in tiles of kDecTile bytes: every
// thread holds 16 of them, counts the varints that end there, and a block scan
// gives each varint its number in the chunk (even: a gap, odd: a step count of
// entry number / 2).  A varint belongs to the thread that holds its last byte,
// which reads the bytes before its own from LDS (the last 16 bytes of the tile
// before are kept).  A second scan turns the chunk's gaps into vertex indices,
// and all threads then lower their entries of g at once.
// The serial part of a chunk is thus two block scans per 8 KiB of payload and
// one scan of its entries, where one thread per chunk walked 4096 entries with
// a dependent byte load per byte and a dependent read of g per entry: bound by
// latency at 443 threads on the whole chip.  1.8 M edits of a 512^3 binary32
// field (5.9 MB of stream): 10.6 ms before, 77 us now; the whole call with its
// copy of the field 10.8 ms before, 0.33 ms now.
// Reads past the payload or indices outside the field set *err; the chunk's
// entries in range may still be written.
constexpr int kDecThreads = 512;
constexpr int kDecBytes = 16;                        // payload bytes per thread and tile
constexpr int kDecTile = kDecThreads * kDecBytes;    // 8 KiB
constexpr int kDecPer = kEditChunk / kDecThreads;    // entries per thread

// Exclusive sum over the kDecThreads threads of a block; *total (all threads).
template <class V>
__device__ __forceinline__ V dec_excl(V v, V* sh, V* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  V x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const V y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  V before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kDecThreads / 64; ++w) {
    const V t = sh[w];
    before += w < wave ? t : V(0);
    all += t;
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

template <class T>
__global__ __launch_bounds__(kDecThreads) void k_edit_decode(const uint8_t* table,
                                                             const uint8_t* payload,
                                                             int64_t payload_bytes, int64_t ne,
                                                             int64_t n, T* g, int* err) {
  // [the 16 bytes before the tile][tile], as 8-byte words
  __shared__ unsigned long long s_raw[(kDecBytes + kDecTile) / 8];
  __shared__ uint32_t s_at[kEditChunk];             // gaps, then vertex indices
  __shared__ unsigned long long s_steps[kEditChunk];
  __shared__ unsigned long long s_sum[kDecThreads / 64];
  __shared__ int s_cnt[kDecThreads / 64];
  constexpr uint32_t kBad = 0xFFFFFFFFu;
  const int tid = threadIdx.x;
  const int64_t c = blockIdx.x;
  const unsigned long long* t = (const unsigned long long*)(table + 16 * c);
  const int64_t start = (int64_t)t[0];
  const unsigned long long first = t[1] + 1ull;  // (all ones: none before)
  const int cnt = (int)((ne - c * kEditChunk) < kEditChunk ? ne - c * kEditChunk : kEditChunk);
  if (start < 0 || start >= payload_bytes) {
    if (tid == 0) *err = 1;
    return;
  }
  const uint8_t* bytes = (const uint8_t*)s_raw;
  bool bad = false;
  if (tid < kDecBytes / 8) s_raw[tid] = 0ull;  // no varint runs into the chunk's first byte
  int found = 0;                               // varints that ended before this tile
  // the payload is 8-byte aligned, and so is every tile
  for (int64_t at = start & ~int64_t(7); found < 2 * cnt; at += kDecTile) {
    if (at >= payload_bytes) {  // the payload ends inside the chunk
      bad = true;
      break;
    }
    __syncthreads();  // the tile before has been read (and its tail copied)
    unsigned long long w[kDecBytes / 8];
#pragma unroll
    for (int k = 0; k < kDecBytes / 8; ++k) {
      const int64_t b = at + tid * kDecBytes + 8 * k;
      w[k] = 0ull;
      if (b + 8 <= payload_bytes) {
        w[k] = *(const unsigned long long*)(payload + b);
      } else {
        for (int j = 0; b + j < payload_bytes; ++j)
          w[k] |= (unsigned long long)payload[b + j] << (8 * j);
      }
      // bytes before the chunk's first one read as ends of other varints
      if (b < start)
        w[k] = start - b >= 8 ? 0ull : w[k] & (~0ull << (8 * (start - b)));
      s_raw[(kDecBytes + tid * kDecBytes) / 8 + k] = w[k];
    }
    int mine = 0;
#pragma unroll
    for (int k = 0; k < kDecBytes / 8; ++k) {
      const int64_t b = at + tid * kDecBytes + 8 * k;
      unsigned long long ends = ~w[k] & 0x8080808080808080ull;
      if (b < start) ends &= start - b >= 8 ? 0ull : ~0ull << (8 * (start - b));
      if (b + 8 > payload_bytes)
        ends &= b >= payload_bytes ? 0ull : ~0ull >> (8 * (8 - (payload_bytes - b)));
      mine += __popcll(ends);
    }
    int all;
    int v = found + dec_excl<int>(mine, s_cnt, &all);  // (its barriers publish s_raw)
    if (mine && v < 2 * cnt) {
      // the part of this thread's first varint that lies before its bytes
      int p = kDecBytes + tid * kDecBytes;
      int q = p;
      while (p - q < 11 && q > 0 && (bytes[q - 1] & 0x80)) --q;
      unsigned long long x = 0;
      int len = 0;
      for (; q < p; ++q, ++len)
        if (len < 10) x |= (unsigned long long)(bytes[q] & 0x7f) << (7 * len);
      for (int k = 0; k < kDecBytes && mine > 0 && v < 2 * cnt; ++k) {
        const int64_t b = at + tid * kDecBytes + k;
        if (b < start) continue;
        const uint8_t y = bytes[p + k];
        if (len < 10) x |= (unsigned long long)(y & 0x7f) << (7 * len);
        ++len;
        if (y & 0x80) continue;
        bad |= len > 10;
        if (v & 1) {
          s_steps[v >> 1] = x;
          bad |= x == 0ull;
        } else {
          const bool in = x < (unsigned long long)n;
          s_at[v >> 1] = in ? (uint32_t)x : kBad;
          bad |= !in;
        }
        ++v;
        --mine;
        x = 0;
        len = 0;
      }
    }
    found += all;
    __syncthreads();  // every thread has read the bytes before its own
    if (tid == kDecThreads - 1)
      for (int k = 0; k < kDecBytes / 8; ++k) s_raw[k] = w[k];
  }
  if (__syncthreads_or(bad)) {
    if (tid == 0) *err = 1;
    return;
  }
  // gaps to vertex indices: entry e edits the vertex after `first` and e + 1
  // gaps and e earlier edits
  unsigned long long sum = 0;
#pragma unroll
  for (int k = 0; k < kDecPer; ++k) {
    const int e = tid * kDecPer + k;
    if (e < cnt) sum += (unsigned long long)s_at[e] + 1ull;
  }
  unsigned long long all;
  unsigned long long i = first + dec_excl<unsigned long long>(sum, s_sum, &all);
#pragma unroll
  for (int k = 0; k < kDecPer; ++k) {
    const int e = tid * kDecPer + k;
    if (e >= cnt) break;
    i += s_at[e];
    const bool in = i < (unsigned long long)n;
    s_at[e] = in ? (uint32_t)i : kBad;
    bad |= !in;
    ++i;
  }
  if (bad) *err = 1;
  __syncthreads();
  const gptr<T> gg = as_global(g);
#pragma unroll
  for (int k = 0; k < kDecPer; ++k) {
    const int e = tid + k * kDecThreads;
    if (e >= cnt || s_at[e] == kBad) continue;
    T out;
    from_order_key(order_key(gg[s_at[e]]) - s_steps[e], &out);
    gg[s_at[e]] = out;
  }
}

// ---- host side -------------------------------------------------------------------
struct EditLayout {
  size_t counts, base, sums, total, idx, len, off, bytes;
  int64_t nblocks, nscan;
};

static size_t al256(size_t v) { return (v + 255) / 256 * 256; }

static EditLayout edit_layout(int64_t n, int64_t cap) {
  EditLayout L;
  L.nblocks = (n + kCountItems - 1) / kCountItems;
  const int64_t items = cap > L.nblocks ? cap : L.nblocks;
  L.nscan = (items + kScanItems - 1) / kScanItems;
  L.counts = 0;
  L.base = L.counts + al256(4 * (size_t)L.nblocks);
  L.sums = L.base + al256(8 * (size_t)L.nblocks);
  L.total = L.sums + al256(8 * (size_t)L.nscan);
  L.idx = L.total + 256;
  L.len = L.idx + al256(4 * (size_t)(cap > 0 ? cap : 1));
  L.off = L.len + al256(4 * (size_t)(cap > 0 ? cap : 1));
  L.bytes = L.off + al256(8 * (size_t)(cap > 0 ? cap : 1));
  return L;
}

size_t edits_workspace_bytes(int64_t n, int64_t cap) { return edit_layout(n, cap).bytes; }

size_t edits_stream_bytes(int64_t ne) {
  const int64_t nch = (ne + kEditChunk - 1) / kEditChunk;
  return 40 + 16 * (size_t)nch + 15 * (size_t)ne;
}

static hipError_t scan_u32(const uint32_t* in, int64_t n, unsigned long long* sums,
                           unsigned long long* total, unsigned long long* out, hipStream_t s) {
  const int64_t nb = (n + kScanItems - 1) / kScanItems;
  if (nb < 1) return hipSuccess;
  hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)nb), dim3(256), 0, s, in, n, sums);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(256), 0, s, sums, nb, total);
  hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(256), 0, s, in, n,
                     (const unsigned long long*)sums, out);
  return hipGetLastError();
}

// Returns 0, or 1 when the edits exceed cap (*ne set), or 2 when the stream
// does not fit out_cap (*nbytes set); hip errors through *herr.
template <class T>
static int encode_t(const T* fhat, const T* g, int64_t n, int64_t cap, char* ws, uint8_t* out,
                    size_t out_cap, int64_t* ne_out, int64_t* nbytes_out, hipError_t* herr,
                    hipStream_t s) {
  const EditLayout L = edit_layout(n, cap);
  uint32_t* counts = (uint32_t*)(ws + L.counts);
  unsigned long long* base = (unsigned long long*)(ws + L.base);
  unsigned long long* sums = (unsigned long long*)(ws + L.sums);
  unsigned long long* total = (unsigned long long*)(ws + L.total);
  uint32_t* idx = (uint32_t*)(ws + L.idx);
  uint32_t* len = (uint32_t*)(ws + L.len);
  unsigned long long* off = (unsigned long long*)(ws + L.off);
  *herr = hipSuccess;
#define EDIT_TRY(x)                        \
  do {                                     \
    hipError_t e_ = (x);                   \
    if (e_ != hipSuccess) {                \
      *herr = e_;                          \
      return -1;                           \
    }                                      \
  } while (0)
  if (L.nblocks > 0) {
    hipLaunchKernelGGL(k_edit_count<T>, dim3((unsigned)L.nblocks), dim3(256), 0, s, fhat, g, n,
                       counts);
    EDIT_TRY(hipGetLastError());
    EDIT_TRY(scan_u32(counts, L.nblocks, sums, total, base, s));
  }
  unsigned long long ne = 0;
  EDIT_TRY(hipMemcpyAsync(&ne, total, 8, hipMemcpyDeviceToHost, s));
  EDIT_TRY(hipStreamSynchronize(s));
  if (L.nblocks == 0) ne = 0;
  *ne_out = (int64_t)ne;
  if ((int64_t)ne > cap) return 1;
  unsigned long long nb = 0;
  if (ne > 0) {
    hipLaunchKernelGGL(k_edit_compact<T>, dim3((unsigned)L.nblocks), dim3(256), 0, s, fhat, g,
                       n, (const unsigned long long*)base, idx, cap);
    EDIT_TRY(hipGetLastError());
    const unsigned grid = (unsigned)((ne + 255) / 256);
    hipLaunchKernelGGL(k_edit_sizes<T>, dim3(grid), dim3(256), 0, s, fhat, g,
                       (const uint32_t*)idx, (int64_t)ne, len);
    EDIT_TRY(hipGetLastError());
    EDIT_TRY(scan_u32(len, (int64_t)ne, sums, total, off, s));
    EDIT_TRY(hipMemcpyAsync(&nb, total, 8, hipMemcpyDeviceToHost, s));
    EDIT_TRY(hipStreamSynchronize(s));
  }
  const int64_t nch = ((int64_t)ne + kEditChunk - 1) / kEditChunk;
  const size_t head = 40 + 16 * (size_t)nch;
  *nbytes_out = (int64_t)(head + nb);
  if (head + nb > out_cap) return 2;
  unsigned char h[40];
  memcpy(h, "PMSE", 4);
  h[4] = 1;
  h[5] = sizeof(T) == 8 ? 1 : 0;
  h[6] = h[7] = 0;
  const unsigned long long nv = (unsigned long long)n;
  const uint32_t chunk = kEditChunk, chunks = (uint32_t)nch;
  memcpy(h + 8, &nv, 8);
  memcpy(h + 16, &ne, 8);
  memcpy(h + 24, &nb, 8);
  memcpy(h + 32, &chunk, 4);
  memcpy(h + 36, &chunks, 4);
  EDIT_TRY(hipMemcpyAsync(out, h, 40, hipMemcpyHostToDevice, s));
  if (ne > 0) {
    const unsigned grid = (unsigned)((ne + 255) / 256);
    hipLaunchKernelGGL(k_edit_write<T>, dim3(grid), dim3(256), 0, s, fhat, g,
                       (const uint32_t*)idx, (int64_t)ne, (const unsigned long long*)off,
                       out + 40, out + head);
    EDIT_TRY(hipGetLastError());
  }
  EDIT_TRY(hipStreamSynchronize(s));  // the header copy reads host memory
#undef EDIT_TRY
  return 0;
}

int edits_encode(int dtype, const void* fhat, const void* g, int64_t n, int64_t cap, void* ws,
                 uint8_t* out, size_t out_cap, int64_t* ne, int64_t* nbytes, hipError_t* herr,
                 hipStream_t s) {
  if (dtype == PMSZ_F32)
    return encode_t<float>((const float*)fhat, (const float*)g, n, cap, (char*)ws, out, out_cap,
                           ne, nbytes, herr, s);
  return encode_t<double>((const double*)fhat, (const double*)g, n, cap, (char*)ws, out, out_cap,
                          ne, nbytes, herr, s);
}

hipError_t edits_decode(int dtype, const uint8_t* table, const uint8_t* payload,
                        int64_t payload_bytes, int64_t ne, int64_t n, void* g, int* err,
                        hipStream_t s) {
  const int64_t nch = (ne + kEditChunk - 1) / kEditChunk;
  if (nch == 0) return hipSuccess;
  if (dtype == PMSZ_F32)
    hipLaunchKernelGGL(k_edit_decode<float>, dim3((unsigned)nch), dim3(kDecThreads), 0, s, table,
                       payload, payload_bytes, ne, n, (float*)g, err);
  else
    hipLaunchKernelGGL(k_edit_decode<double>, dim3((unsigned)nch), dim3(kDecThreads), 0, s, table,
                       payload, payload_bytes, ne, n, (double*)g, err);
  return hipGetLastError();
}

}  // namespace pmsz
