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
// Encoding is a chain of data-parallel passes (find, scan, emit, scan, write);
// decoding runs one block per chunk of the table.
#include <string.h>

#include "launch.hpp"

namespace pmsz {

constexpr int kEditChunk = 4096;    // entries per chunk of the table

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

// Exclusive sum over the THREADS threads of a block; *total (all threads).
template <int THREADS, class V>
__device__ __forceinline__ V block_excl(V v, V* sh, V* total) {
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
  for (int w = 0; w < THREADS / 64; ++w) {
    const V t = sh[w];
    before += w < wave ? t : V(0);
    all += t;
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// ---- encoder passes ----------------------------------------------------------
// The field is cut into spans of kSpan vertices, one block each.
//   find    reads fhat and g once: a bit per changed vertex, and the span's
//           number of changes and last changed vertex
//   scan    rank of each span's first change, and the changed vertex before it
//   emit    gap and steps of every change (gathered from fhat and g at the set
//           bits), listed by rank; the span's payload bytes
//   scan    payload offset of each span
//   write   the listed entries as varints, the chunk table and the header
// Only `find` touches the whole field (2 values per vertex), so the encoder is
// bound by that read; the other passes move about 30 bytes per change and gather
// two lines of the fields for each.  Every load of `find` takes 64 consecutive
// values; count and compaction passes whose threads each took 16 consecutive
// values read the fields twice at 1.1 and 0.5 TB/s.  512^3 binary32, 1.8 M
// changes: find 203 us (5.3 TB/s), emit 81 us, scans 2 x 19 us, write 15 us;
// the call 3.39 ms before, 0.36 ms now.  Spans with many changes are listed word
// by word, and written several entries per thread at a time (a lane per list and one
// entry at a time: 2^18 binary32 values, all changed, 156 us; now 89 us).
constexpr int kSpan = 16384;            // vertices per block
constexpr int kWaveSpan = kSpan / 4;    // per wave: 64 ballots, one per lane
constexpr int kFindLoads = 8;           // ballots whose loads are in flight together
// Changes of 64 vertices that one lane of `emit` lists by itself.  Where the spans
// fill the chip the lanes that wait for the longest list cost their issue slots, else
// only the time of that list (2^27 binary32 values, a tenth changed: 1012 us at 32, 712
// at 12; 2^18: 60 and 76).
constexpr int kDenseWord = 32, kDenseWordFull = 12;
constexpr int64_t kFullSpans = 512;

struct EncSpan {
  uint32_t count, last;           // changes; last changed vertex + 1 (0: none)
  uint32_t rank, prev;            // changes before the span; the last one + 1
  unsigned long long bytes, off;  // payload bytes; those before the span
};
struct EncTotal {
  unsigned long long edits, bytes;
};

// Change bits of the 64 x 64 vertices of a wave's span: bit l of lane k's word
// is vertex v0 + 64 k + l.  Each load instruction reads 64 consecutive values.
template <class T>
__device__ __forceinline__ unsigned long long change_bits(const T* fhat, const T* g, int64_t n,
                                                          int64_t v0) {
  const gptr<const T> a = as_global(fhat);
  const gptr<const T> b = as_global(g);
  const int lane = threadIdx.x & 63;
  unsigned long long mine = 0;
  for (int k0 = 0; k0 < 64; k0 += kFindLoads) {
    if (v0 + 64 * (int64_t)k0 >= n) break;
    T x[kFindLoads], y[kFindLoads];
#pragma unroll
    for (int k = 0; k < kFindLoads; ++k) {
      const int64_t i = v0 + 64 * (k0 + k) + lane;
      const int64_t j = i < n ? i : n - 1;
      x[k] = a[j];
      y[k] = b[j];
    }
#pragma unroll
    for (int k = 0; k < kFindLoads; ++k) {
      const int64_t i = v0 + 64 * (k0 + k) + lane;
      const unsigned long long w = __ballot(i < n && bits_differ<T>(x[k], y[k]));
      if (lane == k0 + k) mine = w;
    }
  }
  return mine;
}

// MAP: the change bits are kept for `emit` (the workspace has room for them).
template <class T, bool MAP>
__global__ __launch_bounds__(256) void k_edit_find(const T* fhat, const T* g, int64_t n,
                                                   EncSpan* spans, unsigned long long* map) {
  __shared__ uint32_t s_cnt[4], s_last[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t v0 = (int64_t)blockIdx.x * kSpan + wave * kWaveSpan;
  const unsigned long long w = change_bits<T>(fhat, g, n, v0);
  if (MAP) as_global(map)[(int64_t)blockIdx.x * 256 + threadIdx.x] = w;
  uint32_t cnt = __popcll(w);
  uint32_t last = w ? (uint32_t)(v0 + 64 * lane + 64 - __clzll(w)) : 0u;
  for (int o = 32; o > 0; o >>= 1) {
    cnt += __shfl_xor(cnt, o, 64);
    const uint32_t l = __shfl_xor(last, o, 64);
    last = l > last ? l : last;
  }
  if (lane == 0) {
    s_cnt[wave] = cnt;
    s_last[wave] = last;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < 4; ++k) {
      cnt += s_cnt[k];
      last = s_last[k] > last ? s_last[k] : last;
    }
    spans[blockIdx.x].count = cnt;
    spans[blockIdx.x].last = last;
  }
}

// One block over all spans.  PASS 0: rank and prev from count and last, the
// number of changes to *total; PASS 1: off from bytes, their sum to *total.
template <int PASS>
__global__ __launch_bounds__(1024) void k_edit_scan(EncSpan* spans, int64_t ns, EncTotal* total) {
  __shared__ unsigned long long s_sum[16];
  __shared__ uint32_t s_max[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t per = (ns + 1023) / 1024;
  const int64_t b0 = threadIdx.x * per, b1 = b0 + per < ns ? b0 + per : ns;
  unsigned long long sum = 0;
  uint32_t top = 0;
  for (int64_t b = b0; b < b1; ++b) {
    if (PASS == 0) {
      sum += spans[b].count;
      top = spans[b].last > top ? spans[b].last : top;
    } else {
      sum += spans[b].bytes;
    }
  }
  unsigned long long x = sum;
  uint32_t m = top;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(x, o, 64);
    const uint32_t z = __shfl_up(m, o, 64);
    if (lane >= o) {
      x += y;
      m = z > m ? z : m;
    }
  }
  if (lane == 63) {
    s_sum[wave] = x;
    s_max[wave] = m;
  }
  // the largest `last` before this thread's spans
  uint32_t prev = __shfl_up(m, 1, 64);
  if (lane == 0) prev = 0;
  __syncthreads();
  unsigned long long run = x - sum, all = 0;
  for (int w = 0; w < 16; ++w) {
    if (w < wave) {
      run += s_sum[w];
      prev = s_max[w] > prev ? s_max[w] : prev;
    }
    all += s_sum[w];
  }
  for (int64_t b = b0; b < b1; ++b) {
    if (PASS == 0) {
      spans[b].rank = (uint32_t)run;
      spans[b].prev = prev;
      run += spans[b].count;
      prev = spans[b].last > prev ? spans[b].last : prev;
    } else {
      spans[b].off = run;
      run += spans[b].bytes;
    }
  }
  if (threadIdx.x == 0) {
    if (PASS == 0) total->edits = all;
    else total->bytes = all;
  }
}

// Lists the entries of a span by rank: index and steps (ranks at or past cap
// are dropped: the caller then writes no stream), and sums their varint
// lengths.
template <class T, bool MAP>
__global__ __launch_bounds__(256) void k_edit_emit(const T* fhat, const T* g, int64_t n,
                                                   EncSpan* spans, const unsigned long long* map,
                                                   uint32_t* idx, unsigned long long* steps,
                                                   int64_t cap, int dense_word) {
  __shared__ unsigned long long sh[4];
  __shared__ uint32_t s_last[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (spans[blockIdx.x].count == 0) {
    if (threadIdx.x == 0) spans[blockIdx.x].bytes = 0;
    return;
  }
  const int64_t v0 = (int64_t)blockIdx.x * kSpan + wave * kWaveSpan;
  const unsigned long long w = MAP ? as_global(map)[(int64_t)blockIdx.x * 256 + threadIdx.x]
                                   : change_bits<T>(fhat, g, n, v0);
  unsigned long long total;
  int64_t r = (int64_t)spans[blockIdx.x].rank +
              (int64_t)block_excl<256, unsigned long long>(__popcll(w), sh, &total);
  // the changed vertex before this thread's word (+ 1)
  uint32_t last = w ? (uint32_t)(v0 + 64 * lane + 64 - __clzll(w)) : 0u;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t l = __shfl_up(last, o, 64);
    if (lane >= o) last = l > last ? l : last;
  }
  if (lane == 63) s_last[wave] = last;
  uint32_t prev = __shfl_up(last, 1, 64);
  if (lane == 0) prev = 0;
  __syncthreads();
  // (in the branches, so that the first gathers do not wait for it)
  auto before = [&]() {
    const uint32_t p = spans[blockIdx.x].prev;
    prev = p > prev ? p : prev;
    for (int k = 0; k < wave; ++k) prev = s_last[k] > prev ? s_last[k] : prev;
  };
  const gptr<const T> a = as_global(fhat);
  const gptr<const T> b = as_global(g);
  unsigned long long len = 0;
  if (__ballot(__popcll(w) > dense_word)) {
    // many changes: word by word, a lane per bit
    before();
    const int32_t r0 = __builtin_amdgcn_readfirstlane((int)r);  // (below 2^31)
    uint32_t seen = 0, last_i = (uint32_t)__builtin_amdgcn_readfirstlane((int)prev);
    for (int k0 = 0; k0 < 64; k0 += kFindLoads) {
      unsigned long long word[kFindLoads], any = 0;
#pragma unroll
      for (int k = 0; k < kFindLoads; ++k) {
        word[k] = (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)w, k0 + k) |
                  (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(w >> 32), k0 + k)
                      << 32;
        any |= word[k];
      }
      if (any == 0) continue;
      T x[kFindLoads], y[kFindLoads];
#pragma unroll
      for (int k = 0; k < kFindLoads; ++k) {
        const int64_t i = v0 + 64 * (k0 + k) + lane;
        const int64_t j = i < n ? i : n - 1;
        x[k] = a[j];
        y[k] = b[j];
      }
#pragma unroll
      for (int k = 0; k < kFindLoads; ++k) {
        const int64_t i0 = v0 + 64 * (k0 + k);
        const unsigned long long below = word[k] & ((1ull << lane) - 1ull);
        if ((word[k] >> lane) & 1ull) {
          const uint32_t was = below ? (uint32_t)(i0 + 64 - __clzll(below)) : last_i;
          const unsigned long long st = order_key(x[k]) - order_key(y[k]);
          len += leb_len((unsigned long long)(i0 + lane - (int64_t)was)) + leb_len(st);
          const int64_t at = (int64_t)r0 + seen + __popcll(below);
          if (at < cap) {
            idx[at] = (uint32_t)(i0 + lane);
            steps[at] = st;
          }
        }
        if (word[k]) last_i = (uint32_t)(i0 + 64 - __clzll(word[k]));
        seen += __popcll(word[k]);
      }
    }
  } else {
    before();
    unsigned long long bits = w;
    while (bits) {
      const int64_t i = v0 + 64 * lane + (__ffsll(bits) - 1);
      bits &= bits - 1;
      const unsigned long long st = order_key(a[i]) - order_key(b[i]);
      len += leb_len((unsigned long long)(i - (int64_t)prev)) + leb_len(st);
      if (r < cap) {
        idx[r] = (uint32_t)i;
        steps[r] = st;
      }
      prev = (uint32_t)(i + 1);
      ++r;
    }
  }
  len = block_sum(len, sh);
  if (threadIdx.x == 0) spans[blockIdx.x].bytes = len;
}

__device__ __forceinline__ uint8_t* put_leb(uint8_t* p, unsigned long long v) {
  while (v >= 0x80ull) {
    *p++ = (uint8_t)(v | 0x80ull);
    v >>= 7;
  }
  *p++ = (uint8_t)v;
  return p;
}

// Header, table and payload.  Writes nothing when the edits exceed cap or the
// stream exceeds out_cap.
template <class T, int THREADS, int U>
__global__ __launch_bounds__(THREADS) void k_edit_write(const EncSpan* spans, const EncTotal* total,
                                                    const uint32_t* idx,
                                                    const unsigned long long* steps, int64_t n,
                                                    int64_t cap, unsigned long long out_cap,
                                                    uint8_t* out) {
  __shared__ unsigned long long sh[THREADS / 64];
  const unsigned long long ne = total->edits, nb = total->bytes;
  const unsigned long long nch = (ne + kEditChunk - 1) / kEditChunk;
  const unsigned long long head = 40 + 16 * nch;
  if (ne > (unsigned long long)cap || head + nb > out_cap) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    // (out is 8-byte aligned) magic, version, type; vertices; edits; payload
    // bytes; chunk and chunks
    unsigned long long* h = (unsigned long long*)out;
    h[0] = 0x45534D50ull | (1ull << 32) | ((unsigned long long)(sizeof(T) == 8) << 40);
    h[1] = (unsigned long long)n;
    h[2] = ne;
    h[3] = nb;
    h[4] = (unsigned long long)kEditChunk | (nch << 32);
  }
  // U entries per thread at a time: their lengths (at most 15 bytes) are scanned together,
  // in 16 bits each
  static_assert(THREADS * 15 < (1 << 16), "a sum of lengths fits its field");
  const EncSpan sp = spans[blockIdx.x];
  unsigned long long at = sp.off;
  for (uint32_t base = 0; base < sp.count; base += THREADS * U) {
    unsigned long long gap[U], st[U], lens = 0;
    uint32_t prev[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k0 = base + THREADS * u, k = k0 + threadIdx.x;
      prev[u] = 0;
      gap[u] = st[u] = 0;
      if (k0 >= sp.count) continue;
      const int64_t r = (int64_t)sp.rank + (k < sp.count ? k : k0);
      prev[u] = r ? idx[r - 1] + 1u : 0u;
      gap[u] = (unsigned long long)(idx[r] - prev[u]);
      st[u] = steps[r];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (base + THREADS * u + threadIdx.x < sp.count)
        lens |= (unsigned long long)(leb_len(gap[u]) + leb_len(st[u])) << (16 * u);
    unsigned long long all;
    const unsigned long long ex = block_excl<THREADS, unsigned long long>(lens, sh, &all);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t k = base + THREADS * u + threadIdx.x;
      const unsigned long long o = at + ((ex >> (16 * u)) & 0xffffull);
      if (k < sp.count) {
        put_leb(put_leb(out + head + o, gap[u]), st[u]);
        const int64_t r = (int64_t)sp.rank + k;
        if (r % kEditChunk == 0) {
          unsigned long long* t = (unsigned long long*)(out + 40 + 16 * (r / kEditChunk));
          t[0] = o;
          t[1] = prev[u] ? (unsigned long long)prev[u] - 1ull : ~0ull;
        }
      }
      at += (all >> (16 * u)) & 0xffffull;
    }
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
constexpr int kVarintMost = 10;                      // bytes of a 64-bit varint

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
  // a varint takes ten bytes at most: a payload of longer ones is read no further
  const int64_t most = 2 * kVarintMost * (int64_t)cnt;
  // the payload is 8-byte aligned, and so is every tile
  for (int64_t at = start & ~int64_t(7); found < 2 * cnt; at += kDecTile) {
    // the payload ends inside the chunk, or its entries cannot be this long
    if (at >= payload_bytes || at >= start + most) {
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
    int v = found + block_excl<kDecThreads, int>(mine, s_cnt, &all);  // (its barriers publish s_raw)
    if (mine && v < 2 * cnt) {
      // the part of this thread's first varint that lies before its bytes
      int p = kDecBytes + tid * kDecBytes;
      int q = p;
      while (p - q < 11 && q > 0 && (bytes[q - 1] & 0x80)) --q;
      unsigned long long x = 0;
      int len = 0;
      for (; q < p; ++q, ++len)
        if (len < kVarintMost) x |= (unsigned long long)(bytes[q] & 0x7f) << (7 * len);
      for (int k = 0; k < kDecBytes && mine > 0 && v < 2 * cnt; ++k) {
        const int64_t b = at + tid * kDecBytes + k;
        if (b < start) continue;
        const uint8_t y = bytes[p + k];
        if (len < kVarintMost) x |= (unsigned long long)(y & 0x7f) << (7 * len);
        ++len;
        if (y & 0x80) continue;
        bad |= len > kVarintMost;
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
  unsigned long long i = first + block_excl<kDecThreads, unsigned long long>(sum, s_sum, &all);
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
// Workspace: [spans][totals][index per edit][change bits, when an edit's four
// bytes of room per edit hold them][steps per edit].
struct EditLayout {
  size_t spans, total, idx, map, steps, bytes;
  int64_t nspans;
  bool keep_map;
};

static size_t al256(size_t v) { return (v + 255) / 256 * 256; }

static EditLayout edit_layout(int64_t n, int64_t cap) {
  EditLayout L;
  L.nspans = (n + kSpan - 1) / kSpan;
  const size_t c = (size_t)(cap > 0 ? cap : 1);
  const int64_t parts = (n + 4095) / 4096;
  const int64_t items = cap > parts ? cap : parts;
  L.spans = 0;
  // (12 bytes per 4096 vertices and 8 per 4096 edits or such parts, each
  // region a multiple of 256: room for a 32-byte span per 16384 vertices)
  const size_t room = al256(4 * (size_t)parts) + al256(8 * (size_t)parts) +
                      al256(8 * (size_t)((items + 4095) / 4096));
  L.total = L.spans + room;
  L.idx = L.total + 256;
  L.map = L.idx + al256(4 * c);
  L.steps = L.map + al256(4 * c);
  L.bytes = L.steps + al256(8 * c);
  L.keep_map = (size_t)L.nspans * (kSpan / 8) <= al256(4 * c);
  return L;
}

size_t edits_workspace_bytes(int64_t n, int64_t cap) { return edit_layout(n, cap).bytes; }

size_t edits_stream_bytes(int64_t ne) {
  const int64_t nch = (ne + kEditChunk - 1) / kEditChunk;
  return 40 + 16 * (size_t)nch + 15 * (size_t)ne;
}

// Returns 0, or 1 when the edits exceed cap (*ne set), or 2 when the stream
// does not fit out_cap (*nbytes set); hip errors through *herr.  Every pass is
// launched by the field's spans and reads the counts on the device, so the
// host waits once, for the totals.
template <class T>
static int encode_t(const T* fhat, const T* g, int64_t n, int64_t cap, char* ws, uint8_t* out,
                    size_t out_cap, int64_t* ne_out, int64_t* nbytes_out, hipError_t* herr,
                    hipStream_t s) {
  const EditLayout L = edit_layout(n, cap);
  EncSpan* spans = (EncSpan*)(ws + L.spans);
  EncTotal* total = (EncTotal*)(ws + L.total);
  uint32_t* idx = (uint32_t*)(ws + L.idx);
  unsigned long long* map = (unsigned long long*)(ws + L.map);
  unsigned long long* steps = (unsigned long long*)(ws + L.steps);
  const dim3 grid((unsigned)L.nspans), block(256);
  *herr = hipSuccess;
#define EDIT_TRY(x)                        \
  do {                                     \
    hipError_t e_ = (x);                   \
    if (e_ != hipSuccess) {                \
      *herr = e_;                          \
      return -1;                           \
    }                                      \
  } while (0)
  if (L.keep_map)
    hipLaunchKernelGGL((k_edit_find<T, true>), grid, block, 0, s, fhat, g, n, spans, map);
  else
    hipLaunchKernelGGL((k_edit_find<T, false>), grid, block, 0, s, fhat, g, n, spans, map);
  EDIT_TRY(hipGetLastError());
  hipLaunchKernelGGL(k_edit_scan<0>, dim3(1), dim3(1024), 0, s, spans, L.nspans, total);
  EDIT_TRY(hipGetLastError());
  const int dense_word = L.nspans < kFullSpans ? kDenseWord : kDenseWordFull;
  if (L.keep_map)
    hipLaunchKernelGGL((k_edit_emit<T, true>), grid, block, 0, s, fhat, g, n, spans,
                       (const unsigned long long*)map, idx, steps, cap, dense_word);
  else
    hipLaunchKernelGGL((k_edit_emit<T, false>), grid, block, 0, s, fhat, g, n, spans,
                       (const unsigned long long*)map, idx, steps, cap, dense_word);
  EDIT_TRY(hipGetLastError());
  hipLaunchKernelGGL(k_edit_scan<1>, dim3(1), dim3(1024), 0, s, spans, L.nspans, total);
  EDIT_TRY(hipGetLastError());
  // (more threads and entries per span where the spans leave the chip idle: the
  // call on 2^18 binary64 values, all changed, takes 110 us this way and 126 with 256
  // threads; on 2^27, one in 74 changed, 888 and 862)
  if (L.nspans < kFullSpans)
    hipLaunchKernelGGL((k_edit_write<T, 512, 4>), grid, dim3(512), 0, s, (const EncSpan*)spans,
                       (const EncTotal*)total, (const uint32_t*)idx,
                       (const unsigned long long*)steps, n, cap, (unsigned long long)out_cap, out);
  else
    hipLaunchKernelGGL((k_edit_write<T, 256, 2>), grid, block, 0, s, (const EncSpan*)spans,
                       (const EncTotal*)total, (const uint32_t*)idx,
                       (const unsigned long long*)steps, n, cap, (unsigned long long)out_cap, out);
  EDIT_TRY(hipGetLastError());
  EncTotal h = {0, 0};
  EDIT_TRY(hipMemcpyAsync(&h, total, sizeof(h), hipMemcpyDeviceToHost, s));
  EDIT_TRY(hipStreamSynchronize(s));
#undef EDIT_TRY
  *ne_out = (int64_t)h.edits;
  if ((int64_t)h.edits > cap) return 1;
  const int64_t nch = ((int64_t)h.edits + kEditChunk - 1) / kEditChunk;
  const size_t size = 40 + 16 * (size_t)nch + (size_t)h.bytes;
  *nbytes_out = (int64_t)size;
  return size > out_cap ? 2 : 0;
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
