// engine.hip -- the persistent correction kernel (gfx950).
//
// One cooperative launch runs the correction loop of Sec. IV-A for one or many
// fields, whose directions of f were computed beforehand (k_dirs_fields, or
// the caller).  Round E (p = E & 1, q = E % 3), for every field still running:
//   detect  directions of g^k, compared with the directions of f; targets are
//           set in the flag bitmap (Sec. IV-A ascending and descending rules,
//           Sec. III-B FPmax rule).  A field's first round sweeps all its
//           tiles and validates fhat; later rounds sweep only the tiles
//           within one vertex of last round's targets, or, when last round
//           flagged few vertices, examine exactly the Freudenthal neighbours
//           of those targets (sparse rounds).
//   barrier
//   apply   for fields with mismatches: count the flagged vertices (|F|) and
//           those already at their bound; unless the field is out of rounds,
//           give every flagged vertex above its bound one halving edit (Eq. 1),
//           list it for a sparse next round and mark the tiles within one
//           vertex of it active.  Either way only vertices whose mismatch can
//           be non-empty are examined, so the result is that of a full sweep.
//   barrier
// The decision of Sec. IV-A's loop (converged, stalled, out of rounds,
// continue) is a pure function of the state at the start of a round and that
// round's counters; every block evaluates it itself when it needs it, and
// block 0 persists it one round later, so no extra barrier is needed.  The
// loop ends when a round edits nothing (every field done) or after
// max_rounds rounds (resumable steps).
#include <map>
#include <mutex>

#include "engine.hpp"
#include "wave_tiles.hpp"

namespace pmsz {

// ---------------------------------------------------------------------------
// Grid barrier for a cooperative launch.  Each block's thread 0 releases its
// writes (one L2 write-back at agent scope) and arrives on one of kBarGroups
// group counters; the last arrival of a group resets it and arrives on the
// top counter, and the last arrival there resets that and publishes the next
// generation with a release store.  The other blocks poll the generation
// word, which no arrival touches, with relaxed loads (they read the coherent
// copy without touching the caches) and acquire once at the end (one cache
// invalidate), so the next phase sees every block's writes.  Spreading the
// arrivals keeps them from serialising on one address.  The spin is bounded:
// after ~4 s the block records an error and the launch winds down instead of
// hanging.
// ---------------------------------------------------------------------------
__device__ __forceinline__ unsigned relaxed_load(const unsigned* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long relaxed_load(const unsigned long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long relaxed_load(gptr<const unsigned long long> p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void relaxed_add(gptr<unsigned long long> p, unsigned long long v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A load of data that another compute unit may have written since this unit
// last invalidated its cache.  CO (the tail rounds of k_tail, below): a
// device-scope load, which skips the unit's cache and reads the XCD's L2 where
// every unit's stores and atomics land; otherwise a plain load (a grid
// barrier's acquire has invalidated the unit's cache).
template <bool CO, class V>
__device__ __forceinline__ V ld(gptr<const V> p) {
  if constexpr (CO) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}

__device__ __forceinline__ void grid_sync(EngineCtl* ctl, unsigned nblocks, unsigned& gen) {
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned target = gen + 1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned groups = nblocks < (unsigned)kBarGroups ? nblocks : (unsigned)kBarGroups;
    const unsigned grp = blockIdx.x % groups;
    const unsigned members = nblocks / groups + (grp < nblocks % groups ? 1u : 0u);
    bool last = false;
    const unsigned arrived =
        __hip_atomic_fetch_add(&ctl->bar[grp].v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (arrived == members - 1) {
      __hip_atomic_store(&ctl->bar[grp].v, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // acq_rel: the reset is ordered before this group's arrival, and the
      // final arrival orders every group's reset before its release below
      const unsigned top = __hip_atomic_fetch_add(&ctl->bar[kBarGroups].v, 1u, __ATOMIC_ACQ_REL,
                                                  __HIP_MEMORY_SCOPE_AGENT);
      if (top == groups - 1) {
        __hip_atomic_store(&ctl->bar[kBarGroups].v, 0u, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl->bar_gen.v, target, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        last = true;
      }
    }
    if (!last) {
      const unsigned long long t0 = wall_clock64();
      while (relaxed_load(&ctl->bar_gen.v) != target) {
        __builtin_amdgcn_s_sleep(1);
        if (wall_clock64() - t0 > 400000000ull) {  // 100 MHz counter: 4 s
          __hip_atomic_store(&ctl->error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    gen = target;
  }
  __syncthreads();
}

// Barrier after the start of a launch.  Release (making this block's writes
// visible to other XCDs) costs an L2 write-back of the whole XCD, so only the
// last block of each XCD to arrive performs it, after every block of that
// XCD has its writes completed in L2 (each wave waits for its stores before
// the block arrives).  Acquire (an invalidate of the compute unit's cache and
// of the XCD's L2) is needed once per compute unit: the blocks resident on
// one unit share its cache, so the first of them past the generation flip
// invalidates and the others wait until it has.  The L1-only invalidate
// does nothing outside thread-group-split mode, and an invalidate per block
// queues 128 of them per XCD (measured: 10.7 us per barrier at 1024 blocks
// against 6.2 us with one per unit).
struct XcdBar {
  unsigned xcc;      // XCD this block runs on
  unsigned members;  // blocks of the launch on it
  unsigned nx;       // XCDs with blocks of the launch
  unsigned cu;       // compute-unit slot: XCD x 256 + HW_ID bits 15:8
  unsigned rank;     // this block's index among the members (k_tail)
};

__device__ __forceinline__ unsigned xcd_of_block() {
  // hardware register XCC_ID, bits 3:0
  return __builtin_amdgcn_s_getreg((3 << 11) | 20) & (unsigned)(kXcdSlots - 1);
}
__device__ __forceinline__ unsigned cu_of_block(unsigned xcc) {
  // hardware register HW_ID, bits 15:8 (CU_ID, SH_ID, SE_ID)
  return xcc * 256u + (__builtin_amdgcn_s_getreg((7 << 11) | (8 << 6) | 4) & 255u);
}

// Bounded spin until *p == target: after ~4 s the block records an error and
// the launch winds down instead of hanging.
__device__ __forceinline__ void spin_until(EngineCtl* ctl, const unsigned* p, unsigned target) {
  const unsigned long long t0 = wall_clock64();
  while (relaxed_load(p) != target) {
    __builtin_amdgcn_s_sleep(1);
    if (wall_clock64() - t0 > 400000000ull) {  // 100 MHz counter: 4 s
      __hip_atomic_store(&ctl->error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
  }
}

__device__ __forceinline__ void xcd_sync(EngineCtl* ctl, const XcdBar& xb, unsigned& gen) {
  __builtin_amdgcn_s_waitcnt(0);  // this wave's stores are complete in L2
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned target = gen + 1;
    bool last = false;
    const unsigned arrived = __hip_atomic_fetch_add(&ctl->xbar[xb.xcc].v, 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
    if (arrived == xb.members - 1) {
      __hip_atomic_store(&ctl->xbar[xb.xcc].v, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // every block of this XCD has arrived: write its L2 back once
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      const unsigned top =
          __hip_atomic_fetch_add(&ctl->xtop.v, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
      if (top == xb.nx - 1) {
        __hip_atomic_store(&ctl->xtop.v, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&ctl->bar_gen.v, target, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        last = true;
      }
    }
    if (!last) spin_until(ctl, &ctl->bar_gen.v, target);
    // one invalidate per compute unit; generations only grow within a launch
    // and the slots are cleared before it, so a claim never matches a stale one
    const unsigned old = __hip_atomic_exchange(&ctl->cu_claim[xb.cu], target, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
    if (old != target) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      __builtin_amdgcn_s_waitcnt(0);  // the invalidate has completed
      __hip_atomic_store(&ctl->cu_done[xb.cu], target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      spin_until(ctl, &ctl->cu_done[xb.cu], target);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
    gen = target;
  }
  __syncthreads();
}

// Barrier of a sparse tail round (tail_round): only the blocks of one XCD
// are left, and every load of data that another unit may have written is a
// device-scope one (ld<true>), which skips the unit's cache and reads the
// XCD's L2.  The barrier then needs neither an L2 write-back nor an
// invalidate, only each wave's stores in L2 before its block arrives.  (An
// agent-scope acquire also drops the XCD's L2: every line read after it came
// from HBM at about 2 us, against about 0.12 us for a device-scope load that
// hits the L2, measured between two units of one XCD.)
__device__ __forceinline__ void tail_sync(EngineCtl* ctl, const XcdBar& xb, unsigned& gen) {
  __builtin_amdgcn_s_waitcnt(0);  // this wave's stores are complete in L2
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned target = gen + 1;
    const unsigned arrived = __hip_atomic_fetch_add(&ctl->xbar[xb.xcc].v, 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
    if (arrived == xb.members - 1) {
      __hip_atomic_store(&ctl->xbar[xb.xcc].v, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_s_waitcnt(0);  // the reset lands before any block passes
      __hip_atomic_store(&ctl->bar_gen.v, target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      spin_until(ctl, &ctl->bar_gen.v, target);
    }
    gen = target;
  }
  __syncthreads();
}

// Census of the launch's blocks per XCD (the XCD counters start cleared),
// ending with a full barrier.
__device__ __forceinline__ XcdBar xcd_census(EngineCtl* ctl, unsigned& gen) {
  XcdBar xb;
  xb.xcc = xcd_of_block();
  xb.cu = cu_of_block(xb.xcc);
  xb.rank = 0;
  if (threadIdx.x == 0)
    __hip_atomic_fetch_add(&ctl->census[xb.xcc], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  grid_sync(ctl, gridDim.x, gen);
  xb.members = __hip_atomic_load(&ctl->census[xb.xcc], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  xb.nx = 0;
  for (int i = 0; i < kXcdSlots; ++i)
    xb.nx += __hip_atomic_load(&ctl->census[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 1u
                                                                                            : 0u;
  return xb;
}

__device__ __forceinline__ bool engine_failed(EngineCtl* ctl) {
  return __hip_atomic_load(&ctl->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// Census of a tail launch (k_tail): block 0 publishes its XCD (the lead,
// where the tail runs), every block reads it and counts itself; the blocks of
// other XCDs then leave, and the lead's blocks wait until every block of the
// launch has counted itself, which fixes their number and their ranks (the
// counters start cleared).  Spins are bounded like the barriers'.  Returns
// false for a block that leaves.
__device__ __forceinline__ bool tail_census(EngineCtl* ctl, XcdBar& xb) {
  __shared__ unsigned s_info[3];  // XCD, rank among the lead XCD's blocks, their number
  if (threadIdx.x == 0) {
    const unsigned xcc = xcd_of_block();
    if (blockIdx.x == 0)
      __hip_atomic_store(&ctl->lead.v, xcc + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long t0 = wall_clock64();
    unsigned lead1;
    while ((lead1 = relaxed_load(&ctl->lead.v)) == 0u) {
      __builtin_amdgcn_s_sleep(1);
      if (wall_clock64() - t0 > 400000000ull) {  // 100 MHz counter: 4 s
        __hip_atomic_store(&ctl->error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
    }
    const unsigned lead = lead1 - 1u;
    unsigned rank = ~0u, members = 0u;
    if (lead1 != 0u && xcc == lead)
      rank = __hip_atomic_fetch_add(&ctl->census[lead], 1u, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
    // counted after the census word (whose add has returned)
    __hip_atomic_fetch_add(&ctl->arrived.v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (rank != ~0u) {
      spin_until(ctl, &ctl->arrived.v, gridDim.x);
      members = relaxed_load(&ctl->census[lead]);
    }
    s_info[0] = xcc;
    s_info[1] = rank;
    s_info[2] = members;
  }
  __syncthreads();
  xb.xcc = s_info[0];
  xb.rank = s_info[1];
  xb.members = s_info[2];
  xb.nx = 1;
  xb.cu = 0;
  return xb.rank != ~0u && !engine_failed(ctl);
}


// Field owning global tile / segment v (fields sorted by base).
__device__ __forceinline__ int field_of_tile(const FieldDesc* fd, int nf, int64_t v) {
  int lo = 0, hi = nf - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (fd[mid].tile_base <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ int field_of_seg(const FieldDesc* fd, int nf, int64_t v) {
  int lo = 0, hi = nf - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (fd[mid].seg_base <= v) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// The loop decision of Sec. IV-A: state at the start of the next round from
// the state at the start of this round and this round's counters.
__device__ __forceinline__ FieldIter next_state(FieldIter s, const CtrSum& c,
                                                int64_t max_iters) {
  if (s.done) return s;
  const bool first = !s.started;
  s.started = 1;
  s.swept += c.swept;
  if (first) s.mism0 = c.mism;
  s.flagged_final = c.nflag;
  s.stalled_final = c.at_lb;
  if (first && (c.bad_nf || c.bad_b)) {
    s.done = 1;
    s.status = c.bad_nf ? PMSZ_ERR_NONFINITE : PMSZ_ERR_INPUT_BOUND;
    s.mism0 = s.flagged_final = s.stalled_final = 0;
  } else if (c.mism == 0) {
    s.done = 1;
    s.status = PMSZ_OK;
  } else if (c.at_lb == c.nflag) {
    s.done = 1;
    s.status = PMSZ_ERR_STALLED;
  } else if ((long long)s.k >= max_iters) {
    s.done = 1;
    s.status = PMSZ_ERR_NOT_CONVERGED;
  } else {
    s.k += 1;
    s.steps += c.nflag - c.at_lb;
    s.flagged_final = s.stalled_final = 0;
  }
  return s;
}

// Whole-struct copies through global-space pointers, member by member (the
// implicit copy operations take generic references).
template <bool CO = false>
__device__ __forceinline__ FieldIter load_iter(gptr<const FieldIter> p) {
  FieldIter r;
  r.k = ld<CO>(&p->k);
  r.steps = ld<CO>(&p->steps);
  r.mism0 = ld<CO>(&p->mism0);
  r.flagged_final = ld<CO>(&p->flagged_final);
  r.stalled_final = ld<CO>(&p->stalled_final);
  r.swept = ld<CO>(&p->swept);
  r.status = ld<CO>(&p->status);
  r.done = ld<CO>(&p->done);
  r.started = ld<CO>(&p->started);
  r.pad = ld<CO>(&p->pad);
  return r;
}
__device__ __forceinline__ void store_iter(gptr<FieldIter> p, const FieldIter& s) {
  p->k = s.k;
  p->steps = s.steps;
  p->mism0 = s.mism0;
  p->flagged_final = s.flagged_final;
  p->stalled_final = s.stalled_final;
  p->swept = s.swept;
  p->status = s.status;
  p->done = s.done;
  p->started = s.started;
  p->pad = s.pad;
}
__device__ __forceinline__ void clear_ctr(gptr<FieldCtr> c) {
  for (int k = 0; k < kCtrSlots; ++k) {
    const gptr<CtrSlot> x = &c->s[k];
    x->mism = x->nflag = x->at_lb = x->bad_nf = x->bad_b = x->swept = x->nlist = 0;
  }
}

// Counter slot of this block.
__device__ __forceinline__ int ctr_slot() { return (int)(blockIdx.x % (unsigned)kCtrSlots); }

// Counters of a finished round, summed over the slots.  They are read only
// after the grid barrier that completed them, whose acquire invalidated this
// unit's caches, so plain loads see the final values; plain loads also let
// the unit's cache serve the blocks that share it (every block of the grid
// reads the same few lines after each barrier, and one L2 channel serves
// each line).
template <bool CO = false>
__device__ __forceinline__ CtrSum load_ctr(gptr<const FieldCtr> c) {
  CtrSum r{0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int k = 0; k < kCtrSlots; ++k) {
    const gptr<const CtrSlot> x = &c->s[k];
    r.mism += ld<CO>(&x->mism);
    r.nflag += ld<CO>(&x->nflag);
    r.at_lb += ld<CO>(&x->at_lb);
    r.bad_nf += ld<CO>(&x->bad_nf);
    r.bad_b += ld<CO>(&x->bad_b);
    r.swept += ld<CO>(&x->swept);
    r.nlist += ld<CO>(&x->nlist);
  }
  return r;
}
// Mismatches of a finished round (the apply pass's only test in later rounds).
template <bool CO = false>
__device__ __forceinline__ unsigned long long load_mism(gptr<const FieldCtr> c) {
  unsigned long long m = 0;
#pragma unroll
  for (int k = 0; k < kCtrSlots; ++k) m += ld<CO>(&c->s[k].mism);
  return m;
}

// Round totals over all fields, summed over the slots (read after the barrier
// that completed them, like the counters).
template <bool CO = false>
__device__ __forceinline__ RoundTot load_tot(const EngineCtl* ctl, int q) {
  RoundTot r{0, 0, 0, 0, {0, 0, 0, 0}};
  const gptr<const RoundTot> t = as_global(&ctl->tot[q][0]);
#pragma unroll
  for (int k = 0; k < kCtrSlots; ++k) {
    r.edits += ld<CO>(&t[k].edits);
    r.swept += ld<CO>(&t[k].swept);
    r.sparse += ld<CO>(&t[k].sparse);
    r.flagged += ld<CO>(&t[k].flagged);
  }
  return r;
}
template <bool CO = false>
__device__ __forceinline__ unsigned long long load_edits(const EngineCtl* ctl, int q) {
  const gptr<const RoundTot> t = as_global(&ctl->tot[q][0]);
  unsigned long long e = 0;
#pragma unroll
  for (int k = 0; k < kCtrSlots; ++k) e += ld<CO>(&t[k].edits);
  return e;
}

// State of a field at the start of round E.
template <bool CO = false>
__device__ __forceinline__ FieldIter state_at(const FieldDesc& d, unsigned long long E,
                                              unsigned long long E0) {
  const gptr<const FieldState> st = as_global((const FieldState*)d.st);
  if (E == E0) return load_iter<CO>(&st->s[E & 1]);
  return next_state(load_iter<CO>(&st->s[(E - 1) & 1]), load_ctr<CO>(&st->c[(E - 1) % 3]),
                    d.max_iters);
}

// Tiles containing a vertex within one step of target t (Freudenthal
// neighbours lie in the 3x3x3 box around t).
struct TileBox {
  int32_t x0, x1, y0, y1, z0, z1;
};

__device__ __forceinline__ TileBox box_of(const TileGeo& G, int32_t t) {
  TileBox b;
  const int32_t row = fdiv(t, G.div_nx);  // y + ny z
  const int32_t x = t - row * G.nx;
  const int32_t xl = x > 0 ? x - 1 : 0, xh = x + 1 < G.nx ? x + 1 : x;
  if (G.ndim == 3) {
    const int32_t z = fdiv(row, G.div_ny), y = row - z * G.ny;
    const int32_t yl = y > 0 ? y - 1 : 0, yh = y + 1 < G.ny ? y + 1 : y;
    const int32_t zl = z > 0 ? z - 1 : 0, zh = z + 1 < G.nz ? z + 1 : z;
    b = {xl / TX, xh / TX, yl / TY, yh / TY, fdiv(zl, G.div_chunk), fdiv(zh, G.div_chunk)};
  } else {
    const int32_t y = row;
    const int32_t yl = y > 0 ? y - 1 : 0, yh = y + 1 < G.ny ? y + 1 : y;
    b = {xl / RX, xh / RX, fdiv(yl, G.div_chunk), fdiv(yh, G.div_chunk), 0, 0};
  }
  return b;
}

// Plain byte stores into the field's activity bytes of the next round: every
// writer stores the same value.  The box spans at most two tiles per axis
// (tile boundaries lie at least two vertices apart), so its tiles are the
// eight corner combinations, duplicates included; all eight bytes are loaded
// before any store, so the loads overlap instead of forming a chain of
// dependent round trips (a store may alias a later load of the same array).
template <bool CO = false>
__device__ __forceinline__ void mark_box(const FieldDesc& d, const TileBox& b, gptr<uint8_t> nxt) {
  int32_t idx[8];
  uint8_t cur[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int32_t bx = (k & 1) ? b.x1 : b.x0, by = (k & 2) ? b.y1 : b.y0,
                  bz = (k & 4) ? b.z1 : b.z0;
    idx[k] = bx + d.geo.tiles_x * (by + d.geo.tiles_y * bz);
    // (the tail stores without reading: its few edits gain more from one
    // round trip less than from the stores a read saves)
    cur[k] = CO ? uint8_t(0) : ld<CO>(nxt + idx[k]);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (!cur[k]) nxt[idx[k]] = 1;
}

// Exclusive prefix sum over the block; *total receives the sum (all threads).
__device__ __forceinline__ int block_scan(int v, int* sh, int* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wave] = x;
  __syncthreads();
  int before = 0, all = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < wave) before += sh[w];
    all += sh[w];
  }
  __syncthreads();
  *total = all;
  return before + x - v;
}

// ---------------------------------------------------------------------------
// Sparse rounds.  A vertex whose mismatch set is non-empty in round E+1 is a
// Freudenthal neighbour of some vertex flagged in round E: either one of its
// neighbours was edited, or nothing around it changed and it flags the same
// target as before, which lies in its own neighbourhood.  So when round E
// flagged few vertices, examining the neighbours of exactly those (the apply
// pass lists them) gives the same flag set as any sweep that covers them.
// Duplicated examinations only repeat idempotent flag writes; the mismatch
// count is then an over-count, which is only ever tested against zero after
// a field's first round.
// ---------------------------------------------------------------------------

// Examinations needed by round E of a field in a sparse round, or -1 when the
// round sweeps its active tiles (first round, or a slot's slice of the target
// list overflowed).  cnt (nullable) receives the targets listed per slot.
template <bool CO = false>
__device__ __forceinline__ long long sparse_items(const FieldDesc& d, const FieldIter& s,
                                                  unsigned long long E, uint32_t* cnt = nullptr) {
  if (!s.started || s.done) return -1;
  const gptr<const FieldCtr> c = &as_global((const FieldState*)d.st)->c[(E + 2) % 3];
  const unsigned long long cap = (unsigned long long)(d.list_cap / list_slices(d.words));
  unsigned long long n = 0;
  bool over = false;
#pragma unroll
  for (int k = 0; k < kCtrSlots; ++k) {
    const unsigned long long nk = ld<CO>(&c->s[k].nlist);
    over |= nk > cap;
    n += nk;
    if (cnt) cnt[k] = (uint32_t)nk;
  }
  if (over) return -1;
  return (long long)n * (d.geo.ndim == 3 ? 15 : 7);
}

// The same count from list lengths loaded beforehand (nk, by load_nlist,
// whose loads then overlap those of the field's state: the tail).
__device__ __forceinline__ long long sparse_items_of(const FieldDesc& d, const FieldIter& s,
                                                     const unsigned long long* nk,
                                                     uint32_t* cnt) {
  if (!s.started || s.done) return -1;
  const unsigned long long cap = (unsigned long long)(d.list_cap / list_slices(d.words));
  unsigned long long n = 0;
  bool over = false;
#pragma unroll
  for (int k = 0; k < kCtrSlots; ++k) {
    over |= nk[k] > cap;
    n += nk[k];
    cnt[k] = (uint32_t)nk[k];
  }
  if (over) return -1;
  return (long long)n * (d.geo.ndim == 3 ? 15 : 7);
}

// List lengths of round E's sparse examination (the previous round's apply
// pass appended the targets), device-scope loads.
__device__ __forceinline__ void load_nlist(const FieldDesc& d, unsigned long long E,
                                           unsigned long long* nk) {
  const gptr<const FieldCtr> c = &as_global((const FieldState*)d.st)->c[(E + 2) % 3];
#pragma unroll
  for (int k = 0; k < kCtrSlots; ++k) nk[k] = ld<true>(&c->s[k].nlist);
}

// Signed vertex offset of a direction code.
__device__ __forceinline__ int32_t code_offset(const TileGeo& G, int code) {
  const int m = code & 7;
  const int32_t o = (m & 1) + ((m >> 1) & 1) * G.nx + ((m >> 2) & 1) * G.sxy;
  return (code & 8) ? -o : o;
}

// Directions of g at vertex v from gathered values: the same upper / lower
// box pair merges, in the same order, as the tile marches.
template <class T, bool CO = false>
__device__ __forceinline__ void gather_dirs(const TileGeo& G, gptr<const T> g, int32_t v,
                                            int32_t x, int32_t y, int32_t z, int& ca, int& cd) {
  const T nan = T(__builtin_nan(""));
  const bool xm = x > 0, xp = x + 1 < G.nx;
  if (G.ndim == 3) {
    const bool ym = y > 0, yp = y + 1 < G.ny, zm = z > 0, zp = z + 1 < G.nz;
    auto up = [&](int bx, int by, int bz) {
      const bool ok = (!bx || xp) && (!by || yp) && (!bz || zp);
      const T val = ok ? ld<CO>(g + (v + bx + by * G.nx + bz * G.sxy)) : nan;
      return ext_of(val, bx | (by << 1) | (bz << 2));
    };
    auto dn = [&](int bx, int by, int bz) {  // vertex v - (1-bx, 1-by, 1-bz)
      const int mx = 1 - bx, my = 1 - by, mz = 1 - bz, m = mx | (my << 1) | (mz << 2);
      const bool ok = (!mx || xm) && (!my || ym) && (!mz || zm);
      const T val = ok ? ld<CO>(g + (v - mx - my * G.nx - mz * G.sxy)) : nan;
      return ext_of(val, m ? (8 | m) : 0);
    };
    const Ext<T> U = merge_up(merge_up(merge_up(up(0, 0, 0), up(1, 0, 0)),
                                       merge_up(up(0, 1, 0), up(1, 1, 0))),
                              merge_up(merge_up(up(0, 0, 1), up(1, 0, 1)),
                                       merge_up(up(0, 1, 1), up(1, 1, 1))));
    const Ext<T> L = merge_dn(merge_dn(merge_dn(dn(0, 0, 0), dn(1, 0, 0)),
                                       merge_dn(dn(0, 1, 0), dn(1, 1, 0))),
                              merge_dn(merge_dn(dn(0, 0, 1), dn(1, 0, 1)),
                                       merge_dn(dn(0, 1, 1), dn(1, 1, 1))));
    const Ext<T> e = merge_up(L, U);
    ca = e.ca;
    cd = e.cd;
  } else {
    const bool ym = y > 0, yp = y + 1 < G.ny;
    auto up = [&](int bx, int by) {
      const bool ok = (!bx || xp) && (!by || yp);
      return ext_of(ok ? ld<CO>(g + (v + bx + by * G.nx)) : nan, bx | (by << 1));
    };
    auto dn = [&](int bx, int by) {
      const int mx = 1 - bx, my = 1 - by, m = mx | (my << 1);
      const bool ok = (!mx || xm) && (!my || ym);
      return ext_of(ok ? ld<CO>(g + (v - mx - my * G.nx)) : nan, m ? (8 | m) : 0);
    };
    const Ext<T> U = merge_up(merge_up(up(0, 0), up(1, 0)), merge_up(up(0, 1), up(1, 1)));
    const Ext<T> L = merge_dn(merge_dn(dn(0, 0), dn(1, 0)), merge_dn(dn(0, 1), dn(1, 1)));
    const Ext<T> e = merge_up(L, U);
    ca = e.ca;
    cd = e.cd;
  }
}

// Examination m of a sparse round: neighbour m % per of the target m / per
// listed by the previous round's apply pass (cnt: targets per list slice).
// Returns the targets the examined vertex flags (-1: none) and its number of
// mismatches.
struct Exam {
  int32_t ta, td;  // ascending-rule and descending-rule targets
  unsigned n;      // mismatches found (0, 1 or 2)
};

template <class T, bool CO = false>
__device__ __forceinline__ Exam sparse_examine(const FieldDesc& d, uint32_t m,
                                               const uint32_t* cnt) {
  const TileGeo& G = d.geo;
  const bool three = G.ndim == 3;
  const uint32_t k = three ? m / 15u : m / 7u;
  const uint32_t j = m - k * (three ? 15u : 7u);
  // the slice holding the k-th listed target
  uint32_t kk = k, at = 0;
  const uint32_t slice = (uint32_t)(d.list_cap / list_slices(d.words));
#pragma unroll
  for (int i = 0; i < kCtrSlots - 1; ++i) {
    const uint32_t ci = cnt[i];
    const bool past = at == (uint32_t)i * slice && kk >= ci;
    kk -= past ? ci : 0u;
    at += past ? slice : 0u;
  }
  const int32_t t = (int32_t)ld<CO>(as_global((const uint32_t*)d.list) + (at + kk));
  // the vertex itself, then its neighbours: 3D codes 1..7, 9..15; 2D 1..3, 9..11
  const int code = three ? (j < 8 ? (int)j : (int)j + 1) : (j < 4 ? (int)j : (int)j + 5);
  // the neighbour's offset
  const int mm = code & 7;
  const int sg = (code & 8) ? -1 : 1;
  const int32_t row = fdiv(t, G.div_nx);  // y + ny z
  const int32_t x = t - row * G.nx;
  const int32_t z = three ? fdiv(row, G.div_ny) : 0;
  const int32_t y = row - z * G.ny;
  const int32_t X = x + sg * (mm & 1), Y = y + sg * ((mm >> 1) & 1), Z = z + sg * ((mm >> 2) & 1);
  Exam ex{-1, -1, 0u};
  // only vertices of the detection box are examined (it lies inside the grid)
  if (X < G.cx0 || X >= G.cx1 || Y < G.cy0 || Y >= G.cy1 || Z < G.cz0 || Z >= G.cz1) return ex;
  const int32_t v = t + code_offset(G, code);
  int ca, cd;
  gather_dirs<T, CO>(G, as_global((const T*)d.g), v, X, Y, Z, ca, cd);
  const int d8 = as_global(d.dirs)[v];
  const int fa = d8 & 15, fd = d8 >> 4;
  // targets are neighbours of v, inside the box for directions made by the
  // direction pass; the range check only guards the bitmap
  const gptr<const T> g = as_global((const T*)d.g);
  if (ca != fa) {
    const int32_t tt = v + code_offset(G, ca);
    if ((uint32_t)tt < (uint32_t)G.n) {
      ex.ta = tt;
      if (d.prop) {
        const int32_t c = v + code_offset(G, fa);
        propose<T>(d.prop, tt, c, ld<CO>(g + c));
      }
    }
    ++ex.n;
  }
  if (cd != fd) {
    const int32_t tt = v + code_offset(G, fd);
    if ((uint32_t)tt < (uint32_t)G.n) {
      ex.td = tt;
      if (d.prop) {
        const int32_t r = v + code_offset(G, cd);
        propose<T>(d.prop, tt, r, ld<CO>(g + r));
      }
    }
    ++ex.n;
  }
  return ex;
}

// Per-thread running count for one field at a time, added to the field's
// counter when the thread moves to another field; `acc_flush` then adds the
// rest with one atomic per block when all threads agree on the field.
struct FieldAcc {
  int f = -1;
  unsigned long long n = 0;
};
template <class Ptr>
__device__ __forceinline__ void acc_add(FieldAcc& acc, int fi, unsigned long long v, Ptr ptr) {
  if (fi != acc.f) {
    if (acc.n) relaxed_add(ptr(acc.f), acc.n);
    acc.f = fi;
    acc.n = 0;
  }
  acc.n += v;
}
// Whole block.  sf (4 ints) and sn (4 counts) are LDS scratch; the caller
// synchronises the block before reusing them.
template <class Ptr>
__device__ __forceinline__ void acc_flush(FieldAcc& acc, Ptr ptr, int* sf,
                                          unsigned long long* sn) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int f0 = acc.n ? acc.f : -1;
  for (int off = 32; off > 0; off >>= 1) f0 = max(f0, __shfl_xor(f0, off, 64));
  const bool agree = __all(acc.f == f0 || acc.n == 0);
  if (!agree && acc.n) relaxed_add(ptr(acc.f), acc.n);
  const unsigned long long w = wave_sum(agree ? acc.n : 0ull);
  if (lane == 0) {
    sf[wave] = (agree && w) ? f0 : -1;
    sn[wave] = w;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 0; i < 4; ++i) {
      if (sf[i] < 0) continue;
      unsigned long long t = sn[i];
      for (int j = i + 1; j < 4; ++j)
        if (sf[j] == sf[i]) {
          t += sn[j];
          sf[j] = -1;
        }
      relaxed_add(ptr(sf[i]), t);
    }
  }
  acc.f = -1;
  acc.n = 0;
}

// Inclusive prefix sums of one value per thread into s_pre; returns the
// total (all threads).  Scans within each wave with shuffles, then adds the
// totals of the waves before it.
__device__ __forceinline__ long long block_prefix(long long v, long long* s_pre) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  long long x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_pre[wave] = x;
  __syncthreads();
  long long before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const long long t = s_pre[w];
    before += w < wave ? t : 0;
    all += t;
  }
  __syncthreads();
  s_pre[tid] = before + x;
  __syncthreads();
  return all;
}
// First entry of s_pre[0..n) exceeding m.
__device__ __forceinline__ int prefix_find(const long long* s_pre, int n, long long m) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (s_pre[mid] > m) hi = mid; else lo = mid + 1;
  }
  return lo;
}

constexpr int kApplyCap = 2048;   // targets per compaction pass
constexpr int kEditUnroll = 2;    // targets per thread with loads in flight together

// Apply pass over bitmap words [w0, w1) of one field: the block reads the
// segment in one sweep (16 words per thread), compacts the set bits into an
// LDS list, and edits the listed targets with all threads at once.
template <class T, bool CO = false>
__device__ __forceinline__ void apply_segment(const FieldDesc& d, int32_t w0, int32_t w1,
                                              bool edit, gptr<uint8_t> nxt, uint32_t* list,
                                              int* scan, long long* lbase_sh, gptr<FieldCtr> cq,
                                              gptr<uint32_t> tlist, unsigned long long& nflag,
                                              unsigned long long& at_lb,
                                              unsigned long long& edits) {
  constexpr int kPer = 16;
  const int tid = threadIdx.x;
  // list slice of this segment (its counter slot for the list length)
  const int nls = list_slices(d.words);
  const int slot = (int)((w0 / kSegWords) % nls);
  const long long slice = d.list_cap / nls;
  // thread t owns words w0 + t + 256 k: each load instruction reads 256
  // consecutive words across the block
  const gptr<uint32_t> bm = as_global(d.bm);
  uint32_t wv[kPer];
  int cnt = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int32_t w = w0 + tid + 256 * k;
    wv[k] = ld<CO>(bm + (w < w1 ? w : w0));
    if (w >= w1) wv[k] = 0u;
    cnt += __popc(wv[k]);
  }
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (wv[k]) bm[w0 + tid + 256 * k] = 0u;
  nflag += (unsigned)cnt;
  int total = 0;
  const int off = block_scan(cnt, scan, &total);
  const gptr<const T> f = as_global((const T*)d.f);
  const gptr<T> g = as_global((T*)d.g);
  const T xi = (T)d.xi_t;
  TileBox last{-1, -1, -1, -1, -1, -1};  // the tile box this thread marked last
  for (int base = 0; base < total; base += kApplyCap) {
    int o = off;
    if (o < base + kApplyCap && o + cnt > base) {
#pragma unroll
      for (int k = 0; k < kPer; ++k) {
        uint32_t bits = wv[k];
        while (bits) {
          const int b = __ffs(bits) - 1;
          bits &= bits - 1;
          if (o >= base && o < base + kApplyCap)
            list[o - base] = (uint32_t)((w0 + tid + 256 * k) * 32 + b);
          ++o;
        }
      }
    }
    const int n = total - base < kApplyCap ? total - base : kApplyCap;
    // In the tail, the first targets' gathers (below) go out before the
    // list-slot atomic, so that the two round trips overlap.
    int32_t t0[kEditUnroll];
    T gt0[kEditUnroll], ft0[kEditUnroll];
    if constexpr (CO) {
      lds_barrier();  // the list is complete
      if (tid < n) {
#pragma unroll
        for (int u = 0; u < kEditUnroll; ++u) {
          const int j = tid + 256 * u;
          t0[u] = (int32_t)list[j < n ? j : tid];
        }
#pragma unroll
        for (int u = 0; u < kEditUnroll; ++u) {
          gt0[u] = ld<CO>(g + t0[u]);
          ft0[u] = f[t0[u]];
        }
      }
    }
    // room in this block's slice of the field's target list for this pass
    // (next round's sparse examination); entries past the slice are
    // dropped, and the count then sends the next round to a tile sweep
    if (edit && tid == 0 && n > 0)
      *lbase_sh = (long long)__hip_atomic_fetch_add(&cq->s[slot].nlist, (unsigned long long)n,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    lds_barrier();
    const long long lbase = edit ? *lbase_sh : 0;
    // kEditUnroll targets per thread at a time: their loads are all issued
    // before any of their stores (the targets are distinct vertices), so a
    // thread keeps several gathers in flight instead of one dependent chain
    // per target
    for (int j0 = tid; j0 < n; j0 += 256 * kEditUnroll) {
      int32_t t[kEditUnroll];
      T gt[kEditUnroll], ft[kEditUnroll];
      if (CO && j0 == tid) {
#pragma unroll
        for (int u = 0; u < kEditUnroll; ++u) {
          t[u] = t0[u];
          gt[u] = gt0[u];
          ft[u] = ft0[u];
        }
      } else {
#pragma unroll
        for (int u = 0; u < kEditUnroll; ++u) {
          const int j = j0 + 256 * u;
          t[u] = (int32_t)list[j < n ? j : j0];
        }
#pragma unroll
        for (int u = 0; u < kEditUnroll; ++u) {
          gt[u] = ld<CO>(g + t[u]);
          ft[u] = f[t[u]];
        }
      }
#pragma unroll
      for (int u = 0; u < kEditUnroll; ++u) {
        const int j = j0 + 256 * u;
        if (j >= n) break;
        const T lb = lower_bound<T>(ft[u], xi);
        const bool above = gt[u] > lb;
        if (d.prop) {
          // targeted edit: the smallest proposal, never below the bound; the
          // proposal slot is reset for the next round
          using K = decltype(prop_key(gt[u]));
          const gptr<K> slot = (gptr<K>)d.prop + t[u];
          if (above && edit) {
            const T pv = prop_value(ld<CO>(slot));
            g[t[u]] = pv > lb ? pv : lb;
          }
          *slot = ~K(0);
        } else if (above && edit) {
          g[t[u]] = halving_edit<T>(gt[u], lb);
        }
        edits += (above && edit) ? 1u : 0u;
        at_lb += above ? 0u : 1u;
        if (edit && lbase + j < slice) tlist[(int64_t)slot * slice + lbase + j] = (uint32_t)t[u];
      }
      if (edit) {
#pragma unroll
        for (int u = 0; u < kEditUnroll; ++u) {
          if (j0 + 256 * u >= n) break;
          // a thread's successive targets lie a few rows apart in a dense
          // round and mostly share their tile box, whose marks are then set
          // already (marks of this round's parity are only ever set here)
          const TileBox b = box_of(d.geo, t[u]);
          if (b.x0 != last.x0 || b.x1 != last.x1 || b.y0 != last.y0 || b.y1 != last.y1 ||
              b.z0 != last.z0 || b.z1 != last.z1) {
            mark_box<CO>(d, b, nxt);
            last = b;
          }
        }
      }
    }
    lds_barrier();
  }
}

// Tile part of round E's detect: the block examines the active tiles among
// first, first + G, first + 2G, ... (activity bytes of round parity E & 1,
// read and cleared 256 at a time, one per thread, and the active ones
// listed); SETS planes are in flight per tile march.
// A block's detect counts for one field, added once per field change.
__device__ __forceinline__ void flush_counts(gptr<CtrSlot> c, unsigned long long m,
                                             unsigned long long nf, unsigned long long nb,
                                             unsigned long long sw, unsigned long long* all_sw) {
  if (m) relaxed_add(&c->mism, m);
  if (nf) relaxed_add(&c->bad_nf, nf);
  if (nb) relaxed_add(&c->bad_b, nb);
  if (sw) {
    relaxed_add(&c->swept, sw);
    atomicAdd(all_sw, sw);
  }
}

// Tile detection of round E over the grid's share of the tiles, each field by
// its state.
template <class T, int SETS>
__device__ void detect_tiles(const EngineArgs& a, TileLds<T>& sm, unsigned long long* red,
                             uint16_t* s_tiles, int* s_scan, unsigned long long* s_acc,
                             unsigned long long E, unsigned long long E0, int64_t first,
                             unsigned G) {
  const int tid = threadIdx.x;
  const int p = (int)(E & 1);
  const int q = (int)(E % 3);
  EngineCtl* ctl = a.ctl;
  // the current field's counts, kept by thread 0 in LDS (registers are the
  // tile march's)
  unsigned long long &acc_m = s_acc[0], &acc_nf = s_acc[1], &acc_nb = s_acc[2],
                     &acc_sw = s_acc[3];
  if (tid == 0) acc_m = acc_nf = acc_nb = acc_sw = 0;
  int cur = -1, cached = -1, cached_kind = -1;
  for (int64_t base = first; base < a.total_tiles; base += (int64_t)G * 256) {
    const int64_t mine = base + (int64_t)tid * G;
    int take = 0;
    if (mine < a.total_tiles) {
      const FieldDesc& d = a.fd[field_of_tile(a.fd, a.nf, mine)];
      const gptr<uint8_t> flag = as_global(d.act) + p * tile_count(d.geo) + (mine - d.tile_base);
      if (*flag) {
        *flag = 0;
        take = 1;
      }
    }
    int n_act = 0;
    const int pos = block_scan(take, s_scan, &n_act);
    if (take) s_tiles[pos] = (uint16_t)tid;
    __syncthreads();
    for (int j = 0; j < n_act; ++j) {
      // uniform over the block: read once and kept in scalar registers
      const int64_t tt = base + (int64_t)__builtin_amdgcn_readfirstlane(s_tiles[j]) * G;
      const int fi = field_of_tile(a.fd, a.nf, tt);
      if (fi != cached) {
        const FieldIter s = state_at(a.fd[fi], E, E0);
        cached = fi;
        cached_kind = (s.done || sparse_items(a.fd[fi], s, E) >= 0) ? -1
                    : s.started ? KIND_NEXT : KIND_FIRST_GIVEN;
      }
      const int kind = cached_kind;
      if (kind < 0) continue;
      const FieldDesc& d = a.fd[fi];
      if (tid == 0 && fi != cur) {
        if (cur >= 0) {
          flush_counts(&as_global(a.fd[cur].st)->c[q].s[ctr_slot()], acc_m, acc_nf, acc_nb,
                       acc_sw, &ctl->tot[q][ctr_slot()].swept);
        }
        acc_m = acc_nf = acc_nb = acc_sw = 0;
        cur = fi;
      }
      const int64_t tile = tt - d.tile_base;
      const T* g = (const T*)d.g;
      const T* f = (const T*)d.f;
      const T xi = (T)d.xi_t;
      TileCounts tc;
      if (d.geo.ndim == 3) {
        if (kind == KIND_NEXT)
          tc = tile3<T, KIND_NEXT, SETS>(sm, red, g, f, d.dirs, d.bm, xi, d.geo, tile, d.prop);
        else
          tc = tile3<T, KIND_FIRST_GIVEN, SETS>(sm, red, g, f, d.dirs, d.bm, xi, d.geo, tile,
                                                d.prop);
      } else {
        if (kind == KIND_NEXT)
          tc = tile2<T, KIND_NEXT, SETS>(sm, red, g, f, d.dirs, d.bm, xi, d.geo, tile, d.prop);
        else
          tc = tile2<T, KIND_FIRST_GIVEN, SETS>(sm, red, g, f, d.dirs, d.bm, xi, d.geo, tile,
                                                d.prop);
      }
      if (tid == 0) {
        acc_m += unpack3(tc, 0);
        acc_nf += unpack3(tc, 1);
        acc_nb += unpack3(tc, 2);
        acc_sw += (unsigned long long)tile_voxels(d.geo, tile);
      }
    }
    __syncthreads();  // s_tiles is rewritten by the next batch
  }
  if (tid == 0 && cur >= 0) {
    flush_counts(&as_global(a.fd[cur].st)->c[q].s[ctr_slot()], acc_m, acc_nf, acc_nb, acc_sw,
                 &ctl->tot[q][ctr_slot()].swept);
  }
}

// Apply pass of a round (parity p, counter set q) on one unit: segment
// u >> plog of the batch's flag bitmaps, part u & (2^plog - 1) of it.  Every
// thread of the block takes part (block reductions inside).
template <class T, bool CO = false>
__device__ __forceinline__ void apply_unit(const EngineArgs& a, int64_t u, int plog, int p, int q,
                                           uint32_t* s_list, int* s_scan, long long* s_lbase,
                                           unsigned long long* red) {
  const int tid = threadIdx.x;
  EngineCtl* ctl = a.ctl;
  const int64_t sg = u >> plog;
  const int32_t part = (int32_t)(u & ((int64_t(1) << plog) - 1));
  const int fi = field_of_seg(a.fd, a.nf, sg);
  const FieldDesc& d = a.fd[fi];
  // the state at the start of the round (persisted before this pass)
  const FieldIter s = load_iter<CO>(&as_global(d.st)->s[p]);
  const gptr<FieldCtr> cq = &as_global(d.st)->c[q];
  const gptr<uint8_t> nxt = as_global(d.act) + (p ^ 1) * tile_count(d.geo);
  const unsigned long long mism = load_mism<CO>(cq);
  bool bad = false;
  if (!s.started) {
    const CtrSum cs = load_ctr<CO>(cq);
    bad = cs.bad_nf || cs.bad_b;
  }
  if (s.done || bad || mism == 0) return;
  const bool edit = (long long)s.k < d.max_iters;
  const int32_t span = (int32_t)(kSegWords >> plog);
  const int32_t w0 = (int32_t)((sg - d.seg_base) * kSegWords) + part * span;
  const int32_t w1 = (w0 + span < d.words) ? w0 + span : (int32_t)d.words;
  if (w0 >= w1) return;  // a part past the end of the field's last segment
  unsigned long long nflag = 0, at_lb = 0, edits = 0;
  apply_segment<T, CO>(d, w0, w1, edit, nxt, s_list, s_scan, s_lbase, cq, as_global(d.list),
                       nflag, at_lb, edits);
  // a segment holds at most 128K vertices: the three counts pack into
  // 21-bit fields of one word for a single block reduction
  const unsigned long long tot =
      block_sum(pack3((unsigned)nflag, (unsigned)at_lb, (unsigned)edits), red);
  if (tid == 0) {
    const unsigned long long nf_ = unpack3(tot, 0), al_ = unpack3(tot, 1),
                             ed_ = unpack3(tot, 2);
    const int slot = ctr_slot();
    if (nf_) {
      relaxed_add(&cq->s[slot].nflag, nf_);
      atomicAdd(&ctl->tot[q][slot].flagged, nf_);
    }
    if (al_) relaxed_add(&cq->s[slot].at_lb, al_);
    if (ed_) atomicAdd(&ctl->tot[q][slot].edits, ed_);
  }
}

// ---------------------------------------------------------------------------
// Apply pass of a plain round (k_apply), by waves.  A wave takes runs of 256-word
// units of the flag bitmaps (four words per lane, the next unit's loads in flight).
// Targets of sparse units gather in an LDS list of the wave's and are edited 64 at a
// time when it is full, the field changes or the wave is done; a unit with more
// targets than the list holds is edited in place, 64 consecutive vertices at a time.
//
// What bounds the pass is memory: a sparse round reads the bitmap, and each
// edit touches a line of f and of g.  With a block per 4096-word segment, every
// segment with a target paid its own chain of dependent round trips (words,
// list slot, values, activity bytes, counters: 10 to 14 us); a
// 1024 x 1024 x 768 binary64 field has eight segments per block, and its rounds of a
// few thousand edits took 0.11 to 0.14 ms.
// ---------------------------------------------------------------------------
constexpr int kUnitWords = 256;
constexpr int kWaveList = kApplyCap / 4;

// What a wave needs of the field it works on, in scalar registers.
template <class T>
struct ApplyField {
  gptr<const T> f;
  gptr<T> g;
  gptr<uint32_t> bm, tlist;
  gptr<uint8_t> nxt;
  gptr<FieldCtr> cq;
  void* prop;
  const FieldDesc* d;
  T xi;
  int64_t slice;
  int32_t words;
  int nls;
  bool edit;
};

// One edit: the value of target t, or its old one; counts what happened.
template <class T>
__device__ __forceinline__ T edited_value(const ApplyField<T>& F, T gt, T ft, T pv, bool& above) {
  const T lb = lower_bound<T>(ft, F.xi);
  above = gt > lb;
  if (!(above && F.edit)) return gt;
  if (F.prop) return pv > lb ? pv : lb;  // the smallest proposal, never below the bound
  return halving_edit<T>(gt, lb);
}

// Edit the n targets of the wave's list.
template <class T>
__device__ __forceinline__ void apply_list(const ApplyField<T>& F, const uint32_t* list, int n,
                                           int slot, unsigned& at_lb, unsigned& edits) {
  const int lane = threadIdx.x & 63;
  constexpr int U = kEditUnroll;
  using K = decltype(prop_key(T(0)));
  long long lbase = 0;
  if (F.edit && lane == 0)
    lbase = (long long)__hip_atomic_fetch_add(&F.cq->s[slot].nlist, (unsigned long long)n,
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  bool based = false;
  for (int j0 = lane; j0 < n; j0 += 64 * U) {
    int32_t t[U];
    T gt[U], ft[U], pv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) t[u] = (int32_t)list[j0 + 64 * u < n ? j0 + 64 * u : j0];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      gt[u] = F.g[t[u]];
      ft[u] = F.f[t[u]];
      pv[u] = F.prop ? prop_value(*((gptr<K>)F.prop + t[u])) : T(0);
    }
    if (!based) {  // (its round trip overlaps the first gathers')
      lbase = __shfl(lbase, 0, 64);
      based = true;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = j0 + 64 * u;
      if (j >= n) break;
      bool above;
      const T v = edited_value<T>(F, gt[u], ft[u], pv[u], above);
      if (above && F.edit) F.g[t[u]] = v;
      if (F.prop) *((gptr<K>)F.prop + t[u]) = ~K(0);  // unset for the next round
      edits += above && F.edit ? 1u : 0u;
      at_lb += above ? 0u : 1u;
      if (F.edit) {
        if (lbase + j < F.slice) F.tlist[(int64_t)slot * F.slice + lbase + j] = (uint32_t)t[u];
        mark_box(*F.d, box_of(F.d->geo, t[u]), F.nxt);
      }
    }
  }
}

// Mark the tiles within one vertex of the vertices v0 .. v1.
__device__ __forceinline__ void mark_range(const TileGeo& G, int32_t v0, int32_t v1,
                                           gptr<uint8_t> nxt) {
  const int32_t r0 = fdiv(v0, G.div_nx), r1 = fdiv(v1, G.div_nx);  // y + ny z
  int32_t xl = 0, xh = G.nx - 1, yl = r0, yh = r1, zl = 0, zh = 0;
  if (r0 == r1) {
    xl = v0 - r0 * G.nx;
    xh = v1 - r0 * G.nx;
  }
  if (G.ndim == 3) {
    zl = fdiv(r0, G.div_ny);
    zh = fdiv(r1, G.div_ny);
    yl = zl == zh ? r0 - zl * G.ny : 0;
    yh = zl == zh ? r1 - zl * G.ny : G.ny - 1;
  }
  auto below = [](int32_t v) { return v > 0 ? v - 1 : 0; };
  auto above = [](int32_t v, int32_t n) { return v + 1 < n ? v + 1 : v; };
  xl = below(xl), xh = above(xh, G.nx), yl = below(yl), yh = above(yh, G.ny);
  int32_t ax, bx, ay, by, az = 0, bz = 0;
  if (G.ndim == 3) {
    ax = xl / TX, bx = xh / TX, ay = yl / TY, by = yh / TY;
    az = fdiv(below(zl), G.div_chunk), bz = fdiv(above(zh, G.nz), G.div_chunk);
  } else {
    ax = xl / RX, bx = xh / RX, ay = fdiv(yl, G.div_chunk), by = fdiv(yh, G.div_chunk);
  }
  const int32_t wx = bx - ax + 1, wy = by - ay + 1, wz = bz - az + 1;
  for (int32_t i = threadIdx.x & 63; i < wx * wy * wz; i += 64) {
    const int32_t x = ax + i % wx, y = ay + i / wx % wy, z = az + i / (wx * wy);
    nxt[x + G.tiles_x * (y + G.tiles_y * z)] = 1;
  }
}

// Edit a unit's targets in place: words w of lane l are w0 + 4 l .., 64
// consecutive vertices per step, loads and stores masked by their offsets.
template <class T>
__device__ __forceinline__ void apply_dense(const ApplyField<T>& F, int32_t w0, const U32x4 w,
                                            int total, int slot, unsigned& at_lb,
                                            unsigned& edits) {
  const int lane = threadIdx.x & 63;
  const int32_t v0 = w0 * 32;
  constexpr uint32_t S = (uint32_t)sizeof(T);
  const Rsrc rg = rsrc_at(F.g + v0), rf = rsrc_at(F.f + v0),
             rp = rsrc_at((gptr<T>)F.prop + v0, F.prop != nullptr);
  long long at = 0;
  if (F.edit) {
    if (lane == 0)
      at = (long long)__hip_atomic_fetch_add(&F.cq->s[slot].nlist, (unsigned long long)total,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    at = __shfl(at, 0, 64);
    mark_range(F.d->geo, v0, tile_end(v0, 32 * kUnitWords, F.d->geo.n) - 1, F.nxt);
  }
  unsigned n_above = 0, n_all = 0;
  for (int l = 0; l < 64; l += 2) {
    unsigned long long m[4];
    uint32_t off[4];
    T gt[4], ft[4], pv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t a = (uint32_t)__builtin_amdgcn_readlane((int)w[2 * (k & 1)], l + (k >> 1));
      const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)w[2 * (k & 1) + 1], l + (k >> 1));
      m[k] = ((unsigned long long)b << 32) | a;
      off[k] = (m[k] >> lane) & 1ull ? (uint32_t)(128 * l + 64 * k + lane) * S : kNoStore;
      buf_load(rg, off[k], 0, gt[k]);
      buf_load(rf, off[k], 0, ft[k]);
      pv[k] = T(0);
      if (F.prop) buf_load(rp, off[k], 0, pv[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool mine = off[k] != kNoStore;
      bool above;
      using K = decltype(prop_key(T(0)));
      const T v = edited_value<T>(F, gt[k], ft[k],
                                  F.prop ? prop_value((K)FP<T>::bits(pv[k])) : T(0), above);
      const unsigned long long up = __ballot(mine && above);
      buf_store(rg, mine && above && F.edit ? off[k] : kNoStore, 0, v);
      if (F.prop) buf_store(rp, off[k], 0, FP<T>::from(~typename FP<T>::U(0)));
      n_above += (unsigned)__builtin_popcountll(up);
      n_all += (unsigned)__builtin_popcountll(m[k]);
      if (F.edit && at < F.slice) {
        const int64_t i = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(m[k] >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m[k], 0));
        if (mine && i < F.slice)
          F.tlist[(int64_t)slot * F.slice + i] = (uint32_t)(v0 + 128 * l + 64 * k + lane);
        at += __builtin_popcountll(m[k]);
      }
    }
  }
  if (lane == 0) {
    edits += F.edit ? n_above : 0u;
    at_lb += n_all - n_above;
  }
}

// The apply pass of a round (parity p, counter set q) on the whole grid.  list:
// kWaveList words per wave; fin, sums: one slot per wave.  Ends with the block in
// step.
template <class T>
__device__ __forceinline__ void apply_pass(const EngineArgs& a, int p, int q, uint32_t* list_all,
                                           int* fin, unsigned long long (*sums)[3]) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  uint32_t* const list = list_all + wave * kWaveList;
  EngineCtl* const ctl = a.ctl;
  const int64_t waves = (int64_t)gridDim.x * 4;
  constexpr int32_t unit = kUnitWords;
  constexpr int32_t per_seg = (int32_t)kSegWords / unit;
  const int64_t units = a.total_segs * per_seg;
  // units of a run: as many as share the waves evenly, within one segment
  int run_log = 0;
  while ((1 << run_log) < per_seg && units >> (run_log + 1) >= waves) ++run_log;
  const int64_t runs = units >> run_log;
  ApplyField<T> F{};
  int cur = -1, fill = 0, slot = 0;
  int64_t seg0 = 0, seg1 = 0;  // the field's segments
  bool idle = true;            // nothing to apply in it
  unsigned nflag = 0, at_lb = 0, edits = 0;
  unsigned long long c_flag = 0, c_lb = 0, c_ed = 0;
  auto flush = [&]() {
    wave_lds_fence();
    if (fill) apply_list<T>(F, list, fill, slot, at_lb, edits);
    wave_lds_fence();
    fill = 0;
  };
  auto add_counts = [&](int fi, unsigned long long nf_, unsigned long long al_,
                        unsigned long long ed_) {
    const gptr<FieldCtr> cq = &as_global(a.fd[fi].st)->c[q];
    const int cs = ctr_slot();
    if (nf_) {
      relaxed_add(&cq->s[cs].nflag, nf_);
      atomicAdd(&ctl->tot[q][cs].flagged, nf_);
    }
    if (al_) relaxed_add(&cq->s[cs].at_lb, al_);
    if (ed_) atomicAdd(&ctl->tot[q][cs].edits, ed_);
  };
  auto sum_counts = [&]() {  // of the current field, into c_*
    c_flag = wave_sum((unsigned long long)nflag);
    c_lb = wave_sum((unsigned long long)at_lb);
    c_ed = wave_sum((unsigned long long)edits);
    nflag = at_lb = edits = 0;
  };
  for (int64_t r = (int64_t)blockIdx.x * 4 + wave; r < runs; r += waves) {
    const int64_t u0 = r << run_log, sg = u0 / per_seg;
    if (cur < 0 || sg < seg0 || sg >= seg1) {
      flush();
      if (cur >= 0) {
        sum_counts();
        if (lane == 0) add_counts(cur, c_flag, c_lb, c_ed);
      }
      cur = __builtin_amdgcn_readfirstlane(field_of_seg(a.fd, a.nf, sg));
      const FieldDesc& d = a.fd[cur];
      F.d = &d;
      F.words = uniform((int32_t)d.words);
      seg0 = d.seg_base;
      seg1 = seg0 + (F.words + kSegWords - 1) / kSegWords;
      const gptr<FieldState> st = as_global(uniform_ptr(d.st));
      // the state at the start of the round (persisted before this pass)
      const FieldIter s = load_iter(&st->s[p]);
      F.cq = &st->c[q];
      bool bad = false;
      if (!s.started) {
        const CtrSum cs = load_ctr((gptr<const FieldCtr>)F.cq);
        bad = cs.bad_nf || cs.bad_b;
      }
      idle = uniform((int32_t)(s.done || bad || load_mism((gptr<const FieldCtr>)F.cq) == 0)) != 0;
      F.edit = uniform((int32_t)((long long)s.k < d.max_iters)) != 0;
      F.f = as_global((const T*)uniform_ptr(d.f));
      F.g = as_global((T*)uniform_ptr(d.g));
      F.bm = as_global(uniform_ptr(d.bm));
      F.tlist = as_global(uniform_ptr(d.list));
      F.nxt = as_global(uniform_ptr(d.act)) + (p ^ 1) * tile_count(d.geo);
      F.prop = uniform_ptr(d.prop);
      F.xi = (T)d.xi_t;
      F.nls = list_slices(F.words);
      F.slice = uniform(d.list_cap) / F.nls;
    }
    if (idle) continue;
    const int32_t seg = (int32_t)(sg - seg0);
    int32_t w0 = seg * (int32_t)kSegWords + (int32_t)(u0 % per_seg) * unit;
    const int32_t wl = 4 * lane;  // this lane's first word of a unit
    // (the bitmap ends on a 256-byte boundary, clear past the field)
    auto load = [&](int32_t at) {
      U32x4 x = {0u, 0u, 0u, 0u};
      if (at + wl < F.words) x = *(gptr<const U32x4>)(F.bm + at + wl);
      return x;
    };
    U32x4 next = load(w0);
    for (int k = 0; k < (1 << run_log); ++k, w0 += unit) {
      const U32x4 w = next;
      if (k + 1 < (1 << run_log)) next = load(w0 + unit);
      const uint32_t any = w.x | w.y | w.z | w.w;
      if (__ballot(any != 0u) == 0ull) continue;
      if (any) *(gptr<U32x4>)(F.bm + w0 + wl) = U32x4{0u, 0u, 0u, 0u};
      const int cnt = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
      nflag += (unsigned)cnt;
      int incl = cnt;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(incl, o, 64);
        if (lane >= o) incl += y;
      }
      const int total = __builtin_amdgcn_readlane(incl, 63);
      if (fill + total > kWaveList) flush();
      if (fill == 0) slot = seg % F.nls;
      if (total > kWaveList) {
        apply_dense<T>(F, w0, w, total, slot, at_lb, edits);
        continue;
      }
      int o = fill + incl - cnt;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        for (uint32_t bits = w[j]; bits; bits &= bits - 1u)
          list[o++] = (uint32_t)((w0 + wl + j) * 32 + __ffs(bits) - 1);
      fill += total;
    }
  }
  flush();
  if (cur >= 0) sum_counts();
  // one set of atomics for the waves that end on the same field
  if (lane == 0) {
    fin[wave] = cur;
    sums[wave][0] = c_flag;
    sums[wave][1] = c_lb;
    sums[wave][2] = c_ed;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 0; i < 4; ++i) {
      const int f = fin[i];
      if (f < 0) continue;
      for (int j = i + 1; j < 4; ++j) {
        if (fin[j] != f) continue;
        for (int k = 0; k < 3; ++k) sums[i][k] += sums[j][k];
        fin[j] = -1;
      }
      add_counts(f, sums[i][0], sums[i][1], sums[i][2]);
    }
  }
  __syncthreads();
}

// The totals of a counter set, by the first threads of a block.
__device__ __forceinline__ void clear_tot(EngineCtl* ctl, int q) {
  const int tid = threadIdx.x;
  if (tid < kCtrSlots) {
    ctl->tot[q][tid].edits = 0;
    ctl->tot[q][tid].swept = 0;
    ctl->tot[q][tid].sparse = 0;
    ctl->tot[q][tid].flagged = 0;
  }
}

// Block 0 at the start of round E: persist the field states of round E, clear
// the next-but-one counters; a field finished at E (stop_on_done) or the
// host's request ends the launch after this round (every block reads the word
// after the detect barrier).  CO as for ld.
template <bool CO>
__device__ __forceinline__ void persist_round(const EngineArgs& a, unsigned long long E,
                                              unsigned long long E0, int p, int qn) {
  const int tid = threadIdx.x;
  EngineCtl* ctl = a.ctl;
  bool stop = false;
  for (int fi = tid; fi < a.nf; fi += 256) {
    const FieldDesc& d = a.fd[fi];
    const gptr<FieldState> st = as_global(d.st);
    bool done;
    if (E > E0) {
      const FieldIter s = state_at<CO>(d, E, E0);
      store_iter(&st->s[p], s);
      stop |= a.stop_on_done && s.done && !ld<CO>(&st->s[p ^ 1].done);
      done = s.done;
    } else {
      done = ld<CO>(&st->s[p].done);
      // a later launch of a step whose tile detection ran as sweeps: a
      // field done at its start finished in the step's earlier launch
      stop |= a.stop_on_done && a.tiles_swept && done;
    }
    // the host asked for the step to end once a field is done (every
    // field of a step was running when it began)
    if (done && a.stop_host &&
        __hip_atomic_load(a.stop_host, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) ==
            kStopWhenDone)
      stop = true;
    clear_ctr(&st->c[qn]);
  }
  if (tid == 0 && a.stop_host &&
      __hip_atomic_load(a.stop_host, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == kStopNow)
    stop = true;
  if (stop) __hip_atomic_store(&ctl->stop.v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  clear_tot(ctl, qn);
}

// ---------------------------------------------------------------------------
// Plain rounds: the kernels of one round of a large batch, each at
// its own occupancy, for the round E that the workspace's epoch names.  The
// detection of fields in tile rounds is k_sweep's, of fields in sparse rounds
// k_sparse's; k_apply applies, and its last block does what the engine's block 0
// and tracer do between rounds.  A kernel with nothing to do returns at once.
// ---------------------------------------------------------------------------
// k_tail takes the rest of the loop after a round with so many edits: the next
// one examines at most 15 neighbours per edit, few enough for the blocks of one
// XCD, and few enough segments to mark for its apply pass.
__device__ __forceinline__ bool tail_takes(const EngineArgs& a, unsigned long long edited) {
  return a.tail_ok && a.nf <= 256 &&
         edited * 15ull <= (unsigned long long)(kTailGrid / 8) * 256ull * kTailExams &&
         (edited <= (unsigned long long)kTailSegs || a.total_segs <= kTailSegs);
}

// End of a plain round, in one block: the state of every field at round E + 1 and
// the counters of round E + 2, as persist_round leaves them; the round's record;
// the epoch.  idle: the plain rounds that follow leave everything as it is, because no
// field is left running (kAllDone), the tail takes the next rounds (kFewEdits; the
// engine launch does nothing either in these two cases), or the next round
// sweeps tiles and its launches have no sweep (kTilesNext).  Other blocks' counts are
// atomics, read past this unit's caches (ld<true>).
__device__ __forceinline__ void round_end(const EngineArgs& a, unsigned long long E) {
  EngineCtl* const ctl = a.ctl;
  const int tid = threadIdx.x;
  const int q = (int)(E % 3), qn = (int)((E + 2) % 3);
  int tiles = 0, sparse = 0;
  // eight lanes per field, one per counter slot: one round trip, few registers
  static_assert(kCtrSlots == 8, "a lane per slot");
  for (int f0 = 0; f0 < a.nf; f0 += 32) {
    const int fi = f0 + (tid >> 3), k = tid & 7;
    const bool mine = fi < a.nf;
    const FieldDesc& d = a.fd[mine ? fi : 0];
    const gptr<FieldState> st = as_global(d.st);
    const gptr<const CtrSlot> c = &st->c[q].s[k];
    CtrSum cs{ld<true>(&c->mism), ld<true>(&c->nflag), ld<true>(&c->at_lb), ld<true>(&c->bad_nf),
              ld<true>(&c->bad_b), ld<true>(&c->swept), ld<true>(&c->nlist)};
    // a slice of the target list overflowed (sparse_items)
    int over = cs.nlist > (unsigned long long)(d.list_cap / list_slices(d.words));
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) {
      cs.mism += __shfl_xor(cs.mism, o, 64);
      cs.nflag += __shfl_xor(cs.nflag, o, 64);
      cs.at_lb += __shfl_xor(cs.at_lb, o, 64);
      cs.bad_nf += __shfl_xor(cs.bad_nf, o, 64);
      cs.bad_b += __shfl_xor(cs.bad_b, o, 64);
      cs.swept += __shfl_xor(cs.swept, o, 64);
      over |= __shfl_xor(over, o, 64);
    }
    if (!mine) continue;
    const gptr<CtrSlot> x = &st->c[qn].s[k];
    x->mism = x->nflag = x->at_lb = x->bad_nf = x->bad_b = x->swept = x->nlist = 0;
    if (k != 0) continue;
    const FieldIter s =
        next_state(load_iter((gptr<const FieldIter>)&st->s[E & 1]), cs, d.max_iters);
    store_iter(&st->s[(E + 1) & 1], s);
    if (s.done) continue;
    if (over) tiles = 1;
    else sparse = 1;
  }
  tiles = __syncthreads_or(tiles);
  sparse = __syncthreads_or(sparse);
  clear_tot(ctl, qn);
  if (tid == 0) {
    RoundTot rt{0, 0, 0, 0, {0, 0, 0, 0}};
#pragma unroll 4
    for (int k = 0; k < kCtrSlots; ++k) {
      const gptr<const RoundTot> t = as_global(&ctl->tot[q][k]);
      rt.edits += ld<true>(&t->edits);
      rt.swept += ld<true>(&t->swept);
      rt.sparse += ld<true>(&t->sparse);
      rt.flagged += ld<true>(&t->flagged);
    }
    ctl->epoch = E + 1;
    ctl->rounds = E + 1;
    ctl->kinds = (tiles ? kKindTiles : 0) | (sparse ? kKindSparse : 0);
    ctl->idle = !(tiles || sparse) ? kAllDone
              : !tiles && tail_takes(a, rt.edits) ? kFewEdits
              : tiles && !a.next_sweep ? kTilesNext : 0;
    if (a.trace && E < kTraceRounds) {
      unsigned long long* t = a.trace + kTraceSlots * E;
      const unsigned long long now = wall_clock64();
      t[2] = now;
      t[3] = rt.swept;
      t[4] = rt.flagged;
      t[5] = rt.edits;
      t[6] = rt.sparse;
      if (E + 1 < kTraceRounds) t[kTraceSlots] = now;  // the next round starts
    }
  }
}

// The block that arrives last of the grid, once its own and every other block's
// stores and atomics are done: the arrival counters of grid_sync, left cleared.
__device__ __forceinline__ bool last_block(EngineCtl* ctl) {
  __shared__ int s_last;
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned groups = gridDim.x < (unsigned)kBarGroups ? gridDim.x : (unsigned)kBarGroups;
    const unsigned grp = blockIdx.x % groups;
    const unsigned members = gridDim.x / groups + (grp < gridDim.x % groups ? 1u : 0u);
    auto arrive = [&](BarWord* w, unsigned n) {
      if (__hip_atomic_fetch_add(&w->v, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != n - 1u)
        return false;
      __hip_atomic_store(&w->v, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return true;
    };
    s_last = arrive(&ctl->bar[grp], members) && arrive(&ctl->bar[kBarGroups], groups);
  }
  __syncthreads();
  return s_last != 0;
}

template <class T>
__global__ __launch_bounds__(256) void k_apply(EngineArgs a) {
  __shared__ uint32_t s_list[kApplyCap];
  __shared__ int s_fin[4];
  __shared__ unsigned long long s_sums[4][3];
  const unsigned long long E = a.ctl->epoch;
  if (a.ctl->idle) return;
  if (a.trace && E < kTraceRounds && blockIdx.x == 0 && threadIdx.x == 0) {
    const unsigned long long now = wall_clock64();
    if (E == 0) {  // round 0 starts here (its detection is timed by its sweep)
      a.trace[kTraceRounds * kTraceSlots] = now;
      a.trace[0] = now;
    }
    a.trace[kTraceSlots * E + 1] = now;
  }
  apply_pass<T>(a, (int)(E & 1), (int)(E % 3), s_list, s_fin, s_sums);
  if (last_block(a.ctl)) round_end(a, E);
}

// Sparse examination of a plain round: the vertices to examine are the
// neighbours of the listed targets (15 in 3D, 7 in 2D, with the target), and
// what decides them lies within two steps of the target: 65 vertices (19),
// which 15 gathers per examined vertex would read 225 times (49).  Sixteen
// (eight) lanes share a target: they stage its surroundings as a 5 x 5 x 5 box in
// LDS, five (three) loads each, and examine one vertex each from there.  The loads
// of the plain gather kept the units' address path busy: 30 M examinations of a
// 1024 x 1024 x 768 binary64 field took 1.6 ms.
constexpr int kBoxN3 = 65, kBoxN2 = 19;
// Box offsets in staging order: coordinates + 2, three bits each.
struct BoxTable {
  uint16_t v[kBoxN3];
};
template <int DIM>
constexpr BoxTable make_box_table() {
  BoxTable t{};
  int n = 0;
  for (int z = DIM == 3 ? -2 : 0; z <= (DIM == 3 ? 2 : 0); ++z)
    for (int y = -2; y <= 2; ++y)
      for (int x = -2; x <= 2; ++x) {
        const int lo = x < y ? (x < z ? x : z) : (y < z ? y : z);
        const int hi = x > y ? (x > z ? x : z) : (y > z ? y : z);
        // a sum of two offsets, each all >= 0 or all <= 0
        if (!(lo < 0 && hi > 0) || (lo == -1 && hi == 1))
          t.v[n++] = (uint16_t)((x + 2) | ((y + 2) << 3) | ((z + 2) << 6));
      }
  return t;
}
__constant__ BoxTable kBox3 = make_box_table<3>();
__constant__ BoxTable kBox2 = make_box_table<2>();

template <int DIM>
struct ExamGeo {
  static constexpr int L = DIM == 3 ? 16 : 8;           // lanes per target
  static constexpr int N = DIM == 3 ? kBoxN3 : kBoxN2;  // vertices staged
  static constexpr int B = DIM == 3 ? 128 : 32;         // box stride in LDS (125, 25)
  static constexpr int K = (N + L - 1) / L;             // loads per lane
  static constexpr int A = 64 / L;                      // targets at once
};
// This lane's vertices of the box.
template <int DIM>
struct BoxLane {
  uint32_t c[ExamGeo<DIM>::K];
};
template <int DIM>
__device__ __forceinline__ BoxLane<DIM> box_lane() {
  using X = ExamGeo<DIM>;
  BoxLane<DIM> b;
  const int me = threadIdx.x & (X::L - 1);
#pragma unroll
  for (int i = 0; i < X::K; ++i)
    b.c[i] = (DIM == 3 ? kBox3 : kBox2).v[me + X::L * i < X::N ? me + X::L * i : X::N - 1];
  return b;
}

// The k-th listed target (the last one past the end).
__device__ __forceinline__ int32_t listed_target(const FieldDesc& d, uint32_t k, uint32_t n,
                                                 const uint32_t* cnt) {
  uint32_t kk = k < n ? k : n - 1u, at = 0;
  const uint32_t slice = (uint32_t)(d.list_cap / list_slices(d.words));
#pragma unroll
  for (int i = 0; i < kCtrSlots - 1; ++i) {
    const uint32_t ci = cnt[i];
    const bool past = at == (uint32_t)i * slice && kk >= ci;
    kk -= past ? ci : 0u;
    at += past ? slice : 0u;
  }
  return (int32_t)as_global((const uint32_t*)d.list)[at + kk];
}

// Examine the surroundings of target t (one per ExamGeo::L lanes; have: there is
// one).
template <class T, int DIM>
__device__ __forceinline__ unsigned examine_target(const FieldDesc& d, const TileGeo& G, int32_t t,
                                                   bool have, const BoxLane<DIM>& lanes, T* box) {
  using GX = ExamGeo<DIM>;
  constexpr int L = GX::L, N = GX::N;
  const int lane = threadIdx.x & 63, me = lane & (L - 1);
  const int32_t row = fdiv(t, G.div_nx);  // y + ny z
  const int32_t x = t - row * G.nx;
  const int32_t z = DIM == 3 ? fdiv(row, G.div_ny) : 0;
  const int32_t y = row - z * G.ny;
  const gptr<const T> g = as_global((const T*)uniform_ptr(d.g));
  T* const mine = box + lane / L * GX::B;
  T val[GX::K];
#pragma unroll
  for (int i = 0; i < GX::K; ++i) {
    const int32_t c = (int32_t)lanes.c[i];
    const int32_t dx = (c & 7) - 2, dy = ((c >> 3) & 7) - 2, dz = DIM == 3 ? (c >> 6) - 2 : 0;
    const bool in = (uint32_t)(x + dx) < (uint32_t)G.nx && (uint32_t)(y + dy) < (uint32_t)G.ny &&
                    (DIM == 2 || (uint32_t)(z + dz) < (uint32_t)G.nz);
    const int32_t v = t + dx + dy * G.nx + (DIM == 3 ? dz * G.sxy : 0);
    val[i] = g[in ? v : t];
    if (!in) val[i] = T(__builtin_nan(""));
  }
  // the vertex examined: code 0 (the target), 1..7, 9..15; 2D 1..3, 9..11
  constexpr int M = DIM == 3 ? 15 : 7;
  const int j = me < M ? me : 0;
  const int code = DIM == 3 ? (j < 8 ? j : j + 1) : (j < 4 ? j : j + 5);
  const int mm = code & 7, sg = (code & 8) ? -1 : 1;
  const int32_t ox = sg * (mm & 1), oy = sg * ((mm >> 1) & 1), oz = sg * ((mm >> 2) & 1);
  const int32_t X = x + ox, Y = y + oy, Z = z + oz;
  const bool look = have && me < M && X >= G.cx0 && X < G.cx1 && Y >= G.cy0 && Y < G.cy1 &&
                    Z >= G.cz0 && Z < G.cz1;
  const int32_t v = t + code_offset(G, code);
  int d8 = 0;
  if (look) d8 = as_global((const uint8_t*)d.dirs)[v];
#pragma unroll
  for (int i = 0; i < GX::K; ++i) {
    const uint32_t c = lanes.c[i];
    if (me + L * i < N)
      mine[(c & 7) + 5 * ((c >> 3) & 7) + (DIM == 3 ? 25 * (c >> 6) : 0)] = val[i];
  }
  wave_lds_fence();
  unsigned found = 0;
  if (look) {
    const T* const at0 = mine + (ox + 2) + 5 * (oy + 2) + (DIM == 3 ? 25 * (oz + 2) : 0);
    auto up = [&](int bx, int by, int bz) {
      return ext_of(at0[bx + 5 * by + 25 * bz], bx | (by << 1) | (bz << 2));
    };
    auto dn = [&](int bx, int by, int bz) {  // the vertex (1-bx, 1-by, 1-bz) back
      const int m = (1 - bx) | ((1 - by) << 1) | (DIM == 3 ? (1 - bz) << 2 : 0);
      return ext_of(at0[-((1 - bx) + 5 * (1 - by) + (DIM == 3 ? 25 * (1 - bz) : 0))],
                    m ? (8 | m) : 0);
    };
    Ext<T> e;
    if constexpr (DIM == 3) {
      const Ext<T> U = merge_up(merge_up(merge_up(up(0, 0, 0), up(1, 0, 0)),
                                         merge_up(up(0, 1, 0), up(1, 1, 0))),
                                merge_up(merge_up(up(0, 0, 1), up(1, 0, 1)),
                                         merge_up(up(0, 1, 1), up(1, 1, 1))));
      const Ext<T> D = merge_dn(merge_dn(merge_dn(dn(0, 0, 0), dn(1, 0, 0)),
                                         merge_dn(dn(0, 1, 0), dn(1, 1, 0))),
                                merge_dn(merge_dn(dn(0, 0, 1), dn(1, 0, 1)),
                                         merge_dn(dn(0, 1, 1), dn(1, 1, 1))));
      e = merge_up(D, U);
    } else {
      const Ext<T> U = merge_up(merge_up(up(0, 0, 0), up(1, 0, 0)),
                                merge_up(up(0, 1, 0), up(1, 1, 0)));
      const Ext<T> D = merge_dn(merge_dn(dn(0, 0, 0), dn(1, 0, 0)),
                                merge_dn(dn(0, 1, 0), dn(1, 1, 0)));
      e = merge_up(D, U);
    }
    const int fa = d8 & 15, fd = d8 >> 4;
    const gptr<uint32_t> bm = as_global(d.bm);
    // targets are neighbours of v, inside the box for directions made by the
    // direction pass; the range check only guards the bitmap
    if (e.ca != fa) {
      const int32_t tt = v + code_offset(G, e.ca);
      if ((uint32_t)tt < (uint32_t)G.n) {
        __hip_atomic_fetch_or(bm + (tt >> 5), 1u << (tt & 31), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
        if (d.prop) {
          const int32_t c = v + code_offset(G, fa);
          propose<T>(d.prop, tt, c, g[c]);
        }
      }
      ++found;
    }
    if (e.cd != fd) {
      const int32_t tt = v + code_offset(G, fd);
      if ((uint32_t)tt < (uint32_t)G.n) {
        __hip_atomic_fetch_or(bm + (tt >> 5), 1u << (tt & 31), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
        if (d.prop) propose<T>(d.prop, tt, v + code_offset(G, e.cd), e.lo);
      }
      ++found;
    }
  }
  wave_lds_fence();  // the box is staged anew
  return found;
}

template <class T, int DIM>
__global__ __launch_bounds__(256) void k_sparse(EngineArgs a) {
  using GX = ExamGeo<DIM>;
  __shared__ long long s_pre[256];
  __shared__ uint32_t s_slot[256 * kCtrSlots];
  __shared__ T s_box[4][GX::A * GX::B];
  EngineCtl* const ctl = a.ctl;
  const unsigned long long E = ctl->epoch;
  if (ctl->idle || !(ctl->kinds & kKindSparse)) return;
  const int q = (int)(E % 3);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t grp = (uint32_t)((tid & 63) / GX::L);
  const BoxLane<DIM> lanes = box_lane<DIM>();
  for (int f0 = 0; f0 < a.nf; f0 += 256) {
    // the groups of targets of up to 256 fields form one index space
    const int fi = f0 + tid;
    long long groups = 0;
    if (fi < a.nf && a.fd[fi].geo.ndim == DIM) {
      const FieldDesc& d = a.fd[fi];
      const long long items = sparse_items(d, state_at(d, E, E), E, s_slot + tid * kCtrSlots);
      if (items > 0) {
        groups = (items / (DIM == 3 ? 15 : 7) + GX::A - 1) / GX::A;
        if (blockIdx.x == 0) {
          relaxed_add(&as_global(d.st)->c[q].s[0].swept, (unsigned long long)items);
          atomicAdd(&ctl->tot[q][0].swept, (unsigned long long)items);
          atomicAdd(&ctl->tot[q][0].sparse, (unsigned long long)items);
        }
      }
    }
    const long long total = block_prefix(groups, s_pre);
    const int nfc = a.nf - f0 < 256 ? a.nf - f0 : 256;
    int cur = -1;
    unsigned found = 0;
    auto flush = [&]() {
      const unsigned long long w = wave_sum((unsigned long long)found);
      if (w && (tid & 63) == 0)
        relaxed_add(&as_global(a.fd[cur].st)->c[q].s[ctr_slot()].mism, w);
      found = 0;
    };
    // a group's field and its targets; the next group's are read while this one's
    // surroundings are examined
    struct Group {
      int f;
      uint32_t n, k;
      int32_t t;
    };
    auto group_at = [&](long long m) {
      Group r;
      r.f = __builtin_amdgcn_readfirstlane(prefix_find(s_pre, nfc, m));
      const uint32_t* const cnt = s_slot + r.f * kCtrSlots;
      r.n = 0;
#pragma unroll
      for (int i = 0; i < kCtrSlots; ++i) r.n += cnt[i];
      r.k = (uint32_t)(m - (r.f ? s_pre[r.f - 1] : 0)) * (uint32_t)GX::A + grp;
      r.t = listed_target(a.fd[f0 + r.f], r.k, r.n, cnt);
      return r;
    };
    long long m = (long long)blockIdx.x * 4 + wave;
    const long long step = (long long)gridDim.x * 4;
    Group now{0, 0, 0, 0};
    if (m < total) now = group_at(m);
    for (; m < total; m += step) {
      Group next = now;
      if (m + step < total) next = group_at(m + step);
      if (f0 + now.f != cur) {
        if (cur >= 0) flush();
        cur = f0 + now.f;
      }
      const FieldDesc& d = a.fd[cur];
      found += examine_target<T, DIM>(d, uniform_geo(d.geo), now.t, now.k < now.n, lanes,
                                      s_box[wave]);
      now = next;
    }
    if (cur >= 0) flush();
    __syncthreads();  // s_pre is rewritten by the next group
  }
}

// LDS of k_tail that a tail round uses.
struct RoundLds {
  long long* pre;           // [256] prefix sums of the fields' examinations
  uint32_t* slot;           // [256 * kCtrSlots] targets listed per slot, per field
  uint32_t* list;           // [kApplyCap] targets of an apply pass
  int* scan;                // [4]
  long long* lbase;         // [1]
  unsigned long long* red;  // [4]
  uint16_t* units;          // [256] marked segments of a batch
};

// One sparse round of the tail (k_tail), on the blocks of the lead XCD
// (rank, members): detection of the listed targets' neighbours, the apply
// pass over the segments that detection marked, and their barriers
// (tail_sync), with every load of data that another unit may have written a
// device-scope one.  Returns 0 when the round ran and the loop goes on, 1
// when the loop ends after it, and 2, before anything has run, when some
// field sweeps tiles in this round (the engine takes that round).  The tail
// holds at most 256 fields.
template <class T>
__device__ __forceinline__ int tail_round(const EngineArgs& a, const XcdBar& xb, unsigned& gen,
                                       unsigned long long& E, unsigned long long E0,
                                       const RoundLds L) {
  const int tid = threadIdx.x;
  EngineCtl* ctl = a.ctl;
  const int p = (int)(E & 1);
  const int q = (int)(E % 3), qn = (int)((E + 1) % 3);
  const bool tracer = a.trace && blockIdx.x == 0 && tid == 0;
  long long items = 0;
  int sweeps = 0;
  if (tid < a.nf) {
    const FieldDesc& d = a.fd[tid];
    unsigned long long nk[kCtrSlots];
    load_nlist(d, E, nk);
    const FieldIter s = state_at<true>(d, E, E0);
    items = sparse_items_of(d, s, nk, L.slot + tid * kCtrSlots);
    if (items < 0) {
      sweeps = !s.done;
      items = 0;
    }
  }
  if (__syncthreads_or(sweeps)) return 2;
  if (tracer && E < kTraceRounds) a.trace[kTraceSlots * E] = wall_clock64();
  if (blockIdx.x == 0) {
    // (the tail's first round is checked against the round before it, which
    // the engine launch ran: a field it finished ends the step after this
    // round, as the engine would have)
    persist_round<true>(a, E, E == E0 && E0 > 0 ? E0 - 1 : E0, p, qn);
    if (tid < a.nf && items > 0) {
      relaxed_add(&as_global(a.fd[tid].st)->c[q].s[0].swept, (unsigned long long)items);
      atomicAdd(&ctl->tot[q][0].swept, (unsigned long long)items);
      atomicAdd(&ctl->tot[q][0].sparse, (unsigned long long)items);
    }
  }
  // ---- detect: the examinations of all fields form one index space
  const long long total = block_prefix(items, L.pre);
  {
    FieldAcc mism;
    auto mism_ptr = [&](int f) { return &as_global(a.fd[f].st)->c[q].s[ctr_slot()].mism; };
    for (long long m = (long long)xb.rank * 256 + tid; m < total;
         m += (long long)xb.members * 256) {
      const int fx = prefix_find(L.pre, a.nf, m);
      const Exam ex = sparse_examine<T, true>(
          a.fd[fx], (uint32_t)(m - (fx ? L.pre[fx - 1] : 0)), L.slot + fx * kCtrSlots);
      acc_add(mism, fx, ex.n, mism_ptr);
      // the flags, and the marks of their segments for the apply pass below
      const gptr<uint32_t> bm = as_global(a.fd[fx].bm);
      const gptr<uint8_t> mk = as_global(a.fd[fx].marks);
      if (ex.ta >= 0) {
        __hip_atomic_fetch_or(bm + (ex.ta >> 5), 1u << (ex.ta & 31), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
        mk[ex.ta >> 17] = 1;
      }
      if (ex.td >= 0) {
        __hip_atomic_fetch_or(bm + (ex.td >> 5), 1u << (ex.td & 31), __ATOMIC_RELAXED,
                              __HIP_MEMORY_SCOPE_AGENT);
        mk[ex.td >> 17] = 1;
      }
    }
    acc_flush(mism, mism_ptr, L.scan, L.red);
  }
  tail_sync(ctl, xb, gen);
  if (engine_failed(ctl)) return 1;
  // written by block 0 before the barrier above
  const bool stop_here =
      __hip_atomic_load(&ctl->stop.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
  if (tracer && E < kTraceRounds) a.trace[kTraceSlots * E + 1] = wall_clock64();
  // ---- apply: the block reads the marks of its segments 256 at a time,
  // clears them, and takes the marked ones whole
  for (int64_t base = xb.rank; base < a.total_segs; base += (int64_t)xb.members * 256) {
    const int64_t mine = base + (int64_t)tid * xb.members;
    int take = 0;
    if (mine < a.total_segs) {
      const FieldDesc& d = a.fd[field_of_seg(a.fd, a.nf, mine)];
      const gptr<uint8_t> mk = as_global(d.marks) + (mine - d.seg_base);
      if (ld<true>(mk)) {
        *mk = 0;
        take = 1;
      }
    }
    int n_take = 0;
    const int pos = block_scan(take, L.scan, &n_take);
    if (take) L.units[pos] = (uint16_t)tid;
    __syncthreads();
    for (int j = 0; j < n_take; ++j) {
      const int64_t u = base + (int64_t)__builtin_amdgcn_readfirstlane(L.units[j]) * xb.members;
      apply_unit<T, true>(a, u, 0, p, q, L.list, L.scan, L.lbase, L.red);
    }
    __syncthreads();  // units is rewritten by the next batch
  }
  tail_sync(ctl, xb, gen);
  if (engine_failed(ctl)) return 1;
  if (tracer && E < kTraceRounds) {
    unsigned long long* t = a.trace + kTraceSlots * E;
    const RoundTot rt = load_tot<true>(ctl, q);
    t[2] = wall_clock64();
    t[3] = rt.swept;
    t[4] = rt.flagged;
    t[5] = rt.edits;
    t[6] = rt.sparse;
  }
  const unsigned long long edited = load_edits<true>(ctl, q);
  ++E;
  return (edited == 0 || stop_here) ? 1 : 0;
}

// WAVES: waves per SIMD, that is the register budget.
template <class T, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_engine(
    EngineArgs a) {
  __shared__ TileLds<T> sm;
  __shared__ unsigned long long red[4];
  __shared__ unsigned long long s_acc[4];
  __shared__ uint16_t s_tiles[256];
  __shared__ long long s_pre[256];
  __shared__ uint32_t s_slot[256 * kCtrSlots];
  __shared__ uint32_t s_list[kApplyCap];
  __shared__ int s_scan[4];
  __shared__ long long s_lbase;
  const unsigned G = gridDim.x;
  const int tid = threadIdx.x;
  for (int k = tid; k < kFlagWords; k += 256) sm.flags[k] = 0u;
  __syncthreads();
  EngineCtl* ctl = a.ctl;
  unsigned gen = relaxed_load(&ctl->bar_gen.v);
  const unsigned long long E0 = ctl->epoch;
  unsigned long long E = E0;
  // After plain rounds that left nothing to do, or the rest to the tail, the
  // launch ends before its first barrier (idle stays, for the blocks that start
  // last).
  const int idle = a.plain ? ctl->idle : 0;
  if (idle == kAllDone || idle == kFewEdits) {
    if (blockIdx.x != 0) return;
    for (int fi = tid; fi < a.nf; fi += 256)
      if (a.out) a.out[fi] = load_iter((gptr<const FieldIter>)&as_global(a.fd[fi].st)->s[E0 & 1]);
    if (tid == 0) {
      ctl->rounds = 0;
      ctl->handoff = idle == kFewEdits ? kHandToTail : 0;
    }
    return;
  }
  const bool tracer = a.trace && blockIdx.x == 0 && tid == 0;
  if (tracer && E0 == 0) a.trace[kTraceRounds * kTraceSlots] = wall_clock64();

  // Fields that have not started: every tile is active in their first round.
  if (a.has_fresh && !a.tiles_swept) {
    for (int64_t tt = (int64_t)blockIdx.x * 256 + tid; tt < a.total_tiles; tt += (int64_t)G * 256) {
      const FieldDesc& d = a.fd[field_of_tile(a.fd, a.nf, tt)];
      const FieldIter s = load_iter(&as_global(d.st)->s[E0 & 1]);
      if (!s.started && !s.done)
        as_global(d.act)[(E0 & 1) * tile_count(d.geo) + (tt - d.tile_base)] = 1;
    }
  }
  // blocks per XCD (its closing barrier also orders the marks above)
  const XcdBar xb = xcd_census(ctl, gen);
  // apply parts per segment: a power of two up to 256 (16 words each), so
  // that the grid's blocks share the segments of small fields
  int parts_log2 = 0;
  while (parts_log2 < 8 && a.total_segs << (parts_log2 + 1) <= (int64_t)G) ++parts_log2;
  // the launch ends to hand its remaining rounds to k_tail
  bool handoff = false;

  for (long long r = 0; a.max_rounds < 0 || r < a.max_rounds; ++r) {
    if (engine_failed(ctl)) break;
    const int p = (int)(E & 1);
    const int q = (int)(E % 3), qn = (int)((E + 1) % 3);
    if (tracer && E < kTraceRounds) a.trace[kTraceSlots * E] = wall_clock64();

    if (blockIdx.x == 0) persist_round<false>(a, E, E0, p, qn);

    // ---- detect ------------------------------------------------------------
    // Sparse rounds first: the examinations of up to 256 fields at a time form
    // one index space (prefix sums in LDS) that the grid strides over.  The
    // mismatch counts are only tested against zero in these rounds.
    int any_tiles = 0;
    bool split_here = false;
    for (int f0 = 0; f0 < a.nf; f0 += 256) {
      const int fi = f0 + tid;
      long long items = 0;
      int sweeps = 0, big = 0;
      if (fi < a.nf) {
        const FieldDesc& d = a.fd[fi];
        const FieldIter s = state_at(d, E, E0);
        items = sparse_items(d, s, E, s_slot + tid * kCtrSlots);
        if (items < 0) {
          sweeps = !s.done;
          big = sweeps && s.started && d.geo.n >= kSplitVoxels;
          items = 0;
        }
      }
      any_tiles |= __syncthreads_or(sweeps);
      // A large tile round is left to plain rounds: every block sees the same
      // states and leaves here, before this round's detection has done anything
      // (the marks of its active tiles stay set for the sweep).
      if (a.split_tiles && (r > 0 || a.plain) && f0 == 0 && __syncthreads_or(big)) {
        split_here = true;
        break;
      }
      if (fi < a.nf && items > 0 && blockIdx.x == 0) {
        const FieldDesc& d = a.fd[fi];
        relaxed_add(&as_global(d.st)->c[q].s[0].swept, (unsigned long long)items);
        atomicAdd(&ctl->tot[q][0].swept, (unsigned long long)items);
        atomicAdd(&ctl->tot[q][0].sparse, (unsigned long long)items);
      }
      const long long total = block_prefix(items, s_pre);
      const int nfc = a.nf - f0 < 256 ? a.nf - f0 : 256;
      FieldAcc mism;
      auto mism_ptr = [&](int f) { return &as_global(a.fd[f].st)->c[q].s[ctr_slot()].mism; };
      for (long long m = (long long)blockIdx.x * 256 + tid; m < total; m += (long long)G * 256) {
        const int lo = prefix_find(s_pre, nfc, m);
        const int fx = f0 + lo;
        const Exam ex = sparse_examine<T>(a.fd[fx], (uint32_t)(m - (lo ? s_pre[lo - 1] : 0)),
                                          s_slot + lo * kCtrSlots);
        acc_add(mism, fx, ex.n, mism_ptr);
        // fire-and-forget flags: the apply pass reads them after the barrier
        const gptr<uint32_t> bm = as_global(a.fd[fx].bm);
        if (ex.ta >= 0)
          __hip_atomic_fetch_or(bm + (ex.ta >> 5), 1u << (ex.ta & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
        if (ex.td >= 0)
          __hip_atomic_fetch_or(bm + (ex.td >> 5), 1u << (ex.td & 31), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
      }
      acc_flush(mism, mism_ptr, s_scan, red);
      __syncthreads();  // s_pre is rewritten by the next group
    }
    if (split_here) break;
    // Tiles: skipped when every running field is in a sparse round (marks
    // left from earlier rounds then only widen a later tile round).
    if (any_tiles && !(r == 0 && a.tiles_swept))
      detect_tiles<T, sets_for<T, KIND_NEXT>()>(a, sm, red, s_tiles, s_scan, s_acc, E, E0,
                                                blockIdx.x, G);
    xcd_sync(ctl, xb, gen);
    if (engine_failed(ctl)) break;
    // written by block 0 before the barrier above
    const bool stop_here =
        __hip_atomic_load(&ctl->stop.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
    if (tracer && E < kTraceRounds) a.trace[kTraceSlots * E + 1] = wall_clock64();

    // ---- apply -------------------------------------------------------------
    // One pass per 4096-word segment of each field's flag bitmap, or per part
    // of one when the grid has more blocks than there are segments (small
    // fields: a segment's edits would otherwise run through one block's
    // threads in a few long chains).
    // (Rounds after an all-sparse detect flag few vertices: whole segments.)
    const int plog = any_tiles ? parts_log2 : 0;
    for (int64_t u = blockIdx.x; u < (a.total_segs << plog); u += G)
      apply_unit<T>(a, u, plog, p, q, s_list, s_scan, &s_lbase, red);
    xcd_sync(ctl, xb, gen);
    if (engine_failed(ctl)) break;
    if (tracer && E < kTraceRounds) {
      unsigned long long* t = a.trace + kTraceSlots * E;
      const RoundTot rt = load_tot(ctl, q);
      t[2] = wall_clock64();
      t[3] = rt.swept;
      t[4] = rt.flagged;
      t[5] = rt.edits;
      t[6] = rt.sparse;
    }
    const unsigned long long edited = load_edits(ctl, q);
    ++E;
    if (edited == 0 || stop_here) break;
    if (tail_takes(a, edited)) {
      handoff = true;
      break;
    }
  }
  // persist the state at the start of the next round, and gather it
  if (blockIdx.x == 0 && !engine_failed(ctl)) {
    for (int fi = tid; fi < a.nf; fi += 256) {
      const FieldDesc& d = a.fd[fi];
      const FieldIter s = state_at(d, E, E0);
      if (E > E0) store_iter(&as_global(d.st)->s[E & 1], s);
      if (a.out) a.out[fi] = s;
    }
    if (tid == 0) {
      ctl->epoch = E;
      ctl->rounds = E - E0;
      ctl->handoff = handoff ? kHandToTail : 0;
      ctl->idle = 0;
      ctl->kinds = kKindTiles | kKindSparse;
    }
    // k_tail's census starts cleared (the XCD arrival counters are cleared
    // already: each barrier's last arrival resets its XCD's)
    if (handoff) {
      if (tid < kXcdSlots) ctl->census[tid] = 0u;
      if (tid == 0) {
        ctl->lead.v = 0u;
        ctl->arrived.v = 0u;
      }
    }
  }
}

// The tail of the correction loop (kHandToTail): the sparse rounds after the
// engine launch that handed them over, on the blocks of one XCD (tail_round),
// until every field is done, a round needs tile sweeps (kHandToEngine: the
// host sweeps and launches the rounds again), or a barrier times out.  Launched after
// every engine launch that may hand over; without a handover it ends at once.
template <class T>
__global__ __launch_bounds__(256) void k_tail(EngineArgs a) {
  __shared__ long long s_pre[256];
  __shared__ uint32_t s_slot[256 * kCtrSlots];
  __shared__ uint32_t s_list[kApplyCap];
  __shared__ int s_scan[4];
  __shared__ long long s_lbase;
  __shared__ unsigned long long red[4];
  __shared__ uint16_t s_units[256];
  EngineCtl* ctl = a.ctl;
  if (ctl->handoff != kHandToTail) return;
  XcdBar xb;
  if (!tail_census(ctl, xb)) return;
  unsigned gen = relaxed_load(&ctl->bar_gen.v);
  const unsigned long long E0 = ctl->epoch;
  unsigned long long E = E0;
  RoundLds L;
  L.pre = s_pre;
  L.slot = s_slot;
  L.list = s_list;
  L.scan = s_scan;
  L.lbase = &s_lbase;
  L.red = red;
  L.units = s_units;
  int rc = 0;
  while (!engine_failed(ctl) && (rc = tail_round<T>(a, xb, gen, E, E0, L)) == 0) {
  }
  // persist the state at the start of the next round, and gather it
  if (blockIdx.x == 0 && !engine_failed(ctl)) {
    const int tid = threadIdx.x;
    for (int fi = tid; fi < a.nf; fi += 256) {
      const FieldDesc& d = a.fd[fi];
      const FieldIter s = state_at<true>(d, E, E0);
      if (E > E0) store_iter(&as_global(d.st)->s[E & 1], s);
      if (a.out) a.out[fi] = s;
      // (round E was handed back before its start: whoever runs it finds the
      // counters of round E + 1 clear, as after a round's start)
      if (rc == 2) clear_ctr(&as_global(d.st)->c[(E + 1) % 3]);
    }
    if (rc == 2) clear_tot(ctl, (int)((E + 1) % 3));
    if (tid == 0) {
      ctl->epoch = E;
      ctl->rounds = E - E0;
      ctl->handoff = rc == 2 ? kHandToEngine : kTailDone;
      ctl->idle = 0;  // (plain rounds may follow)
      ctl->kinds = kKindTiles | kKindSparse;
    }
  }
}

// Directions of f for every field of a batch whose caller gave none, before
// the engine runs: a plain (non-cooperative) grid, one wave per tile or, where the
// tiles are too few to fill the chip, per part of one (128^3 binary32, 256
// tiles: 26 us by tiles, 18 us in eighths).  One kernel per dimension, each taking only its
// own fields.
template <class T, int DIM>
__global__ __launch_bounds__(256) void k_dirs_fields(const FieldDesc* fd, int nf,
                                                     int64_t total_tiles, int32_t parts_log) {
  __shared__ WaveLds<T, DIM, KIND_DIRS> sm[4];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int64_t waves = total_tiles << parts_log;
  const int32_t run = xcd_run(waves);
  const int64_t blocks = tile_blocks(waves);
  for (int64_t vb = blockIdx.x; vb < blocks; vb += gridDim.x) {
    const int64_t w = first_tile(vb, run) + wave;
    if (w >= waves) continue;
    const int64_t tt = w >> parts_log;
    const FieldDesc& d = fd[field_of_tile(fd, nf, tt)];
    if (d.dirs_given || d.geo.ndim != DIM) continue;
    wave_tile<T, KIND_DIRS, false, false, DIM>(
        sm[wave], nullptr, (const T*)d.f, (const T*)nullptr, d.dirs, nullptr, T(0), d.geo,
        (int32_t)(tt - d.tile_base), nullptr, (T*)nullptr, (int32_t)(w - (tt << parts_log)),
        1 << parts_log);
  }
}

// Tile detection of the round the workspace's epoch names, as a plain kernel
// (see engine_sweep in engine.hpp); it adds to the same counters, flag
// bitmaps and totals as the engine's own tile detection.  One tile per wave: a
// wave looks at 64 of its tiles at a time, one per lane, and marches those that
// are its kernel's (every tile of a field in its first round, or the marked tiles of
// a field in a tile round).
// Waves per SIMD of the sweeps: the most that spills next to nothing (a march that
// spills waits for memory in every step: sweeps of a 512^3 binary32 field took
// 0.66 ms at four waves against 0.56 ms at three, of a 1024 x 1024 x 768
// binary64 one 5.2 ms at three against 3.3 ms at two).  The first sweep that also
// makes the directions of f marches two fields and gets one wave less: it reads
// f once for both (1024 x 1024 x 768 binary64: 1.94 ms directions + 4.71 ms
// sweep -> 5.74 ms; 512^3 binary32 is bound by vector instructions either way,
// 0.21 + 0.39 -> 0.59 ms; 256 2D fields 0.59 + 1.21 -> 1.46 ms).
template <class T, int DIM, int KIND>
constexpr int sweep_waves() {
  return (sizeof(T) == 4 ? 4 : 3) - (DIM == 3 ? 1 : 0) - (KIND == KIND_FIRST ? 1 : 0);
}
// COPY (one field, first round): fhat is read from a.src, and the field's g
// written from it on the way.
template <class T, int KIND, bool PROP, bool COPY, int DIM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    sweep_waves<T, DIM, KIND>()))) void k_sweep(EngineArgs a) {
  __shared__ WaveLds<T, DIM, KIND> s_w[4];
  __shared__ int32_t s_delta[16];
  __shared__ int s_cur[4];
  __shared__ unsigned long long s_cnt[4][4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  WaveLds<T, DIM, KIND>& sm = s_w[wave];
  EngineCtl* ctl = a.ctl;
  const unsigned long long E = ctl->epoch;  // written by the previous launch
  if (KIND == KIND_NEXT) {
    // nothing to do in a round without fields in tile rounds (marks that stay
    // set only widen a later one)
    if (a.plain && (ctl->idle || !(ctl->kinds & kKindTiles))) return;
  }
  for (int k = lane; k < (int)(sizeof(sm.flags) / 4); k += 64) sm.flags[k] = 0u;
  if (DIM == 3) set_flag_deltas(s_delta, kRowBits3, kRowBits3 * (TY + 2));
  else set_flag_deltas(s_delta, kRowBits2, 0);
  __syncthreads();
  const int p = (int)(E & 1), q = (int)(E % 3);
  auto counters = [&](int f) { return &as_global(a.fd[f].st)->c[q].s[ctr_slot()]; };
  unsigned long long* const all_sw = &ctl->tot[q][ctr_slot()].swept;
  const int32_t run = xcd_run(a.total_tiles);
  const int64_t blocks = tile_blocks(a.total_tiles);
  const int64_t W = gridDim.x;  // (a multiple of the XCDs)
  int cur = -1;  // the field whose counts these are
  unsigned long long m = 0, nf = 0, nb = 0, sw = 0;
  for (int64_t base = blockIdx.x; base < blocks; base += W * 64) {
    const int64_t mine =
        base + lane * W < blocks ? first_tile(base + lane * W, run) + wave : a.total_tiles;
    int fi = -1;
    bool take = false;
    if (mine < a.total_tiles) {
      fi = field_of_tile(a.fd, a.nf, mine);
      const FieldDesc& d = a.fd[fi];
      if (d.geo.ndim == DIM) {  // (the other dimension's kernel takes the others)
        const FieldIter s = state_at(d, E, E);
        if (KIND != KIND_NEXT) {
          take = !s.started && !s.done;
        } else {
          const gptr<uint8_t> flag = as_global(d.act) + p * tile_count(d.geo) + (mine - d.tile_base);
          if (*flag) {
            *flag = 0;
            take = s.started && !s.done && sparse_items(d, s, E) < 0;
          }
        }
      }
    }
    for (unsigned long long todo = __ballot(take); todo; todo &= todo - 1ull) {
      const int l = __builtin_ctzll(todo);
      const int ft = __builtin_amdgcn_readlane(fi, l);
      const FieldDesc& d = a.fd[ft];
      if (ft != cur) {
        if (cur >= 0 && lane == 0) flush_counts(counters(cur), m, nf, nb, sw, all_sw);
        m = nf = nb = sw = 0;
        cur = ft;
      }
      const int32_t tile =
          (int32_t)(first_tile(base + (int64_t)l * W, run) + wave - d.tile_base);
      const LaneCounts c =
          wave_tile<T, KIND, PROP, COPY, DIM>(sm, s_delta, (const T*)(COPY ? a.src : d.g),
                                              (const T*)d.f, d.dirs, d.bm, (T)d.xi_t, d.geo, tile,
                                              d.prop, (T*)d.g);
      const unsigned long long t = wave_sum(pack3(c.mism, c.nf, c.nb));
      m += uniform((int32_t)unpack3(t, 0));
      nf += uniform((int32_t)unpack3(t, 1));
      nb += uniform((int32_t)unpack3(t, 2));
      sw += (unsigned long long)uniform(tile_voxels(d.geo, tile));
    }
  }
  // the rest, one set of atomics for the waves that end on the same field
  if (lane == 0) {
    s_cur[wave] = cur;
    s_cnt[wave][0] = m;
    s_cnt[wave][1] = nf;
    s_cnt[wave][2] = nb;
    s_cnt[wave][3] = sw;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 0; i < 4; ++i) {
      const int f = s_cur[i];
      if (f < 0) continue;
      for (int j = i + 1; j < 4; ++j) {
        if (s_cur[j] != f) continue;
        for (int k = 0; k < 4; ++k) s_cnt[i][k] += s_cnt[j][k];
        s_cur[j] = -1;
      }
      flush_counts(counters(f), s_cnt[i][0], s_cnt[i][1], s_cnt[i][2], s_cnt[i][3], all_sw);
    }
  }
}

template <class T>
static void dirs_dims(int dims, const FieldDesc* fd, int nf, int64_t total_tiles, hipStream_t s) {
  int32_t parts_log = 0;
  while (parts_log < 3 && total_tiles << (parts_log + 1) <= 2048) ++parts_log;
  int64_t grid = tile_blocks(total_tiles << parts_log);
  if (grid > (1 << 20)) grid = 1 << 20;
  if (dims & 2)
    hipLaunchKernelGGL((k_dirs_fields<T, 2>), dim3((unsigned)grid), dim3(256), 0, s, fd, nf,
                       total_tiles, parts_log);
  if (dims & 4)
    hipLaunchKernelGGL((k_dirs_fields<T, 3>), dim3((unsigned)grid), dim3(256), 0, s, fd, nf,
                       total_tiles, parts_log);
}

hipError_t engine_dirs(int dtype, int dims, const FieldDesc* fd, int nf, int64_t total_tiles,
                       hipStream_t s) {
  if (dtype == PMSZ_F32) dirs_dims<float>(dims, fd, nf, total_tiles, s);
  else dirs_dims<double>(dims, fd, nf, total_tiles, s);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_fill(uint32_t* p, int64_t words, uint32_t v) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t w = (int64_t)blockIdx.x * 256 + threadIdx.x; w < words; w += stride) p[w] = v;
}

hipError_t engine_fill(void* p, size_t bytes, uint32_t v, hipStream_t s) {
  const int64_t words = (int64_t)(bytes / 4);
  int64_t b = (words + 255) / 256;
  if (b < 1) b = 1;
  if (b > 4096) b = 4096;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)b), dim3(256), 0, s, (uint32_t*)p, words, v);
  return hipGetLastError();
}

hipError_t engine_zero(void* p, size_t bytes, hipStream_t s) { return engine_fill(p, bytes, 0u, s); }

// Zero `words` words of p and copy n elements of V from src to dst.
template <class V>
__global__ __launch_bounds__(256) void k_zero_copy(uint32_t* p, int64_t words, V* dst,
                                                   const V* src, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * 256, at = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t i = at; i < n; i += stride) dst[i] = src[i];
  for (int64_t w = at; w < words; w += stride) p[w] = 0u;
}

hipError_t engine_zero_copy(void* p, size_t bytes, void* dst, const void* src, size_t copy_bytes,
                            hipStream_t s) {
  const int64_t words = (int64_t)(bytes / 4);
  const bool wide = ((uintptr_t)dst | (uintptr_t)src | copy_bytes) % 16 == 0;
  const int64_t n = (int64_t)(copy_bytes / (wide ? 16 : 4));
  int64_t b = ((words > n ? words : n) + 255) / 256;
  b = b < 1 ? 1 : b < 4096 ? b : 4096;
  if (wide)
    hipLaunchKernelGGL(k_zero_copy<uint4>, dim3((unsigned)b), dim3(256), 0, s, (uint32_t*)p, words,
                       (uint4*)dst, (const uint4*)src, n);
  else
    hipLaunchKernelGGL(k_zero_copy<uint32_t>, dim3((unsigned)b), dim3(256), 0, s, (uint32_t*)p,
                       words, (uint32_t*)dst, (const uint32_t*)src, n);
  return hipGetLastError();
}

// Cooperative grid: as many resident blocks as the chip holds, but no more
// than there is work for (fewer arrivals make the barrier cheaper).
// Resident blocks per compute unit and compute units of a device, looked up
// once per (device, kernel) under a lock (calls may come from several host
// threads).
struct Occupancy {
  int per_cu = -1, cus = -1;
};
// Resident blocks per compute unit of a 256-thread kernel on a device, and
// the device's compute units (cached per kernel and device).
static hipError_t occupancy_of(const void* kernel, int dev, Occupancy& out) {
  static std::mutex mu;
  static std::map<std::pair<const void*, int>, Occupancy> cache;
  std::lock_guard<std::mutex> lk(mu);
  auto it = cache.find({kernel, dev});
  if (it == cache.end()) {
    Occupancy o;
    hipError_t e = hipDeviceGetAttribute(&o.cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&o.per_cu, kernel, 256, 0);
    if (e != hipSuccess) return e;
    it = cache.emplace(std::make_pair(kernel, dev), o).first;
  }
  out = it->second;
  return hipSuccess;
}
// Waves enough to fill the chip kSweepFill times over, at most one per tile.
constexpr int64_t kSweepFill = 4;
template <class T, int KIND, bool PROP, bool COPY, int DIM>
static hipError_t sweep_t(const EngineArgs& a, hipStream_t s) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  Occupancy occ;
  if ((e = occupancy_of((const void*)k_sweep<T, KIND, PROP, COPY, DIM>, dev, occ)) != hipSuccess)
    return e;
  int64_t grid = kSweepFill * (occ.per_cu > 0 ? occ.per_cu : 1) * (occ.cus > 0 ? occ.cus : 1);
  grid = (grid + kXcds - 1) / kXcds * kXcds;
  if (grid > tile_blocks(a.total_tiles)) grid = tile_blocks(a.total_tiles);
  hipLaunchKernelGGL((k_sweep<T, KIND, PROP, COPY, DIM>), dim3((unsigned)grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <class T, bool PROP, int DIM>
static hipError_t sweep_kind(int kind, const EngineArgs& a, hipStream_t s) {
  if (kind == KIND_NEXT) return sweep_t<T, KIND_NEXT, PROP, false, DIM>(a, s);
  if (kind == KIND_FIRST)
    return a.src ? sweep_t<T, KIND_FIRST, PROP, true, DIM>(a, s)
                 : sweep_t<T, KIND_FIRST, PROP, false, DIM>(a, s);
  return a.src ? sweep_t<T, KIND_FIRST_GIVEN, PROP, true, DIM>(a, s)
               : sweep_t<T, KIND_FIRST_GIVEN, PROP, false, DIM>(a, s);
}

template <class T>
static hipError_t sweep_dims(int kind, bool prop, int dims, const EngineArgs& a, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (dims & 2)
    e = prop ? sweep_kind<T, true, 2>(kind, a, s) : sweep_kind<T, false, 2>(kind, a, s);
  if (e == hipSuccess && (dims & 4))
    e = prop ? sweep_kind<T, true, 3>(kind, a, s) : sweep_kind<T, false, 3>(kind, a, s);
  return e;
}

hipError_t engine_sweep(int dtype, int kind, bool prop, int dims, const EngineArgs& a,
                        hipStream_t s) {
  if (dtype == PMSZ_F32) return sweep_dims<float>(kind, prop, dims, a, s);
  return sweep_dims<double>(kind, prop, dims, a, s);
}

// Resident blocks of a kernel on the current device, at most `most`.
static hipError_t resident(const void* kernel, int64_t most, unsigned* grid) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  Occupancy occ;
  if ((e = occupancy_of(kernel, dev, occ)) != hipSuccess) return e;
  int64_t n = (int64_t)(occ.per_cu > 0 ? occ.per_cu : 1) * (occ.cus > 0 ? occ.cus : 1);
  if (n > most) n = most;
  *grid = (unsigned)(n < 1 ? 1 : n);
  return hipSuccess;
}

template <class T, int DIM>
static hipError_t sparse_t(const EngineArgs& a, hipStream_t s) {
  unsigned grid = 1;
  const hipError_t e = resident((const void*)k_sparse<T, DIM>, a.total_segs * 4, &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_sparse<T, DIM>), dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t engine_sparse(int dtype, int dims, const EngineArgs& a, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (dims & 2) e = dtype == PMSZ_F32 ? sparse_t<float, 2>(a, s) : sparse_t<double, 2>(a, s);
  if (e == hipSuccess && (dims & 4))
    e = dtype == PMSZ_F32 ? sparse_t<float, 3>(a, s) : sparse_t<double, 3>(a, s);
  return e;
}

template <class T>
static hipError_t apply_t(const EngineArgs& a, hipStream_t s) {
  unsigned grid = 1;
  hipError_t e =  // a 256-word unit per wave
      resident((const void*)k_apply<T>, a.total_segs * (kSegWords / kUnitWords) / 4, &grid);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_apply<T>, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}
hipError_t engine_apply(int dtype, const EngineArgs& a, hipStream_t s) {
  return dtype == PMSZ_F32 ? apply_t<float>(a, s) : apply_t<double>(a, s);
}

template <class T, int WAVES>
static hipError_t launch_w(const EngineArgs& a, hipStream_t s, int64_t want, int* grid_out) {
  unsigned grid = 1;
  hipError_t e = resident((const void*)k_engine<T, WAVES>, want, &grid);
  if (e != hipSuccess) return e;
  if (grid_out) *grid_out = (int)grid;
  EngineArgs copy = a;
  void* args[] = {&copy};
  return hipLaunchCooperativeKernel((const void*)k_engine<T, WAVES>, dim3(grid), dim3(256), args,
                                    0, s);
}

template <class T>
static hipError_t launch_t(const EngineArgs& a, hipStream_t s, int* grid_out, bool clear) {
  // the XCD and compute-unit barrier state starts cleared in every launch
  // (the round totals after it are kept: a sweep kernel may have added to
  // the current round's already)
  hipError_t e;
  if (clear &&
      (e = engine_fill(&a.ctl->xbar[0], offsetof(EngineCtl, tot) - offsetof(EngineCtl, xbar), 0u,
                       s)) != hipSuccess)
    return e;
  const int64_t want = a.total_tiles > a.total_segs ? a.total_tiles : a.total_segs;
  // The full register budget (200 registers, two waves per SIMD, so 512 resident
  // blocks) where a grid of a block per tile fits in that, or the launch is left with
  // sparse rounds: the tile march spills at four (three) waves, and a spill's first
  // touch of memory costs a phase microseconds.  Whole calls with four (three) waves
  // and with two, us: 64^3 binary32 (256 tiles) 271 and 265, two of 64^3 (512) 311 and
  // 294, binary64 278 and 265; two of 1337 x 1021 binary64 with dense rounds (536) 472 and
  // 476, two of 100^3 (600) 640 and 656, eight of 100^3 (2400) 1133 and 1218, binary32 1101
  // and 1143; 320^3, sparse after plain rounds, 627 and 593.
  if (a.plain || want <= 512) return launch_w<T, 1>(a, s, want, grid_out);
  return launch_w<T, sizeof(T) == 4 ? 4 : 3>(a, s, want, grid_out);
}

hipError_t engine_launch(int dtype, const EngineArgs& a, hipStream_t s, int* grid_out,
                         bool clear) {
  if (dtype == PMSZ_F32) return launch_t<float>(a, s, grid_out, clear);
  return launch_t<double>(a, s, grid_out, clear);
}

// kTailGrid blocks, all resident (cooperative); an engine launch that hands
// over leaves the census and barrier words of the tail cleared.
template <class T>
static hipError_t tail_t(const EngineArgs& a, hipStream_t s) {
  EngineArgs copy = a;
  void* args[] = {&copy};
  return hipLaunchCooperativeKernel((const void*)k_tail<T>, dim3(kTailGrid), dim3(256), args, 0,
                                    s);
}

hipError_t engine_tail(int dtype, const EngineArgs& a, hipStream_t s) {
  if (dtype == PMSZ_F32) return tail_t<float>(a, s);
  return tail_t<double>(a, s);
}

}  // namespace pmsz
