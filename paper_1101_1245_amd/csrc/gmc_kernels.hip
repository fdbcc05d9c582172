// gmc_kernels.hip -- gfx950 kernels of the coupled photon-electron transport.
//
// A pass kernel transports the particles of ONE type (Sec. II.C.2: photons and
// electrons are never simulated together, which removes the divergence of
// the photon-electron coupling).  Each wavefront owns a contiguous range of
// the work queue; a lane runs events on its particle until it dies, reaches
// the per-visit event cap (the N of Sec. II.C.3) or its per-visit secondary
// budget, and then takes the next particle of the range (lane-level refill,
// the "pool" idea of Sec. II.C.3 inside one launch).  Survivors and
// secondaries go to the wavefront's private segments of two staging queues,
// so no lane ever waits on a shared counter; when a workgroup is done, its
// wavefronts copy their segments into the accumulating queues, one atomic per
// workgroup and queue reserving the room (the stream compaction of Sec.
// II.C.3).  Rare, costly events are sampled by many lanes together: electron
// hard events once enough lanes of the wavefront wait at one, photon
// absorptions, which are parked, at the end.
// Deposits are uint64 fixed-point atomics, so the dose is an exact integer
// sum independent of thread order.  Cross-section and stopping-power tables
// are staged in LDS by every workgroup.
#include <algorithm>
#include <mutex>

#include "gmc_device.hpp"

namespace gmc {
using namespace dev;

// ------------------------------------------------------------------ source
// Primary of history h (Sec. II.C.2, initParticle): parallel beam along +z at
// z = 0, position uniform over the field, energy monoenergetic, triangular or
// tabulated.  Uses the first block (words 0-3) of the history's root stream.
struct Primary { float x, y; uint32_t e; };

// Tabulated spectrum (a histogram): the bin j with C_j <= u < C_j+1 of the
// normalised CDF C at the edges (C_0 = 0, C_n = 1), found by bisection for
// the first edge above u, and the linear inverse inside it, in FP64.
__device__ __forceinline__ uint32_t sample_tabulated(const double* tab, uint32_t n, double u) {
  const double* edge = tab;
  const double* cdf = tab + n + 1;
  uint32_t lo = 0u, hi = n;   // cdf[lo] <= u < cdf[hi]
  while (hi - lo > 1u) {
    const uint32_t mid = (lo + hi) >> 1;
    if (cdf[mid] <= u) lo = mid; else hi = mid;
  }
  const double e = edge[lo] + (u - cdf[lo]) / (cdf[lo + 1] - cdf[lo]) * (edge[lo + 1] - edge[lo]);
  return (uint32_t)__double2uint_rn(e * 134217728.0);
}

__device__ __forceinline__ Primary sample_primary(const DevSource& a, uint32_t key0, uint32_t key1, uint32_t h) {
  const Block blk = philox(0u, 0u, 0u, h, key0, key1);
  const float u0 = to_uniform(blk.w0), u1 = to_uniform(blk.w1), u2 = to_uniform(blk.w2);
  Primary p;
  p.x = a.cx + (u0 - 0.5f) * a.wx;
  p.y = a.cy + (u1 - 0.5f) * a.wy;
  if (a.spectrum == 1) {
    const float lo = a.e_lo, md = a.e_mode, hi = a.e_hi;
    const float fc = (md - lo) / (hi - lo);
    const float e = (u2 < fc) ? lo + sqrtf(u2 * (hi - lo) * (md - lo)) : hi - sqrtf((1.0f - u2) * (hi - lo) * (hi - md));
    p.e = to_lsb(e);
  } else if (a.spectrum == 2) {
    p.e = sample_tabulated(a.tab, a.tab_n, (double)u2);
  } else {
    p.e = a.e_lsb;
  }
  return p;
}

// Batch (off + h) mod K of history h (m = batch_magic(K)): the estimated
// quotient is at most one short, so one conditional subtraction each for the
// remainder and for the offset; no 32-bit sum overflows.  8 instructions where
// the general 32-bit remainder takes about 20.
__device__ __forceinline__ uint32_t batch_of(uint32_t h, uint32_t K, uint32_t m, uint32_t off) {
  uint32_t k = h - __umulhi(h, m) * K;
  k = min(k, k - K);
  k += off;
  return min(k, k - K);
}
// Word of voxel v in the tally line (its batch's line of the target's first
// tile) of a target with K batches.  Lines are counted in 32 bits: 2^32 of
// them are 512 GB.
__device__ __forceinline__ unsigned long long* tally_word(const DevTally& t, uint32_t line, uint32_t K, uint32_t v) {
  return t.base + ((size_t)((v / kTallyBlock) * K + line) * kTallyBlock + (v % kTallyBlock));
}

// Sparse jobs (kMark) mark the lines they add to, for a finalize that reads
// only those.
template <bool kMark>
__device__ __forceinline__ void mark_line(const DevTally& t, uint32_t line) {
  if constexpr (kMark) t.mark[line] = 1;
}
// Offset of voxel v's batch 0 in a tally.
__device__ __forceinline__ size_t vox_off(uint32_t v, uint32_t K) {
  return (size_t)(v / kTallyBlock) * kTallyBlock * K + (v % kTallyBlock);
}

// Tally addition through the global address space: the tally pointers come
// from the beam table, so the compiler cannot tell their address space and
// would issue a flat atomic, which also holds the LDS counter -- every later
// table read in LDS would then wait for the atomic to be acknowledged.
__device__ __forceinline__ void tally_add(unsigned long long* p, unsigned long long v) {
  typedef __attribute__((address_space(1))) unsigned long long global_u64;
  __hip_atomic_fetch_add((global_u64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Admission sizes for both particle types: take the next histories of each
// type while its accumulating buffer holds fewer than `chunk` particles.
__global__ void k_admit_plan(AdmitPlanArgs a) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  for (int t = 0; t < 2; ++t) {
    uint32_t* cnt = t == 0 ? a.count0 : a.count1;
    const uint32_t have = *cnt;
    const uint32_t left = a.total[t] - a.cursor[t];
    uint32_t take = 0;
    if (have < a.chunk) {
      take = min(left, a.chunk);
      take = have < a.cap ? min(take, a.cap - have) : 0u;
    }
    a.out[t].base = have;
    a.out[t].count = take;
    a.out[t].cursor = a.cursor[t];
    a.cursor[t] += take;
    *cnt = have + take;
  }
}

// Primaries of one particle type, written by index.  Primaries that start
// outside the phantom escape and sub-cutoff ones deposit where they enter;
// both are stored with zero energy, which the pass kernels skip.
__global__ void __launch_bounds__(256) k_admit(AdmitArgs a) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  const AdmitPlan pl = *a.plan;
  const bool valid = i < pl.count;
  const uint32_t g = pl.cursor + i;
  uint32_t j = 0;
  if (valid) {   // the segment holding index g: last j with start[j] <= g
    uint32_t lo = 0, hi = a.nb;
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) >> 1;
      if (a.start[mid] <= g) lo = mid; else hi = mid;
    }
    j = lo;
  }
  const uint32_t beam = valid ? a.beam_of[j] : 0u;
  uint32_t h = 0u;   // history number: the beam's first history plus its index in the beam
  Primary p{0.0f, 0.0f, 0u};
  int particle = 0;
  if (valid) {
    const DevSource src = a.sources[beam];
    particle = src.particle;
    h = g - a.start[j] + a.seg_h[j] + src.h0;
    p = sample_primary(src, a.key0, a.beams[beam].key1, h);
  }
  const bool in = valid && inside(a.ph, p.x, p.y, 0.0f);
  const uint32_t cut = particle == 0 ? a.cut.pcut_lsb : a.cut.ecut_lsb;
  const bool keep = in && p.e >= cut;
  const unsigned long long esc = (valid && !in) ? p.e : 0ull;
  if (in && !keep) {
    int ix, iy, iz;
    const uint32_t v = voxel(a.ph, p.x, p.y, 0.0f, ix, iy, iz);
    const DevBeam b = a.beams[beam];
    const DevTally& t = a.tally;
    if (p.e) {
      tally_add(tally_word(t, b.a_line + batch_of(h, t.ka, t.ma, b.a_off), t.ka, v), (unsigned long long)p.e);
      if (t.kb) tally_add(tally_word(t, batch_of(h, t.kb, t.mb, b.b_off), t.kb, v), (unsigned long long)p.e);
    }
  }
  if (valid) {
    const uint32_t slot = pl.base + i;
    if (slot < a.out.cap)
      put(entry<kQGranules>(a.out, slot), p.x, p.y, 0.0f, 0.0f, 0.0f, 1.0f, keep ? p.e : 0u, h, 0u, 0u, 4u, beam);
    else
      ctr_add(a.ctr, C_OVERFLOW, 1ull);
  }
  const unsigned long long ein = wave_sum(valid ? (unsigned long long)p.e : 0ull);
  const unsigned long long es = wave_sum(esc);
  if (lane_id() == 0) {
    if (ein) ctr_add(a.ctr, C_E_IN, ein);
    if (es) ctr_add(a.ctr, C_E_ESC, es);
  }
}

// ------------------------------------------------------------ lane state
struct Lane {
  float x, y, z, u, v, w;
  uint32_t e, beam;
  Stream s;
  uint32_t la, lb;             // this history's batch lines of tally targets a and b
};

// The entry at p (its granule 0).  The lane's pointers into the
// tally are kept as 32-bit line numbers, and the beam table entry is one
// 16-byte read, from LDS where it fits (explicit address spaces: a merged
// pointer would make it a flat load, which waits on both the LDS and the
// memory counters).
__device__ __forceinline__ void load_lane(Lane& L, const uint4* p, const PassArgs& a, const DevBeam* lbeams) {
  const uint4 g0 = p[QG_POS * kQBlock], g1 = p[QG_DIR * kQBlock], g2 = p[QG_STREAM * kQBlock];
  L.x = __uint_as_float(g0.x); L.y = __uint_as_float(g0.y); L.z = __uint_as_float(g0.z);
  L.e = g0.w;
  L.u = __uint_as_float(g1.x); L.v = __uint_as_float(g1.y); L.w = __uint_as_float(g1.z);
  L.beam = g1.w;
  L.s.hist = g2.x; L.s.plo = g2.y; L.s.phi = g2.z; L.s.n = g2.w;
  typedef __attribute__((address_space(3))) const uint4 lds_beam;
  typedef __attribute__((address_space(1))) const uint4 global_beam;
  uint4 b;
  if (a.n_beams <= kLdsBeams) {
    lds_beam* lp = (lds_beam*)lbeams + L.beam;
    b = make_uint4(lp->x, lp->y, lp->z, lp->w);
  } else {
    global_beam* gp = (global_beam*)a.beams + L.beam;
    b = make_uint4(gp->x, gp->y, gp->z, gp->w);
  }
  const DevTally& t = a.tally;
  L.s.k1 = b.x;
  L.la = b.y + batch_of(L.s.hist, t.ka, t.ma, b.z);
  if (t.kb) L.lb = batch_of(L.s.hist, t.kb, t.mb, b.w);
}

__device__ __forceinline__ void store_lane(const Lane& L, uint4* p) {
  put(p, L.x, L.y, L.z, L.u, L.v, L.w, L.e, L.s.hist, L.s.plo, L.s.phi, L.s.n, L.beam);
}

struct Child { float u, v, w; uint32_t e, plo, phi; };

// A wavefront's share of the pass: the work queue's items m are cut into
// chunks (64 items by default) and chunk c goes to wavefront c mod W, so that every
// wavefront gets a slice of every part of the queue -- carried-over
// particles, survivors, the other type's secondaries, new primaries -- whose
// lives differ widely; contiguous shares left many wavefronts idle while a
// few finished theirs.  Loads stay coalesced within a chunk.  [next, end) is
// the wave-uniform cursor over the wavefront's own items, numbered 0..end-1.
struct WaveRange {
  static constexpr bool kStack = false, kMark = false;
  uint32_t next, end, wave, waves, lg;
  const uint4* work;           // the work queue
  uint32_t tail_lanes, tail_min;   // tail requeue (tail_lanes = 0: off)
  // every item of the share has been handed to a lane
  __device__ __forceinline__ bool done() { return next >= end; }
  // whether lanes still busy are requeued: the share (a large one) is done
  // and few are left
  __device__ __forceinline__ bool tail(uint32_t busy) {
    return tail_lanes > 0u && done() && end >= tail_min && busy <= tail_lanes;
  }
  __device__ __forceinline__ uint32_t left() const { return end - next; }
  // the k-th of the next items (k < left())
  __device__ __forceinline__ const uint4* item(uint32_t k) const {
    const uint32_t j = next + k;
    return entry<kQGranules>(work, (((j >> lg) * waves + wave) << lg) + (j & ((1u << lg) - 1u)));
  }
  __device__ __forceinline__ void take(uint32_t n) { next += n; }
};

__device__ __forceinline__ WaveRange wave_range(const PassArgs& a, const PassPlan& P, uint32_t wave, uint32_t waves) {
  const uint32_t lg = P.chunk_log2;
  const uint32_t chunks = (uint32_t)(((uint64_t)P.m + (1u << lg) - 1u) >> lg);
  WaveRange r{0u, 0u, wave, waves, lg, a.work.base, P.admitting ? (uint32_t)a.tail_lanes : 0u, a.tail_min};
  if (wave < chunks) {
    const uint32_t own = (chunks - 1u - wave) / waves + 1u;
    r.end = own << lg;
    if ((chunks - 1u) % waves == wave) r.end -= (chunks << lg) - P.m;   // the last chunk may be partial
  }
  return r;
}

// A wavefront's work in the persistent round kernel: chunks of 2^lg
// consecutive work-queue items claimed one at a time from a device work
// queue.  The m items of a type are split into `parts` contiguous
// partitions, each with its own chunk counter; a wavefront claims from its
// workgroup's partition (block mod parts) first, so most claims are atomics
// on a counter only that workgroup's wavefronts share.  When that partition
// is used up the wavefront steals: its 64 lanes read 64 partitions' counters
// at once (agent-scope loads; a counter only grows, so one that reads
// exhausted is exhausted) and it claims from the first that still has a
// chunk, moving on through all partitions before it gives up.  It never
// claims more than `cap` items in all (the bound its staging segments were
// sized for); the caps add up to more than m, so every item is claimed by
// some wavefront.  No wavefront waits for another.  [next, end) are queue
// indices of the current chunk's items not yet handed out.
struct ClaimRange {
  static constexpr bool kStack = false, kMark = false;
  const uint4* work;          // the work queue
  uint32_t tail_lanes, tail_min;   // as in WaveRange
  uint32_t next, end;
  uint32_t taken, cap;        // items claimed so far, most it may claim
  uint32_t cur;               // partition of the last successful claim
  uint32_t m, parts, lg;
  bool exhausted;             // every partition found used up (or the cap reached)
  uint32_t* ctr;              // [parts] chunk counters of this type

  __device__ __forceinline__ uint32_t lo(uint32_t p) const {
    return (uint32_t)(((uint64_t)m * p) / parts);
  }
  __device__ __forceinline__ uint32_t chunks(uint32_t p) const {
    return (lo(p + 1u) - lo(p) + (1u << lg) - 1u) >> lg;
  }
  // one atomic on partition p's counter (wave-uniform p): true and the
  // chunk set when p still had one
  __device__ __forceinline__ bool grab(uint32_t p) {
    uint32_t c = 0u;
    if (lane_id() == 0u) c = atomicAdd(ctr + p, 1u);
    c = __shfl(c, 0);
    const uint32_t a = lo(p), b = lo(p + 1u);
    const uint64_t first = (uint64_t)a + ((uint64_t)c << lg);
    if (first >= b) return false;
    next = (uint32_t)first;
    end = (uint32_t)min<uint64_t>(first + (1u << lg), b);
    taken += end - next;
    cur = p;
    return true;
  }
  __device__ __forceinline__ void claim() {
    if (exhausted || taken + (1u << lg) > cap) {
      exhausted = true;
      return;
    }
    if (grab(cur)) return;
    // steal: scan the partitions after the current one, 64 at a time
    for (uint32_t base = 1u; base < parts; base += 64u) {
      const uint32_t off = base + lane_id();
      uint32_t p = cur + off;
      if (p >= parts) p -= parts;
      bool avail = false;
      if (off < parts) {
        const uint32_t c = __hip_atomic_load(ctr + p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        avail = c < chunks(p);
      }
      unsigned long long mask = lanes_with(avail);
      while (mask) {
        const int j = __ffsll((long long)mask) - 1;
        const uint32_t pj = (uint32_t)__shfl((int)p, j);
        if (grab(pj)) return;
        mask &= mask - 1ull;
      }
    }
    exhausted = true;
  }
  // wave-uniform: claims the next chunk when the current one is used up
  __device__ __forceinline__ bool done() {
    if (next < end) return false;
    claim();
    return next >= end;
  }
  __device__ __forceinline__ bool tail(uint32_t busy) {
    return tail_lanes > 0u && done() && taken >= tail_min && busy <= tail_lanes;
  }
  __device__ __forceinline__ uint32_t left() const { return end - next; }
  __device__ __forceinline__ const uint4* item(uint32_t k) const { return entry<kQGranules>(work, next + k); }
  __device__ __forceinline__ void take(uint32_t n) { next += n; }
};

__device__ __forceinline__ ClaimRange claim_range(const PassArgs& a, const PassPlan& P, const ClaimType& T,
                                                  uint32_t* ctr, uint32_t block) {
  ClaimRange r;
  r.work = a.work.base;
  r.tail_lanes = P.admitting ? (uint32_t)a.tail_lanes : 0u;
  r.tail_min = a.tail_min;
  r.next = r.end = 0u;
  r.taken = 0u;
  r.cap = T.cap;
  r.m = T.m;
  r.parts = T.parts;
  r.cur = block % T.parts;
  r.lg = P.chunk_log2;
  r.exhausted = T.m == 0u;
  r.ctr = ctr;
  return r;
}

// A wavefront's own stack in the history pool: the entries of its segment of
// one type, newest first.  What its lanes create goes on top of the same
// stacks, so a history's particles are followed depth first and the stacks
// stay short.  The last few busy lanes are put back rather than run out when
// other work waits: a full wavefront of the other type, or (rich) claims of a
// full wavefront, which the pool makes once its two stacks hold fewer than 64.
template <bool kMarks>
struct StackRange {
  static constexpr bool kStack = true, kMark = kMarks;
  WaveSeg& same;
  const WaveSeg& other;
  bool rich;
  uint32_t tail_lanes;
  __device__ __forceinline__ bool done() const { return same.used == 0u; }
  __device__ __forceinline__ bool tail(uint32_t busy) const {
    return done() && busy <= tail_lanes &&
           (other.used >= 64u || (rich && busy + other.used < 64u));
  }
  __device__ __forceinline__ uint32_t left() const { return same.used; }
  __device__ __forceinline__ const uint4* item(uint32_t k) const { return same.at(same.used - 1u - k); }
  __device__ __forceinline__ void take(uint32_t n) {
    same.used -= n;
    wave_fence();   // the entries may be written again by other lanes
  }
};
// Room an iteration of each loop needs.  Electrons: the delta rays and the
// photons of 64 hard events, 64 lanes put back, and as much again in reserve.
// Photons take what their own stack gave; their electrons: 64 recoils, two for
// each photon parked at its absorption, and then the 256 entries that let the
// electron loop start.
template <bool kMarks>
struct ElectronStack : StackRange<kMarks> {
  using StackRange<kMarks>::same;
  using StackRange<kMarks>::other;
  __device__ __forceinline__ bool short_of_room() const {
    return same.used + 192u > same.cap || other.used + 128u > other.cap;
  }
};
template <bool kMarks>
struct PhotonStack : StackRange<kMarks> {
  using StackRange<kMarks>::other;
  __device__ __forceinline__ bool short_of_room(uint32_t parked) const {
    return other.used + 2u * parked + 448u > other.cap;
  }
};

// Lanes without a particle take the next items of the range, in lane order,
// once at least a.refill_lanes of them are idle (one refill then pays the
// load latency for many lanes; with every lane idle it always proceeds).
// Entries with zero energy (primaries settled by the source) are skipped.
// Returns whether this lane took one.
template <class R>
__device__ __forceinline__ bool refill(Lane& L, bool& have, int& events, int& pushes, R& r, const PassArgs& a,
                                       const DevBeam* lbeams) {
  const unsigned long long need = lanes_with(!have);
  if (need == 0 || __popcll(need) < a.refill_lanes || r.done()) return false;
  const uint32_t n = min((uint32_t)__popcll(need), r.left());
  const uint32_t k = rank_in(need);
  const bool took = !have && k < n;
  if (took) {
    load_lane(L, r.item(k), a, lbeams);
    have = L.e != 0;
    if constexpr (!R::kStack) {   // visits are counted where they have a budget
      events = 0;
      pushes = 0;
    }
  }
  r.take(n);
  return took;
}

// Write one entry into a wave segment; a slot beyond the segment (never
// expected: the per-visit budgets bound every segment) is counted, not written.
__device__ __forceinline__ bool seg_ok(const WaveSeg& g, uint32_t slot, unsigned long long* ctr) {
  if (slot < g.cap) return true;
  ctr_add(ctr, C_OVERFLOW, 1ull);
  return false;
}

template <bool kMark>
__device__ __forceinline__ void deposit(const Lane& L, const PassArgs& a, uint32_t v, uint32_t e) {
  if (!e) return;
  tally_add(tally_word(a.tally, L.la, a.tally.ka, v), (unsigned long long)e);
  mark_line<kMark>(a.tally, (v / kTallyBlock) * a.tally.ka + L.la);
  if (a.tally.kb) tally_add(tally_word(a.tally, L.lb, a.tally.kb, v), (unsigned long long)e);
}

// Deposits of the electron loop on their way to the tally.  A 64-bit atomic
// addition to scattered addresses completes at 2.37e10 a second on this chip,
// wherever the words lie; lanes of one instruction that add to the same 64
// bytes count once.  So each lane keeps the sums of the 64-byte segment (8
// voxels, 2 x 1 x 4) its electron is in in a column of LDS, and adds the whole
// segment when the lane deposits in another: an electron makes 0.36 to 0.39
// such additions per step (the tracks of 15 MeV electron and photon beams on
// 0.5 cm water and of 6 MeV photons on 0.25 cm slabs in double precision)
// where it made 0.60 to one voxel each.  Eight lanes add one segment in one
// instruction.  The water job of 5.25e6 electrons and 6.5e7 photons went from
// 33.5 to 29.3 ms, 4e7 photons on 128^3 slabs from 19.7 to 16.6, 256 beamlets
// from 102 to 87.5 (with every addition left out: 20.9, 12.5 and 47).
//
// A column's sums are one particle's deposits, below 2^32 units; a lane that
// takes another particle marks its segment as left (kLeft), so its next
// deposit adds it.  Integer additions make the result independent of when
// they happen.
constexpr uint32_t kLeft = 1u << 31;
struct Column {
  uint32_t* lds;               // the wavefront's columns: [8 words][64 lanes], rotated
  uint32_t seg = ~0u;          // segment of the column (its first voxel / 8), all ones: none
  uint32_t la = 0u, lb = 0u;   // tally lines of targets a and b it belongs to
};
constexpr int kColWords = 8 * 64;   // words of a wavefront's columns
// Word w of lane l: rotated by 8 w, so that both a lane's additions (one word
// each of 64 lanes) and a segment's read-out (8 words of one lane) spread over
// the banks.
__device__ __forceinline__ uint32_t col_at(uint32_t w, uint32_t l) { return w * 64u + ((l + w * 8u) & 63u); }

// The segments of the lanes in m (a ballot), added to the tally and cleared.
// All lanes of the wavefront call this: 8 of them serve one segment.
template <bool kMark>
__device__ __forceinline__ void flush_columns(const Column& c, const DevTally& t, unsigned long long m) {
  const uint32_t lane = lane_id();
  const uint32_t n = (uint32_t)__popcll(m), below = rank_in(m);
  const bool want = (m >> lane) & 1ull;
  // lane j learns the j-th lane of m
  const uint32_t dst = want ? below : n + lane - below;
  const int src = __builtin_amdgcn_ds_permute((int)(dst << 2), (int)lane);
  const uint32_t w = lane & 7u;
  for (uint32_t r = 0u; r < n; r += 8u) {
    const uint32_t j = r + (lane >> 3);
    const uint32_t f = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(j << 2), src);
    const uint32_t half = ((uint32_t)__builtin_amdgcn_ds_bpermute((int)(f << 2), (int)c.seg) & 1u) * 8u + w;
    const uint32_t la = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(f << 2), (int)c.la);
    const uint32_t lb = t.kb ? (uint32_t)__builtin_amdgcn_ds_bpermute((int)(f << 2), (int)c.lb) : 0u;
    if (j < n) {
      const uint32_t e = __hip_atomic_exchange(c.lds + col_at(w, f), 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (e) {
        tally_add(t.base + ((size_t)la * kTallyBlock + half), (unsigned long long)e);
        if (t.kb) tally_add(t.base + ((size_t)lb * kTallyBlock + half), (unsigned long long)e);
      }
      if (w == 0u) mark_line<kMark>(t, la);
    }
  }
}

// One deposit (dep units in voxel v, none where dep is 0) of each lane (all
// lanes call this).
template <bool kMark>
__device__ __forceinline__ void deposit_column(Column& c, const Lane& L, const DevTally& t, uint32_t v, uint32_t dep) {
  const uint32_t seg = v / 8u;
  const bool moved = dep != 0u && seg != c.seg;
  const unsigned long long m = lanes_with(moved && c.seg != ~0u);
  if (m) flush_columns<kMark>(c, t, m);
  if (moved) {
    c.seg = seg;
    c.la = (v / kTallyBlock) * t.ka + L.la;
    if (t.kb) c.lb = (v / kTallyBlock) * t.kb + L.lb;
  }
  if (dep) __hip_atomic_fetch_add(c.lds + col_at(v & 7u, lane_id()), dep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// One photon flight and interaction decision (Sec. II.A, Eqs. 1-3): free path
// with the majorant, then one uniform against the cumulative Compton,
// photoelectric, pair partials of the voxel; fictitious otherwise.
enum { PH_ESCAPE = 0, PH_FICT = 1, PH_COMPTON = 2, PH_PHOTO = 3, PH_PAIR = 4 };

__device__ __forceinline__ int photon_flight(Lane& L, const PassArgs& a, const float* tab, const float* majg,
                                             uint32_t& v0, uint32_t& viol) {
  L.s.align();
  const float ef = (float)L.e * kLsbF;
  const TPos p = tpos_in(a.tab, ef);
  const float muh = majg[p.i];
  if (!(muh > 0.0f)) return PH_ESCAPE;
  const float d = fdiv(-fln(L.s.uniform_at<0>()), muh);
  L.x = fmaf(d, L.u, L.x);
  L.y = fmaf(d, L.v, L.y);
  L.z = fmaf(d, L.w, L.z);
  if (!inside(a.ph, L.x, L.y, L.z)) return PH_ESCAPE;
  int ix, iy, iz;
  v0 = voxel(a.ph, L.x, L.y, L.z, ix, iy, iz);
  const uint2 vx = a.ph.vox[v0];
  const float rho = __uint_as_float(vx.x);
  const float3 c = lerp_ph(tab, (int)vx.y * kNE, p);
  const float mc = rho * c.x, mcp = rho * c.y;
  const float mt = (L.e > a.cut.two_mc2_lsb) ? rho * c.z : mcp;
  if (mt > muh) ++viol;
  const float r = L.s.uniform_at<1>() * muh;
  if (r >= mt) return PH_FICT;
  if (r < mc) return PH_COMPTON;
  if (r < mcp) return PH_PHOTO;
  return PH_PAIR;
}

// End of a pass kernel's workgroup (every thread calls it once, after its
// wavefront's loop): particles m..n-1 of the work queue go to the front of
// the type's new queue (grid-stride over all threads), then one atomic per
// destination reserves room for the workgroup's staged entries and each
// wavefront copies its own segments.  Entries beyond a queue's capacity are
// counted, not written.
__device__ __forceinline__ void copy_entry(const DevQueue& dst, uint32_t d, const uint4* from, unsigned long long* ctr) {
  if (d >= dst.cap) {
    ctr_add(ctr, C_OVERFLOW, 1ull);
    return;
  }
  uint4* to = entry<kQGranules>(dst, d);
  const uint4 g0 = from[0], g1 = from[kQBlock], g2 = from[2 * kQBlock];
  to[0] = g0;
  to[kQBlock] = g1;
  to[2 * kQBlock] = g2;
}

__device__ __forceinline__ void append_outputs(const PassArgs& a, const PassPlan& P, const WaveSeg& gs,
                                               const WaveSeg& go) {
  __shared__ uint32_t s_used[2][16];
  __shared__ uint32_t s_base[2];
  const uint32_t carry = P.n - P.m;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < carry; i += gridDim.x * blockDim.x)
    copy_entry(a.dst_same, i, entry<kQGranules>(a.carry_src, P.m + i), a.ctr);
  const uint32_t wl = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint32_t n0 = min(gs.used, gs.cap), n1 = min(go.used, go.cap);
  if (lane_id() == 0) {
    s_used[0][wl] = n0;
    s_used[1][wl] = n1;
  }
  __syncthreads();
  if (threadIdx.x < 2u) {
    uint32_t tot = 0;
    for (uint32_t w = 0; w < nw; ++w) tot += s_used[threadIdx.x][w];
    s_base[threadIdx.x] = tot ? atomicAdd(threadIdx.x == 0 ? a.cnt_same : a.cnt_other, tot) : 0u;
  }
  __syncthreads();
  uint32_t o0 = s_base[0], o1 = s_base[1];
  for (uint32_t w = 0; w < wl; ++w) {
    o0 += s_used[0][w];
    o1 += s_used[1][w];
  }
  for (uint32_t i = lane_id(); i < n0; i += 64u) copy_entry(a.dst_same, o0 + i, gs.at(i), a.ctr);
  for (uint32_t i = lane_id(); i < n1; i += 64u) copy_entry(a.dst_other, o1 + i, go.at(i), a.ctr);
}

// Photon absorbed in voxel v0 (Sec. II.B.2): photoelectric effect, one
// electron with the whole energy in the Sauter direction; or pair production,
// two electrons sharing E - 2 mc^2 uniformly at opposite azimuths, 2 mc^2 to
// the sink.  Electrons below the cutoff are deposited in v0; those above are
// left in c0 (and c1), nchild of them.
template <bool kMark>
__device__ __forceinline__ void absorb_photon(Lane& L, const PassArgs& a, int kind, uint32_t v0, Child& c0, Child& c1,
                                              int& nchild, unsigned long long& acc_sink) {
  if (kind == PH_PHOTO) {
    const float ef = (float)L.e * kLsbF;
    const float cost = sample_sauter(ef, L.s);
    const float phi = kTwoPi * L.s.uniform();
    c0.u = L.u; c0.v = L.v; c0.w = L.w;
    rotate(c0.u, c0.v, c0.w, cost, phi);
    if (L.e >= a.cut.ecut_lsb) {
      c0.e = L.e;
      child_path(L.s.plo, L.s.phi, L.s.n, 0u, c0.plo, c0.phi);
      nchild = 1;
    } else {
      deposit<kMark>(L, a, v0, L.e);
    }
    return;
  }
  const uint32_t avail = L.e - a.cut.two_mc2_lsb;
  const uint32_t t1 = min((uint32_t)fminf(L.s.uniform_at<2>() * (float)avail, kMaxLsbF), avail);
  const uint32_t t2 = avail - t1;
  const float cs1 = pair_cos((float)t1 * kLsbF, L.s.uniform_at<3>());
  const float cs2 = pair_cos((float)t2 * kLsbF, L.s.uniform_at<0>());
  const float phi = kTwoPi * L.s.uniform_at<1>();
  acc_sink += a.cut.two_mc2_lsb;
  c0.u = L.u; c0.v = L.v; c0.w = L.w;
  rotate(c0.u, c0.v, c0.w, cs1, phi);
  c1.u = L.u; c1.v = L.v; c1.w = L.w;
  rotate(c1.u, c1.v, c1.w, cs2, phi + kPi);
  if (t1 >= a.cut.ecut_lsb) {
    c0.e = t1;
    child_path(L.s.plo, L.s.phi, L.s.n, 0u, c0.plo, c0.phi);
    nchild = 1;
  } else {
    deposit<kMark>(L, a, v0, t1);
  }
  if (t2 >= a.cut.ecut_lsb) {
    c1.e = t2;
    child_path(L.s.plo, L.s.phi, L.s.n, 1u, c1.plo, c1.phi);
    if (nchild == 0) c0 = c1;   // keep the pushed children contiguous
    ++nchild;
  } else {
    deposit<kMark>(L, a, v0, t2);
  }
}

// Push the children of one event (nchild of c0, c1 per lane) to the wave's
// electron staging segment.
__device__ __forceinline__ void push_electrons(const Lane& L, const PassArgs& a, WaveSeg& g, int nchild,
                                               const Child& c0, const Child& c1, uint32_t& sec) {
  const uint32_t before = g.used;
  const WaveSeg::Slots sl = g.append(nchild >= 1, nchild >= 2);
  sec += g.used - before;
  const uint32_t hist = L.s.hist;
  if (nchild >= 1 && seg_ok(g, sl.s0, a.ctr))
    put(g.at(sl.s0), L.x, L.y, L.z, c0.u, c0.v, c0.w, c0.e, hist, c0.plo, c0.phi, 0u, L.beam);
  if (nchild >= 2 && seg_ok(g, sl.s1, a.ctr))
    put(g.at(sl.s1), L.x, L.y, L.z, c1.u, c1.v, c1.w, c1.e, hist, c1.plo, c1.phi, 0u, L.beam);
}

// ------------------------------------------------------------ photon pass
// One Woodcock flight per iteration (Sec. II.B.2).  Photoelectric and pair
// events end the photon: it is parked on a stack at the top of the
// wavefront's photon staging segment (with the interaction type) and the
// lane takes the next photon; once the range is done the wavefront samples
// the parked absorptions 64 at a time, so those two rarer branches do not run
// in most iterations with a few lanes each.  Each photon draws the same words
// in the same order either way.  Segment bound: each photon of the range
// leaves at most one survivor and is parked at most once, within per_wave x 2
// slots.
// Run counters a wavefront accumulates over its loop, added to the run's
// counters once at the end of the kernel: energies and majorant violations
// per lane, event counts over the wavefront (from ballots, in scalar
// registers).
struct WaveTotals {
  unsigned long long esc = 0, sink = 0;
  uint32_t viol = 0;
  uint32_t ev = 0, fict = 0, sec = 0, steps = 0, hard = 0;
  uint32_t real = 0;   // photon flights that end in a real interaction
};
__device__ __forceinline__ uint32_t count_lanes(bool b) { return (uint32_t)__popcll(lanes_with(b)); }

__device__ __forceinline__ void add_totals(const WaveTotals& t, unsigned long long* ctr) {
  const unsigned long long s_esc = wave_sum(t.esc), s_sink = wave_sum(t.sink), s_viol = wave_sum(t.viol);
  if (lane_id() == 0) {
    if (s_esc) ctr_add(ctr, C_E_ESC, s_esc);
    if (s_sink) ctr_add(ctr, C_E_SINK, s_sink);
    if (t.ev) ctr_add(ctr, C_PH_EVENTS, t.ev);
    if (t.fict) ctr_add(ctr, C_FICT, t.fict);
    if (t.real) ctr_add(ctr, C_PH_REAL, t.real);
    if (s_viol) ctr_add(ctr, C_VIOL, s_viol);
    if (t.sec) ctr_add(ctr, C_SEC, t.sec);
    if (t.steps) ctr_add(ctr, C_E_STEPS, t.steps);
    if (t.hard) ctr_add(ctr, C_HARD, t.hard);
  }
}

// The photon transport of one wavefront over its range: photon tables in
// LDS at tab (per material) and majg (majorant), the beam table at lbeams.
template <class R>
__device__ void photon_loop(const PassArgs& a, R& range, WaveSeg& gsame, WaveSeg& gother,
                            const float* tab, const float* majg, const DevBeam* lbeams, WaveTotals& tot) {
  Lane L;
  L.s.k0 = a.key0;
  bool have = false;
  int events = 0, pushes = 0;
  uint32_t npark = 0;   // parked absorptions at the segment's top, wave-uniform

  for (;;) {
    refill(L, have, events, pushes, range, a, lbeams);
    // a refill may bring only zero-energy entries: the wavefront goes on
    // until its range is done
    if (!any_lane(have)) {
      if (range.done()) break;
      continue;
    }
    int nchild = 0;
    Child c0, c1;
    bool surv = false, park = false, flown = false;
    int kind = PH_ESCAPE;
    // tail of the share: with the range empty and few lanes still busy, a
    // photon that lives on after this event is requeued (while primaries
    // remain to be admitted); a stack's are put back at once
    const bool tail = range.tail(count_lanes(have));
    if constexpr (R::kStack) {
      if (tail || range.short_of_room(npark)) {
        const WaveSeg::Slots ss = gsame.append(have, false);
        if (have) store_lane(L, gsame.at(ss.s0));
        break;
      }
    }
    if (have) {
      uint32_t v0 = 0u, dep = 0u;
      kind = photon_flight(L, a, tab, majg, v0, tot.viol);
      flown = true;
      if (kind == PH_ESCAPE) {
        tot.esc += L.e;
        have = false;
      } else if (kind == PH_FICT) {
      } else if (a.cut.mode == 1) {
        dep = L.e;
        have = false;
      } else if (kind == PH_COMPTON) {
        // scattered photon plus recoil electron (momentum conservation)
        const float ef = (float)L.e * kLsbF;
        float eps, cost;
        sample_kn(ef / kMc2, L.s, eps, cost);
        const float phi = kTwoPi * L.s.uniform();
        float nu = L.u, nv = L.v, nw = L.w;
        rotate(nu, nv, nw, cost, phi);
        const uint32_t e1 = min(to_lsb(eps * ef), L.e);
        const uint32_t te = L.e - e1;
        if (te >= a.cut.ecut_lsb) {
          const float e1f = (float)e1 * kLsbF;
          float pu = ef * L.u - e1f * nu, pv = ef * L.v - e1f * nv, pw = ef * L.w - e1f * nw;
          const float inv = rsqrtf(pu * pu + pv * pv + pw * pw);
          c0.u = pu * inv; c0.v = pv * inv; c0.w = pw * inv;
          c0.e = te;
          child_path(L.s.plo, L.s.phi, L.s.n, 0u, c0.plo, c0.phi);
          nchild = 1;
        } else {
          dep = te;
        }
        L.u = nu; L.v = nv; L.w = nw;
        L.e = e1;
        if (e1 < a.cut.pcut_lsb) {
          dep += e1;
          have = false;
        }
      } else {
        // photoelectric absorption or pair production: parked, sampled in the wave's last phase
        park = true;
        have = false;
      }
      deposit<R::kMark>(L, a, v0, dep);
      if constexpr (!R::kStack) {
        pushes += nchild;
        if (have) {
          ++events;
          if (tail || events >= a.max_events || pushes + 2 > a.max_secondaries) {
            surv = true;
            have = false;
          }
        }
      }
    }
    tot.ev += count_lanes(flown);
    tot.fict += count_lanes(flown && kind == PH_FICT);
    tot.real += count_lanes(flown && kind >= PH_COMPTON);
    // secondary electrons to the electron staging segment, survivors to the
    // bottom of the photon one, absorbed photons onto its stack
    push_electrons(L, a, gother, nchild, c0, c1, tot.sec);
    const WaveSeg::Slots ss = gsame.append(surv, false);
    if (surv && seg_ok(gsame, ss.s0, a.ctr)) store_lane(L, gsame.at(ss.s0));
    const unsigned long long pm = lanes_with(park);
    if (park) {
      const uint32_t k = npark + rank_in(pm);
      if (k < gsame.cap && gsame.cap - 1u - k >= gsame.used) {
        uint4* slot = gsame.at(gsame.cap - 1u - k);
        store_lane(L, slot);
        slot[QG_PARK * kQBlock].x = (uint32_t)kind;
      } else {
        ctr_add(a.ctr, C_OVERFLOW, 1ull);
      }
    }
    npark += (uint32_t)__popcll(pm);
  }

  // last phase: the parked absorptions with every lane busy
  if (npark) __threadfence_block();   // a lane may read an entry another lane wrote
  for (uint32_t k0 = 0; k0 < npark; k0 += 64u) {
    const uint32_t k = k0 + lane_id();
    int nchild = 0;
    Child c0, c1;
    if (k < npark) {
      const uint4* slot = gsame.at(gsame.cap - 1u - k);
      load_lane(L, slot, a, lbeams);
      L.s.resume();
      const int kind = (int)slot[QG_PARK * kQBlock].x;
      int ix, iy, iz;
      const uint32_t v0 = voxel(a.ph, L.x, L.y, L.z, ix, iy, iz);
      absorb_photon<R::kMark>(L, a, kind, v0, c0, c1, nchild, tot.sink);
    }
    push_electrons(L, a, gother, nchild, c0, c1, tot.sec);
  }
}

__device__ __forceinline__ void stage_photon_tables(float* dst, const DevTables& t) {
  for (int i = threadIdx.x; i < t.n_mat * kNE; i += blockDim.x) {
    const float4 v = t.ph[i];
    dst[i * kPhRow] = v.x;
    dst[i * kPhRow + 1] = v.y;
    dst[i * kPhRow + 2] = v.z;
  }
}

__global__ void __launch_bounds__(1024) k_photon_pass(PassArgs a) {
  extern __shared__ float4 smem[];
  float* tab = reinterpret_cast<float*>(smem);
  stage_photon_tables(tab, a.tab);
  float* majg = tab + a.tab.n_mat * kNE * kPhRow;
  for (int i = threadIdx.x; i < kNE; i += blockDim.x) majg[i] = a.tab.maj_g[i];
  DevBeam* lbeams = reinterpret_cast<DevBeam*>(majg + kNE);
  if (a.n_beams <= kLdsBeams)
    for (int i = threadIdx.x; i < a.n_beams; i += blockDim.x) lbeams[i] = a.beams[i];
  __syncthreads();

  const uint32_t wave = wave_index();
  const PassPlan P = *a.plan;
  WaveRange range = wave_range(a, P, wave, (gridDim.x * blockDim.x) >> 6);
  WaveSeg gsame = wave_seg(a.stg_same, wave * P.seg_same, P.seg_same);
  WaveSeg gother = wave_seg(a.stg_other, wave * P.seg_other, P.seg_other);
  WaveTotals tot;
  photon_loop(a, range, gsame, gother, tab, majg, lbeams, tot);
  append_outputs(a, P, gsame, gother);
  add_totals(tot, a.ctr);
}

// ---------------------------------------------------------- electron pass
// Hard-event candidate at the end of a step (Sec. II.B.3): accepted with
// Sigma(end) / Sigma_hat, Sigma_hat being the majorant at the step-start
// energy, and split into Moller or bremsstrahlung.  The electron stands at
// the step's end point in voxel v1 with its energy after the step's loss;
// energy below the cutoffs is deposited in v1.  Returns whether the electron
// lives on; a secondary above its cutoff is left in c0 (ctype 0 photon, 1
// electron).
template <bool kMark>
__device__ __forceinline__ bool hard_event(Lane& L, const PassArgs& a, const float4* smem, float sh, uint32_t v1,
                                           Child& c0, int& ctype, bool& hit, uint32_t& c_viol) {
  const float t1f = (float)L.e * kLsbF;
  const float ur = L.s.uniform_at<0>();   // a step ends at a block boundary
  const uint2 vy = a.ph.vox[v1];
  const float rho1 = __uint_as_float(vy.x);
  const float4 t1 = lerp4(smem, (int)vy.y * kNE, tpos_in(a.tab, t1f));
  const float sm = (L.e > a.cut.kcut2_lsb) ? rho1 * t1.y : 0.0f;
  const float sb = (L.e > a.cut.kc_lsb) ? rho1 * t1.z : 0.0f;
  if (sm + sb > sh) ++c_viol;
  const float r = ur * sh;
  if (r < sm) {
    // Moller: binary collision with a free electron at rest
    hit = true;
    const float eps = sample_moller(t1f, a.cut.kcut, L.s);
    const uint32_t wl = min(to_lsb(eps * t1f), L.e);
    const uint32_t tp = L.e - wl;
    const float wf = (float)wl * kLsbF, tpf = (float)tp * kLsbF;
    const float cd = sqrtf(fdiv(wf * (t1f + 2.0f * kMc2), t1f * (wf + 2.0f * kMc2)));
    const float cpp = sqrtf(fdiv(tpf * (t1f + 2.0f * kMc2), t1f * (tpf + 2.0f * kMc2)));
    const float phi = kTwoPi * L.s.uniform();
    c0.u = L.u; c0.v = L.v; c0.w = L.w;
    rotate(c0.u, c0.v, c0.w, cd, phi);
    rotate(L.u, L.v, L.w, cpp, phi + kPi);
    if (wl >= a.cut.ecut_lsb) {
      c0.e = wl;
      child_path(L.s.plo, L.s.phi, L.s.n, 0u, c0.plo, c0.phi);
      ctype = 1;
    } else {
      deposit<kMark>(L, a, v1, wl);
    }
    L.e = tp;
  } else if (r < sm + sb) {
    // bremsstrahlung: electron direction unchanged, photon at mc^2/E
    hit = true;
    const float k = sample_brems(t1f, a.cut.kc, L.s);
    const float phi = kTwoPi * L.s.uniform();
    const uint32_t kl = min(to_lsb(k), L.e);
    c0.u = L.u; c0.v = L.v; c0.w = L.w;
    rotate(c0.u, c0.v, c0.w, __cosf(fdiv(kMc2, t1f + kMc2)), phi);
    if (kl >= a.cut.pcut_lsb) {
      c0.e = kl;
      child_path(L.s.plo, L.s.phi, L.s.n, 0u, c0.plo, c0.phi);
      ctype = 0;
    } else {
      deposit<kMark>(L, a, v1, kl);
    }
    L.e -= kl;
  }
  if (L.e < a.cut.ecut_lsb) {
    deposit<kMark>(L, a, v1, L.e);
    return false;
  }
  return true;
}

// One condensed step per iteration (Sec. II.B.3): e_s = min{d_vox, e_s-max,
// e_hard} (Eq. 4) with e_hard from the majorant at the step-start energy;
// energy loss of Eq. 8 read with the factor s; random hinge at zeta e_s with
// the deflection energy taken before or after the loss at random; the loss is
// deposited in the step-start voxel.
//
// A lane whose step ends at a hard-event candidate waits there with its
// electron until hard_lanes of 64 busy lanes do (or the wavefront leaves the
// loop); then they sample their hard events together and step on.  Sampling
// each where it occurs would run the Moller and bremsstrahlung code in most
// iterations with 3 lanes.  Parking them on a stack in memory, the lane
// going on with another electron, kept more lanes busy, but cost the stores,
// the loads, a refill and, twice, the flush of the lane's column: the water
// job took 29.2 ms so and takes 25.8, 4e7 photons on the 128^3 slabs 16.5 and
// 15.0, 256 beamlets 86 and 75.  A particle's draws and operations, and so
// the dose, are the same either way.
//
// Segment bound: each particle of the range (at most per_wave) leaves at most
// max_secondaries secondaries and one survivor.
// The electron transport of one wavefront over its range: electron tables
// in LDS at tab (per material), maje (hard-event majorant) and ms (screening),
// the beam table at lbeams.
//
// The step is straight-line code under one branch: its lanes differ in which
// of its cases they meet (leaving the phantom, stopping, the coin, small and
// large deflections, the six faces), so branches would run both sides anyway
// and cost the copies and mask work at every join.  Values of lanes that have
// left or stopped are computed along and dropped.  The voxel is looked up
// once, at the start of a step: an electron that leaves the phantom at the
// end of one is found there (or at its hard event).  Against the branching
// form (two lookups, three places of additions): 2594 -> 2156 vector
// instructions and 128 -> 114 registers in the kernel, the water job 42.7 ->
// 41.3 ms, 256 beamlets 136.7 -> 131.0 ms.
template <class R>
__device__ void electron_loop(const PassArgs& a, R& range, WaveSeg& gsame, WaveSeg& gother,
                              const float4* tab, const float* maje, const float* ms, const DevBeam* lbeams,
                              uint32_t* cols, WaveTotals& tot) {
  Lane L;
  L.s.k0 = a.key0;
  Column col{cols};
  bool have = false;
  int events = 0, pushes = 0;
  bool wait = false;               // at a hard event (a lane that waits has an electron)
  float hsh = 0.0f;                // its majorant

  for (;;) {
    if (refill(L, have, events, pushes, range, a, lbeams)) col.seg |= kLeft;
    bool surv = false;
    const uint32_t nb = count_lanes(have), nw = count_lanes(wait);
    if (!nb) {
      if (range.done()) break;
      continue;
    }
    // tail of the share: with the range empty and few lanes still busy, an
    // electron that has stepped in this visit is requeued rather than holding
    // the wavefront for its last few particles -- while primaries remain to be
    // admitted, when a next pass comes anyway; a stack's are put back at once
    bool leave = range.tail(nb);
    if constexpr (R::kStack) leave = leave || range.short_of_room();
    if (nw && (leave || nw * 64u >= nb * (uint32_t)a.hard_lanes)) {
      int ctype = -1;
      bool hit = false;
      Child c0;
      if (wait) {
        wait = false;
        have = false;
        int jx, jy, jz;
        uint32_t v1;
        if (electron_voxel(a.ph, L.x, L.y, L.z, L.u, L.v, L.w, jx, jy, jz, v1)) {
          have = hard_event<R::kMark>(L, a, tab, hsh, v1, c0, ctype, hit, tot.viol);
          if constexpr (!R::kStack) {
            if (ctype >= 0) ++pushes;
            // visit budget spent: requeued
            if (have && (events >= a.max_events || pushes + 1 > a.max_secondaries)) {
              surv = true;
              have = false;
            }
          }
        } else {
          tot.esc += L.e;
        }
      }
      tot.hard += count_lanes(hit);
      tot.sec += count_lanes(ctype >= 0);
      // delta rays to the electron staging segment, photons to the photon one
      const WaveSeg::Slots se = gsame.append(ctype == 1, false);
      if (ctype == 1 && seg_ok(gsame, se.s0, a.ctr))
        put(gsame.at(se.s0), L.x, L.y, L.z, c0.u, c0.v, c0.w, c0.e, L.s.hist, c0.plo, c0.phi, 0u, L.beam);
      const WaveSeg::Slots sg = gother.append(ctype == 0, false);
      if (ctype == 0 && seg_ok(gother, sg.s0, a.ctr))
        put(gother.at(sg.s0), L.x, L.y, L.z, c0.u, c0.v, c0.w, c0.e, L.s.hist, c0.plo, c0.phi, 0u, L.beam);
    }
    if constexpr (R::kStack) {
      if (leave) {
        const WaveSeg::Slots ss = gsame.append(have, false);
        if (have) store_lane(L, gsame.at(ss.s0));
        break;
      }
    } else if (leave && have && events > 0) {
      surv = true;
      have = false;
    }
    bool in = false;
    uint32_t v0 = 0u, dep = 0u;
    if (have && !wait) {
      L.s.align();
      int ix, iy, iz;
      in = electron_voxel(a.ph, L.x, L.y, L.z, L.u, L.v, L.w, ix, iy, iz, v0);
      const uint2 vx = a.ph.vox[v0];
      // the step's four words: one stream block
      const Block rn = philox(L.s.n >> 2, L.s.plo, L.s.phi, L.s.hist, L.s.k0, L.s.k1);
      L.s.n += 4u;
      const float dv = fmaxf(dist_boundary(a.ph, L.x, L.y, L.z, L.u, L.v, L.w, ix, iy, iz), a.ph.skin);
      const float tf = (float)L.e * kLsbF;
      const TPos p0 = tpos_in(a.tab, tf);
      const float sh = maje[p0.i];
      const float ehard = fdiv(-fln(to_uniform(rn.w0)), sh);   // infinite where the majorant is zero
      const float rho0 = __uint_as_float(vx.x);
      const int base0 = (int)vx.y * kNE;
      float es = dv;
      if (a.cut.esmax_gcm2 > 0.0f) {
        asm volatile("");   // rarely set: kept a scalar branch
        const float emax = rho0 > 0.0f ? fdiv(a.cut.esmax_gcm2, rho0) : kInf;
        es = emax < es ? emax : es;
      }
      const bool hard = ehard < es && a.cut.mode != 2;
      es = hard ? ehard : es;
      const float l0 = rho0 * lerp_x(tab, base0, p0);
      const float tm = fmaxf(tf - 0.5f * es * l0, a.cut.emin);
      const float esr = es * rho0;
      const float de = esr * lerp_x(tab, base0, tpos_in(a.tab, tm));
      // the hinge word: fraction zeta from its top bits, deflection-energy coin from bit 0
      const float zeta = to_uniform(rn.w1);
      const float s1 = zeta * es;
      L.x = fmaf(s1, L.u, L.x);
      L.y = fmaf(s1, L.v, L.y);
      L.z = fmaf(s1, L.w, L.z);
      const uint32_t dl = (uint32_t)fminf(de * kInvLsbF, kMaxLsbF);   // de >= 0
      const bool stop = dl >= L.e || L.e - dl < a.cut.ecut_lsb;
      dep = stop ? L.e : dl;
      dep = in ? dep : 0u;
      if (!in) tot.esc += L.e;
      const uint32_t e1 = min(L.e - dl, L.e);   // in range for the lanes that stop, too
      if (a.cut.mode != 2) {
        asm volatile("");
        const float tms = (rn.w1 & 1u) ? (float)e1 * kLsbF : tf;
        const float xx = esr * lerp_w(tab, base0, tpos_in(a.tab, tms));
        // G1 = 1 - exp(-x), by its series where the subtraction would cancel
        const float g1s = xx * (1.0f - 0.5f * xx * (1.0f - xx * (1.0f / 3.0f)));
        const float g1 = xx < 1e-3f ? g1s : 1.0f - fexp(-xx);
        rotate_om(L.u, L.v, L.w, wentzel_om(a.tab, ms, g1, to_uniform(rn.w2)), kTwoPi * to_uniform(rn.w3));
      }
      L.e = e1;
      const float s2 = (1.0f - zeta) * es;
      L.x = fmaf(s2, L.u, L.x);
      L.y = fmaf(s2, L.v, L.y);
      L.z = fmaf(s2, L.w, L.z);
      have = in && !stop;
      wait = have && hard;
      hsh = sh;
      if constexpr (!R::kStack) {
        if (have) ++events;
        if (have && !wait && events >= a.max_events) {
          surv = true;
          have = false;
        }
      }
    }
    tot.steps += count_lanes(in);
    deposit_column<R::kMark>(col, L, a.tally, v0, dep);
    // survivors to the electron staging segment
    if (any_lane(surv)) {
      const WaveSeg::Slots se = gsame.append(surv, false);
      if (surv && seg_ok(gsame, se.s0, a.ctr)) store_lane(L, gsame.at(se.s0));
    }
  }
  const unsigned long long m = lanes_with(col.seg != ~0u);
  if (m) flush_columns<R::kMark>(col, a.tally, m);
}

__global__ void __launch_bounds__(1024) k_electron_pass(PassArgs a) {
  extern __shared__ float4 smem[];
  const int nt = a.tab.n_mat * kNE;
  for (int i = threadIdx.x; i < nt; i += blockDim.x) smem[i] = a.tab.el[i];
  float* maje = reinterpret_cast<float*>(smem + nt);
  float* ms = maje + kNE;
  for (int i = threadIdx.x; i < kNE; i += blockDim.x) maje[i] = a.tab.maj_e[i];
  for (int i = threadIdx.x; i < kNms; i += blockDim.x) ms[i] = a.tab.ms[i];
  DevBeam* lbeams = reinterpret_cast<DevBeam*>(ms + kNms);
  if (a.n_beams <= kLdsBeams)
    for (int i = threadIdx.x; i < a.n_beams; i += blockDim.x) lbeams[i] = a.beams[i];
  uint32_t* cols = reinterpret_cast<uint32_t*>(lbeams + kLdsBeams) + (threadIdx.x >> 6) * kColWords;
  for (int i = lane_id(); i < kColWords; i += 64) cols[i] = 0u;
  __syncthreads();

  const uint32_t wave = wave_index();
  const PassPlan P = *a.plan;
  WaveRange range = wave_range(a, P, wave, (gridDim.x * blockDim.x) >> 6);
  WaveSeg gsame = wave_seg(a.stg_same, wave * P.seg_same, P.seg_same);
  WaveSeg gother = wave_seg(a.stg_other, wave * P.seg_other, P.seg_other);
  WaveTotals tot;
  electron_loop(a, range, gsame, gother, smem, maje, ms, lbeams, cols, tot);
  append_outputs(a, P, gsame, gother);
  add_totals(tot, a.ctr);
}

// ------------------------------------------------------------ round kernel
// End of a round kernel's workgroup: both types' carried-over particles to
// the front of their new queues, then one atomic per type reserves room for
// the workgroup's staged outputs of that type and each wavefront copies its
// segments.
__device__ __forceinline__ void append_round(const RoundArgs& r, const PassPlan& Pe, const PassPlan& Pg,
                                             const WaveSeg& se, const WaveSeg& sg) {
  __shared__ uint32_t s_used[2][16];
  __shared__ uint32_t s_base[2];
  const uint32_t ce = Pe.n - Pe.m, cg = Pg.n - Pg.m;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < ce; i += gridDim.x * blockDim.x)
    copy_entry(r.e.dst_same, i, entry<kQGranules>(r.e.carry_src, Pe.m + i), r.e.ctr);
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < cg; i += gridDim.x * blockDim.x)
    copy_entry(r.g.dst_same, i, entry<kQGranules>(r.g.carry_src, Pg.m + i), r.g.ctr);
  const uint32_t wl = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const uint32_t n0 = min(se.used, se.cap), n1 = min(sg.used, sg.cap);
  if (lane_id() == 0) {
    s_used[0][wl] = n0;
    s_used[1][wl] = n1;
  }
  __syncthreads();
  if (threadIdx.x < 2u) {
    uint32_t tot = 0;
    for (uint32_t w = 0; w < nw; ++w) tot += s_used[threadIdx.x][w];
    s_base[threadIdx.x] = tot ? atomicAdd(threadIdx.x == 0 ? r.e.cnt_same : r.g.cnt_same, tot) : 0u;
  }
  __syncthreads();
  uint32_t o0 = s_base[0], o1 = s_base[1];
  for (uint32_t w = 0; w < wl; ++w) {
    o0 += s_used[0][w];
    o1 += s_used[1][w];
  }
  for (uint32_t i = lane_id(); i < n0; i += 64u) copy_entry(r.e.dst_same, o0 + i, se.at(i), r.e.ctr);
  for (uint32_t i = lane_id(); i < n1; i += 64u) copy_entry(r.g.dst_same, o1 + i, sg.at(i), r.g.ctr);
}

// The persistent round kernel (the batched form's pool of persistent
// wavefronts, Sec. II.C.3): every workgroup stages both table blocks, and
// each wavefront claims chunks of the round's electrons from the device work
// queue until none is left (or its cap is reached), finishes its electrons
// and their hard events, then claims photons the same way.  The
// electron and photon loops are those of the pass kernels; only where their
// items come from differs.  Electron outputs of both phases go to the
// wavefront's electron segment, photon outputs to its photon segment.
__global__ void __launch_bounds__(kRoundMaxBlock) k_round(RoundArgs r) {
  extern __shared__ float4 smem[];
  const int nt = r.e.tab.n_mat * kNE;
  float4* te = smem;
  float* tg = reinterpret_cast<float*>(te + nt);
  float* majg = tg + nt * kPhRow;
  float* maje = majg + kNE;
  float* ms = maje + kNE;
  DevBeam* lbeams = reinterpret_cast<DevBeam*>(ms + kNms);
  stage_photon_tables(tg, r.g.tab);
  for (int i = threadIdx.x; i < nt; i += blockDim.x) te[i] = r.e.tab.el[i];
  for (int i = threadIdx.x; i < kNE; i += blockDim.x) {
    majg[i] = r.g.tab.maj_g[i];
    maje[i] = r.e.tab.maj_e[i];
  }
  for (int i = threadIdx.x; i < kNms; i += blockDim.x) ms[i] = r.e.tab.ms[i];
  if (r.e.n_beams <= kLdsBeams)
    for (int i = threadIdx.x; i < r.e.n_beams; i += blockDim.x) lbeams[i] = r.e.beams[i];
  uint32_t* cols = reinterpret_cast<uint32_t*>(lbeams + kLdsBeams) + (threadIdx.x >> 6) * kColWords;
  for (int i = lane_id(); i < kColWords; i += 64) cols[i] = 0u;
  __syncthreads();

  const uint32_t wave = wave_index();
  const PassPlan Pg = *r.g.plan, Pe = *r.e.plan;
  WaveSeg se = wave_seg(r.e.stg_same, wave * Pe.seg_same, Pe.seg_same);
  WaveSeg sg = wave_seg(r.g.stg_same, wave * Pg.seg_same, Pg.seg_same);
  WaveTotals tot;
  ClaimRange re = claim_range(r.e, Pe, r.claims[1], r.claim_ctr + kMaxClaimParts, blockIdx.x);
  electron_loop(r.e, re, se, sg, te, maje, ms, lbeams, cols, tot);
  ClaimRange rg = claim_range(r.g, Pg, r.claims[0], r.claim_ctr, blockIdx.x);
  photon_loop(r.g, rg, sg, se, tg, majg, lbeams, tot);
  append_round(r, Pe, Pg, se, sg);
  add_totals(tot, r.e.ctr);
}

// ------------------------------------------------------------ history pool
// What a wavefront knows of the claims: how far the cursor of each type had
// come when it last claimed (2^63 and above: none are left).
struct Claims {
  unsigned long long seen[2] = {0ull, 0ull};
};
constexpr unsigned long long kNoneLeft = 1ull << 63;

// The next histories for this wavefront: it claims a share of what remains of
// one particle type (the one whose beams are further behind) with one atomic
// on a 64-bit cursor, samples the primaries on its lanes and puts them on its
// stacks.  Primaries that start outside the phantom escape, sub-cutoff ones
// deposit where they enter.  Returns the number claimed, 0 once none remain
// (or another wavefront has given the job up, which it tells through the
// cursors).
//
// Claim size: half an even share of the rest as last seen, at most kPoolClaim and
// at least an even share of all up to 64, so that large jobs take full
// wavefronts at a time and small ones spread evenly over all wavefronts: their
// time is that of the longest chain of steps in one.  The claim is one
// operation on one hot word: with the cursors read first, and claims of 128,
// the water job took 42.7 ms instead of 34.3.
template <bool kMark>
__device__ uint32_t pool_admit(const PoolArgs& p, WaveSeg& se, WaveSeg& sg, Claims& cl) {
  const PassArgs& a = p.a;
  const unsigned long long l0 = cl.seen[0] < p.total[0] ? p.total[0] - cl.seen[0] : 0ull;
  const unsigned long long l1 = cl.seen[1] < p.total[1] ? p.total[1] - cl.seen[1] : 0ull;
  if (l0 == 0ull && l1 == 0ull) return 0u;
  const int t = l1 && (!l0 || (float)l1 * (float)p.total[0] >= (float)l0 * (float)p.total[1]) ? 1 : 0;
  const unsigned long long total = p.total[t], left = t ? l1 : l0;
  const unsigned long long share = (total + p.waves - 1u) / p.waves;   // an even share of all
  const uint32_t want = (uint32_t)min(max(left / (2ull * p.waves), min(share, 64ull)), (unsigned long long)kPoolClaim);
  unsigned long long g0 = 0ull;
  if (lane_id() == 0u) g0 = atomicAdd(p.cursor[t], (unsigned long long)want);
  g0 = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(g0 >> 32)) << 32) |
       (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)g0);
  cl.seen[t] = g0 + want;
  if (g0 >= total) {   // taken meanwhile; the other type may have some
    if (g0 >= kNoneLeft) cl.seen[1 - t] = kNoneLeft;
    return want;
  }
  const uint32_t n = (uint32_t)min((unsigned long long)want, total - g0);
  const uint32_t* start = p.start[t];
  WaveSeg& seg = t ? se : sg;
  const uint32_t cut = t ? a.cut.ecut_lsb : a.cut.pcut_lsb;
  unsigned long long ein = 0ull, esc = 0ull;
  for (uint32_t i0 = 0u; i0 < n; i0 += 64u) {
    const uint32_t i = i0 + lane_id();
    const bool valid = i < n;
    const uint32_t g = (uint32_t)(p.first[t] + g0) + i;
    uint32_t h = 0u, beam = 0u;   // history number: the beam's first history plus its index in the beam
    Primary pr{0.0f, 0.0f, 0u};
    if (valid) {   // the segment holding index g: last j with start[j] <= g
      uint32_t lo = 0, hi = p.nb[t];
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (start[mid] <= g) lo = mid; else hi = mid;
      }
      beam = p.beam_of[t][lo];
      const DevSource src = p.sources[beam];
      h = g - start[lo] + p.seg_h[t][lo] + src.h0;
      pr = sample_primary(src, a.key0, a.beams[beam].key1, h);
    }
    const bool in = valid && inside(a.ph, pr.x, pr.y, 0.0f);
    const bool keep = in && pr.e >= cut;
    if (valid) ein += pr.e;
    if (valid && !in) esc += pr.e;
    if (in && !keep && pr.e) {
      int ix, iy, iz;
      const uint32_t v = voxel(a.ph, pr.x, pr.y, 0.0f, ix, iy, iz);
      const DevBeam b = a.beams[beam];
      const DevTally& ta = a.tally;
      const uint32_t la = b.a_line + batch_of(h, ta.ka, ta.ma, b.a_off);
      tally_add(tally_word(ta, la, ta.ka, v), (unsigned long long)pr.e);
      mark_line<kMark>(ta, (v / kTallyBlock) * ta.ka + la);
      if (ta.kb) tally_add(tally_word(ta, batch_of(h, ta.kb, ta.mb, b.b_off), ta.kb, v), (unsigned long long)pr.e);
    }
    const WaveSeg::Slots sl = seg.append(keep, false);
    if (keep) put(seg.at(sl.s0), pr.x, pr.y, 0.0f, 0.0f, 0.0f, 1.0f, pr.e, h, 0u, 0u, 4u, beam);
  }
  ein = wave_sum(ein);
  esc = wave_sum(esc);
  if (lane_id() == 0) {
    if (ein) ctr_add(a.ctr, C_E_IN, ein);
    if (esc) ctr_add(a.ctr, C_E_ESC, esc);
  }
  return want;
}

// The history pool: one launch runs a whole job (Sec. II.C.3's pool, with the
// queues made private).  Every workgroup stages both table blocks once; every
// wavefront claims histories, keeps its photons and electrons on two stacks of
// its own and alternates between the electron and the photon loop of the pass
// kernels, always on the type that fills its lanes.  Nothing is shared but the
// claim cursors and the tally: no queue is copied or compacted, no pass waits
// for its slowest wavefront, no launch, plan or host read stands between the
// generations of a cascade, and the phases of different wavefronts, bound by
// instruction issue and by the tally's atomics in turn, overlap on a CU.
// Results are those of the passes bit for bit: a particle's stream and the
// integer tallies do not depend on order.
//
// Measured against the passes (which take 3 to 8 rounds of two passes for the
// smaller jobs, each lasting as long as its longest visit): 2e3 electrons on a
// 33 x 29 x 17 grid 0.94 -> 0.43 ms, 1e6 electrons on 64^3 water 2.07 -> 1.52
// ms, 4e6 photons on the lung box 3.2 -> 2.2 ms, the water job of 5.25e6
// electrons and 6.5e7 photons 41.3 -> 33.5 ms, 4e7 photons on 128^3 slabs 24.1
// -> 19.7 ms, 256 beamlets with per-beamlet doses 131 -> 101 ms.  With the
// columns (see Column) and the waits at hard events (see electron_loop) these
// take 0.23, 1.05, 1.67, 25.1, 14.5 and 74 ms, in calls of their own.
//
// Registers are full: 127 vector registers of 128 (128 in the marking instance),
// with 36 (45) scalar ones kept in lanes of others.  So the stacks' size is a
// constant of the instance (kEntries): as an argument it cost the shorter jobs
// 1 to 2%.
//
// A wavefront whose stacks could overflow (a cascade far beyond what the host's
// rule lets in) sets p.full and ends the claims; the wavefronts then leave as their stacks
// run dry and the host runs the job as passes, which bound their own queues.
template <bool kMark, uint32_t kEntries>
__global__ void __launch_bounds__(1024) k_pool(PoolArgs p) {
  extern __shared__ float4 smem[];
  const PassArgs& a = p.a;
  const int nt = a.tab.n_mat * kNE;
  float4* te = smem;
  float* tg = reinterpret_cast<float*>(te + nt);
  float* majg = tg + nt * kPhRow;
  float* maje = majg + kNE;
  float* ms = maje + kNE;
  DevBeam* lbeams = reinterpret_cast<DevBeam*>(ms + kNms);
  stage_photon_tables(tg, a.tab);
  for (int i = threadIdx.x; i < nt; i += blockDim.x) te[i] = a.tab.el[i];
  for (int i = threadIdx.x; i < kNE; i += blockDim.x) {
    majg[i] = a.tab.maj_g[i];
    maje[i] = a.tab.maj_e[i];
  }
  for (int i = threadIdx.x; i < kNms; i += blockDim.x) ms[i] = a.tab.ms[i];
  if (a.n_beams <= kLdsBeams)
    for (int i = threadIdx.x; i < a.n_beams; i += blockDim.x) lbeams[i] = a.beams[i];
  uint32_t* cols = reinterpret_cast<uint32_t*>(lbeams + kLdsBeams) + (threadIdx.x >> 6) * kColWords;
  for (int i = lane_id(); i < kColWords; i += 64) cols[i] = 0u;
  __syncthreads();

  uint4* own = p.stacks + (size_t)wave_index() * (2u * kPoolStack * kStgGranules);
  WaveSeg se{own, kEntries, 0u}, sg{own + (size_t)kPoolStack * kStgGranules, kEntries, 0u};
  WaveTotals tot;
  Claims cl;
  uint32_t claim = 64u;   // size of the last claim, 0: no histories are left
  for (;;) {
    if (claim && se.used + sg.used < 64u) claim = pool_admit<kMark>(p, se, sg, cl);
    const uint32_t ne = se.used, ng = sg.used;
    if (ne + ng == 0u) {
      if (claim == 0u) break;
      continue;
    }
    const bool rich = claim >= 64u;
    ElectronStack<kMark> re{{se, sg, rich, p.tail_e}};
    PhotonStack<kMark> rg{{sg, se, rich, p.tail_g}};
    // room for an iteration before the loop's own check
    const bool can_e = ne > 0u && ne + 256u <= se.cap && sg.used + 192u <= sg.cap;
    const bool can_g = ng > 0u && !rg.short_of_room(64u);
    if (!can_e && !can_g) {
      if (lane_id() == 0) {
        atomicOr(p.full, 1ull);
        for (int t = 0; t < 2; ++t) atomicOr(p.cursor[t], kNoneLeft);
      }
      break;
    }
    if (can_e && (ne >= 64u || !can_g || ng < 64u)) {
      electron_loop(a, re, se, sg, te, maje, ms, lbeams, cols, tot);
    } else {
      photon_loop(a, rg, sg, se, tg, majg, lbeams, tot);
    }
  }
  add_totals(tot, a.ctr);
}

// ---------------------------------------------------------------- finalize
// Which voxel thread i of a finalize takes: its number u in tile order and v in
// grid order.  Threads run over the tally as it is laid out -- in tile order
// through the library's tallies (whole lines of every batch; the doses of 16
// threads are then written to runs of at least 16 bytes, which the tile's
// neighbours complete), in grid order through the C ABI's -- and v is nvox or
// more where there is no voxel.
struct FinVoxel { uint32_t u, v; };
__device__ __forceinline__ FinVoxel fin_voxel(const FinalizeArgs& a, uint32_t i) {
  if (a.blocked) {
    if (i >= a.tile.n) return FinVoxel{0u, a.nvox};
    uint32_t ix, iy, iz;
    untiled(a.tile, i, ix, iy, iz);
    const bool in = ix < (uint32_t)a.nx && iy < (uint32_t)a.ny && iz < (uint32_t)a.nz;
    return FinVoxel{i, in ? (iz * (uint32_t)a.ny + iy) * (uint32_t)a.nx + ix : a.nvox};
  }
  if (i >= a.nvox) return FinVoxel{0u, a.nvox};
  const uint32_t row = i / (uint32_t)a.nx, iz = row / (uint32_t)a.ny;
  return FinVoxel{tiled(a.tile, i - row * (uint32_t)a.nx, row - iz * (uint32_t)a.ny, iz), i};
}

// Dose per history and batch uncertainty in double precision (Sec. II.D):
// D = sum_k T_k / N converted to Gy; sigma^2 = sum_k n_k^2 (m_k - m)^2 /
// (N^2 (K-1)/K) with m_k = T_k / n_k the batch means, each term formed as
// (T_k - n_k m)^2 (the same quantity, without a division).  The forms below
// return the voxel's deposited energy for the integer ledger and its dose, and
// give the same bits for the same batches.
//
// Where a.clear is set they leave the tally they have read at zero, writing
// only the words that are not: the next job of the workspace then finds its
// tallies clear (the host asks for it where a job touches few words).
struct FinResult {
  unsigned long long e;
  double d;
};

// A voxel's batches in turn: f(k, total over the nsum tallies added, address of
// the first tally's).  kFinFlight loads are issued before the first is used: one
// at a time, a voxel's 1024 batches are 1024 trips to memory in a row (1782
// voxels with 5 beams of 1024 batches, whose finalizes are a few workgroups
// each: 6.7 ms for the call, 4.3 in one launch, and so 2.3).  Four in flight: with
// eight, 33 and 40 slice-major batches on 80^3 voxels take 8% longer.
//
// Several tallies are added with as many loads in flight in a grid of up to
// kFinFewBlocks workgroups (four on a CU), and one at a time in larger ones,
// whose wavefronts hide the latency and lose when they spread over more of the
// tallies at once.  Calls with 33 batches of 256 beams in ms, so and with four
// always: 40 x 50 x 60 voxels 11.2 and 6.3, 60^3 14.4 and 10.2, 80 x 60 x 70 (1313
// workgroups) 18.1 and 20.7, 80^3 23.5 and 38.1, 94 x 111 x 118 62 and 89.
constexpr uint32_t kFinFlight = 4;
constexpr uint32_t kFinFewBlocks = 1024;
template <class F>
__device__ __forceinline__ void for_batches(const FinalizeArgs& a, FinVoxel x, F&& f) {
  unsigned long long* p = a.tally + (a.blocked ? vox_off(x.u, a.K) : (size_t)x.v);
  const size_t step = a.blocked ? kTallyBlock : a.nvox;
  if (a.nsum == 1u) {
    uint32_t k = 0;
    for (; k + kFinFlight <= a.K; k += kFinFlight, p += kFinFlight * step) {
      unsigned long long t[kFinFlight];
#pragma unroll
      for (uint32_t i = 0; i < kFinFlight; ++i) t[i] = p[i * step];
#pragma unroll
      for (uint32_t i = 0; i < kFinFlight; ++i) f(k + i, t[i], p + i * step);
    }
    for (; k < a.K; ++k, p += step) f(k, *p, p);
    return;
  }
  const uint32_t together = gridDim.x <= kFinFewBlocks ? a.nsum : 0u;
  for (uint32_t k = 0; k < a.K; ++k, p += step) {
    unsigned long long s = 0;
    uint32_t j = 0;
    for (; j + kFinFlight <= together; j += kFinFlight) {
      unsigned long long t[kFinFlight];
#pragma unroll
      for (uint32_t i = 0; i < kFinFlight; ++i) t[i] = p[(size_t)(j + i) * a.sum_stride];
#pragma unroll
      for (uint32_t i = 0; i < kFinFlight; ++i) s += t[i];
    }
    for (; j < a.nsum; ++j) s += p[(size_t)j * a.sum_stride];
    f(k, s, p);
  }
}

// General form: any number of batches, nsum tallies added.
__device__ __forceinline__ FinResult finalize_general(const FinalizeArgs& a, FinVoxel x) {
  const uint32_t v = x.v;
  auto leave_at_zero = [&](unsigned long long* p) {
    for (uint32_t j = 0; j < a.nsum; ++j) p[(size_t)j * a.sum_stride] = 0ull;
  };
  unsigned long long s1 = 0;
  for_batches(a, x, [&](uint32_t, unsigned long long t, unsigned long long* p) {
    s1 += t;
    if (t && a.clear && !a.sigma) leave_at_zero(p);
  });
  const double rho = (double)__uint_as_float(a.vox[x.u].x);
  const double conv = rho > 0.0 ? a.conv / rho : 0.0;
  const double m = (double)s1 / a.n_total;
  if (a.dose) a.dose[v] = m * conv;
  if (a.sigma) {
    double acc = 0.0;
    for_batches(a, x, [&](uint32_t k, unsigned long long t, unsigned long long* p) {
      const double nk = a.nk[k];
      if (!(nk > 0.0)) return;   // a batch without histories adds nothing
      const double d = (double)t - nk * m;
      acc += d * d;
      if (t && a.clear) leave_at_zero(p);
    });
    const double var = a.K > 1 ? acc / (a.n_total * a.n_total * (double)(a.K - 1) / (double)a.K) : 0.0;
    a.sigma[v] = sqrt(var) * conv;
  }
  return FinResult{s1, m * conv};
}

// D and sigma of a voxel whose at most KR batches are in registers (zero past
// K), with the general form's operations in the same order.  nk: KR batch
// sizes, zero past K; sigma's sum has no branch: a batch without histories adds
// +0.0 to a sum of non-negative terms, which leaves it as it was.
template <uint32_t KR>
__device__ __forceinline__ FinResult finalize_batches(const FinalizeArgs& a, uint32_t v, float density,
                                                      const unsigned long long (&t)[KR], const double* nk) {
  const double rho = (double)density;
  unsigned long long s1 = 0;
#pragma unroll
  for (uint32_t k = 0; k < KR; ++k) s1 += t[k];
  const double conv = rho > 0.0 ? a.conv / rho : 0.0;
  const double m = (double)s1 / a.n_total;
  double sig = 0.0;
  if (a.sigma) {
    double acc = 0.0;
#pragma unroll
    for (uint32_t k = 0; k < KR; ++k) {
      const double d = (double)t[k] - nk[k] * m;
      const double term = d * d;
      acc += nk[k] > 0.0 ? term : 0.0;
    }
    const double var = a.K > 1 ? acc / (a.n_total * a.n_total * (double)(a.K - 1) / (double)a.K) : 0.0;
    sig = sqrt(var) * conv;
  }
  if (a.dose) a.dose[v] = m * conv;
  if (a.sigma) a.sigma[v] = sig;
  return FinResult{s1, m * conv};
}

// The marked lines of voxel u's tile as a mask of batches (K <= 32), their
// marks cleared; all ones without marks.  After 1e6 photons on 256^3 voxels a
// fifth of the lines are marked: the finalize takes 0.64 ms instead of 1.35.  All lanes of the wavefront call this:
// the 16 of a tile read its marks.
__device__ __forceinline__ uint32_t marked_lines(uint8_t* mark, uint32_t K, uint32_t u, bool valid) {
  if (!mark) return ~0u;
  const uint32_t i = u % kTallyBlock;
  uint8_t* p = mark + (size_t)(u / kTallyBlock) * K + i;
  const bool lo = valid && i < K && p[0], hi = valid && i + 16u < K && p[16];
  if (lo) p[0] = 0;
  if (hi) p[16] = 0;
  const uint32_t tile = lane_id() & 48u;
  return ((uint32_t)(lanes_with(lo) >> tile) & 0xffffu) | (uint32_t)(lanes_with(hi) >> tile) << 16;
}

// The batches of one tally (at most KR of them) from p on: a lane issues every
// load before it uses any.  kTiles: the library's layout, where the batches
// are a line apart and one address with constant offsets reaches all of them
// (and where they may be cleared); else slices of `slice` words.
// lines: those of the batches that may not be zero (all ones where none are
// known to be).
template <uint32_t KR, bool kTiles>
__device__ __forceinline__ void load_batches(unsigned long long (&t)[KR], unsigned long long* p, size_t slice, uint32_t K,
                                             uint32_t lines, bool clear) {
  if constexpr (kTiles) {
    if (__builtin_amdgcn_ballot_w64(lines != ~0u) == 0ull) {
#pragma unroll
      for (uint32_t k = 0; k < KR; ++k) {
        t[k] = 0ull;
        if (k < K) t[k] = p[k * kTallyBlock];
      }
    } else {
#pragma unroll
      for (uint32_t k = 0; k < KR; ++k) {
        t[k] = 0ull;
        if (lines >> k & 1u) t[k] = p[k * kTallyBlock];
      }
    }
    if (clear) {
#pragma unroll
      for (uint32_t k = 0; k < KR; ++k)
        if (t[k]) p[k * kTallyBlock] = 0ull;
    }
  } else {
#pragma unroll
    for (uint32_t k = 0; k < KR; ++k) {
      t[k] = 0ull;
      if (k < K) t[k] = *p;
      p += slice;
    }
  }
}

constexpr uint32_t kFinRegK = 32;
// The batch sizes of a finalize in LDS, zero past K.
__device__ __forceinline__ void stage_nk(double* lds, const FinalizeArgs& a) {
  if (threadIdx.x < kFinRegK) lds[threadIdx.x] = threadIdx.x < a.K ? a.nk[threadIdx.x] : 0.0;
}

// The workgroup's deposited energy to the ledger, and its largest dose to one
// of the kRelBlocks slots that the s reduction starts from (doses are not
// negative, so they order like their bits).  One atomic of each per workgroup.
__device__ __forceinline__ void finalize_totals(const FinalizeArgs& a, unsigned long long e, double d) {
  __shared__ unsigned long long se[4];
  __shared__ double sd[4];
  if (!a.ctr && !a.rel) return;
  e = wave_sum(e);
  for (int off = 32; off > 0; off >>= 1) d = fmax(d, __shfl_xor(d, off));
  if (lane_id() == 0) {
    se[threadIdx.x >> 6] = e;
    sd[threadIdx.x >> 6] = d;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (uint32_t w = 1; w < (blockDim.x >> 6); ++w) {
      e += se[w];
      d = fmax(d, sd[w]);
    }
    const uint32_t slot = blockIdx.x & (kCtrSlots - 1);
    if (e && a.ctr) atomicAdd(&a.ctr[C_E_DEP * kCtrSlots + slot], e);
    if (a.rel && d > 0.0)
      atomicMax(reinterpret_cast<unsigned long long*>(a.rel) + kRelMax + slot, (unsigned long long)__double_as_longlong(d));
  }
}

// One finalize, a thread per voxel (workgroups that take several blocks of
// voxels in turn were 5 to 14% slower).  KR: the width of the register form, 0
// for the general form (more batches than 32, or several tallies added).  One
// instance per width, so that each has the registers of its own width (a lane
// of the one-batch form holds two loads, not thirty-two, and the occupancy that
// hides their latency).  Bound by memory: 32 batches on 256^3 voxels, 4.7 GB, in
// 0.90 ms; 128^3 slice-major, 0.59 GB, in 0.128 ms (a large copy runs at 5.15
// TB/s).
template <uint32_t KR, bool kTiles>
__global__ void __launch_bounds__(256) k_finalize(FinalizeArgs a) {
  __shared__ double nk[kFinRegK];
  if (KR > 0) {
    stage_nk(nk, a);
    __syncthreads();
  }
  FinResult r{0ull, 0.0};
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  const FinVoxel x = fin_voxel(a, i);
  uint32_t lines = ~0u;
  if constexpr (KR > 0 && kTiles) lines = marked_lines(a.mark, a.K, x.u, i < a.tile.n);
  if (x.v < a.nvox) {
    if constexpr (KR > 0) {
      unsigned long long t[KR];
      load_batches<KR, kTiles>(t, a.tally + (kTiles ? vox_off(x.u, a.K) : x.v), a.nvox, a.K, lines, a.clear);
      r = finalize_batches<KR>(a, x.v, __uint_as_float(a.vox[x.u].x), t, nk);
    } else {
      r = finalize_general(a, x);
    }
  }
  finalize_totals(a, r.e, r.d);
}

// The beams of a batched job with a K-batched tally each (K <= KR): one pass
// over the tallies gives every listed beam's dose and sigma and, from the
// batches summed over the beams in registers, the combined ones -- the same
// bits as a finalize each, and the job's own.  Read apart, 16 beams of 32
// batches on 101 x 96 x 83 voxels (3.3 GB) took 1.44 ms for the combined result
// and 0.66 ms for the beams'; together they take 0.74.
template <uint32_t KR>
__global__ void __launch_bounds__(256) k_finalize_beams(FinalizeArgs c, const FinalizeArgs* __restrict__ list) {
  __shared__ double nk[kFinRegK], nkc[kFinRegK];
  stage_nk(nkc, c);
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  const FinVoxel x = fin_voxel(c, i);
  const bool in = x.v < c.nvox;
  const float density = __uint_as_float(c.vox[x.u].x);
  unsigned long long sum[KR];
#pragma unroll
  for (uint32_t k = 0; k < KR; ++k) sum[k] = 0ull;
  for (uint32_t j = 0; j < c.nsum; ++j) {
    const FinalizeArgs a = list[j];
    __syncthreads();   // the batch sizes of the beam before are used
    stage_nk(nk, a);
    __syncthreads();
    const uint32_t lines = marked_lines(a.mark, a.K, x.u, i < c.tile.n);
    if (in) {
      unsigned long long t[KR];
      load_batches<KR, true>(t, a.tally + vox_off(x.u, a.K), 0u, a.K, lines, c.clear);
      finalize_batches<KR>(a, x.v, density, t, nk);
#pragma unroll
      for (uint32_t k = 0; k < KR; ++k) sum[k] += t[k];
    }
  }
  FinResult r{0ull, 0.0};
  if (in) r = finalize_batches<KR>(c, x.v, density, sum, nkc);
  finalize_totals(c, r.e, r.d);
}

// The general form for the beams of a job with more batches than the register
// forms hold, a row of the grid each: one launch (calls with 256 beams of 33
// batches on 25 x 43 x 25 voxels, and with 300 beams of 100 batches on 20^3: 3.9
// and 10.2 ms; with a launch each, of too few workgroups to fill the chip, 15.8
// and 53 where one launch took 9.2 and 29).
__global__ void __launch_bounds__(256) k_finalize_many(const FinalizeArgs* __restrict__ list) {
  const FinalizeArgs a = list[blockIdx.y];
  const FinVoxel x = fin_voxel(a, blockIdx.x * 256u + threadIdx.x);
  if (x.v < a.nvox) finalize_general(a, x);
}

// The one-batch tallies of many beams on one phantom: a thread works out its
// voxel once and takes kFinManyRows beams of it (a row of the grid).  Memory
// bounds it; the doses are not read again here, so they are stored past the
// caches.  256 beams on 6.4e6 voxels (13 GB read, 13 GB written and what the
// beams touched cleared): 16 rows 8.2 ms, 8 7.9, 4 7.8, 2 7.3, 1 8.2; with
// nontemporal stores 16 rows 7.8, 4 7.1, 2 6.7; loads so as well 9.0.
constexpr uint32_t kFinManyRows = 2;
__global__ void __launch_bounds__(256) k_finalize_slices(const FinalizeArgs* __restrict__ list, uint32_t n) {
  const uint32_t j0 = blockIdx.y * kFinManyRows, j1 = min(j0 + kFinManyRows, n);
  const FinalizeArgs a0 = list[j0];
  const FinVoxel x = fin_voxel(a0, blockIdx.x * 256u + threadIdx.x);
  if (x.v >= a0.nvox) return;
  const double rho = (double)__uint_as_float(a0.vox[x.u].x);
  const size_t off = vox_off(x.u, 1u);
  const double conv = rho > 0.0 ? a0.conv / rho : 0.0;
  for (uint32_t j = j0; j < j1; ++j) {
    const FinalizeArgs& a = list[j];
    unsigned long long* p = a.tally + off;
    const unsigned long long t = *p;
    if (a.clear && t) *p = 0ull;
    if (a.dose) __builtin_nontemporal_store((double)t / a.n_total * conv, a.dose + x.v);
    if (a.sigma) a.sigma[x.v] = 0.0;   // no uncertainty from one batch
  }
}

// Eq. 12's s from the largest dose (kRelBlocks slots left by the finalize):
// per-block sums of sigma/D and counts over D > 0.2 D_max, then their totals by
// the last block to finish; every sum in a fixed order.
__device__ __forceinline__ double block_reduce(double v, bool take_max) {
  __shared__ double r[256];
  r[threadIdx.x] = v;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) r[threadIdx.x] = take_max ? fmax(r[threadIdx.x], r[threadIdx.x + h])
                                                       : r[threadIdx.x] + r[threadIdx.x + h];
    __syncthreads();
  }
  const double out = r[0];
  __syncthreads();
  return out;
}

// A thread's voxels are kRelBlocks * 256 apart and added in order; eight of them
// are loaded before the first is used (a 256^3 grid takes 0.08 ms; one at a time
// it took 0.19, and a pass of its own for the maximum 0.10).
__global__ void __launch_bounds__(256) k_rel(const double* __restrict__ dose, const double* __restrict__ sigma,
                                             uint32_t nvox, double* rel, double* out) {
  __shared__ bool last;
  const double cut = 0.2 * block_reduce(rel[kRelMax + threadIdx.x], true);
  double s = 0.0, c = 0.0;
  constexpr uint32_t kStep = kRelBlocks * 256u;
  uint32_t v = blockIdx.x * 256u + threadIdx.x;
  auto add = [&](double d, double sg) {
    if (d > cut) {
      s += sg / d;
      c += 1.0;
    }
  };
  for (; nvox > 7u * kStep && v < nvox - 7u * kStep; v += 8u * kStep) {
    double d[8], g[8];
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) d[j] = dose[v + j * kStep];
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) g[j] = sigma[v + j * kStep];
#pragma unroll
    for (uint32_t j = 0; j < 8u; ++j) add(d[j], g[j]);
    if (v > 0xffffffffu - 8u * kStep) {
      v = nvox;
      break;
    }
  }
  for (; v < nvox; v += kStep) add(dose[v], sigma[v]);
  s = block_reduce(s, false);
  c = block_reduce(c, false);
  if (threadIdx.x == 0) {
    rel[kRelSum + blockIdx.x] = s;
    rel[kRelCount + blockIdx.x] = c;
    __threadfence();
    last = atomicAdd(reinterpret_cast<unsigned long long*>(rel) + kRelDone, 1ull) == gridDim.x - 1u;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  s = block_reduce(__hip_atomic_load(rel + kRelSum + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), false);
  c = block_reduce(__hip_atomic_load(rel + kRelCount + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), false);
  if (threadIdx.x == 0) {
    const double r = c > 0.0 ? s / c : __longlong_as_double(0x7ff8000000000000ll);
    rel[kRelS] = r;
    if (out) *out = r;
  }
}

// --------------------------------------------------- a job's start and end
// What the host gives a job and gets from it goes through pinned memory that
// these kernels read and write themselves: one launch each, in stream order.
// A copy call costs 15 to 30 us of host time and a dispatch of its own; a job
// made eight of them on its way in, two to four on its way out, and waited
// twice more for arguments in the host's memory.  A call with 2e3 electrons,
// whose transport takes 176 us, took 381 us and takes 258; 1e5 photons 372
// and 253; 24 served requests 27.1 and 24.1 ms.
__global__ void __launch_bounds__(256) k_begin(uint4* dst, const uint4* src, uint32_t n16, unsigned long long* ctr,
                                               uint32_t nctr) {
  const uint32_t t = blockIdx.x * 256u + threadIdx.x, step = gridDim.x * 256u;
  for (uint32_t i = t; i < n16; i += step) dst[i] = src[i];
  for (uint32_t i = t; i < nctr; i += step) ctr[i] = 0ull;
}

// Block k < C_COUNT sums counter k; the other blocks copy the results.
__global__ void __launch_bounds__(256) k_report(ReportArgs a) {
  if (blockIdx.x < (uint32_t)C_COUNT) {
    __shared__ unsigned long long part[4];
    const unsigned long long s = wave_sum(a.ctr[blockIdx.x * kCtrSlots + threadIdx.x]);
    if (lane_id() == 0u) part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0u) {
      a.out[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
      if (blockIdx.x == 0u) a.out[C_COUNT] = a.rel ? (unsigned long long)__double_as_longlong(a.rel[kRelS]) : 0ull;
    }
    return;
  }
  double* o = a.h_out;
  for (const double* p : {a.dose, a.sigma}) {
    if (!p) continue;
    for (uint32_t i = (blockIdx.x - C_COUNT) * 256u + threadIdx.x; i < a.nvox; i += (gridDim.x - C_COUNT) * 256u)
      o[i] = p[i];
    o += a.nvox;
  }
}

// ------------------------------------------------------------------ checks
__global__ void k_rng_words(uint32_t key0, uint32_t key1, uint32_t hist, uint32_t plo, uint32_t phi, uint32_t n0,
                            int count, uint32_t* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t n = n0 + (uint32_t)i;
  const Block b = philox(n >> 2, plo, phi, hist, key0, key1);
  const uint32_t j = n & 3u;
  out[i] = j == 0 ? b.w0 : (j == 1 ? b.w1 : (j == 2 ? b.w2 : b.w3));
}

__global__ void k_table_eval(DevTables t, int which, int mat, const float* e, int n, float* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  if (which == 7) {
    const float g1 = e[i];
    out[i] = screening_A(t, t.ms, g1);
    return;
  }
  const TPos p = tpos(t, e[i]);
  if (which <= 2) {
    const float4 c = lerp4(t.ph, mat * kNE, p);
    out[i] = which == 0 ? c.x : (which == 1 ? c.y : c.z);
  } else {
    const float4 c = lerp4(t.el, mat * kNE, p);
    out[i] = which == 3 ? c.x : (which == 4 ? c.y : (which == 5 ? c.z : c.w));
  }
}

// First real photon interaction of each history (checks the stream use, the
// majorant and the table lookups against the oracle history by history).
__global__ void __launch_bounds__(256) k_first_events(PassArgs a, DevSource src, uint32_t h0, uint32_t count,
                                                      float* xyz, uint32_t* nused) {
  extern __shared__ float4 smem[];
  float* tab = reinterpret_cast<float*>(smem);
  stage_photon_tables(tab, a.tab);
  float* majg = tab + a.tab.n_mat * kNE * kPhRow;
  for (int i = threadIdx.x; i < kNE; i += blockDim.x) majg[i] = a.tab.maj_g[i];
  __syncthreads();
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= count) return;
  const uint32_t h = h0 + i;
  const uint32_t key1 = a.beams[0].key1;
  const Primary pr = sample_primary(src, a.key0, key1, h);
  const float nan = __builtin_nanf("");
  xyz[3 * i] = nan; xyz[3 * i + 1] = nan; xyz[3 * i + 2] = nan;
  nused[i] = 0;
  if (!inside(a.ph, pr.x, pr.y, 0.0f) || pr.e < a.cut.pcut_lsb) return;
  Lane L;
  L.x = pr.x; L.y = pr.y; L.z = 0.0f; L.u = 0.0f; L.v = 0.0f; L.w = 1.0f; L.e = pr.e; L.beam = 0;
  L.s.k0 = a.key0; L.s.k1 = key1; L.s.hist = h; L.s.plo = 0; L.s.phi = 0; L.s.n = 4;
  L.la = L.lb = 0u;   // no deposits here
  uint32_t viol = 0;
  for (int guard = 0; guard < (1 << 20); ++guard) {
    uint32_t v0 = 0u;
    const int kind = photon_flight(L, a, tab, majg, v0, viol);
    if (kind == PH_ESCAPE) return;
    if (kind != PH_FICT) {
      xyz[3 * i] = L.x; xyz[3 * i + 1] = L.y; xyz[3 * i + 2] = L.z;
      nused[i] = L.s.n;
      return;
    }
  }
}

__global__ void k_fill_u64(unsigned long long* p, size_t n, unsigned long long v) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// -------------------------------------------------------------- planning
// Sizes of the next pass from the device-resident counts: at most max_items
// particles, and no more than the free space of both destination buffers
// admits under the worst-case per-visit output (the particles left over are
// carried to the next buffer, one slot each).
__global__ void k_plan_pass(PlanArgs a) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const uint32_t n = *a.n_work;
  const uint32_t no = *a.n_other;
  uint64_t m = n < a.max_items ? n : a.max_items;
  // own outputs (carry-over + per-visit budget) must fit the allocated
  // buffer; outputs to the other type only fill it up to its soft capacity,
  // which leaves every type room for a full pass of its own outputs
  if (a.bud_same > 1) {
    const uint64_t lim = n < a.cap ? (uint64_t)(a.cap - n) / (a.bud_same - 1) : 0u;
    if (m > lim) m = lim;
  }
  if (a.bud_other > 0) {
    const uint64_t lim = no < a.cap_other ? (uint64_t)(a.cap_other - no) / a.bud_other : 0u;
    if (m > lim) m = lim;
  }
  // most items a wavefront gets (whole chunks, dealt round-robin)
  const uint64_t chunks = (m + (1u << a.chunk_log2) - 1u) >> a.chunk_log2;
  uint32_t q = (uint32_t)(((chunks + a.waves - 1) / a.waves) << a.chunk_log2);
  if (q == 0u) q = 1u << a.chunk_log2;
  PassPlan P;
  P.n = n;
  P.m = (uint32_t)m;
  *a.n_work = 0u;                 // the work buffer is consumed by this pass
  *a.n_new = n - (uint32_t)m;     // carried-over particles go to the front of the new buffer
  P.per_wave = q;
  P.chunk_log2 = a.chunk_log2;
  P.seg_same = q * (a.bud_same + a.park_slots);
  P.seg_other = q * a.bud_other;
  P.admitting = (a.sched[0] < a.sched[2] || a.sched[1] < a.sched[3]) ? 1u : 0u;
  *a.plan = P;
}

// Sizes of a round (one lane): the electrons' share first, bounded like an
// electron pass (own outputs within the allocated capacity, photons within
// the soft one), then the photons queued at the round's start, bounded so
// that the electrons they create keep the electron queue within the soft
// capacity; the claim caps (an even share of chunks plus one) and the
// segments those caps need; the claim counters are cleared.
__global__ void k_plan_round(RoundPlanArgs a) {
  // every thread of the one workgroup clears claim counters; thread 0 plans
  for (uint32_t i = threadIdx.x; i < 2u * (uint32_t)kMaxClaimParts; i += blockDim.x) a.claim_ctr[i] = 0u;
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const uint32_t ne = *a.n_work[1], ng = *a.n_work[0];
  const uint64_t s = a.sec;
  uint64_t me = ne < a.max_items ? ne : a.max_items;
  if (s > 0) {
    const uint64_t l1 = ne < a.cap ? (uint64_t)(a.cap - ne) / s : 0u;
    const uint64_t l2 = ng < a.cap_soft ? (uint64_t)(a.cap_soft - ng) / s : 0u;
    if (me > l1) me = l1;
    if (me > l2) me = l2;
  }
  uint64_t mg = ng < a.max_items ? ng : a.max_items;
  if (s > 0) {
    const uint64_t held = (uint64_t)ne + me * s;   // most the electron queue holds after the electron phase
    const uint64_t l3 = held < a.cap_soft ? ((uint64_t)a.cap_soft - held) / s : 0u;
    if (mg > l3) mg = l3;
  }
  const uint32_t ch = 1u << a.chunk_log2;
  const uint32_t ms[2] = {(uint32_t)mg, (uint32_t)me};
  const uint32_t ns[2] = {ng, ne};
  uint32_t caps[2];
  for (int t = 0; t < 2; ++t) {
    const uint64_t chunks = ((uint64_t)ms[t] + ch - 1u) >> a.chunk_log2;
    caps[t] = (uint32_t)(((chunks + a.waves - 1u) / a.waves + 1u) << a.chunk_log2);
    // one partition per workgroup, of at least two chunks each
    uint64_t parts = chunks >> 1;
    const uint64_t most = a.blocks < (uint32_t)kMaxClaimParts ? a.blocks : (uint32_t)kMaxClaimParts;
    if (parts > most) parts = most;
    if (parts < 1u) parts = 1u;
    ClaimType c;
    c.cap = caps[t];
    c.m = ms[t];
    c.parts = (uint32_t)parts;
    a.claims[t] = c;
    *a.n_work[t] = 0u;
    *a.n_new[t] = ns[t] - ms[t];
  }
  const uint32_t admitting = (a.sched[0] < a.sched[2] || a.sched[1] < a.sched[3]) ? 1u : 0u;
  // electron outputs: survivors and secondaries of the electron phase, the
  // photon phase's electrons; photon outputs: bremsstrahlung of the electron
  // phase, survivors and the parked stack of the photon phase
  const uint64_t seg_e = (uint64_t)caps[1] * (s + 1u) + (uint64_t)caps[0] * s;
  const uint64_t seg_g = (uint64_t)caps[1] * s + 2ull * caps[0];
  for (int t = 0; t < 2; ++t) {
    PassPlan P;
    P.n = ns[t];
    P.m = ms[t];
    P.per_wave = caps[t];
    P.chunk_log2 = a.chunk_log2;
    P.seg_same = (uint32_t)(t == 1 ? seg_e : seg_g);
    P.seg_other = (uint32_t)(t == 1 ? seg_g : seg_e);
    P.admitting = admitting;
    a.plan[t] = P;
  }
}

// ------------------------------------------------------ energy regrouping
// Sort key: bucket 4 log2(e) + the two bits below the leading one, reversed
// so that the highest energies come first; zero-energy entries go last.
__device__ __forceinline__ uint32_t sort_key(uint32_t e) {
  if (e == 0u) return kSortBuckets - 1u;
  const uint32_t lg = 31u - (uint32_t)__clz(e);
  const uint32_t sub = lg >= 2u ? (e >> (lg - 2u)) & 3u : (e << (2u - lg)) & 3u;
  return (uint32_t)(kSortBuckets - 1) - min((lg << 2) | sub, (uint32_t)(kSortBuckets - 2));
}

// Bucket counts of all entries (grid-stride, one LDS histogram per workgroup).
__global__ void __launch_bounds__(256) k_sort_count(SortArgs a) {
  __shared__ uint32_t h[kSortBuckets];
  for (int b = threadIdx.x; b < kSortBuckets; b += blockDim.x) h[b] = 0u;
  __syncthreads();
  const uint32_t n = *a.n;
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
    atomicAdd(&h[sort_key(entry<kQGranules>(a.src, i)[QG_POS * kQBlock].w)], 1u);
  __syncthreads();
  for (int b = threadIdx.x; b < kSortBuckets; b += blockDim.x)
    if (h[b]) atomicAdd(a.hist + b, h[b]);
}

// Bucket starts (exclusive prefix sum in key order); the counts are cleared
// for the next sort.  One workgroup of kSortBuckets threads.
__global__ void __launch_bounds__(kSortBuckets) k_sort_offsets(SortArgs a) {
  __shared__ uint32_t c[kSortBuckets];
  const int b = threadIdx.x;
  c[b] = a.hist[b];
  __syncthreads();
  uint32_t start = 0u;
  for (int j = 0; j < b; ++j) start += c[j];
  a.cursor[b] = start;
  a.hist[b] = 0u;
}

// Every entry to its bucket: each workgroup counts a tile of entries in LDS,
// reserves room per bucket with one atomic each, and writes its entries
// there (the queue count is unchanged).
constexpr uint32_t kSortTile = 2048;
__global__ void __launch_bounds__(256) k_sort_scatter(SortArgs a) {
  __shared__ uint32_t h[kSortBuckets];
  __shared__ uint32_t base[kSortBuckets];
  const uint32_t n = *a.n;
  for (uint32_t t0 = blockIdx.x * kSortTile; t0 < n; t0 += gridDim.x * kSortTile) {
    const uint32_t t1 = min(t0 + kSortTile, n);
    for (int b = threadIdx.x; b < kSortBuckets; b += blockDim.x) h[b] = 0u;
    __syncthreads();
    for (uint32_t i = t0 + threadIdx.x; i < t1; i += blockDim.x) atomicAdd(&h[sort_key(entry<kQGranules>(a.src, i)[QG_POS * kQBlock].w)], 1u);
    __syncthreads();
    for (int b = threadIdx.x; b < kSortBuckets; b += blockDim.x) {
      base[b] = h[b] ? atomicAdd(a.cursor + b, h[b]) : 0u;
      h[b] = 0u;
    }
    __syncthreads();
    for (uint32_t i = t0 + threadIdx.x; i < t1; i += blockDim.x) {
      const uint32_t key = sort_key(entry<kQGranules>(a.src, i)[QG_POS * kQBlock].w);
      const uint32_t slot = base[key] + atomicAdd(&h[key], 1u);
      const uint4* from = entry<kQGranules>(a.src, i);
      uint4* to = entry<kQGranules>(a.dst, slot);
      for (int g = 0; g < kQGranules; ++g) to[g * kQBlock] = from[g * kQBlock];
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------- launchers
// Tables, majorant, (screening table,) beam table.
size_t photon_lds_bytes(int n_mat) {
  return ((size_t)n_mat * kNE * kPhRow + kNE) * sizeof(float) + kLdsBeams * sizeof(DevBeam);
}
// And the columns of every wavefront.
static size_t electron_lds(int n_mat, int block) {
  return (size_t)n_mat * kNE * sizeof(float4) + (kNE + kNms) * sizeof(float) + kLdsBeams * sizeof(DevBeam) +
         (size_t)(block / 64) * kColWords * sizeof(uint32_t);
}
size_t electron_lds_bytes(int n_mat, int block) { return electron_lds(n_mat, block); }
size_t round_lds_bytes(int n_mat, int block) {
  return electron_lds(n_mat, block) + ((size_t)n_mat * kNE * kPhRow + kNE) * sizeof(float);
}

// The pass kernels' dynamic-LDS limit is raised once, to what the largest
// table set needs (occupancy follows the size each launch asks for), so that
// launches -- also those recorded into a graph -- set no attributes.
static hipError_t lds_limits() {
  static const hipError_t e = [] {
    const int most = (int)kLdsBytes - 512;   // beside the pass kernels' few static words
    for (const void* k : {(const void*)k_photon_pass, (const void*)k_electron_pass, (const void*)k_round}) {
      const hipError_t r = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, most);
      if (r != hipSuccess) return r;
    }
    for (const void* k : {(const void*)k_pool<false, kPoolStack>, (const void*)k_pool<true, kPoolStack>,
                          (const void*)k_pool<false, kPoolStackMin>, (const void*)k_pool<true, kPoolStackMin>}) {
      const hipError_t r = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes);
      if (r != hipSuccess) return r;
    }
    return hipSuccess;
  }();
  return e;
}

hipError_t launch_sort(const SortArgs& a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_sort_count, dim3(grid), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_sort_offsets, dim3(1), dim3(kSortBuckets), 0, s, a);
  hipLaunchKernelGGL(k_sort_scatter, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_plan_pass(const PlanArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_plan_pass, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_admit_plan(const AdmitPlanArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_admit_plan, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_admit(const AdmitArgs& a, uint32_t max_count, hipStream_t s) {
  if (max_count == 0 || a.nb == 0) return hipSuccess;
  const uint32_t grid = (max_count + 255u) / 256u;
  hipLaunchKernelGGL(k_admit, dim3(grid), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_photon_pass(const PassArgs& a, int grid, int block, hipStream_t s) {
  const size_t lds = photon_lds_bytes(a.tab.n_mat);
  const hipError_t e = lds_limits();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_photon_pass, dim3(grid), dim3(block), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_plan_round(const RoundPlanArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_plan_round, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_round(const RoundArgs& a, int grid, int block, hipStream_t s) {
  if (a.e.tab.n_mat > kMaxRoundMat) return hipErrorInvalidValue;
  const size_t lds = round_lds_bytes(a.e.tab.n_mat, block);
  const hipError_t e = lds_limits();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_round, dim3(grid), dim3(block), lds, s, a);
  return hipGetLastError();
}

template <uint32_t kEntries>
static void pool_launch(const PoolArgs& p, int grid, int block, size_t lds, hipStream_t s) {
  if (p.a.tally.mark) hipLaunchKernelGGL((k_pool<true, kEntries>), dim3(grid), dim3(block), lds, s, p);
  else hipLaunchKernelGGL((k_pool<false, kEntries>), dim3(grid), dim3(block), lds, s, p);
}

hipError_t launch_pool(const PoolArgs& p, int grid, int block, bool least, hipStream_t s) {
  if (p.a.tab.n_mat > kMaxRoundMat) return hipErrorInvalidValue;
  const size_t lds = round_lds_bytes(p.a.tab.n_mat, block);
  const hipError_t e = lds_limits();
  if (e != hipSuccess) return e;
  if (least) pool_launch<kPoolStackMin>(p, grid, block, lds, s);
  else pool_launch<kPoolStack>(p, grid, block, lds, s);
  return hipGetLastError();
}

hipError_t launch_electron_pass(const PassArgs& a, int grid, int block, hipStream_t s) {
  const size_t lds = electron_lds_bytes(a.tab.n_mat, block);
  const hipError_t e = lds_limits();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_electron_pass, dim3(grid), dim3(block), lds, s, a);
  return hipGetLastError();
}

// Thread i moves word i of the batches' lines in turn (batch i / n, voxel i mod
// n in tile order): coalesced loads, stores in runs of a tile's row.
__global__ void __launch_bounds__(256) k_tally_to_slices(const unsigned long long* in, unsigned long long* out,
                                                         DevTile tile, int nx, int ny, int nz, uint32_t K) {
  const size_t n = (size_t)tile.n * K, nvox = (size_t)nx * ny * nz;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const uint32_t k = (uint32_t)(i / tile.n), u = (uint32_t)(i % tile.n);
    uint32_t ix, iy, iz;
    untiled(tile, u, ix, iy, iz);
    if (ix < (uint32_t)nx && iy < (uint32_t)ny && iz < (uint32_t)nz)
      out[k * nvox + ((size_t)iz * ny + iy) * nx + ix] = in[vox_off(u, K) + (size_t)k * kTallyBlock];
  }
}

hipError_t launch_tally_to_slices(const unsigned long long* blocked, unsigned long long* slices, const DevTile& tile,
                                  int nx, int ny, int nz, uint32_t K, hipStream_t s) {
  const size_t n = (size_t)tile.n * K;
  if (n == 0) return hipSuccess;
  const int grid = (int)std::min<size_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(k_tally_to_slices, dim3(grid), dim3(256), 0, s, blocked, slices, tile, nx, ny, nz, K);
  return hipGetLastError();
}

// The narrowest register form that holds K batches of one tally, else 0
// (the general form).
static uint32_t finalize_width(uint32_t K, uint32_t nsum) {
  if (nsum != 1u || K < 1u || K > kFinRegK) return 0u;
  return K == 1u ? 1u : K <= 4u ? 4u : K <= 8u ? 8u : K <= 16u ? 16u : kFinRegK;
}

static int finalize_grid(uint32_t n) { return (int)(((size_t)n + 255u) / 256u); }

template <uint32_t KR>
static void finalize_width_launch(const FinalizeArgs& a, int grid, hipStream_t s) {
  if (a.blocked) hipLaunchKernelGGL((k_finalize<KR, true>), dim3(grid), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((k_finalize<KR, false>), dim3(grid), dim3(256), 0, s, a);
}

hipError_t launch_finalize(const FinalizeArgs& a, hipStream_t s) {
  const int grid = finalize_grid(a.blocked ? a.tile.n : a.nvox);
  switch (finalize_width(a.K, a.nsum)) {
    case 1u: finalize_width_launch<1u>(a, grid, s); break;
    case 4u: finalize_width_launch<4u>(a, grid, s); break;
    case 8u: finalize_width_launch<8u>(a, grid, s); break;
    case 16u: finalize_width_launch<16u>(a, grid, s); break;
    case kFinRegK: finalize_width_launch<kFinRegK>(a, grid, s); break;
    default: finalize_width_launch<0u>(a, grid, s); break;
  }
  return hipGetLastError();
}

bool finalize_beams_fit(uint32_t K) { return finalize_width(K, 1u) != 0u; }

hipError_t launch_finalize_beams(const FinalizeArgs& c, const FinalizeArgs* d_list, hipStream_t s) {
  const int grid = finalize_grid(c.tile.n);
  switch (finalize_width(c.K, 1u)) {
    case 1u: hipLaunchKernelGGL(k_finalize_beams<1u>, dim3(grid), dim3(256), 0, s, c, d_list); break;
    case 4u: hipLaunchKernelGGL(k_finalize_beams<4u>, dim3(grid), dim3(256), 0, s, c, d_list); break;
    case 8u: hipLaunchKernelGGL(k_finalize_beams<8u>, dim3(grid), dim3(256), 0, s, c, d_list); break;
    case 16u: hipLaunchKernelGGL(k_finalize_beams<16u>, dim3(grid), dim3(256), 0, s, c, d_list); break;
    case kFinRegK: hipLaunchKernelGGL(k_finalize_beams<kFinRegK>, dim3(grid), dim3(256), 0, s, c, d_list); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_finalize_many(const FinalizeArgs* d_list, uint32_t n, const DevTile& tile, hipStream_t s) {
  constexpr uint32_t kMost = 65535u;   // rows of a grid
  for (uint32_t j0 = 0; j0 < n; j0 += kMost)
    hipLaunchKernelGGL(k_finalize_many, dim3((unsigned)finalize_grid(tile.n), std::min(n - j0, kMost)), dim3(256), 0, s,
                       d_list + j0);
  return hipGetLastError();
}

hipError_t launch_finalize_slices(const FinalizeArgs* d_list, uint32_t n, const DevTile& tile, hipStream_t s) {
  constexpr uint32_t kMost = 65535u * kFinManyRows;   // rows of a grid
  for (uint32_t j0 = 0; j0 < n; j0 += kMost) {
    const uint32_t m = std::min(n - j0, kMost);
    hipLaunchKernelGGL(k_finalize_slices, dim3((unsigned)(((size_t)tile.n + 255) / 256), (m + kFinManyRows - 1u) / kFinManyRows),
                       dim3(256), 0, s, d_list + j0, m);
  }
  return hipGetLastError();
}

hipError_t launch_rel_uncertainty(const double* dose, const double* sigma, uint32_t nvox, double* rel, double* out,
                                  hipStream_t s) {
  static_assert(kRelBlocks == 256 && kCtrSlots == 256, "k_rel reduces one block of 256 partials");
  hipLaunchKernelGGL(k_rel, dim3(kRelBlocks), dim3(256), 0, s, dose, sigma, nvox, rel, out);
  return hipGetLastError();
}

hipError_t launch_begin(void* dst, const void* src, size_t n16, unsigned long long* ctr, uint32_t nctr, hipStream_t s) {
  const size_t n = std::max<size_t>(n16, nctr);
  if (n16 > 0xffffffffull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_begin, dim3((unsigned)std::min<size_t>((n + 255) / 256, 256)), dim3(256), 0, s,
                     static_cast<uint4*>(dst), static_cast<const uint4*>(src), (uint32_t)n16, ctr, nctr);
  return hipGetLastError();
}

hipError_t launch_report(const ReportArgs& a, hipStream_t s) {
  static_assert(kCtrSlots == 256, "k_report sums one block of 256 slots");
  const uint32_t copy = a.dose || a.sigma ? std::min<uint32_t>((a.nvox + 255u) / 256u, 256u) : 0u;
  hipLaunchKernelGGL(k_report, dim3((unsigned)C_COUNT + copy), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_rng_words(uint32_t key0, uint32_t key1, uint32_t hist, uint32_t plo, uint32_t phi, uint32_t n0,
                            int count, uint32_t* out, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_rng_words, dim3((count + 255) / 256), dim3(256), 0, s, key0, key1, hist, plo, phi, n0, count,
                     out);
  return hipGetLastError();
}

hipError_t launch_table_eval(const DevTables& t, int which, int mat, const float* e, int n, float* out,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_table_eval, dim3((n + 255) / 256), dim3(256), 0, s, t, which, mat, e, n, out);
  return hipGetLastError();
}

hipError_t launch_first_events(const PassArgs& a, const DevSource& src, uint32_t h0, uint32_t count, float* xyz,
                               uint32_t* nused, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const size_t lds = photon_lds_bytes(a.tab.n_mat);
  const hipError_t e = hipFuncSetAttribute((const void*)k_first_events, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            (int)photon_lds_bytes(kMaxMat));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_first_events, dim3((count + 255) / 256), dim3(256), lds, s, a, src, h0, count, xyz, nused);
  return hipGetLastError();
}

// Atomic-rate microbenchmark: lane t adds 1 to 64 words of a + (0..mask),
// at hashed addresses (a 32-bit xorshift-multiply finaliser), or (hot > 0)
// to word t mod hot, through the same global atomic as the tallies.
constexpr int kAtomicPerLane = 64;
constexpr int kAtomicBlocks = 4096;
static_assert(kAtomicRateAdds == (uint64_t)kAtomicBlocks * 256u * kAtomicPerLane, "additions per launch");
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352dU;
  x ^= x >> 15;
  x *= 0x846ca68bU;
  x ^= x >> 16;
  return x;
}

__global__ void __launch_bounds__(256) k_atomic_rate(unsigned long long* a, uint32_t mask, uint32_t hot) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  for (int j = 0; j < kAtomicPerLane; ++j) {
    const uint32_t i = hot ? (t & (hot - 1u)) : (mix32(t * 977u + (uint32_t)j * 131071u) & mask);
    tally_add(a + i, 1ull);
  }
}

hipError_t launch_atomic_rate(unsigned long long* a, uint32_t mask, uint32_t hot, hipStream_t s) {
  hipLaunchKernelGGL(k_atomic_rate, dim3(kAtomicBlocks), dim3(256), 0, s, a, mask, hot);
  return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long* p, size_t n, unsigned long long v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

// ------------------------------------------------ allocation-free finalize
// The work memory of gmc_finalize_tally_noalloc lives here instead of in
// memory the library allocates.  Host code never uses the array's name as an
// address: it takes the device address hipGetSymbolAddress returns for the
// current device, once per device, and passes that to the kernels.
static __device__ __align__(256) double scratch[kScratchDoubles];

static std::mutex g_scratch_mu;
static double* g_scratch_addr[kScratchDevices] = {};

hipError_t scratch_resolve(int device) {
  if (device < 0 || device >= kScratchDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch_addr[device]) return hipSuccess;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  if (!p) return hipErrorInvalidSymbol;
  g_scratch_addr[device] = static_cast<double*>(p);
  return hipSuccess;
}

double* scratch_address(int device) {
  if (device < 0 || device >= kScratchDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  return g_scratch_addr[device];
}

// #{h in [h0, h0 + n) : h mod K = k}, from #{h < m : h mod K = k} = (m + K - 1 - k) / K.
// Also clears the work of the s reduction.
__global__ void k_batch_sizes(double* nk, double* rel, unsigned long long h0, unsigned long long n, uint32_t K) {
  const uint32_t k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k < (uint32_t)kRelWords) rel[k] = 0.0;
  if (k < K) nk[k] = (double)((h0 + n + K - 1 - k) / K - (h0 + K - 1 - k) / K);
}

hipError_t launch_batch_sizes(double* nk, double* rel, uint64_t h0, uint64_t n, uint32_t K, hipStream_t s) {
  const uint32_t t = std::max<uint32_t>(K, kRelWords);
  hipLaunchKernelGGL(k_batch_sizes, dim3((t + 255u) / 256u), dim3(256), 0, s, nk, rel, (unsigned long long)h0,
                     (unsigned long long)n, K);
  return hipGetLastError();
}

int max_resident_blocks(int kernel, int block, size_t lds) {
  int per_cu = 0;
  const void* fn = kernel == 0 ? (const void*)k_photon_pass
                   : kernel == 1 ? (const void*)k_electron_pass
                   : kernel == 2 ? (const void*)k_round : (const void*)k_pool<false, kPoolStack>;
  (void)lds_limits();
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, block, lds) != hipSuccess || per_cu <= 0) per_cu = 1;
  int dev = 0, cus = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (cus <= 0) cus = 256;
  return per_cu * cus;
}

}  // namespace gmc
