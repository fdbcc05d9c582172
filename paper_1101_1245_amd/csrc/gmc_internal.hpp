// gmc_internal.hpp -- device-visible data layout shared by the host runtime and
// the gfx950 kernels of the transport engine.
//
// Memory layout in HBM (all linear, no textures):
//  * phantom: one uint2 per voxel {float bits of density, material index},
//    in tiles of 16 voxels, so a voxel costs one 8-byte gather (Sec. II.C.2 keeps
//    composition and density in two 3D textures);
//  * tables: FP32 nodes on a log-energy grid, one float4 per (material, node),
//    staged into LDS by each workgroup;
//  * particles: queues of 48-byte entries in 16-byte granules, two
//    buffers per particle type (one being consumed, one accumulating);
//  * tallies: uint64 fixed-point energy (2^-27 MeV) per (batch, voxel).
//
// Pass sizes live on the device: a one-lane planning kernel reads the queue
// counts and writes a PassPlan that the pass kernel reads, so
// a sequence of passes can be enqueued (or captured in a graph) without the
// host reading counts in between.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gmc {

constexpr int kNE = 1024;               // log-energy nodes on [kEmin, kEmax]
constexpr double kEmin = 1.0e-3;        // MeV
constexpr double kEmax = 32.0;          // MeV (the fixed-point energy range)
constexpr int kNms = 512;               // nodes of the multiple-scattering screening table
constexpr int kMaxMat = 8;
// Voxel order inside the library: voxels in tiles of 16 (kTallyBlock), 2 x 2 x
// 4 along x, y, z where the grid allows it, so that an electron on its way
// (forward peaked along z, the beams' direction) stays in a tile for a few
// voxels.  The phantom and the tallies share the order: the voxel at (x, y, z)
// is number 16 tile + (its place in the tile), tiles x fastest, the grid padded
// to whole tiles.  In a tally, each batch's sums of a tile fill one 128-byte
// line and the tile's K lines are adjacent -- the sum of batch k in voxel v at
// (v / 16) 16 K + 16 k + v mod 16.  Batches never share a line, so the additions
// of a narrow beam's histories to its few voxels do not contend for one, and a
// voxel's batches stay within a few kilobytes.  Half a line, 8 voxels of 2 x 1
// x 4, is the unit the chip's atomics are counted by (see flush_columns).
// The doses and the raw tallies of the C ABI are in grid order ([nz][ny][nx]).
constexpr uint32_t kTallyBlock = 16;
struct DevTile {
  int sx, sy, sz;       // tile of 2^sx x 2^sy x 2^sz voxels, sx + sy + sz = 4
  uint32_t nbx, nby;    // tiles along x and y
  uint32_t n;           // voxels, padded to whole tiles
};
// 2 x 2 x 4, unless another shape of 16 pads the grid to less than 0.85 of that
// (grids of one or a few voxels along an axis).
inline DevTile tile_of(int nx, int ny, int nz) {
  const int best_first[15][3] = {{1, 1, 2}, {1, 2, 1}, {2, 1, 1}, {0, 2, 2}, {2, 0, 2}, {2, 2, 0}, {0, 1, 3}, {1, 0, 3},
                                 {0, 0, 4}, {0, 3, 1}, {3, 0, 1}, {1, 3, 0}, {3, 1, 0}, {0, 4, 0}, {4, 0, 0}};
  DevTile r{};
  double size = 0.0;
  for (const int* s : best_first) {
    const uint64_t bx = ((uint64_t)nx + (1u << s[0]) - 1u) >> s[0], by = ((uint64_t)ny + (1u << s[1]) - 1u) >> s[1],
                   bz = ((uint64_t)nz + (1u << s[2]) - 1u) >> s[2];
    const double n = 16.0 * (double)bx * (double)by * (double)bz;
    if (size > 0.0 && n >= 0.85 * size) continue;
    size = n;
    r = DevTile{s[0], s[1], s[2], (uint32_t)bx, (uint32_t)by, (uint32_t)(bx * by * bz * kTallyBlock)};
  }
  return r;
}
constexpr int kMaxBatches = 1024;
constexpr double kLsbMeV = 1.0 / 134217728.0;   // 2^-27 MeV per energy unit

struct DevPhantom {
  const uint2* vox;     // in tile order
  DevTile tile;
  int nx, ny, nz;
  float dx, dy, dz;
  float idx, idy, idz;
  float lx, ly, lz;
  float skin;         // 1e-4 of the smallest voxel width
};

struct DevTables {
  const float4* ph;     // [n_mat][kNE] {mu_C, mu_C + mu_pe, mu_total, 0} per unit density, cm^2/g
  const float4* el;     // [n_mat][kNE] {L, Sigma_M, Sigma_B, 1/lambda_1} per unit density
  const float* ms;      // [kNms] ln A at evenly spaced logit(G1)
  const float* maj_g;   // [kNE] photon majorant per grid bin, cm^-1
  const float* maj_e;   // [kNE] electron hard-event majorant per grid bin, cm^-1
  int n_mat;
  float lg2_emin;       // log2(kEmin)
  float inv_h2;         // grid nodes per unit of log2 E
  float ms_y0;          // logit(G1) of the first screening node
  float ms_inv_dy;      // nodes per unit of logit(G1)
};

struct DevCuts {
  uint32_t ecut_lsb, pcut_lsb;   // transport cutoffs in energy units
  uint32_t kcut2_lsb, kc_lsb;    // Moller needs T > 2 K_cut; brems needs T > k_c
  uint32_t two_mc2_lsb;          // pair threshold and rest-energy sink
  float kcut, kc;                // MeV
  float esmax_gcm2;              // <= 0: none
  float emin;                    // lowest table energy, MeV
  int mode;                      // 0 full, 1 photon first collision, 2 electron CSDA straight-ahead
};

// Particle queue entries are made of 16-byte granules, kept apart in blocks
// of 64 entries: granule g of entry i is the uint4 at
// (i / 64) 64 G + 64 g + i mod 64, G granules per entry.  A wavefront that
// takes consecutive entries reads each granule as one contiguous kilobyte, a
// few lanes that take or leave entries touch one 16-byte word per granule,
// and one address with the constant offsets g KB reaches the whole entry.  A
// layout of one array per 32-bit word formed 12 to 16 addresses per entry, 3
// instructions each, in passes that are bound by instruction issue: with
// granules (and the 16-byte beam entries below) the 15 MeV water job of 5.25e6
// electrons and 6.5e7 photons went from 50.5 to 42.7 ms, 4e7 photons on the
// 128^3 slabs from 30.9 to 24.9 ms.  Granules: {x, y, z, E}, {u, v, w, beam} and {history,
// stream path (two words), stream word counter}; positions and directions are
// float bits, E is in 2^-27 MeV units.
enum QueueGranule { QG_POS = 0, QG_DIR, QG_STREAM, kQGranules };
// Staging entries carry a granule more for the interaction type of a photon
// parked at its absorption.
constexpr int QG_PARK = kQGranules;
constexpr int kStgGranules = kQGranules + 1;
constexpr int Q_FIELDS = 4 * kQGranules;       // 32-bit words per entry
constexpr int kStgFields = 4 * kStgGranules;
constexpr uint32_t kQBlock = 64;               // entries per block
struct DevQueue {
  uint4* base;
  uint32_t cap;
};

// A beam: its stream key (the high word; the low word is the job's seed) and
// up to two tally targets.  Target a is the beam's own tally (ka batches per
// voxel block, or 1 when only its dose is needed), starting at line a_line of
// the job's tally memory (16 words each, the blocked layout above); target b
// is a combined tally at line 0, batched over all beams' histories (kb batches;
// kb = 0: no such target).  History h of the beam adds to batch (off + h) mod
// K of a target, off < K (the host reduces it); interleaved batches keep every
// run of consecutive histories spread over all K batches, so lanes working on
// neighbouring histories rarely add to the same address.  16 bytes: one LDS
// read per particle taken.
struct DevBeam {
  uint32_t key1;                // Philox key, seed hi ^ beam id
  uint32_t a_line;
  uint32_t a_off, b_off;
};
// The tally targets of a job: the same batch counts for every beam.
struct DevTally {
  unsigned long long* base;
  uint32_t ka, kb;              // batches of targets a and b (kb = 0: no target b)
  uint32_t ma, mb;              // batch_magic of each
  uint8_t* mark;                // a byte per line of target a, set by additions to it (may be null)
};
// Multiplier of the device's h mod K: h - K floor(h m / 2^32) is below 2 K.
inline uint32_t batch_magic(uint32_t K) { return K <= 1u ? 0xffffffffu : (uint32_t)((1ull << 32) / K); }
// Beams whose table the pass kernels keep in LDS (beside the physics tables):
// a particle's refill then reads its beam's key and tally slices without a
// second dependent global load.  Jobs with more beams read it from memory.
constexpr int kLdsBeams = 256;

// A beam's source, on the device for the admission kernel.
struct DevSource {
  int particle, spectrum;
  uint32_t e_lsb;               // monoenergetic energy
  float e_lo, e_mode, e_hi;     // triangular spectrum
  float cx, cy, wx, wy;
  const double* tab;            // tabulated: bin edges [tab_n + 1], then the normalised CDF at them [tab_n + 1]
  uint32_t tab_n;
  uint32_t h0;                  // number of the beam's first history (its stream and batch)
};

// Run counters (energy ledger in 2^-27 MeV units, event counts).  Each counter
// is spread over kCtrSlots words, picked by wavefront, so that the per-wave
// additions at the end of every kernel do not all hit one address;
// launch_report sums the slots.  C_E_DEP is the deposited total summed by the finalize.
// C_POOL_FULL and C_POOL_NEXT (two rows) are the history pool's flag and
// claim cursors, in slot 0 of rows of their own.
enum CounterIndex {
  C_E_IN = 0, C_E_ESC, C_E_SINK, C_PH_EVENTS, C_FICT, C_VIOL, C_E_STEPS, C_HARD, C_SEC, C_OVERFLOW, C_E_DEP,
  C_PH_REAL, C_POOL_FULL, C_POOL_NEXT, C_POOL_NEXT1, C_COUNT
};
constexpr int kCtrSlots = 256;

// Sizes of one pass, written by k_plan_pass.  The work buffer holds n
// particles; this pass transports the first m, dealt to the wavefronts in
// chunks of 2^chunk_log2 (chunk c to wavefront c mod W), at most per_wave
// each; each wavefront has staging segments of seg_same / seg_other slots.
// Particles m..n-1 are carried over to the next buffer.
struct PassPlan {
  uint32_t n, m, per_wave, seg_same, seg_other, chunk_log2;
  uint32_t admitting;   // primaries remain to be admitted: more passes of both types follow
};

// The device work queue of the persistent round kernel, per particle type:
// the round's m items split into `parts` contiguous partitions, partition p
// holding items [m p / parts, m (p+1) / parts) and a chunk counter of its
// own, and the most items one wavefront may claim.  Workgroup b claims from
// partition b mod parts first, so a claim is normally an atomic that only
// its own workgroup's wavefronts share.
constexpr int kMaxClaimParts = 4096;
struct ClaimType {
  uint32_t cap;
  uint32_t m;
  uint32_t parts;
};

struct PlanArgs {
  uint32_t* n_work;             // count of the work buffer (read, then cleared)
  uint32_t* n_new;              // count of the type's new accumulating buffer: set to the carry-over
  const uint32_t* n_other;      // count of the other type's accumulating buffer
  PassPlan* plan;
  uint32_t cap;                 // allocated queue capacity (bounds this type's own outputs)
  uint32_t cap_other;           // soft capacity the outputs to the other type must respect
  uint32_t max_items;           // most particles per pass
  uint32_t waves;               // wavefronts in the pass grid
  uint32_t chunk_log2;          // items per chunk dealt to a wavefront: 2^chunk_log2 (>= 64)
  uint32_t bud_same, bud_other; // per-visit output budgets per particle
  uint32_t park_slots;          // same-type staging slots per particle for parked photons
  const uint32_t* sched;        // admission cursors [2] and totals [2]
};

// A pass kernel's work: each wave of the grid owns its chunks of the work
// queue (at most per_wave items), refills its lanes from them, and appends
// survivors and secondaries to its own segments of two staging queues
// (same type / other type) -- no atomics on shared counters while it
// transports.  When a workgroup is done, one atomic per destination reserves
// room for all of its waves' entries in the accumulating queues and each
// wave copies its segments there; particles the pass did not take (m..n-1)
// are copied to the front of the type's new queue.  Queue order then depends
// on which workgroups finish first; no result does (every particle carries its
// own stream and tallies are integer sums).
struct PassArgs {
  DevPhantom ph;
  DevTables tab;
  DevCuts cut;
  DevQueue work;           // items 0..m-1 of the pass
  DevQueue carry_src;      // items m..n-1, carried over (the work buffer, or the unsorted one)
  const PassPlan* plan;
  DevQueue stg_same;       // survivors and same-type secondaries
  DevQueue stg_other;      // other-type secondaries
  DevQueue dst_same;       // the type's new accumulating queue (carry-over in front)
  DevQueue dst_other;      // the other type's accumulating queue
  uint32_t* cnt_same;      // their counts
  uint32_t* cnt_other;
  const DevBeam* beams;
  int n_beams;
  uint32_t key0;             // Philox key, low word: the same for every beam of a job
  DevTally tally;
  unsigned long long* ctr;   // [C_COUNT][kCtrSlots]
  int max_events;
  int max_secondaries;
  int refill_lanes;          // idle lanes (1..64) that trigger a refill
  int hard_lanes;            // of 64 busy lanes, those at a hard event that sample it together (1..64)
  int tail_lanes;            // requeue the lanes' particles once the share is done and at most this many remain
  uint32_t tail_min;         // ... for shares of at least this many particles
};

// The persistent round kernel: one launch per round transports the
// electrons and then the photons of the round's work queues, every
// wavefront claiming chunks of items from the device work queue (ClaimType
// per type, with its counters) instead of a fixed share.  g and e are the
// photon and electron halves as pass arguments: each reads its own work
// queue and plan; electron outputs go to staging queue 0 (e.stg_same,
// g.stg_other) and photon outputs to staging queue 1.
struct RoundArgs {
  PassArgs g, e;
  const ClaimType* claims;      // [2] photon, electron
  uint32_t* claim_ctr;          // [2][kMaxClaimParts] chunk counters (cleared by the plan)
};

// Sizes of a round: both types' plans as k_plan_pass would make them in
// sequence (electrons first; the photons transported in the round are those
// queued at its start), the per-wavefront claim caps and segments.
struct RoundPlanArgs {
  uint32_t* n_work[2];          // counts of the work buffers (read, then cleared)
  uint32_t* n_new[2];           // counts of the new accumulating buffers: set to the carry-overs
  PassPlan* plan;               // [2]
  ClaimType* claims;            // [2]
  uint32_t* claim_ctr;          // [2][kMaxClaimParts]
  uint32_t cap, cap_soft;       // allocated and soft queue capacity
  uint32_t max_items;           // most particles of a type per round
  uint32_t waves;               // wavefronts of the round grid
  uint32_t blocks;              // workgroups of the round grid
  uint32_t chunk_log2;          // items per claimed chunk: 2^chunk_log2
  uint32_t sec;                 // secondaries per visit
  const uint32_t* sched;        // admission cursors [2] and totals [2]
};

// The history pool: one launch runs a job's histories to the end.  Wavefront
// w of the grid has two stacks of kPoolStack staging entries, electrons then
// photons, from entry 2 kPoolStack w of `stacks`; histories are claimed from
// the cursors.
constexpr uint32_t kPoolStack = 4096;
// Least entries of a stack: a claim on top of 63 entries, and the room each loop
// needs to start (see ElectronStack and PhotonStack).  Ordinary deep cascades
// overfill stacks of this size (tests of the hand-over to the passes).
constexpr uint32_t kPoolStackMin = 640;
constexpr uint32_t kPoolClaim = 256;    // most histories a wavefront claims at once
struct PoolArgs {
  PassArgs a;                   // queues and plan unused
  uint4* stacks;
  unsigned long long* cursor[2];   // histories claimed by this launch, per type
  unsigned long long* full;     // set when a stack could overflow: the job is run as passes
  uint64_t first[2], total[2];  // histories of this launch, per type: total from index first on
  const uint32_t* start[2];     // admission segments per type, as in AdmitArgs
  const uint32_t* beam_of[2];
  const uint32_t* seg_h[2];
  uint32_t nb[2];
  const DevSource* sources;
  uint32_t waves;               // wavefronts of the grid
  uint32_t tail_e, tail_g;      // busy lanes put back when other work waits
};

// Admission of primaries of one particle type.  The histories of all beams of
// that type are numbered consecutively (beam j of the type owns
// [start[j], start[j+1])); each admission takes the next `count` of them,
// stored from `base` on in the type's accumulating buffer.
struct AdmitPlan {
  uint32_t base, count, cursor;
};

struct AdmitPlanArgs {
  uint32_t* cursor;             // next history to admit, per type [2]
  const uint32_t* total;        // histories per type [2]
  uint32_t* count0;             // accumulating photon count
  uint32_t* count1;             // accumulating electron count
  AdmitPlan* out;               // [2]
  uint32_t cap, chunk;          // cap: the soft queue capacity
};

struct AdmitArgs {
  DevPhantom ph;
  DevCuts cut;
  DevQueue out;
  const AdmitPlan* plan;
  const uint32_t* start;        // [nb + 1] first job-wide index of each admission segment of this type
  const uint32_t* beam_of;      // [nb] beam of each segment
  const uint32_t* seg_h;        // [nb] index in its beam of each segment's first history
  uint32_t nb;                  // segments
  const DevBeam* beams;
  const DevSource* sources;     // indexed by beam
  uint32_t key0;                // as in PassArgs
  DevTally tally;
  unsigned long long* ctr;
};

// Energy regrouping of a work queue before its pass (the grouping of
// particles of similar energy that Sec. IV.B proposes against the divergence
// of polyenergetic beams): a counting sort on log-energy buckets, four per
// octave of the 2^-27 MeV units, highest energy first, so that the lanes of a
// chunk hold particles of similar energy and every wavefront takes its
// longest-lived particles first.  Order within a bucket is whatever the
// atomics give: no result depends on queue order.
constexpr int kSortBuckets = 128;
struct SortArgs {
  DevQueue src, dst;            // dst: room for n entries
  const uint32_t* n;            // entries to regroup: the first n of src (the pass's m)
  uint32_t* hist;               // [kSortBuckets] counts; zero before and after a sort
  uint32_t* cursor;             // [kSortBuckets] next free slot of each bucket in dst
};

struct FinalizeArgs {
  unsigned long long* tally;        // nsum tallies sum_stride apart (added), each in the library's layout or [K][nvox]
  uint32_t nsum;
  size_t sum_stride;                // elements between successive tallies
  const uint2* vox;                 // the phantom, in tile order
  DevTile tile;
  int nx, ny, nz;
  const double* nk;                 // histories per batch
  uint32_t nvox, K;
  double n_total, conv;             // conv = LSB * J/MeV / (V * 1e-3 kg/g)
  double* dose;                     // may be null for a beam of several (sigma only)
  double* sigma;                    // may be null
  unsigned long long* ctr;          // [C_COUNT][kCtrSlots], gets C_E_DEP (may be null)
  double* rel;                      // work of the s reduction, gets the largest dose (may be null)
  uint8_t* mark;                    // the tally's marked lines: the others are zero (null: any may not be; else cleared)
  uint32_t clear;                   // 1: the tallies read are left at zero
  uint32_t blocked;                 // 1: the library's layout; 0: slice-major [K][nvox]
};

// Launchers (gmc_kernels.hip).
// LDS of each kernel for n_mat materials and a workgroup of `block` threads.
size_t photon_lds_bytes(int n_mat);
size_t electron_lds_bytes(int n_mat, int block);
hipError_t launch_plan_pass(const PlanArgs& a, hipStream_t s);
hipError_t launch_photon_pass(const PassArgs& a, int grid, int block, hipStream_t s);
size_t round_lds_bytes(int n_mat, int block);
constexpr size_t kLdsBytes = 160u * 1024u;   // of a CU
constexpr int kMaxRoundMat = 4;        // both table blocks of more materials do not fit in LDS
hipError_t launch_plan_round(const RoundPlanArgs& a, hipStream_t s);
hipError_t launch_round(const RoundArgs& a, int grid, int block, hipStream_t s);
// least: only kPoolStackMin entries of each stack are used.
hipError_t launch_pool(const PoolArgs& p, int grid, int block, bool least, hipStream_t s);
hipError_t launch_electron_pass(const PassArgs& a, int grid, int block, hipStream_t s);
hipError_t launch_admit_plan(const AdmitPlanArgs& a, hipStream_t s);
hipError_t launch_admit(const AdmitArgs& a, uint32_t max_count, hipStream_t s);
hipError_t launch_finalize(const FinalizeArgs& a, hipStream_t s);
// Whether launch_finalize_beams takes K batches.
bool finalize_beams_fit(uint32_t K);
// The combined finalize c of nsum tallies and a finalize of each, whose
// arguments are at d_list in device memory (their tallies in the library's
// layout; a null dose or sigma is not wanted).  c.clear is every tally's.
hipError_t launch_finalize_beams(const FinalizeArgs& c, const FinalizeArgs* d_list, hipStream_t s);
// n finalizes of one phantom of any number of batches, arguments at d_list.
hipError_t launch_finalize_many(const FinalizeArgs* d_list, uint32_t n, const DevTile& tile, hipStream_t s);
// n finalizes of one-batch tallies of one phantom, arguments at d_list.
hipError_t launch_finalize_slices(const FinalizeArgs* d_list, uint32_t n, const DevTile& tile, hipStream_t s);
// A tally in the library's layout (K batches) rewritten slice-major, [K][nz][ny][nx].
hipError_t launch_tally_to_slices(const unsigned long long* blocked, unsigned long long* slices, const DevTile& tile,
                                  int nx, int ny, int nz, uint32_t K, hipStream_t s);
hipError_t launch_rng_words(uint32_t key0, uint32_t key1, uint32_t hist, uint32_t plo, uint32_t phi, uint32_t n0,
                            int count, uint32_t* out, hipStream_t s);
hipError_t launch_table_eval(const DevTables& t, int which, int mat, const float* e, int n, float* out,
                             hipStream_t s);
hipError_t launch_first_events(const PassArgs& a, const DevSource& src, uint32_t h0, uint32_t count, float* xyz,
                               uint32_t* nused, hipStream_t s);
hipError_t launch_sort(const SortArgs& a, int grid, hipStream_t s);
constexpr uint64_t kAtomicRateAdds = 4096ull * 256ull * 64ull;   // additions per microbenchmark launch
// Eq. 12's s of a dose and sigma array: mean sigma/D over voxels with
// D > 0.2 D_max, by fixed-order reductions (the same inputs give the same
// bits).  Work of kRelWords doubles, cleared before the finalize that leaves
// the largest dose in it: s, a count of finished blocks, kRelBlocks maxima,
// sums and counts.
constexpr int kRelBlocks = 256;
constexpr int kRelS = 0, kRelDone = 1, kRelMax = 2, kRelSum = kRelMax + kRelBlocks, kRelCount = kRelSum + kRelBlocks,
              kRelWords = kRelCount + kRelBlocks;
// s also goes to *out (pinned host memory) unless that is null.
hipError_t launch_rel_uncertainty(const double* dose, const double* sigma, uint32_t nvox, double* rel, double* out,
                                  hipStream_t s);
// A job's start: n16 16-byte units from pinned host memory, and nctr words cleared.
hipError_t launch_begin(void* dst, const void* src, size_t n16, unsigned long long* ctr, uint32_t nctr, hipStream_t s);
// A job's end, to pinned host memory: the sum of each counter's slots and s
// (from rel, unless that is null: 0), and nvox values of each of dose and
// sigma that is not null, one after the other.
struct ReportArgs {
  const unsigned long long* ctr;
  const double* rel;
  unsigned long long* out;
  const double* dose;
  const double* sigma;
  double* h_out;
  uint32_t nvox;
};
hipError_t launch_report(const ReportArgs& a, hipStream_t s);
hipError_t launch_atomic_rate(unsigned long long* a, uint32_t mask, uint32_t hot, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long* p, size_t n, unsigned long long v, hipStream_t s);
// kernel: 0 photon pass, 1 electron pass, 2 round kernel, 3 history pool
int max_resident_blocks(int kernel, int block, size_t lds);

// Largest workgroup of the round kernel: it holds the electron and the photon
// loop, whose registers together exceed what a 1024-thread workgroup leaves
// each lane (128), so it is bounded at 512 threads (up to 256 registers)
// rather than spill.
constexpr int kRoundMaxBlock = 512;

// Work memory of the allocation-free finalize: a file-scope device array of
// the kernels' source, one copy per device, never freed.  It holds the
// histories per batch (kMaxBatches doubles) and then the s reduction's work.
constexpr size_t kScratchDoubles = (size_t)kMaxBatches + kRelWords;
constexpr int kScratchDevices = 64;
// Resolve the array's address on `device` (which must be current): done once
// per device, at context creation.
hipError_t scratch_resolve(int device);
// Its address on `device` (nullptr before scratch_resolve succeeded there).
double* scratch_address(int device);
// nk[k] = histories of [h0, h0 + n) in batch k (h mod K), k < K; clears rel.
hipError_t launch_batch_sizes(double* nk, double* rel, uint64_t h0, uint64_t n, uint32_t K, hipStream_t s);

}  // namespace gmc
