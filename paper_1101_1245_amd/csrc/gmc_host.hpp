// gmc_host.hpp -- host-side state of the engine: table and phantom objects,
// the per-run workspace (particle queues, counters, tallies, stream and
// events), the transport engine's interface, and the context behind the
// C ABI.  Shared by gmc_engine.cpp (engine, blocking forms, autotuner),
// gmc_server.cpp (served form) and gmc_runtime.cpp (ABI entry points).
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "gmc_internal.hpp"
#include "gmc_tables.hpp"
#include "gpumcd.h"

namespace gmc {

struct TablesObj {
  gmc_physics phys{};
  double kcut = 0, kc = 0;
  double margin = 1.001;         // majorant safety factor
  HostTables host;
  float4* d_ph = nullptr;
  float4* d_el = nullptr;
  float* d_ms = nullptr;
};

struct PhantomObj {
  int nx = 0, ny = 0, nz = 0;
  double dx = 0, dy = 0, dz = 0;
  uint2* d_vox = nullptr;
  std::vector<double> rho_max;   // per material index 0..255
  int max_mat = 0;
  DevTile tile{};
  size_t nvox() const { return (size_t)nx * ny * nz; }
  // voxels of a tally in the library's layout (padded to whole tiles)
  size_t tally_vox() const { return tile.n; }
};

struct MajObj {
  float* d_g = nullptr;
  float* d_e = nullptr;
};

struct QueueBuf {
  DevQueue q{};
  void* base = nullptr;
};

constexpr uint32_t kMinSoftCap = 1u << 23;
constexpr uint32_t kMaxSoftCap = 1u << 25;
constexpr uint32_t kMaxWaves = 1u << 15;
constexpr int kSortGrid = 2048;              // workgroups of the regrouping kernels
constexpr double kAutotuneBudgetS = 10.0;   // default wall-clock budget of one tuning
constexpr double kTuneTrials = 24.0;        // about how many candidates one tuning runs
constexpr uint64_t kTuneMinSample = 1ull << 25;   // 8 chunks of the largest candidate
// Of 64 busy lanes of an electron wavefront, those waiting at a hard event that
// start it for all of them: the water job took 27.1 ms at 8, 26.4 at 12, 26.1
// at 16, 26.0 at 20 and 24, 26.1 at 32; 1e6 electrons 1164, 1129, 1119, 1109,
// 1116 and 1137 us.
constexpr int kHardLanes = 20;
// Smallest share of a pass (particles per wavefront) whose tail is requeued.
constexpr uint32_t kTailMinItems = 256u;
// Busy lanes of a pool wavefront's electron / photon loop that are put back
// when its stack is empty and other work waits.
constexpr uint32_t kPoolTailE = 40u;
constexpr uint32_t kPoolTailG = 32u;
// Admission segments of a job with several beams of a type: at least this
// many histories each, at most kMaxAdmitSegments per type.
constexpr uint64_t kAdmitSegment = 4096u;
constexpr uint64_t kMaxAdmitSegments = 1u << 16;

// Device control block of a workspace: queue counts [type][buffer],
// admission cursor and histories per type, the last pass plans and
// admissions.  One copy of it is the host's view of a job's progress.
struct Control {
  uint32_t counts[4];
  uint32_t sched[4];            // cursor[2], total[2]
  PassPlan plan[2];
  AdmitPlan adm[2];
  ClaimType claim[2];           // the round kernel's work queue per type
  bool done() const {
    return sched[0] == sched[2] && sched[1] == sched[3] && counts[0] == 0 && counts[1] == 0 && counts[2] == 0 &&
           counts[3] == 0;
  }
};

// Everything one running job needs on the device, with the stream it runs
// on.  The context has one for the blocking forms; the server has one per
// slot.  Buffers only grow (released by ws_trim or ws_free).
struct Workspace {
  int device = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::string err;
  uint32_t cap = 0;              // allocated particles per queue buffer
  uint32_t cap_soft = 0;         // what admission and other-type outputs may fill
  QueueBuf qbuf[2][2];          // [type: 0 photon, 1 electron][2 buffers]
  int acc[2] = {0, 0};          // buffer of each type that accumulates
  QueueBuf stg[2];              // staging: [0] same type, [1] other type
  uint32_t stg_cap = 0;
  QueueBuf sorted;              // a work buffer regrouped by energy (when sorting)
  uint32_t sorted_cap = 0;
  uint32_t* d_sort = nullptr;   // [2][kSortBuckets]: bucket counts, bucket cursors
  Control* d_ctl = nullptr;
  Control* h_ctl = nullptr;     // pinned host copy
  unsigned long long* d_ctr = nullptr;   // [C_COUNT][kCtrSlots], then the kRelWords of d_srel
  unsigned long long* h_ctr = nullptr;   // pinned: the counters' sums and s (kCtrCopy words), written by launch_report
  unsigned long long* d_tally = nullptr;
  size_t tally_elems = 0;
  uint8_t* d_mark = nullptr;    // a byte per 16 words of the tally: lines a sparse job has added to
  size_t mark_cap = 0;
  bool mark_dirty = false, marking = false;   // not all zero; in use by the job
  size_t tally_dirty_to = 0;    // words that are zero once the job's finalizes have cleared its own
  size_t tally_clean = 0;       // its first words known to be zero between jobs (the finalizes leave them so)
  // A job's inputs (beams, sources, spectra, admission segments, batch sizes,
  // finalize arguments): put together in h_up and brought to d_up in one piece.
  char* h_up = nullptr;         // pinned up to kUpPinned, else ordinary memory
  char* d_up = nullptr;
  size_t up_cap = 0;
  bool up_busy = false;         // the device may still read them
  double* h_out = nullptr;      // pinned: small results on their way to host memory
  size_t out_cap = 0;
  uint4* d_pool = nullptr;      // the history pool's stacks
  size_t pool_waves = 0;        // wavefronts they are sized for
  bool least_stacks = false;    // its jobs use only kPoolStackMin entries of each
  std::atomic<uint64_t>* pool_launches = nullptr;   // counts the pool's launches (the context's)
  bool pool_timed = false;      // kev0/kev1 bracket a pool launch not yet added to t_pass
  uint32_t* d_claim = nullptr;  // [2][kMaxClaimParts] chunk counters of the round kernel's work queue
  double* d_nk = nullptr;
  double* d_srel = nullptr;     // work of the s reduction, s first, behind the counters
  bool want_s = false;          // the last job's combined result has an s
  double* h_nk = nullptr;       // pinned batch sizes for the finalize
  double* d_dose = nullptr;
  double* d_sigma = nullptr;
  size_t out_elems = 0;
  std::map<std::vector<int>, int> resident;    // (kernel, block, materials) -> resident workgroups
  hipEvent_t ev0 = nullptr, ev1 = nullptr;     // around a whole job
  hipEvent_t kev0 = nullptr, kev1 = nullptr;   // around a pass launch (plain form)
  hipEvent_t ev_ctl = nullptr;                 // after a control-block copy
  std::vector<hipEvent_t> gev;                 // pairs around the passes of a captured graph
  double t_pass[3] = {0.0, 0.0, 0.0};          // summed photon pass, electron pass, round kernel durations, s
  uint64_t n_pass[3] = {0, 0, 0};
};

int wfail(Workspace* w, int code, const std::string& msg);

#define WS_TRY(w, expr)                                                                  \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess)                                                                \
      return ::gmc::wfail(w, e_ == hipErrorOutOfMemory ? GMC_ENOMEM : GMC_EDEVICE,      \
                          std::string(#expr) + ": " + hipGetErrorString(e_));           \
  } while (0)

// Wait for the null stream.  A workspace's own stream is non-blocking and does
// not follow it, so every call that reads or writes a caller's device memory
// does this first: the null stream may still be producing the inputs, or using
// the memory that an allocator has handed out again for the results.
hipError_t wait_null_stream();
// stream null: the workspace creates (and owns) a non-blocking stream.
int ws_init(Workspace* w, int device, hipStream_t stream);
void ws_free(Workspace* w);
// Release the job-sized buffers (tallies, marks, outputs); keep queues, staging
// and the pool's stacks.
void ws_trim(Workspace* w);
// Release queues and staging; release the pool's stacks.
void ws_drop_queues(Workspace* w);
void ws_drop_pool(Workspace* w);
size_t ws_device_bytes(const Workspace& w);
// What a job needs of a workspace: the stacks of a history pool (pool) or the
// queues and staging of the passes, its tallies, and the marks of their lines.
struct JobBytes {
  bool pool = false;
  size_t form = 0, tally = 0, marks = 0;
  size_t total() const { return form + tally + marks; }
};
// Device memory a workspace holds once it has run such a job (buffers only grow).
size_t ws_device_bytes(const Workspace& w, const JobBytes& job);
// Bytes of the marks for the lines of `words` words of a tally.
inline size_t mark_bytes(size_t words) { return (words / kTallyBlock + 7u) / 8u * 8u; }
int ws_ensure_tally(Workspace* w, size_t elems);
// Enqueue what is needed for the first elems words of the tally to be zero;
// they count as dirty until ws_tally_cleared says that every word a job may
// have written was left at zero.
int ws_clear_tally(Workspace* w, size_t elems);
void ws_tally_cleared(Workspace* w);
// Clear marks for the lines of `words` words of the tally, null where there is no
// memory for them.
uint8_t* ws_marks(Workspace* w, size_t words);
// Whether a job's finalizes leave its tallies at zero, rather than the next job
// clearing them: where it touches few of their words.  A clearing store of the
// finalize is paid for each word touched, a clearing pass for every word: 1e6
// photons on 256^3 voxels 0.18 ms against 0.71, 16 beams of 6e5 histories in
// all on 101 x 96 x 83 voxels 0.05 against 0.56, 5.8e7 histories of 256 beams
// 2.0 against 2.6; 4e7 photons on 128^3 slabs, where most words are touched,
// 0.08 against 0.07.  A history makes about 20 additions.
inline bool clears_sparsely(uint64_t n_hist, size_t tally_elems) { return 20.0 * (double)n_hist < (double)tally_elems; }
// Whether a job's transport marks the lines it adds to and its finalize reads
// only those: the finalize then takes less and the transport, which stores a
// byte per addition, more.  15 MeV photons on 256^3 voxels and 32 batches, in
// us of the call: 3e5 histories (1790 words each) 1850 -> 1420, 1e6 (537)
// 2830 -> 2570, 2e6 (268) 4010 -> 4210; on 128^3 1e5 (671) 583 -> 506, 2.5e5
// (268) 800 -> 760, 5e5 (134) 855 -> 871.  15 MeV electrons on 256^3: 2000 words
// each 2320 -> 1870, 405 5010 -> 4970, 268 6540 -> 6780.  16 beams with a tally
// each on 101 x 96 x 83 gain at fewer words too, which the rule leaves: 405 words
// 2150 -> 1940 (electrons) and 1600 -> 1360 (photons), 134 4110 -> 4020 and 2200
// -> 2070.
inline bool marks_lines(uint64_t n_hist, size_t tally_elems) { return 400.0 * (double)n_hist < (double)tally_elems; }
int ws_ensure_out(Workspace* w, size_t elems);
// Room for `bytes` in h_up and d_up (an earlier upload has been read).
int ws_reserve_upload(Workspace* w, size_t bytes);
// Enqueue the upload of its first `bytes`, and the clearing of the counters.
int ws_upload(Workspace* w, size_t bytes);
constexpr size_t kUpPinned = 1u << 20;
// Results up to this many bytes reach host memory through h_out.
constexpr size_t kOutPinned = 1u << 20;

// Engine knobs (gmc_tuning with defaults filled in).
struct Tune {
  int events, secondaries, chunk, block, pass_items, wave_items, rounds, refill;
  int sort;            // 1: energy regrouping before every pass
  int tail_g, tail_e;  // tail requeue lanes of the photon / electron pass (0: off)
  int queue;           // soft queue capacity (0: from the chunk)
  int persistent;      // 1: one persistent round kernel per round
  int aggregate;       // of no effect (reported back as set)
  bool pool;           // no knob of the passes is set: the job may run as a history pool
};
Tune resolve_tuning(const gmc_tuning* t);
gmc_tuning default_tuning();

// Queue capacity (allocated and soft) and staging slots the engine uses for a tuning.
void queue_sizes(Workspace* w, const Tune& tu, int n_mat, uint32_t* cap, uint32_t* cap_soft, uint32_t* stg);
// Whether a tuning runs rounds as the persistent kernel for n_mat materials.
bool uses_round(const Tune& tu, int n_mat);

int check_source(std::string* err, const gmc_source* s);
// Highest and mean kinetic energy of a (checked) source's spectrum, MeV.
double source_emax(const gmc_source& s);
double source_emean(const gmc_source& s);
// Edges then the normalised CDF at them (C_0 = 0, C_n = 1) of a tabulated spectrum.
void tabulated_cdf(const gmc_source& s, std::vector<double>* out);
uint32_t mev_to_lsb(double e);
DevPhantom dev_phantom(const PhantomObj& p);
DevCuts dev_cuts(const TablesObj& t);
DevSource dev_source(const gmc_source& s);
DevTables dev_tables(const TablesObj& t, const MajObj& m);

// One transport job: its beams, their sources and tally targets.  Histories
// of each particle type are numbered consecutively over the beams of that
// type (start[t][j] is the first history of the j-th beam of type t).
struct Job {
  const PhantomObj* P = nullptr;
  const TablesObj* T = nullptr;
  MajObj maj;
  uint32_t key0 = 0;                  // stream key, low word (the seed's)
  DevTally tally{};
  std::vector<DevBeam> beams;
  std::vector<DevSource> sources;
  std::vector<double> tab;            // tabulated spectra: per such beam, edges then normalised CDF
  std::vector<size_t> tab_off;        // per beam: offset in tab (tabulated beams only)
  // admission segments per type: segment j covers job-wide indices
  // [start[j], start[j+1]), histories seg_h[j] ... of beam beam_of[j]
  std::vector<uint32_t> start[2], beam_of[2], seg_h[2];
  uint32_t total[2] = {0, 0};
  std::vector<double> nk;             // histories per batch of the combined result
  std::vector<FinalizeArgs> fin;      // finalizes of single beams (nk is set on upload)
  std::vector<double> fin_nk;         // their histories per batch, fin_k each
  uint32_t fin_k = 0;
};

// How a job tallies (the plain form and the served form use kCombined with
// one beam).
enum TallyMode {
  kCombined,       // one tally [K][nvox] batched over all histories: no per-beam doses
  kBeamBatched,    // a [K][nvox] tally per beam; the combined result is their sum
  kBeamPlusComb    // a [1][nvox] tally per beam plus a combined [K][nvox] one (two additions per deposit)
};

// Beams, sources and tally targets of a job in workspace w (tallies at
// w->d_tally, laid out per mode).
void build_job(Job* J, Workspace* w, const PhantomObj& P, const TablesObj& T, const MajObj& maj,
               const gmc_source* srcs, const uint64_t* n_hist, int n_beams, uint64_t seed, TallyMode mode);
size_t job_tally_elems(TallyMode mode, const PhantomObj& P, uint32_t K, size_t n_beams);

// Workgroup size of a pass kernel: the requested one as far as LDS has room for
// its wavefronts' columns, or (requested 0) the smallest of 256 / 512 / 640 /
// 1024 threads that keeps the most wavefronts resident (with many materials the
// LDS tables, one copy per workgroup, limit 256-thread workgroups to half the
// occupancy registers allow; beside the tables of eight materials there is room
// for ten wavefronts' columns: 1e6 electrons take 2.11 ms there and 1.85 with
// seven materials and 16 wavefronts, 2.54 and 2.48 before there were columns).
// The round kernel's is kRoundMaxBlock.
int pass_block(Workspace* w, int kernel, int requested, int n_mat);
// Wavefronts of a pass grid (resident workgroups x waves per workgroup, at
// most kMaxWaves).  The round kernel's are at most 8 on a CU, as many as one
// workgroup of kRoundMaxBlock threads: its wavefronts claim chunks from each
// other's workgroups, and with more of them, in more workgroups, they spend a
// round of few chunks on that.  With 16 on a CU (512 threads, one material)
// 1e6 photons in water took 3.66 ms and take 1.45, 1e6 electrons 3.7 and 1.8,
// 2e7 photons 22 and 13; 8 in workgroups of 256 take 2.3, 2.9 and 14.8.
uint32_t pass_waves(Workspace* w, int kernel, int block, int n_mat);

struct Engine {
  Workspace* w = nullptr;
  Tune tu{};
  bool round = false;             // rounds as one persistent kernel (tu.persistent and the tables fit)
  int round_block = 0;            // its workgroup size, grid, wavefronts
  uint32_t round_blocks = 0, round_waves = 0;
  int block[2] = {0, 0};          // workgroup size of each pass kernel
  PassArgs proto{};
  AdmitArgs adm[2]{};
  PoolArgs pool{};
  uint32_t total[2] = {0, 0};
  uint32_t waves[2] = {0, 0};     // wavefronts of each pass grid
  uint32_t blocks[2] = {0, 0};
  uint32_t bud_same[2] = {0, 0}, bud_other[2] = {0, 0};
  const double* nk = nullptr;             // the job's nk, fin_nk and fin in device memory
  const double* fin_nk = nullptr;
  const FinalizeArgs* fin = nullptr;
};

// Queues, staging, inputs and counters of a job (enqueued on w->stream).
// pool: for a history pool (its stacks, no queues).
int engine_setup(Workspace* w, Engine& E, const Job& J, const Tune& tu, bool pool);
// Whether a job runs as a history pool.  The pool is the better form of every
// job the passes' knobs are left alone for (measured at k_pool), as long as
// both types' tables fit in LDS and the cascades fit its stacks: a wavefront
// holds the delta rays of its 64 electrons, about 0.077 R / K_cut each over a
// range of R = E / 2 cm, so K_cut >= 0.0016 E keeps them to 25 each.
bool uses_pool(const Tune& tu, const TablesObj& T, const gmc_source* srcs, int n_beams);
// The grid of a pool launch over n histories (the engine's comment says why),
// and the bytes of its stacks.
struct PoolGrid {
  uint32_t blocks, waves_per_block;
  uint32_t waves() const { return blocks * waves_per_block; }
};
PoolGrid pool_grid(Workspace* w, int n_mat, uint64_t n);
inline size_t pool_bytes(size_t waves) { return waves * 2u * kPoolStack * kStgGranules * sizeof(uint4); }
// Enqueue a pool launch over histories [first, first + count) of each type.
int engine_launch_pool(Engine& E, const uint64_t first[2], const uint64_t count[2]);
// Plain form: run to the end, host reads after admission and electron pass.
int engine_run_plain(Engine& E, uint64_t* rounds);
// Capture 2 * tu.rounds rounds (with event pairs around the passes) on
// w->stream into an executable graph.
int engine_capture(Engine& E, hipGraphExec_t* exec, int* rounds_per_replay);
// Batched form: capture, then replay until done (blocking).
int engine_run_graph(Engine& E, uint64_t* rounds);
// Enqueue a copy of the control block to w->h_ctl and record w->ev_ctl.
int enqueue_control_copy(Workspace* w);
// After a replay's control copy completed: check it and add the pass times;
// *done tells whether the job finished (a job that cannot progress any more
// returns GMC_EOVERFLOW).
int after_replay(Engine& E, int rounds_per_replay, bool* done);

// Histories per batch for interleaved batches: n_k += #{h in [h0, h0 + n) : h mod K = k}.
void add_batch_sizes(std::vector<double>& nk, uint64_t h0, uint64_t n, uint32_t K);
// Gy per tally unit (2^-27 MeV) per unit density of a voxel of P.
double dose_per_lsb(const PhantomObj& P);
// Enqueue dose and sigma of one tally; nk is in device memory.
// `ledger`: the combined result of a job, with its deposited energy and s.
// `blocked`: the tally is in the library's layout (else slice-major, as the C
// ABI's raw tallies are); `clear`: it is left at zero.
int finalize(Workspace* w, const PhantomObj& P, unsigned long long* tally, uint32_t K, const double* nk, uint64_t n,
             double* d_dose, double* d_sigma, bool ledger, bool blocked, bool clear, uint8_t* mark);
// Words of h_ctr: the counters' sums and s.
constexpr size_t kCtrCopy = (size_t)C_COUNT + 1;
// kPoolFull: the job overfilled a history pool's stacks and must run as passes.
constexpr int kPoolFull = 1;
// h_ctr -> stats, ledger check.
int stats_from_counters(Workspace* w, gmc_run_stats* stats, uint64_t n_hist, uint64_t rounds, double t_total_s,
                        double t_device_s);

// Job class of the autotuner's cache.
std::vector<int> job_class(const PhantomObj& P, const TablesObj& T, const gmc_source* srcs, const uint64_t* n_hist,
                           int n_beams);

struct Server;

}  // namespace gmc

struct gmc_context {
  int device = 0;
  std::string err;
  std::mutex mu;   // guards the maps and the tuning cache (the server thread reads them)
  int32_t next_id = 1;
  std::map<int32_t, std::unique_ptr<gmc::TablesObj>> tables;
  std::map<int32_t, std::unique_ptr<gmc::PhantomObj>> phantoms;
  std::map<std::pair<int32_t, int32_t>, gmc::MajObj> majorants;
  std::map<std::vector<int>, gmc_tuning> tuned;   // autotuner choices per job class
  std::map<int32_t, int> refs;                     // server requests holding a tables / phantom id
  gmc::Workspace ws;                               // the blocking forms' workspace
  hipStream_t gstream = nullptr;                   // owned stream the batched form captures on
  hipEvent_t join = nullptr;
  gmc::Server* server = nullptr;                   // owned; see server_destroy
  std::atomic<bool> least_stacks{false};           // of the jobs from here on
  std::atomic<uint64_t> pool_launches{0};          // of this context and its server
};

namespace gmc {
int cfail(gmc_context* c, int code, const std::string& msg);
// Majorants of a (phantom, tables) pair, built and uploaded once (locks c->mu).
int get_majorants(gmc_context* c, int32_t pid, int32_t tid, const PhantomObj& p, const TablesObj& t, MajObj* out,
                  std::string* err);
// Blocking run of a job in the context's workspace (the plain and batched forms).
// tally_out (single-beam plain runs): the raw [K][nvox] batch tallies are
// copied there too (host or device per tally_kind); dose may then be NULL.
int run_job(gmc_context* c, int32_t phantom_id, int32_t tables_id, const gmc_source* srcs, const uint64_t* n_hist,
            int n_beams, uint64_t seed, double* const* dose_per_beam, double* const* sigma_per_beam, double* dose,
            double* sigma, int out_kind, const gmc_tuning* tuning, gmc_run_stats* stats, bool batched,
            uint64_t* tally_out = nullptr, int tally_kind = GMC_HOST);
// per_beam: tune the job as run with per-beam outputs (their tally layout),
// a job class of its own.
int autotune(gmc_context* c, int32_t phantom_id, int32_t tables_id, const gmc_source* srcs, const uint64_t* n_hist,
             int n_beams, double budget_s, gmc_tuning* out, gmc_autotune_report* rep, bool per_beam = false);
// Served form (gmc_server.cpp).
void server_destroy(gmc_context* c);
}  // namespace gmc
