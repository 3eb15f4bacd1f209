// Host side of the C boundary declared in include/dpllm.h: argument checks, the model object,
// load-time re-tiling, launch planning and kernel launches.  No kernel arithmetic lives here.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/dpllm.h"
#include "aux_kernels.hpp"
#include "chain_kernel.hpp"
#include "gemv_lane.hpp"
#include "layout.hpp"
#include "selector_kernels.hpp"

using namespace dpllm;

// Scratch of dpllm_estimate_noalloc: the partial dot products of one projection selector (rank up to
// kStaticMaxRank, every column chunking) or its sum x^2.  Every GPU the library runs on holds its own copy of the
// array until the process ends.  In host code the name is only a stand-in: the device address comes from
// hipGetSymbolAddress, once per device (static_scratch_ptr), and only that pointer is handed to kernels.
constexpr int kStaticMaxRank = 256;
constexpr size_t kStaticScratchSlots = (size_t)kSelMaxChunks * kStaticMaxRank;
static __device__ __align__(256) double scratch[kStaticScratchSlots];

namespace {

struct Pair {
  bool set = false;
  int l = 0, h = 0, kind = DPLLM_SEL_NONE, r = 0;
  const uint16_t* G = nullptr;
  float alpha = 0.f, beta = 0.f, T = 0.f;
};

struct TargetEntry {   // what a linear runs under one of the targets 1 .. DPLLM_MAX_TARGETS - 1
  bool set = false;
  int slot = 0;
  float T = 0.f;
};

struct Linear {
  bool loaded = false;
  LinearLayout L;
  char* arena = nullptr;
  Pair sel[DPLLM_MAX_PAIRS];
  int active = -1;                     // the pair of target 0
  TargetEntry tgt[DPLLM_MAX_TARGETS];  // [0] unused
  const void* sel_input = nullptr;     // decode step: the selector reads this vector instead of the linear's input
  int find_pair(int l, int h) const {
    for (int i = 0; i < DPLLM_MAX_PAIRS; ++i)
      if (sel[i].set && sel[i].l == l && sel[i].h == h) return i;
    return -1;
  }
  // what the launches are sized for: the properties of all pairs the linear holds, whichever is in use
  int max_rowgroups() const {
    int g = 0;
    for (const Pair& s : sel)
      if (s.set) g = std::max(g, sel_rowgroups_of(s.kind, s.r));
    return g;
  }
  int part_k() const {   // the bitwidth the work of a step launch is cut for: the larger one of the pair of target 0
    return active >= 0 ? sel[active].h : L.p;
  }
};

// A decode step is cut into phases: maximal runs of consecutive linears none of which reads or overwrites
// what an earlier linear of the run writes.  Inside a phase all selectors run in one launch and all GEMVs
// in another; phases run one after the other on the stream, so the result equals running the linears strictly
// in order.  Small GEMV launches take the decisions themselves (decides), those with little selector work run the
// selectors as well (fused).
struct Phase {
  int sel_first = 0, sel_count = 0;     // slice of the device selector job table
  int part_first = 0, part_count = 0;   // slice of the device selector part table
  int member_first = 0;                 // slice of the device table of group members
  int gemv_first = 0, gemv_count = 0;   // slice of the device GEMV job table (streaming kernel, one launch)
  int blocks = 0;                       // workgroups of that launch
  int block_first = 0;                  // slice of the device workgroup-to-job table
  bool estimators = true;               // under some target a job of the selector launch has an estimator (else the launch is skipped)
  bool may_estimate = true;             // ... under some pair its linear holds: what a captured step has to be able to follow
  int groups = 1;                       // column groups per wavefront of that launch (see gemv_narrow)
  bool may_decide = false;              // the GEMV launch is small enough to take the decisions of its linears
  bool decides = false;                 // a whole step takes them there
  bool fused = false;                   // ... and runs the selectors of this slice there too
  int task_first = 0, task_count = 0;   // slice of the device table of selector tasks
};
constexpr int kMaxGroups = 8;           // column groups per wavefront, at most
constexpr int kSelPolls = 64;           // polls of about a microsecond before a workgroup computes missing products itself
constexpr int kChainPatience = 1 << 21;   // polls of about a microsecond in a whole step before a wavefront of gemv_chain_kernel gives up
constexpr size_t kSelOneSlots = (size_t)kSelMaxChunks * kSelMaxRank;

struct StepPlan {
  bool valid = false;
  uint64_t version = 0;
  std::vector<const void*> xs;
  std::vector<void*> ys;
  int32_t* k_dev = nullptr;
  float* e_dev = nullptr;
  std::vector<Phase> phases;
  size_t slots = 0;      // partial dot products of all selectors; emptied at the start of a whole step if
  bool fused = false;    //   any of its phases runs selectors inside its GEMV launch
  bool idle = false;     // some phase has no estimator under any target, though its linears hold pairs with one
  bool captured = false; // a graph may hold launches of this plan
  bool chain = false;    // a whole step is one launch (gemv_chain_kernel)
  int chain_grid = 0;
  size_t chain_slots = 0, chain_mail = 0;   // 64-bit words
};

// The caller's workspace, carved once by dpllm_set_workspace.  Offsets in bytes, every region 256-byte aligned.
struct Workspace {
  char* base = nullptr;
  size_t bytes = 0;
  size_t est_ws = 0;                         // dpllm_estimate in two launches: kSelOneSlots fp64
  size_t est_sets = 0, est_slots_cap = 0;    // dpllm_estimate in one: [kEstRing] of a header, whose first dword is the captured call
                                             //   that does not rely on its slots any more, and uint64 [cap][2], empty between calls
  size_t est_set_words() const { return kEstHeader + 2 * est_slots_cap; }
  size_t target = 0;                         // the number of the active target
  size_t sel_params = 0;                     // SelParams [DPLLM_MAX_TARGETS][n]
  size_t sel_active = 0;                     // SelParams [n]: the row of the active target
  size_t sel_tasks = 0, sel_tasks_cap = 0;   // SelTask [cap]
  size_t sel_jobs = 0, sel_members = 0;      // SelJob [n], int32 [n]
  size_t sel_parts = 0, sel_parts_cap = 0;   // SelPart [cap]
  size_t sel_ws = 0, sel_ws_cap = 0;         // fp64 [cap]
  size_t gemv_jobs = 0;                      // GemvJob [n]
  size_t block_jobs = 0, block_jobs_cap = 0; // int32 [cap]
  size_t chain_state = 0;                    // uint32 [kChainLevelCounts + n]
  size_t chain_levels = 0, chain_jobs = 0;   // ChainLevel [n + 1], ChainJob [n]
  size_t chain_mail = 0, chain_mail_cap = 0; // 64-bit words [cap]
  size_t total = 0;
  template <class T>
  T* at(size_t off) const { return reinterpret_cast<T*>(base + off); }
};

}  // namespace

struct dpllm_model {
  std::vector<Linear> linears;
  std::string err;
  uint64_t version = 1;            // bumped by every call that changes what the launch plan depends on
  bool params_dirty = true;        // the device table of selector parameters is behind the host's
  StepPlan plan;
  Workspace ws;
  // host copies of what the plan puts into the workspace (kept so that the asynchronous copies have a source)
  std::vector<SelJob> h_sel_jobs;
  std::vector<SelPart> h_sel_parts;
  std::vector<int32_t> h_sel_members;
  std::vector<GemvJob> h_gemv_jobs;
  std::vector<int32_t> h_block_jobs;
  std::vector<ChainLevel> h_chain_levels;
  std::vector<ChainJob> h_chain_jobs;
  std::vector<SelParams> h_params;
  uint32_t est_turn = 0;           // the number of the last estimate; they take turns in the sets of slots,
  hipStream_t ws_stream = nullptr; //   which dpllm_set_workspace empties on this stream:
  hipEvent_t ws_event = nullptr;   //   done for every stream to see once the event has passed
  bool est_ready = false;
  int polls = kSelPolls;           // < 0: the selector tasks are left out of the launches (dpllm_debug_set_polls)
  int chain_mode = 0;              // 1: one launch wherever gemv_chain_kernel serves the step, -1: nowhere (dpllm_debug_set_one_launch)
  int chain_seats = 0;             // of the first level of such a launch, at most (0: all)
  int launches = 0;                // kernels of the last step
  int device = 0;
};

namespace {

int fail(dpllm_model* m, int code, const char* fmt, ...) {
  if (m) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    m->err = buf;
  }
  return code;
}

int hip_fail(dpllm_model* m, hipError_t e, const char* what) {
  return fail(m, DPLLM_EHIP, "%s: %s", what, hipGetErrorString(e));
}

#define HIP_TRY(m, call)                                 \
  do {                                                   \
    hipError_t e__ = (call);                             \
    if (e__ != hipSuccess) return hip_fail(m, e__, #call); \
  } while (0)

int check_shape(int out, int in, int p, int kmin) {
  if (out < 1 || in < 32 || in % 32 != 0) return DPLLM_ESHAPE;
  if (p < 1 || p > DPLLM_MAX_BITS || kmin < 1 || kmin > p) return DPLLM_ERANGE;
  return DPLLM_OK;
}

// Makes `slot` the linear's pair under target 0.  The work of a step is cut for the h of that pair, so the next step plans anew
// where it changes; but not while a graph may hold launches of the present plan: they serve every pair, and replayed under
// another one they have to find their own tables (a plan for another h has another number of workgroups).
void use_pair(dpllm_model* m, Linear* lin, int slot) {
  if (lin->active < 0 || (lin->sel[lin->active].h != lin->sel[slot].h && !(m->plan.valid && m->plan.captured))) m->version++;
  lin->active = slot;
}

Linear* get_linear(dpllm_model* m, int id, int* rc) {
  if (!m) { *rc = DPLLM_EINVAL; return nullptr; }
  if (id < 0 || id >= (int)m->linears.size()) { *rc = fail(m, DPLLM_EINVAL, "linear id %d out of range", id); return nullptr; }
  Linear* lin = &m->linears[id];
  if (!lin->loaded) { *rc = fail(m, DPLLM_ESTATE, "linear %d is not loaded", id); return nullptr; }
  return lin;
}

// ---- workspace ------------------------------------------------------------------------------------------------
// slices of a row of G, at most
int sel_slices(int in) { return (in + kSelTaskCols - 1) / kSelTaskCols; }

// slots of an estimate in one launch: 16 rows of G in chunks of 512 columns and more
size_t est_slots_of(const Linear& lin, int rowgroups) {
  return (size_t)std::min(rowgroups * kSelPartRows, kEstMaxRank) * std::min(kEstChunks, (lin.L.in + kSelChunkStep - 1) / kSelChunkStep);
}

// 64-bit words of a linear's mailbox (whole lines: no two linears share one)
size_t mail_words(const LinearLayout& L) { return align_up((size_t)L.rows_padded * 2, kAlign) / 8; }

// Sized for any launch plan over the linears as they stand (shapes, pairs): the caps are upper bounds.
Workspace carve_workspace(const dpllm_model* m) {
  Workspace w;
  const size_t n = m->linears.size();
  size_t parts = 0, slots = 0, blocks = 0, tasks = 0, est = 0, mail = 0;
  for (const Linear& lin : m->linears) {
    if (!lin.loaded) continue;
    if (lin.max_rowgroups() > 0) est = std::max(est, est_slots_of(lin, lin.max_rowgroups()));
    mail += mail_words(lin.L);
    const size_t rg = (size_t)std::max(1, lin.max_rowgroups());
    parts += rg * kSelMaxChunks + 1;
    slots += rg * kSelPartRows * std::max(kSelMaxChunks, kSelCopies * sel_slices(lin.L.in));
    tasks += rg * kSelPartRows * sel_slices(lin.L.in);
    blocks += (size_t)lin.L.nrq * kMaxGroups;
  }
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes, kAlign); return o; };
  w.est_ws = take(sizeof(double) * kSelOneSlots);
  w.est_slots_cap = est;
  w.est_sets = take(sizeof(uint64_t) * kEstRing * w.est_set_words());
  w.target = take(sizeof(int32_t));
  w.sel_params = take(sizeof(SelParams) * DPLLM_MAX_TARGETS * n);
  w.sel_active = take(sizeof(SelParams) * n);
  w.sel_tasks_cap = tasks;
  w.sel_tasks = take(sizeof(SelTask) * tasks);
  w.sel_jobs = take(sizeof(SelJob) * n);
  w.sel_members = take(sizeof(int32_t) * n);
  w.sel_parts_cap = parts;
  w.sel_parts = take(sizeof(SelPart) * parts);
  w.sel_ws_cap = slots;
  w.sel_ws = take(sizeof(double) * slots);
  w.gemv_jobs = take(sizeof(GemvJob) * n);
  w.block_jobs_cap = blocks;
  w.block_jobs = take(sizeof(int32_t) * blocks);
  w.chain_state = take(sizeof(uint32_t) * (kChainLevelCounts + n));
  w.chain_levels = take(sizeof(ChainLevel) * (n + 1));
  w.chain_jobs = take(sizeof(ChainJob) * n);
  w.chain_mail_cap = mail;
  w.chain_mail = take(sizeof(uint64_t) * mail);
  w.total = off;
  return w;
}

// ---- selector ---------------------------------------------------------------------------------------------
SelParams make_params(const Pair& s, float T) {
  SelParams P;
  P.G = s.G;
  P.T = T; P.alpha = s.alpha; P.beta = s.beta;
  P.r = s.r; P.l = s.l; P.h = s.h; P.kind = s.kind;
  return P;
}

// cols: columns of a chunk (a multiple of 512), more where the columns would be cut into more than `most` of them
SelJob make_sel_job(const Linear& lin, int linear, int rowgroups, const void* x, float* e_dev, int32_t* k_dev, int cols, int most = kSelMaxChunks) {
  SelJob j;
  j.x = (const uint16_t*)x;
  j.e_out = e_dev;
  j.k_out = k_dev;
  j.ws = nullptr;
  j.in = lin.L.in;
  j.linear = linear;
  j.nchunks = 1;
  j.chunk_cols = lin.L.in;
  if (rowgroups > 0) {
    const int least = ((lin.L.in + most - 1) / most + kSelChunkStep - 1) / kSelChunkStep * kSelChunkStep;
    j.chunk_cols = std::min(std::max(cols, least), (lin.L.in + kSelChunkStep - 1) / kSelChunkStep * kSelChunkStep);
    j.nchunks = (lin.L.in + j.chunk_cols - 1) / j.chunk_cols;
  }
  j.ws_rows = std::max(1, rowgroups) * kSelPartRows;
  j.row_each = 0;
  return j;
}

// ---- GEMV -------------------------------------------------------------------------------------------------
GemvJob make_gemv_job(const Linear& lin, int k, const int32_t* k_dev, const void* x, void* y) {
  GemvJob j;
  j.arena = lin.arena;
  j.x = (const uint16_t*)x;
  j.y = (uint16_t*)y;
  j.k_dev = k_dev;
  j.has_fin = 0;
  j.fin = SelFinish{};
  j.plane_stride_u4 = (uint32_t)(lin.L.plane_bytes / 16);
  for (int kk = 1; kk <= kKMax; ++kk)
    j.lut_at[kk - 1] = (kk >= lin.L.kmin && kk <= lin.L.p) ? lin.L.lut_at(kk) : 0u;
  j.k = k;
  j.kmin = lin.L.kmin; j.p = lin.L.p;
  j.out = lin.L.out; j.ncw = lin.L.ncw; j.nrq = lin.L.nrq; j.ncc = lin.L.ncc;
  j.nblocks = lin.L.nrq;
  j.block_start = 0;
  j.nsamples = 1;
  return j;
}

// Blocks of 64 rows one workgroup (eight wavefronts) streams.  A workgroup should run for the better part of a
// hundred microseconds (about 1 MiB of planes): shorter ones pay their start-up (job record, tables, first
// loads: a few microseconds of an otherwise idle slot) too often, longer ones leave the chip half empty at the
// end of the launch (measured on the 7B step: 0.25 MiB 496 us, 0.375 MiB 480, 0.75 MiB 471, 1 MiB 468, 2 MiB
// 477, 4 MiB 546); and a launch wants at least a few workgroups per compute unit.
constexpr long kLaneGroupBytes = 1048576;
// Where a whole step takes the decisions of a launch's linears and runs its selectors.  us per level at rank r with
// launches in front for parts and decisions / a part launch and the decision in the prologue of every workgroup /
// everything inside the GEMV launch:
//   7B q, k, v (192 workgroups)       r = 64: 15.8 / 15.1 / 13.0, 256: 17.0 / 16.0 / 15.3, 384: 18.2 / 16.7 / 17.7
//   7B down (256, 11008 columns)      r = 64: 15.5 / 16.0 / 12.2, 1024: 25.9 / 21.2 / 19.1
//   7B gate, up (344)                 r = 64: 18.5 / 18.1 / 17.1, 128: 19.0 / 18.5 / 16.7, 192: 19.2 / 18.4 / 18.7, 512: 21.3 / 19.5 / 22.4
//   70B gate, up (896, 8192 columns)  r = 64: 47.3 / 49.2 / 47.1, 512: 54.3 / 54.5 / 55.3
//   a 7B block at once (664)          r = 64: 40.5 / 41.6 / 42.2, 256: 45.8 / 45.9 / 52.9, 1024: 59.3 / 57.3 / 617
//   two of them (1328)                r = 64: 53.0 / 55.8 / 55.6
// The 256 workgroups that share the selectors inside work their rows off one after the other, the rest of the launch waits,
// and who has waited too long computes every product of its linear (the 617 us).  A level between others of a chain gains
// a little more from being one launch: chained 7B / 8B block with the lines at 4, 6, 8 rows each (up to 256 workgroups) and
// 1, 2, 4 slices of 4096 columns (up to 512), r = 256: 52.5 / 53.7, 51.3 / 53.1, 51.4 / 53.1; r = 512: 61.2 / 64.0, 60.4 /
// 62.6, 61.2 / 64.3.  Repeating the decision in every workgroup pays up to 512.  (One 70B block at once with every second
// linear on the linear regression is the exception seen: 110.5 us in front, 107.3 inside.)
constexpr int kDecideMaxBlocks = 1024, kPrologueMaxBlocks = 512;
bool runs_selectors(int blocks, long rows, long slices) {
  if (blocks <= kSelTaskGroups) return rows <= 6L * kSelTaskGroups;
  return slices <= (blocks <= kPrologueMaxBlocks ? 2L : 1L) * kSelTaskGroups;
}
int pick_blocks_per_group(const LinearLayout& L, int k, long total_blocks, long group_bytes = kLaneGroupBytes) {
  const long bytes_per_block = 64L * L.in * k / 8;
  long r = std::min<long>(16, std::max<long>(1, group_bytes / std::max<long>(1, bytes_per_block)));
  while (r > 1 && total_blocks / r < 1024) --r;
  return (int)r;
}

// Column groups per wavefront (rows per workgroup = 64 / groups) of a launch whose linears have `blocks64` blocks of 64
// rows in all (times the passes of a batch), the shortest row ncc column tiles: the most that leave at most one
// workgroup per compute unit.  The bitwidth is not looked at: it moves no line by much.  us per launch in a graph, one linear, k = 3 / 4 / 6 / 8,
// with one, two, four and eight groups:
//   4096 x 4096     6.2 / 7.2 / 11.2 / 12.8,   4.9 / 5.6 / 7.6 / 8.8,     4.6 / 4.9 / 6.3 / 7.4,     6.9 / 7.5 / 9.3 / 11.0
//   4096 x 11008    12.6 / 14.5 / 24.3 / 26.9, 9.2 / 10.5 / 15.2 / 16.5,  7.5 / 8.6 / 11.7 / 13.3,   9.7 / 11.2 / 14.4 / 16.9
//   8192 x 8192     11.1 / 12.4 / 19.6 / 22.2, 9.0 / 10.1 / 14.4 / 16.5,  9.4 / 10.3 / 14.6 / 16.6,  14.9 / 17.1 / 22.0 / 26.7
//   11008 x 4096    7.2 / 8.3 / 12.3 / 14.4,   7.5 / 8.6 / 12.8 / 15.1,   8.3 / 9.1 / 12.1 / 14.6,   17.5 / 19.2 / 23.7 / 28.8
//   16384 x 4096    8.5 / 10.0 / 14.2 / 17.4,  9.2 / 10.2 / 14.7 / 17.3,  10.6 / 11.9 / 15.9 / 19.5, 23.5 / 25.7 / 31.5 / 38.5
//   1024 x 8192     9.3 / 10.9 / 18.0 / 20.2,  6.6 / 7.6 / 10.9 / 12.1,   5.1 / 5.4 / 7.3 / 8.4,     4.2 / 4.7 / 5.7 / 6.8
// (129 to 172 blocks at k = 5, 6, 7 would gain 2 to 4 per cent with four.)  Eight groups only where every wavefront gets a step
// (1024 x 4096: 4.4 us with four, 4.3 with eight; a batch of four 5.2, 5.6).  A batch of four, one / two / four / eight groups: 8192 x 8192 k = 3 11.3 /
// 9.3 / 11.8 / 20.4, k = 6 20.0 / 15.0 / 18.2 / 27.3; 14336 x 4096 k = 3 8.2 / 10.6 / 14.8 / 25.8, k = 6 13.6 / 16.8 / 22.0 / 35.0; 4096 x 4096 k = 6 11.3 / 8.1 /
// 6.9 / 11.1; four / eight: 640 x 14336 k = 3 7.9 / 7.5, 192 x 14336 k = 6 12.2 / 9.9, 419 x 28672 k = 8 20.1 / 17.3 (workgroups that split the columns of
// 64 rows, with a hand-over through memory that calls would share, take 11.4 and 18.0 us for the last two: every
// workgroup reads all activations here).  A batch at k = 4 takes four at most (`most`; gemv_lone where the device says k): what a lane holds of a sample
// comes from two places there, and with 8 rows to a workgroup each wavefront fetches, sorts and exchanges that for eight tiles a step.  k = 4, B = 2,
// 4, four / eight: 500 x 8192 6.1 / 6.3, 6.3 / 7.9; 1000 x 11008 7.3 / 7.7, 7.5 / 9.8; 2048 x 14336 8.7 / 8.6, 9.0 / 11.1; 1024 x 28672 11.9 / 12.1, 12.6 /
// 16.2; at k = 2, 3 eight are 0 to 10 per cent ahead, at k >= 5 9 to 20.
int pick_groups(long blocks64, int ncc, int most = 8) {
  int g = 1;
  while (g < 4 && blocks64 * g * 2 <= 256) g *= 2;
  if (g == 4 && most == 8 && blocks64 * 8 <= 256 && ncc >= 8 * kLaneWaves) g = 8;
  return g;
}

void launch_lane(const LinearLayout& L, const char* arena, int groups, int nb, int nblocks, int passes, hipStream_t st, int k, const int32_t* k_dev,
                 const void* x, void* y, int nrhs) {
  const uint32_t bits = LaneBits{k, L.kmin, L.p, nrhs}.pack();
  const uint32_t lut = k_dev ? L.lut_at(L.kmin) - ((uint32_t)L.nrq << (L.kmin - 1)) : L.lut_at(k);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)(nblocks * passes)), dim3(kLaneThreads), 0, st, arena, (const uint16_t*)x, (uint16_t*)y, k_dev,
                       (uint32_t)(L.plane_bytes / 16), lut, bits, L.out, L.ncw, nblocks);
  };
  if (nb == 1) {
    switch (groups) {
      case 1: go(gemv_lane_kernel<1, 1>); break;
      case 2: go(gemv_lane_kernel<1, 2>); break;
      case 4: go(gemv_lane_kernel<1, 4>); break;
      default: go(gemv_lane_kernel<1, 8>); break;
    }
  } else if (nb == 4) {
    switch (groups) {
      case 1: go(gemv_lane_kernel<4, 1>); break;
      case 2: go(gemv_lane_kernel<4, 2>); break;
      case 4: go(gemv_lane_kernel<4, 4>); break;
      default: go(gemv_lane_kernel<4, 8>); break;
    }
  } else {
    switch (groups) {
      case 1: go(gemv_lane_kernel<8, 1>); break;
      case 2: go(gemv_lane_kernel<8, 2>); break;
      default: go(gemv_lane_kernel<8, 4>); break;
    }
  }
}

// fewer workgroups than compute units: more of them help with the selectors
void launch_step(int groups, int blocks, hipStream_t st, const GemvJob* jobs, const int32_t* block_jobs, const SelParams* active,
                 const SelTask* tasks, int ntasks, int polls) {
  if (polls < 0) ntasks = 0;
  const unsigned grid = (unsigned)std::max(blocks, std::min(ntasks, kSelTaskGroups));
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kLaneThreads), 0, st, tasks, jobs, block_jobs, active, ntasks, kSelTaskGroups, blocks, polls);
  };
  switch (groups) {
    case 1: go(gemv_step_kernel<1>); break;
    case 2: go(gemv_step_kernel<2>); break;
    case 4: go(gemv_step_kernel<4>); break;
    default: go(gemv_step_kernel<8>); break;
  }
}

void launch_chain(const dpllm_model* m, const Workspace& W, const StepPlan& P, hipStream_t st) {
  uint32_t* state = W.at<uint32_t>(W.chain_state);
  hipLaunchKernelGGL(chain_reset_kernel, dim3(512), dim3(256), 0, st, W.at<uint64_t>(W.sel_ws), P.chain_slots, W.at<uint64_t>(W.chain_mail), P.chain_mail, state,
                     m->h_chain_levels.size() - 1 + kChainLevelCounts);
  hipLaunchKernelGGL(gemv_chain_kernel, dim3((unsigned)P.chain_grid), dim3(kLaneThreads), 0, st, (const ChainLevel*)W.at<ChainLevel>(W.chain_levels),
                     (const ChainJob*)W.at<ChainJob>(W.chain_jobs), (const SelParams*)W.at<SelParams>(W.sel_active), (const SelTask*)W.at<SelTask>(W.sel_tasks),
                     state, (int)m->h_chain_levels.size() - 1, (int)m->h_chain_jobs.size(), kChainPatience, m->chain_seats);
}

// One linear, B right-hand sides.  Five to eight of them share one pass over the planes where two passes of four would be
// more workgroups than there are compute units; below that the second pass runs beside the first one.  us per call of
// B = 8, two passes / one: 14336 x 4096 k = 3 10.9 / 8.8, 11008 x 4096 k = 3 11.3 / 8.4, k = 5 18.7 / 12.5, k = 8 25.0 / 15.3.
// Up to 128 row blocks both passes fit, with twice the rows to a workgroup that one pass takes (64 / 1 and 64 / 2; up to 64 blocks
// 64 / 2 and 64 / 4): twice the lookups in a workgroup for the same sums.  One pass pays where lookups are what a step consists of
// (k >= 5) and where every wavefront has a step or several.  65 to 128 blocks: 8192 x 8192 k = 3 11.2 / 9.6, k = 4 12.3 / 11.0, k = 5 19.0 / 13.9,
// k = 8 22.4 / 17.5; 6000 x 4096 k = 3 7.2 / 6.6, k = 4 8.1 / 7.3; 5000 x 2048 k = 2 5.2 / 5.2, k = 4 5.9 / 5.6,
// k = 5 7.8 / 6.5, k = 8 9.9 / 7.9; 8192 x 1024 k = 3 4.3 / 5.0, k = 5 5.7 / 6.0, k = 8 7.4 / 7.1.  33 to 64: 4096 x 14336 k = 3 10.9 / 11.5, k = 5 17.4 /
// 16.0, k = 8 20.5 / 18.8; 4096 x 4096 k = 3 5.8 / 6.2, k = 4 6.2 / 7.6, k = 5 7.9 / 7.5; 4096 x 28672 k = 3 18.2 / 17.4, k = 4 19.4 / 23.3, k = 6 31.8 /
// 25.0; 3000 x 2048 k = 3 4.9 / 5.4, k = 5 6.1 / 6.2.  Fewer: 1000 x 4096 k = 5 6.2 / 7.1, 1500 x 14336 k = 3 8.6 / 11.1.
// Where the device says k the launch is the one for the widest bitwidth, and up to k = 4 its workgroups run the two passes (gemv_two_passes): B = 8,
// named / device / one pass, 4096 x 14336 k = 3 10.6 / 11.1 / 11.5, 4096 x 4096 k = 4 6.0 / 6.2 / 7.6, 8192 x 2048 k = 3 5.2 / 5.2 / 5.7.
int launch_gemv(dpllm_model* m, const Linear& lin, int k, const int32_t* k_dev, const void* x, void* y, int B, hipStream_t st) {
  const int blocks = lin.L.nrq;
  const bool deep = (k_dev ? lin.L.p : k) >= 5, wide = lin.L.ncc >= kLaneWideTiles;
  const bool one_pass = blocks > 128 || (blocks > 64 && (deep || wide)) || (blocks > 32 && deep && wide);
  const int nb = B == 1 ? 1 : B <= 4 || !one_pass ? 4 : 8;
  const int passes = (B + nb - 1) / nb;
  const int groups = nb == 8 ? (blocks > 128 ? 1 : blocks > 64 ? 2 : 4) : pick_groups((long)blocks * passes, lin.L.ncc, B > 1 && !k_dev && k == 4 ? 4 : 8);
  int nblocks = (lin.L.out + 64 / groups - 1) / (64 / groups);
  if (nb == 8 && k_dev) nblocks = (lin.L.out + 128 / groups - 1) / (128 / groups) * 2;   // (whole halves: gemv_two_passes)
  if (groups == 1) {
    const int rpb = pick_blocks_per_group(lin.L, k_dev ? lin.L.p : k, lin.L.nrq);
    nblocks = (lin.L.nrq + rpb - 1) / rpb;
  }
  launch_lane(lin.L, lin.arena, groups, nb, nblocks, passes, st, k, k_dev, x, y, B);
  HIP_TRY(m, hipGetLastError());
  return DPLLM_OK;
}

// ---- decode-step planning ------------------------------------------------------------------------------------
bool overlap(const void* a, size_t an, const void* b, size_t bn) {
  uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
  return a0 < b0 + bn && b0 < a0 + an;
}

// the table of selector parameters: row t = what every linear runs under target t (rows of targets that hold no
// entry of their own for a linear repeat target 0)
void fill_params(dpllm_model* m) {
  const size_t n = m->linears.size();
  m->h_params.assign((size_t)DPLLM_MAX_TARGETS * n, SelParams{});
  for (size_t i = 0; i < n; ++i) {
    const Linear& lin = m->linears[i];
    if (!lin.loaded || lin.active < 0) continue;
    const Pair& base = lin.sel[lin.active];
    for (int t = 0; t < DPLLM_MAX_TARGETS; ++t) {
      const TargetEntry& e = lin.tgt[t];
      const bool own = t > 0 && e.set && lin.sel[e.slot].set;
      m->h_params[(size_t)t * n + i] = own ? make_params(lin.sel[e.slot], e.T) : make_params(base, base.T);
    }
  }
}

void activate(const dpllm_model* m, int target, hipStream_t st) {
  const Workspace& W = m->ws;
  const int n = (int)m->linears.size();
  hipLaunchKernelGGL(selector_activate_kernel, dim3(std::min(n, 256)), dim3(256), 0, st, (const SelParams*)W.at<SelParams>(W.sel_params),
                     W.at<SelParams>(W.sel_active), n, (const GemvJob*)W.at<GemvJob>(W.gemv_jobs), W.at<SelTask>(W.sel_tasks),
                     W.at<int32_t>(W.target), target);
}

int upload_params(dpllm_model* m, hipStream_t st) {
  fill_params(m);
  // a selector launch none of whose linears has an estimator under any target has nothing to compute
  const size_t n = m->linears.size();
  m->plan.idle = false;
  for (Phase& ph : m->plan.phases) {
    ph.estimators = ph.may_estimate = false;
    for (int j = ph.sel_first; j < ph.sel_first + ph.sel_count && !ph.estimators; ++j) {
      const int linear = m->h_sel_jobs[j].linear;
      for (int t = 0; t < DPLLM_MAX_TARGETS && !ph.estimators; ++t)
        ph.estimators = m->h_params[(size_t)t * n + linear].kind != DPLLM_SEL_NONE;
      for (const Pair& s : m->linears[linear].sel) ph.may_estimate |= s.set && s.kind != DPLLM_SEL_NONE;
    }
    m->plan.idle |= ph.may_estimate && !ph.estimators;
  }
  HIP_TRY(m, hipMemcpyAsync(m->ws.at<SelParams>(m->ws.sel_params), m->h_params.data(), sizeof(SelParams) * m->h_params.size(),
                            hipMemcpyHostToDevice, st));
  activate(m, -1, st);
  HIP_TRY(m, hipGetLastError());
  m->params_dirty = false;
  return DPLLM_OK;
}

// Which chained steps are one launch.  The rule looks at shapes and at the ranks of all attached pairs, never at the pairs in use:
// a graph that holds a captured step follows those, and both kinds of step share the table of tasks.  us a step in a graph, a
// launch per level / one in all (8 blocks of a Transformer with d model and f hidden features, rank 64, at 3 and 4 bits; 7 and 8):
//   levels: 24 and more.  d = 4096, f = 11008 276 / 257 and 436 / 410 with 24 of them.
//   weights of a level, on average: 64 million.  4096, 11008 (51) 1420 / 1290 (32 blocks) and 587 / 555; 4096, 14336 with grouped
//     queries (55) 374 / 353 and 604 / 578; 3584, 18944 (64) 426 / 402 and 669 / 650; 4096, 16384 (67) 384 / 366 and 648 / 656; 4096,
//     22016 (84) 473 / 441 and 768 / 785; 8192, 8192 (117) 553 / 531 and 946 / 993.  Larger ones the streaming kernel decodes with
//     twice the wavefronts.
//   evenness: eight wavefronts share the columns in chunks of 512, so the one with the most may have up to 1.2 times its share (on
//     average over the rows).  3840, 10240 (1.10) 358 / 334 and 547 / 518; 3584, 18944 (1.13) above; 3072, 8192 (1.26) 295 / 292 and
//     418 / 447; 4608, 12288 (1.6) 441 / 463 and 690 / 781; 5120, 13824 (1.5) 454 / 530 and 746 / 976; 2560, 6912 (1.5) 287 / 275 and 394 /
//     393; 1024, 2816 202 / 203 and 266 / 280; 2048, 16384 302 / 323 and 453 / 516.
//   selectors: a task (row of G times 4096 columns) to a workgroup and level, on average.  4096, 11008 at rank 96 (0.84 of that) 375 / 366, 128
//     (1.1) 374 / 388, 256 399 / 439, 1024 612 / 786; 4096, 14336 at 96 (0.94) 385 / 384,
//     and 489 / 465 at 5 and 6 bits with selectors a level early; 4096, 4096 at 144 (0.98) 312 / 315, and 383 / 376 at 5 and 6 bits.
constexpr int kChainMinLevels = 24;
constexpr double kChainLevelWeights = 64e6, kChainUneven = 1.2;
bool chain_pays(const dpllm_model* m, int levels) {
  double weights = 0, even = 0, dealt = 0, tasks = 0;
  for (const Linear& lin : m->linears) {
    const LinearLayout& L = lin.L;
    const int chunks = (L.in + kChainChunk - 1) / kChainChunk;
    weights += (double)L.out * L.in;
    even += (double)L.out * L.ncc / kLaneWaves;
    dealt += (double)L.out * ((chunks + kLaneWaves - 1) / kLaneWaves) * (kChainChunk / 128);
    tasks += (double)lin.max_rowgroups() * kSelPartRows * sel_slices(L.in);
  }
  return levels >= kChainMinLevels && weights <= kChainLevelWeights * levels && dealt <= kChainUneven * even && tasks <= (double)kChainGrid * levels;
}

// Plans a whole step as one launch of gemv_chain_kernel.  false: the step is none that it serves.  fins: SelFinish of every linear.
// It serves steps of several levels in which every vector is either never written or, from a multiple of eight elements on,
// part of the result of one earlier linear, and no two results share memory: what a level reads then comes from mailboxes and
// from buffers that stay as they are, and it does not matter that the last workgroups of a level may still be at work when the
// first ones have begun a later one.
bool plan_chain(dpllm_model* m, const void* const* xs, void* const* ys, const std::vector<std::pair<int, int>>& bounds,
                const std::vector<int>& phase_of, std::vector<SelFinish>& fins) {
  const int n = (int)m->linears.size(), levels = (int)bounds.size();
  const Workspace& W = m->ws;
  StepPlan& P = m->plan;
  if (m->chain_mode < 0 || (m->chain_mode == 0 && !chain_pays(m, levels))) return false;
  for (const auto& [id, end] : bounds)
    if (end - id > kChainLevelJobs) return false;
  // the results by address
  struct Range { uintptr_t at, end; int id; };
  std::vector<Range> out(n);
  for (int j = 0; j < n; ++j) out[j] = {(uintptr_t)ys[j], (uintptr_t)ys[j] + (size_t)m->linears[j].L.out * 2, j};
  std::sort(out.begin(), out.end(), [](const Range& a, const Range& b) { return a.at < b.at; });
  for (int i = 1; i < n; ++i)
    if (out[i].at < out[i - 1].end) return false;
  // the linear that writes a vector (-1: none), and whether the step can be served
  auto writer = [&](const void* p, int in, int reader, int* from) {
    const uintptr_t a = (uintptr_t)p, e = a + (size_t)in * 2;
    auto it = std::upper_bound(out.begin(), out.end(), a, [](uintptr_t v, const Range& r) { return v < r.end; });   // the first that ends behind a
    *from = -1;
    if (it == out.end() || it->at >= e) return true;
    *from = it->id;
    return it->at <= a && e <= it->end && (a - it->at) % 16 == 0 && it->id < reader;
  };
  std::vector<size_t> mail_at(n, 0);
  std::vector<char> read(n, 0);
  size_t mail = 0;
  for (int j = 0; j < n; ++j) {
    mail_at[j] = mail;
    mail += mail_words(m->linears[j].L);
  }
  if (mail > W.chain_mail_cap) return false;
  std::vector<ChainLevel>& lv = m->h_chain_levels;
  std::vector<ChainJob>& jobs = m->h_chain_jobs;
  lv.assign(levels + 1, ChainLevel{});
  jobs.assign(n, ChainJob{});
  size_t slots = 0, ntasks = 0;
  for (ChainLevel& l : lv) std::fill(std::begin(l.unit_start), std::end(l.unit_start), 0x7fffffff);
  std::vector<std::vector<int>> tasks_of(levels);   // linears whose tasks run in a level
  for (int j = 0; j < n; ++j) {
    const Linear& lin = m->linears[j];
    ChainLevel& l = lv[phase_of[j]];
    const int first = bounds[phase_of[j]].first;
    l.job_first = first;
    l.job_count++;
    const void* sx = lin.sel_input ? lin.sel_input : xs[j];
    int from, sel_from;
    if (!writer(xs[j], lin.L.in, j, &from) || !writer(sx, lin.L.in, j, &sel_from)) return false;
    auto place = [&](int w, const void* p) {
      return (const uint16_t*)(W.at<uint64_t>(W.chain_mail) + mail_at[w]) + ((const char*)p - (const char*)ys[w]) / 2;
    };
    ChainJob& c = jobs[j];
    c.arena = lin.arena;
    c.x = from < 0 ? (const uint16_t*)xs[j] : place(from, xs[j]);
    c.x_handed = from >= 0;
    if (from >= 0) read[from] = 1;
    c.y = (uint16_t*)ys[j];
    c.e_out = P.e_dev + j;
    c.k_out = P.k_dev + j;
    if (lin.L.total_bytes >> 32) return false;   // (32-bit offsets)
    c.plane_bytes = (uint32_t)lin.L.plane_bytes;
    c.out = lin.L.out; c.ncw = lin.L.ncw; c.ncc = lin.L.ncc;
    for (int k = lin.L.kmin; k <= lin.L.p; ++k) c.lut_off[k - 1] = (uint32_t)lin.L.lut_offset[k];
    bool any = false, linreg = false;
    for (const Pair& s : lin.sel) {
      if (!s.set) continue;
      any |= s.kind != DPLLM_SEL_NONE;
      linreg |= s.kind == DPLLM_SEL_LINREG;
    }
    SelFinish f{};
    f.e_out = c.e_out; f.k_out = c.k_out;
    f.x = sel_from < 0 ? (const uint16_t*)sx : place(sel_from, sx);
    f.x_handed = sel_from >= 0;
    if (sel_from >= 0) read[sel_from] = 1;
    f.in = lin.L.in; f.linear = j; f.copies = kSelCopies; f.squares = linreg;
    const int slices = sel_slices(lin.L.in);
    f.chunk_cols = ((lin.L.in + slices - 1) / slices + kSelChunkStep - 1) / kSelChunkStep * kSelChunkStep;
    f.nchunks = (lin.L.in + f.chunk_cols - 1) / f.chunk_cols;
    f.task_rows = any ? std::max(1, lin.max_rowgroups() * kSelPartRows) : 0;
    f.ws_rows = std::max(1, f.task_rows);
    f.ws = W.at<double>(W.sel_ws) + slots;
    c.slots = (const uint64_t*)f.ws;
    c.slot_rows = f.ws_rows; c.nchunks = f.nchunks;
    slots += align_up((size_t)f.ws_rows * f.nchunks * kSelCopies, 16);
    fins[j] = f;
    if (!any) continue;
    // a selector whose vector is there a level earlier runs in that level
    const int ready = sel_from < 0 ? 0 : phase_of[sel_from] + 1, q = phase_of[j];
    tasks_of[ready < q ? q - 1 : q].push_back(j);
  }
  for (int l = 0; l < levels; ++l) {
    lv[l].task_first = (int32_t)ntasks;
    for (int j : tasks_of[l]) {
      fins[j].task_first = (int)ntasks;
      ntasks += (size_t)fins[j].task_rows * fins[j].nchunks;
    }
    lv[l].task_count = (int32_t)ntasks - lv[l].task_first;
  }
  if (ntasks > W.sel_tasks_cap || slots > W.sel_ws_cap) return false;
  // rows of a block: the makespan of a level in tiles a wavefront decodes, and about 0.6 of one for every block
  for (int i = 0; i < levels; ++i) {
    ChainLevel& l = lv[i];
    double best = 1e300;
    for (int lg = 2; lg >= 0; --lg) {
      int units = 0, widest = 0;
      for (int j = bounds[i].first; j < bounds[i].second; ++j) {
        const LinearLayout& L = m->linears[j].L;
        units += (L.out + (64 >> lg) - 1) / (64 >> lg);
        widest = std::max(widest, L.in);
      }
      const double chunks = (widest + kChainChunk * kLaneWaves - 1) / (kChainChunk * kLaneWaves);
      const double est = (units + kChainGrid - 1) / kChainGrid * (chunks * (4 >> lg) + 0.6);
      if (est < best) { best = est; l.log_groups = lg; }
    }
    for (int j = bounds[i].first; j < bounds[i].second; ++j) {
      l.unit_start[j - bounds[i].first] = l.units;
      l.units += (m->linears[j].L.out + (64 >> l.log_groups) - 1) / (64 >> l.log_groups);
    }
  }
  int grid = 1;
  for (int j = 0; j < n; ++j) jobs[j].mail = read[j] ? W.at<uint64_t>(W.chain_mail) + mail_at[j] : nullptr;
  for (const ChainLevel& l : lv) grid = std::max(grid, std::max(l.units, 0) + l.task_count);
  P.chain_grid = std::min(grid, kChainGrid);
  P.chain_slots = slots;
  P.chain_mail = mail;
  return true;
}

int build_plan(dpllm_model* m, const void* const* xs, void* const* ys, int32_t* k_dev, float* e_dev, hipStream_t st) {
  const int n = (int)m->linears.size();
  const Workspace& W = m->ws;
  StepPlan& P = m->plan;
  P.valid = P.captured = false;
  P.xs.assign(xs, xs + n);
  P.ys.assign(ys, ys + n);
  P.k_dev = k_dev;
  P.e_dev = e_dev;
  P.phases.clear();
  std::vector<SelJob>& sel_jobs = m->h_sel_jobs;
  std::vector<SelPart>& sel_parts = m->h_sel_parts;
  std::vector<int32_t>& sel_members = m->h_sel_members;
  std::vector<GemvJob>& gemv_jobs = m->h_gemv_jobs;
  std::vector<int32_t>& block_jobs = m->h_block_jobs;
  gemv_jobs.clear(); block_jobs.clear();
  // phases: maximal runs of consecutive linears that do not depend on one another
  std::vector<std::pair<int, int>> bounds;
  std::vector<int> phase_of(n, 0);
  for (int id = 0; id < n;) {
    int end = id + 1;
    for (; end < n; ++end) {  // extend the phase while linear `end` is independent of all of [id, end)
      const Linear& le = m->linears[end];
      bool dep = false;
      for (int j = id; j < end && !dep; ++j) {
        const Linear& lj = m->linears[j];
        dep = overlap(xs[end], (size_t)le.L.in * 2, ys[j], (size_t)lj.L.out * 2) ||
              (le.sel_input && overlap(le.sel_input, (size_t)le.L.in * 2, ys[j], (size_t)lj.L.out * 2)) ||
              (lj.sel_input && overlap(ys[end], (size_t)le.L.out * 2, lj.sel_input, (size_t)lj.L.in * 2)) ||
              overlap(ys[end], (size_t)le.L.out * 2, xs[j], (size_t)lj.L.in * 2) ||
              overlap(ys[end], (size_t)le.L.out * 2, ys[j], (size_t)lj.L.out * 2);
      }
      if (dep) break;
    }
    for (int j = id; j < end; ++j) phase_of[j] = (int)bounds.size();
    bounds.emplace_back(id, end);
    id = end;
  }
  // the GEMV launch of every phase
  for (const auto& [id, end] : bounds) {
    Phase ph;
    ph.gemv_first = (int)gemv_jobs.size();
    ph.block_first = (int)block_jobs.size();
    long total_rq = 0, lane_groups = 0;
    for (int j = id; j < end; ++j) total_rq += m->linears[j].L.nrq;
    int min_ncc = m->linears[id].L.ncc;
    for (int j = id; j < end; ++j) min_ncc = std::min(min_ncc, m->linears[j].L.ncc);
    ph.groups = pick_groups(total_rq, min_ncc);
    // The chip runs 512 workgroups at a time.  A launch of a few such rounds loses the unfilled part of its last
    // round (2.7 rounds cost 3): the work per workgroup is scaled, between half and one and a half times the
    // usual megabyte, to the value with the smallest estimate of rounds x (start-up + work of a workgroup).
    long base_bytes = kLaneGroupBytes;
    {
      double best = 1e300;
      for (int pct = 50; pct <= 150; pct += 5) {
        const long gb = kLaneGroupBytes * pct / 100;
        long groups = 0;
        for (int j = id; j < end; ++j) {
          const Linear& lin = m->linears[j];
          const int rpb = pick_blocks_per_group(lin.L, lin.part_k(), total_rq, gb);
          groups += (lin.L.nrq + rpb - 1) / rpb;
        }
        const double rounds = std::ceil(groups / 512.0);
        const double est = rounds * (4.0 + 85.0 * pct / 100) * (1.0 + 0.0005 * std::abs(pct - 100));   // ties: the usual size
        if (est < best) { best = est; base_bytes = gb; lane_groups = groups; }
      }
    }
    std::vector<long> bytes_after(end - id, 0);   // plane bytes of the launch that follow linear j
    {
      long acc = 0;
      for (int j = end - 1; j >= id; --j) {
        const Linear& lin = m->linears[j];
        bytes_after[j - id] = acc;
        acc += (long)lin.L.nrq * 64 * lin.L.in * lin.part_k() / 8;
      }
    }
    // Large launches: the linears dispatched last (one round of workgroups: two on each of 256 compute units)
    // get workgroups of half the usual work, so that the chip drains in less time at the end of the launch
    // (measured on the 7B step: 0.5 - 0.8 % of the launch; quarters and eighths did not add to that).
    const bool taper = lane_groups >= 2048;
    int blocks = 0;
    for (int j = id; j < end; ++j) {
      const Linear& lin = m->linears[j];
      GemvJob gj = make_gemv_job(lin, 0, k_dev + j, xs[j], ys[j]);
      long group_bytes = base_bytes;
      if (taper && bytes_after[j - id] < 512 * base_bytes) group_bytes /= 2;
      const int rpb = pick_blocks_per_group(lin.L, lin.part_k(), total_rq, group_bytes);
      gj.nblocks = ph.groups > 1 ? (lin.L.out + 64 / ph.groups - 1) / (64 / ph.groups) : (lin.L.nrq + rpb - 1) / rpb;
      gj.block_start = blocks;
      blocks += gj.nblocks;
      block_jobs.insert(block_jobs.end(), gj.nblocks, (int32_t)(gemv_jobs.size() - ph.gemv_first));
      gemv_jobs.push_back(gj);
    }
    ph.gemv_count = (int)gemv_jobs.size() - ph.gemv_first;
    ph.blocks = blocks;
    ph.may_decide = blocks < kDecideMaxBlocks;
    // a selector that reads what its own linear writes has to be done before the GEMV launch starts
    for (int j = id; j < end; ++j) {
      const Linear& lin = m->linears[j];
      if (lin.sel_input && overlap(lin.sel_input, (size_t)lin.L.in * 2, ys[j], (size_t)lin.L.out * 2)) ph.may_decide = false;
    }
    P.phases.push_back(ph);
  }
  std::vector<SelFinish> fins(n);
  P.chain = plan_chain(m, xs, ys, bounds, phase_of, fins);
  // the selectors of every phase, at most twice: a workspace handed over before the selectors were attached may hold
  // their parts but not the tasks of the launches that run them
  for (bool tasks = !P.chain;; tasks = false) {
    // A selector that reads its own input buffer (asynchronous estimation, Sec. 5.2) does not have to run right
    // before its linear: any phase from which on nothing writes that buffer before the linear runs will do.  It
    // joins the latest such phase that launches selectors anyway (for linears that estimate from their immediate
    // input), so that its own phase starts with the GEMV; without such a phase it stays where it is, and so it does where
    // the GEMV launch of its own phase does not take the decision (the launch that does serves the selectors of its phase).
    sel_jobs.clear(); sel_parts.clear(); sel_members.clear();
    size_t ws_slots = 0, ntasks = 0;
    P.fused = false;
    std::vector<char> has_selectors(bounds.size(), 0);
    for (int j = 0; j < n; ++j)
      if (!m->linears[j].sel_input) has_selectors[phase_of[j]] = 1;
    std::vector<std::vector<int>> sel_of_phase(bounds.size());
    std::vector<char> ahead(bounds.size(), 0);   // a selector of the phase runs with an earlier one
    for (int j = 0; j < n; ++j) {
      const Linear& lin = m->linears[j];
      int q = phase_of[j];
      if (lin.sel_input && P.phases[q].may_decide) {
        int first = q;   // earliest phase the selector may run in
        while (first > 0) {
          bool written = false;
          for (int i = bounds[first - 1].first; i < bounds[first - 1].second && !written; ++i)
            written = overlap(lin.sel_input, (size_t)lin.L.in * 2, ys[i], (size_t)m->linears[i].L.out * 2);
          if (written) break;
          --first;
        }
        while (q > first && !has_selectors[q]) --q;
        if (!has_selectors[q]) q = phase_of[j];
        has_selectors[q] = 1;
      }
      sel_of_phase[q].push_back(j);
      if (q != phase_of[j]) ahead[phase_of[j]] = 1;
    }
    for (size_t pi = 0; pi < bounds.size(); ++pi) {
      Phase& ph = P.phases[pi];
      ph.sel_first = (int)sel_jobs.size();
      ph.sel_count = (int)sel_of_phase[pi].size();
      ph.part_first = (int)sel_parts.size();
      long launch_rowgroups = 0, launch_slices = 0;
      for (int j : sel_of_phase[pi]) {
        launch_rowgroups += m->linears[j].max_rowgroups();
        launch_slices += (long)m->linears[j].max_rowgroups() * kSelPartRows * sel_slices(m->linears[j].L.in);
      }
      // Parts of a launch are of one size, the smallest that lets all of them run at once (1280: five wavefronts per SIMD): rows of different
      // lengths cut into the same number of chunks, as they were, leave the long parts to the end.  us of the selectors of 8 blocks of 70B,
      // then -> now: 25.7 -> 21.1, every second linear on the linear regression 18.6 -> 15.2; 32 blocks of 7B 29.6 with parts of 4096 columns (1152 of
      // them), 31.6 of 2048, 33.9 of 1024.
      int chunk_cols = kSelChunkStep;
      for (; chunk_cols < kSelTaskCols; chunk_cols += kSelChunkStep) {
        long parts = 0;
        for (int j : sel_of_phase[pi])
          parts += (long)m->linears[j].max_rowgroups() * std::min(kSelMaxChunks, (m->linears[j].L.in + chunk_cols - 1) / chunk_cols);
        if (parts <= 1280) break;
      }
      const bool small = runs_selectors(ph.blocks, launch_rowgroups * kSelPartRows, launch_slices);
      ph.fused = tasks && ph.may_decide && small;
      ph.decides = ph.may_decide && (small || ahead[pi] || ph.blocks <= kPrologueMaxBlocks);
      // Selectors inside the GEMV launch: a task is a row of G times a slice of at most 4096 columns (one load per
      // wavefront), or more where there are more rows than workgroups to share them out to.
      ph.task_first = (int)ntasks;
      const long slices_each = std::max<long>(1, kSelTaskGroups / std::max<long>(1, launch_rowgroups * kSelPartRows));
      for (size_t local = 0; local < sel_of_phase[pi].size(); ++local) {
        const int j = sel_of_phase[pi][local];
        const Linear& lin = m->linears[j];
        const int rowgroups = lin.max_rowgroups();
        SelJob sj = make_sel_job(lin, j, rowgroups, lin.sel_input ? lin.sel_input : xs[j], e_dev + j, k_dev + j, chunk_cols);
        for (int part = 0; part < rowgroups * sj.nchunks; ++part) sel_parts.push_back(SelPart{(int)local, part, j, 0, 0, 0});
        sj.ws = W.at<double>(W.sel_ws) + ws_slots;
        SelFinish fin = sel_finish_of(sj);
        if (ph.fused) fin.copies = kSelCopies;
        if (ph.fused && rowgroups > 0) {
          const long slices = std::min<long>(sel_slices(lin.L.in), slices_each);
          fin.chunk_cols = (int)((lin.L.in + slices - 1) / slices + kSelChunkStep - 1) / kSelChunkStep * kSelChunkStep;
          fin.nchunks = (lin.L.in + fin.chunk_cols - 1) / fin.chunk_cols;
          fin.task_first = (int)ntasks;
          fin.task_rows = rowgroups * kSelPartRows;
          ntasks += (size_t)fin.task_rows * fin.nchunks;
        }
        ws_slots += (size_t)sj.ws_rows * (rowgroups > 0 ? std::max(sj.nchunks, fin.copies * fin.nchunks) : 1);
        gemv_jobs[j].has_fin = 1;                 // (the jobs of all linears, in their order)
        gemv_jobs[j].fin = fin;
        sel_jobs.push_back(sj);
      }
      ph.task_count = (int)ntasks - ph.task_first;
      // groups of jobs that read the same vector: one more part each, which adds up x^2 once for the members whose
      // estimator is the linear regression
      ph.member_first = (int)sel_members.size();
      for (int a = 0; a < ph.sel_count; ++a) {
        const SelJob& ja = sel_jobs[ph.sel_first + a];
        bool head = true;
        for (int b = 0; b < a && head; ++b) head = sel_jobs[ph.sel_first + b].x != ja.x || sel_jobs[ph.sel_first + b].in != ja.in;
        if (!head) continue;
        const int first = (int)sel_members.size() - ph.member_first;
        for (int b = a; b < ph.sel_count; ++b) {
          const SelJob& jb = sel_jobs[ph.sel_first + b];
          if (jb.x == ja.x && jb.in == ja.in) sel_members.push_back(b);
        }
        sel_parts.push_back(SelPart{a, -1, ja.linear, (int)sel_members.size() - ph.member_first - first, first, 0});
      }
      ph.part_count = (int)sel_parts.size() - ph.part_first;
      if (ph.task_count > 0) P.fused = true;
    }
    const bool fits = sel_parts.size() <= W.sel_parts_cap && ws_slots <= W.sel_ws_cap && ntasks <= W.sel_tasks_cap &&
                      block_jobs.size() <= W.block_jobs_cap;
    P.slots = ws_slots;
    if (fits) break;
    if (!P.fused)
      return fail(m, DPLLM_ESTATE, "workspace too small for this step (set after the model changed?): call dpllm_workspace_bytes and "
                                   "dpllm_set_workspace again");
  }
  if (P.chain) {   // (the launches of a step in parts, the only others of this plan, do not read them)
    for (int j = 0; j < n; ++j) gemv_jobs[j].fin = fins[j];
    HIP_TRY(m, hipMemcpyAsync(W.at<ChainLevel>(W.chain_levels), m->h_chain_levels.data(), sizeof(ChainLevel) * m->h_chain_levels.size(), hipMemcpyHostToDevice, st));
    HIP_TRY(m, hipMemcpyAsync(W.at<ChainJob>(W.chain_jobs), m->h_chain_jobs.data(), sizeof(ChainJob) * n, hipMemcpyHostToDevice, st));
  }
  // The tables may still be read by a step enqueued earlier on this stream: the copies are ordered behind it.
  if (!sel_parts.empty())
    HIP_TRY(m, hipMemcpyAsync(W.at<SelPart>(W.sel_parts), sel_parts.data(), sizeof(SelPart) * sel_parts.size(), hipMemcpyHostToDevice, st));
  if (!block_jobs.empty())
    HIP_TRY(m, hipMemcpyAsync(W.at<int32_t>(W.block_jobs), block_jobs.data(), sizeof(int32_t) * block_jobs.size(), hipMemcpyHostToDevice, st));
  HIP_TRY(m, hipMemcpyAsync(W.at<SelJob>(W.sel_jobs), sel_jobs.data(), sizeof(SelJob) * sel_jobs.size(), hipMemcpyHostToDevice, st));
  HIP_TRY(m, hipMemcpyAsync(W.at<int32_t>(W.sel_members), sel_members.data(), sizeof(int32_t) * sel_members.size(), hipMemcpyHostToDevice, st));
  if (!gemv_jobs.empty())
    HIP_TRY(m, hipMemcpyAsync(W.at<GemvJob>(W.gemv_jobs), gemv_jobs.data(), sizeof(GemvJob) * gemv_jobs.size(), hipMemcpyHostToDevice, st));
  P.version = m->version;
  P.valid = true;
  m->params_dirty = true;   // the phases' estimator flags and the tasks are worked out with the parameter table
  return DPLLM_OK;
}

// device address of `scratch` on the current device, looked up on the first call on that device
constexpr int kMaxDevices = 64;
int static_scratch_ptr(dpllm_model* m, double** out) {
  static double* ptr[kMaxDevices] = {};
  int dev = 0;
  HIP_TRY(m, hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(m, DPLLM_EINVAL, "device %d outside [0,%d)", dev, kMaxDevices);
  if (!ptr[dev]) {
    void* p = nullptr;
    HIP_TRY(m, hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(m, DPLLM_EHIP, "hipGetSymbolAddress returned a null address");
    ptr[dev] = (double*)p;
  }
  *out = ptr[dev];
  return DPLLM_OK;
}

bool capturing(hipStream_t st) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &s) != hipSuccess) { (void)hipGetLastError(); return false; }
  return s != hipStreamCaptureStatusNone;
}

// Whether an event has passed.  A query is not allowed, and can spoil the capture, while some stream is captured in the global
// mode by any thread; this one has nothing to do with a capture.
bool passed(hipEvent_t event) {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
  const bool done = hipEventQuery(event) == hipSuccess;
  if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
  (void)hipGetLastError();
  return done;
}

}  // namespace

extern "C" {

int dpllm_model_create(dpllm_model** out, int n_linears) {
  if (!out || n_linears < 1) return DPLLM_EINVAL;
  *out = nullptr;
  dpllm_model* m = new (std::nothrow) dpllm_model();
  if (!m) return DPLLM_EINVAL;
  m->linears.resize(n_linears);
  if (hipGetDevice(&m->device) != hipSuccess) {
    (void)hipGetLastError();
    delete m;
    return DPLLM_EHIP;
  }
  *out = m;
  return DPLLM_OK;
}

void dpllm_model_destroy(dpllm_model* m) {
  if (m && m->ws_event) (void)hipEventDestroy(m->ws_event);
  delete m;
}

const char* dpllm_last_error(const dpllm_model* m) { return m ? m->err.c_str() : "null model"; }

int dpllm_linear_device_bytes(int out, int in, int p, int kmin, size_t* bytes) {
  if (!bytes) return DPLLM_EINVAL;
  int rc = check_shape(out, in, p, kmin);
  if (rc != DPLLM_OK) return rc;
  *bytes = LinearLayout::make(out, in, p, kmin).total_bytes;
  return DPLLM_OK;
}

int dpllm_debug_locate(int out, int in, int p, int kmin, int plane, int row, int col, size_t* byte_offset, int* bit) {
  if (!byte_offset || !bit) return DPLLM_EINVAL;
  int rc = check_shape(out, in, p, kmin);
  if (rc != DPLLM_OK) return rc;
  if (plane < 0 || plane >= p || row < 0 || row >= out || col < 0 || col >= in) return DPLLM_ERANGE;
  const LinearLayout L = LinearLayout::make(out, in, p, kmin);
  // the word of the tile, the column's position inside it, and the rotation of plane b (see layout_device.hpp)
  const size_t word = plane_word_index(row, col / 32, L.ncc);
  *byte_offset = (size_t)plane * L.plane_bytes + word * 4;
  *bit = ((col_to_pos(col % 32) - plane) % 32 + 32) % 32;
  return DPLLM_OK;
}

int dpllm_workspace_bytes(const dpllm_model* m, size_t* bytes) {
  if (!m || !bytes) return DPLLM_EINVAL;
  *bytes = carve_workspace(m).total;
  return DPLLM_OK;
}

int dpllm_set_workspace(dpllm_model* m, void* ws_dev, size_t bytes, void* stream) {
  if (!m) return DPLLM_EINVAL;
  if (!ws_dev) return fail(m, DPLLM_EINVAL, "null workspace");
  if ((uintptr_t)ws_dev % kAlign) return fail(m, DPLLM_EINVAL, "workspace not %zu-byte aligned", kAlign);
  Workspace w = carve_workspace(m);
  if (bytes < w.total) return fail(m, DPLLM_ESTATE, "workspace holds %zu bytes, %zu needed", bytes, w.total);
  w.base = (char*)ws_dev;
  w.bytes = bytes;
  hipStream_t st = (hipStream_t)stream;
  if (capturing(st)) w.est_slots_cap = 0;   // (emptied by a replay at some time to come: no estimate relies on it)
  else if (w.est_slots_cap > 0 && !m->ws_event) HIP_TRY(m, hipEventCreateWithFlags(&m->ws_event, hipEventDisableTiming));
  // the target starts at zero, the jobs without tasks, the slots of lone estimates empty; everything else is written before it is used
  struct { size_t off, words; } zero[] = {{w.target, 1}, {w.gemv_jobs, sizeof(GemvJob) / 4 * m->linears.size()}, {w.est_sets, w.est_slots_cap > 0 ? w.est_set_words() * kEstRing * 2 : 0}};
  for (const auto& z : zero)
    if (z.words > 0)
      hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((z.words + 255) / 256)), dim3(256), 0, st, w.at<uint32_t>(z.off), z.words, 0u);
  HIP_TRY(m, hipGetLastError());
  if (w.est_slots_cap > 0) HIP_TRY(m, hipEventRecord(m->ws_event, st));
  m->ws_stream = st;
  m->est_ready = false;
  m->ws = w;
  m->params_dirty = true;
  m->version++;
  return DPLLM_OK;
}

int dpllm_load_linear(dpllm_model* m, int id, int out, int in, int p, int kmin, const uint32_t* planes,
                      const uint16_t* const* luts, int src_on_device, void* dev_arena, size_t arena_bytes,
                      void* stream) {
  if (!m) return DPLLM_EINVAL;
  if (id < 0 || id >= (int)m->linears.size()) return fail(m, DPLLM_EINVAL, "linear id %d out of range", id);
  if (!planes || !luts || !dev_arena) return fail(m, DPLLM_EINVAL, "null pointer");
  if (src_on_device != 0 && src_on_device != 1) return fail(m, DPLLM_EINVAL, "src_on_device must be 0 or 1");
  int rc = check_shape(out, in, p, kmin);
  if (rc != DPLLM_OK) return fail(m, rc, "bad shape out=%d in=%d p=%d kmin=%d", out, in, p, kmin);
  for (int k = kmin; k <= p; ++k)
    if (!luts[k - kmin]) return fail(m, DPLLM_EINVAL, "null table for k=%d", k);
  if ((uintptr_t)dev_arena % kAlign) return fail(m, DPLLM_EINVAL, "arena not %zu-byte aligned", kAlign);
  LinearLayout L = LinearLayout::make(out, in, p, kmin);
  if (arena_bytes < L.total_bytes)
    return fail(m, DPLLM_ESTATE, "arena holds %zu bytes, %zu needed", arena_bytes, L.total_bytes);
  hipStream_t st = (hipStream_t)stream;

  const size_t plane_words = (size_t)p * out * L.ncw;
  size_t lut_elems_total = 0;
  for (int k = kmin; k <= p; ++k) lut_elems_total += (size_t)out << k;
  const uint32_t* d_planes = planes;
  void* staging = nullptr;
  if (!src_on_device) {   // host sources pass through a device staging buffer that lives for the length of this call
    HIP_TRY(m, hipMalloc(&staging, plane_words * 4 + lut_elems_total * 2));
    hipError_t e = hipMemcpyAsync(staging, planes, plane_words * 4, hipMemcpyHostToDevice, st);
    char* dst = (char*)staging + plane_words * 4;
    for (int k = kmin; k <= p && e == hipSuccess; ++k) {
      size_t bytes = ((size_t)out << k) * 2;
      e = hipMemcpyAsync(dst, luts[k - kmin], bytes, hipMemcpyHostToDevice, st);
      dst += bytes;
    }
    if (e != hipSuccess) { (void)hipFree(staging); return hip_fail(m, e, "hipMemcpyAsync"); }
    d_planes = (const uint32_t*)staging;
  }
  {
    size_t n = (size_t)L.nrq * L.ncc * 64 * p;
    hipLaunchKernelGGL(retile_planes_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, d_planes,
                       (uint4*)dev_arena, p, out, L.ncw, L.ncc, L.nrq, L.plane_bytes / 16);
  }
  const char* lsrc = staging ? (const char*)staging + plane_words * 4 : nullptr;
  for (int k = kmin; k <= p; ++k) {
    const uint16_t* src = staging ? (const uint16_t*)lsrc : luts[k - kmin];
    size_t n = (size_t)L.rows_padded << k;
    hipLaunchKernelGGL(copy_lut_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, src,
                       (uint16_t*)((char*)dev_arena + L.lut_offset[k]), out, L.rows_padded, 1 << k);
    if (staging) lsrc += ((size_t)out << k) * 2;
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (staging) (void)hipFree(staging);
  if (e != hipSuccess) return hip_fail(m, e, "load kernels");
  Linear& lin = m->linears[id];
  lin = Linear();
  lin.loaded = true;
  lin.L = L;
  lin.arena = (char*)dev_arena;
  m->version++;
  m->params_dirty = true;
  return DPLLM_OK;
}

int dpllm_set_selector(dpllm_model* m, int id, int l, int h, int kind, const void* G_dev, int r, float alpha,
                       float beta, float T) {
  int rc = DPLLM_OK;
  Linear* lin = get_linear(m, id, &rc);
  if (!lin) return rc;
  if (l < lin->L.kmin || h > lin->L.p || l > h) return fail(m, DPLLM_ERANGE, "pair (%d,%d) outside [%d,%d]", l, h, lin->L.kmin, lin->L.p);
  if (std::isnan(T)) return fail(m, DPLLM_EINVAL, "threshold is NaN");
  if (kind == DPLLM_SEL_PROJ) {
    if (!G_dev) return fail(m, DPLLM_EINVAL, "G is null");
    if (r < 1 || r > DPLLM_MAX_RANK) return fail(m, DPLLM_ERANGE, "rank %d outside [1,%d]", r, DPLLM_MAX_RANK);
    if ((uintptr_t)G_dev % 16) return fail(m, DPLLM_EINVAL, "G not 16-byte aligned");
  } else if (kind == DPLLM_SEL_LINREG) {
    if (std::isnan(alpha) || std::isnan(beta)) return fail(m, DPLLM_EINVAL, "alpha/beta NaN");
  } else if (kind == DPLLM_SEL_NONE) {
    if (l != h) return fail(m, DPLLM_EINVAL, "kind none needs l == h");
  } else {
    return fail(m, DPLLM_EINVAL, "unknown selector kind %d", kind);
  }
  int slot = lin->find_pair(l, h);
  if (slot < 0)
    for (int i = 0; i < DPLLM_MAX_PAIRS && slot < 0; ++i)
      if (!lin->sel[i].set) slot = i;
  if (slot < 0) return fail(m, DPLLM_ESTATE, "linear %d already holds %d pairs", id, DPLLM_MAX_PAIRS);
  Pair& s = lin->sel[slot];
  // the launch plan is sized by the kinds and ranks of all pairs of the linear: it survives a change of G, alpha, beta or T
  const bool same_shape = s.set && s.kind == kind && sel_rowgroups_of(s.kind, s.r) == sel_rowgroups_of(kind, r);
  s.set = true; s.l = l; s.h = h; s.kind = kind; s.r = kind == DPLLM_SEL_PROJ ? r : 0; s.G = (const uint16_t*)G_dev;
  s.alpha = alpha; s.beta = beta; s.T = T;
  if (!same_shape) m->version++;
  use_pair(m, lin, slot);
  m->params_dirty = true;
  return DPLLM_OK;
}

int dpllm_set_threshold(dpllm_model* m, int id, int l, int h, float T) {
  int rc = DPLLM_OK;
  Linear* lin = get_linear(m, id, &rc);
  if (!lin) return rc;
  if (std::isnan(T)) return fail(m, DPLLM_EINVAL, "threshold is NaN");
  int slot = lin->find_pair(l, h);
  if (slot < 0) return fail(m, DPLLM_ESTATE, "pair (%d,%d) not set on linear %d", l, h, id);
  lin->sel[slot].T = T;
  m->params_dirty = true;
  return DPLLM_OK;
}

int dpllm_set_active_pair(dpllm_model* m, int id, int l, int h) {
  int rc = DPLLM_OK;
  Linear* lin = get_linear(m, id, &rc);
  if (!lin) return rc;
  int slot = lin->find_pair(l, h);
  if (slot < 0) return fail(m, DPLLM_ESTATE, "pair (%d,%d) not set on linear %d", l, h, id);
  use_pair(m, lin, slot);
  m->params_dirty = true;
  return DPLLM_OK;
}

int dpllm_set_target_entry(dpllm_model* m, int target, int id, int l, int h, float T) {
  int rc = DPLLM_OK;
  Linear* lin = get_linear(m, id, &rc);
  if (!lin) return rc;
  if (target < 1 || target >= DPLLM_MAX_TARGETS) return fail(m, DPLLM_EINVAL, "target %d outside [1,%d]", target, DPLLM_MAX_TARGETS - 1);
  if (std::isnan(T)) return fail(m, DPLLM_EINVAL, "threshold is NaN");
  int slot = lin->find_pair(l, h);
  if (slot < 0) return fail(m, DPLLM_ESTATE, "pair (%d,%d) not set on linear %d", l, h, id);
  lin->tgt[target].set = true;
  lin->tgt[target].slot = slot;
  lin->tgt[target].T = T;
  m->params_dirty = true;
  return DPLLM_OK;
}

int dpllm_set_target(dpllm_model* m, int target, void* stream) {
  if (!m) return DPLLM_EINVAL;
  if (target < 0 || target >= DPLLM_MAX_TARGETS) return fail(m, DPLLM_EINVAL, "target %d outside [0,%d]", target, DPLLM_MAX_TARGETS - 1);
  if (!m->ws.base) return fail(m, DPLLM_ESTATE, "no workspace set");
  activate(m, target, (hipStream_t)stream);
  HIP_TRY(m, hipGetLastError());
  return DPLLM_OK;
}

int dpllm_set_selector_input(dpllm_model* m, int id, const void* xsel_dev) {
  int rc = DPLLM_OK;
  Linear* lin = get_linear(m, id, &rc);
  if (!lin) return rc;
  if ((uintptr_t)xsel_dev % 16) return fail(m, DPLLM_EINVAL, "selector input not 16-byte aligned");
  lin->sel_input = xsel_dev;
  m->version++;
  return DPLLM_OK;
}

constexpr int kSelParts = 1152;   // parts of a lone estimate with many rows, about

// The job of a lone estimate.  Up to the ranks that one launch serves, the columns are cut into no more chunks than its last workgroup
// collects at a time; the ways an estimate may take share the cut, and with it the bits.  us of a dpllm_estimate in a graph, up to 32 chunks /
// 12: rank 64 of 8192 columns 4.9 / 4.5, 11008 5.3 / 4.8, 14336 6.3 / 5.2, 28672 6.9 / 6.2; rank 256 of 8192 6.9 / 5.3, 28672 11.3 / 7.8 (8 chunks: rank 64 of
// 5120 4.4 where 12 take 4.1, of 28672 6.7).
static SelJob lone_job(const Linear& lin, int id, int rowgroups, const void* x_dev, float* e_dev, int32_t* k_dev) {
  const bool few = rowgroups * kSelPartRows <= kEstMaxRank;
  const long want = std::min<long>(few ? kEstChunks : kSelMaxChunks, kSelParts / std::max(1, rowgroups));
  const int cols = (int)((lin.L.in + want - 1) / want + kSelChunkStep - 1) / kSelChunkStep * kSelChunkStep;
  SelJob j = make_sel_job(lin, id, rowgroups, x_dev, e_dev, k_dev, std::min(cols, kSelTaskCols), few ? kEstChunks : kSelMaxChunks);
  j.row_each = few;
  return j;
}

// the two launches of a lone estimate: the parts leave their partial results in `slots`, the decide kernel finishes
static int launch_estimate(dpllm_model* m, const Linear& lin, int id, const Pair& sel, const void* x_dev, float* e_dev, int32_t* k_dev,
                           double* slots, hipStream_t st) {
  const int rowgroups = sel_rowgroups_of(sel.kind, sel.r);
  SelJob j = lone_job(lin, id, rowgroups, x_dev, e_dev, k_dev);
  j.ws = slots;
  const SelParams P = make_params(sel, sel.T);
  const int parts = j.row_each ? (sel.r + kSelPartWaves - 1) / kSelPartWaves : rowgroups;
  const int blocks = sel.kind == DPLLM_SEL_PROJ ? parts * j.nchunks : sel.kind == DPLLM_SEL_LINREG ? 1 : 0;
  if (blocks > 0)
    hipLaunchKernelGGL(selector_part_kernel, dim3(blocks), dim3(kSelPartThreads), 0, st, (const SelJob*)nullptr,
                       (const SelPart*)nullptr, (const int32_t*)nullptr, (const SelParams*)nullptr, j, P);
  hipLaunchKernelGGL(selector_decide_kernel, dim3(1), dim3(kSelDecideThreads), 0, st, (const SelJob*)nullptr,
                     (const SelParams*)nullptr, j, P);
  HIP_TRY(m, hipGetLastError());
  return DPLLM_OK;
}

// one launch, with slots of the workspace; false: the rank is beyond what its last workgroup collects at a time, a pair attached
// after the workspace was handed over needs more slots, or they may not be empty yet
static bool launch_estimate_once(dpllm_model* m, const Linear& lin, int id, const Pair& sel, const void* x_dev, float* e_dev, int32_t* k_dev,
                                 hipStream_t st) {
  const Workspace& W = m->ws;
  const int rowgroups = sel_rowgroups_of(sel.kind, sel.r);
  SelJob j = lone_job(lin, id, rowgroups, x_dev, e_dev, k_dev);
  if (lin.L.ncw > kEstMaxWords || (sel.kind == DPLLM_SEL_PROJ && (sel.r > kEstMaxRank || (size_t)j.ws_rows * j.nchunks > W.est_slots_cap))) return false;
  if (!m->est_ready && sel.kind == DPLLM_SEL_PROJ) {
    // the slots are empty for work behind dpllm_set_workspace on its stream, for any other once that has been seen to be done
    if (!capturing(st) && passed(m->ws_event)) m->est_ready = true;
    if (!m->est_ready && st != m->ws_stream) return false;
  }
  if (sel.kind == DPLLM_SEL_PROJ && (++m->est_turn == kEstAll || m->est_turn == 0)) m->est_turn = 1;   // (0: an empty slot)
  const unsigned set = m->est_turn % kEstRing;
  const int polls = m->polls == kSelPolls ? kEstPolls : std::max(m->polls, 0);
  const int parts = sel.kind == DPLLM_SEL_PROJ ? (sel.r + kEstPartRows - 1) / kEstPartRows * j.nchunks : 1;
  const bool proj = sel.kind == DPLLM_SEL_PROJ;
  const EstShape shape{lin.L.ncw, proj ? j.nchunks : 0, proj ? j.ws_rows : 0};
  const EstPair pair{proj ? j.chunk_cols : 0, proj ? sel.r : 0, sel.kind, proj && capturing(st), sel.l, sel.h};
  hipLaunchKernelGGL(selector_estimate_kernel, dim3(parts), dim3(kSelPartThreads), 0, st, sel.G, (const uint16_t*)x_dev,
                     W.at<uint64_t>(W.est_sets) + set * W.est_set_words() + kEstHeader, e_dev, k_dev, shape.pack(), pair.pack(), m->est_turn, sel.T, polls, sel.alpha,
                     sel.beta);
  return true;
}

static int check_estimate_args(dpllm_model* m, int id, int l, int h, const void* x_dev, float* e_dev, int32_t* k_dev, Linear** lin,
                               int* slot) {
  int rc = DPLLM_OK;
  *lin = get_linear(m, id, &rc);
  if (!*lin) return rc;
  if (!x_dev || !e_dev || !k_dev) return fail(m, DPLLM_EINVAL, "null pointer");
  if ((uintptr_t)x_dev % 16) return fail(m, DPLLM_EINVAL, "x not 16-byte aligned");
  *slot = (*lin)->find_pair(l, h);
  if (*slot < 0) return fail(m, DPLLM_ESTATE, "pair (%d,%d) not set on linear %d", l, h, id);
  return DPLLM_OK;
}

int dpllm_estimate(dpllm_model* m, int id, int l, int h, const void* x_dev, float* e_dev, int32_t* k_dev,
                   void* stream) {
  Linear* lin = nullptr;
  int slot = -1;
  int rc = check_estimate_args(m, id, l, h, x_dev, e_dev, k_dev, &lin, &slot);
  if (rc != DPLLM_OK) return rc;
  if (!m->ws.base) return fail(m, DPLLM_ESTATE, "no workspace set");
  if (launch_estimate_once(m, *lin, id, lin->sel[slot], x_dev, e_dev, k_dev, (hipStream_t)stream)) {
    HIP_TRY(m, hipGetLastError());
    return DPLLM_OK;
  }
  return launch_estimate(m, *lin, id, lin->sel[slot], x_dev, e_dev, k_dev, m->ws.at<double>(m->ws.est_ws), (hipStream_t)stream);
}

int dpllm_estimate_noalloc(dpllm_model* m, int id, int l, int h, const void* x_dev, float* e_dev, int32_t* k_dev,
                           void* stream) {
  Linear* lin = nullptr;
  int slot = -1;
  int rc = check_estimate_args(m, id, l, h, x_dev, e_dev, k_dev, &lin, &slot);
  if (rc != DPLLM_OK) return rc;
  const Pair& sel = lin->sel[slot];
  if (sel.kind == DPLLM_SEL_PROJ && sel.r > kStaticMaxRank)
    return fail(m, DPLLM_ERANGE, "rank %d beyond the static scratch (at most %d): use dpllm_estimate with a workspace", sel.r, kStaticMaxRank);
  double* slots = nullptr;
  rc = static_scratch_ptr(m, &slots);
  if (rc != DPLLM_OK) return rc;
  // nothing in the scratch has to start at zero: every slot the decide kernel reads is written by the parts of
  // this call first (the previous call's contents are never read)
  return launch_estimate(m, *lin, id, sel, x_dev, e_dev, k_dev, slots, (hipStream_t)stream);
}

int dpllm_gemv(dpllm_model* m, int id, int k, const int32_t* k_dev, const void* x_dev, void* y_dev, int B,
               void* stream) {
  int rc = DPLLM_OK;
  Linear* lin = get_linear(m, id, &rc);
  if (!lin) return rc;
  if (!x_dev || !y_dev) return fail(m, DPLLM_EINVAL, "null pointer");
  if ((uintptr_t)x_dev % 16) return fail(m, DPLLM_EINVAL, "x not 16-byte aligned");
  if (B < 1 || B > DPLLM_MAX_BATCH) return fail(m, DPLLM_ESHAPE, "batch %d outside [1,%d]", B, DPLLM_MAX_BATCH);
  if (overlap(x_dev, (size_t)B * lin->L.in * 2, y_dev, (size_t)B * lin->L.out * 2)) return fail(m, DPLLM_EINVAL, "x and y overlap");
  if (k >= 0) {
    if (k < lin->L.kmin || k > lin->L.p) return fail(m, DPLLM_ERANGE, "k=%d outside [%d,%d]", k, lin->L.kmin, lin->L.p);
    return launch_gemv(m, *lin, k, nullptr, x_dev, y_dev, B, (hipStream_t)stream);
  }
  if (!k_dev) return fail(m, DPLLM_EINVAL, "k < 0 needs k_dev");
  return launch_gemv(m, *lin, 0, k_dev, x_dev, y_dev, B, (hipStream_t)stream);
}

int dpllm_decode_step_parts(dpllm_model* m, const void* const* xs, void* const* ys, int32_t* k_dev, float* e_dev,
                            int parts, void* stream) {
  if (!m) return DPLLM_EINVAL;
  if (parts < 1 || parts > (DPLLM_STEP_SELECT | DPLLM_STEP_GEMV)) return fail(m, DPLLM_EINVAL, "bad parts %d", parts);
  if (!xs || !ys || !k_dev || !e_dev) return fail(m, DPLLM_EINVAL, "null pointer");
  if (!m->ws.base) return fail(m, DPLLM_ESTATE, "no workspace set");
  const int n = (int)m->linears.size();
  hipStream_t st = (hipStream_t)stream;
  StepPlan& P = m->plan;
  bool reuse = P.valid && P.version == m->version && P.k_dev == k_dev && P.e_dev == e_dev &&
               std::equal(xs, xs + n, P.xs.begin()) && std::equal(ys, ys + n, P.ys.begin());
  const bool in_capture = capturing(st);
  if ((!reuse || m->params_dirty) && in_capture)
    return fail(m, DPLLM_ESTATE, "the model changed since its last step: run one step outside stream capture first");
  if (!reuse) {
    for (int id = 0; id < n; ++id) {
      const Linear& lin = m->linears[id];
      if (!lin.loaded) return fail(m, DPLLM_ESTATE, "linear %d is not loaded", id);
      if (lin.active < 0) return fail(m, DPLLM_ESTATE, "linear %d has no selector", id);
      if (!xs[id] || !ys[id]) return fail(m, DPLLM_EINVAL, "null x or y for linear %d", id);
      if ((uintptr_t)xs[id] % 16) return fail(m, DPLLM_EINVAL, "x of linear %d not 16-byte aligned", id);
      if (overlap(xs[id], (size_t)lin.L.in * 2, ys[id], (size_t)lin.L.out * 2)) return fail(m, DPLLM_EINVAL, "x and y of linear %d overlap", id);
    }
    int rc = build_plan(m, xs, ys, k_dev, e_dev, st);
    if (rc != DPLLM_OK) return rc;
  }
  if (m->params_dirty) {
    int rc = upload_params(m, st);
    if (rc != DPLLM_OK) return rc;
  }
  const Workspace& W = m->ws;
  SelJob none{};
  SelParams pnone{};
  const SelParams* active = W.at<SelParams>(W.sel_active);
  const bool both = parts == (DPLLM_STEP_SELECT | DPLLM_STEP_GEMV);
  // a captured step is replayed under pairs and targets chosen later: it holds the selectors of every pair
  const bool all = P.idle && in_capture;
  P.captured |= in_capture;
  m->launches = 0;
  if (both && P.chain) {
    launch_chain(m, W, P, st);
    m->launches = 2;
    HIP_TRY(m, hipGetLastError());
    return DPLLM_OK;
  }
  if (both && P.fused && P.slots > 0) {   // the slots the fused launches collect start empty
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((P.slots * 2 + 255) / 256)), dim3(256), 0, st,
                       W.at<uint32_t>(W.sel_ws), P.slots * 2, (uint32_t)kSelEmpty);
    ++m->launches;
  }
  for (const Phase& ph : P.phases) {
    const bool decides = both && ph.decides && !P.chain, fused = both && ph.fused, estimators = ph.estimators || (all && ph.may_estimate);
    const SelJob* jobs = W.at<SelJob>(W.sel_jobs) + ph.sel_first;
    const SelPart* sel_parts = W.at<SelPart>(W.sel_parts) + ph.part_first;
    if ((parts & DPLLM_STEP_SELECT) && !fused && ph.sel_count > 0) {
      if (estimators)
        hipLaunchKernelGGL(selector_part_kernel, dim3(ph.part_count), dim3(kSelPartThreads), 0, st, jobs, sel_parts,
                           (const int32_t*)(W.at<int32_t>(W.sel_members) + ph.member_first), active, none, pnone);
      if (!decides)
        hipLaunchKernelGGL(selector_decide_kernel, dim3(ph.sel_count), dim3(kSelDecideThreads), 0, st, jobs, active, none, pnone);
      m->launches += estimators + !decides;
    }
    if (!(parts & DPLLM_STEP_GEMV)) continue;
    launch_step(ph.groups, ph.blocks, st, W.at<GemvJob>(W.gemv_jobs) + ph.gemv_first, W.at<int32_t>(W.block_jobs) + ph.block_first,
                decides ? active : nullptr, W.at<SelTask>(W.sel_tasks) + ph.task_first, fused && estimators ? ph.task_count : 0, m->polls);
    ++m->launches;
  }
  HIP_TRY(m, hipGetLastError());
  return DPLLM_OK;
}

int dpllm_decode_step(dpllm_model* m, const void* const* xs, void* const* ys, int32_t* k_dev, float* e_dev,
                      void* stream) {
  return dpllm_decode_step_parts(m, xs, ys, k_dev, e_dev, DPLLM_STEP_SELECT | DPLLM_STEP_GEMV, stream);
}

int dpllm_debug_unpack(dpllm_model* m, int id, int k, uint8_t* idx_dev, void* stream) {
  int rc = DPLLM_OK;
  Linear* lin = get_linear(m, id, &rc);
  if (!lin) return rc;
  if (!idx_dev) return fail(m, DPLLM_EINVAL, "null pointer");
  if (k < 1 || k > lin->L.p) return fail(m, DPLLM_ERANGE, "k=%d outside [1,%d]", k, lin->L.p);
  size_t n = (size_t)lin->L.out * lin->L.ncw;
  hipLaunchKernelGGL(debug_unpack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                     (const uint32_t*)lin->arena, lin->L.plane_bytes / 4, lin->L.p, k, lin->L.out, lin->L.ncw, lin->L.ncc, idx_dev);
  HIP_TRY(m, hipGetLastError());
  return DPLLM_OK;
}

int dpllm_debug_set_polls(dpllm_model* m, int polls) {
  if (!m) return DPLLM_EINVAL;
  if (polls < -1) return fail(m, DPLLM_EINVAL, "polls %d below -1", polls);
  m->polls = polls;
  return DPLLM_OK;
}

int dpllm_debug_set_one_launch(dpllm_model* m, int mode, int seats) {
  if (!m) return DPLLM_EINVAL;
  if (mode < -1 || mode > 1) return fail(m, DPLLM_EINVAL, "mode %d outside [-1,1]", mode);
  if (seats < 0) return fail(m, DPLLM_EINVAL, "seats %d below 0", seats);
  m->chain_mode = mode;
  m->chain_seats = seats;
  m->version++;
  return DPLLM_OK;
}

int dpllm_debug_step_launches(const dpllm_model* m, int* launches) {
  if (!m || !launches) return DPLLM_EINVAL;
  *launches = m->launches;
  return DPLLM_OK;
}

int dpllm_debug_copy(void* dst_dev, const void* src_dev, size_t bytes, void* stream) {
  if (!dst_dev || !src_dev || bytes % 16 || ((uintptr_t)dst_dev | (uintptr_t)src_dev) % 16) return DPLLM_EINVAL;
  hipLaunchKernelGGL(plain_copy_kernel, dim3(256 * 16), dim3(256), 0, (hipStream_t)stream, (const uint4*)src_dev,
                     (uint4*)dst_dev, bytes / 16);
  return hipGetLastError() == hipSuccess ? DPLLM_OK : DPLLM_EHIP;
}

int dpllm_debug_read(const void* src_dev, size_t bytes, void* sink_dev, void* stream) {
  if (!src_dev || !sink_dev || bytes % 16 || ((uintptr_t)src_dev | (uintptr_t)sink_dev) % 16) return DPLLM_EINVAL;
  hipLaunchKernelGGL(plain_read_kernel, dim3(256 * 8), dim3(256), 0, (hipStream_t)stream, (const uint4*)src_dev,
                     bytes / 16, (uint4*)sink_dev);
  return hipGetLastError() == hipSuccess ? DPLLM_OK : DPLLM_EHIP;
}

}  // extern "C"
