// A whole decode step whose levels depend on one another, in one launch: the workgroups stay from the first level to the
// last and hand the results of a level over to the next one themselves.
//
// What bounds a chained step is not the weights (a 7B block: 13 us at the rate of a plain read) but what a level waits for.
// With a launch per level that is the gap between launches 1.5 us, job and task records 0.8, products of the selector stored
// and seen 3, first planes and tables 2, and 192 or 344 workgroups on 256 compute units.  Here a wavefront asks for its next
// planes, also those of the next level, before it decodes the ones it has; records travel a level ahead; the tables of both
// bitwidths stand before the decision falls; and the rows of a level are dealt out in blocks of 64, 32 or 16, whichever ends
// first.  Measured inside (7B, k = 3 / 4, us after the last result of the level before): that result seen 1.2, products of the
// selector stored 1.9, seen and decided 3.5, first tile decoded 5; a level ends at 5 (o), 10 (q, k, v; down) and 16 (gate, up).
// us a step, a launch per level -> now, eager and in a graph: 7B, 32 blocks at 3 and 4 bits 1419 -> 1281 and 1420 -> 1283, with most
// selectors a level early 1381 -> 1206 and 1380 -> 1205, at 5 and 6 bits 1987 -> 1696 and 1989 -> 1700; 8B, 16 blocks at 5 and 6 bits,
// selectors early, 969 -> 842 and 970 -> 845.  Where 0.53 of the linears run at 4 bits and their weights are quantised Gaussians (bench.py's
// workload, in a graph) 1318 -> 1304, selectors early 1247 -> 1167, none 1060 -> 905: what a level waits for its selector is not less than
// with a launch per level, but weighs more.  What is left is that wait, and decode at two wavefronts per SIMD (an instruction in five
// cycles).
// Not served (chain_pays, plan_chain): few levels, whose start (number, first records: 8 us) weighs more; large levels, which the
// streaming kernel decodes with twice the wavefronts; columns that eight wavefronts cannot share evenly in chunks; high ranks.
// Tried and taken back: two workgroups per compute unit with 128 registers (spills; 1790 us), planes asked for two blocks
// ahead of tables that are built between two barriers (1560), table rows of the next level asked for before its tasks (no
// change), more copies of the results (no change), longer and shorter pauses between polls (no change).
//
// Hand-over.  A result that a later level reads goes into a mailbox as well as into the caller's buffer: four fp16 in a
// 64-bit word that is its own flag (kMailEmpty, two NaN that no writer stores, until the value is there).  Partial products of
// selectors travel through their slots in the same way (selector_kernels.hpp).  Both sides use relaxed atomics on that one
// word, so nothing rests on the order of two memory locations and no fence is needed (a device-scope release writes back the
// die's whole L2).  chain_reset_kernel empties both before the launch.
//
// Who takes part.  Every workgroup that starts takes a number.  A level is dealt out to the workgroups that have a number by the
// time somebody settles it (one compare-and-swap per level; everybody else reads how many they are): the first level when the last
// of the grid has started, or somebody has waited about 50 us for it, and from then on every level while the level before is being
// worked on, until all of the grid take part.  So every wait is for a workgroup that is running and works its levels off in order
// (tasks, then rows): the lowest level that is not finished is always one that its workgroups can finish, however many workgroups
// the chip has room for beside other work; and those that find a place later join at the next level.  us a chained 7B step beside
// work on another stream, median and worst, a launch per level / this launch with the workgroups of its first level only / now:
// copies of 1 GiB 2870, 3090 / 2360, 2390 / 2360, 2380; matrix products of 8192^3 (it waits for them to end) / 2600 .. 4700, 9600 / 2870,
// 3830; of 2048^3 2900, 3250 / 1540 .. 1700, 2060 / 1340, 1420.
//
// A workgroup is eight wavefronts, one workgroup to a compute unit (LDS), and up to 256 registers.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "gemv_lane.hpp"

namespace dpllm {

constexpr int kChainChunk = 512;           // columns: four tiles, what a wavefront parks at a time
constexpr int kChainGrid = 256;            // one workgroup per compute unit
constexpr int kChainLevelJobs = 56;        // linears of a level, at most
constexpr uint32_t kMailEmpty = 0xffffffffu;   // the low half of a mailbox word nobody has written
constexpr int kChainEnrolPolls = 64;       // of about a microsecond
constexpr int kChainLevelCounts = 32;      // state words: [0] workgroups that have started, [32 + l] how many level l is dealt out to

// One level: 64 dwords, which a wavefront holds in one register (lane i = dword i) and reads with v_readlane.
struct ChainLevel {
  int32_t job_first, job_count;            // linears job_first .. + job_count
  int32_t units;                           // blocks of 64 >> log_groups rows
  int32_t task_first, task_count;          // selector tasks: of this level's linears, and of the next one's whose vector is there by now
  int32_t log_groups;                      // column groups of a wavefront: 1, 2 or 4
  int32_t unused[2];                       // (unit_start begins at lane 8)
  int32_t unit_start[kChainLevelJobs];     // first block of every linear; 0x7fffffff past the last one
};
static_assert(sizeof(ChainLevel) == 256, "one dword per lane");

// One linear: 32 dwords, read the same way, in a register with the 16 of its selector parameters.
struct alignas(64) ChainJob {
  const char* arena;
  const uint16_t* x;                       // the vector, or its place in the mailbox of the linear that writes it
  uint16_t* y;
  uint64_t* mail;                          // nullptr: no later level reads the result
  const uint64_t* slots;                   // [kSelCopies][nchunks][slot_rows] partial products of the selector
  float* e_out;
  int32_t* k_out;
  uint32_t plane_bytes;
  int32_t x_handed;                        // x lies in a mailbox; 0: the caller's buffer, always there
  int32_t out, ncw, ncc;
  int32_t slot_rows, nchunks;
  uint32_t lut_off[kKMax];
};
static_assert(sizeof(ChainJob) == 128 && sizeof(SelParams) == 64, "dwords of a job record");
#define DPLLM_CJ(field) (int)(offsetof(ChainJob, field) / 4)
#define DPLLM_CP(field) (int)(32 + offsetof(SelParams, field) / 4)
#define DPLLM_CL(field) (int)(offsetof(ChainLevel, field) / 4)
#define DPLLM_CT(field) (int)(offsetof(SelTask, field) / 4)

__device__ __forceinline__ uint32_t rec_u32(uint32_t rec, int i) { return (uint32_t)__builtin_amdgcn_readlane((int)rec, i); }
template <class T>
__device__ __forceinline__ T* rec_ptr(uint32_t rec, int i) {
  return reinterpret_cast<T*>((uint64_t)rec_u32(rec, i + 1) << 32 | rec_u32(rec, i));
}

__device__ __forceinline__ uint64_t mail_load(const DPLLM_GLOBAL uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Empties slots and mailboxes; no workgroup has started and no level is settled.
__global__ void __launch_bounds__(256) chain_reset_kernel(uint64_t* slots, size_t nslots, uint64_t* mail, size_t nmail, uint32_t* state, size_t nstate) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, n = (size_t)gridDim.x * 256;
  for (size_t j = i; j < nslots; j += n) slots[j] = kSelEmpty;
  for (size_t j = i; j < nmail; j += n) mail[j] = ~0ull;
  for (size_t j = i; j < nstate; j += n) state[j] = 0;
}

// How many workgroups level `level` is dealt out to: as many as have started by now, unless it is settled.  most: 0 for no bound.
__device__ __forceinline__ int chain_settle(DPLLM_GLOBAL uint32_t* state, int level, int most) {
  DPLLM_GLOBAL uint32_t* at = state + kChainLevelCounts + level;
  uint32_t count = __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (count != 0) return (int)count;
  uint32_t started = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (most > 0) started = min(started, (uint32_t)most);
  return (int)(__hip_atomic_compare_exchange_strong(at, &count, started, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? started : count);
}

// Thread 0 of a workgroup: its number, the first level it takes part in and how many that one is dealt out to; number < 0: none.
__device__ __forceinline__ void chain_enrol(DPLLM_GLOBAL uint32_t* state, int grid, int seats, int nlevels, int patience, int& number, int& level, int& count) {
  const DPLLM_GLOBAL uint32_t* counts = state + kChainLevelCounts;
  number = (int)__hip_atomic_fetch_add(state, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  level = 0;
  count = number + 1 == grid ? chain_settle(state, 0, seats) : 0;
  for (int left = kChainEnrolPolls; count == 0; --left) {
    count = left > 0 ? (int)__hip_atomic_load(counts, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : chain_settle(state, 0, seats);
    if (count == 0) __builtin_amdgcn_s_sleep(2);
  }
  // not among them: a later level.  While fewer than the grid take part, those that do settle every level, so this ends
  while (number >= count) {
    if (++level == nlevels || patience < 0) {
      number = -1;
      return;
    }
    while ((count = (int)__hip_atomic_load(counts + level, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0 && --patience >= 0) __builtin_amdgcn_s_sleep(8);
  }
}

// Where the planes of one step (as many column tiles as column groups) of a wavefront lie, nb of them: all offsets are 32-bit
// bytes from the arena (plan_chain sees to that), so that a load takes one addition and no 64-bit arithmetic.
struct ChainAt {
  const char* arena;
  uint32_t plane, at;                      // from one plane to the next; the lane's part of plane 0
  int nb;
};
// the first step of chunk `chunk` of block `block`
__device__ __forceinline__ ChainAt chain_at(uint32_t rec, int log_groups, int block, int chunk, int nb, int lane) {
  const int ncc = (int)rec_u32(rec, DPLLM_CJ(ncc)), rows = 64 >> log_groups;
  const uint32_t at = (uint32_t)min(4 * chunk + (lane >> (6 - log_groups)), ncc - 1) * 1024u + (uint32_t)(lane & (rows - 1)) * 16u +
                      (uint32_t)(block >> log_groups) * ncc * 1024u + (uint32_t)(block & ((1 << log_groups) - 1)) * rows * 16u;
  return {rec_ptr<const char>(rec, DPLLM_CJ(arena)), rec_u32(rec, DPLLM_CJ(plane_bytes)), at, nb};
}
// Asks for them.  Loads are never predicated (registers that are loaded on one of two ways are copied where the ways meet, and
// the copy waits for the load): past nb plane 0 is read once more, out of the vector cache.
template <int H>
__device__ __forceinline__ void chain_load_planes(u32x4 (&T)[H], const ChainAt& p) {
#pragma unroll
  for (int b = 0; b < H; ++b)
    T[b] = load_stream(reinterpret_cast<const DPLLM_GLOBAL u32x4*>(as_global(p.arena) + (p.at + (b < p.nb ? (uint32_t)b * p.plane : 0u))));
}

// the lane's eight columns of a vector from column c on (clamped: n is a multiple of 32)
__device__ __forceinline__ u32x4 chain_load_x(const DPLLM_GLOBAL uint64_t* x, int c, int n) {
  const DPLLM_GLOBAL uint64_t* p = x + (min(c, n - 8) >> 2);
  const uint64_t a = mail_load(p), b = mail_load(p + 1);
  return u32x4{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
}
__device__ __forceinline__ bool chain_here(const u32x4& v) { return v.x != kMailEmpty && v.z != kMailEmpty; }

// The estimate and the decision of a linear from its selector's slots (kind 1: the squares of the rows' products; kind 2:
// row 0 holds the sum of squares), by the whole workgroup; a barrier for what it has in LDS as well.  sh: as in selector_gather.
// look: the wavefront's first batch, asked for earlier (chain_look).
constexpr int kChainBatch = 4;
struct ChainSlots {
  const DPLLM_GLOBAL uint64_t* at;
  int nchunks, rows, r;                    // r: rows that count
};
__device__ __forceinline__ ChainSlots chain_slots(uint32_t rec, int number) {
  const int nchunks = (int)rec_u32(rec, DPLLM_CJ(nchunks)), rows = (int)rec_u32(rec, DPLLM_CJ(slot_rows));
  return {as_global(rec_ptr<const uint64_t>(rec, DPLLM_CJ(slots))) + (size_t)(number & (kSelCopies - 1)) * nchunks * rows, nchunks, rows,
          (int)rec_u32(rec, DPLLM_CP(kind)) == 1 ? (int)rec_u32(rec, DPLLM_CP(r)) : 1};
}
__device__ __forceinline__ void chain_look(const ChainSlots& s, int t, int c0, uint64_t (&v)[kChainBatch]) {
#pragma unroll
  for (int i = 0; i < kChainBatch; ++i) v[i] = mail_load(s.at + (size_t)min(c0 + i, s.nchunks - 1) * s.rows + min(t, s.r - 1));
}
__device__ __forceinline__ int chain_decide(uint32_t rec, const ChainSlots& s, const uint64_t (&look)[kChainBatch], int& patience, int tid, double* sh, bool write) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int kind = (int)rec_u32(rec, DPLLM_CP(kind));
  double e = 0.0;
  if (kind != 0) {
    double part = 0.0;
    for (int t0 = wave * 64; t0 < s.r; t0 += kLaneThreads) {
      double g = 0.0;
      for (int c0 = 0; c0 < s.nchunks; c0 += kChainBatch) {
        uint64_t v[kChainBatch];
#pragma unroll
        for (int i = 0; i < kChainBatch; ++i) v[i] = look[i];
        bool again = t0 >= kLaneThreads || c0 > 0;
        for (;;) {
          if (again) chain_look(s, t0 + lane, c0, v);
          bool all = true;
#pragma unroll
          for (int i = 0; i < kChainBatch; ++i) all = all && v[i] != kSelEmpty;
          if (__all(all) || --patience < 0) break;
          if (again) __builtin_amdgcn_s_sleep(1);
          again = true;
        }
#pragma unroll
        for (int i = 0; i < kChainBatch; ++i)
          if (c0 + i < s.nchunks) g += __builtin_bit_cast(double, v[i]);
      }
      part += t0 + lane >= s.r ? 0.0 : kind == 1 ? g * g : g;
    }
    part = wave_sum_f64(part);
    if (lane == 0) sh[16 + wave] = part;
    lds_barrier();
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kLaneWaves; ++w) sum += sh[16 + w];
    e = sqrt(sum);
    if (kind == 2) {
      const float alpha = __builtin_bit_cast(float, rec_u32(rec, DPLLM_CP(alpha))), beta = __builtin_bit_cast(float, rec_u32(rec, DPLLM_CP(beta)));
      e = (double)alpha * e + (double)beta;
    }
  } else {
    lds_barrier();
  }
  const float T = __builtin_bit_cast(float, rec_u32(rec, DPLLM_CP(T)));
  const int k = (int)rec_u32(rec, kind != 0 && e > (double)T ? DPLLM_CP(h) : DPLLM_CP(l));
  if (write && tid == 0) {
    *as_global(rec_ptr<float>(rec, DPLLM_CJ(e_out))) = (float)e;
    *as_global(rec_ptr<int32_t>(rec, DPLLM_CJ(k_out))) = k;
  }
  return __builtin_amdgcn_readfirstlane(k);
}

// One selector task (a slice of at most 4096 columns), by the whole workgroup: g = the lane's eight columns of the row of G
// (asked for before).  G at x itself: the sum of squares (linear regression).  v: the lane's columns of x.
__device__ __forceinline__ sel_u32x4 chain_task_g(uint32_t rec, int wave, int lane) {
  const uint16_t* g = rec_ptr<const uint16_t>(rec, DPLLM_CT(g));
  sel_u32x4 v = {0u, 0u, 0u, 0u};
  const int cols = (int)rec_u32(rec, DPLLM_CT(cols));
  if (g != nullptr && g != rec_ptr<const uint16_t>(rec, DPLLM_CT(x)) && wave * kSelChunkStep < cols)
    v = __builtin_nontemporal_load((const DPLLM_SEL_GLOBAL sel_u32x4*)(g + min(wave * kSelChunkStep + lane * 8, cols - 8)));
  return v;
}
__device__ __forceinline__ void chain_task(uint32_t rec, sel_u32x4 g, int& patience, int tid, double* sh, int& turn, u32x4& v) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const uint16_t* gp = rec_ptr<const uint16_t>(rec, DPLLM_CT(g));
  if (gp == nullptr) return;
  const uint16_t* xp = rec_ptr<const uint16_t>(rec, DPLLM_CT(x));
  const int cols = (int)rec_u32(rec, DPLLM_CT(cols)), handed = (int)rec_u32(rec, DPLLM_CT(x_handed));
  double acc = 0.0;
  if (wave * kSelChunkStep < cols) {
    const DPLLM_GLOBAL uint64_t* x = as_global(reinterpret_cast<const uint64_t*>(xp));
    const int c = wave * kSelChunkStep + lane * 8;
    for (;;) {
      v = chain_load_x(x, c, cols);
      if (handed == 0 || __all(chain_here(v)) || --patience < 0) break;
      __builtin_amdgcn_s_sleep(1);
    }
    const sel_u32x4 xv = v, gv = gp == xp ? xv : g;
    if (c < cols) {
      const __half* gh = reinterpret_cast<const __half*>(&gv);
      const __half* xh = reinterpret_cast<const __half*>(&xv);
#pragma unroll
      for (int i = 0; i < 8; ++i) acc = fma((double)__half2float(gh[i]), (double)__half2float(xh[i]), acc);
    }
  }
  acc = wave_sum_f64(acc);
  if (lane == 0) sh[turn + wave] = acc;
  lds_barrier();
  if (tid < kSelCopies) {
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < 8; ++w) sum += sh[turn + w];
    DPLLM_GLOBAL uint64_t* slot = as_global(rec_ptr<uint64_t>(rec, DPLLM_CT(slot)));
    __hip_atomic_store(slot + (size_t)tid * rec_u32(rec, DPLLM_CT(copy_stride)), __builtin_bit_cast(uint64_t, sel_storable(sum)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  turn ^= 8;
}

// LDS: two tables and the partial sums of two blocks (one is worked on, the other one's table is being built or its sums are
// being added up), activation slots, shared words
constexpr int kChainRedOffset = 2 * kLaneTableBytes;
constexpr int kChainXOffset = kChainRedOffset + 2 * kLaneRedBytes;
constexpr int kChainXBytes = 4 * kLaneGroupStride;   // per wavefront: the four tiles of a chunk
constexpr int kChainLdsBytes = kChainXOffset + kLaneWaves * kChainXBytes + kSelSharedBytes;
static_assert(kChainLdsBytes <= 163840, "LDS of a compute unit");

// The sums of a block's rows, by one wavefront: to the caller's buffer, and to the mailbox if a later level reads them.
template <int G>
__device__ __forceinline__ void chain_store(uint32_t rec, int block, int buffer, int lane, const char* lds) {
  const float* red = reinterpret_cast<const float*>(lds + kChainRedOffset + buffer * kLaneRedBytes);
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < kLaneWaves; ++w) s += red[w * 64 + lane];
  constexpr int rows = 64 / G;
  if constexpr (G > 1) s = sum_groups<G>(s);   // row lane mod `rows`, in every lane
  const uint32_t bits = __builtin_bit_cast(uint16_t, (_Float16)s);
  const int row = block * rows + lane % rows;
  const bool inside = row < (int)rec_u32(rec, DPLLM_CJ(out));
  uint64_t* mail = rec_ptr<uint64_t>(rec, DPLLM_CJ(mail));
  if (mail != nullptr) {
    // lane 4 q stores rows 4 q .. + 3
    const int v = !inside ? 0 : bits == 0xffffu ? 0xfe00 : (int)bits;
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_update_dpp(0, v, 0x00, 0xf, 0xf, true), r1 = (uint32_t)__builtin_amdgcn_update_dpp(0, v, 0x55, 0xf, 0xf, true);
    const uint32_t r2 = (uint32_t)__builtin_amdgcn_update_dpp(0, v, 0xaa, 0xf, 0xf, true), r3 = (uint32_t)__builtin_amdgcn_update_dpp(0, v, 0xff, 0xf, 0xf, true);
    if (lane < rows && (lane & 3) == 0)
      __hip_atomic_store(as_global(mail) + row / 4,
                         (uint64_t)(r2 | r3 << 16) << 32 | (r0 | r1 << 16), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (lane < rows && inside) as_global(rec_ptr<uint16_t>(rec, DPLLM_CJ(y)))[row] = (uint16_t)bits;
}

// The tables of the rows of a block (row: the lane's) at lo and hi bits, in buffers 0 and 1.  Neighbouring bitwidths are asked for
// together.
template <int H>
__device__ __forceinline__ void chain_tables(uint32_t rec, int lo, int hi, int row, int wave, int lane, char* lds) {
  const char* arena = rec_ptr<const char>(rec, DPLLM_CJ(arena));
  auto lut = [&](int bits) { return as_global(reinterpret_cast<const uint16_t*>(arena + rec_u32(rec, DPLLM_CJ(lut_off) + bits - 1))); };
  const uint32_t mine = (uint32_t)lane * 4;
  const bool pair = hi == lo + 1;
  auto build = [&](auto kc, uint32_t lanecol, bool both) {
    constexpr int K = decltype(kc)::value, K1 = K < H ? K + 1 : K;
    if constexpr (K <= H) {
      LaneLut<K> L;
      lane_fetch_lut<K>(L, lut(K), row, wave);
      if (both) {
        LaneLut<K1> L1;
        lane_fetch_lut<K1>(L1, lut(K1), row, wave);
        lane_build_table<K>(L, wave, lanecol, lds);
        lane_build_table<K1>(L1, wave, mine + kLaneTableBytes, lds);
      } else {
        lane_build_table<K>(L, wave, lanecol, lds);
      }
    }
  };
  auto at = [&](int bits, uint32_t lanecol, bool both) {
    switch (bits) {
      case 1: build(std::integral_constant<int, 1>{}, lanecol, both); break;
      case 2: build(std::integral_constant<int, 2>{}, lanecol, both); break;
      case 3: build(std::integral_constant<int, 3>{}, lanecol, both); break;
      case 4: build(std::integral_constant<int, 4>{}, lanecol, both); break;
      case 5: build(std::integral_constant<int, 5>{}, lanecol, both); break;
      case 6: build(std::integral_constant<int, 6>{}, lanecol, both); break;
      case 7: build(std::integral_constant<int, 7>{}, lanecol, both); break;
      default: build(std::integral_constant<int, 8>{}, lanecol, both); break;
    }
  };
  at(lo, mine, pair);
  if (hi != lo && !pair) at(hi, mine + kLaneTableBytes, false);
}

// The blocks [block, block + blocks) of a linear at K bits, 64 / G rows each, in the wavefront's chunks [c0, c1) of the columns (at
// most one unless MULTI).  T holds the planes of the first step, x the lane's columns of chunk c0; the table of the first block
// stands in `buffer`.  What comes next (the following step or block, or `next` behind the run) is asked for as soon as its
// registers are free, and the next block's table is built while this one is decoded.
template <int K, int H, int G, bool MULTI>
__device__ __forceinline__ void chain_run(u32x4 (&T)[H], uint32_t rec, int block, int blocks, u32x4 x, const DPLLM_GLOBAL uint64_t* xw,
                                          int c0, int c1, int buffer, const ChainAt& next, int tid, char* lds) {
  constexpr int S = 4 / G, rows = 64 / G;   // steps of a chunk
  constexpr int kLog = G == 1 ? 0 : G == 2 ? 1 : 2;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, group = lane / rows;
  const int ncw = (int)rec_u32(rec, DPLLM_CJ(ncw)), ncc = (int)rec_u32(rec, DPLLM_CJ(ncc)), n = (c1 - c0) * S;
  char* ready = lds + kChainXOffset + wave * kChainXBytes;
  const char* xmine = ready + group * kLaneGroupStride + (lane & 3) * 16;
  const char* arena = rec_ptr<const char>(rec, DPLLM_CJ(arena));
  const uint32_t plane = rec_u32(rec, DPLLM_CJ(plane_bytes));
  const DPLLM_GLOBAL char* lut = as_global(arena + rec_u32(rec, DPLLM_CJ(lut_off) + K - 1));
  const int last = block + blocks - 1, tile0 = 4 * c0 + group, in_block = lane % rows;
  auto park = [&](int chunk) {
    const uint32_t v[4] = {x.x, x.y, x.z, x.w};
    narrow_park<K, 4>(v, chunk * kChainChunk + lane * 8 < ncw * 32, lane, ready);
  };
  LaneLut<K> L;                            // the wavefront's part of the next block's table rows
  auto fetch_lut = [&](int b) {
    lane_fetch_lut_at<K>(L, lut + ((uint32_t)(b * rows + in_block) << (K + 1)), wave);
  };
  fetch_lut(min(block + 1, last));
  // behind step q of block b
  auto ask = [&](u32x4 (&t)[H], int b, int q) {
    const bool inner = q + 1 < n, again = inner || b < last;
    if (!inner && b < last) lane_build_table<K>(L, wave, (uint32_t)lane * 4 + (uint32_t)(buffer ^ 1) * kLaneTableBytes, lds);
    const int nb = inner ? b : b + 1, nq = inner ? q + 1 : 0;
    if constexpr (MULTI) {                 // the chunk behind this one
      const int chunk = c0 + q / S + 1;
      x = chain_load_x(xw, (chunk < c1 ? chunk : c0) * kChainChunk + lane * 8, ncw * 32);
    }
    fetch_lut(min(nb + 1, last));
    const uint32_t at = (uint32_t)min(tile0 + nq * G, ncc - 1) * 1024u + (uint32_t)in_block * 16u + ((uint32_t)(nb >> kLog) * ncc * 1024u + (uint32_t)(nb & (G - 1)) * rows * 16u);
    chain_load_planes<H>(t, ChainAt{again ? arena : +next.arena, again ? +plane : +next.plane, again ? +at : +next.at, again ? (n > 0 ? K : 0) : +next.nb});
  };
  LaneMasks<K> M;
  if constexpr (K <= 6) M.init();
  const uint32_t mask = LaneDecode<K>::pair ? LaneDecode<K>::pair_mask : 0;
  const bool short_row = 4 * c1 > ncc;     // some lanes have no tile in the last step or steps: they decode another one and drop it
  for (int b = block; b <= last; ++b) {
    const uint32_t lanecol = (uint32_t)lane * 4 + (uint32_t)buffer * kLaneTableBytes;
    float* red = reinterpret_cast<float*>(lds + kChainRedOffset + buffer * kLaneRedBytes);
    if (!MULTI && b == block && n > 0) park(c0);
    LaneAcc<1> acc;
    acc.zero();
    float sum = 0.f;
    uint32_t addr[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) addr[i] = lanecol;
#pragma unroll 1
    for (int q = 0; q < n; ++q) {
      if (MULTI && q % S == 0) park(c0 + q / S);
      const int tile = 4 * c0 + q * G;
      LaneX<K, 1, G> xs;
      xs.mine = xmine + q % S * G * kLaneGroupStride;
      lane_compute<K, 1, G, true, false>(T, lanecol, lds, xs, acc, addr, mask, M, ncw - (tile + group) * 4, (tile + G) * 4 > ncw,
                                  [&](u32x4 (&t)[H]) { ask(t, b, q); });
      acc.settle();
      if (short_row && tile + group < ncc) sum = acc.sum(0);
    }
    if (n <= 0) ask(T, b, 0);
    red[wave * 64 + lane] = short_row ? sum : acc.sum(0);
    lds_barrier();
    if (wave == (b & (kLaneWaves - 1))) chain_store<G>(rec, b, buffer, lane, lds);
    buffer ^= 1;
  }
}

// The levels of a step from `first` on.  H: the largest bitwidth of the active pairs, rounded up to 4, 6 or 8 (registers of the
// planes asked for ahead); number, first, count: as chain_enrol gives them.
template <int H>
__device__ __forceinline__ void chain_levels(const ChainLevel* levels, const ChainJob* jobs, const SelParams* active, const SelTask* tasks, DPLLM_GLOBAL uint32_t* state,
                                             int nlevels, int patience, int number, int first, int count, int tid, char* lds) {
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int lane = tid & 63;
  double* sh = reinterpret_cast<double*>(lds + kChainLdsBytes - kSelSharedBytes);
  auto load_level = [&](int l) { return as_global(reinterpret_cast<const uint32_t*>(levels + min(l, nlevels)))[lane]; };   // (the one behind the last is empty)
  auto load_job = [&](int j) {
    const uint32_t* p = lane < 32 ? reinterpret_cast<const uint32_t*>(jobs + j) + lane : reinterpret_cast<const uint32_t*>(active + j) + (lane & 15);
    return *as_global(p);
  };
  auto load_task = [&](int t) { return as_global(reinterpret_cast<const uint32_t*>(tasks + t))[lane & 15]; };
  // this workgroup's blocks [u0, u1) of a level that is dealt out to `count`; units / count as a product: exact for fewer than
  // 2^24 units (count <= 256)
  auto inverse = [](int count) { return count > 1 ? 0xffffffffu / (uint32_t)count + 1 : 0; };
  uint32_t per_count = inverse(count), per_count1 = per_count;   // of this level, of the next one
  auto share = [&](uint32_t lev, int count, uint32_t per_count, int& u0, int& u1) {
    const int units = (int)rec_u32(lev, DPLLM_CL(units)), base = count > 1 ? (int)__umulhi((uint32_t)units, per_count) : units, extra = units - base * count;
    u0 = number * base + min(number, extra);
    u1 = u0 + base + (number < extra ? 1 : 0);
  };
  // which linear of the level block u belongs to, as its block number `block`; its last one is end - 1
  auto job_of = [&](uint32_t lev, int u, int& block, int& end) {
    const int j = __popcll(__ballot(lane >= 8 && (int)lev <= u)) - 1;
    block = u - (int)rec_u32(lev, 8 + j);
    end = j + 1 < kChainLevelJobs ? (int)rec_u32(lev, 8 + min(j + 1, kChainLevelJobs - 1)) : 0x7fffffff;
    return (int)rec_u32(lev, DPLLM_CL(job_first)) + j;
  };
  auto steps = [&](uint32_t rec, int& c0, int& c1) {
    const int chunks = ((int)rec_u32(rec, DPLLM_CJ(ncc)) + 3) / 4;
    c0 = wave * chunks / kLaneWaves;
    c1 = (wave + 1) * chunks / kLaneWaves;
  };
  uint32_t lev = load_level(first), lev1 = load_level(first + 1);
  uint32_t trec = 0;
  sel_u32x4 tg = {0u, 0u, 0u, 0u};
  // tasks go to the workgroups that have the fewest rows first; this workgroup's first one of a level (without one: any, unused)
  auto task_of = [&](uint32_t lev, int count) {
    const int mirror = count - 1 - number;
    return mirror < (int)rec_u32(lev, DPLLM_CL(task_count)) ? (int)rec_u32(lev, DPLLM_CL(task_first)) + mirror : 0;
  };
  bool task_here = count - 1 - number < (int)rec_u32(lev, DPLLM_CL(task_count));
  if (task_here) {
    trec = load_task(task_of(lev, count));
    tg = chain_task_g(trec, wave, lane);
  }
  u32x4 T[H];
#pragma unroll
  for (int b = 0; b < H; ++b) T[b] = u32x4{0u, 0u, 0u, 0u};
  uint32_t rec = 0;                        // the linear T's planes belong to
  int block = 0, end = 0, c0 = 0, c1 = 0;  // its block, the end of its blocks in its level, the wavefront's chunks of its columns
  auto first_rows = [&](uint32_t lev, int u) {
    rec = load_job(job_of(lev, u, block, end));
    steps(rec, c0, c1);
    chain_load_planes<H>(T, chain_at(rec, (int)rec_u32(lev, DPLLM_CL(log_groups)), block, c0, c0 < c1 ? (int)rec_u32(rec, DPLLM_CP(h)) : 0, lane));
  };
  {
    int u0, u1;
    share(lev, count, per_count, u0, u1);
    if (u0 < u1) first_rows(lev, u0);
  }
  int turn = 0;
  for (int l = first; l < nlevels; ++l) {
    // how many the next level is dealt out to (a workgroup that has joined stays: all of the grid do from some level on)
    int count1 = count;
    if (count < (int)gridDim.x && l + 1 < nlevels) {
      int* word = reinterpret_cast<int*>(lds + kChainLdsBytes) - 1;
      if (tid == 0) *word = chain_settle(state, l + 1, 0);
      lds_barrier();
      count1 = __builtin_amdgcn_readfirstlane(*word);
      lds_barrier();
      per_count1 = inverse(count1);
    }
    // records of the levels behind this one
    uint32_t lev2 = load_level(l + 2), trec1 = load_task(task_of(lev1, count1));
    const bool task1 = count1 - 1 - number < (int)rec_u32(lev1, DPLLM_CL(task_count));
    int u0, u1, n0, n1;
    share(lev, count, per_count, u0, u1);
    share(lev1, count1, per_count1, n0, n1);
    u32x4 task_x = {0u, 0u, 0u, 0u};       // the vector of the workgroup's first task, if it is one slice, and where it lies
    const uint16_t* task_at = nullptr;
    int task_cols = 0;
    if (task_here) {
      chain_task(trec, tg, patience, tid, sh, turn, task_x);
      if (rec_ptr<const uint16_t>(trec, DPLLM_CT(g)) != nullptr) task_at = rec_ptr<const uint16_t>(trec, DPLLM_CT(x));
      task_cols = (int)rec_u32(trec, DPLLM_CT(cols));
      const int tasks_here = (int)rec_u32(lev, DPLLM_CL(task_count)), first_task = (int)rec_u32(lev, DPLLM_CL(task_first));
      for (int t = 2 * count - 1 - number; t < tasks_here; t += count) {
        const uint32_t r = load_task(first_task + t);
        u32x4 unused = task_x;
        chain_task(r, chain_task_g(r, wave, lane), patience, tid, sh, turn, unused);
      }
    }
    const int lg = (int)rec_u32(lev, DPLLM_CL(log_groups)), lg1 = (int)rec_u32(lev1, DPLLM_CL(log_groups));
    for (int u = u0; u < u1;) {            // run by run of blocks of one linear
      asm volatile("" : "+v"(tid), "+v"(lane));   // what is worked out from them is worked out again, not kept in registers
      const int blocks = min(u1, end) - u;
      // a look at the vector and at the products of the selector, the tables of both bitwidths
      const int lo = (int)rec_u32(rec, DPLLM_CP(l)), hi = (int)rec_u32(rec, DPLLM_CP(h)), row = block * (64 >> lg) + (lane & ((64 >> lg) - 1));
      const int x_handed = (int)rec_u32(rec, DPLLM_CJ(x_handed)), in = (int)rec_u32(rec, DPLLM_CJ(ncw)) * 32;
      const uint16_t* xp = rec_ptr<const uint16_t>(rec, DPLLM_CJ(x));
      const DPLLM_GLOBAL uint64_t* xw = as_global(reinterpret_cast<const uint64_t*>(xp));
      const int c = c0 * kChainChunk + lane * 8;
      const u32x4 x_look = chain_load_x(xw, c, in);
      const ChainSlots slots = chain_slots(rec, number);
      uint64_t look[kChainBatch] = {};
      if (wave * 64 < slots.r) chain_look(slots, wave * 64 + lane, 0, look);
      // what comes next: another linear of the level, or the first block of the next level
      const bool same_level = u + blocks < u1, any_next = same_level || n0 < n1;
      int next_block = 0, next_end = 0;
      uint32_t next_rec = load_job(any_next ? job_of(same_level ? lev : lev1, same_level ? u + blocks : n0, next_block, next_end) : 0);
      chain_tables<H>(rec, lo, hi, row, wave, lane, lds);
      // the vector
      const bool have_x = c0 >= c1 || (xp == task_at && task_cols == in && c0 == wave && c1 == wave + 1);
      u32x4 x = have_x ? task_x : x_look;
      if (!have_x && (c1 - c0 > 1 || (x_handed != 0 && !__all(chain_here(x))))) {
        for (;;) {
          x = chain_load_x(xw, c, in);
          bool here = chain_here(x);
          for (int sc = c0 + 1; sc < c1 && x_handed != 0; sc += 2) {
            const u32x4 p = chain_load_x(xw, c + (sc - c0) * kChainChunk, in), q = chain_load_x(xw, c + (min(sc + 1, c1 - 1) - c0) * kChainChunk, in);
            here = here && chain_here(p) && chain_here(q);
          }
          if (x_handed == 0 || __all(here) || --patience < 0) break;
          __builtin_amdgcn_s_sleep(1);
        }
      }
      // what was asked for on the way is waited for here, where there is nothing else in flight, not behind the planes and stores
      // to come
      asm volatile("" : "+v"(next_rec), "+v"(lev2), "+v"(trec1));
      int nc0, nc1;
      steps(next_rec, nc0, nc1);
      const ChainAt next = chain_at(next_rec, same_level ? lg : lg1, next_block, nc0, any_next && nc0 < nc1 ? (int)rec_u32(next_rec, DPLLM_CP(h)) : 0, lane);
      const int k = chain_decide(rec, slots, look, patience, tid, sh, block == 0);
      auto run = [&](auto kc) {
        constexpr int K = decltype(kc)::value;
        if constexpr (K <= H) {
          auto go = [&](auto gc) {
            constexpr int G = decltype(gc)::value;
            if (in <= kChainChunk * kLaneWaves) chain_run<K, H, G, false>(T, rec, block, blocks, x, xw, c0, c1, k != lo, next, tid, lds);
            else chain_run<K, H, G, true>(T, rec, block, blocks, x, xw, c0, c1, k != lo, next, tid, lds);
          };
          if (lg == 0) go(std::integral_constant<int, 1>{});
          else if (lg == 1) go(std::integral_constant<int, 2>{});
          else go(std::integral_constant<int, 4>{});
        }
      };
      switch (k) {
        case 1: run(std::integral_constant<int, 1>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        case 7: run(std::integral_constant<int, 7>{}); break;
        default: run(std::integral_constant<int, 8>{}); break;
      }
      rec = next_rec;
      block = next_block;
      end = next_end;
      c0 = nc0;
      c1 = nc1;
      u += blocks;
    }
    // no rows here: the first ones of the next level are asked for now
    if (u0 >= u1) {
      asm volatile("" : "+v"(lev2), "+v"(trec1));
      if (n0 < n1) first_rows(lev1, n0);
    }
    task_here = task1;
    trec = trec1;
    if (task1) tg = chain_task_g(trec, wave, lane);
    lev = lev1;
    lev1 = lev2;
    count = count1;
    per_count = per_count1;
  }
  // cannot be, by what chain_enrol promises; if it is, a bitwidth says so
  if (patience < 0 && lane == 0) {
    const uint32_t* p = reinterpret_cast<const uint32_t*>(jobs);
    *as_global(reinterpret_cast<int32_t*>((uint64_t)p[DPLLM_CJ(k_out) + 1] << 32 | p[DPLLM_CJ(k_out)])) = -1;
  }
}

// The active pairs say on the device how many planes are asked for ahead, whatever other pairs a linear holds: every plane beyond
// those of a step is a load for nothing in each row block.  7B, 32 blocks at 3 and 4 bits, us a step with pairs of up to 8 bits
// attached as well: 1485 with a kernel for the largest attached pair, 1310 with the active ones' (1338 with a launch per level).
// The pairs are read while thread 0 enrols the workgroup.  All three variants have the registers and the LDS of the
// largest; one workgroup fills a compute unit either way.
__global__ void __launch_bounds__(kLaneThreads, 2) gemv_chain_kernel(const ChainLevel* levels, const ChainJob* jobs, const SelParams* active, const SelTask* tasks,
                                                                     uint32_t* state, int nlevels, int njobs, int patience, int seats) {
  __shared__ __attribute__((aligned(256))) char lds[kChainLdsBytes];
  if ((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds != 0u) return;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int* seat = reinterpret_cast<int*>(lds + kChainLdsBytes - kSelSharedBytes);   // number, first level, count, largest bitwidth class of every wavefront
  int h = 0;
  for (int j = tid; j < njobs; j += kLaneThreads) h = max(h, *as_global(&active[j].h));
  if (tid == 0) {
    chain_enrol((DPLLM_GLOBAL uint32_t*)state, (int)gridDim.x, seats, nlevels, patience, seat[0], seat[1], seat[2]);
  }
  const int mine = __any(h > 6) ? 2 : __any(h > 4) ? 1 : 0;
  if ((tid & 63) == 0) seat[3 + wave] = mine;
  lds_barrier();
  const int number = __builtin_amdgcn_readfirstlane(seat[0]), first = __builtin_amdgcn_readfirstlane(seat[1]), count = __builtin_amdgcn_readfirstlane(seat[2]);
  int size = 0;
#pragma unroll
  for (int w = 0; w < kLaneWaves; ++w) size = max(size, seat[3 + w]);
  size = __builtin_amdgcn_readfirstlane(size);
  lds_barrier();
  if (number < 0) return;
  if (size == 0) chain_levels<4>(levels, jobs, active, tasks, (DPLLM_GLOBAL uint32_t*)state, nlevels, patience, number, first, count, tid, lds);
  else if (size == 1) chain_levels<6>(levels, jobs, active, tasks, (DPLLM_GLOBAL uint32_t*)state, nlevels, patience, number, first, count, tid, lds);
  else chain_levels<8>(levels, jobs, active, tasks, (DPLLM_GLOBAL uint32_t*)state, nlevels, patience, number, first, count, tid, lds);
}

}  // namespace dpllm
