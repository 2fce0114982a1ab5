// MAP accepting-cycle detection for MI355X (gfx950, CDNA4): HIP kernels and
// the C ABI declared in include/mapcheck.h.
//
// Method: Barnat, Brim, Ceska, "DiVinE-CUDA", PDMC 2009, Section 2.  MAP runs on
// the transposed state graph, so on the generated graph G a vertex v keeps
//   map(v) = max{ a accepting : v reaches a along >= 1 edge },
// the least fixpoint of  map(v) = max over edges v->w of max(map(w), [w in A]*w),
// computed by repeated sparse (max, id) matrix-vector products ("sweeps") over
// the pull CSR of G (row v = successors of v).  The fixpoint is unique, so any
// monotone schedule -- in place, stale reads across workgroups, any order --
// reaches the same vector; only the sweep count depends on the schedule.
//
// Device data layout (workspace):
//   ctrl   control block: grid-barrier counters, per-epoch reduction slots,
//          the asynchronous change counter and quiet reports, and the
//          iteration-tag epoch kept across calls;
//   pv     uint32[n]: bit 31 = vertex is accepting in the current iteration,
//          low bits (the bit length of n) = current map value (id, 0 = none),
//          the bits between = tag of the iteration that wrote the word;
//   accw   uint8[n]: working accepting flags, stripped between iterations;
//   frontier lists, change bitmaps and the CSR build's scratch (see layout()).
//
// One cooperative persistent kernel runs the whole outer loop (reset, sweeps
// to the fixpoint, detect, strip, next iteration) with grid barriers between
// phases; a small graph is solved by one workgroup in an ordinary launch.  The
// host enqueues one launch per call (two where it cannot tell how dense a small
// graph is) and never synchronizes.
// Sweeps pull over the CSR (staged in LDS where a workgroup's slice fits,
// streamed otherwise); on large graphs the streamed sweeps can switch to
// pushing from the rows that grew over the transposed CSR.  The CSR itself is
// built on the device, by per-row cursors or a radix sort.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "mapcheck.h"

namespace {

constexpr int kWave = 64;
constexpr int kBlock = 1024;  // threads per workgroup of the loop kernel (one per CU)
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kTileRows = 128;    // rows per wave tile
constexpr int kFiltRows = 128;    // rows per wave tile of the filtered sweeps
constexpr int kFiltAlign = 4;      // filtered sweeps: a wave's rows begin at a multiple of this
constexpr int kFoldWords = 16384;  // filtered sweeps: words of the bitmap in LDS (64 KiB)
constexpr int kBandCount = 11;     // banded sweeps: bands
constexpr int kBandPasses = 64;    // banded sweeps: passes over a band
constexpr int kBandGrow = 64;      // banded sweeps: begun from this share of the rows on where the frontier doubles
constexpr int kBandLeave = 128;    // banded sweeps: a band is left once fewer than this share of its rows grew
constexpr int kBandWrong = 1 << 17;  // banded sweeps: at most this share of the sampled edges points the other way
constexpr int32_t kBandMinN = 3 << 21;  // banded sweeps: fewer rows are swept faster whole
constexpr int kFoldMinWords = 512;   // filtered sweeps: a smaller bitmap is read where it is
constexpr int kFoldDiv = 4;        // filtered sweeps: a folded bitmap has at most this share of its bits set
constexpr int kTileEdges = 512;   // stream mode: edges staged in LDS per wave (2 KiB)
constexpr int kRowsPerLane = kTileRows / kWave;
constexpr int kEdgesPerLane = kTileEdges / kWave;
constexpr int kResRowsPerLane = 4;                     // resident mode: rows per lane
constexpr int kResWaveRows = kWave * kResRowsPerLane;  // resident mode: rows per wave
constexpr int kResEdges = 24576;                        // resident mode: CSR edges per block in LDS
constexpr int kGatherBatch = 6;                         // resident mode: gathers in flight per lane
constexpr int kLocalPasses = 4;                         // resident mode: LDS-only passes after a sweep
constexpr int kSortSlots = 1024;                        // resident mode: bitonic sort width (>= 64 * kGatherBatch)
constexpr int kSortPerLane = kSortSlots / kWave;
static_assert(kSortSlots >= kWave * kGatherBatch, "sort must cover a gather batch");
constexpr uint32_t kAllFlags =
    MAP_FLAG_DENSE_ONLY | MAP_FLAG_NO_TRACE_DIGEST | MAP_FLAG_STREAM | MAP_FLAG_SYNC_SWEEPS | MAP_FLAG_PUSH |
    MAP_FLAG_EARLY | MAP_FLAG_NO_FILTER |
    MAP_FLAG_DIRECTION;
constexpr uint32_t kAccBit = 0x80000000u;
// Direction switch: push rounds while the previous sweep grew fewer than
// n / kPushNear rows, or n / kPushFar where a workgroup has kPushFarRows rows or
// more: a push round is a chain of atomics of much the same length everywhere, a
// pull takes as long as a workgroup's rows.  n / 8, 16: digraph of 1.1M vertices
// (4,300 rows each) 0.94, 0.87 ms, 4M 1.95, 1.93; 16M vertices 4.10, 4.11; a batch
// of 64 graphs of 200,000 to 10^6, one workgroup each, 6.47, 6.66 (n / 4, 32, 64
// in a batch of 512: 8.8, 11.7, 16.5 against 8.8 and 9.7).
constexpr int kPushNear = 16, kPushFar = 8;
constexpr int64_t kPushFarRows = 1 << 16;
// Likewise an iteration begins with a push round from the accepting vertices
// (fewer than the same share) only where the pull over a workgroup's rows costs
// more than the reset pass, its barrier and the round: DAGs of 1.1M, 2M, 4M
// vertices (4,300, 7,800, 15,600 rows) 607, 692, 762 us, with a pull 575, 686,
// 832; one workgroup with 10^6 rows 0.05 ms against 0.8.
constexpr int64_t kPushResetRows = 1 << 13;
constexpr int kHubEdges = 64;  // stream tiles: default edges of a row in a staged chunk above which a wave folds it

// Global-memory views of device pointers, for out-of-line functions where the
// address space of a pointer loaded from an argument struct is not inferred.
typedef __attribute__((address_space(1))) uint32_t g_u32;
typedef __attribute__((address_space(1))) uint8_t g_u8;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) u32x4 g_u32x4;
typedef __attribute__((address_space(1))) const int32_t g_ci32;
typedef __attribute__((address_space(1))) const uint8_t g_cu8;
constexpr uint32_t kValMask = 0x7fffffffu;
constexpr int kStripes = 16;
constexpr int kSets = 3;
constexpr int kMaxGroups = 8;  // barrier arrival groups (one per XCD)
constexpr int kMaxBlocks = 2048;  // upper bound on the loop kernel's grid
constexpr int kMaxGang = 256;     // upper bound on the blocks that share one graph of a batch
// Bound on one barrier wait, in ticks of the 100 MHz device wall clock (10 s):
// far beyond any legitimate phase, so a broken launch exits instead of hanging.
constexpr uint64_t kWaitTicks = 1000000000ull;
// Bound on the asynchronous sweeping of one fixpoint computation (60 s of
// device wall clock): a sweep loop that has not settled by then (a livelock)
// ends the launch with MAP_EDEVICE instead of running on.
constexpr uint64_t kIterTicks = 6000000000ull;

// Windowed iterations (win_body).
constexpr int kWinWords = 7;
constexpr int kWinBits = 32 * kWinWords;
constexpr int kWinRows = 4;                     // rows per thread
constexpr int kWinMaxRows = kBlock * kWinRows;  // rows per block
constexpr int kWinBlockEdges = 24576;           // edges per block, in registers: 25 slots of one per thread
constexpr int kWinSlots = kWinBlockEdges / kBlock + 1;
constexpr int kWinFronts = 64;                  // ids of the last strip that guide the choice of a window
constexpr int kWinList = 8192;                  // different records that a workgroup can simulate
constexpr int kWinListRows = kWinList / kBlock;
constexpr int kWinPasses = 3;                   // passes over a block's own edges per sweep
// Windows pay when a strip removes few flags: at most an eighth of a window.
constexpr uint32_t kWinDel = kWinBits / 8;
constexpr uint32_t kWinMinLeft = 2 * kWinDel;  // accepting vertices left: fewer end soon anyway
constexpr int kWinShort = 4;                   // a window of fewer iterations did not pay
constexpr int kWinShorts = 3;                  // so many of them in a row end the windows
constexpr int kWinFirstShorts = 2;             // the same before any has paid (or one of a single iteration)
constexpr int kWinBackoff = 32;                // plain iterations before they are tried again, doubled each time

// ------------------------------------------------------------------ ctrl --

struct alignas(128) Stripe {
  unsigned long long digest;
  unsigned long long sweeps;  // sweeps of the blocks of this stripe in the iteration
  uint32_t count;
  int32_t witness;
  uint32_t nonzero;
  uint32_t pad[25];
};

struct alignas(128) Line64 {
  unsigned long long v;
  unsigned long long pad[15];
};

// Control block of one set of cooperating blocks: the whole grid for a single
// graph, or the gang of blocks that solves one graph of a batch.  Q bounds the
// number of blocks in the set.
template <int Q>
struct alignas(256) CtrlT {
  Line64 grp[kMaxGroups];  // barrier arrivals per group: high 32 = arrivals, low 32 = payload sum
  Line64 top;              // arrivals of the group leaders
  alignas(128) uint32_t gen;       // barrier generation
  uint32_t payload;                // payload sum of the last completed barrier
  int32_t abort;                   // set when a barrier wait exceeded its bound
  uint32_t pad0[29];
  Stripe sets[kSets][kStripes];    // per-epoch reductions
  // Asynchronous fixpoint: change counter, per-block quiet reports
  // {iteration, counter + 1} and the iteration whose fixpoint is established.
  alignas(128) uint32_t dirty;
  uint32_t pad1[31];
  alignas(128) uint32_t done;
  uint32_t pad2[31];
  alignas(128) uint32_t fcount[2];  // push and lasso: entries appended to frontier 0 / 1
  uint32_t hit;                     // lasso: smallest vertex whose edge reached the target, or kNoHit
  uint32_t bad;                     // lasso and trim: an edge endpoint outside 0..n-1 was read
  unsigned long long scanned;       // lasso: edges examined
  uint32_t kept;                    // trim: vertices kept
  uint32_t acc_kept;                // trim: accepting vertices kept
  uint32_t early;                   // MAP_FLAG_EARLY: largest id seen equal to its own value (0: none)
  uint32_t pad3[23];
  unsigned long long quiet[Q];
};
using Ctrl = CtrlT<kMaxBlocks>;
using GangCtrl = CtrlT<kMaxGang>;
constexpr size_t kCtrlBytes = 32768;
// The last line of a single graph's control region holds the tag epoch, which
// outlives the call (the per-call clear stops before it): the first iteration
// tag of a call follows the last one of the previous call on the workspace.
constexpr size_t kEpochOff = kCtrlBytes - 256;
static_assert(sizeof(Ctrl) <= kEpochOff, "ctrl block too large");
constexpr size_t kGangCtrlBytes = sizeof(GangCtrl);
// Arrays of control blocks are indexed with GangCtrl pointers and cleared in
// kGangCtrlBytes units: the two strides must agree.
static_assert(kGangCtrlBytes % 256 == 0, "control blocks are 256-byte multiples");

// Completes this wave's global writes before a workgroup barrier after which
// the workgroup's leader publishes them to other workgroups (an agent-scope
// release, then an atomic).  On gfx950 a workgroup-scope release waits only
// for LDS operations (the waves of a workgroup share one CU's L1), and the
// leader's agent-scope release -- an L2 write-back (`buffer_wbl2 sc1`) and a
// wait on the leader's own wave's memory operations -- is documented to order
// only that wave's operations.  Waiting here for every vector memory operation
// of every wave (`s_waitcnt vmcnt(0)`: each store acknowledged by L2) puts all
// of them in L2 before the barrier, so the leader's write-back that follows the
// barrier covers them.
__device__ __forceinline__ void wave_writes_done() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0x0F70);  // gfx9 encoding of vmcnt(0), expcnt and lgkmcnt left at their maxima
}

__device__ __forceinline__ uint32_t ld_agent(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------- wave reductions --

// Max over the 64 lanes with DPP row operations (GFX9 row_bcast), result in
// every lane.
__device__ __forceinline__ int wave_max_i32(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x140, 0xF, 0xF, false));  // row_mirror
  x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x142, 0xA, 0xF, false));  // row_bcast:15
  x = max(x, __builtin_amdgcn_update_dpp(x, x, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return __builtin_amdgcn_readlane(x, 63);
}

// Max over the 64 lanes of values below 2^31 (map values and ids), result in
// every lane: the same DPP row operations as wave_max_i32.
__device__ __forceinline__ uint32_t wave_max_u31(uint32_t x) { return (uint32_t)wave_max_i32((int)x); }

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, kWave);
  return x;
}

// SplitMix64 finalizer (Steele, Lea & Flood, OOPSLA 2014), the per-vertex term
// of the order-independent map digest.
__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ------------------------------------------------------------ grid barrier --

template <typename C>
struct Grid {
  C* c;
  uint32_t gen;      // generation this block expects to complete next
  int nblocks;
  int group;         // arrival group of this block
  int group_size;    // blocks in this group
  int ngroups;
  int rank;          // index of this block in the set
};

// Grid-wide barrier with a summed 32-bit payload.  Every thread must call it.
// Returns false if the wait exceeded its bound (the kernel must then exit).
//
// Ordering: every wave completes its global writes (wave_writes_done) before
// the workgroup barrier; the block's leader then issues one agent-scope release
// fence before its arrival; the last arrival of a group and the last group
// leader acquire before forwarding; waiters poll with relaxed loads (no cache
// invalidation per poll) and acquire once when the generation moves.
template <typename C>
__device__ __forceinline__ bool grid_sync_inline(Grid<C>& g, uint32_t payload, uint32_t* total) {
  __shared__ uint32_t s_total;
  __shared__ int s_ok;
  if (g.nblocks == 1) {
    // A single block: a workgroup barrier orders everything it shares.
    __syncthreads();
    if (threadIdx.x < kStripes) {
      Stripe& s = g.c->sets[(g.gen + 2) % kSets][threadIdx.x];
      __hip_atomic_store(&s.digest, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&s.sweeps, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      st_agent(&s.count, 0u);
      __hip_atomic_store(&s.witness, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      st_agent(&s.nonzero, 0u);
    }
    __syncthreads();
    g.gen++;
    if (total) *total = payload;
    return true;
  }
  wave_writes_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    C* c = g.c;
    int ok = 1;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    const unsigned long long inc = (1ull << 32) | payload;
    unsigned long long old = __hip_atomic_fetch_add(&c->grp[g.group].v, inc, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
    if ((int)(old >> 32) == g.group_size - 1) {
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const uint32_t gsum = (uint32_t)old + payload;
      __hip_atomic_store(&c->grp[g.group].v, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      unsigned long long old2 = __hip_atomic_fetch_add(&c->top.v, (1ull << 32) | gsum, __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT);
      if ((int)(old2 >> 32) == g.ngroups - 1) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __hip_atomic_store(&c->top.v, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        st_agent(&c->payload, (uint32_t)old2 + gsum);
        __hip_atomic_store(&c->gen, g.gen + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    const uint64_t t0 = wall_clock64();
    while (ld_agent(&c->gen) == g.gen) {
      __builtin_amdgcn_s_sleep(1);
      if (wall_clock64() - t0 > kWaitTicks || ld_agent((const uint32_t*)&c->abort)) {
        ok = 0;
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (!ok) st_agent((uint32_t*)&c->abort, 1u);
    if (total) s_total = ok ? ld_agent(&c->payload) : 0u;
    s_ok = ok;
  }
  __syncthreads();
  // Epoch E+1 writes set (E+1)%3 and reads set E%3; set (E-1)%3 was last read
  // during epoch E, so block 0 clears it now for epoch E+2.
  if (g.rank == 0 && threadIdx.x < kStripes) {
    Stripe& s = g.c->sets[(g.gen + 2) % kSets][threadIdx.x];
    __hip_atomic_store(&s.digest, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&s.sweeps, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    st_agent(&s.count, 0u);
    __hip_atomic_store(&s.witness, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    st_agent(&s.nonzero, 0u);
  }
  g.gen++;
  if (total) *total = s_total;
  return s_ok != 0;
}

// The same where few values live across a barrier: left to the compiler, which
// calls it out of line when there are many.  The loop bodies take the inline
// form: a called barrier makes them save most of their registers to memory
// around each, over 1 us a sweep (filtered sweeps of 4M vertices 34.0 us each
// with called barriers, 32.4 inlined).
template <typename C>
__device__ bool grid_sync(Grid<C>& g, uint32_t payload, uint32_t* total) {
  return grid_sync_inline(g, payload, total);
}

// ------------------------------------------------------------- the kernel --

struct LoopArgs {
  int32_t n;
  int32_t ntiles;
  const int32_t* row_ptr;
  const int32_t* col;
  const uint8_t* acc_in;  // A_1 (detect) or the accepting set (propagate)
  uint32_t* pv;
  uint8_t* accw;
  Ctrl* ctrl;
  map_result* result;
  uint64_t* trace;
  int32_t trace_cap;
  uint8_t* acc_out;
  int32_t* map_out;
  int32_t max_iter;
  int32_t propagate;  // 1: one fixpoint of acc_in, write map_out
  int32_t digest;     // 1: compute the trace digest
  int32_t force_stream;  // 1: never stage the CSR in LDS
  int32_t sync_sweeps;   // 1: a grid barrier after every sweep instead of the asynchronous fixpoint
  uint32_t val_mask;     // bits of a packed word holding the map value
  uint32_t tag_mask;     // bits holding the iteration tag (0: untagged, n >= 2^30)
  uint32_t tag_shift;    // lowest bit of the tag
  uint32_t* epoch;       // single graph: the workspace's tag epoch word (else null)
  int32_t push;          // 1: frontier sweeps over the transposed CSR (barrier per round)
  int32_t early;         // 1: stop once a value equals its own row's id (MAP_FLAG_EARLY)
  const int32_t* rrow_ptr;  // push: transposed CSR (row w = predecessors of w)
  const int32_t* rcol;
  int32_t* front[2];     // push: frontier lists, int32[n] each
  uint32_t* mark;        // push: round in which a vertex last joined a frontier
  // Filtered stream sweeps (every block streams, barrier per sweep): three
  // change bitmaps of one bit per vertex (the rows that grew in a sweep) and
  // the bitmap of the current accepting set; null where no workspace holds them.
  uint32_t* chg;         // [3][words]; single graph: [4][words]
  uint32_t* accb;        // [words]
  int64_t words;         // 32-bit words per bitmap
  int32_t filt;          // 1: run the filtered stream kernel
  int32_t dopt;          // filtered stream kernel: small frontiers run as push rounds (transposed CSR, front[])
  int32_t hub;           // stream tiles: rows with more edges in a staged chunk are folded by the whole wave
  int32_t gate;          // 1: map_small_kernel and map_loop_kernel are both launched, small_takes says whose graph it is
  struct WinCtl* win;    // windowed iterations: control words and the rows' records, or null
  struct WinRec* win_rec;
};

// Windowed iterations: what a row sends, or reaches.
struct alignas(16) WinRec {
  uint32_t w[8];  // w[0..6]: bit 31 - i of word q = the window's id number 32 q + i; w[7]: the largest id below the window
};

// Windowed iterations: reductions of one iteration over the blocks (as Stripe)
// and the words the blocks exchange when a window is chosen.
struct alignas(128) WinRed {
  uint32_t img[8];
  unsigned long long dig;
  int32_t wit;
  uint32_t nz;
  uint32_t low;
  uint32_t pad[19];
};
struct WinCtl {
  WinRed red[kSets][kStripes];
  uint32_t count[kMaxGang];   // accepting rows of each block
  uint32_t ids[kWinBits];
  uint32_t moved[kSets][32];         // blocks that raised a row in a sweep, one bit each (8 words)
  uint32_t fronts;                   // entries of `front`
  uint32_t front[kWinFronts];        // ids stripped last: block << 16 | accepting rows above in the block
  uint32_t listed;                   // entries of `list`
  uint32_t pad[30];
  unsigned long long dig[kWinBits];  // digests of the simulated iterations
  WinRec list[kWinList];             // different records of the graph (w[7]: see win_body)
};
constexpr size_t kWinCtlBytes = (sizeof(WinCtl) + 255) & ~(size_t)255;
constexpr int32_t kWinMaxN = kMaxGang * kWinMaxRows;  // 2^20: a successor and a row offset share 32 bits
static_assert(kWinMaxN <= 1 << 20 && kWinMaxRows <= 1 << 12, "an edge is one register");

// A function that is called out of line finds its arguments in vector registers
// and memory, and the compiler takes them as different in every lane and of
// unknown address space.  These make them uniform over the wave again, in scalar
// registers, and the pointers global.  Measured on the loop bodies: 13,000
// vertices 271 us without, 226 with; 700,000 vertices 619 and 506 (inlined into
// the kernel: 222 and 493); 512 graphs in one batch 24.6 and 22.5 ms.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <typename T>
__device__ __forceinline__ T* uniform(T* p) {
  const uint64_t x = reinterpret_cast<uint64_t>(p);
  const uint64_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
  const uint64_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32));
  return (T*)(__attribute__((address_space(1))) T*)(lo | hi << 32);
}
__device__ __forceinline__ LoopArgs uniform(const LoopArgs& a) {
  constexpr int kWords = sizeof(LoopArgs) / 4;
  static_assert(sizeof(LoopArgs) % 4 == 0, "copied in words");
  uint32_t w[kWords];
  __builtin_memcpy(w, &a, sizeof a);
#pragma unroll
  for (int i = 0; i < kWords; ++i) w[i] = (uint32_t)uniform((int)w[i]);
  LoopArgs u;
  __builtin_memcpy(&u, w, sizeof u);
  u.row_ptr = uniform(u.row_ptr);
  u.col = uniform(u.col);
  u.acc_in = uniform(u.acc_in);
  u.pv = uniform(u.pv);
  u.accw = uniform(u.accw);
  u.ctrl = uniform(u.ctrl);
  u.result = uniform(u.result);
  u.trace = uniform(u.trace);
  u.acc_out = uniform(u.acc_out);
  u.map_out = uniform(u.map_out);
  u.epoch = uniform(u.epoch);
  u.rrow_ptr = uniform(u.rrow_ptr);
  u.rcol = uniform(u.rcol);
  u.front[0] = uniform(u.front[0]);
  u.front[1] = uniform(u.front[1]);
  u.mark = uniform(u.mark);
  u.chg = uniform(u.chg);
  u.accb = uniform(u.accb);
  u.win = uniform(u.win);
  u.win_rec = uniform(u.win_rec);
  return u;
}

// What survives between the loop's two ways of iterating.
struct LoopState {
  int32_t k;        // iterations made
  uint32_t count;   // |A_k|, before the strip of iteration k
  uint32_t gen;     // barrier generation
  int32_t resumed;  // 1: the working flags and iterations so far stand
  int32_t win_from; // windows are tried from this iteration on
  int32_t backoff;  // plain iterations before the next try
  // Of the windows (here and not in registers: seldom read).
  int32_t shorts;   // short windows in a row
  int32_t paid;     // 1: some window since the last plain iteration paid
  int64_t sweeps;
};

// Rows per block of the windowed iterations (whole words of a row bitmap).
__device__ __forceinline__ int64_t win_rows(int32_t n, int nb) { return (((int64_t)n + nb - 1) / nb + 31) & ~(int64_t)31; }

// Row ownership: the rows are cut into one contiguous range per block and,
// inside it, one contiguous range per wave.  A wave is the only writer of the
// packed values of its rows for the whole launch.
//
// Two sweep modes, chosen per block at launch:
//   resident  the block's slice of the CSR (column indices plus, per edge, the
//             row's offset inside its wave) is staged in LDS once; the wave's
//             packed values live in registers; a sweep is one batch of gathers
//             per lane, reduced per row with LDS atomic max.
//   stream    row offsets and column indices are streamed from HBM in tiles of
//             kTileRows rows, gathered values staged in LDS, reduced per row.
struct TileLds {
  int32_t rp[kTileRows + 1];
  uint32_t val[kTileEdges];
};

// Filtered sweeps: a wave's staged chunk, and the bitmap of the rows that send,
// folded to kFoldWords words (bit v of the fold: a vertex congruent to v sends).
struct FiltLds {
  uint32_t val[kWavesPerBlock][kTileEdges];
  uint32_t bits[kFoldWords];
};

struct ResLds {
  // Staged edges of each wave: first those to rows of other blocks, as
  // (successor << 8) | row offset in the wave, sorted by successor in gather
  // batches; then those to rows of this block, as successor - block base,
  // grouped by row in row order.
  uint32_t e[kResEdges];
  uint16_t lrow[kWavesPerBlock * kResWaveRows];  // first in-block edge of each row of the block
  uint32_t best[kWavesPerBlock][kResWaveRows];
  uint32_t pv[kWavesPerBlock * kResWaveRows];  // the block's own packed values (row - block base)
};

// A graph of at most kSmallN vertices solved by one workgroup (small_body):
// what every vertex sends stays in LDS, and up to kSmallEdges edges per thread
// stay in registers.
constexpr int kSmallRows = 12;                // rows per thread
constexpr int kSmallN = kBlock * kSmallRows;  // 12,288 vertices
constexpr int kSmallEdges = 48;               // edges per thread: 49,152 in all
constexpr int kSmallBatch = 8;                // edges of a thread relaxed together
// Times a wave goes over its edges between two workgroup barriers, for m edges:
// with few edges per thread the barriers cost more than another round (1,000
// vertices, K = 8: 186 us with 1 round, 133 us with 16); from 16 edges per
// thread on a round costs more than the barriers (12,288 vertices, 37,000
// edges: 105 us with 1, 116 us with 16).
__device__ __forceinline__ int small_rounds(int m) { return max(1, min(16, 32 * kBlock / max(m, 1))); }
static_assert(kSmallEdges % kSmallBatch == 0, "whole batches");
struct SmallLds {
  union {
    struct {
      uint32_t sent[kSmallN + 4];     // what each vertex sends; entry n stays 0 (padding, columns outside 0..n-1)
      uint32_t own[kSmallN];          // map values of the accepting rows that send their own id
      uint32_t del[kSmallN / 32];     // flags to strip after the iteration
    };
    uint16_t row_of[kBlock * kSmallEdges];  // set-up: the row of each edge
  };
  int32_t rp[kSmallN + 1];            // row starts, relative to the first
};

// Windowed iterations (win_body): per row what it reaches of the kWinBits
// largest accepting ids, one bit each, and the largest other accepting id.
struct WinLds {
  union {
    struct {
      WinRec rec[kWinMaxRows];    // what the block's rows send; after the fixpoint what they reach
      uint32_t own[kWinMaxRows];  // reached ids of the rows below the window that send their own
    };
    struct {  // set-up
      uint32_t stage[kWinBlockEdges];
      uint16_t row_of[kWinBlockEdges];
    };
  };
  uint32_t chg[2][kWinMaxRows / 32];  // rows raised: consumed by the current pass, collected for the next
  uint32_t pub[kWinMaxRows / 32];     // rows raised since they were last written to memory
  uint32_t acc[kWinMaxRows / 32];     // accepting rows
  uint32_t accs[kWinMaxRows / 32];    // accepting rows in the words above
  uint32_t suf[kMaxGang];             // accepting rows in the blocks above
  uint32_t fp[kWinFronts], fl[kWinFronts];  // fronts: accepting rows above, ids taken
  uint32_t ids[kWinBits];             // the window's ids, descending
  uint32_t img[8];                    // image of an iteration inside the window
  uint32_t moved[kMaxGang / 32];      // blocks that raised a row in the last sweep
  uint32_t alive[8];                  // window ids that still accept
  uint32_t self[8];                   // window ids that reach themselves
  uint8_t widx[kWinMaxRows];          // a row's number in the window, or 255
};

union BlockLds {
  TileLds tile[kWavesPerBlock];
  FiltLds filt;
  ResLds res;
  SmallLds small;
  WinLds win;
};

struct WaveRows {
  int64_t rb0, rb1;  // rows of this block
  int64_t r0, r1;  // rows of this wave
  int32_t we0, we1;  // resident: edge range of the wave inside the block's LDS slice
  int32_t wr;        // resident: [we0, wr) edges to rows of other blocks, [wr, we1) to rows of this block
  bool resident;
  bool ascending;    // stream: sweep tiles in increasing row order (most edges point to lower rows)
};

// The block's LDS, at namespace scope so that out-of-line sweep functions
// address it directly (LDS instructions, not generic pointers).  In resident
// mode g_lds.res.pv holds the block's own packed values, the only copy a wave
// reads its rows from.
__shared__ BlockLds g_lds;
// MAP_FLAG_EARLY: the largest id of a row of this block whose value equals
// its own id (0: none), found by a scan of the block's rows after each sweep.
__shared__ uint32_t g_early;
// Resident asynchronous bodies: where each wave's edges to other blocks' rows
// start in the staged slice, and the prefix sums of their counts, so that the
// block's remote edges can be shared evenly over its waves.
__shared__ int32_t g_rseg[kWavesPerBlock];
__shared__ int32_t g_rpre[kWavesPerBlock + 1];

#ifdef MAPCHECK_PHASES
// Phase clocks of the loop kernel, in a build made only to measure where the
// time goes (libmapcheck_phases.so): thread 0 of each block adds the device
// wall-clock ticks since its previous mark to the phase a mark names, and counts
// events; the block writes its totals to g_phase_out when it finishes.
enum PhaseSlot {
  kPhSetup, kPhRemote, kPhLocal, kPhStream, kPhReport, kPhWait, kPhDetect, kPhOther,
  kPhSweeps, kPhLocalPasses, kPhQuiet, kPhIters, kPhRemoteWait, kPhGather, kPhSlots = 16
};
__shared__ uint64_t g_ph[kPhSlots];
__shared__ uint64_t g_ph_t;
__device__ uint64_t g_phase_out[kMaxBlocks * kPhSlots];
__device__ int32_t g_phase_blocks;  // workgroups of the run that wrote it
__device__ __forceinline__ void ph_start() {
  if (threadIdx.x == 0) {
    for (int i = 0; i < kPhSlots; ++i) g_ph[i] = 0;
    g_ph_t = wall_clock64();
  }
}
__device__ __forceinline__ void ph_mark(int slot) {
  if (threadIdx.x == 0) {
    const uint64_t t = wall_clock64();
    g_ph[slot] += t - g_ph_t;
    g_ph_t = t;
  }
}
__device__ __forceinline__ void ph_count(int slot, uint64_t d) {
  if (threadIdx.x == 0) g_ph[slot] += d;
}
__device__ __forceinline__ void ph_store(int b, int nb) {
  if (threadIdx.x == 0 && b < kMaxBlocks) {
    for (int i = 0; i < kPhSlots; ++i) g_phase_out[(size_t)b * kPhSlots + i] = g_ph[i];
    if (b == 0) g_phase_blocks = nb;
  }
}
#define PH_START() ph_start()
#define PH_MARK(slot) ph_mark(slot)
#define PH_COUNT(slot, d) ph_count((slot), (d))
#define PH_STORE(b, nb) ph_store((b), (nb))
#else
#define PH_START() ((void)0)
#define PH_MARK(slot) ((void)0)
#define PH_COUNT(slot, d) ((void)0)
#define PH_STORE(b, nb) ((void)0)
#endif

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Layout of a packed value word for ids 1..n: the value takes the bit length
// of n, the accepting flag bit 31, and the iteration tag the bits between
// (none when n >= 2^30, one bit -- the iteration parity -- when n >= 2^29).
__host__ __device__ inline void word_layout(int32_t n, uint32_t* vmask, uint32_t* tmask, uint32_t* tshift) {
  int vbits = 0;
  while (vbits < 31 && ((uint32_t)n >> vbits) != 0u) ++vbits;
  if (vbits >= 31) {
    *vmask = kValMask;
    *tmask = 0u;
    *tshift = 31u;
    return;
  }
  *vmask = (1u << vbits) - 1u;
  *tmask = kValMask & ~*vmask;
  *tshift = (uint32_t)vbits;
}

// Tag of the words written in iteration k (k >= 1) of a call whose epoch is
// `base`.  With two or more tag bits the tags run through 1 .. 2^T - 1 (tag 0,
// the launch-start clear, is never current), consecutive iterations differ,
// and a call starts right after the tags its predecessor on the workspace
// used; with one bit the tag is the parity of k.
__device__ __forceinline__ uint32_t iter_tag(uint32_t tmask, uint32_t tshift, uint32_t base, int32_t k) {
  if (tmask == 0u) return 0u;
  const uint32_t span = tmask >> tshift;
  if (span == 1u) return (k & 1) ? tmask : 0u;
  return (1u + (base + (uint32_t)k - 1u) % span) << tshift;
}

// Fold of one staged chunk of a stream tile into the maxima of the rows a lane
// owns: a row with at most `hub` edges in the chunk is folded by its own lane;
// each longer row is folded by the whole wave -- every lane takes every 64th of
// its edges, then a DPP max gives the row's maximum to its lane.
template <int kRows>
__device__ __forceinline__ void fold_chunk(const uint32_t* val, const int32_t* lo, const int32_t* hi, int32_t c0,
                                          int cnt, int hub, int lane, uint32_t* best) {
#pragma unroll
  for (int j = 0; j < kRows; ++j) {
    const int b = max(lo[j] - c0, 0), e = min(hi[j] - c0, cnt);
    const bool longrow = e - b > hub;
    uint32_t m = best[j];
    if (!longrow)
      for (int k = b; k < e; ++k) m = max(m, val[k]);
    unsigned long long lr = __ballot(longrow);
    while (lr) {
      const int src = __ffsll(lr) - 1;
      lr &= lr - 1;
      const int bb = __shfl(b, src, kWave), ee = __shfl(e, src, kWave);
      uint32_t x = 0;
      for (int k = bb + lane; k < ee; k += kWave) x = max(x, val[k]);
      x = wave_max_u31(x);
      if (lane == src) m = max(m, x);
    }
    best[j] = m;
  }
}

// Value that successor w (0-based) sends along an edge: its map value, or its
// own id if it is accepting and larger.  A word tagged with another iteration
// has not been reset in this iteration yet and sends 0, a valid lower bound
// (its owner's reset sweep then counts as a change, so the reader sweeps again
// once the true value is there).
__device__ __forceinline__ uint32_t sent_word(uint32_t x, int32_t w, uint32_t cur, uint32_t vmask, uint32_t tmask) {
  const uint32_t id = (uint32_t)w + 1u;
  if ((x & tmask) != cur) return 0u;
  const uint32_t m = x & vmask;
  return (x & kAccBit) ? (m > id ? m : id) : m;
}

// What successor w sends in the first sweep of an iteration (map = 0 everywhere).
__device__ __forceinline__ uint32_t sent_first(const uint8_t* acc, int32_t w) {
  return ((g_cu8*)acc)[w] ? (uint32_t)w + 1u : 0u;
}

// Stream mode, rows [r0, r1) with r1 - r0 <= kTileRows, processed by one wave.
// kFirst: the sweep that starts an iteration from map = 0 (successors send their
// id if accepting, every row is written).  Otherwise a row is written only when
// its value grows.  Returns nonzero (wave-uniform) if some row changed.
template <bool kFirst, bool kHub>
__device__ uint32_t sweep_tile(const LoopArgs& a, const uint8_t* acc, int64_t r0, int64_t r1, TileLds& L, int lane,
                               uint32_t cur, uint32_t* acc_count) {
  const int nr = (int)(r1 - r0);
  g_ci32* row_ptr = (g_ci32*)a.row_ptr;
  g_ci32* colp = (g_ci32*)a.col;
  g_u32* pv = (g_u32*)a.pv;
  g_cu8* gacc = (g_cu8*)acc;
  const uint32_t n = (uint32_t)a.n, vmask = a.val_mask, tmask = a.tag_mask;
  for (int i = lane; i <= nr; i += kWave) L.rp[i] = __builtin_nontemporal_load(row_ptr + r0 + i);
  wave_lds_sync();
  const int32_t e0 = L.rp[0], e1 = L.rp[nr];
  int32_t lo[kRowsPerLane], hi[kRowsPerLane];
  uint32_t best[kRowsPerLane], old[kRowsPerLane];
#pragma unroll
  for (int j = 0; j < kRowsPerLane; ++j) {
    int r = lane + j * kWave;
    lo[j] = r < nr ? L.rp[r] : 0;
    hi[j] = r < nr ? L.rp[r + 1] : 0;
    best[j] = 0;
    old[j] = (!kFirst && r < nr) ? pv[r0 + r] : 0u;
  }
  // (Unsigned: a step past the last of 2^31 - 1 edges stays above it.)
  for (uint32_t c0 = (uint32_t)e0; c0 < (uint32_t)e1; c0 += kTileEdges) {
    const int cnt = (int)min((uint32_t)kTileEdges, (uint32_t)e1 - c0);
    int32_t w[kEdgesPerLane];
#pragma unroll
    for (int u = 0; u < kEdgesPerLane; ++u) {
      int i = lane + u * kWave;
      w[u] = i < cnt ? __builtin_nontemporal_load(colp + c0 + i) : -1;
    }
#pragma unroll
    for (int u = 0; u < kEdgesPerLane; ++u) {
      int i = lane + u * kWave;
      uint32_t x = 0;
      if ((uint32_t)w[u] < n) x = kFirst ? sent_first(acc, w[u]) : sent_word(pv[w[u]], w[u], cur, vmask, tmask);
      if (i < cnt) L.val[i] = x;
    }
    wave_lds_sync();
    if (kHub) {
      fold_chunk<kRowsPerLane>(L.val, lo, hi, (int32_t)c0, cnt, a.hub, lane, best);
    } else {
#pragma unroll
      for (int j = 0; j < kRowsPerLane; ++j) {
        int b = max(lo[j] - (int32_t)c0, 0), e = min(hi[j] - (int32_t)c0, cnt);
        uint32_t m = best[j];
        for (int k = b; k < e; ++k) m = max(m, L.val[k]);
        best[j] = m;
      }
    }
    wave_lds_sync();
  }
  uint32_t changed = 0, nacc = 0;
#pragma unroll
  for (int j = 0; j < kRowsPerLane; ++j) {
    int r = lane + j * kWave;
    if (r < nr) {
      int64_t v = r0 + r;
      if (kFirst) {
        uint32_t isacc = gacc[v] ? 1u : 0u;
        nacc += isacc;
        pv[v] = (isacc << 31) | cur | best[j];
        changed |= (best[j] | isacc) != 0;
      } else if (best[j] > (old[j] & vmask)) {
        pv[v] = (old[j] & ~vmask) | best[j];
        changed = 1;
      }
    }
  }
  if (acc_count) *acc_count += nacc;
  return __ballot(changed) != 0;
}

// Resident mode: one pass over the wave's staged edges to rows of other
// blocks, folding what each successor sends into best[row] with LDS atomic
// max.  kSrc 0: first sweep of an iteration (successors send their id if
// accepting); 1: the successors' packed values, gathered from memory.
template <int kSrc>
__device__ __forceinline__ void gather_range(const uint8_t* acc, int32_t e0, int32_t e1, uint32_t* best,
                                             const LoopArgs& a, int lane, uint32_t cur) {
  ResLds& R = g_lds.res;
  g_u32* pv = (g_u32*)a.pv;
  const uint32_t n = (uint32_t)a.n, vmask = a.val_mask, tmask = a.tag_mask;
  for (int32_t k0 = e0; k0 < e1; k0 += kWave * kGatherBatch) {
    uint32_t e[kGatherBatch];
#pragma unroll
    for (int u = 0; u < kGatherBatch; ++u) {
      const int32_t k = k0 + lane + u * kWave;
      e[u] = k < e1 ? R.e[k] : 0xffffffffu;
    }
    uint32_t x[kGatherBatch];
#pragma unroll
    for (int u = 0; u < kGatherBatch; ++u) {
      x[u] = 0;
      const uint32_t w = e[u] >> 8;
      if (e[u] != 0xffffffffu && w < n) {
        if (kSrc == 0) x[u] = sent_first(acc, (int32_t)w);
        else x[u] = sent_word(pv[w], (int32_t)w, cur, vmask, tmask);
      }
    }
#pragma unroll
    for (int u = 0; u < kGatherBatch; ++u) {
      if (x[u] != 0) atomicMax(&best[e[u] & 0xffu], x[u]);
    }
  }
}

// Resident mode, kBal: the pass over the block's edges to other blocks' rows,
// shared evenly over the block's waves (the waves' staged lists taken as one
// list of g_rpre[16] edges), each value folded with an LDS atomic max into the
// maxima of its row's wave.  Every wave must have cleared its maxima before
// (block barrier), and the rows are updated after another block barrier.
template <int kSrc>
__device__ __forceinline__ void gather_block(const uint8_t* acc, uint32_t* best_all, const LoopArgs& a, int wib,
                                             int lane, uint32_t cur) {
  ResLds& R = g_lds.res;
  g_u32* pv = (g_u32*)a.pv;
  const uint32_t n = (uint32_t)a.n, vmask = a.val_mask, tmask = a.tag_mask;
  const int32_t total = g_rpre[kWavesPerBlock];
  const int32_t share = (total + kWavesPerBlock - 1) / kWavesPerBlock;
  const int32_t lo = min(total, wib * share), hi = min(total, lo + share);
  // The list that holds the wave's first edge (the last one whose prefix sum
  // does not exceed it), found once: a lane's later edges only move forward.
  int w_lo = 0;
  while (w_lo + 1 < kWavesPerBlock && lo >= g_rpre[w_lo + 1]) ++w_lo;
  for (int32_t g0 = lo; g0 < hi; g0 += kWave * kGatherBatch) {
    uint32_t e[kGatherBatch];
    int32_t seg[kGatherBatch];
    int w = w_lo;  // the list a lane's next edge lies in (its edges increase)
#pragma unroll
    for (int u = 0; u < kGatherBatch; ++u) {
      const int32_t gi = g0 + lane + u * kWave;
      e[u] = 0xffffffffu;
      seg[u] = 0;
      if (gi < hi) {
        while (gi >= g_rpre[w + 1]) ++w;
        e[u] = R.e[g_rseg[w] + (gi - g_rpre[w])];
        seg[u] = w;
      }
    }
    uint32_t x[kGatherBatch];
#pragma unroll
    for (int u = 0; u < kGatherBatch; ++u) {
      x[u] = 0;
      const uint32_t wv = e[u] >> 8;
      if (e[u] != 0xffffffffu && wv < n) {
        if (kSrc == 0) x[u] = sent_first(acc, (int32_t)wv);
        else x[u] = sent_word(pv[wv], (int32_t)wv, cur, vmask, tmask);
      }
    }
#pragma unroll
    for (int u = 0; u < kGatherBatch; ++u) {
      if (x[u] != 0) atomicMax(&best_all[seg[u] * kResWaveRows + (e[u] & 0xffu)], x[u]);
    }
  }
}

// Rows of the wave in the order values travel: a row takes values from its
// successors, so when the block's edges mostly point to higher rows values
// flow downwards and the rows go from high to low.
__device__ __forceinline__ int row_step(const WaveRows& W, int jj) {
  return W.ascending ? jj : kResRowsPerLane - 1 - jj;
}

// Resident mode, edges to rows of this block: every lane folds the successors
// of its own rows from the block's LDS values, row by row in the order values
// travel, so rows raised earlier in the pass are seen later in it.  No
// atomics: a row's in-block edges are contiguous.  Returns nonzero
// (wave-uniform) if some row grew.
__device__ uint32_t local_pass(const LoopArgs& a, const WaveRows& W, int lane, uint32_t cur) {
  ResLds& R = g_lds.res;
  g_u32* pv = (g_u32*)a.pv;
  const uint32_t vmask = a.val_mask, tmask = a.tag_mask, base = (uint32_t)W.rb0;
  const int32_t nrow = (int32_t)(W.r1 - W.r0), r0 = (int32_t)(W.r0 - W.rb0);
  uint32_t changed = 0;
#pragma unroll
  for (int jj = 0; jj < kResRowsPerLane; ++jj) {
    const int32_t i = lane + row_step(W, jj) * kWave;
    if (i < nrow) {
      const int32_t li = r0 + i;
      const int32_t k1 = i + 1 < nrow ? (int32_t)R.lrow[li + 1] : W.we1;
      uint32_t b = 0;
      for (int32_t k = R.lrow[li]; k < k1; ++k) {
        const uint32_t t = R.e[k];
        b = max(b, sent_word(R.pv[t], (int32_t)(base + t), cur, vmask, tmask));
      }
      const uint32_t old = R.pv[li];
      if (b > (old & vmask)) {
        const uint32_t x = (old & ~vmask) | b;
        pv[(int64_t)base + li] = x;
        R.pv[li] = x;
        changed = 1;
      }
    }
  }
  return __ballot(changed) != 0;
}

// kBal: the balanced layout of the resident slice, used by the asynchronous
// bodies.  Its in-block edge entries carry the successor's row offset in the
// block (low 16 bits) and the edge's own row offset in the wave (high 16 bits);
// otherwise an entry is the successor's row offset alone.
__device__ __forceinline__ uint32_t in_succ(uint32_t e) { return e & 0xffffu; }
__device__ __forceinline__ uint32_t in_row(uint32_t e) { return e >> 16; }

// Resident mode, edges to rows of this block, balanced over the lanes (kBal).
// The wave's rows are taken in groups of 64 in the order values travel, so a
// group sees the rows the groups before it raised in the same pass.  A group's
// in-block edges are contiguous (grouped by row) and the lanes share them
// evenly: lane l folds edges l, l + 64, ... into the group's per-row maxima
// with an LDS atomic max, so a row of high degree costs its group a few more
// edges per lane instead of holding up one lane for all of them.  Every
// in-block row carries the current iteration's tag here (the reset sweep wrote
// them all before the first pass), so no tag is compared.  Returns nonzero
// (wave-uniform) if some row grew.
__device__ uint32_t local_pass_bal(const LoopArgs& a, const WaveRows& W, int wib, int lane) {
  ResLds& R = g_lds.res;
  uint32_t* best = R.best[wib];
  g_u32* pv = (g_u32*)a.pv;
  const uint32_t vmask = a.val_mask, base = (uint32_t)W.rb0;
  const int32_t nrow = (int32_t)(W.r1 - W.r0), r0 = (int32_t)(W.r0 - W.rb0);
  uint32_t changed = 0;
  for (int jj = 0; jj < kResRowsPerLane; ++jj) {
    const int32_t g0 = row_step(W, jj) * kWave;  // first row of the group in the wave
    if (g0 >= nrow) continue;                    // wave-uniform
    const int32_t g1 = min(g0 + kWave, nrow);
    const int32_t k0 = R.lrow[r0 + g0];
    const int32_t k1 = g1 < nrow ? (int32_t)R.lrow[r0 + g1] : W.we1;
    best[g0 + lane] = 0;
    wave_lds_sync();
    for (int32_t k = k0 + lane; k < k1; k += kWave) {
      const uint32_t e = R.e[k];
      const uint32_t t = in_succ(e);
      const uint32_t x = R.pv[t];
      const uint32_t m = x & vmask, id = base + t + 1u;
      const uint32_t sv = (x & kAccBit) ? max(m, id) : m;
      if (sv) atomicMax(&best[in_row(e)], sv);
    }
    wave_lds_sync();
    const int32_t i = g0 + lane;
    if (i < g1) {
      const int32_t li = r0 + i;
      const uint32_t b = best[i];
      const uint32_t old = R.pv[li];
      if (b > (old & vmask)) {
        const uint32_t x = (old & ~vmask) | b;
        pv[(int64_t)base + li] = x;
        R.pv[li] = x;
        changed = 1;
      }
    }
    wave_lds_sync();
  }
  return __ballot(changed) != 0;
}

// Resident mode: the pass over the wave's edges to other blocks' rows.
// kFirst: the reset sweep, which also folds the in-block edges (successors
// send their id if accepting) and writes every row.  Otherwise a row is
// written only when its value grows.  Returns nonzero (wave-uniform) if some
// row changed.
template <bool kFirst, bool kBal>
__device__ uint32_t sweep_resident(const LoopArgs& a, const uint8_t* acc, const WaveRows& W, int wib, int lane,
                                   uint32_t cur, uint32_t* acc_count) {
  ResLds& R = g_lds.res;
  uint32_t* best = R.best[wib];
  g_u32* pv = (g_u32*)a.pv;
  g_cu8* gacc = (g_cu8*)acc;
  const uint32_t vmask = a.val_mask, base = (uint32_t)W.rb0;
  const int32_t nrow = (int32_t)(W.r1 - W.r0), r0 = (int32_t)(W.r0 - W.rb0);
#pragma unroll
  for (int j = 0; j < kResRowsPerLane; ++j) best[lane + j * kWave] = 0;
  if (kBal) {
    __syncthreads();  // every wave's maxima cleared before any wave folds into them
    gather_block<kFirst ? 0 : 1>(acc, &R.best[0][0], a, wib, lane, cur);
    if (!kFirst) PH_MARK(kPhGather);
  } else {
    wave_lds_sync();
    gather_range<kFirst ? 0 : 1>(acc, W.we0, W.wr, best, a, lane, cur);
  }
  if (kFirst && kBal) {
    // In-block successors send their id if accepting: folded like the remote
    // edges, shared evenly over the lanes.
    for (int32_t k = W.wr + lane; k < W.we1; k += kWave) {
      const uint32_t e = R.e[k];
      const uint32_t x = sent_first(acc, (int32_t)(base + in_succ(e)));
      if (x) atomicMax(&best[in_row(e)], x);
    }
  }
  if (kBal) __syncthreads();  // every wave's folds into these maxima are done
  else wave_lds_sync();
  uint32_t changed = 0, nacc = 0;
#pragma unroll
  for (int j = 0; j < kResRowsPerLane; ++j) {
    const int32_t i = lane + j * kWave;
    if (i < nrow) {
      const int32_t li = r0 + i;
      const int64_t v = (int64_t)base + li;
      uint32_t b = best[i];
      if (kFirst) {
        if (!kBal) {
          const int32_t k1 = i + 1 < nrow ? (int32_t)R.lrow[li + 1] : W.we1;
          for (int32_t k = R.lrow[li]; k < k1; ++k) b = max(b, sent_first(acc, (int32_t)(base + R.e[k])));
        }
        uint32_t isacc = gacc[v] ? 1u : 0u;
        nacc += isacc;
        const uint32_t x = (isacc << 31) | cur | b;
        pv[v] = x;
        R.pv[li] = x;
        changed |= (b | isacc) != 0;
      } else {
        const uint32_t old = R.pv[li];
        if (b > (old & vmask)) {
          const uint32_t x = (old & ~vmask) | b;
          pv[v] = x;
          R.pv[li] = x;
          changed = 1;
        }
      }
    }
  }
  if (acc_count) *acc_count += nacc;
  return __ballot(changed) != 0;
}

// One sweep of the block's rows.  Every thread of the block calls it.
// Resident mode: the pass over edges to other blocks' rows (every edge in the
// reset sweep), then up to kLocalPasses LDS passes over in-block edges, which
// stop once a pass changes nothing in the block.  *local_fix (block-uniform)
// records that the last LDS pass changed nothing: while it holds and the first
// pass changes nothing, the block's values are at the fixpoint of the values
// gathered, and the LDS passes are skipped.  Always inline: where the compiler
// called it, a sweep of 300,000 vertices took 23.3 us, and 17.7 inlined (a
// barrier after each).
template <bool kFirst, bool kBal>
__device__ __forceinline__ uint32_t sweep_rows(const LoopArgs& a, const uint8_t* acc, const WaveRows W, int wib, int lane,
                               uint32_t cur, uint32_t* acc_count, bool* local_fix) {
  __shared__ uint32_t s_any;
  if (W.resident) {
    uint32_t ch = sweep_resident<kFirst, kBal>(a, acc, W, wib, lane, cur, acc_count);
    PH_MARK(kPhRemote);
    if (threadIdx.x == 0) s_any = 0;
    __syncthreads();
    if (ch && lane == 0) atomicOr(&s_any, 1u);
    __syncthreads();
    const bool run = kFirst || s_any != 0 || !*local_fix;
    *local_fix = false;
    PH_MARK(kPhRemoteWait);
    if (run) {
      for (int p = 0; p < kLocalPasses; ++p) {
        __syncthreads();  // every thread has read s_any; the previous pass's LDS values are complete
        if (threadIdx.x == 0) s_any = 0;
        __syncthreads();
        const uint32_t lc = kBal ? local_pass_bal(a, W, wib, lane) : local_pass(a, W, lane, cur);
        if (lc && lane == 0) atomicOr(&s_any, 1u);
        ch |= lc;
        __syncthreads();
        PH_COUNT(kPhLocalPasses, 1);
        if (s_any == 0) {
          *local_fix = true;
          break;
        }
      }
    } else {
      *local_fix = true;
    }
    __syncthreads();  // every thread has read s_any
    PH_MARK(kPhLocal);
    return ch;
  }
  uint32_t ch = 0;
  if (W.r1 > W.r0) {
    // Tiles in the order values travel: a row takes values from its
    // successors, so when most edges point to higher rows values flow from
    // high ids to low and the tiles go downwards, otherwise upwards; a tile
    // then sees the values its neighbours produced earlier in the same sweep.
    const int64_t last = W.r0 + ((W.r1 - W.r0 - 1) / kTileRows) * kTileRows;
    if (W.ascending) {
      for (int64_t t0 = W.r0; t0 <= last; t0 += kTileRows)
        ch |= sweep_tile<kFirst, kBal>(a, acc, t0, min(W.r1, t0 + kTileRows), g_lds.tile[wib], lane, cur, acc_count);
    } else {
      for (int64_t t0 = last; t0 >= W.r0; t0 -= kTileRows)
        ch |= sweep_tile<kFirst, kBal>(a, acc, t0, min(W.r1, t0 + kTileRows), g_lds.tile[wib], lane, cur, acc_count);
    }
  }
  PH_MARK(kPhStream);
  return ch;
}

// Appends v (where take) to frontier F with one counter update per wave;
// returns the number appended by the wave (wave-uniform).
__device__ __forceinline__ uint32_t frontier_append(int32_t* F, uint32_t* cnt, bool take, int32_t v, int lane) {
  const uint64_t m = __ballot(take);
  if (m == 0) return 0;
  const int first = __ffsll((unsigned long long)m) - 1;
  uint32_t base = 0;
  if (lane == first) base = __hip_atomic_fetch_add(cnt, (uint32_t)__popcll(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  base = (uint32_t)__shfl((int)base, first, kWave);
  const uint64_t below = lane ? (~0ull >> (kWave - lane)) : 0ull;
  if (take) F[base + (uint32_t)__popcll(m & below)] = v;
  return (uint32_t)__popcll(m);
}

// Sets, with one atomic per 32-bit word, the bits of bitmap `mark` for the
// rows v0 + l (l = 0..63) whose lane l is set in m (wave-uniform m).
__device__ __forceinline__ void mark_rows(uint32_t* mark, int64_t v0, unsigned long long m, int lane) {
  if (m == 0) return;
  const uint32_t sh = (uint32_t)(v0 & 31);
  const int64_t w0 = v0 >> 5;
  const unsigned long long lo = m << sh;
  uint32_t part = 0;
  if (lane == 0) part = (uint32_t)lo;
  else if (lane == 1) part = (uint32_t)(lo >> 32);
  else if (lane == 2) part = sh ? (uint32_t)(m >> (64 - sh)) : 0u;
  if (part) atomicOr(&mark[w0 + lane], part);
}

__device__ __forceinline__ bool bit_set(const uint32_t* b, uint32_t v) { return (b[v >> 5] >> (v & 31)) & 1u; }

// Lane of this wave whose slice of the combined list holds slot q: the last
// lane whose first slot is <= q (binary search over the lanes with shuffles;
// every lane of the wave must call it).
__device__ __forceinline__ int slot_owner(uint32_t q, uint32_t first) {
  int lo = 0;
#pragma unroll
  for (int step = kWave / 2; step > 0; step >>= 1) {
    const uint32_t f = (uint32_t)__shfl((int)first, lo + step, kWave);
    if (f <= q) lo += step;
  }
  return lo;
}

// Filtered stream mode, direction switch (dopt): a sweep whose frontier (the
// rows that grew in the previous sweep, set in `keep`) is small runs as a
// push round over the transposed CSR instead of a pull over every row.  A
// wave takes 64 words of `keep` at a time and deals their set rows out to its
// lanes; a lane raises each predecessor v of its row w with an atomic max of
// what w sends, behind v's
// own accepting bit and the iteration tag (the reset sweep wrote every row
// with both, so the words compare by value); a predecessor that grows is set
// in `mark`.  A row with more than kPushHub predecessors is queued in LDS and
// pushed by the whole wave after the step (64 predecessors at a time), so it
// does not hold up its wave.  The result is that of the filtered pull: both
// fold, into each row, what its grown successors send.  Returns the wave's
// count of raises that grew a row (a row raised twice counts twice: an upper
// bound on the next frontier, zero exactly when nothing grew).
constexpr int32_t kPushHub = 64;
__shared__ int32_t g_hubq[kWavesPerBlock][kWave];
__shared__ uint32_t g_hubn[kWavesPerBlock];

__device__ __forceinline__ bool push_raise(const LoopArgs& a, uint32_t* mark, int32_t v, uint32_t x, uint32_t cur) {
  if ((uint32_t)v >= (uint32_t)a.n) return false;
  const uint32_t word = (bit_set(a.accb, (uint32_t)v) ? kAccBit : 0u) | cur | x;
  const uint32_t old = __hip_atomic_fetch_max(&a.pv[v], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if ((old & a.val_mask) >= x) return false;
  atomicOr(&mark[v >> 5], 1u << (v & 31));
  return true;
}

__device__ __forceinline__ uint32_t push_round_filt(const LoopArgs& a, const uint32_t* keep, uint32_t* mark,
                                                    uint32_t cur, int64_t gw, int64_t nw, int wib, int lane) {
  g_u32* pvg = (g_u32*)a.pv;
  g_ci32* rrow = (g_ci32*)a.rrow_ptr;
  g_ci32* rcol = (g_ci32*)a.rcol;
  const uint32_t n = (uint32_t)a.n;
  uint32_t grew = 0;
  // Which of the wave's next eight steps find a row set: the words of eight
  // steps read together (small frontiers leave most words empty; a wave with one
  // step would only read its words twice).
  const bool ahead = a.words > nw * kWave;
  uint32_t live = ~0u;
  int it = 0;
  for (int64_t w0 = gw * kWave; w0 < a.words; w0 += nw * kWave, ++it) {
    if (ahead && (it & 7) == 0) {
      uint32_t x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int64_t wi = w0 + i * nw * kWave + lane;
        x[i] = wi < a.words ? keep[wi] : 0u;
      }
      live = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) live |= __ballot(x[i] != 0) != 0 ? 1u << i : 0u;
    }
    if (((live >> (it & 7)) & 1u) == 0) continue;
    if (lane == 0) g_hubn[wib] = 0;
    wave_lds_sync();
    // The rows set in the wave's 64 words, dealt out one per lane per step
    // (rows that grow together sit in the same words).
    const int64_t wi = w0 + lane;
    const uint32_t bits = wi < a.words ? keep[wi] : 0u;
    const uint32_t c = (uint32_t)__popc(bits);
    uint32_t incl = c;
    for (int off = 1; off < kWave; off <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)incl, off, kWave);
      if (lane >= off) incl += y;
    }
    const uint32_t first = incl - c;
    const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
    for (uint32_t s0 = 0; s0 < total; s0 += kWave) {
      const uint32_t q = s0 + (uint32_t)lane;
      const int o = slot_owner(q, first);
      const uint32_t ob = (uint32_t)__shfl((int)bits, o, kWave);
      const uint32_t of = (uint32_t)__shfl((int)first, o, kWave);
      if (q >= total) continue;
      uint32_t b = ob;
      for (uint32_t t = of; t < q; ++t) b &= b - 1u;  // drop the owner's set bits before this slot's
      const uint32_t w = (uint32_t)((w0 + o) << 5) + (uint32_t)__builtin_ctz(b);
      if (w >= n) continue;
      const int32_t k0 = rrow[w], k1 = rrow[w + 1];
      if (k1 - k0 > kPushHub) {
        const uint32_t hq = atomicAdd(&g_hubn[wib], 1u);
        if (hq < (uint32_t)kWave) {
          g_hubq[wib][hq] = (int32_t)w;
          continue;
        }
      }
      const uint32_t x = sent_word(pvg[w], (int32_t)w, cur, a.val_mask, a.tag_mask);
      if (!x) continue;
      for (int32_t k = k0; k < k1; ++k) grew += push_raise(a, mark, rcol[k], x, cur) ? 1u : 0u;
    }
    wave_lds_sync();
    const uint32_t hubs = min(g_hubn[wib], (uint32_t)kWave);
    for (uint32_t h = 0; h < hubs; ++h) {  // wave-uniform: the whole wave pushes each queued row
      const uint32_t w = (uint32_t)g_hubq[wib][h];
      const uint32_t x = sent_word(pvg[w], (int32_t)w, cur, a.val_mask, a.tag_mask);
      if (!x) continue;
      const uint32_t k1 = (uint32_t)rrow[w + 1];
      for (uint32_t k = (uint32_t)rrow[w] + (uint32_t)lane; k < k1; k += kWave) grew += push_raise(a, mark, rcol[k], x, cur) ? 1u : 0u;
    }
    wave_lds_sync();  // the queue is read before the next step clears it
  }
  return wave_sum_u32(grew);
}

// Brings `keep` into LDS for a filtered sweep (every thread of the block).  The
// successors of a sweep are anywhere, so their bits cost a 64-byte request each
// that the first-level cache seldom holds, and the second level not either
// where 32 workgroups bring 32 bitmaps of their own.  A bitmap of more than
// kFoldWords words is folded, and a set bit then only says that the successor
// may have grown: its value is read, which can do no harm.  The fold is used
// while few of its bits are set (a quarter at most) and reading the whole
// bitmap, coalesced, costs less than the bits of the block's edges (a word is
// 1/16 of a 64-byte request; the line is drawn at 8 words per edge).  A bitmap of
// 2 KB stays in the first-level cache: 5,000 vertices, streamed, 189 us with its
// copy and 181 without; of 7.5 KB 303 and 315 us (60,000 vertices).
__device__ __forceinline__ bool fold_bits(const LoopArgs& a, const uint32_t* keep, uint32_t size, int32_t edges) {
  if (a.words <= kFoldMinWords) return false;
  if (a.words > kFoldWords && ((int64_t)size * kFoldDiv > kFoldWords * 32 || a.words > (int64_t)edges * 8)) return false;
  g_u32* src = (g_u32*)const_cast<uint32_t*>(keep);
  constexpr int kPer = 8;
  __syncthreads();  // the sweep before has been read
  for (int p0 = threadIdx.x; p0 < kFoldWords && p0 < a.words; p0 += kPer * kBlock) {
    uint32_t x[kPer] = {};
    for (int64_t q0 = p0; q0 < a.words; q0 += kFoldWords) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) x[i] |= q0 + i * kBlock < a.words ? src[q0 + i * kBlock] : 0u;
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) g_lds.filt.bits[p0 + i * kBlock] = x[i];
  }
  __syncthreads();
  return true;
}

// Filtered stream mode (every block streams its rows, a grid barrier after
// every sweep): one sweep of the wave's rows in tiles, in the order values
// travel.  Like sweep_tile, but an edge's successor w is gathered only if its
// bit is set in `keep` -- in the reset sweep the accepting set (w sends its
// id), later the rows that grew in the previous sweep (w sends its value).  A
// successor left out either sends nothing new (not accepting) or has not grown
// since the previous sweep, whose rows already folded in its value: the
// fixpoint is unchanged.  The rows that grow (in the reset sweep: that get a
// nonzero value) are set in `mark` for the next sweep.  Returns the rows that
// grew (the wave's count).
//
// A tile is a chain of dependent reads -- row offsets, successors, their bits,
// the values behind the set ones -- and a wave holds one tile, so the chain and
// not the bytes is what a sweep costs unless most rows grow.  The row offsets
// are therefore read two tiles ahead and the successors one tile ahead, which
// leaves the bits and the values, and a tile none of whose bits is set ends
// after the bits.  Measured (3.3M vertices, 4.2M edges, 256 workgroups, a
// handful of rows growing): 55 us a sweep, reading ahead 46, bits in LDS 26.
enum class Pull { kReset, kGrown, kAll };
// The rows of a pull, and where the sending rows lie: tiles t0, t0 + step, ...
// of [r0, r1); only successors base <= w < base + span are looked at.
struct PullRows {
  int64_t r0, r1, t0, step;
  bool ascending;
  uint32_t base, span;
};

// kReset: the first sweep of an iteration.  kGrown: `keep` are the rows that
// grew.  kAll (banded sweeps): every successor's value is read, and the
// successors on the far side of the band (above it where bands ascend) are
// set in `keep` for the sweep after the bands.
template <Pull kPull>
__device__ __forceinline__ uint32_t sweep_stream_filt(const LoopArgs& a, const PullRows& W, int wib, int lane,
                                                      uint32_t cur, uint32_t* keep, uint32_t* mark, uint32_t size,
                                                      int32_t edges) {
  constexpr bool kFirst = kPull == Pull::kReset, kAll = kPull == Pull::kAll;
  uint32_t grown = 0;
  const bool fold = !kAll && uniform(fold_bits(a, keep, size, edges) ? 1 : 0);
  const int64_t tiles = (W.r1 - W.r0 + kFiltRows - 1) / kFiltRows;
  const int nt = uniform(W.t0 < tiles ? (int)((tiles - W.t0 + W.step - 1) / W.step) : 0);
  if (nt > 0) {
    constexpr int kRows = kFiltRows / kWave;
    FiltLds& L = g_lds.filt;
    const bool exact = a.words <= kFoldWords;
    g_ci32* row_ptr = (g_ci32*)a.row_ptr;
    g_ci32* colp = (g_ci32*)a.col;
    g_u32* pv = (g_u32*)a.pv;
    g_u32* keepg = (g_u32*)keep;
    const uint32_t base = W.base, span = W.span, vmask = a.val_mask, tmask = a.tag_mask;
    auto first_row = [&](int t) { return W.r0 + (W.t0 + (W.ascending ? t : nt - 1 - t) * W.step) * kFiltRows; };
    auto rows_of = [&](int64_t r0) { return (int)min((int64_t)kFiltRows, W.r1 - r0); };
    // Row offsets of tile t: entry lane + 64 j, past the end the last one.
    auto load_rp = [&](int t, int32_t* rp) {
      const int64_t r0 = first_row(t);
      const int nr = rows_of(r0);
#pragma unroll
      for (int j = 0; j <= kRows; ++j) rp[j] = __builtin_nontemporal_load(row_ptr + r0 + min(lane + j * kWave, nr));
    };
    auto load_col = [&](int32_t c0, int32_t e1, uint32_t* w) {
#pragma unroll
      for (int u = 0; u < kEdgesPerLane; ++u) {
        const int32_t k = lane + u * kWave;
        w[u] = k < e1 - c0 ? (uint32_t)__builtin_nontemporal_load(colp + c0 + k) : 0xffffffffu;
      }
    };
    int32_t rp[kRows + 1], rpn[kRows + 1];
    uint32_t w[kEdgesPerLane], wn[kEdgesPerLane];
    load_rp(0, rp);
    if (nt > 1) load_rp(1, rpn);
    load_col(uniform(rp[0]), uniform(rp[kRows]), w);
    for (int t = 0; t < nt; ++t) {
      const int64_t r0 = first_row(t);
      const int nr = rows_of(r0);
      const int32_t e0 = uniform(rp[0]), e1 = uniform(rp[kRows]);
      int32_t lo[kRows], hi[kRows];
      uint32_t best[kRows];
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        const int32_t nx = __shfl(rp[j + 1], 0, kWave), dn = __shfl_down(rp[j], 1, kWave);
        lo[j] = rp[j];
        hi[j] = lane == kWave - 1 ? nx : dn;
        best[j] = 0;
      }
      bool hit = false;  // wave-uniform: some successor of the tile sends
      for (int32_t c0 = e0;;) {
        uint32_t bits[kEdgesPerLane];
        if (kAll) {
          const uint32_t n = (uint32_t)a.n, far = W.ascending ? (uint32_t)W.r1 : 0u;
          const uint32_t nfar = W.ascending ? n - (uint32_t)W.r1 : (uint32_t)W.r0;
#pragma unroll
          for (int u = 0; u < kEdgesPerLane; ++u) {
            bits[u] = w[u] < n ? 1u : 0u;
            if (w[u] - far < nfar) atomicOr(&keep[w[u] >> 5], 1u << (w[u] & 31));
          }
        } else if (fold) {
#pragma unroll
          for (int u = 0; u < kEdgesPerLane; ++u)
            bits[u] = w[u] - base < span ? L.bits[(w[u] >> 5) & (kFoldWords - 1)] >> (w[u] & 31) : 0u;
          if (kFirst && !exact) {
#pragma unroll
            for (int u = 0; u < kEdgesPerLane; ++u)
              if (bits[u] & 1u) bits[u] = keepg[w[u] >> 5] >> (w[u] & 31);
          }
        } else {
#pragma unroll
          for (int u = 0; u < kEdgesPerLane; ++u)
            bits[u] = w[u] - base < span ? keepg[w[u] >> 5] >> (w[u] & 31) : 0u;
        }
        const bool lastc = e1 - c0 <= kTileEdges;
        if (!lastc) {
          load_col(c0 + kTileEdges, e1, wn);
        } else if (t + 1 < nt) {
          // The next tile's successors and the row offsets of the one after (no
          // reads past the last tile: the values' would wait behind them).
          load_col(uniform(rpn[0]), uniform(rpn[kRows]), wn);
#pragma unroll
          for (int j = 0; j <= kRows; ++j) rp[j] = rpn[j];
          load_rp(min(t + 2, nt - 1), rpn);
        }
        uint32_t some = 0;
#pragma unroll
        for (int u = 0; u < kEdgesPerLane; ++u) some |= bits[u];
        if (__ballot(some & 1u) != 0) {
          uint32_t x[kEdgesPerLane];
#pragma unroll
          for (int u = 0; u < kEdgesPerLane; ++u) {
            x[u] = 0;
            if (bits[u] & 1u) x[u] = kFirst ? w[u] + 1u : sent_word(pv[w[u]], (int32_t)w[u], cur, vmask, tmask);
          }
#pragma unroll
          for (int u = 0; u < kEdgesPerLane; ++u) L.val[wib][lane + u * kWave] = x[u];
          wave_lds_sync();
          fold_chunk<kRows>(L.val[wib], lo, hi, c0, min(kTileEdges, e1 - c0), a.hub, lane, best);
          wave_lds_sync();
          hit = true;
        }
#pragma unroll
        for (int u = 0; u < kEdgesPerLane; ++u) w[u] = wn[u];
        if (lastc) break;
        c0 += kTileEdges;
      }
      if (!kFirst && !hit) continue;
      uint32_t old[kRows];
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        const int r = lane + j * kWave;
        old[j] = r >= nr ? 0u : kFirst ? keepg[(r0 + r) >> 5] >> ((r0 + r) & 31) : pv[r0 + r];
      }
#pragma unroll
      for (int j = 0; j < kRows; ++j) {
        const int r = lane + j * kWave;
        bool grew = false;
        if (r < nr) {
          if (kFirst) {
            pv[r0 + r] = (old[j] << 31) | cur | best[j];
            grew = best[j] != 0;
          } else if (best[j] > (old[j] & vmask)) {
            pv[r0 + r] = (old[j] & ~vmask) | best[j];
            grew = true;
          }
        }
        const unsigned long long gm = __ballot(grew);
        mark_rows(mark, r0 + j * kWave, gm, lane);
        grown += (uint32_t)__popcll(gm);
      }
    }
  }
  PH_MARK(kPhStream);
  return grown;
}

// Clears this block's share of the words of bitmap b (word-striped over the grid).
__device__ __forceinline__ void clear_share(uint32_t* b, int64_t words, int blk, int nb) {
  for (int64_t i = (int64_t)blk * kBlock + threadIdx.x; i < words; i += (int64_t)nb * kBlock) b[i] = 0u;
}

// Filtered stream mode: passes over all rows take kQuads times 4 (flags: 16)
// consecutive rows per lane at a time, their loads before their stores.  With a
// row per lane at a time one workgroup that solves a large graph has too few
// bytes in flight, and such a pass is a chain of memory latencies (10^6
// vertices in one of 256 workgroups: from the last sweep of an iteration to the
// first of the next 3.2 ms; eight rows per lane, one by one, 0.96; so 0.39).
// A wave's rows begin at a multiple of kFiltAlign, which is all that 16-byte
// accesses need, and the arrays of the workspace at one of 256 bytes.  (Rounded
// to 32, a sixth of the workgroups of a graph with 130 rows per wave had none:
// 300,000 vertices, streamed, 376 us, so 364.)
constexpr int kQuads = 4;
constexpr int kRowBatch = 8;  // output passes

// The accepting flags as a bitmap (and, where accw is given, copied there as 0
// or 1); the waves take every nw-th batch of vertices.  Returns the wave's count
// of accepting vertices in every lane.
__device__ __forceinline__ uint32_t build_accb(const uint8_t* acc, uint8_t* accw, uint32_t* accb, int64_t n, int64_t gw,
                                               int64_t nw, int lane) {
  constexpr int64_t kStep = kWave * 16 * kQuads;
  g_cu8* src = (g_cu8*)acc;
  const bool wide = ((uintptr_t)acc & 15) == 0;  // the caller's flags may lie anywhere
  uint32_t cnt = 0;
  for (int64_t b0 = gw * kStep; b0 < n; b0 += nw * kStep) {
    u32x4 x[kQuads];
#pragma unroll
    for (int j = 0; j < kQuads; ++j) {
      const int64_t v = b0 + (j * kWave + lane) * 16;
      x[j] = u32x4{0u, 0u, 0u, 0u};
      if (wide && v + 16 <= n) {
        x[j] = *(g_u32x4*)(src + v);
      } else if (v < n) {
        uint32_t y[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (v + i < n) y[i >> 2] |= (uint32_t)src[v + i] << (8 * (i & 3));
        x[j] = u32x4{y[0], y[1], y[2], y[3]};
      }
    }
#pragma unroll
    for (int j = 0; j < kQuads; ++j) {
      const int64_t v = b0 + (j * kWave + lane) * 16;
      uint32_t y[4] = {x[j].x, x[j].y, x[j].z, x[j].w}, half = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t t = ((((y[i] & 0x7f7f7f7fu) + 0x7f7f7f7fu) | y[i]) >> 7) & 0x01010101u;  // 1 per nonzero byte
        y[i] = t;
        half |= ((t | t >> 7 | t >> 14 | t >> 21) & 15u) << (4 * i);
      }
      if (accw && v + 16 <= n) {
        *(g_u32x4*)(accw + v) = u32x4{y[0], y[1], y[2], y[3]};
      } else if (accw && v < n) {
        for (int i = 0; i < 16 && v + i < n; ++i) accw[v + i] = (uint8_t)((half >> i) & 1u);
      }
      cnt += (uint32_t)__popc(half);
      const uint32_t other = (uint32_t)__shfl_xor((int)half, 1, kWave);
      if ((lane & 1) == 0 && v < n) accb[v >> 5] = half | other << 16;
    }
  }
  return wave_sum_u32(cnt);
}

// Map 0 for the rows [r0, r1): the reset alone, where the accepting vertices
// then push what they send.
__device__ __forceinline__ void reset_rows(const LoopArgs& a, int64_t r0, int64_t r1, uint32_t cur, int lane) {
  g_u32* pv = (g_u32*)a.pv;
  for (int64_t b0 = r0; b0 < r1; b0 += kWave * 4 * kQuads) {
    uint32_t w[kQuads];
#pragma unroll
    for (int j = 0; j < kQuads; ++j) {
      const int64_t v = b0 + (j * kWave + lane) * 4;
      w[j] = v < r1 ? a.accb[v >> 5] >> (v & 31) : 0u;
    }
#pragma unroll
    for (int j = 0; j < kQuads; ++j) {
      const int64_t v = b0 + (j * kWave + lane) * 4;
      if (v + 4 <= r1) {
        *(g_u32x4*)(pv + v) = u32x4{w[j] << 31 | cur, (w[j] >> 1) << 31 | cur, (w[j] >> 2) << 31 | cur, (w[j] >> 3) << 31 | cur};
      } else {
        for (int i = 0; i < 4 && v + i < r1; ++i) pv[v + i] = (w[j] >> i) << 31 | cur;
      }
    }
  }
}

// Calls f(v, packed value of v) for every row v of the wave (lane-strided),
// kBatch rows of a lane loaded together.
template <int kBatch = 1, typename F>
__device__ __forceinline__ void for_own_rows(const LoopArgs& a, const WaveRows& W, int lane, F f) {
  if (kBatch > 1) {
    g_u32* pv = (g_u32*)a.pv;
    for (int64_t v0 = W.r0 + lane; v0 < W.r1; v0 += kWave * kBatch) {
      uint32_t x[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) x[j] = v0 + j * kWave < W.r1 ? pv[v0 + j * kWave] : 0u;
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (v0 + j * kWave < W.r1) f(v0 + j * kWave, x[j]);
    }
  } else if (W.resident) {
#pragma unroll
    for (int j = 0; j < kResRowsPerLane; ++j) {
      int64_t v = W.r0 + lane + j * kWave;
      if (v < W.r1) f(v, g_lds.res.pv[v - W.rb0]);
    }
  } else {
    for (int64_t v = W.r0 + lane; v < W.r1; v += kWave) f(v, a.pv[v]);
  }
}

// Resident mode set-up: sort each gather batch of the wave's edges by target
// (key = target << 8 | row offset), so that the 64 lanes of one gather
// instruction read neighbouring addresses and touch few cache lines.  Bitonic
// network over kSortSlots keys held kSortSlots / 64 per lane (element i lives
// in lane i % 64, slot i / 64); padding keys are 0xffffffff and sort last.
__device__ void sort_gather_batches(int32_t we0, int32_t we1, int lane) {
  ResLds& R = g_lds.res;
  for (int32_t k0 = we0; k0 < we1; k0 += kWave * kGatherBatch) {
    const int cnt = (int)min((int32_t)(kWave * kGatherBatch), we1 - k0);
    uint32_t key[kSortPerLane];
#pragma unroll
    for (int u = 0; u < kSortPerLane; ++u) {
      const int i = lane + u * kWave;
      key[u] = i < cnt ? R.e[k0 + i] : 0xffffffffu;
    }
#pragma unroll
    for (int k = 2; k <= kSortSlots; k <<= 1) {
#pragma unroll
      for (int j = k >> 1; j > 0; j >>= 1) {
        if (j >= kWave) {
          const int ju = j / kWave;
#pragma unroll
          for (int u = 0; u < kSortPerLane; ++u) {
            if (u & ju) continue;
            const int i = lane + u * kWave;
            const bool asc = (i & k) == 0;
            const uint32_t x = key[u], y = key[u | ju];
            const bool sw = asc ? (x > y) : (x < y);
            key[u] = sw ? y : x;
            key[u | ju] = sw ? x : y;
          }
        } else {
#pragma unroll
          for (int u = 0; u < kSortPerLane; ++u) {
            const int i = lane + u * kWave;
            const uint32_t y = (uint32_t)__shfl_xor((int)key[u], j, kWave);
            const bool asc = (i & k) == 0;
            const bool lower = (i & j) == 0;
            const uint32_t lo = min(key[u], y), hi = max(key[u], y);
            key[u] = (lower == asc) ? lo : hi;
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kSortPerLane; ++u) {
      const int i = lane + u * kWave;
      if (i < cnt) R.e[k0 + i] = key[u];
    }
  }
}

// Banded sweeps (filtered stream mode of the whole device): where nearly all
// edges point one way, the rows are swept once in kBandCount bands in the order
// values travel, each by the whole grid and with a barrier after it.  A band's
// first pass reads every successor's value: those before the band have theirs
// already, so only edges inside the band are taken again, in passes over the
// band's rows that look at successors grown in the pass before, until few grow.
// The rows grown in a band's last pass, and the successors on the far side of
// the band, are left to the sweeps that follow.  An edge is so read about once
// where the plain sweeps read it as often as its successor grows.  Used once
// per iteration, when a frontier has become too large for push rounds or is
// about to (from n / 64 rows where it doubles: frontiers that shrink from
// there are cheaper swept or pushed).  Bands end at n / 2^(5 - i/2) rows, so the
// edges inside a band are few.  Measured (33.5M vertices, 134M edges downwards,
// detection): 14.7 ms without, 6.7 so; begun at n / 8 rows only 1 ms more; 5, 7,
// 9, 15 bands 8.2, 7.2, 6.8, 6.9; left at 1/16, 1/32, 1/64 of a band's
// rows (15 bands) 7.3, 7.2, 7.0, at 1/512 (9 bands) 7.2.  Smaller graphs of the
// kind have too little in a band to fill the device, and its eleven barriers and
// more cost them more than whole sweeps (without / with bands, direction switch
// off and on): 2M vertices 1.29 / 2.10 and 1.61 / 2.13 ms, 4M 2.61 / 3.06 and
// 2.25 / 2.48, 6M 3.68 / 3.70 and 2.78 / 2.64, 8M 4.92 / 4.05 and 3.55 / 2.70;
// the line lies at 6.3M (kBandMinN), and below it runs a kernel without them.
// Edges the other way bring values back into bands that are done: of 6.4M
// vertices' edges 1 in 10^6 and 1 in 330,000 wrong 2.72 and 4.49 ms with bands, 3.29
// and 5.42 without; 1 in 10^5 21.6 and 15.6, 1 in 3,000 (8M) 8.3 and 5.9 (16M 25.3
// and 18.2), 1 in 100 5.8 and 4.8.  The line is 1 in 131,072 of the sample (eight
// rows per thread).
__device__ __forceinline__ int64_t band_end(int32_t n, int band) {
  if (band < 0) return 0;
  if (band >= kBandCount - 1) return n;
  const int up = kBandCount - 1 - band;
  const uint64_t x = (uint64_t)n >> (up >> 1);
  return (int64_t)(((up & 1) ? x * 46341 >> 16 : x) & ~(uint64_t)31);
}
__device__ __forceinline__ PullRows band_rows(int32_t n, int band, int dir) {
  PullRows r = {};
  const int64_t lo = band_end(n, band - 1), hi = band_end(n, band);
  const int64_t m = ((int64_t)n + 31) & ~(int64_t)31;  // bands of rows n..1 begin at multiples of 32, too
  r.r0 = dir > 0 ? lo : band == kBandCount - 1 ? 0 : m - ((hi + 31) & ~(int64_t)31);
  r.r1 = dir > 0 ? hi : min((int64_t)n, m - lo);
  r.ascending = dir > 0;
  return r;
}

// The whole MAP computation for one graph, run by `nb` cooperating blocks of
// which this is block `b`; `logical` is the block's position in row order.
// Every block of the set must call it; c is the set's zeroed control block.
// kAsync selects the fixpoint control at compile time: asynchronous sweeps with
// quiescence detection, or a grid barrier after every sweep (required for a
// single block, for untagged values, and with MAP_FLAG_SYNC_SWEEPS).
// kWin: st carries the loop's state in and out; returns true when the next
// iterations are to be windowed (win_body), false when the run has ended.
template <typename C, bool kAsync, bool kEarly, bool kFilt = false, bool kWin = false, bool kBands = false>
__device__ __forceinline__ bool map_body(const LoopArgs& a, C* c, const int nb, const int b, const int logical,
                         LoopState* st = nullptr) {
  BlockLds& S = g_lds;
  __shared__ uint32_t s_red[kWavesPerBlock];
  __shared__ unsigned long long s_red64[kWavesPerBlock];
  __shared__ int32_t s_wit[kWavesPerBlock];

  const int lane = threadIdx.x & (kWave - 1);
  // In a scalar register, and with it the wave's row ranges, which would
  // otherwise fill the vector registers and be spilled across the barriers
  // (push rounds at 1.1M vertices 13.1 us each, so 11.7; asynchronous detection
  // of 300,000 vertices 375 us, so 359).
  const int wib = uniform((int)(threadIdx.x / kWave));
  // The asynchronous bodies use the balanced layout of the resident slice and
  // LDS pass; the barrier-mode bodies keep the per-lane row fold.
  constexpr bool kBal = kAsync;
  if (!kWin || !st->resumed) PH_START();
  if (kEarly && threadIdx.x == 0) g_early = 0;  // ordered before its first use by the set-up's barriers
  // Tag epoch of this call: left by the previous call on the workspace (an
  // earlier kernel); block 0 writes the next one only after the first grid
  // barrier, which every block reaches after this read.
  const uint32_t tbase = a.epoch ? *a.epoch : 0u;

  // Row ranges of this block and wave.
  int64_t rows_per_block = ((int64_t)a.n + nb - 1) / nb;
  int64_t rows_per_wave = (rows_per_block + kWavesPerBlock - 1) / kWavesPerBlock;
  if (kFilt) {
    rows_per_wave = (rows_per_wave + kFiltAlign - 1) / kFiltAlign * kFiltAlign;
    rows_per_block = rows_per_wave * kWavesPerBlock;
  }
  const int64_t rb0 = min((int64_t)a.n, (int64_t)logical * rows_per_block);
  const int64_t rb1 = min((int64_t)a.n, rb0 + rows_per_block);
  const int push_div = rows_per_block >= kPushFarRows ? kPushFar : kPushNear;
  WaveRows W;
  W.rb0 = rb0;
  W.rb1 = rb1;
  W.r0 = min(rb1, rb0 + (int64_t)wib * rows_per_wave);
  W.r1 = min(rb1, W.r0 + rows_per_wave);
  W.we0 = W.we1 = 0;
  int32_t block_edges;
  uint32_t dir_down = 0, dir_up = 0;  // kBands: sampled edges of the block to lower and to higher rows
  {
    const int32_t eb0 = a.row_ptr[rb0], eb1 = a.row_ptr[rb1];
    block_edges = eb1 - eb0;
    // n < 2^24 keeps every staged remote key (successor << 8 | row offset)
    // below 0xffffffff, the padding key of the sort and the gather.
    W.resident = !kFilt && !a.force_stream && a.n < (1 << 24) && rows_per_wave <= kResWaveRows &&
                 (int64_t)eb1 - eb0 <= kResEdges;
    W.wr = 0;
    {
      // Direction of the block's edges, from up to 8 rows per thread.
      __shared__ uint32_t s_dir[2];
      if (threadIdx.x < 2) s_dir[threadIdx.x] = 0;
      __syncthreads();
      uint32_t down = 0, up = 0;
      for (int64_t r = rb0 + threadIdx.x, i = 0; r < rb1 && i < 8; r += kBlock, ++i) {
        const int32_t k1 = a.row_ptr[r + 1];
        for (int32_t k = a.row_ptr[r]; k < k1; ++k) {
          if ((int64_t)a.col[k] < r) ++down;
          else if ((int64_t)a.col[k] > r) ++up;
        }
      }
      down = wave_sum_u32(down);
      up = wave_sum_u32(up);
      if (lane == 0) {
        atomicAdd(&s_dir[0], down);
        atomicAdd(&s_dir[1], up);
      }
      __syncthreads();
      W.ascending = s_dir[0] > s_dir[1];
      dir_down = s_dir[0];
      dir_up = s_dir[1];
      __syncthreads();
    }
    if (W.resident) {
      // Each wave stages its rows' edges in its part of the block's slice:
      // first the edges to rows of other blocks (gathered from memory each
      // sweep), then the edges to rows of this block grouped by row (folded
      // from LDS by the row's lane).
      W.we0 = a.row_ptr[W.r0] - eb0;
      W.we1 = a.row_ptr[W.r1] - eb0;
      const uint32_t base = (uint32_t)rb0, span = (uint32_t)(rb1 - rb0);
      const uint64_t below = lane ? (~0ull >> (kWave - lane)) : 0ull;
      uint32_t nr = 0;
      for (int64_t r = W.r0 + lane; r < W.r1; r += kWave) {
        const int32_t k1 = a.row_ptr[r + 1];
        for (int32_t k = a.row_ptr[r]; k < k1; ++k) nr += (uint32_t)a.col[k] - base >= span ? 1u : 0u;
      }
      W.wr = W.we0 + (int32_t)wave_sum_u32(nr);
      int32_t nrem = 0, lrun = W.wr;
      for (int64_t rc = W.r0; rc < W.r1; rc += kWave) {
        const int64_t r = rc + lane;
        int32_t k = 0, k1 = 0;
        if (r < W.r1) {
          k = a.row_ptr[r];
          k1 = a.row_ptr[r + 1];
        }
        uint32_t dl = 0;
        for (int32_t kk = k; kk < k1; ++kk) dl += (uint32_t)a.col[kk] - base < span ? 1u : 0u;
        uint32_t incl = dl;
        for (int off = 1; off < kWave; off <<= 1) {
          const uint32_t y = (uint32_t)__shfl_up((int)incl, off, kWave);
          if (lane >= off) incl += y;
        }
        int32_t lpos = lrun + (int32_t)(incl - dl);
        if (r < W.r1) S.res.lrow[r - rb0] = (uint16_t)lpos;
        lrun += (int32_t)__shfl((int)incl, kWave - 1, kWave);
        const uint32_t off = (uint32_t)(r - W.r0);
        for (;;) {
          const bool act = k < k1;
          if (__ballot(act) == 0) break;
          const int32_t t = act ? a.col[k] : 0;
          const bool rem = act && (uint32_t)t - base >= span;
          const uint64_t mr = __ballot(rem);
          if (rem) S.res.e[W.we0 + nrem + __popcll(mr & below)] = ((uint32_t)t << 8) | off;
          nrem += __popcll(mr);
          if (act && !rem) S.res.e[lpos++] = (kBal ? (off << 16) : 0u) | ((uint32_t)t - base);
          k += act ? 1 : 0;
        }
      }
      wave_lds_sync();
      // A scalar branch, so that the call starts a block of its own: in the
      // block that ends the divergent loops above, the compiler has placed
      // copies of registers that live across the call before it restores the
      // lanes that left those loops (the copies then miss every lane).
      if (__builtin_amdgcn_readfirstlane(W.wr - W.we0) > 0) sort_gather_batches(W.we0, W.wr, lane);
    }
    __syncthreads();
    if (kBal && W.resident) {  // block-uniform
      if (lane == 0) {
        g_rseg[wib] = W.we0;
        g_rpre[wib + 1] = W.wr - W.we0;
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        g_rpre[0] = 0;
        for (int i = 1; i <= kWavesPerBlock; ++i) g_rpre[i] += g_rpre[i - 1];
      }
      __syncthreads();
    }
  }

  Grid<C> g;
  g.c = c;
  g.gen = kWin ? st->gen : 0;
  g.nblocks = nb;
  g.ngroups = min(nb, kMaxGroups);
  g.group = b % g.ngroups;
  g.group_size = nb / g.ngroups + ((b % g.ngroups) < (nb % g.ngroups) ? 1 : 0);
  g.rank = b;
  uint8_t* acc = a.propagate ? const_cast<uint8_t*>(a.acc_in) : a.accw;
  const PullRows own = {W.r0, W.r1, 0, 1, W.ascending, 0u, (uint32_t)a.n};  // kFilt

  // Block-level sum of per-wave u32 values followed by one striped atomic.
  auto block_add_count = [&](uint32_t x, int set) {
    x = wave_sum_u32(x);
    if (lane == 0) s_red[wib] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t t = 0;
      for (int i = 0; i < kWavesPerBlock; ++i) t += s_red[i];
      if (t) __hip_atomic_fetch_add(&c->sets[set][b % kStripes].count, t, __ATOMIC_RELAXED,
                                    __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  };
  // Reads of a completed set (after the barrier that closed it).
  auto read_count = [&](int set) {
    uint32_t t = lane < kStripes ? ld_agent(&c->sets[set][lane].count) : 0u;
    return wave_sum_u32(t);
  };
  // Any wave of the block changed a row: one flag per block.  Each wave first
  // completes its writes, so that the leader's release after this barrier
  // (change report, or grid barrier) covers every wave's new values.
  auto block_any = [&](uint32_t ch) {
    if (lane == 0) s_red[wib] = ch;
    wave_writes_done();
    __syncthreads();
    uint32_t any = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) any |= s_red[i];
    __syncthreads();
    return any ? 1u : 0u;
  };
  // Filtered stream sweeps report how many rows grew (the barrier sums them):
  // the next sweep's frontier size.
  auto block_count = [&](uint32_t x) {
    if (lane == 0) s_red[wib] = x;
    wave_writes_done();
    __syncthreads();
    uint32_t t = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) t += s_red[i];
    __syncthreads();
    return t;
  };

  uint32_t count_prev = 0;  // |A_k| of the last completed iteration
  uint32_t rtag = 0;        // push: frontier round, the same in every block
  uint32_t cnt_next = 0;    // kFilt: |A_k| of the iteration that begins
  int band_dir = 0;         // kBands: the way nearly all edges point (1: to lower rows), or 0
  uint32_t gsw = 0;         // filtered stream sweeps: sweeps so far, the same in every block
  int32_t k = 0;
  int64_t total_sweeps = 0;  // whole-graph sweeps, summed over the iterations
  int32_t status = MAP_OK, found = 0, witness = 0;
  int32_t left = 0;
  bool acc_from_pv = false;  // acc_out comes from the accepting bits of the packed values
  bool ok = true;
  uint32_t tot = 0;
  bool win_ok = false;              // kWin: every block's edges fit the windowed iterations' registers
  uint32_t del1 = ~0u, del2 = ~0u;  // kWin: flags removed by iterations k - 1 and k - 2
  const bool resumed = kWin && st->resumed;
  if (resumed) {
    k = st->k;
    total_sweeps = st->sweeps;
  }
  // Asynchronous sweeps need the iteration tag; without it (n >= 2^30) every
  // sweep ends with a grid barrier.
  constexpr bool sync = !kAsync;

  {
    // Own packed values start in iteration 0 (tag 0), so no value left in the
    // workspace by an earlier call is mistaken for one of this call; A_1 is
    // copied to the working flags and counted.
    uint32_t cnt = 0;
    if (kFilt) {
      // Only the bitmap of A_1: a packed value is read in an iteration after
      // its reset alone, and the reset writes every row.
      const uint32_t c = build_accb(a.acc_in, a.propagate ? nullptr : a.accw, a.accb, a.n,
                                    (int64_t)b * kWavesPerBlock + wib, (int64_t)nb * kWavesPerBlock, lane);
      cnt = lane == 0 ? c : 0u;
    }
    for (int64_t v = W.r0 + lane; !kFilt && v < W.r1; v += kWave) {
      a.pv[v] = 0u;
      if (a.push) a.mark[v] = 0u;
      if (!a.propagate && !resumed) {
        uint8_t x = a.acc_in[v] ? 1 : 0;
        a.accw[v] = x;
        cnt += x;
      }
    }
    if (kFilt) clear_share(a.chg, 3 * a.words, b, nb);
    block_add_count(cnt, g.gen % kSets);
    if (kBands && threadIdx.x == 0) {
      Stripe& st0 = c->sets[g.gen % kSets][b % kStripes];
      __hip_atomic_fetch_add(&st0.digest, (unsigned long long)dir_down, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_add(&st0.sweeps, (unsigned long long)dir_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (kWin && threadIdx.x == 0) {
      const int64_t rpb = win_rows(a.n, nb), w0 = min((int64_t)a.n, logical * rpb), w1 = min((int64_t)a.n, w0 + rpb);
      if (!a.win || a.propagate || rpb > kWinMaxRows || nb > kMaxGang ||
          (int64_t)a.row_ptr[w1] - a.row_ptr[w0] > kWinBlockEdges)
        __hip_atomic_fetch_add(&c->sets[g.gen % kSets][b % kStripes].nonzero, 1u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
    ok = grid_sync_inline(g, 0, nullptr);
    if (!ok) goto aborted;
    count_prev = resumed ? st->count : read_count((g.gen - 1) % kSets);
    cnt_next = count_prev;
    if (kBands) {
      const int set = (g.gen - 1) % kSets;
      const unsigned long long dn = wave_sum_u64(
          lane < kStripes ? __hip_atomic_load(&c->sets[set][lane].digest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull);
      const unsigned long long up = wave_sum_u64(
          lane < kStripes ? __hip_atomic_load(&c->sets[set][lane].sweeps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull);
      band_dir = uniform(up * kBandWrong <= dn ? 1 : dn * kBandWrong <= up ? -1 : 0);
    }
    if (kWin) {
      const uint32_t t = lane < kStripes ? ld_agent(&c->sets[(g.gen - 1) % kSets][lane].nonzero) : 0u;
      win_ok = wave_sum_u32(t) == 0;
    }
    PH_MARK(kPhSetup);
    if (!a.propagate && count_prev == 0) { left = 0; goto done; }
  }

  for (;;) {
    k++;
    // Iteration tag: values written in iteration k carry the tag of k; a
    // reader that finds another tag takes the reset value instead.
    const uint32_t cur = iter_tag(a.tag_mask, a.tag_shift, tbase, k);
    uint32_t nacc = 0;       // accepting rows of this block in A_k (reset sweep)
    uint32_t cnt_k = kFilt ? cnt_next : 0u;  // |A_k|
    int64_t s = 0;           // sweeps of this block in iteration k
    int band = -1, pass = 0; // kBands: the band being swept and its passes so far
    bool banded = false;
    uint32_t tot_prev = cnt_k;  // kBands: the frontier before the last
    bool local_fix = false;  // resident: the block's values are at the fixpoint of its in-block edges
    // One loop for both fixpoint controls, so that each sweep variant is
    // inlined once.
    //  - sync: a grid barrier after every sweep carries the changed count.
    //  - asynchronous (the reset is each block's first sweep): blocks sweep
    //    their rows without waiting for one another; values only grow, so
    //    reads of stale remote values are safe.  A sweep that changed
    //    something releases its writes and bumps `dirty`; a sweep that changed
    //    nothing, started after reading dirty == d (then an acquire), reports
    //    quiet {k, d+1}.  When every block reports quiet for the current value
    //    of `dirty`, no change happened while any of those sweeps ran and every
    //    change before them was visible to them, so all rows are at the
    //    fixpoint: block 0 then publishes done = k.
    const uint32_t tag = (uint32_t)k;
    uint32_t d_seen = 0xffffffffu;  // async: counter value of this block's last quiet sweep (wave 0)
    // Async: start of this fixpoint computation on the device wall clock
    // (wave 0), against which kIterTicks bounds the sweeping.
    const uint64_t t_iter = wall_clock64();
    // After a sweep: the barrier (sync) or the change / quiet report (async).
    // Returns false when the launch must stop.
    auto report = [&](uint32_t any, uint32_t d0) -> bool {
      // A row that reached its own id in this sweep (block_any's barrier has
      // ordered every wave's record before this read); published before the
      // barrier or the release below.
      if (kEarly && threadIdx.x == 0 && g_early)
        __hip_atomic_fetch_max(&c->early, g_early, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (sync) {
        const bool counts = !kFilt && s == 1 && !a.propagate;
        if (counts) block_add_count(nacc, g.gen % kSets);
        if (!grid_sync_inline(g, any, &tot)) return false;
        if (counts) cnt_k = read_count((g.gen - 1) % kSets);
        return true;
      }
      if (threadIdx.x == 0) {
        if (any) {
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
          __hip_atomic_fetch_add(&c->dirty, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
          __hip_atomic_store(&c->quiet[b], ((unsigned long long)tag << 32) | (uint32_t)(d0 + 1u),
                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
      if (wib == 0) d_seen = any ? 0xffffffffu : d0;
      return true;
    };
    // MAP_FLAG_EARLY: after a sweep, the block's rows whose value is their
    // own id (kept out of the sweep code, whose register allocation it would
    // otherwise share); block_any's barrier orders the records before report
    // reads them.
    auto early_scan = [&]() {
      if (!kEarly) return;
      for_own_rows(a, W, lane, [&](int64_t v, uint32_t x) {
        if ((x & a.val_mask) == (uint32_t)v + 1u) atomicMax(&g_early, (uint32_t)v + 1u);
      });
    };
    // Sum over the block of a per-wave count (every thread gets it).
    auto block_sum_waves = [&](uint32_t x) {
      if (lane == 0) s_red[wib] = x;
      __syncthreads();
      uint32_t t = 0;
      for (int i = 0; i < kWavesPerBlock; ++i) t += s_red[i];
      __syncthreads();
      return t;
    };
    if (sync && a.push) {
      // Frontier rounds over the transposed CSR: every vertex whose value grew
      // sends its new value to each predecessor with an atomic max on the
      // packed word (same accepting bit and tag, so the words compare by
      // value); the predecessors that grew form the next frontier.  A grid
      // barrier ends each round and carries the size of the next frontier.
      // The reset gives every row map 0 and puts the accepting rows in the
      // first frontier (they send their own id).
      g_u32* pvg = (g_u32*)a.pv;
      g_cu8* gacc = (g_cu8*)acc;
      ++rtag;
      if (b == 0 && threadIdx.x == 0) st_agent(&c->fcount[1], 0u);
      uint32_t napp = 0;
      for (int64_t v0 = W.r0; v0 < W.r1; v0 += kWave) {
        const int64_t v = v0 + lane;
        uint32_t isacc = 0;
        if (v < W.r1) {
          isacc = gacc[v] ? 1u : 0u;
          pvg[v] = (isacc << 31) | cur;
          if (isacc) a.mark[v] = rtag;
        }
        nacc += isacc;
        napp += frontier_append(a.front[0], &c->fcount[0], isacc != 0, (int32_t)v, lane);
      }
      if (!a.propagate) block_add_count(nacc, g.gen % kSets);
      uint32_t bapp = block_sum_waves(napp);
      if (!grid_sync_inline(g, bapp, &tot)) goto aborted;
      if (!a.propagate) cnt_k = read_count((g.gen - 1) % kSets);
      s = 1;
      int fc = 0;
      uint32_t S = tot;
      const int64_t gw = (int64_t)b * kWavesPerBlock + wib, nw = (int64_t)nb * kWavesPerBlock;
      while (S > 0) {
        if (s > (int64_t)a.n + 1) { status = MAP_ENOTCONVERGED; break; }
        ++rtag;
        // This round reads frontier fc; its counter is next written in the
        // round after (the barrier ending this round orders the clear).
        if (b == 0 && threadIdx.x == 0) st_agent(&c->fcount[fc], 0u);
        const int32_t* F = a.front[fc];
        int32_t* Fn = a.front[fc ^ 1];
        uint32_t* cn = &c->fcount[fc ^ 1];
        napp = 0;
        for (int64_t i0 = gw * kWave; i0 < (int64_t)S; i0 += nw * kWave) {
          const int64_t i = i0 + lane;
          int32_t k = 0, k1 = 0;
          uint32_t x = 0;
          if (i < (int64_t)S) {
            const int32_t w = F[i];
            x = sent_word(pvg[w], w, cur, a.val_mask, a.tag_mask);
            if (x) {
              k = a.rrow_ptr[w];
              k1 = a.rrow_ptr[w + 1];
            }
          }
          for (;;) {
            const bool act = k < k1;
            if (__ballot(act) == 0) break;
            bool grew = false;
            int32_t v = 0;
            if (act) {
              v = a.rcol[k++];
              const uint32_t word = ((gacc[v] ? 1u : 0u) << 31) | cur | x;
              const uint32_t old = __hip_atomic_fetch_max(&a.pv[v], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              grew = (old & a.val_mask) < x &&
                     __hip_atomic_exchange(&a.mark[v], rtag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != rtag;
            }
            napp += frontier_append(Fn, cn, grew, v, lane);
          }
        }
        bapp = block_sum_waves(napp);
        if (!grid_sync_inline(g, bapp, &tot)) goto aborted;
        S = tot;
        fc ^= 1;
        s++;
      }
    } else {
    {
      // The reset sweep of iteration k.
      uint32_t d0 = 0;
      if (!sync) {
        if (threadIdx.x == 0) {
          s_red[1] = ld_agent(&c->dirty);
          __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        d0 = s_red[1];
        __syncthreads();
      }
      PH_MARK(kPhOther);
      uint32_t c1;
      if (kFilt) {
        // Sweep gsw reads the rows that grew in sweep gsw - 1 (the reset sweep:
        // the accepting set), marks its own in bitmap gsw % 3 and clears
        // bitmap (gsw + 1) % 3 for the next sweep.
        clear_share(a.chg + ((gsw + 1) % 3) * a.words, a.words, b, nb);
        uint32_t* markb = a.chg + (gsw % 3) * a.words;
        // (A scalar branch, as the one on the frontier's size below: the same in every lane.)
        if (uniform(a.dopt && rows_per_block >= kPushResetRows && (int64_t)cnt_k * push_div < (int64_t)a.n ? 1 : 0)) {
          // Few accepting vertices: the reset, then a push round from them,
          // instead of a pull over every row (10^6 vertices, one workgroup:
          // 0.05 ms against 0.8; 33.5M vertices, 256 workgroups: 0.1 against 0.34).
          reset_rows(a, W.r0, W.r1, cur, lane);
          if (!grid_sync_inline(g, 0, nullptr)) goto aborted;
          c1 = push_round_filt(a, a.accb, markb, cur, (int64_t)b * kWavesPerBlock + wib,
                               (int64_t)nb * kWavesPerBlock, wib, lane);
        } else {
          c1 = sweep_stream_filt<Pull::kReset>(a, own, wib, lane, cur, a.accb, markb, cnt_k, block_edges);
        }
        ++gsw;
      } else {
        c1 = sweep_rows<true, kBal>(a, acc, W, wib, lane, cur, &nacc, &local_fix);
      }
      s = 1;
      early_scan();
      const uint32_t any1 = kFilt ? block_count(c1) : block_any(c1);
      if (!report(any1, d0)) goto aborted;
      PH_MARK(kPhReport);
      PH_COUNT(kPhSweeps, 1);
      PH_COUNT(kPhQuiet, any1 ? 0 : 1);
    }
    for (;;) {
      uint32_t d0 = 0;
      if (sync) {
        if (tot == 0 && !(kBands && band >= 0)) break;
        if (kEarly && ld_agent(&c->early)) break;  // read after the barrier: the same in every block
        if (s > (int64_t)a.n + 1) { status = MAP_ENOTCONVERGED; break; }
      } else {
        if (wib == 0) {
          uint32_t cmd = 0;  // 0 sweep, 1 done, 2 abort
          const uint64_t t0 = wall_clock64();
          for (;;) {
            if (ld_agent(&c->done) == tag) { cmd = 1; break; }
            if (kEarly && ld_agent(&c->early)) { cmd = 1; break; }
            // Sweeping that has not settled within kIterTicks ends the launch,
            // however often the counter moves.
            if (wall_clock64() - t_iter > kIterTicks) { cmd = 2; break; }
            const uint32_t d = ld_agent(&c->dirty);
            if (d != d_seen) { cmd = 0; d0 = d; break; }
            if (b == 0) {
              const unsigned long long want = ((unsigned long long)tag << 32) | (uint32_t)(d + 1u);
              bool mine = true;
              for (int i = lane; i < nb; i += kWave)
                mine &= __hip_atomic_load(&c->quiet[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == want;
              if (__ballot(!mine) == 0 && ld_agent(&c->dirty) == d) {
                if (lane == 0) __hip_atomic_store(&c->done, tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                cmd = 1;
                break;
              }
            }
            if (wall_clock64() - t0 > kWaitTicks || ld_agent((const uint32_t*)&c->abort)) { cmd = 2; break; }
            __builtin_amdgcn_s_sleep(1);
          }
          if (lane == 0) {
            if (cmd == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (cmd == 2) st_agent((uint32_t*)&c->abort, 1u);
            s_red[0] = cmd;
            s_red[1] = d0;
          }
        }
        __syncthreads();
        const uint32_t cmd = s_red[0];
        d0 = s_red[1];
        __syncthreads();
        PH_MARK(kPhWait);
        if (cmd == 2) goto aborted;
        if (cmd == 1) break;
      }
      uint32_t c2;
      if (kFilt) {
        uint32_t* markb = a.chg + (gsw % 3) * a.words;
        uint32_t* keepb = a.chg + ((gsw + 2) % 3) * a.words;
        uint32_t* restb = a.chg + 3 * a.words;  // kBands: rows that some row may not have folded in when the bands end
        PullRows rows = own;
        if (kBands) {
          const int heavy = uniform(band < 0 && !banded && band_dir != 0 && ((int64_t)tot * push_div >= (int64_t)a.n ||
                                      ((int64_t)tot * kBandGrow >= (int64_t)a.n && tot / 2 > tot_prev)) ? 1 : 0);
          tot_prev = tot;
          const int leave = uniform(band >= 0 && (pass >= kBandPasses || (int64_t)tot * kBandLeave <=
                                                      band_end(a.n, band) - band_end(a.n, band - 1)) ? 1 : 0);
          if (heavy || leave) {
            if (heavy) {
              clear_share(restb, a.words, b, nb);
              banded = true;
            } else {
              // Of the band's rows, those that grew in its last pass are left over.
              const PullRows r = band_rows(a.n, band, band_dir);
              for (int64_t i = (r.r0 >> 5) + (int64_t)b * kBlock + threadIdx.x; i < ((r.r1 + 31) >> 5); i += (int64_t)nb * kBlock)
                if (keepb[i]) atomicOr(&restb[i], keepb[i]);
            }
            pass = 0;
            if (++band == kBandCount) band = -1;
            if (heavy || band < 0) {
              // The bitmap is clear (complete) in every block; the barrier carries its size.
              uint32_t left_over = 0;
              if (!heavy) {
                if (!grid_sync_inline(g, 0, nullptr)) goto aborted;
                for (int64_t i = (int64_t)b * kBlock + threadIdx.x; i < a.words; i += (int64_t)nb * kBlock)
                  left_over += (uint32_t)__popc(ld_agent(&restb[i]));
              }
              if (!grid_sync_inline(g, block_count(wave_sum_u32(left_over)), &tot)) goto aborted;
              if (!heavy && uniform((int)tot) == 0) break;
              keepb = restb;
            }
          }
          if (band >= 0) {
            rows = band_rows(a.n, band, band_dir);
            rows.t0 = (int64_t)b * kWavesPerBlock + wib;
            rows.step = (int64_t)nb * kWavesPerBlock;
            rows.base = (uint32_t)rows.r0;
            rows.span = (uint32_t)(rows.r1 - rows.r0);
          }
        }
        clear_share(a.chg + ((gsw + 1) % 3) * a.words, a.words, b, nb);
        // tot: the rows that grew in the previous sweep (an upper bound after a
        // push round), the same in every block
        if (kBands && uniform(band >= 0 && pass == 0 ? 1 : 0)) {
          c2 = sweep_stream_filt<Pull::kAll>(a, rows, wib, lane, cur, restb, markb, 0u, 0);
          s += band == 0 ? 0 : -1;
        } else if (uniform(a.dopt && band < 0 && (int64_t)tot * push_div < (int64_t)a.n ? 1 : 0)) {
          const int64_t gw = (int64_t)b * kWavesPerBlock + wib, nw = (int64_t)nb * kWavesPerBlock;
          c2 = push_round_filt(a, keepb, markb, cur, gw, nw, wib, lane);
          PH_MARK(kPhStream);
        } else {
          c2 = sweep_stream_filt<Pull::kGrown>(a, rows, wib, lane, cur, keepb, markb, tot, band < 0 ? block_edges : 0);
          s += band < 0 ? 0 : -1;
        }
        pass++;
        ++gsw;
      } else {
        c2 = sweep_rows<false, kBal>(a, acc, W, wib, lane, cur, nullptr, &local_fix);
      }
      s++;
      early_scan();
      const uint32_t any2 = kFilt ? block_count(c2) : block_any(c2);
      if (!report(any2, d0)) goto aborted;
      PH_MARK(kPhReport);
      PH_COUNT(kPhSweeps, 1);
      PH_COUNT(kPhQuiet, any2 ? 0 : 1);
    }
    }
    // Asynchronous mode: |A_k| is reduced together with the detect pass (same
    // barrier epoch).
    if (!sync && !a.propagate) block_add_count(nacc, g.gen % kSets);
    if (status != MAP_OK) { total_sweeps += s; left = (int32_t)count_prev; acc_from_pv = !a.propagate; break; }
    if (a.propagate) {
      // The blocks' sweep counts, summed at one more barrier.
      if (threadIdx.x == 0 && s)
        __hip_atomic_fetch_add(&c->sets[g.gen % kSets][b % kStripes].sweeps, (unsigned long long)s,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      ok = grid_sync_inline(g, 0, nullptr);
      if (!ok) goto aborted;
      unsigned long long sw = lane < kStripes ? __hip_atomic_load(&c->sets[(g.gen - 1) % kSets][lane].sweeps,
                                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
      total_sweeps += ((int64_t)wave_sum_u64(sw) + nb / 2) / nb;
      break;
    }

    // Detect and strip: witness = max v with map(v) == v; every nonzero map
    // value loses its accepting flag (the flags of this iteration stay in the
    // packed values).
    {
      int32_t wit = 0;
      unsigned long long dig = 0;
      uint32_t nz = 0;
      const bool want_digest = a.digest != 0;
      auto note = [&](int64_t v, uint32_t mv) {
        const uint32_t id = (uint32_t)v + 1u;
        if (mv == id) wit = max(wit, (int32_t)id);
        if (want_digest) dig += mix64(((unsigned long long)id << 32) | mv);
        nz |= mv;
      };
      if (W.resident) {
        // The flag of every map value is cleared without reading it first: no
        // load waits here, and the stores complete before the barrier below
        // (rows that share a map value clear it more than once, harmlessly).
#pragma unroll
        for (int j = 0; j < kResRowsPerLane; ++j) {
          const int64_t v = W.r0 + lane + j * kWave;
          const uint32_t mv = v < W.r1 ? g_lds.res.pv[v - W.rb0] & a.val_mask : 0u;
          if (v < W.r1) note(v, mv);
          if (mv) acc[mv - 1] = 0;
        }
      } else if (kFilt) {
        g_u32* pv = (g_u32*)a.pv;
        g_u8* gacc = (g_u8*)acc;
        for (int64_t b0 = W.r0; b0 < W.r1; b0 += kWave * 4 * kQuads) {
          uint32_t mv[4 * kQuads];
          uint8_t f[4 * kQuads];
#pragma unroll
          for (int j = 0; j < kQuads; ++j) {
            const int64_t v = b0 + (j * kWave + lane) * 4;
            u32x4 x = {0u, 0u, 0u, 0u};
            if (v + 4 <= W.r1) {
              x = *(g_u32x4*)(pv + v);
            } else {
              if (v < W.r1) x.x = pv[v];
              if (v + 1 < W.r1) x.y = pv[v + 1];
              if (v + 2 < W.r1) x.z = pv[v + 2];
            }
            mv[4 * j] = x.x & a.val_mask;
            mv[4 * j + 1] = x.y & a.val_mask;
            mv[4 * j + 2] = x.z & a.val_mask;
            mv[4 * j + 3] = x.w & a.val_mask;
          }
#pragma unroll
          for (int i = 0; i < 4 * kQuads; ++i) {
            const int64_t v = b0 + ((i >> 2) * kWave + lane) * 4 + (i & 3);
            if (v < W.r1) note(v, mv[i]);
            f[i] = mv[i] ? gacc[mv[i] - 1] : (uint8_t)0;
          }
#pragma unroll
          for (int i = 0; i < 4 * kQuads; ++i)
            if (f[i]) gacc[mv[i] - 1] = 0;
        }
      } else {
        for_own_rows(a, W, lane, [&](int64_t v, uint32_t x) {
          const uint32_t mv = x & a.val_mask;
          note(v, mv);
          // Many vertices share a map value: read before writing.
          if (mv != 0 && acc[mv - 1]) acc[mv - 1] = 0;
        });
      }
      wit = wave_max_i32(wit);
      if (want_digest) dig = wave_sum_u64(dig);
      const uint32_t wnz = __ballot(nz != 0) != 0 ? 1u : 0u;
      if (lane == 0) { s_wit[wib] = wit; s_red64[wib] = dig; s_red[wib] = wnz; }
      __syncthreads();
      if (threadIdx.x == 0) {
        int32_t bw = 0;
        unsigned long long bd = 0;
        uint32_t bn = 0;
        for (int i = 0; i < kWavesPerBlock; ++i) { bw = max(bw, s_wit[i]); bd += s_red64[i]; bn |= s_red[i]; }
        Stripe& st = c->sets[g.gen % kSets][b % kStripes];
        if (bw) __hip_atomic_fetch_max(&st.witness, bw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bd) __hip_atomic_fetch_add(&st.digest, bd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (s) __hip_atomic_fetch_add(&st.sweeps, (unsigned long long)s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bn) __hip_atomic_fetch_add(&st.nonzero, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      ok = grid_sync_inline(g, 0, nullptr);
      if (!ok) goto aborted;
      const int set = (g.gen - 1) % kSets;
      // Lane i of every wave reads stripe i; the wave combines them.
      int32_t w2 = 0;
      unsigned long long d2 = 0, sw2 = 0;
      uint32_t nz2 = 0, cnt2 = 0;
      if (lane < kStripes) {
        Stripe& st = c->sets[set][lane];
        w2 = __hip_atomic_load(&st.witness, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        d2 = __hip_atomic_load(&st.digest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sw2 = __hip_atomic_load(&st.sweeps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        nz2 = ld_agent(&st.nonzero);
        cnt2 = ld_agent(&st.count);
      }
      w2 = wave_max_i32(w2);
      d2 = wave_sum_u64(d2);
      sw2 = wave_sum_u64(sw2);
      nz2 = wave_sum_u32(nz2);
      cnt2 = wave_sum_u32(cnt2);
      if (!sync) cnt_k = cnt2;
      PH_MARK(kPhDetect);
      PH_COUNT(kPhIters, 1);
      // MAP_FLAG_EARLY: a published early hit (every block's publication
      // precedes its arrival at the barrier above) is a cycle vertex too.
      if (kEarly) w2 = max(w2, (int32_t)ld_agent(&c->early));
      const bool leader = b == 0 && threadIdx.x == 0;
      if (k >= 2 && cnt_k == 0) {
        // No accepting vertex was left after iteration k-1: iteration k did not happen.
        if (leader && a.trace && k - 1 <= a.trace_cap) a.trace[(int64_t)(k - 2) * 3 + 0] = (uint64_t)count_prev;
        k--;
        left = 0;
        break;
      }
      // Whole-graph sweeps of iteration k: the blocks' sweeps over their
      // count, rounded (in barrier mode every block's count).
      const int64_t sweeps_k = ((int64_t)sw2 + nb / 2) / nb;
      total_sweeps += sweeps_k;
      if (leader && a.trace) {
        if (k >= 2 && k - 1 <= a.trace_cap) a.trace[(int64_t)(k - 2) * 3 + 0] = (uint64_t)(count_prev - cnt_k);
        if (k <= a.trace_cap) {
          uint64_t* row = a.trace + (int64_t)(k - 1) * 3;
          row[0] = 0;
          row[1] = (uint64_t)sweeps_k;
          row[2] = want_digest ? d2 : 0ull;
        }
      }
      if (w2 > 0) {  // some vertex is its own maximal accepting predecessor
        found = 1;
        witness = w2;
        left = (int32_t)cnt_k;
        acc_from_pv = true;
        break;
      }
      if (nz2 == 0) { left = (int32_t)cnt_k; break; }  // every map value is 0: nothing to strip
      if (a.max_iter > 0 && k >= a.max_iter) {
        // Cap reached: count the accepting set left after this strip.
        uint32_t cnt = 0;
        for (int64_t v = W.r0 + lane; v < W.r1; v += kWave) cnt += a.accw[v];
        block_add_count(cnt, g.gen % kSets);
        ok = grid_sync_inline(g, 0, nullptr);
        if (!ok) goto aborted;
        const uint32_t nxt = read_count((g.gen - 1) % kSets);
        if (leader && a.trace && k <= a.trace_cap) a.trace[(int64_t)(k - 1) * 3 + 0] = (uint64_t)(cnt_k - nxt);
        left = (int32_t)nxt;
        if (nxt != 0) status = MAP_ENOTCONVERGED;
        break;
      }
      if (kWin) {
        // Two strips in a row that removed few flags: the next ones will be
        // small too, and one window covers several of them.
        del2 = del1;
        del1 = k >= 2 ? count_prev - cnt_k : ~0u;
        if (win_ok && k >= st->win_from && del1 <= kWinDel && del2 <= kWinDel && cnt_k >= kWinMinLeft) {
          st->k = k;
          st->count = cnt_k;
          st->gen = g.gen;
          st->sweeps = total_sweeps;
          return true;
        }
      }
      if (kFilt) {
        // The accepting set of the next iteration as a bitmap, complete in
        // every block before the reset reads it; the barrier carries its size.
        const uint32_t bc = block_count(build_accb(a.accw, nullptr, a.accb, a.n, (int64_t)b * kWavesPerBlock + wib,
                                                   (int64_t)nb * kWavesPerBlock, lane));
        if (!grid_sync_inline(g, bc, &cnt_next)) goto aborted;
        if (cnt_next == 0) {  // no accepting vertex is left: iteration k + 1 does not happen
          if (leader && a.trace && k <= a.trace_cap) a.trace[(int64_t)(k - 1) * 3 + 0] = (uint64_t)cnt_k;
          left = 0;
          break;
        }
      }
      count_prev = cnt_k;
    }
  }

done:
  // Outputs: map vector (propagate) or the accepting set at exit (detect).
  if (a.propagate && a.map_out) {
    for_own_rows<kFilt ? kRowBatch : 1>(a, W, lane, [&](int64_t v, uint32_t x) { a.map_out[v] = (int32_t)(x & a.val_mask); });
  }
  if (!a.propagate && a.acc_out) {
    for_own_rows<kFilt ? kRowBatch : 1>(a, W, lane, [&](int64_t v, uint32_t x) {
      a.acc_out[v] = acc_from_pv ? (uint8_t)(x >> 31) : a.accw[v];
    });
  }
  if (b == 0 && threadIdx.x == 0) {
    // Words now carry the tags of iterations k and, where a reset was cut
    // short, k - 1: the next call's first tag is past both.
    if (a.epoch) *a.epoch = tbase + (uint32_t)k + 1u;
    a.result->found = found;
    a.result->witness = witness;
    a.result->iterations = a.propagate ? 0 : k;
    a.result->status = status;
    a.result->sweeps = total_sweeps;
    a.result->accepting_left = a.propagate ? 0 : left;
    a.result->reserved = 0;
  }
  PH_MARK(kPhOther);
  PH_STORE(b, nb);
  return false;

aborted:
  if (threadIdx.x == 0) {
    __hip_atomic_store(&a.result->status, (int32_t)MAP_EDEVICE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  return false;
}

// ------------------------------------------------------ windowed iterations --

// Adds what record x brings to row `row` of the block; marks the row in `chg`
// and `pub` when it grew.
__device__ __forceinline__ void win_fold(WinLds& S, uint32_t row, const uint32_t* x, uint32_t* chg) {
  WinRec& r = S.rec[row];
  const uint4 y0 = *reinterpret_cast<const uint4*>(&r.w[0]), y1 = *reinterpret_cast<const uint4*>(&r.w[4]);
  const uint32_t y[8] = {y0.x, y0.y, y0.z, y0.w, y1.x, y1.y, y1.z, y1.w};
  uint32_t any = x[7] > y[7] ? 1u : 0u;
#pragma unroll
  for (int q = 0; q < kWinWords; ++q) any |= x[q] & ~y[q];
  if (!any) return;
#pragma unroll
  for (int q = 0; q < kWinWords; ++q)
    if (x[q] & ~y[q]) atomicOr(&r.w[q], x[q]);
  if (x[7] > y[7]) atomicMax(&r.w[7], x[7]);
  const uint32_t bit = 1u << (row & 31u);
  if (!(chg[row >> 5] & bit)) atomicOr(&chg[row >> 5], bit);
  if (!(S.pub[row >> 5] & bit)) atomicOr(&S.pub[row >> 5], bit);
}

// The iterations of one window on the list of the graph's different records,
// by one workgroup (every block runs them for itself): at most `most`, and up
// to the first that strips an id outside the window, finds a cycle or maps
// nothing.  S.alive is updated; iteration t's image goes to S.own[7 t ..].
__device__ __noinline__ int win_simulate(const WinCtl* wc, const uint32_t nlist, const int most) {
  WinLds& S = g_lds.win;
  __shared__ uint32_t s_img[2][8];
  __shared__ uint32_t s_halt;
  const int tid = threadIdx.x;
  uint32_t x[kWinListRows][8], alive[kWinWords];
#pragma unroll
  for (int i = 0; i < kWinListRows; ++i) {
#pragma unroll
    for (int q = 0; q < 8; ++q) x[i][q] = 0;
    const uint32_t e = (uint32_t)(tid + i * kBlock);
    if (e < nlist) {
      const uint4* p = reinterpret_cast<const uint4*>(&wc->list[e]);
      const uint4 x0 = p[0], x1 = p[1];
      x[i][0] = x0.x, x[i][1] = x0.y, x[i][2] = x0.z, x[i][3] = x0.w;
      x[i][4] = x1.x, x[i][5] = x1.y, x[i][6] = x1.z, x[i][7] = x1.w;
    }
  }
#pragma unroll
  for (int q = 0; q < kWinWords; ++q) alive[q] = S.alive[q];
  if (tid < 16) s_img[tid >> 3][tid & 7] = 0;
  if (tid == 0) s_halt = 0;
  __syncthreads();
  int T = 0;
  for (; T < kWinBits && T < most; ++T) {
    uint32_t* img = s_img[T & 1];
    bool halt = false;
#pragma unroll
    for (int i = 0; i < kWinListRows; ++i) {
      if ((uint32_t)(i * kBlock) >= nlist) continue;
      int q = -1;
      uint32_t word = 0;
#pragma unroll
      for (int t = kWinWords - 1; t >= 0; --t)
        if (x[i][t] & alive[t]) {
          q = t;
          word = x[i][t] & alive[t];
        }
      const uint32_t tail = x[i][7];
      if (q >= 0) {
        const int c = __builtin_clz(word);
        const uint32_t bit = 0x80000000u >> c;
        if (!(img[q] & bit)) atomicOr(&img[q], bit);
        halt = halt || (tail >> 31 ? (tail & 255u) == (uint32_t)(32 * q + c) : tail > S.ids[32 * q + c]);
      } else {
        halt = halt || (tail && !(tail >> 31));
      }
    }
    if (__ballot(halt) && (tid & (kWave - 1)) == 0) s_halt = 1;
    __syncthreads();
    uint32_t any = 0;
#pragma unroll
    for (int q = 0; q < kWinWords; ++q) {
      const uint32_t im = img[q];
      any |= im;
      if (!s_halt) alive[q] &= ~im;
    }
    if (s_halt || !any) break;  // uniform
    // The other image is free: every thread read it before this barrier.
    if (tid < kWinWords) {
      S.own[T * kWinWords + tid] = img[tid];
      s_img[(T & 1) ^ 1][tid] = 0;
    }
    __syncthreads();
  }
  if (tid == 0)
#pragma unroll
    for (int q = 0; q < kWinWords; ++q) S.alive[q] = alive[q];
  __syncthreads();
  return T;
}

// Outer iterations in windows, for graphs whose strips remove only a few flags
// each, so that hundreds of iterations follow one another (config 2: 8 of
// 10,000 flags per strip, K = 1,286).  Such an iteration is bound by the
// latency of its chain of sweeps across blocks (about 160 us at 2^20 vertices),
// not by bytes.  One window takes the chain once for many iterations: S = kWinBits
// accepting ids of A_k, mostly the largest; every vertex v computes
//   mask(v) = the ids of S it reaches over at least one edge (a bit each),
//   low(v)  = the largest id of A_k \ S it reaches,
// one fixpoint of OR and max over the same edges.  Reaching does not depend on
// the flags, so for every following iteration j, while only flags of S have
// been removed,
//   map_j(v) = the larger of low(v) and the largest id of mask(v) that is
//              still accepting,
// and an iteration is the image of one pass over the records.  When an iteration strips
// an id outside the window, or no id of the window is left, the next window is
// chosen.  Most rows reach the same part of the window (some 4,000 different
// records in a million rows of config 2), so the iterations need no barrier
// either: every block runs them on the list of the different records.  Results are those of the plain loop, iteration by iteration.
// A record (mask and low: 32 bytes) is read with two 16-byte loads; the block's
// records fill 128 KB of LDS and its edges, (successor << 12) | row, stay in
// registers.  224 bits and the low word make a whole record of 32 bytes: half
// the bits would take the chain twice as often, twice as many do not fit.
// Measured (2^20 vertices, 4.2M edges, K = 1,286): 45.9 ms against 212 ms of
// asynchronous sweeps per iteration; 62 windows of about 10 sweeps (40 us
// each: the slowest block's passes and the barrier) and 20 iterations.  150,001
// vertices (K = 110 and more, digests on): 2.84 ms against 8.5 ms.  Passes per
// sweep 2 / 3 / 4 / 8: 45.5 / 43.8 / 44.0 / 49.2 ms.
// Returns true to go back to the plain loop: where strips jump about among the
// ids a window lasts one iteration, and where values travel from block to block
// and back its fixpoint, a barrier per sweep, takes several times as long as one
// of asynchronous sweeps.  A path through 900 accepting vertices in random order
// of ids (13,000 vertices, K = 51): 35.9 ms without windows, 42.3 so; through
// 1,500 (20,011 vertices, K = 72) 75 and 94, 206 when three short windows were
// taken at a time and tried again after four iterations.  Leaving after any one
// short window costs some state spaces their windows for a while (159,262 states
// 5.5 ms against 4.4).  (Giving a fixpoint up after four times the plain
// iteration's sweeps, or six times its time, gained no more than its code cost
// where windows pay, half a percent.)
__device__ __noinline__ bool win_body(const LoopArgs& a_, const int nb_, const int b_, const int logical_, LoopState* st) {
  const LoopArgs a = uniform(a_);
  const int nb = uniform(nb_), b = uniform(b_), logical = uniform(logical_);
  WinLds& S = g_lds.win;
  __shared__ uint32_t s_cnt[2];
  __shared__ uint32_t s_red[kWavesPerBlock];
  __shared__ unsigned long long s_red64[kWavesPerBlock];
  __shared__ int32_t s_wit[kWavesPerBlock];
  __shared__ uint32_t s_low[kWavesPerBlock];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wib = tid / kWave;
  const int32_t n = a.n;
  const int64_t rpb = win_rows(n, nb);
  const int32_t rb0 = (int32_t)min((int64_t)n, logical * rpb), rb1 = (int32_t)min((int64_t)n, rb0 + rpb);
  const int nrow = rb1 - rb0;
  WinCtl* wc = a.win;
  WinRec* grec = a.win_rec;
  Grid<Ctrl> g;
  g.c = a.ctrl;
  g.gen = st->gen;
  g.nblocks = nb;
  g.ngroups = min(nb, kMaxGroups);
  g.group = b % g.ngroups;
  g.group_size = nb / g.ngroups + ((b % g.ngroups) < (nb % g.ngroups) ? 1 : 0);
  g.rank = b;
  const uint32_t per_inv = (uint32_t)(((1ull << 32) + rpb - 1) / rpb);  // row -> block, exact below 2^20 rows
  const bool leader = b == 0 && tid == 0;
  auto clear_red = [&](int set) {
    if (b == 0)
      for (int i = tid; i < kStripes * (int)(sizeof(WinRed) / 4) + kMaxGang / 32; i += kBlock)
        st_agent(i < kMaxGang / 32 ? &wc->moved[set][i] : reinterpret_cast<uint32_t*>(&wc->red[set][0]) + (i - kMaxGang / 32), 0u);
  };
  // Barrier; the reduction set of epoch E is written in E, read after the
  // barrier that ends E and cleared by block 0 after the one that ends E + 1.
  auto sync = [&](uint32_t payload, uint32_t* total) {
    const bool ok = grid_sync(g, payload, total);
    clear_red((g.gen + 1) % kSets);
    return ok;
  };
  auto block_sum = [&](uint32_t x) {
    x = wave_sum_u32(x);
    if (lane == 0) s_red[wib] = x;
    __syncthreads();
    uint32_t t = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) t += s_red[i];
    __syncthreads();
    return t;
  };

  // Set-up: the block's edges into registers, those to other blocks' rows in
  // the first nr slots, then those to its own.
  uint32_t edge[kWinSlots];
  int nrem, nloc, nr;
  {
    const int32_t e0 = a.row_ptr[rb0];
    const int m = a.row_ptr[rb1] - e0;
    if (tid < 2) s_cnt[tid] = 0;
    for (int r0 = wib * kWave; r0 < nrow; r0 += kBlock) {
      const int r = r0 + lane;
      const int kb = r < nrow ? a.row_ptr[rb0 + r] - e0 : 0, ke = r < nrow ? a.row_ptr[rb0 + r + 1] - e0 : 0;
      const bool longrow = ke - kb > kWave;
      if (!longrow)
        for (int k = kb; k < ke; ++k) S.row_of[k] = (uint16_t)r;
      unsigned long long lr = __ballot(longrow);
      while (lr) {
        const int src = __ffsll(lr) - 1;
        lr &= lr - 1;
        const int bb = __shfl(kb, src, kWave), ee = __shfl(ke, src, kWave);
        for (int k = bb + lane; k < ee; k += kWave) S.row_of[k] = (uint16_t)(r0 + src);
      }
    }
    __syncthreads();
    const unsigned long long below = lane ? (~0ull >> (kWave - lane)) : 0ull;
    for (int k0 = wib * kWave; k0 < m; k0 += kBlock) {
      const int k = k0 + lane;
      const uint32_t w = k < m ? (uint32_t)a.col[e0 + k] : 0xffffffffu;
      const bool in = w < (uint32_t)n, local = in && w - (uint32_t)rb0 < (uint32_t)nrow;
      const unsigned long long mr = __ballot(in && !local), ml = __ballot(local);
      uint32_t pr = 0, pl = 0;
      if (lane == 0) {
        pr = atomicAdd(&s_cnt[0], (uint32_t)__popcll(mr));
        pl = atomicAdd(&s_cnt[1], (uint32_t)__popcll(ml));
      }
      pr = (uint32_t)__shfl((int)pr, 0, kWave);
      pl = (uint32_t)__shfl((int)pl, 0, kWave);
      if (in) {
        const uint32_t row = S.row_of[k];
        if (local) S.stage[kWinBlockEdges - 1 - (pl + (uint32_t)__popcll(ml & below))] = ((w - (uint32_t)rb0) << 12) | row;
        else S.stage[pr + (uint32_t)__popcll(mr & below)] = (w << 12) | row;
      }
    }
    __syncthreads();
    nrem = (int)s_cnt[0];
    nloc = (int)s_cnt[1];
    nr = (nrem + kBlock - 1) / kBlock;
    // The block's own edges in the order values travel: from the high rows
    // down when most successors are higher.
    uint32_t higher = 0;
    for (int i = tid; i < nloc; i += kBlock) {
      const uint32_t e = S.stage[kWinBlockEdges - 1 - i];
      higher += (e >> 12) > (e & 0xfffu) ? 1u : 0u;
    }
    const bool down = 2 * block_sum(higher) > (uint32_t)nloc;
#pragma unroll
    for (int j = 0; j < kWinSlots; ++j) {
      const int i = tid + (j < nr ? j : j - nr) * kBlock;
      edge[j] = 0;
      if (j < nr ? i < nrem : i < nloc)
        edge[j] = S.stage[j < nr ? i : kWinBlockEdges - 1 - (down ? nloc - 1 - i : i)];
    }
    __syncthreads();
  }
  // Number of the edge in slot j among its kind; valid if below the count.
  auto valid = [&](int j) { return j < nr ? tid + j * kBlock < nrem : tid + (j - nr) * kBlock < nloc; };
  if (b == 0)
    for (int s = 0; s < kSets; ++s) clear_red(s);

  int32_t k = st->k, found = 0, witness = 0, status = MAP_OK, left = 0;
  uint32_t count = st->count;  // accepting vertices left
  uint32_t before = count;     // |A_k|
  int64_t total_sweeps = st->sweeps;
  bool pending = true;         // the trace row of iteration k still lacks its removals
  bool capped = false;
  const bool want_digest = a.digest != 0;
  uint32_t accb = 0;            // accepting flags of the thread's rows at the window's choice
  uint32_t widx = 0xffffffffu;  // a byte per row: its number in the window, or 255
  int windows = 0;
  if (leader) st_agent(&wc->fronts, 0u);
  if (!sync(0, nullptr)) goto aborted;
  PH_MARK(kPhSetup);
  for (;;) {
    // Accepting rows, and the fronts: the ids that the last strip removed.
    const uint32_t accold = accb;
    accb = 0;
    if (tid < kWinMaxRows / 32) S.acc[tid] = 0;
    if (tid == 0) s_cnt[0] = 0;
    __syncthreads();
    uint32_t frontb = 0;
#pragma unroll
    for (int j = 0; j < kWinRows; ++j) {
      const int r = tid + j * kBlock;
      const bool acc = r < nrow && a.accw[rb0 + r] != 0;
      if (acc) accb |= 1u << j;
      const unsigned long long m = __ballot(acc);
      if (lane < 2 && m) S.acc[(j * kBlock + wib * kWave) / 32 + lane] = lane ? (uint32_t)(m >> 32) : (uint32_t)m;
      if (r < nrow && !acc) {
        const uint32_t i = (widx >> (8 * j)) & 255u;
        const bool gone = windows == 0 ? a.pv[rb0 + r] >> 31 != 0   // the plain loop's strip
                          : i != 255u  ? (S.img[i >> 5] << (i & 31u)) >> 31 != 0
                                       : (accold >> j) & 1u;
        if (gone) frontb |= 1u << j;
      }
    }
    if (frontb) atomicAdd(&s_cnt[0], (uint32_t)__popc(frontb));
    __syncthreads();
    if (wib == 0) {  // accepting rows in the words above each word: two words per lane
      const uint32_t lo = (uint32_t)__popc(S.acc[2 * lane]), hi = (uint32_t)__popc(S.acc[2 * lane + 1]);
      uint32_t incl = lo + hi;
      for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_down((int)incl, off, kWave);
        if (lane + off < kWave) incl += y;
      }
      S.accs[2 * lane] = incl - lo;
      S.accs[2 * lane + 1] = incl - lo - hi;
    }
    if (tid == kWave) {
      s_cnt[1] = s_cnt[0] ? __hip_atomic_fetch_add(&wc->fronts, s_cnt[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
      s_cnt[0] = 0;
    }
    __syncthreads();
    // Accepting rows of the block above its row r.
    auto rank_of = [&](int r) { return S.accs[r >> 5] + (uint32_t)__popc(S.acc[r >> 5] & ~(0xffffffffu >> (31 - (r & 31)))); };
#pragma unroll
    for (int j = 0; j < kWinRows; ++j)
      if ((frontb >> j) & 1u) {
        const uint32_t at = s_cnt[1] + atomicAdd(&s_cnt[0], 1u);
        if (at < (uint32_t)kWinFronts) st_agent(&wc->front[at], (uint32_t)logical << 16 | rank_of(tid + j * kBlock));
      }
    if (tid == 0) st_agent(&wc->count[logical], S.accs[0] + (uint32_t)__popc(S.acc[0]));
    if (b == 0 && tid < kWinBits) st_agent(&wc->ids[tid], 0u);
    if (!sync(0, nullptr)) goto aborted;
    uint32_t total = 0;
    for (int i = lane; i < nb; i += kWave) total += ld_agent(&wc->count[i]);
    total = wave_sum_u32(total);
    if (pending && leader && a.trace && k <= a.trace_cap)
      a.trace[(int64_t)(k - 1) * 3] = (uint64_t)(count - total);
    if (capped || total == 0) {
      left = (int32_t)total;
      if (capped && total != 0) status = MAP_ENOTCONVERGED;
      break;
    }
    if (st->shorts >= (st->paid ? kWinShorts : kWinFirstShorts)) goto plain;
    count = total;
    ++windows;
    // The window: as many ids below each front as fill it, the same number for
    // each (those next to be stripped; the largest ids when there is no front).
    if (wib == 0) {
      uint32_t c[4], sum = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        c[i] = 4 * lane + i < nb ? ld_agent(&wc->count[4 * lane + i]) : 0u;
        sum += c[i];
      }
      uint32_t incl = sum;
      for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_down((int)incl, off, kWave);
        if (lane + off < kWave) incl += y;
      }
      uint32_t run = incl - sum;
#pragma unroll
      for (int i = 3; i >= 0; --i) {
        S.suf[4 * lane + i] = run;
        run += c[i];
      }
      wave_lds_sync();
      const uint32_t nf = ld_agent(&wc->fronts);
      const bool top = nf == 0 || nf > (uint32_t)kWinFronts;  // wave-uniform
      uint32_t P = 0xffffffffu;
      if (top) P = lane == 0 ? 0u : P;
      else if ((uint32_t)lane < nf) {
        const uint32_t f = ld_agent(&wc->front[lane]);
        P = S.suf[f >> 16] + (f & 0xffffu);
      }
      uint32_t gap = P < total ? total - P : 0u;  // ids from this front to the next
      for (int i = 0; i < kWave; ++i) {
        const uint32_t o = (uint32_t)__shfl((int)P, i, kWave);
        if (o > P) gap = min(gap, o - P);
        else if (o == P && i < lane) gap = 0;
      }
      uint32_t D = 0;
      for (uint32_t step = 1u << 20; step; step >>= 1)
        if (wave_sum_u32(min(D + step, gap)) <= (uint32_t)kWinBits) D += step;
      S.fp[lane] = P;
      S.fl[lane] = min(D, gap);
    }
    __syncthreads();
    widx = 0xffffffffu;
#pragma unroll
    for (int j = 0; j < kWinRows; ++j) {
      const int r = tid + j * kBlock;
      WinRec x = {};
      if ((accb >> j) & 1u) {
        const uint32_t R = S.suf[logical] + rank_of(r);  // accepting ids above
        uint32_t rank = 0;
        bool in = false;
        for (int i = 0; i < kWinFronts; ++i) {
          const uint32_t P = S.fp[i], len = S.fl[i];
          if (P > R) continue;
          in = in || R - P < len;
          rank += min(R - P, len);
        }
        if (!in) rank = ~0u;
        if (rank < (uint32_t)kWinBits) {
          widx ^= (255u ^ rank) << (8 * j);
          x.w[0] = rank < 32 ? 0x80000000u >> rank : 0u;
#pragma unroll
          for (int q = 1; q < kWinWords; ++q) x.w[q] = (rank >> 5) == (uint32_t)q ? 0x80000000u >> (rank & 31u) : 0u;
          st_agent(&wc->ids[rank], (uint32_t)(rb0 + r) + 1u);
        } else {
          x.w[7] = (uint32_t)(rb0 + r) + 1u;
        }
      }
      if (r < nrow) {
        S.rec[r] = x;
        grec[rb0 + r] = x;
        S.widx[r] = (uint8_t)(widx >> (8 * j));
      }
    }
    // Every accepting row has something to send.
    if (tid < kWinMaxRows / 32) {
      S.chg[0][tid] = S.acc[tid];
      S.chg[1][tid] = 0;
      S.pub[tid] = 0;
    }
    if (tid < 8) S.self[tid] = 0;
    if (b == 0) {  // every block has read the last window's list and digests
      if (tid == 0) st_agent(&wc->listed, 0u);
      if (tid < kWinBits) __hip_atomic_store(&wc->dig[tid], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (!sync(0, nullptr)) goto aborted;
    if (leader) st_agent(&wc->fronts, 0u);
    for (int i = tid; i < kWinBits; i += kBlock) S.ids[i] = ld_agent(&wc->ids[i]);
    PH_MARK(kPhOther);

    // Fixpoint: gathers from other blocks' rows, then passes over the block's
    // own edges from rows raised in the pass before, then a grid barrier.
    int32_t s = 0;
    int cb = 0;  // S.chg[cb]: rows raised and not yet looked at
    if (tid < kMaxGang / 32) S.moved[tid] = ~0u;
    __syncthreads();
    for (;;) {
      constexpr int kBatch = 4;
#pragma unroll
      for (int j0 = 0; j0 < kWinSlots; j0 += kBatch) {
        if (j0 >= nr) continue;
        uint4 x0[kBatch], x1[kBatch];
        bool go[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          if (j0 + u >= kWinSlots) continue;
          asm volatile("" : "+v"(edge[j0 + u]));
          x0[u] = x1[u] = make_uint4(0, 0, 0, 0);
          go[u] = false;
          if (j0 + u < nr && valid(j0 + u)) {
            const uint32_t src = edge[j0 + u] >> 12, blk = __umulhi(src, per_inv);
            go[u] = (S.moved[blk >> 5] >> (blk & 31u)) & 1u;
            if (go[u]) {
              const uint4* p = reinterpret_cast<const uint4*>(grec + src);
              x0[u] = p[0];
              x1[u] = p[1];
            }
          }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          if (j0 + u >= kWinSlots) continue;
          const uint32_t x[8] = {x0[u].x, x0[u].y, x0[u].z, x0[u].w, x1[u].x, x1[u].y, x1[u].z, x1[u].w};
          if (go[u]) win_fold(S, edge[j0 + u] & 0xfffu, x, S.chg[cb]);
        }
      }
      __syncthreads();
      PH_MARK(kPhRemote);
      bool open = true;  // rows raised in the last pass remain to be looked at
      for (int p = 0; p < kWinPasses && open; ++p) {
        uint32_t* cur = S.chg[cb];
        uint32_t* nxt = S.chg[cb ^ 1];
#pragma unroll
        for (int j = 0; j < kWinSlots; ++j) {
          if (j < nr || (j - nr) * kBlock >= nloc) continue;
          asm volatile("" : "+v"(edge[j]));  // nothing derived from it is kept across the passes
          const uint32_t src = edge[j] >> 12, row = edge[j] & 0xfffu;
          if (valid(j) && (((cur[src >> 5] | nxt[src >> 5]) >> (src & 31u)) & 1u)) {
            const WinRec& r = S.rec[src];
            const uint4 x0 = *reinterpret_cast<const uint4*>(&r.w[0]), x1 = *reinterpret_cast<const uint4*>(&r.w[4]);
            const uint32_t x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
            win_fold(S, row, x, nxt);
          }
        }
        __syncthreads();
        uint32_t more = 0;
        if (tid < kWinMaxRows / 32) {
          cur[tid] = 0;
          more = nxt[tid];
        }
        open = __syncthreads_or((int)more) != 0;
        cb ^= 1;
        PH_COUNT(kPhLocalPasses, 1);
      }
      PH_MARK(kPhLocal);
      // Rows that grew go to memory.
      uint32_t any = open ? 1u : 0u;
#pragma unroll
      for (int j = 0; j < kWinRows; ++j) {
        const int r = tid + j * kBlock;
        if (r < nrow && ((S.pub[r >> 5] >> (r & 31)) & 1u)) {
          grec[rb0 + r] = S.rec[r];
          any = 1;
        }
      }
      any = __syncthreads_or((int)any) != 0 ? 1u : 0u;
      if (tid < kWinMaxRows / 32) S.pub[tid] = 0;
      uint32_t tot = 0;
      uint32_t* mv = wc->moved[g.gen % kSets];
      if (tid == 0 && any)
        __hip_atomic_fetch_or(&mv[logical >> 5], 1u << (logical & 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!sync(any, &tot)) goto aborted;
      if (tid < kMaxGang / 32) S.moved[tid] = ld_agent(&mv[tid]);
      PH_MARK(kPhReport);
      PH_COUNT(kPhSweeps, 1);
      PH_COUNT(kPhQuiet, any ? 0 : 1);
      ++s;
      if (tot == 0) break;
      __syncthreads();
    }

    // What accepting rows reach rather than send: a window row's own bit only
    // if some successor sends it, a lower row's word only from its successors.
#pragma unroll
    for (int j = 0; j < kWinRows; ++j)
      if (tid + j * kBlock < nrow) S.own[tid + j * kBlock] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kWinSlots; ++j) {
      if (!valid(j)) continue;
      asm volatile("" : "+v"(edge[j]));
      const uint32_t row = edge[j] & 0xfffu, src = edge[j] >> 12;
      if (!((S.acc[row >> 5] >> (row & 31u)) & 1u)) continue;
      const WinRec* x = j < nr ? grec + src : &S.rec[src];
      const uint32_t i = S.widx[row];
      if (i < (uint32_t)kWinBits) {
        const uint32_t bit = 0x80000000u >> (i & 31u);
        if (x->w[i >> 5] & bit) atomicOr(&S.self[i >> 5], bit);
      } else if (S.rec[row].w[7] == (uint32_t)rb0 + row + 1u) {
        atomicMax(&S.own[row], x->w[7]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kWinRows; ++j) {
      const int r = tid + j * kBlock;
      if (r < nrow && ((accb >> j) & 1u)) {
        const uint32_t i = (widx >> (8 * j)) & 255u;
        if (i < (uint32_t)kWinBits) {
          const uint32_t bit = 0x80000000u >> (i & 31u);
          if (!(S.self[i >> 5] & bit)) S.rec[r].w[i >> 5] &= ~bit;
        } else if (S.rec[r].w[7] == (uint32_t)(rb0 + r) + 1u) {
          S.rec[r].w[7] = S.own[r];
        }
      }
    }
    __syncthreads();

    PH_MARK(kPhOther);
    // Iterations inside the window.
    uint32_t alive[kWinWords];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kWinWords; ++q) alive[q] = __brev((uint32_t)__ballot(lane < 32 && S.ids[32 * q + (lane & 31)] != 0));
    int iters = 0;
    bool end = false, stop = false;
    {
      // Different records of the whole graph: a block drops rows whose record
      // it has already met (a small hash table that may miss some), the rest
      // go to one list.  A window row that reaches itself has an entry of its
      // own too, with bit 31 and its number in w[7].
      uint32_t* tab = S.own;
      for (int i = tid; i < kWinMaxRows; i += kBlock) tab[i] = 0;
      if (tid == 0) s_cnt[0] = 0;
      __syncthreads();
      uint32_t takes = 0, place[kWinRows];
#pragma unroll
      for (int j = 0; j < kWinRows; ++j) {
        const int r = tid + j * kBlock;
        if (r >= nrow) continue;
        const WinRec x = S.rec[r];
        uint32_t h = x.w[7];
#pragma unroll
        for (int q = 0; q < kWinWords; ++q) h = (h ^ x.w[q]) * 0x9E3779B1u;
        h ^= h >> 15;
        bool take = true;
        for (int t = 0; t < 4 && take; ++t) {
          uint32_t* slot = &tab[(h + t) & (kWinMaxRows - 1)];
          uint32_t o = *slot;  // most rows find their record here: no atomic
          if (o == 0) o = atomicCAS(slot, 0u, (uint32_t)r + 1u);
          if (o == 0) break;
          const WinRec& y = S.rec[o - 1];
          bool same = true;
#pragma unroll
          for (int q = 0; q < 8; ++q) same = same && y.w[q] == x.w[q];
          if (same) take = false;
        }
        const uint32_t i = (widx >> (8 * j)) & 255u;
        if (take) takes |= 1u << j;
        if (i < (uint32_t)kWinBits && ((S.self[i >> 5] << (i & 31u)) >> 31)) takes |= 16u << j;
      }
#pragma unroll
      for (int j = 0; j < kWinRows; ++j) {
        place[j] = 0;
        if ((takes >> j) & 17u) place[j] = atomicAdd(&s_cnt[0], (uint32_t)__popc((takes >> j) & 17u));
      }
      __syncthreads();
      if (tid == 0) s_cnt[1] = s_cnt[0] ? __hip_atomic_fetch_add(&wc->listed, s_cnt[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kWinRows; ++j) {
        uint32_t at = s_cnt[1] + place[j];
        WinRec x;
        if ((takes >> j) & 17u) x = S.rec[tid + j * kBlock];
        if ((takes >> j) & 1u) {
          if (at < (uint32_t)kWinList) wc->list[at] = x;
          ++at;
        }
        if ((takes >> j) & 16u) {
          x.w[7] = 0x80000000u | ((widx >> (8 * j)) & 255u);
          if (at < (uint32_t)kWinList) wc->list[at] = x;
        }
      }
      if (!sync(0, nullptr)) goto aborted;
      const uint32_t nlist = ld_agent(&wc->listed);
      int T = 0;
      if (nlist <= (uint32_t)kWinList) {
        if (tid < kWinWords) S.alive[tid] = 0;
        __syncthreads();
        if (tid == 0)
#pragma unroll
          for (int q = 0; q < kWinWords; ++q) S.alive[q] = alive[q];
        __syncthreads();
        T = win_simulate(wc, nlist, a.max_iter > 0 ? a.max_iter - k - 1 : kWinBits);
        uint32_t gone = 0, last = 0;
#pragma unroll
        for (int q = 0; q < kWinWords; ++q) {
          const uint32_t w = S.alive[q];
          gone += (uint32_t)__popc(alive[q] & ~w);
          alive[q] = w;
          if (T > 0) last += (uint32_t)__popc(S.own[(T - 1) * kWinWords + q]);
        }
        if (T > 0) before = count - gone + last;
        count -= gone;
        if (a.trace && b == 0)
          for (int t = tid; t < T && k + t < a.trace_cap; t += kBlock) {
            uint32_t ndel = 0;
            for (int q = 0; q < kWinWords; ++q) ndel += (uint32_t)__popc(S.own[t * kWinWords + q]);
            uint64_t* row = a.trace + (int64_t)(k + t) * 3;
            row[0] = ndel;
            row[1] = (uint64_t)(t ? 1 : s);
            row[2] = 0;
          }
      }
      if (want_digest && T > 0) {
        // Digests of those iterations: a row's word of the window only moves on.
        unsigned long long* dg = reinterpret_cast<unsigned long long*>(S.own + kWinBits * (kWinWords + 1));
        for (int t = tid; t < T; t += kBlock) dg[t] = 0;
        uint32_t live[kWinWords], cur = 0;  // cur: a byte per row, its current word
#pragma unroll
        for (int q = 0; q < kWinWords; ++q) live[q] = __brev((uint32_t)__ballot(lane < 32 && S.ids[32 * q + (lane & 31)] != 0));
        if (tid < kWinWords) S.img[tid] = live[0];
#pragma unroll
        for (int q = 1; q < kWinWords; ++q)
          if (tid == q) S.img[q] = live[q];
        __syncthreads();
        for (int t = 0; t < T; ++t) {
          unsigned long long dig = 0;
#pragma unroll
          for (int j = 0; j < kWinRows; ++j) {
            const int r = tid + j * kBlock;
            if (r >= nrow) continue;
            uint32_t q = (cur >> (8 * j)) & 255u, word = 0;
            while (q < (uint32_t)kWinWords && !(word = S.rec[r].w[q] & S.img[q])) ++q;
            cur = (cur & ~(255u << (8 * j))) | (q << (8 * j));
            const uint32_t mv = word ? S.ids[32 * q + __builtin_clz(word)] : 0u;  // low is 0 here
            dig += mix64(((unsigned long long)((uint32_t)(rb0 + r) + 1u) << 32) | mv);
          }
          dig = wave_sum_u64(dig);
          if (lane == 0) atomicAdd(&dg[t], dig);
          __syncthreads();
          if (tid < kWinWords) S.img[tid] &= ~S.own[t * kWinWords + tid];
          __syncthreads();
        }
        for (int t = tid; t < T; t += kBlock)
          __hip_atomic_fetch_add(&wc->dig[t], dg[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!sync(0, nullptr)) goto aborted;
        if (b == 0 && a.trace)
          for (int t = tid; t < T; t += kBlock)
            if (k + t < a.trace_cap)
              a.trace[(int64_t)(k + t) * 3 + 2] = __hip_atomic_load(&wc->dig[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (T > 0) {
        pending = false;
        k += T;
        iters = T;
        total_sweeps += s + (T - 1);
        uint32_t open = 0;
#pragma unroll
        for (int q = 0; q < kWinWords; ++q) open |= alive[q];
        end = open == 0;
        __syncthreads();
        if (tid < kWinWords) S.img[tid] = S.own[(T - 1) * kWinWords + tid];  // the last strip, for the next window
      }
      PH_MARK(kPhDetect);
      PH_COUNT(kPhIters, T);
    }
    while (!end) {
      if (tid < 8) S.img[tid] = 0;
      __syncthreads();
      int32_t wit = 0;
      unsigned long long dig = 0;
      uint32_t nz = 0, low = 0, lows[kWinRows];
#pragma unroll
      for (int j = 0; j < kWinRows; ++j) {
        const int r = tid + j * kBlock;
        lows[j] = 0;
        if (r >= nrow) continue;
        const uint4 x0 = *reinterpret_cast<const uint4*>(&S.rec[r].w[0]), x1 = *reinterpret_cast<const uint4*>(&S.rec[r].w[4]);
        const uint32_t x[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
        int q = -1;
        uint32_t word = 0;
#pragma unroll
        for (int t = kWinWords - 1; t >= 0; --t)
          if (x[t] & alive[t]) {
            q = t;
            word = x[t] & alive[t];
          }
        uint32_t mv = x[7];
        const uint32_t id = (uint32_t)(rb0 + r) + 1u;
        const int i = q >= 0 ? __builtin_clz(word) : 0;
        const uint32_t top = q >= 0 ? S.ids[32 * q + i] : 0u;
        if (top > mv) {
          mv = top;
          const uint32_t bit = 0x80000000u >> i;
          if (!(S.img[q] & bit)) atomicOr(&S.img[q], bit);
        } else {
          lows[j] = mv;
          low |= mv;
        }
        if (mv == id) wit = max(wit, (int32_t)id);
        if (want_digest) dig += mix64(((unsigned long long)id << 32) | mv);
        nz |= mv;
      }
      wit = wave_max_i32(wit);
      if (want_digest) dig = wave_sum_u64(dig);
      const uint32_t wnz = __ballot(nz != 0) != 0 ? 1u : 0u, wlow = __ballot(low != 0) != 0 ? 1u : 0u;
      if (lane == 0) {
        s_wit[wib] = wit;
        s_red64[wib] = dig;
        s_red[wib] = wnz;
        s_low[wib] = wlow;
      }
      __syncthreads();
      WinRed& red = wc->red[g.gen % kSets][b % kStripes];
      if (tid < kWinWords) {
        if (S.img[tid]) __hip_atomic_fetch_or(&red.img[tid], S.img[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (tid == kWave) {
        int32_t bw = 0;
        unsigned long long bd = 0;
        uint32_t bn = 0, bl = 0;
        for (int i = 0; i < kWavesPerBlock; ++i) {
          bw = max(bw, s_wit[i]);
          bd += s_red64[i];
          bn |= s_red[i];
          bl |= s_low[i];
        }
        if (bw) __hip_atomic_fetch_max(&red.wit, bw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bd) __hip_atomic_fetch_add(&red.dig, bd, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bn) __hip_atomic_fetch_or(&red.nz, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (bl) __hip_atomic_fetch_or(&red.low, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (!sync(0, nullptr)) goto aborted;
      // Lane i of every wave reads stripe i; the wave combines them.
      const WinRed* rd = &wc->red[(g.gen - 1) % kSets][lane & (kStripes - 1)];
      int32_t w2 = __hip_atomic_load(&rd->wit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned long long d2 = __hip_atomic_load(&rd->dig, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint32_t flags2 = ld_agent(&rd->nz) | (ld_agent(&rd->low) << 1), im[kWinWords], ndel = 0;
#pragma unroll
      for (int q = 0; q < kWinWords; ++q) im[q] = ld_agent(&rd->img[q]);
      w2 = wave_max_i32(w2);
      if (lane >= kStripes) d2 = 0;
      if (want_digest) d2 = wave_sum_u64(d2);
      for (int off = 1; off < kStripes; off <<= 1) {
        flags2 |= (uint32_t)__shfl_xor((int)flags2, off, kWave);
#pragma unroll
        for (int q = 0; q < kWinWords; ++q) im[q] |= (uint32_t)__shfl_xor((int)im[q], off, kWave);
      }
#pragma unroll
      for (int q = 0; q < kWinWords; ++q) ndel += (uint32_t)__popc(im[q]);
      PH_MARK(kPhDetect);
      PH_COUNT(kPhIters, 1);
      ++k;
      // The window's sweeps belong to its first iteration; a later one is one
      // pass over the records.
      before = count;
      const int32_t sk = iters == 0 ? s : 1;
      total_sweeps += sk;
      ++iters;
      stop = w2 > 0 || !(flags2 & 1u);
      const bool lowered = !stop && (flags2 & 2u);
      if (leader && a.trace && k <= a.trace_cap) {
        uint64_t* row = a.trace + (int64_t)(k - 1) * 3;
        row[0] = stop || lowered ? 0ull : (uint64_t)ndel;
        row[1] = (uint64_t)sk;
        row[2] = want_digest ? d2 : 0ull;
      }
      pending = lowered;
      if (stop) {
        found = w2 > 0 ? 1 : 0;
        witness = w2;
        left = (int32_t)count;
        break;
      }
      uint32_t open = 0;
      __syncthreads();
      if (tid == 0)
#pragma unroll
        for (int q = 0; q < kWinWords; ++q) S.img[q] = im[q];  // the last strip, for the next window
#pragma unroll
      for (int q = 0; q < kWinWords; ++q) {
        alive[q] &= ~im[q];
        open |= alive[q];
      }
      if (lowered) {
        // Ids below the window lose their flags in memory; the count of A_{k+1}
        // follows with the next window.
#pragma unroll
        for (int j = 0; j < kWinRows; ++j)
          if (lows[j]) a.accw[lows[j] - 1] = 0;
      } else {
        count -= ndel;
      }
      if (a.max_iter > 0 && k >= a.max_iter) capped = true;
      end = lowered || capped || open == 0;
    }
    // The window's removed ids lose their flags in memory.
#pragma unroll
    for (int j = 0; j < kWinRows; ++j) {
      const uint32_t i = (widx >> (8 * j)) & 255u;
      if (i >= (uint32_t)kWinBits) continue;
      uint32_t live = 0;
#pragma unroll
      for (int q = 0; q < kWinWords; ++q) live |= (i >> 5) == (uint32_t)q ? alive[q] & (0x80000000u >> (i & 31u)) : 0u;
      if (!live) a.accw[rb0 + tid + j * kBlock] = 0;
    }
    if (stop) break;
    if (iters < kWinShort) {
      st->shorts += iters == 1 && !st->paid ? kWinFirstShorts : 1;
    } else {
      st->shorts = 0;
      st->paid = 1;
    }
    // Flags that other blocks removed are read next.
    if (pending && !sync(0, nullptr)) goto aborted;
  }
  // Outputs (the accepting flags in memory are those at exit; each thread
  // reads rows that it wrote itself, or that a barrier ordered).
  if (a.acc_out)
#pragma unroll
    for (int j = 0; j < kWinRows; ++j) {
      const int r = tid + j * kBlock;
      if (r < nrow) a.acc_out[rb0 + r] = a.accw[rb0 + r];
    }
  if (leader) {
    if (a.epoch) *a.epoch += (uint32_t)k + 1u;
    a.result->found = found;
    a.result->witness = witness;
    a.result->iterations = k;
    a.result->status = status;
    a.result->sweeps = total_sweeps;
    a.result->accepting_left = left;
    a.result->reserved = 0;
  }
  PH_MARK(kPhOther);
  PH_STORE(b, nb);
  return false;
plain:  // k iterations have been made
  st->k = k;
  st->count = before;
  st->gen = g.gen;
  st->sweeps = total_sweeps;
  st->resumed = 1;
  st->backoff = max(kWinBackoff, 2 * st->backoff);
  st->win_from = k + st->backoff;
  st->shorts = st->paid = 0;
  return true;
aborted:
  if (tid == 0) __hip_atomic_store(&a.result->status, (int32_t)MAP_EDEVICE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return false;
}

// ------------------------------------------------- one workgroup, all in LDS --

// Streamed sweep of small_body: g lanes (a power of two near an eighth of the
// mean degree) fold each row, two rows at a time with eight columns of each per
// lane in flight; rows longer than the wave's stride are folded by the whole
// wave.  A row that sends its own id records its maximum in `own` as it goes:
// the last sweep, which raises nothing, leaves the map value there.
__device__ __forceinline__ uint32_t small_stream(const LoopArgs& a, int32_t base, int g, bool ascending, int wib,
                                                 int lane) {
  SmallLds& S = g_lds.small;
  g_ci32* col = (g_ci32*)(a.col + base);
  const int n = a.n, per = kBlock / g, sub = lane & (g - 1);
  const int steps = (n + per - 1) / per;
  uint32_t changed = 0;
  for (int it = 0; it < steps; it += 2) {
    int r[2];
    uint32_t k[2], e[2];  // unsigned: a step past the last of 2^31 - 1 edges stays above it
    uint32_t x[2] = {0u, 0u};
    bool longrow[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int st = it + p < steps ? (ascending ? it + p : steps - 1 - it - p) : steps;
      r[p] = st * per + wib * (kWave / g) + lane / g;
      k[p] = e[p] = 0;
      if (r[p] < n) {
        k[p] = (uint32_t)S.rp[r[p]];
        e[p] = (uint32_t)max(S.rp[r[p] + 1], S.rp[r[p]]);
      }
      longrow[p] = e[p] - k[p] > (uint32_t)(kSmallBatch * kWave);
      if (longrow[p]) e[p] = k[p];
      k[p] += (uint32_t)sub;
    }
    while (__ballot(k[0] < e[0] || k[1] < e[1])) {
      uint32_t w[2][kSmallBatch];
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int u = 0; u < kSmallBatch; ++u) w[p][u] = k[p] + u * g < e[p] ? (uint32_t)col[k[p] + u * g] : (uint32_t)n;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int u = 0; u < kSmallBatch; ++u) x[p] = max(x[p], S.sent[min(w[p][u], (uint32_t)n)]);
        k[p] += (uint32_t)(kSmallBatch * g);
      }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      for (int off = 1; off < g; off <<= 1) x[p] = max(x[p], (uint32_t)__shfl_xor((int)x[p], off, kWave));
      unsigned long long lr = __ballot(longrow[p] && sub == 0);
      while (lr) {
        const int src = __ffsll(lr) - 1;
        lr &= lr - 1;
        const int rr = __shfl(r[p], src, kWave);
        uint32_t y = 0;
        const uint32_t e1 = (uint32_t)S.rp[rr + 1];
        for (uint32_t kk = (uint32_t)(S.rp[rr] + lane); kk < e1; kk += kSmallBatch * kWave) {
          uint32_t w[kSmallBatch];
#pragma unroll
          for (int u = 0; u < kSmallBatch; ++u) w[u] = kk + u * kWave < e1 ? (uint32_t)col[kk + u * kWave] : (uint32_t)n;
#pragma unroll
          for (int u = 0; u < kSmallBatch; ++u) y = max(y, S.sent[min(w[u], (uint32_t)n)]);
        }
        y = wave_max_u31(y);
        if (lane == src) x[p] = y;
      }
      if (r[p] < n && sub == 0) {
        const uint32_t old = S.sent[r[p]];
        if (x[p] > old) {
          S.sent[r[p]] = x[p];
          changed = 1;
        } else if (old == (uint32_t)r[p] + 1u) {
          S.own[r[p]] = x[p];
        }
      }
    }
  }
  return changed;
}

// The whole MAP computation of a graph of n <= kSmallN vertices by one
// workgroup, results as map_body's.  Such a graph is latency-bound: over
// several workgroups every sweep pays gathers through memory and releases or
// grid barriers (about 10 us); here a sweep is one pass over LDS between two
// workgroup barriers, and the launch needs neither the cooperative queue (17 us
// more than an ordinary launch) nor a cleared control block.  An edge is one
// register, the two byte offsets (4 row) << 16 | 4 successor, edge t + 1024 j in
// thread t: the work of a
// sweep is even whatever the degrees, and both values of eight edges per
// thread are read together, so LDS throughput bounds the sweep, not its
// latency.  A vertex's value is what it sends, max(map, own id if accepting),
// raised in place with LDS atomic maxima; values only grow, so the order
// inside a sweep does not matter, and the sweep that raises nothing is the
// fixpoint.  Only an accepting vertex whose map value is at most its own id
// hides that value: one more pass folds those (own).  Graphs of more than
// 49,152 edges stream their columns instead (small_stream).
// One detection, back to back, against several workgroups with asynchronous
// sweeps: 10,000 vertices and 25,000 random edges 64 us (205 us before), 1,000
// vertices and 2,500 edges 18 us (80), 10,000 vertices and 12,500 edges of a DAG
// with K = 3 90 us (278).  Streamed, 100,000 edges: 138 us (244); small_takes
// draws the line for more.  12,288 vertices is what fits the LDS beside the row
// starts.
__device__ __forceinline__ void small_body(const LoopArgs& a) {
  SmallLds& S = g_lds.small;
  __shared__ uint32_t s_red[kWavesPerBlock];
  __shared__ unsigned long long s_red64[kWavesPerBlock];
  __shared__ int32_t s_wit[kWavesPerBlock];
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wib = tid / kWave;
  const int n = a.n;
  PH_START();
  auto block_sum = [&](uint32_t x) {
    x = wave_sum_u32(x);
    if (lane == 0) s_red[wib] = x;
    __syncthreads();
    uint32_t t = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) t += s_red[i];
    __syncthreads();
    return t;
  };
  const int32_t base = a.row_ptr[0];
  const int64_t m64 = (int64_t)a.row_ptr[n] - base;
  const bool staged = m64 >= 0 && m64 <= kBlock * kSmallEdges;
  const int m = staged ? (int)m64 : 0;
  const int rounds = small_rounds(m);
  int g = 1;  // streamed: lanes per row
  while (g < kWave && (int64_t)g * kSmallBatch * n < m64) g <<= 1;
#pragma unroll 4
  for (int r = tid; r <= n; r += kBlock) S.rp[r] = a.row_ptr[r] - base;
  __syncthreads();
  // Values go the way the rows are taken: upwards when most edges point down
  // (one edge per thread sampled).
  bool ascending;
  auto vote = [&](int row, int64_t k, bool any) {
    const int c = any ? a.col[base + k] : row;
    const uint32_t down = block_sum((c < row ? 1u : 0u) | (c > row ? 0x10000u : 0u));
    ascending = (down & 0xffffu) > down >> 16;
  };
  uint32_t edge[kSmallEdges];
  if (!staged) {
    const int row = (int)((int64_t)tid * n / kBlock);
    vote(row, S.rp[row], S.rp[row] < S.rp[row + 1]);
  } else {
    for (int r0 = wib * kWave; r0 < n; r0 += kBlock) {
      const int r = r0 + lane;
      const int b = r < n ? max(S.rp[r], 0) : 0, e = r < n ? min(S.rp[r + 1], m) : 0;
      const bool longrow = e - b > kWave;
      if (!longrow)
        for (int k = b; k < e; ++k) S.row_of[k] = (uint16_t)r;
      unsigned long long lr = __ballot(longrow);
      while (lr) {
        const int src = __ffsll(lr) - 1;
        lr &= lr - 1;
        const int bb = __shfl(b, src, kWave), ee = __shfl(e, src, kWave);
        for (int k = bb + lane; k < ee; k += kWave) S.row_of[k] = (uint16_t)(r0 + src);
      }
    }
    __syncthreads();
    const int sample = (int)((int64_t)tid * m / kBlock);
    vote(m ? (int)S.row_of[sample] : 0, sample, m != 0);
    const uint32_t pad = ((uint32_t)n << 18) | ((uint32_t)n << 2);  // an edge that changes nothing
#pragma unroll
    for (int j0 = 0; j0 < kSmallEdges; j0 += kSmallBatch) {
#pragma unroll
      for (int u = 0; u < kSmallBatch; ++u) edge[j0 + u] = pad;
      if (j0 * kBlock >= m) continue;
#pragma unroll
      for (int u = 0; u < kSmallBatch; ++u) {
        const int t = tid + (j0 + u) * kBlock, k = ascending ? t : m - 1 - t;
        if (t < m) edge[j0 + u] = ((uint32_t)S.row_of[k] << 18) | min((uint32_t)a.col[base + k], (uint32_t)n) << 2;
      }
    }
    __syncthreads();
  }
  // One sweep over the staged edges; kOwn: only the maxima of the rows that
  // send their own id.
  auto sent_at = [&](uint32_t offset) { return reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(S.sent) + offset); };
  auto relax = [&](auto kOwn) -> uint32_t {
    uint32_t changed = 0;
#pragma unroll
    for (int j0 = 0; j0 < kSmallEdges; j0 += kSmallBatch) {
      if (j0 * kBlock >= m) continue;
      uint32_t x[kSmallBatch], y[kSmallBatch];
#pragma unroll
      for (int u = 0; u < kSmallBatch; ++u) {
        // Opaque to the optimizer: it would keep both LDS addresses of every
        // edge in registers across the sweeps, and spill them.
        asm volatile("" : "+v"(edge[j0 + u]));
        x[u] = *sent_at(edge[j0 + u] & 0xffffu);
        y[u] = *sent_at(edge[j0 + u] >> 16);
      }
#pragma unroll
      for (int u = 0; u < kSmallBatch; ++u) {
        if (decltype(kOwn)::value) {
          const uint32_t r = edge[j0 + u] >> 18;
          if (x[u] && y[u] == r + 1u) atomicMax(&S.own[r], x[u]);
        } else if (x[u] > y[u]) {
          atomicMax(sent_at(edge[j0 + u] >> 16), x[u]);
          changed = 1;
        }
      }
    }
    return changed;
  };
  uint32_t accbits = 0;  // accepting flags of the thread's rows tid + 1024 j
#pragma unroll 4
  for (int j = 0; j < kSmallRows; ++j) {
    const int r = tid + j * kBlock;
    if (r < n && a.acc_in[r]) accbits |= 1u << j;
  }
  if (tid < kSmallN / 32) S.del[tid] = 0;
  if (tid == 0) S.sent[n] = 0;
  // Map value of row r after the fixpoint.
  auto map_of = [&](int r) {
    const uint32_t x = S.sent[r];
    return x == (uint32_t)r + 1u ? S.own[r] : x;
  };
  int32_t k = 0, found = 0, witness = 0, status = MAP_OK, left = 0;
  int64_t total = 0;
  uint32_t count = block_sum((uint32_t)__popc(accbits));
  const bool want_digest = a.digest != 0;
  PH_MARK(kPhSetup);
  while (a.propagate || count != 0) {
    ++k;
#pragma unroll 1
    for (int j = 0; j < kSmallRows && j * kBlock < n; ++j) {
      const int r = tid + j * kBlock;
      if (r < n) {
        S.sent[r] = ((accbits >> j) & 1u) ? (uint32_t)r + 1u : 0u;
        S.own[r] = 0;
      }
    }
    __syncthreads();
    PH_MARK(kPhOther);
    int32_t s = 0;
    if (staged) {
      uint32_t again;
      do {
        ++s;
        again = 0;
        for (int round = 0; round < rounds; ++round) {
          const uint32_t ch = relax(std::false_type());
          again |= ch;
          PH_COUNT(kPhLocalPasses, 1);
          if (__ballot(ch != 0) == 0) break;
        }
      } while (__syncthreads_or((int)again));
      relax(std::true_type());
      __syncthreads();
      PH_MARK(kPhLocal);
    } else {
      do ++s;
      while (__syncthreads_or((int)small_stream(a, base, g, ascending, wib, lane)));
      PH_MARK(kPhStream);
    }
    PH_COUNT(kPhSweeps, s);
    PH_COUNT(kPhQuiet, 1);
    total += s;
    if (a.propagate) break;
    // Witness, digest, and the flags this iteration strips.
    int32_t wit = 0;
    unsigned long long dig = 0;
    uint32_t nz = 0;
#pragma unroll 1
    for (int j = 0; j < kSmallRows && j * kBlock < n; ++j) {
      const int r = tid + j * kBlock;
      if (r < n) {
        const uint32_t id = (uint32_t)r + 1u, mv = map_of(r);
        if (mv == id) wit = max(wit, (int32_t)id);
        if (want_digest) dig += mix64(((unsigned long long)id << 32) | mv);
        if (mv) {
          const uint32_t bit = 1u << ((mv - 1u) & 31u);
          uint32_t* w = &S.del[(mv - 1u) >> 5];
          if (!(*w & bit)) atomicOr(w, bit);  // many rows share a value: read before writing
        }
        nz |= mv;
      }
    }
    wit = wave_max_i32(wit);
    if (want_digest) dig = wave_sum_u64(dig);
    const uint32_t wnz = __ballot(nz != 0) != 0 ? 1u : 0u;
    if (lane == 0) {
      s_wit[wib] = wit;
      s_red64[wib] = dig;
      s_red[wib] = wnz;
    }
    __syncthreads();
    wit = 0;
    dig = 0;
    nz = 0;
    for (int i = 0; i < kWavesPerBlock; ++i) {
      wit = max(wit, s_wit[i]);
      dig += s_red64[i];
      nz |= s_red[i];
    }
    __syncthreads();
    uint32_t next = count;
    if (wit == 0 && nz != 0) {
#pragma unroll 1
      for (int j = 0; j < kSmallRows && j * kBlock < n; ++j) {
        const int r = tid + j * kBlock;
        if (r < n && ((S.del[r >> 5] >> (r & 31)) & 1u)) accbits &= ~(1u << j);
      }
      next = block_sum((uint32_t)__popc(accbits));  // its barriers order the reads of del before the clear
      if (tid < kSmallN / 32) S.del[tid] = 0;
    }
    if (tid == 0 && a.trace && k <= a.trace_cap) {
      uint64_t* row = a.trace + (int64_t)(k - 1) * 3;
      row[0] = (uint64_t)(count - next);
      row[1] = (uint64_t)s;
      row[2] = want_digest ? dig : 0ull;
    }
    count = next;
    left = (int32_t)count;
    PH_MARK(kPhDetect);
    PH_COUNT(kPhIters, 1);
    if (wit > 0) {
      found = 1;
      witness = wit;
      break;
    }
    if (nz == 0) break;
    if (a.max_iter > 0 && k >= a.max_iter) {
      if (count != 0) status = MAP_ENOTCONVERGED;
      break;
    }
  }
#pragma unroll 1
  for (int j = 0; j < kSmallRows && j * kBlock < n; ++j) {
    const int r = tid + j * kBlock;
    if (r < n) {
      if (a.propagate && a.map_out) a.map_out[r] = (int32_t)map_of(r);
      if (!a.propagate && a.acc_out) a.acc_out[r] = (uint8_t)((accbits >> j) & 1u);
    }
  }
  if (tid == 0) {
    a.result->found = found;
    a.result->witness = witness;
    a.result->iterations = a.propagate ? 0 : k;
    a.result->status = status;
    a.result->sweeps = total;
    a.result->accepting_left = a.propagate ? 0 : left;
    a.result->reserved = 0;
  }
  PH_MARK(kPhOther);
  PH_STORE(0, 1);
  __syncthreads();
}

// One workgroup solves a graph of at most kSmallN vertices unless its
// arguments ask for another control: streamed sweeps, a barrier per sweep,
// frontier rounds or early detection.
__host__ __device__ inline bool small_fits(const LoopArgs& a) {
  return a.n <= kSmallN && !a.force_stream && !a.sync_sweeps && !a.push && !a.early;
}

// Whether one workgroup is the better choice for such a graph of m edges, too,
// where a launch of its own could share it out to g workgroups (one per 2,048
// vertices).  It streams the columns of a dense graph as fast as they come out
// of the L2 of its XCD (4 MB): with more columns the workgroups, each on an XCD
// of its own, are ahead while their shares fit theirs, and four of them always.
// Detection by one workgroup / by g (random digraphs): 12,288 vertices, 262,000
// edges 216 / 215 us, 786,000 edges 559 / 574, 1.05M 918 / 681, 10M 9.8 / 5.4 ms;
// 4,096 vertices, 1.05M 866 / 1,138 us, 1.8M 2,221 / 1,725, 4M 3.9 / 6.1 ms; 6,144
// vertices, 1.5M 1,914 / 1,269 us, 4M 4.2 / 4.0 ms, 10M 8.9 / 10.8.
// Where the host cannot bound the edges both kernels are launched and the other
// one returns at once (gate): 2,049 to 12,288 vertices then take 12 us more when
// several workgroups run, 20 us when one does.
constexpr int64_t kSmallStream = 3 << 18;  // edges: 3 MB of columns
__host__ __device__ inline bool small_takes(int32_t n, int64_t m) {
  constexpr int kRows = kWavesPerBlock * kTileRows;
  const int64_t g = (n + kRows - 1) / kRows;
  return g == 1 || m <= kSmallStream || (g < 4 && m > g << 20);
}

__global__ void __launch_bounds__(kBlock) map_small_kernel(LoopArgs a) {
  if (a.gate && !small_takes(a.n, (int64_t)a.row_ptr[a.n] - a.row_ptr[0])) return;
  small_body(a);
}

// The asynchronous loop, out of line so that its register allocation is not
// shared with the windowed iterations (inlined beside the call of win_body its
// values live across the call are spilled: 853 accesses of scratch memory
// instead of 134).
__device__ __noinline__ bool map_body_async(const LoopArgs& a, const int nb, const int b, const int logical,
                                            LoopState* st) {
  const LoopArgs u = uniform(a);
  return map_body<Ctrl, true, false, false, true>(u, u.ctrl, uniform(nb), uniform(b), uniform(logical), st);
}

// kEarly: MAP_FLAG_EARLY (a separate instantiation, so that the plain loop
// carries none of its code).
template <bool kAsync, bool kEarly, bool kFilt = false, bool kBands = false>
__global__ void __launch_bounds__(kBlock) map_loop_kernel(LoopArgs a) {
  const int nb = gridDim.x;
  const int b = blockIdx.x;
  // XCD-aware numbering: consecutive hardware block ids land on different
  // XCDs; give each XCD a contiguous range of logical blocks (and rows).
  const int logical = (nb % kMaxGroups == 0) ? (b % kMaxGroups) * (nb / kMaxGroups) + b / kMaxGroups : b;
  if constexpr (kAsync && !kEarly && !kFilt) {
    if (a.gate && small_takes(a.n, (int64_t)a.row_ptr[a.n] - a.row_ptr[0])) return;
    // By reference to the kernel's own copy, every thread would write that copy
    // to scratch memory first: 10 us a launch.
    __shared__ LoopArgs s_args;
    if (threadIdx.x == 0) s_args = a;
    __syncthreads();
    LoopState st = {};
    while (uniform((int)map_body_async(s_args, nb, b, logical, &st)))
      if (!uniform((int)win_body(s_args, nb, b, logical, &st))) break;
  } else {
    map_body<Ctrl, kAsync, kEarly, kFilt, false, kBands>(a, a.ctrl, nb, b, logical);
  }
}

// ------------------------------------------------------------------ batch --

struct BatchArgs {
  int32_t count;
  const map_graph_desc* graphs;
  map_result* results;
  const int32_t* item_start;  // [count + 1]: first work item of each graph
  const int64_t* scratch_off;  // [count]: byte offset of each graph's scratch
  GangCtrl* gctrl;             // [count]
  char* scratch;
  uint32_t* next_item;
  int32_t* status;             // MAP_ENOSPC when the scratch does not fit
  uint32_t flags;
};

// One graph of a batch, out of line so that its register allocation is not
// shared with the work-queue loop around it.
__device__ __noinline__ void map_body_gang_async(const LoopArgs& a, GangCtrl* c, int nb, int rank) {
  map_body<GangCtrl, true, false>(uniform(a), uniform(c), uniform(nb), uniform(rank), uniform(rank));
}
__device__ __noinline__ void map_body_gang_sync(const LoopArgs& a, GangCtrl* c, int nb, int rank) {
  map_body<GangCtrl, false, false>(uniform(a), uniform(c), uniform(nb), uniform(rank), uniform(rank));
}
__device__ __noinline__ void map_body_gang_sync_early(const LoopArgs& a, GangCtrl* c, int nb, int rank) {
  map_body<GangCtrl, false, true>(uniform(a), uniform(c), uniform(nb), uniform(rank), uniform(rank));
}
__device__ __noinline__ void map_body_gang_filt(const LoopArgs& a, GangCtrl* c, int nb, int rank) {
  map_body<GangCtrl, false, false, true>(uniform(a), uniform(c), uniform(nb), uniform(rank), uniform(rank));
}
__device__ __noinline__ void small_body_gang(const LoopArgs& a) { small_body(uniform(a)); }
// One graph solved by a gang, in the fixpoint control and mode its arguments ask
// for.  MAP_FLAG_EARLY always runs with a grid barrier after every sweep: the
// asynchronous early body is not built (its builds hung on the device).
__device__ __forceinline__ void map_body_gang(const LoopArgs& a, GangCtrl* c, int nb, int rank) {
  const bool async = nb > 1 && !a.sync_sweeps && a.tag_mask;
  if (nb == 1 && small_fits(a)) {
    small_body_gang(a);
  } else if (a.early) {
    map_body_gang_sync_early(a, c, nb, rank);
  } else if (a.filt) {
    map_body_gang_filt(a, c, nb, rank);
  } else {
    if (async) map_body_gang_async(a, c, nb, rank);
    else map_body_gang_sync(a, c, nb, rank);
  }
}

// --------------------------------------------------------- counterexample --

// Barrier state of a launch whose blocks all cooperate on one control block,
// in hardware block order.
__device__ __forceinline__ Grid<Ctrl> whole_grid(Ctrl* c) {
  Grid<Ctrl> g;
  g.c = c;
  g.gen = 0;
  g.nblocks = gridDim.x;
  g.ngroups = min((int)gridDim.x, kMaxGroups);
  g.group = blockIdx.x % g.ngroups;
  g.group_size = gridDim.x / g.ngroups + ((blockIdx.x % g.ngroups) < (gridDim.x % g.ngroups) ? 1 : 0);
  g.rank = blockIdx.x;
  return g;
}

// Arguments of the lasso search: a shortest path from `init` to the witness
// and a shortest cycle through it, by breadth-first search over successors.
struct LassoArgs {
  int32_t n;
  const int32_t* row_ptr;  // pull CSR of G: row v = successors of v
  const int32_t* col;
  int32_t w;               // witness, 0-based
  int32_t init;            // initial vertex, 0-based, or -1
  int32_t* path;           // ids out
  int32_t cap;
  map_lasso_result* result;
  uint64_t* parent;        // [n]: level << 32 | (1 + the vertex it was reached from); the start
                           // level 0 with low word -1; unreached kUnreached
  int32_t* front[2];       // frontiers [n]
  Ctrl* ctrl;
};

// Sum over the block of a per-wave u32 (every thread gets it).
__device__ uint32_t lasso_block_sum(uint32_t x) {
  __shared__ uint32_t s_part[kWavesPerBlock];
  const int lane = threadIdx.x & (kWave - 1), wib = threadIdx.x / kWave;
  if (lane == 0) s_part[wib] = x;
  __syncthreads();
  uint32_t t = 0;
  for (int i = 0; i < kWavesPerBlock; ++i) t += s_part[i];
  __syncthreads();
  return t;
}

// Flattened frontier expansion, shared by the counterexample search and the
// pruning.  A wave takes 64 frontier vertices at a time; an inclusive scan of
// their degrees across the wave gives each vertex the first slot of its edges
// in the wave's combined list, and lane l examines slots q0 + l + 64 s (s <
// kExpandPerLane) of that list.  The wave thus issues the reads and atomics of
// up to 64 * kExpandPerLane edges together, instead of one edge per lane per
// step, and appends what it claimed with one counter update per chunk.
constexpr int kExpandPerLane = 4;
constexpr uint64_t kUnreached = ~0ull;    // lasso parent word of a vertex not reached
constexpr uint32_t kDirectSize = 16384;  // lasso: frontiers below it claim without reading first
constexpr uint32_t kNoHit = 0xffffffffu;  // lasso: no edge has entered the target yet

// A block's appends to the next frontier, staged in LDS and moved there with one
// update of the frontier's counter per block and round.  (One update per wave
// and step went to one address 10,000 times in a large round, some 10 ns each:
// a search round of 277,000 vertices took 95 us, so 50, and a whole
// counterexample in 2^20 states 658 and 492; the pruning of 2^20 states, with
// its first frontier and its sums collected the same way, 433 and 221.)  What does not fit is appended by its wave.
// Fewer than kStageBlocks workgroups append wave by wave (kStaged false): the
// counter is not contended, and the stage's barriers cost up to 4% of the pruning
// of 5,000 vertices.  In instantiations of their own: asked at run time it cost
// the pruning of 2^20 vertices 1 to 2% and the search of them 0.5%.
constexpr uint32_t kStage = 8192;
constexpr int kStageBlocks = 8;
__shared__ int32_t g_stage[kStage];
__shared__ uint32_t g_staged, g_stage_end, g_stage_base;

// Before the first append of a kernel, followed by a barrier.
__device__ __forceinline__ void stage_clear() {
  if (threadIdx.x == 0) {
    g_staged = 0;
    g_stage_end = kStage;
  }
}

// Appends x[s] for every s with take[s]; returns the number appended by the
// wave (wave-uniform).
template <bool kStaged, int N>
__device__ __forceinline__ uint32_t stage_append(int32_t* F, uint32_t* cnt, const bool* take, const int32_t* x,
                                                 int lane) {
  uint32_t c = 0;
#pragma unroll
  for (int s = 0; s < N; ++s) c += take[s] ? 1u : 0u;
  uint32_t incl = c;
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)incl, off, kWave);
    if (lane >= off) incl += y;
  }
  const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
  if (total == 0) return 0;
  uint32_t base = 0;
  if (kStaged) {
    if (lane == 0) base = atomicAdd(&g_staged, total);
    base = (uint32_t)__shfl((int)base, 0, kWave);
  }
  if (kStaged && base <= kStage - total) {  // total <= 64 N
    base += incl - c;
#pragma unroll
    for (int s = 0; s < N; ++s)
      if (take[s]) g_stage[base++] = x[s];
  } else {
    if (lane == 0) {
      if (kStaged) atomicMin(&g_stage_end, base);  // the staged entries end here: whoever came later did not fit either
      base = __hip_atomic_fetch_add(cnt, total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    base = (uint32_t)__shfl((int)base, 0, kWave) + (incl - c);
#pragma unroll
    for (int s = 0; s < N; ++s)
      if (take[s]) F[base++] = x[s];
  }
  return total;
}

// Moves the staged entries to frontier F (every thread of the block).
template <bool kStaged>
__device__ __forceinline__ void stage_flush(int32_t* F, uint32_t* cnt) {
  if (!kStaged) return;
  __syncthreads();
  const uint32_t m = min(g_staged, g_stage_end);
  if (threadIdx.x == 0 && m) g_stage_base = __hip_atomic_fetch_add(cnt, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  const uint32_t base = g_stage_base;
  for (uint32_t i = threadIdx.x; i < m; i += kBlock) F[base + i] = g_stage[i];
  __syncthreads();
  stage_clear();
}

// Breadth-first search from `from` until an edge enters `to`, run by every
// thread of the grid.  The start is marked reached (level 0) but an edge into
// `to` is taken before that mark is looked at, so from == to finds a shortest
// cycle.  Each round expands one frontier: a wave takes 64 frontier vertices
// and a lane walks its vertex's successors.  A successor not reached in an
// earlier round takes, by an atomic minimum on its 64-bit parent word (round
// in the high half), the smallest frontier vertex with an edge to it; the
// lane whose minimum found the word unreached appends it to the next
// frontier.  An edge into `to` takes the minimum of its source into c->hit.
// The parents, the last vertex and so the path therefore depend only on the
// edge set, not on the column order or the schedule: walking back from `to`,
// each step goes to the smallest vertex of the level before.  A grid barrier
// ends each round and carries the size of the next frontier.  Returns the
// length of a shortest path of >= 1 edge, 0 if `to` is not reached, -1 if a
// barrier wait gave up (the launch must stop); *last (every block) is the
// vertex whose edge entered `to`.
template <bool kStaged>
__device__ int32_t lasso_bfs(const LassoArgs& a, Grid<Ctrl>& g, int32_t from, int32_t to, int32_t* last,
                             unsigned long long* scanned, int32_t* levels) {
  Ctrl* c = a.ctrl;
  const int lane = threadIdx.x & (kWave - 1), wib = threadIdx.x / kWave;
  const int64_t gw = (int64_t)g.rank * kWavesPerBlock + wib, nw = (int64_t)g.nblocks * kWavesPerBlock;
  for (int64_t v = (int64_t)g.rank * kBlock + threadIdx.x; v < a.n; v += (int64_t)g.nblocks * kBlock)
    a.parent[v] = v == from ? 0xffffffffull : kUnreached;  // the start: level 0, low word -1
  if (g.rank == 0 && threadIdx.x == 0) {
    st_agent(&c->hit, kNoHit);
    st_agent(&c->fcount[0], 0u);
    st_agent(&c->fcount[1], 0u);
    a.front[0][0] = from;
  }
  if (!grid_sync(g, 0, nullptr)) return -1;
  uint64_t* parent = a.parent;
  uint32_t size = 1;
  int fc = 0;
  for (int32_t level = 1;; ++level) {
    // This round reads frontier fc and appends to fc ^ 1, whose counter was
    // cleared before the barrier that opened the round; fc's counter is
    // appended to in the next round, after the barrier that closes this one.
    if (g.rank == 0 && threadIdx.x == 0) st_agent(&c->fcount[fc], 0u);
    const int32_t* F = a.front[fc];
    int32_t* Fn = a.front[fc ^ 1];
    uint32_t* cn = &c->fcount[fc ^ 1];
    const bool direct = size < kDirectSize;
    uint32_t napp = 0;
    for (int64_t i0 = gw * kWave; i0 < (int64_t)size; i0 += nw * kWave) {
      const int64_t i = i0 + lane;
      int32_t u = 0, k = 0;
      uint32_t deg = 0;
      if (i < (int64_t)size) {
        u = F[i];
        if ((uint32_t)u < (uint32_t)a.n) {
          k = a.row_ptr[u];
          deg = (uint32_t)(a.row_ptr[u + 1] - k);
        } else {
          st_agent(&c->bad, 1u);
        }
      }
      uint32_t incl = deg;
      for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, off, kWave);
        if (lane >= off) incl += y;
      }
      const uint32_t first = incl - deg;
      const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
      for (uint32_t q0 = 0; q0 < total; q0 += kWave * kExpandPerLane) {
        int32_t v[kExpandPerLane], src[kExpandPerLane];
        bool ok[kExpandPerLane], take[kExpandPerLane];
        uint32_t pw[kExpandPerLane];
#pragma unroll
        for (int s = 0; s < kExpandPerLane; ++s) {
          const uint32_t q = q0 + (uint32_t)(s * kWave + lane);
          const int o = slot_owner(q, first);
          const int32_t ko = __shfl(k, o, kWave);
          const uint32_t fo = (uint32_t)__shfl((int)first, o, kWave);
          src[s] = __shfl(u, o, kWave);
          ok[s] = q < total;
          v[s] = ok[s] ? a.col[ko + (int32_t)(q - fo)] : 0;
        }
        // Plain reads of the round in a parent word: words set in an earlier
        // round are final (they precede a barrier) and are skipped; an
        // unreached word or one of this round takes the atomic minimum.  In a
        // small round every word takes it at once: a minimum leaves an earlier
        // round's word as it is, and the read is a link of the round's chain
        // (counterexample in 2^20 states 485 us with the read, 450 without).
#pragma unroll
        for (int s = 0; s < kExpandPerLane; ++s) {
          pw[s] = 0u;
          if (!ok[s]) continue;
          ++*scanned;
          if ((uint32_t)v[s] >= (uint32_t)a.n) {
            st_agent(&c->bad, 1u);
            ok[s] = false;
          } else if (v[s] == to) {
            __hip_atomic_fetch_min(&c->hit, (uint32_t)src[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok[s] = false;
          } else {
            pw[s] = direct ? (uint32_t)level : (uint32_t)(parent[v[s]] >> 32);
          }
        }
#pragma unroll
        for (int s = 0; s < kExpandPerLane; ++s) {
          take[s] = false;
          if (ok[s] && pw[s] >= (uint32_t)level) {
            const uint64_t claim = ((uint64_t)(uint32_t)level << 32) | (uint32_t)(src[s] + 1);
            take[s] = __hip_atomic_fetch_min(&parent[v[s]], claim, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                      kUnreached;
          }
        }
        napp += stage_append<kStaged, kExpandPerLane>(Fn, cn, take, v, lane);
      }
    }
    uint32_t tot = 0;
    stage_flush<kStaged>(Fn, cn);
    if (!grid_sync(g, lasso_block_sum(napp), &tot)) return -1;
    *levels += 1;
    const uint32_t h = ld_agent(&c->hit), bad = ld_agent(&c->bad);
    if (bad) return 0;
    if (h != kNoHit) {
      *last = (int32_t)h;
      return level;
    }
    if (tot == 0) return 0;
    size = tot;
    fc ^= 1;
  }
}

// Walks parent words back from `x` and writes path[hi], path[hi-1], ...,
// path[lo] (ids); the word of the vertex written at path[lo] must name `root`.
// Single thread.  Returns false if the chain does not end there.
__device__ bool lasso_walk(const LassoArgs& a, int32_t x, int32_t hi, int32_t lo, int32_t root) {
  for (int32_t i = hi; i >= lo; --i) {
    if ((uint32_t)x >= (uint32_t)a.n) return false;
    a.path[i] = x + 1;
    const int32_t p = (int32_t)(uint32_t)__hip_atomic_load(&a.parent[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (i == lo) return p == root + 1 || (p == -1 && x == root);
    if (p <= 0) return false;
    x = p - 1;
  }
  return true;
}

template <bool kStaged>
__global__ void __launch_bounds__(kBlock) map_lasso_kernel(LassoArgs a) {
  Grid<Ctrl> g = whole_grid(a.ctrl);
  const bool leader = blockIdx.x == 0 && threadIdx.x == 0;
  unsigned long long scanned = 0;
  int32_t levels = 0, S = 0, L = -1, last = 0;
  int32_t status = MAP_OK;
  bool written = false;
  stage_clear();  // ordered before its first use by the barriers that open a search
  if (a.init >= 0 && a.init != a.w) {
    S = lasso_bfs<kStaged>(a, g, a.init, a.w, &last, &scanned, &levels);
    if (S < 0) goto aborted;
    if (S == 0) {
      S = -1;
      status = MAP_ENOPATH;
    } else if (leader && (int64_t)S + 1 <= a.cap) {
      // s_S = w, s_{S-1} = last, ..., s_0 = init (parent word -1)
      a.path[S] = a.w + 1;
      if (!lasso_walk(a, last, S - 1, 0, a.init)) status = MAP_EDEVICE;
    }
    // The stem's parent words are read above before the next search clears them.
    if (!grid_sync(g, 0, nullptr)) goto aborted;
  }
  if (status == MAP_OK) {
    L = lasso_bfs<kStaged>(a, g, a.w, a.w, &last, &scanned, &levels);
    if (L < 0) goto aborted;
    if (L == 0) {
      L = -1;
      status = MAP_ENOPATH;
    } else if ((int64_t)S + L + 1 > a.cap) {
      status = MAP_ENOSPC;
    } else if (leader) {
      // c_L = w, c_{L-1} = last, ..., c_1 (parent word names w)
      a.path[S + L] = a.w + 1;
      if (S == 0) a.path[0] = a.w + 1;
      if (L > 1 && !lasso_walk(a, last, S + L - 1, S + 1, a.w)) status = MAP_EDEVICE;
      if (L == 1 && last != a.w) status = MAP_EDEVICE;
      written = status == MAP_OK;
    }
  }
  {
    // Edges examined (below 2^32: each at most once in a search): one atomic
    // per block, read after a last barrier.
    const uint32_t ws = lasso_block_sum(wave_sum_u32((uint32_t)scanned));
    if (threadIdx.x == 0 && ws)
      __hip_atomic_fetch_add(&a.ctrl->scanned, (unsigned long long)ws, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (!grid_sync(g, 0, nullptr)) goto aborted;
  }
  if (leader) {
    if (ld_agent(&a.ctrl->bad)) status = MAP_ERANGE_DEV;
    map_lasso_result* r = a.result;
    r->status = status;
    r->stem_len = status == MAP_ENOPATH && S < 0 ? -1 : S;
    r->cycle_len = L;
    r->path_len = written && status == MAP_OK ? S + L + 1 : 0;
    r->edges_scanned = (int64_t)__hip_atomic_load(&a.ctrl->scanned, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    r->levels = levels;
    r->reserved = 0;
  }
  return;
aborted:
  if (leader) {
    a.result->status = MAP_EDEVICE;
    a.result->path_len = 0;
  }
}

// ---------------------------------------------------------------- pruning --

// Arguments of the trim of cycle-free vertices.
struct TrimArgs {
  int32_t n;
  const int32_t* row_ptr;  // pull CSR of G: row v = successors
  const int32_t* col;
  const int32_t* rrow_ptr; // transposed CSR: row v = predecessors
  const int32_t* rcol;
  const uint8_t* acc_in;   // or nullptr
  uint8_t* keep_out;
  uint8_t* acc_out;        // or nullptr
  map_trim_result* result;
  uint32_t* indeg;         // [n] in-edges from vertices not removed
  uint32_t* outdeg;        // [n] out-edges to vertices not removed
  uint32_t* removed;       // [n] 1 once removed (claimed by compare-and-swap)
  int32_t* front[2];
  Ctrl* ctrl;
};

// Removes, while one exists, a vertex with no remaining predecessor or no
// remaining successor (parallel edges counted with multiplicity), in rounds:
// the first frontier is every vertex with no in-edge or no out-edge; a round
// takes a frontier of removed vertices, subtracts each one's out-edges from
// its successors' in-counts and its in-edges from its predecessors'
// out-counts, and a vertex whose count reaches 0 is claimed (compare-and-swap
// on its removed word) and appended to the next frontier.  A grid barrier
// ends each round and carries the next frontier's size.  A vertex on a cycle
// always keeps an in-edge and an out-edge from the cycle, so it is never
// removed.
template <bool kStaged>
__global__ void __launch_bounds__(kBlock) map_trim_kernel(TrimArgs a) {
  Grid<Ctrl> g = whole_grid(a.ctrl);
  Ctrl* c = a.ctrl;
  const int lane = threadIdx.x & (kWave - 1), wib = threadIdx.x / kWave;
  const int64_t gw = (int64_t)g.rank * kWavesPerBlock + wib, nw = (int64_t)g.nblocks * kWavesPerBlock;
  const bool leader = blockIdx.x == 0 && threadIdx.x == 0;
  int32_t rounds = 0;
  uint32_t napp = 0, size = 0, kept = 0, acc_kept = 0;
  int fc = 0;
  // Counts, and the first frontier into front[0] (counter fcount[0], zero),
  // kExpandPerLane vertices of a lane at a time.
  stage_clear();
  __syncthreads();
  for (int64_t v0 = gw * (kWave * kExpandPerLane); v0 < a.n; v0 += nw * (kWave * kExpandPerLane)) {
    int32_t x[kExpandPerLane];
    bool take[kExpandPerLane];
    uint32_t in[kExpandPerLane], out[kExpandPerLane];
#pragma unroll
    for (int s = 0; s < kExpandPerLane; ++s) {
      const int64_t v = v0 + s * kWave + lane;
      x[s] = (int32_t)v;
      in[s] = v < a.n ? (uint32_t)(a.rrow_ptr[v + 1] - a.rrow_ptr[v]) : 1u;
      out[s] = v < a.n ? (uint32_t)(a.row_ptr[v + 1] - a.row_ptr[v]) : 1u;
    }
#pragma unroll
    for (int s = 0; s < kExpandPerLane; ++s) {
      const int64_t v = v0 + s * kWave + lane;
      take[s] = in[s] == 0 || out[s] == 0;
      if (v < a.n) {
        a.indeg[v] = in[s];
        a.outdeg[v] = out[s];
        a.removed[v] = take[s] ? 1u : 0u;
      }
    }
    napp += stage_append<kStaged, kExpandPerLane>(a.front[0], &c->fcount[0], take, x, lane);
  }
  stage_flush<kStaged>(a.front[0], &c->fcount[0]);
  if (!grid_sync(g, lasso_block_sum(napp), &size)) goto aborted;
  while (size > 0) {
    // Frontier fc is read and fc ^ 1 appended to (its counter is zero: it was
    // cleared in the round that read it, before the barrier that closed it).
    if (g.rank == 0 && threadIdx.x == 0) st_agent(&c->fcount[fc], 0u);
    const int32_t* F = a.front[fc];
    int32_t* Fn = a.front[fc ^ 1];
    uint32_t* cn = &c->fcount[fc ^ 1];
    napp = 0;
    for (int64_t i0 = gw * kWave; i0 < (int64_t)size; i0 += nw * kWave) {
      const int64_t i = i0 + lane;
      // A removed vertex's out-edges then its in-edges, flattened across the
      // wave (slots [0, dout) of a vertex are col entries, the rest rcol).
      int32_t k = 0, r = 0;
      uint32_t dout = 0, deg = 0;
      if (i < (int64_t)size) {
        const int32_t v = F[i];
        if ((uint32_t)v < (uint32_t)a.n) {
          k = a.row_ptr[v];
          r = a.rrow_ptr[v];
          dout = (uint32_t)(a.row_ptr[v + 1] - k);
          deg = dout + (uint32_t)(a.rrow_ptr[v + 1] - r);
        } else {
          st_agent(&c->bad, 1u);
        }
      }
      uint32_t incl = deg;
      for (int off = 1; off < kWave; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, off, kWave);
        if (lane >= off) incl += y;
      }
      const uint32_t first = incl - deg;
      const uint32_t total = (uint32_t)__shfl((int)incl, kWave - 1, kWave);
      for (uint32_t q0 = 0; q0 < total; q0 += kWave * kExpandPerLane) {
        int32_t x[kExpandPerLane];
        bool ok[kExpandPerLane], out_e[kExpandPerLane], take[kExpandPerLane];
        uint32_t old[kExpandPerLane];
#pragma unroll
        for (int s = 0; s < kExpandPerLane; ++s) {
          const uint32_t q = q0 + (uint32_t)(s * kWave + lane);
          const int o = slot_owner(q, first);
          const int32_t ko = __shfl(k, o, kWave), ro = __shfl(r, o, kWave);
          const uint32_t fo = (uint32_t)__shfl((int)first, o, kWave);
          const uint32_t dout_o = (uint32_t)__shfl((int)dout, o, kWave);
          const uint32_t j = q - fo;
          ok[s] = q < total;
          out_e[s] = j < dout_o;
          x[s] = ok[s] ? (out_e[s] ? a.col[ko + (int32_t)j] : a.rcol[ro + (int32_t)(j - dout_o)]) : 0;
        }
#pragma unroll
        for (int s = 0; s < kExpandPerLane; ++s) {
          old[s] = 0u;
          if (!ok[s]) continue;
          if ((uint32_t)x[s] >= (uint32_t)a.n) {
            st_agent(&c->bad, 1u);
            ok[s] = false;
            continue;
          }
          uint32_t* cnt = out_e[s] ? &a.indeg[x[s]] : &a.outdeg[x[s]];
          old[s] = __hip_atomic_fetch_sub(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int s = 0; s < kExpandPerLane; ++s) {
          take[s] = false;
          if (ok[s] && old[s] == 1u) {
            uint32_t zero = 0;
            take[s] = __hip_atomic_compare_exchange_strong(&a.removed[x[s]], &zero, 1u, __ATOMIC_RELAXED,
                                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
        napp += stage_append<kStaged, kExpandPerLane>(Fn, cn, take, x, lane);
      }
    }
    stage_flush<kStaged>(Fn, cn);
    if (!grid_sync(g, lasso_block_sum(napp), &size)) goto aborted;
    ++rounds;
    fc ^= 1;
  }
  // Outputs and counts.
  for (int64_t v = (int64_t)g.rank * kBlock + threadIdx.x; v < a.n; v += (int64_t)g.nblocks * kBlock) {
    const uint32_t keep = ld_agent(&a.removed[v]) ? 0u : 1u;
    a.keep_out[v] = (uint8_t)keep;
    kept += keep;
    if (a.acc_out) {
      const uint32_t ak = keep && a.acc_in[v] ? 1u : 0u;
      a.acc_out[v] = (uint8_t)ak;
      acc_kept += ak;
    }
  }
  kept = lasso_block_sum(wave_sum_u32(kept));
  acc_kept = lasso_block_sum(wave_sum_u32(acc_kept));
  if (threadIdx.x == 0) {
    if (kept) __hip_atomic_fetch_add(&c->kept, kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (acc_kept) __hip_atomic_fetch_add(&c->acc_kept, acc_kept, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (!grid_sync(g, 0, nullptr)) goto aborted;
  if (leader) {
    a.result->status = ld_agent(&c->bad) ? MAP_ERANGE_DEV : MAP_OK;
    a.result->kept = (int32_t)ld_agent(&c->kept);
    a.result->accepting_kept = (int32_t)ld_agent(&c->acc_kept);
    a.result->rounds = rounds;
  }
  return;
aborted:
  if (leader) a.result->status = MAP_EDEVICE;
}

// Scratch of one graph of a batch: the packed values (4n bytes), the working
// accepting flags (n), and with MAP_GRAPH_FILTER the three change bitmaps and
// the accepting bitmap of the filtered sweeps (ceil(n / 32) words each); every
// part 256-aligned.
__host__ __device__ inline int64_t gang_bitmap_bytes(int64_t n) { return ((((n + 31) / 32) * 4) + 255) & ~(int64_t)255; }
__host__ __device__ inline int64_t gang_scratch_bytes(int64_t n, int32_t options) {
  n = n < 1 ? 1 : n;
  const int64_t base = ((n * 4 + 255) & ~(int64_t)255) + ((n + 255) & ~(int64_t)255);
  return base + ((options & MAP_GRAPH_FILTER) ? 4 * gang_bitmap_bytes(n) : 0);
}

// Loop arguments of one graph solved by a gang, on its scratch.
__device__ LoopArgs gang_args(int32_t n, const int32_t* row_ptr, const int32_t* col, const int32_t* rrow_ptr,
                              const int32_t* rcol, const uint8_t* acc0, char* scratch, map_result* result,
                              uint32_t flags, int32_t options) {
  LoopArgs a;
  a.n = n;
  a.ntiles = (int32_t)(((int64_t)n + kTileRows - 1) / kTileRows);
  a.row_ptr = row_ptr;
  a.col = col;
  a.acc_in = acc0;
  a.pv = reinterpret_cast<uint32_t*>(scratch);
  a.accw = reinterpret_cast<uint8_t*>(scratch + (((size_t)n * 4 + 255) & ~(size_t)255));
  a.ctrl = nullptr;
  a.result = result;
  a.trace = nullptr;
  a.trace_cap = 0;
  a.acc_out = nullptr;
  a.map_out = nullptr;
  a.max_iter = 0;
  a.propagate = 0;
  a.digest = 0;
  a.force_stream = (flags & MAP_FLAG_STREAM) ? 1 : 0;
  a.sync_sweeps = (flags & MAP_FLAG_SYNC_SWEEPS) ? 1 : 0;
  word_layout(n, &a.val_mask, &a.tag_mask, &a.tag_shift);
  a.epoch = nullptr;
  a.push = 0;
  a.early = (flags & MAP_FLAG_EARLY) ? 1 : 0;
  a.rrow_ptr = nullptr;
  a.rcol = nullptr;
  a.front[0] = a.front[1] = nullptr;
  a.mark = nullptr;
  a.chg = nullptr;
  a.accb = nullptr;
  a.win = nullptr;
  a.win_rec = nullptr;
  a.gate = 0;
  a.words = 0;
  a.filt = 0;
  a.dopt = 0;
  if ((options & MAP_GRAPH_FILTER) && !a.early) {
    // Filtered stream sweeps, a barrier after each (the change bitmaps follow
    // the working flags).
    const int64_t off = (((int64_t)n * 4 + 255) & ~(int64_t)255) + (((int64_t)n + 255) & ~(int64_t)255);
    const int64_t bb = gang_bitmap_bytes(n);
    a.chg = reinterpret_cast<uint32_t*>(scratch + off);
    a.accb = reinterpret_cast<uint32_t*>(scratch + off + 3 * bb);
    a.words = ((int64_t)n + 31) / 32;
    a.filt = 1;
    if ((options & MAP_GRAPH_DIRECTION) && rrow_ptr && rcol) {
      // Direction switch: small frontiers run as push rounds.
      a.dopt = 1;
      a.rrow_ptr = rrow_ptr;
      a.rcol = rcol;
    }
  }
  // Per-graph options of a batch (map_graph_desc.options): long-row threshold,
  // barrier per sweep, streamed CSR (filtered sweeps and the direction switch
  // above).
  a.hub = (options & MAP_GRAPH_HUB_MASK) ? (options & MAP_GRAPH_HUB_MASK) : kHubEdges;
  if (options & MAP_GRAPH_SYNC_SWEEPS) a.sync_sweeps = 1;
  if (options & MAP_GRAPH_STREAM) a.force_stream = 1;
  return a;
}

// Persistent work queue over the graphs of a batch.  Graph g is solved by
// item_start[g+1] - item_start[g] blocks (its gang); each block pops one item
// (graph, rank) at a time.  Items of a gang are consecutive in the queue, so a
// gang is always completed by blocks that free up, and it never waits on a
// later one.
__global__ void __launch_bounds__(kBlock) map_batch_kernel(BatchArgs ba) {
  __shared__ int32_t s_item;
  const int32_t total = ba.item_start[ba.count];
  if (__hip_atomic_load(ba.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != MAP_OK) {
    for (int32_t gi = blockIdx.x * blockDim.x + threadIdx.x; gi < ba.count; gi += gridDim.x * blockDim.x)
      ba.results[gi].status = MAP_ENOSPC;
    return;
  }
  for (;;) {
    if (threadIdx.x == 0) s_item = (int32_t)__hip_atomic_fetch_add(ba.next_item, 1u, __ATOMIC_RELAXED,
                                                                   __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int32_t item = s_item;
    __syncthreads();
    if (item >= total) break;
    int32_t lo = 0, hi = ba.count;  // largest gi with item_start[gi] <= item
    while (hi - lo > 1) {
      const int32_t mid = (lo + hi) >> 1;
      if (ba.item_start[mid] <= item) lo = mid; else hi = mid;
    }
    const int32_t gi = lo;
    const int nb = ba.item_start[gi + 1] - ba.item_start[gi];
    const int rank = item - ba.item_start[gi];
    const map_graph_desc d = ba.graphs[gi];
    if (d.n < 1 || d.n > 0x7ffffffe || !d.row_ptr || !d.col || !d.accepting0) {
      if (rank == 0 && threadIdx.x == 0) {
        ba.results[gi].status = MAP_EINVAL;
        ba.results[gi].found = ba.results[gi].witness = ba.results[gi].iterations = 0;
      }
      continue;
    }
    char* base = ba.scratch + ba.scratch_off[gi];
    const LoopArgs a = gang_args(d.n, d.row_ptr, d.col, d.rrow_ptr, d.rcol, d.accepting0, base, ba.results + gi,
                                 ba.flags, d.options);
    map_body_gang(a, ba.gctrl + gi, nb, rank);
  }
}

// ----------------------------------------------------------------- engine --
//
// A persistent server kernel: one cooperative launch that runs until the host
// asks it to stop.  The host posts jobs (an edge list to turn into a CSR and
// check) into fine-grained host memory; a job whose gang has g workgroups
// takes g consecutive tickets, each naming (job slot, rank).  Workgroups take
// tickets in order from a device counter, so, as in the batch queue, every gang
// is completed by workgroups that free up and never waits on a later ticket.
// Only the workgroup holding the first unpublished ticket polls host memory; it
// mirrors the host's ticket count into device memory for the other waiters.

struct EngineShared {          // fine-grained host memory, shared with the host
  unsigned long long tail;     // tickets published by the host
  uint32_t stop;               // host: exit once every published ticket is taken
  uint32_t expired;            // device: the idle bound elapsed and the engine exited
  uint32_t pad[28];
};
static_assert(sizeof(EngineShared) == 128, "shared block is one 128-byte line");

struct alignas(128) EngineDev {  // device memory
  unsigned long long head;       // next ticket to hand out
  unsigned long long pad0[15];
  unsigned long long mirror;     // the host's ticket count as last seen by the polling workgroup
  unsigned long long pad1[15];
  uint32_t quit;                 // 1: no further ticket will be published
  uint32_t pad2[31];
};

// A job as the engine reads it: the caller's map_job with its inputs resolved
// to device addresses, and whether the edge list lies in host memory.
struct EngineJob {
  map_job j;
  uint64_t host_edges;
};
static_assert(sizeof(EngineJob) % 8 == 0, "jobs are read as 64-bit words");

struct EngineArgs {
  EngineShared* sh;                // device address of the shared host block
  const unsigned long long* ring;  // [ring_cap] host: (slot << 32) | rank
  const EngineJob* jobs;           // [slots] host
  map_result* hres;                // [slots] host: status MAP_PENDING until the job is done
  EngineDev* dev;
  GangCtrl* bctrl;                 // [slots] barriers of the CSR build
  GangCtrl* mctrl;                 // [slots] barriers of the MAP loop
  map_result* dres;                // [slots] device results
  unsigned long long* ready;       // [slots] first ticket + 1 of the job whose control blocks are zeroed
  int32_t ring_cap;
  int32_t slots;
  uint64_t idle_ticks;             // idle bound in device wall-clock ticks
  uint32_t flags;
};


__device__ uint32_t block_sum_u32(uint32_t x) {
  __shared__ uint32_t s_bs[kWavesPerBlock];
  x = wave_sum_u32(x);
  if ((threadIdx.x & (kWave - 1)) == 0) s_bs[threadIdx.x / kWave] = x;
  __syncthreads();
  uint32_t t = 0;
  for (int i = 0; i < kWavesPerBlock; ++i) t += s_bs[i];
  __syncthreads();
  return t;
}

// Inclusive scan of one value per thread over the block; *total = block sum.
__device__ uint32_t block_scan_u32(uint32_t x, uint32_t* total) {
  __shared__ uint32_t s_ws[kWavesPerBlock];
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t y = (uint32_t)__shfl_up((int)x, off, kWave);
    if (lane >= off) x += y;
  }
  if (lane == kWave - 1) s_ws[w] = x;
  __syncthreads();
  uint32_t pre = 0, tot = 0;
  for (int i = 0; i < kWavesPerBlock; ++i) {
    const uint32_t v = s_ws[i];
    pre += i < w ? v : 0u;
    tot += v;
  }
  __syncthreads();
  *total = tot;
  return x + pre;
}

template <typename C>
__device__ Grid<C> make_grid(C* c, int nb, int b) {
  Grid<C> g;
  g.c = c;
  g.gen = 0;
  g.nblocks = nb;
  g.ngroups = min(nb, kMaxGroups);
  g.group = b % g.ngroups;
  g.group_size = nb / g.ngroups + ((b % g.ngroups) < (nb % g.ngroups) ? 1 : 0);
  g.rank = b;
  return g;
}

// Calls f(src[e], dst[e]) for the edges e = gt, gt + gs, ... of [0, m), and
// copies them to copy_src / copy_dst when those are given.  The arrays may
// live in host memory, where every load is a bus round trip, so when both are
// 16-byte aligned they are read four edges at a time with two such loads per
// array in flight.
template <typename F>
__device__ __forceinline__ void for_edges(const int32_t* src, const int32_t* dst, int64_t m, int64_t gt,
                                          int64_t gs, int32_t* copy_src, int32_t* copy_dst, F f) {
  int64_t e0 = 0;
  if (((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) & 15) == 0) {
    const int64_t q = m / 4;
    const int4* s4 = reinterpret_cast<const int4*>(src);
    const int4* d4 = reinterpret_cast<const int4*>(dst);
    int64_t i = gt;
    for (; i + gs < q; i += 2 * gs) {
      const int4 a = s4[i], b = d4[i], c = s4[i + gs], d = d4[i + gs];
      if (copy_src) {
        reinterpret_cast<int4*>(copy_src)[i] = a;
        reinterpret_cast<int4*>(copy_dst)[i] = b;
        reinterpret_cast<int4*>(copy_src)[i + gs] = c;
        reinterpret_cast<int4*>(copy_dst)[i + gs] = d;
      }
      f(a.x, b.x);
      f(a.y, b.y);
      f(a.z, b.z);
      f(a.w, b.w);
      f(c.x, d.x);
      f(c.y, d.y);
      f(c.z, d.z);
      f(c.w, d.w);
    }
    if (i < q) {
      const int4 a = s4[i], b = d4[i];
      if (copy_src) {
        reinterpret_cast<int4*>(copy_src)[i] = a;
        reinterpret_cast<int4*>(copy_dst)[i] = b;
      }
      f(a.x, b.x);
      f(a.y, b.y);
      f(a.z, b.z);
      f(a.w, b.w);
    }
    e0 = q * 4;
  }
  for (int64_t e = e0 + gt; e < m; e += gs) {
    const int32_t a = src[e], b = dst[e];
    if (copy_src) {
      copy_src[e] = a;
      copy_dst[e] = b;
    }
    f(a, b);
  }
}

// Pull CSR of a job's edge list, built by its gang: the same arrays that
// map_build_csr produces, up to the order of columns inside a row.  cursor is
// int32[n] and part uint32[nb] of scratch.  With stage_src / stage_dst (edge
// list in host memory) the histogram pass also copies the edges there, so the
// bus is crossed once and the scatter reads device memory.  Returns false if a
// gang barrier timed out; *bad = edges with an endpoint outside 1..n (the CSR
// is then unspecified and the gang stops after the histogram).
__device__ bool gang_build_csr(const map_job& j, int32_t* cursor, uint32_t* part, int32_t* stage_src,
                               int32_t* stage_dst, Grid<GangCtrl>& g, int nb, int rank, uint32_t* bad,
                               int32_t* rp, int32_t* col, const int32_t* esrc, const int32_t* edst, bool swap) {
  const int32_t n = j.n;
  const int64_t m = j.m;
  const int64_t gt = (int64_t)rank * kBlock + threadIdx.x, gs = (int64_t)nb * kBlock;
  for (int64_t i = gt; i <= n; i += gs) rp[i] = 0;
  if (!grid_sync(g, 0u, nullptr)) return false;
  // Degree histogram: the count of row v (vertex v+1) lands at rp[v+1].
  uint32_t nbad = 0;
  for_edges(esrc, edst, m, gt, gs, stage_src, stage_dst, [&](int32_t s, int32_t d) {
    if (s < 1 || s > n || d < 1 || d > n) {
      ++nbad;
      return;
    }
    __hip_atomic_fetch_add(&rp[swap ? d : s], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  });
  nbad = block_sum_u32(nbad);
  uint32_t tot = 0;
  if (!grid_sync(g, nbad, &tot)) return false;
  *bad = tot;
  if (tot) return true;
  // Inclusive scan of rp[0..n]: chunk totals, then each block scans its chunk
  // from the sum of the chunks before it.
  const int64_t len = (int64_t)n + 1, chunk = (len + nb - 1) / nb;
  const int64_t lo = min(len, (int64_t)rank * chunk), hi = min(len, lo + chunk);
  uint32_t sum = 0;
  for (int64_t i = lo + threadIdx.x; i < hi; i += kBlock) sum += (uint32_t)rp[i];
  sum = block_sum_u32(sum);
  if (threadIdx.x == 0) st_agent(&part[rank], sum);
  if (!grid_sync(g, 0u, nullptr)) return false;
  uint32_t off = 0;
  for (int i = threadIdx.x; i < rank; i += kBlock) off += ld_agent(&part[i]);
  off = block_sum_u32(off);
  for (int64_t base = lo; base < hi; base += kBlock) {
    const int64_t i = base + threadIdx.x;
    uint32_t piece = 0;
    const uint32_t incl = block_scan_u32(i < hi ? (uint32_t)rp[i] : 0u, &piece);
    if (i < hi) rp[i] = (int32_t)(off + incl);
    off += piece;
  }
  if (!grid_sync(g, 0u, nullptr)) return false;
  for (int64_t r = gt; r < n; r += gs) cursor[r] = rp[r];
  if (!grid_sync(g, 0u, nullptr)) return false;
  const int32_t* src = stage_src ? stage_src : esrc;
  const int32_t* dst = stage_src ? stage_dst : edst;
  for_edges(src, dst, m, gt, gs, nullptr, nullptr, [&](int32_t s, int32_t d) {
    const int32_t r = swap ? d : s, c = swap ? s : d;
    const int32_t pos = __hip_atomic_fetch_add(&cursor[r - 1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    col[pos] = c - 1;
  });
  return grid_sync(g, 0u, nullptr);
}

// One ticket of a job: rank `rank` of its gang.  Rank 0 zeroes the job's
// control blocks before any rank uses them, and publishes the result to host
// memory after every other rank has left the job.
__device__ __noinline__ void engine_job(const EngineArgs& ea, int slot, int rank, unsigned long long start) {
  constexpr int kJobWords = (int)(sizeof(EngineJob) / 8);
  __shared__ unsigned long long s_job[kJobWords];
  __shared__ int s_ready;
  if (threadIdx.x < kJobWords)
    s_job[threadIdx.x] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(ea.jobs + slot) + threadIdx.x,
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __syncthreads();
  EngineJob ej;
  memcpy(&ej, s_job, sizeof(ej));
  const map_job& j = ej.j;
  const int nb = max(1, min(j.gang, min((int)gridDim.x, kMaxGang)));
  GangCtrl* bc = ea.bctrl + slot;
  GangCtrl* mcx = ea.mctrl + slot;
  map_result* res = ea.dres + slot;
  char* sc = static_cast<char*>(j.scratch);
  // Scratch: packed values | working flags | bitmaps of the filtered sweeps |
  // scan partials | staged edge list (src, dst) | transposed CSR.
  const size_t pv_bytes = ((size_t)j.n * 4 + 255) & ~(size_t)255;
  const size_t acc_bytes = ((size_t)j.n + 255) & ~(size_t)255;
  const size_t bm_bytes = 4 * (size_t)gang_bitmap_bytes(j.n);
  const size_t edge_bytes = ((size_t)j.m * 4 + 255) & ~(size_t)255;
  char* part = sc + pv_bytes + acc_bytes + bm_bytes;
  char* stage = part + (size_t)kMaxGang * 4;
  int32_t* rrow = reinterpret_cast<int32_t*>(stage + 2 * edge_bytes);
  int32_t* rcol = reinterpret_cast<int32_t*>(stage + 2 * edge_bytes + (((size_t)j.n * 4 + 4 + 255) & ~(size_t)255));
  const bool dir = (ea.flags & MAP_FLAG_DIRECTION) != 0;

  if (rank == 0) {
    uint32_t* pb = reinterpret_cast<uint32_t*>(bc);
    uint32_t* pm = reinterpret_cast<uint32_t*>(mcx);
    for (int i = threadIdx.x; i < (int)(kGangCtrlBytes / 4); i += kBlock) {
      pb[i] = 0u;
      pm[i] = 0u;
    }
    if (threadIdx.x < 8) reinterpret_cast<uint32_t*>(res)[threadIdx.x] = 0u;
    wave_writes_done();
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __hip_atomic_store(ea.ready + slot, start + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_ready = 1;
    }
  } else if (threadIdx.x == 0) {
    int ok = 1;
    const uint64_t t0 = wall_clock64();
    while (__hip_atomic_load(ea.ready + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != start + 1) {
      __builtin_amdgcn_s_sleep(2);
      if (wall_clock64() - t0 > kWaitTicks) {
        ok = 0;
        break;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    s_ready = ok;
  }
  __syncthreads();
  bool ok = s_ready != 0;
  uint32_t bad = 0;
  if (ok) {
    Grid<GangCtrl> g = make_grid(bc, nb, rank);
    int32_t* ss = ej.host_edges ? reinterpret_cast<int32_t*>(stage) : nullptr;
    int32_t* sd = ej.host_edges ? reinterpret_cast<int32_t*>(stage + edge_bytes) : nullptr;
    ok = gang_build_csr(j, reinterpret_cast<int32_t*>(sc), reinterpret_cast<uint32_t*>(part), ss, sd, g, nb, rank,
                        &bad, j.row_ptr, j.col, j.src, j.dst, false);
    // MAP_FLAG_DIRECTION: the transposed CSR too, from the staged copy of a
    // host edge list.
    if (ok && bad == 0 && dir)
      ok = gang_build_csr(j, reinterpret_cast<int32_t*>(sc), reinterpret_cast<uint32_t*>(part), nullptr, nullptr, g,
                          nb, rank, &bad, rrow, rcol, ss ? ss : j.src, ss ? sd : j.dst, true);
  }
  if (ok && bad == 0) {
    const LoopArgs a = gang_args(j.n, j.row_ptr, j.col, dir ? rrow : nullptr, dir ? rcol : nullptr, j.accepting0, sc,
                                 res, ea.flags, dir ? (MAP_GRAPH_FILTER | MAP_GRAPH_DIRECTION) : 0);
    map_body_gang(a, mcx, nb, rank);
  }
  // Leave the job: release this block's writes, then report (ranks > 0) or
  // wait for the others and publish the result (rank 0).
  wave_writes_done();
  __syncthreads();
  if (threadIdx.x == 0) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (rank != 0) {
      __hip_atomic_fetch_add(&bc->dirty, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      int waited = 1;
      const uint64_t t0 = wall_clock64();
      while (ld_agent(&bc->dirty) != (uint32_t)(nb - 1)) {
        __builtin_amdgcn_s_sleep(2);
        if (wall_clock64() - t0 > kWaitTicks) {
          waited = 0;
          break;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      const int32_t* d = reinterpret_cast<const int32_t*>(res);
      int32_t r[8];
      for (int i = 0; i < 8; ++i) r[i] = __hip_atomic_load(d + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool broken = !ok || !waited || ld_agent((const uint32_t*)&bc->abort) ||
                          ld_agent((const uint32_t*)&mcx->abort);
      if (broken || bad) {
        for (int i = 0; i < 8; ++i) r[i] = 0;
        r[3] = broken ? MAP_EDEVICE : MAP_ERANGE_DEV;
      }
      int32_t* h = reinterpret_cast<int32_t*>(ea.hres + slot);
      for (int i = 0; i < 8; ++i)
        if (i != 3) __hip_atomic_store(h + i, r[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
      __hip_atomic_store(h + 3, r[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
  __syncthreads();
}

__global__ void __launch_bounds__(kBlock) map_engine_kernel(EngineArgs ea) {
  __shared__ int32_t s_slot, s_rank, s_quit;
  __shared__ unsigned long long s_start;
  for (;;) {
    if (threadIdx.x == 0) {
      const unsigned long long t =
          __hip_atomic_fetch_add(&ea.dev->head, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      int quit = 0;
      uint64_t t0 = wall_clock64();
      unsigned long long seen = ~0ull;
      for (;;) {
        const unsigned long long mir = __hip_atomic_load(&ea.dev->mirror, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t < mir) break;
        if (ld_agent(&ea.dev->quit)) {
          quit = 1;
          break;
        }
        if (mir != seen) {  // progress: restart the idle clock
          seen = mir;
          t0 = wall_clock64();
        }
        if (t == mir) {
          // This block holds the first unpublished ticket: it polls the host.
          unsigned long long tail = __hip_atomic_load(&ea.sh->tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          if (tail == mir && __hip_atomic_load(&ea.sh->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM)) {
            // The host publishes before it stops: read the count once more.
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
            tail = __hip_atomic_load(&ea.sh->tail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            if (tail == mir) {
              st_agent(&ea.dev->quit, 1u);
              quit = 1;
              break;
            }
          }
          if (tail > mir) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
            __hip_atomic_store(&ea.dev->mirror, tail, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            continue;
          }
        }
        if (wall_clock64() - t0 > ea.idle_ticks) {
          st_agent(&ea.dev->quit, 1u);
          __hip_atomic_store(&ea.sh->expired, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
          quit = 1;
          break;
        }
        if (t == mir) __builtin_amdgcn_s_sleep(1);
        else __builtin_amdgcn_s_sleep(8);
      }
      s_quit = quit;
      if (!quit) {
        // Acquire the host's writes of the ticket, its job and the job's device
        // buffers (filled by copies the host waited for before publishing).
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "");
        const unsigned long long e = __hip_atomic_load(ea.ring + (t % (unsigned long long)ea.ring_cap),
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        s_slot = (int32_t)(e >> 32);
        s_rank = (int32_t)(e & 0xffffffffu);
        s_start = t - (e & 0xffffffffu);
      }
    }
    __syncthreads();
    const int quit = s_quit, slot = s_slot, rank = s_rank;
    const unsigned long long start = s_start;
    __syncthreads();
    if (quit) break;
    if (slot >= 0 && slot < ea.slots) engine_job(ea, slot, rank, start);
  }
}

// Batch set-up (one block): gang sizes -> work item offsets, scratch offsets,
// and the scratch size check.
__global__ void __launch_bounds__(1024) batch_plan(int32_t count, const map_graph_desc* graphs,
                                                   const int32_t* gang, int32_t* item_start, int64_t* scratch_off,
                                                   size_t scratch_bytes, int32_t max_gang, int32_t* status,
                                                   uint32_t* next_item) {
  __shared__ int64_t part_i[1024];
  __shared__ int64_t part_b[1024];
  const int64_t per = ((int64_t)count + 1023) / 1024;
  const int64_t lo = (int64_t)threadIdx.x * per, hi = min((int64_t)count, lo + per);
  int64_t si = 0, sb = 0;
  for (int64_t i = lo; i < hi; ++i) {
    int32_t gsz = gang ? gang[i] : 1;
    gsz = max(1, min(gsz, max_gang));
    si += gsz;
    sb += gang_scratch_bytes(graphs[i].n, graphs[i].options);
  }
  part_i[threadIdx.x] = si;
  part_b[threadIdx.x] = sb;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int64_t yi = threadIdx.x >= off ? part_i[threadIdx.x - off] : 0;
    const int64_t yb = threadIdx.x >= off ? part_b[threadIdx.x - off] : 0;
    __syncthreads();
    part_i[threadIdx.x] += yi;
    part_b[threadIdx.x] += yb;
    __syncthreads();
  }
  int64_t pi = threadIdx.x ? part_i[threadIdx.x - 1] : 0;
  int64_t pb = threadIdx.x ? part_b[threadIdx.x - 1] : 0;
  for (int64_t i = lo; i < hi; ++i) {
    item_start[i] = (int32_t)pi;
    scratch_off[i] = pb;
    int32_t gsz = gang ? gang[i] : 1;
    pi += max(1, min(gsz, max_gang));
    pb += gang_scratch_bytes(graphs[i].n, graphs[i].options);
  }
  if (threadIdx.x == 1023) {
    item_start[count] = (int32_t)part_i[1023];
    *status = (size_t)part_b[1023] <= scratch_bytes ? MAP_OK : MAP_ENOSPC;
    *next_item = 0;
  }
}

// --------------------------------------------------------------- CSR build --

// CSR build: the path a build takes, chosen on the device (csr_pick) and read
// by every kernel of both paths, which return at once when it is not theirs.
constexpr int32_t kBuildAtomic = 1;  // per-row cursors, one atomic per run of equal keys, then row ordering
constexpr int32_t kBuildRadix = 2;   // stable radix sort by key (keys mostly differ from their neighbour's)
constexpr int32_t kBuildSorted = 3;  // keys ascend already: one pass, given up at the first edge that breaks the order

// One orientation of a build (the pull CSR: key = source; the transposed one:
// key = target) and its share of the workspace.  The kernels of the cursor
// path take both at once, blockIdx.y naming the side.
struct BuildSide {
  const int32_t* key;
  const int32_t* other;
  int32_t* row_ptr;
  int32_t* col;
  int32_t* cursor;  // [n + 1], then the lists of longer rows; sorted path: long gaps of the row pointers
  int32_t* sums;
  int32_t* counts;  // two list counts, the build path, the path if the keys turn out unsorted, the long gaps
  int32_t* ids;     // edge index of every slot
};
struct BuildArgs {
  BuildSide side[2];
  int32_t n;
  int32_t vec;  // 1: the edge arrays and columns are 16-byte aligned
  int64_t m;
  int32_t* status;
};
__device__ __forceinline__ bool build_is(const BuildSide& b, int32_t path) {
  return __hip_atomic_load(&b.counts[2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == path;
}
constexpr int kScanThreads = 256;
constexpr int kScanPer = 16;
constexpr int kScanTile = kScanThreads * kScanPer;

__global__ void fill_u32(uint32_t* p, int64_t count, uint32_t val) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = val;
}

// Clears the row pointers for the cursor path's histogram (and for an empty
// edge list); on the sorted path fills their long gaps, a piece per workgroup.
__global__ void csr_zero(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (build_is(sd, kBuildSorted)) {
    const int32_t pieces = sd.counts[4];
    for (int32_t i = blockIdx.x; i < pieces; i += gridDim.x) {
      const int32_t b = sd.cursor[3 * (int64_t)i], e = sd.cursor[3 * (int64_t)i + 1], x = sd.cursor[3 * (int64_t)i + 2];
      for (int64_t r = (int64_t)b + threadIdx.x; r < e; r += blockDim.x) sd.row_ptr[r] = x;
    }
  }
  if (!build_is(sd, kBuildAtomic)) return;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i <= a.n; i += (int64_t)gridDim.x * blockDim.x)
    sd.row_ptr[i] = 0;
}

// Runs of equal keys among a wave's 64 consecutive edges.  Edge lists in
// generation order come grouped by source, so one atomic per run instead of
// one per edge takes most of the atomic traffic out of the build; on lists in
// random order nearly every run has length 1 and nothing changes.  A run
// starts at a valid lane whose key differs from the previous lane's (or whose
// previous lane is invalid, or at lane 0) and ends before the next start or
// invalid lane.  All 64 lanes must call it (the wave walks the edges in
// wave-aligned steps).
struct KeyRun {
  bool head;  // this lane starts a run
  int len;    // head: lanes in the run
  int first;  // valid lane: the lane that starts its run
};

__device__ __forceinline__ KeyRun key_run(bool valid, int32_t k, int lane) {
  const int32_t pk = __shfl_up(k, 1, kWave);
  const int pv = __shfl_up(valid ? 1 : 0, 1, kWave);
  const bool head = valid && (lane == 0 || pv == 0 || pk != k);
  const unsigned long long heads = __ballot(head);
  const unsigned long long stops = heads | ~__ballot(valid);
  const unsigned long long upto = (2ull << lane) - 1ull;  // lanes 0..lane (all 64 for lane 63)
  const unsigned long long after = stops & ~upto;
  KeyRun r;
  r.head = head;
  r.len = (after ? __builtin_ctzll(after) : kWave) - lane;
  const unsigned long long before = heads & upto;
  r.first = before ? 63 - __builtin_clzll(before) : lane;
  return r;
}

// Degree histogram of the key endpoint: cnt[key] += (edges with that key)
// (cnt = row_ptr, so row v's count lands at index v+1 for 1-based key v+1).
__global__ void csr_hist(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (!build_is(sd, kBuildAtomic)) return;
  const int32_t n = a.n;
  const int64_t m = a.m;
  const int32_t* __restrict__ key = sd.key;
  const int32_t* __restrict__ other = sd.other;
  int32_t* cnt = sd.row_ptr;
  int32_t* status = a.status;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t w0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); w0 < m; w0 += stride) {
    const int64_t i = w0 + lane;
    int32_t k = 0;
    bool valid = false;
    if (i < m) {
      const int32_t o = other[i];
      k = key[i];
      valid = k >= 1 && k <= n && o >= 1 && o <= n;
      if (!valid) __hip_atomic_store(status, (int32_t)MAP_ERANGE_DEV, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const KeyRun r = key_run(valid, k, lane);
    if (r.head) atomicAdd(&cnt[k], r.len);
  }
}

// In-place inclusive scan of each tile of kScanTile elements; tile totals to sums.
__device__ __forceinline__ void scan_tile(int32_t* a, int64_t len, int32_t* sums) {
  __shared__ int32_t part[kScanThreads];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanPer;
  int32_t x[kScanPer];
  int32_t run = 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    int64_t i = base + j;
    run += (i < len) ? a[i] : 0;
    x[j] = run;
  }
  part[threadIdx.x] = run;
  __syncthreads();
  for (int off = 1; off < kScanThreads; off <<= 1) {
    int32_t y = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
    __syncthreads();
    part[threadIdx.x] += y;
    __syncthreads();
  }
  int32_t pre = threadIdx.x ? part[threadIdx.x - 1] : 0;
#pragma unroll
  for (int j = 0; j < kScanPer; ++j) {
    int64_t i = base + j;
    if (i < len) a[i] = x[j] + pre;
  }
  if (threadIdx.x == kScanThreads - 1) sums[blockIdx.x] = part[kScanThreads - 1];
}

__global__ void __launch_bounds__(kScanThreads) scan_tiles(const int32_t* gate, int32_t want, int32_t* a, int64_t len,
                                                          int32_t* sums) {
  if (*gate == want) scan_tile(a, len, sums);
}

__global__ void __launch_bounds__(kScanThreads) rows_scan_tiles(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (build_is(sd, kBuildAtomic)) scan_tile(sd.row_ptr, (int64_t)a.n + 1, sd.sums);
}

// Exclusive scan of the tile totals by one workgroup.
__device__ __forceinline__ void scan_totals(int32_t* sums, int64_t count) {
  __shared__ int32_t part[1024];
  const int64_t per = (count + 1023) / 1024;
  const int64_t lo = (int64_t)threadIdx.x * per, hi = min(count, lo + per);
  int32_t run = 0;
  for (int64_t i = lo; i < hi; ++i) run += sums[i];
  part[threadIdx.x] = run;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    int32_t y = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
    __syncthreads();
    part[threadIdx.x] += y;
    __syncthreads();
  }
  int32_t pre = threadIdx.x ? part[threadIdx.x - 1] : 0;
  for (int64_t i = lo; i < hi; ++i) {
    int32_t v = sums[i];
    sums[i] = pre;
    pre += v;
  }
}

__global__ void __launch_bounds__(1024) scan_sums(const int32_t* gate, int32_t want, int32_t* sums, int64_t count) {
  if (*gate == want) scan_totals(sums, count);
}

__global__ void __launch_bounds__(1024) rows_scan_sums(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (build_is(sd, kBuildAtomic)) scan_totals(sd.sums, ((int64_t)a.n + kScanTile) / kScanTile);
}

// Row pointers complete, and copied to the cursors.
__global__ void __launch_bounds__(kScanThreads) rows_scan_add(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (!build_is(sd, kBuildAtomic)) return;
  const int64_t tile = blockIdx.x, len = (int64_t)a.n + 1;
  const int32_t pre = sd.sums[tile];
  for (int64_t i = tile * kScanTile + threadIdx.x; i < min(len, (tile + 1) * kScanTile); i += blockDim.x) {
    const int32_t x = sd.row_ptr[i] + pre;
    sd.row_ptr[i] = x;
    sd.cursor[i] = x;
  }
}

__global__ void scan_add(const int32_t* gate, int32_t want, int32_t* a, int64_t len, const int32_t* sums) {
  if (*gate != want) return;
  const int64_t tile = blockIdx.x;
  const int32_t pre = sums[tile];
  if (pre == 0) return;
  for (int64_t i = tile * kScanTile + threadIdx.x; i < min(len, (tile + 1) * kScanTile); i += blockDim.x) a[i] += pre;
}

// col[cursor[key-1]++] = other-1 and ids[same slot] = edge index for every
// in-range edge; a run of equal keys reserves its slots with one atomic and
// fills them in edge order.  The order of the runs inside a row depends on the
// schedule; the csr_order_* kernels then put every row whose edge indices are
// out of order in edge order.
__global__ void csr_scatter(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (!build_is(sd, kBuildAtomic)) return;
  const int32_t n = a.n;
  const int64_t m = a.m;
  const int32_t* __restrict__ key = sd.key;
  const int32_t* __restrict__ other = sd.other;
  int32_t* cursor = sd.cursor;
  int32_t* col = sd.col;
  int32_t* ids = sd.ids;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t w0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); w0 < m; w0 += stride) {
    const int64_t i = w0 + lane;
    int32_t k = 0, o = 0;
    bool valid = false;
    if (i < m) {
      k = key[i];
      o = other[i];
      valid = k >= 1 && k <= n && o >= 1 && o <= n;
    }
    const KeyRun r = key_run(valid, k, lane);
    int32_t pos = 0;
    if (r.head) pos = atomicAdd(&cursor[k - 1], r.len);
    pos = __shfl(pos, r.first, kWave) + (lane - r.first);
    if (valid) {
      col[pos] = o - 1;
      ids[pos] = (int32_t)i;
    }
  }
}

// Putting each row in edge order: rows of at most kOrderShort edges by one
// lane, rows of at most 64 by one wave, longer rows by one workgroup.  A row
// whose edge indices already ascend (the usual case for edge lists grouped by
// source, where one wave's run fills most rows) is only read.
constexpr int kOrderShort = 16;
constexpr int kOrderChunk = 4096;   // long rows: entries sorted in LDS at a time
constexpr int kOrderThreads = 1024;
constexpr int kOrderLongGrid = 256;

// Appends `val` for every lane with `take` to list[count...] (from the back,
// list[back - 1 - index], when back > 0).  All 64 lanes must call it.
__device__ void wave_list_append(bool take, int32_t val, int32_t* list, int32_t* count, int64_t back, int lane) {
  const unsigned long long mask = __ballot(take);
  if (!mask) return;
  const int leader = __builtin_ctzll(mask);
  int32_t base = 0;
  if (lane == leader) base = atomicAdd(count, __popcll(mask));
  base = __shfl(base, leader, kWave);
  const int64_t idx = base + __popcll(mask & ((1ull << lane) - 1ull));
  if (take) list[back > 0 ? back - 1 - idx : idx] = val;
}

// A row of 2..W edges in one lane: its edge indices are loaded together (no
// branch between the loads, so their latencies overlap) and, unless they
// ascend, each column is written at the rank of its edge index in the row.
template <int W>
__device__ __forceinline__ void order_short_row(int32_t b, int32_t d, int32_t* col, const int32_t* __restrict__ ids) {
  int32_t e[W];
#pragma unroll
  for (int k = 0; k < W; ++k) e[k] = k < d ? ids[b + k] : INT32_MAX;
  bool sorted = true;
#pragma unroll
  for (int k = 1; k < W; ++k) sorted = sorted && e[k - 1] < e[k];
  if (sorted) return;
  int32_t o[W];
#pragma unroll
  for (int k = 0; k < W; ++k) o[k] = k < d ? col[b + k] : 0;
#pragma unroll
  for (int k = 0; k < W; ++k) {
    int rank = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) rank += e[q] < e[k] ? 1 : 0;
    if (k < d) col[b + rank] = o[k];
  }
}

// One lane per row of 2..kOrderShort edges (order_short_row, at the width of
// the wave's longest such row).  Rows of kOrderShort+1..64 edges go to the
// front of `lists` (count counts[0]), longer ones to its back (n entries,
// count counts[1]); both counts start at zero.  Waves step over the rows in
// grid strides (the launch grid is capped).
__global__ void csr_order_rows(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (!build_is(sd, kBuildAtomic)) return;
  const int32_t n = a.n;
  const int32_t* __restrict__ row_ptr = sd.row_ptr;
  int32_t* col = sd.col;
  const int32_t* __restrict__ ids = sd.ids;
  int32_t* lists = sd.cursor;  // the cursors are spent
  int32_t* counts = sd.counts;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r0 = (int64_t)blockIdx.x * blockDim.x + (threadIdx.x & ~(kWave - 1)); r0 < n; r0 += stride) {
    const int64_t r = r0 + lane;
    int32_t b = 0, d = 0;
    if (r < n) {
      b = row_ptr[r];
      d = row_ptr[r + 1] - b;
    }
    wave_list_append(d > kOrderShort && d <= kWave, (int32_t)r, lists, &counts[0], 0, lane);
    wave_list_append(d > kWave, (int32_t)r, lists, &counts[1], n, lane);
    const bool mine = d >= 2 && d <= kOrderShort;
    int dm = mine ? d : 0;  // longest short row of the wave
    for (int off = kWave / 2; off > 0; off >>= 1) dm = max(dm, __shfl_xor(dm, off, kWave));
    if (!mine) continue;
    if (dm <= 4)
      order_short_row<4>(b, d, col, ids);
    else if (dm <= 8)
      order_short_row<8>(b, d, col, ids);
    else
      order_short_row<kOrderShort>(b, d, col, ids);
  }
}

// One wave per listed row of kOrderShort+1..64 edges: lane l holds entry l;
// unless the edge indices ascend, each lane counts the lanes with a smaller
// one and writes its column there.
__device__ __forceinline__ void order_mid_rows(const BuildSide& sd) {
  const int32_t* __restrict__ row_ptr = sd.row_ptr;
  int32_t* col = sd.col;
  const int32_t* __restrict__ ids = sd.ids;
  const int32_t* __restrict__ lists = sd.cursor;
  const int32_t* __restrict__ counts = sd.counts;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t gw = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = (int64_t)gridDim.x * blockDim.x / kWave;
  const int32_t cnt = counts[0];
  for (int64_t li = gw; li < cnt; li += nw) {
    const int32_t r = lists[li];
    const int32_t b = row_ptr[r], d = row_ptr[r + 1] - b;
    const int32_t e = lane < d ? ids[b + lane] : INT32_MAX;
    const int32_t prev = __shfl_up(e, 1, kWave);
    if (!__ballot(lane > 0 && lane < d && prev > e)) continue;
    const int32_t o = lane < d ? col[b + lane] : 0;
    int rank = 0;
#pragma unroll
    for (int q = 0; q < kWave; ++q) rank += __builtin_amdgcn_readlane(e, q) < e ? 1 : 0;
    if (lane < d) col[b + rank] = o;  // every lane's read precedes (the ranks depend on all of them)
  }
}

// Compare-exchange step of an ascending bitonic sort over se/so[0, S): pairs
// (i, i ^ (k - 1)) on the first step of merge size k, else (i, i + j); the
// smaller edge index goes to the lower position.
__device__ void order_lds_step(int32_t* se, int32_t* so, int S, int k, int j, bool first) {
  for (int t = threadIdx.x; t < S / 2; t += blockDim.x) {
    const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
    const int p = first ? (i ^ (k - 1)) : (i + j);
    const int32_t x = se[i], y = se[p];
    if (x > y) {
      se[i] = y;
      se[p] = x;
      const int32_t z = so[i];
      so[i] = so[p];
      so[p] = z;
    }
  }
  __syncthreads();
}

// The same step over a whole row in global memory (E edge indices, O columns,
// d entries, P the power of two the network spans).  Positions d and beyond
// stand for +infinity: a pair that reaches one never exchanges.
__device__ void order_global_step(int32_t* E, int32_t* O, int64_t d, int64_t P, int64_t k, int64_t j, bool first) {
  for (int64_t t = threadIdx.x; t < P / 2; t += blockDim.x) {
    const int64_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
    const int64_t p = first ? (i ^ (k - 1)) : (i + j);
    if (p >= d) continue;
    const int32_t x = E[i], y = E[p];
    if (x > y) {
      E[i] = y;
      E[p] = x;
      const int32_t z = O[i];
      O[i] = O[p];
      O[p] = z;
    }
  }
  __syncthreads();
}

// Entries [c0, c0 + S) of a row through LDS: either a whole bitonic sort of
// the chunk (k == 0) or the steps j = S/2 .. 1 of merge size k.  The entries
// below d go back to E and O, or only to O on the chunk's last pass.
__device__ void order_lds_chunk(int32_t* se, int32_t* so, int32_t* E, int32_t* O, int64_t d, int64_t c0, int S,
                                int64_t k, bool last) {
  for (int i = threadIdx.x; i < S; i += blockDim.x) {
    const int64_t g = c0 + i;
    se[i] = g < d ? E[g] : INT32_MAX;
    so[i] = g < d ? O[g] : 0;
  }
  __syncthreads();
  if (k == 0) {
    for (int kk = 2; kk <= S; kk <<= 1) {
      order_lds_step(se, so, S, kk, kk >> 1, true);
      for (int j = kk >> 2; j > 0; j >>= 1) order_lds_step(se, so, S, kk, j, false);
    }
  } else {
    for (int j = S >> 1; j > 0; j >>= 1) order_lds_step(se, so, S, 0, j, false);
  }
  for (int i = threadIdx.x; i < S; i += blockDim.x) {
    const int64_t g = c0 + i;
    if (g >= d) break;
    if (!last) E[g] = se[i];
    O[g] = so[i];
  }
  __syncthreads();
}

// One workgroup per listed row of more than 64 edges (from the back of
// `lists`, count counts[1]) whose edge indices do not ascend: an ascending
// bitonic sort of (edge index, column) pairs, in LDS for rows of up to
// kOrderChunk entries, else chunks sorted in LDS and merged by steps over the
// row in global memory (the row's edge indices are scratch).  The rows of up
// to 64 edges go first, one per wave.
__global__ void __launch_bounds__(kOrderThreads) csr_order_listed(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (!build_is(sd, kBuildAtomic)) return;
  order_mid_rows(sd);
  const int32_t n = a.n;
  const int32_t* __restrict__ row_ptr = sd.row_ptr;
  int32_t* col = sd.col;
  int32_t* ids = sd.ids;
  const int32_t* __restrict__ lists = sd.cursor;
  const int32_t* __restrict__ counts = sd.counts;
  __shared__ int32_t se[kOrderChunk];
  __shared__ int32_t so[kOrderChunk];
  const int32_t cnt = counts[1];
  for (int32_t li = blockIdx.x; li < cnt; li += gridDim.x) {
    const int32_t r = lists[(int64_t)n - 1 - li];
    const int64_t b = row_ptr[r];
    const int64_t d = (int64_t)row_ptr[r + 1] - b;
    int32_t* E = ids + b;
    int32_t* O = col + b;
    int descents = 0;
    for (int64_t i = 1 + threadIdx.x; i < d; i += blockDim.x) descents |= E[i - 1] > E[i] ? 1 : 0;
    if (!__syncthreads_or(descents)) continue;
    if (d <= kOrderChunk) {
      int S = 2 * kWave;
      while (S < d) S <<= 1;
      order_lds_chunk(se, so, E, O, d, 0, S, 0, true);
      continue;
    }
    int64_t P = kOrderChunk;
    while (P < d) P <<= 1;
    for (int64_t c0 = 0; c0 < d; c0 += kOrderChunk) order_lds_chunk(se, so, E, O, d, c0, kOrderChunk, 0, false);
    for (int64_t k = 2 * (int64_t)kOrderChunk; k <= P; k <<= 1) {
      order_global_step(E, O, d, P, k, k >> 1, true);
      for (int64_t j = k >> 2; j >= kOrderChunk; j >>= 1) order_global_step(E, O, d, P, k, j, false);
      for (int64_t c0 = 0; c0 < d; c0 += kOrderChunk) order_lds_chunk(se, so, E, O, d, c0, kOrderChunk, k, k == P);
    }
  }
}

// Picks each side's build path from 1024 evenly spaced pairs of neighbouring
// edges, and sets the list counts and the status.  No pair descends: the list
// is taken as sorted by the key (csr_sorted, which checks every edge).
// Otherwise, when most pairs differ in key, runs of equal keys are short and
// every edge would take its own atomic, so the radix sort (bandwidth-bound) is
// taken, from kRadixMinEdges edges: below, its kernels are not even launched
// (their twenty-odd launches cost more than the atomics they would save).
constexpr int64_t kRadixMinEdges = 1 << 20;
__global__ void __launch_bounds__(1024) csr_pick(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  __shared__ uint32_t s_diff, s_down;
  if (threadIdx.x == 0) s_diff = s_down = 0;
  __syncthreads();
  uint32_t d = 0, down = 0;
  if (a.m > 1) {
    const int64_t i = (a.m - 1) * (int64_t)threadIdx.x / 1024;
    d = sd.key[i] != sd.key[i + 1] ? 1u : 0u;
    down = sd.key[i] > sd.key[i + 1] ? 1u : 0u;
  }
  d = wave_sum_u32(d);
  down = wave_sum_u32(down);
  if ((threadIdx.x & (kWave - 1)) == 0) {
    if (d) atomicAdd(&s_diff, d);
    if (down) atomicAdd(&s_down, down);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const int32_t path = a.m >= kRadixMinEdges && 2 * s_diff > 1024 ? kBuildRadix : kBuildAtomic;
    sd.counts[0] = sd.counts[1] = sd.counts[4] = 0;
    sd.counts[2] = a.m > 0 && s_down == 0 ? kBuildSorted : path;
    sd.counts[3] = path;
    if (blockIdx.y == 0) *a.status = MAP_OK;
  }
}

// Row pointers of the rows [r0, r1) of each lane set to `val`: a few by the
// lane, a longer run by the whole wave (one lane alone takes 20 ns a row, and
// the rows after the last edge of a growing graph are many).  All lanes call it.
constexpr int kRowGap = 8;
__device__ __forceinline__ void fill_rows(int32_t* row_ptr, int32_t r0, int32_t r1, int32_t val, int lane) {
  const bool longrun = r1 - r0 > kRowGap;
  if (!longrun)
    for (int32_t r = r0; r < r1; ++r) row_ptr[r] = val;
  unsigned long long lr = __ballot(longrun);
  while (lr) {
    const int src = __ffsll(lr) - 1;
    lr &= lr - 1;
    const int32_t b = __shfl(r0, src, kWave), e = __shfl(r1, src, kWave), x = __shfl(val, src, kWave);
    for (int64_t r = (int64_t)b + lane; r < e; r += kWave) row_ptr[r] = x;
  }
}

// The same for the sorted path, with gaps of more than kRowLong rows put down
// for csr_zero in pieces, three words of the cursors each: a list of few edges
// over many rows has few waves here (4M rows, 1,000 edges: 496 us when a wave
// filled each of its gaps, 47 us so).  An ascending list has at most
// n / kRowLong + n / kRowPiece pieces; false if they pass the cursors' end, which
// shows that the list does not ascend.  All lanes call it.
constexpr int kRowLong = 512;
constexpr int kRowPiece = 16384;
__device__ __forceinline__ bool fill_or_list(const BuildSide& sd, int32_t n, int32_t r0, int32_t r1, int32_t val,
                                             int lane) {
  const bool far = r1 - r0 > kRowLong;
  fill_rows(sd.row_ptr, r0, far ? r0 : r1, val, lane);
  if (!__ballot(far)) return true;
  const int64_t len = max((int64_t)kRowPiece, (int64_t)n / 256);
  const uint32_t mine = far ? (uint32_t)((r1 - r0 + len - 1) / len) : 0u;
  uint32_t upto = mine;
  for (int d = 1; d < kWave; d *= 2) {
    const uint32_t v = __shfl_up(upto, d, kWave);
    if (lane >= d) upto += v;
  }
  const uint32_t total = __shfl(upto, kWave - 1, kWave);
  uint32_t at = 0;
  if (lane == 0)
    at = __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(&sd.counts[4]), total, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
  at = __shfl(at, 0, kWave);
  if (3 * ((uint64_t)at + total) > (uint64_t)n + 1) return false;
  int32_t* p = sd.cursor + 3 * (int64_t)(at + upto - mine);
  for (int64_t lo = r0; mine && lo < r1; lo += len, p += 3) {
    p[0] = (int32_t)lo;
    p[1] = (int32_t)min((int64_t)r1, lo + len);
    p[2] = val;
  }
  return true;
}

// Sorted path: columns copied and row pointers read off the keys in one pass,
// four consecutive edges per thread (16-byte loads and stores where the arrays
// allow them).  An edge whose key is below its predecessor's, or that has an
// endpoint outside 1..n, ends the attempt: the side's path becomes the other
// one that was picked, whose kernels follow and overwrite everything.  Edge
// lists in generation order (by source) take this path for the pull CSR.
// 134M edges in 0.35 ms (5.0 TB/s with the row pointers; histogram, scan,
// cursors and row ordering took 1.9 ms), 4M in 15 us.
__global__ void __launch_bounds__(256) csr_sorted(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  if (!build_is(sd, kBuildSorted)) return;
  const int32_t n = a.n;
  const int64_t m = a.m, quads = (m + 3) / 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, gs = (int64_t)gridDim.x * blockDim.x;
  bool bad = false;
  for (int64_t q0 = gt - lane; q0 < quads; q0 += gs) {  // whole waves
    const int64_t i0 = 4 * (q0 + lane);
    int32_t k[4] = {0, 0, 0, 0}, o[4];
    int32_t prev = 0;
    const int cnt = (int)max((int64_t)0, min((int64_t)4, m - i0));
    if (cnt > 0 && i0) prev = sd.key[i0 - 1];
    if (a.vec && cnt == 4) {
      const int4 kk = *reinterpret_cast<const int4*>(sd.key + i0), oo = *reinterpret_cast<const int4*>(sd.other + i0);
      k[0] = kk.x, k[1] = kk.y, k[2] = kk.z, k[3] = kk.w;
      o[0] = oo.x, o[1] = oo.y, o[2] = oo.z, o[3] = oo.w;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (u < cnt) k[u] = sd.key[i0 + u];
        o[u] = u < cnt ? sd.other[i0 + u] : 1;
      }
    }
    int32_t from[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      from[u] = k[u];
      if (u < cnt) {
        if (k[u] < 1 || k[u] > n || o[u] < 1 || o[u] > n || k[u] < prev || prev < 0) bad = true;
        from[u] = prev;
        prev = k[u];
      }
    }
    if (__ballot(bad)) break;
    if (a.vec && cnt == 4) {
      *reinterpret_cast<int4*>(sd.col + i0) = make_int4(o[0] - 1, o[1] - 1, o[2] - 1, o[3] - 1);
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (u < cnt) sd.col[i0 + u] = o[u] - 1;
    }
    // Rows from - 1 + 1 .. k - 1 (0-based) start at the edge; before the first
    // edge `from` is 0.
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (!fill_or_list(sd, n, from[u], k[u], (int32_t)(i0 + u), lane)) bad = true;
  }
  if (bad) __hip_atomic_store(&sd.counts[2], sd.counts[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // The rows after the last edge, by the whole grid.
  for (int64_t r = (int64_t)max(sd.key[m - 1], 0) + gt; r <= n; r += gs) sd.row_ptr[r] = (int32_t)m;
}

// Small builds: one workgroup per side sorts the whole edge list by key in LDS
// (least significant digit first, stable, from one buffer to another) and
// writes row pointers and columns.  The code is kept short (no unrolled steps):
// a lone launch finds the instruction cache cold.  An edge is one word, key << 14 | value;
// edges with an endpoint outside 1..n take key n and sort last.  The general
// paths make ten launches; this is one.
// Both orientations of 1,000 vertices: 14 us, 86 us before (twenty-five
// launches); 18,432 edges are what two buffers of LDS hold.
constexpr int kTinyEdges = 18432;
static_assert(kSmallN < (1 << 14), "keys 0..n and values share a word");
__global__ void __launch_bounds__(kBlock) csr_small(BuildArgs a) {
  const BuildSide& sd = a.side[blockIdx.y];
  __shared__ uint32_t buf[2][kTinyEdges];
  __shared__ uint32_t off[kWavesPerBlock][128];
  __shared__ uint32_t loc[128];
  __shared__ uint32_t s_bad;
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wib = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = a.n, m = (int)a.m;
  // Wave w holds edges [w * per, (w + 1) * per), 64 per step.
  const int steps = (m + kBlock - 1) / kBlock, per = steps * kWave;
  const unsigned long long below = lane ? (~0ull >> (kWave - lane)) : 0ull;
  if (tid == 0) s_bad = 0;
  __syncthreads();
#pragma unroll 4
  for (int i = tid; i < m; i += kBlock) {
    const int32_t k = sd.key[i], o = sd.other[i];
    const bool ok = k >= 1 && k <= n && o >= 1 && o <= n;
    buf[0][i] = ok ? (uint32_t)(k - 1) << 14 | (uint32_t)(o - 1) : (uint32_t)n << 14;
    if (!ok) s_bad = 1;
  }
  int bits = 1, cur = 0;
  while ((1 << bits) <= n) ++bits;
  for (int lo = 0; lo < bits; lo += 7, cur ^= 1) {
    const int width = min(7, bits - lo);
    const uint32_t mask = (1u << width) - 1u;
    for (int i = tid; i < kWavesPerBlock * 128; i += kBlock) off[i / 128][i % 128] = 0;
    __syncthreads();
    for (int u = 0; u < steps; ++u) {
      const int i = wib * per + u * kWave + lane;
      if (i < m) atomicAdd(&off[wib][(buf[cur][i] >> (14 + lo)) & mask], 1u);
    }
    __syncthreads();
    if (tid < 128) {
      uint32_t run = 0;
#pragma unroll 1
      for (int w = 0; w < kWavesPerBlock; ++w) {
        const uint32_t c = off[w][tid];
        off[w][tid] = run;
        run += c;
      }
      loc[tid] = run;
    }
    __syncthreads();
    if (wib == 0) {  // exclusive scan of the digit totals, two per lane
      const uint32_t x = loc[2 * lane], y = loc[2 * lane + 1];
      uint32_t incl = x + y;
      for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t z = (uint32_t)__shfl_up((int)incl, o, kWave);
        if (lane >= o) incl += z;
      }
      loc[2 * lane] = incl - x - y;
      loc[2 * lane + 1] = incl - y;
    }
    __syncthreads();
    for (int u = 0; u < steps; ++u) {
      const int i = wib * per + u * kWave + lane;
      const bool ok = i < m;
      const uint32_t e = ok ? buf[cur][i] : 0u;
      const uint32_t d = (e >> (14 + lo)) & mask;
      unsigned long long peers = __ballot(ok);
      for (int bit = 0; bit < width; ++bit) {
        const unsigned long long one = __ballot(ok && ((d >> bit) & 1u));
        peers &= ((d >> bit) & 1u) ? one : ~one;
      }
      const uint32_t rank = (uint32_t)__popcll(peers & below);
      if (ok) buf[cur ^ 1][loc[d] + off[wib][d] + rank] = e;
      wave_lds_sync();  // every lane has read off before the group's lowest lane advances it
      if (ok && rank == 0) off[wib][d] += (uint32_t)__popcll(peers);
      wave_lds_sync();
    }
    __syncthreads();
  }
  for (int i0 = tid - lane; i0 <= m; i0 += kBlock) {
    const int i = i0 + lane;
    const int prev = i == 0 || i > m ? -1 : (int)(buf[cur][i - 1] >> 14);
    const uint32_t x = i < m ? buf[cur][i] : 0u;
    const int key = i < m ? (int)(x >> 14) : i == m ? n : -2;
    fill_rows(sd.row_ptr, prev + 1, key + 1, i, lane);
    if (i < m && key < n) sd.col[i] = (int32_t)(x & 0x3fffu);
  }
  if (tid == 0 && blockIdx.y == 0) *a.status = s_bad ? MAP_ERANGE_DEV : MAP_OK;
}

// Radix path: a least-significant-digit radix sort of (key - 1, other - 1)
// pairs by key, stable in every pass, so each row lists its columns in edge
// order; an edge with an endpoint outside 1..n gets key n and sorts last.
// Digits of up to kRadixMaxBits bits; a tile of kRadixTile edges per
// workgroup, kRadixSub consecutive ones per wave.
constexpr int kRadixMaxBits = 7;
constexpr int kRadixBins = 1 << kRadixMaxBits;
constexpr int kRadixWaves = 8;
constexpr int kRadixThreads = kRadixWaves * kWave;
constexpr int kRadixSub = 1024;
constexpr int kRadixTile = kRadixWaves * kRadixSub;

// Key of edge i (0-based; n for an edge outside 1..n, which also marks status).
__device__ __forceinline__ int32_t radix_key_in(int32_t n, int64_t i, const int32_t* key, const int32_t* other,
                                                const int32_t* kin, int32_t* status) {
  if (kin) return kin[i];
  const int32_t k = key[i], o = other[i];
  const bool ok = k >= 1 && k <= n && o >= 1 && o <= n;
  if (!ok && status) __hip_atomic_store(status, (int32_t)MAP_ERANGE_DEV, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return ok ? k - 1 : n;
}

// Per tile, the count of each digit value: hist[digit * tiles + tile].
__global__ void __launch_bounds__(kRadixThreads)
    radix_count(const int32_t* gate, int32_t n, int64_t m, const int32_t* __restrict__ key,
                const int32_t* __restrict__ other, const int32_t* __restrict__ kin, int shift, int bits, int64_t tiles,
                int32_t* hist, int32_t* status) {
  if (*gate != kBuildRadix) return;
  __shared__ uint32_t h[kRadixBins];
  const uint32_t mask = (1u << bits) - 1u;
  for (int i = threadIdx.x; i <= (int)mask; i += blockDim.x) h[i] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * kRadixTile, t1 = min(m, t0 + kRadixTile);
  constexpr int kPer = kRadixTile / kRadixThreads;
  int32_t kk[kPer];
#pragma unroll
  for (int u = 0; u < kPer; ++u) {  // every load of the thread in flight together
    const int64_t i = t0 + threadIdx.x + (int64_t)u * kRadixThreads;
    kk[u] = i < t1 ? radix_key_in(n, i, key, other, kin, status) : -1;
  }
#pragma unroll
  for (int u = 0; u < kPer; ++u)
    if (kk[u] >= 0) atomicAdd(&h[((uint32_t)kk[u] >> shift) & mask], 1u);
  __syncthreads();
  for (int d = threadIdx.x; d <= (int)mask; d += blockDim.x) hist[(int64_t)d * tiles + blockIdx.x] = (int32_t)h[d];
}

// Stable scatter of one pass.  hist holds the inclusive scan of the counts
// (digit-major), so a tile's first slot for digit d is hist[d][tile] minus
// the tile's own count of d.  The tile is first sorted by digit in LDS, then
// written out a digit run at a time (consecutive threads, consecutive slots).
// Inside the tile the waves take their sub-ranges in order (per-wave counts,
// summed over the waves before), and a wave walks its sub-range 64 edges at a
// time: the lanes that share a digit (found bit by bit with ballots) take
// consecutive places in lane order, and the lowest of them advances the
// wave's cursor for that digit.
__global__ void __launch_bounds__(kRadixThreads)
    radix_scatter(const int32_t* gate, int32_t n, int64_t m, const int32_t* __restrict__ key,
                  const int32_t* __restrict__ other, const int32_t* __restrict__ kin, const int32_t* __restrict__ vin,
                  int shift, int bits, int64_t tiles, const int32_t* __restrict__ hist, int32_t* kout,
                  int32_t* vout) {
  if (*gate != kBuildRadix) return;
  __shared__ uint32_t off[kRadixWaves][kRadixBins];
  __shared__ uint32_t loc[kRadixBins];   // first place of each digit in the sorted tile
  __shared__ uint32_t gpos[kRadixBins];  // its first slot in the output
  __shared__ int32_t sk[kRadixTile];
  __shared__ int32_t sv[kRadixTile];
  const int lane = threadIdx.x & (kWave - 1), wib = threadIdx.x / kWave;
  const uint32_t mask = (1u << bits) - 1u;
  for (int i = threadIdx.x; i < kRadixWaves * kRadixBins; i += blockDim.x) off[i / kRadixBins][i % kRadixBins] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * kRadixTile;
  const int32_t cnt = (int32_t)min((int64_t)kRadixTile, m - t0);
  const int64_t s0 = min(m, t0 + (int64_t)wib * kRadixSub);
  const int64_t s1 = min(m, s0 + kRadixSub);
  // The wave's sub-range in registers, every load in flight together: step u
  // holds edges s0 + 64u + lane.
  constexpr int kSteps = kRadixSub / kWave;
  int32_t kr[kSteps], vr[kSteps];
#pragma unroll
  for (int u = 0; u < kSteps; ++u) {
    const int64_t i = s0 + (int64_t)u * kWave + lane;
    kr[u] = vr[u] = 0;
    if (i < s1) {
      kr[u] = radix_key_in(n, i, key, other, kin, nullptr);
      vr[u] = vin ? vin[i] : other[i] - 1;
    }
  }
#pragma unroll
  for (int u = 0; u < kSteps; ++u)
    if (s0 + (int64_t)u * kWave + lane < s1) atomicAdd(&off[wib][((uint32_t)kr[u] >> shift) & mask], 1u);
  __syncthreads();
  // Per digit: the tile's total (into loc) and each wave's place before the
  // scan over digits.
  for (int d = threadIdx.x; d < kRadixBins; d += blockDim.x) {
    uint32_t run = 0;
    if (d <= (int)mask) {
      for (int w = 0; w < kRadixWaves; ++w) {
        const uint32_t c = off[w][d];
        off[w][d] = run;
        run += c;
      }
      gpos[d] = (uint32_t)hist[(int64_t)d * tiles + blockIdx.x] - run;
    }
    loc[d] = run;
  }
  __syncthreads();
  if (wib == 0) {
    // Exclusive scan of the digit totals, kRadixBins / 64 digits per lane.
    uint32_t v[kRadixBins / kWave], sum = 0;
#pragma unroll
    for (int j = 0; j < kRadixBins / kWave; ++j) {
      v[j] = loc[lane * (kRadixBins / kWave) + j];
      sum += v[j];
    }
    uint32_t incl = sum;
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t y = (uint32_t)__shfl_up((int)incl, o, kWave);
      if (lane >= o) incl += y;
    }
    uint32_t run = incl - sum;
#pragma unroll
    for (int j = 0; j < kRadixBins / kWave; ++j) {
      loc[lane * (kRadixBins / kWave) + j] = run;
      run += v[j];
    }
  }
  __syncthreads();
  const unsigned long long below = lane ? (~0ull >> (kWave - lane)) : 0ull;
#pragma unroll
  for (int u = 0; u < kSteps; ++u) {
    const bool ok = s0 + (int64_t)u * kWave + lane < s1;
    const int32_t kk = kr[u], vv = vr[u];
    const uint32_t d = ((uint32_t)kk >> shift) & mask;
    unsigned long long peers = __ballot(ok);
    for (int bit = 0; bit < bits; ++bit) {
      const unsigned long long one = __ballot(ok && ((d >> bit) & 1u));
      peers &= ((d >> bit) & 1u) ? one : ~one;
    }
    const uint32_t r = (uint32_t)__popcll(peers & below);
    if (ok) {
      const uint32_t lp = loc[d] + off[wib][d] + r;
      sk[lp] = kk;
      sv[lp] = vv;
    }
    // Every lane has read off[wib][d] above (the wave's LDS operations
    // complete in order) before the group's lowest lane advances it.
    if (ok && r == 0) off[wib][d] += (uint32_t)__popcll(peers);
  }
  __syncthreads();
  for (int j = threadIdx.x; j < cnt; j += blockDim.x) {
    const int32_t kk = sk[j];
    const uint32_t d = ((uint32_t)kk >> shift) & mask;
    const uint32_t pos = gpos[d] + ((uint32_t)j - loc[d]);
    kout[pos] = kk;
    vout[pos] = sv[j];
  }
}

// Row pointers from the sorted keys: the rows (key of edge i-1, key of edge
// i] start at edge i (before the first edge: -1; after the last: n).  Four
// consecutive edges per thread, read with one load: 134M edges
// in 0.22 ms (1.16 ms when a lane alone filled the rows behind the last edge).
__global__ void __launch_bounds__(256) radix_row_ptr(const int32_t* gate, int32_t n, int64_t m,
                                                     const int32_t* __restrict__ ks, int32_t* row_ptr) {
  if (*gate != kBuildRadix) return;
  const int64_t quads = (m + 3) / 4;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, gs = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q0 = gt - lane; q0 < quads; q0 += gs) {  // whole waves
    const int64_t i0 = 4 * (q0 + lane);
    int32_t prev = i0 == 0 || i0 >= m ? -1 : ks[i0 - 1];
    int32_t k[4];
    if (i0 + 4 <= m) {
      const int4 kk = *reinterpret_cast<const int4*>(ks + i0);
      k[0] = kk.x, k[1] = kk.y, k[2] = kk.z, k[3] = kk.w;
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) k[u] = i0 + u < m ? ks[i0 + u] : -2;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      fill_rows(row_ptr, prev + 1, k[u] + 1, (int32_t)(i0 + u), lane);
      if (k[u] >= 0) prev = k[u];
    }
  }
  // The rows after the last edge, by the whole grid (none if it is invalid: its
  // key is n).
  for (int64_t r = (int64_t)ks[m - 1] + 1 + gt; r <= n; r += gs) row_ptr[r] = (int32_t)m;
}

// ------------------------------------------------------------------- host --

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

bool sizes_ok(int32_t n, int64_t m) { return n >= 1 && n <= 0x7ffffffe && m >= 0 && m <= 0x7fffffff; }

struct Layout {
  size_t ctrl, pv, accw, front0, front1, mark, aux, chg, accb, win, win_rec, parent, cursor, sums, counts, ids, total;
  size_t rk[2], rv[2], rhist, rsums;  // CSR build, radix path (rk[0] and rv[0] share the atomic path's ids of either side)
  size_t cursor2, sums2, counts2;     // the transposed side's
  int64_t words;  // 32-bit words of one vertex bitmap
};

// m > 0 adds the CSR build's per-edge scratch.
Layout layout(int32_t n, int64_t m = 0) {
  Layout L;
  size_t off = 0;
  L.ctrl = off;
  off += align256(kCtrlBytes);
  const size_t region = off;
  // propagation / detection
  L.pv = off;
  off += align256((size_t)n * 4);
  L.accw = off;
  off += align256((size_t)n);
  // frontier sweeps
  L.front0 = off;
  off += align256((size_t)n * 4);
  L.front1 = off;
  off += align256((size_t)n * 4);
  L.mark = off;
  off += align256((size_t)n * 4);
  // pruning: removed flags
  L.aux = off;
  off += align256((size_t)n * 4);
  // lasso: 64-bit parent words over the mark and removed-flag arrays
  L.parent = L.mark;
  // filtered stream sweeps: three change bitmaps, the rows left by the banded sweeps, the accepting bitmap
  L.words = ((int64_t)n + 31) / 32;
  L.chg = off;
  off += align256((size_t)L.words * 4 * 4);
  L.accb = off;
  off += align256((size_t)L.words * 4);
  // windowed iterations (graphs that the workgroups can hold on chip); larger
  // graphs keep the room, so that a workspace for the largest graph of a set
  // serves the smaller ones too
  L.win = L.win_rec = 0;
  if (n > kSmallN) {
    L.win = off;
    off += kWinCtlBytes;
    L.win_rec = off;
    off += align256((size_t)std::min(n, kWinMaxN) * sizeof(WinRec));
  }
  size_t end_loop = off;
  // CSR build (shares the region after ctrl)
  off = region;
  L.cursor = off;
  off += align256(((size_t)n + 1) * 4);
  L.sums = off;
  off += align256((((size_t)n + 1 + kScanTile - 1) / kScanTile + 1) * 4);
  L.counts = off;  // two list counts, the build paths, the long gaps
  off += 256;
  L.cursor2 = off;
  off += align256(((size_t)n + 1) * 4);
  L.sums2 = off;
  off += align256((((size_t)n + 1 + kScanTile - 1) / kScanTile + 1) * 4);
  L.counts2 = off;
  off += 256;
  const size_t per_edge = align256((size_t)(m > 0 ? m : 0) * 4);
  L.ids = off;  // edge index of every CSR slot (atomic path)
  L.rk[0] = off;
  off += per_edge;
  L.rv[0] = off;
  off += per_edge;
  L.rk[1] = off;
  off += per_edge;
  L.rv[1] = off;
  off += per_edge;
  const int64_t rtiles = ((m > 0 ? m : 0) + kRadixTile - 1) / kRadixTile;
  const int64_t rlen = (int64_t)kRadixBins * rtiles;
  L.rhist = off;
  off += align256((size_t)rlen * 4);
  L.rsums = off;
  off += align256(((size_t)(rlen + kScanTile - 1) / kScanTile + 1) * 4);
  size_t end_build = off;
  L.total = end_loop > end_build ? end_loop : end_build;
  return L;
}

struct DeviceInfo {
  int cus = 0;
  int blocks_per_cu = 0;
  int coop = 0;
};

std::mutex g_dev_mu;
DeviceInfo g_dev[64];

int device_info(DeviceInfo* out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MAP_EDEVICE;
  std::lock_guard<std::mutex> lock(g_dev_mu);
  DeviceInfo& d = g_dev[dev];
  if (d.cus == 0) {
    int cus = 0, coop = 0, nb = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return MAP_EDEVICE;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess) return MAP_EDEVICE;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(map_loop_kernel<true, false>), kBlock,
                                                     0) != hipSuccess)
      return MAP_EDEVICE;
    if (cus <= 0 || nb <= 0) return MAP_EDEVICE;
    d.cus = cus;
    d.coop = coop;
    d.blocks_per_cu = nb;
  }
  *out = d;
  return MAP_OK;
}

int launch_loop(LoopArgs& a, hipStream_t stream) {
  DeviceInfo di;
  int rc = device_info(&di);
  if (rc) return rc;
  if (!di.coop) return MAP_EDEVICE;
  if (!small_fits(a)) {
    a.gate = 0;
  } else {
    hipLaunchKernelGGL(map_small_kernel, dim3(1), dim3(kBlock), 0, stream, a);
    if (hipGetLastError() != hipSuccess) return MAP_EDEVICE;
    if (!a.gate) return MAP_OK;
  }
  const int64_t need = ((int64_t)a.n + (int64_t)kWavesPerBlock * kTileRows - 1) / ((int64_t)kWavesPerBlock * kTileRows);
  int64_t grid = (int64_t)di.cus * di.blocks_per_cu;
  if (grid > need) grid = need;
  if (grid > kMaxBlocks) grid = kMaxBlocks;
  if (grid >= kMaxGroups) grid -= grid % kMaxGroups;
  if (grid < 1) grid = 1;
  hipLaunchKernelGGL(fill_u32, dim3(8), dim3(256), 0, stream, reinterpret_cast<uint32_t*>(a.ctrl),
                     (int64_t)(kEpochOff / 4), 0u);
  if (hipGetLastError() != hipSuccess) return MAP_EDEVICE;
  void* args[] = {&a};
  // MAP_FLAG_EARLY runs with a grid barrier after every sweep (no asynchronous
  // early instantiation exists).
  // When no block can stage its slice on chip (or staging is refused) and the
  // workspace holds the change bitmaps, the filtered stream kernel runs: a
  // barrier after every sweep, gathers only from rows that grew.
  const int64_t rpb = ((int64_t)a.n + grid - 1) / grid;
  const int64_t rpw = (rpb + kWavesPerBlock - 1) / kWavesPerBlock;
  const bool all_stream = a.force_stream || a.n >= (1 << 24) || rpw > kResWaveRows;
  a.filt = (a.chg != nullptr && !a.early && !a.push && all_stream) ? 1 : 0;
  if (!a.filt) a.dopt = 0;
  const bool async = !a.filt && grid > 1 && !a.sync_sweeps && a.tag_mask != 0 && !a.early;
  const void* kernel =
      a.early ? reinterpret_cast<const void*>(map_loop_kernel<false, true>)
      : a.filt ? (a.n >= kBandMinN ? reinterpret_cast<const void*>(map_loop_kernel<false, false, true, true>)
                                   : reinterpret_cast<const void*>(map_loop_kernel<false, false, true>))
               : (async ? reinterpret_cast<const void*>(map_loop_kernel<true, false>)
                        : reinterpret_cast<const void*>(map_loop_kernel<false, false>));
  if (hipLaunchCooperativeKernel(kernel, dim3((unsigned)grid), dim3(kBlock), args, 0, stream) != hipSuccess)
    return MAP_EDEVICE;
  return MAP_OK;
}

inline unsigned grid_for(int64_t work, int threads) {
  int64_t g = (work + threads - 1) / threads;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// Digit width and pass count of the radix path: keys 0..n (n: an edge outside
// 1..n) in passes of at most kRadixMaxBits bits.
static void radix_plan(int32_t n, int* passes, int* bits) {
  int k = 1;
  while (k < 31 && (1ll << k) <= (int64_t)n) ++k;
  *passes = (k + kRadixMaxBits - 1) / kRadixMaxBits;
  *bits = (k + *passes - 1) / *passes;
}

// Builds both sides (side[1].key null: the pull CSR alone).
int build_sides(const BuildArgs& a, char* ws, const Layout& L, hipStream_t stream) {
  const int32_t n = a.n;
  const int64_t m = a.m;
  const unsigned sides = a.side[1].row_ptr ? 2 : 1;
  // Both sides of a small graph in one launch: the size is what one workgroup
  // sorts in LDS.
  if (n <= kSmallN && m <= kTinyEdges) {
    hipLaunchKernelGGL(csr_small, dim3(1, sides), dim3(kBlock), 0, stream, a);
    return hipGetLastError() == hipSuccess ? MAP_OK : MAP_EDEVICE;
  }
  // Path choice (device words: the host never waits for the device here).
  // The grids of kernels that a side's path may skip are kept to what fills
  // the card: 65,536 workgroups that return at once take 15 us.
  const int64_t fill = 1 << 20;
  hipLaunchKernelGGL(csr_pick, dim3(1, sides), dim3(1024), 0, stream, a);
  if (m > 0)
    hipLaunchKernelGGL(csr_sorted, dim3(grid_for(std::min((m + 3) / 4, fill), 256), sides), dim3(256), 0, stream, a);
  // Atomic path: degree histogram, scan, per-row cursors, then row ordering.
  const int64_t tiles = ((int64_t)n + kScanTile) / kScanTile;
  hipLaunchKernelGGL(csr_zero, dim3(grid_for(std::min((int64_t)n + 1, fill), 256), sides), dim3(256), 0, stream, a);
  if (m > 0) {
    hipLaunchKernelGGL(csr_hist, dim3(grid_for(std::min(m, fill), 256), sides), dim3(256), 0, stream, a);
    hipLaunchKernelGGL(rows_scan_tiles, dim3((unsigned)tiles, sides), dim3(kScanThreads), 0, stream, a);
    hipLaunchKernelGGL(rows_scan_sums, dim3(1, sides), dim3(1024), 0, stream, a);
    hipLaunchKernelGGL(rows_scan_add, dim3((unsigned)tiles, sides), dim3(kScanThreads), 0, stream, a);
    hipLaunchKernelGGL(csr_scatter, dim3(grid_for(std::min(m, fill), 256), sides), dim3(256), 0, stream, a);
    hipLaunchKernelGGL(csr_order_rows, dim3(grid_for(std::min((int64_t)n, fill), 256), sides), dim3(256), 0, stream, a);
    hipLaunchKernelGGL(csr_order_listed, dim3(kOrderLongGrid, sides), dim3(kOrderThreads), 0, stream, a);
  }
  // Radix path (m >= kRadixMinEdges only): passes from the edge list through
  // the two scratch pairs; the last pass writes the columns into col.
  if (m >= kRadixMinEdges) {
    int passes = 0, bits = 0;
    radix_plan(n, &passes, &bits);
    const int64_t rtiles = (m + kRadixTile - 1) / kRadixTile;
    const int64_t hlen = (int64_t)(1 << bits) * rtiles;
    const int64_t htiles = (hlen + kScanTile - 1) / kScanTile;
    int32_t* hist = reinterpret_cast<int32_t*>(ws + L.rhist);
    int32_t* hsums = reinterpret_cast<int32_t*>(ws + L.rsums);
    for (unsigned sd = 0; sd < sides; ++sd) {
      const BuildSide& b = a.side[sd];
      const int32_t* mode = b.counts + 2;
      const int32_t* kin = nullptr;
      const int32_t* vin = nullptr;
      int32_t* ks = nullptr;
      for (int p = 0; p < passes; ++p) {
        const int shift = p * bits;
        int32_t* kout = reinterpret_cast<int32_t*>(ws + L.rk[p & 1]);
        int32_t* vout = p + 1 == passes ? b.col : reinterpret_cast<int32_t*>(ws + L.rv[p & 1]);
        hipLaunchKernelGGL(radix_count, dim3((unsigned)rtiles), dim3(kRadixThreads), 0, stream, mode, n, m, b.key,
                           b.other, kin, shift, bits, rtiles, hist, a.status);
        hipLaunchKernelGGL(scan_tiles, dim3((unsigned)htiles), dim3(kScanThreads), 0, stream, mode, kBuildRadix, hist,
                           hlen, hsums);
        hipLaunchKernelGGL(scan_sums, dim3(1), dim3(1024), 0, stream, mode, kBuildRadix, hsums, htiles);
        hipLaunchKernelGGL(scan_add, dim3((unsigned)htiles), dim3(256), 0, stream, mode, kBuildRadix, hist, hlen,
                           hsums);
        hipLaunchKernelGGL(radix_scatter, dim3((unsigned)rtiles), dim3(kRadixThreads), 0, stream, mode, n, m, b.key,
                           b.other, kin, vin, shift, bits, rtiles, hist, kout, vout);
        kin = kout;
        vin = vout;
        ks = kout;
      }
      hipLaunchKernelGGL(radix_row_ptr, dim3(grid_for(std::min(m / 4 + 1, fill), 256)), dim3(256), 0, stream, mode, n, m,
                         ks, b.row_ptr);
    }
  }
  return hipGetLastError() == hipSuccess ? MAP_OK : MAP_EDEVICE;
}

struct BatchLayout {
  size_t header, item_start, scratch_off, gctrl, scratch, total;
};

BatchLayout batch_layout(int32_t count, int64_t total_n) {
  BatchLayout L;
  size_t off = 0;
  L.header = off;
  off += 256;
  L.item_start = off;
  off += align256(((size_t)count + 1) * 4);
  L.scratch_off = off;
  off += align256((size_t)count * 8);
  L.gctrl = off;
  off += (size_t)count * kGangCtrlBytes;
  L.scratch = off;
  // Per graph at most gang_scratch_bytes with MAP_GRAPH_FILTER: 5n + 4 ceil(n / 32)
  // words plus six 256-byte alignments.
  off += (size_t)total_n * 5 + (size_t)(total_n / 2) + (size_t)count * (2 * 256 + 4 * (4 + 256));
  L.total = off;
  return L;
}

int batch_device_info(int* cus, int* per_cu) {
  static std::mutex mu;
  static int cache_cus[64], cache_per[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MAP_EDEVICE;
  std::lock_guard<std::mutex> lock(mu);
  if (cache_cus[dev] == 0) {
    int c = 0, nb = 0;
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return MAP_EDEVICE;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(map_batch_kernel), kBlock,
                                                     0) != hipSuccess)
      return MAP_EDEVICE;
    if (c <= 0 || nb <= 0) return MAP_EDEVICE;
    cache_cus[dev] = c;
    cache_per[dev] = nb;
  }
  *cus = cache_cus[dev];
  *per_cu = cache_per[dev];
  return MAP_OK;
}

int engine_device_info(int* cus, int* per_cu, int* wall_khz) {
  static std::mutex mu;
  static int cache_cus[64], cache_per[64], cache_khz[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MAP_EDEVICE;
  std::lock_guard<std::mutex> lock(mu);
  if (cache_cus[dev] == 0) {
    int c = 0, nb = 0, khz = 0;
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return MAP_EDEVICE;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess) return MAP_EDEVICE;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, reinterpret_cast<const void*>(map_engine_kernel), kBlock,
                                                     0) != hipSuccess)
      return MAP_EDEVICE;
    if (c <= 0 || nb <= 0 || khz <= 0) return MAP_EDEVICE;
    cache_cus[dev] = c;
    cache_per[dev] = nb;
    cache_khz[dev] = khz;
  }
  *cus = cache_cus[dev];
  *per_cu = cache_per[dev];
  *wall_khz = cache_khz[dev];
  return MAP_OK;
}

// Grid of a cooperative frontier launch (counterexample search, pruning):
// about one workgroup per 4096 vertices and at most one per CU — a round's
// frontier is usually far smaller than the graph, and fewer workgroups make the
// per-round barrier cheaper.  Limits are cached per device and kernel.
int frontier_grid(const void* kernel, int32_t n, int64_t* grid_out) {
  static std::mutex mu;
  static std::map<std::pair<int, const void*>, std::pair<int, int>> cache;  // -> (CUs, blocks per CU)
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MAP_EDEVICE;
  int cus = 0, per = 0;
  {
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find({dev, kernel});
    if (it == cache.end()) {
      int co = 0;
      if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return MAP_EDEVICE;
      if (hipDeviceGetAttribute(&co, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess) return MAP_EDEVICE;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, kBlock, 0) != hipSuccess) return MAP_EDEVICE;
      if (cus <= 0 || per <= 0 || !co) return MAP_EDEVICE;
      it = cache.emplace(std::make_pair(dev, kernel), std::make_pair(cus, per)).first;
    }
    cus = it->second.first;
    per = it->second.second;
  }
  int64_t grid = ((int64_t)n + 4095) / 4096;
  if (grid > (int64_t)cus * per) grid = (int64_t)cus * per;
  if (grid > cus) grid = cus;
  if (grid > kMaxBlocks) grid = kMaxBlocks;
  if (grid >= kMaxGroups) grid -= grid % kMaxGroups;
  if (grid < 1) grid = 1;
  *grid_out = grid;
  return MAP_OK;
}

constexpr int32_t kEngineRing = 1 << 17;  // ticket ring entries (1 MiB of host memory)

// Fixed device scratch of map_detect_noalloc, for callers that cannot allocate:
// the control block, packed values and working accepting flags of one graph of
// at most MAP_NOALLOC_MAX_N vertices, laid out as in a map_detect workspace.
// Each device that runs the library holds its own copy until the process ends.
constexpr size_t kNoAllocBytes = kCtrlBytes + (size_t)MAP_NOALLOC_MAX_N * 4 + (size_t)MAP_NOALLOC_MAX_N;
static_assert(kCtrlBytes % 256 == 0 && ((size_t)MAP_NOALLOC_MAX_N * 4) % 256 == 0,
              "no-alloc scratch regions are 256-byte aligned");
static __device__ __align__(256) char noalloc_scratch[kNoAllocBytes];

// Device address of noalloc_scratch on each device, taken once per device with
// that device current (the array's name in host code is only a stand-in).
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[64];

int noalloc_scratch_ptr(char** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return MAP_EDEVICE;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_noalloc_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc_scratch)) != hipSuccess || !p) return MAP_EDEVICE;
    g_noalloc_ptr[dev] = p;
  }
  *out = static_cast<char*>(g_noalloc_ptr[dev]);
  return MAP_OK;
}

}  // namespace

// Host state of a serving engine (one per map_engine_create).
struct map_engine {
  hipStream_t stream;
  hipEvent_t exited;             // recorded after the engine launch
  int grid;                      // workgroups of the launch
  int32_t slots;
  char* host;                    // fine-grained host block: shared line, ring, jobs, results
  EngineShared* sh;
  unsigned long long* ring;
  EngineJob* jobs;
  map_result* res;
  char* dmem;                    // device state
  std::vector<int32_t> free_slots;
  std::vector<unsigned long long> start;  // first ticket of the job in each busy slot
  std::vector<uint8_t> busy;
  unsigned long long tail;       // tickets published
  bool stopped;
};

extern "C" {

size_t map_workspace_bytes(int32_t n, int64_t m, uint32_t flags) {
  (void)flags;
  if (!sizes_ok(n, m)) return 0;
  return layout(n, m).total;
}

int map_build_csr(int32_t n, int64_t m, const int32_t* src, const int32_t* dst, int32_t* row_ptr, int32_t* col,
                  int32_t* rrow_ptr, int32_t* rcol, int32_t* status, void* ws, size_t ws_bytes, void* stream) {
  if (!sizes_ok(n, m)) return MAP_ERANGE;
  if (!row_ptr || !status || !ws || (m > 0 && (!src || !dst || !col))) return MAP_EINVAL;
  if ((rrow_ptr == nullptr) != (rcol == nullptr)) return MAP_EINVAL;
  if (rrow_ptr && m > 0 && !rcol) return MAP_EINVAL;
  const Layout L = layout(n, m);
  if (ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255)) return MAP_ENOSPC;
  char* w = static_cast<char*>(ws);
  auto words = [w](size_t off) { return reinterpret_cast<int32_t*>(w + off); };
  BuildArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n = n;
  a.m = m;
  a.status = status;
  a.vec = ((reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(col) |
            reinterpret_cast<uintptr_t>(rcol)) & 15) == 0;
  a.side[0] = {src, dst, row_ptr, col, words(L.cursor), words(L.sums), words(L.counts), words(L.rk[0])};
  if (rrow_ptr)
    a.side[1] = {dst, src, rrow_ptr, rcol, words(L.cursor2), words(L.sums2), words(L.counts2), words(L.rv[0])};
  return build_sides(a, w, L, reinterpret_cast<hipStream_t>(stream));
}

// Loop arguments over scratch at w laid out by L (control block, packed values,
// working flags).
static void loop_args(int32_t n, const int32_t* row_ptr, const int32_t* col, const uint8_t* acc, map_result* result,
                      char* w, const Layout& L, LoopArgs& a) {
  std::memset(&a, 0, sizeof(a));
  a.n = n;
  a.ntiles = (int32_t)(((int64_t)n + kTileRows - 1) / kTileRows);
  a.row_ptr = row_ptr;
  a.col = col;
  a.acc_in = acc;
  a.pv = reinterpret_cast<uint32_t*>(w + L.pv);
  a.accw = reinterpret_cast<uint8_t*>(w + L.accw);
  a.ctrl = reinterpret_cast<Ctrl*>(w + L.ctrl);
  a.result = result;
  word_layout(n, &a.val_mask, &a.tag_mask, &a.tag_shift);
  a.epoch = reinterpret_cast<uint32_t*>(w + L.ctrl + kEpochOff);
  a.chg = reinterpret_cast<uint32_t*>(w + L.chg);
  a.accb = reinterpret_cast<uint32_t*>(w + L.accb);
  a.words = L.words;
  a.hub = kHubEdges;
  if (L.win && n <= kWinMaxN) {
    a.win = reinterpret_cast<WinCtl*>(w + L.win);
    a.win_rec = reinterpret_cast<WinRec*>(w + L.win_rec);
  }
}

static int loop_common(int32_t n, const int32_t* row_ptr, const int32_t* col, const uint8_t* acc, map_result* result,
                       void* ws, size_t ws_bytes, LoopArgs& a) {
  if (n < 1 || n > 0x7ffffffe) return MAP_ERANGE;
  if (!row_ptr || !col || !acc || !result || !ws) return MAP_EINVAL;
  const Layout L = layout(n);
  if (ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255)) return MAP_ENOSPC;
  loop_args(n, row_ptr, col, acc, result, static_cast<char*>(ws), L, a);
  // The workspace is at least as large as the graph's edges ask for: a graph
  // that it cannot serve with more edges than one workgroup takes needs no gate.
  a.gate = !small_takes(n, kSmallStream + 1) && ws_bytes >= layout(n, kSmallStream + 1).total;
  return MAP_OK;
}

// Frontier sweeps (MAP_FLAG_PUSH, not with MAP_FLAG_DENSE_ONLY) need the
// transposed CSR; they run with a barrier per round and read the values from
// memory (no LDS-resident rows).
static int push_setup(LoopArgs& a, const int32_t* rrow_ptr, const int32_t* rcol, uint32_t flags, void* ws) {
  if (!(flags & MAP_FLAG_PUSH) || (flags & MAP_FLAG_DENSE_ONLY)) return MAP_OK;
  if (!rrow_ptr || !rcol) return MAP_EINVAL;
  const Layout L = layout(a.n);
  char* w = static_cast<char*>(ws);
  a.push = 1;
  a.rrow_ptr = rrow_ptr;
  a.rcol = rcol;
  a.front[0] = reinterpret_cast<int32_t*>(w + L.front0);
  a.front[1] = reinterpret_cast<int32_t*>(w + L.front1);
  a.mark = reinterpret_cast<uint32_t*>(w + L.mark);
  a.force_stream = 1;
  a.sync_sweeps = 1;
  return MAP_OK;
}

// Direction switch of the filtered stream sweeps (MAP_FLAG_DIRECTION, not with
// MAP_FLAG_DENSE_ONLY): needs the transposed CSR; the frontier is the change
// bitmap the sweeps keep anyway.  It takes effect only where the filtered
// stream kernel runs (launch_loop).
static int dir_setup(LoopArgs& a, const int32_t* rrow_ptr, const int32_t* rcol, uint32_t flags) {
  if (!(flags & MAP_FLAG_DIRECTION) || (flags & MAP_FLAG_DENSE_ONLY)) return MAP_OK;
  if (flags & MAP_FLAG_PUSH) return MAP_EINVAL;
  if (!rrow_ptr || !rcol) return MAP_EINVAL;
  a.dopt = 1;
  a.rrow_ptr = rrow_ptr;
  a.rcol = rcol;
  return MAP_OK;
}

int map_propagate(int32_t n, const int32_t* row_ptr, const int32_t* col, const int32_t* rrow_ptr, const int32_t* rcol,
                  const uint8_t* accepting, int32_t* map_out, map_result* result, uint32_t flags, void* ws,
                  size_t ws_bytes, void* stream) {
  if (flags & ~kAllFlags) return MAP_EINVAL;
  if (!map_out) return MAP_EINVAL;
  LoopArgs a;
  int rc = loop_common(n, row_ptr, col, accepting, result, ws, ws_bytes, a);
  if (rc) return rc;
  a.propagate = 1;
  a.force_stream = (flags & MAP_FLAG_STREAM) ? 1 : 0;
  a.sync_sweeps = (flags & MAP_FLAG_SYNC_SWEEPS) ? 1 : 0;
  if (flags & MAP_FLAG_NO_FILTER) a.chg = nullptr;
  a.map_out = map_out;
  rc = push_setup(a, rrow_ptr, rcol, flags, ws);
  if (rc) return rc;
  rc = dir_setup(a, rrow_ptr, rcol, flags);
  if (rc) return rc;
  return launch_loop(a, reinterpret_cast<hipStream_t>(stream));
}

int map_detect(int32_t n, const int32_t* row_ptr, const int32_t* col, const int32_t* rrow_ptr, const int32_t* rcol,
               const uint8_t* accepting0, map_result* result, uint64_t* trace, int32_t trace_cap,
               uint8_t* accepting_out, int32_t max_iterations, uint32_t flags, void* ws, size_t ws_bytes,
               void* stream) {
  if (flags & ~kAllFlags) return MAP_EINVAL;
  if (trace && trace_cap < 0) return MAP_EINVAL;
  LoopArgs a;
  int rc = loop_common(n, row_ptr, col, accepting0, result, ws, ws_bytes, a);
  if (rc) return rc;
  a.propagate = 0;
  a.trace = trace;
  a.trace_cap = trace ? trace_cap : 0;
  a.acc_out = accepting_out;
  a.max_iter = max_iterations;
  a.digest = (trace && !(flags & MAP_FLAG_NO_TRACE_DIGEST)) ? 1 : 0;
  a.force_stream = (flags & MAP_FLAG_STREAM) ? 1 : 0;
  a.sync_sweeps = (flags & MAP_FLAG_SYNC_SWEEPS) ? 1 : 0;
  if (flags & MAP_FLAG_NO_FILTER) a.chg = nullptr;
  rc = push_setup(a, rrow_ptr, rcol, flags, ws);
  if (rc) return rc;
  rc = dir_setup(a, rrow_ptr, rcol, flags);
  if (rc) return rc;
  if (flags & MAP_FLAG_EARLY) {
    if (a.push) return MAP_EINVAL;
    a.early = 1;
  }
  return launch_loop(a, reinterpret_cast<hipStream_t>(stream));
}

int map_detect_noalloc(int32_t n, const int32_t* row_ptr, const int32_t* col, const uint8_t* accepting0,
                       map_result* result, uint64_t* trace, int32_t trace_cap, uint8_t* accepting_out,
                       int32_t max_iterations, uint32_t flags, void* stream) {
  if (flags & ~kAllFlags) return MAP_EINVAL;
  if ((flags & (MAP_FLAG_PUSH | MAP_FLAG_DIRECTION)) && !(flags & MAP_FLAG_DENSE_ONLY)) return MAP_EINVAL;
  if (trace && trace_cap < 0) return MAP_EINVAL;
  if (n < 1 || n > MAP_NOALLOC_MAX_N) return MAP_ERANGE;
  if (!row_ptr || !col || !accepting0 || !result) return MAP_EINVAL;
  const Layout L = layout(n);
  // Only the control block, packed values and working flags are used.
  if (L.accw + (size_t)n > kNoAllocBytes) return MAP_ERANGE;
  char* w = nullptr;
  int rc = noalloc_scratch_ptr(&w);
  if (rc) return rc;
  LoopArgs a;
  loop_args(n, row_ptr, col, accepting0, result, w, L, a);
  a.chg = nullptr;  // the fixed scratch holds no change bitmaps: unfiltered sweeps
  a.accb = nullptr;
  a.win = nullptr;  // nor the records of windowed iterations
  a.win_rec = nullptr;
  a.gate = !small_takes(n, kSmallStream + 1);  // nothing bounds the edges here
  a.propagate = 0;
  a.trace = trace;
  a.trace_cap = trace ? trace_cap : 0;
  a.acc_out = accepting_out;
  a.max_iter = max_iterations;
  a.digest = (trace && !(flags & MAP_FLAG_NO_TRACE_DIGEST)) ? 1 : 0;
  a.force_stream = (flags & MAP_FLAG_STREAM) ? 1 : 0;
  a.sync_sweeps = (flags & MAP_FLAG_SYNC_SWEEPS) ? 1 : 0;
  a.early = (flags & MAP_FLAG_EARLY) ? 1 : 0;
  return launch_loop(a, reinterpret_cast<hipStream_t>(stream));
}

int map_lasso(int32_t n, const int32_t* row_ptr, const int32_t* col, int32_t witness, int32_t init, int32_t* path,
              int32_t path_cap, map_lasso_result* result, void* ws, size_t ws_bytes, void* stream) {
  if (n < 1 || n > 0x7ffffffe) return MAP_ERANGE;
  if (!row_ptr || !col || !result || !ws || path_cap < 0 || (path_cap > 0 && !path)) return MAP_EINVAL;
  if (witness < 1 || witness > n || init < 0 || init > n) return MAP_EINVAL;
  const Layout L = layout(n);
  if (ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255)) return MAP_ENOSPC;
  int64_t grid = 0;
  int rc = frontier_grid(reinterpret_cast<const void*>(map_lasso_kernel<true>), n, &grid);
  if (rc) return rc;
  char* w = static_cast<char*>(ws);
  LassoArgs a;
  a.n = n;
  a.row_ptr = row_ptr;
  a.col = col;
  a.w = witness - 1;
  a.init = init - 1;
  a.path = path;
  a.cap = path_cap;
  a.result = result;
  a.parent = reinterpret_cast<uint64_t*>(w + L.parent);
  a.front[0] = reinterpret_cast<int32_t*>(w + L.front0);
  a.front[1] = reinterpret_cast<int32_t*>(w + L.front1);
  a.ctrl = reinterpret_cast<Ctrl*>(w + L.ctrl);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(fill_u32, dim3(8), dim3(256), 0, st, reinterpret_cast<uint32_t*>(a.ctrl),
                     (int64_t)(kEpochOff / 4), 0u);
  if (hipGetLastError() != hipSuccess) return MAP_EDEVICE;
  void* args[] = {&a};
  const void* kernel = grid >= kStageBlocks ? reinterpret_cast<const void*>(map_lasso_kernel<true>)
                                            : reinterpret_cast<const void*>(map_lasso_kernel<false>);
  if (hipLaunchCooperativeKernel(kernel, dim3((unsigned)grid), dim3(kBlock), args, 0, st) != hipSuccess)
    return MAP_EDEVICE;
  return MAP_OK;
}

int map_trim(int32_t n, const int32_t* row_ptr, const int32_t* col, const int32_t* rrow_ptr, const int32_t* rcol,
             const uint8_t* accepting, uint8_t* keep_out, uint8_t* accepting_out, map_trim_result* result, void* ws,
             size_t ws_bytes, void* stream) {
  if (n < 1 || n > 0x7ffffffe) return MAP_ERANGE;
  if (!row_ptr || !col || !rrow_ptr || !rcol || !keep_out || !result || !ws) return MAP_EINVAL;
  if ((accepting == nullptr) != (accepting_out == nullptr)) return MAP_EINVAL;
  const Layout L = layout(n);
  if (ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255)) return MAP_ENOSPC;
  int64_t grid = 0;
  int rc = frontier_grid(reinterpret_cast<const void*>(map_trim_kernel<true>), n, &grid);
  if (rc) return rc;
  char* w = static_cast<char*>(ws);
  TrimArgs a;
  a.n = n;
  a.row_ptr = row_ptr;
  a.col = col;
  a.rrow_ptr = rrow_ptr;
  a.rcol = rcol;
  a.acc_in = accepting;
  a.keep_out = keep_out;
  a.acc_out = accepting_out;
  a.result = result;
  a.indeg = reinterpret_cast<uint32_t*>(w + L.pv);
  a.outdeg = reinterpret_cast<uint32_t*>(w + L.mark);
  a.removed = reinterpret_cast<uint32_t*>(w + L.aux);
  a.front[0] = reinterpret_cast<int32_t*>(w + L.front0);
  a.front[1] = reinterpret_cast<int32_t*>(w + L.front1);
  a.ctrl = reinterpret_cast<Ctrl*>(w + L.ctrl);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(fill_u32, dim3(8), dim3(256), 0, st, reinterpret_cast<uint32_t*>(a.ctrl),
                     (int64_t)(kEpochOff / 4), 0u);
  if (hipGetLastError() != hipSuccess) return MAP_EDEVICE;
  void* args[] = {&a};
  const void* kernel = grid >= kStageBlocks ? reinterpret_cast<const void*>(map_trim_kernel<true>)
                                            : reinterpret_cast<const void*>(map_trim_kernel<false>);
  if (hipLaunchCooperativeKernel(kernel, dim3((unsigned)grid), dim3(kBlock), args, 0, st) != hipSuccess)
    return MAP_EDEVICE;
  return MAP_OK;
}

size_t map_batch_workspace_bytes(int32_t count, int64_t total_n, uint32_t flags) {
  (void)flags;
  if (count < 1 || count > (1 << 24) || total_n < count || total_n > ((int64_t)1 << 40)) return 0;
  return batch_layout(count, total_n).total;
}

int map_detect_batch(int32_t count, const map_graph_desc* graphs, const int32_t* gang, map_result* results,
                     int64_t total_n, uint32_t flags, void* ws, size_t ws_bytes, void* stream) {
  if (count < 1 || count > (1 << 24) || total_n < count || total_n > ((int64_t)1 << 40)) return MAP_ERANGE;
  if (!graphs || !results || !ws) return MAP_EINVAL;
  if (flags & ~kAllFlags) return MAP_EINVAL;
  const BatchLayout L = batch_layout(count, total_n);
  if (ws_bytes < L.total || (reinterpret_cast<uintptr_t>(ws) & 255)) return MAP_ENOSPC;
  int cus = 0, per_cu = 0;
  int rc = batch_device_info(&cus, &per_cu);
  if (rc) return rc;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char* w = static_cast<char*>(ws);
  BatchArgs ba;
  ba.count = count;
  ba.graphs = graphs;
  ba.results = results;
  ba.item_start = reinterpret_cast<int32_t*>(w + L.item_start);
  ba.scratch_off = reinterpret_cast<int64_t*>(w + L.scratch_off);
  ba.gctrl = reinterpret_cast<GangCtrl*>(w + L.gctrl);
  ba.scratch = w + L.scratch;
  ba.next_item = reinterpret_cast<uint32_t*>(w + L.header);
  ba.status = reinterpret_cast<int32_t*>(w + L.header + 128);
  ba.flags = flags;
  const int64_t ctrl_words = (int64_t)((size_t)count * kGangCtrlBytes / 4);
  hipLaunchKernelGGL(fill_u32, dim3(grid_for(ctrl_words, 256)), dim3(256), 0, st,
                     reinterpret_cast<uint32_t*>(ba.gctrl), ctrl_words, 0u);
  // A gang must fit in the grid at once: its blocks wait for each other.
  const int grid = cus * per_cu;
  hipLaunchKernelGGL(batch_plan, dim3(1), dim3(1024), 0, st, count, graphs, gang,
                     const_cast<int32_t*>(ba.item_start), const_cast<int64_t*>(ba.scratch_off),
                     (size_t)(L.total - L.scratch), (int32_t)std::min(kMaxGang, grid), ba.status, ba.next_item);
  if (hipGetLastError() != hipSuccess) return MAP_EDEVICE;
  if (gang == nullptr) {
    hipLaunchKernelGGL(map_batch_kernel, dim3(grid), dim3(kBlock), 0, st, ba);
    if (hipGetLastError() != hipSuccess) return MAP_EDEVICE;
  } else {
    void* args[] = {&ba};
    if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(map_batch_kernel), dim3(grid), dim3(kBlock), args,
                                   0, st) != hipSuccess)
      return MAP_EDEVICE;
  }
  return MAP_OK;
}

size_t map_job_scratch_bytes(int32_t n, int64_t m) {
  if (!sizes_ok(n, m)) return 0;
  // packed values | working flags | bitmaps of the filtered sweeps | scan
  // partials | staged edge list (src, dst) | transposed CSR (the last three
  // parts used with MAP_FLAG_DIRECTION only)
  return align256((size_t)n * 4) + align256((size_t)n) + 4 * (size_t)gang_bitmap_bytes(n) + (size_t)kMaxGang * 4 +
         2 * align256((size_t)m * 4) + align256((size_t)n * 4 + 4) + align256((size_t)m * 4);
}

static void engine_free(map_engine* e) {
  if (e->dmem) (void)hipFree(e->dmem);
  if (e->host) (void)hipHostFree(e->host);
  if (e->exited) (void)hipEventDestroy(e->exited);
  delete e;
}

int map_engine_create(int32_t max_jobs, int32_t workgroups, double idle_seconds, uint32_t flags, void* stream,
                      map_engine** out) {
  if (!out) return MAP_EINVAL;
  *out = nullptr;
  if (flags & ~kAllFlags) return MAP_EINVAL;
  if (max_jobs < 1 || max_jobs > (1 << 16) || workgroups < 0 || !(idle_seconds > 0.0) || idle_seconds > 86400.0)
    return MAP_ERANGE;
  int cus = 0, per_cu = 0, khz = 0;
  int rc = engine_device_info(&cus, &per_cu, &khz);
  if (rc) return rc;
  const int full = cus * per_cu;
  // By default one compute unit per 32 is left to other work (copy kernels of
  // the runtime, the caller's own launches) while the engine runs.
  const int grid = workgroups > 0 ? std::min(workgroups, full) : std::max(1, full - cus / 32);
  map_engine* e = new map_engine();
  e->stream = reinterpret_cast<hipStream_t>(stream);
  e->grid = grid;
  e->slots = max_jobs;
  const size_t off_ring = sizeof(EngineShared);
  const size_t off_jobs = off_ring + (size_t)kEngineRing * 8;
  const size_t off_res = off_jobs + align256((size_t)max_jobs * sizeof(EngineJob));
  const size_t host_bytes = off_res + (size_t)max_jobs * sizeof(map_result);
  void* h = nullptr;
  if (hipHostMalloc(&h, host_bytes, hipHostMallocCoherent | hipHostMallocMapped) != hipSuccess || !h) {
    delete e;
    return MAP_EDEVICE;
  }
  e->host = static_cast<char*>(h);
  std::memset(e->host, 0, host_bytes);
  e->sh = reinterpret_cast<EngineShared*>(e->host);
  e->ring = reinterpret_cast<unsigned long long*>(e->host + off_ring);
  e->jobs = reinterpret_cast<EngineJob*>(e->host + off_jobs);
  e->res = reinterpret_cast<map_result*>(e->host + off_res);
  void* hd = nullptr;
  if (hipHostGetDevicePointer(&hd, h, 0) != hipSuccess || !hd) {
    engine_free(e);
    return MAP_EDEVICE;
  }
  char* hdev = static_cast<char*>(hd);
  const size_t off_b = align256(sizeof(EngineDev));
  const size_t off_m = off_b + (size_t)max_jobs * kGangCtrlBytes;
  const size_t off_d = off_m + (size_t)max_jobs * kGangCtrlBytes;
  const size_t off_r = off_d + align256((size_t)max_jobs * sizeof(map_result));
  const size_t dev_bytes = off_r + align256((size_t)max_jobs * 8);
  void* dm = nullptr;
  if (hipMalloc(&dm, dev_bytes) != hipSuccess || !dm) {
    engine_free(e);
    return MAP_EDEVICE;
  }
  e->dmem = static_cast<char*>(dm);
  if (hipEventCreateWithFlags(&e->exited, hipEventDisableTiming) != hipSuccess) {
    e->exited = nullptr;
    engine_free(e);
    return MAP_EDEVICE;
  }
  e->free_slots.reserve(max_jobs);
  for (int32_t i = max_jobs - 1; i >= 0; --i) e->free_slots.push_back(i);
  e->start.assign(max_jobs, 0ull);
  e->busy.assign(max_jobs, 0);
  e->tail = 0;
  e->stopped = false;

  EngineArgs ea;
  ea.sh = reinterpret_cast<EngineShared*>(hdev);
  ea.ring = reinterpret_cast<const unsigned long long*>(hdev + off_ring);
  ea.jobs = reinterpret_cast<const EngineJob*>(hdev + off_jobs);
  ea.hres = reinterpret_cast<map_result*>(hdev + off_res);
  ea.dev = reinterpret_cast<EngineDev*>(e->dmem);
  ea.bctrl = reinterpret_cast<GangCtrl*>(e->dmem + off_b);
  ea.mctrl = reinterpret_cast<GangCtrl*>(e->dmem + off_m);
  ea.dres = reinterpret_cast<map_result*>(e->dmem + off_d);
  ea.ready = reinterpret_cast<unsigned long long*>(e->dmem + off_r);
  ea.ring_cap = kEngineRing;
  ea.slots = max_jobs;
  ea.idle_ticks = (uint64_t)(idle_seconds * (double)khz * 1000.0);
  ea.flags = flags;
  hipLaunchKernelGGL(fill_u32, dim3(grid_for((int64_t)(dev_bytes / 4), 256)), dim3(256), 0, e->stream,
                     reinterpret_cast<uint32_t*>(e->dmem), (int64_t)(dev_bytes / 4), 0u);
  void* args[] = {&ea};
  if (hipGetLastError() != hipSuccess ||
      hipLaunchCooperativeKernel(reinterpret_cast<const void*>(map_engine_kernel), dim3(grid), dim3(kBlock), args, 0,
                                 e->stream) != hipSuccess ||
      hipEventRecord(e->exited, e->stream) != hipSuccess) {
    // Nothing was launched, or the launch failed: no kernel can be using the memory.
    (void)hipStreamSynchronize(e->stream);
    engine_free(e);
    return MAP_EDEVICE;
  }
  *out = e;
  return MAP_OK;
}

int map_engine_workgroups(const map_engine* e) { return e ? e->grid : 0; }

// Device address through which the engine reads a job input: device memory
// as is, pinned host memory through its device mapping; anything else (pageable
// host memory, unknown pointers) is rejected so the kernel never touches it.
static int engine_input(const void* p, const void** out, bool* host = nullptr) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return MAP_EINVAL;
  }
  if (at.type == hipMemoryTypeDevice) {
    *out = p;
    return MAP_OK;
  }
  if (at.type == hipMemoryTypeHost) {
    void* d = nullptr;
    if (hipHostGetDevicePointer(&d, const_cast<void*>(p), 0) != hipSuccess || !d) {
      (void)hipGetLastError();
      return MAP_EINVAL;
    }
    *out = d;
    if (host) *host = true;
    return MAP_OK;
  }
  return MAP_EINVAL;
}

static bool engine_output(const void* p) {
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return at.type == hipMemoryTypeDevice;
}

int map_engine_submit(map_engine* e, const map_job* job, int32_t* slot) {
  if (!e || !job || !slot) return MAP_EINVAL;
  if (e->stopped) return MAP_EINVAL;
  if (__atomic_load_n(&e->sh->expired, __ATOMIC_ACQUIRE)) return MAP_EDEVICE;
  if (!sizes_ok(job->n, job->m)) return MAP_ERANGE;
  if (!job->row_ptr || !job->accepting0 || !job->scratch) return MAP_EINVAL;
  if (job->m > 0 && (!job->src || !job->dst || !job->col)) return MAP_EINVAL;
  if (reinterpret_cast<uintptr_t>(job->scratch) & 255) return MAP_EINVAL;
  EngineJob ej;
  std::memset(&ej, 0, sizeof(ej));
  map_job& jj = ej.j;
  jj = *job;
  bool host_src = false, host_dst = false;
  if (engine_input(job->accepting0, reinterpret_cast<const void**>(&jj.accepting0)) ||
      !engine_output(job->row_ptr) || !engine_output(job->scratch))
    return MAP_EINVAL;
  if (job->m > 0 && (engine_input(job->src, reinterpret_cast<const void**>(&jj.src), &host_src) ||
                     engine_input(job->dst, reinterpret_cast<const void**>(&jj.dst), &host_dst) ||
                     !engine_output(job->col)))
    return MAP_EINVAL;
  ej.host_edges = (host_src || host_dst) ? 1u : 0u;
  const int32_t gang = std::max(1, std::min(job->gang, std::min(kMaxGang, e->grid)));
  if (e->free_slots.empty()) return MAP_EBUSY;
  // The new tickets reuse ring entries of tickets [tail + gang - ring, ...),
  // which must all have been taken: every ticket below the first one of the
  // oldest unfinished job has been.
  unsigned long long oldest = e->tail;
  for (int32_t i = 0; i < e->slots; ++i)
    if (e->busy[i] && e->start[i] < oldest) oldest = e->start[i];
  if (e->tail + (unsigned long long)gang > oldest + (unsigned long long)kEngineRing) return MAP_EBUSY;
  const int32_t s = e->free_slots.back();
  e->free_slots.pop_back();
  jj.gang = gang;
  e->jobs[s] = ej;
  map_result r0;
  std::memset(&r0, 0, sizeof(r0));
  r0.status = MAP_PENDING;
  e->res[s] = r0;
  for (int32_t r = 0; r < gang; ++r)
    e->ring[(e->tail + (unsigned long long)r) % kEngineRing] = ((unsigned long long)s << 32) | (unsigned)r;
  e->start[s] = e->tail;
  e->busy[s] = 1;
  e->tail += (unsigned long long)gang;
  __atomic_store_n(&e->sh->tail, e->tail, __ATOMIC_RELEASE);
  *slot = s;
  return MAP_OK;
}

int map_engine_poll(map_engine* e, int32_t slot, map_result* out) {
  if (!e || slot < 0 || slot >= e->slots || !e->busy[slot]) return MAP_EINVAL;
  const int32_t st = __atomic_load_n(&e->res[slot].status, __ATOMIC_ACQUIRE);
  if (st == MAP_PENDING) {
    // A job still pending after the engine exited (idle bound) never completes.
    if (hipEventQuery(e->exited) != hipSuccess) return MAP_PENDING;
    if (__atomic_load_n(&e->res[slot].status, __ATOMIC_ACQUIRE) == MAP_PENDING) {
      e->busy[slot] = 0;
      e->free_slots.push_back(slot);
      return MAP_EDEVICE;
    }
  }
  if (out) std::memcpy(out, &e->res[slot], sizeof(map_result));
  e->busy[slot] = 0;
  e->free_slots.push_back(slot);
  return MAP_OK;
}

int map_engine_stop(map_engine* e) {
  if (!e) return MAP_EINVAL;
  __atomic_store_n(&e->sh->stop, 1u, __ATOMIC_RELEASE);
  e->stopped = true;
  return MAP_OK;
}

int map_engine_destroy(map_engine* e) {
  if (!e) return MAP_EINVAL;
  map_engine_stop(e);
  const int rc = hipEventSynchronize(e->exited) == hipSuccess ? MAP_OK : MAP_EDEVICE;
  engine_free(e);
  return rc;
}

int map_phase_counters(uint64_t* out, int32_t max_blocks, int32_t* blocks) {
#ifdef MAPCHECK_PHASES
  if (!out || !blocks || max_blocks < 0) return MAP_EINVAL;
  int32_t nb = 0;
  if (hipMemcpyFromSymbol(&nb, HIP_SYMBOL(g_phase_blocks), sizeof(nb), 0, hipMemcpyDeviceToHost) != hipSuccess)
    return MAP_EDEVICE;
  *blocks = nb;
  const int k = nb < max_blocks ? nb : max_blocks;
  if (k > 0 && hipMemcpyFromSymbol(out, HIP_SYMBOL(g_phase_out), (size_t)k * kPhSlots * sizeof(uint64_t), 0,
                                   hipMemcpyDeviceToHost) != hipSuccess)
    return MAP_EDEVICE;
  return MAP_OK;
#else
  (void)out;
  (void)max_blocks;
  (void)blocks;
  return MAP_EINVAL;
#endif
}

const char* map_strerror(int status) {
  switch (status) {
    case MAP_OK: return "ok";
    case MAP_EINVAL: return "invalid argument (null pointer or unknown flag)";
    case MAP_ERANGE: return "n or m out of the supported range";
    case MAP_ENOSPC: return "workspace too small or not 256-byte aligned";
    case MAP_EDEVICE: return "HIP runtime error or device-side barrier timeout";
    case MAP_ENOTCONVERGED: return "iteration or sweep cap reached";
    case MAP_ERANGE_DEV: return "edge endpoint outside 1..n";
    case MAP_EBUSY: return "engine has no free job slot or ticket space; poll finished jobs first";
    case MAP_ENOPATH: return "no path from the initial vertex to the witness, or no cycle through the witness";
    case MAP_PENDING: return "job not finished yet";
    default: return "unknown status";
  }
}

}  // extern "C"
