// Persistent recurrent kernels: interface used by the layer drivers.
#pragma once

#include "common.hpp"

// Barrier of the steps: every thread's LDS accesses are done, while its global
// stores and prefetches stay in flight (the fence of __syncthreads would wait
// for them at each step).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}


// ---------------------------------------------------------------------------
// Exchange words: agent-scope relaxed 8-byte atomics (coherent per location
// over the whole GPU).  A member whose group sits on one XCD publishes with
// plain stores instead: they stay in that XCD's L2, where the readers'
// agent-scope loads (which pass the CU's own cache by) find them, while an
// agent-scope store goes through to memory.  Every word carries its tag, so a
// reader can only be late, never wrong.  Measured at H = 512 per step of the
// backward: 2.26 -> 2.01 us (8 rows per workgroup), 3.34 -> 2.83 (16), 5.4 ->
// 4.7 (32); loads with weaker scopes or non-temporal accesses were slower.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t ll_load(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ll_store64(uint64_t* p, uint64_t v, bool local) {
  if (local)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  else
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

#define PERSIST_SPIN_LIMIT (1u << 18)
// Polls word j at base[off[j]] until all carry `want` (one already holding
// it is not read again); gives up after PERSIST_SPIN_LIMIT polls, or at once when
// any wait anywhere has given up, so every wave ends.
template <int N>
__device__ __forceinline__ void poll_tagged(uint64_t (&wv)[N], const uint64_t* base, const uint32_t (&off)[N],
                                            uint32_t want, int* status) {
  for (unsigned it = 0;; ++it) {
    bool bad = false;
#pragma unroll
    for (int j = 0; j < N; ++j) bad |= (uint32_t)(wv[j] >> 32) != want;
    if (!bad) break;
    if (it > PERSIST_SPIN_LIMIT ||
        ((it & 63) == 63 && __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
      __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      break;
    }
    __builtin_amdgcn_s_sleep(1);
#pragma unroll
    for (int j = 0; j < N; ++j)
      if ((uint32_t)(wv[j] >> 32) != want) wv[j] = ll_load(base + off[j]);
  }
}

// ---------------------------------------------------------------------------
// Groups.  The members of a group wait for each other at every step, so they
// may start only when all of them run, and a launch cannot count on that:
// launches of other streams, graphs or processes may hold the CUs that some of
// its workgroups need, and need the CUs that the others hold.  So the members
// first meet at the group's word.  When the last one has arrived the group runs
// as planned; a member that has waited `wait` ticks before that may decide
// (one compare-and-swap, so the two outcomes exclude each other) that the
// group runs on it alone: the others leave their CUs, now or when they
// arrive, and it does every member's part of every step in turn, by the same
// code and through the same exchange words, bit for bit with the same results.
// No launch then depends on what else runs on the device.  Meeting costs a
// launch of two steps 0.3-0.8 us; what a group costs that runs alone (50 us a
// step at H = 512) matters only beside launches that hold CUs for longer than
// the wait.
//
// Word: arrivals in bits 0-7, the sum of the arrivals' XCD numbers in bits
// 8-19 and of their squares in bits 20-35 (equal numbers: count * squares ==
// sum * sum), the deciding member in bits 48-55, bit 62 once it has decided.
// Two sets of words, used by launches of even and odd position in the call;
// each launch clears the other set for the next.
// ---------------------------------------------------------------------------
#define GROUP_SET 512
#define GROUP_WORDS (2 * GROUP_SET)   // in front of the exchange words
#define GROUP_ALONE_BIT (1ull << 62)
enum { GROUP_APART = 0, GROUP_LOCAL = 1, GROUP_ALONE = 2, GROUP_LEAVE = 3 };

__device__ __forceinline__ uint32_t xcd_id() {
  return __builtin_amdgcn_s_getreg(20 | (3 << 11));   // HW_REG_XCC_ID, bits 0-3
}
// Group and member of a workgroup.  Workgroup i runs on XCD i % 8, and each XCD
// starts its workgroups in order.  So the groups come in blocks of eight, one
// on each XCD, whose members follow each other there (what is left of a number
// of groups that 8 does not divide is spread over the XCDs): the exchange of
// nearly every group stays on one XCD, and few groups of a launch at a time
// have only a part of their members running.
__device__ __forceinline__ void group_of(int NG, int members, int* g, int* mem) {
  const int i = blockIdx.x, whole = NG / 8 * 8;
  if (i < whole * members) {
    *g = (i & 7) + 8 * ((i >> 3) / members);
    *mem = (i >> 3) % members;
  } else {
    *g = whole + (i - whole * members) % (NG - whole);
    *mem = (i - whole * members) / (NG - whole);
  }
}
// This workgroup arrives at its group's word (every thread calls it).  With no
// wait at all, the group's first member decides here, before it arrives.
__device__ __forceinline__ void group_arrive(uint64_t* words, uint32_t seq, int g, int mem, uint32_t wait) {
  if (blockIdx.x == 0 && threadIdx.x < GROUP_SET) words[((seq + 1) & 1) * GROUP_SET + threadIdx.x] = 0;
  if (threadIdx.x == 0) {
    const uint64_t x = xcd_id();
    if (wait == 0) {
      uint64_t none = 0;
      __hip_atomic_compare_exchange_strong(words + (seq & 1) * GROUP_SET + g, &none,
                                           GROUP_ALONE_BIT | (uint64_t)mem << 48, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
    }
    __hip_atomic_fetch_add(words + (seq & 1) * GROUP_SET + g, 1ull | x << 8 | x * x << 20, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
  }
}
// (a call of its own: inlined, it costs the forward's steps scalar registers)
static __device__ __attribute__((noinline)) void group_decide(uint64_t* p, uint32_t lo, uint32_t hi, int mem) {
  uint64_t seen = (uint64_t)hi << 32 | lo;
  __hip_atomic_compare_exchange_strong(p, &seen, seen | GROUP_ALONE_BIT | (uint64_t)mem << 48, __ATOMIC_RELAXED,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The group's word as group_meet takes it first; asked for ahead, its latency
// passes behind other work.
__device__ __forceinline__ uint64_t group_word(const uint64_t* words, uint32_t seq, int g) {
  return ll_load(words + (seq & 1) * GROUP_SET + g);
}
// How the group runs: GROUP_LOCAL (all its members, on one XCD), GROUP_APART
// (all, on several), GROUP_ALONE (this workgroup does all the work) or
// GROUP_LEAVE (another one does); the same for every wave of the workgroup.
// wait: 100 MHz ticks.
__device__ __forceinline__ int group_meet(uint64_t v, uint64_t* words, uint32_t seq, int g, int mem, int members,
                                          uint32_t wait) {
  uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  auto open = [&]() { return (lo & 255u) != (uint32_t)members && !(hi & (uint32_t)(GROUP_ALONE_BIT >> 32)); };
  if (open()) {
    uint64_t* p = words + (seq & 1) * GROUP_SET + g;
    const uint32_t t0 = (uint32_t)__builtin_amdgcn_s_memrealtime();
    do {
      if ((uint32_t)__builtin_amdgcn_s_memrealtime() - t0 >= wait) group_decide(p, lo, hi, mem);
      v = ll_load(p);
      lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
      hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    } while (open());
  }
  if (hi & (uint32_t)(GROUP_ALONE_BIT >> 32)) return (int)(hi >> 16 & 255u) == mem ? GROUP_ALONE : GROUP_LEAVE;
  const uint32_t sum = lo >> 8 & 4095u, sq = lo >> 20 | (hi & 15u) << 12;
  return (uint32_t)members * sq == sum * sum ? GROUP_LOCAL : GROUP_APART;
}
// The passes of a group that runs alone are calls of their own (not inlined),
// so that they take no registers from the steps before them; their arguments
// come in vector registers and are made scalar again.  The compiler would also
// keep what the passes derive from the kernel's argument and the thread's
// number in registers across the loop over them, so each pass reads the
// argument anew and takes the thread's number as unknown (KNOWN: below 512, said
// where that shortens the code; it lengthens the float32 kernels and makes the
// 32-row forward spill).
typedef __attribute__((address_space(3))) char* lds_base_t;
__device__ __forceinline__ int scalar(int v) { return __builtin_amdgcn_readfirstlane(v); }
// (in a kernel: its only argument where it lies; its address taken instead would move it to the stack)
template <class Args>
__device__ __forceinline__ const Args* kernel_args() { return (const Args*)__builtin_amdgcn_kernarg_segment_ptr(); }
template <class Args>
__device__ __forceinline__ Args pass_args(const Args* at) {
  const uint64_t v = (uint64_t)at;
  uint64_t u = (uint64_t)(uint32_t)scalar((int)(v >> 32)) << 32 | (uint32_t)scalar((int)v);
  asm volatile("" : "+s"(u));
  typedef const __attribute__((address_space(4))) Args* const_args_t;
  Args a;
  __builtin_memcpy(&a, (const void*)(const_args_t)u, sizeof(Args));
  return a;
}
template <bool ONE, bool KNOWN = true>
__device__ __forceinline__ int pass_thread() {
  int t = threadIdx.x;
  if constexpr (ONE) asm volatile("" : "+v"(t));
  return KNOWN ? t & 511 : t;
}
// A member's registers between the steps of a group that runs alone: 8 floats
// per thread, by group, member and thread.
#define GROUP_STATE 8
__device__ __forceinline__ float* group_state(float* st, int g, int mem, int members) {
  return st + (((int64_t)g * members + mem) * 512 + threadIdx.x) * GROUP_STATE;
}

struct PersistArgs {
  bf16* Y;            // layer output [M][2H] (forward: read h_prev, write h)
  const bf16* W;      // bf16 parameter copy (flat layout)
  int64_t whh0, whh1; // element offsets of W_hh for the two directions
  bf16* Gx;           // forward: input projection incl. both biases [M][8H] (written by the
                      // kernel itself when Xin is set, else read only)
  // forward, optional: the layer input and W_ih, so that each workgroup
  // computes the input projection of its own rows and gate columns before
  // the steps (instead of a separate product launch); null Xin: Gx is given
  const bf16* Xin;    // layer input [M][ldx] (bf16, 16-byte aligned rows)
  int64_t ldx;
  const bf16* Wih;    // W_ih of direction 0 [4H][ldw]; direction 1 at Wih + wih_d
  int64_t ldw, wih_d;
  const float* bih;   // b_ih and b_hh of direction 0 [4H]; direction 1 at + b_d
  const float* bhh;
  int64_t b_d;
  int Kin;            // input width (a multiple of 8; zero k past the operands' ends)
  // backward, optional: dy as ndy split-K partial sums (partial s of frame f,
  // unit column c at DYP[s * dy_kstride + f * 2H + c]) instead of DY; the
  // kernel sums its own rows' and units' entries in split order (the order
  // of the separate reduction) before the steps, into LDS
  const float* DYP;
  int ndy;
  int64_t dy_kstride;
  float* C;           // cell states [M][2H] (forward writes, backward reads)
  bf16* G;            // gate pre-activations [M][2][H][4] (direction, unit, gate i/f/g/o; forward writes, backward reads)
  bf16* DA;           // backward: gate pre-activation gradients [M][8H]
  const float* DY;    // backward: gradient reaching the layer output [M][2H]
  uint64_t* words;    // the groups' words (GROUP_WORDS)
  uint64_t* X;        // step-exchange words behind them (see lstm_persist.hip)
  float* state;       // registers of groups that run alone (see group_state)
  float* DBP;         // backward, optional: sums of da over each workgroup's rows and all steps
                      // [persist_bias_rows][8H] (per launch: its first row)
  int* status;        // recurrence status block (sticky flag, see persist_status_reset)
  uint32_t tag;       // caller: the layer's position in the order the call runs the layers
  int Tn, B, H;
  int b0, rows, NS;   // batch chunk handled by one launch (filled in by persist_layer)
  int NG;             // groups of the launch: 2 NS, or more with padding (persist_groups)
  uint32_t seq;       // the launch's position among the call's launches (filled in by persist_layer)
  uint32_t wait;      // ticks a member waits for its group (filled in by persist_layer)
};

// Exchange buffer: the groups' words, then 2 slots x 2 directions x row quads x (H/64 members, rounded up) x H
// units words of 8 bytes (the backward's partial sums: four rows per word, one
// where 64 does not divide H; the forward uses H/4 words per row, never more).
static inline size_t persist_xch_bytes(int B, int H) {
  const size_t members = (H + 63) / 64;
  size_t rows = 256 / (2 * members) * (H % 64 ? 16 : 32);   // the most of one launch on 256 CUs
  if (rows > (size_t)B) rows = B;
  const size_t bwd = (size_t)2 * 2 * ((rows + 3) / 4) * members * H * 8 * (H % 64 ? 4 : 1);
  const size_t fwd = (size_t)2 * 2 * rows * (H / 4 > 0 ? H / 4 : 1) * 8;
  return (bwd > fwd ? bwd : fwd) + GROUP_WORDS * 8;
}
// PersistArgs::state: of each workgroup that waits for others (256 CUs).
static inline size_t persist_state_bytes(int B, int H) {
  const size_t members = (H + 63) / 64;
  if (members < 2) return 0;
  size_t slices = (B + 7) / 8;
  if (slices > 256 / (2 * members)) slices = 256 / (2 * members);
  return 2 * slices * members * 512 * GROUP_STATE * 4;
}

// Whether the backward can take dy as split-K partials (its summed dy of all
// steps must fit the LDS beside the step buffers).
bool persist_bwd_dy_partials_ok(int H, int B, int T);
// True if the persistent kernels handle this H (a multiple of 32, at most
// 512: a member's 256 W_hh rows fit in its registers; the last member may own
// 32 units); any T.
bool persist_supported(int H, int T);
// Whether a forward of so few steps (two or more) is faster as one launch per
// step than with W_hh staged for the whole chunk.  At widths that 64 does not
// divide only: the others' exchange has always run at any T.  One launch per
// step / persistent, two layers, us: H = 480, B = 128, T = 2 43.6 / 50.8, T = 3
// 57.2 / 55.8; where a layer takes several persistent launches later, above all
// where the last is nearly empty: H = 224, B = 520, T = 5 94 / 106, B = 600 116 /
// 106; H = 480, B = 300, T = 3 94 / 129, T = 4 125 / 141.
bool persist_short_fwd(int H, int B, int T);
// Whether the forward computes the input projection (K columns) itself.  A
// workgroup runs it in passes of 176 rows at one workgroup per CU, so it pays
// where the workgroups fill most of the chip and the passes are mostly full
// (fused / separate product, us, two layers at H = 512: B = 100 (208 workgroups
// of 8 rows) T = 2 57 / 47, T = 12 101 / 100, T = 21 139 / 147, T = 64 368 / 370;
// B = 250 (256 of 16) T = 12 157 / 143, T = 21 222 / 231; with 104 workgroups at
// H = 256, B = 100, T = 40 196 / 184), and where there is next to nothing to
// multiply (one layer of 40 or 128 columns, T = 2, B = 4 to 100: 16.2-19.5 /
// 17.8-19.7; T = 8 25-32 / 25-30).
bool persist_fuse_gx(int H, int B, int T, int K);
// Rows of the BPTT's bias partial sums (PersistArgs::DBP): one per slice of 8,
// 16 or 32 batch rows.
int persist_bias_rows(int H, int B);
// Status block (PERSIST_STATUS_BYTES at the end of the activation
// workspace): an int flag set by any exchange wait that gives up, an int set by
// any group that ran alone, and a tag that marks the block initialised.  Both
// are sticky across calls.
#define PERSIST_STATUS_BYTES 256
// Clears the exchange words (and, for the forward, initialises the status
// block of a fresh workspace); once per forward or backward call, before
// its first persist_layer.
hipError_t persist_clear(bool backward, const PersistArgs& a, hipStream_t s);
// Initialises the status block if it is fresh (a forward call that does not
// take the persistent path, or whose exchange clear failed).
hipError_t persist_status_init(int* status, hipStream_t s);
// Clears the flag (after blstm_recurrence_ok has read it).
hipError_t persist_status_reset(int* status, hipStream_t s);
// Runs every step of one layer, both directions; hipSuccess or the error of
// the launch that failed.  The layers of one call carry tags 0, 1, 2, ...
// in the order they run (an exchange word tells its launch from the two
// before it by the launch's position modulo 4).
hipError_t persist_layer(bool backward, PersistArgs a, hipStream_t s);

// ---------------------------------------------------------------------------
// float32 persistent kernels (lstm_persist32.hip): the same split, exchange
// protocol, status block and launch rules with float32 operands.
// ---------------------------------------------------------------------------
struct Persist32Args {
  float* Y;             // forward: layer output [M][2H]
  const float* W;       // parameters (flat layout)
  int64_t whh0, whh1;   // element offsets of W_hh for the two directions
  const float* Gx;      // forward: input projection incl. both biases [M][8H]
  float* C;             // cell states [M][2H] (forward writes, backward reads)
  float* G;             // gate pre-activations [M][2][H][4] (forward writes, backward reads)
  float* DA;            // backward: gate pre-activation gradients [M][8H]
  const float* DY;      // backward: gradient reaching the layer output [M][2H]
  float* DBP;           // backward: sums of da over each workgroup's rows and all steps
                        // [cdiv(B, persist32_rows_per_workgroup)][8H]
  uint64_t* words;      // the groups' words (GROUP_WORDS)
  uint64_t* X;          // step-exchange words behind them
  float* state;         // registers of groups that run alone (see group_state)
  int* status;          // recurrence status block
  uint32_t tag0;        // caller: the layer's position in the call; per launch: the tag before its first step's
  int Tn, B, H;
  int b0, rows, NS, NG; // filled in by persist32_layer, as are
  uint32_t seq, wait;   // the launch's position in the call, the ticks a member waits for its group
};

// True if these kernels handle this H (a multiple of 16 up to 512).
bool persist32_supported(int H);
int persist32_rows_per_workgroup(int H, int B);
size_t persist32_xch_bytes(int B, int H);
size_t persist32_state_bytes(int B, int H);
hipError_t persist32_clear(bool backward, const Persist32Args& a, hipStream_t s);
hipError_t persist32_layer(bool backward, Persist32Args a, hipStream_t s);

// Compute units of the current device (0: unknown); one persistent workgroup
// runs on each.
int persist_max_wg();
// Groups a launch of `groups` groups of `members` workgroups is laid out for:
// a multiple of 8, which puts each on one XCD (see group_of; workgroup i runs
// on XCD i % 8, measured; the kernels check), where that many fit the chip at
// one workgroup per CU.  Workgroups of the groups past the real ones return at
// once.
int persist_groups(int groups, int members);
// Ticks a member waits for its group before it decides to run it alone (1 ms;
// ADPSGD_BLSTM_GROUP_WAIT_US sets another time, for tests).
uint32_t persist_group_wait();
// Launches a kernel whose workgroups wait for each other: plain when the
// occupancy query shows the whole grid resident at once on an idle device,
// else cooperative.  args: the kernel's only argument.
hipError_t persist_launch(const char* name, const void* fn, dim3 grid, int threads, size_t lds, void* args,
                          hipStream_t s);
// Zeroes n16 16-byte pieces at p (may be none) and, if status is given,
// initialises the status block of a fresh workspace.
hipError_t persist_clear_words(void* p, int64_t n16, int* status, hipStream_t s);
