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

// Placement words in front of the exchange words, one per workgroup of a
// launch: (launch mark << 32) | XCD.
#define PERSIST_PLACE_WORDS 1024
__device__ __forceinline__ uint32_t xcd_id() {
  return __builtin_amdgcn_s_getreg(20 | (3 << 11));   // HW_REG_XCC_ID, bits 0-3
}
// Announces this workgroup's XCD (one thread, at the kernel's start).
__device__ __forceinline__ void place_announce(uint64_t* place, uint32_t mark) {
  __hip_atomic_store(place + blockIdx.x, ((uint64_t)mark << 32) | xcd_id(), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
// Whether every member of the group (workgroups g, g + ng, ...; at most 64)
// runs on this XCD; all lanes of every wave call it, and get one answer.
__device__ __forceinline__ bool place_local(const uint64_t* place, uint32_t mark, int g, int ng, int members,
                                            int* status) {
  const int lane = threadIdx.x & 63;
  const uint64_t* p = place + g + (int64_t)(lane < members ? lane : 0) * ng;
  uint64_t v = ll_load(p);
  for (unsigned it = 0; !__all((uint32_t)(v >> 32) == mark); ++it) {
    if (it > PERSIST_SPIN_LIMIT ||
        ((it & 63) == 63 && __hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
      __hip_atomic_store(status, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
    v = ll_load(p);
  }
  return __all((uint32_t)v == xcd_id());
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
  uint64_t* place;    // placement words (PERSIST_PLACE_WORDS)
  uint64_t* X;        // step-exchange words behind them (see lstm_persist.hip)
  float* DBP;         // backward, optional: sums of da over each workgroup's rows and all steps
                      // [cdiv(B, rows per workgroup)][8H] (see persist_rows_per_workgroup)
  int* status;        // recurrence status block (sticky flag, see persist_status_reset)
  uint32_t tag;       // caller: the layer's position in the order the call runs the layers
  int Tn, B, H;
  int b0, rows, NS;   // batch chunk handled by one launch (filled in by persist_layer)
  int NG;             // groups of the launch: 2 NS, or more with padding (persist_groups)
  uint32_t seq;       // the launch's position among the call's launches (filled in by persist_layer)
};

// At most this many batch slices of 8, 16 or 32 rows per launch, so one
// launch covers at most PERSIST_MAX_ROWS rows.
#define PERSIST_MAX_SLICES 32
#define PERSIST_MAX_ROWS (PERSIST_MAX_SLICES * 32)
// Exchange buffer: the placement words, then 2 slots x 2 directions x row quads x (H/64 members, rounded up) x H
// units words of 8 bytes (the backward's partial sums: four rows per word, one
// where 64 does not divide H; the forward uses H/4 words per row, never more).
static inline size_t persist_xch_bytes(int B, int H) {
  const size_t rows = B < PERSIST_MAX_ROWS ? B : PERSIST_MAX_ROWS;
  const size_t members = (H + 63) / 64;
  const size_t bwd = (size_t)2 * 2 * ((rows + 3) / 4) * members * H * 8 * (H % 64 ? 4 : 1);
  const size_t fwd = (size_t)2 * 2 * rows * (H / 4 > 0 ? H / 4 : 1) * 8;
  return (bwd > fwd ? bwd : fwd) + PERSIST_PLACE_WORDS * 8;
}

// Whether the backward can take dy as split-K partials (its summed dy of all
// steps must fit the LDS beside the step buffers).
bool persist_bwd_dy_partials_ok(int H, int B, int T);
// True if the persistent kernels handle this H (a multiple of 32, at most
// 512: a member's 256 W_hh rows fit in its registers; the last member may own
// 32 units); any T.
bool persist_supported(int H, int T);
// Workgroups of a layer's largest launch for this H and B.
int persist_workgroups(int H, int B);
// Batch rows per persistent workgroup (8, 16 or 32) for this H and B: the row
// block of the BPTT's bias partial sums (PersistArgs::DBP).
int persist_rows_per_workgroup(int H, int B);
// Status block (PERSIST_STATUS_BYTES at the end of the activation
// workspace): an int flag set by any exchange wait that gives up, and a tag
// that marks the block initialised.  The flag is sticky across calls.
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
  uint64_t* place;      // placement words (PERSIST_PLACE_WORDS)
  uint64_t* X;          // step-exchange words behind them
  int* status;          // recurrence status block
  uint32_t tag0;        // caller: the layer's position in the call; per launch: the tag before its first step's
  int Tn, B, H;
  int b0, rows, NS, NG; // filled in by persist32_layer
};

// True if these kernels handle this H (a multiple of 16 up to 512).
bool persist32_supported(int H);
int persist32_rows_per_workgroup(int H, int B);
size_t persist32_xch_bytes(int B, int H);
hipError_t persist32_clear(bool backward, const Persist32Args& a, hipStream_t s);
hipError_t persist32_layer(bool backward, Persist32Args a, hipStream_t s);

// Compute units of the current device (0: unknown); one persistent workgroup
// runs on each.
int persist_max_wg();
// Groups a launch of `groups` groups of `members` workgroups is laid out for.
// Member m of group g is workgroup g + m NG, and workgroup i runs on XCD i % 8
// (measured; the kernels check), so an NG of a multiple of 8 puts a group on
// one XCD: workgroups of the groups past the real ones return at once.  Not
// padded where the padding would not fit the chip at one workgroup per CU.
int persist_groups(int groups, int members);
// Launches a kernel whose workgroups wait for each other: plain when the
// occupancy query shows the whole grid resident at once, else cooperative.
// args: the kernel's only argument.
hipError_t persist_launch(const char* name, const void* fn, dim3 grid, int threads, size_t lds, void* args,
                          hipStream_t s);
// Zeroes n16 16-byte pieces at p (may be none) and, if status is given,
// initialises the status block of a fresh workspace.
hipError_t persist_clear_words(void* p, int64_t n16, int* status, hipStream_t s);
