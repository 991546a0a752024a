// Single-launch paged attention for one mixed continuous-batching iteration:
// the decode share (one query token per decoding request) and the prefill
// share (a chunk of prompt tokens, causal over the prompt's cached prefix plus
// the chunk) of Eq. 1, Sec. 2.1, served by one grid.
//
// Grid: the work list's prefill units first, one 256-thread workgroup each,
// then decode units: four per workgroup (one per wavefront), or one
// (dlfp::decode_by_workgroup says when).
//
// Prefill unit = (sequence, KV head, tile of 128 query rows, key split).
// Rows are the tile's tokens x the g query heads sharing the KV head, so each
// K/V tile staged in LDS serves all g heads (grouped-query sharing in LDS).
// Each wavefront owns 32 rows and computes, per 64-key tile,
//   S^T = K Q^T        (v_mfma_f32_32x32x16_bf16, fp32 accumulation)
//   online softmax     (exp2 domain; each lane owns one row, so row max and
//                       sum need only one exchange with lane ^ 32)
//   O^T += V^T P^T     (P rounded to bf16; V pages are stored transposed, so
//                       the operand is read straight from LDS)
// Working with S^T and O^T keeps every row statistic lane-local, and the
// accumulator layout of S^T is already the B-operand layout of the PV
// product, so P never leaves registers.  K/V tiles are double-buffered in LDS
// (one barrier per tile), with XOR swizzles that keep the 16 lanes of each
// LDS access phase on distinct banks.  Tiles of at most 32 rows, where three
// of the four wavefronts would idle, split the keys over the wavefronts
// instead (prefill_small).
//
// Decode unit = (sequence, KV head, key split).  Memory-bound: pages of K and V
// reach LDS by fully coalesced, non-temporal 16-byte copies while earlier ones
// are consumed by 16x16 matrix products whose columns are the grouped heads.
//
// Split-K: a unit whose rows are split over several key ranges writes
// (unnormalised O, running max, running sum) to its workspace slot, releases,
// and bumps its group's counter; the last arriver acquires and merges all
// splits in split-index order (deterministic), writes the output and resets
// the counter to zero for the next launch.
//
// The same kernel, instantiated with APP, also writes the iteration's new
// keys and values into the cache (the append and the attention in one
// launch): a decode unit takes its own new token from k_new / v_new into its
// staged last page and stores it to its slot; leading append workgroups write
// the prompt tokens, and prefill units wait for them before loading a page
// that holds a new token (units of at most 32 rows take the new tokens from
// k_new / v_new and do not wait).  Instantiated with MIXED (a launch with both
// shares), the prefill tile loop issues its QK products in the order that
// suits a wavefront sharing its SIMD with a decode wavefront.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "dlfp.h"
#include "dlfp_internal.h"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

constexpr int D = DLFP_HEAD_DIM;
constexpr int PAGE = DLFP_PAGE_SIZE;
constexpr int PAGE_ELEMS = PAGE * D;          // bf16 elements per (block, head) page
constexpr int KV_TILE = 64;                   // keys per prefill tile (4 pages)
constexpr int THREADS = 256;
constexpr int PRE_PTAB = DLFP_MAX_PREFILL_UNIT_KEYS / PAGE;  // block ids of one prefill unit
constexpr int PRE_LDS = 4 * KV_TILE * D * 2 + PRE_PTAB * 4;  // 64 KiB of K/V tiles + 8 KiB
constexpr int DEC_PTAB = DLFP_MAX_DECODE_UNIT_KEYS / PAGE;   // block ids of one decode unit
// Per decode wavefront: two slots of (K page, V page), block ids.
constexpr int DEC_PAGE_SLOT = 2 * PAGE_ELEMS * 2;  // K and V page, 8 KiB
constexpr int DEC_WAVE_LDS = 2 * DEC_PAGE_SLOT + DEC_PTAB * 4;
// Per wavefront of a wide decode unit: a key slot and a value slot of two pages
// each, ids of its pages.
constexpr int WIDE_SLOT = 2 * PAGE_ELEMS * 2;
constexpr int WIDE_WAVE_LDS = 2 * WIDE_SLOT + DEC_PTAB;  // a quarter of a unit's pages, 4 bytes each
constexpr int LDS_BYTES = PRE_LDS > 4 * DEC_WAVE_LDS ? PRE_LDS : 4 * DEC_WAVE_LDS;
// Two workgroups per CU (160 KiB of LDS).
static_assert(2 * (LDS_BYTES + 16) <= 160 * 1024, "two workgroups must share a CU");
// Small prefill units: rows, keys of a block, and per wave one slot each of a
// block's keys and values plus the ids of its pages (two per block, every
// fourth block of the unit).
constexpr int SMALL_ROWS = 32, SMALL_KEYS = 32;
constexpr int SMALL_SLOT = SMALL_KEYS * D * 2;
constexpr int SMALL_WAVE_LDS = 2 * SMALL_SLOT + DLFP_MAX_PREFILL_UNIT_KEYS / PAGE / 4 * 4;
constexpr float NEG_BIG = -1.0e30f;
constexpr float LOG2E = 1.4426950408889634f;
static_assert(4 * WIDE_WAVE_LDS <= LDS_BYTES, "wide decode slices must fit the shared buffer");
static_assert(4 * SMALL_WAVE_LDS <= LDS_BYTES, "small prefill slices must fit the shared buffer");
static_assert(4 * 1024 * 16 + 2 * 4 * 32 * 4 <= LDS_BYTES, "partial results of the four waves");

struct Args {
  const int32_t* work;
  const int32_t* block_table;
  const uint16_t* q;
  const uint16_t* kc;
  const uint16_t* vc;
  void* out;
  float* ws;
  int32_t max_blocks;
  int32_t num_blocks;
  int32_t hq;
  int32_t hkv;
  int32_t num_units;
  int32_t num_prefill;
  int32_t out_f32;
  int32_t decode_waves;  // wavefronts of the decode workgroups of this launch
  int32_t decode_static; // decode units handed out by position, the rest by queue
  int32_t lead;          // prefill workgroups before the first decode workgroup
  int32_t decode_lead;   // decode workgroups before the remaining prefill ones
  int32_t deep;          // decode wavefronts keep two pages in flight
  int32_t wide;          // wavefronts of the workgroup of a decode unit; 0: a wavefront each
  float scale_log2;      // softmax scale * log2(e)
  // Append launches only: this iteration's keys and values [tokens][hkv][128],
  // the leading workgroups that write the append records stored after the
  // units, and the prefill units that wait for them.
  const uint16_t* k_new;
  const uint16_t* v_new;
  int32_t app_wgs;
  int32_t num_append;
  int32_t num_waiting;
};

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                         __builtin_bit_cast(bf16x2_t, b), c, false);
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  bf16x2_t v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

// TWO: the decode products take a probability in two bf16 terms, at no matrix
// product more: the columns that a unit's heads (at most 8 of 16) leave idle hold
// the same heads again.  Columns 0-7 take a probability's upper half, cut off, and
// columns 8-15 (`low`) the rest, which is then positive; at least the least normal
// number, so that the product with an infinite value is that infinity in both.  A
// row is then 3e-6 to 5e-6 off in the 2-norm where one rounded term leaves 1.1e-3
// to 1.6e-3.  Launches of decode units alone take two terms (1000 batches 1.01x
// the time, those of up to 8 us 1.02x, from 60 us on the same), and all units with
// one query head per KV head; beside prefill tiles the instructions come out of
// the tiles' time and power (Qwen3-8B, 128 decoders beside 1999 tokens: 1.006x).
template <int G>
constexpr bool two_terms(bool alone) {
  return alone || G == 1;
}
__device__ __forceinline__ uint32_t pack_term(float p0, float p1, bool low) {
  typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
  const uint32_t b0 = __builtin_bit_cast(uint32_t, p0), b1 = __builtin_bit_cast(uint32_t, p1);
  const uint32_t upper = __builtin_amdgcn_perm(b1, b0, 0x07060302u);
  const uint32_t rest = pack_bf16(p0 - __builtin_bit_cast(float, b0 & 0xFFFF0000u),
                                  p1 - __builtin_bit_cast(float, b1 & 0xFFFF0000u));
  const u16x2_t least = {0x0080, 0x0080};
  const u16x2_t kept = __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, rest), least);
  return low ? __builtin_bit_cast(uint32_t, kept) : upper;
}
// x plus the x of lane ^ 8 (rows of 16 lanes rotated by 8).  The sum is made
// here and not where its lanes are used, which keeps it one instruction.
__device__ __forceinline__ float sum_xor8(float x) {
  float y = x + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x128,
                                                                   0xF, 0xF, true));
  asm volatile("" : "+v"(y));
  return y;
}

__device__ __forceinline__ float fexp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float shfl_xor(float x, int m) { return __shfl_xor(x, m); }

// Combine a value with the one of lane ^ 16 (or lane ^ 32) by the gfx950
// permlane swaps (VALU, no LDS round trip): swapping two copies of a value
// leaves the lane's own value in one register and its partner's in the
// other.  Written as assembly because the compiler reads both results of
// the swap builtin from one register, losing the partner's value.
__device__ __forceinline__ void swap16(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void swap32(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float max_xor16(float x) {
  float a = x, b = x;
  swap16(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float max_xor32(float x) {
  float a = x, b = x;
  swap32(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float sum_xor16(float x) {
  float a = x, b = x;
  swap16(a, b);
  return a + b;
}
__device__ __forceinline__ float sum_xor32(float x) {
  float a = x, b = x;
  swap32(a, b);
  return a + b;
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Work records are read-only for the launch: read through the constant
// address space, so that a wave-uniform record comes in with scalar loads
// (one round trip for all its fields).
typedef const __attribute__((address_space(4))) int32_t* record_ptr;
__device__ __forceinline__ record_ptr as_record(const int32_t* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (record_ptr)(((uint64_t)hi << 32) | lo);
}
// A whole record in one scalar load.
typedef int32_t record_t __attribute__((ext_vector_type(16), aligned(4)));
__device__ __forceinline__ record_t load_record(const int32_t* p) {
  return *(const __attribute__((address_space(4))) record_t*)as_record(p);
}

// Lanes of one wavefront hand data to each other through LDS.  The hardware
// runs a wave's LDS operations in order; this keeps the compiler from moving a
// lane's LDS accesses across the hand-off (it reasons per lane, so a store to
// an address the lane itself never reads would otherwise be free to move).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int* group_counter_ptr(float* ws, int grp) {
  return reinterpret_cast<int*>(reinterpret_cast<char*>(ws) + DLFP_WORKSPACE_HEADER) + grp;
}

// Header words of the workspace: the decode queue's next ticket and the
// count of decode wavefronts that found it empty.
__device__ __forceinline__ int* header_word(float* ws, int i) { return reinterpret_cast<int*>(ws) + i; }
constexpr int HDR_TICKET = DLFP_WORKSPACE_TICKET_WORD;
constexpr int HDR_DONE = DLFP_WORKSPACE_DONE_WORD;
// Append launches: append workgroups finished, waiting prefill units finished.
constexpr int HDR_APPEND = DLFP_WORKSPACE_APPEND_WORD;
constexpr int HDR_WAITED = DLFP_WORKSPACE_WAITED_WORD;

// Error word values: 1 = a block id outside the pool, 2 = a wait for the
// append records ran out.
__device__ __forceinline__ void raise_error(float* ws, int code = 1) {
  __hip_atomic_store(reinterpret_cast<int*>(ws), code, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Append launches.  A prefill unit polls the count of finished append
// workgroups (device-coherent loads, so a stale L2 line is never returned)
// until all have counted themselves; the append workgroups come first in the
// grid and wait for nothing, so they are dispatched before any waiting unit
// and the count is reached.  The poll is bounded all the same: after about
// a second it raises error 2 and goes on.  A waiting unit counts itself on
// a second word once its loop is done (it never polls again); the last one
// zeroes both words for the next launch.  None of these units reads a page that
// holds a new token before its wait, so it meets no old copy of one in its L2.
// (Tiles of at most 32 rows and decode units do read such pages beside the
// stores; they put the new tokens in from k_new and v_new, and no later launch
// sees those copies: a launch begins with its L2s invalidated.)
constexpr int APPEND_SPIN_LIMIT = 1 << 20;

__device__ __forceinline__ void wait_for_appends(const Args& a) {
  const int* done = header_word(a.ws, HDR_APPEND);
  const int need = a.app_wgs;
  for (int spins = 0;; ++spins) {
    const int n = uniform(__hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    if (n >= need) break;
    if (spins == APPEND_SPIN_LIMIT) {
      if ((threadIdx.x & 63) == 0) raise_error(a.ws, 2);
      break;
    }
    __builtin_amdgcn_s_sleep(8);
  }
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// Split-K partial results cross workgroups (and XCDs, whose L2s are not
// coherent with each other).  They are written with device-coherent stores
// (the sc1 policy: written through to the device coherence point) and read
// back with device-coherent loads (which do not return stale L2 lines), both
// through a buffer resource bounded to the group's slots.  Before a unit
// bumps its group counter it waits until all its vector-memory operations,
// stores included, have completed; the last arriver issues its loads only
// after the counter read has returned.  This orders the exchange without
// writing back or invalidating whole L2 caches per unit.
constexpr int CPOL_SC1 = 16;  // cache-policy bit: coherent at device scope

// Loads past the group's slots return zero: a batch of a decode merge may reach
// past the last split (a repeated split with a weight of zero would make an
// infinite partial value a NaN, as the masked keys of a prefill tile make one).
struct Slots {
  __amdgpu_buffer_rsrc_t r;
};

__device__ __forceinline__ Slots group_slots(float* ws, int group_off, int nsplits,
                                             int slot_floats) {
  return Slots{__builtin_amdgcn_make_buffer_rsrc(ws + group_off, 0, nsplits * slot_floats * 4,
                                                 0x00020000)};
}
__device__ __forceinline__ void pstore4(Slots s, int float_off, f32x4_t v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), s.r, float_off * 4, 0,
                                         CPOL_SC1);
}
__device__ __forceinline__ void pstore2(Slots s, int float_off, f32x2_t v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), s.r, float_off * 4, 0,
                                        CPOL_SC1);
}
__device__ __forceinline__ void pstore1(Slots s, int float_off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), s.r, float_off * 4, 0,
                                        CPOL_SC1);
}
__device__ __forceinline__ f32x4_t pload4(Slots s, int float_off) {
  return __builtin_bit_cast(f32x4_t,
                            __builtin_amdgcn_raw_buffer_load_b128(s.r, float_off * 4, 0, CPOL_SC1));
}
__device__ __forceinline__ f32x2_t pload2(Slots s, int float_off) {
  return __builtin_bit_cast(f32x2_t,
                            __builtin_amdgcn_raw_buffer_load_b64(s.r, float_off * 4, 0, CPOL_SC1));
}
__device__ __forceinline__ float pload1(Slots s, int float_off) {
  return __builtin_bit_cast(float,
                            __builtin_amdgcn_raw_buffer_load_b32(s.r, float_off * 4, 0, CPOL_SC1));
}
// Floats per partial slot: O (rows x 128), m[rows], l[rows], padded to 256 bytes.
__device__ __forceinline__ int slot_floats_for(int rows) {
  return (rows * (D + 2) + 63) / 64 * 64;
}
// Wait for every outstanding vector-memory operation of this wave (on gfx9 the
// vector-memory counter covers stores) and keep the compiler from moving
// memory operations across the wait.
__device__ __forceinline__ void wait_memory_complete() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0), expcnt and lgkmcnt unconstrained
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}
// Wait until at most N of this wave's copies are in flight; until its LDS
// reads have returned.
template <int N>
__device__ __forceinline__ void wait_copies() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ int arrive(float* ws, int grp) {
  return __hip_atomic_fetch_add(group_counter_ptr(ws, grp), 1, __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ int* group_counter(float* ws, int grp) {
  return group_counter_ptr(ws, grp);
}

// Workgroups are dealt round-robin over the 8 XCDs; map them so that each XCD
// gets a contiguous range of prefill units (same KV head -> same L2).
__device__ __forceinline__ int xcd_remap(int b, int n) {
  const int x = b & 7, i = b >> 3;
  const int per = n >> 3, rem = n & 7;
  return x * per + min(x, rem) + i;
}

// Store 4 consecutive output values of one row.
__device__ __forceinline__ void store4(const Args& a, int64_t elem, float v0, float v1, float v2,
                                       float v3) {
  if (a.out_f32) {
    f32x4_t v = {v0, v1, v2, v3};
    *reinterpret_cast<f32x4_t*>(static_cast<float*>(a.out) + elem) = v;
  } else {
    u32x2_t v = {pack_bf16(v0, v1), pack_bf16(v2, v3)};
    *reinterpret_cast<u32x2_t*>(static_cast<uint16_t*>(a.out) + elem) = v;
  }
}

__device__ __forceinline__ void store2(const Args& a, int64_t elem, float v0, float v1) {
  if (a.out_f32) {
    f32x2_t v = {v0, v1};
    *reinterpret_cast<f32x2_t*>(static_cast<float*>(a.out) + elem) = v;
  } else {
    *reinterpret_cast<uint32_t*>(static_cast<uint16_t*>(a.out) + elem) = pack_bf16(v0, v1);
  }
}

// ---------------------------------------------------------------- prefill

// Prefill LDS map: K tiles in two slots at 0 and 16 KiB, V^T tiles in two
// slots at 32 and 48 KiB, the unit's block ids from 64 KiB.
constexpr int TILE_BYTES = KV_TILE * D * 2;  // 16 KiB: 64 keys of K, or of V^T
constexpr int V_BASE = 2 * TILE_BYTES;
constexpr int PTAB_BASE = 4 * TILE_BYTES;
// A running row maximum is only raised once a tile's maximum exceeds it by
// more than this many powers of two, so probabilities stay below 2^8 and the
// accumulators are rescaled rarely (the final division by the row sum makes
// the result independent of the reference maximum).
constexpr float RESCALE_LOG2 = 8.f;

// V^T rows (dims) store their two 16-byte halves swapped when bits 2 and 3
// of the dim differ; 8 (or 16) consecutive dims then cover every LDS bank
// once for each half.
__device__ __forceinline__ int vt_swz(int d) { return ((d >> 2) ^ (d >> 3)) & 1; }

// Position of token slot t inside a V^T row of the cache: slots 4-7 and 8-11
// trade places (bits 2 and 3 swap), matching the key order of the
// S^T accumulator rows that become the PV operand.
__device__ __forceinline__ int vt_pos(int t) { return (t & 3) | ((t & 4) << 1) | ((t & 8) >> 1); }

typedef __attribute__((address_space(3))) char* lds_ptr_t;
// One 16-byte piece per lane, global to LDS without registers: lane l's piece
// lands at LDS byte address lds + 16 l (lds is wave-uniform).  Completion is
// counted by the vector-memory counter; the caller waits for it explicitly
// (wait_memory_complete) before the barrier that publishes the tile.  The
// copy is written as assembly so that the compiler, which cannot tell the
// ring slots apart, does not wait for it before every LDS read.
__device__ __forceinline__ void lds_copy16(const char* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(src), "s"(lds)
               : "memory", "m0");
}
// The same copy from a wave-uniform base and a lane's byte offset (the address
// costs no vector instruction).
__device__ __forceinline__ const char* uniform_ptr(const void* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const char*>(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void lds_copy16(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}
// The same copy marked non-temporal, for the decode share's pages: each is
// read once per launch, so streaming them past the caches keeps the prefill
// share's K/V tiles (read by many query tiles) resident in L2 and raises the
// decode share's own HBM rate (Qwen3-32B decode-only 5.91 -> 6.49 TB/s).
__device__ __forceinline__ void lds_copy16_nt(const char* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt"
               :
               : "v"(src), "s"(lds)
               : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_addr(char* p) {
  return (uint32_t)(uintptr_t)(lds_ptr_t)p;
}

// Keep the elements of a 16-bit-element vector whose key index is below
// limit; key_of(e) gives element e's key.
template <typename F>
__device__ __forceinline__ u32x4_t mask_elems(u32x4_t v, int limit, F key_of) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const uint32_t lo = key_of(2 * w) < limit ? 0x0000FFFFu : 0u;
    const uint32_t hi = key_of(2 * w + 1) < limit ? 0xFFFF0000u : 0u;
    v[w] &= (lo | hi);
  }
  return v;
}

// Last arriver's merge of a prefill group: every split's (O, m, l) in split
// order with an online rescale.  TPR threads per row; a row's 128 values are
// 32 four-float pieces (chunk c = piece / 2, half = piece % 2 of the partial
// layout), and the thread with index sub in its row takes pieces
// sub + TPR i.  The loads of NB splits (pieces, maxima and sums) are issued
// before any is consumed, so a batch costs about one memory round trip; NB is
// chosen so that a batch holds about 136 registers.  Every load instruction
// of a wavefront reads whole contiguous runs of the partial layout.
template <int G, int TPR>
__device__ __forceinline__ void prefill_merge(const Args& a, const Slots sl, int slot_floats,
                                              int nsplits, int rows, int row0, int kh) {
  constexpr int NP = 32 / TPR;             // pieces per thread
  constexpr int PP = NP < 8 ? NP : 8;      // pieces per pass
  constexpr int PASSES = NP / PP;
  constexpr int NB = 32 / PP;              // splits per batch
  const int tid = threadIdx.x;
  if (tid >= TPR * rows) return;
  const int row = tid / TPR, sub = tid % TPR;
  const int64_t orow = ((int64_t)(row0 + row / G) * a.hq + kh * G + row % G) * D;
  for (int pass = 0; pass < PASSES; ++pass) {
    float M = NEG_BIG, lsum = 0.f;
    f32x4_t acc[PP];
#pragma unroll
    for (int i = 0; i < PP; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < nsplits; j += NB) {
      float mj[NB], lj[NB];
      f32x4_t x[NB][PP];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int b = min(j + u, nsplits - 1) * slot_floats;
        mj[u] = pload1(sl, b + rows * D + row);
        lj[u] = pload1(sl, b + rows * D + rows + row);
#pragma unroll
        for (int i = 0; i < PP; ++i) {
          const int piece = sub + TPR * (pass * PP + i);
          x[u][i] = pload4(sl, b + (((piece >> 1) * rows + row) * 8 + 4 * (piece & 1)));
        }
      }
      float mn = M;
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (j + u < nsplits) mn = fmaxf(mn, mj[u]);
      const float rs = fexp2(M - mn);
      M = mn;
      lsum *= rs;
#pragma unroll
      for (int i = 0; i < PP; ++i) acc[i] *= rs;
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const float w = j + u < nsplits ? fexp2(mj[u] - mn) : 0.f;
        lsum += w * lj[u];
#pragma unroll
        for (int i = 0; i < PP; ++i) acc[i] += w * x[u][i];
      }
    }
    const float inv = 1.f / lsum;
#pragma unroll
    for (int i = 0; i < PP; ++i) {
      // piece -> chunk c = 4 mb + g4 and half h -> dims 32 mb + 8 g4 + 4 h
      const int piece = sub + TPR * (pass * PP + i);
      const int c = piece >> 1;
      const int dim = 32 * (c >> 2) + 8 * (c & 3) + 4 * (piece & 1);
      store4(a, orow + dim, acc[i][0] * inv, acc[i][1] * inv, acc[i][2] * inv, acc[i][3] * inv);
    }
  }
}

// MIXED: the launch also has decode units (the issue order of the tile loop).
template <int G, bool APP, bool MIXED, class R>
__device__ void prefill_unit(const Args& a, const int32_t* it, const R f, char* smem, int* flag) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int col = lane & 31, hi = lane >> 5;
  const int s = f[DLFP_W_SEQ], kh = f[DLFP_W_KVHEAD];
  const int t0 = f[DLFP_W_QTOK0], nt = f[DLFP_W_QNTOK];
  const int kb = f[DLFP_W_KVBEGIN], ke = f[DLFP_W_KVEND];
  const int nsplits = f[DLFP_W_NSPLITS];
  // First packed row and first position of the sequence's new tokens.
  const int q0 = f[DLFP_W_QROW0] - t0, pos0 = f[DLFP_W_QPOS0] - t0;
  const int32_t* bt = a.block_table + (int64_t)s * a.max_blocks;

  const int r = wave * 32 + col;       // this lane's row within the tile
  const int tr = r / G, hh = r % G;    // token within the unit, head within the group
  const bool row_ok = tr < nt;
  const int lim = row_ok ? min(pos0 + t0 + tr + 1, ke) : 0;  // keys < lim are visible
  const int wave_tok0 = uniform((wave * 32) / G);
  const bool wave_active = wave_tok0 < nt;
  const int wave_lim_min = min(pos0 + t0 + wave_tok0 + 1, ke);

  // Q^T as the B operand: lane holds dims [16kk + 8hi, +8) of its row.
  // Rows past the unit's tokens load the first row's query; they are never stored.
  bf16x8_t qf[8];
  {
    const int64_t qrow = ((int64_t)(q0 + t0 + (row_ok ? tr : 0)) * a.hq + kh * G + hh) * D;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      qf[kk] = *reinterpret_cast<const bf16x8_t*>(a.q + qrow + 16 * kk + 8 * hi);
  }

  const int ntiles = (ke - kb + KV_TILE - 1) / KV_TILE;
  const int first_page = kb / PAGE, last_page = (ke - 1) / PAGE;
  // Append launches: the first tile with a page at or past the one holding
  // the sequence's first new token (the unit waits before loading it).
  int wait_tile = ntiles;
  if constexpr (APP) {
    const int newp = pos0 / PAGE;
    if (a.app_wgs > 0 && last_page >= newp)
      wait_tile = max(0, (newp - first_page) >> 2);  // wave 3's page
  }
  int32_t* ptab = reinterpret_cast<int32_t*>(smem + PTAB_BASE);
  for (int i = tid; i <= last_page - first_page; i += THREADS) ptab[i] = bt[first_page + i];
  wait_memory_complete();  // queries and block ids resident before the KV pipeline starts
  __syncthreads();

  // Copies: wave w moves page w of each 64-key tile, its 16 K rows and its
  // 128 V^T rows, as four 1 KiB pieces each.  K row R keeps 16-byte chunk x
  // at position x ^ (R & 15); V^T row d keeps half h at position h ^ vt_swz(d).
  uint32_t koff[4], voff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rr = 4 * i + (lane >> 4);
    koff[i] = rr * 256 + (((lane & 15) ^ rr) << 4);
    const int d = 32 * i + (lane >> 1);
    voff[i] = d * 32 + (((lane & 1) ^ vt_swz(d)) << 4);
  }
  // Straight-line on purpose: a page past the unit's last key re-reads its
  // last page (every key there is masked), and a block id outside the pool is
  // replaced by block 0 after raising the error word.
  // Block id of this wave's page of tile t, and its element offset (same in
  // both caches).
  auto page_id = [&](int t) {
    return ptab[min(first_page + 4 * t + wave, last_page) - first_page];
  };
  auto page_off = [&](int id) -> int64_t {
    const int raw = uniform(id);
    const bool ok = (unsigned)raw < (unsigned)a.num_blocks;
    if (!ok && lane == 0) raise_error(a.ws);
    return ((int64_t)(ok ? raw : 0) * a.hkv + kh) * PAGE_ELEMS;
  };
  const uint32_t lds_wave = lds_addr(smem) + uniform(wave) * (PAGE * 256);
  auto issue_k = [&](int64_t off, int slot) {
    const char* src = uniform_ptr(a.kc + off);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds_copy16(src, koff[i], lds_wave + slot * TILE_BYTES + i * 1024);
  };
  auto issue_v = [&](int64_t off, int slot) {
    const char* src = uniform_ptr(a.vc + off);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      lds_copy16(src, voff[i], lds_wave + V_BASE + slot * TILE_BYTES + i * 1024);
  };
  // Values past the unit's last key are zeroed in LDS (a probability of 0
  // times a NaN left in an unused slot would still be NaN).
  auto zero_v_tail = [&](int slot, int k0) {
    const int pg = tid >> 6;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int d = 2 * (tid & 63) + (c >> 1), h = c & 1;
      char* p = smem + V_BASE + slot * TILE_BYTES + pg * (PAGE * 256) + d * 32 + (h << 4);
      const int half = h ^ vt_swz(d);
      const int key0 = k0 + pg * PAGE;
      *reinterpret_cast<u32x4_t*>(p) = mask_elems(*reinterpret_cast<const u32x4_t*>(p), ke,
                                                   [&](int e) { return key0 + vt_pos(8 * half + e); });
    }
  };

  // Per-lane LDS offsets.  K: chunk (2kk + hi) of row R = 32 kb2 + col sits at
  // ((2kk + hi) ^ (col & 15)) << 4, i.e. kbase ^ (kk << 5).  V^T: half hi of
  // dim row d = 32 mb + col, at a lane-constant offset plus immediates.
  const int kbase = col * 256 + ((hi ^ (col & 15)) << 4);
  const int vbase = V_BASE + col * 32 + ((hi ^ vt_swz(col)) << 4);

  float m_run = NEG_BIG, l_run = 0.f;
  f32x16_t o[4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) o[mb] = f32x16_t{};
  const float c = a.scale_log2;

  // S^T = K Q^T for the 64 keys of the tile in K slot `slot`: two 32-key
  // accumulators advanced alternately.  sacc[kb2][rr] holds key
  // 32 kb2 + 8 (rr / 4) + 4 hi + rr % 4 of this lane's row.
  auto qk = [&](f32x16_t* sacc, int slot) {
    sacc[0] = f32x16_t{};
    sacc[1] = f32x16_t{};
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const char* kp = smem + slot * TILE_BYTES + (kbase ^ (kk << 5));
      const bf16x8_t k0f = *reinterpret_cast<const bf16x8_t*>(kp);
      const bf16x8_t k1f = *reinterpret_cast<const bf16x8_t*>(kp + 32 * 256);
      sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k0f, qf[kk], sacc[0], 0, 0, 0);
      sacc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k1f, qf[kk], sacc[1], 0, 0, 0);
    }
  };
  // Causal and tail mask for a tile starting at key k0 (raw scores).
  auto mask = [&](f32x16_t* sacc, int k0) {
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) {
        const int key = k0 + kb2 * 32 + 8 * (rr >> 2) + 4 * hi + (rr & 3);
        sacc[kb2][rr] = key < lim ? sacc[kb2][rr] : -__builtin_inff();
      }
  };
  // Row maximum of a tile (raw scores), this half of the row; in four chains
  // where the products do not wait for anything else (beside decode wavefronts
  // one chain is 0.5% faster).
  auto rowmax = [&](const f32x16_t* sacc) {
    if constexpr (MIXED) {
      float mx = -__builtin_inff();
#pragma unroll
      for (int i = 0; i < 32; ++i) mx = fmaxf(mx, sacc[i >> 4][i & 15]);
      return mx;
    }
    float m4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      m4[i] = fmaxf(sacc[i >> 1][8 * (i & 1)], sacc[i >> 1][8 * (i & 1) + 1]);
#pragma unroll
    for (int rr = 2; rr < 8; ++rr)
#pragma unroll
      for (int i = 0; i < 4; ++i) m4[i] = fmaxf(m4[i], sacc[i >> 1][8 * (i & 1) + rr]);
    return fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
  };
  // Raise the reference maximum where a tile's row maximum (mx: of one half of
  // the row) exceeds it by more than RESCALE_LOG2 (scaled units); the
  // accumulators follow.
  auto rebase = [&](float mx) {
    const float m_tile = max_xor32(mx) * c;
    if (__builtin_amdgcn_ballot_w64(m_tile > m_run + RESCALE_LOG2)) {
      const float m_new = m_tile > m_run + RESCALE_LOG2 ? m_tile : m_run;
      const float alpha = fexp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) o[mb] *= alpha;
    }
  };
  // P^T = exp2(S^T c - m) rounded to bf16, as the B operands of the four
  // 16-key steps k0 .. k1 - 1 of PV; pf[kk] holds keys 16 kk + {0-3, 8-11} + 4 hi.
  auto probs = [&](const f32x16_t* sacc, bf16x8_t* pf, int k0, int k1) {
#pragma unroll
    for (int kk = k0; kk < k1; ++kk) {
      u32x4_t pk;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float p0 = fexp2(__builtin_fmaf(sacc[kk >> 1][8 * (kk & 1) + 2 * w], c, -m_run));
        const float p1 = fexp2(__builtin_fmaf(sacc[kk >> 1][8 * (kk & 1) + 2 * w + 1], c, -m_run));
        pk[w] = pack_bf16(p0, p1);
      }
      pf[kk] = __builtin_bit_cast(bf16x8_t, pk);
    }
  };
  // Row sum of the rounded probabilities (this half of the row).
  auto rowsum = [&](const bf16x8_t* pf) {
    constexpr uint32_t ONES = 0x3F803F80u;  // two bf16 1.0
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const u32x4_t pk = __builtin_bit_cast(u32x4_t, pf[kk]);
#pragma unroll
      for (int w = 0; w < 4; ++w) l_run = dot2(pk[w], ONES, l_run);
    }
  };
  // O^T += V^T P^T over the 16-key steps k0 .. k1 - 1 of the tile in V slot `slot`.
  auto pv = [&](const bf16x8_t* pf, int slot, int k0, int k1) {
#pragma unroll
    for (int kk = k0; kk < k1; ++kk)
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        const bf16x8_t vf = *reinterpret_cast<const bf16x8_t*>(
            smem + vbase + slot * TILE_BYTES + kk * (PAGE * 256) + mb * 1024);
        o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[kk], o[mb], 0, 0, 0);
      }
  };
  const bool tail = kb + ntiles * KV_TILE > ke;  // the last tile reaches past the unit's keys

  // Prologue: tiles 0 (K and V) and 1 (K) in flight, then S_0.  off_next
  // carries the page of tile j + 1 from the step that loaded its keys to the
  // step that loads its values.
  // The wait for the append records sits outside the tile loop (which is
  // split there): inside it, the poll's control flow costs the loop body its
  // partial LDS waits.  Tile t's keys are issued in the prologue (t < 2) or
  // by step t - 2.
  if constexpr (APP) {
    if (wait_tile <= 1) wait_for_appends(a);
  }
  int64_t off_next = page_off(page_id(0));
  issue_k(off_next, 0);
  issue_v(off_next, 0);
  if (ntiles > 1) {
    off_next = page_off(page_id(1));
    issue_k(off_next, 1);
  }
  wait_memory_complete();
  __syncthreads();
  if (tail && ntiles == 1) {
    zero_v_tail(0, kb);
    __syncthreads();
  }
  f32x16_t sa[2], sb[2];
  if (wave_active) {
    qk(sa, 0);
    if (kb + KV_TILE > wave_lim_min) mask(sa, kb);
    rebase(rowmax(sa));
  }
  __syncthreads();  // K slot 0 is refilled below
  int id2 = page_id(2);  // read a step before its use

  // Iteration j: loads of K_{j+2} and V_{j+1} go out; S_{j+1} = K_{j+1} Q^T
  // runs on the matrix cores while probabilities of tile j are formed (without
  // decode units the first half of them, the second half beside the first half
  // of O += V_j P_j, and the row maxima of tile j + 1 beside its second half:
  // the exponentials outlast the QK products); then O += V_j P_j.  Large
  // launches are bound by the clock the power limit leaves (1.7 of 2.4 GHz).
  // With that order, the addresses of the copies in scalar registers and the
  // block ids read a step ahead: prefill alone, 2048 tokens over 6144 keys
  // (g = 2) 131.6 -> 128.2 us, 4096 over 8192 (g = 8) 1192 -> 1157 us; beside decode
  // units, in their order, 8192 tokens over 16384 6727 -> 6587 us.
  auto step = [&](int j, f32x16_t* cur, f32x16_t* nxt, auto parity) {
    constexpr int PAR = decltype(parity)::value;  // j & 1
    constexpr int FIRST = MIXED ? 4 : 2;  // 16-key steps whose exponentials run beside QK
    const bool more = j + 1 < ntiles;
    if (more) issue_v(off_next, PAR ^ 1);
    if (j + 2 < ntiles) {
      off_next = page_off(id2);
      issue_k(off_next, PAR);
    }
    id2 = page_id(j + 3);
    if (wave_active) {
      bf16x8_t pf[4];
      // On the last tile this reads a stale slot; the result is not used, and
      // keeping it unconditional lets the products overlap the exponentials.
      qk(nxt, PAR ^ 1);
      probs(cur, pf, 0, FIRST);
      // The key operands of the QK products are read four products ahead, one
      // per product, and the exponentials fill the gaps between the products.
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      // The PV products and row sums run at raised wave priority: the SIMD
      // arbiter then keeps feeding the matrix core of the wave that is past
      // its exponentials while the other waves of the CU finish theirs
      // (measured 4-7% more prefill throughput on long chunks).
      __builtin_amdgcn_s_setprio(1);
      // Issue order of the raised-priority phase (s_setprio ends a scheduling
      // region): the value operands four products ahead, VALU work between.
      float mx;
      if constexpr (MIXED) {
        pv(pf, PAR, 0, 4);
        rowsum(pf);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      } else {
        probs(cur, pf, FIRST, 4);
        pv(pf, PAR, 0, FIRST);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 1);
#pragma unroll
        for (int i = 0; i < 4 * FIRST; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
          __builtin_amdgcn_sched_group_barrier(0x002, 5, 1);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        pv(pf, PAR, FIRST, 4);
        rowsum(pf);
        mx = rowmax(nxt);
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 2);
#pragma unroll
        for (int i = 0; i < 16 - 4 * FIRST; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 2);
          __builtin_amdgcn_sched_group_barrier(0x002, 5, 2);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 2);
        }
      }
      __builtin_amdgcn_s_setprio(0);
      if (more) {
        const int k1 = kb + (j + 1) * KV_TILE;
        const bool masked = k1 + KV_TILE > wave_lim_min;
        if (masked) mask(nxt, k1);
        if (MIXED || masked) mx = rowmax(nxt);
        rebase(mx);
      }
    }
    wait_memory_complete();
    __syncthreads();
    if (tail && j + 2 == ntiles) {  // V of the last tile has landed
      zero_v_tail(PAR ^ 1, kb + (ntiles - 1) * KV_TILE);
      __syncthreads();
    }
  };
  const std::integral_constant<int, 0> even;
  const std::integral_constant<int, 1> odd;
  int j = 0;
  if constexpr (APP) {
    if (wait_tile > 1 && wait_tile < ntiles) {
      const int jw = wait_tile - 2;  // the step that issues tile wait_tile
      for (; j + 1 < jw; j += 2) {
        step(j, sa, sb, even);
        step(j + 1, sb, sa, odd);
      }
      if (j < jw) step(j++, sa, sb, even);
      wait_for_appends(a);
      if (j & 1) step(j++, sb, sa, odd);
    }
  }
  for (; j < ntiles; j += 2) {
    step(j, sa, sb, even);
    if (j + 1 < ntiles) step(j + 1, sb, sa, odd);
  }

  // A waiting unit counts itself past its wait; the count returns while the
  // results are stored, and the last such unit zeroes the append words.
  int waited = -1;
  if constexpr (APP) {
    if (wait_tile < ntiles && tid == 0)
      waited = __hip_atomic_fetch_add(header_word(a.ws, HDR_WAITED), 1, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
  }
  auto reset_append_words = [&]() {
    if constexpr (APP) {
      if (waited >= 0 && waited == a.num_waiting - 1) {
        __hip_atomic_store(header_word(a.ws, HDR_APPEND), 0, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(header_word(a.ws, HDR_WAITED), 0, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  };

  l_run = sum_xor32(l_run);
  const int rows = nt * G;
  // o[mb][rr] = O[row][32 mb + 8 (rr / 4) + 4 hi + rr % 4]
  if (nsplits == 1) {
    if (row_ok) {
      const float inv = 1.f / l_run;
      const int64_t orow = ((int64_t)(q0 + t0 + tr) * a.hq + kh * G + hh) * D;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
          store4(a, orow + mb * 32 + 8 * g4 + 4 * hi, o[mb][4 * g4] * inv,
                 o[mb][4 * g4 + 1] * inv, o[mb][4 * g4 + 2] * inv, o[mb][4 * g4 + 3] * inv);
    }
    reset_append_words();
    return;
  }

  // Partial result: O as 16 chunks c = 4 mb + g4 of [rows][2][4] floats (chunk
  // c, row r, half h holds dims 32 mb + 8 g4 + 4 h .. + 3), so that a wave's
  // store and the merge's loads each cover a contiguous kilobyte; then
  // m[rows] and l[rows].
  const int slot_floats = slot_floats_for(rows);
  const Slots sl = group_slots(a.ws, it[DLFP_W_WSGROUP], nsplits, slot_floats);
  const int my = it[DLFP_W_SPLIT] * slot_floats;
  if (row_ok) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4_t v = {o[mb][4 * g4], o[mb][4 * g4 + 1], o[mb][4 * g4 + 2],
                           o[mb][4 * g4 + 3]};
        pstore4(sl, my + ((4 * mb + g4) * rows + r) * 8 + 4 * hi, v);
      }
    if (hi == 0) {
      pstore1(sl, my + rows * D + r, m_run);
      pstore1(sl, my + rows * D + rows + r, l_run);
    }
  }
  wait_memory_complete();
  reset_append_words();
  __syncthreads();  // every wave of the unit has completed its stores
  const int grp = it[DLFP_W_GROUP];
  if (tid == 0) *flag = arrive(a.ws, grp) == nsplits - 1;
  __syncthreads();
  if (!*flag) return;

  // Last arriver: merge every split of the group (threads per row chosen so
  // that the whole workgroup takes part).
  if (rows > 64)
    prefill_merge<G, 2>(a, sl, slot_floats, nsplits, rows, q0 + t0, kh);
  else if (rows > 32)
    prefill_merge<G, 4>(a, sl, slot_floats, nsplits, rows, q0 + t0, kh);
  else
    prefill_merge<G, 8>(a, sl, slot_floats, nsplits, rows, q0 + t0, kh);
  if (tid == 0)
    __hip_atomic_store(group_counter(a.ws, grp), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Prefill unit of at most 32 query rows: the launches too small to fill the
// chip, which last as long as their longest unit takes from its first load to
// its store.  One wavefront's accumulators hold all rows, so the four
// wavefronts split the keys: wavefront w takes 32-key blocks w, w + 4, ... of
// the unit, each through one key slot and one value slot of its own (a slot is
// refilled as soon as its reads have returned), without a barrier until the
// four partial results are added through LDS.  A unit then takes 6.1 us and
// 6.4 us per 1024 keys (the 128-row code with one of its wavefronts at work:
// 10 us and 14 us), and new tokens are read where the caller put them, which
// takes the append and the wait for it (4.7 us) off the path.  20 new tokens
// and one decoder, g = 2: 9.5 -> 6.0 us; 128 tokens over 1000 cached, prefill
// alone: 18.7 -> 13.9 us; with 4 decoders over 384 cached: 17.2 -> 9.5 us.
template <int G, bool APP>
__device__ void prefill_small(const Args& a, record_t f, char* smem, int* flag) {
  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  const int col = lane & 31, hi = lane >> 5;
  const int s = f[DLFP_W_SEQ], kh = f[DLFP_W_KVHEAD];
  const int t0 = f[DLFP_W_QTOK0], nt = f[DLFP_W_QNTOK];
  const int kb = f[DLFP_W_KVBEGIN], ke = f[DLFP_W_KVEND];
  const int nsplits = f[DLFP_W_NSPLITS], grp = f[DLFP_W_GROUP];
  const int wsgroup = f[DLFP_W_WSGROUP], split = f[DLFP_W_SPLIT];
  const int row0 = f[DLFP_W_QROW0], first_pos = f[DLFP_W_QPOS0];
  const int32_t* bt = a.block_table + (int64_t)s * a.max_blocks;

  const int tr = col / G, hh = col % G;
  const bool row_ok = tr < nt;
  const int lim = row_ok ? min(first_pos + tr + 1, ke) : 0;  // keys < lim are visible
  const int lim_min = min(first_pos + 1, ke);

  const int first_page = kb / PAGE, last_page = (ke - 1) / PAGE;
  const int blocks = (ke - kb + SMALL_KEYS - 1) / SMALL_KEYS;
  const int mine = blocks > wave ? (blocks - wave + 3) / 4 : 0;
  // This wavefront's page h of its block i; past the unit's last page, that page.
  auto page_index = [&](int i, int h) { return min(2 * (wave + 4 * i) + h, last_page - first_page); };

  char* wl = smem + wave * SMALL_WAVE_LDS;
  int32_t* ptab = reinterpret_cast<int32_t*>(wl + 2 * SMALL_SLOT);
  bf16x8_t qf[8];
  {
    const int64_t qrow = ((int64_t)(row0 + (row_ok ? tr : 0)) * a.hq + kh * G + hh) * D;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      qf[kk] = *reinterpret_cast<const bf16x8_t*>(a.q + qrow + 16 * kk + 8 * hi);
  }
  // Block ids of this wavefront's pages, two per block.
  for (int x = lane; x < 2 * mine; x += 64) ptab[x] = bt[first_page + page_index(x >> 1, x & 1)];
  wait_memory_complete();
  wave_sync();

  uint32_t koff[4], voff[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int rr = 4 * i + (lane >> 4);
    koff[i] = rr * 256 + (((lane & 15) ^ rr) << 4);
    const int d = 32 * i + (lane >> 1);
    voff[i] = d * 32 + (((lane & 1) ^ vt_swz(d)) << 4);
  }
  const uint32_t lds_wave = (uint32_t)uniform((int)lds_addr(wl));
  // Element offset of a page (same in both caches).
  auto page_off = [&](int raw) -> int64_t {
    const bool ok = (unsigned)raw < (unsigned)a.num_blocks;
    if (!ok && lane == 0) raise_error(a.ws);
    return ((int64_t)(ok ? raw : 0) * a.hkv + kh) * PAGE_ELEMS;
  };
  auto issue = [&](const uint16_t* cache, const uint32_t* off, int64_t p0, int64_t p1, uint32_t dst) {
    const char* s0 = reinterpret_cast<const char*>(cache + p0);
    const char* s1 = reinterpret_cast<const char*>(cache + p1);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds_copy16(s0 + off[i], dst + i * 1024);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds_copy16(s1 + off[i], dst + (4 + i) * 1024);
  };

  // Blocks that hold new tokens are "fresh" and come first, then the old ones
  // (the same order whether the tokens are in the cache or not).  In an append
  // launch every unit is small and takes new tokens from k_new and v_new, so
  // none waits for the append records.
  const int pos0 = first_pos - t0;
  const bool direct = APP && a.app_wgs > 0;
  const int fresh_block = max(0, (pos0 - kb) / SMALL_KEYS);  // the block holding position pos0
  const int old = min(mine, fresh_block > wave ? (fresh_block - wave + 3) / 4 : 0);
  auto first_key = [&](int i) { return kb + (wave + 4 * i) * SMALL_KEYS; };
  // Block of step j of the loop over cached blocks.
  const int steps = direct ? old : mine;
  auto block_of = [&](int j) { return direct ? j : j + old < mine ? j + old : j + old - mine; };
  const int kbase = col * 256 + ((hi ^ (col & 15)) << 4);
  const int vbase = SMALL_SLOT + col * 32 + ((hi ^ vt_swz(col)) << 4);
  const float c = a.scale_log2;
  float m_run = NEG_BIG, l_run = 0.f;
  f32x16_t o[4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb) o[mb] = f32x16_t{};

  // Scores of a block's keys into probabilities, then O^T += V^T P^T over the
  // value slot.
  bf16x8_t pf[2];
  auto softmax = [&](f32x16_t sacc, int k0) {
    if (k0 + SMALL_KEYS > lim_min) {
#pragma unroll
      for (int rr = 0; rr < 16; ++rr)
        sacc[rr] = k0 + 8 * (rr >> 2) + 4 * hi + (rr & 3) < lim ? sacc[rr] : -__builtin_inff();
    }
    float mx = -__builtin_inff();
#pragma unroll
    for (int rr = 0; rr < 16; ++rr) mx = fmaxf(mx, sacc[rr]);
    const float m_tile = max_xor32(mx) * c;
    if (__builtin_amdgcn_ballot_w64(m_tile > m_run + RESCALE_LOG2)) {
      const float m_new = m_tile > m_run + RESCALE_LOG2 ? m_tile : m_run;
      const float alpha = fexp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) o[mb] *= alpha;
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      u32x4_t pk;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const float p0 = fexp2(__builtin_fmaf(sacc[8 * kk + 2 * w], c, -m_run));
        const float p1 = fexp2(__builtin_fmaf(sacc[8 * kk + 2 * w + 1], c, -m_run));
        pk[w] = pack_bf16(p0, p1);
        l_run = dot2(pk[w], 0x3F803F80u, l_run);  // two bf16 1.0
      }
      pf[kk] = __builtin_bit_cast(bf16x8_t, pk);
    }
  };
  auto pv = [&]() {
    bf16x8_t vf[8];
#pragma unroll
    for (int x = 0; x < 8; ++x)
      vf[x] = *reinterpret_cast<const bf16x8_t*>(wl + vbase + (x >> 2) * (PAGE * 256) +
                                                 (x & 3) * 1024);
#pragma unroll
    for (int x = 0; x < 8; ++x)
      o[x & 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[x], pf[x >> 2], o[x & 3], 0, 0, 0);
    wait_lds();  // the value slot is free
  };

  int64_t p0 = 0, p1 = 0;  // page offsets of the block going out
  if (steps > 0) {
    const int i = block_of(0);
    p0 = page_off(uniform(ptab[2 * i]));
    p1 = page_off(uniform(ptab[2 * i + 1]));
    issue(a.kc, koff, p0, p1, lds_wave);
  }
  // Fresh blocks first, while the first old one's keys are in flight: the key
  // operand straight from its rows (of the cache or, from position pos0 on, of
  // k_new; keys past the unit's last re-read that one and are masked), the
  // values of dims 2 lane and 2 lane + 1 gathered from v_new (or from their
  // page) and packed into the value slot.
  for (int i = direct ? old : mine; i < mine; ++i) {
    const int k0 = first_key(i);
    const int64_t f0 = page_off(uniform(ptab[2 * i])), f1 = page_off(uniform(ptab[2 * i + 1]));
    // Row of the sequence's first new token in k_new and v_new, this KV head.
    const int64_t new0 = ((int64_t)(row0 - t0) * a.hkv + kh) * D, stride = (int64_t)a.hkv * D;
    const int key = min(k0 + col, ke - 1);
    const uint16_t* krow = key < pos0 ? a.kc + (col < PAGE ? f0 : f1) + (col % PAGE) * D
                                      : a.k_new + new0 + (key - pos0) * stride;
    bf16x8_t kf[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      kf[kk] = *reinterpret_cast<const bf16x8_t*>(krow + 16 * kk + 8 * hi);
    uint32_t x[2][PAGE];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int t = 0; t < PAGE; ++t)
        x[h][t] = *reinterpret_cast<const uint32_t*>(
            a.v_new + new0 + (min(max(k0 + PAGE * h + t, pos0), ke - 1) - pos0) * stride + 2 * lane);
    f32x16_t sacc = f32x16_t{};
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], sacc, 0, 0, 0);
    softmax(sacc, k0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int key0 = k0 + PAGE * h;
      if (key0 < pos0) {  // the page's first tokens are old ones
        const u32x4_t* row =
            reinterpret_cast<const u32x4_t*>(a.vc + (h ? f1 : f0) + (2 * lane) * PAGE);
        const u32x4_t w0[2] = {row[0], row[1]}, w1[2] = {row[2], row[3]};
#pragma unroll
        for (int t = 0; t < PAGE; ++t) {
          const int sp = vt_pos(t);
          const uint32_t lo = w0[sp >> 3][(sp & 7) >> 1], up = w1[sp >> 3][(sp & 7) >> 1];
          const uint32_t was =
              (sp & 1) ? (lo >> 16) | (up & 0xFFFF0000u) : (lo & 0xFFFFu) | (up << 16);
          x[h][t] = key0 + t < pos0 ? was : x[h][t];
        }
      }
      char* vl = wl + SMALL_SLOT + h * (PAGE * 256);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        u32x4_t d0, d1;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int ta = vt_pos(8 * half + 2 * w), tb = vt_pos(8 * half + 2 * w + 1);
          const uint32_t xa = key0 + ta < ke ? x[h][ta] : 0u, xb = key0 + tb < ke ? x[h][tb] : 0u;
          d0[w] = (xa & 0xFFFFu) | (xb << 16);
          d1[w] = (xa >> 16) | (xb & 0xFFFF0000u);
        }
        const int d = 2 * lane;
        *reinterpret_cast<u32x4_t*>(vl + d * 32 + ((half ^ vt_swz(d)) << 4)) = d0;
        *reinterpret_cast<u32x4_t*>(vl + (d + 1) * 32 + ((half ^ vt_swz(d + 1)) << 4)) = d1;
      }
    }
    wave_sync();
    pv();
  }

  if (steps > 0) issue(a.vc, voff, p0, p1, lds_wave + SMALL_SLOT);
  for (int j = 0; j < steps; ++j) {
    const int k0 = first_key(block_of(j));
    const bool more = j + 1 < steps;
    wait_copies<8>();  // in flight, oldest first: this block's keys, its values
    f32x16_t sacc = f32x16_t{};
    {
      bf16x8_t kf[8];
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        kf[kk] = *reinterpret_cast<const bf16x8_t*>(wl + (kbase ^ (kk << 5)));
#pragma unroll
      for (int kk = 0; kk < 8; ++kk)
        sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk], qf[kk], sacc, 0, 0, 0);
    }
    wait_lds();  // the key slot is free
    if (more) {
      const int i = block_of(j + 1);
      p0 = page_off(uniform(ptab[2 * i]));
      p1 = page_off(uniform(ptab[2 * i + 1]));
      issue(a.kc, koff, p0, p1, lds_wave);
    }
    softmax(sacc, k0);
    if (more)
      wait_copies<8>();  // the values; behind them the next block's keys
    else
      wait_copies<0>();
    if (k0 + SMALL_KEYS > ke) {
      // Values past the unit's last key are zeroed (a probability of 0 times a
      // NaN left in an unused slot would still be NaN).
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int pg = x >> 2, d = 2 * lane + ((x >> 1) & 1), h = x & 1;
        char* p = wl + SMALL_SLOT + pg * (PAGE * 256) + d * 32 + (h << 4);
        const int half = h ^ vt_swz(d), key0 = k0 + pg * PAGE;
        *reinterpret_cast<u32x4_t*>(p) =
            mask_elems(*reinterpret_cast<const u32x4_t*>(p), ke,
                       [&](int e) { return key0 + vt_pos(8 * half + e); });
      }
      wave_sync();
    }
    pv();
    if (more) issue(a.vc, voff, p0, p1, lds_wave + SMALL_SLOT);
  }

  // Add the four wavefronts' results through LDS.  Piece (c, hi) of a row holds
  // dims 32 (c / 4) + 8 (c % 4) + 4 hi .. + 3; thread (row, sub) of the sum takes
  // chunks 2 sub and 2 sub + 1, 16 consecutive dims; the row is XORed with the
  // chunk so that both sides spread over the banks.
  l_run = sum_xor32(l_run);
  __syncthreads();  // every wavefront is done with its slots
  f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);
  float* stat = reinterpret_cast<float*>(smem + 4 * 1024 * 16);  // m[4][32], l[4][32]
  auto at = [](int w, int ch, int h, int row) {
    return w * 1024 + ch * 64 + h * 32 + (row ^ (((ch >> 1) & 7) << 1));
  };
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4)
      red[at(wave, 4 * mb + g4, hi, col)] = f32x4_t{o[mb][4 * g4], o[mb][4 * g4 + 1],
                                                   o[mb][4 * g4 + 2], o[mb][4 * g4 + 3]};
  if (hi == 0) {
    stat[wave * 32 + col] = m_run;
    stat[128 + wave * 32 + col] = l_run;
  }
  __syncthreads();
  const int row = tid >> 3, sub = tid & 7, rows = nt * G;
  float M = NEG_BIG, L = 0.f, wgt[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) M = fmaxf(M, stat[w * 32 + row]);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    wgt[w] = fexp2(stat[w * 32 + row] - M);
    L += wgt[w] * stat[128 + w * 32 + row];
  }
  f32x4_t acc[4];  // pieces (2 sub, 0), (2 sub, 1), (2 sub + 1, 0), (2 sub + 1, 1)
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    acc[x] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) acc[x] += wgt[w] * red[at(w, 2 * sub + (x >> 1), x & 1, row)];
  }
  if (nsplits == 1) {
    if (row < rows) {
      const float inv = 1.f / L;
      const int64_t orow = ((int64_t)(row0 + row / G) * a.hq + kh * G + row % G) * D + 16 * sub;
#pragma unroll
      for (int x = 0; x < 4; ++x)
        store4(a, orow + 4 * x, acc[x][0] * inv, acc[x][1] * inv, acc[x][2] * inv, acc[x][3] * inv);
    }
    return;
  }
  const int slot_floats = slot_floats_for(rows);
  const Slots sl = group_slots(a.ws, wsgroup, nsplits, slot_floats);
  const int my = split * slot_floats;
  if (row < rows) {
#pragma unroll
    for (int x = 0; x < 4; ++x)
      pstore4(sl, my + ((2 * sub + (x >> 1)) * rows + row) * 8 + 4 * (x & 1), acc[x]);
    if (sub == 0) {
      pstore1(sl, my + rows * D + row, M);
      pstore1(sl, my + rows * D + rows + row, L);
    }
  }
  wait_memory_complete();
  __syncthreads();  // every wave of the unit has completed its stores
  if (tid == 0) *flag = arrive(a.ws, grp) == nsplits - 1;
  __syncthreads();
  if (!*flag) return;
  prefill_merge<G, 8>(a, sl, slot_floats, nsplits, rows, row0, kh);
  if (tid == 0)
    __hip_atomic_store(group_counter(a.ws, grp), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Last arriver of a decode split group: merges the group's partial results
// (O[G][128], m[G], l[G] per split, in split order) into the output.  Lane
// `lane` writes dims 2 lane and 2 lane + 1 of every head; obase is the
// element offset of those dims of the group's first head.
template <int G>
__device__ __forceinline__ void decode_merge(const Args& a, const Slots sl, int slot_floats,
                                             int nsplits, int64_t obase, int grp) {
  const int lane = threadIdx.x & 63;
  // Entry f = j G + h stands for head h of split j.  Per batch
  // of up to 64 entries, lane e loads entry e's maximum and row sum while
  // every lane loads its two dims of the batch's entries (in groups of 16,
  // only as many groups as the batch has entries), so a batch costs one
  // memory round trip; the running per-head maximum rescales what earlier
  // batches summed, and entries are accumulated in split order.
  const int nf = nsplits * G;
  float M[G], lsum[G], acc0[G], acc1[G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    M[h] = NEG_BIG;
    lsum[h] = acc0[h] = acc1[h] = 0.f;
  }
  for (int f0 = 0; f0 < nf; f0 += 64) {
    const int n = min(64, nf - f0);
    const int fl = f0 + lane;
    const int lbase = (fl / G) * slot_floats + G * D + fl % G;
    const float mf = lane < n ? pload1(sl, lbase) : NEG_BIG;
    const float lf = pload1(sl, lbase + G);
    f32x2_t v[4][16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (16 * q < n) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int fe = f0 + 16 * q + e;
          v[q][e] = pload2(sl, (fe / G) * slot_floats + (fe % G) * D + 2 * lane);
        }
      }
    }
    // Batch maximum of head lane % G (f0 is a multiple of 64, so entry
    // f0 + e belongs to head e % G).
    float bm = mf;
#pragma unroll
    for (int sh = G; sh < 64; sh <<= 1) bm = fmaxf(bm, shfl_xor(bm, sh));
    float mh = NEG_BIG;
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float mnew = fmaxf(M[h], __builtin_bit_cast(float, __builtin_amdgcn_readlane(
                                                                  __builtin_bit_cast(int, bm), h)));
      const float rs = fexp2(M[h] - mnew);
      M[h] = mnew;
      lsum[h] *= rs;
      acc0[h] *= rs;
      acc1[h] *= rs;
      if (lane % G == h) mh = mnew;
    }
    const float wf = lane < n ? fexp2(mf - mh) : 0.f;
    const float wl = wf * lf;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (16 * q < n) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int src = 16 * q + e;  // weights of entries past the batch are zero
          const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(
                                                        __builtin_bit_cast(int, wf), src));
          const float lw = __builtin_bit_cast(float, __builtin_amdgcn_readlane(
                                                         __builtin_bit_cast(int, wl), src));
          lsum[e % G] += lw;
          acc0[e % G] += w * v[q][e][0];
          acc1[e % G] += w * v[q][e][1];
        }
      }
    }
  }
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float inv = 1.f / lsum[h];
    store2(a, obase + h * D, acc0[h] * inv, acc1[h] * inv);
  }
  if (lane == 0)
    __hip_atomic_store(group_counter(a.ws, grp), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- decode

typedef short s16x4_t __attribute__((ext_vector_type(4)));

// Decode unit of a wavefront (in a launch whose decode workgroups drain a
// queue).  The unit's g heads are the columns of 16x16 matrix
// products (twice, 8 apart, with TWO; the others have zero queries): per page,
// the scores are S^T = K Q^T (four v_mfma_f32_16x16x32_bf16 over the 128
// dims) and the output advances by O^T += V^T P^T (eight
// v_mfma_f32_16x16x16_bf16 over the page's 16 keys), so the VALU only forms
// the softmax.  Lane l owns column l % 16 and accumulator rows
// 4 (l / 16) .. + 3.  Row r of the K operand (and so of S^T) is token slot
// vt_pos(r) of the page: a lane's four rows are then four consecutive
// positions of a value-page row (the cache keeps V^T pages with slot t at
// position vt_pos(t)), so the probabilities go from the score accumulator
// straight into the B operand of the PV product, and a lane's V^T operand is
// one 8-byte LDS read.  Per-head maxima combine the four lane groups with
// permlane swaps; the reference maximum is raised lazily, as in the prefill
// tiles.
//
// Wave-private LDS slice: two page slots, each a K page (row R keeps its
// 16-byte chunk x at position x ^ R) and a V^T page (32-byte row d keeps its
// two halves swapped when bit 3 of d is set; either way the lanes that LDS
// serves together read distinct banks), then the unit's block ids.  Pages
// reach a slot by direct global-to-LDS copies (no registers, no staging
// writes).  Asked for two pages in flight, page p + 2 is issued as soon as page
// p has been consumed; otherwise page p + 1 when page p has landed: a deeper
// queue makes the prefill tiles wait longer for their loads (measured 3.6-5.5%
// longer iterations for chunks of 64-256 tokens).  A block id outside the pool
// is replaced by block 0 after raising the error word.
// Returns the next queue ticket's pending value when asked to take one (see
// the kernel's decode loop): the ticket is taken a few pages before the unit
// ends, so that its round trip overlaps the unit's last pages.
template <int G, bool APP, bool TWO>
__device__ int decode_unit(const Args& a, const int32_t* it_g, char* wl, bool take_ticket) {
  static_assert(G >= 1 && G <= 8, "heads must fit half of the 16 columns");
  const int lane = threadIdx.x & 63;
  const int col = lane & 15, gq = lane >> 4, head = TWO ? col & 7 : col;
  const record_ptr it = as_record(it_g);
  const int s = it[DLFP_W_SEQ], kh = it[DLFP_W_KVHEAD];
  const int kb = it[DLFP_W_KVBEGIN], ke = it[DLFP_W_KVEND];
  const int nsplits = it[DLFP_W_NSPLITS];
  const int tok = it[DLFP_W_QROW0];
  const int newpos = it[DLFP_W_QPOS0];
  const int first_blk = it[DLFP_W_PAGE0], second_blk = it[DLFP_W_PAGE1];
  const int grp = it[DLFP_W_GROUP], wsgroup = it[DLFP_W_WSGROUP], split = it[DLFP_W_SPLIT];
  const int32_t* bt = a.block_table + (int64_t)s * a.max_blocks;
  int32_t* ptab = reinterpret_cast<int32_t*>(wl + 2 * DEC_PAGE_SLOT);

  const bool deep = a.deep != 0;
  const int p_begin = kb / PAGE, p_end = (ke + PAGE - 1) / PAGE;
  const int npages = p_end - p_begin;
  uint32_t kofs[4], vofs[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ck = 64 * j + lane;  // LDS chunk this lane fills
    const int R = ck >> 4, xs = ck & 15;
    kofs[j] = R * 256 + ((xs ^ R) << 4);
    const int d = ck >> 1, hs = ck & 1;
    vofs[j] = d * 32 + ((hs ^ ((d >> 3) & 1)) << 4);
  }
  const uint32_t lds_wave = (uint32_t)uniform((int)lds_addr(wl));
  auto issue_block = [&](int raw, int slot) {
    const bool ok = (unsigned)raw < (unsigned)a.num_blocks;
    if (!ok && lane == 0) raise_error(a.ws);
    const int64_t base = ((int64_t)(ok ? raw : 0) * a.hkv + kh) * PAGE_ELEMS;
    const char* ksrc = reinterpret_cast<const char*>(a.kc + base);
    const char* vsrc = reinterpret_cast<const char*>(a.vc + base);
    const uint32_t dst = lds_wave + uniform(slot) * DEC_PAGE_SLOT;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      lds_copy16_nt(ksrc + kofs[j], dst + j * 1024);
      lds_copy16_nt(vsrc + vofs[j], dst + PAGE_ELEMS * 2 + j * 1024);
    }
  };
  auto issue = [&](int p, int slot) { issue_block(uniform(ptab[p - p_begin]), slot); };
  auto wait_page = [&](bool next_in_flight) {
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    if (next_in_flight)
      __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt(8)
    else
      __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
  };

  // Prologue (one round trip after the work record): the first page, the
  // queries as the B operand (lane holds dims 32 kk + 8 (l / 16) .. + 8 of head
  // column l % 16 (l % 8 with TWO), zero past the unit's g heads), the unit's block ids and
  // (append launches) the new token's key row and value pair.
  issue_block(first_blk, 0);
  bf16x8_t qb[4];
  {
    const uint16_t* qp = a.q + ((int64_t)tok * a.hq + kh * G + min(head, G - 1)) * D + 8 * gq;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(qp + 32 * kk);
      qb[kk] = __builtin_bit_cast(bf16x8_t, head < G ? v : u32x4_t{0u, 0u, 0u, 0u});
    }
  }
  constexpr int PTV = DEC_PTAB / 64;
  int ptv[PTV];
#pragma unroll
  for (int k = 0; k < PTV; ++k) {
    const int i = lane + 64 * k;
    ptv[k] = i < npages ? bt[p_begin + i] : 0;
  }
  const bool own_new = APP && newpos < ke;
  const int new_page = newpos / PAGE, new_off = newpos % PAGE;
  u32x4_t kn = {0u, 0u, 0u, 0u};
  uint32_t vn = 0u;
  if (own_new) {
    const int64_t src = ((int64_t)tok * a.hkv + kh) * D;
    if (lane < 16) kn = *reinterpret_cast<const u32x4_t*>(a.k_new + src + 8 * lane);
    vn = *reinterpret_cast<const uint32_t*>(a.v_new + src + 2 * lane);
  }
  if (deep && npages > 1) issue_block(second_blk, 1);
  wait_memory_complete();
#pragma unroll
  for (int k = 0; k < PTV; ++k)
    if (lane + 64 * k < npages) ptab[lane + 64 * k] = ptv[k];
  wave_sync();
  if (own_new) {
    const int raw = ptab[new_page - p_begin];
    if ((unsigned)raw < (unsigned)a.num_blocks) {
      const int64_t base = ((int64_t)raw * a.hkv + kh) * PAGE_ELEMS;
      uint16_t* kc = const_cast<uint16_t*>(a.kc);
      uint16_t* vc = const_cast<uint16_t*>(a.vc);
      if (lane < 16) *reinterpret_cast<u32x4_t*>(kc + base + new_off * D + 8 * lane) = kn;
      vc[base + (2 * lane) * PAGE + vt_pos(new_off)] = (uint16_t)(vn & 0xFFFFu);
      vc[base + (2 * lane + 1) * PAGE + vt_pos(new_off)] = (uint16_t)(vn >> 16);
    }
  }

  float m_run = NEG_BIG, l_run = 0.f;
  f32x4_t o[8];
#pragma unroll
  for (int mb = 0; mb < 8; ++mb) o[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const float c = a.scale_log2;
  int ticket_v = 0;
  const int ticket_page = max(p_begin, p_end - 4);
  // This lane's K operand row (token slot vt_pos(col)), the token slot of its
  // first accumulator row (vt_pos(4 gq)), and its V^T operand's byte offset
  // inside a 16-row block (row col, positions 4 gq .. + 3).
  const int ra = vt_pos(col);
  const int slot0 = vt_pos(4 * gq);
  const int vbyte = col * 32 + (((gq >> 1) ^ ((col >> 3) & 1)) << 4) + 8 * (gq & 1);

  auto process = [&](int p, int slot) {
    char* kl = wl + slot * DEC_PAGE_SLOT;
    char* vl = kl + PAGE_ELEMS * 2;
    wait_page(deep && p + 1 < p_end);
    wave_sync();
    if (!deep && p + 1 < p_end) issue(p + 1, slot ^ 1);  // that slot was consumed
    if (take_ticket && p == ticket_page && lane == 0)
      ticket_v = __hip_atomic_fetch_add(header_word(a.ws, HDR_TICKET), 1, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
    if (p * PAGE + PAGE > ke) {
      // Values past the unit's last key are zeroed (a probability of 0 times
      // a NaN left in an unused slot would still be NaN).
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int ck = 64 * j + lane;
        const int d = ck >> 1, h = (ck & 1) ^ ((d >> 3) & 1);
        u32x4_t* v = reinterpret_cast<u32x4_t*>(vl + ck * 16);
        *v = mask_elems(*v, ke, [&](int e) { return p * PAGE + vt_pos(8 * h + e); });
      }
    }
    if (own_new && p == new_page) {
      if (lane < 16)
        *reinterpret_cast<u32x4_t*>(kl + new_off * 256 + ((lane ^ new_off) << 4)) = kn;
      const int sp = vt_pos(new_off), half = sp >> 3;
      const int d0 = 2 * lane, d1 = 2 * lane + 1;
      *reinterpret_cast<uint16_t*>(vl + d0 * 32 + ((half ^ ((d0 >> 3) & 1)) << 4) + 2 * (sp & 7)) =
          (uint16_t)(vn & 0xFFFFu);
      *reinterpret_cast<uint16_t*>(vl + d1 * 32 + ((half ^ ((d1 >> 3) & 1)) << 4) + 2 * (sp & 7)) =
          (uint16_t)(vn >> 16);
    }
    wave_sync();  // fixed-up page visible to every lane

    // S^T = K Q^T: rows = token slots vt_pos(r), columns = heads.
    f32x4_t sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const bf16x8_t kf =
          *reinterpret_cast<const bf16x8_t*>(kl + ra * 256 + (((4 * kk + gq) ^ ra) << 4));
      sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qb[kk], sacc, 0, 0, 0);
    }
    // Rows 4 gq + i hold slots slot0 + i; keys at or past ke are masked.
    float sc[4];
    float mx = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      sc[i] = p * PAGE + slot0 + i < ke ? sacc[i] : -__builtin_inff();
      mx = fmaxf(mx, sc[i]);
    }
    mx = max_xor32(max_xor16(mx));
    const float m_tile = mx * c;
    if (__builtin_amdgcn_ballot_w64(m_tile > m_run + RESCALE_LOG2)) {
      const float m_new = m_tile > m_run + RESCALE_LOG2 ? m_tile : m_run;
      const float alpha = fexp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) o[mb] *= alpha;
    }
    // P^T: this lane's keys of its column, its term of each, the B operand.
    u32x2_t pk;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const float e0 = fexp2(__builtin_fmaf(sc[2 * w], c, -m_run));
      const float e1 = fexp2(__builtin_fmaf(sc[2 * w + 1], c, -m_run));
      pk[w] = TWO ? pack_term(e0, e1, col >= 8) : pack_bf16(e0, e1);
      l_run = dot2(pk[w], 0x3F803F80u, l_run);  // two bf16 1.0
    }
    const s16x4_t pb = __builtin_bit_cast(s16x4_t, pk);
    // O^T += V^T P^T, eight blocks of 16 dims.
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) {
      const s16x4_t vf = *reinterpret_cast<const s16x4_t*>(vl + mb * 512 + vbyte);
      o[mb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vf, pb, o[mb], 0, 0, 0);
    }
    wave_sync();  // every lane done reading the slot before it is refilled
    if (deep && p + 2 < p_end) issue(p + 2, slot);
  };

  for (int p = p_begin; p < p_end; p += 2) {
    process(p, 0);
    if (p + 1 < p_end) process(p + 1, 1);
  }

  // Row sums: each lane group holds a quarter of the keys of its head (the two
  // columns of a head a term each).
  float l_tot = sum_xor32(sum_xor16(l_run));
  if constexpr (TWO) {
    l_tot = sum_xor8(l_tot);
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[mb][i] = sum_xor8(o[mb][i]);
  }
  // o[mb][i] = O[head col][16 mb + 4 gq + i]
  if (nsplits == 1) {
    if (col < G) {
      const float inv = 1.f / l_tot;
      const int64_t orow = ((int64_t)tok * a.hq + kh * G + col) * D + 4 * gq;
#pragma unroll
      for (int mb = 0; mb < 8; ++mb)
        store4(a, orow + 16 * mb, o[mb][0] * inv, o[mb][1] * inv, o[mb][2] * inv,
               o[mb][3] * inv);
    }
    return ticket_v;
  }

  // Partial: O[G][128], m[G], l[G].
  const int slot_floats = slot_floats_for(G);
  const Slots sl = group_slots(a.ws, wsgroup, nsplits, slot_floats);
  const int my = split * slot_floats;
  if (col < G) {
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) pstore4(sl, my + col * D + 16 * mb + 4 * gq, o[mb]);
    if (gq == 0) {
      pstore1(sl, my + G * D + col, m_run);
      pstore1(sl, my + G * D + G + col, l_tot);
    }
  }
  wait_memory_complete();
  int old = 0;
  if (lane == 0) old = arrive(a.ws, grp);
  old = __shfl(old, 0);
  if (old != nsplits - 1) return ticket_v;
  decode_merge<G>(a, sl, slot_floats, nsplits, ((int64_t)tok * a.hq + kh * G) * D + 2 * lane,
                  grp);
  return ticket_v;
}

// Decode unit of a whole workgroup ("wide").  Wavefront w takes the unit's
// 32-key blocks (two pages) w, w + NW, ..., so all finish together and the unit's
// partial results meet in LDS; only the parts of a range that the split policy
// cut (it weighs parts from 192 keys on) are merged across workgroups, by the
// last of them to finish.  Against one unit per wavefront (each of the four then merged
// through device memory, 2-5 us) decode-only launches take: 4 sequences of
// 64-256 keys 10.2 -> 5.7 us, one of 8000 keys (g = 4) 26.0 -> 13 us, 100 of
// 300-2400 keys 115.8 -> 93 us, 256 of 2048-16384 keys (g = 8) 1567 -> 1490 us.
//
// The unit's g heads are the columns of 16x16 matrix products (twice, 8 apart,
// with TWO; the others have zero queries).  Per block the scores are S^T = K Q^T (two independent
// chains of four v_mfma_f32_16x16x32_bf16 over the 128 dims) and the output
// advances by O^T += V^T P^T (eight of them over the 32 keys), half the
// products, LDS reads and softmax steps per key of 16-key blocks.  Lane l owns
// column l % 16; its group q = l / 16 owns the eight keys at positions
// 8 (q / 2) .. + 7 of page q % 2 (position p of a page holds token slot
// vt_pos(p)).  Row r of the K operand of chain b is position
// 8 (r / 8) + 4 b + r % 4 of page r / 4 % 2: the accumulator rows 4 q .. + 3 of
// both chains are then exactly the group's keys, so the probabilities go from
// the score accumulators straight into the B operand, and its V^T operand is
// one 16-byte LDS read per 16 dims.
//
// Wave-private LDS slice: one key slot and one value slot of two pages each,
// then the ids of the wavefront's pages.  A slot is refilled with the next
// block as soon as its reads have returned, so its copies fly while the other
// half of the step runs; four wavefronts then keep 64 KiB in flight, what a CU
// can have outstanding (measured: a workgroup of four wavefronts alone on its
// CU reads 67 GB/s, one of eight the same).  K row R of
// page h keeps its 16-byte chunk x at position x ^ R ^ 8 h; V^T row d (32 bytes)
// its two halves swapped when vt_swz(d): the lanes that LDS serves together
// read distinct banks.
template <int G, bool APP, int NW, bool TWO>
__device__ void decode_wide(const Args& a, const int32_t* it_g, char* smem, int* flag) {
  static_assert(G >= 1 && G <= 8 && G * 32 <= NW * 64, "heads");
  const int tid = threadIdx.x, wave = uniform(tid >> 6), lane = tid & 63;
  char* wl = smem + wave * WIDE_WAVE_LDS;
  const int col = lane & 15, gq = lane >> 4, head = TWO ? col & 7 : col;
  const record_ptr it = as_record(it_g);
  const int s = it[DLFP_W_SEQ], kh = it[DLFP_W_KVHEAD];
  const int kb = it[DLFP_W_KVBEGIN], ke = it[DLFP_W_KVEND];
  const int nsplits = it[DLFP_W_NSPLITS];
  const int tok = it[DLFP_W_QROW0];
  const int newpos = it[DLFP_W_QPOS0];
  const int grp = it[DLFP_W_GROUP], wsgroup = it[DLFP_W_WSGROUP], split = it[DLFP_W_SPLIT];
  const int32_t* bt = a.block_table + (int64_t)s * a.max_blocks;
  int32_t* ptab = reinterpret_cast<int32_t*>(wl + 2 * WIDE_SLOT);

  const int first_page = kb / PAGE;
  const int npages = (ke + PAGE - 1) / PAGE - first_page, nblocks = (npages + 1) >> 1;
  const int mine = nblocks > wave ? (nblocks - wave + NW - 1) / NW : 0;
  // Page h of this wavefront's block i (the unit's last page past its end);
  // whether the block has both pages.
  auto page_of = [&](int i, int h) { return min(2 * (wave + NW * i) + h, npages - 1); };
  auto has_both = [&](int i) { return 2 * (wave + NW * i) + 1 < npages; };

  uint32_t kofs[2][4], vofs[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int ck = 64 * j + lane;  // LDS chunk of a page this lane fills
    const int R = ck >> 4, xs = ck & 15;
    kofs[0][j] = R * 256 + ((xs ^ R) << 4);
    kofs[1][j] = R * 256 + ((xs ^ R ^ 8) << 4);
    const int d = ck >> 1, hs = ck & 1;
    vofs[j] = d * 32 + ((hs ^ vt_swz(d)) << 4);
  }
  const uint32_t lds_wave = (uint32_t)uniform((int)lds_addr(wl));
  // Element offset of a page (same in both caches); a block id outside the
  // pool is replaced by block 0 after raising the error word.
  auto page_off = [&](int raw) -> int64_t {
    const bool ok = (unsigned)raw < (unsigned)a.num_blocks;
    if (!ok && lane == 0) raise_error(a.ws);
    return ((int64_t)(ok ? raw : 0) * a.hkv + kh) * PAGE_ELEMS;
  };
  auto copy_page = [&](const uint16_t* page, const uint32_t* off, uint32_t dst) {
    const char* src = reinterpret_cast<const char*>(page);
#pragma unroll
    for (int j = 0; j < 4; ++j) lds_copy16_nt(src + off[j], dst + j * 1024);
  };
  // A last block of one page leaves the other half of its slots as it is (its
  // keys are masked, its values zeroed).
  auto issue_k = [&](int64_t p0, int64_t p1, bool both) {
    copy_page(a.kc + p0, kofs[0], lds_wave);
    if (both) copy_page(a.kc + p1, kofs[1], lds_wave + WIDE_SLOT / 2);
  };
  auto issue_v = [&](int64_t p0, int64_t p1, bool both) {
    copy_page(a.vc + p0, vofs, lds_wave + WIDE_SLOT);
    if (both) copy_page(a.vc + p1, vofs, lds_wave + WIDE_SLOT + WIDE_SLOT / 2);
  };
  // Prologue, after the work record: wavefront 0's first block (the ids of the
  // unit's first two pages come with the record).
  int64_t p0 = 0, p1 = 0;
  if (wave == 0) {
    p0 = page_off(it[DLFP_W_PAGE0]);
    p1 = npages > 1 ? page_off(it[DLFP_W_PAGE1]) : p0;
    issue_k(p0, p1, npages > 1);
    issue_v(p0, p1, npages > 1);
  }
  // With it go out the ids of the wavefront's pages, the queries as the B
  // operand (lane holds dims 32 kk + 8 gq .. + 7 of its head column, zero past
  // the g heads) and (append launches, the wavefront with the unit's last
  // block) the new token's key row (lanes 0-15, 16 bytes each) and its values of
  // dims 2 lane, 2 lane + 1.
  for (int x = lane; x < 2 * mine; x += 64) ptab[x] = bt[first_page + page_of(x >> 1, x & 1)];
  bf16x8_t qb[4];
  {
    const uint16_t* qp = a.q + ((int64_t)tok * a.hq + kh * G + min(head, G - 1)) * D + 8 * gq;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const u32x4_t v = *reinterpret_cast<const u32x4_t*>(qp + 32 * kk);
      qb[kk] = __builtin_bit_cast(bf16x8_t, head < G ? v : u32x4_t{0u, 0u, 0u, 0u});
    }
  }
  const bool own_new =
      APP && newpos < ke && mine > 0 && wave + NW * (mine - 1) == nblocks - 1;
  const int new_half = (newpos / PAGE - first_page) & 1, new_off = newpos % PAGE;
  u32x4_t kn = {0u, 0u, 0u, 0u};
  uint32_t vn = 0u;
  if (own_new) {
    const int64_t src = ((int64_t)tok * a.hkv + kh) * D;
    if (lane < 16) kn = *reinterpret_cast<const u32x4_t*>(a.k_new + src + 8 * lane);
    vn = *reinterpret_cast<const uint32_t*>(a.v_new + src + 2 * lane);
  }
  wait_memory_complete();
  wave_sync();

  if (wave != 0 && mine > 0) {
    p0 = page_off(uniform(ptab[0]));
    p1 = page_off(uniform(ptab[1]));
    issue_k(p0, p1, has_both(0));
    issue_v(p0, p1, has_both(0));
  }
  // The new token goes to its slot (and into the landed pages below).
  if (own_new) {
    const int raw = uniform(ptab[2 * (mine - 1) + new_half]);
    if ((unsigned)raw < (unsigned)a.num_blocks) {
      const int64_t base = ((int64_t)raw * a.hkv + kh) * PAGE_ELEMS;
      uint16_t* kc = const_cast<uint16_t*>(a.kc);
      uint16_t* vc = const_cast<uint16_t*>(a.vc);
      if (lane < 16) *reinterpret_cast<u32x4_t*>(kc + base + new_off * D + 8 * lane) = kn;
      vc[base + (2 * lane) * PAGE + vt_pos(new_off)] = (uint16_t)(vn & 0xFFFFu);
      vc[base + (2 * lane + 1) * PAGE + vt_pos(new_off)] = (uint16_t)(vn >> 16);
    }
  }

  float m_run = NEG_BIG, l_run = 0.f;
  f32x4_t o[8];
#pragma unroll
  for (int mb = 0; mb < 8; ++mb) o[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const float c = a.scale_log2;
  // This lane's K operand rows: page and slot of row `col` of each chain.
  const int kpage = (col >> 2) & 1;
  int krow[2], kxor[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int R = vt_pos(8 * (col >> 3) + 4 * b + (col & 3));
    krow[b] = kpage * (WIDE_SLOT / 2) + R * 256;
    kxor[b] = R ^ (kpage << 3);
  }
  // Accumulator row 4 gq + i of chain b is key key_of[b] + i of the block.
  const int key_of[2] = {16 * (gq & 1) + vt_pos(8 * (gq >> 1)),
                         16 * (gq & 1) + vt_pos(8 * (gq >> 1) + 4)};
  // V^T operand: row col of a 16-dim block, page gq % 2, half gq / 2.
  const int vbyte = WIDE_SLOT + (gq & 1) * (WIDE_SLOT / 2) + col * 32 +
                    (((gq >> 1) ^ vt_swz(col)) << 4);

  for (int i = 0; i < mine; ++i) {
    const int base = kb + 2 * PAGE * (wave + NW * i);  // first key of the block
    const bool more = i + 1 < mine, tail = base + 2 * PAGE > ke;
    // In flight, oldest first: this block's keys, its values (eight copies
    // each; a block of one page, only ever the last, has four).
    if (has_both(i))
      wait_copies<8>();
    else
      wait_copies<0>();
    if (own_new && !more) {
      if (lane < 16)
        *reinterpret_cast<u32x4_t*>(wl + new_half * (WIDE_SLOT / 2) + new_off * 256 +
                                    ((lane ^ new_off ^ (new_half << 3)) << 4)) = kn;
      wave_sync();
    }
    f32x4_t sacc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    {
      bf16x8_t kf[2][4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          kf[b][kk] = *reinterpret_cast<const bf16x8_t*>(wl + krow[b] +
                                                         (((4 * kk + gq) ^ kxor[b]) << 4));
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int b = 0; b < 2; ++b)
          sacc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[b][kk], qb[kk], sacc[b], 0, 0, 0);
    }
    wait_lds();  // the key slot is free
    const bool both = has_both(i + 1);
    if (more) {
      p0 = page_off(uniform(ptab[2 * i + 2]));
      p1 = page_off(uniform(ptab[2 * i + 3]));
      issue_k(p0, p1, both);
    }
    float sc[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) sc[x] = sacc[x >> 2][x & 3];
    if (tail) {
#pragma unroll
      for (int x = 0; x < 8; ++x)
        sc[x] = base + key_of[x >> 2] + (x & 3) < ke ? sc[x] : -__builtin_inff();
    }
    float mx = -__builtin_inff();
#pragma unroll
    for (int x = 0; x < 8; ++x) mx = fmaxf(mx, sc[x]);
    const float m_tile = max_xor32(max_xor16(mx)) * c;
    if (__builtin_amdgcn_ballot_w64(m_tile > m_run + RESCALE_LOG2)) {
      const float m_new = m_tile > m_run + RESCALE_LOG2 ? m_tile : m_run;
      const float alpha = fexp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < 8; ++mb) o[mb] *= alpha;
    }
    // P^T: this lane's keys of its column, its term of each, the B operand.
    u32x4_t pk;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float e0 = fexp2(__builtin_fmaf(sc[2 * w], c, -m_run));
      const float e1 = fexp2(__builtin_fmaf(sc[2 * w + 1], c, -m_run));
      pk[w] = TWO ? pack_term(e0, e1, col >= 8) : pack_bf16(e0, e1);
      l_run = dot2(pk[w], 0x3F803F80u, l_run);  // two bf16 1.0
    }
    const bf16x8_t pb = __builtin_bit_cast(bf16x8_t, pk);
    // The values; behind them the next block's keys may be in flight.
    if (more && both)
      wait_copies<8>();
    else
      wait_copies<0>();
    if (tail) {
      // Values past the unit's last key are zeroed (a probability of 0 times
      // a NaN left in an unused slot would still be NaN).
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int ck = 64 * (j & 3) + lane, d = ck >> 1, h = (ck & 1) ^ vt_swz(d);
        u32x4_t* v = reinterpret_cast<u32x4_t*>(wl + WIDE_SLOT + (j >> 2) * (WIDE_SLOT / 2) +
                                                ck * 16);
        *v = mask_elems(*v, ke,
                        [&](int e) { return base + PAGE * (j >> 2) + vt_pos(8 * h + e); });
      }
      wave_sync();
    }
    if (own_new && !more) {
      const int sp = vt_pos(new_off), half = sp >> 3, d0 = 2 * lane, d1 = 2 * lane + 1;
      char* vl = wl + WIDE_SLOT + new_half * (WIDE_SLOT / 2) + 2 * (sp & 7);
      *reinterpret_cast<uint16_t*>(vl + d0 * 32 + ((half ^ vt_swz(d0)) << 4)) =
          (uint16_t)(vn & 0xFFFFu);
      *reinterpret_cast<uint16_t*>(vl + d1 * 32 + ((half ^ vt_swz(d1)) << 4)) =
          (uint16_t)(vn >> 16);
      wave_sync();
    }
    // O^T += V^T P^T, eight blocks of 16 dims.
    {
      bf16x8_t vf[8];
#pragma unroll
      for (int mb = 0; mb < 8; ++mb)
        vf[mb] = *reinterpret_cast<const bf16x8_t*>(wl + vbyte + mb * 512);
#pragma unroll
      for (int mb = 0; mb < 8; ++mb)
        o[mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[mb], pb, o[mb], 0, 0, 0);
    }
    wait_lds();  // the value slot is free
    if (more) issue_v(p0, p1, both);
  }

  // Each lane group holds a quarter of its head's keys.  Then the wavefronts'
  // results are added through LDS: quad (head, 4 mb + gq) holds dims
  // 16 mb + 4 gq .. + 3 of the head, thread (h, q4) sums quad q4 of head h.
  // Two terms: the columns of a head are added before.
  float l_tot = sum_xor32(sum_xor16(l_run));
  if constexpr (TWO) {
    l_tot = sum_xor8(l_tot);
#pragma unroll
    for (int mb = 0; mb < 8; ++mb)
#pragma unroll
      for (int i = 0; i < 4; ++i) o[mb][i] = sum_xor8(o[mb][i]);
  }
  wait_memory_complete();
  __syncthreads();  // every wavefront is done with its slots
  f32x4_t* red = reinterpret_cast<f32x4_t*>(smem);
  float* stat = reinterpret_cast<float*>(smem + NW * G * 512);  // m[NW][G], l[NW][G]
  auto at = [](int w, int h, int q) { return (w * G + h) * 32 + (q ^ ((h & 7) << 2)); };
  if (col < G) {
#pragma unroll
    for (int mb = 0; mb < 8; ++mb) red[at(wave, col, 4 * mb + gq)] = o[mb];
    if (gq == 0) {
      stat[wave * G + col] = m_run;
      stat[NW * G + wave * G + col] = l_tot;
    }
  }
  __syncthreads();
  const int h = tid >> 5, q4 = tid & 31;
  const bool act = tid < G * 32;
  const int64_t out_elem = ((int64_t)tok * a.hq + kh * G + h) * D + 4 * q4;
  float M = NEG_BIG, L = 0.f;
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  if (act) {
#pragma unroll
    for (int w = 0; w < NW; ++w) M = fmaxf(M, stat[w * G + h]);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float e = fexp2(stat[w * G + h] - M);
      L += e * stat[NW * G + w * G + h];
      acc += e * red[at(w, h, q4)];
    }
    if (nsplits == 1) {
      const float inv = 1.f / L;
      store4(a, out_elem, acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
    }
  }
  if (nsplits == 1) return;

  // Partial: O[G][128], m[G], l[G]; the last arriver merges in split order.
  const int slot_floats = slot_floats_for(G);
  const Slots sl = group_slots(a.ws, wsgroup, nsplits, slot_floats);
  const int my = split * slot_floats;
  if (act) {
    pstore4(sl, my + h * D + 4 * q4, acc);
    if (q4 == 0) {
      pstore1(sl, my + G * D + h, M);
      pstore1(sl, my + G * D + G + h, L);
    }
  }
  wait_memory_complete();
  __syncthreads();  // every wave of the unit has completed its stores
  if (tid == 0) *flag = arrive(a.ws, grp) == nsplits - 1;
  __syncthreads();
  if (!*flag) return;
  if (act) {
    // Batches of NB splits: all loads of a batch go out before any is used.
    constexpr int NB = 16;
    M = NEG_BIG;
    L = 0.f;
    acc = f32x4_t{0.f, 0.f, 0.f, 0.f};
    for (int j = 0; j < nsplits; j += NB) {
      float mj[NB], lj[NB];
      f32x4_t x[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const int b = (j + u) * slot_floats;
        mj[u] = pload1(sl, b + G * D + h);
        lj[u] = pload1(sl, b + G * D + G + h);
        x[u] = pload4(sl, b + h * D + 4 * q4);
      }
      float mn = M;
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (j + u < nsplits) mn = fmaxf(mn, mj[u]);
      const float rs = fexp2(M - mn);
      M = mn;
      L *= rs;
      acc *= rs;
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const float e = j + u < nsplits ? fexp2(mj[u] - mn) : 0.f;
        L += e * lj[u];
        acc += e * x[u];
      }
    }
    const float inv = 1.f / L;
    store4(a, out_elem, acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv);
  }
  if (tid == 0)
    __hip_atomic_store(group_counter(a.ws, grp), 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------- append

// Append workgroup (append launches): each wavefront writes whole append
// records, one at a time -- one run of a prompt sequence's new tokens inside
// one page, for one KV head.  Key rows: lane covers 16-byte chunk lane % 16
// of rows 4 j + lane / 16.  Values: lane owns dims 2 lane and 2 lane + 1 and
// gathers them with one 4-byte load per token (a wavefront reads the whole
// 256-byte value row); a record that fills its page is written as whole
// 32-byte V^T rows, any other as one 2-byte value per token and dim (the
// page's other slots are left alone).  Every load of a record is issued
// before its stores.  The stores are ordinary ones, which the XCD's L2
// combines into whole lines (written through one by one, the half-line
// pieces cost a read-modify-write each at the memory side; measured 60-70 us
// for a 2048-token chunk).  When prefill units of the launch wait for the
// records, the workgroup then writes its L2 back (an agent-scope release) and
// counts itself done.

template <bool DIRECT>
__device__ void append_records(const Args& a) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint16_t* kc = const_cast<uint16_t*>(a.kc);
  uint16_t* vc = const_cast<uint16_t*>(a.vc);
  const int x16 = lane & 15;
  for (int r = blockIdx.x * 4 + wave; r < a.num_append; r += 4 * a.app_wgs) {
    const int32_t* it = a.work + (int64_t)(a.num_units + r) * DLFP_WORK_INTS;
    const int s = uniform(it[DLFP_W_SEQ]), kh = uniform(it[DLFP_W_KVHEAD]);
    const int n = uniform(it[DLFP_W_QNTOK]), row0 = uniform(it[DLFP_W_QROW0]);
    const int pos = uniform(it[DLFP_W_QPOS0]);
    const int o0 = pos % PAGE, o1 = o0 + n;
    const int raw = uniform(a.block_table[(int64_t)s * a.max_blocks + pos / PAGE]);
    if ((unsigned)raw >= (unsigned)a.num_blocks || o1 > PAGE) {
      if (lane == 0) raise_error(a.ws);
      continue;
    }
    const int64_t base = ((int64_t)raw * a.hkv + kh) * PAGE_ELEMS;
    // token row of slot o in k_new / v_new: row0 + o - o0
    const int64_t src0 = ((int64_t)(row0 - o0) * a.hkv + kh) * D;
    const int64_t tok_stride = (int64_t)a.hkv * D;
    u32x4_t kr[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = 4 * j + (lane >> 4);
      kr[j] = o >= o0 && o < o1
                  ? *reinterpret_cast<const u32x4_t*>(a.k_new + src0 + o * tok_stride + 8 * x16)
                  : u32x4_t{0u, 0u, 0u, 0u};
    }
    uint32_t x[PAGE];
#pragma unroll
    for (int o = 0; o < PAGE; ++o)
      x[o] = o >= o0 && o < o1
                 ? *reinterpret_cast<const uint32_t*>(a.v_new + src0 + o * tok_stride + 2 * lane)
                 : 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int o = 4 * j + (lane >> 4);
      if (o >= o0 && o < o1) *reinterpret_cast<u32x4_t*>(kc + base + o * D + 8 * x16) = kr[j];
    }
    uint16_t* row = vc + base + (2 * lane) * PAGE;  // rows 2 lane and 2 lane + 1
    if (o0 == 0 && o1 == PAGE) {
      // position 2 w + i of a row holds slot vt_pos(2 w + i)
      u32x4_t lo[2], hi[2];
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const uint32_t xa = x[vt_pos(2 * w)], xb = x[vt_pos(2 * w + 1)];
        lo[w >> 2][w & 3] = (xa & 0xFFFFu) | (xb << 16);
        hi[w >> 2][w & 3] = (xa >> 16) | (xb & 0xFFFF0000u);
      }
      u32x4_t* dst = reinterpret_cast<u32x4_t*>(row);
      dst[0] = lo[0];
      dst[1] = lo[1];
      dst[2] = hi[0];
      dst[3] = hi[1];
    } else {
#pragma unroll
      for (int o = 0; o < PAGE; ++o)
        if (o >= o0 && o < o1) {
          row[vt_pos(o)] = (uint16_t)(x[o] & 0xFFFFu);
          row[PAGE + vt_pos(o)] = (uint16_t)(x[o] >> 16);
        }
    }
  }
  if (a.num_waiting > 0 && !(DIRECT && a.work[DLFP_W_PAGE0])) {
    wait_memory_complete();  // this wavefront's stores have reached the L2
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // write the L2 back
      __hip_atomic_fetch_add(header_word(a.ws, HDR_APPEND), 1, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// The append records alone, as a launch of their own (one record per
// wavefront) ahead of the attention launch.
__global__ __launch_bounds__(THREADS) void append_records_kernel(Args a) {
  append_records<false>(a);
}

// ---------------------------------------------------------------- kernel

// Grid: `lead` prefill workgroups, `decode_lead` decode workgroups, the other
// prefill workgroups, the other decode workgroups.  The prefill unit of
// workgroup b (after the append workgroups), or -1 - d for decode workgroup d.
// The i-th prefill workgroup takes unit xcd_remap(i): decode_lead is a multiple
// of 8, so it runs on XCD i % 8 either way.
__device__ __forceinline__ int prefill_of(const Args& a, int b) {
  const int np = a.num_prefill, L = a.lead, DL = a.decode_lead;
  if (b < L) return xcd_remap(b, np);
  if (b < L + DL) return L - 1 - b;
  if (b < np + DL) return xcd_remap(b - DL, np);
  return np - 1 - b;
}

// Prefill units, and decode units of a workgroup each (DECODE).  Units of few
// rows (the records say so, for all units or none) take the code made for
// them; a record comes in whole, so the choice costs no round trip.
template <int G, bool APP, bool DECODE>
__global__ __launch_bounds__(THREADS, 2) void attention_wide_kernel(Args a) {
  __shared__ __attribute__((aligned(16))) char smem[LDS_BYTES];
  __shared__ int flag;
  int b = blockIdx.x;
  if constexpr (APP) {
    if (b < a.app_wgs) {
      append_records<true>(a);
      return;
    }
    b -= a.app_wgs;
  }
  const int u = prefill_of(a, b);
  if (u >= 0) {
    const int32_t* rec = a.work + (int64_t)u * DLFP_WORK_INTS;
    const record_t f = load_record(rec);
    if (f[DLFP_W_PAGE0])
      prefill_small<G, APP>(a, f, smem, &flag);
    else
      prefill_unit<G, APP, DECODE>(a, rec, f, smem, &flag);
  } else if constexpr (DECODE) {
    decode_wide<G, APP, 4, two_terms<G>(false)>(a, a.work + (int64_t)(a.num_prefill - 1 - u) * DLFP_WORK_INTS, smem,
                           &flag);
  }
}

// Decode workgroup d of a launch whose wavefronts drain a queue of decode units.
template <int G, bool APP, bool TWO>
__device__ __forceinline__ void decode_queue(const Args& a, int d, char* smem) {
  // Decode wavefront w of decode workgroup d starts with unit 4 d + w when
  // that is one of the first decode_static units (the workgroups resident
  // from the start); the other units form a queue that wavefronts drain one
  // ticket at a time as they finish, so none idles while units remain (a
  // workgroup's slot frees only when all four of its wavefronts are done),
  // and a workgroup that only becomes resident later takes tickets from the
  // start instead of holding units back to the tail.  The last workgroup to
  // finish resets the header words for the next launch.
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  char* wl = smem + wave * DEC_WAVE_LDS;
  const int ndec = a.num_units - a.num_prefill;
  const bool queue = ndec > a.decode_static;
  auto ticket = [&]() {
    int nt = 0;
    if (lane == 0)
      nt = a.decode_static + __hip_atomic_fetch_add(header_word(a.ws, HDR_TICKET), 1,
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return uniform(__shfl(nt, 0));
  };
  int t = d * 4 + wave;
  if (queue && t >= a.decode_static) t = ticket();
  while (t < ndec) {
    // In queue mode the unit takes the next ticket itself near its end.
    const int32_t* rec = a.work + (int64_t)(a.num_prefill + t) * DLFP_WORK_INTS;
    int pending;
    pending = decode_unit<G, APP, TWO>(a, rec, wl, queue);
    wave_sync();
    if (!queue) break;
    t = a.decode_static + uniform(__shfl(pending, 0));
  }
  if (queue) {
    __syncthreads();
    if (threadIdx.x == 0) {
      const int d = __hip_atomic_fetch_add(header_word(a.ws, HDR_DONE), 1, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
      if (d == a.decode_waves / 4 - 1) {
        __hip_atomic_store(header_word(a.ws, HDR_TICKET), 0, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(header_word(a.ws, HDR_DONE), 0, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
}

// Prefill units of any height beside wavefronts that drain a queue of decode
// units.
template <int G, bool APP>
__global__ __launch_bounds__(THREADS, 2) void attention_mixed_kernel(Args a) {
  __shared__ __attribute__((aligned(16))) char smem[LDS_BYTES];
  __shared__ int flag;
  int b = blockIdx.x;
  if constexpr (APP) {
    // Append workgroups first (a multiple of 8, so the XCD of every later
    // workgroup is unchanged by the offset).
    if (b < a.app_wgs) {
      append_records<false>(a);
      return;
    }
    b -= a.app_wgs;
  }
  const int u = prefill_of(a, b);
  if (u >= 0) {
    const int32_t* rec = a.work + (int64_t)u * DLFP_WORK_INTS;
    prefill_unit<G, APP, true>(a, rec, rec, smem, &flag);
  } else {
    decode_queue<G, APP, two_terms<G>(false)>(a, -1 - u, smem);
  }
}

// Launches of many short decode units alone.
template <int G, bool APP>
__global__ __launch_bounds__(THREADS, 2) void decode_queue_kernel(Args a) {
  __shared__ __attribute__((aligned(16))) char smem[4 * DEC_WAVE_LDS];
  decode_queue<G, APP, two_terms<G>(true)>(a, blockIdx.x, smem);
}

// Launches without prefill units, but for many short units: one wide decode unit
// per workgroup, longest first.
template <int G, bool APP, int NW>
__global__ __launch_bounds__(NW * 64, 2) void decode_kernel(Args a) {
  __shared__ __attribute__((aligned(16))) char smem[NW * WIDE_WAVE_LDS];
  __shared__ int flag;
  decode_wide<G, APP, NW, two_terms<G>(true)>(a, a.work + (int64_t)blockIdx.x * DLFP_WORK_INTS, smem, &flag);
}

// Workspace of dlfp_append_attention_mixed_static: a fixed array in device
// memory, one copy per GPU the library runs on, held until the process ends.
// Host code must not pass the array's name to a kernel (on the host it only
// stands for the symbol); static_workspace() below looks up its device address
// once per device.
__device__ __align__(256) char scratch[DLFP_STATIC_WORKSPACE_BYTES];

__global__ void fill_zero_kernel(int* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Compute units of the current device (queried once per device).
int compute_units() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cached[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

template <int G, bool APP>
hipError_t launch(const Args& a, int grid, hipStream_t stream) {
  if (a.num_prefill == 0 && a.wide == 4)
    decode_kernel<G, APP, 4><<<a.num_units, 4 * 64, 0, stream>>>(a);
  else if (a.num_prefill == 0 && a.wide == 8)
    decode_kernel<G, APP, 8><<<a.num_units, 8 * 64, 0, stream>>>(a);
  else if (a.num_prefill == 0)
    decode_queue_kernel<G, APP><<<grid, THREADS, 0, stream>>>(a);
  else if (a.num_units == a.num_prefill)
    attention_wide_kernel<G, APP, false><<<grid, THREADS, 0, stream>>>(a);
  else if (a.wide)
    attention_wide_kernel<G, APP, true><<<grid, THREADS, 0, stream>>>(a);
  else
    attention_mixed_kernel<G, APP><<<grid, THREADS, 0, stream>>>(a);
  return hipGetLastError();
}

template <int G>
hipError_t launch_g(const Args& a, int grid, bool app, hipStream_t stream) {
  return app ? launch<G, true>(a, grid, stream) : launch<G, false>(a, grid, stream);
}

// Validation, grid and launch shared by the entry points; `app` selects the
// fused append (k_new / v_new are ignored without it).  A batch without units
// returns DLFP_OK after its counts are checked, before any pointer is.
int launch_mixed(const dlfp_dims* dims, const dlfp_meta* meta, const int32_t* d_work,
                 const int32_t* d_block_table, int32_t max_blocks, int32_t num_blocks,
                 const void* q, bool app, const void* k_new, const void* v_new,
                 const void* k_cache,
                 const void* v_cache, float scale, void* out, int32_t out_dtype, void* workspace,
                 size_t workspace_bytes, hipStream_t stream) {
  int g = 0;
  const int st = dlfp::check_dims(dims, &g);
  if (st != DLFP_OK) return st;
  if (!meta) return DLFP_EINVAL;
  if (out_dtype != 0 && out_dtype != 1) return DLFP_EINVAL;
  if (!(scale > 0.f) || !(scale < 3.0e38f)) return DLFP_EINVAL;
  if (meta->num_units < 0 || meta->num_prefill_units < 0 ||
      meta->num_prefill_units > meta->num_units || meta->num_groups < 0)
    return DLFP_EINVAL;
  if (app && (meta->num_append < 0 || meta->num_waiting_units < 0 ||
              (meta->num_append > 0 && meta->num_waiting_units == 0) ||
              meta->num_waiting_units > meta->num_prefill_units))
    return DLFP_EINVAL;
  if (meta->num_units == 0) return DLFP_OK;
  if (meta->prefill_lead_units < 0 || meta->prefill_lead_units > meta->num_prefill_units ||
      (meta->decode_pages_in_flight != 1 && meta->decode_pages_in_flight != 2))
    return DLFP_EINVAL;
  if (!d_work || !d_block_table || !q || !k_cache || !v_cache || !out || !workspace)
    return DLFP_EINVAL;
  if (app && (!k_new || !v_new)) return DLFP_EINVAL;
  if (max_blocks <= 0 || num_blocks <= 0) return DLFP_EINVAL;
  if ((int64_t)workspace_bytes < meta->workspace_bytes ||
      workspace_bytes < (size_t)DLFP_WORKSPACE_PARTIALS)
    return DLFP_ENOSPC;
  if (meta->num_groups > DLFP_MAX_GROUPS) return DLFP_EINVAL;
  Args a;
  a.work = d_work;
  a.block_table = d_block_table;
  a.q = static_cast<const uint16_t*>(q);
  a.kc = static_cast<const uint16_t*>(k_cache);
  a.vc = static_cast<const uint16_t*>(v_cache);
  a.out = out;
  a.ws = static_cast<float*>(workspace);
  a.max_blocks = max_blocks;
  a.num_blocks = num_blocks;
  a.hq = dims->num_q_heads;
  a.hkv = dims->num_kv_heads;
  a.num_units = meta->num_units;
  a.num_prefill = meta->num_prefill_units;
  a.out_f32 = out_dtype;
  a.scale_log2 = scale * LOG2E;
  a.k_new = static_cast<const uint16_t*>(k_new);
  a.v_new = static_cast<const uint16_t*>(v_new);
  a.num_append = app ? meta->num_append : 0;
  a.num_waiting = app ? meta->num_waiting_units : 0;
  a.app_wgs = dlfp::append_workgroups(a.num_append);
  if (a.num_append > 0 && a.app_wgs == 0) {
    Args r = a;
    r.app_wgs = (a.num_append + 3) / 4;
    r.num_waiting = 0;
    (void)hipGetLastError();
    append_records_kernel<<<r.app_wgs, THREADS, 0, stream>>>(r);
    if (hipGetLastError() != hipSuccess) return DLFP_EHIP;
    a.num_append = 0;
    a.num_waiting = 0;
  }
  // Wavefronts' decode units beside prefill units: enough workgroups to fill the
  // slots, fewer when there are fewer units; they drain the decode queue.  Only
  // those that find a slot left by the append and prefill workgroups from the
  // start (at least 64) get units by position.
  const int cus = compute_units();
  const int decode_units = meta->num_units - meta->num_prefill_units;
  const int ahead = meta->num_prefill_units + a.app_wgs;
  a.wide = dlfp::decode_by_workgroup(*meta, cus) ? 4 : 0;
  // Without prefill units: eight wavefronts to a unit while the units are few
  // and long (a compute unit's workgroup then finishes its unit soonest: 512
  // units of 512-2048 keys, g = 2, 53.8 us against 58.1 with four), four, two
  // workgroups to a compute unit, when they run in several rounds (one's
  // prologue and sum then hide behind the other: 3656 units of the Qwen3-8B
  // decoders 394 us against 406 with eight) or are short: a wavefront's part of
  // up to 128 keys is a block at most either way (0.92x), and from one unit per
  // compute unit on the larger workgroups take turns (up to 128 keys 0.65-0.75x,
  // 256 0.8x, 512 0.88x, 1024 0.95x).
  const bool several = meta->num_units > 4 * cus;
  const bool shorter = meta->decode_split_tokens <= (meta->num_units > cus ? 1024 : 128);
  if (a.wide && meta->num_prefill_units == 0 && !several && !shorter) a.wide = 8;
  const int decode_wgs = a.wide ? decode_units : std::min((decode_units + 3) / 4, 2 * cus);
  const int slots = ahead < 2 * cus ? std::max(2 * cus - ahead, 64) : 2 * cus;
  a.decode_waves = 4 * decode_wgs;
  a.decode_static = std::min(decode_units, 4 * std::min(decode_wgs, slots));
  a.lead = meta->num_prefill_units;
  a.decode_lead = 0;
  a.deep = meta->decode_pages_in_flight == 2;
  if (meta->prefill_lead_units < meta->num_prefill_units && decode_wgs >= 8) {
    // the leading decode workgroups are resident from the start and take their
    // units by position; the ones after the other prefill units take tickets
    a.lead = meta->prefill_lead_units;
    a.decode_lead = std::min(decode_wgs, cus) / 8 * 8;
    a.decode_static = std::min(decode_units, 4 * a.decode_lead);
  }
  const int grid = a.app_wgs + meta->num_prefill_units + decode_wgs;
  (void)hipGetLastError();
  hipError_t e;
  switch (g) {
    case 1: e = launch_g<1>(a, grid, app, stream); break;
    case 2: e = launch_g<2>(a, grid, app, stream); break;
    case 4: e = launch_g<4>(a, grid, app, stream); break;
    default: e = launch_g<8>(a, grid, app, stream); break;
  }
  return e == hipSuccess ? DLFP_OK : DLFP_EHIP;
}

// Device address of `scratch` on the current device, looked up (and its
// header and counter region zeroed by a fill kernel on `stream`) on the first
// call for that device.  Launches leave the header and counters zero again.
int static_workspace(void** ptr, hipStream_t stream) {
  static std::mutex mu;
  static void* addr[64] = {nullptr};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return DLFP_EHIP;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return DLFP_EHIP;
    const int64_t n = DLFP_WORKSPACE_PARTIALS / 4;
    (void)hipGetLastError();
    fill_zero_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(static_cast<int*>(p), n);
    if (hipGetLastError() != hipSuccess) return DLFP_EHIP;
    addr[dev] = p;
  }
  *ptr = addr[dev];
  return DLFP_OK;
}

}  // namespace

extern "C" int dlfp_attention_mixed(const dlfp_dims* dims, const dlfp_meta* meta,
                                    const int32_t* d_work,
                                    const int32_t* d_block_table, int32_t max_blocks,
                                    int32_t num_blocks, const void* q, const void* k_cache,
                                    const void* v_cache, float scale, void* out,
                                    int32_t out_dtype, void* workspace, size_t workspace_bytes,
                                    hipStream_t stream) {
  return launch_mixed(dims, meta, d_work, d_block_table, max_blocks, num_blocks, q, false,
                      nullptr, nullptr, k_cache, v_cache, scale, out, out_dtype, workspace,
                      workspace_bytes, stream);
}

extern "C" int dlfp_append_attention_mixed(const dlfp_dims* dims, const dlfp_meta* meta,
                                           const int32_t* d_work, const int32_t* d_block_table,
                                           int32_t max_blocks, int32_t num_blocks, const void* q,
                                           const void* k_new, const void* v_new, void* k_cache,
                                           void* v_cache, float scale, void* out,
                                           int32_t out_dtype, void* workspace,
                                           size_t workspace_bytes, hipStream_t stream) {
  return launch_mixed(dims, meta, d_work, d_block_table, max_blocks, num_blocks, q, true,
                      k_new, v_new, k_cache, v_cache, scale, out, out_dtype, workspace,
                      workspace_bytes, stream);
}

extern "C" int dlfp_append_attention_mixed_static(const dlfp_dims* dims, const dlfp_meta* meta,
                                                  const int32_t* d_work,
                                                  const int32_t* d_block_table,
                                                  int32_t max_blocks, int32_t num_blocks,
                                                  const void* q, const void* k_new,
                                                  const void* v_new, void* k_cache,
                                                  void* v_cache, float scale, void* out,
                                                  int32_t out_dtype, hipStream_t stream) {
  if (!meta) return DLFP_EINVAL;
  if (meta->workspace_bytes > (int64_t)DLFP_STATIC_WORKSPACE_BYTES) return DLFP_ENOSPC;
  if (meta->num_units == 0)  // checks the counts only; no set-up, no launch
    return launch_mixed(dims, meta, d_work, d_block_table, max_blocks, num_blocks, q, true,
                        k_new, v_new, k_cache, v_cache, scale, out, out_dtype, nullptr, 0,
                        stream);
  void* ws = nullptr;
  const int st = static_workspace(&ws, stream);
  if (st != DLFP_OK) return st;
  return launch_mixed(dims, meta, d_work, d_block_table, max_blocks, num_blocks, q, true, k_new,
                      v_new, k_cache, v_cache, scale, out, out_dtype, ws,
                      DLFP_STATIC_WORKSPACE_BYTES, stream);
}

extern "C" int dlfp_workspace_init(void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (!workspace) return DLFP_EINVAL;
  const int64_t bytes = DLFP_WORKSPACE_PARTIALS;
  if ((int64_t)workspace_bytes < bytes) return DLFP_ENOSPC;
  const int64_t n = bytes / 4;
  (void)hipGetLastError();
  fill_zero_kernel<<<(unsigned)((n + 255) / 256), 256, 0, stream>>>(static_cast<int*>(workspace),
                                                                     n);
  return hipGetLastError() == hipSuccess ? DLFP_OK : DLFP_EHIP;
}

extern "C" int dlfp_workspace_error(const void* workspace, int32_t* host_error,
                                    hipStream_t stream) {
  if (!workspace || !host_error) return DLFP_EINVAL;
  if (hipStreamSynchronize(stream) != hipSuccess) return DLFP_EHIP;
  if (hipMemcpy(host_error, workspace, sizeof(int32_t), hipMemcpyDeviceToHost) != hipSuccess)
    return DLFP_EHIP;
  return DLFP_OK;
}
