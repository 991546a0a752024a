// Paged KV append: write this iteration's new keys and values into their
// pages (the PagedAttention cache write; the cache layout is the one the
// attention launch reads, declared in dlfp.h).
//
// One workgroup of 128 threads serves a block of 16 consecutive packed tokens of
// one KV head.  Keys keep their token-row layout: 16 threads copy one 256-byte
// row with 16-byte loads and stores.  Values go into the transposed page
// [dim][position], token slot t at position vt_pos(t) (slots 4-7 and 8-11
// trade places): thread d gathers dimension d of 16 tokens (256-byte coalesced
// reads per token) and, when they fill one page in slot order -- the common
// case inside a prefill chunk -- writes its whole 32-byte row, so the workgroup
// stores the 4 KiB page contiguously.  Otherwise each token's value lands with a
// 2-byte store at its position, each of which costs the memory side a
// read-modify-write of its line.  A prompt's chunk rarely starts at a page, so
// the page that a block writes is the full one that begins in it, wherever that
// is: it ends in the next block, whose workgroup finds it by the same rule and
// leaves its tokens out.  The launch is bound by its round trips (slots, tokens,
// stores) up to about 2000 tokens and by its bytes from there.  Against pages
// only where a block is one, with 8 heads: 2048 tokens from position 4099 9.9 ->
// 6.7 us, 8192 from 1001 28.3 -> 15.7; from 4096, where a page's values are
// loaded beside the slots, 2048 tokens 4.84 -> 4.23 and 8192 11.8 -> 11.3 (one
// slot load per wavefront, contiguous stores of the value rows).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "dlfp.h"
#include "dlfp_internal.h"

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int D = DLFP_HEAD_DIM;
constexpr int PAGE = DLFP_PAGE_SIZE;
constexpr int TOK = 16;      // tokens per workgroup
constexpr int THREADS = 128;

// Position of token slot t in a value page row (bits 2 and 3 swap).
__device__ __forceinline__ int vt_pos(int t) { return (t & 3) | ((t & 4) << 1) | ((t & 8) >> 1); }

__global__ __launch_bounds__(THREADS) void kv_append_kernel(
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new,
    const int32_t* __restrict__ slots, uint16_t* __restrict__ k_cache,
    uint16_t* __restrict__ v_cache, int num_tokens, int hkv, int64_t num_slots) {
  const int t0 = blockIdx.x * TOK;
  const int h = blockIdx.y;
  const int tid = threadIdx.x;
  const int nt = min(TOK, num_tokens - t0);

  // The loads of the block are issued before any store (one memory round
  // trip): slots, two 16-byte key chunks per thread (tokens tid / 16 and
  // tid / 16 + 8, chunk tid % 16) and the 16 values of dimension d = tid.
  // Lane l of a wavefront has the slot of token t0 - 16 + l: the block before,
  // this one, the one after.
  const int lane = tid & 63;
  const int tl = t0 - TOK + lane;
  const bool real = tl >= 0 && tl < num_tokens && lane < 3 * TOK;
  const int slot_l = real ? slots[tl] : -1;
  const int c = tid & 15;
  u32x4_t kv[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int tt = (tid >> 4) + 8 * j;
    kv[j] = tt < nt ? *reinterpret_cast<const u32x4_t*>(k_new + ((int64_t)(t0 + tt) * hkv + h) * D + c * 8)
                    : u32x4_t{0u, 0u, 0u, 0u};
  }
  const int d = tid;
  uint16_t vals[TOK];
#pragma unroll
  for (int tt = 0; tt < TOK; ++tt)
    vals[tt] = tt < nt ? v_new[((int64_t)(t0 + tt) * hkv + h) * D + d] : 0;

  // Keys: token rows, 16-byte chunks.
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int tt = (tid >> 4) + 8 * j;
    const int slot = __shfl(slot_l, TOK + tt);
    if (tt < nt && slot >= 0 && (int64_t)slot < num_slots) {
      const int64_t blk = slot / PAGE, off = slot % PAGE;
      *reinterpret_cast<u32x4_t*>(k_cache + ((blk * hkv + h) * PAGE + off) * D + c * 8) = kv[j];
    }
  }

  // Lanes whose token begins a page of the pool that the 15 tokens after it
  // fill in slot order.
  const int next = __shfl_down(slot_l, 1);
  const bool goes_on = real && lane + 1 < 3 * TOK && tl + 1 < num_tokens && slot_l >= 0 &&
                       (int64_t)next == (int64_t)slot_l + 1;
  uint64_t run = __builtin_amdgcn_ballot_w64(goes_on);  // 1, then 2, 4, 8, 15 steps
  run &= run >> 1;
  run &= run >> 2;
  run &= run >> 4;
  run &= run >> 7;
  const uint64_t begins = run & __builtin_amdgcn_ballot_w64(
      slot_l >= 0 && slot_l % PAGE == 0 && (int64_t)slot_l + PAGE <= num_slots);
  // The page beginning in a block, relative to it (at most one: the next of a
  // run begins 16 tokens later); TOK: none.
  auto page_of = [&](int block) {
    const uint32_t b = (uint32_t)(begins >> (TOK * block)) & 0xFFFFu;
    return b ? __builtin_ctz(b) : TOK;
  };
  const int before = page_of(0), here = page_of(1);

  // Values, thread d dimension d: the block's tokens in neither its page nor the
  // one from the block before, then its page.
  const int first = before < TOK ? before : 0;
  if (first < here) {
#pragma unroll
    for (int tt = 0; tt < TOK; ++tt) {
      const int slot = __builtin_amdgcn_readlane(slot_l, TOK + tt);
      if (tt >= first && tt < here && tt < nt && slot >= 0 && (int64_t)slot < num_slots) {
        const int64_t blk = slot / PAGE, off = slot % PAGE;
        v_cache[((blk * hkv + h) * D + d) * PAGE + vt_pos((int)off)] = vals[tt];
      }
    }
  }
  if (here < TOK) {
    if (here > 0) {
#pragma unroll
      for (int tt = 0; tt < TOK; ++tt)
        vals[tt] = v_new[((int64_t)(t0 + here + tt) * hkv + h) * D + d];
    }
    const int64_t blk = __builtin_amdgcn_readlane(slot_l, TOK + here) / PAGE;
    u32x4_t lo, hi;
#pragma unroll
    for (int w = 0; w < 4; ++w) {  // position p holds slot vt_pos(p)
      lo[w] = (uint32_t)vals[vt_pos(2 * w)] | ((uint32_t)vals[vt_pos(2 * w + 1)] << 16);
      hi[w] = (uint32_t)vals[vt_pos(8 + 2 * w)] | ((uint32_t)vals[vt_pos(8 + 2 * w + 1)] << 16);
    }
    // Lanes trade halves of rows, so that a store covers a contiguous kilobyte.
    u32x4_t* dst = reinterpret_cast<u32x4_t*>(v_cache + ((blk * hkv + h) * D + (tid & 64)) * PAGE);
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      u32x4_t x;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t l = __shfl(lo[w], 32 * p + (lane >> 1)), u = __shfl(hi[w], 32 * p + (lane >> 1));
        x[w] = lane & 1 ? u : l;
      }
      dst[64 * p + lane] = x;
    }
  }
}

}  // namespace

extern "C" int dlfp_kv_append(const dlfp_dims* dims, int32_t num_tokens, const void* k_new,
                              const void* v_new, const int32_t* slot_mapping, void* k_cache,
                              void* v_cache, int32_t num_blocks, hipStream_t stream) {
  int g = 0;
  const int st = dlfp::check_dims(dims, &g);
  if (st != DLFP_OK) return st;
  if (num_tokens < 0 || num_blocks < 0) return DLFP_EINVAL;
  if (num_tokens == 0) return DLFP_OK;
  if (!k_new || !v_new || !slot_mapping || !k_cache || !v_cache) return DLFP_EINVAL;
  (void)hipGetLastError();
  const dim3 grid((num_tokens + TOK - 1) / TOK, dims->num_kv_heads);
  kv_append_kernel<<<grid, THREADS, 0, stream>>>(
      static_cast<const uint16_t*>(k_new), static_cast<const uint16_t*>(v_new), slot_mapping,
      static_cast<uint16_t*>(k_cache), static_cast<uint16_t*>(v_cache), num_tokens,
      dims->num_kv_heads, (int64_t)num_blocks * PAGE);
  return hipGetLastError() == hipSuccess ? DLFP_OK : DLFP_EHIP;
}
