// Dense projections of one transformer layer's tokens, for the full-iteration
// latency of Eq. 1: the iteration cost the controller observes includes the
// linear layers, whose work grows with the prefill chunk p_t (Sec. 2.1), not
// only the attention.
//
//   out[m][n] = sum_k x[m][k] w[n][k]      (bf16 in, fp32 accumulation)
//
// x is row-major with row stride ldx (elements), w is [n][k] (a linear layer's
// weight as stored: one row per output feature), out row-major with row stride
// ldo.  The products are computed as out^T = w x^T on
// v_mfma_f32_32x32x16_bf16, so that a lane's accumulator holds four
// consecutive features of one token.  Two kernels share the operand layout:
//
//  - split_kernel (few output tiles): the wavefronts of a workgroup compute
//    the same tile over different 64-deep K steps, each from its own LDS ring
//    without a barrier, and add their results through LDS at the end;
//  - tile_kernel (many output tiles): the wavefronts own parts of the tile and
//    share LDS stages, one barrier per 64-deep K step.
//
// Stages are filled by direct global-to-LDS copies of whole 128-byte row
// segments: a copy instruction that covers 8 rows of 128 bytes moves 64 bytes
// per clock and CU, one of 16 rows of 64 bytes half of that (measured from L2,
// 34 against 17 TB/s over the chip), so the K step is 64 and never 32.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "dlfp.h"

namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int N_UNIT = 128;            // n is a multiple of this
constexpr int KSTEP = 64;              // k per LDS stage
constexpr int ROW_BYTES = KSTEP * 2;   // one 64-deep row of a stage
constexpr int COPY_ROWS = 8;           // rows of one copy instruction (64 lanes x 16 bytes)
constexpr int LDS_MAX = 160 * 1024;

typedef __attribute__((address_space(3))) char* lds_ptr_t;

__device__ __forceinline__ uint32_t lds_addr(char* p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_ptr_t)p);
}

// 16 bytes per lane from global memory straight into LDS at lds + 16 lane:
// base is wave-uniform, off the lane's byte offset.  The caller waits for the
// vector-memory counter before the data is read.
__device__ __forceinline__ void lds_copy16(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(off), "s"(base), "s"(lds)
               : "memory", "m0");
}
__device__ __forceinline__ void lds_copy16(const char* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
               :
               : "v"(src), "s"(lds)
               : "memory", "m0");
}

// Wait until at most N of this wave's vector-memory operations are in flight.
template <int N>
__device__ __forceinline__ void wait_copies() {
  static_assert(N <= 63, "the counter has six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// The same, then meet the other waves; every LDS read of this wave has returned.
template <int N>
__device__ __forceinline__ void wait_copies_barrier() {
  static_assert(N <= 63, "the counter has six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Leave min(later, MOST) stages of L copies each in flight.
template <int MOST, int L, bool BARRIER>
__device__ __forceinline__ void wait_stages(int later) {
  if constexpr (MOST > 0) {
    if (later < MOST) return wait_stages<MOST - 1, L, BARRIER>(later);
  }
  if constexpr (BARRIER)
    wait_copies_barrier<MOST * L>();
  else
    wait_copies<MOST * L>();
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  bf16x2_t v;
  v[0] = (__bf16)lo;
  v[1] = (__bf16)hi;
  return __builtin_bit_cast(uint32_t, v);
}

struct LinArgs {
  const uint16_t* x;
  const uint16_t* w;
  void* out;
  int32_t m, n, k, ldx, ldo, out_f32;
  int32_t wide;  // bf16 output rows take 16-byte stores
};

// LDS layout of a stage: row r (64 k values, 128 bytes) keeps its 16-byte
// chunk c at position c ^ swz(r).  LDS serves sixteen lanes of a 16-byte read
// from 64 banks at once; two rows fill the banks, so the lanes that read the
// same chunk of sixteen rows are spread by bits 1-3 of the row (bits 0-2
// measured 1-4% slower: the even rows of a group then share positions).
__device__ __forceinline__ int swz(int row) { return (row >> 1) & 7; }

// Eight consecutive features of a token.
__device__ __forceinline__ void store8(const LinArgs& a, int m, int n, f32x4_t lo, f32x4_t hi) {
  const int64_t e = (int64_t)m * a.ldo + n;
  if (a.out_f32) {
    f32x4_t* o = reinterpret_cast<f32x4_t*>(static_cast<float*>(a.out) + e);
    o[0] = lo;
    o[1] = hi;
    return;
  }
  uint16_t* o = static_cast<uint16_t*>(a.out) + e;
  const u32x4_t v = {pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]),
                     pack_bf16(hi[2], hi[3])};
  if (a.wide) {
    *reinterpret_cast<u32x4_t*>(o) = v;
  } else {
    reinterpret_cast<u32x2_t*>(o)[0] = u32x2_t{v[0], v[1]};
    reinterpret_cast<u32x2_t*>(o)[1] = u32x2_t{v[2], v[3]};
  }
}

// Per-lane byte offsets of the copies of ROWS rows by one wave: copy i covers
// rows first(i) .. + 8, lane l the 16-byte chunk that belongs at position
// l % 8 of row l / 8.  Rows past `last` re-read it (never stored).
template <int COUNT, typename F>
__device__ __forceinline__ void copy_offsets(uint32_t (&off)[COUNT], int lane, int ld, int last,
                                             F first) {
#pragma unroll
  for (int i = 0; i < COUNT; ++i) {
    const int r = first(i) + (lane >> 3);
    off[i] = (uint32_t)(min(r, last) * ld * 2 + (((lane & 7) ^ swz(r)) << 4));
  }
}

// ---------------------------------------------------------------- split K

// One TN x TM tile per workgroup; wave w computes K steps w, w + WAVES, ...
// from its own ring of STAGES stages.  Few tiles leave most CUs one workgroup
// or none, and the launch is then bound by how fast a CU fills its LDS and by
// the memory latency in front of it: the ring keeps 64 KiB and more in flight
// per CU with no barrier to wait at, and every LDS byte is read once.
template <int TN, int TM, int WAVES, int STAGES>
__global__ __launch_bounds__(64 * WAVES) void split_kernel(LinArgs a) {
  constexpr int BN = TN / 32, BM = TM / 32;
  constexpr int NL = TN / COPY_ROWS, ML = TM / COPY_ROWS, L = NL + ML;
  constexpr int STAGE = (TN + TM) * ROW_BYTES;
  constexpr int RING = WAVES * STAGES * STAGE, RESULT = WAVES * TN * TM * 4;
  constexpr int LDS = RING > RESULT ? RING : RESULT;
  static_assert(LDS <= LDS_MAX, "LDS");
  __shared__ __attribute__((aligned(16))) char smem[LDS];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n0 = blockIdx.x * TN, m0 = blockIdx.y * TM;
  uint32_t woff[NL], xoff[ML];
  copy_offsets(woff, lane, a.k, TN - 1, [](int i) { return COPY_ROWS * i; });
  copy_offsets(xoff, lane, a.ldx, a.m - 1 - m0, [](int i) { return COPY_ROWS * i; });
  const char* wbase = reinterpret_cast<const char*>(a.w + (int64_t)n0 * a.k);
  const char* xbase = reinterpret_cast<const char*>(a.x + (int64_t)m0 * a.ldx);
  char* ring = smem + wave * (STAGES * STAGE);
  const uint32_t lds0 = lds_addr(ring);
  const int total = a.k / KSTEP;
  const int mine = total > wave ? (total - wave + WAVES - 1) / WAVES : 0;
  auto issue = [&](int i, int slot) {
    const int64_t ko = (int64_t)(wave + WAVES * i) * ROW_BYTES;
    const uint32_t d = lds0 + slot * STAGE;
#pragma unroll
    for (int j = 0; j < NL; ++j) lds_copy16(wbase + ko, woff[j], d + j * 1024);
#pragma unroll
    for (int j = 0; j < ML; ++j) lds_copy16(xbase + ko, xoff[j], d + (NL + j) * 1024);
  };

  f32x16_t acc[BN][BM];
#pragma unroll
  for (int i = 0; i < BN; ++i)
#pragma unroll
    for (int j = 0; j < BM; ++j) acc[i][j] = f32x16_t{};
  // Operand reads: lane l takes row (l % 32) of a 32-row block and k
  // 8 (l / 32) .. + 8 of each 16-deep product.
  const int lr = lane & 31, lh = lane >> 5;
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < mine) issue(s, s);
  int slot = 0;
  for (int i = 0; i < mine; ++i) {
    wait_stages<STAGES - 1, L, false>(mine - 1 - i);
    const char* wl = ring + slot * STAGE + lr * ROW_BYTES;
    const char* xl = wl + TN * ROW_BYTES;
#pragma unroll
    for (int kk = 0; kk < KSTEP / 16; ++kk) {
      const int c = ((2 * kk + lh) ^ swz(lr)) << 4;
      bf16x8_t wf[BN], xf[BM];
#pragma unroll
      for (int q = 0; q < BN; ++q)
        wf[q] = *reinterpret_cast<const bf16x8_t*>(wl + 32 * q * ROW_BYTES + c);
#pragma unroll
      for (int q = 0; q < BM; ++q)
        xf[q] = *reinterpret_cast<const bf16x8_t*>(xl + 32 * q * ROW_BYTES + c);
#pragma unroll
      for (int q = 0; q < BN; ++q)
#pragma unroll
        for (int t = 0; t < BM; ++t)
          acc[q][t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[q], xf[t], acc[q][t], 0, 0, 0);
    }
    wait_lds();  // the slot's reads have returned before it is refilled
    if (i + STAGES < mine) issue(i + STAGES, slot);
    slot = slot + 1 == STAGES ? 0 : slot + 1;
  }

  // Sum over the waves, in wave order.  A wave's accumulators are groups of
  // four features: group (q, t, g) of lane l holds features
  // 32 q + 8 g + 4 (l / 32) .. + 3 of token 32 t + l % 32.  A thread then sums
  // and stores eight consecutive features, neighbouring threads the next ones
  // of the same token; the lane index is XORed with g and q so that both the
  // writes and these reads spread over the banks.
  wait_copies_barrier<0>();  // every wave is done with its ring
  constexpr int GROUPS = TN * TM / 4;
  f32x4_t* res = reinterpret_cast<f32x4_t*>(smem);
  auto at = [](int q, int t, int g, int l) {
    return ((q * BM + t) * 4 + g) * 64 + (l ^ (g << 2) ^ ((q & 1) << 1));
  };
#pragma unroll
  for (int q = 0; q < BN; ++q)
#pragma unroll
    for (int t = 0; t < BM; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        res[wave * GROUPS + at(q, t, g, lane)] =
            f32x4_t{acc[q][t][4 * g], acc[q][t][4 * g + 1], acc[q][t][4 * g + 2],
                    acc[q][t][4 * g + 3]};
  __syncthreads();
  for (int u = tid; u < GROUPS / 2; u += 64 * WAVES) {
    const int g = u & 3, q = (u >> 2) % BN, tok = (u >> 2) / BN;
    const int ilo = at(q, tok >> 5, g, tok & 31), ihi = at(q, tok >> 5, g, 32 + (tok & 31));
    f32x4_t lo = res[ilo], hi = res[ihi];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      lo += res[w * GROUPS + ilo];
      hi += res[w * GROUPS + ihi];
    }
    if (m0 + tok < a.m) store8(a, m0 + tok, n0 + 32 * q + 8 * g, lo, hi);
  }
}

// ---------------------------------------------------------------- tiles

// TN x TM tile per workgroup of WN x WM waves, STAGES shared LDS stages.  The
// operands of a 16-deep product are read from LDS while the one before it is
// on the matrix cores, across the stage barrier too.  FAR: 64-bit row offsets
// (row strides of 4 Mi elements and more).
template <int TN, int TM, int WN, int WM, int STAGES, bool FAR = false>
__global__ __launch_bounds__(64 * WN * WM, 2) void tile_kernel(LinArgs a, int gm, int gn) {
  constexpr int WAVES = WN * WM, BN = TN / WN / 32, BM = TM / WM / 32, KK = KSTEP / 16;
  constexpr int NL = TN / (COPY_ROWS * WAVES), ML = TM / (COPY_ROWS * WAVES), L = NL + ML;
  static_assert(NL * COPY_ROWS * WAVES == TN && ML * COPY_ROWS * WAVES == TM, "copies");
  constexpr int STAGE = (TN + TM) * ROW_BYTES;
  static_assert(STAGES * STAGE <= LDS_MAX, "LDS");
  __shared__ __attribute__((aligned(16))) char smem[STAGES * STAGE];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // Workgroups are dealt round-robin over the 8 XCDs: each takes a contiguous
  // range of tiles, which walk the feature tiles in bands of 8 token tiles, so
  // the tiles running on an XCD share rows and weights in its L2.
  const int tiles = gm * gn, x = blockIdx.x & 7;
  const int t = x * (tiles >> 3) + min(x, tiles & 7) + (blockIdx.x >> 3);
  constexpr int BAND = 8;
  const int first = t / (BAND * gn) * BAND, h = min(BAND, gm - first), in = t - first * gn;
  const int n0 = (in / h) * TN, m0 = (first + in % h) * TM;

  const char* wbase = reinterpret_cast<const char*>(a.w + (int64_t)n0 * a.k);
  const char* xbase = reinterpret_cast<const char*>(a.x + (int64_t)m0 * a.ldx);
  const int xlast = a.m - 1 - m0;
  uint32_t woff[NL], xoff[ML];
  if constexpr (!FAR) {
    copy_offsets(woff, lane, a.k, TN - 1, [&](int i) { return COPY_ROWS * (i * WAVES + wave); });
    copy_offsets(xoff, lane, a.ldx, xlast, [&](int i) { return COPY_ROWS * (i * WAVES + wave); });
  }
  const uint32_t lds0 = lds_addr(smem) + wave * 1024;
  auto issue = [&](int ks, int slot) {
    const int64_t ko = (int64_t)ks * ROW_BYTES;
    const uint32_t d = lds0 + slot * STAGE;
    if constexpr (FAR) {
      auto src = [&](const char* base, int i, int64_t ld, int last) {
        const int r = COPY_ROWS * (i * WAVES + wave) + (lane >> 3);
        return base + ko + min(r, last) * ld * 2 + (((lane & 7) ^ swz(r)) << 4);
      };
#pragma unroll
      for (int j = 0; j < NL; ++j) lds_copy16(src(wbase, j, a.k, TN - 1), d + j * WAVES * 1024);
#pragma unroll
      for (int j = 0; j < ML; ++j)
        lds_copy16(src(xbase, j, a.ldx, xlast), d + TN * ROW_BYTES + j * WAVES * 1024);
    } else {
#pragma unroll
      for (int j = 0; j < NL; ++j) lds_copy16(wbase + ko, woff[j], d + j * WAVES * 1024);
#pragma unroll
      for (int j = 0; j < ML; ++j)
        lds_copy16(xbase + ko, xoff[j], d + TN * ROW_BYTES + j * WAVES * 1024);
    }
  };

  f32x16_t acc[BN][BM];
#pragma unroll
  for (int i = 0; i < BN; ++i)
#pragma unroll
    for (int j = 0; j < BM; ++j) acc[i][j] = f32x16_t{};
  const int lr = lane & 31, lh = lane >> 5, wn = wave / WM, wm = wave % WM;
  const char* wl = smem + (wn * BN * 32 + lr) * ROW_BYTES;
  const char* xl = smem + (TN + wm * BM * 32 + lr) * ROW_BYTES;
  bf16x8_t wf[2][BN], xf[2][BM];
  auto read = [&](int slot, int kk, int set) {
    const int c = slot * STAGE + (((2 * kk + lh) ^ swz(lr)) << 4);
#pragma unroll
    for (int q = 0; q < BN; ++q)
      wf[set][q] = *reinterpret_cast<const bf16x8_t*>(wl + 32 * q * ROW_BYTES + c);
#pragma unroll
    for (int q = 0; q < BM; ++q)
      xf[set][q] = *reinterpret_cast<const bf16x8_t*>(xl + 32 * q * ROW_BYTES + c);
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int q = 0; q < BN; ++q)
#pragma unroll
      for (int u = 0; u < BM; ++u)
        acc[q][u] =
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][q], xf[set][u], acc[q][u], 0, 0, 0);
  };

  const int steps = a.k / KSTEP;
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < steps) issue(s, s);
  wait_stages<STAGES - 1, L, true>(steps - 1);
  read(0, 0, 0);
  int slot = 0;
  for (int ks = 0; ks < steps; ++ks) {
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      if (kk + 1 < KK) {
        read(slot, kk + 1, (kk + 1) & 1);
      } else if (ks + 1 < steps) {
        // Stage ks + 1 has landed and no wave reads stage ks any more; its
        // slot takes stage ks + STAGES.
        const int next = slot + 1 == STAGES ? 0 : slot + 1;
        wait_stages<STAGES - 2, L, true>(steps - 2 - ks);
        read(next, 0, 0);
        if (ks + STAGES < steps) issue(ks + STAGES, slot);
        slot = next;
      }
      multiply(kk & 1);
    }
  }

  // Through the wave's slice of LDS, so that whole runs of a row are stored
  // (straight from the accumulators a store covers 16 bytes of 32 rows; on
  // m = 8192, n = 6144, k = 1024 the launch took 13% longer with those).
  constexpr int SLICE = STAGES * STAGE / WAVES / 16 * 16;
  constexpr int FB = 2;                    // 32-feature blocks per pass
  constexpr int RB = FB * 32 * 4 + 16;     // fp32 row of a pass, padded off the banks
  static_assert(BN % FB == 0 || BN == 1, "passes");
  constexpr int B = BN < FB ? BN : FB;
  static_assert(SLICE >= 32 * RB, "epilogue slice");
  wait_copies_barrier<0>();
  char* mine = smem + wave * SLICE;
#pragma unroll
  for (int j = 0; j < BM; ++j)
#pragma unroll
    for (int p = 0; p < BN / B; ++p) {
#pragma unroll
      for (int i = 0; i < B; ++i)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x16_t& c = acc[p * B + i][j];
          *reinterpret_cast<f32x4_t*>(mine + lr * RB + (32 * i + 8 * g + 4 * lh) * 4) =
              f32x4_t{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
        }
      wait_lds();
      constexpr int PER_ROW = B * 4, ROWS = 64 / PER_ROW;  // lanes per row, rows per store
#pragma unroll
      for (int r0 = 0; r0 < 32; r0 += ROWS) {
        const int r = r0 + lane / PER_ROW, f = 8 * (lane % PER_ROW);
        const f32x4_t* v = reinterpret_cast<const f32x4_t*>(mine + r * RB + f * 4);
        const int m = m0 + 32 * (wm * BM + j) + r;
        if (m < a.m) store8(a, m, n0 + 32 * (wn * BN + p * B) + f, v[0], v[1]);
      }
      wait_lds();
    }
}

template <int TN, int TM, int WAVES, int STAGES>
void launch_split(const LinArgs& a, hipStream_t stream) {
  const dim3 grid(a.n / TN, (a.m + TM - 1) / TM);
  split_kernel<TN, TM, WAVES, STAGES><<<grid, 64 * WAVES, 0, stream>>>(a);
}
template <int TN, int TM, int WN, int WM, int STAGES, bool FAR = false>
void launch_tile(const LinArgs& a, hipStream_t stream) {
  const int gm = (a.m + TM - 1) / TM, gn = a.n / TN;
  tile_kernel<TN, TM, WN, WM, STAGES, FAR><<<gm * gn, 64 * WN * WM, 0, stream>>>(a, gm, gn);
}

// Which kernel and tile: the one whose estimated time is lowest.  With
// r = ceil(tiles / 256) rounds over the CUs and s = k / 64 K steps the estimate
// is start + step s + (round + work s) r microseconds, fitted to 660 launches of
// 1-8192 tokens times 24 (n, k), the Qwen3-0.6B, 8B and 32B projections among them
// (relative errors; sizes where a variant takes over 1.8 times the best one's
// time count little).  There the choice is within 0.4% of the fastest variant on
// average, and against one 128 x 128 tile for every size, as before, the launches
// take 0.42x of the time (geometric mean) and none takes longer: n = k = 1024
// 11.0 -> 3.3 us at m = 32, 14.3 -> 6.3 us at m = 545, 28.2 -> 21.3 us at
// m = 8192; n = 6144, k = 1024, m = 8192 141.5 -> 104.5 us; n = 1024, k = 3072,
// m = 545 36.9 -> 12.1 us; n = 5120, k = 8192, m = 4096 384 -> 353 us.  (A row's
// sum over k runs in another order in another kernel, so its last bit can depend
// on the number of rows.)  Small tiles win where the tiles are few, since
// every CU then fills its LDS side by side; large ones where the tiles fill
// the chip, since each operand byte then serves more products.
struct Variant {
  int tn, tm;
  float start, step, round, work;
  void (*launch)(const LinArgs&, hipStream_t);
};
constexpr Variant VARIANTS[] = {
    {32, 32, 1.35f, -0.024f, 0.80f, 0.120f, launch_split<32, 32, 8, 2>},
    {64, 32, 1.30f, -0.029f, 1.05f, 0.170f, launch_split<64, 32, 4, 3>},
    {64, 64, 1.44f, -0.043f, 1.64f, 0.231f, launch_split<64, 64, 4, 2>},
    {128, 64, 1.79f, 0.065f, 0.91f, 0.305f, launch_tile<128, 64, 2, 2, 3>},
    {128, 128, 1.05f, -0.060f, 2.41f, 0.545f, launch_tile<128, 128, 2, 4, 4>},
    {128, 256, 0.54f, -0.142f, 3.93f, 0.942f, launch_tile<128, 256, 2, 4, 3>},
    {256, 256, -0.42f, -0.277f, 6.99f, 1.657f, launch_tile<256, 256, 2, 4, 2>},
};
constexpr int CUS = 256;
// Row strides from here on take 64-bit offsets (255 rows of 2 bytes each fit
// 32 bits below).
constexpr int FAR_STRIDE = 1 << 22;

void launch_linear(const LinArgs& a, hipStream_t stream) {
  if (std::max(a.ldx, a.k) >= FAR_STRIDE) return launch_tile<64, 64, 2, 2, 4, true>(a, stream);
  const Variant* best = nullptr;
  float least = 0.f;
  for (const Variant& v : VARIANTS) {
    if (a.n % v.tn) continue;
    const int64_t tiles = ((int64_t)a.m + v.tm - 1) / v.tm * (a.n / v.tn);
    const float rounds = (float)((tiles + CUS - 1) / CUS), steps = (float)(a.k / KSTEP);
    const float t = v.start + v.step * steps + (v.round + v.work * steps) * rounds;
    if (!best || t < least) {
      best = &v;
      least = t;
    }
  }
  best->launch(a, stream);
}

}  // namespace

extern "C" int dlfp_linear_bf16(int32_t m, int32_t n, int32_t k, const void* x, int32_t ldx,
                                const void* w, void* out, int32_t ldo, int32_t out_dtype,
                                hipStream_t stream) {
  if (m < 0 || n <= 0 || k <= 0) return DLFP_EINVAL;
  if (out_dtype != 0 && out_dtype != 1) return DLFP_EINVAL;
  if (n % N_UNIT || k % KSTEP) return DLFP_EUNSUPPORTED;
  if (ldx < k || ldo < n || ldx % 8 || ldo % 4) return DLFP_EINVAL;
  if (m == 0) return DLFP_OK;
  if (!x || !w || !out) return DLFP_EINVAL;
  if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(w)) & 15) return DLFP_EINVAL;
  if (reinterpret_cast<uintptr_t>(out) & (out_dtype ? 15 : 7)) return DLFP_EINVAL;
  const bool wide = (reinterpret_cast<uintptr_t>(out) & 15) == 0 && ldo % 8 == 0;
  const LinArgs a{static_cast<const uint16_t*>(x), static_cast<const uint16_t*>(w), out, m, n, k,
                  ldx, ldo, out_dtype, wide};
  (void)hipGetLastError();
  launch_linear(a, stream);
  return hipGetLastError() == hipSuccess ? DLFP_OK : DLFP_EHIP;
}
