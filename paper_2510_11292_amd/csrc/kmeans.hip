// Prefill-stage k-means of prompt keys (Section 4.2 prefill stage; Algorithm 1
// store_cache prefill branch), one independent problem per (sequence, layer,
// KV head) slice.
//
// Per Lloyd iteration:
//   prep     centroid operand for the matrix cores: -2 * op(c) laid out as MFMA
//            A-fragments (op = bf16 RNE rounding for bf16 keys, identity for fp32),
//            plus ||op(c)||^2 (float64 sum, rounded to fp32).
//   assign   D = ||op(c)||^2 - 2 op(c).k on MFMA (the norm enters as the
//            accumulator input), running argmin per key kept in registers;
//            the counts follow (a block histogram, later each moved key).
//   scatter  scan of the counts -> CSR offsets, and key ids into their cluster's
//            member range (order unspecified).
//   sum      centroid = float64 sum of members / count, rounded once to fp32;
//            empty clusters keep their centroid.  Sums of bf16 or fp32 inputs
//            are exact in float64 at these sizes, so the order is irrelevant.
//            The same kernel writes the next iteration's operand (prep runs
//            once, before the first iteration).
// From the second iteration on (bf16) the assignment starts each key's running
// minimum at a bound from its previous centroid, so the index search runs
// only for tiles that hold a closer centroid, and only the clusters that a key
// entered or left are scattered and recomputed.  In large calls, from the
// fourth iteration on, only those clusters' centroids are swept, and the few
// keys for which that is not enough take a launch of their own.
// After the last iteration, finalize sorts each member range ascending (the
// perm output), writes the unit table, and pack copies K/V rows into the pool.
#include "common.h"

namespace louiskv {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int kTileC = 32;                 // centroids per MFMA tile (rows of D)
constexpr int kBf16Steps = 8;              // 32x32x16 MFMAs per 128-wide dot product
constexpr int kBf16TileU4 = kBf16Steps * 64;       // uint4 per bf16 operand tile (8 KB)
constexpr int kF32TileU4 = 16 * 64;                // uint4 per fp32 operand tile (16 KB)

#ifndef LKV_BF16_KEY_TILES
#define LKV_BF16_KEY_TILES 4
#endif
#ifndef LKV_BF16_STAGE_TILES
#define LKV_BF16_STAGE_TILES 2
#endif
#ifndef LKV_ASSIGN_WAVES
#define LKV_ASSIGN_WAVES 4
#endif
constexpr int kAssignThreads = 256;                          // fp32 kernel block
constexpr int kBf16Waves = LKV_ASSIGN_WAVES;                 // waves sharing one LDS stage
constexpr int kBf16Threads = 64 * kBf16Waves;
constexpr int kBf16KeyTiles = LKV_BF16_KEY_TILES;            // 32-key tiles held per wave
constexpr int kBf16KeysPerBlock = kBf16Waves * 32 * kBf16KeyTiles;
constexpr int kBf16StageTiles = LKV_BF16_STAGE_TILES;        // centroid tiles per LDS stage
constexpr int kF32KeysPerBlock = 4 * 32;           // one 32-key tile per wave
constexpr int kF32StageTiles = 2;

__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Workgroups are dealt to the 8 XCDs round-robin by block id.  Renumber the
// first 8*floor(n/8) blocks so that consecutive logical blocks (the blocks of
// one slice) run on the same XCD and share its L2; the tail keeps its id.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_local_block(int b, int n) {
  const int q = n / kXcds;
  if (b >= q * kXcds) return b;
  return (b % kXcds) * q + b / kXcds;
}

template <class T>
__global__ void init_centroids_kernel(const T* __restrict__ keys, const int32_t* __restrict__ init_idx,
                                      float* __restrict__ reps, int n_tokens, int n_clusters,
                                      int units_cap, int64_t n_rows) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int lane = threadIdx.x & 63;
  const int64_t s = row / n_clusters;
  const int c = (int)(row - s * n_clusters);
  int t = init_idx[s * n_clusters + c];
  t = t < 0 ? 0 : (t >= n_tokens ? n_tokens - 1 : t);
  const T* src = keys + ((size_t)s * n_tokens + t) * kHeadDim;
  float* dst = reps + ((size_t)s * units_cap + c) * kHeadDim;
  dst[2 * lane] = load_as_f32(src, 2 * lane);
  dst[2 * lane + 1] = load_as_f32(src, 2 * lane + 1);
}

// One wave per padded centroid row.  Writes the A-fragments of -2*op(c) and
// ||op(c)||^2; padding rows get a zero operand and +inf norm so they never win.
//
// Dimension k of a centroid maps to MFMA operand position (lane half h, step,
// element): bf16: k = 64h + 8*step + e; fp32: k = 64h + step.  The key operand
// uses the same map, so each product pairs equal dimensions.
template <bool kBf16>
__global__ void prep_operand_kernel(const float* __restrict__ reps, int units_cap, int n_clusters,
                                    int n_ctiles, uint4* __restrict__ frag, float* __restrict__ cnorm,
                                    int32_t* __restrict__ counts, int32_t* __restrict__ cursor,
                                    int32_t* __restrict__ dirty, int64_t n_rows) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n_rows) return;
  const int lane = threadIdx.x & 63;
  const int cpad = n_ctiles * kTileC;
  const int64_t s = row / cpad;
  const int c = (int)(row - s * cpad);
  const bool real = c < n_clusters;
  float v0 = 0.f, v1 = 0.f;
  if (real) {
    const float* src = reps + ((size_t)s * units_cap + c) * kHeadDim;
    v0 = src[2 * lane];
    v1 = src[2 * lane + 1];
  }
  if (kBf16) {
    v0 = bf16_to_f32(f32_to_bf16(v0));
    v1 = bf16_to_f32(f32_to_bf16(v1));
  }
  double nrm = wave_sum((double)v0 * v0 + (double)v1 * v1);
  const int t = c / kTileC, ci = c % kTileC;
  const int k0 = 2 * lane, h = k0 >> 6;
  const int flane = h * 32 + ci;
  if (kBf16) {
    const int step = (k0 & 63) >> 3, e = k0 & 7;
    uint16_t* f = reinterpret_cast<uint16_t*>(frag + ((size_t)s * n_ctiles + t) * kBf16TileU4);
    const uint32_t lo = f32_to_bf16(-2.f * v0), hi = f32_to_bf16(-2.f * v1);
    *reinterpret_cast<uint32_t*>(f + ((size_t)(step * 64 + flane) * 8 + e)) = lo | (hi << 16);
  } else {
    float* f = reinterpret_cast<float*>(frag + ((size_t)s * n_ctiles + t) * kF32TileU4);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int step = (k0 + q) & 63;
      f[((size_t)(step >> 2) * 64 + flane) * 4 + (step & 3)] = -2.f * (q ? v1 : v0);
    }
  }
  if (lane == 0) {
    cnorm[(size_t)s * cpad + c] = real ? (float)nrm : __builtin_inff();
    if (real && counts) {
      counts[(size_t)s * n_clusters + c] = 0;
      cursor[(size_t)s * n_clusters + c] = 0;
      dirty[(size_t)s * n_clusters + c] = 0;
    }
  }
}

// Block histogram of chosen clusters, merged into counts[slice][*].
__device__ __forceinline__ void block_histogram(int* hist, bool lds_ok, int n_clusters, int32_t* counts_slice,
                                                const int* idx, const bool* valid, int n_local) {
  const int tid = threadIdx.x;
  if (lds_ok) {
    for (int i = tid; i < n_clusters; i += blockDim.x) hist[i] = 0;
    __syncthreads();
    for (int q = 0; q < n_local; ++q)
      if (valid[q]) atomicAdd(&hist[idx[q]], 1);
    __syncthreads();
    for (int i = tid; i < n_clusters; i += blockDim.x)
      if (hist[i]) atomicAdd(&counts_slice[i], hist[i]);
  } else {
    for (int q = 0; q < n_local; ++q)
      if (valid[q]) atomicAdd(&counts_slice[idx[q]], 1);
  }
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr int kBf16Ring = 4;                          // LDS stage buffers in flight
constexpr int kBf16StageBytes = kBf16StageTiles * kBf16TileU4 * 16 + 64 * 4;
// DMA instructions each wave issues per stage: its share of the operand tiles
// plus one copy of the stage's norms (every wave writes the same norms, so the
// count is the same for all waves and vmcnt thresholds are uniform).
constexpr int kBf16DmaPerWave = kBf16StageTiles * (kBf16TileU4 / 64) / kBf16Waves + 1;
static_assert(kBf16StageTiles * (kBf16TileU4 / 64) % kBf16Waves == 0, "operand copies must split evenly");
static_assert(kBf16StageTiles * kTileC <= 64, "one 64-lane copy carries a stage's norms");

// Asynchronous copy of stage `st` (centroid operand tiles and their norms)
// straight from global memory into an LDS stage buffer; 64 lanes x 16 bytes
// per instruction, completion tracked by vmcnt.  The tile count is padded to
// whole stages, so every stage copies the same amount.
// Copies [q0, q1) of the wave's kBf16DmaPerWave instructions for stage st
// (the last one carries the norms), so a stage's copy can be spread out.
//
// The copies are written as inline assembly (scalar base address, per-lane
// offset, LDS destination in M0) rather than with the compiler builtin: the
// builtin makes the compiler track the LDS writes itself, and at the loop
// header it cannot tell the ring buffers apart and drains every copy in
// flight (vmcnt(0)) once per pass of the ring.  Written this way the compiler
// sees no memory operation, and the sweep's explicit vmcnt waits and barriers
// are the only synchronisation, as intended.
__device__ __forceinline__ void dma_16b(const void* base, uint32_t lane_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_addr)
               : "memory", "m0");
}
__device__ __forceinline__ void dma_4b(const void* base, uint32_t lane_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dword %0, %1" ::"v"(lane_off), "s"(base), "s"(lds_addr)
               : "memory", "m0");
}

__device__ __forceinline__ void stage_async_part(const uint4* fslice, const float* cslice, int st, char* buf,
                                                 int wave, int lane, int q0, int q1) {
  const uint4* src = fslice + (size_t)st * kBf16StageTiles * kBf16TileU4;
#pragma unroll
  for (int q = 0; q < kBf16DmaPerWave - 1; ++q) {
    if (q < q0 || q >= q1) continue;
    const int i = wave + q * kBf16Waves;   // wave-uniform
    dma_16b(src + i * 64, lane * 16, (uint32_t)(uintptr_t)(buf + i * 1024));
  }
  if (q1 == kBf16DmaPerWave) {
    const int c = lane % (kBf16StageTiles * kTileC);
    dma_4b(cslice + st * kBf16StageTiles * kTileC, c * 4,
           (uint32_t)(uintptr_t)(buf + kBf16StageTiles * kBf16TileU4 * 16));
  }
}

__device__ __forceinline__ void stage_async(const uint4* fslice, const float* cslice, int st, char* buf, int wave,
                                            int lane) {
  stage_async_part(fslice, cslice, st, buf, wave, lane, 0, kBf16DmaPerWave);
}

__device__ __forceinline__ void wait_vm_stages(int k) {
  // at most k later stages' copies may still be in flight
  if (k >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kBf16DmaPerWave) : "memory");
  else if (k == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kBf16DmaPerWave) : "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Tile epilogue of the running argmin.  The lane's 16 results of a tile
// (rows ascending with v) are reduced to their minimum with min3 (8 ops); only
// when that beats the running best does the lane search for the lowest row
// holding it.  Because tiles are visited in ascending order and only a
// strictly smaller value replaces the best, the result is the lowest index
// among equal minima.  The search is skipped by a wave-uniform branch (taken
// when any lane improved) and applied with per-lane selects, so EXEC is never
// narrowed while matrix instructions are in flight.
// Row of result register v within the lane's half of a 32x32 tile.
#define LKV_ROW(v) (8 * ((v) >> 2) + ((v) & 3))

__device__ __forceinline__ float tile_min(const floatx16& x) {
  const float a = __builtin_fminf(__builtin_fminf(x[0], x[1]), x[2]);
  const float b = __builtin_fminf(__builtin_fminf(x[3], x[4]), x[5]);
  const float c = __builtin_fminf(__builtin_fminf(x[6], x[7]), x[8]);
  const float d = __builtin_fminf(__builtin_fminf(x[9], x[10]), x[11]);
  const float e = __builtin_fminf(__builtin_fminf(x[12], x[13]), x[14]);
  const float f = __builtin_fminf(__builtin_fminf(a, b), c);
  const float g = __builtin_fminf(__builtin_fminf(d, e), x[15]);
  return __builtin_fminf(f, g);
}

// Lowest row of the tile holding the value m (the lane's minimum).  All
// compares go first, each into its own SGPR pair, then the selects from the
// highest row down; written as a plain select chain the compiler pairs every
// compare with its select through VCC and pads each pair with wait states.
#define LKV_CMP(v) asm("v_cmp_eq_f32_e64 %0, %1, %2" : "=s"(e##v) : "v"(x[v]), "v"(m))
#define LKV_CND(v, row) asm("v_cndmask_b32_e64 %0, %1, " #row ", %2" : "=v"(id) : "v"(id), "s"(e##v))
__device__ __forceinline__ int tile_find(const floatx16& x, float m) {
  uint64_t e0, e1, e2, e3, e4, e5, e6, e7, e8, e9, e10, e11, e12, e13, e14;
  LKV_CMP(0); LKV_CMP(1); LKV_CMP(2); LKV_CMP(3); LKV_CMP(4); LKV_CMP(5); LKV_CMP(6); LKV_CMP(7);
  LKV_CMP(8); LKV_CMP(9); LKV_CMP(10); LKV_CMP(11); LKV_CMP(12); LKV_CMP(13); LKV_CMP(14);
  int id = LKV_ROW(15);
  // rows LKV_ROW(14..0) = 26 25 24 19 18 17 16 11 10 9 8 3 2 1 0
  LKV_CND(14, 26); LKV_CND(13, 25); LKV_CND(12, 24); LKV_CND(11, 19); LKV_CND(10, 18); LKV_CND(9, 17);
  LKV_CND(8, 16); LKV_CND(7, 11); LKV_CND(6, 10); LKV_CND(5, 9); LKV_CND(4, 8); LKV_CND(3, 3); LKV_CND(2, 2);
  LKV_CND(1, 1); LKV_CND(0, 0);
  return id;
}
#undef LKV_CMP
#undef LKV_CND

// The second smallest of the lane's 16 results (equal to the smallest where
// two are): the medians of the five triples that tile_min takes the minima of,
// merged pair by pair.  A NaN among the results can only make it smaller.
__device__ __forceinline__ float tile_second(const floatx16& x) {
  float m = x[15], t = __builtin_inff();
#pragma unroll
  for (int v = 0; v < 15; v += 3) {
    const float a = __builtin_fminf(__builtin_fminf(x[v], x[v + 1]), x[v + 2]);
    const float b = __builtin_amdgcn_fmed3f(x[v], x[v + 1], x[v + 2]);
    t = __builtin_fminf(__builtin_fminf(t, b), __builtin_fmaxf(m, a));
    m = __builtin_fminf(m, a);
  }
  return t;
}

// The smallest float above x (x not NaN; +inf stays).
__device__ __forceinline__ float next_up(float x) {
  const int i = __float_as_int(x);
  if (x == __builtin_inff()) return x;
  return __int_as_float(x == 0.f ? 1 : i > 0 ? i + 1 : i - 1);
}

// One stage of the bf16 sweep.  `cur` holds stage st (its copy was waited
// for); the copy of stage st + kBf16Ring - 1 goes into `nxt`, the buffer that
// stage st - 1 used.
// kSecond: sec collects the minimum over every centroid but the winner (a
// starting bound, bidx -1, is no centroid's value and stays out of it); it
// costs one minimum per tile outside the search branch.
template <int kKT, bool kSecond>
__device__ __forceinline__ void bf16_stage(const char* cur, char* nxt, const uint4* fslice,
                                           const float* cslice, int st, int n_stages, int wave, int lane, int h,
                                           const bf16x8_t (&b)[kKT][kBf16Steps], float (&best)[kKT],
                                           int (&bidx)[kKT], float (&sec)[kKT]) {
  wait_vm_stages(min(kBf16Ring - 2, n_stages - 1 - st));
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();   // stage st is in LDS for all waves; stage st-1's buffer is free
  const bool copy_next = st + kBf16Ring - 1 < n_stages;
  const uint4* s_frag = reinterpret_cast<const uint4*>(cur);
  const float* s_cn = reinterpret_cast<const float*>(cur + kBf16StageTiles * kBf16TileU4 * 16);
  const int t0 = st * kBf16StageTiles;
#pragma unroll
  for (int tt = 0; tt < kBf16StageTiles; ++tt) {
    // spread the copy of stage st + kBf16Ring - 1 over the stage's tiles
    if (copy_next) {
      const int per = (kBf16DmaPerWave + kBf16StageTiles - 1) / kBf16StageTiles;
      stage_async_part(fslice, cslice, st + kBf16Ring - 1, nxt, wave, lane, tt * per,
                       min(kBf16DmaPerWave, (tt + 1) * per));
    }
    bf16x8_t a[kBf16Steps];
#pragma unroll
    for (int s = 0; s < kBf16Steps; ++s)
      a[s] = __builtin_bit_cast(bf16x8_t, s_frag[(tt * kBf16Steps + s) * 64 + lane]);
    floatx16 cn;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 x = *reinterpret_cast<const float4*>(&s_cn[tt * kTileC + 8 * g + 4 * h]);
      cn[4 * g + 0] = x.x; cn[4 * g + 1] = x.y; cn[4 * g + 2] = x.z; cn[4 * g + 3] = x.w;
    }
    const int cbase = (t0 + tt) * kTileC + 4 * h;
    // independent accumulation chains (one per key tile), interleaved step by
    // step so consecutive MFMAs never wait on each other
    floatx16 acc[kKT];
#pragma unroll
    for (int kt = 0; kt < kKT; ++kt)
      acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b[kt][0], cn, 0, 0, 0);
#pragma unroll
    for (int s = 1; s < kBf16Steps; ++s)
#pragma unroll
      for (int kt = 0; kt < kKT; ++kt)
        acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[s], b[kt][s], acc[kt], 0, 0, 0);
#pragma unroll
    for (int kt = 0; kt < kKT; ++kt) {
      const float m = tile_min(acc[kt]);
      const bool better = m < best[kt];
      // wave-uniform branch: EXEC stays all-ones, lanes select their update.
      // The predicate goes through an opaque register so the compiler cannot
      // turn the selects back into an EXEC-masked block.
      if (__builtin_amdgcn_ballot_w64(better)) {
        int sel = better ? 1 : 0;
        int id = cbase + tile_find(acc[kt], m);
        float m2 = kSecond ? tile_second(acc[kt]) : 0.f;
        asm volatile("" : "+v"(sel), "+v"(id), "+v"(m2));
        if constexpr (kSecond) {
          const float won = __builtin_fminf(__builtin_fminf(sec[kt], m2), bidx[kt] >= 0 ? best[kt] : __builtin_inff());
          sec[kt] = sel ? won : __builtin_fminf(sec[kt], m);
        }
        bidx[kt] = sel ? id : bidx[kt];
        best[kt] = sel ? m : best[kt];
      } else if constexpr (kSecond) {
        sec[kt] = __builtin_fminf(sec[kt], m);
      }
    }
  }
}

// The whole sweep over the centroid stages.  The four ring buffers are
// restrict parameters of this one inlined function, so every asynchronous
// copy and every LDS read below carries alias scopes that tell the compiler
// which buffer it touches; it then waits only where the code says so instead
// of draining all copies in flight before each read.  best/bidx come in
// holding the starting bound (and -1).
template <int kKT, bool kSecond>
__device__ __forceinline__ void bf16_sweep(char* __restrict__ r0, char* __restrict__ r1, char* __restrict__ r2,
                                           char* __restrict__ r3, const uint4* fslice, const float* cslice,
                                           int n_stages, int wave, int lane, int h,
                                           const bf16x8_t (&b)[kKT][kBf16Steps], float (&best)[kKT],
                                           int (&bidx)[kKT], float (&sec)[kKT]) {
  // the first kBf16Ring - 1 stages were copied by the caller (bf16_prologue)
  for (int st = 0; st < n_stages; st += kBf16Ring) {
    bf16_stage<kKT, kSecond>(r0, r3, fslice, cslice, st, n_stages, wave, lane, h, b, best, bidx, sec);
    if (st + 1 >= n_stages) break;
    bf16_stage<kKT, kSecond>(r1, r0, fslice, cslice, st + 1, n_stages, wave, lane, h, b, best, bidx, sec);
    if (st + 2 >= n_stages) break;
    bf16_stage<kKT, kSecond>(r2, r1, fslice, cslice, st + 2, n_stages, wave, lane, h, b, best, bidx, sec);
    if (st + 3 >= n_stages) break;
    bf16_stage<kKT, kSecond>(r3, r2, fslice, cslice, st + 3, n_stages, wave, lane, h, b, best, bidx, sec);
  }
}

// Copies of the first kBf16Ring - 1 stages, issued before anything else the
// block loads, so their latency overlaps the key loads and the bound.
__device__ __forceinline__ void bf16_prologue(char* __restrict__ r0, char* __restrict__ r1, char* __restrict__ r2,
                                              const uint4* fslice, const float* cslice, int n_stages, int wave,
                                              int lane) {
  stage_async(fslice, cslice, 0, r0, wave, lane);
  if (n_stages > 1) stage_async(fslice, cslice, 1, r1, wave, lane);
  if (n_stages > 2) stage_async(fslice, cslice, 2, r2, wave, lane);
}

// What the assignment of a bf16 clustering reads and writes.
struct AssignArgs {
  const uint16_t* keys;
  const uint4* frag;
  const float* cnorm;
  int32_t *assign, *counts;
  int n_tokens, n_clusters, n_ctiles, blocks_per_slice, hist_in_lds;
  uint4* kswz;
  int kswz_mode;
  // from the second iteration of a clustering on (kTrack)
  int32_t* dirty;          // out: clusters that a key entered or left
  float *best, *sec;       // per key: D to its cluster, and a lower bound on D to every other
  const int32_t *ndirty, *dmap, *dlist;   // the clusters recomputed since the last assignment
  int32_t* recorded;       // per slice, two entries used in turn: the last assignment left `best` and `sec`
  int turn;
  int part_percent, record_percent;
  const uint4* cfrag;      // their operands, compacted in ascending order
  const float* ccnorm;
  int32_t *fail, *nfail;   // out: keys left to assign_rest_kernel
};

// A key's move from cluster `from` to `to`: both are recomputed, and counted
// anew (row: the slice's first cluster).
__device__ __forceinline__ void move_key(const AssignArgs& a, size_t row, int from, int to) {
  a.dirty[row + to] = 1;
  atomicAdd(&a.counts[row + to], 1);
  if (from >= 0 && from < a.n_clusters) {
    a.dirty[row + from] = 1;
    atomicSub(&a.counts[row + from], 1);
  }
}

// Sweep over the recomputed clusters alone up to this share of all of them
// (percent); above, the full sweep costs no more and leaves no key over.
// Above the second share the next one will most likely be full too, and a full
// sweep that records takes 5-12% longer, so it records nothing.  The shares fall
// by about ten points an iteration, by more at first where the clusters are well
// apart.  In calls of few (key, centroid) pairs a sweep is short against the
// launch for the left-over keys, and both lines lie lower: a whole call at 70
// and 82 against 80 and 95, keys with noise 0.65 around their centres: 1002 us
// against 1035 for 16 slices of 20480 keys in 640 clusters, 858 against 876 for
// 10 of 25600 in 800, 962 against 978 for 8 of 32768 in 1024, the same for 40 of
// 20480 in 640; noise 0.45, 64 of 32768 in 1024: 5.01 ms against 4.88.
constexpr int kPartPercent = 80, kPartPercentFew = 70;
constexpr int kRecordPercent = 95, kRecordPercentFew = 82;
constexpr double kFewPairs = 1e9;

// Modes of the bf16 assignment: on its own or first of a clustering; later
// iterations, which start from the last assignment (kTrack in the kernel); and
// those that also record `best` and `sec` and may sweep the recomputed
// clusters alone.
constexpr int kAssignPlain = 0, kAssignMoves = 1, kAssignRecord = 2;

// bf16 keys: each wave holds kBf16KeyTiles tiles of 32 keys as MFMA B operands
// for the whole sweep; centroid tiles stream through a ring of kBf16Ring LDS
// stage buffers, copied kBf16Ring - 1 stages ahead.  Lane l owns key column
// l % 32 and rows 8*(v/4) + 4*(l/32) + (v%4) of each 32x32 result, so the
// argmin over a tile is in-lane; the two lane halves merge at the end.
//
// kAssignRecord (third iteration on).  D(k, c) depends on the key and on c's
// operand alone, so it changes only for the clusters the last update
// recomputed.  Every such assignment records, per key, D to its cluster
// (best) and a lower bound on D to all others (sec); the next one then has to
// evaluate the recomputed clusters only:
//  - the key's own cluster was not recomputed: `best` still holds, the
//    clusters not recomputed are no nearer than before, and the argmin is the
//    lower of `best` and the recomputed clusters' minimum (ties to the lower
//    id: the sweep starts just above `best`, so an equal value is found);
//  - it was: the recomputed clusters' minimum is the argmin if it is below
//    `sec`, which bounds every other cluster; if not, the key goes to the
//    fail list and assign_rest_kernel sweeps all centroids for it.
// Both compare the same matrix-core values as the full sweep, so assignments,
// and with them all outputs, are the same bit for bit.  On the benchmark's
// keys (32768 around 1024 centres) 93, 74, 51, 40, 27, 19, 15 and 10% of the
// clusters are recomputed before iterations 3 to 10, and 1.4% of the keys or
// fewer are left over: the ten assignments of 256 such slices take 2.13, 1.83,
// 1.9, 1.6, 1.2, .96, .78, .68, .62 and .59 ms where ten full sweeps took 18.3,
// those of 8 slices 473 us where they took 685 (MI355X).
template <int kMode>
__global__ __launch_bounds__(kBf16Threads, 8 / kBf16Waves)
void assign_bf16_kernel(const AssignArgs a) {
  constexpr bool kTrack = kMode >= kAssignMoves, kRecord = kMode == kAssignRecord;
  __shared__ __align__(16) char s_ring0[kBf16StageBytes];
  __shared__ __align__(16) char s_ring1[kBf16StageBytes];
  __shared__ __align__(16) char s_ring2[kBf16StageBytes];
  __shared__ __align__(16) char s_ring3[kBf16StageBytes];
  static_assert(kBf16Ring == 4, "the stage loop below is unrolled for four buffers");

  const int n_tokens = a.n_tokens, n_clusters = a.n_clusters;
  const int lb = xcd_local_block(blockIdx.x, gridDim.x);
  const int slice = lb / a.blocks_per_slice;
  const int kb = lb - slice * a.blocks_per_slice;
  // the wave index lives in an SGPR (it addresses the copies every stage)
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5,
            j = lane & 31;
  const int key_base = kb * kBf16KeysPerBlock + wave * (32 * kBf16KeyTiles);
  const uint16_t* kslice = a.keys + (size_t)slice * n_tokens * kHeadDim;
  const uint4* fslice = a.frag + (size_t)slice * a.n_ctiles * kBf16TileU4;
  const float* cslice = a.cnorm + (size_t)slice * a.n_ctiles * kTileC;
  int32_t* assign = a.assign + (size_t)slice * n_tokens;
  // the operands swept: all of the slice's, or the recomputed ones
  bool some = false, record = false;
  const uint4* fsweep = fslice;
  const float* csweep = cslice;
  int n_stages = a.n_ctiles / kBf16StageTiles;   // n_ctiles is padded to whole stages
  if constexpr (kRecord) {
    const int nd = __builtin_amdgcn_readfirstlane(a.ndirty[slice]);
    const int had = __builtin_amdgcn_readfirstlane(a.recorded[2 * slice + (a.turn ^ 1)]);
    some = had && nd * 100 <= n_clusters * a.part_percent;
    record = some || nd * 100 <= n_clusters * a.record_percent;
    if (kb == 0 && tid == 0) a.recorded[2 * slice + a.turn] = record ? 1 : 0;
    if (some) {
      if (nd == 0) return;                        // no centroid changed, so no key does
      fsweep = a.cfrag + (size_t)slice * a.n_ctiles * kBf16TileU4;
      csweep = a.ccnorm + (size_t)slice * a.n_ctiles * kTileC;
      n_stages = (nd + kBf16StageTiles * kTileC - 1) / (kBf16StageTiles * kTileC);
    }
  }

  // Start-up latency is the block's fixed cost, so the loads that do not
  // depend on each other are issued together: the ring's first copies, the
  // previous assignment (for the bound), then the keys.
  bf16_prologue(s_ring0, s_ring1, s_ring2, fsweep, csweep, n_stages, wave, lane);
  int zp[kBf16KeyTiles];
#pragma unroll
  for (int kt = 0; kt < kBf16KeyTiles; ++kt) {
    const int key = key_base + kt * 32 + j;
    zp[kt] = (kTrack && key < n_tokens) ? assign[key] : -1;
  }
  // Key operands.  In B-operand order a load instruction touches 64 rows
  // (16 bytes of each), which makes the block's start slow; so the first
  // iteration of a prefill also stores the operands in that order (kswz_mode
  // 1, one contiguous KiB per instruction, padding keys zero), and the later
  // iterations read them back contiguously (kswz_mode 2).
  bf16x8_t b[kBf16KeyTiles][kBf16Steps];
  uint4* zs =
      a.kswz + (((size_t)slice * a.blocks_per_slice + kb) * kBf16Waves + wave) * (kBf16KeyTiles * kBf16Steps * 64);
  if (a.kswz_mode == 2) {
#pragma unroll
    for (int kt = 0; kt < kBf16KeyTiles; ++kt)
#pragma unroll
      for (int s = 0; s < kBf16Steps; ++s) b[kt][s] = __builtin_bit_cast(bf16x8_t, zs[(kt * kBf16Steps + s) * 64 + lane]);
  } else {
#pragma unroll
    for (int kt = 0; kt < kBf16KeyTiles; ++kt) {
      const int key = key_base + kt * 32 + j;
      const uint4* src = reinterpret_cast<const uint4*>(kslice + (size_t)key * kHeadDim + 64 * h);
#pragma unroll
      for (int s = 0; s < kBf16Steps; ++s) {
        uint4 v = key < n_tokens ? src[s] : make_uint4(0, 0, 0, 0);
        b[kt][s] = __builtin_bit_cast(bf16x8_t, v);
      }
    }
    if (a.kswz_mode == 1) {
#pragma unroll
      for (int kt = 0; kt < kBf16KeyTiles; ++kt)
#pragma unroll
        for (int s = 0; s < kBf16Steps; ++s) zs[(kt * kBf16Steps + s) * 64 + lane] = __builtin_bit_cast(uint4, b[kt][s]);
    }
  }
  // Starting bound.  From the second Lloyd iteration on, assign holds the
  // previous assignment; the key's distance to that centroid (computed on the
  // VALU over the same bf16 operands) plus a margin is an upper bound on the
  // matrix-core value of its nearest centroid: both evaluations of D differ
  // from the exact value by at most ~60 x 2^-24 x (||c||^2 + 2 sum|c_i k_i|)
  // <= 7.2e-6 (||c||^2 + ||k||^2), and the margin is 3e-5 of that.  Tiles whose
  // minimum does not beat the bound skip the index search; the nearest
  // centroid's value is strictly below it, so the result is unchanged.
  // In a sweep over the recomputed clusters the bound is the recorded `best`
  // (own cluster not recomputed) or `sec`.
  float best[kBf16KeyTiles], sec[kBf16KeyTiles];
  int bidx[kBf16KeyTiles];
#pragma unroll
  for (int kt = 0; kt < kBf16KeyTiles; ++kt) {
    bidx[kt] = -1;
    best[kt] = __builtin_inff();
    sec[kt] = __builtin_inff();
    const bool have = kTrack && zp[kt] >= 0 && zp[kt] < n_clusters;
    if (some) {
      const int key = key_base + kt * 32 + j;
      if (have)
        best[kt] = a.dmap[(size_t)slice * n_clusters + zp[kt]] < 0 ? next_up(a.best[(size_t)slice * n_tokens + key])
                                                                   : a.sec[(size_t)slice * n_tokens + key];
    } else if (kTrack && __builtin_amdgcn_ballot_w64(have)) {
      typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
      const int zc = have ? zp[kt] : 0;
      // the lane's 64 dimensions of -2 op(c): A-fragment row zc % 32, half h
      const uint4* f = fslice + (size_t)(zc / kTileC) * kBf16TileU4 + (zc % kTileC) + 32 * h;
      float p = 0.f, kk = 0.f;
#pragma unroll
      for (int s = 0; s < kBf16Steps; ++s) {
        const uint4 fa = f[s * 64];
        const uint4 kv = __builtin_bit_cast(uint4, b[kt][s]);
        const uint32_t fw[4] = {fa.x, fa.y, fa.z, fa.w};
        const uint32_t kw[4] = {kv.x, kv.y, kv.z, kv.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const bf16x2_t kq = __builtin_bit_cast(bf16x2_t, kw[q]);
          p = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, fw[q]), kq, p, false);
          kk = __builtin_amdgcn_fdot2_f32_bf16(kq, kq, kk, false);
        }
      }
      p += __shfl_xor(p, 32, kWave);
      kk += __shfl_xor(kk, 32, kWave);
      const float cn = cslice[zc];
      const float u = cn + p + 3e-5f * (cn + kk);
      if (have && u < __builtin_inff()) best[kt] = u;   // false for NaN
    }
  }
  // the key operands are complete before the sweep starts, so no key load is
  // pending inside the stage loop (the loop then only waits for its copies);
  // the compiler does not read that wait, so every key register is also used
  // here, which makes it complete the loads before the loop, not inside it
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int kt = 0; kt < kBf16KeyTiles; ++kt)
#pragma unroll
    for (int s = 0; s < kBf16Steps; ++s) asm volatile("" ::"v"(b[kt][s]));
  if (kRecord && record)
    bf16_sweep<kBf16KeyTiles, true>(s_ring0, s_ring1, s_ring2, s_ring3, fsweep, csweep, n_stages, wave, lane, h, b,
                                    best, bidx, sec);
  else
    bf16_sweep<kBf16KeyTiles, false>(s_ring0, s_ring1, s_ring2, s_ring3, fsweep, csweep, n_stages, wave, lane, h, b,
                                     best, bidx, sec);

  int zi[kBf16KeyTiles];
  bool zv[kBf16KeyTiles];
#pragma unroll
  for (int kt = 0; kt < kBf16KeyTiles; ++kt) {
    const float ob = __shfl_xor(best[kt], 32, kWave);
    const int oi = __shfl_xor(bidx[kt], 32, kWave);
    const float os = kRecord ? __shfl_xor(sec[kt], 32, kWave) : 0.f;
    // a half with no value below its starting bound holds index -1
    const bool other = bidx[kt] < 0 || (oi >= 0 && (ob < best[kt] || (ob == best[kt] && oi < bidx[kt])));
    if constexpr (kRecord) {
      const float lost = other ? (bidx[kt] >= 0 ? best[kt] : __builtin_inff()) : (oi >= 0 ? ob : __builtin_inff());
      sec[kt] = __builtin_fminf(__builtin_fminf(sec[kt], os), lost);
    }
    if (other) {
      best[kt] = ob;
      bidx[kt] = oi;
    }
    const int key = key_base + kt * 32 + j;
    zv[kt] = (h == 0) && key < n_tokens;
    if constexpr (kTrack) {
      const size_t kr = (size_t)slice * n_tokens + key, cr = (size_t)slice * n_clusters;
      int id = bidx[kt];
      float bv = best[kt], sv = sec[kt];
      bool left = false;
      if (some) {
        if (zv[kt]) {
          if (id >= 0) id = a.dlist[cr + id];
          const float bo = a.best[kr], so = a.sec[kr];
          if (a.dmap[cr + zp[kt]] < 0) {
            if (id >= 0 && (bv < bo || (bv == bo && id < zp[kt]))) {
              sv = __builtin_fminf(__builtin_fminf(so, bo), sv);
            } else {
              sv = __builtin_fminf(__builtin_fminf(so, id >= 0 ? bv : __builtin_inff()), sv);
              bv = bo;
              id = zp[kt];
            }
          } else {
            left = id < 0;
            sv = __builtin_fminf(so, sv);
          }
        }
        const uint64_t m = __builtin_amdgcn_ballot_w64(left);
        if (m) {
          int at = 0;
          if (lane == (int)__builtin_ctzll(m)) at = atomicAdd(&a.nfail[slice], __popcll(m));
          at = __shfl(at, (int)__builtin_ctzll(m), kWave);
          if (left)
            a.fail[(size_t)slice * n_tokens + at +
                   __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0))] = key;
        }
      } else if (id < 0) {
        id = 0;   // only reachable with non-finite inputs
        bv = __builtin_inff();
      }
      if (zv[kt] && !left) {
        assign[key] = id;
        if (kRecord && record) {
          a.best[kr] = bv;
          a.sec[kr] = sv;
        }
        // a key that changed cluster marks both clusters for the update and
        // moves from one's count to the other's
        if (id != zp[kt]) move_key(a, cr, zp[kt], id);
      }
    } else {
      if (bidx[kt] < 0) bidx[kt] = 0;   // only reachable with non-finite inputs
      zi[kt] = bidx[kt];
      if (zv[kt]) assign[key] = bidx[kt];
    }
  }
  if (!kTrack && a.counts) {
    __syncthreads();
    block_histogram(reinterpret_cast<int*>(s_ring0), a.hist_in_lds, n_clusters,
                    a.counts + (size_t)slice * n_clusters, zi, zv, kBf16KeyTiles);
  }
}

// The keys that a sweep over the recomputed clusters left over: 32 kKT of a
// slice's list per block, each of its NW waves sweeps every NW-th centroid
// tile for all of them straight from L2, and the waves' results merge in LDS.
// The keys are few and scattered: a block per 512 of them, as above, would
// leave most of the chip idle and its one long sweep would be the iteration's
// time.  A wave's first two tiles are loaded before anything about the keys is
// known.  Few slices: 32 keys a block for the shortest chain; many slices: 64
// keys a block, so that a tile is read from L2 half as often.
template <int kKT, int NW>
__global__ __launch_bounds__(64 * NW)
void assign_rest_kernel(const AssignArgs a, int parts) {
  constexpr int kKeys = 32 * kKT;
  __shared__ float s_best[NW][kKeys], s_sec[NW][kKeys];
  __shared__ int s_idx[NW][kKeys];
  const int slice = blockIdx.x / parts;
  const int part = blockIdx.x - slice * parts;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5,
            j = lane & 31;
  const int32_t* list = a.fail + (size_t)slice * a.n_tokens;
  const uint16_t* kslice = a.keys + (size_t)slice * a.n_tokens * kHeadDim;
  const uint4* fslice = a.frag + (size_t)slice * a.n_ctiles * kBf16TileU4;
  const float* cslice = a.cnorm + (size_t)slice * a.n_ctiles * kTileC;
  auto load_tile = [&](int t, bf16x8_t (&x)[kBf16Steps]) {
    const uint4* f = fslice + (size_t)min(t, a.n_ctiles - 1) * kBf16TileU4 + lane;
#pragma unroll
    for (int s = 0; s < kBf16Steps; ++s) x[s] = __builtin_bit_cast(bf16x8_t, f[s * 64]);
  };
  bf16x8_t x0[kBf16Steps], x1[kBf16Steps];
  load_tile(w, x0);
  const int nf = min(a.nfail[slice], a.n_tokens);
  for (int k0 = part * kKeys; k0 < nf; k0 += parts * kKeys) {
    bf16x8_t b[kKT][kBf16Steps];
    float best[kKT], sec[kKT];
    int bidx[kKT];
#pragma unroll
    for (int kt = 0; kt < kKT; ++kt) {
      const int key = list[min(k0 + kt * 32 + j, nf - 1)];
      const uint4* src = reinterpret_cast<const uint4*>(kslice + (size_t)key * kHeadDim + 64 * h);
#pragma unroll
      for (int s = 0; s < kBf16Steps; ++s) b[kt][s] = __builtin_bit_cast(bf16x8_t, src[s]);
      best[kt] = sec[kt] = __builtin_inff();
      bidx[kt] = -1;
    }
    if (k0 != part * kKeys) load_tile(w, x0);
    auto tile = [&](int t, const bf16x8_t (&x)[kBf16Steps]) {
      floatx16 cn;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 v = *reinterpret_cast<const float4*>(cslice + t * kTileC + 8 * g + 4 * h);
        cn[4 * g + 0] = v.x; cn[4 * g + 1] = v.y; cn[4 * g + 2] = v.z; cn[4 * g + 3] = v.w;
      }
      floatx16 acc[kKT];
#pragma unroll
      for (int kt = 0; kt < kKT; ++kt) acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], b[kt][0], cn, 0, 0, 0);
#pragma unroll
      for (int s = 1; s < kBf16Steps; ++s)
#pragma unroll
        for (int kt = 0; kt < kKT; ++kt)
          acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[s], b[kt][s], acc[kt], 0, 0, 0);
#pragma unroll
      for (int kt = 0; kt < kKT; ++kt) {
        const float m = tile_min(acc[kt]);
        float m2 = tile_second(acc[kt]);
        int id = t * kTileC + 4 * h + tile_find(acc[kt], m);
        int sel = m < best[kt] ? 1 : 0;
        asm volatile("" : "+v"(sel), "+v"(id), "+v"(m2));
        const float won = __builtin_fminf(__builtin_fminf(sec[kt], m2), best[kt]);   // best is +inf until one is found
        sec[kt] = sel ? won : __builtin_fminf(sec[kt], m);
        bidx[kt] = sel ? id : bidx[kt];
        best[kt] = sel ? m : best[kt];
      }
    };
    for (int t = w; t < a.n_ctiles; t += 2 * NW) {
      load_tile(t + NW, x1);
      tile(t, x0);
      if (t + 2 * NW < a.n_ctiles) load_tile(t + 2 * NW, x0);
      if (t + NW < a.n_ctiles) tile(t + NW, x1);
    }
    __syncthreads();   // the last round's results have been read
#pragma unroll
    for (int kt = 0; kt < kKT; ++kt) {
      const float ob = __shfl_xor(best[kt], 32, kWave), os = __shfl_xor(sec[kt], 32, kWave);
      const int oi = __shfl_xor(bidx[kt], 32, kWave);
      const bool other = bidx[kt] < 0 || (oi >= 0 && (ob < best[kt] || (ob == best[kt] && oi < bidx[kt])));
      if (h == 0) {
        s_best[w][kt * 32 + j] = other ? ob : best[kt];
        s_idx[w][kt * 32 + j] = other ? oi : bidx[kt];
        s_sec[w][kt * 32 + j] = __builtin_fminf(__builtin_fminf(sec[kt], os), other ? best[kt] : ob);
      }
    }
    __syncthreads();
    if (tid < kKeys && k0 + tid < nf) {
      const int key = list[k0 + tid];
      const size_t kr = (size_t)slice * a.n_tokens + key;
      const int old = a.assign[kr];
      float bv = __builtin_inff(), sv = __builtin_inff();
      int id = -1;
#pragma unroll
      for (int q = 0; q < NW; ++q) {
        const float ob = s_best[q][tid];
        const int oi = s_idx[q][tid];
        const bool other = oi >= 0 && (id < 0 || ob < bv || (ob == bv && oi < id));
        sv = __builtin_fminf(__builtin_fminf(sv, s_sec[q][tid]), other ? bv : ob);
        if (other) {
          bv = ob;
          id = oi;
        }
      }
      if (id < 0) id = 0;   // only reachable with non-finite inputs
      a.assign[kr] = id;
      a.best[kr] = bv;
      a.sec[kr] = sv;
      if (id != old) move_key(a, (size_t)slice * a.n_clusters, old, id);
    }
  }
}

// fp32 keys: the same scheme with 32x32x2 fp32 MFMAs (64 steps per dot product)
// and one 32-key tile per wave.
__global__ __launch_bounds__(kAssignThreads, 2)
void assign_f32_kernel(const float* __restrict__ keys, const uint4* __restrict__ frag,
                       const float* __restrict__ cnorm, int32_t* __restrict__ assign,
                       int32_t* __restrict__ counts, int n_tokens, int n_clusters, int n_ctiles,
                       int blocks_per_slice, int hist_in_lds) {
  extern __shared__ __align__(16) char smem[];
  uint4* s_frag = reinterpret_cast<uint4*>(smem);
  float* s_cn = reinterpret_cast<float*>(smem + kF32StageTiles * kF32TileU4 * 16);

  const int slice = blockIdx.x / blocks_per_slice;
  const int kb = blockIdx.x - slice * blocks_per_slice;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, h = lane >> 5, j = lane & 31;
  const int key = kb * kF32KeysPerBlock + wave * 32 + j;
  const float* kslice = keys + (size_t)slice * n_tokens * kHeadDim;

  float b[64];
  {
    const float4* src = reinterpret_cast<const float4*>(kslice + (size_t)key * kHeadDim + 64 * h);
#pragma unroll
    for (int s4 = 0; s4 < 16; ++s4) {
      float4 v = key < n_tokens ? src[s4] : make_float4(0.f, 0.f, 0.f, 0.f);
      b[4 * s4 + 0] = v.x; b[4 * s4 + 1] = v.y; b[4 * s4 + 2] = v.z; b[4 * s4 + 3] = v.w;
    }
  }
  float best = __builtin_inff();
  int bidx = 0;
  const uint4* fslice = frag + (size_t)slice * n_ctiles * kF32TileU4;
  const float* cslice = cnorm + (size_t)slice * n_ctiles * kTileC;
  for (int t0 = 0; t0 < n_ctiles; t0 += kF32StageTiles) {
    const int nt = min(kF32StageTiles, n_ctiles - t0);
    __syncthreads();
    for (int i = tid; i < nt * kF32TileU4; i += kAssignThreads) s_frag[i] = fslice[(size_t)t0 * kF32TileU4 + i];
    for (int i = tid; i < nt * kTileC; i += kAssignThreads) s_cn[i] = cslice[t0 * kTileC + i];
    __syncthreads();
    for (int tt = 0; tt < nt; ++tt) {
      floatx16 acc;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 x = *reinterpret_cast<const float4*>(&s_cn[tt * kTileC + 8 * g + 4 * h]);
        acc[4 * g + 0] = x.x; acc[4 * g + 1] = x.y; acc[4 * g + 2] = x.z; acc[4 * g + 3] = x.w;
      }
#pragma unroll
      for (int s4 = 0; s4 < 16; ++s4) {
        const float4 a4 = __builtin_bit_cast(float4, s_frag[(tt * 16 + s4) * 64 + lane]);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.x, b[4 * s4 + 0], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.y, b[4 * s4 + 1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.z, b[4 * s4 + 2], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a4.w, b[4 * s4 + 3], acc, 0, 0, 0);
      }
      const int cbase = (t0 + tt) * kTileC + 4 * h;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float x = acc[v];
        const int c = cbase + 8 * (v >> 2) + (v & 3);
        if (x < best) { best = x; bidx = c; }
      }
    }
  }
  const float ob = __shfl_xor(best, 32, kWave);
  const int oi = __shfl_xor(bidx, 32, kWave);
  if (ob < best || (ob == best && oi < bidx)) { best = ob; bidx = oi; }
  const bool valid = (h == 0) && key < n_tokens;
  if (valid) assign[(size_t)slice * n_tokens + key] = bidx;
  if (counts) {
    __syncthreads();
    int zi[1] = {bidx};
    bool zv[1] = {valid};
    block_histogram(reinterpret_cast<int*>(smem), hist_in_lds, n_clusters,
                    counts + (size_t)slice * n_clusters, zi, zv, 1);
  }
}

constexpr int kCountKeys = 1024;

// counts[s][c] = number of keys with assign == c (used by the standalone update).
__global__ void count_kernel(const int32_t* __restrict__ assign, int32_t* __restrict__ counts, int n_tokens,
                             int n_clusters, int blocks_per_slice, int hist_in_lds) {
  extern __shared__ __align__(16) char smem[];
  const int slice = blockIdx.x / blocks_per_slice;
  const int kb = blockIdx.x - slice * blocks_per_slice;
  int zi[4];
  bool zv[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = kb * kCountKeys + q * 256 + threadIdx.x;
    zv[q] = i < n_tokens;
    zi[q] = zv[q] ? assign[(size_t)slice * n_tokens + i] : 0;
    zv[q] = zv[q] && zi[q] >= 0 && zi[q] < n_clusters;
  }
  block_histogram(reinterpret_cast<int*>(smem), hist_in_lds, n_clusters,
                  counts + (size_t)slice * n_clusters, zi, zv, 4);
}

// Per slice: offsets[c] = sum of counts[<c], offsets[C] = total; cursor =
// offsets.  Only for more clusters than scatter_kernel scans in LDS.
__global__ __launch_bounds__(1024)
void scan_kernel(const int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
                 int32_t* __restrict__ cursor, int n_clusters) {
  __shared__ int s_warp[16];
  __shared__ int s_carry;
  const int slice = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int32_t* cnt = counts + (size_t)slice * n_clusters;
  int32_t* off = offsets + (size_t)slice * (n_clusters + 1);
  int32_t* cur = cursor + (size_t)slice * n_clusters;
  if (tid == 0) s_carry = 0;
  __syncthreads();
  for (int base = 0; base < n_clusters; base += 1024) {
    const int c = base + tid;
    const int v = c < n_clusters ? cnt[c] : 0;
    int x = v;  // inclusive wave scan
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o, kWave);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_warp[w] = x;
    __syncthreads();
    int wprefix = 0;
    for (int q = 0; q < w; ++q) wprefix += s_warp[q];
    const int carry = s_carry;
    const int excl = carry + wprefix + x - v;
    if (c < n_clusters) {
      off[c] = excl;
      cur[c] = excl;
    }
    __syncthreads();
    if (tid == 1023) s_carry = excl + v;
    __syncthreads();
  }
  if (tid == 0) off[n_clusters] = s_carry;
}

constexpr int kScatterKeys = 1024;   // keys per block (scatter_kernel: 256 * its kPer)

// members[s][cursor[z]++] = i for every key i, with cursors from scan_kernel.
__global__ void scatter_global_kernel(const int32_t* __restrict__ assign, int32_t* __restrict__ cursor,
                                      int32_t* __restrict__ members, int n_tokens, int n_clusters,
                                      int blocks_per_slice) {
  const int slice = blockIdx.x / blocks_per_slice;
  const int kb = blockIdx.x - slice * blocks_per_slice;
  int32_t* cur = cursor + (size_t)slice * n_clusters;
  int32_t* mem = members + (size_t)slice * n_tokens;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int i = kb * kScatterKeys + q * 256 + threadIdx.x;
    const int z = i < n_tokens ? assign[(size_t)slice * n_tokens + i] : -1;
    if (z >= 0 && z < n_clusters) mem[atomicAdd(&cur[z], 1)] = i;   // same keys as the count
  }
}

// Exclusive block-wide scan of one value per thread (256 threads); returns
// the total.  s_w: 4 ints of LDS.
__device__ __forceinline__ int block256_scan(int v, int* s_w, int& excl) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o, kWave);
    if (lane >= o) x += y;
  }
  __syncthreads();   // s_w of an earlier scan has been read
  if (lane == 63) s_w[w] = x;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int t = s_w[q];
    before += q < w ? t : 0;
    total += t;
  }
  excl = before + x - v;
  return total;
}

// CSR offsets and member lists in one launch: every block scans its slice's
// counts in LDS (C ints from L2; a launch of its own for the scan cost 3-5 us
// an iteration), then places its 1024 keys: members[s][offsets[z] + k] = i, k
// unique per key (an LDS count per block, one global atomic per block and
// cluster on `cursor`, which is zero before the launch and cleared again by
// the update).  Block 0 of a slice writes the offsets.
// With `dirty` only the keys of flagged clusters are placed, the ones the
// update reads, and block 0 writes the list of those clusters in ascending
// order, each one's place in it (dmap, -1 for the others) and its length, and
// empties the list of left-over keys for the next assignment.
template <int kPer>
__global__ __launch_bounds__(256)
void scatter_kernel(const int32_t* __restrict__ assign, const int32_t* __restrict__ counts,
                    int32_t* __restrict__ cursor, int32_t* __restrict__ offsets, int32_t* __restrict__ members,
                    int n_tokens, int n_clusters, int blocks_per_slice, const int32_t* __restrict__ dirty,
                    int32_t* __restrict__ dlist, int32_t* __restrict__ dmap, int32_t* __restrict__ ndirty,
                    int32_t* __restrict__ nfail, uint4* __restrict__ cfrag, float* __restrict__ ccnorm, int n_ctiles,
                    int place_all, int32_t* __restrict__ clear_recorded) {
  extern __shared__ __align__(16) char smem[];
  __shared__ int s_w[4];
  int* hist = reinterpret_cast<int*>(smem);
  int* base = hist + n_clusters;
  const int slice = blockIdx.x / blocks_per_slice;
  const int kb = blockIdx.x - slice * blocks_per_slice;
  const int tid = threadIdx.x;
  const size_t crow = (size_t)slice * n_clusters;
  const int32_t* dr = dirty ? dirty + crow : nullptr;
  int32_t* mem = members + (size_t)slice * n_tokens;
  int z[kPer], pos[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int i = kb * (256 * kPer) + q * 256 + tid;
    z[q] = i < n_tokens ? assign[(size_t)slice * n_tokens + i] : -1;
    if (z[q] >= n_clusters) z[q] = -1;   // same keys as the count
  }
  // counts, the top bit set for the clusters not to be placed
  constexpr int kSkip = 1 << 31;
  for (int i = tid; i < n_clusters; i += 256) hist[i] = counts[crow + i] | (dr && !dr[i] ? kSkip : 0);
  __syncthreads();
  // a thread's run of consecutive clusters
  const int per = (n_clusters + 255) / 256;
  const int c0 = min(tid * per, n_clusters), c1 = min(c0 + per, n_clusters);
  int sum = 0;
  int nd = 0;
  for (int c = c0; c < c1; ++c) {
    sum += hist[c] & ~kSkip;
    nd += hist[c] >= 0;
  }
  int at;
  const int total = block256_scan(sum, s_w, at);
  for (int c = c0; c < c1; ++c) {
    const int n = hist[c];
    base[c] = at | (n & kSkip);
    hist[c] = 0;
    at += n & ~kSkip;
  }
  __syncthreads();
  if (kb == 0) {
    int32_t* off = offsets + (size_t)slice * (n_clusters + 1);
    for (int i = tid; i < n_clusters; i += 256) off[i] = base[i] & ~kSkip;
    if (tid == 0) off[n_clusters] = total;
    if (dr) {
      int k;
      const int all = block256_scan(nd, s_w, k);
      for (int c = c0; c < c1; ++c) {
        const bool d = base[c] >= 0;
        dmap[crow + c] = d ? k : -1;
        if (d) dlist[crow + k++] = c;
      }
      // the compacted operand's last stage is padded with rows that never win
      constexpr int kStageC = kBf16StageTiles * kTileC;
      const int pad = cfrag ? (all + kStageC - 1) / kStageC * kStageC - all : 0;
      for (int i = tid; i < pad * 16; i += 256) {
        const int r = all + i / 16, q = i % 16;   // 16-byte piece q of row r
        cfrag[((size_t)slice * n_ctiles + r / kTileC) * kBf16TileU4 + (q & 7) * 64 + (q >> 3) * 32 + r % kTileC] =
            make_uint4(0, 0, 0, 0);
        if (q == 0) ccnorm[(size_t)slice * n_ctiles * kTileC + r] = __builtin_inff();
      }
      if (tid == 0) {
        ndirty[slice] = all;
        nfail[slice] = 0;
        if (clear_recorded) clear_recorded[2 * slice] = clear_recorded[2 * slice + 1] = 0;
      }
    }
  }
  if (dr && !place_all) {
#pragma unroll
    for (int q = 0; q < kPer; ++q)
      if (z[q] >= 0 && base[z[q]] < 0) z[q] = -1;
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) pos[q] = z[q] >= 0 ? atomicAdd(&hist[z[q]], 1) : 0;
  __syncthreads();
  for (int i = tid; i < n_clusters; i += 256)
    if (hist[i]) base[i] = (base[i] & ~kSkip) + atomicAdd(&cursor[crow + i], hist[i]);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q)
    if (z[q] >= 0) mem[base[z[q]] + pos[q]] = kb * (256 * kPer) + q * 256 + tid;
}

// Mean of a cluster's member keys, float64 sum; kSplit waves per (slice,
// cluster).  A key row is read as 16-byte pieces: kLpr lanes per row, so one
// wave load covers kRpl rows and kUnroll loads are in flight; each lane
// accumulates its dims in float64, the row groups are summed across lanes and
// the waves' parts through LDS at the end.  Where waves share a cluster, and in
// bf16 where one has kBatchIdsMembers members or more on average, a wave loads
// each batch's ids with the rows of the batch before; otherwise 64 ids at a time,
// a lane each, handed out by shuffles.
// One wave a cluster reads the rows at the rate HBM gives them once there are
// clusters enough to fill the chip; below that the longest member list is the
// kernel's time, and a block's waves share it.
// With dirty only the flagged clusters are recomputed (a cluster that no key
// entered or left keeps its members, hence its mean and the operand prepared
// from it) and their flags cleared for the next assignment; with dlist (many
// clusters in all) each wave takes every `stride_e`-th cluster of the slice's
// list, without it a wave or block per cluster looks at its flag, which is one
// dependent load less (8192 clusters: 13.3 us against 16.7).  The flag is the
// place in the list, or where the scatter wrote none (more clusters than it
// scans in LDS) `dirty` itself.
// With frag given, the wave also writes the next iteration's matrix operand
// for this centroid (-2 op(c) in A-fragment order, and ||op(c)||^2), the work
// prep_operand_kernel does for the first iteration.  The clusters' scatter
// cursors, and with zero_counts their counts, are cleared for the next
// iteration.
template <class T>
struct UpdateArgs {
  const T* keys;
  const int32_t *members, *offsets;
  int32_t *counts, *cursor;
  const float* cin;
  float* cout;
  int stride, n_tokens, n_clusters;
  int blocks_per_slice, stride_e;      // entries (clusters) a slice's waves or blocks take at once
  uint4* frag;
  float* cnorm;
  int n_ctiles, zero_counts;
  int32_t *dirty, *dlist, *dmap, *ndirty;
  uint4* cfrag;       // the recomputed clusters' operands in list order, or NULL
  float* ccnorm;
};

template <class T, int kSplit, bool kBatchIds = (kSplit > 1)>
__global__ __launch_bounds__((kSplit > 4 ? 64 * kSplit : 256))
void centroid_update_kernel(const UpdateArgs<T> a) {
  constexpr int kDims = 16 / sizeof(T);          // dims per 16-byte piece (8 bf16, 4 fp32)
  constexpr int kLpr = kHeadDim / kDims;         // lanes per row
  constexpr int kRpl = kWave / kLpr;             // rows per wave load
  constexpr int kUnroll = sizeof(T) == 2 || kSplit == 1 ? 4 : 8;
  constexpr int kBatch = kRpl * kUnroll;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t s = blockIdx.x / a.blocks_per_slice;
  const int blk = (int)(blockIdx.x - s * a.blocks_per_slice);
  const int part = kSplit > 1 ? w : 0;
  const int lane = threadIdx.x & 63;
  const int sub = lane % kLpr, grp = lane / kLpr;
  const int n_entries = a.dlist ? a.ndirty[s] : a.n_clusters;
  const bool track = a.dirty != nullptr;
  const size_t crow = (size_t)s * a.n_clusters;
  for (int e = kSplit > 1 ? blk : blk * 4 + w; e < n_entries; e += a.stride_e) {
    const int c = a.dlist ? a.dlist[crow + e] : e;
    // place in the slice's list, or -1
    const int slot = !track ? 0 : a.dlist ? e : a.dmap ? a.dmap[crow + c] : a.dirty[crow + c] ? 0 : -1;
    const bool clean = slot < 0;
    if (kSplit == 1 && clean) continue;   // before anything else is loaded: most waves of late iterations end here
    const int n = a.counts[crow + c];
    const int off = a.offsets[(size_t)s * (a.n_clusters + 1) + c];
    float* dst = a.cout + ((size_t)s * a.stride + c) * kHeadDim;
    if constexpr (kSplit > 1) __syncthreads();   // every wave has read the count and the flag before one clears them
    if (clean) continue;
    // after the row loads, which would otherwise wait for these stores (a wave's
    // memory operations complete in order)
    auto clear = [&]() {
      if (lane == 0 && part == 0) {
        if (track) a.dirty[crow + c] = 0;
        if (a.cursor) a.cursor[crow + c] = 0;
        if (a.zero_counts) a.counts[crow + c] = 0;
      }
    };
    if (n == 0) {
      clear();
      // empty: the centroid (and its operand from the previous preparation) stay
      if (a.cin != a.cout && part == 0) {
        const float* src = a.cin + ((size_t)s * a.stride + c) * kHeadDim;
        dst[2 * lane] = src[2 * lane];
        dst[2 * lane + 1] = src[2 * lane + 1];
      }
      // in the list all the same: its operand goes to its place there
      if (a.cfrag && a.frag && part == 0 && lane < 16) {
        const int at = (lane & 7) * 64 + (lane >> 3) * 32;
        a.cfrag[((size_t)s * a.n_ctiles + slot / kTileC) * kBf16TileU4 + at + slot % kTileC] =
            a.frag[((size_t)s * a.n_ctiles + c / kTileC) * kBf16TileU4 + at + c % kTileC];
        if (lane == 0)
          a.ccnorm[(size_t)s * a.n_ctiles * kTileC + slot] = a.cnorm[(size_t)s * a.n_ctiles * kTileC + c];
      }
      continue;
    }
    const int32_t* mem = a.members + (size_t)s * a.n_tokens + off;
    const T* kslice = a.keys + (size_t)s * a.n_tokens * kHeadDim;
    double acc[kDims];
#pragma unroll
    for (int d = 0; d < kDims; ++d) acc[d] = 0.0;
    auto load_row = [&](int id, bool ok) {
      return ok ? reinterpret_cast<const uint4*>(kslice + (size_t)id * kHeadDim)[sub] : make_uint4(0, 0, 0, 0);
    };
    auto add_rows = [&](const uint4 (&x)[kUnroll]) {
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const T* v = reinterpret_cast<const T*>(&x[u]);
#pragma unroll
        for (int d = 0; d < kDims; ++d) acc[d] += (double)load_as_f32(v, d);
      }
    };
    if constexpr (!kBatchIds) {
      static_assert(kSplit == 1, "a wave's own members");
      int next = lane < n ? mem[lane] : 0;
      for (int m0 = 0; m0 < n; m0 += kWave) {   // 64 member ids at a time, a lane each
        const int mine = next;
        const int cnt = min(kWave, n - m0);
        if (m0 + kWave < n) next = m0 + kWave + lane < n ? mem[m0 + kWave + lane] : 0;   // ahead of the rows
        for (int q = 0; q < cnt; q += kBatch) {
          uint4 x[kUnroll];
#pragma unroll
          for (int u = 0; u < kUnroll; ++u) {
            const int r = q + u * kRpl + grp;
            x[u] = load_row(__shfl(mine, r & (kWave - 1), kWave), r < cnt);
          }
          add_rows(x);
        }
      }
    } else {
      int tok[kUnroll];
      auto load_ids = [&](int m0) {
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
          const int r = m0 + u * kRpl + grp;
          tok[u] = r < n ? mem[r] : -1;
        }
      };
      load_ids(part * kBatch);
      for (int m0 = part * kBatch; m0 < n; m0 += kSplit * kBatch) {
        uint4 x[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) x[u] = load_row(tok[u], tok[u] >= 0);
        load_ids(m0 + kSplit * kBatch);
        add_rows(x);
      }
    }
    clear();
#pragma unroll
    for (int o = kLpr; o < kWave; o <<= 1)
#pragma unroll
      for (int d = 0; d < kDims; ++d) acc[d] += __shfl_xor(acc[d], o, kWave);
    if constexpr (kSplit > 1) {
      __shared__ double s_part[kSplit - 1][kHeadDim];
      if (part > 0 && grp == 0)
#pragma unroll
        for (int d = 0; d < kDims; ++d) s_part[part - 1][kDims * sub + d] = acc[d];
      __syncthreads();
      if (part > 0) continue;
      for (int q = 0; q < kSplit - 1; ++q)
#pragma unroll
        for (int d = 0; d < kDims; ++d) acc[d] += s_part[q][kDims * sub + d];
    }
    if (grp != 0) continue;
    // lanes 0..kLpr-1 hold dims kDims*lane ..
    float mean[kDims];
#pragma unroll
    for (int d = 0; d < kDims; ++d) mean[d] = (float)(acc[d] / (double)n);
    float4* d4 = reinterpret_cast<float4*>(dst + kDims * sub);
#pragma unroll
    for (int d = 0; d < kDims; d += 4) d4[d / 4] = make_float4(mean[d], mean[d + 1], mean[d + 2], mean[d + 3]);
    if (!a.frag) continue;
    // next iteration's operand: same layout and values as prep_operand_kernel
    const int t = c / kTileC, ci = c % kTileC;
    const int d0 = kDims * sub, hh = d0 >> 6;
    const int flane = hh * 32 + ci;
    double nrm = 0.0;
    if (sizeof(T) == 2) {
      uint32_t wd[4];
#pragma unroll
      for (int d = 0; d < 8; d += 2) {
        const float o0 = bf16_to_f32(f32_to_bf16(mean[d])), o1 = bf16_to_f32(f32_to_bf16(mean[d + 1]));
        nrm += (double)o0 * o0 + (double)o1 * o1;
        wd[d / 2] = (uint32_t)f32_to_bf16(-2.f * o0) | ((uint32_t)f32_to_bf16(-2.f * o1) << 16);
      }
      const int step = (d0 & 63) >> 3;
      const uint4 op = make_uint4(wd[0], wd[1], wd[2], wd[3]);
      a.frag[((size_t)s * a.n_ctiles + t) * kBf16TileU4 + step * 64 + flane] = op;
      if (a.cfrag)
        a.cfrag[((size_t)s * a.n_ctiles + slot / kTileC) * kBf16TileU4 + step * 64 + hh * 32 + slot % kTileC] = op;
    } else {
#pragma unroll
      for (int d = 0; d < kDims; ++d) nrm += (double)mean[d] * mean[d];
      const int step = d0 & 63;   // 4 consecutive steps, one float4 of the fp32 layout
      float* f = reinterpret_cast<float*>(a.frag + ((size_t)s * a.n_ctiles + t) * kF32TileU4);
      *reinterpret_cast<float4*>(f + ((size_t)(step >> 2) * 64 + flane) * 4) =
          make_float4(-2.f * mean[0], -2.f * mean[1], -2.f * mean[2], -2.f * mean[3]);
    }
#pragma unroll
    for (int o = 1; o < kLpr; o <<= 1) nrm += __shfl_xor(nrm, o, kWave);
    if (sub == 0) {
      a.cnorm[(size_t)s * a.n_ctiles * kTileC + c] = (float)nrm;
      if (a.cfrag) a.ccnorm[(size_t)s * a.n_ctiles * kTileC + slot] = (float)nrm;
    }
  }
}

// One wave per (slice, cluster): member ids sorted ascending into perm, and the
// unit-table entry.  Up to 64 members sit in one register a lane and a member's
// rank is the number of smaller ids (a readlane and a compare for each member;
// ids are distinct).  Larger clusters go through a bitmap of kFinalIds token
// ids in the wave's LDS, window by window: a set bit's position among the set
// bits is its rank, so the cost is the members plus a pass over the bitmap
// whatever the cluster's size.  Ranks counted through ds_bpermute, and above
// 64 members with a global load per pair of members, took 151 us for 8 slices
// of 4096 float32 keys in 64 clusters (now 9.6), 40 us for 8 of 32768 bf16 keys
// in 1024 (9.7) and 232 us for 256 such slices (112).
constexpr int kFinalIds = 16384;                 // ids per window: 2 KiB of LDS a wave
constexpr int kFinalWords = kFinalIds / 32;
constexpr int kFinalPerLane = kFinalWords / 64;   // consecutive words a lane emits

__global__ __launch_bounds__(256)
void finalize_kernel(const int32_t* __restrict__ members, const int32_t* __restrict__ offsets,
                     const int32_t* __restrict__ counts, int32_t* __restrict__ perm,
                     int32_t* __restrict__ unit_start, int32_t* __restrict__ unit_size, int units_cap, int n_tokens,
                     int n_clusters, int64_t n_rows) {
  __shared__ uint32_t s_bits[4][kFinalWords];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row = (int64_t)blockIdx.x * 4 + w;
  if (row >= n_rows) return;
  const int lane = threadIdx.x & 63;
  const int64_t s = row / n_clusters;
  const int c = (int)(row - s * n_clusters);
  const int n = counts[s * n_clusters + c];
  const int off = offsets[s * (n_clusters + 1) + c];
  if (lane == 0) {
    unit_start[s * units_cap + c] = off;
    unit_size[s * units_cap + c] = n;
  }
  const int32_t* mem = members + (size_t)s * n_tokens + off;
  int32_t* out = perm + (size_t)s * n_tokens + off;
  if (n <= kWave) {
    const int mine = lane < n ? mem[lane] : 0x7fffffff;
    int rank = 0;
    for (int q = 0; q < n; ++q) rank += __builtin_amdgcn_readlane(mine, q) < mine;
    if (lane < n) out[rank] = mine;
    return;
  }
  // the wave's own slot, so no block barrier: a wave's LDS operations complete
  // in order, the fences keep the compiler from reordering them
  uint32_t* bits = s_bits[w];
  int done = 0;   // members of the windows before this one
  for (int base = 0; base < n_tokens; base += kFinalIds) {
#pragma unroll
    for (int i = 0; i < kFinalPerLane; ++i) bits[i * 64 + lane] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int i = lane; i < n; i += kWave) {
      const int id = mem[i] - base;
      if (id >= 0 && id < kFinalIds) atomicOr(&bits[id >> 5], 1u << (id & 31));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t word[kFinalPerLane];
    int cnt = 0;
#pragma unroll
    for (int i = 0; i < kFinalPerLane; ++i) {
      word[i] = bits[lane * kFinalPerLane + i];
      cnt += __popc(word[i]);
    }
    int incl = cnt;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    int at = done + incl - cnt;
    done += __shfl(incl, kWave - 1, kWave);
#pragma unroll
    for (int i = 0; i < kFinalPerLane; ++i) {
      uint32_t x = word[i];
      while (x) {
        out[at++] = base + (lane * kFinalPerLane + i) * 32 + __builtin_ctz(x);
        x &= x - 1;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// ---------------------------------------------------------------------------
// Clustering of a short prompt in one launch: a block per slice runs the
// initial centroids, every Lloyd iteration and the CSR, perm and unit outputs,
// its keys in registers as matrix B operands (wave w holds the 32-key tiles
// w, w + 16, ..) and the centroid operands, the assignment, counts and member
// lists in LDS.  The launches above take 3-8 us each whatever their size, four
// an iteration; here an iteration is a chain of barriers and one gather of
// the member rows of the clusters that keys entered or left, from L2.  Same
// matrix-core values, order of ties and means as those launches, so the same
// outputs.  8 slices of 500 keys in 16 clusters: 175 -> 67 us, 256 of 1024 keys
// in 32: 445 -> 181 us (sixteen waves; eight took 74 and 202).  It serves what
// fits one block's registers (1024 keys) and a few operand tiles; a block per
// slice is also fastest where slices are few, as the launches it replaces are
// latency alone there, and at its limits: 1024 keys in 128 clusters, 1, 8, 64,
// 256 and 512 slices: 218 -> 157, 229 -> 166, 281 -> 178, 499 -> 209 and 853 ->
// 382 us; 512 keys in 128: 202 -> 102, .., 556 -> 247.
struct SmallArgs {
  const uint16_t* keys;
  const int32_t* init_idx;
  float* reps;
  int32_t *unit_start, *unit_size, *assign, *perm;
  int n_tokens, n_clusters, units_cap, n_iters;
};

constexpr int kSmallWaves = 16;
constexpr int kSmallKeys = 32 * 2 * kSmallWaves;   // 1024: two key tiles a wave
constexpr int kSmallTiles = 4;                     // centroid tiles (32 KiB of operands)
constexpr int kSmallClusters = kSmallTiles * kTileC;

// Lane l < 16 holds dims 8 l .. 8 l + 7 of a centroid: its operand -2 op(c)
// into row `c` of the A-fragment tiles and ||op(c)||^2 (every lane of the 16).
__device__ __forceinline__ void small_operand(const float (&v)[8], int c, int l, uint4* s_frag, float* s_cn) {
  uint32_t wd[4];
  double nrm = 0.0;
#pragma unroll
  for (int d = 0; d < 8; d += 2) {
    const float o0 = bf16_to_f32(f32_to_bf16(v[d])), o1 = bf16_to_f32(f32_to_bf16(v[d + 1]));
    nrm += (double)o0 * o0 + (double)o1 * o1;
    wd[d / 2] = (uint32_t)f32_to_bf16(-2.f * o0) | ((uint32_t)f32_to_bf16(-2.f * o1) << 16);
  }
  s_frag[(c / kTileC) * kBf16TileU4 + (l & 7) * 64 + (l >> 3) * 32 + c % kTileC] = make_uint4(wd[0], wd[1], wd[2], wd[3]);
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) nrm += __shfl_xor(nrm, o, kWave);
  if (l == 0) s_cn[c] = (float)nrm;
}

template <int kKT>
__global__ __launch_bounds__(64 * kSmallWaves)
void lloyd_small_kernel(const SmallArgs a) {
  __shared__ uint4 s_frag[kSmallTiles * kBf16TileU4];
  __shared__ float s_cn[kSmallClusters];
  __shared__ int s_assign[kSmallKeys], s_mem[kSmallKeys];
  __shared__ int s_cnt[kSmallClusters], s_off[kSmallClusters], s_cur[kSmallClusters], s_dirty[kSmallClusters];
  __shared__ uint32_t s_bits[kSmallWaves][kSmallKeys / 32];
  constexpr int kRows = kKT == 1 ? 8 : 4;   // row loads in flight a lane
  const int64_t s = blockIdx.x;
  const int N = a.n_tokens, C = a.n_clusters;
  const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5,
            j = lane & 31, sub = lane & 15, grp = lane >> 4;
  const int n_tiles = (C + kTileC - 1) / kTileC;
  const uint16_t* kslice = a.keys + (size_t)s * N * kHeadDim;
  float* reps = a.reps + (size_t)s * a.units_cap * kHeadDim;

  // the keys, and the initial centroids (four a wave at a time)
  bf16x8_t b[kKT][kBf16Steps];
#pragma unroll
  for (int kt = 0; kt < kKT; ++kt) {
    const int key = 32 * (w + kt * kSmallWaves) + j;
    const uint4* src = reinterpret_cast<const uint4*>(kslice + (size_t)key * kHeadDim + 64 * h);
#pragma unroll
    for (int t = 0; t < kBf16Steps; ++t)
      b[kt][t] = __builtin_bit_cast(bf16x8_t, key < N ? src[t] : make_uint4(0, 0, 0, 0));
  }
  for (int c0 = 4 * w; c0 < n_tiles * kTileC; c0 += 4 * kSmallWaves) {
    const int c = c0 + grp;
    float v[8] = {};
    if (c < C) {
      const int t = min(max(a.init_idx[s * C + c], 0), N - 1);
      const uint4 x = reinterpret_cast<const uint4*>(kslice + (size_t)t * kHeadDim)[sub];
      const uint16_t* e = reinterpret_cast<const uint16_t*>(&x);
#pragma unroll
      for (int d = 0; d < 8; ++d) v[d] = bf16_to_f32(e[d]);
      float4* dst = reinterpret_cast<float4*>(reps + (size_t)c * kHeadDim + 8 * sub);
      dst[0] = make_float4(v[0], v[1], v[2], v[3]);
      dst[1] = make_float4(v[4], v[5], v[6], v[7]);
    }
    small_operand(v, c, sub, s_frag, s_cn);
    if (c >= C && sub == 0) s_cn[c] = __builtin_inff();   // padding rows never win
  }
  for (int i = tid; i < kSmallKeys; i += 64 * kSmallWaves) s_assign[i] = -1;
  if (tid < kSmallClusters) {
    s_cnt[tid] = 0;
    s_dirty[tid] = 1;
  }
  __syncthreads();

  for (int it = 0; it < a.n_iters; ++it) {
    const bool last = it + 1 == a.n_iters;
    float best[kKT];
    int bidx[kKT];
#pragma unroll
    for (int kt = 0; kt < kKT; ++kt) {
      best[kt] = __builtin_inff();
      bidx[kt] = -1;
    }
    for (int t = 0; t < n_tiles; ++t) {
      floatx16 cn;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 x = *reinterpret_cast<const float4*>(&s_cn[t * kTileC + 8 * g + 4 * h]);
        cn[4 * g + 0] = x.x; cn[4 * g + 1] = x.y; cn[4 * g + 2] = x.z; cn[4 * g + 3] = x.w;
      }
      floatx16 acc[kKT];
#pragma unroll
      for (int q = 0; q < kBf16Steps; ++q) {
        const bf16x8_t x = __builtin_bit_cast(bf16x8_t, s_frag[t * kBf16TileU4 + q * 64 + lane]);
#pragma unroll
        for (int kt = 0; kt < kKT; ++kt)
          acc[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, b[kt][q], q == 0 ? cn : acc[kt], 0, 0, 0);
      }
#pragma unroll
      for (int kt = 0; kt < kKT; ++kt) {
        const float m = tile_min(acc[kt]);
        int id = t * kTileC + 4 * h + tile_find(acc[kt], m);
        int sel = m < best[kt] ? 1 : 0;
        asm volatile("" : "+v"(sel), "+v"(id));
        bidx[kt] = sel ? id : bidx[kt];
        best[kt] = sel ? m : best[kt];
      }
    }
#pragma unroll
    for (int kt = 0; kt < kKT; ++kt) {
      const float ob = __shfl_xor(best[kt], 32, kWave);
      const int oi = __shfl_xor(bidx[kt], 32, kWave);
      if (bidx[kt] < 0 || (oi >= 0 && (ob < best[kt] || (ob == best[kt] && oi < bidx[kt])))) bidx[kt] = oi;
      if (bidx[kt] < 0) bidx[kt] = 0;   // only reachable with non-finite inputs
      const int key = 32 * (w + kt * kSmallWaves) + j;
      if (h == 0 && key < N) {
        const int old = s_assign[key], id = bidx[kt];
        if (id != old) {
          s_assign[key] = id;
          s_dirty[id] = 1;
          atomicAdd(&s_cnt[id], 1);
          if (old >= 0) {
            s_dirty[old] = 1;
            atomicSub(&s_cnt[old], 1);
          }
        }
      }
    }
    __syncthreads();
    if (w == 0) {   // offsets: lane l scans clusters 2l, 2l + 1
      const int c0 = 2 * lane;
      const int n0 = c0 < C ? s_cnt[c0] : 0, n1 = c0 + 1 < C ? s_cnt[c0 + 1] : 0;
      int x = n0 + n1;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
      }
      s_off[c0] = s_cur[c0] = x - n0 - n1;
      s_off[c0 + 1] = s_cur[c0 + 1] = x - n1;
    }
    __syncthreads();
    for (int i = tid; i < N; i += 64 * kSmallWaves) {
      const int z = s_assign[i];
      if (last || s_dirty[z]) s_mem[atomicAdd(&s_cur[z], 1)] = i;
    }
    __syncthreads();
    // means of the flagged clusters, one wave each, 4 kRows rows in flight
    for (int c = w; c < C; c += kSmallWaves) {
      const int n = s_cnt[c];
      const bool flagged = s_dirty[c] != 0;
      if (!flagged || n == 0) {
        if (lane == 0) s_dirty[c] = 0;
        continue;
      }
      const int off = s_off[c];
      double acc[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) acc[d] = 0.0;
      for (int m0 = 0; m0 < n; m0 += 4 * kRows) {
        uint4 x[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          const int r = m0 + 4 * u + grp;
          x[u] = r < n ? reinterpret_cast<const uint4*>(kslice + (size_t)s_mem[off + r] * kHeadDim)[sub]
                       : make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          const uint16_t* e = reinterpret_cast<const uint16_t*>(&x[u]);
#pragma unroll
          for (int d = 0; d < 8; ++d) acc[d] += (double)bf16_to_f32(e[d]);
        }
      }
#pragma unroll
      for (int o = 16; o < kWave; o <<= 1)
#pragma unroll
        for (int d = 0; d < 8; ++d) acc[d] += __shfl_xor(acc[d], o, kWave);
      float mean[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) mean[d] = (float)(acc[d] / (double)n);
      if (grp == 0) {
        float4* dst = reinterpret_cast<float4*>(reps + (size_t)c * kHeadDim + 8 * sub);
        dst[0] = make_float4(mean[0], mean[1], mean[2], mean[3]);
        dst[1] = make_float4(mean[4], mean[5], mean[6], mean[7]);
        small_operand(mean, c, sub, s_frag, s_cn);
      }
      if (lane == 0) s_dirty[c] = 0;
    }
    __syncthreads();
  }

  // outputs: members of each cluster in ascending order through a bitmap
  for (int i = tid; i < N; i += 64 * kSmallWaves) a.assign[(size_t)s * N + i] = s_assign[i];
  uint32_t* bits = s_bits[w];
  for (int c = w; c < C; c += kSmallWaves) {
    const int n = s_cnt[c], off = s_off[c];
    if (lane == 0) {
      a.unit_start[s * a.units_cap + c] = off;
      a.unit_size[s * a.units_cap + c] = n;
    }
    if (lane < kSmallKeys / 32) bits[lane] = 0u;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int i = lane; i < n; i += kWave) {
      const int id = s_mem[off + i];
      atomicOr(&bits[id >> 5], 1u << (id & 31));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t x = lane < kSmallKeys / 32 ? bits[lane] : 0u;
    int incl = __popc(x);
    const int mine = incl;
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
      const int y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += y;
    }
    int at = off + incl - mine;
    while (x) {
      a.perm[(size_t)s * N + at++] = 32 * lane + __builtin_ctz(x);
      x &= x - 1;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// pool[s][r] = src[s][perm[s][r]] for r < n_tokens; 16 lanes per row.  The
// first `blocks` blocks write the pool of src, the others (values given) that
// of src2: one launch for keys and values.
template <class T>
__global__ void pack_pool_kernel(const T* __restrict__ src, const T* __restrict__ src2,
                                 const int32_t* __restrict__ perm, T* __restrict__ pool, T* __restrict__ pool2,
                                 int64_t pool_rows, int n_tokens, int64_t n_rows, int blocks) {
  // 16 rows per block of 256 per round; a grid smaller than n_rows / 16
  // blocks strides over the rest (a pack that shares the chip with clustering)
  const int sub = threadIdx.x & 15;
  const bool second = (int)blockIdx.x >= blocks;
  const int blk = second ? blockIdx.x - blocks : blockIdx.x;
  const T* from = second ? src2 : src;
  T* to = second ? pool2 : pool;
  for (int64_t g = (int64_t)blk * 16 + (threadIdx.x >> 4); g < n_rows; g += (int64_t)blocks * 16) {
    const int64_t s = g / n_tokens;
    const int r = (int)(g - s * n_tokens);
    const int tok = min(max(perm[s * n_tokens + r], 0), n_tokens - 1);   // perm may come from the caller
    constexpr int kU4 = kHeadDim * sizeof(T) / 16;
    const uint4* a = reinterpret_cast<const uint4*>(from + ((size_t)s * n_tokens + tok) * kHeadDim);
    uint4* b = reinterpret_cast<uint4*>(to + ((size_t)s * pool_rows + r) * kHeadDim);
#pragma unroll
    for (int q = sub; q < kU4; q += 16) b[q] = a[q];
  }
}

__global__ void fill_i32_kernel(int32_t* __restrict__ p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Page-level index: one wave per (slice, page).  Lane l sums dims 2l, 2l+1 of
// the page's keys in float64 (row order) and writes their mean rounded once
// to float32; the page's K/V rows are copied to the pool in token order.
template <class T>
__global__ __launch_bounds__(256)
void page_units_kernel(const T* __restrict__ keys, const T* __restrict__ values, int n_tokens, int page_len,
                       int n_pages, int64_t n_items, float* __restrict__ reps, int units_cap,
                       int32_t* __restrict__ unit_start, int32_t* __restrict__ unit_size, T* __restrict__ k_pool,
                       T* __restrict__ v_pool, int64_t pool_rows) {
  const int64_t item = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (item >= n_items) return;
  const int lane = threadIdx.x & 63;
  const int64_t s = item / n_pages;
  const int p = (int)(item - s * n_pages);
  const int a = p * page_len;
  const int len = min(page_len, n_tokens - a);
  double x0 = 0.0, x1 = 0.0;
  for (int r = 0; r < len; ++r) {
    const size_t o = ((size_t)s * n_tokens + a + r) * kHeadDim + 2 * lane;
    x0 += (double)load_as_f32(keys, o);
    x1 += (double)load_as_f32(keys, o + 1);
    if (k_pool) {
      const size_t po = ((size_t)s * pool_rows + a + r) * kHeadDim + 2 * lane;
      k_pool[po] = keys[o];
      k_pool[po + 1] = keys[o + 1];
      if (v_pool) {
        v_pool[po] = values[o];
        v_pool[po + 1] = values[o + 1];
      }
    }
  }
  float* rep = reps + ((size_t)s * units_cap + p) * kHeadDim;
  rep[2 * lane] = (float)(x0 / (double)len);
  rep[2 * lane + 1] = (float)(x1 / (double)len);
  if (lane == 0) {
    unit_start[s * units_cap + p] = a;
    unit_size[s * units_cap + p] = len;
  }
}

// ------------------------------------------------------------------ host side

struct Ws {
  uint4* frag;
  float* cnorm;
  int32_t* counts;
  int32_t* offsets;
  int32_t* cursor;
  int32_t* members;
  int32_t* dirty;    // per cluster: a key entered or left it in the last assignment
  int32_t* dlist;    // the flagged clusters of a slice, ascending
  int32_t* ndirty;   // their number
  int32_t* dmap;     // per cluster: its place in dlist, or -1
  // calls that record (see records()):
  uint4* cfrag;      // the listed clusters' operands and norms, compacted
  float* ccnorm;
  float *best, *sec;     // per key: D to its cluster, a lower bound on D to every other
  int32_t *fail, *nfail; // keys left over by a sweep over the listed clusters, their number
  int32_t* recorded;     // per slice, by the iteration's parity: it recorded best and sec
  uint4* kswz;   // bf16 key operands in B-operand order (kswz_mode of the assignment)
  size_t bytes;
};

// Centroid tiles per slice; bf16 pads to whole LDS stages (padding rows have a
// zero operand and an infinite norm, so they never win).
int n_ctiles_for(int n_clusters, int dtype) {
  const int t = ceil_div(n_clusters, kTileC);
  return dtype == LOUISKV_BF16 ? ceil_div(t, kBf16StageTiles) * kBf16StageTiles : t;
}

constexpr size_t kMaxHistLds = 64 * 1024;

// Whether the scatter scans the counts in LDS (two ints a cluster); above,
// the scan is a launch of its own and no list of the flagged clusters is made.
bool scatter_in_lds(int C) { return (size_t)C * 8 <= kMaxHistLds; }

// Assignments record (and sweep the recomputed clusters alone) from this
// iteration on, where nearly every cluster moves before; a call of fewer
// (key, centroid) pairs does not: its sweep is short, and the launch for the
// left-over keys (8-10 us) takes back what the shorter sweeps give.  A whole
// call with against without, by the noise of the keys around their centres:
//                                     pairs    0.3    0.45    0.65    1.0
//    8 slices of 20011 keys in  625   1.0e8   0.93    0.99    1.05   1.02
//   16           16640          520   1.4e8   0.92    1.00    1.05   1.01
//   16           20480          640   2.1e8   0.92    1.01    1.04   1.01
//   10           25600          800   2.0e8   0.91    0.99    1.03   1.00
//   24           20480          640   3.1e8   0.90    0.96    1.00   0.99
//    8           32768         1024   2.7e8   0.88    0.97    1.01   0.98
//   40           20480          640   5.2e8   0.88    0.94    0.99   0.98
//   64           32768         1024   2.1e9   0.79    0.86    0.95   0.93
// The line lies where the gain on keys well apart begins to outweigh what
// overlapping ones lose.
// Nor does one of few clusters: what recording costs is per key, what it saves
// per (key, centroid) pair (10% longer at 166 clusters, 256 slices of 4000 keys;
// 2% longer at 520, 40 of 25000 keys; 11, 6, 0 and 1% shorter at 520, 40 of
// 16640, for the four noises above).
constexpr int kFirstRecord = 2;
constexpr double kRecordPairs = 1.5e8;
constexpr int kRecordClusters = 640;
bool records(int64_t S, int N, int C, int dtype) {
  return dtype == LOUISKV_BF16 && scatter_in_lds(C) && C >= kRecordClusters &&
         (double)S * N * C >= kRecordPairs;
}

Ws carve(void* base, int64_t n_slices, int n_tokens, int n_clusters, int dtype) {
  Carver cv(base);
  const int n_ctiles = n_ctiles_for(n_clusters, dtype);
  const int tile_u4 = dtype == LOUISKV_BF16 ? kBf16TileU4 : kF32TileU4;
  Ws w;
  w.frag = cv.take<uint4>((size_t)n_slices * n_ctiles * tile_u4);
  w.cnorm = cv.take<float>((size_t)n_slices * n_ctiles * kTileC);
  w.counts = cv.take<int32_t>((size_t)n_slices * n_clusters);
  w.offsets = cv.take<int32_t>((size_t)n_slices * (n_clusters + 1));
  w.cursor = cv.take<int32_t>((size_t)n_slices * n_clusters);
  w.members = cv.take<int32_t>((size_t)n_slices * n_tokens);
  w.dirty = cv.take<int32_t>((size_t)n_slices * n_clusters);
  w.dlist = cv.take<int32_t>((size_t)n_slices * n_clusters);
  w.ndirty = cv.take<int32_t>((size_t)n_slices);
  w.dmap = cv.take<int32_t>((size_t)n_slices * n_clusters);
  w.nfail = cv.take<int32_t>((size_t)n_slices);
  w.recorded = cv.take<int32_t>((size_t)n_slices * 2);
  const size_t bf = records(n_slices, n_tokens, n_clusters, dtype) ? 1 : 0;
  w.cfrag = cv.take<uint4>(bf * n_slices * n_ctiles * tile_u4);
  w.ccnorm = cv.take<float>(bf * n_slices * n_ctiles * kTileC);
  w.best = cv.take<float>(bf * n_slices * n_tokens);
  w.sec = cv.take<float>(bf * n_slices * n_tokens);
  w.fail = cv.take<int32_t>(bf * n_slices * n_tokens);
  w.kswz = dtype == LOUISKV_BF16
               ? cv.take<uint4>((size_t)n_slices * ceil_div(n_tokens, kBf16KeysPerBlock) * kBf16KeysPerBlock * 16)
               : nullptr;
  w.bytes = align_up(cv.used, 256);
  return w;
}

// Waves per cluster of the update, by the clusters of the whole call: one each
// fills the chip from kSplit4Clusters on.  Below that the four waves of a block
// share a cluster's members where it has enough on average for the longest lists
// to be the kernel's time: one per kSplit4Bf16 or kSplit4F32 clusters of the
// call (fewer clusters leave the waves' places empty anyway).  Below
// kSplit16Clusters sixteen waves do from kSplit16Bf16 or kSplit16F32 members on.
// Whole clusterings, us with one / four / sixteen waves (keys 0.3 around their
// centres; overlapping keys gain more from the split), by members on average:
//   clusters          4               16               64               300
//   bf16   512                  200/ 188/ 219   240/ 212/ 239    669/ 427/ 430
//         1000   333/337/398    202/ 195/ 260   287/ 231/ 283    827/ 557/ 592
//         2000   242/256/376    269/ 267/ 390   431/ 353/ 464   1365/1039/1143
//         4000   352/380/619    395/ 405/ 648   794/ 652/ 875   3454/2604/2710
//   f32    512   198/195/236    256/ 216/ 251   640/ 365/ 315   3338/1370/ 873
//         1000   270/267/363    363/ 299/ 399  1263/ 625/ 604   4525/2214/1683
//         2000   401/432/624    600/ 504/ 768  1891/1278/1363   8984/5392/4763
//         4000   723/784/1204  1238/1181/1719  4489/3432/3775
// (An update of clusters of one size gains less: 4000 of 16 float32 keys take 20
// us with one wave and 31 with four; 1000 of 64 25 and 19.)
constexpr int64_t kSplit4Clusters = 4096;
constexpr int kSplit4Bf16 = 128, kSplit4F32 = 256;
constexpr int64_t kSplit16Clusters = 1024;
constexpr int kSplit16Bf16 = 256, kSplit16F32 = 64;
// One wave a cluster in bf16: ids a batch at a time from this many members on
// (long lists end sooner: clusterings of 16 slices of 20000 keys in 256 clusters
// 804 us against 818 with 64 ids at a time, 8 of 20011 in 625 705 against 712;
// an update of 16000 clusters of 4 keys 26.1 against 25.2, of 20 34.7 and 34.6).
// Float32 rows are two a load, and 64 ids at a time are faster throughout (16000
// clusters of 48 keys 108 us against 122).
constexpr int kBatchIdsMembers = 20;
// From this many clusters on a wave takes four of a list's clusters in turn (not
// where every cluster is recomputed): late iterations list a few percent of
// them, and waves that find nothing to do are then a quarter as many.
constexpr int64_t kShareClusters = 65536;
// Scatter blocks of 4096 keys instead of 1024 once that leaves the chip full.
constexpr int64_t kWideScatterBlocks = 4096;
// A block of assign_rest_kernel for this many of a slice's keys (32 at a
// time; about 1% of the keys come to it, more only make the blocks loop), or
// two blocks a slice from kRestManySlices on, where the slices fill the chip.
constexpr int kRestKeysPerBlock = 2048;
constexpr int64_t kRestManySlices = 64;

// clear: the counts, scatter cursors and flags of a new clustering start at zero.
int launch_prep(const float* reps, int stride, int64_t S, int C, int dtype, const Ws& w, bool clear,
                hipStream_t st) {
  const int n_ctiles = n_ctiles_for(C, dtype);
  const int64_t rows = S * n_ctiles * kTileC;
  const int grid = (int)((rows + 3) / 4);
  if (dtype == LOUISKV_BF16)
    prep_operand_kernel<true><<<grid, 256, 0, st>>>(reps, stride, C, n_ctiles, w.frag, w.cnorm,
                                                     clear ? w.counts : nullptr, w.cursor, w.dirty, rows);
  else
    prep_operand_kernel<false><<<grid, 256, 0, st>>>(reps, stride, C, n_ctiles, w.frag, w.cnorm,
                                                      clear ? w.counts : nullptr, w.cursor, w.dirty, rows);
  LKV_CHECK_LAUNCH();
  return LOUISKV_OK;
}

// kswz_mode: 0 keys only, 1 keys and store the operand copy, 2 read the copy
// (bf16 path only).  mode (bf16): from kAssignMoves on, assign holds the
// previous iteration's result, whose counts are kept up to date and whose
// clusters that a key enters or leaves are flagged; with kAssignRecord the
// update has listed the clusters it recomputed, and where the assignment
// before recorded the sweep leaves out the others.  it: the iteration.
int launch_assign(const void* keys, int dtype, int64_t S, int N, int C, const Ws& w, int32_t* assign,
                  bool with_counts, int kswz_mode, hipStream_t st, int mode = kAssignPlain, int it = 0) {
  const int n_ctiles = n_ctiles_for(C, dtype);
  if (dtype == LOUISKV_BF16) {
    AssignArgs a{};
    a.keys = static_cast<const uint16_t*>(keys);
    a.frag = w.frag;
    a.cnorm = w.cnorm;
    a.assign = assign;
    a.counts = with_counts ? w.counts : nullptr;
    a.n_tokens = N;
    a.n_clusters = C;
    a.n_ctiles = n_ctiles;
    a.blocks_per_slice = ceil_div(N, kBf16KeysPerBlock);
    a.hist_in_lds = (size_t)C * 4 <= (size_t)kBf16StageBytes ? 1 : 0;
    a.kswz = w.kswz;
    a.kswz_mode = kswz_mode;
    a.dirty = w.dirty;
    a.best = w.best;
    a.sec = w.sec;
    a.ndirty = w.ndirty;
    a.recorded = w.recorded;
    a.turn = it & 1;
    const bool few = (double)S * N * C < kFewPairs;
    a.part_percent = few ? kPartPercentFew : kPartPercent;
    a.record_percent = few ? kRecordPercentFew : kRecordPercent;
    a.dmap = w.dmap;
    a.dlist = w.dlist;
    a.cfrag = w.cfrag;
    a.ccnorm = w.ccnorm;
    a.fail = w.fail;
    a.nfail = w.nfail;
    const unsigned grid = (unsigned)(S * a.blocks_per_slice);
    if (mode == kAssignRecord)
      assign_bf16_kernel<kAssignRecord><<<grid, kBf16Threads, 0, st>>>(a);
    else if (mode == kAssignMoves)
      assign_bf16_kernel<kAssignMoves><<<grid, kBf16Threads, 0, st>>>(a);
    else
      assign_bf16_kernel<kAssignPlain><<<grid, kBf16Threads, 0, st>>>(a);
    if (mode == kAssignRecord && it > kFirstRecord) {
      LKV_CHECK_LAUNCH();
      if (S >= kRestManySlices)
        assign_rest_kernel<2, 8><<<(unsigned)(2 * S), 512, 0, st>>>(a, 2);
      else {
        const int parts = ceil_div(N, kRestKeysPerBlock);
        assign_rest_kernel<1, 8><<<(unsigned)(S * parts), 512, 0, st>>>(a, parts);
      }
    }
  } else {
    const int bps = ceil_div(N, kF32KeysPerBlock);
    size_t lds = (size_t)kF32StageTiles * (kF32TileU4 * 16 + kTileC * 4);
    const bool hist_lds = (size_t)C * 4 <= std::max(lds, kMaxHistLds);
    if (with_counts && hist_lds) lds = std::max(lds, (size_t)C * 4);
    assign_f32_kernel<<<(unsigned)(S * bps), kAssignThreads, lds, st>>>(
        static_cast<const float*>(keys), w.frag, w.cnorm, assign, with_counts ? w.counts : nullptr, N, C,
        n_ctiles, bps, hist_lds ? 1 : 0);
  }
  LKV_CHECK_LAUNCH();
  return LOUISKV_OK;
}

// list: only the flagged clusters' members are placed and the list of those
// clusters is written (all: every key is placed all the same; first: nothing
// has been recorded yet).
int launch_scan_scatter(const int32_t* assign, int64_t S, int N, int C, const Ws& w, bool list, bool all, bool first,
                        hipStream_t st) {
  const int bps = ceil_div(N, kScatterKeys);
  const bool rec = list && records(S, N, C, LOUISKV_BF16);
  if (scatter_in_lds(C)) {
#define LKV_SCATTER(PER)                                                                                           \
  scatter_kernel<PER><<<(unsigned)(S * ceil_div(N, 256 * PER)), 256, (size_t)C * 8, st>>>(                          \
      assign, w.counts, w.cursor, w.offsets, w.members, N, C, ceil_div(N, 256 * PER), list ? w.dirty : nullptr,      \
      w.dlist, w.dmap, w.ndirty, w.nfail, rec ? w.cfrag : nullptr, w.ccnorm, n_ctiles_for(C, LOUISKV_BF16), all ? 1 : 0,           \
      first ? w.recorded : nullptr)
    if (S * bps >= kWideScatterBlocks) {
      LKV_SCATTER(16);
    } else {
      LKV_SCATTER(4);
    }
#undef LKV_SCATTER
  } else {
    scan_kernel<<<(unsigned)S, 1024, 0, st>>>(w.counts, w.offsets, w.cursor, C);
    LKV_CHECK_LAUNCH();
    scatter_global_kernel<<<(unsigned)(S * bps), 256, 0, st>>>(assign, w.cursor, w.members, N, C, bps);
  }
  LKV_CHECK_LAUNCH();
  return LOUISKV_OK;
}

// Centroid update; with prep_next, also the next iteration's operand (the
// work of launch_prep for the iterations after the first).  zero_counts: the
// next assignment counts from zero.  flagged: only the clusters that the
// assignment flagged (the others keep centroid and operand).
template <class T>
int launch_sum_t(const void* keys, int64_t S, int N, int C, int n_ctiles, const Ws& w, const float* cin, float* cout,
                 int stride, bool prep_next, bool zero_counts, bool flagged, hipStream_t st) {
  const bool list = flagged && scatter_in_lds(C);
  UpdateArgs<T> a{};
  a.keys = static_cast<const T*>(keys);
  a.members = w.members;
  a.offsets = w.offsets;
  a.counts = w.counts;
  a.cursor = scatter_in_lds(C) ? w.cursor : nullptr;
  a.cin = cin;
  a.cout = cout;
  a.stride = stride;
  a.n_tokens = N;
  a.n_clusters = C;
  a.frag = prep_next ? w.frag : nullptr;
  a.cnorm = w.cnorm;
  a.n_ctiles = n_ctiles;
  a.zero_counts = zero_counts ? 1 : 0;
  a.dirty = flagged ? w.dirty : nullptr;
  a.ndirty = w.ndirty;
  a.dmap = list ? w.dmap : nullptr;
  a.cfrag = list && records(S, N, C, LOUISKV_BF16) ? w.cfrag : nullptr;
  a.ccnorm = w.ccnorm;
  const int64_t rows = S * C;
  const int members = N / C;
  constexpr bool kBf16 = sizeof(T) == 2;
  if (rows < kSplit4Clusters && (int64_t)members * (kBf16 ? kSplit4Bf16 : kSplit4F32) >= rows) {
    a.blocks_per_slice = a.stride_e = C;
    if (rows < kSplit16Clusters && members >= (kBf16 ? kSplit16Bf16 : kSplit16F32))
      centroid_update_kernel<T, 16><<<(unsigned)rows, 1024, 0, st>>>(a);
    else
      centroid_update_kernel<T, 4><<<(unsigned)rows, 256, 0, st>>>(a);
  } else {
    const int per = list && rows >= kShareClusters ? 4 : 1;   // clusters a wave takes when all are listed
    a.dlist = per > 1 ? w.dlist : nullptr;
    a.blocks_per_slice = ceil_div(C, 4 * per);
    a.stride_e = 4 * a.blocks_per_slice;
    const unsigned grid = (unsigned)(S * a.blocks_per_slice);
    if constexpr (kBf16) {
      if (members >= kBatchIdsMembers)
        centroid_update_kernel<T, 1, true><<<grid, 256, 0, st>>>(a);
      else
        centroid_update_kernel<T, 1><<<grid, 256, 0, st>>>(a);
    } else {
      centroid_update_kernel<T, 1><<<grid, 256, 0, st>>>(a);
    }
  }
  LKV_CHECK_LAUNCH();
  return LOUISKV_OK;
}

int launch_sum(const void* keys, int dtype, int64_t S, int N, int C, const Ws& w, const float* cin, float* cout,
               int stride, bool prep_next, bool zero_counts, bool flagged, hipStream_t st) {
  const int n_ctiles = n_ctiles_for(C, dtype);
  return dtype == LOUISKV_BF16
             ? launch_sum_t<uint16_t>(keys, S, N, C, n_ctiles, w, cin, cout, stride, prep_next, zero_counts, flagged, st)
             : launch_sum_t<float>(keys, S, N, C, n_ctiles, w, cin, cout, stride, prep_next, zero_counts, flagged, st);
}

constexpr int64_t kMaxPackGrid = 1 << 20;   // blocks a pool; they stride over more rows

// Prompt K/V rows in perm order into the pools (each cluster one contiguous run).
int launch_pack(const void* keys, const void* values, int dtype, int64_t S, int N, const int32_t* perm, void* k_pool,
                void* v_pool, int64_t pool_rows, hipStream_t s, int max_grid = 0) {
  const int64_t prow = S * N;
  int pgrid = (int)std::min<int64_t>((prow + 15) / 16, kMaxPackGrid);
  if (max_grid > 0) pgrid = std::min(pgrid, max_grid);
  if (!k_pool) {   // values alone
    keys = values;
    k_pool = v_pool;
    v_pool = nullptr;
  }
  if (!k_pool) return LOUISKV_OK;
  const unsigned grid = (unsigned)pgrid * (v_pool ? 2u : 1u);
  if (dtype == LOUISKV_BF16)
    pack_pool_kernel<uint16_t><<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(keys),
                                                    static_cast<const uint16_t*>(values), perm,
                                                    static_cast<uint16_t*>(k_pool), static_cast<uint16_t*>(v_pool),
                                                    pool_rows, N, prow, pgrid);
  else
    pack_pool_kernel<float><<<grid, 256, 0, s>>>(static_cast<const float*>(keys), static_cast<const float*>(values),
                                                 perm, static_cast<float*>(k_pool), static_cast<float*>(v_pool),
                                                 pool_rows, N, prow, pgrid);
  LKV_CHECK_LAUNCH();
  return LOUISKV_OK;
}


// Initial centroids, n_iters Lloyd iterations and the CSR/perm outputs, for
// arguments already validated (no pool write).
int run_cluster(const void* keys, int dtype, int64_t S, int N, int C, int n_iters, const int32_t* init_idx,
                float* reps, int units_cap, int32_t* unit_start, int32_t* unit_size, int32_t* assign, int32_t* perm,
                void* const* iter_events, const Ws& w, hipStream_t s) {
  int st;
  if (dtype == LOUISKV_BF16 && N <= kSmallKeys && C <= kSmallClusters && !iter_events) {
    SmallArgs a{static_cast<const uint16_t*>(keys), init_idx, reps, unit_start, unit_size, assign, perm, N, C,
                units_cap, n_iters};
    if (N <= kSmallKeys / 2)
      lloyd_small_kernel<1><<<(unsigned)S, 64 * kSmallWaves, 0, s>>>(a);
    else
      lloyd_small_kernel<2><<<(unsigned)S, 64 * kSmallWaves, 0, s>>>(a);
    LKV_CHECK_LAUNCH();
    return LOUISKV_OK;
  }
  {
    const int64_t rows = S * C;
    const int grid = (int)((rows + 3) / 4);
    if (dtype == LOUISKV_BF16)
      init_centroids_kernel<uint16_t><<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(keys), init_idx, reps,
                                                            N, C, units_cap, rows);
    else
      init_centroids_kernel<float><<<grid, 256, 0, s>>>(static_cast<const float*>(keys), init_idx, reps, N,
                                                         C, units_cap, rows);
    LKV_CHECK_LAUNCH();
  }
  // the first operand comes from the initial centroids; after that each
  // update writes the next one (and clears the counts) as it goes
  if ((st = launch_prep(reps, units_cap, S, C, dtype, w, true, s))) return st;
  for (int it = 0; it < n_iters; ++it) {
    if (iter_events) LKV_CHECK_HIP(hipEventRecord(reinterpret_cast<hipEvent_t>(iter_events[2 * it]), s));
    // from the second iteration on (bf16), the assignment flags the clusters
    // that keys entered or left, keeps the counts up to date, and the update
    // recomputes only those clusters
    const bool track = dtype == LOUISKV_BF16 && it > 0;
    const bool list = track && scatter_in_lds(C);
    const bool last = it + 1 == n_iters;
    const bool record = it >= kFirstRecord && records(S, N, C, dtype);
    const int mode = !track ? kAssignPlain : record ? kAssignRecord : kAssignMoves;
    if ((st = launch_assign(keys, dtype, S, N, C, w, assign, true, it == 0 ? 1 : 2, s, mode, it)))
      return st;
    if (iter_events) LKV_CHECK_HIP(hipEventRecord(reinterpret_cast<hipEvent_t>(iter_events[2 * it + 1]), s));
    if ((st = launch_scan_scatter(assign, S, N, C, w, list, last, it < kFirstRecord, s))) return st;
    if ((st = launch_sum(keys, dtype, S, N, C, w, reps, reps, units_cap, !last, !last && dtype != LOUISKV_BF16, track,
                         s)))
      return st;
  }
  {
    const int64_t rows = S * C;
    finalize_kernel<<<(int)((rows + 3) / 4), 256, 0, s>>>(w.members, w.offsets, w.counts, perm, unit_start,
                                                          unit_size, units_cap, N, C, rows);
    LKV_CHECK_LAUNCH();
  }
  return LOUISKV_OK;
}

int check_common(const void* keys, int dtype, int64_t S, int N, int d, int C) {
  if (!keys) return fail(LOUISKV_ERR_NULL, "keys is NULL");
  if (dtype != LOUISKV_F32 && dtype != LOUISKV_BF16) return fail(LOUISKV_ERR_DTYPE, "unknown dtype %d", dtype);
  if (d != kHeadDim) return fail(LOUISKV_ERR_UNSUPPORTED, "head dim %d not supported (only 128)", d);
  if (S < 1 || N < 1) return fail(LOUISKV_ERR_SHAPE, "n_slices=%lld n_tokens=%d must be >= 1", (long long)S, N);
  if (C < 1 || C > N) return fail(LOUISKV_ERR_SHAPE, "n_clusters=%d must be in [1, n_tokens=%d]", C, N);
  if ((int64_t)S * ceil_div(N, kBf16KeysPerBlock) > (int64_t)INT32_MAX / 2 ||
      (int64_t)S * ceil_div(N, kF32KeysPerBlock) > (int64_t)INT32_MAX / 2)
    return fail(LOUISKV_ERR_SHAPE, "problem too large for one launch");
  return LOUISKV_OK;
}

}  // namespace
}  // namespace louiskv

using namespace louiskv;

extern "C" size_t louiskv_cluster_prefill_workspace_size(int64_t n_slices, int32_t n_tokens, int32_t d,
                                                         int32_t n_clusters, int32_t dtype) {
  (void)d;
  if (n_slices < 1 || n_tokens < 1 || n_clusters < 1) return 0;
  return carve(nullptr, n_slices, n_tokens, n_clusters, dtype == LOUISKV_BF16 ? LOUISKV_BF16 : LOUISKV_F32).bytes;
}

extern "C" int louiskv_cluster_prefill(const void* keys, int32_t dtype, int64_t n_slices, int32_t n_tokens,
                                       int32_t d, int32_t n_clusters, int32_t n_iters, const int32_t* init_idx,
                                       float* reps, int32_t units_cap, int32_t* unit_start, int32_t* unit_size,
                                       int32_t* assign, int32_t* perm, const void* values, void* k_pool,
                                       void* v_pool, int64_t pool_rows, int32_t pool_on_host,
                                       void* const* iter_events, void* workspace, size_t workspace_bytes,
                                       void* stream) {
  int st = check_common(keys, dtype, n_slices, n_tokens, d, n_clusters);
  if (st) return st;
  if (!init_idx || !reps || !unit_start || !unit_size || !assign || !perm)
    return fail(LOUISKV_ERR_NULL, "init_idx, reps, unit_start, unit_size, assign and perm are required");
  if (n_iters < 1) return fail(LOUISKV_ERR_SHAPE, "n_iters=%d must be >= 1", n_iters);
  if (units_cap < n_clusters) return fail(LOUISKV_ERR_SHAPE, "units_cap=%d < n_clusters=%d", units_cap, n_clusters);
  if (v_pool && !values) return fail(LOUISKV_ERR_NULL, "v_pool given without values");
  if ((k_pool || v_pool) && pool_rows < n_tokens)
    return fail(LOUISKV_ERR_SHAPE, "pool_rows=%lld < n_tokens=%d", (long long)pool_rows, n_tokens);
  if (pool_on_host && ((st = device_view_of_host_pool(k_pool, &k_pool)) || (st = device_view_of_host_pool(v_pool, &v_pool))))
    return st;
  const Ws need = carve(nullptr, n_slices, n_tokens, n_clusters, dtype);
  if (!workspace || workspace_bytes < need.bytes)
    return fail(LOUISKV_ERR_WORKSPACE, "workspace needs %zu bytes, got %zu", need.bytes, workspace_bytes);
  const Ws w = carve(workspace, n_slices, n_tokens, n_clusters, dtype);
  hipStream_t s = as_stream(stream);
  if ((st = run_cluster(keys, dtype, n_slices, n_tokens, n_clusters, n_iters, init_idx, reps, units_cap, unit_start,
                        unit_size, assign, perm, iter_events, w, s)))
    return st;
  return launch_pack(keys, values, dtype, n_slices, n_tokens, perm, k_pool, v_pool, pool_rows, s);
}

namespace louiskv {
namespace {

size_t esize_of(int dtype) { return dtype == LOUISKV_BF16 ? 2 : 4; }

// Workspace of the pipelined prefill: the clustering workspace of one chunk,
// then (copy-engine writes only) one chunk of staged pool rows.
size_t pipelined_bytes(int64_t chunk, int N, int C, int dtype, bool staged) {
  size_t b = carve(nullptr, chunk, N, C, dtype).bytes;
  if (staged) b += align_up((size_t)chunk * N * kHeadDim * esize_of(dtype), 256);
  return b;
}

// Largest pack grid while the pack shares the chip with the clustering of
// the next chunk: enough rows in flight for the host link, few CUs held.
constexpr int kOverlapPackGrid = 256;
// Keys and values of a chunk in one launch hold twice that: faster where a
// chunk has many rows to write to HBM, slower where the next chunk's clustering
// is short of blocks or the host link sets the pace anyway.  Whole calls, one
// launch against two: 64 slices of 32768 keys in chunks of 32 slices 4.29 ms
// against 4.47, 256 in chunks of 8 24.5 against 24.3; 32 in chunks of 8 into a
// host pool 12.5 against 12.1.
constexpr int64_t kOverlapPackBothRows = 1 << 19;

}  // namespace
}  // namespace louiskv

extern "C" size_t louiskv_cluster_prefill_pipelined_workspace_size(int64_t slices_per_chunk, int32_t n_tokens,
                                                                   int32_t d, int32_t n_clusters, int32_t dtype,
                                                                   int32_t pool_on_host, int32_t copy_engine) {
  (void)d;
  if (slices_per_chunk < 1 || n_tokens < 1 || n_clusters < 1) return 0;
  const int dt = dtype == LOUISKV_BF16 ? LOUISKV_BF16 : LOUISKV_F32;
  return pipelined_bytes(slices_per_chunk, n_tokens, n_clusters, dt, pool_on_host && copy_engine);
}

extern "C" int louiskv_cluster_prefill_pipelined(
    const void* keys, int32_t dtype, int64_t n_slices, int32_t n_tokens, int32_t d, int32_t n_clusters,
    int32_t n_iters, const int32_t* init_idx, float* reps, int32_t units_cap, int32_t* unit_start,
    int32_t* unit_size, int32_t* assign, int32_t* perm, const void* values, void* k_pool, void* v_pool,
    int64_t pool_rows, int32_t pool_on_host, int64_t slices_per_chunk, int32_t copy_engine,
    void* const* chunk_events, int64_t n_events, void* workspace, size_t workspace_bytes, void* stream,
    void* copy_stream) {
  int st = check_common(keys, dtype, n_slices, n_tokens, d, n_clusters);
  if (st) return st;
  if (!init_idx || !reps || !unit_start || !unit_size || !assign || !perm || !k_pool)
    return fail(LOUISKV_ERR_NULL, "init_idx, reps, unit_start, unit_size, assign, perm and k_pool are required");
  if (n_iters < 1) return fail(LOUISKV_ERR_SHAPE, "n_iters=%d must be >= 1", n_iters);
  if (units_cap < n_clusters) return fail(LOUISKV_ERR_SHAPE, "units_cap=%d < n_clusters=%d", units_cap, n_clusters);
  if (v_pool && !values) return fail(LOUISKV_ERR_NULL, "v_pool given without values");
  if (pool_rows < n_tokens)
    return fail(LOUISKV_ERR_SHAPE, "pool_rows=%lld < n_tokens=%d", (long long)pool_rows, n_tokens);
  if (slices_per_chunk < 1) return fail(LOUISKV_ERR_SHAPE, "slices_per_chunk=%lld must be >= 1",
                                        (long long)slices_per_chunk);
  const int64_t chunk = std::min(slices_per_chunk, n_slices);
  const int64_t n_chunks = (n_slices + chunk - 1) / chunk;
  if (!chunk_events || n_events < n_chunks + 1)
    return fail(LOUISKV_ERR_NULL, "chunk_events must hold n_chunks + 1 = %lld events, got %lld",
                (long long)(n_chunks + 1), (long long)n_events);
  for (int64_t i = 0; i <= n_chunks; ++i)
    if (!chunk_events[i]) return fail(LOUISKV_ERR_NULL, "chunk_events[%lld] is NULL", (long long)i);
  void* k_dev = k_pool;
  void* v_dev = v_pool;
  if (pool_on_host && ((st = device_view_of_host_pool(k_pool, &k_dev)) || (st = device_view_of_host_pool(v_pool, &v_dev))))
    return st;
  const bool staged = pool_on_host && copy_engine;
  const size_t need = pipelined_bytes(chunk, n_tokens, n_clusters, dtype, staged);
  if (!workspace || workspace_bytes < need)
    return fail(LOUISKV_ERR_WORKSPACE, "workspace needs %zu bytes, got %zu", need, workspace_bytes);
  const Ws w = carve(workspace, chunk, n_tokens, n_clusters, dtype);
  void* staging = static_cast<char*>(workspace) + w.bytes;
  hipStream_t s = as_stream(stream);
  hipStream_t cp = as_stream(copy_stream);
  const size_t es = esize_of(dtype);
  const size_t row_bytes = (size_t)kHeadDim * es;
  for (int64_t i = 0; i < n_chunks; ++i) {
    const int64_t c0 = i * chunk;
    const int64_t n = std::min(chunk, n_slices - c0);
    const size_t kv_off = (size_t)c0 * n_tokens * row_bytes;
    const size_t pool_off = (size_t)c0 * pool_rows * row_bytes;
    const void* keys_c = static_cast<const char*>(keys) + kv_off;
    const void* vals_c = values ? static_cast<const char*>(values) + kv_off : nullptr;
    int32_t* perm_c = perm + c0 * n_tokens;
    if ((st = run_cluster(keys_c, dtype, n, n_tokens, n_clusters, n_iters, init_idx + c0 * n_clusters,
                          reps + c0 * units_cap * kHeadDim, units_cap, unit_start + c0 * units_cap,
                          unit_size + c0 * units_cap, assign + c0 * n_tokens, perm_c, nullptr, w, s)))
      return st;
    // the pool write of this chunk waits for its clustering only and runs
    // beside the clustering of the next chunks
    LKV_CHECK_HIP(hipEventRecord(reinterpret_cast<hipEvent_t>(chunk_events[i]), s));
    LKV_CHECK_HIP(hipStreamWaitEvent(cp, reinterpret_cast<hipEvent_t>(chunk_events[i]), 0));
    if (!staged) {
      void* kp = static_cast<char*>(k_dev) + pool_off;
      void* vp = v_dev ? static_cast<char*>(v_dev) + pool_off : nullptr;
      const bool both = !pool_on_host && n * n_tokens >= kOverlapPackBothRows;
      if ((st = launch_pack(keys_c, vals_c, dtype, n, n_tokens, perm_c, kp, both ? vp : nullptr, pool_rows, cp,
                            kOverlapPackGrid)))
        return st;
      if (vp && !both &&
          (st = launch_pack(nullptr, vals_c, dtype, n, n_tokens, perm_c, nullptr, vp, pool_rows, cp, kOverlapPackGrid)))
        return st;
      continue;
    }
    // copy engine: permute into HBM staging, then one pitched copy over the host link
    for (int which = 0; which < 2; ++which) {
      void* host = which == 0 ? k_pool : v_pool;
      if (!host) continue;
      const void* src = which == 0 ? keys_c : vals_c;
      if ((st = launch_pack(src, nullptr, dtype, n, n_tokens, perm_c, staging, nullptr, n_tokens, cp))) return st;
      LKV_CHECK_HIP(hipMemcpy2DAsync(static_cast<char*>(host) + pool_off, (size_t)pool_rows * row_bytes, staging,
                                     (size_t)n_tokens * row_bytes, (size_t)n_tokens * row_bytes, (size_t)n,
                                     hipMemcpyDeviceToHost, cp));
    }
  }
  LKV_CHECK_HIP(hipEventRecord(reinterpret_cast<hipEvent_t>(chunk_events[n_chunks]), cp));
  LKV_CHECK_HIP(hipStreamWaitEvent(s, reinterpret_cast<hipEvent_t>(chunk_events[n_chunks]), 0));
  return LOUISKV_OK;
}

extern "C" int louiskv_page_prefill(const void* keys, const void* values, int32_t dtype, int64_t n_slices,
                                    int32_t n_tokens, int32_t d, int32_t page_len, float* reps, int32_t units_cap,
                                    int32_t* unit_start, int32_t* unit_size, void* k_pool, void* v_pool,
                                    int64_t pool_rows, int32_t pool_on_host, void* stream) {
  if (!keys || !reps || !unit_start || !unit_size)
    return fail(LOUISKV_ERR_NULL, "keys, reps, unit_start and unit_size are required");
  if (v_pool && !values) return fail(LOUISKV_ERR_NULL, "v_pool given without values");
  if (v_pool && !k_pool) return fail(LOUISKV_ERR_NULL, "v_pool given without k_pool");
  if (dtype != LOUISKV_F32 && dtype != LOUISKV_BF16) return fail(LOUISKV_ERR_DTYPE, "unknown dtype %d", dtype);
  if (d != kHeadDim) return fail(LOUISKV_ERR_UNSUPPORTED, "head dim %d not supported (only 128)", d);
  if (n_slices < 1 || n_tokens < 1 || page_len < 1)
    return fail(LOUISKV_ERR_SHAPE, "n_slices=%lld n_tokens=%d page_len=%d", (long long)n_slices, n_tokens, page_len);
  const int n_pages = ceil_div(n_tokens, page_len);
  if (units_cap < n_pages) return fail(LOUISKV_ERR_SHAPE, "units_cap=%d < %d pages", units_cap, n_pages);
  if (k_pool && pool_rows < n_tokens)
    return fail(LOUISKV_ERR_SHAPE, "pool_rows=%lld < n_tokens=%d", (long long)pool_rows, n_tokens);
  const int64_t items = n_slices * n_pages;
  if ((items + 3) / 4 > INT32_MAX) return fail(LOUISKV_ERR_SHAPE, "problem too large for one launch");
  int st;
  if (pool_on_host && ((st = device_view_of_host_pool(k_pool, &k_pool)) || (st = device_view_of_host_pool(v_pool, &v_pool))))
    return st;
  hipStream_t s = as_stream(stream);
  const unsigned grid = (unsigned)((items + 3) / 4);
  if (dtype == LOUISKV_BF16)
    page_units_kernel<uint16_t><<<grid, 256, 0, s>>>(static_cast<const uint16_t*>(keys),
                                                      static_cast<const uint16_t*>(values), n_tokens, page_len,
                                                      n_pages, items, reps, units_cap, unit_start, unit_size,
                                                      static_cast<uint16_t*>(k_pool), static_cast<uint16_t*>(v_pool),
                                                      pool_rows);
  else
    page_units_kernel<float><<<grid, 256, 0, s>>>(static_cast<const float*>(keys), static_cast<const float*>(values),
                                                   n_tokens, page_len, n_pages, items, reps, units_cap, unit_start,
                                                   unit_size, static_cast<float*>(k_pool), static_cast<float*>(v_pool),
                                                   pool_rows);
  LKV_CHECK_LAUNCH();
  return LOUISKV_OK;
}

extern "C" int louiskv_pack_pool(const void* keys, const void* values, int32_t dtype, int64_t n_slices,
                                 int32_t n_tokens, int32_t d, const int32_t* perm, void* k_pool, void* v_pool,
                                 int64_t pool_rows, int32_t pool_on_host, void* stream) {
  if (!keys || !perm || !k_pool) return fail(LOUISKV_ERR_NULL, "keys, perm and k_pool are required");
  if (v_pool && !values) return fail(LOUISKV_ERR_NULL, "v_pool given without values");
  if (dtype != LOUISKV_F32 && dtype != LOUISKV_BF16) return fail(LOUISKV_ERR_DTYPE, "unknown dtype %d", dtype);
  if (d != kHeadDim) return fail(LOUISKV_ERR_UNSUPPORTED, "head dim %d not supported (only 128)", d);
  if (n_slices < 1 || n_tokens < 1 || pool_rows < n_tokens)
    return fail(LOUISKV_ERR_SHAPE, "n_slices=%lld n_tokens=%d pool_rows=%lld", (long long)n_slices, n_tokens,
                (long long)pool_rows);
  int st;
  if (pool_on_host && ((st = device_view_of_host_pool(k_pool, &k_pool)) || (st = device_view_of_host_pool(v_pool, &v_pool))))
    return st;
  return launch_pack(keys, values, dtype, n_slices, n_tokens, perm, k_pool, v_pool, pool_rows, as_stream(stream));
}

extern "C" int louiskv_kmeans_assign(const void* keys, int32_t dtype, int64_t n_slices, int32_t n_tokens, int32_t d,
                                     int32_t n_clusters, const float* centroids, int32_t centroid_stride,
                                     int32_t* assign, void* workspace, size_t workspace_bytes, void* stream) {
  int st = check_common(keys, dtype, n_slices, n_tokens, d, n_clusters);
  if (st) return st;
  if (!centroids || !assign) return fail(LOUISKV_ERR_NULL, "centroids and assign are required");
  if (centroid_stride < n_clusters) return fail(LOUISKV_ERR_SHAPE, "centroid_stride < n_clusters");
  const Ws need = carve(nullptr, n_slices, n_tokens, n_clusters, dtype);
  if (!workspace || workspace_bytes < need.bytes)
    return fail(LOUISKV_ERR_WORKSPACE, "workspace needs %zu bytes, got %zu", need.bytes, workspace_bytes);
  const Ws w = carve(workspace, n_slices, n_tokens, n_clusters, dtype);
  hipStream_t s = as_stream(stream);
  if ((st = launch_prep(centroids, centroid_stride, n_slices, n_clusters, dtype, w, false, s))) return st;
  return launch_assign(keys, dtype, n_slices, n_tokens, n_clusters, w, assign, false, 0, s);
}

extern "C" int louiskv_kmeans_update(const void* keys, int32_t dtype, int64_t n_slices, int32_t n_tokens, int32_t d,
                                     int32_t n_clusters, const int32_t* assign, const float* centroids_in,
                                     float* centroids_out, int32_t centroid_stride, int32_t* counts,
                                     void* workspace, size_t workspace_bytes, void* stream) {
  int st = check_common(keys, dtype, n_slices, n_tokens, d, n_clusters);
  if (st) return st;
  if (!assign || !centroids_in || !centroids_out) return fail(LOUISKV_ERR_NULL, "assign and centroids are required");
  if (centroid_stride < n_clusters) return fail(LOUISKV_ERR_SHAPE, "centroid_stride < n_clusters");
  const Ws need = carve(nullptr, n_slices, n_tokens, n_clusters, dtype);
  if (!workspace || workspace_bytes < need.bytes)
    return fail(LOUISKV_ERR_WORKSPACE, "workspace needs %zu bytes, got %zu", need.bytes, workspace_bytes);
  const Ws w = carve(workspace, n_slices, n_tokens, n_clusters, dtype);
  hipStream_t s = as_stream(stream);
  {
    // a fill kernel rather than a memset node, so the call stays safe to capture
    const int64_t n = n_slices * n_clusters;
    const unsigned grid = (unsigned)((n + 255) / 256);
    fill_i32_kernel<<<grid, 256, 0, s>>>(w.counts, 0, n);
    LKV_CHECK_LAUNCH();
    fill_i32_kernel<<<grid, 256, 0, s>>>(w.cursor, 0, n);
    LKV_CHECK_LAUNCH();
  }
  const int bps = ceil_div(n_tokens, kCountKeys);
  const bool lds_ok = (size_t)n_clusters * 4 <= kMaxHistLds;
  count_kernel<<<(unsigned)(n_slices * bps), 256, lds_ok ? (size_t)n_clusters * 4 : 0, s>>>(
      assign, w.counts, n_tokens, n_clusters, bps, lds_ok ? 1 : 0);
  LKV_CHECK_LAUNCH();
  if ((st = launch_scan_scatter(assign, n_slices, n_tokens, n_clusters, w, false, true, false, s))) return st;
  if ((st = launch_sum(keys, dtype, n_slices, n_tokens, n_clusters, w, centroids_in, centroids_out,
                       centroid_stride, false, false, false, s)))
    return st;
  if (counts)
    LKV_CHECK_HIP(hipMemcpyAsync(counts, w.counts, sizeof(int32_t) * n_slices * n_clusters,
                                 hipMemcpyDeviceToDevice, s));
  return LOUISKV_OK;
}
