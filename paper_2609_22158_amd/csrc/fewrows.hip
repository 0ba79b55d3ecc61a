// Token saliency of few window rows: K read once, its logits kept.
//
// With at most 8 window rows the sweeps are streams of K (2 d bytes per key)
// with almost no arithmetic, and the logits of a key (4 R bytes) are smaller
// than its row. row_logits_kernel reads K once, writes the logits and the
// chunk's per-row (max, sum) partials; row_sums_kernel merges the partials of
// its (sequence, head) into the row LSEs and sums exp2(c z - lse) over the rows
// of each key. The logits of 16 keys are one tile: for each quad of rows, the
// keys' four logits. Bound by the K stream. Saliency of the 32-layer 32k cache
// (8 KV heads, d 128), both sweeps in one launch and this form: one query per
// head (R = 4) 601 -> 409 us (K at 5.7 TB/s and 27 us for the sums), R = 8
// 602 -> 460; d 64: 316 -> 238 and 316 -> 277; one layer of 8192 tokens
// 17.6 -> 12.4 (a launch less).
#include "common.h"
#include "internal.h"
#include "saliency_chunks.h"

#include <math.h>

#include <type_traits>

namespace stepkv {
namespace {

typedef float f32x4_t __attribute__((__vector_size__(4 * sizeof(float))));

constexpr int kThreads = 256;
constexpr int kRing = 3;  // tiles per wave in its K ring

// XOR swizzle of the 16-byte pieces of row r of a tile: the 16 rows of a
// fragment read fall on distinct bank groups.
template <int D>
__device__ __forceinline__ int swz(int r) {
  return D == 128 ? (r & 15) : ((r >> 1) & 7);
}

template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// The fragments at addr[ks] + OFF in LDS. The reads and their wait are one
// block: the compiler takes an asm's outputs as written when it ends. (In
// assembly, so that no wait for the whole K ring is put in front of them.)
template <int OFF>
__device__ __forceinline__ void read_fragments(const uint32_t (&addr)[4], bf16x8_t (&f)[4]) {
  asm volatile(
      "ds_read_b128 %0, %4 offset:%8\n\tds_read_b128 %1, %5 offset:%8\n\t"
      "ds_read_b128 %2, %6 offset:%8\n\tds_read_b128 %3, %7 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3])
      : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "n"(OFF)
      : "memory");
}
template <int OFF>
__device__ __forceinline__ void read_fragments(const uint32_t (&addr)[2], bf16x8_t (&f)[2]) {
  asm volatile(
      "ds_read_b128 %0, %2 offset:%4\n\tds_read_b128 %1, %3 offset:%4\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(f[0]), "=&v"(f[1])
      : "v"(addr[0]), "v"(addr[1]), "n"(OFF)
      : "memory");
}

constexpr int kFewRows = 8;      // most rows taken
constexpr int kMaxFewRows = 16;  // rows of the MFMA tile and of a partial

// First logit slot of sequence s: whole tiles that no other sequence's reach.
__device__ __forceinline__ size_t logit_slot(int s, int seq0) {
  return (size_t)(seq0 & ~15) + 16 * (size_t)s;
}

// One workgroup per (head, chunk). Each wave takes every fourth tile of 16
// keys through a ring of its own in LDS (global_load_lds: whole rows, fully
// coalesced; loading the MFMA operand straight to registers, 64 bytes of a row
// at a time, took 498 us against 409). The tile is the B operand of
// v_mfma_f32_16x16x32_bf16, where lane group g holds the 16-byte pieces 4 ks + g
// of its row (the window rows take the same order); lane l then holds key
// l % 16 for rows 4 (l / 16) + 0..3. Rings of 2 and 4 tiles: 413 and 404 us here,
// 52 and 57 against 52 on three layers (fewer workgroups fit a CU).
template <int D, int RQ, bool CAUSAL>
__global__ __launch_bounds__(kThreads) void row_logits_kernel(SaliencyArgs a, int lh0) {
  constexpr int KS = D / 32;
  __shared__ __attribute__((aligned(16))) uint8_t kring[(kThreads / kWave) * kRing * 32 * D];
  __shared__ float2 part[kThreads / kWave][kMaxFewRows];
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int c16 = lane & 15, g4 = lane >> 4;
  const int lr = blockIdx.x / a.total_chunks, g = blockIdx.x - lr * a.total_chunks;
  const int lh = lh0 + lr;
  const ChunkLoc loc = find_chunk(a, g);
  const int l = lh / a.Hkv, h = lh - l * a.Hkv;
  const int key0 = (g - loc.first) * a.chunk;
  const int nkeys = min(a.chunk, loc.ns - key0);
  const int ntiles = (nkeys + 15) / 16;
  const uint16_t* __restrict__ kb = a.k + ((size_t)lh * a.ntot + loc.seq0 + key0) * D;
  float* __restrict__ lg = a.logits + ((size_t)lr * a.logit_slots + logit_slot(loc.s, loc.seq0) +
                                       key0) * (4 * RQ) + 64 * g4 + 4 * c16;
  // K ring of this wave in LDS: kRing tiles of 16 rows, each row's 16-byte pieces
  // XOR-swizzled
  constexpr int PR = D / 8, RPI = kWave / PR, NL = 16 / RPI, TB = 16 * 2 * D;
  uint8_t* ring = kring + wave * (kRing * TB);
  const int lrow = lane / PR, lpiece = lane % PR;
  const uint32_t ring_lds = static_cast<uint32_t>(
      reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)ring));
  uint32_t fa[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) fa[ks] = ring_lds + c16 * (2 * D) + 16 * ((4 * ks + g4) ^ swz<D>(c16));
  auto issue = [&](int t, auto slot_c) __attribute__((always_inline)) {
    constexpr int slot = decltype(slot_c)::value;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int r = i * RPI + lrow;
      const int key = min(16 * t + r, nkeys - 1);
      __builtin_amdgcn_global_load_lds(
          static_cast<const void*>(kb + (size_t)key * D + 8 * (lpiece ^ swz<D>(r))),
          (__attribute__((address_space(3))) void*)(ring + slot * TB + i * (16 * kWave)), 16, 0, 2);
    }
  };
  const int mytiles = wave < ntiles ? (ntiles - wave + 3) / 4 : 0;  // tiles wave + 4 i
  static_for<0, kRing - 1>([&](auto ic) __attribute__((always_inline)) {
    if (decltype(ic)::value < mytiles) issue(wave + 4 * decltype(ic)::value, ic);
  });
  bf16x8_t qa[KS];
  {
    const int w = c16 / a.G, gg = c16 - w * a.G;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qa[ks] = bf16x8_t{};
      if (c16 < a.R)
        qa[ks] = *reinterpret_cast<const bf16x8_t*>(
            a.q + ((((size_t)l * a.S + loc.s) * a.W + w) * a.Hq + h * a.G + gg) * D + 32 * ks +
            8 * g4);
    }
  }
  int last_seen[4];  // causal tail: the last key of the sequence that row 4 g4 + i sees
#pragma unroll
  for (int i = 0; i < 4; ++i) last_seen[i] = loc.ns - a.W + (4 * g4 + i) / a.G;
  float m[4], z[4];  // log2-domain reference and sum of exp2(c logit - m) per row
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    m[i] = -INFINITY;
    z[i] = 0.f;
  }
  auto compute = [&](int t, const bf16x8_t(&f)[KS]) __attribute__((always_inline)) {
    f32x4_t acc = f32x4_t{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa[ks], f[ks], acc, 0, 0, 0);
    if (g4 < RQ) {
      const int key = 16 * t + c16;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (key >= nkeys || (CAUSAL && key0 + key > last_seen[i])) acc[i] = -INFINITY;
        const float x = acc[i] * a.c;
        const float mn = fmaxf(m[i], x);
        const float ref = mn == -INFINITY ? 0.f : mn;  // no key seen yet: every term is 0
        z[i] = fmaf(z[i], fast_exp2(m[i] - ref), fast_exp2(fmaf(acc[i], a.c, -ref)));
        m[i] = mn;
      }
      *reinterpret_cast<f32x4_t*>(lg + (size_t)t * (64 * RQ)) = acc;
    }
  };
  for (int i0 = 0; i0 < mytiles; i0 += kRing) {
    static_for<0, kRing>([&](auto ic) __attribute__((always_inline)) {
      constexpr int u = decltype(ic)::value;
      const int i = i0 + u;
      if (i >= mytiles) return;
      if (i + kRing - 1 < mytiles)
        issue(wave + 4 * (i + kRing - 1), std::integral_constant<int, (u + kRing - 1) % kRing>{});
      const int ahead = min(kRing - 1, mytiles - 1 - i);
      // stores of logits count too: this waits for a little more than the tile
      wait_tiles<NL, kRing - 1>(ahead);
      bf16x8_t f[KS];
      read_fragments<u * TB>(fa, f);
      compute(wave + 4 * i, f);
    });
  }
  // merge the 16 lanes of each row, then the waves
  auto merge = [](float& M, float& Z, float mo, float zo) {
    const float mn = fmaxf(M, mo);
    if (mn != -INFINITY) {
      Z = Z * fast_exp2(M - mn) + zo * fast_exp2(mo - mn);
      M = mn;
    }
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      const float mo = __shfl_xor(m[i], o, kWave), zo = __shfl_xor(z[i], o, kWave);
      merge(m[i], z[i], mo, zo);
    }
    if (c16 == 0) part[wave][4 * g4 + i] = make_float2(m[i], z[i]);
  }
  __syncthreads();
  if (tid < kMaxFewRows) {
    float2 p = part[0][tid];
#pragma unroll
    for (int w = 1; w < kThreads / kWave; ++w) merge(p.x, p.y, part[w][tid].x, part[w][tid].y);
    a.partial[((size_t)lh * a.total_chunks + g) * kMaxFewRows + tid] = p;
  }
}

// One workgroup per (head, chunk) of the launch, the heads in reverse (the
// logits written last are still in the caches).
template <int RQ>
__global__ __launch_bounds__(kThreads) void row_sums_kernel(SaliencyArgs a, int lh0, int heads) {
  __shared__ float2 part[kThreads / kWave][kMaxFewRows];
  const int tid = threadIdx.x, lane = tid & 63;
  const int b = blockIdx.x / a.total_chunks, g = blockIdx.x - b * a.total_chunks;
  const int lr = heads - 1 - b, lh = lh0 + lr;
  const ChunkLoc loc = find_chunk(a, g);
  const int nch = chunks_of(a, loc.s);
  const int key0 = (g - loc.first) * a.chunk;
  const int nkeys = min(a.chunk, loc.ns - key0);
  // the row LSEs: thread t merges row t % 16 of chunks t / 16, t / 16 + 16, ..
  const int row = tid & 15;
  const float2* __restrict__ pp =
      a.partial + ((size_t)lh * a.total_chunks + loc.first) * kMaxFewRows + row;
  float M = -INFINITY, Z = 0.f;
  auto merge = [&](float mo, float zo) {
    const float mn = fmaxf(M, mo);
    if (mn != -INFINITY) {
      Z = Z * exp2f(M - mn) + zo * exp2f(mo - mn);
      M = mn;
    }
  };
  for (int c = tid >> 4; c < nch; c += kThreads / 16) {
    const float2 p = pp[(size_t)c * kMaxFewRows];
    merge(p.x, p.y);
  }
#pragma unroll
  for (int o = 16; o < kWave; o <<= 1) {
    const float mo = __shfl_xor(M, o, kWave), zo = __shfl_xor(Z, o, kWave);
    merge(mo, zo);
  }
  if (lane < 16) part[tid >> 6][row] = make_float2(M, Z);
  __syncthreads();
  M = -INFINITY;
  Z = 0.f;
#pragma unroll
  for (int w = 0; w < kThreads / kWave; ++w) merge(part[w][row].x, part[w][row].y);
  // +inf for padding rows and rows that see no key (probability 0), as store_row_lse
  const float l2 = row < a.R && Z > 0.f ? M + log2f(Z) : INFINITY;
  float lse[4 * RQ];
#pragma unroll
  for (int r = 0; r < 4 * RQ; ++r) lse[r] = __shfl(l2, r, kWave);
  const float* __restrict__ lg =
      a.logits + ((size_t)lr * a.logit_slots + logit_slot(loc.s, loc.seq0) + key0) * (4 * RQ);
  float* __restrict__ out = a.sal + (size_t)lh * a.ntot + loc.seq0 + key0;
  for (int e = tid; e < nkeys; e += kThreads) {
    const float* __restrict__ p = lg + (size_t)(e >> 4) * (64 * RQ) + 4 * (e & 15);
    f32x4_t v[RQ];
#pragma unroll
    for (int q = 0; q < RQ; ++q) v[q] = *reinterpret_cast<const f32x4_t*>(p + 64 * q);
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < RQ; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) sum += fast_exp2(fmaf(v[q][i], a.c, -lse[4 * q + i]));
    out[e] = sum;
  }
}

template <int D, int RQ>
hipError_t launch_few_rows_q(const SaliencyArgs& a, int lh0, int heads, hipStream_t st) {
  const dim3 grid((unsigned)heads * (unsigned)a.total_chunks);
  if (a.causal)
    hipLaunchKernelGGL((row_logits_kernel<D, RQ, true>), grid, dim3(kThreads), 0, st, a, lh0);
  else
    hipLaunchKernelGGL((row_logits_kernel<D, RQ, false>), grid, dim3(kThreads), 0, st, a, lh0);
  hipLaunchKernelGGL(row_sums_kernel<RQ>, grid, dim3(kThreads), 0, st, a, lh0, heads);
  return hipGetLastError();
}

template <int D>
hipError_t launch_few_rows_d(const SaliencyArgs& a, int lh0, int heads, hipStream_t st) {
  return a.R <= 4 ? launch_few_rows_q<D, 1>(a, lh0, heads, st)
                  : launch_few_rows_q<D, 2>(a, lh0, heads, st);
}

}  // namespace

// At R = 16 the logits (64 bytes per key, written and read) cost what the second
// read of K from the Infinity Cache does: 603 against 602 us at d 128, 320
// against 317 at d 64.
bool few_rows(int R) { return R <= kFewRows; }
int few_rows_quads(int R) { return R <= 4 ? 1 : 2; }

hipError_t launch_few_rows(const SaliencyArgs& a, int d, int lh0, int heads, hipStream_t st) {
  return d == 128 ? launch_few_rows_d<128>(a, lh0, heads, st)
                  : launch_few_rows_d<64>(a, lh0, heads, st);
}

}  // namespace stepkv
