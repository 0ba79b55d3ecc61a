// Global top-B selection (Sec. 5.2 last paragraph, Algorithm 1 phase 3) and
// the retained-row plan of eq. problem, one workgroup per (sequence, head).
//
// Scores map to order-preserving uint32 keys (NaN -> -inf, -0 -> +0). A radix
// search finds the key tau of the B-th largest prunable score and how many
// tokens equal to tau must be kept. It counts 2048 equal bins between a lower
// bound for tau and the largest key, then searches the bin that holds the
// B-th key: that bin's few keys are gathered into LDS, and ballots rank up to
// 64 of them at once. The write-out walks positions in order: tokens above tau
// are kept, tokens equal to tau are kept while their rank among equals is below
// that count (lower positions first), protected tokens are always kept.
//
// A thread holds runs of four consecutive positions (4 tid + 4096 b in block
// b): one 16-byte load of scores and one 4-byte load of protected flags per
// run. Rows of up to 65536 tokens keep their keys in registers, in code
// for 1, 2, 4, 8 or 16 blocks chosen by the row's own length; longer rows are
// read again in every phase, 8 blocks at a time. In a batch of 2 to 64
// sequences the workgroups take the rows of the longest sequences first.
//
// What bounds it: vector issue on the one CU that holds a row and, for few or
// short rows, the chain of loads, barriers and LDS round trips; so scans and
// reductions run on DPP, a phase takes one or two barriers, and ties that are
// all kept take a cheaper write-out. Times of stepkv_select, before (one
// position per slot of 1024, up to three radix passes over all keys) and now:
// 256 rows of 32768 tokens 21.4 -> 12.7 us, one such row 17.5 -> 10.9, 256 rows
// of 16384 21.7 -> 10.5, 16 sequences of 4k to 32k tokens x 112 heads
// 163 -> 81, 8 rows of 60000 136 -> 21, 64 rows of 131071 360 -> 70.
#include "common.h"
#include "internal.h"

#include <type_traits>

namespace stepkv {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr int kBlock = 4 * kThreads;  // positions of one block: four per thread
constexpr int kCachedBlocks = 16;     // blocks held in registers (rows of up to 65536 tokens)
constexpr int kStreamBlocks = 8;      // blocks per pass over a longer row

// A protected token holds this key: above every score's key
// (+inf maps to 0xFF800000), so it is kept by the same test as a score above
// tau; positions past the sequence hold 0. Neither is a candidate.
constexpr uint32_t kProtKey = 0xFFFFFFFFu;
// No score maps to key 1 (it would be a NaN's), so `key == 1` is never a tie.
constexpr uint32_t kNoKey = 1u;

constexpr int kDigitBits = 11;
constexpr int kBins = 1 << kDigitBits;
constexpr int kList = 1024;  // keys of one bin that the search takes into LDS
static_assert(kBins == 2 * kThreads, "each thread owns two bins");

// Inclusive prefix sum over the wave in lane order (DPP row shifts, then the
// row totals broadcast to the rows above: no LDS round trip).
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}

// Maximum (MAX) or minimum over the wave, in every lane.
template <bool MAX>
__device__ __forceinline__ uint32_t wave_extreme(uint32_t v) {
  auto pick = [](uint32_t a, int b) { return MAX ? max(a, (uint32_t)b) : min(a, (uint32_t)b); };
  v = pick(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x111, 0xf, 0xf, false));
  v = pick(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x112, 0xf, 0xf, false));
  v = pick(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x114, 0xf, 0xf, false));
  v = pick(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x118, 0xf, 0xf, false));
  v = pick(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xa, 0xf, false));
  v = pick(v, __builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xc, 0xf, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The median of three (v_med3_u32).
__device__ __forceinline__ uint32_t median(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));
}

// Lanes of one bin from which a wave adds to the histogram by groups: LDS
// atomics of many lanes on one word run one after another (256 rows of 32768
// scores with a handful of distinct values: 80 us without the groups, 30 with).
constexpr int kClustered = 16;

// Add one to h[bin] for every active lane, the first two distinct bins with one
// atomic each.
__device__ __forceinline__ void hist_add_grouped(uint32_t* h, bool active, uint32_t bin, int lane) {
  uint64_t rest = ballot(active);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    if (rest == 0ull) return;
    const int leader = __builtin_ctzll(rest);
    const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
    const uint64_t same = ballot(bin == lb) & rest;
    if (lane == leader) atomicAdd(&h[lb], (uint32_t)__popcll(same));
    rest &= ~same;
  }
  if ((rest >> lane) & 1ull) atomicAdd(&h[bin], 1u);
}

// Kept candidates of one slot grouped by step: one atomic per step per wave.
__device__ __forceinline__ void count_kept_steps(int32_t* kept, int nsteps, int k, int lane) {
  const bool ok = k >= 0 && k < nsteps;
  uint64_t pend = ballot(ok);
  while (pend) {
    const int leader = __builtin_ctzll(pend);
    const int kk = __shfl(k, leader, kWave);
    const uint64_t grp = ballot(ok && k == kk);
    if (lane == leader) atomicAdd(&kept[kk], (int)__popcll(grp));
    pend &= ~grp;
  }
}

struct RowSetup {
  int s, lh, seq0, ns, B, nsteps;
  int32_t* kept;
};

// Rows of the sequence of rank q when the sequences are ordered by decreasing
// length (equal lengths by index), for batches of 2 to 64 sequences:
// workgroups are dispatched in block order, so the rows of the longest
// sequences start first and the shortest fill the end of the launch. Every
// wave computes it from one round of loads of the sequence offsets.
__device__ __forceinline__ void longest_first(const SelectArgs& a, int q, RowSetup& r) {
  const int lane = threadIdx.x & 63;
  const bool in = lane < a.S;
  const int c0 = in ? a.cu_seqlens[lane] : 0;
  const int len = in ? a.cu_seqlens[lane + 1] - c0 : -1;
  int rank = 0;
  for (int j = 0; j < a.S; ++j) {
    const int lj = __shfl(len, j, kWave);
    rank += (lj > len || (lj == len && j < lane)) ? 1 : 0;
  }
  // ranks are a permutation of 0 .. S-1
  r.s = uniform(__builtin_ctzll(ballot(in && rank == q)));
  r.seq0 = uniform(__shfl(c0, r.s, kWave));
  r.ns = uniform(__shfl(len, r.s, kWave));
}

__device__ __forceinline__ RowSetup row_setup(const SelectArgs& a) {
  RowSetup r;
  const int q = blockIdx.x / a.LH;
  r.lh = blockIdx.x - q * a.LH;
  if (a.S > 1 && a.S <= kWave) {
    longest_first(a, q, r);
  } else {
    r.s = q;
    r.seq0 = a.cu_seqlens[r.s];
    r.ns = a.cu_seqlens[r.s + 1] - r.seq0;
  }
  r.B = a.budgets ? max(1, a.budgets[r.s]) : a.budget;
  const int st0 = a.kept ? a.cu_steps[r.s] : 0;
  r.nsteps = a.kept ? a.cu_steps[r.s + 1] - st0 : 0;
  r.kept = a.kept ? a.kept + (size_t)r.lh * a.total_steps + st0 : nullptr;
  if (r.kept) {
    for (int k = threadIdx.x; k < r.nsteps; k += kThreads) r.kept[k] = 0;
    __threadfence();  // the zeros reach L2 before any wave's atomics below
  }
  return r;
}

__device__ __forceinline__ int budget_of(const SelectArgs& a, int s) {
  return a.budgets ? max(1, a.budgets[s]) : a.budget;
}

// Protected tokens of sequence s, counted by one wave: 16 at a time from
// aligned 16-byte words, the unaligned head and tail one byte at a time.
__device__ __forceinline__ int count_protected(const SelectArgs& a, int s) {
  const int lane = threadIdx.x & 63;
  const int seq0 = a.cu_seqlens[s], ns = a.cu_seqlens[s + 1] - seq0;
  const int misal = (int)(reinterpret_cast<uintptr_t>(a.prot + seq0) & 15);
  const int head = min(ns, (16 - misal) & 15);
  const int nvec = (ns - head) / 16;
  int np = 0;
  if (lane < head) np += a.prot[seq0 + lane] != 0;
  const uint4* vp = reinterpret_cast<const uint4*>(a.prot + seq0 + head);
#pragma unroll 4
  for (int i = lane; i < nvec; i += kWave) {
    const uint4 w = vp[i];
    const uint32_t x[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {  // one bit per nonzero byte
      uint32_t b = x[c] | (x[c] >> 4);
      b |= b >> 2;
      b |= b >> 1;
      np += __builtin_popcount(b & 0x01010101u);
    }
  }
  for (int i = head + 16 * nvec + lane; i < ns; i += kWave) np += a.prot[seq0 + i] != 0;
  return __builtin_amdgcn_readlane((int)wave_scan((uint32_t)np), 63);
}

// Retained rows of the sequences t0 <= t < t1, t = t0 + wave + 16 k per wave
// (cu_retained[s+1] - cu_retained[s] = n_protected_s + min(B_s, N_s - n_protected_s)),
// summed over the workgroup. Block-uniform call.
__device__ __forceinline__ int retained_between(const SelectArgs& a, int t0, int t1, uint32_t* scratch) {
  const int wave = uniform(threadIdx.x >> 6);
  int acc = 0;
  for (int t = t0 + wave; t < t1; t += kWaves) {
    const int nt = a.cu_seqlens[t + 1] - a.cu_seqlens[t];
    const int np = count_protected(a, t);
    acc += np + min(budget_of(a, t), nt - np);
  }
  if ((threadIdx.x & 63) == 0) scratch[wave] = (uint32_t)acc;
  __syncthreads();
  int sum = 0;
  for (int w = 0; w < kWaves; ++w) sum += (int)scratch[w];
  __syncthreads();
  return sum;
}

// Without heads there are no selection workgroups; one workgroup writes the plan.
__global__ __launch_bounds__(kThreads) void retained_plan_kernel(SelectArgs a) {
  __shared__ uint32_t scratch[kWaves];
  int acc = 0;
  if (threadIdx.x == 0) a.cu_retained[0] = 0;
  for (int s = 0; s < a.S; ++s) {
    acc += retained_between(a, s, s + 1, scratch);
    if (threadIdx.x == 0) a.cu_retained[s + 1] = acc;
  }
}

// The same plan from the selection workgroups of head 0: the workgroup of
// sequence s counts the protected tokens of the sequences before it, one
// sequence per wave (none with a single sequence), and adds its own sequence
// once its candidate count npr = N_s - n_protected_s is known.
__device__ __forceinline__ void write_retained(const SelectArgs& a, int s, int before, int ns,
                                               int npr, int B) {
  if (threadIdx.x == 0) {
    if (s == 0) a.cu_retained[0] = 0;
    a.cu_retained[s + 1] = before + (ns - npr) + min(B, npr);
  }
}

struct Scratch {
  uint32_t hist[kBins];  // bins of the search; clear on entry to every count
  uint32_t list[kList];  // the keys of the bin searched last
  uint32_t cnt[kCachedBlocks * kWaves];  // write-out: per (block, wave) sure | ties << 16
  uint32_t red[4][kWaves];
  uint32_t wtot[kWaves];
  uint32_t found[3];  // bin, rank within it, keys in it
  uint32_t nlist;
};

// Order-preserving key of a score: NaN -> -inf and -0 -> +0 in float
// arithmetic, then the sign flip.
__device__ __forceinline__ uint32_t order_key(float p) {
  const uint32_t u = __float_as_uint(fmaxf(p, -INFINITY) + 0.0f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// Keys of NB blocks from P and prot (at the first block's base), whose first
// `rem` positions exist: keys[4 b + e] is position 4096 b + 4 tid + e. Every
// load of 4 blocks is issued before any is used (8 took 0.4 us more on a row of
// 32768 tokens); whole blocks take one 16-byte and one 4-byte load per thread
// (any alignment of P and prot).
template <int NB>
__device__ __forceinline__ void load_keys(const float* __restrict__ P,
                                          const uint8_t* __restrict__ prot, int rem,
                                          uint32_t* keys) {
  if constexpr (NB > 4) {
    load_keys<4>(P, prot, rem, keys);
#pragma unroll
    for (int j = 0; j < 16; ++j) asm volatile("" : "+v"(keys[j]));
    load_keys<NB - 4>(P + 4 * kBlock, prot + 4 * kBlock, rem - 4 * kBlock, keys + 16);
    return;
  }
  const int p4 = 4 * (int)threadIdx.x;
  float pv[4 * NB];
  uint32_t pw[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int left = rem - kBlock * b;  // uniform
    pw[b] = 0u;
    if (left >= kBlock) {
      __builtin_memcpy(&pv[4 * b], P + kBlock * b + p4, 16);
      __builtin_memcpy(&pw[b], prot + kBlock * b + p4, 4);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) pv[4 * b + e] = 0.f;
      if (left > 0) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int i = kBlock * b + min(p4 + e, left - 1);
          pv[4 * b + e] = P[i];
          pw[b] |= (uint32_t)prot[i] << (8 * e);
        }
      }
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int left = rem - kBlock * b;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      keys[4 * b + e] = ((pw[b] >> (8 * e)) & 0xFFu) == 0u ? order_key(pv[4 * b + e]) : kProtKey;
    }
    if (left < kBlock) {  // uniform: positions past the sequence
#pragma unroll
      for (int e = 0; e < 4; ++e) keys[4 * b + e] = p4 + e < left ? keys[4 * b + e] : 0u;
    }
  }
}

// One (sequence, head) row of ns tokens. STREAM: the keys are read again in
// every phase, kStreamBlocks blocks at a time; otherwise NB blocks hold the row.
template <int NB, bool STREAM>
struct Row {
  static constexpr int NK = 4 * NB;
  using Keys = uint32_t[NK];
  Scratch& sh;
  const float* __restrict__ P;
  const uint8_t* __restrict__ prot;
  const int32_t* __restrict__ sid;
  int32_t* __restrict__ out;
  int32_t* __restrict__ kept;  // or null
  int ns, nsteps;

  // f(segment) over the row's segments of NB blocks with their keys in `keys`
  template <typename F>
  __device__ __forceinline__ void each(Keys& keys, F&& f) const {
    if constexpr (STREAM) {
      const int nseg = (ns - 1) / (kBlock * NB) + 1;
      for (int sg = 0; sg < nseg; ++sg) {
        load_keys<NB>(P + (size_t)sg * (kBlock * NB), prot + (size_t)sg * (kBlock * NB),
                      ns - sg * (kBlock * NB), keys);
        f(sg);
      }
    } else {
      // fresh compares in every phase rather than lane masks held across phases
#pragma unroll
      for (int j = 0; j < NK; ++j) asm volatile("" : "+v"(keys[j]));
      f(0);
    }
  }

  // Candidates (npr, of this wave), the largest candidate key + 1 and this
  // thread's M-th largest key + 1 (0 or 1: fewer than M candidates). In the +1
  // domain a protected token is 0 and a position past the sequence 1.
  template <int M>
  __device__ __forceinline__ void survey(Keys& keys, int& npr, uint32_t& kmax1, uint32_t& mth1) const {
    uint32_t top[M];  // the largest so far, in descending order
#pragma unroll
    for (int q = 0; q < M; ++q) top[q] = 0u;
    each(keys, [&](int) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < NK; ++j) {
        const uint32_t x = keys[j] + 1u;
        npr += __popcll(ballot(x > 1u));
#pragma unroll
        for (int q = M - 1; q > 0; --q) top[q] = median(top[q - 1], top[q], x);
        top[0] = max(top[0], x);
      }
    });
    kmax1 = top[0];
    mth1 = top[M - 1];
  }

  // The bin holding the krem-th largest counted key (sh.hist, cleared while it
  // is read): thread t owns bins kBins - 1 - 2t and kBins - 2 - 2t, so that the
  // prefix in thread order counts the keys from the top.
  __device__ __forceinline__ void find_bin(int krem) const {
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int b0 = kBins - 2 - 2 * tid;
    uint2* hp = reinterpret_cast<uint2*>(&sh.hist[b0]);
    const uint2 c = *hp;
    *hp = make_uint2(0u, 0u);
    const uint32_t own = c.x + c.y;
    const uint32_t incl = wave_scan(own);
    if (lane == 63) sh.wtot[wave] = incl;
    __syncthreads();
    const uint32_t tot = wave_scan(lane < kWaves ? sh.wtot[lane] : 0u);
    const uint32_t before = wave ? (uint32_t)__builtin_amdgcn_readlane((int)tot, wave - 1) : 0u;
    const uint32_t above = before + incl - own, k = (uint32_t)krem;
    if (above < k && k <= above + own) {
      const bool hi = k <= above + c.y;
      sh.found[0] = (uint32_t)(hi ? b0 + 1 : b0);
      sh.found[1] = hi ? k - above : k - above - c.y;
      sh.found[2] = hi ? c.y : c.x;
      sh.nlist = 0u;
    }
    __syncthreads();
  }

  // The key tau of the krem-th largest of the candidates with keys in
  // [lo, lo + span] (span > 0) and the number `need` of tokens equal to tau
  // that are kept; need = 0 when every tie is kept, with tau then one below
  // that key. sh.hist is clear and visible on entry.
  __device__ __forceinline__ void search(Keys& keys, uint32_t lo, uint32_t span, int krem,
                                         uint32_t& tau, int& need) const {
    const int tid = threadIdx.x, lane = tid & 63;
    int shift, n;
    // the bin found last becomes the range; true when it is a single key
    auto narrow = [&]() __attribute__((always_inline)) {
      find_bin(krem);
      lo += uniform((int)sh.found[0]) << shift;
      krem = uniform((int)sh.found[1]);
      n = uniform((int)sh.found[2]);
      span = (1u << shift) - 1u;
      tau = lo;
      need = krem;
      return shift == 0;
    };
    do {  // count the row's keys (again only while a bin holds more than kList)
      shift = max(0, 32 - kDigitBits - __builtin_clz(span));
      each(keys, [&](int) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {  // keys 0 and kProtKey fall outside
          uint32_t d[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) d[e] = keys[4 * b + e] - lo;
          const uint64_t act = ballot(d[0] <= span);
          bool clustered = false;  // many lanes share the first lane's bin
          if (act != 0ull) {
            const uint32_t lead =
                (uint32_t)__builtin_amdgcn_readlane((int)d[0], __builtin_ctzll(act)) >> shift;
            clustered = __popcll(ballot(d[0] >> shift == lead)) >= kClustered;
          }
          if (clustered) {
#pragma unroll
            for (int e = 0; e < 4; ++e) hist_add_grouped(sh.hist, d[e] <= span, d[e] >> shift, lane);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (d[e] <= span) atomicAdd(&sh.hist[d[e] >> shift], 1u);
          }
        }
      });
      __syncthreads();
      if (narrow()) return;
    } while (n > kList);
    each(keys, [&](int) __attribute__((always_inline)) {  // the bin's keys into LDS, in any order
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        uint32_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) d[e] = keys[4 * b + e] - lo;
        if (min(min(d[0], d[1]), min(d[2], d[3])) <= span) {  // few runs hold one
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (d[e] <= span) sh.list[atomicAdd(&sh.nlist, 1u)] = lo + d[e];
        }
      }
    });
    __syncthreads();
    const int nlist = n;
    while (n > kWave) {
      shift = max(0, 32 - kDigitBits - __builtin_clz(span));
      const uint32_t d = tid < nlist ? sh.list[tid] - lo : 0u;
      if (tid < nlist && d <= span) atomicAdd(&sh.hist[d >> shift], 1u);
      __syncthreads();
      if (narrow()) return;
      if (n <= kWave) {  // the list's keys in the bin, to its front
        const uint32_t key = tid < nlist ? sh.list[tid] : 0u;
        __syncthreads();
        if (tid < nlist && key - lo <= span) sh.list[atomicAdd(&sh.nlist, 1u)] = key;
        __syncthreads();
      }
    }
    // rank the last keys: lane l holds key l, wave w ranks keys w, w + 16, ..
    const int wave = uniform(tid >> 6);
    const uint32_t mine = lane < n ? sh.list[lane] : 0u;  // 0: below every candidate
    for (int i = wave; i < n; i += kWaves) {
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)mine, i);
      const int gt = __popcll(ballot(mine > o)), ge = __popcll(ballot(mine >= o));
      if (gt < krem && krem <= ge && lane == 0) {  // equal keys write equal values
        sh.found[0] = o;
        sh.found[1] = (uint32_t)(krem - gt);
        sh.found[2] = (uint32_t)(ge - gt);
      }
    }
    __syncthreads();
    tau = (uint32_t)uniform((int)sh.found[0]);
    need = uniform((int)sh.found[1]);
    if (need == uniform((int)sh.found[2])) {  // every tie is kept: all above tau - 1
      --tau;
      need = 0;
    }
  }

  // Ordered write-out. Per (block, wave) the numbers of sure keeps and of ties
  // go to LDS, in position order; every wave scans them and ranks its own
  // tokens with ballots (a lane's four positions follow each other). A tie is
  // kept when fewer than `need` ties precede it, so the tokens kept before
  // position p are the sure keeps before p plus min(ties before p, need).
  // Without TIES only keys above t_sure are kept.
  template <bool TIES>
  __device__ __forceinline__ void write_out(Keys& keys, uint32_t t_sure, int need) const {
    const uint32_t t_tie = TIES ? t_sure : kNoKey;
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    int sure0 = 0, tie0 = 0;  // sure keeps and ties of the segments before this one
    each(keys, [&](int sg) __attribute__((always_inline)) {
      uint32_t cw = 0u;  // lane b: block b of this wave
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        uint32_t cs = 0u, ct = 0u;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          cs += (uint32_t)__popcll(ballot(keys[4 * b + e] > t_sure));
          if (TIES) ct += (uint32_t)__popcll(ballot(keys[4 * b + e] == t_tie));
        }
        uint32_t c = cs | (ct << 16);
        asm volatile("" : "+s"(c));  // counted here, so that no ballot outlives its block
        cw = lane == b ? c : cw;
      }
      if (STREAM) __syncthreads();  // the counts of the segment before this one are read
      if (lane < NB) sh.cnt[lane * kWaves + wave] = cw;
      __syncthreads();
      // four (block, wave) pairs per lane, in position order
      uint4 c4 = make_uint4(0u, 0u, 0u, 0u);
      if (lane < 4 * NB) c4 = reinterpret_cast<const uint4*>(sh.cnt)[lane];
      const uint32_t own = (c4.x + c4.y) + (c4.z + c4.w);
      const uint32_t incl = wave_scan(own);
      const int sub = wave & 3;  // this wave's pair of block b is the sub-th of lane 4 b + wave / 4
      const uint32_t base_lane = incl - own + (sub > 0 ? c4.x : 0u) + (sub > 1 ? c4.y : 0u) +
                                 (sub > 2 ? c4.z : 0u);
      int tid_w = 4 * tid;
      asm volatile("" : "+v"(tid_w));  // positions made here, not carried from the top
#pragma unroll
      for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int e = 0; e < 4; ++e) asm volatile("" : "+v"(keys[4 * b + e]));
        uint64_t bs[4], bt[4];
        uint64_t any = 0ull, anyt = 0ull;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bs[e] = ballot(keys[4 * b + e] > t_sure);
          bt[e] = TIES ? ballot(keys[4 * b + e] == t_tie) : 0ull;
          any |= bs[e];
          anyt |= bt[e];
        }
        if ((any | anyt) == 0ull) continue;
        const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)base_lane, 4 * b + (wave >> 2));
        int s_before = sure0 + (int)(base & 0xFFFFu), t_before = tie0 + (int)(base >> 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) s_before += lanes_below(bs[e]);
        if (TIES && anyt != 0ull) {
#pragma unroll
          for (int e = 0; e < 4; ++e) t_before += lanes_below(bt[e]);
        }
        const int i0 = tid_w + kBlock * b + (STREAM ? sg * (kBlock * NB) : 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t key = keys[4 * b + e];
          const bool sure = key > t_sure, tie = TIES && key == t_tie;
          const bool keep = sure || (tie && t_before < need);
          if (keep) out[s_before + (TIES ? min(t_before, need) : 0)] = i0 + e;
          s_before += sure ? 1 : 0;
          if (TIES) t_before += tie ? 1 : 0;
          if (kept) {
            const bool cand = key - 1u < kProtKey - 1u;
            count_kept_steps(kept, nsteps, (keep && cand) ? sid[i0 + e] : -1, lane);
          }
        }
      }
      if (STREAM) {
        const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        sure0 += (int)(all & 0xFFFFu);  // at most 32768 tokens a segment: both halves fit
        tie0 += (int)(all >> 16);
      }
    });
  }

  // The row's selection from its keys (STREAM: read from memory here).
  __device__ __forceinline__ void run(const SelectArgs& a, const RowSetup& r, int plan_before,
                                      Keys& keys) const {
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    // A lower bound for tau: each thread holding at least m candidates has m
    // of them at or above its m-th largest, so at least m times as many
    // candidates as there are such threads lie at or above the smallest of
    // those m-th largest keys; when ktake is within that number, tau lies there
    // too and the search skips every key below it. m = 1, 2, 4 or 8, the least
    // for which the budget can be within the bound.
    const int m = r.B <= kThreads ? 1 : (r.B <= 2 * kThreads ? 2 : (r.B <= 4 * kThreads ? 4 : 8));
    int npr = 0;  // wave total
    uint32_t kmax1, mth1;
    if (m == 1) survey<1>(keys, npr, kmax1, mth1);
    else if (m == 2) survey<2>(keys, npr, kmax1, mth1);
    else if (m == 4) survey<4>(keys, npr, kmax1, mth1);
    else survey<8>(keys, npr, kmax1, mth1);
    const bool has = mth1 > 1u;  // this thread holds at least m candidates
    const uint32_t nthr = (uint32_t)__popcll(ballot(has));
    kmax1 = wave_extreme<true>(kmax1);
    const uint32_t tmin = wave_extreme<false>(has ? mth1 - 1u : 0xFFFFFFFFu);
    reinterpret_cast<uint2*>(sh.hist)[tid] = make_uint2(0u, 0u);
    if (lane == 0) {
      sh.red[0][wave] = (uint32_t)npr;
      sh.red[1][wave] = kmax1;
      sh.red[2][wave] = tmin;
      sh.red[3][wave] = nthr;
    }
    __syncthreads();
    // the four results at once, one per row of 16 lanes: sums in rows 0 and 3,
    // maxima in rows 1 and 2 (of the complement for the minimum)
    const int row16 = lane >> 4;
    uint32_t v = (&sh.red[0][0])[lane];
    if (row16 == 2) v = ~v;
    const bool sums = row16 == 0 || row16 == 3;
    auto fold = [&](int t) { v = sums ? v + (uint32_t)t : max(v, (uint32_t)t); };
    fold(__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));  // row_shr:1
    fold(__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));  // row_shr:2
    fold(__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));  // row_shr:4
    fold(__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));  // row_shr:8
    npr = __builtin_amdgcn_readlane((int)v, 15);
    const uint32_t kmax = (uint32_t)__builtin_amdgcn_readlane((int)v, 31) - 1u;  // with candidates
    const uint32_t bound = ~(uint32_t)__builtin_amdgcn_readlane((int)v, 47);
    const int nthr_all = __builtin_amdgcn_readlane((int)v, 63);
    const int ktake = min(r.B, npr);
    const bool take_all = ktake == npr;
    if (r.lh == 0) write_retained(a, r.s, plan_before, r.ns, npr, r.B);

    uint32_t tau = 0u;
    int need = 0;
    if (!take_all) {
      uint32_t lbound = bound;  // tau >= lbound
      if (ktake > m * nthr_all) {  // no bound: the smallest candidate key
        uint32_t lowest = 0xFFFFFFFFu;
        each(keys, [&](int) __attribute__((always_inline)) {
#pragma unroll
          for (int j = 0; j < NK; ++j) lowest = min(lowest, keys[j] - 1u);  // 0 wraps to the top
        });
        lowest = wave_extreme<false>(lowest);
        __syncthreads();  // sh.red is read
        if (lane == 0) sh.red[0][wave] = lowest;
        __syncthreads();
        lbound = wave_extreme<false>(sh.red[0][lane & (kWaves - 1)]) + 1u;
      }
      if (lbound == kmax) {
        tau = kmax;  // every candidate from the bound up ties
        need = ktake;
      } else {
        search(keys, lbound, kmax - lbound, ktake, tau, need);
      }
    }
    // keys above tau (0: every token) are kept, and the first `need` equal to it
    if (need > 0) write_out<true>(keys, tau, need);
    else write_out<false>(keys, tau, 0);
  }
};

template <int NB, bool STREAM>
__device__ __forceinline__ void run_row(const SelectArgs& a, const RowSetup& r, int plan_before,
                                        Scratch& sh) {
  const size_t row = (size_t)r.lh * a.ntot + r.seq0;
  const Row<NB, STREAM> w{sh,           a.scores + row, a.prot + r.seq0, a.step_ids + r.seq0,
                          a.idx + row, r.kept,         r.ns,            r.nsteps};
  typename Row<NB, STREAM>::Keys keys;
  if constexpr (!STREAM) load_keys<NB>(w.P, w.prot, w.ns, keys);
  w.run(a, r, plan_before, keys);
}

// Rows of up to NB blocks: the code for the least of 1, 2, 4, .. NB blocks that
// holds this row.
template <int NB>
__device__ __forceinline__ void select_row(const SelectArgs& a, const RowSetup& r, int plan_before,
                                           Scratch& sh) {
  if constexpr (NB > 1) {
    if (r.ns <= kBlock * (NB / 2)) {
      select_row<NB / 2>(a, r, plan_before, sh);
      return;
    }
  }
  run_row<NB, false>(a, r, plan_before, sh);
}

template <int NB>
__global__ __launch_bounds__(kThreads) void select_cached_kernel(SelectArgs a) {
  __shared__ __attribute__((aligned(16))) Scratch sh;
  const RowSetup r = row_setup(a);
  const int plan_before = r.lh == 0 ? retained_between(a, 0, r.s, sh.wtot) : 0;
  select_row<NB>(a, r, plan_before, sh);
}

// Rows past 65536 tokens (and the shorter ones beside them) from memory.
__global__ __launch_bounds__(kThreads) void select_stream_kernel(SelectArgs a) {
  __shared__ __attribute__((aligned(16))) Scratch sh;
  const RowSetup r = row_setup(a);
  const int plan_before = r.lh == 0 ? retained_between(a, 0, r.s, sh.wtot) : 0;
  if (r.ns <= kBlock * kStreamBlocks) {
    select_row<kStreamBlocks>(a, r, plan_before, sh);
    return;
  }
  run_row<kStreamBlocks, true>(a, r, plan_before, sh);
}

// ---------------------------------------------------------------- priority and selection
// The priority (as the kernels of fuse.hip, value for value) and the selection
// of one row by one workgroup: the saliency of the row stays in registers, is
// pooled there (neighbouring runs come from the next lane by DPP and, at the
// ends of a wave, from LDS) and becomes P, which is written once and ranked from
// the registers. The row is not read again, and one launch takes the place of
// two to four. Bound by vector issue on the row's CU (about 55 instructions per
// position), for short rows by the chain of loads and barriers. Priority and
// selection before (separate launches) and now: 256 rows of 32768 tokens
// 33 + 25 -> 27 us, of 16384 22 + 24 -> 19, 8 rows of 8192 10 + 21 -> 10, 2 rows
// of 1024 9.5 + 20 -> 7.7, 16 sequences of 4k to 32k tokens x 112 heads
// 98 + 206 -> 152. Rows of up to 8 blocks, pooling windows of up to 9 and up to
// kRankSteps steps per sequence (the table of step utilities in LDS). 1024
// threads leave each 128 VGPRs: code for 8 blocks takes 113 to 121 of them up to
// windows of 5, all and 4 more in scratch at 7, and 21 to 26 in scratch at 9, all
// with about 20 scalars kept in vector lanes; code for 4 blocks takes 54 to 80
// (72 at a window of 7, so that one workgroup is resident on a CU, not two).
// Rows of 16 blocks would spill most of theirs.
constexpr int kRankSteps = 4096;
constexpr int kRankHalf = 4;
constexpr int kRankBlocks = 8;

// What rank_row holds in place of U for a protected token or a position past
// the sequence: below every U, which is a sum of exponentials (0 or more, or NaN
// of any payload), so u < 0 means masked and the maximum from 0 passes it over.
constexpr float kNoU = -1.f;

// The masked saliency at the ends of every wave's 256 positions, where the
// neighbouring wave's pooling reads it: run q of 256 positions is entry q + 1,
// its first four positions, then its last four; entries 0 and 16 NB + 1 stay 0.
struct Edges {
  float4 e[kRankBlocks * kWaves + 2][2];
};

template <int NB, int HALF, bool FLAGS>
__device__ __forceinline__ void rank_row(const FuseArgs& f, const SelectArgs& a, const RowSetup& r,
                                         int plan_before, float* bu_lds, Edges& ed, Scratch& sh) {
  if constexpr (NB > 1) {
    if (r.ns <= kBlock * (NB / 2)) {
      rank_row<NB / 2, HALF, FLAGS>(f, a, r, plan_before, bu_lds, ed, sh);
      return;
    }
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int p4 = 4 * tid;
  const size_t row = (size_t)r.lh * a.ntot + r.seq0;
  const float* __restrict__ A = f.sal + row;
  const uint8_t* __restrict__ prot = a.prot + r.seq0;
  const int st0 = f.cu_steps[r.s], nsteps = f.cu_steps[r.s + 1] - st0;

  // ---- every load of the row, issued before any is used
  float u[NB][4];  // the saliency, then U
  uint32_t pw[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int left = r.ns - kBlock * b;  // uniform
    pw[b] = 0xFFFFFFFFu;                 // past the sequence: not prunable
#pragma unroll
    for (int e = 0; e < 4; ++e) u[b][e] = 0.f;
    if (left >= kBlock) {
      __builtin_memcpy(u[b], A + kBlock * b + p4, 16);
      __builtin_memcpy(&pw[b], prot + kBlock * b + p4, 4);
    } else if (left > 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (p4 + e < left) {
          u[b][e] = A[kBlock * b + p4 + e];
          pw[b] = (pw[b] & ~(0xFFu << (8 * e))) | ((uint32_t)prot[kBlock * b + p4 + e] << (8 * e));
        }
      }
    }
  }
  // beta S of every step, and beta 0 for ids out of range
  for (int k = tid; k <= nsteps; k += kThreads) bu_lds[k] = f.beta * (k < nsteps ? f.util[st0 + k] : 0.f);
  if (tid < 2) ed.e[tid ? NB * kWaves + 1 : 0][tid ? 0 : 1] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int e = 0; e < 4; ++e) u[b][e] = ((pw[b] >> (8 * e)) & 0xFFu) == 0u ? u[b][e] : 0.f;
  }
  const bool edge = lane == 0 || lane == 63;
  if (HALF > 0) {
    if (edge) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
        ed.e[b * kWaves + wave + 1][lane ? 1 : 0] = make_float4(u[b][0], u[b][1], u[b][2], u[b][3]);
    }
    __syncthreads();
  }

  // ---- pooling in place, left to right as every pooling kernel adds, and the maximum
  float m = 0.f;  // U >= 0, and Th = 0 everywhere when the maximum is 0
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    float v[12];  // positions p4 - 4 .. p4 + 7
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 + e] = u[b][e];
    if (HALF > 0) {
      float4 h = make_float4(0.f, 0.f, 0.f, 0.f);  // lane 0: the run before, lane 63: the run after
      if (edge) h = ed.e[b * kWaves + wave + (lane ? 2 : 0)][lane ? 0 : 1];
      const float he[4] = {h.x, h.y, h.z, h.w};
      // wave_shr:1 and wave_shl:1; the lane without a source keeps its halo
#pragma unroll
      for (int e = 4 - HALF; e < 4; ++e)
        v[e] = __int_as_float(__builtin_amdgcn_update_dpp(
            __float_as_int(he[e]), __float_as_int(v[4 + e]), 0x138, 0xf, 0xf, false));
#pragma unroll
      for (int e = 0; e < HALF; ++e)
        v[8 + e] = __int_as_float(__builtin_amdgcn_update_dpp(
            __float_as_int(he[e]), __float_as_int(v[4 + e]), 0x130, 0xf, 0xf, false));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float acc = v[4 + e - HALF];
#pragma unroll
      for (int o = 1; o <= 2 * HALF; ++o) acc += v[4 + e - HALF + o];
      u[b][e] = ((pw[b] >> (8 * e)) & 0xFFu) == 0u ? acc : kNoU;
      m = fmaxf(m, u[b][e]);
    }
  }
  // step ids, on their way while the maximum is reduced
  const int32_t* __restrict__ sid = a.step_ids + r.seq0;
  int kk[NB][4];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int left = r.ns - kBlock * b, i0 = kBlock * b + p4;  // left: uniform
#pragma unroll
    for (int e = 0; e < 4; ++e) kk[b][e] = -1;
    if (left >= kBlock) {
      __builtin_memcpy(kk[b], sid + i0, 16);
    } else if (left > 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (p4 + e < left) kk[b][e] = sid[i0 + e];
    }
  }
  // non-negative floats order as their bits
  const uint32_t wm = wave_extreme<true>(__float_as_uint(m));
  if (lane == 0) sh.wtot[wave] = wm;
  __syncthreads();
  const float M = __uint_as_float(wave_extreme<true>(sh.wtot[lane & (kWaves - 1)]));
  const float inv = M > 0.f ? 1.0f / M : 0.f;

  // ---- P, written once; its keys take the place of U
  float* __restrict__ out = f.scores + row;
  typename Row<NB, false>::Keys keys;
  uint64_t bad_id = 0ull, bad_nf = 0ull;  // wave masks of STEPKV_FLAG_* conditions
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int left = r.ns - kBlock * b, i0 = kBlock * b + p4;
    float pv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool pr = !(u[b][e] < 0.f);
      const float bu = bu_lds[min((uint32_t)kk[b][e], (uint32_t)nsteps)];
      const float p = fmaf(f.alpha, u[b][e] * inv, bu);
      if (FLAGS) {
        bad_id |= ballot(pr && (uint32_t)kk[b][e] >= (uint32_t)nsteps);
        bad_nf |= ballot(pr && !finite(p));
      }
      pv[e] = pr ? p : -INFINITY;
      keys[4 * b + e] = pr ? order_key(p) : kProtKey;
    }
    if (FLAGS) asm volatile("" : "+s"(bad_id), "+s"(bad_nf));  // no ballot outlives its block
    if (left >= kBlock) {
      __builtin_memcpy(out + i0, pv, 16);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (p4 + e < left) out[i0 + e] = pv[e];
        else keys[4 * b + e] = 0u;  // past the sequence
      }
    }
  }
  if (FLAGS) report_masks(f.status, bad_id, bad_nf);
  const Row<NB, false> w{sh, nullptr, prot, sid, a.idx + row, nullptr, r.ns, 0};
  w.run(a, r, plan_before, keys);
}

template <int NB, int HALF, bool FLAGS>
__global__ __launch_bounds__(kThreads) void rank_kernel(FuseArgs f, SelectArgs a) {
  __shared__ __attribute__((aligned(16))) Scratch sh;
  __shared__ Edges ed;
  extern __shared__ float bu_lds[];  // [max_steps + 1]
  const RowSetup r = row_setup(a);
  const int plan_before = r.lh == 0 ? retained_between(a, 0, r.s, sh.wtot) : 0;
  rank_row<NB, HALF, FLAGS>(f, a, r, plan_before, bu_lds, ed, sh);
}

}  // namespace

bool rank_fits(const FuseArgs& f) {
  return !f.stats && f.half <= kRankHalf && f.max_steps <= kRankSteps &&
         f.max_len <= kBlock * kRankBlocks;
}

hipError_t launch_rank(const FuseArgs& f, const SelectArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)a.S * (unsigned)a.LH), block(kThreads);
  const size_t dyn = sizeof(float) * ((size_t)f.max_steps + 1);
  const int blocks = (a.max_len + kBlock - 1) / kBlock;
  auto go = [&](auto half_c, auto flags_c) {
    constexpr int H = decltype(half_c)::value;
    constexpr bool F = decltype(flags_c)::value;
    if (blocks <= 1) hipLaunchKernelGGL((rank_kernel<1, H, F>), grid, block, dyn, st, f, a);
    else if (blocks <= 4) hipLaunchKernelGGL((rank_kernel<4, H, F>), grid, block, dyn, st, f, a);
    else hipLaunchKernelGGL((rank_kernel<kRankBlocks, H, F>), grid, block, dyn, st, f, a);
  };
  auto with_flags = [&](auto half_c) {
    if (f.status) go(half_c, std::true_type{});
    else go(half_c, std::false_type{});
  };
  switch (f.half) {
    case 0: with_flags(std::integral_constant<int, 0>{}); break;
    case 1: with_flags(std::integral_constant<int, 1>{}); break;
    case 2: with_flags(std::integral_constant<int, 2>{}); break;
    case 3: with_flags(std::integral_constant<int, 3>{}); break;
    default: with_flags(std::integral_constant<int, 4>{}); break;
  }
  return hipGetLastError();
}

// The least kernel that holds the longest row: code for more blocks takes more
// registers (82 for 8 blocks against 45 for up to 4, which lets two workgroups
// share a CU). With 16 blocks the 64 keys of a thread and the rest exceed its 128
// VGPRs: 58 are spilled to scratch, and it is still faster than reading the row
// again (8 rows of 60000, budget 2048: 26 us, streamed 36). Past 16 blocks they cannot be held.
hipError_t launch_select(const SelectArgs& a, hipStream_t st) {
  if (a.S * a.LH == 0) {
    hipLaunchKernelGGL(retained_plan_kernel, dim3(1), dim3(kThreads), 0, st, a);
    return hipGetLastError();
  }
  const dim3 grid((unsigned)a.S * (unsigned)a.LH), block(kThreads);
  const int blocks = (a.max_len + kBlock - 1) / kBlock;
  if (blocks <= 1) hipLaunchKernelGGL(select_cached_kernel<1>, grid, block, 0, st, a);
  else if (blocks <= 4) hipLaunchKernelGGL(select_cached_kernel<4>, grid, block, 0, st, a);
  else if (blocks <= 8) hipLaunchKernelGGL(select_cached_kernel<8>, grid, block, 0, st, a);
  else if (blocks <= kCachedBlocks)
    hipLaunchKernelGGL(select_cached_kernel<kCachedBlocks>, grid, block, 0, st, a);
  else hipLaunchKernelGGL(select_stream_kernel, grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace stepkv
