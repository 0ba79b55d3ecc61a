// Which (sequence, key chunk) a saliency workgroup works on, from the chunk
// list of SaliencyArgs (chunks of the sequences in order).
#pragma once

#include "common.h"
#include "internal.h"

namespace stepkv {

// Key chunks of sequence s: ceil(N_s / chunk), from cu_seqlens (s may differ
// between lanes) ...
__device__ __forceinline__ int chunks_in_memory(const SaliencyArgs& a, int s) {
  return (a.cu_seqlens[s + 1] - a.cu_seqlens[s] + a.chunk - 1) / a.chunk;
}

// ... or, for a wave-uniform s, from the argument tables when the batch has them.
__device__ __forceinline__ int chunks_of(const SaliencyArgs& a, int s) {
  if (a.S <= SaliencyArgs::kArgSeqs) return a.chunk_first[s + 1] - a.chunk_first[s];
  return chunks_in_memory(a, s);
}

// The sequence s holding global chunk g (chunks of the sequences in order) and
// its first global chunk: a wave-wide prefix over 64 sequences at a time, in
// every wave (g is below the chunk total, so some sequence holds it).
__device__ __forceinline__ void locate_chunk(const SaliencyArgs& a, int g, int& s_out,
                                             int& first_out) {
  const int lane = threadIdx.x & 63;
  int base = 0;
  s_out = a.S - 1;
  first_out = 0;
  for (int s0 = 0; s0 < a.S; s0 += kWave) {
    const int sq = s0 + lane;
    const int cnt = sq < a.S ? chunks_in_memory(a, sq) : 0;
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int o = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += o;
    }
    const int total = __shfl(incl, kWave - 1, kWave);
    if (g < base + total) {
      const int first = __builtin_ctzll(ballot(base + incl > g));
      s_out = s0 + first;
      first_out = base + __shfl(incl - cnt, first, kWave);
      return;
    }
    base += total;
  }
}

// Global chunk g (wave-uniform): its sequence s, the sequence's first global
// chunk, first key and length. Batches of up to kArgSeqs sequences search the
// argument tables (five scalar loads); larger ones take locate_chunk and read
// cu_seqlens.
struct ChunkLoc {
  int s, first, seq0, ns;
};

__device__ __forceinline__ ChunkLoc find_chunk(const SaliencyArgs& a, int g) {
  ChunkLoc r;
  if (a.S <= SaliencyArgs::kArgSeqs) {
    // the last s with chunk_first[s] <= g (a sequence without keys has no
    // chunk, so the search passes over it)
    int lo = 0;
#pragma unroll
    for (int step = SaliencyArgs::kArgSeqs / 2; step > 0; step >>= 1)
      if (a.chunk_first[lo + step] <= g) lo += step;
    r.s = lo;
    r.first = a.chunk_first[lo];
    r.seq0 = a.seq_first[lo];
    r.ns = a.seq_first[lo + 1] - r.seq0;
  } else {
    locate_chunk(a, g, r.s, r.first);
    r.s = uniform(r.s);
    r.first = uniform(r.first);
    // read into scalar registers: a value either branch may give stays scalar
    r.seq0 = uniform(a.cu_seqlens[r.s]);
    r.ns = uniform(a.cu_seqlens[r.s + 1]) - r.seq0;
  }
  return r;
}

// The first global chunk of sequence s: the chunks of the sequences before it.
__device__ __forceinline__ int first_chunk(const SaliencyArgs& a, int s) {
  if (a.S <= SaliencyArgs::kArgSeqs) return a.chunk_first[s];
  const int lane = threadIdx.x & 63;
  int acc = 0;
  for (int s0 = 0; s0 < s; s0 += kWave) {
    int cnt = s0 + lane < s ? chunks_in_memory(a, s0 + lane) : 0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, kWave);
    acc += cnt;
  }
  return acc;
}

}  // namespace stepkv
