// Chunk length of a ragged batch, fitted by the kernel that works on the chunks.
//
// The host knows the longest sequence a cache can hold, not the lengths: chunks cut for the former leave compute units
// without work (short sequences use few of their slots) or some with twice the work of the others (the chunks of all
// sequences are a little more than a round).  The lengths of up to 64 sequences are one register per lane, so every
// wavefront fits the chunk length and finds its own chunk by itself: one more round trip to memory and 1 us for a few
// sequences, 4 us for 60.  Whole steps: fp32, 8 sequences of 300 to 2048 tokens x 128 heads 89.5 -> 76.9 us (the uniform
// chunks were 344 workgroups for 256 CUs); without the kernels in front that planned or ordered the chunks, four query tokens
// for 16 sequences of 1000 to 4093 93.4 -> 92.1 us, 4 sequences of 64K to 128K 148.2 -> 146.5.
#pragma once

#include "mlra_internal.h"

namespace mlra {
namespace chunk_fit {

constexpr int kMaxSeqs = 64;
constexpr int kTokens = 64;      // chunk lengths are multiples of this ("tiles")

struct Chunk {
  int seq, split;
};

// The chunk length in tokens.  n: this lane's sequence length, 0 from n_seqs on.  Each chunk is the work of `wgs`
// workgroups, `cus` of them run at a time, and a workgroup costs its tiles and `overhead` tiles more.  Lane k prices chunks
// of c_min + k step tiles (c_min: what the workspace has slots for).  Workgroups go out longest first: rounds of whole
// chunks, then the sequences' last pieces beside the whole chunks of the last round.  Pieces that find no room there come
// second on the units with the shortest first ones; both are about as long as the pieces are at that place if these spread
// evenly over the lengths up to a whole chunk.  No launch is shorter than the mean over the units.  The cheapest length
// wins, among equals the longest, for the fewest partials.  Every wavefront of a launch computes the same: it runs the same
// instructions on the same lengths.
// SHARED: a compute unit runs several workgroups at a time, which share its matrix pipe: their start-ups overlap, and one
// alone takes 8 % longer for its tiles (fp32 kernel, 8 sequences of 8192: 222 us in one round of long chunks, 213 in two of
// half the length).
template <bool SHARED>
__device__ __forceinline__ int fit_length(int n, int n_seqs, int wgs, int cus, int c_min, int overhead) {
  const int lane = threadIdx.x & 63, tiles = chunks_of(n, kTokens);
  int longest = max(tiles, c_min);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) longest = max(longest, __shfl_xor(longest, o));
  longest = min(longest, 0x7fffffff / kTokens);          // (in tokens it fits an int; c_min is no more than this)
  const int c = min(c_min + lane * ((c_min + 31) / 32), longest);
  const float c_inv = 1.f / (float)c;
  unsigned total = 0;
  int whole = 0, units = 0;
  for (int i = 0; i < n_seqs; ++i) {
    const int t = __builtin_amdgcn_readlane(tiles, i);
    const float x = (float)t;
    total += (unsigned)t;
    whole += (int)((x + 0.5f) * c_inv);                  // (rounding may miss by one from 2^20 tiles on: a price only)
    units += t > 0 ? (int)((x - 0.5f) * c_inv) + 1 : 0;
  }
  const float at_once = (float)cus / (float)wgs, cost = (float)overhead, w = (float)whole, u = (float)units;
  const float full = floorf(w / at_once), rests = u - w, per_round = SHARED ? 0.f : cost, one = (float)c + per_round;
  const float room = (full + 1.f) * at_once - w;        // places beside the whole chunks of the last round
  float last = room < at_once || rests > 0.f ? one : 0.f;
  if (rests > room) last = fmaxf(last, 2.f * ((float)c * (1.f - room / rests) + per_round));
  float price = fmaxf(full * one + last, u > at_once ? ((float)total + u * per_round) / at_once : 0.f);
  if (SHARED) price = price * (full * one + last < 1.5f * one ? 1.08f : 1.f) + cost;
  unsigned best = (unsigned)fminf(8.f * price, 67000000.f) << 6 | (unsigned)(63 - lane);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) best = min(best, (unsigned)__shfl_xor((int)best, o));
  return __builtin_amdgcn_readlane(c, 63 - (best & 63)) * kTokens;
}

// Chunks of `chunk` tokens in the whole batch.
__device__ __forceinline__ int count(int n, int chunk) {
  int units = chunks_of(n, chunk);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) units += __shfl_xor(units, o);
  return __builtin_amdgcn_readfirstlane(units);
}

// Chunk `index` (< count) of the batch: all whole chunks, then what is left of the sequences, longest first.
__device__ __forceinline__ Chunk find(int n, int n_seqs, int chunk, int index) {
  const int lane = threadIdx.x & 63;
  const int whole = n / chunk, rest = n - whole * chunk;
  int upto = whole;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int a = __shfl_up(upto, o);
    if (lane >= o) upto += a;
  }
  const int n_whole = __builtin_amdgcn_readlane(upto, 63);
  if (index < n_whole) {                 // (uniform) the first lane whose running count exceeds the index
    const int seq = __builtin_ctzll(__ballot(upto > index) | (1ull << 63));
    return Chunk{seq, index - (__builtin_amdgcn_readlane(upto, seq) - __builtin_amdgcn_readlane(whole, seq))};
  }
  int rank = 0;
  for (int i = 0; i < n_seqs; ++i) {
    const int r = __builtin_amdgcn_readlane(rest, i);
    rank += (r > rest || (r == rest && i < lane)) ? 1 : 0;
  }
  const int seq = __builtin_ctzll(__ballot(rest > 0 && rank == index - n_whole) | (1ull << 63));
  return Chunk{seq, __builtin_amdgcn_readlane(whole, seq)};
}

}  // namespace chunk_fit
}  // namespace mlra
