// The two per-head projections around the decode kernel for every shape outside the bf16 fast paths (any dims, fp32
// or bf16 storage), on v_mfma_f32_16x16x4_f32: everything is multiplied and accumulated in fp32.
//   * absorb_q:  q~_b[i] = W^UK_(b),(i) q_i                                        (Step 1, Section 2.1, per block)
//   * merge + up-projection + block sum:  out[i] = out_scale * sum_b z_b[i] W^UV_(b),(i)   (Step 3, Eq. (5), Eq. (6))
// Both take 16 sequences as the MFMA M dimension, so that a weight element is read once per 16 sequences.
#include "f32_tile.h"

namespace mlra {
namespace {

using namespace f32_tile;

constexpr float kLn2 = 0.6931471805599453f;

// four elements of a row of `len` from k on, zero beyond its end (no conditional loads: the address is clamped)
template <bool VEC, typename T>
__device__ __forceinline__ typename RawOf<T>::type load_row4(const T* row, int k, int len) {
  typename RawOf<T>::type x;
  if constexpr (VEC) {
    x.load(row + min(k, len - 4));
  } else {
    x.zero();
#pragma unroll
    for (int e = 0; e < 4; ++e) x.set(e, row[min(k + e, len - 1)]);
  }
  return x;
}
__device__ __forceinline__ f32x4 cut_row4(f32x4 v, int k, int len) {
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = k + e < len ? v[e] : 0.f;
  return v;
}

// ------------------------------------------------------------------------------------------------
// absorb_q.  One workgroup per (head, block, 16 sequences); wave w produces channel tiles w and w + 4 of every eight
// (SPLIT, for blocks of at most two tiles: every wave produces both, from a quarter of the k groups each, and the four
// parts are added through LDS).
// Query rows are the A operand, weight rows (one per latent channel, contiguous along d_h) the B operand; k is dealt
// as 16 i + 4 q + j (q = lane / 16, j = step), so that both are read four elements at a time, straight from global
// memory: a weight element is used by one workgroup only, and U k groups (3 U loads) are in flight per wave.
// Every MFMA starts from zero and the partial sums of four products are added as a tree: chained through one
// accumulator, 128 products have a rounding error of sqrt(64.5) roundings (2.0e-7 of the result, 2-norm), as a tree of
// sqrt(7.5) (7.3e-8; a dot product split over 64 lanes, one workgroup per sequence, had 7.35e-8).
// Bound by the weights' stream at small batches: 8 sequences, 128 heads, 4 blocks x 128 channels in fp32 (33.5 MB)
// take 9.5 us; one workgroup per sequence, which read them once each, took 53.
// ------------------------------------------------------------------------------------------------
template <typename T, bool VEC, int U, bool SPLIT>   // U: k groups in flight
__global__ __launch_bounds__(256) void absorb_q_f32_kernel(const T* __restrict__ q_nope, const T* __restrict__ w_uk,
                                                           T* __restrict__ q_abs, int batch, int h, int d_h,
                                                           int n_blocks, int groups, int d_cb, float fold,
                                                           const T* __restrict__ q_rope, T* __restrict__ q_rope_out,
                                                           int d_r) {
  typedef typename RawOf<T>::type Raw;
  const int head = blockIdx.x, b = blockIdx.y, m0 = blockIdx.z * 16, tid = threadIdx.x;
  const int n_seq = min(16, batch - m0), q_heads = h * groups;
  if (b == n_blocks) {   // (launched only when the softmax scale is folded in) the RoPE queries of this head
    for (int id = tid; id < n_seq * groups * d_r; id += 256) {
      const int c = id % d_r, grp = id / d_r % groups, s = m0 + id / (d_r * groups);
      const size_t off = ((size_t)s * q_heads + grp * h + head) * d_r + c;
      store_f32(q_rope_out, off, load_f32(q_rope, off) * fold);
    }
    return;
  }
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), q = lane >> 4, r16 = lane & 15;
  const int q_head = (b / (n_blocks / groups)) * h + head;   // Eq. (6): block b serves the heads of its group
  const size_t ldw = (size_t)h * d_h;
  const T* const qrow = q_nope + ((size_t)(m0 + min(r16, n_seq - 1)) * q_heads + q_head) * d_h;
  constexpr int TS = SPLIT ? 1 : 4;      // distance of this wave's two channel tiles
  for (int ct0 = SPLIT ? 0 : wave; ct0 * 16 < d_cb; ct0 += 8) {
    const T* wrow[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
      wrow[t] = w_uk + ((size_t)b * d_cb + min((ct0 + TS * t) * 16 + r16, d_cb - 1)) * ldw + (size_t)head * d_h;
    f32x4 acc[2] = {};
    for (int k0 = SPLIT ? wave * 16 * U : 0; k0 < d_h; k0 += (SPLIT ? 64 : 16) * U) {
      Raw a[U], w[U][2];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int k = k0 + 16 * i + 4 * q;
        a[i] = load_row4<VEC>(qrow, k, d_h);
#pragma unroll
        for (int t = 0; t < 2; ++t) w[i][t] = load_row4<VEC>(wrow[t], k, d_h);
      }
      __builtin_amdgcn_sched_barrier(0);
      f32x4 sum[2][U];
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int k = k0 + 16 * i + 4 * q;
        const f32x4 av = cut_row4(a[i].get(), k, d_h);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const f32x4 wv = cut_row4(w[i][t].get(), k, d_h);
          f32x4 part[4];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            part[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[e], wv[e], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
          sum[t][i] = (part[0] + part[1]) + (part[2] + part[3]);
#pragma unroll
          for (int s = 1; (i + 1) % (2 * s) == 0 && s < U; s *= 2) sum[t][i + 1 - 2 * s] += sum[t][i + 1 - s];
        }
        __builtin_amdgcn_sched_barrier(0);   // (or all 64 partial sums would be held at once)
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[t] += sum[t][0];
    }
    if constexpr (SPLIT) {
      __shared__ __attribute__((aligned(16))) f32x4 part[2][4][64];
#pragma unroll
      for (int t = 0; t < 2; ++t) part[t][wave][lane] = acc[t];
      __syncthreads();
      if (wave >= 2) return;               // wave t adds and stores tile t
      acc[0] = (part[wave][0][lane] + part[wave][1][lane]) + (part[wave][2][lane] + part[wave][3][lane]);
    }
#pragma unroll
    for (int t = 0; t < (SPLIT ? 1 : 2); ++t) {
      const int c = (SPLIT ? wave : ct0 + 4 * t) * 16 + r16;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (c < d_cb && 4 * q + i < n_seq)
          store_f32(q_abs, (((size_t)(m0 + 4 * q + i) * n_blocks + b) * h + head) * d_cb + c, acc[t][i] * fold);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// merge + up-projection.  One workgroup per (output head, 16 sequences, 64 output columns); the head's latent channels
// (all blocks of its group, R of them) go through in slabs of at most SLAB:
//   1. this wave's share of the slab's W^UV rows is fetched into registers (in flight during 2 and 3);
//   2. sixteen lanes per (sequence, block), four pairs at a time (one thread, if there are at most four slots), reduce
//      the chunks' (m, l) to the maximum m* and 1 / L in LDS, and write the log-sum-exp;
//   3. z = sum_k 2^(m_k - m*) Z_k / L of the slab is built in LDS, a thread's four-channel pieces side by side (eight
//      single channels, if the rows are not made of runs of four); with few sequences the chunks of a piece are dealt to
//      several threads (KP of them) and added in LDS;
//   4. out += z W^UV: z rows (sequences) are the A operand, W^UV rows the B operand (k dealt as 16 i + 4 q + j; column
//      tile ct takes columns 4 c + ct, so that a lane reads four consecutive ones), the four waves take every
//      fourth k group each and are added through LDS at the end.
// Bound by the streams of the weights and the partials: on the shape above (33.5 MB + 16.8 MB of partials in eight
// chunks) 20.6 us; one workgroup per (head, sequence) took 63.  A slab of 512 takes 300 to 354 registers per wave, most of
// them weights; heads of few channels have one of 128 (up to 157 registers, a quarter of the LDS), see the rule below.
// ------------------------------------------------------------------------------------------------
constexpr int kSlabBlocks = 64, kChannels = 8;

template <typename T, typename TO, bool VEC, int SLAB>
__global__ __launch_bounds__(256) void merge_upproj_f32_kernel(
    const float* __restrict__ part_z, const float* __restrict__ part_ml, const int32_t* __restrict__ seq_lens,
    const T* __restrict__ w_uv, TO* __restrict__ out, float* __restrict__ lse, int batch, int h, int d_h, int n_blocks,
    int d_cb, int n_splits, int chunk, const int32_t* __restrict__ fitted_chunk, float out_scale, int groups,
    const T* __restrict__ gate) {
  typedef typename RawOf<T>::type Raw;
  constexpr int kZPitch = SLAB + 4, kPieces = SLAB / 64, kZRows = 16 * kZPitch, kExchange = 4 * 16 * 68;
  static_assert(16 * SLAB / 4 <= kPieces * 256, "every piece of a slab needs a thread");
  static_assert(kPieces * 256 * 4 <= kZRows && kChannels * 256 <= kZRows, "the chunk parts are exchanged in the z rows' space");
  __shared__ __attribute__((aligned(16))) float zs[kZRows > kExchange ? kZRows : kExchange];   // (the waves' sums as well)
  __shared__ float mtab[16 * kSlabBlocks], itab[16 * kSlabBlocks];
  __shared__ int act[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, r16 = lane & 15;
  // output head blockIdx.x = grp * h + head; its branches are the bpg blocks of group grp (Eq. (6); one group of all
  // blocks is Eq. (5))
  const int head = blockIdx.x % h, grp = blockIdx.x / h, m0 = blockIdx.y * 16, col0 = blockIdx.z * 64;
  const int bpg = n_blocks / groups, b0 = grp * bpg, R = bpg * d_cb;
  const int n_seq = min(16, batch - m0);
  const size_t ldw = (size_t)h * d_h;
  // (at most kSlabBlocks blocks per slab: with fewer than nine channels a block, a slab is whole blocks)
  const int slab = min(SLAB, kSlabBlocks * d_cb);
  const T* const wcol = w_uv + (size_t)b0 * d_cb * ldw + (size_t)head * d_h;
  f32x4 acc[4] = {opaque_zero4(), opaque_zero4(), opaque_zero4(), opaque_zero4()};
  if (fitted_chunk) chunk = *fitted_chunk;   // (the decode kernel's own choice)
  if (tid < 16) {
    const int n = tid < n_seq ? seq_lens[m0 + tid] : 0;
    act[tid] = min(n_splits, chunks_of(n, chunk));
  }

  for (int r0 = 0; r0 < R; r0 += slab) {
    const int len = min(slab, R - r0);
    // 1. (a row past the slab repeats its last row; z is zero there, and so is the row once it is used)
    constexpr int KG = SLAB / 16 / 4;
    Raw w[VEC ? KG : 1][4];
    auto fetch_w = [&](int i, Raw (&x)[4]) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int r = r0 + min((4 * i + wave) * 16 + 4 * q + j, len - 1);
        x[j] = load_row4<VEC>(wcol + (size_t)r * ldw, col0 + 4 * r16, d_h);
      }
    };
    if constexpr (VEC) {                             // (element loads would not fit the registers beside 3.)
#pragma unroll
      for (int i = 0; i < KG; ++i)
        if ((4 * i + wave) * 16 < len) fetch_w(i, w[i]);   // (uniform per wave)
    }
    // 2.
    const int blk0 = r0 / d_cb, nblk = (r0 + len - 1) / d_cb - blk0 + 1;
    const int n_pairs = n_seq * nblk;
    auto ml_of = [&](int sl, int bb) {
      return part_ml + ((((size_t)(m0 + sl) * n_blocks + b0 + blk0 + bb) * n_splits) * h + head) * 2;
    };
    auto put_pair = [&](int sl, int bb, float m_star, float L) {
      mtab[sl * kSlabBlocks + bb] = m_star;
      itab[sl * kSlabBlocks + bb] = L > 0.f ? 1.f / L : 0.f;
      if (lse && blockIdx.z == 0 && (blk0 + bb) * d_cb >= r0)
        lse[((size_t)(m0 + sl) * n_blocks + b0 + blk0 + bb) * h + head] = L > 0.f ? (m_star + log2f(L)) * kLn2 : -INFINITY;
    };
    if (n_splits <= 4) {       // a thread per pair, its chunks and the length fetched at once
      for (int pair = tid; pair < n_pairs; pair += 256) {
        const int sl = pair / nblk, bb = pair - sl * nblk;
        const float* ml = ml_of(sl, bb);
        const int n_act = min(n_splits, chunks_of(seq_lens[m0 + sl], chunk));
        float2 got[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) got[k] = *(const float2*)(ml + (size_t)min(k, n_splits - 1) * h * 2);
        float m_star = kNegBig, L = 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k < n_act) m_star = fmaxf(m_star, got[k].x);
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (k < n_act) L += exp2f(got[k].x - m_star) * got[k].y;
        put_pair(sl, bb, m_star, L);
      }
    } else {
      __syncthreads();         // (act)
      for (int pair0 = tid >> 4; pair0 < n_pairs; pair0 += 64) {
        float2 first[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int pair = min(pair0 + 16 * i, n_pairs - 1), sl = pair / nblk;
          first[i] = *(const float2*)(ml_of(sl, pair - sl * nblk) + (size_t)min(r16, n_splits - 1) * h * 2);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int pair = pair0 + 16 * i, sl = pair / nblk, bb = pair - sl * nblk;
          if (pair >= n_pairs) break;
          const int n_act = act[sl];
          const float* ml = ml_of(sl, bb);
          float m_star = r16 < n_act ? fmaxf(kNegBig, first[i].x) : kNegBig, L = 0.f;
          for (int k = r16 + 16; k < n_act; k += 16) m_star = fmaxf(m_star, ml[(size_t)k * h * 2]);
#pragma unroll
          for (int o = 8; o > 0; o >>= 1) m_star = fmaxf(m_star, __shfl_xor(m_star, o));
          if (r16 < n_act) L = exp2f(first[i].x - m_star) * first[i].y;
          for (int k = r16 + 16; k < n_act; k += 16) {
            const float2 got = *(const float2*)(ml + (size_t)k * h * 2);
            L += exp2f(got.x - m_star) * got.y;
          }
#pragma unroll
          for (int o = 8; o > 0; o >>= 1) L += __shfl_xor(L, o);
          if (r16 == 0) put_pair(sl, bb, m_star, L);
        }
      }
    }
    __syncthreads();           // the tables and act are there; the previous slab's z rows are no longer read
    // 3.  (zero: rows past the batch, channels past the slab's end up to its last k group's)
    const int pad = (len + 15) / 16 * 16;
    if constexpr (VEC) {
      const int per_row = len / 4, items = n_seq * per_row;
      int max_act = 0;
      for (int sl = 0; sl < n_seq; ++sl) max_act = max(max_act, act[sl]);
      const int KP = max(1, min(kPieces * 256 / items, max_act));
      f32x4 z[kPieces];
      const float* src[kPieces];
      const float* mls[kPieces];
      int n_act[kPieces], kfirst[kPieces];
      float m_star[kPieces];
#pragma unroll
      for (int u = 0; u < kPieces; ++u) {
        const int id = tid + 256 * u, kp = id / items, it = id - kp * items;
        const int sl = it / per_row, r = r0 + 4 * (it - sl * per_row), b = b0 + r / d_cb;
        const bool live = kp < KP;
        z[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        kfirst[u] = kp;
        n_act[u] = live ? act[sl] : 0;
        const size_t unit0 = ((size_t)(m0 + sl) * n_blocks + b) * n_splits;
        src[u] = part_z + (live ? (unit0 * h + head) * d_cb + r % d_cb : 0);
        mls[u] = part_ml + (live ? (unit0 * h + head) * 2 : 0);
        m_star[u] = live ? mtab[sl * kSlabBlocks + r / d_cb - blk0] : 0.f;
      }
      for (int k = 0; k < max_act; k += KP) {
        f32x4 v[kPieces];
        float m[kPieces];
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
          const int kk = k + kfirst[u];
          const size_t at = kk < n_act[u] ? (size_t)kk * h : 0;
          v[u] = *(const f32x4*)(src[u] + at * d_cb);
          m[u] = mls[u][at * 2];
        }
#pragma unroll
        for (int u = 0; u < kPieces; ++u) {
          const bool on = k + kfirst[u] < n_act[u];
          const float wk = exp2f(m[u] - m_star[u]);
#pragma unroll
          for (int e = 0; e < 4; ++e) z[u][e] += on ? wk * v[u][e] : 0.f;
        }
      }
      if (KP > 1) {       // (uniform) add the chunk parts
#pragma unroll
        for (int u = 0; u < kPieces; ++u)
          if (kfirst[u] < KP) *(f32x4*)(zs + 4 * (tid + 256 * u)) = z[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kPieces; ++u)
          if (tid + 256 * u < items)
            for (int kp = 1; kp < KP; ++kp) z[u] += *(const f32x4*)(zs + 4 * (tid + 256 * u + kp * items));
        __syncthreads();
      }
#pragma unroll
      for (int u = 0; u < kPieces; ++u) {
        const int it = tid + 256 * u;
        if (it < items) {
          const int sl = it / per_row, c = 4 * (it - sl * per_row);
          *(f32x4*)(zs + sl * kZPitch + c) = z[u] * itab[sl * kSlabBlocks + (r0 + c) / d_cb - blk0];
        }
      }
      for (int t = tid; t < 16 * (pad / 4); t += 256) {
        const int sl = t / (pad / 4), c = 4 * (t - sl * (pad / 4));
        if (sl >= n_seq || c >= len) *(f32x4*)(zs + sl * kZPitch + c) = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    } else {              // (rows that are not made of aligned runs of four: one channel at a time, eight in flight)
      const int items = n_seq * len;
      int max_act = 0;
      for (int sl = 0; sl < n_seq; ++sl) max_act = max(max_act, act[sl]);
      const int KP = max(1, min(256 * kChannels / items, max_act)), total = items * KP;   // (KP > 1: one pass)
      for (int base = tid; base - tid < total; base += 256 * kChannels) {
        const int np = min(kChannels, (total - (base - tid) + 255) / 256);   // (uniform)
        const float* src[kChannels];
        const float* mls[kChannels];
        float z[kChannels], m_star[kChannels];
        int n_act[kChannels], at[kChannels], zrow[kChannels], kfirst[kChannels];
#pragma unroll
        for (int u = 0; u < kChannels; ++u) {
          if (u >= np) break;
          const int id = min(base + 256 * u, total - 1), kp = id / items, it = id - kp * items;
          const int sl = it / len, c = it - sl * len, bb = (r0 + c) / d_cb;
          const size_t unit0 = ((size_t)(m0 + sl) * n_blocks + b0 + bb) * n_splits;
          src[u] = part_z + (unit0 * h + head) * d_cb + r0 + c - bb * d_cb;
          mls[u] = part_ml + (unit0 * h + head) * 2;
          kfirst[u] = kp;
          n_act[u] = act[sl];
          at[u] = sl * kSlabBlocks + bb - blk0;
          zrow[u] = sl * kZPitch + c;
          m_star[u] = mtab[at[u]];
          z[u] = 0.f;
        }
        for (int k = 0; k < max_act; k += KP) {
          float v[kChannels], m[kChannels];
#pragma unroll
          for (int u = 0; u < kChannels; ++u) {
            if (u >= np) break;
            const size_t o = k + kfirst[u] < n_act[u] ? (size_t)(k + kfirst[u]) * h : 0;
            v[u] = src[u][o * d_cb];
            m[u] = mls[u][o * 2];
          }
#pragma unroll
          for (int u = 0; u < kChannels; ++u) {
            if (u >= np) break;
            z[u] += k + kfirst[u] < n_act[u] ? exp2f(m[u] - m_star[u]) * v[u] : 0.f;
          }
        }
        if (KP > 1) {     // (uniform) add the chunk parts
#pragma unroll
          for (int u = 0; u < kChannels; ++u)
            if (u < np && base + 256 * u < total) zs[base + 256 * u] = z[u];
          __syncthreads();
#pragma unroll
          for (int u = 0; u < kChannels; ++u)
            if (u < np && base + 256 * u < items)
              for (int kp = 1; kp < KP; ++kp) z[u] += zs[base + 256 * u + kp * items];
          __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < kChannels; ++u)
          if (u < np && base + 256 * u < items) zs[zrow[u]] = z[u] * itab[at[u]];
      }
      for (int t = tid; t < 16 * pad; t += 256) {
        const int sl = t / pad, c = t - sl * pad;
        if (sl >= n_seq || c >= len) zs[sl * kZPitch + c] = 0.f;
      }
    }
    __syncthreads();
    // 4.
    auto multiply = [&](int i, const Raw (&x)[4]) {
      const int k = (4 * i + wave) * 16 + 4 * q;
      const f32x4 a = *(const f32x4*)(zs + r16 * kZPitch + k);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 wv = x[j].get();
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          const float wx = k + j < len ? wv[ct] : 0.f;
          acc[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], wx, acc[ct], 0, 0, 0);
        }
      }
    };
    if constexpr (VEC) {
#pragma unroll
      for (int i = 0; i < KG; ++i)
        if ((4 * i + wave) * 16 < len) multiply(i, w[i]);
    } else {
#pragma unroll 1
      for (int i = 0; i < KG; ++i)
        if ((4 * i + wave) * 16 < len) {
          fetch_w(i, w[0]);
          multiply(i, w[0]);
        }
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i)
    *(f32x4*)(zs + (wave * 16 + 4 * q + i) * 68 + 4 * r16) = f32x4{acc[0][i], acc[1][i], acc[2][i], acc[3][i]};
  __syncthreads();
  const int cols = min(64, d_h - col0);
  for (int id = tid; id < n_seq * 64; id += 256) {
    const int sl = id >> 6, j = id & 63;
    if (j >= cols) continue;
    float v = 0.f;
#pragma unroll
    for (int g = 0; g < 4; ++g) v += zs[(g * 16 + sl) * 68 + j];
    const size_t o = ((size_t)(m0 + sl) * h * groups + blockIdx.x) * d_h + col0 + j;
    store_f32(out, o, v * out_scale * (gate ? load_f32(gate, o) : 1.f));   // gate: Appendix E, O^attn = Attention . G
  }
}

// runs of four elements at `p` and at every multiple of four elements from it are aligned for one load
bool aligned4(const void* p, int dtype) { return (uintptr_t)p % (dtype == MLRA_BF16 ? 8 : 16) == 0; }

}  // namespace

int launch_absorb_q_f32(int batch, int h, int d_h, int n_blocks, int groups, int d_cb, const void* q_nope,
                        const void* w_uk, void* q_abs, int dtype, hipStream_t stream, float fold, const void* q_rope,
                        void* q_rope_out, int d_r) {
  const dim3 grid(h, n_blocks + (q_rope_out ? 1 : 0), (batch + 15) / 16);
  const bool vec = d_h % 4 == 0 && aligned4(q_nope, dtype) && aligned4(w_uk, dtype);
#define MLRA_ABSORB_U(T, VEC, U, SPLIT)                                                                              \
  absorb_q_f32_kernel<T, VEC, U, SPLIT><<<grid, 256, 0, stream>>>(                                                   \
      (const T*)q_nope, (const T*)w_uk, (T*)q_abs, batch, h, d_h, n_blocks, groups, d_cb, fold, (const T*)q_rope,    \
      (T*)q_rope_out, d_r)
  // As many k groups at a time as a short row has: the rest of a step is multiplied with zeros (16 sequences, 128 heads,
  // 4 blocks x 128 channels, d_h = 64: 6.7 us with four groups, 9.9 with eight); element loads go four groups at a time.
  // Long rows of narrow blocks are shared by the waves (60 sequences x 8 heads x 4 channels, d_h = 256: 4.3 us, by one
  // wave 6.7).
#define MLRA_ABSORB(T, VEC)                                                 \
  do {                                                                      \
    if (d_h <= 32) MLRA_ABSORB_U(T, VEC, 2, false);                         \
    else if (d_h <= 64) MLRA_ABSORB_U(T, VEC, 4, false);                    \
    else if (d_cb <= 32 && d_h <= 128) MLRA_ABSORB_U(T, VEC, 2, true);      \
    else if (d_cb <= 32) MLRA_ABSORB_U(T, VEC, 4, true);                    \
    else MLRA_ABSORB_U(T, VEC, (VEC ? 8 : 4), false);                       \
  } while (0)
  if (dtype == MLRA_BF16) {
    if (vec) MLRA_ABSORB(bf16_t, true); else MLRA_ABSORB(bf16_t, false);
  } else {
    if (vec) MLRA_ABSORB(float, true); else MLRA_ABSORB(float, false);
  }
#undef MLRA_ABSORB
#undef MLRA_ABSORB_U
  return check_launch();
}

int launch_merge_upproj_f32(const DecodeArgs& a) {
  const dim3 grid(a.h * a.groups, (a.batch + 15) / 16, (a.d_h + 63) / 64);
  const bool vec = a.d_h % 4 == 0 && a.d_cb % 4 == 0 && aligned4(a.w_uv, a.dtype);
  // One small slab where it holds all channels of a head: several workgroups then share a CU (510 sequences, 32 heads,
  // one block of 4 channels, d_h = 256: 33 us, with the large slab 107; one workgroup per head and sequence 41).
  const bool small = a.n_blocks / a.groups * a.d_cb <= 128;
#define MLRA_MERGE(T, TO, VEC)                                \
  do {                                                        \
    if (small) MLRA_MERGE_SLAB(T, TO, VEC, 128);              \
    else MLRA_MERGE_SLAB(T, TO, VEC, 512);                    \
  } while (0)
#define MLRA_MERGE_SLAB(T, TO, VEC, SLAB)                                                                           \
  merge_upproj_f32_kernel<T, TO, VEC, SLAB><<<grid, 256, 0, a.stream>>>(                                            \
      a.part_z, a.part_ml, a.seq_lens, (const T*)a.w_uv, (TO*)a.out, a.lse, a.batch, a.h, a.d_h, a.n_blocks, a.d_cb, \
      a.plan.n_splits, a.plan.chunk_tokens, a.fitted ? a.chunk_tab : nullptr, a.out_scale, a.groups, (const T*)a.gate)
#define MLRA_MERGE_OUT(T, VEC)                                  \
  do {                                                          \
    if (a.out_dtype == MLRA_BF16) MLRA_MERGE(T, bf16_t, VEC);   \
    else MLRA_MERGE(T, float, VEC);                             \
  } while (0)
  if (a.dtype == MLRA_BF16) {
    if (vec) MLRA_MERGE_OUT(bf16_t, true); else MLRA_MERGE_OUT(bf16_t, false);
  } else {
    if (vec) MLRA_MERGE_OUT(float, true); else MLRA_MERGE_OUT(float, false);
  }
#undef MLRA_MERGE_OUT
#undef MLRA_MERGE
#undef MLRA_MERGE_SLAB
  return check_launch();
}

}  // namespace mlra
