// MFMA kernels for the two per-head projections around the decode kernel (bf16, d_h = 128):
//   * absorb_q:  q~_b[i] = W^UK_(b),(i) q_i                (Step 1, Section 2.1, per block)
//   * merge + up-projection + block sum:  out[i] = out_scale * sum_b z_b[i] W^UV_(b),(i)
//     (log-sum-exp merge of the context chunks, then Step 3 and the block sum of Eq. (5) as one
//      contraction over all n_blocks * d_cb latent channels)
// Both are batched over sequences as the MFMA M dimension so that each weight element is read once
// per workgroup, and both put the head index on the grid.
#include "mlra_internal.h"

namespace mlra {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kDh = 128;
constexpr float kNegBig = -1.0e30f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ int swz(int t) { return ((t & 3) << 1) | ((t >> 2) & 1); }

// Zero that the compiler cannot fold: an accumulator initialised from it is a real register operand, so
// every MFMA is emitted in the tied form (destination = accumulator input) and its destination can
// never be placed on top of its A / B operands.
__device__ __forceinline__ f32x16 opaque_zero() {
  float z = 0.f;
  asm volatile("" : "+v"(z));
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = z;
  return acc;
}

__device__ __forceinline__ short4v lds_tr16(const void* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)p);
}

// ------------------------------------------------------------------------------------------------
// absorb_q.  One workgroup per (head, block, 128 channels, 64 sequences); wave w produces the 32-channel tile ct0 + w of
// its four: out[seq][c] = sum_p q[seq][p] W[c][p].  An MFMA operand wants sixteen bytes of
// each of 32 rows per lane group, and rows of q (one per sequence) and of W (one per channel) lie 32 KiB
// apart: read in that shape, every load instruction touches 64 cache lines for 1 KiB.  So both are fetched
// as whole 256-byte rows (sixteen lanes a row), laid into LDS with a chunk swizzle, and the operands are
// read from there; the 64 query rows are fetched once per workgroup instead of once per wave.  The results
// pass through LDS as well, so that they leave as whole 16-byte pieces of the q_abs rows.  Larger batches
// put their 64-sequence tiles on the grid (the weights of a head are then read once from HBM and again
// from L2).
// ------------------------------------------------------------------------------------------------
constexpr int kAbsPitch = 128 * 2 + 16;   // bytes per staged sequence row (128 channels; +16: rows on different banks)
constexpr int kAbsQ = 64 * 256;           // LDS: the 64 query rows of the head ...
constexpr int kAbsW = 4 * 32 * 256;       // ... and 32 weight rows per wave (the result staging reuses this part)
static_assert(64 * kAbsPitch <= kAbsW, "the staged results must fit the weight rows' space");

__global__ __launch_bounds__(256) void absorb_q_mfma_kernel(const bf16_t* __restrict__ q_nope,
                                                            const bf16_t* __restrict__ w_uk,
                                                            bf16_t* __restrict__ q_abs, int batch, int h,
                                                            int n_blocks, int groups, int d_cb, float fold,
                                                            const bf16_t* __restrict__ q_rope,
                                                            bf16_t* __restrict__ q_rope_out, int d_r, int n_pass) {
  // h: heads per block; q_nope holds groups * h heads and block b reads those of its group (Eq. (6))
  // fold: factor applied to the absorbed queries before they are rounded (1, or tau log2(e) when the
  // softmax scale is folded into the queries); the workgroups behind those of the blocks (launched only
  // then) apply it to the RoPE queries of head blockIdx.x of every group.
  // Blocks wider than 128 channels (MLA, GLA-2) have one workgroup per 128 of them (n_pass).  One that walked its
  // block's passes had them one after the other, each a round trip to memory: 128 sequences, 128 heads, one block of 512
  // channels 17.4 -> 15.4 us.
  __shared__ __attribute__((aligned(16))) unsigned char smem[kAbsQ + kAbsW];
  if (blockIdx.y == (unsigned)(n_blocks * n_pass)) {
    const int m0r = blockIdx.z * 64, q_heads_r = h * groups, per_row = d_r >> 3;   // d_r % 8 == 0 (launcher)
    for (int id = threadIdx.x; id < 64 * groups * per_row; id += 256) {
      const int pc = id % per_row, grp = (id / per_row) % groups, s_ = m0r + id / (per_row * groups);
      if (s_ >= batch) continue;
      const size_t off = ((size_t)s_ * q_heads_r + grp * h + blockIdx.x) * d_r + pc * 8;
      bf16x8 v = *(const bf16x8*)(q_rope + off);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = (__bf16)((float)v[e] * fold);
      *(bf16x8*)(q_rope_out + off) = v;
    }
    return;
  }
  unsigned char* const qs = smem;
  unsigned char* const ws = smem + kAbsQ;
  unsigned char* const stage = ws;
  const int head = blockIdx.x, b = blockIdx.y / n_pass, first = 4 * (blockIdx.y % n_pass);
  const int q_head = (b / (n_blocks / groups)) * h + head, q_heads = h * groups;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, c32 = lane & 31;
  const size_t ldw = (size_t)h * kDh;
  const int m0 = blockIdx.z * 64;      // 64 sequences per workgroup
  // rows are stored with 16-byte chunk c at position c ^ (row % 16): the sixteen lanes that a 128-bit LDS
  // read serves together (rows 0-3, 12-15, 20-27 of one chunk column, and so on) then hit sixteen positions
  const int ld_chunk = tid & 15, ld_row = tid >> 4;          // loads: thread = (row % 16 of its pass, chunk)
  bf16x8 qld[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int seq = min(m0 + 16 * i + ld_row, batch - 1);
    qld[i] = *(const bf16x8*)(q_nope + ((size_t)seq * q_heads + q_head) * kDh + ld_chunk * 8);
  }
  bf16x8 areg[2][8];
  for (int ct0 = first; ct0 * 32 < d_cb; ct0 += 4 * n_pass) {
    const int ct = ct0 + wave;
    const bool live = ct * 32 < d_cb;                       // (uniform per wave)
    // this wave's 32 weight rows (a wave past the last channel tile repeats the last row and stores nothing)
    bf16x8 wld[8];
    {
      const int wl_chunk = lane & 15, wl_row = lane >> 4;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = min(ct * 32 + 4 * i + wl_row, d_cb - 1);
        wld[i] = *(const bf16x8*)(w_uk + ((size_t)b * d_cb + c) * ldw + (size_t)head * kDh + wl_chunk * 8);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = 4 * i + wl_row;
        *(bf16x8*)(ws + wave * (32 * 256) + r * 256 + ((wl_chunk ^ (r & 15)) << 4)) = wld[i];
      }
    }
    if (ct0 == first) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * i + ld_row;
        *(bf16x8*)(qs + r * 256 + ((ld_chunk ^ (r & 15)) << 4)) = qld[i];
      }
    }
    __syncthreads();
    bf16x8 breg[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      breg[ks] = *(const bf16x8*)(ws + wave * (32 * 256) + c32 * 256 + (((2 * ks + g) ^ (c32 & 15)) << 4));
    if (ct0 == first) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int ks = 0; ks < 8; ++ks)
          areg[t][ks] = *(const bf16x8*)(qs + (32 * t + c32) * 256 + (((2 * ks + g) ^ (c32 & 15)) << 4));
    }
    __syncthreads();      // every wave holds its operands: the weight rows' space becomes the result staging
    const int pass_ch = min(128, d_cb - ct0 * 32);          // channels this pass produces
    f32x16 acc[2] = {opaque_zero(), opaque_zero()};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(areg[0][ks], breg[ks], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(areg[1][ks], breg[ks], acc[1], 0, 0, 0);
    }
    if (live) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = 32 * t + (r >> 2) * 8 + g * 4 + (r & 3);
          *(bf16_t*)(stage + row * kAbsPitch + (wave * 32 + c32) * 2) = f32_to_bf16(acc[t][r] * fold);
        }
    }
    __syncthreads();
    // 64 rows x (pass_ch / 8) 16-byte pieces, one piece per thread and step
    const int pieces = pass_ch >> 3;
    for (int id = tid; id < 64 * pieces; id += 256) {
      const int row = id / pieces, pc = id - row * pieces, s_ = m0 + row;
      if (s_ < batch)
        *(bf16x8*)(q_abs + (((size_t)s_ * n_blocks + b) * h + head) * d_cb + ct0 * 32 + pc * 8) =
            *(const bf16x8*)(stage + row * kAbsPitch + pc * 16);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------------
// merge + up-projection.  One workgroup per (head, tile of up to 32 sequences), two of them resident per CU.
//   phase 0: the first 256 rows of this head's W^UV slice are fetched into registers, so that they are in flight while
//            phase 1 runs;
//   phase 1: merged z of the 32 sequences for all R = n_blocks * d_cb latent channels, rounded to bf16, is built in LDS
//            (row = sequence).  kDirect: every sequence has one chunk and the decode kernel has normalised and rounded
//            its row, which is only copied.  kRows / kItems: z = sum_k w_k z_k over the chunks, whose partials are
//            normalised bf16 rows / fp32 Z; a thread takes U items (sequence, 8 channels) at a time and the first
//            KK chunks of each are in flight while sixteen lanes (a thread, if there are at most
//            four slots) per (sequence, block) turn the chunks' (m, l) into the
//            weights w_k = 2^(m_k - m*) (l_k) / L in LDS and write the log-sum-exp;
//   phase 2: out[seq][j] = sum_r z[seq][r] W^UV[r][head*128 + j]; W^UV goes through LDS 128 rows at a time (the rows
//            after the next 128 are fetched into the registers that were just stored) and reaches the MFMA B operand
//            through transpose reads; wave w owns output columns [32 w, 32 w + 32).
// Bound by latency: a chain of a few round trips to memory per workgroup, which the second workgroup of the CU fills.
// One kernel for all three forms held the registers of the largest (448), so that a CU had one workgroup.
// Kernel times, before -> after the forms were split (128 heads, 512 latent channels): 128 sequences with gate and
// log-sum-exp 41 -> 19 us, 64 sequences 15.6 -> 13.0, 4 sequences of up to 128K in 32 chunk slots 22.4 -> 17.4, one
// sequence in 12 chunks 11.5 -> 8.9, fp32 partials of 128 sequences in 4 slots 32.9 -> 26.9.  Lane groups for two slots as
// well cost a step on 44 decode units 4 us (57.0 against 52.6): the shuffles of a pair take longer than its two loads.
// ------------------------------------------------------------------------------------------------
constexpr int kWRows = 128;       // W^UV rows in LDS at a time (32 KiB); twice as many in registers
enum MergeMode { kDirect, kRows, kItems };

template <typename TO, int MODE, int U, int KK>
__global__ __launch_bounds__(256, 2) void merge_upproj_mfma_kernel(
    const float* __restrict__ part_z, const float* __restrict__ part_ml, const int32_t* __restrict__ seq_lens,
    const bf16_t* __restrict__ w_uv, TO* __restrict__ out, float* __restrict__ lse, int batch, int h, int nb_total,
    int d_cb, int n_splits, int chunk, const int32_t* __restrict__ chunk_tab, float out_scale,
    const bf16_t* __restrict__ gate, int spw, int q_group, unsigned q_magic) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  // blockIdx.z = head group (Eq. (6)); one group of all blocks is Eq. (5).  h: heads per block; this
  // workgroup's head is h * group + head in out, and its branches are blocks [b0, b0 + n_blocks).
  const int n_blocks = nb_total / gridDim.z, b0 = blockIdx.z * n_blocks;
  const int R = n_blocks * d_cb;
  const int zpitch = R + 8;                               // bf16 elements per z row (+16 B against conflicts)
  const int units_per_seq = n_blocks * n_splits;
  unsigned char* wt = smem;                               // [kWRows][256 B], 16-byte chunks swizzled
  bf16_t* zt = (bf16_t*)(smem + kWRows * 256);            // [32][zpitch]
  float* wtab = (float*)(smem + kWRows * 256 + (size_t)32 * zpitch * 2);   // [32][units_per_seq] (not kDirect)
  // spw: sequences per workgroup (32, or fewer for small batches so that more workgroups share the merge;
  // the rest of the 32 MFMA rows is zero padding)
  const int head = blockIdx.x, m0 = blockIdx.y * spw;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, c32 = lane & 31;
  const size_t ldw = (size_t)h * kDh;
  const int n_valid = min(spw, batch - m0);
  const int items_per_row = R / 8, n_items = n_valid * items_per_row;

  // ---- phase 0: thread t owns 16-byte chunk t % 16 of rows t / 16 + 16 i of each part
  bf16x8 wreg[2][kWRows / 16];
  const bf16_t* wsrc = w_uv + ((size_t)b0 * d_cb + (tid >> 4)) * ldw + (size_t)head * kDh + (tid & 15) * 8;
  auto fetch_w = [&](int part, bf16x8 (&reg)[kWRows / 16]) {
#pragma unroll
    for (int i = 0; i < kWRows / 16; ++i)
      if (part * kWRows + 16 * i < R) reg[i] = *(const bf16x8*)(wsrc + (size_t)(part * kWRows + 16 * i) * ldw);
  };
  fetch_w(0, wreg[0]);
  fetch_w(1, wreg[1]);

  // ---- phase 1
  // q_group > 1: entries [i q_group, (i + 1) q_group) of the batch are the queries of one sequence, which share a length
  // (q_magic = 2^32 / q_group rounded up: an exact quotient for 16-bit numbers)
  auto len_of = [&](int seq) {
    if (q_group == 1) return seq_lens[seq];
    const int own = (int)__umulhi((unsigned)seq, q_magic);
    return max(0, seq_lens[own] - (q_group - 1 - (seq - own * q_group)));
  };
  auto active_chunks = [&](int seq) {
    const int ch = chunk_tab ? chunk_tab[seq] : chunk;
    return min(n_splits, chunks_of(len_of(seq), ch));
  };
  bf16x8 zero8;
#pragma unroll
  for (int e = 0; e < 8; ++e) zero8[e] = (__bf16)0.0f;
  // rows of sequences past the batch feed MFMA rows that are never stored; they only have to be finite
  for (int t = n_items + tid; t < 32 * items_per_row; t += 256)
    *(bf16x8*)(zt + (t / items_per_row) * zpitch + (t % items_per_row) * 8) = zero8;
  if constexpr (MODE == kDirect) {
    const bf16_t* zn = (const bf16_t*)part_z;
    for (int base = tid; base < n_items; base += U * 256) {
      bf16x8 row[U];
      int n[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int item = min(base + u * 256, n_items - 1), sl = item / items_per_row, r0 = (item % items_per_row) * 8;
        row[u] = *(const bf16x8*)(zn + (((size_t)(m0 + sl) * nb_total + b0 + r0 / d_cb) * h + head) * d_cb + r0 % d_cb);
        n[u] = len_of(m0 + sl);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int item = base + u * 256;
        // (what a sequence without tokens leaves in the workspace is discarded)
        if (item < n_items)
          *(bf16x8*)(zt + (item / items_per_row) * zpitch + (item % items_per_row) * 8) = n[u] > 0 ? row[u] : zero8;
      }
    }
    if (lse)
      for (int t = tid; t < n_valid * n_blocks; t += 256) {
        const int seq = m0 + t / n_blocks, b = b0 + t % n_blocks;
        const float2 ml = *(const float2*)(part_ml + (((size_t)seq * nb_total + b) * h + head) * 2);
        lse[((size_t)seq * nb_total + b) * h + head] =
            len_of(seq) > 0 && ml.y > 0.f ? (ml.x + log2f(ml.y)) * kLn2 : -INFINITY;
      }
  } else {
    const size_t z_stride = (size_t)h * d_cb;
    bool have_weights = false;
    for (int base0 = 0; base0 < n_items; base0 += U * 256) {
      const int base = base0 + tid;
      size_t pz[U];
      const float* wk[U];
      int na[U], sl[U], r0[U], kmax = 0;
      float z[U][8];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int item = min(base + u * 256, n_items - 1);
        sl[u] = item / items_per_row;
        r0[u] = (item % items_per_row) * 8;
        const int b = r0[u] / d_cb, c0 = r0[u] % d_cb;
        na[u] = base + u * 256 < n_items ? active_chunks(m0 + sl[u]) : 0;
        kmax = max(kmax, na[u]);
        pz[u] = ((((size_t)(m0 + sl[u]) * nb_total + b0 + b) * n_splits) * h + head) * d_cb + c0;
        wk[u] = wtab + sl[u] * units_per_seq + b * n_splits;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[u][e] = 0.f;
      }
      typedef __attribute__((ext_vector_type(MODE == kRows ? 4 : 8))) float raw_t;   // eight channels as stored
      raw_t raw[KK][U];
      auto load_chunks = [&](int k0) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const size_t at = pz[u] + (k0 + kk < na[u] ? k0 + kk : 0) * z_stride;   // (chunk 0's slot always exists)
            if constexpr (MODE == kRows) raw[kk][u] = *(const raw_t*)((const bf16_t*)part_z + at);
            else raw[kk][u] = *(const raw_t*)(part_z + at);
          }
      };
      load_chunks(0);
      if (!have_weights) {     // (uniform) weights of all (sequence, block) pairs, once
        have_weights = true;
        const int n_pairs = n_valid * n_blocks;
        if constexpr (KK == 2) {
          // at most four slots: one thread per pair, all of them in its registers
          for (int pair = tid; pair < n_pairs; pair += 256) {
            const int ps = pair / n_blocks, b = pair - ps * n_blocks, seq = m0 + ps, active = active_chunks(seq);
            const float* ml = part_ml + ((((size_t)seq * nb_total + b0 + b) * n_splits) * h + head) * 2;
            float2 got[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) got[k] = *(const float2*)(ml + (size_t)min(k, n_splits - 1) * h * 2);
            float m_star = kNegBig, L = 0.f, w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (k < active) m_star = fmaxf(m_star, got[k].x);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              w[k] = k < active ? exp2f(got[k].x - m_star) : 0.f;
              if (k < active) L += w[k] * got[k].y;
              if (MODE == kRows) w[k] *= got[k].y;
            }
            const float inv = L > 0.f ? 1.f / L : 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (k < active) wtab[ps * units_per_seq + b * n_splits + k] = w[k] * inv;
            if (lse)
              lse[((size_t)seq * nb_total + b0 + b) * h + head] = L > 0.f ? (m_star + log2f(L)) * kLn2 : -INFINITY;
          }
        } else {
        // (four pairs of a lane group at a time, so that their loads overlap; chunk l16 of each stays in a register,
        // and only chunks from 16 on are read twice)
        const int l16 = lane & 15;
        for (int pair0 = tid >> 4; pair0 < n_pairs; pair0 += 64) {
          float2 first[4];
          int active[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int pair = min(pair0 + 16 * i, n_pairs - 1), ps = pair / n_blocks, b = pair - ps * n_blocks;
            active[i] = active_chunks(m0 + ps);
            first[i] = *(const float2*)(part_ml + ((((size_t)(m0 + ps) * nb_total + b0 + b) * n_splits +
                                                    min(l16, n_splits - 1)) * h + head) * 2);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int pair = pair0 + 16 * i, ps = pair / n_blocks, b = pair - ps * n_blocks, seq = m0 + ps;
            if (pair >= n_pairs) break;
            const float* ml = part_ml + ((((size_t)seq * nb_total + b0 + b) * n_splits) * h + head) * 2;
            float* wrow = wtab + ps * units_per_seq + b * n_splits;
            float m_star = l16 < active[i] ? fmaxf(kNegBig, first[i].x) : kNegBig, L = 0.f, w0 = 0.f;
            for (int k = l16 + 16; k < active[i]; k += 16) m_star = fmaxf(m_star, ml[(size_t)k * h * 2]);
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) m_star = fmaxf(m_star, __shfl_xor(m_star, o));
            // (a partial that arrives normalised, z_k / l_k, carries its row sum in its weight)
            if (l16 < active[i]) {
              w0 = exp2f(first[i].x - m_star);
              L = w0 * first[i].y;
              if (MODE == kRows) w0 = L;
            }
            for (int k = l16 + 16; k < active[i]; k += 16) {
              const float2 got = *(const float2*)(ml + (size_t)k * h * 2);
              const float w = exp2f(got.x - m_star);
              L += w * got.y;
              wrow[k] = MODE == kRows ? w * got.y : w;
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) L += __shfl_xor(L, o);
            const float inv = L > 0.f ? 1.f / L : 0.f;
            if (l16 < active[i]) wrow[l16] = w0 * inv;
            for (int k = l16 + 16; k < active[i]; k += 16) wrow[k] *= inv;
            if (lse && l16 == 0)
              lse[((size_t)seq * nb_total + b0 + b) * h + head] = L > 0.f ? (m_star + log2f(L)) * kLn2 : -INFINITY;
          }
        }
        }
        __syncthreads();
      }
      for (int k0 = 0; k0 < kmax; k0 += KK) {
        if (k0 > 0) load_chunks(k0);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const bool on = k0 + kk < na[u];
            const float w = on ? wk[u][k0 + kk] : 0.f;
            // (an inactive chunk has weight 0; what its slot holds may be anything, NaN included)
            if constexpr (MODE == kRows) {
              const bf16x8 row = __builtin_bit_cast(bf16x8, raw[kk][u]);
#pragma unroll
              for (int e = 0; e < 8; ++e) z[u][e] += w != 0.f ? w * (float)row[e] : 0.f;
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e) z[u][e] += on ? w * raw[kk][u][e] : 0.f;
            }
          }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (base + u * 256 < n_items) {
          bf16x8 packed;
#pragma unroll
          for (int e = 0; e < 8; ++e) packed[e] = (__bf16)z[u][e];
          *(bf16x8*)(zt + sl[u] * zpitch + r0[u]) = packed;
        }
    }
  }

  // ---- phase 2 ----
  // The gate values of this lane's outputs are fetched here, all sixteen at once (rows past the batch repeat the last
  // one): fetched one by one between the stores at the end, each was a round trip to memory of its own (12 us of 39 on
  // 128 sequences).
  const int j = wave * 32 + c32;
  auto out_at = [&](int r) {             // accumulator register r: offset of its sequence slot in out and gate
    const int sl = (r >> 2) * 8 + g * 4 + (r & 3), s = m0 + min(sl, n_valid - 1);
    return ((size_t)s * h * gridDim.z + blockIdx.z * h + head) * kDh + j;
  };
  bf16_t gate_v[16];
  if (gate) {
#pragma unroll
    for (int r = 0; r < 16; ++r) gate_v[r] = gate[out_at(r)];
  }
  f32x16 acc = opaque_zero();
  // transpose-read offsets: the 16 lanes of a block fetch 4 consecutive rows x 16 output columns
  unsigned tr_off[2];
  {
    const int k = (lane & 15) >> 2, seg = lane & 3, hb = (lane >> 4) & 1;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int row = 8 * g + 4 * half + k;                 // + 16 per MFMA k-step (same swizzle: row & 7)
      const int cc = 4 * wave + 2 * hb + (seg >> 1);
      tr_off[half] = row * 256 + ((cc ^ swz(row & 7)) << 4) + ((seg & 1) << 3);
    }
  }
  auto part_step = [&](int part, bf16x8 (&reg)[kWRows / 16]) {
    const int row_base = part * kWRows;
    if (row_base >= R) return;                              // (uniform)
    __syncthreads();   // phase 1 done / previous rows consumed
#pragma unroll
    for (int i = 0; i < kWRows / 16; ++i) {
      const int row = (tid >> 4) + 16 * i, cc = tid & 15;
      if (row_base + 16 * i < R) *(bf16x8*)(wt + row * 256 + ((cc ^ swz(row & 7)) << 4)) = reg[i];
    }
    if (row_base + 2 * kWRows < R) fetch_w(part + 2, reg);
    __syncthreads();
    const int rows = min(kWRows, R - row_base);
    auto k_step = [&](int ks) {
      const bf16x8 a = *(const bf16x8*)(zt + c32 * zpitch + row_base + ks * 16 + g * 8);
      const short4v lo = lds_tr16(wt + ks * 16 * 256 + tr_off[0]);
      const short4v hi = lds_tr16(wt + ks * 16 * 256 + tr_off[1]);
      const bf16x8 bm = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bm, acc, 0, 0, 0);
    };
    if (rows == kWRows) {
      // straight-line, so that the LDS reads of later steps are issued ahead of the MFMAs of earlier ones
#pragma unroll
      for (int ks = 0; ks < kWRows / 16; ++ks) k_step(ks);
    } else {
      for (int ks = 0; ks < rows / 16; ++ks) k_step(ks);
    }
  };
  for (int part = 0; part * kWRows < R; part += 2) {
    part_step(part, wreg[0]);
    part_step(part + 1, wreg[1]);
  }
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int sl = (r >> 2) * 8 + g * 4 + (r & 3);
    if (sl < n_valid)
      store_f32(out, out_at(r), acc[r] * out_scale * (gate ? bf16_to_f32(gate_v[r]) : 1.f));   // gate: Appendix E
  }
}

}  // namespace

bool absorb_q_mfma_supported(int d_h, int d_cb, int dtype) {
  return dtype == MLRA_BF16 && d_h == kDh && d_cb % 32 == 0;
}

int launch_absorb_q_mfma(int batch, int h, int d_h, int n_blocks, int groups, int d_cb, const void* q_nope,
                         const void* w_uk, void* q_abs, hipStream_t stream, float fold, const void* q_rope,
                         void* q_rope_out, int d_r) {
  (void)d_h;
  int n_pass = (d_cb + 127) / 128;
  if ((long)n_blocks * n_pass > 65534) n_pass = 1;   // (a grid dimension)
  dim3 grid(h, n_blocks * n_pass + (q_rope_out ? 1 : 0), (batch + 63) / 64);
  absorb_q_mfma_kernel<<<grid, 256, 0, stream>>>((const bf16_t*)q_nope, (const bf16_t*)w_uk, (bf16_t*)q_abs, batch, h,
                                                 n_blocks, groups, d_cb, fold, (const bf16_t*)q_rope,
                                                 (bf16_t*)q_rope_out, d_r, n_pass);
  return check_launch();
}

// Dynamic LDS of the merge + up-projection kernel: the weight rows, the normalised z rows of 32 sequences and, when
// there is something to merge, the weights of every (sequence, block, chunk).
static size_t merge_upproj_lds_bytes(const DecodeArgs& a, bool direct) {
  const int bpg = a.n_blocks / a.groups, R = bpg * a.d_cb;
  return (size_t)kWRows * 256 + (size_t)32 * (R + 8) * 2 + (direct ? 0 : (size_t)32 * bpg * a.plan.n_splits * sizeof(float));
}
constexpr size_t kMergeLdsLimit = 160 * 1024;

// Up to 1024 latent channels and 128 (block, chunk) slots per sequence, and at most 98,176 bytes of both at 64 per z
// channel and 256 per slot; everything else takes the fp32 epilogue (and fp32 partials).  This is no limit of the kernel:
// with 128 bytes per slot and 32 KiB of weights it occupies up to 112 KiB of LDS here, and 256 slots at 512 channels (one
// sequence of 8K tokens and up, four blocks) would fit; whether it is the better epilogue there has not been measured.
bool merge_upproj_mfma_supported(const DecodeArgs& a) {
  const int bpg = a.n_blocks / a.groups;
  return a.dtype == MLRA_BF16 && a.d_h == kDh && a.d_cb % 32 == 0 && bpg * a.d_cb <= 1024 &&
         bpg * a.plan.n_splits <= 128 && 64L * (bpg * a.d_cb + 8) + 256L * bpg * a.plan.n_splits <= 98176;
}

template <typename TO, int MODE, int U, int KK>
static int launch_merge_as(const DecodeArgs& a, dim3 grid, int spw) {
  static PerDeviceSetup setup;
  int setup_dev = -1;
  if (setup.needed(&setup_dev)) {
    if (hipFuncSetAttribute((const void*)merge_upproj_mfma_kernel<TO, MODE, U, KK>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMergeLdsLimit) != hipSuccess)
      return MLRA_ERR_LAUNCH;
    setup.done(setup_dev);
  }
  const int q_group = a.fitted ? a.q_group : 1;
  const int32_t* const chunk_tab = a.balanced || a.fitted ? a.chunk_tab : nullptr;
  MLRA_LAUNCH_TIMED(a.t_epi, (merge_upproj_mfma_kernel<TO, MODE, U, KK>), grid, dim3(256),
                    merge_upproj_lds_bytes(a, MODE == kDirect), a.stream, (const float*)a.part_z,
                    (const float*)a.part_ml, a.seq_lens, (const bf16_t*)a.w_uv, (TO*)a.out, a.lse, a.batch, a.h,
                    a.n_blocks, a.d_cb, a.plan.n_splits, a.plan.chunk_tokens, chunk_tab, a.out_scale,
                    (const bf16_t*)a.gate, spw, q_group, 0xffffffffu / (unsigned)q_group + 1u);
  return check_launch();
}

template <typename TO>
static int launch_merge_typed(const DecodeArgs& a, dim3 grid, int spw) {
  // U items per thread and step: many chunks (small batches) go one item per thread with all loads on its chunks, few
  // chunks several items
  // (KK = 2: at most four slots.  Among them are the forms that leave a batch of nearly equal lengths uncut, of which one
  // or two are used)
  if (a.rows_bf16) {
    if (a.plan.n_splits == 1) return launch_merge_as<TO, kDirect, 8, 1>(a, grid, spw);
    if (a.plan.n_splits > 8) return launch_merge_as<TO, kRows, 1, 16>(a, grid, spw);
    if (a.plan.n_splits > 4) return launch_merge_as<TO, kRows, 2, 8>(a, grid, spw);
    return launch_merge_as<TO, kRows, 4, 2>(a, grid, spw);
  }
  if (a.plan.n_splits > 4) return launch_merge_as<TO, kItems, 1, 8>(a, grid, spw);
  return launch_merge_as<TO, kItems, 4, 2>(a, grid, spw);
}

int launch_merge_upproj_mfma(const DecodeArgs& a) {
  // small batches: fewer sequences per workgroup while that brings more workgroups onto idle CUs (not below 8: with 4 or
  // 2, 4 sequences of up to 128K took the same 17 us; two workgroups per CU instead of one cost 64 sequences 3 us)
  int spw = 32;
  while (spw > 8 && (long)a.h * a.groups * ((a.batch + spw - 1) / spw) < a.cus) spw /= 2;
  const dim3 grid(a.h, (a.batch + spw - 1) / spw, a.groups);
  return a.out_dtype == MLRA_BF16 ? launch_merge_typed<bf16_t>(a, grid, spw) : launch_merge_typed<float>(a, grid, spw);
}

}  // namespace mlra
