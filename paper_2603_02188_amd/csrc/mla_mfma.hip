// MFMA decode kernel for the MLA comparison: one 512-dim latent plus a 64-dim RoPE key per token
// (Section 2.1, Steps 1-3 with d_c = 512; bf16 caches).
//
// One workgroup (4 wavefronts) owns one (sequence, context chunk, 64 query heads) and walks the
// chunk in tiles of 32 tokens [C | K^RoPE] that stream HBM -> LDS with direct-to-LDS loads.  Most launches run on
// mla_pipe_kernel, described there; mla_mfma_kernel, two stages deep with two workgroups per CU or four stages deep with
// one, keeps the shapes named in mla_mfma_stages.  In the latter the two products split the work differently:
//   * scores and softmax by heads: wave w owns heads [16 w, 16 w + 16) and computes their complete scores
//     S^T = [C | K^R] [q~ | q^R]^T over all 576 channels with 16x16x32 MFMAs (tokens x heads), so the
//     softmax of a head is computed once, by one wave, with its running maximum and sum in that wave;
//   * values by channels: wave w accumulates Z_w^T += C_w^T P^T for channels [128 w, 128 w + 128) and all
//     64 heads (32x32x16 MFMAs; C_w^T from LDS transpose reads of the same tile), so the 64 x 512
//     accumulator is spread over the four waves (128 registers each).
// Between the two, the probabilities P^T (bf16, 4 KiB per tile) go through LDS in the layout of the second
// product's B operand, together with the factors by which a wave lowered the weight of its heads'
// history when their running maximum grew (refreshed lazily, so almost always none).  Two workgroup
// barriers per tile: one hands the landed tile and the freed stage around, one publishes P^T.
// A wave's chain through a tile (LDS latencies, softmax, the hand-overs) is 2.5 times the 1088 cycles of matrix pipe in
// it, so a second workgroup on the CU matters more than deeper buffering: the two-stage form takes 256 registers per wave,
// all of them (accumulators 128, queries 72, the rest operands in flight), and whatever can be recomputed is, because a
// spill inside the loop also waits for the tile loads (six registers are spilled in front of it and reloaded after it;
// the build fails if the loop holds a scratch access).  64 heads x 512 + 64 channels, two stages against four stages of
// the same width with one workgroup per CU: 256 sequences of 2176 tokens x 128 heads 222 -> 185 us, 128 sequences of 512 to 8192 in chunks 275 -> 221, 128
// sequences of 4352 (one workgroup per CU) 221 -> 212.  Measured and not kept: 16-token tiles in four stages
// (198 / 237 / 250 us), two groups of four waves one barrier apart in one workgroup (223 / 260 / 215), 32 heads x 16
// tokens per wave (216 / 264 / 214), the channels of the scores split over two waves (224 / 265 / 298).
// The two head halves of a sequence are placed on the same XCD (ids 8 apart), so the cache is fetched
// from HBM once.  Partials go to the workspace in the layout of the MLRA path with n_blocks = 1,
// d_cb = 512.
#include "chunk_fit.h"
#include "mfma_tile.h"

#include <type_traits>

namespace mlra {
namespace {

using namespace mfma_tile;

constexpr int kMDc = 512;                          // latent channels
constexpr int kMTok = 32;                          // tokens per tile
constexpr int kMHeads = 64;                        // query heads per workgroup
constexpr int kMLatBytes = kMTok * kMDc * 2;       // 32 KiB
constexpr int kMRopeBytes = kMTok * kDr * 2;       //  4 KiB
constexpr int kMStage = kMLatBytes + kMRopeBytes;  // 36 KiB
constexpr int kMPBytes = 4 * 1024;                 // P^T: [2 head tiles][2 token halves][64 lanes][16 B]
// LDS: the stages, P^T, the rescale factors ([64 heads] floats) and the four waves' flags
constexpr int mla_lds_bytes(int stages) { return stages * kMStage + kMPBytes + kMHeads * 4 + 4 * 4; }
static_assert(2 * mla_lds_bytes(2) <= 160 * 1024 && mla_lds_bytes(4) <= 160 * 1024, "two workgroups per CU / one");
constexpr int kMLoads = 9;                         // direct-to-LDS loads per wave and tile

// start-up and write-out of a workgroup in the time of 64 tokens (15 us, 2.3 us)
constexpr int kMFitOverhead = 6;

typedef const __attribute__((address_space(3))) bf16x8* lds_bf16x8_ptr;
typedef const __attribute__((address_space(3))) unsigned char* lds_byte_ptr;

// The four lanes c16, c16 + 16, c16 + 32, c16 + 48 hold parts of one head: these combine them in every
// lane without a trip through LDS.  v_permlane16_swap exchanges the odd 16-lane rows of its first operand
// with the even rows of its second, v_permlane32_swap the upper half of the first with the lower half of
// the second; applied to two copies of a value, every lane ends up with its own and its partner's.
__device__ __forceinline__ void row_pairs(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void half_pairs(float& a, float& b) {
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ float head_max(float v) {
  float a = v, b = v;
  row_pairs(a, b);
  a = fmaxf(a, b);
  b = a;
  half_pairs(a, b);
  return fmaxf(a, b);
}
__device__ __forceinline__ float head_sum(float v) {
  float a = v, b = v;
  row_pairs(a, b);
  a += b;
  b = a;
  half_pairs(a, b);
  return a + b;
}

typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

// false: an empty slot.  FIT: the kernel takes fitted launches as well.
template <bool FIT>
__device__ __forceinline__ bool mla_unit(const MfmaParams& p, int& hgrp, int& seq, int& split, int& chunk_len) {
  // workgroup -> (sequence, chunk, head half); the halves of one (sequence, chunk) get ids 8 apart
  const int n_hg = (p.h + kMHeads - 1) / kMHeads;
  int n_units = p.n_splits * p.batch, fit_len = 0;
  if (FIT && p.chunk_out) {    // one chunk length fitted to the lengths (chunk_fit.h), left for the merge
    const int i = threadIdx.x & 63;
    fit_len = i < p.batch ? max(0, min(p.seq_lens[i], p.max_pages * p.page_size)) : 0;
    chunk_len = chunk_fit::fit_length<false>(fit_len, p.batch, n_hg, p.cus, p.fit_min, kMFitOverhead);
    if (blockIdx.x == 0 && (int)threadIdx.x < p.batch) p.chunk_out[threadIdx.x] = chunk_len;
    n_units = chunk_fit::count(fit_len, chunk_len);
    if ((int)blockIdx.x >= n_units * n_hg) return false;
  }
  const int full_units = n_units & ~7;
  int wg = blockIdx.x, su;
  if (wg < full_units * n_hg) {
    const int r = wg >> 3;
    hgrp = r % n_hg;
    su = (r / n_hg) * 8 + (wg & 7);
  } else {
    wg -= full_units * n_hg;
    su = full_units + wg / n_hg;
    hgrp = wg % n_hg;
  }
  if (FIT && p.chunk_out) {
    const chunk_fit::Chunk c = chunk_fit::find(fit_len, p.batch, chunk_len, su);
    seq = c.seq;
    split = c.split;
  } else if (p.unit_tab) {     // chunk lengths follow the sequence lengths: active units listed first
    const int code = p.unit_tab[su];
    if (code < 0) return false;
    seq = code >> 10;
    split = code & 1023;
    chunk_len = p.chunk_tab[seq];
  } else {
    // longest sequences first, and with several slots per sequence all first chunks, then all second ones, ...: the
    // slots that shorter sequences leave empty come late and in runs.  (Sequence by sequence they lie between the others,
    // and CUs that were dealt empty ones stay idle while others get a second workgroup: 50 sequences of 1666 to 5000
    // tokens x 64 heads, whole step 98 us against 83.)
    const int slot = p.split_major ? su % p.batch : su / p.n_splits;
    split = p.split_major ? su / p.batch : su % p.n_splits;
    seq = p.seq_order ? p.seq_order[slot] : slot;
    chunk_len = p.chunk;
  }
  return true;
}

__device__ __forceinline__ f32x16 opaque_zero16() {
  float z = 0.f;
  asm volatile("" : "+v"(z));
  f32x16 v;
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = z;
  return v;
}

template <int STAGES>
__global__ __launch_bounds__(256, STAGES == 2 ? 2 : 1) void mla_mfma_kernel(MfmaParams p) {
  static_assert(STAGES == 2 || STAGES == 4, "a power of two, and the waits below");
  constexpr int kMPOff = STAGES * kMStage, kMAOff = kMPOff + kMPBytes, kMFOff = kMAOff + kMHeads * 4;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int hgrp, seq, split, chunk_len;
  if (!mla_unit<false>(p, hgrp, seq, split, chunk_len)) return;
  const int n = ((const_i32_ptr)p.seq_lens)[seq];
  const int t0 = split * chunk_len;
  if (t0 >= n) return;
  const int t1 = t0 + min(n - t0, chunk_len);
  const int ntiles = (t1 - t0 + kMTok - 1) / kMTok;
  const int nvalid_last = t1 - t0 - (ntiles - 1) * kMTok;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 5, c32 = lane & 31;         // 32x32 MFMA roles (values)
  const int q4 = lane >> 4, c16 = lane & 15;        // 16x16 MFMA roles (scores)
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const float sc = p.scale_log2;
  const int head_base = hgrp * kMHeads;

  // ---- this wave's 16 heads, complete: absorbed (512) and RoPE (64) query channels as B operands of the
  // 16x16x32 MFMA (lane: head c16, eight channels from 32 ks + 8 q4)
  bf16x8 qreg[18];
  {
    const int head = min(head_base + 16 * wave + c16, p.h - 1);
    const bf16_t* qa = p.q_abs + ((size_t)seq * p.h + head) * kMDc + q4 * 8;
    const bf16_t* qr = p.q_rope + ((size_t)seq * p.h + head) * kDr + q4 * 8;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) qreg[ks] = *(const bf16x8*)(qa + ks * 32);
    qreg[16] = *(const bf16x8*)qr;
    qreg[17] = *(const bf16x8*)(qr + 32);
  }
  // consumed here, before any direct-to-LDS load is in flight (a compiler-placed wait would drain them)
#pragma unroll
  for (int ks = 0; ks < 18; ++ks) asm volatile("" : "+v"(qreg[ks]));

  // ---- tile loads.  Latent rows are 1 KiB: one load moves one token row (lane i: 16-byte chunk i, i.e.
  // 256-byte sub-row i / 16, stored at chunk position (i % 16) ^ lat_swz(token) inside the sub-row);
  // wave w loads tokens 8w .. 8w+7 and RoPE rows 8w .. 8w+7 (one load).
  const const_i32_ptr pt_row = (const_i32_ptr)(p.page_table + (size_t)seq * p.max_pages);
  const size_t lat_page_bytes = (size_t)p.page_size * (kMDc * 2);
  const size_t rope_page_bytes = (size_t)p.page_size * (kDr * 2);
  // (the swizzle of a row is uniform, so the lane offset of load i is one exclusive or away from 16 lane)
  // Tiles are issued in order, nine loads each (0..7: latent rows, 8: the RoPE rows).  Pages hold whole tiles, and the id
  // of the page after the current one is always loaded already.
  int iss_tok = t0, iss_page_at = t0 / p.page_size, iss_slot = t0 % p.page_size, iss_stage = 0;
  unsigned iss_page = (unsigned)pt_row[iss_page_at];
  unsigned iss_page_next = (unsigned)pt_row[min(iss_page_at + 1, p.max_pages - 1)];
  const unsigned lane16 = lane * 16;
  auto issue_tile = [&]() {
    const char* const lat = (const char*)p.latent + iss_page * lat_page_bytes + (size_t)iss_slot * (kMDc * 2);
    const char* const rope = (const char*)p.rope + iss_page * rope_page_bytes + (size_t)iss_slot * (kDr * 2);
    const int last = min(kMTok, t1 - iss_tok) - 1;     // rows past it re-read it (finite values, weight 0 later)
    const unsigned dst = lds_base + iss_stage * kMStage;
#pragma unroll
    for (int i = 0; i < kMLoads; ++i) {
      unsigned l16 = lane16;
      asm volatile("" : "+v"(l16));    // (or the offsets of all nine loads would be kept in registers: there are none left)
      if (i < 8) {
        const int t = 8 * wave_u + i;
        set_m0(dst + t * 1024);
        lds_dma16<0>(lat + (size_t)min(t, last) * 1024, l16 ^ (unsigned)(lat_swz(t) << 4));
      } else {
        const int t = 8 * wave_u + (l16 >> 7);       // lane / 8 rows on
        set_m0(dst + kMLatBytes + wave_u * 1024);
        lds_dma16<0>(rope, (unsigned)min(t, last) * (kDr * 2) + ((l16 & 0x70) ^ (rope_swz(t) << 4)));
      }
    }
    iss_tok += kMTok;
    iss_slot += kMTok;
    iss_stage = (iss_stage + 1) & (STAGES - 1);
    if (iss_slot == p.page_size) {
      iss_slot = 0;
      ++iss_page_at;
      iss_page = iss_page_next;
      iss_page_next = (unsigned)pt_row[min(iss_page_at + 1, p.max_pages - 1)];
    }
  };

  // ---- per-lane LDS read offsets inside a stage (XOR swizzle, see mfma_tile.h and decode_mfma.hip).
  // Scores, A operand of the 16x16x32 MFMA: lane = operand row c16 (+ 16 th) and eight channels from
  // 32 ks + 8 q4, i.e. 16-byte chunk 4 ks + q4 of the token row: sub-row ks / 4, chunk 4 (ks % 4) + q4.
  // A 128-bit LDS read is served sixteen lanes a cycle, and the sixteen are lanes 0-3, 12-15, 20-27 (then
  // 4-11, 16-19, 28-31; the same in the upper half): rows 4..11 of one chunk column meet rows 0-3 and 12-15
  // of the neighbouring column.  With operand row r holding token r ^ 8 (r in 4..7 or 12..15), i.e. rows
  // 4..11 = tokens 8..15, the chunk positions c ^ lat_swz(t) of such a group are all different (measured:
  // 4.6 instead of 8 cycles per read).  Output rows 4 q4 .. + 3 are then tokens 4 q4t .. + 3.
  const int k_tok = c16 ^ ((c16 & 4) << 1);
  const int q4t = q4 ^ ((q4 & 1) << 1);
  // (the swizzles repeat every 16 tokens: token half th is th * 16 rows further on)
  const unsigned k_lat_off = k_tok * 1024 + ((q4 ^ lat_swz(k_tok)) << 4);                      // ^ ((ks % 4) << 6), + 256 (ks / 4)
  const unsigned k_rope_off = kMLatBytes + k_tok * (kDr * 2) + ((q4 ^ rope_swz(k_tok)) << 4);  // ^ (kr << 6)
  // Values: lane group's token ta = 8 half + 4 g + k of 16; half 1 is 8 rows on and flips bit 1 of the swizzle.
  unsigned v_off;                                                             // ^ (mt << 6), + 16 KiB ss
  {
    const int k = (lane & 15) >> 2, seg = lane & 3, hb = (lane >> 4) & 1, ta = 4 * g + k;
    v_off = ta * 1024 + wave * 256 + (((2 * hb + (seg >> 1)) ^ lat_swz(ta)) << 4) + ((seg & 1) << 3);
  }
  // P^T: the B operand (head tile w / 2, token half th) pairs with the transposed value operand, whose
  // lane group g holds tokens 4 g .. 4 g + 3 and 8 + 4 g .. 8 + 4 g + 3 of the 16.  This lane's four
  // probabilities (tokens 4 q4t .. + 3 of the half, head 16 w + c16) are therefore the first (q4t < 2) or
  // second four of lane n + 32 (q4t % 2), n = 16 (w % 2) + c16.
  const unsigned p_wr_off = (wave >> 1) * 2048 + (16 * (wave & 1) + c16 + 32 * (q4t & 1)) * 16 + (q4t >> 1) * 8;  // + 1024 th

  float m_run = kNegBig, l_run = 0.f;      // of head 16 w + c16 (the four lanes of a head hold equal m)
  f32x16 zacc[4][2];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt)
#pragma unroll
      for (int i = 0; i < 16; ++i) zacc[mt][nt][i] = 0.f;

  for (int jj = 0; jj < STAGES - 1 && jj < ntiles; ++jj) issue_tile();
  for (int j = 0; j < ntiles; ++j) {
    // tile j landed in this wave's share (the tiles issued after it may still be in flight) ...
    if (STAGES > 2 && j + 2 < ntiles) wait_vm_lgkm<2 * kMLoads>();
    else if (STAGES > 2 && j + 1 < ntiles) wait_vm_lgkm<kMLoads>();
    else wait_vm_lgkm<0>();
    // ... and in everybody's; every wave is also done with tile j-1, whose stage is refilled now
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (j + STAGES - 1 < ntiles) issue_tile();
    const unsigned base = lds_base + (j & (STAGES - 1)) * kMStage;

    // ---- scores of this wave's 16 heads: 36 MFMAs
    f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    {
      auto k_read = [&](int i) {     // i = 2 ks + th
        const int ks = i >> 1, th = i & 1;
        const unsigned addr = ks < 16 ? ((base + k_lat_off) ^ ((ks & 3) << 6)) + (ks >> 2) * 256 + th * 16 * 1024
                                      : ((base + k_rope_off) ^ ((ks - 16) << 6)) + th * 16 * (kDr * 2);
        return *(lds_bf16x8_ptr)(size_t)addr;
      };
      // (the order is pinned: left to itself, the scheduler reads one operand at a time and waits for it)
      constexpr int kAhead = STAGES == 2 ? 5 : 12;
      bf16x8 ka[36];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 36; ++i) ka[i] = k_read(i);
#pragma unroll
      for (int i = 0; i < 36; ++i) s[i & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[i], qreg[i >> 1], s[i & 1], 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
      for (int i = 0; i < 36 - kAhead; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, kAhead, 0);
      __builtin_amdgcn_sched_barrier(0);
    }

    // ---- softmax of the 16 heads (running maximum refreshed lazily, see decode_mfma.hip)
    float mx = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])),
                     fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    mx = head_max(mx);
    const float cand = mx * sc;
    const bool grow = cand > m_run + kLazy;
    const bool any_grow = __any(grow);
    float alpha = 1.f;
    if (any_grow) {
      const float m_new = grow ? cand : m_run;
      alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
      m_run = m_new;
    }
    const int valid = (j == ntiles - 1) ? nvalid_last : kMTok;
    const float neg_m = -m_run;
#pragma unroll
    for (int th = 0; th < 2; ++th) {
      float pe[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        pe[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[th][i], sc, neg_m));
        if (16 * th + 4 * q4t + i >= valid) pe[i] = 0.f;     // rows past a ragged end are copies of the last valid row
        l_run += pe[i];
      }
      typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
      const bf16x4 pk = {(__bf16)pe[0], (__bf16)pe[1], (__bf16)pe[2], (__bf16)pe[3]};
      *(bf16x4*)(smem + kMPOff + th * 1024 + p_wr_off) = pk;
    }
    if (q4 == 0) ((float*)(smem + kMAOff))[16 * wave + c16] = alpha;
    if (lane == 0) ((int*)(smem + kMFOff))[wave_u] = any_grow ? 1 : 0;

    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");     // P^T, the factors and the flags of every wave are visible

    // P^T and value operands of the first token half are on their way while the flags are looked at
    bf16x8 pb[2], va[4];
    auto read_half = [&](int ss) {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
        pb[nt] = *(const bf16x8*)(smem + kMPOff + (nt * 2 + ss) * 1024 + lane * 16);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const short4v lo = lds_tr16((lds_byte_ptr)(size_t)((base + v_off) ^ (mt << 6)) + ss * 16 * 1024);
        const short4v hi = lds_tr16((lds_byte_ptr)(size_t)((base + v_off) ^ (mt << 6) ^ 32) + (ss * 16 + 8) * 1024);
        va[mt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
    };
    const int4 fl = *(const int4*)(smem + kMFOff);
    read_half(0);
    __builtin_amdgcn_sched_barrier(0);
    // ---- a head's history loses weight when its maximum grew: the owner of the head said by how much
    {
      if (__builtin_amdgcn_readfirstlane(fl.x | fl.y | fl.z | fl.w)) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const float a_h = ((const float*)(smem + kMAOff))[nt * 32 + c32];
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int i = 0; i < 16; ++i) zacc[mt][nt][i] *= a_h;
        }
      }
    }
    // ---- values: Z_w^T += C_w^T P^T
#pragma unroll
    for (int ss = 0; ss < 2; ++ss) {
      if (ss == 1) read_half(1);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        zacc[mt][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[mt], pb[0], zacc[mt][0], 0, 0, 0);
        zacc[mt][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[mt], pb[1], zacc[mt][1], 0, 0, 0);
      }
    }
  }

  // ---- write the chunk's partial: every wave its 128 channels of all 64 heads, and (m, l) of its 16 heads
  l_run = head_sum(l_run);
  const size_t unit = (size_t)seq * p.n_splits + split;
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int head = head_base + nt * 32 + c32;
    if (head < p.h) {
      float* dst = p.part_z + (unit * p.h + head) * kMDc + wave * 128 + g * 4;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x4 v = {zacc[mt][nt][r4 * 4], zacc[mt][nt][r4 * 4 + 1], zacc[mt][nt][r4 * 4 + 2],
                           zacc[mt][nt][r4 * 4 + 3]};
          *(f32x4*)(dst + mt * 32 + r4 * 8) = v;
        }
    }
  }
  {
    const int head = head_base + 16 * wave + c16;
    if (q4 == 0 && head < p.h) {
      p.part_ml[(unit * p.h + head) * 2 + 0] = m_run;
      p.part_ml[(unit * p.h + head) * 2 + 1] = l_run;
    }
  }
}

// ------------------------------------------------------------------------------------------------
// The pipelined form: one workgroup of four waves per CU, four stages, and in each step the scores of one tile and the value
// product of the tile before it, so that a wave has matrix work while its softmax, its hand-overs and its LDS reads are on
// their way.  Against the form above:
//   * scores and softmax by 32 heads x 16 tokens per wave (two groups of 16 heads share an operand read, 18 reads a tile
//     instead of 36); the two waves of a head exchange their maxima over LDS and refresh the reference alike;
//   * P^T, maxima and factors in two copies, so that one barrier hands over maxima, tile and freed stage and a second
//     one P^T; neither has a wait behind it that matters;
//   * everything a lane keeps per head is held for both of its groups in one register, masks and row clamps are only in the
//     copy of the step that meets the chunk's last tile, factors are stored only when a maximum moved: 287 instructions a tile,
//     52 of them MFMAs (430 in a first version, 300 us against 238 of the whole step below).
// Bound by instruction issue of the one wave per SIMD: 2250 cycles a tile with 1088 of matrix pipe in them; without the tile
// loads, the score reads or the value reads it takes 5 to 10 % less each.  Per workgroup another 15 us of start-up and
// write-out.  HBM traffic is that of the cache once (0.68 GB on 128 sequences of 512 to 8192, two-stage form 1.01).
// Whole steps, against the better of the two older forms: 128 sequences of 512 to 8192 x 128 heads 247.4 -> 236.2 us, x 64
// heads 222 -> 190, 128 of 4352 x 128 heads 262 -> 222, 64 of 6000 186 -> 158, one of 4000 41.3 -> 38.2.
// Measured and not kept: eight waves, two per SIMD, with half of the scores and channels each (260 us on the first shape
// against 238), P^T read behind the first barrier and no second one (238), all loads of a tile behind the value product (243).
// ------------------------------------------------------------------------------------------------
template <int N>
__device__ __forceinline__ void wait_lgkm() { asm volatile("s_waitcnt lgkmcnt(%0)" : : "n"(N) : "memory"); }

// LDS of the pipelined kernel: the stages and, twice (tiles of even and odd number), P^T, the rescale factors, the tile
// maxima of the four waves and the number of the last tile in which a wave's maxima grew.
constexpr int kPStages = 4;
constexpr int kPPOff = kPStages * kMStage, kPAOff = kPPOff + 2 * kMPBytes, kPXOff = kPAOff + 2 * kMHeads * 4,
              kPFOff = kPXOff + 2 * 4 * 32 * 4, kPLds = kPFOff + 2 * 4 * 4;
static_assert(kPLds <= 160 * 1024, "one workgroup per CU");

__global__ __launch_bounds__(256, 1) void mla_pipe_kernel(MfmaParams p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int hgrp, seq, split, chunk_len;
  if (!mla_unit<true>(p, hgrp, seq, split, chunk_len)) return;
  const int n = ((const_i32_ptr)p.seq_lens)[seq];
  const int t0 = split * chunk_len;
  if (n <= 0 || (unsigned)t0 >= (unsigned)n) return;   // (unplanned slots reach beyond 2^31 in the widest caches)
  const int t1 = t0 + min(n - t0, chunk_len);
  const int ntiles = (t1 - t0 + kMTok - 1) / kMTok;
  const int nvalid_last = t1 - t0 - (ntiles - 1) * kMTok;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int g = lane >> 5, c32 = lane & 31;         // 32x32 MFMA roles (values)
  const int q4 = lane >> 4, c16 = lane & 15;        // 16x16 MFMA roles (scores)
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int hg = wave & 1, th = wave >> 1;          // scores: heads [32 hg, + 32), tokens [16 th, + 16) of the tile
  const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const float sc = p.scale_log2;
  const int head_base = hgrp * kMHeads;

  // ---- tile loads.  Latent rows are 1 KiB: one load moves one token row (lane i: 16-byte chunk i, i.e. 256-byte sub-row
  // i / 16, stored at chunk position (i % 16) ^ lat_swz(token) inside the sub-row); wave w loads tokens 8 w .. + 7 (parts
  // 0..7) and RoPE rows 8 w .. + 7 (part 8).  Tiles are issued in order, in parts that sit behind different MFMAs; the id of
  // the page after the current one is always loaded already (pages hold whole tiles).
  const const_i32_ptr pt_row = (const_i32_ptr)(p.page_table + (size_t)seq * p.max_pages);
  const size_t lat_page_bytes = (size_t)p.page_size * (kMDc * 2);
  const size_t rope_page_bytes = (size_t)p.page_size * (kDr * 2);
  int iss_tok = t0, iss_page_at = t0 / p.page_size, iss_slot = t0 % p.page_size;
  unsigned iss_page = (unsigned)pt_row[iss_page_at];
  unsigned iss_page_next = (unsigned)pt_row[min(iss_page_at + 1, p.max_pages - 1)];
  unsigned lat_voff[8], rope_voff;
#pragma unroll
  for (int i = 0; i < 8; ++i) lat_voff[i] = ((lane * 16) ^ (unsigned)(lat_swz(8 * wave + i) << 4)) + (i & 4) * 1024;
  rope_voff = (8 * wave + (lane >> 3)) * (kDr * 2) + (((lane * 16) & 0x70) ^ (rope_swz(8 * wave + (lane >> 3)) << 4));
  const char* iss_lat = nullptr;
  const char* iss_rope = nullptr;
  unsigned iss_dst = lds_base;
  auto issue_begin = [&]() {
    iss_lat = (const char*)p.latent + iss_page * lat_page_bytes + (size_t)(iss_slot + 8 * wave_u) * (kMDc * 2);   // (pages of 4 GiB)
    iss_rope = (const char*)p.rope + iss_page * rope_page_bytes + (size_t)iss_slot * (kDr * 2);
  };
  auto issue_part = [&](int i) {       // of a full tile (the instruction offset moves both sides)
    if (i == 0 || i == 4) set_m0(iss_dst + wave_u * 8192 + i * 1024);
    if (i == 8) set_m0(iss_dst + kMLatBytes + wave_u * 1024);
    if (i == 8) lds_dma16<0>(iss_rope, rope_voff);
    else if ((i & 3) == 0) lds_dma16<0>(iss_lat, lat_voff[i]);
    else if ((i & 3) == 1) lds_dma16<1024>(iss_lat, lat_voff[i]);
    else if ((i & 3) == 2) lds_dma16<2048>(iss_lat, lat_voff[i]);
    else lds_dma16<3072>(iss_lat, lat_voff[i]);
  };
  auto issue_part_any = [&](int i) {   // rows past the chunk's end re-read its last one (finite values, weight 0 later)
    const int last = min(kMTok, t1 - iss_tok) - 1;
    if (i < 8) {
      const int t = 8 * wave_u + i;
      set_m0(iss_dst + t * 1024);
      lds_dma16<0>(iss_lat + (long)(min(t, last) - 8 * wave_u) * 1024, lat_voff[i] - (i & 4) * 1024);
    } else {
      const int t = 8 * wave + (lane >> 3);
      set_m0(iss_dst + kMLatBytes + wave_u * 1024);
      lds_dma16<0>(iss_rope, rope_voff - (unsigned)(t - min(t, last)) * (kDr * 2));
    }
  };
  auto issue_end = [&]() {
    iss_tok += kMTok;
    iss_slot += kMTok;
    iss_dst = iss_dst == lds_base + (kPStages - 1) * kMStage ? lds_base : iss_dst + kMStage;
    if (iss_slot == p.page_size) {
      iss_slot = 0;
      ++iss_page_at;
      iss_page = iss_page_next;
      iss_page_next = (unsigned)pt_row[min(iss_page_at + 1, p.max_pages - 1)];
    }
  };

  // ---- query operands of this wave's 32 heads, two groups of 16
  bf16x8 qreg[2][18];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int head = min(head_base + 32 * hg + 16 * i + c16, p.h - 1);
    const bf16_t* qa = p.q_abs + ((size_t)seq * p.h + head) * kMDc + q4 * 8;
    const bf16_t* qr = p.q_rope + ((size_t)seq * p.h + head) * kDr + q4 * 8;
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) qreg[i][ks] = *(const bf16x8*)(qa + ks * 32);
    qreg[i][16] = *(const bf16x8*)qr;
    qreg[i][17] = *(const bf16x8*)(qr + 32);
  }
  auto issue_whole = [&]() {
    issue_begin();
#pragma unroll
    for (int i = 0; i < kMLoads; ++i) issue_part_any(i);
    issue_end();
  };
  // the first tile is requested behind the queries and waited for with them; they go into the accumulation file
  issue_whole();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int ks = 0; ks < 18; ++ks) asm volatile("" : "+a"(qreg[i][ks]));
  __builtin_amdgcn_sched_barrier(0);
  const int n_pro = min(ntiles, kPStages);
  for (int jj = 1; jj < n_pro; ++jj) issue_whole();
  if (tid < 8) ((int*)(smem + kPFOff))[tid] = -1;

  // ---- per-lane LDS read offsets inside a stage (see mla_mfma_kernel; this wave's 16 tokens only)
  const int k_tok = c16 ^ ((c16 & 4) << 1);
  const int q4t = q4 ^ ((q4 & 1) << 1);
  const unsigned k_lat_off = (16 * th + k_tok) * 1024 + ((q4 ^ lat_swz(k_tok)) << 4);                     // ^ ((ks % 4) << 6), + 256 (ks / 4)
  const unsigned k_rope_off = kMLatBytes + (16 * th + k_tok) * (kDr * 2) + ((q4 ^ rope_swz(k_tok)) << 4); // ^ (kr << 6)
  unsigned v_off;                                                             // ^ (mt << 6), + 16 KiB ss
  {
    const int k = (lane & 15) >> 2, seg = lane & 3, hb = (lane >> 4) & 1, ta = 4 * g + k;
    v_off = ta * 1024 + wave * 256 + (((2 * hb + (seg >> 1)) ^ lat_swz(ta)) << 4) + ((seg & 1) << 3);
  }
  // this lane's four probabilities of head group i go to + 256 i
  const unsigned p_wr_off = hg * 2048 + th * 1024 + (c16 + 32 * (q4t & 1)) * 16 + (q4t >> 1) * 8;

  // Per-head values (16 lanes a group) are kept for both groups in one register: lanes with even q4 hold group 0, odd q4
  // group 1.  both() spreads such a register.
  float m_run = kNegBig, mx = 0.f;
  float neg_m[2] = {-kNegBig, -kNegBig}, l_run[2] = {0.f, 0.f};
  auto both = [&](float x, float& g0, float& g1) {
    g0 = g1 = x;
    row_pairs(g0, g1);
  };
  f32x16 zacc[4][2];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) zacc[mt][nt] = opaque_zero16();

  constexpr int kAhead = 10;           // score operands read in the step before
  bf16x8 ka[18];
  short4v vlo[2][4], vhi[2][4];
  f32x4 s[2];
  auto k_read = [&](unsigned base, int ks) {
    const unsigned addr = ks < 16 ? ((base + k_lat_off) ^ ((ks & 3) << 6)) + (ks >> 2) * 256
                                  : ((base + k_rope_off) ^ ((ks - 16) << 6));
    ka[ks] = *(lds_bf16x8_ptr)(size_t)addr;
  };
  auto v_read = [&](unsigned base, int i) {     // i = 8 ss + 2 mt + half
    const int ss = i >> 3, mt = (i >> 1) & 3;
    if ((i & 1) == 0) vlo[ss][mt] = lds_tr16((lds_byte_ptr)(size_t)((base + v_off) ^ (mt << 6)) + ss * 16 * 1024);
    else vhi[ss][mt] = lds_tr16((lds_byte_ptr)(size_t)((base + v_off) ^ (mt << 6) ^ 32) + (ss * 16 + 8) * 1024);
  };
  bf16x8 pb[2][2];
  auto p_read = [&](int par, int i) {           // i = 2 nt + ss
    pb[i & 1][i >> 1] = *(const bf16x8*)(smem + kPPOff + par * kMPBytes + i * 1024 + lane * 16);
  };
  // scores of a tile (its first operands already read), with the operands of the value product of the tile before it and, ISSUE, the
  // second half of the loads of the tile after next
  auto scores = [&](unsigned kb, unsigned vb, int par, auto with_v, auto issue, bool rest) {
    constexpr bool ISSUE = decltype(issue)::value;
    s[0] = s[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < 18; ++m) {
      s[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[m], qreg[0][m], s[0], 0, 0, 0);
      s[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[m], qreg[1][m], s[1], 0, 0, 0);
      if (m + kAhead < 18) k_read(kb, m + kAhead);
      if (decltype(with_v)::value && m < 16) v_read(vb, m);
      if (decltype(with_v)::value && m >= 10 && m < 14) p_read(par, m - 10);
      if (m % 3 == 1 && m < 15) {
        if (ISSUE) issue_part(4 + m / 3);
        else if (rest) issue_part_any(4 + m / 3);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (ISSUE || rest) issue_end();
  };
  // the tile's maxima over this wave's 16 tokens, for the wave with the other 16 as well
  auto publish_max = [&](int par) {
    float a = fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3]));
    float b = fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3]));
    row_pairs(a, b);
    a = fmaxf(a, b);
    b = a;
    half_pairs(a, b);
    mx = fmaxf(a, b);
    ((float*)(smem + kPXOff))[(par * 4 + wave) * 32 + c32] = mx;
  };
  // The reference maxima (refreshed lazily, see decode_mfma.hip) from both halves' maxima; when one moves, its factor is
  // left for the waves that hold the head's history (both halves store the same).
  auto refresh = [&](float partner, int par, int tile) {
    const float cand = fmaxf(mx, partner) * sc;
    const bool grow = cand > m_run + kLazy;
    if (__builtin_expect(__any(grow), 0)) {
      const float m_new = grow ? cand : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      float a0, a1;
      both(alpha, a0, a1);
      l_run[0] *= a0;
      l_run[1] *= a1;
      both(-m_new, neg_m[0], neg_m[1]);
      ((float*)(smem + kPAOff))[par * kMHeads + 32 * hg + c32] = alpha;
      ((int*)(smem + kPFOff))[par * 4 + wave] = tile;
    }
  };
  float pe[2][4];
  auto soften = [&](int e, int valid) {        // valid: tokens of the tile (kMTok: no mask)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      pe[i][e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i][e], sc, neg_m[i]));
      if (valid < kMTok && 16 * th + 4 * q4t + e >= valid) pe[i][e] = 0.f;    // rows past a ragged end are copies of its last one
      l_run[i] += pe[i][e];
    }
  };
  auto store_p = [&](int par) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const bf16x4 pk = {(__bf16)pe[i][0], (__bf16)pe[i][1], (__bf16)pe[i][2], (__bf16)pe[i][3]};
      *(bf16x4*)(smem + kPPOff + par * kMPBytes + i * 256 + p_wr_off) = pk;
    }
  };
  auto rescale = [&](int2 grown, int par, int tile) {      // a head's history loses weight when its maximum grew
    const int g0 = __builtin_amdgcn_readfirstlane(grown.x), g1 = __builtin_amdgcn_readfirstlane(grown.y);
    if (__builtin_expect(g0 == tile || g1 == tile, 0)) {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        const float a_h = (nt == 0 ? g0 : g1) == tile ? ((const float*)(smem + kPAOff))[par * kMHeads + nt * 32 + c32] : 1.f;
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int i = 0; i < 16; ++i) zacc[mt][nt][i] *= a_h;
      }
    }
  };
  auto pv = [&](int m) {             // m = 4 ss + mt
    const int ss = m >> 2, mt = m & 3;
    const bf16x8 va = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vlo[ss][mt], vhi[ss][mt], 0, 1, 2, 3, 4, 5, 6, 7));
    zacc[mt][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[ss][0], zacc[mt][0], 0, 0, 0);
    zacc[mt][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[ss][1], zacc[mt][1], 0, 0, 0);
  };
  auto hand_over = [&]() {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto partner_max = [&](int par) { return ((const float*)(smem + kPXOff))[(par * 4 + (wave ^ 2)) * 32 + c32]; };
  auto grown_at = [&](int par) { return *(const int2*)(smem + kPFOff + par * 16); };   // waves 0, 1: heads 0..31, 32..63
  auto after = [&](unsigned st) { return st == lds_base + (kPStages - 1) * kMStage ? lds_base : st + kMStage; };

  // ---- prologue: scores and probabilities of tile 0
  if (ntiles > 3) wait_vm_lgkm<3 * kMLoads>();
  else if (ntiles > 2) wait_vm_lgkm<2 * kMLoads>();
  else if (ntiles > 1) wait_vm_lgkm<kMLoads>();
  else wait_vm_lgkm<0>();
  hand_over();
#pragma unroll
  for (int i = 0; i < kAhead; ++i) k_read(lds_base, i);
  scores(lds_base, 0u, 0, std::false_type{}, std::false_type{}, false);
  publish_max(0);
  if (ntiles > 3) wait_vm_lgkm<2 * kMLoads>();
  else if (ntiles > 2) wait_vm_lgkm<kMLoads>();
  else wait_vm_lgkm<0>();
  hand_over();                       // the maxima are visible, tile 1 has landed
  refresh(partner_max(0), 0, 0);
#pragma unroll
  for (int e = 0; e < 4; ++e) soften(e, ntiles == 1 ? nvalid_last : kMTok);
  store_p(0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < kAhead; ++i) k_read(lds_base + kMStage, i);   // (one tile: whatever the stage holds, unused)

  // ---- step j: scores of tile j + 1 while the operands of tile j's value product are read; one barrier; the value product
  // of tile j, with the softmax of tile j + 1 and the first operands of tile j + 2 between its MFMAs; one barrier, behind
  // which P^T of tile j + 1 is there.  The loads of tile j + 4 are spread over the second half of the step and the first
  // half of the next.
  bool rest = false;                 // the second half of a tile's loads is due
  unsigned st_cur = lds_base;
  __builtin_amdgcn_sched_barrier(0);
  wait_lgkm<kAhead>();
  hand_over();                       // P^T of tile 0
  auto step = [&](auto issue, int j) {
    constexpr bool ISSUE = decltype(issue)::value;         // tiles j + 3 and j + 4 exist and are no last ones
    const int par = j & 1, next = par ^ 1;
    const unsigned st_next = after(st_cur), st_then = after(st_next);
    __builtin_amdgcn_sched_barrier(0);
    const int2 grown = grown_at(par);
    scores(st_next, st_cur, par, std::true_type{}, issue, rest);
    publish_max(next);
    // tile j + 2 has landed in this wave's share, its reads of tile j are done, the maxima are stored
    if (ISSUE || j + 3 < ntiles) wait_vm_lgkm<kMLoads>();
    else wait_vm_lgkm<0>();
    hand_over();
    const float partner = partner_max(next);
    rest = ISSUE || j + 4 < ntiles;
    const int valid = !ISSUE && j + 2 == ntiles ? nvalid_last : kMTok;
    rescale(grown, par, j);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      pv(m);
      if (m == 0 && (ISSUE || rest)) issue_begin();
      if (m == 1) refresh(partner, next, j + 1);
      if (m >= 2 && m < 6) soften(m - 2, valid);
      if (m == 5) store_p(next);
      if ((m & 1) == 1) {
        if (ISSUE) issue_part(m >> 1);
        else if (rest) issue_part_any(m >> 1);
      }
      if (m >= 3) {
        k_read(st_then, 2 * (m - 3));
        k_read(st_then, 2 * (m - 3) + 1);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    wait_lgkm<4>();                  // (all but the last two pieces' reads: P^T is stored)
    hand_over();
    st_cur = st_next;
  };
  {
    int j = 0;
    if (ntiles > 1) step(std::false_type{}, j++);
    for (; j + 5 < ntiles; ++j) step(std::true_type{}, j);
    for (; j + 1 < ntiles; ++j) step(std::false_type{}, j);
  }
  {
    const int j = ntiles - 1, par = j & 1;
    const int2 grown = grown_at(par);
#pragma unroll
    for (int i = 0; i < 16; ++i) v_read(st_cur, i);
#pragma unroll
    for (int i = 0; i < 4; ++i) p_read(par, i);
    rescale(grown, par, j);
#pragma unroll
    for (int m = 0; m < 8; ++m) pv(m);
    hand_over();                     // (every wave is past the last maxima: their space is used below)
  }

  // ---- write the chunk's partial: every wave its 128 channels of all 64 heads, and (m, l) of the heads, whose sums over
  // the two token halves meet in LDS
  const size_t unit = (size_t)seq * p.n_splits + split;
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int head = head_base + nt * 32 + c32;
    if (head < p.h) {
      float* dst = p.part_z + (unit * p.h + head) * kMDc + wave * 128 + g * 4;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          const f32x4 v = {zacc[mt][nt][r4 * 4], zacc[mt][nt][r4 * 4 + 1], zacc[mt][nt][r4 * 4 + 2],
                           zacc[mt][nt][r4 * 4 + 3]};
          *(f32x4*)(dst + mt * 32 + r4 * 8) = v;
        }
    }
  }
  float* const lbuf = (float*)(smem + kPXOff);       // (free since the barrier above)
#pragma unroll
  for (int i = 0; i < 2; ++i) l_run[i] = head_sum(l_run[i]);
  if (th == 1 && lane < 32) lbuf[hg * 32 + lane] = lane < 16 ? l_run[0] : l_run[1];
  __syncthreads();
  if (th == 0 && lane < 32) {
    const int head = head_base + 32 * hg + lane;
    if (head < p.h) {
      p.part_ml[(unit * p.h + head) * 2 + 0] = m_run;
      p.part_ml[(unit * p.h + head) * 2 + 1] = (lane < 16 ? l_run[0] : l_run[1]) + lbuf[hg * 32 + lane];
    }
  }
}

}  // namespace

bool mla_mfma_supported(const DecodeArgs& a) {
  return a.dtype == MLRA_BF16 && a.n_blocks == 1 && a.d_cb == kMDc && a.d_r == kDr && a.page_size % kMTok == 0 &&
         a.plan.chunk_tokens % kMTok == 0;
}

template <int STAGES>
static int launch_mla_as(const DecodeArgs& a, const MfmaParams& p, unsigned n_wg) {
  static PerDeviceSetup setup;
  int setup_dev = -1;
  if (setup.needed(&setup_dev)) {
    if (hipFuncSetAttribute((const void*)mla_mfma_kernel<STAGES>, hipFuncAttributeMaxDynamicSharedMemorySize,
                            mla_lds_bytes(STAGES)) != hipSuccess)
      return MLRA_ERR_LAUNCH;
    setup.done(setup_dev);
  }
  MLRA_LAUNCH_TIMED(a.t_main, mla_mfma_kernel<STAGES>, dim3(n_wg), dim3(256), mla_lds_bytes(STAGES), a.stream, p);
  return check_launch();
}

// The pipelined kernel has one workgroup per CU, 15 us of start-up and write-out each and 1.15 us per tile; the two-stage
// kernel overlaps the start-up of one workgroup with another's tiles, 1.5 us each.  So the latter keeps launches of more
// workgroups than CUs in short chunks, where these are not fitted (whole steps, two-stage against pipelined: 100 sequences of
// 300 to 900 x 128 heads in chunks of 512 87 against 91 us, 140 of 2000 x 64 heads in chunks of 1024 130 against 143; with
// long ones 256 of 2176 x 128 heads 265 against 257).  Planned chunks of one head group go to the four-stage kernel where the
// batch is no more than a round, which is as many sequences as CUs (smaller batches are cut without a plan): left uncut, equal
// lengths of 2000 to 3000 tokens take 1 to 2 % less in it (256 of 2176 x 64 heads, whole call, four-stage against pipelined 159
// against 162 us, of 2000 x 16 heads 129 against 130).  Elsewhere it is behind: 256 of 8000 x 64 heads 458 against 447, of 512 to
// 4096 190 against 187, of 300 with 16 of 8192 among them 128 against 109.
int mla_mfma_stages(const DecodeArgs& a) {
  const int n_hg = (a.h + kMHeads - 1) / kMHeads;
  if (a.balanced && n_hg == 1 && a.batch <= a.cus) return 4;
  return !a.balanced && !a.fitted && (long)a.plan.n_splits * n_hg * a.batch > a.cus && a.plan.chunk_tokens < 1280 ? 2 : 0;
}

int launch_mla_mfma(const DecodeArgs& a) {
  MfmaParams p;
  p.latent = (const bf16_t*)a.latent;
  p.rope = (const bf16_t*)a.rope;
  p.page_table = a.page_table;
  p.seq_lens = a.seq_lens;
  p.seq_order = nullptr;   // set below when the launch needs more than one round of workgroups
  p.chunk_tab = a.balanced ? a.chunk_tab : nullptr;
  p.unit_tab = a.balanced ? a.unit_tab : nullptr;
  p.q_abs = (const bf16_t*)a.q_abs;
  p.q_rope = (const bf16_t*)a.q_rope;
  p.part_z = a.part_z;
  p.part_ml = a.part_ml;
  p.page_size = a.page_size;
  p.max_pages = a.max_pages;
  p.n_blocks = 1;
  p.h = a.h;
  p.groups = a.groups;
  p.n_splits = a.plan.n_splits;
  p.chunk = a.plan.chunk_tokens;
  p.batch = a.batch;
  p.scale_log2 = softmax_scale_log2(a.softmax_scale);
  p.rows_bf16 = 0;
  if (a.fitted) {
    p.fit_min = a.fit_tiles;
    p.cus = a.cus;
    p.chunk_out = a.chunk_tab;
  }
  const int n_hg = (a.h + kMHeads - 1) / kMHeads;
  const long long n_wg = (long long)a.plan.n_splits * n_hg * a.batch;
  if (n_wg <= 0 || n_wg > 0x7fffffffLL) return MLRA_ERR_SHAPE;
  if (!a.balanced && !a.fitted && (n_wg > a.cus || a.q_group > 1) && launch_seq_order(a) == MLRA_OK) p.seq_order = a.seq_order;
  // (the query tokens of one sequence are kept side by side in the order)
  p.split_major = p.seq_order && a.q_group <= 1;
  const int stages = mla_mfma_stages(a);
  if (stages == 4) return launch_mla_as<4>(a, p, (unsigned)n_wg);
  if (stages == 2) return launch_mla_as<2>(a, p, (unsigned)n_wg);
  static PerDeviceSetup setup;
  int setup_dev = -1;
  if (setup.needed(&setup_dev)) {
    if (hipFuncSetAttribute((const void*)mla_pipe_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kPLds) != hipSuccess)
      return MLRA_ERR_LAUNCH;
    setup.done(setup_dev);
  }
  MLRA_LAUNCH_TIMED(a.t_main, mla_pipe_kernel, dim3((unsigned)n_wg), dim3(256), kPLds, a.stream, p);
  return check_launch();
}


// Fitted chunk lengths where the slots are more than a round of workgroups: whole steps of 30 sequences of 2500 tokens x 128
// heads 92.7 -> 72.7 us (300 slots for 256 CUs; 87.2 in the two-stage kernel), 59 of 2836 x 64 heads 103.0 -> 82.9 (99.4).
bool mla_mfma_fits_chunks(const DecodeArgs& a) {
  const long slots = (long)a.plan.n_splits * a.batch * ((a.h + kMHeads - 1) / kMHeads);
  return a.batch > 1 && a.batch <= chunk_fit::kMaxSeqs && a.q_group == 1 && a.plan.n_splits > 1 && a.plan.target_chunks == 0 &&
         slots > a.cus;
}
}  // namespace mlra
