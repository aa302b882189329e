// Decode kernel for every shape outside the bf16 fast paths' dimensions (fp32 caches; bf16 caches of other
// head, latent or RoPE sizes or other page sizes), on the fp32 matrix instructions.
// Everything is computed in fp32, bf16 is only a storage type here: v_mfma_f32_16x16x4_f32 multiplies and
// accumulates in fp32, at 64 flop per cycle and SIMD.
//
// One workgroup (4 wavefronts) owns one (context chunk, block, 16 HT heads) and walks the chunk in tiles of TT tokens
// [C_b | K^RoPE], staged as fp32 in LDS (key and value at once).  The four waves are HT head tiles of 16 heads x
// TG = 4 / HT token groups; a wave scores its heads against its share of the tile's tokens, keeps its own running
// maximum, sum and Z, and the token groups are merged through LDS at the end.
//   * scores transposed, S^T = K Q^T (16 tokens x 16 heads): in the result, lane l holds head l % 16 and tokens
//     4 (l / 16) + i in register i.  That is the B operand of Z^T += V^T P^T if step i of that product takes tokens
//     4 q + i (q = lane / 16 is the MFMA's k index), so the probabilities never leave their registers.
//   * k indices are dealt so that every LDS read is 128 bits wide: step j of k group i takes k = 16 i + 4 q + j (a
//     lane reads four consecutive channels of a token row for four score MFMAs), and channel tile ct of a 64-channel
//     group takes channels 4 r + ct (a lane reads four consecutive channels of a token row for four value MFMAs).
//   * rows are 16 KG + 4 floats apart: 4 modulo 16, which spreads both kinds of reads over the banks.
//   * the next tile is in flight in registers while a tile is worked on; the addresses of its rows come from a
//     table in LDS that is computed one more tile ahead (one page lookup per token, not one per lane).
// Bound by the matrix pipe: a tile of 64 tokens x 192 channels x 64 heads is 10240 cycles of MFMA per SIMD against
// 2500 of LDS reads and 48 KiB of loads.  fp32, 4 blocks x 128 channels, 128 heads: 100 TFLOP/s on 8 sequences of 8192
// tokens (of 157 nominal), 58 us on 8 of 300 to 2048 (the VALU kernel it replaces: 1710 us), of which about 12 us are
// start-up, write-out and the launch; with chunks fitted to the lengths (chunk_fit.h) 46 us.
#include "chunk_fit.h"
#include "f32_tile.h"

namespace mlra {
namespace {

using namespace f32_tile;

struct F32Params {
  const void* latent;
  const void* rope;
  const int32_t* page_table;
  const int32_t* seq_lens;
  const void* q_abs;
  const void* q_rope;
  float* part_z;
  float* part_ml;
  int32_t* chunk_tab;   // non-null: the chunk length is fitted to the lengths (chunk_fit.h) and left here for the merge
  int page_size, max_pages, n_blocks, groups, d_cb, d_r, h, n_splits, chunk, n_hg, batch, fit_min, cus;
  float scale_log2;
};

template <int KG, int NCT, int TT>
constexpr size_t f32_lds_bytes() {
  // (a tile narrower than its 64-channel value groups is read past its rows' ends: into the next rows, and after the last
  // one into the merge buffer's space; those channels are not stored)
  const size_t tile = (size_t)TT * (16 * KG + 4) * 4, merge = (size_t)64 * (64 * NCT + 4) * 4;
  return (tile > merge ? tile : merge) + 4 * TT * sizeof(long long) + 2 * 64 * sizeof(float);
}

template <typename T, bool VEC, int KG, int NCT, int TT, int HT>
__global__ __launch_bounds__(256) void decode_f32_kernel(F32Params p) {
  typedef typename RawOf<T>::type Raw;
  constexpr int TG = 4 / HT, NTT = TT / 16 / TG;             // token groups; 16-token tiles per wave
  static_assert(NTT >= 1, "every wave needs a token tile");
  constexpr int P = 16 * KG + 4, ZP = 64 * NCT + 4;          // floats per tile row / merge row
  constexpr int V4 = 4 * KG;                                 // four-element pieces per tile row
  constexpr int LPR = V4 <= 8 ? 8 : V4 <= 32 ? 32 : 64, RPI = 64 / LPR;   // lanes per row, rows per load instruction
  constexpr int CI = (V4 + LPR - 1) / LPR, NR = TT / (4 * RPI);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  float* const tile = (float*)smem;
  constexpr size_t kMain = f32_lds_bytes<KG, NCT, TT>() - 4 * TT * sizeof(long long) - 2 * 64 * sizeof(float);
  long long* const row_off = (long long*)(smem + kMain);     // [2 tiles][latent, rope][TT] element offsets of the rows
  float* const mbuf = (float*)(row_off + 4 * TT);            // [4 waves][16 heads]
  float* const lbuf = mbuf + 64;

  // workgroup -> (chunk, sequence, block, head group).  Ids go round-robin over the eight XCDs: the head groups of
  // one (chunk, sequence, block) read the same rows and get ids 8 apart (one XCD, one L2), and the chunk is the
  // slowest index, so that the chunk slots that a ragged batch leaves empty are spread over the XCDs evenly.
  // (A grid that one dimension does not hold is cut into rows of a multiple of eight; the last one is padded.)
  int wg = blockIdx.y * gridDim.x + blockIdx.x, units = p.n_splits * p.batch * p.n_blocks, chunk = p.chunk, len = 0;
  if (__builtin_expect(p.chunk_tab != nullptr, 0)) {
    const int lane = threadIdx.x & 63;
    len = lane < p.batch ? max(0, min(p.seq_lens[lane], p.max_pages * p.page_size)) : 0;
    chunk = chunk_fit::fit_length<true>(len, p.batch, p.n_blocks * p.n_hg, p.cus, p.fit_min, 1);
    if (wg == 0 && (int)threadIdx.x < p.batch) p.chunk_tab[threadIdx.x] = chunk;
    units = chunk_fit::count(len, chunk) * p.n_blocks;
  }
  if (wg >= units * p.n_hg) return;
  const int full = units & ~7;
  int u, hg;
  if (wg < full * p.n_hg) {
    const int r = wg >> 3;
    hg = r % p.n_hg;
    u = (r / p.n_hg) * 8 + (wg & 7);
  } else {
    wg -= full * p.n_hg;
    u = full + wg / p.n_hg;
    hg = wg % p.n_hg;
  }
  const int b = u % p.n_blocks;
  int s = u / p.n_blocks % p.batch, split = u / p.n_blocks / p.batch;
  if (__builtin_expect(p.chunk_tab != nullptr, 0)) {
    const chunk_fit::Chunk c = chunk_fit::find(len, p.batch, chunk, u / p.n_blocks);
    s = c.seq;
    split = c.split;
  }
  const int n = p.seq_lens[s];
  const int t0 = split * chunk;
  if (n <= 0 || (unsigned)t0 >= (unsigned)n) return;   // (slots beyond the capacity)
  const int t1 = t0 + min(n - t0, chunk);
  const int ntiles = (t1 - t0 + TT - 1) / TT;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane >> 4, r16 = lane & 15;
  const int ht = wave / TG, tg = wave % TG;
  const int d_cb = p.d_cb, D = p.d_cb + p.d_r;
  const T* const latent = (const T*)p.latent;
  const T* const rope = (const T*)p.rope;

  // Where the rows of a tile lie: thread i < TT looks token i's page up (page_of) one tile before it writes the two
  // offsets to LDS (row_table), so that no lookup waits behind a tile's loads.  Slots past the chunk repeat its last
  // row: finite wherever the chunk is, and their weight is 0.
  auto page_of = [&](int j) {
    const int tok = min(t0 + j * TT + tid % TT, t1 - 1);
    return p.page_table[(size_t)s * p.max_pages + tok / p.page_size];
  };
  auto row_table = [&](int j, int page_id) {
    if (tid < TT) {
      const long long page = page_id;
      const int slot = min(t0 + j * TT + tid, t1 - 1) % p.page_size;
      row_off[(j & 1) * 2 * TT + tid] = ((page * p.n_blocks + b) * p.page_size + slot) * d_cb;
      row_off[(j & 1) * 2 * TT + TT + tid] = (page * p.page_size + slot) * p.d_r - d_cb;
    }
  };
  // Loads: lane = (row of the instruction, four-element piece of [latent | rope]).  No load is conditional (a piece
  // past the row's end reads element 0 and is replaced by zero), so that a whole tile's are in flight together.
  Raw pre[NR][CI];
  const int ld_row = lane / LPR, ld_k4 = lane % LPR;
  auto fetch = [&](int j) {            // tile j into registers
#pragma unroll
    for (int c = 0; c < CI; ++c) {
      const int k = 4 * (ld_k4 + c * LPR);
      if constexpr (VEC) {
        const bool in_rope = k >= d_cb && k < D;
        const long long* off = row_off + (j & 1) * 2 * TT + (in_rope ? TT : 0) + wave * NR * RPI + ld_row;
        const T* base = (in_rope ? rope : latent) + (k < D ? k : 0);
#pragma unroll
        for (int r = 0; r < NR; ++r) pre[r][c].load(base + off[r * RPI]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool in_rope = k + e >= d_cb && k + e < D;
          const long long* off = row_off + (j & 1) * 2 * TT + (in_rope ? TT : 0) + wave * NR * RPI + ld_row;
          const T* base = (in_rope ? rope : latent) + (k + e < D ? k + e : 0);
#pragma unroll
          for (int r = 0; r < NR; ++r) pre[r][c].set(e, base[off[r * RPI]]);
        }
      }
    }
  };
  auto put = [&]() {                   // registers into the LDS tile
#pragma unroll
    for (int c = 0; c < CI; ++c) {
      const int k = 4 * (ld_k4 + c * LPR);
      if (k < 4 * V4) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          f32x4 v = pre[r][c].get();
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = k + e < D ? v[e] : 0.f;
          *(f32x4*)(tile + ((wave * NR + r) * RPI + ld_row) * P + k) = v;
        }
      }
    }
  };

  row_table(0, page_of(0));
  row_table(1, page_of(1));
  int page_next = page_of(2);
  // queries of this wave's head tile (a head past the last repeats it and is not stored)
  const int head0 = hg * 16 * HT;
  f32x4 qf[KG];
  {
    const int head = min(head0 + 16 * ht + r16, p.h - 1);
    const T* qa = (const T*)p.q_abs + (((size_t)s * p.n_blocks + b) * p.h + head) * d_cb;
    const T* qr = (const T*)p.q_rope + ((size_t)s * p.h * p.groups + (b / (p.n_blocks / p.groups)) * p.h + head) * p.d_r;
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      const int k = 16 * i + 4 * q;
      Raw x;
      if constexpr (VEC) {
        x.load(k < d_cb ? qa + k : qr + (k < D ? k - d_cb : 0));
      } else {
        x.zero();
#pragma unroll
        for (int e = 0; e < 4; ++e) x.set(e, k + e < d_cb ? qa[k + e] : qr[k + e < D ? k + e - d_cb : 0]);
      }
      qf[i] = x.get();
#pragma unroll
      for (int e = 0; e < 4; ++e) qf[i][e] = k + e < D ? qf[i][e] : 0.f;
    }
  }
  __syncthreads();
  fetch(0);

  float m_run = kNegBig, l_run = 0.f;   // of head r16 (equal in the head's four lanes) / of this lane's tokens
  f32x4 z[NCT][4];
#pragma unroll
  for (int m = 0; m < NCT; ++m)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) z[m][ct] = opaque_zero4();

  for (int j = 0; j < ntiles; ++j) {
    __syncthreads();                    // the tile's readers are done; row tables are visible
    put();
    __syncthreads();
    if (j + 1 < ntiles) {
      row_table(j + 2, page_next);      // into the half that fetch(j) read, two barriers ago
      page_next = page_of(j + 3);
      fetch(j + 1);
    }
    const int valid = t1 - (t0 + j * TT);
    const int tok0 = tg * NTT * 16;     // first token of this wave's share
    f32x4 sc[NTT];
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt) sc[tt] = opaque_zero4();
    const float* krow = tile + (tok0 + r16) * P + 4 * q;
#pragma unroll
    for (int i = 0; i < KG; ++i) {
      f32x4 kf[NTT];
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt) kf[tt] = *(const f32x4*)(krow + tt * 16 * P + 16 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int tt = 0; tt < NTT; ++tt)
          sc[tt] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[tt][e], qf[i][e], sc[tt], 0, 0, 0);
    }
    float mx = -INFINITY, lowest = INFINITY;
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float x = sc[tt][i] * p.scale_log2;
        lowest = fminf(lowest, x);
        sc[tt][i] = tok0 + tt * 16 + 4 * q + i < valid ? x : -INFINITY;
        mx = fmaxf(mx, sc[tt][i]);
      }
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);
    const float alpha = exp2f(m_run - m_new);
    m_run = m_new;
    l_run *= alpha;
#pragma unroll
    for (int m = 0; m < NCT; ++m)
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) z[m][ct] *= alpha;
    // The exponential instruction returns zero below 2^-126; exp2f spends a few more on a denormal result, and the values can
    // make such a weight count.  Only a tile that holds one pays for it, the bits of the others are the same either way.
    // 8 sequences of 300 to 2048: kernel 47.3 us with exp2f throughout, 45.8 with the instruction throughout; the whole step
    // takes as long with this test in it as with the latter (75.0 us).
    if (__builtin_expect(__any(lowest - m_new < -126.f), 0)) {
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[tt][i] = exp2f(sc[tt][i] - m_new);
    } else {
#pragma unroll
      for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
        for (int i = 0; i < 4; ++i) sc[tt][i] = __builtin_amdgcn_exp2f(sc[tt][i] - m_new);   // masked rows: 2^(-inf) = 0
    }
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i) l_run += sc[tt][i];
    const float* vrow = tile + (tok0 + 4 * q) * P + 4 * r16;
#pragma unroll
    for (int tt = 0; tt < NTT; ++tt)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int m = 0; m < NCT; ++m) {
          const f32x4 vf = *(const f32x4*)(vrow + (tt * 16 + i) * P + 64 * m);
#pragma unroll
          for (int ct = 0; ct < 4; ++ct)
            z[m][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[ct], sc[tt][i], z[m][ct], 0, 0, 0);
        }
  }

  // ---- merge the token groups and write the chunk's partial (not normalised, maximum and sum in the log2 domain)
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
  __syncthreads();
  if (q == 0) {
    mbuf[wave * 16 + r16] = m_run;
    lbuf[wave * 16 + r16] = l_run;
  }
  __syncthreads();
  float m_star = kNegBig;
#pragma unroll
  for (int g = 0; g < TG; ++g) m_star = fmaxf(m_star, mbuf[(ht * TG + g) * 16 + r16]);
  const float w = exp2f(m_run - m_star);
#pragma unroll
  for (int m = 0; m < NCT; ++m)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *(f32x4*)(tile + (wave * 16 + r16) * ZP + 64 * m + 16 * q + 4 * i) =
          f32x4{z[m][0][i] * w, z[m][1][i] * w, z[m][2][i] * w, z[m][3][i] * w};
  __syncthreads();
  const int nh = min(16 * HT, p.h - head0);
  const size_t unit = ((size_t)s * p.n_blocks + b) * p.n_splits + split;
  constexpr int C4 = 16 * NCT;          // four-channel pieces per head row of the merge buffer
  const int c = 4 * (tid % C4);
  float* const dst = p.part_z + (unit * p.h + head0) * d_cb + c;
#pragma unroll
  for (int hh = tid / C4; hh < 16 * HT; hh += 256 / C4) {
    if (hh >= nh || c >= d_cb) break;
    const float* src = tile + ((hh >> 4) * TG * 16 + (hh & 15)) * ZP + c;
    f32x4 acc = *(const f32x4*)src;
#pragma unroll
    for (int g = 1; g < TG; ++g) acc += *(const f32x4*)(src + g * 16 * ZP);
    if constexpr (VEC) {
      *(f32x4*)(dst + (size_t)hh * d_cb) = acc;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < d_cb) dst[(size_t)hh * d_cb + e] = acc[e];
    }
  }
  if (tid < nh) {
    const int at = (tid >> 4) * TG * 16 + (tid & 15);
    float ms = kNegBig, L = 0.f;
#pragma unroll
    for (int g = 0; g < TG; ++g) ms = fmaxf(ms, mbuf[at + g * 16]);
#pragma unroll
    for (int g = 0; g < TG; ++g) L += lbuf[at + g * 16] * exp2f(mbuf[at + g * 16] - ms);
    p.part_ml[(unit * p.h + head0 + tid) * 2 + 0] = ms;
    p.part_ml[(unit * p.h + head0 + tid) * 2 + 1] = L;
  }
}

template <typename T, bool VEC, int KG, int NCT, int TT, int HT>
int launch_one(const DecodeArgs& a, const F32Params& p) {
  constexpr size_t lds = f32_lds_bytes<KG, NCT, TT>();
  if (lds > 64 * 1024) {
    static PerDeviceSetup setup;
    int dev = -1;
    if (setup.needed(&dev)) {
      if (hipFuncSetAttribute((const void*)decode_f32_kernel<T, VEC, KG, NCT, TT, HT>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return MLRA_ERR_LAUNCH;
      setup.done(dev);
    }
  }
  const long long wgs = (long long)a.plan.n_splits * a.n_blocks * a.batch * p.n_hg;
  // A dimension of a launch holds fewer than 2^32 threads (more wrap around without an error): rows of 2^23 workgroups.
  constexpr long long kRow = 1 << 23;
  if (wgs > 0x7fffffffLL - kRow) return MLRA_ERR_LAUNCH;
  const dim3 grid((unsigned)(wgs < kRow ? wgs : kRow), (unsigned)((wgs + kRow - 1) / kRow));
  decode_f32_kernel<T, VEC, KG, NCT, TT, HT><<<grid, 256, lds, a.stream>>>(p);
  return check_launch();
}

template <typename T, bool VEC>
int launch_typed(const DecodeArgs& a, F32Params& p, int ht) {
  const int D = a.d_cb + a.d_r;
  p.n_hg = (a.h + 16 * ht - 1) / (16 * ht);
  // Tiles of 32 channels for the smallest blocks: with 96, most loads and three quarters of the score MFMAs are padding
  // (184 bf16 sequences of 194 tokens x 64 blocks of 4 + 2 channels: 153 us, with 96 channels 289, the plain kernel 148).
  if (D <= 32)
    return ht == 4   ? launch_one<T, VEC, 2, 1, 64, 4>(a, p)
           : ht == 2 ? launch_one<T, VEC, 2, 1, 64, 2>(a, p)
                     : launch_one<T, VEC, 2, 1, 64, 1>(a, p);
  if (a.d_cb <= 64 && D <= 96)
    return ht == 4   ? launch_one<T, VEC, 6, 1, 64, 4>(a, p)
           : ht == 2 ? launch_one<T, VEC, 6, 1, 64, 2>(a, p)
                     : launch_one<T, VEC, 6, 1, 64, 1>(a, p);
  if (a.d_cb <= 128 && D <= 192)
    return ht == 4   ? launch_one<T, VEC, 12, 2, 64, 4>(a, p)
           : ht == 2 ? launch_one<T, VEC, 12, 2, 64, 2>(a, p)
                     : launch_one<T, VEC, 12, 2, 64, 1>(a, p);
  if (ht == 1) p.n_hg = (a.h + 31) / 32;      // (32-token tiles: at most two token groups)
  return ht == 4 ? launch_one<T, VEC, 20, 4, 32, 4>(a, p) : launch_one<T, VEC, 20, 4, 32, 2>(a, p);
}

}  // namespace

// Queries and accumulators live in registers: (d_cb + d_r) / 4 + d_cb / 4 of them per lane, beside the tile in flight.
bool decode_f32_supported(const DecodeArgs& a) { return a.d_cb <= 256 && a.d_cb + a.d_r <= 320; }

// Head tiles of 16 per workgroup: 64 heads where that gives every CU a workgroup (a tile is then staged for four head
// tiles at once: 59 against 61 us with 32 and 77 with 16 on 8 sequences of 300 to 2048), fewer where it would leave CUs
// idle (8 sequences of 256 tokens: 15 us with 32 heads, 22 with 64).
static int head_tiles(const DecodeArgs& a) {
  const int n_ht = (a.h + 15) / 16;
  const long units = (long)a.plan.n_splits * a.n_blocks * a.batch;
  int ht = n_ht >= 4 ? 4 : n_ht >= 2 ? 2 : 1;
  while (ht > 1 && units * ((n_ht + ht - 1) / ht) < a.cus) ht >>= 1;
  return ht;
}

// Fitted chunk lengths (at most 64 sequences, whose lengths the kernel then knows) pay where the slots are more than a round
// of workgroups, so that a longer chunk can bring a ragged batch down to one, and a chunk is long against the fit itself,
// which takes 1 us for a few sequences and 4 for 60.  Whole steps, fp32, 128 heads, 4 x 128 channels: 8 sequences of 300 to
// 2048 90.8 -> 78.0 us, 16 of 100 to 560 77.7 -> 66.1; with one round of slots 4 of 500 to 1000 48.7 -> 50.0, with chunks
// of 9000 cycles (12 heads, 64 channels) 60 of 200 to 900 38.8 -> 43.0.
bool decode_f32_fits_chunks(const DecodeArgs& a) {
  if (a.batch < 2 || a.batch > chunk_fit::kMaxSeqs || a.plan.n_splits < 2 || a.q_group > 1) return false;
  const int ht = head_tiles(a), D = a.d_cb + a.d_r;
  const long wgs = (long)a.plan.n_splits * a.n_blocks * a.batch * ((a.h + 16 * ht - 1) / (16 * ht));
  const int k16 = D <= 32 ? 2 : a.d_cb <= 64 && D <= 96 ? 6 : a.d_cb <= 128 && D <= 192 ? 12 : 20, v64 = (a.d_cb + 63) / 64;
  const long cycles = 32L * ht * (4 * k16 + 16 * v64) * (a.plan.chunk_tokens / chunk_fit::kTokens);   // matrix pipe, per chunk
  return wgs > a.cus && cycles >= 12000;
}

int launch_decode_f32(const DecodeArgs& a) {
  F32Params p;
  p.latent = a.latent;
  p.rope = a.rope;
  p.page_table = a.page_table;
  p.seq_lens = a.seq_lens;
  p.q_abs = a.q_abs;
  p.q_rope = a.q_rope;
  p.part_z = a.part_z;
  p.part_ml = a.part_ml;
  p.page_size = a.page_size;
  p.max_pages = a.max_pages;
  p.n_blocks = a.n_blocks;
  p.groups = a.groups;
  p.d_cb = a.d_cb;
  p.d_r = a.d_r;
  p.h = a.h;
  p.batch = a.batch;
  p.n_splits = a.plan.n_splits;
  p.chunk = a.plan.chunk_tokens;
  p.scale_log2 = softmax_scale_log2(a.softmax_scale);
  p.chunk_tab = a.fitted ? a.chunk_tab : nullptr;
  p.fit_min = a.fit_tiles;
  p.cus = a.cus;
  // four-element loads: every row and every head's query starts on a multiple of four elements, and so do the bases
  const uintptr_t bases = (uintptr_t)a.latent | (uintptr_t)a.rope | (uintptr_t)a.q_abs | (uintptr_t)a.q_rope;
  const bool vec = a.d_cb % 4 == 0 && a.d_r % 4 == 0 && bases % (a.dtype == MLRA_BF16 ? 8 : 16) == 0;
  const int ht = head_tiles(a);
  if (a.dtype == MLRA_BF16) return vec ? launch_typed<bf16_t, true>(a, p, ht) : launch_typed<bf16_t, false>(a, p, ht);
  return vec ? launch_typed<float, true>(a, p, ht) : launch_typed<float, false>(a, p, ht);
}

}  // namespace mlra
