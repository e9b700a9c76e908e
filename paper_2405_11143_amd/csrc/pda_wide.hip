// Pass 1 for steps with more than 4 query chunks per sequence (chunked and
// fresh prefill, long drafts: Section 3.2) and no shared-prefix groups.
//
// A work item is (partition of a context, sequence, KV head, group of up to 8
// or 16 chunks), as in pda_partition.hip; a workgroup of 4 wavefronts takes 8
// chunks of it (an item of 16 is two workgroups), and each wavefront two
// neighbouring chunks, 32 query rows.  Chunked prefill is bound by the matrix
// cores and, with them busy, by the chip's power: the clock falls to about 1.8
// GHz with the MFMA pipes busy on 59% of the cycles, VALU instructions issued on
// 52% and both at once on 25%.  Fresh prompts (pipes 24% busy) wait for the starts
// and ends of many short items.  What follows from that:
//  * Both products on MFMA f32_32x32x16_bf16, transposed as in pda_wave.h
//    (S^T = K Q^T, O^T = V^T P^T): one instruction of 32 cycles keeps a SIMD's
//    pipe full from a single wavefront and leaves room for 4-6 VALU
//    instructions under it, where the 16-row instructions of 16 cycles left
//    2-3 and the softmax added to their time instead of hiding under it.  The
//    lane's 16 scores (one query row) are already its P^T fragments, as the
//    k order of the second product is free.
//  * The scores of step s + 1 are formed while step s is folded, so that the
//    24 MFMAs and the softmax of a step are one stretch without a branch
//    (1561 -> 1501 us on the step below).
//  * K and V tiles go straight from memory to LDS (16 bytes per lane), a
//    32-token step at a time in four buffers: one step is folded, the next
//    one's scores are formed, two are in flight.  Through registers (two
//    buffers of 64 tokens) the same fold took 1731 us: the LDS writes and the
//    registers' loads waited on each other.
//  * Cached loads: each tile is read by every workgroup that shares the
//    (sequence, KV head), and 89% of the requests hit the XCD's L2
//    (non-temporal loads: 48%, 1734 us).
//  * Two independent workgroups of 4 wavefronts per compute unit; one of 8,
//    which halves the tile loads but keeps its wavefronts in step, took
//    1585 us.
// 32 sequences of 1024-8192 tokens, 512 of them new, 32 / 8 heads, D = 128:
// 1853 -> 1586 us against 8 wavefronts of two 16-row tiles each (738 TFLOP/s
// of attention, 1107 issued with P in two halves); 64 new tokens over 64
// contexts of up to 16384: 706 -> 622 us; 48 prompts of up to 1024 tokens
// (28 / 4 heads), the append of their K and V among it: 754 -> 432 us.
#include "pda_wave.h"

namespace pda {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kTileRows = 32;          // query rows of a wavefront: two 16-row chunks
constexpr int kWgChunks = 2 * kWaves;  // chunks of a workgroup
constexpr int kStageBlocks = 2;        // blocks of a staged step: 32 tokens
constexpr int kBuffers = 4;            // one step folded, the next one's scores formed, two in flight
constexpr int kWindow = 1024;          // block ids held in LDS at a time
constexpr float kExactMax = 128.f;     // running maxima whose rounding is below P's resolution

template <int D>
struct WideLds {
  static constexpr int kTilePieces = 2 * D;  // 16-byte pieces of a K or V tile
  static constexpr int kBlockPieces = 2 * kTilePieces;
  union {
    uint4 buf[kBuffers][kStageBlocks][kBlockPieces];
    f32x4_t o[kWaves][kTileRows][D / 4];
  };
  int ids[kWindow];
};

// 16 bytes per lane from k + k_off and v + v_off straight into LDS, at k_lds and
// v_lds plus 16 lane.  The compiler does not count these loads: the caller waits
// with wait_loads.  (It counts the builtin's, and waits for all of them before
// every LDS read: no load would stay in flight.)  M0, which names the LDS
// address, belongs to the compiler: it gets back what it held.
__device__ __forceinline__ void load_to_lds(const char* k, int k_off, unsigned k_lds, const char* v, int v_off,
                                            unsigned v_lds) {
  unsigned m0;
  asm volatile("s_mov_b32 %0, m0\n\t"
               "s_mov_b32 m0, %5\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3\n\t"
               "s_mov_b32 m0, %6\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %4\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(m0)
               : "v"(k_off), "v"(v_off), "s"(k), "s"(v), "s"(k_lds), "s"(v_lds)
               : "memory");
}
template <int N>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

template <int D>
__global__ void __launch_bounds__(kWaves * kWaveSize) __attribute__((amdgpu_waves_per_eu(2)))
wide_kernel(const StepArgs a) {
  using S = WideLds<D>;
  constexpr int KS = D / 16;  // score MFMA k-steps
  constexpr int VT = D / 32;  // output tiles of 32 columns
  constexpr int kTileBytes = kBlockTokens * D * 2;
  __shared__ __align__(16) S st;

  // an item of 16 chunks is two workgroups, next to each other on one XCD
  const int halves = a.chunks_per_group / kWgChunks;
  const int bid = blockIdx.x;
  const int slot = halves == 2 ? (bid >> 4) * 8 + (bid & 7) : bid;
  const int half = halves == 2 ? (bid >> 3) & 1 : 0;
  if (slot >= a.num_regular_items) return;
  const int item = a.order ? a.order[slot] : slot;
  if ((unsigned)item >= (unsigned)a.num_regular_items) return;

  const int Hq = a.num_q_heads;
  const int G = a.group;
  const int HC = a.num_kv_heads * a.num_chunk_groups;
  const int gc = item % HC;
  const int b = (item / HC) % a.num_seqs;
  const int p = item / (HC * a.num_seqs);
  const int g = gc / a.num_chunk_groups;
  const int cg = gc % a.num_chunk_groups;
  const int nq = a.num_query_tokens;
  const int Tp = a.partition_tokens;
  const int item_first = cg * a.chunks_per_group;
  const int item_end = min(a.num_query_chunks, item_first + a.chunks_per_group);
  const int c_first = item_first + half * kWgChunks;
  const int c_end = min(item_end, c_first + kWgChunks);
  if (c_first >= c_end) return;
  const int tid = threadIdx.x;
  const int lane = tid & (kWaveSize - 1);
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5;       // which half of the k-groups the lane holds
  const int col = lane & 31;      // the lane's row of the tile

  int L = a.lens[b];
  L = L < 0 ? 0 : (L > a.max_context_len ? a.max_context_len : L);
  auto parts_of = [&](int c) {
    const int lv = chunk_visible(a, L, c);
    return lv > 0 ? (lv + Tp - 1) / Tp : 0;
  };
  if (p == 0) {  // chunks that see nothing: zero rows
    for (int c = c_first; c < c_end; ++c) {
      if (chunk_visible(a, L, c) > 0) break;  // later chunks see more
      const int i0 = c * a.query_chunk;
      const int rows = min(a.query_chunk, nq - i0) * G;
      for (int i = tid; i < rows * (D / 4); i += kWaves * kWaveSize) {
        const int r = i / (D / 4);
        store_nt4(a.out + (((size_t)b * nq + i0 + r / G) * Hq + (size_t)g * G + r % G) * D + 4 * (i % (D / 4)), 0.f, 0.f,
                  0.f, 0.f);
      }
    }
  }
  if (p >= parts_of(c_end - 1)) return;  // the last chunk sees the most

  // ---- this wavefront's tile: chunks ca and ca + 1 ----
  const int ca = c_first + 2 * w;
  const bool active = ca < c_end;
  const int cb = ca + 1 < c_end ? ca + 1 : ca;
  const int t_pe = (p + 1) * Tp;  // tokens at or past it belong to the next partition
  const int my_c = active ? (col < 16 ? ca : cb) : c_first;
  const int my_i0 = my_c * a.query_chunk;
  const int my_rows = min(a.query_chunk, nq - my_i0) * G;
  const int my_r = (col & 15) % my_rows;  // lane rows past the chunk's last one repeat real rows
  const int my_qi = my_i0 + my_r / G;
  const int limit = min(L - (nq - 1 - my_qi), t_pe);  // the lane's row sees tokens below it
  const int l_first = min(chunk_visible(a, L, ca) - min(a.query_chunk, nq - ca * a.query_chunk) + 1, t_pe);
  const int l_vis_a = min(max(chunk_visible(a, L, ca), 0), t_pe);
  const int l_vis = min(max(chunk_visible(a, L, cb), 0), t_pe);

  float scale = a.scale_log2;
  const unsigned flip = scale < 0.f ? 0x80008000u : 0u;
  const unsigned keep = scale == 0.f ? 0u : 0xffffffffu;  // a zero scale: zero scores, whatever is masked
  scale = keep ? fabsf(scale) : 1.f;
  bf16x8_t q[KS];
  {
    const uint16_t* qp = a.q + (((size_t)b * nq + my_qi) * Hq + (size_t)g * G + my_r % G) * D + 8 * hh;
#pragma unroll
    for (int c = 0; c < KS; ++c) {
      uint4 u = *reinterpret_cast<const uint4*>(qp + 16 * c);
      u.x = (u.x ^ flip) & keep, u.y = (u.y ^ flip) & keep, u.z = (u.z ^ flip) & keep, u.w = (u.w ^ flip) & keep;
      q[c] = __builtin_bit_cast(bf16x8_t, u);
    }
  }
  f32x16_t o[VT];
#pragma unroll
  for (int t = 0; t < VT; ++t)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[t][i] = 0.f;
  // The running maximum before scaling, and scaled and rounded.  A step that
  // moves the maximum takes its probabilities as exp2((s - m_raw) * scale): the
  // row's largest score gets exactly 1, so a row that sees one token returns its
  // V row bit for bit, and scores of any size cancel.  The other steps take them
  // as exp2(s * scale - m_run), in one instruction less per score, as long as
  // the rounding of m_run (up to kExactMax: below 2^-17, the resolution of P) is
  // all that the two differ by.
  float m_raw = fmaxf(-1e30f / scale, -__FLT_MAX__), m_run = mul_rounded(m_raw, scale), l_run = 0.f;

  const char* kpool = reinterpret_cast<const char*>(a.k) + (size_t)g * kTileBytes;
  const char* vpool = reinterpret_cast<const char*>(a.v) + (size_t)g * kTileBytes;
  const int32_t* table_row = a.table + (size_t)b * a.max_blocks_per_seq;
  const size_t block_bytes = (size_t)a.num_kv_heads * kTileBytes;
  const int J0 = p * Tp / kBlockTokens;
  auto vis_blocks = [&](int c) { return (min(max(chunk_visible(a, L, c), 0), t_pe) + kBlockTokens - 1) / kBlockTokens; };
  const int J1 = vis_blocks(c_end - 1);
  bool bad = false;  // a block id outside the pool, anywhere the item looks

  // Staging: 1 KiB of a tile per load instruction.  A tile is KPT of them; at
  // D = 128 wavefront w takes the w-th of every tile of the step, at D = 64
  // half w % 2 of the tiles of block w / 2.  K lands as it lies in memory; in
  // a V row the 16-byte pieces are permuted, so that the 4 rows of a
  // transposed read fall on disjoint banks.
  constexpr int KPT = kTileBytes / 1024;
  constexpr int kStepLoads = kStageBlocks * 2 * KPT / kWaves;  // per wavefront
  constexpr int RP = D / 8;                                    // pieces of a V row
  const int k_load = (w % KPT) * 1024 + lane * 16;
  const int v_row = lane / RP;  // (mod 4: a wavefront's KiB starts at a multiple of 4 rows)
  const int v_load = (w % KPT) * 1024 + v_row * (2 * D) + 16 * ((lane % RP) ^ (D == 128 ? 4 * (v_row & 3) : 4 * ((v_row >> 1) & 1)));
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)&st.buf[0][0][0]) +
                        (w % KPT) * 1024;
  int ids = 0;  // lane x: the id of block 64 (block / 64) + x of the window
  auto issue = [&](int step) {
    const int j = min(step * kStageBlocks, kWindow - kStageBlocks);  // steps past the window load what nothing folds
    if (j % kWaveSize == 0) ids = st.ids[j + lane];
    const unsigned dst = lds0 + (step % kBuffers) * (kStageBlocks * S::kBlockPieces * 16);
#pragma unroll
    for (int s = 0; s < kStageBlocks; ++s) {
      if (KPT * 2 == kWaves && (w >> 1) != s) continue;  // D = 64
      const size_t off = (size_t)(unsigned)__builtin_amdgcn_readlane(ids, j % kWaveSize + s) * block_bytes;
      const unsigned at = dst + s * (S::kBlockPieces * 16);
      load_to_lds(kpool + off, k_load, at, vpool + off, v_load, at + kTileBytes);
    }
  };

  typedef short v4s_t __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) v4s_t lds_v4s_t;
  const int k_piece = (col >> 4) * S::kBlockPieces + hh * 16 + (lane & 15);
  // transposed V reads: source lane s of each 16 points at row 4 hh + s / 4, columns 16 u + 4 (s % 4)
  const int s16 = lane & 15;
  const int tr_row = (4 * hh + s16 / 4) * D + 16 * ((lane >> 4) & 1) + 4 * (s16 & 3);
  int tr_off[VT];  // (with the row's permutation of pieces)
#pragma unroll
  for (int t = 0; t < VT; ++t) tr_off[t] = tr_row + 32 * (t ^ (D == 128 ? s16 / 4 : s16 / 8));

  f32x16_t s;  // scores of the step to fold: reg i is token tok0 + 8 (i / 4) + 4 hh + i % 4
  float top;   // the largest of them
  auto scores = [&](const uint4* blocks) {
    f32x16_t x;
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = 0.f;
#pragma unroll
    for (int c = 0; c < KS; ++c)
      x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, blocks[k_piece + 32 * c]), q[c], x, 0, 0, 0);
    return x;
  };
  auto largest = [&] {
    float x = max3(s[0], s[1], s[2]);
#pragma unroll
    for (int i = 3; i + 1 < 15; i += 2) x = max3(x, s[i], s[i + 1]);
    top = max3(x, s[15], s[15]);
    asm volatile("" : "+v"(top));  // the MFMA results are first read in their own basic block
  };
  auto mask = [&](int tok0) {
    if (tok0 + 32 > l_first) {  // wavefront-uniform: some row does not see some of these tokens
      asm volatile("");  // a branch: as selects the masking would run on every step
      const int rel = limit - (tok0 + 4 * hh);
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (8 * (i / 4) + i % 4 >= rel) s[i] = -__builtin_huge_valf();
      largest();
    }
  };
  // o += p V of the tokens [l_vis_a, l_vis) of a step, one after the other,
  // for the second chunk's rows (never reached with finite values).
  auto add_apart = [&](int tok0, const uint4* blocks, float ref) {
    for (int x = max(tok0, l_vis_a) - tok0; x < min(32, l_vis - tok0); ++x) {
      float sx = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) sx = i == 4 * (x / 8) + x % 4 ? s[i] : sx;
      const float mine = exp2_fast(fmaf(sx, scale, -ref));
      const float other = __shfl_xor(mine, 32);
      const float px = (x / 4) % 2 == hh ? mine : other;
      const int perm = D == 128 ? 4 * (x & 3) : 4 * ((x >> 1) & 1);
      const uint2* row = reinterpret_cast<const uint2*>(blocks + (x / 16) * S::kBlockPieces + S::kTilePieces + (x % 16) * RP);
#pragma unroll
      for (int t = 0; t < VT; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint2 v = row[2 * ((4 * t + k) ^ perm) + hh];  // columns 32 t + 8 k + 4 hh .. + 3
          const float vv[4] = {__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16),
                               __uint_as_float(v.y & 0xffff0000u)};
#pragma unroll
          for (int e = 0; e < 4; ++e) o[t][4 * k + e] = col < 16 ? o[t][4 * k + e] : fmaf(px, vv[e], o[t][4 * k + e]);
        }
    }
  };
  // Fold the step whose scores are in s (32 tokens from tok0 on, two blocks of
  // a buffer), and form the scores of the next one (in next_blocks).
  auto fold = [&](int tok0, const uint4* blocks, const uint4* next_blocks) {
    auto v_frag = [&](int m, int t) {
      const uint16_t* v0 = reinterpret_cast<const uint16_t*>(blocks + S::kTilePieces + m * S::kBlockPieces) + tr_off[t];
      const uint2 x = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)v0));
      const uint2 y = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_t*)(v0 + 8 * D)));
      return make_uint4(x.x, x.y, y.x, y.y);
    };
    uint4 vf[2][VT];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int t = 0; t < VT; ++t) vf[m][t] = v_frag(m, t);
    bool apart = false;
    if (tok0 + 32 > l_vis_a) {  // wavefront-uniform: some V rows are not for every row of the tile
      asm volatile("");
      // Rows [l_vis_a, l_vis) are the second chunk's own.  When they are
      // finite the first chunk's zero probabilities leave them out; otherwise
      // they are added apart, to the second chunk only.
      for (int x = max(tok0, l_vis_a); x < min(tok0 + 32, l_vis); ++x) {
        const unsigned* row = reinterpret_cast<const unsigned*>(blocks + ((x - tok0) / 16) * S::kBlockPieces + S::kTilePieces + ((x - tok0) % 16) * RP);
        const unsigned e = row[lane & (D / 2 - 1)] & 0x7f807f80u;
        apart |= __builtin_amdgcn_ballot_w64((e & 0x7f800000u) == 0x7f800000u || (e & 0x7f80u) == 0x7f80u) != 0;
      }
      // V rows that no row of the tile sees are zeroed, whatever they hold.
      const int vrel = (apart ? l_vis_a : l_vis) - (tok0 + 4 * hh);
      auto word = [&](unsigned v, int t0) {
        return v & ((t0 < vrel ? 0x0000ffffu : 0u) | (t0 + 1 < vrel ? 0xffff0000u : 0u));
      };
#pragma unroll
      for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int t = 0; t < VT; ++t)
          vf[m][t] = make_uint4(word(vf[m][t].x, 16 * m), word(vf[m][t].y, 16 * m + 2), word(vf[m][t].z, 16 * m + 8),
                                word(vf[m][t].w, 16 * m + 10));
    }
    float ref = m_run;
    if (__builtin_amdgcn_ballot_w64(fmaf(top, scale, -m_run) > 8.f || fabsf(m_run) > kExactMax) != 0) {
      const float mn = fmaxf(m_raw, fmaxf(top, __shfl_xor(top, 32)));
      const float al = exp2_fast((m_raw - mn) * scale);
      m_raw = mn;
      m_run = mul_rounded(mn, scale);
      ref = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] -= m_raw;
      l_run *= al;
#pragma unroll
      for (int t = 0; t < VT; ++t) o[t] *= al;
    }
    if (apart) add_apart(tok0, blocks, ref);
    const f32x16_t ns = scores(next_blocks);
    bf16x8_t bh[2], bl[2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      float pr[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) pr[i] = exp2_fast(fmaf(s[8 * m + i], scale, -ref));
      l_run += ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
      unsigned hw[4], lw[4];
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const unsigned h0 = __float_as_uint(pr[2 * h]) & 0xffff0000u;
        const unsigned h1 = __float_as_uint(pr[2 * h + 1]) & 0xffff0000u;
        hw[h] = pack_halves(__float_as_uint(pr[2 * h]), __float_as_uint(pr[2 * h + 1]), true);
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        const bf16x2_t l2 = {(__bf16)(pr[2 * h] - __uint_as_float(h0)), (__bf16)(pr[2 * h + 1] - __uint_as_float(h1))};
        lw[h] = __builtin_bit_cast(unsigned, l2);
      }
      bh[m] = __builtin_bit_cast(bf16x8_t, make_uint4(hw[0], hw[1], hw[2], hw[3]));
      bl[m] = __builtin_bit_cast(bf16x8_t, make_uint4(lw[0], lw[1], lw[2], lw[3]));
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        const bf16x8_t av = __builtin_bit_cast(bf16x8_t, vf[m][t]);
        o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bh[m], o[t], 0, 0, 0);
        o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bl[m], o[t], 0, 0, 0);
      }
    s = ns;
    largest();
    mask(tok0 + 32);
  };

  for (int jw = J0; jw < J1; jw += kWindow) {
    const int jwe = min(J1, jw + kWindow);
    // (as many as the steps and the loads issued past them read, by 64)
    const int n_ids = min(kWindow, (jwe - jw + kBuffers * kStageBlocks + kWaveSize) / kWaveSize * kWaveSize);
    for (int x = tid; x < n_ids; x += kWaves * kWaveSize) {
      const int id = table_row[min(jw + x, jwe - 1)];  // past the end: the last block again (masked)
      const bool ok = (unsigned)id < (unsigned)a.num_blocks;  // never read outside the pool
      bad |= !ok;
      st.ids[x] = ok ? id : 0;
    }
    __syncthreads();
    const int nsteps = (jwe - jw + kStageBlocks - 1) / kStageBlocks;
#pragma unroll
    for (int x = 0; x < kBuffers - 1; ++x) issue(x);
    wait_loads<(kBuffers - 2) * kStepLoads>();
    __syncthreads();
    if (active) {
      s = scores(st.buf[0][0]);
      largest();
      mask(jw * kBlockTokens);
    }
    for (int step = 0; step < nsteps; ++step) {
      // the next step's loads of this wavefront, and behind the barrier those
      // of the others; the last step's buffer is free then
      wait_loads<(kBuffers - 3) * kStepLoads>();
      __syncthreads();
      issue(step + kBuffers - 1);
      const int tok0 = (jw + step * kStageBlocks) * kBlockTokens;
      if (active && tok0 < l_vis)  // wavefront-uniform
        fold(tok0, st.buf[step % kBuffers][0], st.buf[(step + 1) % kBuffers][0]);
    }
    wait_loads<0>();
    __syncthreads();
  }
  // the other workgroup of the item may look further: its ids count as well
  for (int j = J1 + tid; j < vis_blocks(item_end - 1); j += kWaves * kWaveSize)
    bad |= (unsigned)table_row[j] >= (unsigned)a.num_blocks;
  const bool any_bad = __syncthreads_or(bad ? 1 : 0) != 0;  // (and the staging area is free)

  l_run += __shfl_xor(l_run, 32);
  const int my_parts = parts_of(my_c);
  const bool single = my_parts == 1;
  const float mul = any_bad ? __builtin_nanf("") : single && l_run > 0.f ? 1.f / l_run : 1.f;
  const int swz = col & (D / 4 - 1);  // 16-byte units of a row permuted: conflict-free
#pragma unroll
  for (int t = 0; t < VT; ++t)
#pragma unroll
    for (int k = 0; k < 4; ++k)
      st.o[w][col][(8 * t + 2 * k + hh) ^ swz] =
          f32x4_t{o[t][4 * k] * mul, o[t][4 * k + 1] * mul, o[t][4 * k + 2] * mul, o[t][4 * k + 3] * mul};
  __syncthreads();
  if (!active) return;
  for (int x = lane; x < kTileRows * (D / 4); x += kWaveSize) {
    const int r32 = x / (D / 4);
    const int d0 = 4 * (x % (D / 4));
    const int c = r32 < 16 ? ca : ca + 1;
    if (c >= c_end) continue;
    const int i0 = c * a.query_chunk;
    const int h = r32 & 15;
    if (h >= min(a.query_chunk, nq - i0) * G) continue;
    const int cparts = parts_of(c);
    if (p >= cparts) continue;  // the chunk sees nothing in this partition
    const size_t row = ((size_t)b * nq + i0 + h / G) * Hq + (size_t)g * G + h % G;
    const f32x4_t v = st.o[w][r32][(d0 / 4) ^ (r32 & (D / 4 - 1))];
    if (cparts == 1)
      store_nt4(a.out + row * D + d0, v[0], v[1], v[2], v[3]);
    else
      *reinterpret_cast<f32x4_t*>(a.part_o + (row * a.slots_per_row + p) * D + d0) = v;
  }
  if (hh == 0 && (col & 15) < my_rows && (col < 16 || ca + 1 < c_end) && p < my_parts && !single) {
    const size_t row = ((size_t)b * nq + my_qi) * Hq + (size_t)g * G + my_r % G;
    a.part_m[row * a.slots_per_row + p] = m_run;
    a.part_l[row * a.slots_per_row + p] = l_run;
  }
}

template <int D>
hipError_t launch_d(const StepArgs& a, hipStream_t stream) {
  const unsigned items = (unsigned)a.num_regular_items;
  const unsigned grid = a.chunks_per_group > kWgChunks ? (items + 7) / 8 * 16 : items;
  hipLaunchKernelGGL(wide_kernel<D>, dim3(grid), dim3(kWaves * kWaveSize), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_wide(const StepArgs& a, int head_dim, hipStream_t stream) {
  if (head_dim == 64) return launch_d<64>(a, stream);
  if (head_dim == 128) return launch_d<128>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace pda
