// Pass 2 of paged decode attention: merge partial softmax states.
//
// A context split into partitions k = 0..n-1 leaves, per query head, the
// partition's reference maximum m_k (log2 domain), denominator l_k and
// unnormalised output O_k (a partition that the row does not reach has
// m_k = -1e30, l_k = 0, O_k = 0).  Softmax over the whole context is recovered
// exactly by rescaling every partition to the common maximum M = max_k m_k:
//   out = sum_k 2^(m_k - M) O_k / sum_k 2^(m_k - M) l_k.
// Both sums run in a fixed order, so the result is reproducible.  One
// wavefront per output row (sequence, new token, query head), 4 rows per
// workgroup.
//
// A small step's merge is a chain of memory latencies, so the chain is kept
// short.  A row's states sit in its own slots_per_row slots (its group's prefix
// partitions, then its own), whatever it sees: the maxima and denominators of
// all slots (one per lane) and the outputs of the first kSpec are loaded
// before the row's length is known, and slots that turn out to hold nothing
// get weight 0 and are left out by selection.  Outputs are read 16 bytes per
// lane, several slots per instruction, and past the first kSpec slots
// kInFlight instructions at a time.
//
// With many rows (several new tokens per sequence) the merge streams tens to
// hundreds of MB, and what counts is the wavefronts in flight and the vector
// instructions of a row: rows of up to kFewSlots or kSpec slots have variants
// without the loop over further slots (22 and 33 VGPRs at D = 128 against 73: 8
// wavefronts per SIMD instead of 6; 83 and 5 when this was measured), and
// whatever is the same for a wavefront is scalar (169 and 210 vector
// instructions).  Whole steps, one kernel for all against these: 64 new tokens over 64 long contexts (131072 rows of 2 slots)
// 616 -> 601 us, 4 over 188 (12032 rows of 6) 56.8 -> 55.8, 11 over 22 (9680 of
// 6) 53.2 -> 52.3, 4 over 303 (19392 of 3) 44.5 -> 43.2.  That is what such steps
// took before outputs were loaded early (55.9, 52.3, 44.0): the early loads are
// for small steps.  Lengths first where rows are many was measured as well: 12
// new tokens over 77 (29568 rows of 2, most of them whole) +-0, the other two
// 56.0 -> 56.5 and 52.6 -> 53.5, 64 over 64 610 -> 600.
#include "pda_internal.h"

namespace pda {
namespace {

// Maximum over the wavefront's first LANES lanes (a power of two; the others hold
// less); every lane gets the same value.
template <int LANES>
__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 1; o < LANES; o <<= 1) x = fmaxf(x, __shfl_xor(x, o));
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// Sum over them in a fixed butterfly order (the others hold 0); every lane gets
// the same bits.
template <int LANES>
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 1; o < LANES; o <<= 1) x += __shfl_xor(x, o);
  return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

__device__ __forceinline__ int clamped_len(const StepArgs& a, int b) {
  const int L = a.lens[b];
  return L < 0 ? 0 : (L > a.max_context_len ? a.max_context_len : L);
}

constexpr int kMergeRows = 4;  // rows (wavefronts) per workgroup
constexpr int kFewSlots = 4;   // slots per row of the smallest variant
constexpr int kSpec = 8;       // slots whose outputs are loaded before the length is known
constexpr int kInFlight = 4;   // output loads in flight past them

// Output row (b, i, h), row = (b * n + i) * Hq + h, has its partial states
// at slots row * S .. row * S + S - 1 (S = slots_per_row): first the prefix
// partitions of its group, then, from slot row * S + Pp, its own partitions
// (as many as the query chunk of new token i sees after the prefix).
// SPEC slots are loaded early; MORE: a row may have more of them.
template <int D, int SPEC, bool MORE>
__global__ void __launch_bounds__(kMergeRows * kWaveSize) __attribute__((amdgpu_waves_per_eu(MORE ? 5 : 8)))
merge_kernel(const StepArgs a) {
  constexpr int LPS = D / 4;             // lanes per slot: 4 columns each
  constexpr int SPI = kWaveSize / LPS;   // slots per load instruction
  constexpr int NS = SPEC / SPI;
  constexpr int LANES = MORE ? kWaveSize : SPEC;  // lanes that hold a slot's state
  // (the same for the whole wavefront: its divisions and addresses are scalar)
  const int row = blockIdx.x * kMergeRows + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWaveSize - 1);
  if ((size_t)row >= (size_t)a.num_seqs * a.num_query_tokens * a.num_q_heads) return;  // spare wavefronts
  const int i = (row / a.num_q_heads) % a.num_query_tokens;
  const int b = row / (a.num_q_heads * a.num_query_tokens);
  const int S = a.slots_per_row;
  const size_t first = (size_t)row * S;
  const int sub = lane / LPS;         // the lane's slot of a load instruction
  const int d0 = 4 * (lane % LPS);    // its columns
  const float* src = a.part_o + (first + sub) * D + d0;  // slot s + sub at src + s * D
  constexpr float kNone = -__builtin_huge_valf();

  float m_first = kNone, l_first = 0.f;
  if (lane < S) {
    m_first = a.part_m[first + lane];
    l_first = a.part_l[first + lane];
  }
  f32x4_t o_s[NS];
#pragma unroll
  for (int x = 0; x < NS; ++x)
    if (x * SPI + sub < S) o_s[x] = *reinterpret_cast<const f32x4_t*>(src + (size_t)(x * SPI) * D);

  const int L = clamped_len(a, b);
  const int vis = chunk_visible(a, L, i / a.query_chunk);
  if (vis <= 0) return;  // pass 1 wrote zeros
  const int Tp = a.partition_tokens;
  const int t0 = min(seq_prefix_len(a, b), vis);
  const int n_pre = (t0 + Tp - 1) / Tp;
  const int n_own = (vis - t0 + Tp - 1) / Tp;
  if (n_pre == 0 && n_own <= 1) return;  // pass 1 wrote the final row
  const int own = a.prefix_partitions, own_end = own + n_own;
  auto valid = [&](int s) { return s < n_pre || (s >= own && s < own_end); };
  // the maximum and the denominator of slots s0 .. s0 + 63, one per lane
  auto state = [&](int s0, float& m, float& l) {
    const int s = s0 + lane;
    if (s0 == 0) {
      m = m_first, l = l_first;
    } else if (s < S) {
      m = a.part_m[first + s], l = a.part_l[first + s];
    }
    if (!valid(s)) m = kNone, l = 0.f;
  };
  const int state_end = MORE ? own_end : 1;  // (without MORE the first kWaveSize slots are all)
  float M = kNone;
  for (int s0 = 0; s0 < state_end; s0 += kWaveSize) {
    float m = kNone, l = 0.f;
    state(s0, m, l);
    M = fmaxf(M, m);
  }
  M = wave_max<LANES>(M);
  f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
  float lpart = 0.f;
  auto add = [&](bool in, float wgt, const f32x4_t& v) {
    if (in) {
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(wgt, v[e], acc[e]);
    }
  };
  for (int s0 = 0; s0 < state_end; s0 += kWaveSize) {
    float m = kNone, l = 0.f;
    state(s0, m, l);
    const float wgt = __builtin_amdgcn_exp2f(m - M);  // 2^(m - M), 0 for a slot that holds nothing
    lpart = fmaf(wgt, l, lpart);
    const int end = min(kWaveSize, own_end - s0);
    int x0 = 0;
    if (s0 == 0) {
#pragma unroll
      for (int x = 0; x < NS; ++x) {
        auto of_lane = [&](int i) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, wgt), i)); };
        float w_x = of_lane(x * SPI);  // the weight of slot x SPI + sub
#pragma unroll
        for (int i = 1; i < SPI; ++i) w_x = sub == i ? of_lane(x * SPI + i) : w_x;
        add(valid(x * SPI + sub), w_x, o_s[x]);
      }
      x0 = SPEC;
    }
    for (; MORE && x0 < end; x0 += kInFlight * SPI) {
      f32x4_t v[kInFlight];
      auto slot = [&](int x) { return x0 + x * SPI + sub; };  // of these 64
      auto in = [&](int x) { return slot(x) < kWaveSize && valid(s0 + slot(x)); };
#pragma unroll
      for (int x = 0; x < kInFlight; ++x)
        if (in(x)) v[x] = *reinterpret_cast<const f32x4_t*>(src + (size_t)(s0 + x0 + x * SPI) * D);
#pragma unroll
      for (int x = 0; x < kInFlight; ++x) add(in(x), __shfl(wgt, slot(x) & (kWaveSize - 1)), v[x]);
    }
  }
#pragma unroll
  for (int o = LPS; o < kWaveSize; o <<= 1)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += __shfl_xor(acc[e], o);
  const float lsum = wave_sum<LANES>(lpart);
  const bool pos = lsum > 0.f;  // 0: the row sees nothing
  if (sub == 0) {
    float* orow = a.out + (size_t)row * D + d0;
    store_nt4(orow, pos ? acc[0] / lsum : acc[0], pos ? acc[1] / lsum : acc[1], pos ? acc[2] / lsum : acc[2],
              pos ? acc[3] / lsum : acc[3]);
  }
}

template <int D>
void launch_d(const StepArgs& a, unsigned grid, hipStream_t stream) {
  const dim3 threads(kMergeRows * kWaveSize);
  if (a.slots_per_row <= kFewSlots)
    hipLaunchKernelGGL((merge_kernel<D, kFewSlots, false>), dim3(grid), threads, 0, stream, a);
  else if (a.slots_per_row <= kSpec)
    hipLaunchKernelGGL((merge_kernel<D, kSpec, false>), dim3(grid), threads, 0, stream, a);
  else
    hipLaunchKernelGGL((merge_kernel<D, kSpec, true>), dim3(grid), threads, 0, stream, a);
}

}  // namespace

hipError_t launch_merge(const StepArgs& a, int head_dim, hipStream_t stream) {
  const unsigned rows = (unsigned)a.num_seqs * (unsigned)a.num_query_tokens * (unsigned)a.num_q_heads;
  const unsigned grid = (rows + kMergeRows - 1) / kMergeRows;
  if (head_dim == 64)
    launch_d<64>(a, grid, stream);
  else if (head_dim == 128)
    launch_d<128>(a, grid, stream);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace pda
