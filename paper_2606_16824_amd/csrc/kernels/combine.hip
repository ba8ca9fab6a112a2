// Split-K merge of extend / decode partials.
#include <hip/hip_runtime.h>

#include "../cw_internal.h"
#include "../plan_expand.h"

namespace cw {
namespace {

constexpr float kLn2 = 0.69314718055994531f;
constexpr int kFewParts = 4;  // up to this many partials per row: combine_few_kernel

// N consecutive elements of the partials' O, as they are stored (bf16 or fp32) ...
template <int N, bool F32>
struct Raw {
  typedef uint32_t words __attribute__((ext_vector_type(F32 ? N : N / 2)));
  words w = words(0u);
  __device__ __forceinline__ void load(const void* base, size_t elem) {
    w = *reinterpret_cast<const words*>(static_cast<const uint8_t*>(base) + elem * (F32 ? 4 : 2));
  }
  // ... and element e as fp32.
  __device__ __forceinline__ float operator[](int e) const {
    if constexpr (F32) return __uint_as_float(w[e]);
    else return __uint_as_float(e % 2 ? w[e / 2] & 0xFFFF0000u : w[e / 2] << 16);
  }
};

// The merge group of workgroup block `grp`.
template <int AP>
__device__ __forceinline__ CombineGroup group_of(const ExtendParams& p, const PlanArg<AP>& ap, int grp) {
  if constexpr (AP != kPlanInMemory) {
    if (p.ap_desc > 0) {  // a decode plan in compact form: the group is rebuilt (each wave searches)
      const ExpandDesc& d = *reinterpret_cast<const ExpandDesc*>(ap.bytes + p.ap_desc);
      const DecodeRec* rec = reinterpret_cast<const DecodeRec*>(ap.bytes + d.rec_off);
      const int b = wave_last_at_most(d.n_seqs, grp, static_cast<int>(threadIdx.x % 64),
                                      [&](int k) { return rec[k].group_off; });
      return expand_group_at(rec, grp, b, d.rows);
    }
  }
  return plan_ptr<AP>(ap, p.ap_groups, p.groups)[grp];
}

// Both kernels merge the split-K partials of query rows: weights 2^(m_c - max m),
// O = sum w_c O_c / sum w_c l_c, in a fixed order, no atomics.

// Few partials per row (at most kFewParts): a workgroup of 256 lanes covers 8 rows of
// 32 lanes, and every load is issued before the first use, so a row waits for one
// memory latency instead of one per partial.  Traffic bound for the extends.
template <int D, bool F32, int AP>
__global__ __launch_bounds__(256) void combine_few_kernel(ExtendParams p, PlanArg<AP> ap) {
  constexpr int ROWS = 8;
  constexpr int PER = D / 32;  // dims per lane
  const int wg_per_group = (p.part_rows + ROWS - 1) / ROWS;
  const CombineGroup cg = group_of<AP>(p, ap, blockIdx.x / wg_per_group);
  const int lr = (blockIdx.x % wg_per_group) * ROWS + threadIdx.x / 32;
  if (lr >= cg.rows) return;
  const int d0 = (threadIdx.x % 32) * PER;
  float mc[kFewParts], lc[kFewParts];
  Raw<PER, F32> oc[kFewParts];
#pragma unroll
  for (int c = 0; c < kFewParts; ++c) {
    mc[c] = -INFINITY;
    lc[c] = 0.f;
    if (c < cg.n_parts) {
      const size_t pr = size_t(cg.part0 + c) * p.part_rows + lr;
      const float2 ml = *reinterpret_cast<const float2*>(p.part_ml + pr * 2);
      mc[c] = ml.x;
      lc[c] = ml.y;
      oc[c].load(p.part_o, pr * D + d0);
    }
  }
  float m = -INFINITY, L = 0.f, acc[PER];
#pragma unroll
  for (int e = 0; e < PER; ++e) acc[e] = 0.f;
#pragma unroll
  for (int c = 0; c < kFewParts; ++c) m = fmaxf(m, mc[c]);
#pragma unroll
  for (int c = 0; c < kFewParts; ++c) {
    const float w = c < cg.n_parts ? __builtin_amdgcn_exp2f(mc[c] - m) : 0.f;
    L += w * lc[c];
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] += w * oc[c][e];
  }
  const SeqInfo sq = plan_ptr<AP>(ap, p.ap_seqs, p.seqs)[cg.seq];
  const int G = p.gqa_group, hq = p.num_kv_heads * G;
  const int r = cg.q_row0 + lr;
  const int t = r / G, g = r - t * G;
  const float inv = 1.f / L;
  uint16_t* orow = static_cast<uint16_t*>(p.out) + (size_t(sq.cu + t) * hq + size_t(cg.kvh) * G + g) * D + d0;
#pragma unroll
  for (int e = 0; e < PER; ++e) orow[e] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(acc[e] * inv));
  if (p.lse != nullptr && threadIdx.x % 32 == 0)
    p.lse[size_t(sq.cu + t) * hq + size_t(cg.kvh) * G + g] = (m + log2f(L)) * kLn2;
}

// Many partials per row (decodes of long prefixes): a workgroup per row.  Few rows
// and a chain of latencies, so every slice of D / 8 lanes (16 bytes of a partial each)
// issues the loads of kBatch partials at once: with 8, up to 128 partials (256 at D =
// 64) in one round, with 4 half as many but fewer empty loads.  The slices are then
// merged through LDS, one dim per lane.  Step times, before with four partials of 8
// bytes per lane in flight in slices of 32 lanes: a decode of 131072 keys (64 rows of
// 94 partials) 94.5 -> 89.4 us; of 1700 keys (32 rows of 27) 11.9 -> 10.2 us of GPU
// time; 48 decodes over fp8 pages (1536 rows of up to 33) 277.5 -> 277.0 us, with
// batches of 8 278.2.
template <int D, int kBatch, bool F32, int AP>
__global__ __launch_bounds__(256) void combine_many_kernel(ExtendParams p, PlanArg<AP> ap) {
  constexpr int LANES = D / 8, SLICES = 256 / LANES;
  __shared__ float sh_o[SLICES][D];
  __shared__ float sh_m[SLICES], sh_l[SLICES];
  const CombineGroup cg = group_of<AP>(p, ap, blockIdx.x / p.part_rows);
  const int lr = blockIdx.x % p.part_rows;
  if (lr >= cg.rows) return;  // (uniform)
  const int slice = threadIdx.x / LANES, d0 = (threadIdx.x % LANES) * 8;
  float m = -INFINITY, L = 0.f, acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
  for (int c0 = slice; c0 < cg.n_parts; c0 += kBatch * SLICES) {
    float2 ml[kBatch];
    Raw<8, F32> oc[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int c = c0 + k * SLICES;
      ml[k] = make_float2(-INFINITY, 0.f);
      if (c < cg.n_parts) {
        const size_t pr = size_t(cg.part0 + c) * p.part_rows + lr;
        ml[k] = *reinterpret_cast<const float2*>(p.part_ml + pr * 2);
        oc[k].load(p.part_o, pr * D + d0);
      }
    }
    float m_new = m;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) m_new = fmaxf(m_new, ml[k].x);
    const float a = __builtin_amdgcn_exp2f(m - m_new);
    L *= a;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= a;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const float w = c0 + k * SLICES < cg.n_parts ? __builtin_amdgcn_exp2f(ml[k].x - m_new) : 0.f;
      L += w * ml[k].y;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += w * oc[k][e];
    }
    m = m_new;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) sh_o[slice][d0 + e] = acc[e];
  if (threadIdx.x % LANES == 0) {
    sh_m[slice] = m;
    sh_l[slice] = L;
  }
  __syncthreads();
  const int d = threadIdx.x;
  if (d >= D) return;
  float mstar = -INFINITY;
#pragma unroll
  for (int s = 0; s < SLICES; ++s) mstar = fmaxf(mstar, sh_m[s]);
  float Lt = 0.f, out = 0.f;
#pragma unroll
  for (int s = 0; s < SLICES; ++s) {
    const float w = sh_m[s] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(sh_m[s] - mstar);
    Lt += w * sh_l[s];
    out += w * sh_o[s][d];
  }
  const SeqInfo sq = plan_ptr<AP>(ap, p.ap_seqs, p.seqs)[cg.seq];
  const int G = p.gqa_group, hq = p.num_kv_heads * G;
  const int r = cg.q_row0 + lr;
  const int t = r / G, g = r - t * G;
  const size_t row = size_t(sq.cu + t) * hq + size_t(cg.kvh) * G + g;
  static_cast<uint16_t*>(p.out)[row * D + d] = __builtin_bit_cast(uint16_t, static_cast<__bf16>(out / Lt));
  if (p.lse != nullptr && d == 0) p.lse[row] = (mstar + log2f(Lt)) * kLn2;
}

}  // namespace

hipError_t launch_combine(const ExtendParams& p, int head_dim, int max_parts, hipStream_t stream,
                          const ArgPlanBuf* ap) {
  if (p.n_groups <= 0) return hipSuccess;
  const bool many = max_parts > kFewParts;
  const int rows_per_wg = many ? 1 : 8;
  const dim3 grid(p.n_groups * ((p.part_rows + rows_per_wg - 1) / rows_per_wg));
#define CW_COMBINE_AP(K_, ...)                                                                         \
  do {                                                                                                 \
    if (ap && ap->small())                                                                             \
      hipLaunchKernelGGL((K_<__VA_ARGS__, kPlanInSmallArgs>), grid, dim3(256), 0, stream, p, ap->small_plan()); \
    else if (ap)                                                                                       \
      hipLaunchKernelGGL((K_<__VA_ARGS__, kPlanInArgs>), grid, dim3(256), 0, stream, p, ap->plan);              \
    else                                                                                               \
      hipLaunchKernelGGL((K_<__VA_ARGS__, kPlanInMemory>), grid, dim3(256), 0, stream, p, NoArgPlan{});         \
  } while (0)
#define CW_COMBINE(K_, ...)                                  \
  do {                                                       \
    if (p.part_f32) CW_COMBINE_AP(K_, __VA_ARGS__, true);    \
    else CW_COMBINE_AP(K_, __VA_ARGS__, false);              \
  } while (0)
  if (head_dim == 64) {
    if (max_parts > 128) CW_COMBINE(combine_many_kernel, 64, 8);
    else if (many) CW_COMBINE(combine_many_kernel, 64, 4);
    else CW_COMBINE(combine_few_kernel, 64);
  } else if (head_dim == 128) {
    if (max_parts > 64) CW_COMBINE(combine_many_kernel, 128, 8);
    else if (many) CW_COMBINE(combine_many_kernel, 128, 4);
    else CW_COMBINE(combine_few_kernel, 128);
  } else {
    return hipErrorInvalidValue;
  }
#undef CW_COMBINE
#undef CW_COMBINE_AP
  return hipGetLastError();
}

}  // namespace cw
