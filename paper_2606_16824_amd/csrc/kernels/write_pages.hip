// Scatter of new K/V rows into their page-pool slots (bf16 copy or fp8
// quantise-on-write).
//
// Bound by memory: k_new / v_new are read once and the pool rows written once, in
// contiguous 16-byte pieces (8 elements of one (token, kv head) row of K and of V).
// What held it back was not the bytes but the way to them: each piece searched its
// sequence, then its page, then its scales, one dependent load after the other, and
// quantised with a division per element.  So a wave takes kPieces * 64 consecutive
// pieces: it issues all its K/V loads first, finds the sequence of its first token
// once (64 sequences per load and ballot) and steps on from there, and reads page
// ids and scales of all its pieces together.  The pool rows are stored with the
// nontemporal hint: they are whole lines that nothing reads before the next step.
// 27408 tokens of 12 sequences, 8 kv heads of 128, call time with the new K/V in
// the memory-side cache: fp8 pages (168 MB) 54.8 us before, 47.3 with the above,
// 42.0 with the sequences in the kernel arguments, 34.6 with nontemporal stores
// (from HBM 55.0 -> 38.0 us, 4.4 TB/s; a plain copy reaches 4.7); bf16 pages 48.8
// -> 34.3 us.  2 pieces per lane: 42.0, 4: 42.6, 8: 44.6 us (fewer waves to hide the
// latencies).  Nontemporal loads cost 4 us: the new K/V have just been written.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "../cw_internal.h"
#include "../plan_expand.h"
#include "page_write.h"

namespace cw {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kPieces = 2;  // 16-byte pieces of K and of V per lane and pass
constexpr int kThreads = 256;
constexpr int kWavePieces = 64 * kPieces;

template <int D, int P, bool FP8, int AP>
__global__ __launch_bounds__(kThreads) void write_pages_kernel(WriteParams p, PlanArg<AP> ap) {
  constexpr int CH = D / 8;  // pieces per (token, kv head) row
  const SeqInfo* seqs = plan_ptr<AP>(ap, 0, p.seqs);
  const int hkv = p.num_kv_heads;
  const uint32_t row = static_cast<uint32_t>(hkv) * CH;  // pieces per token
  const float inv_row = 1.f / static_cast<float>(row);
  const int64_t total = int64_t(p.total_tokens) * row;
  const int lane = threadIdx.x % 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const u32x4* k_new = static_cast<const u32x4*>(p.k_new);
  const u32x4* v_new = static_cast<const u32x4*>(p.v_new);
  const int64_t stride = int64_t(gridDim.x) * (kThreads / 64) * kWavePieces;
  for (int64_t base = (int64_t(blockIdx.x) * (kThreads / 64) + wave) * kWavePieces; base < total; base += stride) {
    u32x4 kx[kPieces], vx[kPieces];
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      const int64_t idx = base + 64 * u + lane;
      if (idx < total) {
        kx[u] = k_new[idx];
        vx[u] = v_new[idx];
      }
    }
    const int tok0 = static_cast<int>(base / row);
    const uint32_t rem = static_cast<uint32_t>(base - int64_t(tok0) * row);
    // sequence owning the wave's first token: the last one whose first row is <= it
    const int s0 = wave_last_at_most(p.num_seqs, tok0, lane, [&](int k) { return seqs[k].cu; });
    int h[kPieces], c8[kPieces], slot[kPieces], pg[kPieces];
    float ks[kPieces], vs[kPieces];
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      // rem + the lane's pieces < 2^15, so the fp32 quotient's floor is exact
      const uint32_t r = rem + 64 * u + lane;
      const uint32_t dt = static_cast<uint32_t>((static_cast<float>(r) + 0.5f) * inv_row);
      const uint32_t in_row = r - dt * row;
      const int tok = min(tok0 + static_cast<int>(dt), p.total_tokens - 1);  // (idle lanes: any valid token)
      h[u] = static_cast<int>(in_row / CH);
      c8[u] = static_cast<int>(in_row % CH);
      int s = s0;
      while (s + 1 < p.num_seqs && seqs[s + 1].cu <= tok) ++s;
      const SeqInfo sq = seqs[s];
      const int pos = sq.lp + (tok - sq.cu);
      slot[u] = pos % P;
      pg[u] = p.block_table[size_t(sq.bt_row) * p.bt_stride + pos / P];
    }
#pragma unroll
    for (int u = 0; u < kPieces; ++u) {
      ks[u] = vs[u] = 1.f;
      if constexpr (FP8) {
        const size_t si = size_t(pg[u]) * hkv + h[u];
        ks[u] = p.k_scale[si];
        vs[u] = p.v_scale[si];
      }
    }
#pragma unroll
    for (int u = 0; u < kPieces; ++u)
      if (base + 64 * u + lane < total)
        pw::put_piece<D, P, FP8, true>(p, kx[u], vx[u], h[u], c8[u], pg[u], slot[u], ks[u], vs[u]);
  }
}

template <int D, int P, bool FP8>
hipError_t launch_t(const WriteParams& p, hipStream_t stream, const ArgPlanBuf* ap) {
  const int64_t total = int64_t(p.total_tokens) * p.num_kv_heads * (D / 8);
  constexpr int kBlockPieces = kThreads / 64 * kWavePieces;
  const int64_t blocks = std::min<int64_t>((total + kBlockPieces - 1) / kBlockPieces, 65536);
  const dim3 grid(static_cast<unsigned>(blocks));
  if (ap != nullptr && ap->small())
    hipLaunchKernelGGL((write_pages_kernel<D, P, FP8, kPlanInSmallArgs>), grid, dim3(kThreads), 0, stream, p,
                       ap->small_plan());
  else if (ap != nullptr)
    hipLaunchKernelGGL((write_pages_kernel<D, P, FP8, kPlanInArgs>), grid, dim3(kThreads), 0, stream, p, ap->plan);
  else
    hipLaunchKernelGGL((write_pages_kernel<D, P, FP8, kPlanInMemory>), grid, dim3(kThreads), 0, stream, p,
                       NoArgPlan{});
  return hipGetLastError();
}

}  // namespace

hipError_t launch_write_pages(const WriteParams& p, int head_dim, int page_size, bool fp8,
                              hipStream_t stream, const ArgPlanBuf* ap) {
  if (p.total_tokens <= 0) return hipSuccess;
#define CW_CASE(D_, P_)                                                                          \
  if (head_dim == D_ && page_size == P_)                                                         \
    return fp8 ? launch_t<D_, P_, true>(p, stream, ap) : launch_t<D_, P_, false>(p, stream, ap);
  CW_CASE(64, 16)
  CW_CASE(64, 64)
  CW_CASE(128, 16)
  CW_CASE(128, 64)
#undef CW_CASE
  return hipErrorInvalidValue;
}

}  // namespace cw
