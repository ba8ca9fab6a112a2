// Scatter of one 16-byte piece of a new K/V row into its page-pool slot (bf16
// copy, or fp8 quantise-on-write with the page's scale), shared by the
// stand-alone page-write kernel and the fused writes of the extend and decode
// kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "../cw_internal.h"

namespace cw {
namespace pw {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Eight bf16 -> eight e4m3fn codes of clamp(x / s, -448, 448), nearest-even, the
// quotient an IEEE fp32 division.  The scale is the same for all eight, so its
// reciprocal r is divided out once and each quotient is x r, corrected once with
// the remainder of a fused multiply-add (Markstein): five operations per element
// against about fourteen of a division each.
//  The codes are those of the division.  The corrected quotient is RN(x / s (1 +
// d)) with |d| <= 2^-46, so it differs from RN(x / s) only where x / s lies that close
// to the midpoint of two fp32 numbers, and then matters only where one of them is a
// tie of the code, a number C of 5 significant bits.  With S and X the integer
// significands of s (24 bits) and x (8 bits), that is |S (C 2^20 +- 1) - X 2^j| <= 32:
// then S = a 2^20 + t with |t| <= 32, a <= 15, and t C +- a = 0, which C >= 16 rules out.
//  The first quotient is clamped to +-1024 (whose code is that of +-448), so the
// remainder of a huge x is its own size and the corrected quotient infinite at most;
// a NaN ends as -448, as from the division; quotients small enough for a
// remainder to underflow have the code of zero; and -0 keeps its sign (its remainder
// enters as -0).  Scales outside [2^-60, 2^60] take the division.
__device__ __forceinline__ u32x2 quantise8(u32x4 x, float s) {
  u32x2 out;
  float f[8];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    f[2 * e] = __uint_as_float(x[e] << 16);
    f[2 * e + 1] = __uint_as_float(x[e] & 0xFFFF0000u);
  }
  if (s >= 0x1p-60f && s <= 0x1p60f) {
    const float r = __fdiv_rn(1.f, s);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float q = __builtin_amdgcn_fmed3f(f[e] * r, -1024.f, 1024.f);
      f[e] = __builtin_amdgcn_fmed3f(fmaf(-fmaf(s, q, -f[e]), r, q), -448.f, 448.f);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = fminf(fmaxf(__fdiv_rn(f[e], s), -448.f), 448.f);
  }
#pragma unroll
  for (int w = 0; w < 2; ++w) {
    int packed = __builtin_amdgcn_cvt_pk_fp8_f32(f[4 * w], f[4 * w + 1], 0, false);
    packed = __builtin_amdgcn_cvt_pk_fp8_f32(f[4 * w + 2], f[4 * w + 3], packed, true);
    out[w] = static_cast<uint32_t>(packed);
  }
  return out;
}

template <bool NT, class T>
__device__ __forceinline__ void put(T* dst, T x) {
  if constexpr (NT) __builtin_nontemporal_store(x, dst);
  else *dst = x;
}

// One piece, read already, into slot `slot` of physical page `pg`; fp8 pools
// quantise with the page's scales ks, vs.  NT: stores with the nontemporal hint.
template <int D, int P, bool FP8, bool NT>
__device__ __forceinline__ void put_piece(const WriteParams& p, u32x4 kx, u32x4 vx, int h, int c8, int pg,
                                          int slot, float ks, float vs) {
  const size_t dst = ((size_t(pg) * p.num_kv_heads + h) * P + slot) * D + c8 * 8;
  if constexpr (FP8) {
    put<NT>(reinterpret_cast<u32x2*>(static_cast<uint8_t*>(p.k_pool) + dst), quantise8(kx, ks));
    put<NT>(reinterpret_cast<u32x2*>(static_cast<uint8_t*>(p.v_pool) + dst), quantise8(vx, vs));
  } else {
    put<NT>(reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.k_pool) + dst), kx);
    put<NT>(reinterpret_cast<u32x4*>(static_cast<uint16_t*>(p.v_pool) + dst), vx);
  }
}

// Elements c8 * 8 .. c8 * 8 + 7 of K and V of new row (tok, kv head h) into slot
// `slot` of physical page `pg`; fp8 pools quantise with the page's scales ks, vs.
template <int D, int P, bool FP8>
__device__ __forceinline__ void store_piece(const WriteParams& p, int tok, int h, int c8, int pg,
                                            int slot, float ks, float vs) {
  const int hkv = p.num_kv_heads;
  const size_t src = (size_t(tok) * hkv + h) * D + c8 * 8;
  const u32x4 kx = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(p.k_new) + src);
  const u32x4 vx = *reinterpret_cast<const u32x4*>(static_cast<const uint16_t*>(p.v_new) + src);
  put_piece<D, P, FP8, false>(p, kx, vx, h, c8, pg, slot, ks, vs);
}

// Piece `idx` of the flat [token, kv head, D / 8] order: the 8 elements
// c8 * 8 .. c8 * 8 + 7 of K and of V for (token, kv head) go to slot
// (Lp + i) % P of page block_table[b][(Lp + i) / P], where token = cu_b + i.
template <int D, int P, bool FP8>
__device__ __forceinline__ void write_piece(const WriteParams& p, int64_t idx) {
  constexpr int CH = D / 8;  // 8-element pieces per row
  const int hkv = p.num_kv_heads;
  const int c8 = static_cast<int>(idx % CH);
  const int64_t rest = idx / CH;
  const int h = static_cast<int>(rest % hkv);
  const int tok = static_cast<int>(rest / hkv);
  // sequence owning this token: the last one whose first row is <= tok
  int lo = 0, hi = p.num_seqs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (p.seqs[mid].cu <= tok) lo = mid;
    else hi = mid - 1;
  }
  const SeqInfo sq = p.seqs[lo];
  const int pos = sq.lp + (tok - sq.cu);
  const int pg = p.block_table[size_t(sq.bt_row) * p.bt_stride + pos / P];
  if constexpr (FP8) {
    const size_t si = size_t(pg) * hkv + h;
    store_piece<D, P, FP8>(p, tok, h, c8, pg, pos % P, p.k_scale[si], p.v_scale[si]);
  } else {
    store_piece<D, P, FP8>(p, tok, h, c8, pg, pos % P, 1.f, 1.f);
  }
}

}  // namespace pw
}  // namespace cw
