// What the bf16 MFMA kernels share: operand types, row exchanges, the tile order of the projections and a step of attention.
#pragma once
#include "vvs_device.h"

namespace vvs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // 16 bytes as a native vector (plain register moves)

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

// Maximum / sum over the four lanes l % 16 + 16 j of a wave (the four 16-lane rows), left in all four, with gfx950's row
// swaps: v_permlane16_swap exchanges the odd rows of its first operand with the even rows of its second, v_permlane32_swap
// the upper half of the first with the lower half of the second - given the same value twice they return (x of the
// even / lower partner, x of the odd / upper partner) in every lane.  Plain VALU instructions: the LDS crossbar that a
// __shfl_xor goes through costs a round trip per step of these dependent chains.  Same order of additions as
// x += xor16(x); x += xor32(x).
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float rows_max(float x) {
  uintx2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
  p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
__device__ __forceinline__ float rows_sum(float x) {
  uintx2 p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Tile order of the projection launches.  Workgroups are dealt to the 8 XCDs round-robin by linear id, and each XCD has its own
// L2.  Column tiles are taken in groups of 8 (one per XCD); inside a group the row tiles of one column tile get ids 8 apart:
// they run at the same time on the same XCD, so a weight tile is fetched from memory once and then hits in that XCD's L2.  A
// last group of fewer columns is dealt over all XCDs.
__device__ __forceinline__ void tile_of(int id, int MT, int NT, int* tile_m, int* tile_n) {
  const int grp = id / (8 * MT), rem = id % (8 * MT), cols = min(8, NT - grp * 8);
  *tile_m = rem / cols;
  *tile_n = grp * 8 + rem % cols;
}

// K and V of 32-key step STEP of the head whose caches start at kb and vb, into the operand registers of lane `lane`
#define VVS_ATTN_LOAD(STEP, KF, VF)                                                                                   \
  {                                                                                                                   \
    _Pragma("unroll") for (int t = 0; t < 2; ++t)                                                                     \
        _Pragma("unroll") for (int kd = 0; kd < KD; ++kd)                                                             \
            KF[t][kd] = as_bf16x8(*(const uint4*)(kb + ((((size_t)(STEP) * 2 + t) * KD + kd) * 64 + lane) * 8));      \
    _Pragma("unroll") for (int dt = 0; dt < DT; ++dt)                                                                 \
        VF[dt] = as_bf16x8(*(const uint4*)(vb + (((size_t)(STEP) * DT + dt) * 64 + lane) * 8));                       \
  }

// One 32-key step of the attention kernels for NQB blocks of 16 queries: scores S^T = K Q^T (lane = query l % 16, key
// group g = l / 16, 8 consecutive keys per lane), online softmax, O^T += V^T P^T.  The tree mask only touches a step that
// reaches past the cached length S (tail).
// The softmax weights are not rounded to bf16 (the definition keeps them exact): each un-normalised weight e goes into the
// P V product as the sum of two bf16 values, hi = bf16(e) and lo = bf16(e - hi) (e to 2^-17), with two MFMAs per V block -
// the matrix cores idle in these kernels anyway - and the normaliser sums the fp32 weights themselves.
template <int NQB, int KD, int DT>
__device__ __forceinline__ void attn_step(const bf16x8 (&kf)[2][KD], const bf16x8 (&vf)[DT], const bf16x8 (&qf)[NQB][KD],
                                          const uint64_t (&mask)[NQB], float (&m_run)[NQB], float (&l_run)[NQB], floatx4 (&o)[NQB][DT],
                                          int key0, int S, int n_keys, bool tail, int g, float c_exp) {
#pragma unroll
  for (int qb = 0; qb < NQB; ++qb) {
    floatx4 s2[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      s2[t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kd = 0; kd < KD; ++kd) s2[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][kd], qf[qb][kd], s2[t], 0, 0, 0);
    }
    float sv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) sv[i] = s2[i >> 2][i & 3];
    if (tail) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int key = key0 + 8 * g + i;
        bool vis = key < S;
        if (!vis && key < n_keys) vis = (mask[qb] >> (key - S)) & 1ull;
        if (!vis) sv[i] = -INFINITY;
      }
    }
    float mx = sv[0];
#pragma unroll
    for (int i = 1; i < 8; ++i) mx = fmaxf(mx, sv[i]);
    mx = rows_max(mx);
    const float m_new = fmaxf(m_run[qb], mx);
    const float m_safe = m_new == -INFINITY ? 0.f : m_new;
    const float alpha = __builtin_amdgcn_exp2f((m_run[qb] - m_safe) * c_exp);
    const float mc = m_safe * c_exp;
    uint32_t pk[4], pl[4];
    float rs = 0.f;
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
      // hardware exp2 (arguments <= 0 up to the rounding of the fused multiply-add)
      const float e0 = __builtin_amdgcn_exp2f(fmaf(sv[i], c_exp, -mc)), e1 = __builtin_amdgcn_exp2f(fmaf(sv[i + 1], c_exp, -mc));
      const uint32_t pp = pack2bf(e0, e1);
      rs += e0 + e1;
      pk[i >> 1] = pp;
      pl[i >> 1] = pack2bf(e0 - __uint_as_float(pp << 16), e1 - __uint_as_float(pp & 0xFFFF0000u));
    }
    rs = rows_sum(rs);
    l_run[qb] = l_run[qb] * alpha + rs;
    m_run[qb] = m_new;
    const bf16x8 pf = as_bf16x8(make_uint4(pk[0], pk[1], pk[2], pk[3]));
    const bf16x8 pfl = as_bf16x8(make_uint4(pl[0], pl[1], pl[2], pl[3]));
    // the running maximum rarely moves after the first steps: the accumulators are only rescaled when some query's did
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) o[qb][dt][rr] *= alpha;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      o[qb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pf, o[qb][dt], 0, 0, 0);
      o[qb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pfl, o[qb][dt], 0, 0, 0);
    }
  }
}

}  // namespace vvs
