// Split-K joint attention of one work item (Eq. (1)) of the per-phase kernels.
//
// A work item is (agent b, head h, a range of rows, a tile of 16 queries).  Per 32-row tile:
//   S^T = K Q^T on MFMA (A operand: 16 rows x 32 channels straight from memory in 16-byte loads; B operand:
//   the 16 queries, kept in registers); scores arrive in log2 units (q is pre-scaled by log2(e)/sqrt(Dh));
//   online softmax with the row max reduced over the 4 lanes sharing a query (xor 16, xor 32);
//   P (bf16/f16) is re-used in place as the A operand of O += P V: the lane's own 8 scores are rows
//   {4g..4g+3, 16+4g..16+4g+3}, and V is loaded as exactly those 8 rows x 8 channels per lane (each load
//   instruction reads 4 whole 256-byte rows) and transposed 8x8 in registers, so MFMA k (k = 0..7)
//   produces output channels 8c + k.
// fp8 rows are decoded to fp16 in registers (exact) and use fp16 MFMA; the per-(agent, layer, head) scale of the keys
// multiplies the scores, that of the values the output once the cached rows are done.
#pragma once

#include "common.h"

namespace fsx {

// 16 queries' fragments (B operand), bf16 (KT 0) or fp16 (KT 1), from the fp32 row at q (zeros where not valid).
template <int KT>
__device__ __forceinline__ void load_q_frag(const float* __restrict__ q, int64_t row, bool valid, int grp,
                                            uint4 qf[4]) {
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
    if (valid) {
      const float* p = q + row + 32 * kb + 8 * grp;
      lo = *reinterpret_cast<const float4*>(p);
      hi = *reinterpret_cast<const float4*>(p + 4);
    }
    if (KT == 0)
      qf[kb] = make_uint4(pack_bf16x2(lo.x, lo.y), pack_bf16x2(lo.z, lo.w), pack_bf16x2(hi.x, hi.y),
                          pack_bf16x2(hi.z, hi.w));
    else
      qf[kb] = make_uint4(pack_f16x2(lo.x, lo.y), pack_f16x2(lo.z, lo.w), pack_f16x2(hi.x, hi.y),
                          pack_f16x2(hi.z, hi.w));
  }
}

// 16-byte group of 8 consecutive channels of one row -> 8 x 16-bit MFMA operand values.
template <int KT>
__device__ __forceinline__ uint4 load8(const char* p) {
  if constexpr (KT == 0) {
    return *reinterpret_cast<const uint4*>(p);
  } else {
    const uint2 raw = *reinterpret_cast<const uint2*>(p);
    return make_uint4(e4m3x2_to_f16x2(raw.x, false), e4m3x2_to_f16x2(raw.x, true), e4m3x2_to_f16x2(raw.y, false),
                      e4m3x2_to_f16x2(raw.y, true));
  }
}

// Running state of 16 queries: accumulator k holds channel 8c + k of queries 4 grp + i; m (log2 units) and the lane's
// share of the sum l belong to query c.
struct AttnState {
  f32x4 o[8];
  float m, l;
};

// Adds rows [i0, i1) of one (agent, head) to the state; row i lives at base + slot(i) * row_bytes, where
// slot(i) = (start + i) mod cap for a ring and i for the new tokens' own rows.  The query of lane column c sees only
// rows i <= qmax0 + c (a causal mask among new rows; pass a large qmax0 for none).  The tiles are taken from tile `rot`
// on, wrapping around.
template <int KT, bool RING>
__device__ __forceinline__ void attn_rows(const char* __restrict__ kbase, const char* __restrict__ vbase, int64_t row_bytes,
                                          int64_t start, int64_t cap, int i0, int i1, int rot, const uint4 qf[4], float kscale,
                                          int lane, AttnState& st, int qmax0 = 1 << 30) {
  constexpr int ES = KT == 0 ? 2 : 1;
  const int c = lane & 15, grp = lane >> 4;
  const int qmax = qmax0 + c;
  auto roff = [&](int i) -> int64_t {
    int64_t slot = i;
    if (RING) {
      slot = start + i;
      if (slot >= cap) slot -= cap;
    }
    return slot * row_bytes;
  };
  const int n = (i1 - i0 + 31) / 32;
  for (int u = 0; u < n; ++u) {
    const int r0 = i0 + 32 * (u + rot < n ? u + rot : u + rot - n);
    uint4 kf[2][4];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      const int i = r0 + 16 * rt + c;
      const char* p = kbase + roff(i < i1 ? i : i0);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) kf[rt][kb] = load8<KT>(p + (32 * kb + 8 * grp) * ES);
    }
    uint4 vr[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int rr = r0 + (j < 4 ? 4 * grp + j : 16 + 4 * grp + (j - 4));
      vr[j] = load8<KT>(vbase + roff(rr < i1 ? rr : i0) + 8 * c * ES);
    }
    f32x4 s[2];
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      s[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
        s[rt] = KT == 0 ? mfma_bf16(kf[rt][kb], qf[kb], s[rt]) : mfma_f16(kf[rt][kb], qf[kb], s[rt]);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rr = r0 + 16 * rt + 4 * grp + i;
        const float v = rr < i1 && rr <= qmax ? s[rt][i] * kscale : -INFINITY;
        s[rt][i] = v;
        mx = fmaxf(mx, v);
      }
    mx = rows_max(mx);
    const float m_new = fmaxf(st.m, mx);
    const float alpha = exp2f(st.m - m_new);
    float p[8], ps = 0.f;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        p[rt * 4 + i] = exp2f(s[rt][i] - m_new);
        ps += p[rt * 4 + i];
      }
    st.l = st.l * alpha + ps;
    st.m = m_new;
    uint4 pf;
    if (KT == 0)
      pf = make_uint4(pack_bf16x2(p[0], p[1]), pack_bf16x2(p[2], p[3]), pack_bf16x2(p[4], p[5]),
                      pack_bf16x2(p[6], p[7]));
    else
      pf = make_uint4(pack_f16x2(p[0], p[1]), pack_f16x2(p[2], p[3]), pack_f16x2(p[4], p[5]), pack_f16x2(p[6], p[7]));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a_i = col_pick(alpha, grp, i);
#pragma unroll
      for (int k = 0; k < 8; ++k) st.o[k][i] *= a_i;
    }
    uint4 vt[8];
    transpose8x8_b16(vr, vt);
#pragma unroll
    for (int k = 0; k < 8; ++k) st.o[k] = KT == 0 ? mfma_bf16(pf, vt[k], st.o[k]) : mfma_f16(pf, vt[k], st.o[k]);
  }
}

}  // namespace fsx
