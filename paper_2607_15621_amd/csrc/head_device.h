// The paper's waypoint head (Sec. 3.1): the last n_queries expert tokens are learnable waypoint queries, each
// decoded to one (x, y) waypoint by a two-layer head -- final RMSNorm, Linear(d -> hidden) + bias, GELU (exact erf
// form), Linear(hidden -> 2) + bias.  Shared by the persistent tick kernel (which reads its tile-major residual and
// splits an agent's hidden units over workgroups) and the per-op paths (row-major residual, one workgroup per agent).
#pragma once

#include "common.h"

namespace fsx {

constexpr int QH_MAX_QUERIES = 8;

struct QueryHead {
  const void* w1;   // [hidden][d] (wdtype)
  const float* b1;  // [hidden]
  const void* w2;   // [2][hidden] (wdtype)
  const float* b2;  // [2]
  int hidden;
  int wdtype;       // FSX_F32 or FSX_BF16
};

__device__ __forceinline__ float qh_weight(const void* w, int wdtype, int64_t i) {
  return wdtype == FSX_BF16 ? bf16_to_f32(reinterpret_cast<const uint16_t*>(w)[i]) : reinterpret_cast<const float*>(w)[i];
}

// The mean-pool head of one agent of the per-op paths (blockIdx.x; residual h [M][d], S rows per agent): W_head times the
// mean over the first T tokens of RMSNorm(h) * g_final.  xm: d floats of LDS; 256 threads.  A token's scale is one wave's
// work (one workgroup-wide sum per token after another took 22 us at T = 10, d = 512, now 14).
__device__ __forceinline__ void mean_head_wg(const float* __restrict__ h, int S, int T, int d, float eps,
                                             const float* __restrict__ gfin, const void* __restrict__ w, int wdtype, int n_out,
                                             float* __restrict__ wp, float* xm) {
  constexpr int TB = 16;
  __shared__ float rs[TB];
  const int b = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float* hb = h + (int64_t)b * S * d;
  for (int t0 = 0; t0 < T; t0 += TB) {
    for (int t = t0 + wave; t < min(t0 + TB, T); t += 4) {
      const float* hr = hb + (int64_t)t * d;
      float ss = 0.f;
#pragma unroll 8
      for (int n = lane; n < d; n += WAVE) ss += hr[n] * hr[n];
      ss = wave_sum(ss);
      if (lane == 0) rs[t - t0] = 1.0f / sqrtf(ss / (float)d + eps);
    }
    __syncthreads();
    for (int n = threadIdx.x; n < d; n += blockDim.x) {
      const float gn = gfin[n];
      float acc = t0 ? xm[n] : 0.f;
#pragma unroll 5
      for (int t = t0; t < min(t0 + TB, T); ++t) acc += hb[(int64_t)t * d + n] * rs[t - t0] * gn;
      xm[n] = acc;
    }
    __syncthreads();
  }
  for (int o = wave; o < n_out; o += 4) {
    float acc = 0.f;
#pragma unroll 8
    for (int n = lane; n < d; n += WAVE) acc += xm[n] * qh_weight(w, wdtype, (int64_t)o * d + n);
    acc = wave_sum(acc);
    if (lane == 0) wp[(int64_t)b * n_out + o] = acc / (float)T;
  }
}

// Hidden units [64 g0, 64 g1) (groups of 64; units past `hidden` count nothing) of one agent's head, summed into the
// 2 nq outputs without b2: emit(q, c, v) is called by lane 0 of a wave for every query q and coordinate c.
// row(t, col): residual of expert token t (0 <= t < T), column col.  lds: nq * (d + 256) floats.  `ready()` runs after
// the first group's weights have been issued and before the rows are read (the tick kernel's wait for its last layer);
// false makes the call return without emitting.  Ends with a barrier; every thread of the 256 must call it.
//
// Lane l of every wave owns unit 64 g + l and the four waves split the columns, so a unit's dot products need no
// cross-lane sums: a lane loads its quarter of the unit's W1 row (16 loads of 16 bytes at d = 512, all issued at
// once) and multiplies it by the normalised query rows, which LDS broadcasts.  The earlier form (one wave per unit,
// one 2-byte load per lane and step, a 64-lane sum per query) was a chain of 128 load latencies per wave: 840 us per
// tick at hidden 512 (4 agents) against the mean-pool head's 10.
template <typename Row, typename Ready, typename Emit>
__device__ void query_head_part(Row row, int T, int nq, int d, float eps, const float* __restrict__ gfin,
                                const QueryHead& qh, int g0, int g1, Ready ready, Emit emit, float* lds) {
  constexpr int CH = 16;  // 16-byte chunks of W1 a lane holds: 128 columns
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int hid = qh.hidden;
  float* x = lds;              // [nq][d] normalised query rows
  float* part = lds + nq * d;  // [4 waves][nq][64 units] partial dot products
  const bool vec = qh.wdtype == FSX_BF16 && d % 32 == 0;  // whole 16-byte chunks in every wave's columns
  const int cq = vec ? d / 4 : (d + 3) / 4, c0 = wave * cq, c1 = min(d, c0 + cq);
  uint4 w[CH];
  auto load_w = [&](int g, int cb) {
    const int j = min(64 * g + lane, hid - 1);
    const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(qh.w1) + (int64_t)j * d + cb);
#pragma unroll
    for (int i = 0; i < CH; ++i) w[i] = cb + 8 * i < c1 ? ld_global(p + i) : make_uint4(0, 0, 0, 0);
  };
  if (vec && g0 < g1) load_w(g0, c0);
  if (!ready()) return;
  for (int q = wave; q < nq; q += 4) {
    float ss = 0.f;
    for (int cb = 0; cb < d; cb += 8 * WAVE) {  // eight columns per lane at a time, every load issued before any is used
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = cb + i * WAVE + lane;
        v[i] = row(T - nq + q, c < d ? c : d - 1);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = cb + i * WAVE + lane;
        if (c < d) {
          x[q * d + c] = v[i];
          ss += v[i] * v[i];
        }
      }
    }
    const float r = 1.0f / sqrtf(wave_sum(ss) / (float)d + eps);
    for (int c = lane; c < d; c += WAVE) x[q * d + c] *= r * gfin[c];  // this wave's own stores
  }
  __syncthreads();
  float osum[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
  for (int g = g0; g < g1; ++g) {
    const int j = 64 * g + lane, jj = min(j, hid - 1);
    const float b1 = qh.b1[jj], wx = qh_weight(qh.w2, qh.wdtype, jj), wy = qh_weight(qh.w2, qh.wdtype, (int64_t)hid + jj);
    float acc[QH_MAX_QUERIES];
#pragma unroll
    for (int q = 0; q < QH_MAX_QUERIES; ++q) acc[q] = 0.f;
    if (vec) {
      for (int cb = c0; cb < c1; cb += 8 * CH) {
        if (g != g0 || cb != c0) load_w(g, cb);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          if (cb + 8 * i < c1) {
            const uint32_t u[4] = {w[i].x, w[i].y, w[i].z, w[i].w};
            float wf[8];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              wf[2 * e] = __uint_as_float(u[e] << 16);
              wf[2 * e + 1] = __uint_as_float(u[e] & 0xFFFF0000u);
            }
#pragma unroll
            for (int q = 0; q < QH_MAX_QUERIES; ++q)
              if (q < nq) {
                const float4* xq = reinterpret_cast<const float4*>(x + q * d + cb + 8 * i);
                const float4 a = xq[0], b = xq[1];
                acc[q] += wf[0] * a.x + wf[1] * a.y + wf[2] * a.z + wf[3] * a.w + wf[4] * b.x + wf[5] * b.y +
                          wf[6] * b.z + wf[7] * b.w;
              }
          }
        }
      }
    } else {
      for (int c = c0; c < c1; ++c) {
        const float wv = qh_weight(qh.w1, qh.wdtype, (int64_t)jj * d + c);
#pragma unroll
        for (int q = 0; q < QH_MAX_QUERIES; ++q)
          if (q < nq) acc[q] += wv * x[q * d + c];
      }
    }
#pragma unroll
    for (int q = 0; q < QH_MAX_QUERIES; ++q)
      if (q < nq) part[(wave * nq + q) * 64 + lane] = acc[q];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int q = wave + 4 * i;
      if (q < nq) {
        const float u = part[q * 64 + lane] + part[(nq + q) * 64 + lane] + part[(2 * nq + q) * 64 + lane] +
                        part[(3 * nq + q) * 64 + lane] + b1;
        const float a = j < hid ? 0.5f * u * (1.0f + erff(u * 0.70710678118654752f)) : 0.f;
        osum[i][0] += a * wx;
        osum[i][1] += a * wy;
      }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = wave + 4 * i;
    if (q < nq) {
      const float vx = wave_sum(osum[i][0]), vy = wave_sum(osum[i][1]);
      if (lane == 0) {
        emit(q, 0, vx);
        emit(q, 1, vy);
      }
    }
  }
  __syncthreads();
}

// The whole head of one agent on one workgroup: out(o, v) stores output o = 2q + {0: x, 1: y}.
template <typename Row, typename Out>
__device__ void query_head_wg(Row row, int T, int nq, int d, float eps, const float* __restrict__ gfin,
                              const QueryHead& qh, Out out, float* lds) {
  query_head_part(row, T, nq, d, eps, gfin, qh, 0, (qh.hidden + 63) / 64, [] { return true; },
                  [&](int q, int c, float v) { out(2 * q + c, v + qh.b2[c]); }, lds);
}

}  // namespace fsx
