// Per-op kernels of the expert tick (Sec. 3.1, Eq. (1)) for any shape and for fp32 weights.  Every value is computed in
// fp32; these kernels serve the fp32 expert (whose tolerance needs fp32 arithmetic end to end) and shapes the fused bf16
// path does not cover.  Same readings as the fused path: pre-norm RMSNorm, rotary pairs (j, j + Dh/2), scale 1/sqrt(Dh),
// SwiGLU, mean-pool head.
//
// Such experts are small, so a tick is bound by the number of launches (about 4 us each) and by the longest chain of
// dependent loads in one: five launches per layer (norm + q/k/v + rotary, attention, O + residual, norm + gate/up +
// SwiGLU, down + residual), each of whose sums is split over the lanes of a wave.  With one thread per output and 14
// launches per layer the smallest expert (2 layers, width 64, one agent over 40 rows) took 1,547 us, of which 1,270 were
// the attention's 50 dependent rows per thread; now 64 us.

#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace fsx {

__device__ __forceinline__ float ld(const void* p, int dtype, int64_t i) {
  if (dtype == FSX_BF16) return bf16_to_f32(((const uint16_t*)p)[i]);
  if (dtype == FSX_FP8_E4M3) return e4m3_to_f32(((const uint8_t*)p)[i]);
  return ((const float*)p)[i];
}

__global__ void g_embed(const void* tokens, int dtype, TickParams tp, Dims dm, GenericWorkspace ws) {
  const int m = blockIdx.x;
  const int b = m / tp.S, t = m % tp.S;
  for (int n = threadIdx.x; n < dm.d; n += blockDim.x) ws.h[(int64_t)m * dm.d + n] = ld(tokens, dtype, (int64_t)m * dm.d + n);
  const int half = dm.Dh / 2;
  for (int j = threadIdx.x; j < half; j += blockDim.x) {
    double cs = 1.0, sn = 0.0;
    if (dm.rope_base > 0.f) {
      const double ang = (double)(tp.pos[b] + t) * pow((double)dm.rope_base, -2.0 * (double)j / (double)dm.Dh);
      cs = cos(ang);
      sn = sin(ang);
    }
    ws.rope[((int64_t)m * half + j) * 2] = (float)cs;
    ws.rope[((int64_t)m * half + j) * 2 + 1] = (float)sn;
  }
}

// Four consecutive elements (16, 8 or 4 bytes, aligned to that), or one.
template <int DT>
__device__ __forceinline__ float4 ld4(const void* p, int64_t i) {
  if constexpr (DT == FSX_F32) {
    return *reinterpret_cast<const float4*>((const float*)p + i);
  } else if constexpr (DT == FSX_BF16) {
    const uint2 v = *reinterpret_cast<const uint2*>((const uint16_t*)p + i);
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                       __uint_as_float(v.y & 0xFFFF0000u));
  } else {
    const uint32_t v = *reinterpret_cast<const uint32_t*>((const uint8_t*)p + i);
    const f16x2 lo = __builtin_bit_cast(f16x2, e4m3x2_to_f16x2(v, false)), hi = __builtin_bit_cast(f16x2, e4m3x2_to_f16x2(v, true));
    return make_float4((float)lo[0], (float)lo[1], (float)hi[0], (float)hi[1]);
  }
}
// VW = 4 or 1 elements in the first places of a float4.
template <int DT, int VW>
__device__ __forceinline__ float4 ldv(const void* p, int64_t i) {
  if constexpr (VW == 4)
    return ld4<DT>(p, i);
  else
    return make_float4(ld(p, DT, i), 0.f, 0.f, 0.f);
}

enum { GEPI_QKV = 0, GEPI_SWIGLU = 1, GEPI_RESIDUAL = 2 };
constexpr int64_t GRID_MAX = 1 << 22;  // workgroups of a launch; they loop over what is beyond
constexpr int PR_ROWS = 8;   // rows of a projection workgroup
constexpr int PR_KC = 512;   // columns of x staged at a time

struct ProjArgs {
  const float* x;      // [M][K]
  const float* gain;   // RMSNorm of x with this gain first (null: x as it is)
  const void* w[3];    // QKV: wq, wk, wv; SWIGLU: gate, up; RESIDUAL: w[0]
  float* out[3];       // QKV: q, k, v [M][A]; SWIGLU: [M][N]; RESIDUAL: h [M][N], added to
  float* hidden;       // RESIDUAL: a copy of the new h (optional)
  const float* rope;   // [M][Dh/2][2]
  int M, N, K;         // N: columns of one output
  int A, Dh;
  float eps;
};

// out = epilogue(norm(x) W^T).  Workgroup = 8 rows x 8 pairs of columns, a pair being what one epilogue needs: (j, j + Dh/2)
// of a head, gate and up of one unit, two neighbours.  The 16 lanes of a row of lanes split K (VW elements each, so their
// loads are consecutive), one column per row of lanes; the rows of x pass through LDS, normalised on the way.  The rows of
// a small expert fill only a few tiles, so the tile is kept small (8 x 16) to spread them: 10 rows of the smallest expert
// are 48 workgroups for q/k/v and 64 for gate/up.
template <int EPI, int WDT, int VW>
__global__ __launch_bounds__(256) void g_proj(ProjArgs a) {
  __shared__ __align__(16) float xs[PR_ROWS][PR_KC];
  __shared__ float rs[PR_ROWS], red[PR_ROWS][17];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, ksl = lane & 15, grp = lane >> 4;
  const int K = a.K;
  const int pairs = EPI == GEPI_QKV ? 3 * (a.A / 2) : (EPI == GEPI_SWIGLU ? a.N : (a.N + 1) / 2);
  // column of pair u, member mem: weight matrix sec, row col
  auto column = [&](int u, int mem, int& sec, int& col) {
    if (EPI == GEPI_QKV) {
      const int half = a.Dh / 2, p = u % (a.A / 2);
      sec = u / (a.A / 2);
      col = p / half * a.Dh + p % half + mem * half;
    } else if (EPI == GEPI_SWIGLU) {
      sec = mem;
      col = u;
    } else {
      sec = 0;
      col = 2 * u + mem;
    }
  };
  const int cblk = (pairs + 7) / 8;
  const int64_t tiles = (int64_t)cblk * ((a.M + PR_ROWS - 1) / PR_ROWS);
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int u0 = (int)(tile % cblk) * 8, row0 = (int)(tile / cblk) * PR_ROWS;
    int sec, col;
    column(min(u0 + wave * 2 + (grp >> 1), pairs - 1), grp & 1, sec, col);
    const void* w = EPI == GEPI_RESIDUAL ? a.w[0] : (sec == 0 ? a.w[0] : (sec == 1 ? a.w[1] : a.w[2]));
    const int64_t wrow = (int64_t)min(col, a.N - 1) * K;
    float acc[PR_ROWS];
#pragma unroll
    for (int r = 0; r < PR_ROWS; ++r) acc[r] = 0.f;
    constexpr int NS = PR_KC / (16 * VW);  // steps of a chunk
    constexpr int UB = NS < 8 ? NS : 8;    // weight loads in flight
    for (int k0 = 0; k0 < K; k0 += PR_KC) {
      const int kn = min(PR_KC, K - k0);
      float4 wv[UB];
      auto load_w = [&](int s0) {
#pragma unroll
        for (int s = 0; s < UB; ++s) {
          const int k = (s0 + s) * 16 * VW + ksl * VW;
          wv[s] = k < kn ? ldv<WDT, VW>(w, wrow + k0 + k) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
      };
      load_w(0);
      if (k0 == 0) {  // each row's RMSNorm scale: two rows per wave
        for (int r = wave; r < PR_ROWS; r += 4) {
          float ss = 0.f;
          if (a.gain && row0 + r < a.M)
            for (int k = lane; k < K; k += WAVE) {
              const float v = a.x[(int64_t)(row0 + r) * K + k];
              ss += v * v;
            }
          ss = wave_sum(ss);
          if (lane == 0) rs[r] = a.gain ? 1.0f / sqrtf(ss / (float)K + a.eps) : 1.f;
        }
      }
      __syncthreads();  // the scales; the chunk before has been read
      for (int r = wave; r < PR_ROWS; r += 4)
        for (int k = lane; k < kn; k += WAVE) {
          const float v = row0 + r < a.M ? a.x[(int64_t)(row0 + r) * K + k0 + k] : 0.f;
          xs[r][k] = a.gain ? v * rs[r] * a.gain[k0 + k] : v;
        }
      __syncthreads();
      for (int s0 = 0; s0 < NS && s0 * 16 * VW < kn; s0 += UB) {
        if (s0) load_w(s0);
#pragma unroll
        for (int s = 0; s < UB; ++s) {
          const int k = (s0 + s) * 16 * VW + ksl * VW;
          if (k < kn) {
#pragma unroll
            for (int r = 0; r < PR_ROWS; ++r) {
              if constexpr (VW == 4) {
                const float4 xv = *reinterpret_cast<const float4*>(&xs[r][k]);
                acc[r] += xv.x * wv[s].x + xv.y * wv[s].y + xv.z * wv[s].z + xv.w * wv[s].w;
              } else {
                acc[r] += xs[r][k] * wv[s].x;
              }
            }
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < PR_ROWS; ++r) {
      acc[r] = row_sum16(acc[r]);
      if (ksl == 0) red[r][wave * 4 + grp] = acc[r];
    }
    __syncthreads();
    const int r = threadIdx.x >> 4, i = threadIdx.x & 15, m = row0 + r, u = u0 + (i >> 1), mem = i & 1;
    if (r < PR_ROWS && m < a.M && u < pairs) {
      const float v = red[r][i], other = red[r][i ^ 1];
      column(u, mem, sec, col);
      if (EPI == GEPI_QKV) {
        float y = v;
        if (sec < 2) {
          const float* cs = a.rope + ((int64_t)m * (a.Dh / 2) + u % (a.A / 2) % (a.Dh / 2)) * 2;
          y = mem ? v * cs[0] + other * cs[1] : v * cs[0] - other * cs[1];
          if (sec == 0) y *= 1.0f / sqrtf((float)a.Dh);
        }
        (sec == 0 ? a.out[0] : (sec == 1 ? a.out[1] : a.out[2]))[(int64_t)m * a.A + col] = y;
      } else if (EPI == GEPI_SWIGLU) {
        if (mem == 0) a.out[0][(int64_t)m * a.N + col] = v / (1.0f + expf(-v)) * other;
      } else if (col < a.N) {
        const int64_t o = (int64_t)m * a.N + col;
        const float y = a.out[0][o] + v;
        a.out[0][o] = y;
        if (a.hidden) a.hidden[o] = y;
      }
    }
    __syncthreads();
  }
}

struct GAttnArgs {
  CacheView cv;
  const float* q;  // [M][A] rotated, scaled by 1/sqrt(Dh)
  const float* k;
  const float* v;
  float* out;
  int H, Dh;
};

__device__ __forceinline__ float wave_max(float v) {
#define FSX_ROR_MAX(ctrl) \
  v = vmax(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, 0xF, 0xF, false)))
  FSX_ROR_MAX(0x128);
  FSX_ROR_MAX(0x124);
  FSX_ROR_MAX(0x122);
  FSX_ROR_MAX(0x121);
#undef FSX_ROR_MAX
  return rows_max(v);
}

// One tile of n <= 64 rows (lane r's row at element krow of kbase; row r of the tile at vrow(r) of vbase) into a wave's
// running state: scores with one row per lane, then the values with lpr lanes per row (VW channels each) and 64 / lpr
// rows at a time.  The weights cross through the wave's own 64 floats of LDS.
template <int DT, int VW, typename VRow>
__device__ __forceinline__ void g_attn_tile(const float* __restrict__ q, int Dh, const void* kbase, int64_t krow, float ks,
                                            const void* vbase, VRow vrow, float vs, int n, int ch, int lpr, int lane,
                                            float* p_lds, float& m, float& l, float4& o) {
  float s = 0.f;
  for (int c0 = 0; c0 < Dh; c0 += 8 * VW) {
    float4 kv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      kv[j] = c0 + j * VW < Dh ? ldv<DT, VW>(kbase, krow + c0 + j * VW) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int c = c0 + j * VW;
      if (c < Dh) {
        s += q[c] * kv[j].x;
        if constexpr (VW == 4) s += q[c + 1] * kv[j].y + q[c + 2] * kv[j].z + q[c + 3] * kv[j].w;
      }
    }
  }
  s *= ks;
  const float m_new = fmaxf(m, wave_max(lane < n ? s : -INFINITY));
  const float mz = m_new == -INFINITY ? 0.f : m_new;  // rows that all score -inf weigh nothing yet
  const float alpha = expf(m - mz);
  const float p = lane < n ? expf(s - mz) : 0.f;
  l = l * alpha + wave_sum(p);
  m = m_new;
  o.x *= alpha;
  o.y *= alpha;
  o.z *= alpha;
  o.w *= alpha;
  p_lds[lane] = p;
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  const int rps = WAVE / lpr;
  if (ch < Dh) {
    for (int r0 = lane / lpr; r0 < n; r0 += 8 * rps) {
      float4 vv[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) vv[j] = ldv<DT, VW>(vbase, vrow(min(r0 + j * rps, n - 1)) + ch);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (r0 + j * rps < n) {
          const float pj = p_lds[r0 + j * rps] * vs;
          o.x += pj * vv[j].x;
          if constexpr (VW == 4) {
            o.y += pj * vv[j].y;
            o.z += pj * vv[j].z;
            o.w += pj * vv[j].w;
          }
        }
      }
    }
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// One workgroup per (query, head, 64 VW output channels): its four waves take 64-row tiles of [cache rows ; own rows] in
// turn, each with an online softmax, and merge their states.
template <int CDT, int VW>
__global__ __launch_bounds__(256) void g_attention(GAttnArgs a, TickParams tp) {
  __shared__ float p_lds[4][WAVE], ml[4][2];
  __shared__ float4 part[4][WAVE];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int A = a.H * a.Dh, Dh = a.Dh;
  for (int64_t item = blockIdx.x; item < (int64_t)tp.M * a.H; item += gridDim.x) {
    const int h = (int)(item % a.H), row = (int)(item / a.H), b = row / tp.S;
    const int c_first = blockIdx.y * WAVE * VW, nc = min(Dh - c_first, WAVE * VW);
    int lpr = 1;  // lanes per row of values
    while (lpr * VW < nc) lpr *= 2;
    const int ch = c_first + lane % lpr * VW;
    const float* q = a.q + (int64_t)row * A + (int64_t)h * Dh;
    const int L = tp.len[b], nct = (L + 63) / 64, nt = nct + (tp.S + 63) / 64;
    const int64_t hb = cache_head_base(a.cv, b, a.cv.layer, h);
    float ks = 1.f, vs = 1.f;
    if (CDT == FSX_FP8_E4M3 && L > 0) {
      ks = a.cv.k_scale[cache_scale_index(a.cv, b, a.cv.layer, h)];
      vs = a.cv.v_scale[cache_scale_index(a.cv, b, a.cv.layer, h)];
    }
    float m = -INFINITY, l = 0.f;
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int ti = wave; ti < nt; ti += 4) {
      if (ti < nct) {
        const int r0 = ti * 64, n = min(64, L - r0);
        auto off = [&](int r) {
          int64_t slot = tp.start[b] + r0 + r;
          if (slot >= a.cv.cap) slot -= a.cv.cap;
          return hb + slot * a.cv.rs;
        };
        g_attn_tile<CDT, VW>(q, Dh, a.cv.k, off(min(lane, n - 1)), ks, a.cv.v, off, vs, n, ch, lpr, lane, p_lds[wave], m, l, o);
      } else {
        const int r0 = (ti - nct) * 64, n = min(64, tp.S - r0);
        auto off = [&](int r) { return ((int64_t)b * tp.S + r0 + r) * A + (int64_t)h * Dh; };
        g_attn_tile<FSX_F32, VW>(q, Dh, a.k, off(min(lane, n - 1)), 1.f, a.v, off, 1.f, n, ch, lpr, lane, p_lds[wave], m, l, o);
      }
    }
    part[wave][lane] = o;
    if (lane == 0) {
      ml[wave][0] = m;
      ml[wave][1] = l;
    }
    __syncthreads();
    const int c = threadIdx.x;  // channel c_first + c
    if (c < nc) {
      float M = -INFINITY;
      for (int w = 0; w < 4; ++w) M = fmaxf(M, ml[w][0]);
      const float mz = M == -INFINITY ? 0.f : M;
      float sum = 0.f, y = 0.f;
      for (int w = 0; w < 4; ++w) {
        if (w >= nt) continue;
        const float f = expf(ml[w][0] - mz);
        sum += ml[w][1] * f;
        float yw = 0.f;
        for (int g = 0; g < WAVE / lpr; ++g) yw += reinterpret_cast<const float*>(&part[w][g * lpr + c / VW])[c % VW];
        y += yw * f;
      }
      a.out[(int64_t)row * A + (int64_t)h * Dh + c_first + c] = y * (1.0f / sum);
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void g_head(const float* h, int S, int T, int d, float eps, const float* gfin, const void* w,
                                              int wdtype, int n_out, float* wp) {
  extern __shared__ float xm[];
  mean_head_wg(h, S, T, d, eps, gfin, w, wdtype, n_out, wp, xm);
}

// Four elements per load where the rows allow it: K a multiple of four and every matrix aligned to that.
template <int EPI>
static void launch_proj(const ProjArgs& p, int wdt, int n_w, int64_t pairs, hipStream_t s) {
  const int es = wdt == FSX_BF16 ? 2 : 4;
  bool vec = p.K % 4 == 0;
  for (int i = 0; i < n_w; ++i) vec = vec && reinterpret_cast<uintptr_t>(p.w[i]) % (4 * es) == 0;
  const auto fn = wdt == FSX_BF16 ? (vec ? g_proj<EPI, FSX_BF16, 4> : g_proj<EPI, FSX_BF16, 1>)
                                  : (vec ? g_proj<EPI, FSX_F32, 4> : g_proj<EPI, FSX_F32, 1>);
  const int64_t tiles = (pairs + 7) / 8 * ((p.M + PR_ROWS - 1) / PR_ROWS);
  hipLaunchKernelGGL(fn, dim3((unsigned)std::min(tiles, GRID_MAX)), dim3(256), 0, s, p);
}

template <int VW>
static void launch_g_attention(const GAttnArgs& a, const TickParams& tp, hipStream_t s) {
  const auto fn = a.cv.dtype == FSX_BF16 ? g_attention<FSX_BF16, VW>
                                         : (a.cv.dtype == FSX_FP8_E4M3 ? g_attention<FSX_FP8_E4M3, VW> : g_attention<FSX_F32, VW>);
  hipLaunchKernelGGL(fn, dim3((unsigned)std::min((int64_t)tp.M * a.H, GRID_MAX), (unsigned)((a.Dh + WAVE * VW - 1) / (WAVE * VW))), dim3(256), 0, s, a, tp);
}

hipError_t generic_tick(const GenericWeights* L, const float* final_norm, const void* head_w, const QueryHead& qhead,
                        int wdt,
                        const void* tokens, const CacheView& cv0, const TickParams& tp, const Dims& dm,
                        const GenericWorkspace& ws, float* waypoints, float* hidden, hipStream_t s) {
  const int M = tp.M, d = dm.d, A = dm.A, F = dm.F;
  hipLaunchKernelGGL(g_embed, dim3(M), dim3(128), 0, s, tokens, wdt, tp, dm, ws);
  for (int l = 0; l < dm.n_layers; ++l) {
    ProjArgs p{};
    p.M = M; p.A = A; p.Dh = dm.Dh; p.eps = dm.eps; p.rope = ws.rope;
    p.x = ws.h; p.gain = L[l].attn_norm; p.N = A; p.K = d;
    p.w[0] = L[l].wq; p.w[1] = L[l].wk; p.w[2] = L[l].wv;
    p.out[0] = ws.q; p.out[1] = ws.k; p.out[2] = ws.v;
    launch_proj<GEPI_QKV>(p, wdt, 3, 3 * (int64_t)(A / 2), s);
    GAttnArgs at{cv0, ws.q, ws.k, ws.v, ws.attn, dm.H, dm.Dh};
    at.cv.layer = l;
    // heads of a multiple of four channels: every row of cache and workspace is aligned to four elements
    if (dm.Dh % 4 == 0)
      launch_g_attention<4>(at, tp, s);
    else
      launch_g_attention<1>(at, tp, s);
    p.x = ws.attn; p.gain = nullptr; p.N = d; p.K = A;
    p.w[0] = L[l].wo; p.out[0] = ws.h;
    launch_proj<GEPI_RESIDUAL>(p, wdt, 1, (d + 1) / 2, s);
    p.x = ws.h; p.gain = L[l].ffn_norm; p.N = F; p.K = d;
    p.w[0] = L[l].wg; p.w[1] = L[l].wu; p.out[0] = ws.g;
    launch_proj<GEPI_SWIGLU>(p, wdt, 2, F, s);
    p.x = ws.g; p.gain = nullptr; p.N = d; p.K = F;
    p.w[0] = L[l].wd; p.out[0] = ws.h; p.hidden = hidden ? hidden + (int64_t)l * M * d : nullptr;
    launch_proj<GEPI_RESIDUAL>(p, wdt, 1, (d + 1) / 2, s);
  }
  if (dm.head_kind == 1) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_query_head((const float*)ws.h, tp, dm, final_norm, qhead, waypoints, s);
  }
  hipLaunchKernelGGL(g_head, dim3(tp.B), dim3(256), d * sizeof(float), s, (const float*)ws.h, tp.S, tp.T, d, dm.eps,
                     final_norm, head_w, wdt, dm.n_out, waypoints);
  return hipGetLastError();
}

}  // namespace fsx
