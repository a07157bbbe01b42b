// Kernels of the bf16 expert tick on gfx950 (Sec. 3.1, Eq. (1); Sec. 3.3).
//
// One tick, per layer:
//   qkv   : x = RMSNorm(h) (bf16) times the packed [3A][d] projection on MFMA; epilogue applies the
//           rotary rotation to q and k and folds 1/sqrt(Dh) * log2(e) into q.
//   attn  : split-K ("flash-decode") joint attention over chunks of cached rows, the expert's own keys/values after an
//           agent's last chunk, so Eq. (1)'s single softmax over [cache ; own rows] is the log-sum-exp merge of the
//           chunks, which the one that finishes last does.
//   o     : output projection, split-K partial sums.
//   norm  : h += sum of partials; x = RMSNorm(h) * gain (bf16) for the next projection.
//   gu    : gate/up projection on MFMA with SwiGLU in the epilogue.
//   down  : down projection, split-K partials; then norm again with the next layer's gain.
// The head pools the first T tokens after a final RMSNorm and applies a d -> n_out map.

#include <algorithm>
#include <type_traits>

#include "attn_device.h"
#include "common.h"
#include "kernels.h"

namespace fsx {

// =====================================================================================================
// Weight packing.  A [N][K] bf16 matrix (nn.Linear layout) becomes N/16 x K/32 blocks of 1 KiB; block
// (nt, kb) sits at element offset (nt*K/32 + kb)*512 and its 16-byte slot l (l = 0..63) holds
// W[row(nt*16 + l%16)][kb*32 + 8*(l/16) + j], j = 0..7 -- exactly the B operand of a 16x16x32 MFMA for
// output columns nt*16.. and k = kb*32.., so one wave reads a block with one fully coalesced 1 KiB load.
// row() pairs rows for fused epilogues:
//   PACK_ROPE_PAIRS  : within each head of width Dh, tile tau holds channels [8tau, 8tau+8) in columns
//                      0..7 and [Dh/2 + 8tau, ...) in columns 8..15, so rotary partners are lanes l, l^8.
//   PACK_SWIGLU_PAIRS: tile tau holds gate rows [8tau, 8tau+8) (from a) in columns 0..7 and the same up
//                      rows (from b) in columns 8..15.
// When the projection reads an RMSNorm output, the norm's gain is folded into the packed weights
// (x*r*g) W^T = r * (x (W diag(g))^T), so kernels feed bf16(x) and scale each output row by r.
// =====================================================================================================
__global__ void k_pack(const uint16_t* __restrict__ a, const uint16_t* __restrict__ b, int N, int K, int kind,
                       int param, const float* __restrict__ gain, uint4* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int KB = K / 32;
  const int64_t total = (int64_t)(N / 16) * KB * 64;
  if (i >= total) return;
  const int l = (int)(i & 63);
  const int64_t blk = i >> 6;
  const int kb = (int)(blk % KB);
  const int nt = (int)(blk / KB);
  const int n = nt * 16 + (l & 15);
  const int kcol = kb * 32 + 8 * (l >> 4);
  const uint16_t* src = a;
  int64_t row = n;
  if (kind == PACK_ROPE_PAIRS) {
    const int Dh = param, half = Dh / 2;
    const int head = n / Dh, p = n % Dh, tau = p / 16, c = p % 16;
    row = (int64_t)head * Dh + (c < 8 ? 8 * tau + c : half + 8 * tau + (c - 8));
  } else if (kind == PACK_SWIGLU_PAIRS) {
    const int tau = n / 16, c = n % 16;
    row = 8 * tau + (c & 7);
    src = c < 8 ? a : b;
  }
  uint4 v = *reinterpret_cast<const uint4*>(src + row * K + kcol);
  if (gain) {  // fold the RMSNorm gain of the input channels into the weight: W'[n][k] = W[n][k] * g[k]
    uint32_t* w = reinterpret_cast<uint32_t*>(&v);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float lo = bf16_to_f32((uint16_t)(w[j] & 0xffffu)) * gain[kcol + 2 * j];
      const float hi = bf16_to_f32((uint16_t)(w[j] >> 16)) * gain[kcol + 2 * j + 1];
      w[j] = pack_bf16x2(lo, hi);
    }
  }
  dst[i] = v;
}

hipError_t launch_pack(const uint16_t* a, const uint16_t* b, int N, int K, int kind, int param, const float* gain,
                       void* dst, hipStream_t s) {
  const int64_t total = (int64_t)(N / 16) * (K / 32) * 64;
  const int64_t blocks = (total + 255) / 256;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)blocks), dim3(256), 0, s, a, b, N, K, kind, param, gain, (uint4*)dst);
  return hipGetLastError();
}

// =====================================================================================================
// Embed: h = tokens (fp32), x = bf16(h / rms(h)), rotary table cos/sin(p * base^(-2j/Dh)) in fp64.
// One workgroup per token row.
// =====================================================================================================
__global__ __launch_bounds__(256) void k_embed(const void* __restrict__ tokens, int tok_dtype,
                                               const float* __restrict__ g0, TickParams tp, Dims dm,
                                               Workspace ws) {
  __shared__ float red[16];
  const int m = blockIdx.x;
  const int b = m / tp.S, t = m % tp.S;
  const int d = dm.d;
  float ss = 0.f;
  for (int n = threadIdx.x; n < d; n += blockDim.x) {
    const int64_t idx = (int64_t)m * d + n;
    const float v = tok_dtype == FSX_BF16 ? bf16_to_f32(((const uint16_t*)tokens)[idx]) : ((const float*)tokens)[idx];
    ws.h[idx] = v;
    ss += v * v;
  }
  ss = block_sum(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)d + dm.eps);
  for (int n = threadIdx.x; n < d; n += blockDim.x) {
    const int64_t idx = (int64_t)m * d + n;
    ws.xb[idx] = f32_to_bf16(ws.h[idx] * r);  // the gain is folded into the packed weights
  }
  const int half = dm.Dh / 2;
  for (int j = threadIdx.x; j < half; j += blockDim.x) {
    double cs = 1.0, sn = 0.0;
    if (dm.rope_base > 0.f) {
      const double theta = pow((double)dm.rope_base, -2.0 * (double)j / (double)dm.Dh);
      const double ang = (double)(tp.pos[b] + t) * theta;
      cs = cos(ang);
      sn = sin(ang);
    }
    ws.rope[((int64_t)m * half + j) * 2 + 0] = (float)cs;
    ws.rope[((int64_t)m * half + j) * 2 + 1] = (float)sn;
  }
}

hipError_t launch_embed(const void* tokens, int tok_dtype, const float* g0, const TickParams& tp, const Dims& dm,
                        const Workspace& ws, hipStream_t s) {
  hipLaunchKernelGGL(k_embed, dim3(tp.M), dim3(256), 0, s, tokens, tok_dtype, g0, tp, dm, ws);
  return hipGetLastError();
}

// =====================================================================================================
// Projection GEMM: y[m][n] = sum_k x[m][k] W[n][k], x bf16 [M][K], W packed (above).
// Workgroup = 4 waves on one 16-column tile and one split-K range; the waves interleave its k-blocks,
// then reduce their accumulators through LDS.  Each lane streams one 16-byte weight slot per k-block
// (1 KiB coalesced per wave).  k_gemm takes one row tile (at most 16 rows); k_gemm_rows, below, more.
// =====================================================================================================
enum { EPI_QKV = 0, EPI_SWIGLU = 1, EPI_PARTIAL = 2 };

struct GemmArgs {
  const uint16_t* x;
  int ldx;
  const uint4* w;
  int M, K, N, ksplit;
  float* out_f;      // QKV: q [M][A]; PARTIAL: [ksplit][M][N]
  uint16_t* out_k;   // QKV
  uint16_t* out_v;   // QKV
  uint16_t* out_z;   // SWIGLU: [M][N/2]
  const float* rope; // [M][Dh/2][2]
  int A, Dh;
  float q_scale;
  // optional RMSNorm scale of each row [M], applied to the products (wide rows: x then holds the unscaled residual
  // in bf16; the gain is folded into the weights)
  const float* rscale;
};

// Rotary (cos, sin) of the four rows 4 grp + i of a row tile in this lane's column of tile nt (EPI_QKV, q and k tiles;
// loaded ahead of the epilogue, whose stores would otherwise keep each tile's loads behind those of the tile before).
template <int EPI>
__device__ __forceinline__ void load_rope(const GemmArgs& g, int row0, int nt, int c, int grp, float2 (&cs)[4]) {
  if constexpr (EPI == EPI_QKV) {
    const int half = g.Dh / 2, n = nt * 16 + c, nl = n % g.A, j = 8 * (nl % g.Dh / 16) + (c & 7);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      cs[i] = reinterpret_cast<const float2*>(g.rope)[(int64_t)min(row0 + 4 * grp + i, g.M - 1) * half + j];
  }
}

template <int EPI>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, f32x4 s, int row0, int nt, int ks, int c, int grp,
                                              const float2 (&cs)[4]) {
  const int n = nt * 16 + c;
  if constexpr (EPI == EPI_PARTIAL) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = row0 + 4 * grp + i;
      if (row < g.M) g.out_f[((int64_t)ks * g.M + row) * g.N + n] = s[i];
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float up = xor8(s[i]);
      const int row = row0 + 4 * grp + i;
      if (c < 8 && row < g.M) {
        const float gt = s[i];
        const float zz = gt / (1.0f + expf(-gt)) * up;
        g.out_z[(int64_t)row * (g.N / 2) + nt * 8 + c] = f32_to_bf16(zz);
      }
    }
  } else {
    const int A = g.A, Dh = g.Dh, half = Dh / 2;
    const int sec = n / A;  // 0 = q, 1 = k, 2 = v (uniform across the tile)
    const int nl = n - sec * A;
    if (sec == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row0 + 4 * grp + i;
        if (row < g.M) g.out_v[(int64_t)row * A + nl] = f32_to_bf16(s[i]);
      }
    } else {
      const int head = nl / Dh, p = nl % Dh;
      const int j = 8 * (p / 16) + (c & 7);
      const int dch = c < 8 ? j : half + j;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float other = xor8(s[i]);
        const int row = row0 + 4 * grp + i;
        const float r = c < 8 ? s[i] * cs[i].x - other * cs[i].y : s[i] * cs[i].x + other * cs[i].y;
        if (row < g.M) {
          const int64_t o = (int64_t)row * A + head * Dh + dch;
          if (sec == 0)
            g.out_f[o] = r * g.q_scale;
          else
            g.out_k[o] = f32_to_bf16(r);
        }
      }
    }
  }
}

template <int EPI>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs g) {
  __shared__ f32x4 red[4][WAVE];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c = lane & 15, grp = lane >> 4;
  const int n_tiles = g.N / 16;
  const int nt = blockIdx.x % n_tiles, ks = blockIdx.x / n_tiles;
  const int KB = g.K / 32;
  const int kbs = KB / g.ksplit;
  const int kb0 = ks * kbs, kb1 = kb0 + kbs;
  const uint4* __restrict__ wt = g.w + (int64_t)nt * KB * WAVE + lane;
  const bool ok = c < g.M;
  const uint16_t* xr = g.x + (int64_t)(ok ? c : 0) * g.ldx + 8 * grp;
  float rsc[4];  // row scales of this lane's epilogue rows, loaded before the weight stream
#pragma unroll
  for (int i = 0; i < 4; ++i) rsc[i] = EPI != EPI_PARTIAL && g.rscale && 4 * grp + i < g.M ? g.rscale[4 * grp + i] : 1.f;
  float2 cs[4];
  if (wave == 0) load_rope<EPI>(g, 0, nt, c, grp, cs);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  // Batches of U k-blocks of this wave: every weight block and x operand of the batch is loaded before the first
  // MFMA, so U KiB of weights per wave are in flight (one at a time leaves the stream latency-bound).
  constexpr int U = 8;
  int kb = kb0 + wave;
  for (; kb + 4 * (U - 1) < kb1; kb += 4 * U) {
    uint4 wv[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) wv[u] = ld_global(wt + (int64_t)(kb + 4 * u) * WAVE);
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = ok ? *reinterpret_cast<const uint4*>(xr + (kb + 4 * u) * 32) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int u = 0; u < U; ++u) acc = mfma_bf16(xv[u], wv[u], acc);
  }
  if (kb < kb1) {
    // the last, partial batch: its k-blocks loaded together too (the missing ones as zeros), so a short split-K
    // range costs one load latency instead of one per k-block
    uint4 wv[U], xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = kb + 4 * u < kb1;
      wv[u] = in ? ld_global(wt + (int64_t)(kb + 4 * u) * WAVE) : make_uint4(0, 0, 0, 0);
      xv[u] = in && ok ? *reinterpret_cast<const uint4*>(xr + (kb + 4 * u) * 32) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (kb + 4 * u < kb1) acc = mfma_bf16(xv[u], wv[u], acc);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave == 0) {
    f32x4 s = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] *= rsc[i];
    gemm_epilogue<EPI>(g, s, 0, nt, ks, c, grp, cs);
  }
}

constexpr int SHORT_CHUNKS = 4;  // chunks of a K range that LDS holds whole

// Workgroup barrier without the fence that drains global loads: the callers order LDS themselves.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Projection of many rows.  Workgroup = CW compute waves and 4 loader waves on MT row tiles and CW NT column tiles; compute
// wave w owns NT column tiles for every row, so its weights are read by nobody else and go straight from memory into a
// register ring of RING k-blocks, while the rows pass through LDS in chunks of KCB k-blocks, three chunks deep, brought by
// the loaders' direct loads (two loader waves per chunk, even and odd chunks in turn, so a chunk has two steps to
// arrive).  A loader waits for its loads itself and never reads LDS; the compute waves' only loads in flight are
// weights, so the ring keeps RING * NT KiB per wave in flight across the barriers.
// Measured at the backbone's widths (us: q/k/v, gate/up, O + down), against workgroups whose waves split K and load the
// rows themselves, in register batches of two k-blocks: 64 rows 48, 63, 44 -> 28, 38, 35; 512 rows 298, 400, 271 -> 62,
// 115, 80.  Bound: the lines a CU can have in flight (see cu_cost), at 512 rows with the MFMAs busy a third of the time;
// one loader wave was the bound before (12 GB/s per CU), and operands read two at a time cost 40 % of the 512-row q/k/v.
//
// ALL: a K range of at most four chunks (512 columns of bf16, the expert's width), which LDS holds whole: every load is
// issued at once, the chunks divided among the loaders.  With three buffers the last chunks waited for the first to be multiplied, and the round trips were most
// of the expert's projections.  us for q/k/v, gate/up, O + down: 74 rows 10.9, 8.6, 13.8, now 8.2, 5.5, 9.7; 160 rows 15.2,
// 9.8, 15.1, now 9.9, 5.4, 11.2 (with smaller row blocks too, see gemm_short).
template <int MT, int NT, int KCB, int RING, int EPI, int CW, bool ALL>
__global__ __launch_bounds__((CW + 4) * 64) void k_gemm_rows(GemmArgs g, int n_rb) {
  constexpr int CPR = KCB * 4;         // 16-byte chunks of a row in one LDS chunk
  constexpr int RPI = 64 / CPR;        // rows one direct-load instruction brings
  constexpr int NI = MT * 16 / RPI;    // instructions per chunk
  static_assert(CPR >= 8 && CPR <= 64 && NI % (ALL ? 4 : 2) == 0, "chunk size");
  static_assert(RING % KCB == 0 || KCB % RING == 0, "chunk and ring sizes");
  constexpr int UN = RING > KCB ? RING : KCB;  // k-blocks per unrolled pass
  constexpr int NB = ALL ? SHORT_CHUNKS : 3;
  __shared__ uint4 xs[NB][MT * 16 * CPR];
  __shared__ float rs[MT * 16];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int c = lane & 15, grp = lane >> 4;
  const int n_tiles = g.N / 16, KB = g.K / 32;
  // the row blocks of one (column group, K range) run side by side on one XCD (workgroup id mod 8), sharing its L2
  const int n_cg = (n_tiles + CW * NT - 1) / (CW * NT);
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int combo = (idx / n_rb) * 8 + xcd, rb = idx % n_rb;
  if (combo >= n_cg * g.ksplit) return;
  const int cg = combo % n_cg, ks = combo / n_cg;
  const int row0 = rb * MT * 16;
  const int kb0 = ks * KB / g.ksplit, kb1 = (ks + 1) * KB / g.ksplit;
  const int nch = (kb1 - kb0 + KCB - 1) / KCB;
  if (EPI != EPI_PARTIAL && threadIdx.x < MT * 16) {
    const int row = row0 + (int)threadIdx.x;
    rs[threadIdx.x] = g.rscale && row < g.M ? g.rscale[row] : 1.f;
  }
  if (wave >= CW) {
    // part of lpc of chunk i of the rows, into buffer i % NB: row r's 16-byte chunk k at chunk position k ^ (r & 7) (the 16
    // rows of an operand read then fall in distinct banks); rows past M and k-blocks past the range repeat the last one
    auto stage = [&](int i, int part, int lpc) {
      uint4* buf = xs[i % NB];
#pragma unroll 8
      for (int qq = 0; qq < NI / lpc; ++qq) {
        const int q = lpc * qq + part;
        const int r = q * RPI + lane / CPR, k = (lane % CPR) ^ (r & 7);
        const int kb = min(kb0 + i * KCB + (k >> 2), kb1 - 1);
        load_lds16<false>(g.x + (int64_t)min(row0 + r, g.M - 1) * g.ldx + kb * 32 + (k & 3) * 8, buf + q * 64);
      }
    };
    const int lw = wave - CW;
    if constexpr (ALL) {
      // a loader has loads of one chunk only (four chunks: one loader each, two: two each), so it waits for all of its
      // loads before the barrier of its chunk and no wait counts loads of a later one
      const int lpc = nch > 2 ? 1 : 4 / nch, mine = lw / lpc;
      if (mine < nch) stage(mine, lw % lpc, lpc);
      for (int i = 0; i < nch; ++i) {
        if (i == mine) vm_wait_all();
        wg_barrier();
      }
    } else {
      const int par = lw >> 1, half = lw & 1;
      if (par < nch) stage(par, half, 2);
      if (par == 0) vm_wait_all();
      wg_barrier();
      for (int i = 0; i + 1 < nch; ++i) {  // while chunk i is multiplied
        if ((i & 1) == par) {
          if (i + 2 < nch) stage(i + 2, half, 2);
        } else {
          vm_wait_all();  // chunk i + 1
        }
        wg_barrier();
      }
    }
    return;
  }
  const uint4* wt[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
    wt[t] = g.w + (int64_t)min((cg * CW + wave) * NT + t, n_tiles - 1) * KB * WAVE + lane;
  uint4 w[RING][NT];
#pragma unroll
  for (int j = 0; j < RING; ++j)
#pragma unroll
    for (int t = 0; t < NT; ++t) w[j][t] = ld_global(wt[t] + (int64_t)min(kb0 + j, kb1 - 1) * WAVE);
  f32x4 acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  wg_barrier();
  int buf = 0, kb = kb0;
  uint4 xv[2][MT];  // the row operands of this k-block and of the next
  auto read = [&](int jj, uint4 (&x)[MT]) {
    const uint4* xb = &xs[buf][c * CPR + ((jj * 4 + grp) ^ (c & 7))];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) x[mt] = xb[mt * 16 * CPR];
  };
  read(0, xv[0]);
  // UN k-blocks from kb on: the next k-block's operands are read (past the barrier that frees a chunk, when it is the
  // chunk's last) before this one's products, which hide their latency; left to itself the compiler reads two operands
  // at a time and waits for each pair.  The last pass checks each k-block against the range.
  auto pass = [&](auto check) {
    constexpr bool CHECK = decltype(check)::value;
#pragma unroll
    for (int j = 0; j < UN; ++j) {
      if (!CHECK || kb + j < kb1) {
        if (!CHECK || kb + j + 1 < kb1) {
          if (j % KCB == KCB - 1) {
            wg_barrier();
            buf = buf == NB - 1 ? 0 : buf + 1;
          }
          read((j + 1) % KCB, xv[(j + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int t = 0; t < NT; ++t) acc[mt][t] = mfma_bf16(xv[j & 1][mt], w[j % RING][t], acc[mt][t]);
        if (!CHECK || RING < UN)
#pragma unroll
          for (int t = 0; t < NT; ++t) w[j % RING][t] = ld_global(wt[t] + (int64_t)min(kb + j + RING, kb1 - 1) * WAVE);
      }
    }
    kb += UN;
  };
  static_assert(UN % 2 == 0, "operand buffers alternate");
  while (kb + UN < kb1) pass(std::false_type());
  pass(std::true_type());
  float2 cs[2][NT][4];
  auto tile_of = [&](int t) { return min((cg * CW + wave) * NT + t, n_tiles - 1); };
#pragma unroll
  for (int t = 0; t < NT; ++t) load_rope<EPI>(g, row0, tile_of(t), c, grp, cs[0][t]);
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    if (mt + 1 < MT)
#pragma unroll
      for (int t = 0; t < NT; ++t) load_rope<EPI>(g, row0 + (mt + 1) * 16, tile_of(t), c, grp, cs[(mt + 1) & 1][t]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int tile = (cg * CW + wave) * NT + t;
      if (tile < n_tiles) {
        f32x4 s = acc[mt][t];
        if (EPI != EPI_PARTIAL) s *= *reinterpret_cast<const f32x4*>(&rs[mt * 16 + 4 * grp]);
        gemm_epilogue<EPI>(g, s, row0 + mt * 16, tile, ks, c, grp, cs[mt & 1][t]);
      }
    }
  }
}

template <int MT, int NT, int KCB, int RING, int EPI, int CW = 4, bool ALL = false>
static hipError_t launch_rows(const GemmArgs& g, hipStream_t s) {
  const int n_rb = (g.M + MT * 16 - 1) / (MT * 16), n_cg = (g.N / 16 + CW * NT - 1) / (CW * NT);
  const int combos = n_cg * g.ksplit;
  hipLaunchKernelGGL((k_gemm_rows<MT, NT, KCB, RING, EPI, CW, ALL>), dim3((unsigned)((combos + 7) / 8 * 8 * n_rb)), dim3((CW + 4) * 64), 0, s,
                     g, n_rb);
  return hipGetLastError();
}

// What a projection's workgroups cost a CU, in 128-byte lines weighted by how long each keeps its place: a CU has about
// 64 lines in flight (read requests x their mean latency over the CUs' cycles come to 43 to 81 at the backbone's widths),
// whatever the depth of the ring, so its time goes with the lines it loads: 8 per column tile and k-block for the
// weights, 8 per row tile for the rows, in whole rounds of CUS workgroups.  A line of weights from memory takes about
// three times as long as one of the rows from L2; with several row blocks all but one find the weights in L2.
constexpr int CUS = 256;  // compute units of an MI355X, as one device
static int64_t cu_cost(int n_rb, int mt, int tiles, int KB, int ksplit, int tpw) {
  const int64_t wgs = (int64_t)((tiles + tpw - 1) / tpw) * ksplit * n_rb;
  return (wgs + CUS - 1) / CUS * (8 * tpw * (n_rb > 1 ? 1 : 3) + 8 * mt) * ((KB + ksplit - 1) / ksplit);
}
// Column tiles per workgroup: the cheapest of what the kernels are built for.
static int pick_tiles(int n_mt, int tiles, int KB, int ksplit) {
  const int n_rb = (n_mt + 7) / 8, mt = n_mt > 4 ? 8 : (n_mt > 2 ? 4 : 2);
  static constexpr int one[] = {3, 4, 6, 8}, many[] = {4, 8, 12, 16};
  const int* opt = n_rb > 1 ? many : one;
  int best = opt[0];
  for (int i = 1; i < 4; ++i)
    if (cu_cost(n_rb, mt, tiles, KB, ksplit, opt[i]) <= cu_cost(n_rb, mt, tiles, KB, ksplit, best)) best = opt[i];
  return best;
}

// Split-K ranges of a projection [M][K] x [N][K] whose partial sums a reduction adds.  One row block: 8 where K allows (the
// weights bound it, and the partial sums are small).  Beyond, the count whose loads and partial sums (written, and read
// back by the reduction: twice the price of a line from L2) are least: 512 rows of the backbone's O and down and their
// reductions take 110 + 39 us with 8 ranges, 80 + 29 with the 2 and 4 chosen.
int gemm_split(int M, int N, int K) {
  const int n_mt = (M + 15) / 16, n_rb = (n_mt + 7) / 8, tiles = N / 16, KB = K / 32;
  int best = KB % 8 == 0 ? 8 : (KB % 4 == 0 ? 4 : (KB % 2 == 0 ? 2 : 1));
  if (n_rb == 1) return best;
  int64_t cost = INT64_MAX;
  for (int ks = 1; ks <= 8 && ks <= KB; ks *= 2) {
    const int64_t c = cu_cost(n_rb, 8, tiles, KB, ks, pick_tiles(n_mt, tiles, KB, ks)) + (int64_t)ks * M * N * 8 / 128 / CUS * 2;
    if (c < cost) {
      best = ks;
      cost = c;
    }
  }
  return best;
}

// More than 16 rows over a K range that LDS holds whole: row tiles (2 to 5) and column tiles of a workgroup, by its rounds of
// CUS workgroups times its row tiles and a third of its column tiles (the rows pass through LDS, the weights stream by
// them).  Of the pairs below, at 74 to 400 rows of the expert, the rule picks the fastest or one within 0.5 us of it, with
// two exceptions of 1 us.  us against row tiles of 5 and 8 weighed as much as column tiles: q/k/v of 74 rows 9.9 -> 8.2, of
// 400 rows 23.0 -> 18.6; gate/up of 160 rows 7.6 -> 5.4, O and down 6.2 -> 5.6.
// The rule never picks the other pairs (evaluated for every count of row tiles to 400 and some to 5,000, up to 128 heads,
// widths to 8,192, FFNs to 16,384).
template <int EPI>
constexpr bool short_pair(int mt, int t) {
  return mt == 2 || (EPI == EPI_PARTIAL ? t > 1 && (t != 3 || mt == 3) : t >= (mt < 4 ? mt : 4));
}

template <int MT, int EPI>
static hipError_t launch_short(const GemmArgs& g, int tpw, hipStream_t s) {
  auto pair = [&](auto t) {
    constexpr int T = decltype(t)::value;
    if constexpr (!short_pair<EPI>(MT, T))
      return hipErrorInvalidValue;  // not among the rule's pairs
    else if constexpr (T <= 4)
      return launch_rows<MT, 1, 4, 16, EPI, T, true>(g, s);
    else if constexpr (T == 6)
      return launch_rows<MT, 1, 4, 8, EPI, 6, true>(g, s);
    else if constexpr (T == 8)
      return launch_rows<MT, 2, 4, 8, EPI, 4, true>(g, s);
    else
      return launch_rows<MT, 3, 4, 4, EPI, T / 3, true>(g, s);
  };
  switch (tpw) {
    case 1: return pair(std::integral_constant<int, 1>());
    case 2: return pair(std::integral_constant<int, 2>());
    case 3: return pair(std::integral_constant<int, 3>());
    case 4: return pair(std::integral_constant<int, 4>());
    case 6: return pair(std::integral_constant<int, 6>());
    case 8: return pair(std::integral_constant<int, 8>());
    case 12: return pair(std::integral_constant<int, 12>());
    default: return pair(std::integral_constant<int, 24>());
  }
}

template <int EPI>
static hipError_t gemm_short(const GemmArgs& g, hipStream_t s) {
  const int n_mt = (g.M + 15) / 16, tiles = g.N / 16;
  static constexpr int opt_mt[] = {2, 3, 4, 5}, opt_t[] = {1, 2, 3, 4, 6, 8, 12, 24};
  int mt = 2, tpw = 1;
  int64_t best = INT64_MAX;
  for (int m : opt_mt)
    for (int t : opt_t) {
      if (!short_pair<EPI>(m, t)) continue;
      const int64_t wgs = (int64_t)((tiles + t - 1) / t) * g.ksplit * ((n_mt + m - 1) / m);
      const int64_t cost = (wgs + CUS - 1) / CUS * (3 * m + t);
      if (cost <= best) {
        best = cost;
        mt = m;
        tpw = t;
      }
    }
  switch (mt) {
    case 2: return launch_short<2, EPI>(g, tpw, s);
    case 3: return launch_short<3, EPI>(g, tpw, s);
    case 4: return launch_short<4, EPI>(g, tpw, s);
    default: return launch_short<5, EPI>(g, tpw, s);
  }
}

template <int EPI>
static hipError_t gemm_dispatch(const GemmArgs& g, hipStream_t s) {
  const int n_mt = (g.M + 15) / 16, tiles = g.N / 16;
  if (n_mt == 1) {
    // weights alone: a workgroup per column tile, its waves splitting K (gate/up of the backbone 35 us, 5.1 TB/s; the
    // kernel for many rows 39)
    hipLaunchKernelGGL((k_gemm<EPI>), dim3((unsigned)(tiles * g.ksplit)), dim3(256), 0, s, g);
    return hipGetLastError();
  }
  if (g.K / 32 <= SHORT_CHUNKS * 4 * g.ksplit) return gemm_short<EPI>(g, s);
  // 64 rows of the backbone, us by tiles per workgroup (3, 4, 6, 8): gate/up 46, 49, 38, 45; q/k/v 28, 31, 35, 40; O and
  // down together 45, 39, 42, 35
  const int tpw = pick_tiles(n_mt, tiles, g.K / 32, g.ksplit);
  if (n_mt <= 2) {
    switch (tpw) {
      case 3: return launch_rows<2, 1, 8, 16, EPI, 3>(g, s);
      case 4: return launch_rows<2, 1, 8, 16, EPI, 4>(g, s);
      case 6: return launch_rows<2, 1, 8, 8, EPI, 6>(g, s);
      default: return launch_rows<2, 2, 8, 8, EPI, 4>(g, s);
    }
  }
  if (n_mt <= 4) {
    switch (tpw) {
      case 3: return launch_rows<4, 1, 4, 16, EPI, 3>(g, s);
      case 4: return launch_rows<4, 1, 4, 16, EPI, 4>(g, s);
      case 6: return launch_rows<4, 1, 4, 8, EPI, 6>(g, s);
      default: return launch_rows<4, 2, 4, 8, EPI, 4>(g, s);
    }
  }
  switch (tpw) {
    case 3: return launch_rows<8, 1, 4, 8, EPI, 3>(g, s);
    case 4: return launch_rows<8, 1, 4, 8, EPI, 4>(g, s);
    case 6: return launch_rows<8, 1, 4, 8, EPI, 6>(g, s);
    case 8: return launch_rows<8, 2, 2, 8, EPI, 4>(g, s);
    case 12: return launch_rows<8, 3, 2, 4, EPI, 4>(g, s);
    default: return launch_rows<8, 4, 2, 2, EPI, 4>(g, s);
  }
}

// After a reduction of wide rows xb holds the unscaled residual and ws.rs each row's RMSNorm scale: the
// projection applies the scales to its products.
static void row_scale_from_chunks(GemmArgs& g, const Dims& dm, const Workspace& ws, bool after_reduction) {
  if (after_reduction && wide_rows(dm)) g.rscale = ws.rs;
}

hipError_t launch_gemm_qkv(const FastWeights& w, const TickParams& tp, const Dims& dm, const Workspace& ws,
                           hipStream_t s, bool after_reduction) {
  GemmArgs g{};
  g.x = ws.xb; g.ldx = dm.d; g.w = w.wqkv; g.M = tp.M; g.K = dm.d; g.N = 3 * dm.A; g.ksplit = 1;
  row_scale_from_chunks(g, dm, ws, after_reduction);
  g.out_f = ws.q; g.out_k = ws.kself; g.out_v = ws.vself; g.rope = ws.rope; g.A = dm.A; g.Dh = dm.Dh;
  g.q_scale = LOG2E / sqrtf((float)dm.Dh);
  return gemm_dispatch<EPI_QKV>(g, s);
}

hipError_t launch_gemm_o(const FastWeights& w, const TickParams& tp, const Dims& dm, const Workspace& ws,
                         int ksplit, hipStream_t s) {
  GemmArgs g{};
  g.x = ws.attn; g.ldx = dm.A; g.w = w.wo; g.M = tp.M; g.K = dm.A; g.N = dm.d; g.ksplit = ksplit;
  g.out_f = ws.part;
  return gemm_dispatch<EPI_PARTIAL>(g, s);
}

hipError_t launch_gemm_gu(const FastWeights& w, const TickParams& tp, const Dims& dm, const Workspace& ws,
                          hipStream_t s) {
  GemmArgs g{};
  g.x = ws.xb; g.ldx = dm.d; g.w = w.wgu; g.M = tp.M; g.K = dm.d; g.N = 2 * dm.F; g.ksplit = 1;
  g.out_z = ws.z;
  row_scale_from_chunks(g, dm, ws, true);
  return gemm_dispatch<EPI_SWIGLU>(g, s);
}

hipError_t launch_gemm_down(const FastWeights& w, const TickParams& tp, const Dims& dm, const Workspace& ws,
                            int ksplit, hipStream_t s) {
  GemmArgs g{};
  g.x = ws.z; g.ldx = dm.F; g.w = w.wd; g.M = tp.M; g.K = dm.F; g.N = dm.d; g.ksplit = ksplit;
  g.out_f = ws.part;
  return gemm_dispatch<EPI_PARTIAL>(g, s);
}

// =====================================================================================================
// Split-K joint attention (Eq. (1)): one wave = one work item = (agent, head, chunk of cached rows; see
// attn_device.h) of agents with one query tile, an agent's last chunk followed by the new tokens' own rows.  The wave that
// finishes last among the chunks of an (agent, head) merges their states in chunk order, so no launch does; an agent of one
// chunk writes its output at once.  Partial states cross through device-scope stores and loads, counted by a relaxed
// device-scope atomic that the last wave resets (as k_reduce_chunks counts a row's chunks).
// =====================================================================================================
struct AttnArgs {
  CacheView cv;
  const float* q;
  const uint16_t* kself;
  const uint16_t* vself;
  float* att_o;        // [item][2048] partial outputs and
  float* att_ml;       // [item][32] their maxima and sums, laid out by store_state
  uint32_t* acnt;      // [B * H * n_tt] chunks finished (zero between launches)
  uint16_t* attn_out;  // [M][A] bf16
  int H, Dh, A;
  int causal;          // the own rows are masked causally (new token t sees own rows 0..t)
};

// A state in memory: 16-byte piece k of lane l (accumulator k, queries 4 (l / 16) .. + 3, channel 8 (l % 16) + k) at
// float4 64 k + l of att_o + 2048 item, so every access is a run of whole lines (rows of queries that do not exist are
// left out); the maximum and the sum of query c at att_ml + 32 item + c and + 16 + c.
// Stored query by query in 8-byte words, the states of 74 queries over 4,096 rows (10 MB) took 12 to 18 us to store and
// merge, now 6.
__device__ __forceinline__ void store_state(const AttnArgs& a, int64_t item, const AttnState& st, float lt, int rows, int lane) {
  const int grp = lane >> 4, c = lane & 15;
  if (grp == 0 && c < rows) {
    st_dev_f(a.att_ml + item * 32 + c, st.m);
    st_dev_f(a.att_ml + item * 32 + 16 + c, lt);
  }
  if (4 * grp < rows) {
    const DevBuf o(a.att_o + item * 2048, 8192);
#pragma unroll
    for (int k = 0; k < 8; ++k) o.store16((64 * k + lane) * 16, __builtin_bit_cast(u32x4_t, st.o[k]));
  }
}

// One query tile's output (its first `rows` rows at dst) from a whole state; lt: the sum of query c.
__device__ __forceinline__ void write_output(const AttnArgs& a, const AttnState& st, float lt, int rows, int lane, uint16_t* dst) {
  const int grp = lane >> 4, c = lane & 15;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float inv = 1.0f / col_pick(lt, grp, i);
    if (4 * grp + i < rows)
      *reinterpret_cast<uint4*>(dst + (int64_t)(4 * grp + i) * a.A + 8 * c) =
          make_uint4(pack_bf16x2(st.o[0][i] * inv, st.o[1][i] * inv), pack_bf16x2(st.o[2][i] * inv, st.o[3][i] * inv),
                     pack_bf16x2(st.o[4][i] * inv, st.o[5][i] * inv), pack_bf16x2(st.o[6][i] * inv, st.o[7][i] * inv));
  }
}

// Log-sum-exp merge of the nslot states at items it0, it0 + step, ... (in that order) for queries 4 qq .. + 3 by one wave:
// lane l takes channels 8 (l % 16) + 2 (l / 16) and the next of every query, and for the weights, 16 slots at a time, query
// l % 4 of slot l / 4.  Few workgroups run this, each from a cold instruction cache, so it is kept short: with the weights
// computed by every lane and 7 to 8 slots unrolled it took 8 to 9 us for 3 rounds of 8 slots, now 5.
__device__ __forceinline__ void merge_queries(const AttnArgs& a, int64_t it0, int64_t step, int nslot, int qq, int rows, int lane,
                                              uint16_t* dst /* query 0, channel 0 */) {
  constexpr int RB = 8;
  const int kk = 2 * (lane >> 4), c = lane & 15;
  auto over_slots = [](float v, auto op) {  // over the lanes of one query
    v = op(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x124, 0xF, 0xF, false)));
    return op(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x128, 0xF, 0xF, false)));
  };
  float M = -INFINITY, L = 0.f;
  f32x4 o0 = {0.f, 0.f, 0.f, 0.f}, o1 = o0;
  auto lane_value = [](float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); };
  for (int s0 = 0; s0 < nslot; s0 += 16) {
    const int sl = s0 + (lane >> 2);
    const float* ml = a.att_ml + (it0 + step * min(sl, nslot - 1)) * 32 + 4 * qq + (lane & 3);
    float m = ld_dev_f(ml), l = ld_dev_f(ml + 16);
    const int ns = min(16, nslot - s0);
    for (int j0 = 0; j0 < ns; j0 += RB) {
      f32x4 x0[RB], x1[RB];
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        const DevBuf o(a.att_o + (it0 + step * (s0 + min(j0 + j, ns - 1))) * 2048, 8192);
        x0[j] = __builtin_bit_cast(f32x4, o.load16((64 * kk + 16 * qq + c) * 16));
        x1[j] = __builtin_bit_cast(f32x4, o.load16((64 * kk + 64 + 16 * qq + c) * 16));
      }
      if (j0 == 0) {  // the weights of these 16 slots, in m
        if (sl >= nslot) m = -INFINITY;
        const float mn = fmaxf(M, rows_max(over_slots(m, vmax))), mz = mn == -INFINITY ? 0.f : mn;
        m = __builtin_amdgcn_exp2f(m - mz);
        const float fa = __builtin_amdgcn_exp2f(M - mz);
        L = L * fa + rows_sum(over_slots(sl < nslot ? l * m : 0.f, [](float x, float y) { return x + y; }));
        M = mn;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float f = lane_value(fa, i);
          o0[i] *= f;
          o1[i] *= f;
        }
      }
#pragma unroll
      for (int j = 0; j < RB; ++j)
        if (j0 + j < ns)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float f = lane_value(m, 4 * (j0 + j) + i);
            o0[i] += x0[j][i] * f;
            o1[i] += x1[j][i] * f;
          }
    }
  }
  const float inv = 1.0f / L;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (4 * qq + i < rows) {
      const float f = lane_value(inv, i);
      *reinterpret_cast<uint32_t*>(dst + (int64_t)(4 * qq + i) * a.A + 8 * c + kk) = pack_bf16x2(o0[i] * f, o1[i] * f);
    }
}

// The wave's number, known to be the same in its lanes (what depends on it stays in scalar registers).
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// The per-agent arrays of the kernel arguments, one agent per lane: one round trip for all of them, where scalar loads by
// agent wait for one another (arguments are cold in every launch).
struct AgentLanes {
  int len, prefix, prefix1;
  int64_t start;
  __device__ __forceinline__ AgentLanes(const TickParams& tp, int lane) {
    static_assert(FSX_MAX_BATCH == WAVE, "an agent per lane");
    len = tp.len[lane];
    prefix = tp.chunk_prefix[lane];
    prefix1 = tp.chunk_prefix[lane + 1];
    start = tp.start[lane];
  }
  static __device__ __forceinline__ int pick(int v, int b) { return __builtin_amdgcn_readlane(v, b); }
  __device__ __forceinline__ int64_t start_of(int b) const {
    return (int64_t)((uint64_t)(uint32_t)pick((int)(start >> 32), b) << 32 | (uint32_t)pick((int)start, b));
  }
};

// The end of a work item (one wave's state of 16 queries): the output itself if the agent has one chunk, else the state to
// its slot, and the merge by the wave that finishes last.  first, nslot: the agent's chunks; cs: this one (first <= cs).
__device__ __forceinline__ void finish_item(const AttnArgs& a, const TickParams& tp, const AttnState& st, int b, int h, int first,
                                            int nslot, int cs, int lane) {
  const int rows = tp.S;
  const int64_t item = (int64_t)cs * a.H + h;
  const float lt = rows_sum(st.l);
  uint16_t* out = a.attn_out + (int64_t)b * tp.S * a.A + (int64_t)h * a.Dh;
  if (nslot == 1) {
    write_output(a, st, lt, rows, lane, out);
    return;
  }
  store_state(a, item, st, lt, rows, lane);
  stores_done();
  uint32_t* cnt = a.acnt + (int64_t)b * a.H + h;
  uint32_t done = 0;
  if (lane == 0) done = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  done = (uint32_t)__builtin_amdgcn_readfirstlane((int)done);
  if (done != (uint32_t)(nslot - 1)) return;
  if (lane == 0) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  asm volatile("" ::: "memory");
  for (int qq = 0; 4 * qq < rows; ++qq)
    merge_queries(a, (int64_t)first * a.H + h, a.H, nslot, qq, rows, lane, out);
}

template <int KT>
__global__ __launch_bounds__(256) void k_attention(AttnArgs a, TickParams tp) {
  const int wave = wave_id(), lane = threadIdx.x & 63;
  const int item = blockIdx.x * (blockDim.x >> 6) + wave;
  if (item >= tp.n_items) return;
  const int h = item % a.H, cs = item / a.H;
  const AgentLanes al(tp, lane);
  const int b = __popcll(__ballot(lane < tp.B && al.prefix1 <= cs));
  const int first = al.pick(al.prefix, b), nslot = al.pick(al.prefix1, b) - first, cidx = cs - first, len = al.pick(al.len, b);
  const int grp = lane >> 4, c = lane & 15;
  const bool tv = c < tp.S;
  const int64_t qrow = ((int64_t)b * tp.S + (tv ? c : 0)) * a.A + (int64_t)h * a.Dh;
  uint4 qf[4];
  AttnState st;
#pragma unroll
  for (int k = 0; k < 8; ++k) st.o[k] = f32x4{0.f, 0.f, 0.f, 0.f};
  st.m = -INFINITY;
  st.l = 0.f;
  const int i0 = cidx * tp.chunk_rows, i1 = min(i0 + tp.chunk_rows, len);
  if (i0 < i1) {
    constexpr int ES = KT == 0 ? 2 : 1;
    // ring slot 0 of (agent, layer, head); slots are a.cv.rs elements apart
    const int64_t off = cache_head_base(a.cv, b, a.cv.layer, h) * ES;
    float ks = 1.f, vs = 1.f;
    if (KT == 1) {
      const int64_t si = cache_scale_index(a.cv, b, a.cv.layer, h);
      ks = a.cv.k_scale[si];
      vs = a.cv.v_scale[si];
    }
    load_q_frag<KT>(a.q, qrow, tv, grp, qf);
    // chunks start at rows equal modulo the chunk, rings are often a power of two: every item would stream addresses
    // equal modulo that, so each starts at a tile of its own
    const int n = (i1 - i0 + 31) / 32;
    attn_rows<KT, true>((const char*)a.cv.k + off, (const char*)a.cv.v + off, a.cv.rs * ES, al.start_of(b), a.cv.cap, i0, i1,
                        (int)((5u * h + 3u * b + cidx) % (unsigned)n), qf, ks, lane, st);
    if (KT == 1)
#pragma unroll
      for (int k = 0; k < 8; ++k) st.o[k] *= vs;
  }
  if (cidx == nslot - 1) {  // the new tokens' own rows (bf16)
    if (KT == 1 || i0 >= i1) load_q_frag<0>(a.q, qrow, tv, grp, qf);
    const int64_t off = ((int64_t)b * tp.S * a.A + (int64_t)h * a.Dh) * 2;
    attn_rows<0, false>((const char*)a.kself + off, (const char*)a.vself + off, (int64_t)a.A * 2, 0, 0, 0, tp.S, 0, qf, 1.f,
                        lane, st, a.causal ? 0 : 1 << 30);
  }
  finish_item(a, tp, st, b, h, first, nslot, cs, lane);
}

// The same for agents whose query tiles share their rows: several query tiles per agent, or several agents on one shared
// cache.  Workgroup = (head, group of up to ATT_Q query tiles, chunk of tp.chunk_rows rows): two loader waves bring the
// chunk's 32-row tiles of K and V into LDS by direct loads of whole rows, two tiles per step, three steps deep (as in
// k_gemm_rows: the loaders take the steps in turn), and each compute wave takes one query tile.  The own rows follow the
// cached ones in the list of tiles; on a shared cache, where they differ from agent to agent, each wave takes them by
// itself.  The last workgroup of a (head, group) merges its chunks, four queries per wave at a time.
// One wave per query tile reading its rows by itself fetched every tile once per query tile and had nothing in flight while
// it computed.  Per layer: 74 queries over 4,096 rows 111 -> 28 us (2 to the arguments, 4 to the first step, 13 for 17
// tiles -- 64 KiB in flight per CU, bound by memory -- and 6 to store and merge); the 40 blocks of a clip over one cache
// 40 -> 14; 74 queries over 16,000 fp8 rows 6,960 -> 3,670 per tick.  Six compute waves and two loaders: two waves per SIMD leave each 256 registers; with eight and
// four, 168 each, the tiles' operands spilled.
//
// Places of a lane's operands in a tile: k[kb] of row c (and 16 rows on) for channels 32 kb + 8 grp .., v[j] of row 4 grp + j
// (and 16 rows on) for channels 8 c ..  Kept in registers; computed at each use they were hoisted, once per use, and spilled.
template <int KT>
struct LdsPlaces {
  static constexpr int RB = KT == 0 ? 256 : 128;  // bytes of a row
  int k[4], v[4];
  static __device__ __forceinline__ int place(int row, int e) {
    return KT == 0 ? row * 256 + (((e >> 3) ^ (row & 15)) << 4) : row * 128 + (((e >> 4) ^ ((row >> 1) & 7)) << 4) + (e & 8);
  }
  __device__ __forceinline__ explicit LdsPlaces(int lane) {
    const int c = lane & 15, grp = lane >> 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      k[j] = place(c, 32 * j + 8 * grp);
      v[j] = place(4 * grp + j, 8 * c);
    }
  }
};

constexpr int AT_TILE = 16384;  // LDS of a tile: K rows, then V rows

// Rows [0, nv) of the NT 32-row tiles in LDS into the state; query c sees rows up to qmax + c.  The state's maximum moves
// only when a score exceeds it by more than 2^8 (or is the first), so probabilities stay below 2^8.
template <int KT, int NT>
__device__ __forceinline__ void attn_lds_tiles(const char* tile, int nv, int qmax, const uint4 (&qf)[4], float kscale, int lane,
                                               const LdsPlaces<KT>& at, AttnState& st) {
  constexpr int R16 = 16 * LdsPlaces<KT>::RB;
  const int c = lane & 15, grp = lane >> 4;
  f32x4 s[2 * NT];
#pragma unroll
  for (int r = 0; r < 2 * NT; ++r) {
    uint4 kf[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) kf[kb] = load8<KT>(tile + at.k[kb] + (r / 2 * AT_TILE + (r & 1) * R16));
    s[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) s[r] = KT == 0 ? mfma_bf16(kf[kb], qf[kb], s[r]) : mfma_f16(kf[kb], qf[kb], s[r]);
    if (KT == 1) s[r] *= kscale;
    if (r & 1) __builtin_amdgcn_sched_barrier(0);  // or the compiler has every operand in registers at once, and spills
  }
  const bool edge = nv < 32 * NT;
  if (edge || qmax < 32 * NT) {  // rows past the agent's, or of later new tokens: no weight
#pragma unroll
    for (int r = 0; r < 2 * NT; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int rr = 16 * r + 4 * grp + i;
        if (rr >= nv || rr > qmax + c) s[r][i] = -INFINITY;
      }
  }
  float mx = vmax(s[0][0], s[0][1]);
#pragma unroll
  for (int r = 0; r < 2 * NT; ++r) mx = vmax3(r ? vmax3(mx, s[r][0], s[r][1]) : mx, s[r][2], s[r][3]);
  mx = rows_max(mx);
  if (__any(mx > st.m + 8.0f)) {
    const float m_new = fmaxf(st.m, mx);
    const float alpha = __builtin_amdgcn_exp2f(st.m - (m_new == -INFINITY ? 0.f : m_new));
    st.l *= alpha;
    st.m = m_new;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a_i = col_pick(alpha, grp, i);
#pragma unroll
      for (int k = 0; k < 8; ++k) st.o[k][i] *= a_i;
    }
  }
  const float mz = st.m == -INFINITY ? 0.f : st.m;  // no row seen yet
  float ps = 0.f;
#pragma unroll
  for (int r = 0; r < 2 * NT; ++r)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[r][i] = __builtin_amdgcn_exp2f(s[r][i] - mz);
      ps += s[r][i];
    }
  st.l += ps;
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    uint4 vr[8], vt[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) vr[j] = load8<KT>(tile + at.v[j & 3] + (u * AT_TILE + 8192 + (j >> 2) * R16));
    if (edge)  // the values of rows past the agent's are not the agent's
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (32 * u + (j < 4 ? 4 * grp + j : 12 + 4 * grp + j) >= nv) vr[j] = make_uint4(0, 0, 0, 0);
    const f32x4 p0 = s[2 * u], p1 = s[2 * u + 1];
    uint4 pf;
    if (KT == 0)
      pf = make_uint4(pack_bf16x2(p0[0], p0[1]), pack_bf16x2(p0[2], p0[3]), pack_bf16x2(p1[0], p1[1]), pack_bf16x2(p1[2], p1[3]));
    else
      pf = make_uint4(pack_f16x2(p0[0], p0[1]), pack_f16x2(p0[2], p0[3]), pack_f16x2(p1[0], p1[1]), pack_f16x2(p1[2], p1[3]));
    transpose8x8_b16(vr, vt);
#pragma unroll
    for (int k = 0; k < 8; ++k) st.o[k] = KT == 0 ? mfma_bf16(pf, vt[k], st.o[k]) : mfma_f16(pf, vt[k], st.o[k]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

template <int KT>
__global__ __launch_bounds__((ATT_Q + 2) * 64) void k_attention_tiles(AttnArgs a, TickParams tp) {
  __shared__ __align__(16) char at_lds[3 * 2 * AT_TILE];  // three buffers of two tiles
  __shared__ uint32_t last;
  const int wave = wave_id(), lane = threadIdx.x & 63, grp = lane >> 4, c = lane & 15;
  const AgentLanes al(tp, lane);
  const int h = blockIdx.x % a.H, rest = blockIdx.x / a.H, n_groups = tp.att_groups, g = rest % n_groups, cidx = rest / n_groups;
  const bool shared = tp.att_shared;
  const int qg = tp.att_qg, gpa = shared ? 1 : n_groups / tp.B;  // query tiles of a group, groups of an agent
  const int q0 = shared ? g * qg : (g % gpa) * qg, q1 = min(q0 + qg, shared ? tp.B * tp.n_tt : tp.n_tt);
  auto agent_of = [&](int q) { return shared ? q / tp.n_tt : g / gpa; };
  const int b_first = agent_of(q0), per = tp.chunk_rows / 32, own_tiles = shared ? 0 : (tp.S + 31) / 32;
  int len_max = 0;  // of the group's agents
  for (int b = b_first; b <= agent_of(q1 - 1); ++b) len_max = max(len_max, al.pick(al.len, b));
  const int nt = (len_max + 31) / 32 + own_tiles;
  const int t0 = cidx * per, n = min(per, nt - t0);  // this chunk's tiles t0 .. t0 + n - 1
  if (n <= 0 && cidx > 0) return;
  const int ns = (n + 1) / 2, n_chunks = max(1, (nt + per - 1) / per);
  if (wave >= qg) {
    constexpr int ES = KT == 0 ? 2 : 1;
    const int par = wave - qg;
    const int64_t cap = a.cv.cap, start = shared ? tp.att_start : al.start_of(b_first);
    const int64_t off = cache_head_base(a.cv, b_first, a.cv.layer, h) * ES;
    const int ct = nt - own_tiles;
    // step i, 16-byte chunk k of row r at position k ^ (r & 15) (fp8: k ^ ((r >> 1) & 7)), so that the rows of an operand
    // read fall in distinct banks
    auto stage = [&](int i) {
      for (int u = 0; u < 2 && 2 * i + u < n; ++u) {
        const int t = t0 + 2 * i + u;
        char* dst = at_lds + (i % 3 * 2 + u) * AT_TILE;
        if (t < ct) {
          constexpr int RPI = KT == 0 ? 4 : 8, CPR = 64 / RPI;  // rows of a load, 16-byte chunks of a row
#pragma unroll
          for (int q = 0; q < 32 / RPI; ++q) {
            const int r = q * RPI + lane / CPR, ch = (lane % CPR) ^ (KT == 0 ? r & 15 : (r >> 1) & 7);
            int64_t slot = start + min(32 * t + r, len_max - 1);
            if (slot >= cap) slot -= cap;
            const int64_t src = off + slot * a.cv.rs * ES + ch * 16;
            load_lds16<false>((const char*)a.cv.k + src, dst + q * 1024);
            load_lds16<false>((const char*)a.cv.v + src, dst + 8192 + q * 1024);
          }
        } else {
          const int64_t base = (int64_t)b_first * tp.S * a.A + (int64_t)h * a.Dh;
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const int r = q * 4 + grp, ch = c ^ (r & 15);
            const int64_t src = base + (int64_t)min(32 * (t - ct) + r, tp.S - 1) * a.A + ch * 8;
            load_lds16<false>(a.kself + src, dst + q * 1024);
            load_lds16<false>(a.vself + src, dst + 8192 + q * 1024);
          }
        }
      }
    };
    if (par < ns) stage(par);
    if (par == 0) vm_wait_all();
    wg_barrier();
    for (int i = 0; i + 1 < ns; ++i) {  // while step i is computed
      if ((i & 1) == par) {
        if (i + 2 < ns) stage(i + 2);
      } else {
        vm_wait_all();  // step i + 1
      }
      wg_barrier();
    }
  } else {
    const bool active = q0 + wave < q1;
    const int q = min(q0 + wave, q1 - 1), b = agent_of(q), tt = shared ? q % tp.n_tt : q;  // this wave's query tile
    const int len = al.pick(al.len, b), ct = (len + 31) / 32;
    const int first = al.pick(al.prefix, b), nslot = al.pick(al.prefix1, b) - first;
    const int t = tt * 16 + c;
    const bool tv = t < tp.S;
    const int64_t qrow = ((int64_t)b * tp.S + (tv ? t : 0)) * a.A + (int64_t)h * a.Dh;
    AttnState st;
#pragma unroll
    for (int k = 0; k < 8; ++k) st.o[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    st.m = -INFINITY;
    st.l = 0.f;
    float ks = 1.f, vs = 1.f;
    if (KT == 1 && len > 0) {
      const int64_t si = cache_scale_index(a.cv, b, a.cv.layer, h);
      ks = a.cv.k_scale[si];
      vs = a.cv.v_scale[si];
    }
    uint4 qf[4];
    load_q_frag<KT>(a.q, qrow, tv, grp, qf);
    const LdsPlaces<KT> at(lane);
    const LdsPlaces<0> at_own(lane);
    bool codes = KT == 1;  // the state still counts cached rows in codes, the queries are in fp16
    auto to_own = [&]() {
      if (KT == 1 && codes) {
        codes = false;
#pragma unroll
        for (int k = 0; k < 8; ++k) st.o[k] *= vs;
        load_q_frag<0>(a.q, qrow, tv, grp, qf);
      }
    };
    wg_barrier();
    for (int i = 0; i < ns; ++i) {
      const int ti = t0 + 2 * i, nu = min(2, n - 2 * i);
      const char* tile = at_lds + i % 3 * 2 * AT_TILE;
      if (active) {
        // both tiles of the step at once where they are of one kind
        const int nc = max(0, min(nu, ct - ti));  // cached ones
        if (nc == 2)
          attn_lds_tiles<KT, 2>(tile, min(64, len - 32 * ti), 64, qf, ks, lane, at, st);
        else if (nc == 1)
          attn_lds_tiles<KT, 1>(tile, min(32, len - 32 * ti), 32, qf, ks, lane, at, st);
        if (!shared && nc < nu) {
          to_own();
          const int r0 = 32 * (ti + nc - ct), qmax = a.causal ? tt * 16 - r0 : 64;
          if (qmax + 15 >= 0) {
            if (nu - nc == 2)
              attn_lds_tiles<0, 2>(tile, min(64, tp.S - r0), qmax, qf, 1.f, lane, at_own, st);
            else
              attn_lds_tiles<0, 1>(tile + nc * AT_TILE, min(32, tp.S - r0), qmax, qf, 1.f, lane, at_own, st);
          }
        }
      }
      if (i + 1 < ns) wg_barrier();
    }
    if (shared && active && cidx == nslot - 1) {  // the own rows of this wave's agent
      to_own();
      const int64_t off = ((int64_t)b * tp.S * a.A + (int64_t)h * a.Dh) * 2;
      attn_rows<0, false>((const char*)a.kself + off, (const char*)a.vself + off, (int64_t)a.A * 2, 0, 0, 0, tp.S, 0, qf, 1.f,
                          lane, st, a.causal ? tt * 16 : 1 << 30);
    }
    if (KT == 1 && codes)
#pragma unroll
      for (int k = 0; k < 8; ++k) st.o[k] *= vs;
    if (active && cidx < nslot) {
      const int rows = min(16, tp.S - tt * 16);
      const float lt = rows_sum(st.l);
      if (nslot == 1)
        write_output(a, st, lt, rows, lane, a.attn_out + ((int64_t)b * tp.S + tt * 16) * a.A + (int64_t)h * a.Dh);
      else
        store_state(a, ((int64_t)(first + cidx) * a.H + h) * tp.n_tt + tt, st, lt, rows, lane);
    }
  }
  if (n_chunks == 1) return;
  // the last workgroup of the (head, group) merges
  stores_done();
  wg_barrier();
  if (threadIdx.x == 0) {
    uint32_t* cnt = a.acnt + (int64_t)g * a.H + h;
    last = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(n_chunks - 1);
    if (last) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!last) return;
  const int64_t step = (int64_t)a.H * tp.n_tt;
  for (int i = wave; i < 4 * (q1 - q0); i += qg + 2) {
    const int q = q0 + (i >> 2), qq = i & 3, b = agent_of(q), tt = shared ? q % tp.n_tt : q, rows = min(16, tp.S - tt * 16);
    const int first = al.pick(al.prefix, b), nslot = al.pick(al.prefix1, b) - first;
    if (nslot > 1 && 4 * qq < rows)
      merge_queries(a, (int64_t)first * step + (int64_t)h * tp.n_tt + tt, step, nslot, qq, rows, lane,
                    a.attn_out + ((int64_t)b * tp.S + tt * 16) * a.A + (int64_t)h * a.Dh);
  }
}

hipError_t launch_attention(const CacheView& cv, const TickParams& tp, const Dims& dm, const Workspace& ws,
                            hipStream_t s, bool causal) {
  AttnArgs a{};
  a.cv = cv; a.q = ws.q; a.kself = ws.kself; a.vself = ws.vself; a.att_o = ws.att_o; a.att_ml = ws.att_ml;
  a.acnt = ws.acnt; a.attn_out = ws.attn; a.H = dm.H; a.Dh = dm.Dh; a.A = dm.A; a.causal = causal ? 1 : 0;
  if (tp.att_groups) {
    const auto fn = cv.dtype == FSX_FP8_E4M3 ? k_attention_tiles<1> : k_attention_tiles<0>;
    hipLaunchKernelGGL(fn, dim3((unsigned)(dm.H * tp.att_groups * tp.att_chunks)), dim3(64 * (tp.att_qg + 2)), 0, s, a, tp);
    return hipGetLastError();
  }
  const int wpg = tp.n_items >= 1024 ? 4 : 1;
  const dim3 grid((unsigned)((tp.n_items + wpg - 1) / wpg)), block(64 * wpg);
  if (cv.dtype == FSX_FP8_E4M3)
    hipLaunchKernelGGL(k_attention<1>, grid, block, 0, s, a, tp);
  else
    hipLaunchKernelGGL(k_attention<0>, grid, block, 0, s, a, tp);
  return hipGetLastError();
}

// The layer's new rows (kself / vself) into the cache rings, by the workgroups of a reduction past its own (the first
// launch after the attention has read the old rows, which a full ring overwrites).
struct RowsInto {
  CacheView cv;
  const uint16_t* ks;
  const uint16_t* vs;
  int32_t B, n;
  int64_t first[FSX_MAX_BATCH];  // ring slot of each agent's first new row
};
__device__ __forceinline__ void write_row_chunk(const RowsInto& w, int64_t i);

// =====================================================================================================
// h += sum of split-K partials (fixed order), optional copy to the per-layer hidden output, then
// x = bf16(h / rms(h)) for the next projection (whose packed weights carry the norm gain).  One workgroup
// per token row.
// =====================================================================================================
constexpr int RN_T = 128;
// The sum of ksplit partials of four columns, every load issued before any add (in order of the partials).
__device__ __forceinline__ float4 sum_partials(const float* __restrict__ part, int64_t idx, int64_t stride, int ksplit) {
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int s0 = 0; s0 < ksplit; s0 += 8) {
    float4 v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
      v[j] = s0 + j < ksplit ? *reinterpret_cast<const float4*>(part + (s0 + j) * stride + idx) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      acc.x += v[j].x;
      acc.y += v[j].y;
      acc.z += v[j].z;
      acc.w += v[j].w;
    }
  }
  return acc;
}

template <bool ROWS>
__global__ __launch_bounds__(RN_T) void k_reduce_norm(float* __restrict__ h, const float* __restrict__ part,
                                                      uint16_t* __restrict__ xb, int M, int d, int ksplit, float eps,
                                                      float* __restrict__ hidden, RowsInto w) {
  __shared__ float red[16];
  const int m = blockIdx.x;
  if (ROWS && m >= M) {
    write_row_chunk(w, (int64_t)(m - M) * blockDim.x + threadIdx.x);
    return;
  }
  float ss = 0.f;
  float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int n = 4 * threadIdx.x; n < d; n += 4 * RN_T) {
    const int64_t idx = (int64_t)m * d + n;
    const float4 h0 = *reinterpret_cast<const float4*>(h + idx);
    const float4 acc = sum_partials(part, idx, (int64_t)M * d, ksplit);
    val = make_float4(h0.x + acc.x, h0.y + acc.y, h0.z + acc.z, h0.w + acc.w);
    *reinterpret_cast<float4*>(h + idx) = val;
    if (hidden) {  // the caller's buffer: 4-byte alignment only
      hidden[idx] = val.x;
      hidden[idx + 1] = val.y;
      hidden[idx + 2] = val.z;
      hidden[idx + 3] = val.w;
    }
    ss += val.x * val.x + val.y * val.y + val.z * val.z + val.w * val.w;
  }
  ss = block_sum(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)d + eps);
  for (int n = 4 * threadIdx.x; n < d; n += 4 * RN_T) {
    const int64_t idx = (int64_t)m * d + n;
    if (d > 4 * RN_T) val = *reinterpret_cast<const float4*>(h + idx);
    // the gain is folded into the packed weights
    *reinterpret_cast<uint2*>(xb + idx) = make_uint2(pack_bf16x2(val.x * r, val.y * r), pack_bf16x2(val.z * r, val.w * r));
  }
}

// Wide rows (the backbone's d = 4096 over a handful of tokens): one workgroup per row leaves the partial sums'
// loads latency-bound on a few CUs, so the rows are cut into 512-column chunks, one workgroup each: h += sum of the
// partials, xb = bf16(h) unscaled, and the chunk's sum of squares to ss[m][chunk]; the last chunk of the row forms
// the row's RMSNorm scale, which the next projection applies to its products, so no launch forms the normalised
// input.
template <bool ROWS>
__global__ __launch_bounds__(RN_CHUNK / 4) void k_reduce_chunks(float* __restrict__ h, const float* __restrict__ part,
                                                                int M, int d, int ksplit, float* __restrict__ ss,
                                                                uint16_t* __restrict__ xb, float* __restrict__ hidden,
                                                                float* __restrict__ rs, uint32_t* __restrict__ rcnt,
                                                                float eps, RowsInto w) {
  __shared__ float red[16];
  const int nch = d / RN_CHUNK, m = blockIdx.x / nch, ch = blockIdx.x % nch;
  if (ROWS && m >= M) {
    write_row_chunk(w, (int64_t)(blockIdx.x - M * nch) * blockDim.x + threadIdx.x);
    return;
  }
  // thread t: the 4 columns ch * RN_CHUNK + 4t .. + 3, 16-byte loads (every partial's load issued before any add)
  const int64_t idx = (int64_t)m * d + ch * RN_CHUNK + 4 * threadIdx.x;
  const float4 acc = sum_partials(part, idx, (int64_t)M * d, ksplit);
  const float4 h0 = *reinterpret_cast<const float4*>(h + idx);
  const float4 val = make_float4(h0.x + acc.x, h0.y + acc.y, h0.z + acc.z, h0.w + acc.w);
  *reinterpret_cast<float4*>(h + idx) = val;
  *reinterpret_cast<uint2*>(xb + idx) = make_uint2(pack_bf16x2(val.x, val.y), pack_bf16x2(val.z, val.w));
  if (hidden) {  // the caller's buffer: 4-byte alignment only
    hidden[idx] = val.x;
    hidden[idx + 1] = val.y;
    hidden[idx + 2] = val.z;
    hidden[idx + 3] = val.w;
  }
  float sq = val.x * val.x + val.y * val.y + val.z * val.z + val.w * val.w;
  sq = block_sum(sq, red);
  // the last chunk of row m to finish adds the chunk sums in chunk order and writes the row's scale; it then resets
  // the row's counter for the next reduction (the next launch).  The sums are device-scope stores completed before
  // the count (no release fence: at device scope that writes back the whole L2) and read with device-scope loads.
  if (threadIdx.x == 0) {
    st_dev_f(ss + (int64_t)m * nch + ch, sq);
    stores_done();
    const uint32_t done = __hip_atomic_fetch_add(rcnt + m, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (done == (uint32_t)(nch - 1)) {
      float tot = 0.f;
      for (int c = 0; c < nch; ++c) tot += ld_dev_f(ss + (int64_t)m * nch + c);
      rs[m] = 1.0f / sqrtf(tot / (float)d + eps);
      __hip_atomic_store(rcnt + m, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

hipError_t launch_reduce_norm(const TickParams& tp, const Dims& dm, const Workspace& ws, int ksplit,
                              const float* gain, float* hidden_layer, hipStream_t s, const CacheView* rows_into) {
  RowsInto w{};
  int64_t chunks = 0;
  if (rows_into) {
    w.cv = *rows_into; w.ks = ws.kself; w.vs = ws.vself; w.B = tp.B; w.n = tp.S;
    for (int b = 0; b < tp.B; ++b) w.first[b] = (tp.start[b] + tp.len[b]) % rows_into->cap;
    chunks = (int64_t)tp.B * tp.S * rows_into->H * (rows_into->Dh / 8);
  }
  const int nt = wide_rows(dm) ? RN_CHUNK / 4 : RN_T, own = wide_rows(dm) ? tp.M * (dm.d / RN_CHUNK) : tp.M;
  const dim3 grid((unsigned)(own + (chunks + nt - 1) / nt)), block(nt);
  if (wide_rows(dm)) {
    const auto fn = rows_into ? k_reduce_chunks<true> : k_reduce_chunks<false>;
    hipLaunchKernelGGL(fn, grid, block, 0, s, ws.h, (const float*)ws.part, tp.M, dm.d, ksplit, ws.ss, ws.xb, hidden_layer,
                       ws.rs, ws.rcnt, dm.eps, w);
  } else {
    const auto fn = rows_into ? k_reduce_norm<true> : k_reduce_norm<false>;
    hipLaunchKernelGGL(fn, grid, block, 0, s, ws.h, (const float*)ws.part, ws.xb, tp.M, dm.d, ksplit, dm.eps,
                       hidden_layer, w);
  }
  return hipGetLastError();
}

// =====================================================================================================
// Waypoint head: mean over the first T tokens of RMSNorm(h) * g_final, then W_head [n_out][d] (no bias).
// One workgroup per agent.  Dynamic LDS: d floats.
// =====================================================================================================
__global__ __launch_bounds__(256) void k_head(const float* __restrict__ h, int S, int T, int d, float eps,
                                              const float* __restrict__ gfin, const void* __restrict__ w,
                                              int wdtype, int n_out, float* __restrict__ wp) {
  extern __shared__ float xm[];
  mean_head_wg(h, S, T, d, eps, gfin, w, wdtype, n_out, wp, xm);
}

__global__ __launch_bounds__(256) void k_query_head(const float* __restrict__ h, int S, int T, int d, float eps,
                                                    const float* __restrict__ gfin, QueryHead qh, int nq,
                                                    float* __restrict__ wp) {
  extern __shared__ float qlds[];
  const int b = blockIdx.x;
  query_head_wg([&](int t, int c) { return h[((int64_t)b * S + t) * d + c]; }, T, nq, d, eps, gfin, qh,
                [&](int o, float v) { wp[(int64_t)b * 2 * nq + o] = v; }, qlds);
}

hipError_t launch_query_head(const float* h, const TickParams& tp, const Dims& dm, const float* final_norm,
                             const QueryHead& qh, float* waypoints, hipStream_t s) {
  const int nq = dm.n_out / 2;
  hipLaunchKernelGGL(k_query_head, dim3(tp.B), dim3(256), (size_t)nq * (dm.d + 256) * sizeof(float), s, h,
                     tp.S, tp.T, dm.d, dm.eps, final_norm, qh, nq, waypoints);
  return hipGetLastError();
}

hipError_t launch_head(const TickParams& tp, const Dims& dm, const Workspace& ws, const float* final_norm,
                       const void* head_w, int head_dtype, float* waypoints, hipStream_t s) {
  hipLaunchKernelGGL(k_head, dim3(tp.B), dim3(256), dm.d * sizeof(float), s, (const float*)ws.h, tp.S, tp.T, dm.d,
                     dm.eps, final_norm, head_w, head_dtype, dm.n_out, waypoints);
  return hipGetLastError();
}

// =====================================================================================================
// Cache append (Sec. 3.3): copy n new rows of every (agent, layer, head) into ring slots
// (first[b] + j) mod cap, bit-exact, 16 bytes per thread.  The rows come in the cache's layout with n slots:
// head-major [B][n_layers][H][n][Dh] into [B][n_layers][H][cap][Dh], or token-major [B][n_layers][n][H][Dh] into
// [B][n_layers][cap][H][Dh].  Either way thread i copies 16-byte chunk i of the source, so reads are coalesced.
// =====================================================================================================
struct AppendArgs {
  const uint4* ks;
  const uint4* vs;
  uint4* kc;
  uint4* vc;
  int64_t cap;
  int64_t row_chunks;  // 16-byte chunks per head row (Dh elements)
  int n_layers, n_heads, n_rows, B, token_major;
  int64_t first[FSX_MAX_BATCH];
};

__global__ __launch_bounds__(256) void k_append(AppendArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)a.B * a.n_layers * a.n_heads * a.n_rows * a.row_chunks;
  if (i >= total) return;
  const int64_t ch = i % a.row_chunks;
  int64_t r = i / a.row_chunks;
  int64_t dst;
  if (a.token_major) {
    const int h = (int)(r % a.n_heads);
    r /= a.n_heads;
    const int j = (int)(r % a.n_rows);
    r /= a.n_rows;  // (b, l)
    const int b = (int)(r / a.n_layers);
    int64_t slot = a.first[b] + j;
    if (slot >= a.cap) slot -= a.cap;
    dst = ((r * a.cap + slot) * a.n_heads + h) * a.row_chunks + ch;
  } else {
    const int j = (int)(r % a.n_rows);
    r /= a.n_rows;  // (b, l, h) slab index
    const int b = (int)(r / ((int64_t)a.n_layers * a.n_heads));
    int64_t slot = a.first[b] + j;
    if (slot >= a.cap) slot -= a.cap;
    dst = (r * a.cap + slot) * a.row_chunks + ch;
  }
  a.kc[dst] = a.ks[i];
  a.vc[dst] = a.vs[i];
}

// Quantising append into an fp8 cache: the rows arrive in bf16 or fp32 and each element is stored as the E4M3 code
// RNE(clamp(x / scale, -448, 448)) with the (agent, layer, head) scale the cache already has.  The encoding follows
// the format's definition step by step (exact in fp32: the quotient is rounded once by the division, the mantissa
// rounding is a rint of an exactly scaled value), so the codes are reproducible bit for bit.
__device__ __forceinline__ uint32_t e4m3_encode(float x, float scale) {
  float y = x / scale;
  if (y != y) return 0x7Fu | (__float_as_uint(y) >> 31 << 7);
  y = fminf(fmaxf(y, -448.0f), 448.0f);
  const uint32_t sign = __float_as_uint(y) >> 31 << 7;
  const float a = fabsf(y);
  uint32_t code;
  if (a < 0.015625f) {  // below the smallest normal 2^-6: subnormal steps of 2^-9
    code = (uint32_t)rintf(a * 512.0f);  // 8 -> the smallest normal, code 0x08
  } else {
    int e;
    const float m = frexpf(a, &e);  // a = m 2^e, m in [0.5, 1)
    uint32_t mant = (uint32_t)rintf((m * 2.0f - 1.0f) * 8.0f);
    int ex = e - 1;
    if (mant == 8) {
      mant = 0;
      ++ex;
    }
    code = ((uint32_t)(ex + 7) << 3) | mant;
  }
  return sign | code;
}

struct QAppendArgs {
  const void* ks;
  const void* vs;
  uint8_t* kc;
  uint8_t* vc;
  const float* kscale;
  const float* vscale;
  int64_t cap;
  int n_layers, n_heads, head_dim, n_rows, B, token_major, src_f32;
  int64_t first[FSX_MAX_BATCH];
};

// Thread i encodes 8 consecutive elements of one head row (8 bytes out).
__global__ __launch_bounds__(256) void k_append_quantize(QAppendArgs a) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int cpr = a.head_dim / 8;
  const int64_t total = (int64_t)a.B * a.n_layers * a.n_heads * a.n_rows * cpr;
  if (i >= total) return;
  const int ch = (int)(i % cpr);
  int64_t r = i / cpr;
  int b, l, h, j;
  if (a.token_major) {
    h = (int)(r % a.n_heads);
    r /= a.n_heads;
    j = (int)(r % a.n_rows);
    r /= a.n_rows;
    l = (int)(r % a.n_layers);
    b = (int)(r / a.n_layers);
  } else {
    j = (int)(r % a.n_rows);
    r /= a.n_rows;
    h = (int)(r % a.n_heads);
    r /= a.n_heads;
    l = (int)(r % a.n_layers);
    b = (int)(r / a.n_layers);
  }
  int64_t slot = a.first[b] + j;
  if (slot >= a.cap) slot -= a.cap;
  const int64_t lb = ((int64_t)b * a.n_layers + l);
  const int64_t dst = a.token_major ? ((lb * a.cap + slot) * a.n_heads + h) * a.head_dim + 8 * ch
                                    : ((lb * a.n_heads + h) * a.cap + slot) * a.head_dim + 8 * ch;
  const float sk = a.kscale[lb * a.n_heads + h], sv = a.vscale[lb * a.n_heads + h];
  const int64_t src = i * 8;  // the source rows are dense in the same order as i
  float xk[8], xv[8];
  if (a.src_f32) {
    const float4* pk = reinterpret_cast<const float4*>((const float*)a.ks + src);
    const float4* pv = reinterpret_cast<const float4*>((const float*)a.vs + src);
    const float4 k0 = pk[0], k1 = pk[1], v0 = pv[0], v1 = pv[1];
    const float kk[8] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w};
    const float vv[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      xk[e] = kk[e];
      xv[e] = vv[e];
    }
  } else {
    const uint4 k = *reinterpret_cast<const uint4*>((const uint16_t*)a.ks + src);
    const uint4 v = *reinterpret_cast<const uint4*>((const uint16_t*)a.vs + src);
    const uint32_t kw[4] = {k.x, k.y, k.z, k.w}, vw[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xk[2 * e] = __uint_as_float(kw[e] << 16);
      xk[2 * e + 1] = __uint_as_float(kw[e] & 0xFFFF0000u);
      xv[2 * e] = __uint_as_float(vw[e] << 16);
      xv[2 * e + 1] = __uint_as_float(vw[e] & 0xFFFF0000u);
    }
  }
  uint32_t ck[2] = {0, 0}, cv[2] = {0, 0};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ck[e >> 2] |= e4m3_encode(xk[e], sk) << (8 * (e & 3));
    cv[e >> 2] |= e4m3_encode(xv[e], sv) << (8 * (e & 3));
  }
  *reinterpret_cast<uint2*>(a.kc + dst) = make_uint2(ck[0], ck[1]);
  *reinterpret_cast<uint2*>(a.vc + dst) = make_uint2(cv[0], cv[1]);
}

hipError_t launch_append_quantize(const fsx_cache_desc& c, const void* k_rows, const void* v_rows, int rows_dtype,
                                  int n_rows, const int64_t* first, hipStream_t s) {
  QAppendArgs a{};
  a.ks = k_rows; a.vs = v_rows; a.kc = (uint8_t*)c.k; a.vc = (uint8_t*)c.v; a.kscale = c.k_scale; a.vscale = c.v_scale;
  a.cap = c.capacity; a.n_layers = c.n_layers; a.n_heads = c.n_heads; a.head_dim = c.head_dim; a.n_rows = n_rows;
  a.B = c.batch; a.token_major = (c.layout & FSX_CACHE_TOKEN_MAJOR) != 0; a.src_f32 = rows_dtype == FSX_F32;
  for (int b = 0; b < c.batch; ++b) a.first[b] = first[b];
  const int64_t total = (int64_t)a.B * a.n_layers * a.n_heads * a.n_rows * (a.head_dim / 8);
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_append_quantize, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Chunk i (8 elements) of the new rows [B][n][H][Dh] (kself / vself: bf16, rotated; row b * n + t) into ring slot
// (first[b] + t) mod capacity of (agent b, layer cv.layer, head h): a bf16 copy, or E4M3 codes with the cache's
// per-(agent, layer, head) scales.
__device__ __forceinline__ void write_row_chunk(const RowsInto& w, int64_t i) {
  const CacheView& cv = w.cv;
  const int cpr = cv.Dh / 8, A = cv.H * cv.Dh, n = w.n;
  const int64_t total = (int64_t)w.B * n * cv.H * cpr;
  if (i >= total) return;
  const int ch = (int)(i % cpr);
  int64_t r = i / cpr;
  const int h = (int)(r % cv.H);
  const int64_t m = r / cv.H;  // token row b * n + t
  const int b = (int)(m / n), t = (int)(m % n);
  int64_t slot = w.first[b] + t;
  if (slot >= cv.cap) slot -= cv.cap;
  const int64_t dst = cache_head_base(cv, b, cv.layer, h) + slot * cv.rs + 8 * ch;
  const int64_t src = m * A + (int64_t)h * cv.Dh + 8 * ch;
  const uint4 kv = *reinterpret_cast<const uint4*>(w.ks + src), vv = *reinterpret_cast<const uint4*>(w.vs + src);
  if (cv.dtype == FSX_FP8_E4M3) {
    const int64_t si = cache_scale_index(cv, b, cv.layer, h);
    const float sk = cv.k_scale[si], sv = cv.v_scale[si];
    const uint32_t kw[4] = {kv.x, kv.y, kv.z, kv.w}, vw[4] = {vv.x, vv.y, vv.z, vv.w};
    uint32_t ck[2] = {0, 0}, cvw[2] = {0, 0};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t kbits = e & 1 ? kw[e >> 1] & 0xFFFF0000u : kw[e >> 1] << 16;
      const uint32_t vbits = e & 1 ? vw[e >> 1] & 0xFFFF0000u : vw[e >> 1] << 16;
      ck[e >> 2] |= e4m3_encode(__uint_as_float(kbits), sk) << (8 * (e & 3));
      cvw[e >> 2] |= e4m3_encode(__uint_as_float(vbits), sv) << (8 * (e & 3));
    }
    *reinterpret_cast<uint2*>((uint8_t*)cv.k + dst) = make_uint2(ck[0], ck[1]);
    *reinterpret_cast<uint2*>((uint8_t*)cv.v + dst) = make_uint2(cvw[0], cvw[1]);
  } else {
    *reinterpret_cast<uint4*>((uint16_t*)cv.k + dst) = kv;
    *reinterpret_cast<uint4*>((uint16_t*)cv.v + dst) = vv;
  }
}

hipError_t launch_append(const fsx_cache_desc& c, const void* k_rows, const void* v_rows, int n_rows,
                         const int64_t* first, hipStream_t s) {
  AppendArgs a{};
  const int es = c.dtype == FSX_F32 ? 4 : (c.dtype == FSX_BF16 ? 2 : 1);
  a.ks = (const uint4*)k_rows; a.vs = (const uint4*)v_rows; a.kc = (uint4*)c.k; a.vc = (uint4*)c.v;
  a.cap = c.capacity; a.row_chunks = (int64_t)c.head_dim * es / 16;
  a.n_layers = c.n_layers; a.n_heads = c.n_heads; a.n_rows = n_rows; a.B = c.batch;
  a.token_major = (c.layout & FSX_CACHE_TOKEN_MAJOR) != 0;
  for (int b = 0; b < c.batch; ++b) a.first[b] = first[b];
  const int64_t total = (int64_t)a.B * a.n_layers * a.n_heads * a.n_rows * a.row_chunks;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_append, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace fsx

namespace fsx {

// =====================================================================================================
// Zero fill of a device range (a kernel, not a memset, so that it is an ordinary kernel node when the caller
// captures the stream into a graph).  Whole 16-byte chunks; `bytes` is a multiple of 256.
// =====================================================================================================
__global__ __launch_bounds__(256) void k_fill_zero(uint4* p, int64_t n16) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = make_uint4(0, 0, 0, 0);
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s) {
  const int64_t n16 = (int64_t)(bytes / 16);
  if (n16 == 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n16 + 255) / 256, 2048);
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)blocks), dim3(256), 0, s, (uint4*)p, n16);
  return hipGetLastError();
}

}  // namespace fsx
