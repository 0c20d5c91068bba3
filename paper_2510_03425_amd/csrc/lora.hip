// Rank-r LoRA products on MFMA (gfx950): the adapter's down-projection u = X A^T, the
// gradient projection du = s dY B (both "rows": r <= 16 outputs per token, reduction over
// the model dimension), and the weight gradients dB = s dY^T u, dA = du^T X ("outer":
// reduction over tokens). Up to three projections that share a stage of the layer (q, k,
// v; gate, up) run in one launch.
//
// The 16-bit activation / gradient operand is used as stored; the fp32 adapter weights
// (A, B) and fp32 u / du enter the MFMA as a hi + lo pair of 16-bit values (two MFMAs),
// which keeps their operand rounding near 2^-17 instead of 2^-9.
//
// "rows" keeps the whole reduction inside one workgroup (its waves split K, partial
// tiles summed through LDS in wave order). "outer" splits the token range over
// the grid when there are many tokens; the split partials are then summed in split
// order by a small reduce kernel. Both are deterministic.
#include <algorithm>

#include "device_common.h"
#include "mebp_internal.h"

namespace mebp {
namespace {

typedef uint16_t u16;

template <class Op>
DEV void split_hi_lo(const float (&f)[8], uint4& hi, uint4& lo) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = Op::pack(f[2 * i], f[2 * i + 1]);
    l[i] = Op::pack(f[2 * i] - Op::lo(h[i]), f[2 * i + 1] - Op::hi(h[i]));
  }
  hi = make_uint4(h[0], h[1], h[2], h[3]);
  lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// ------------------------------------------------------------------------------ rows
// out[m][j] = s * sum_k X[m][k] W(j,k); workgroup = 16 RT rows x 16 outputs and LR_WAVES waves
// that take interleaved 64-wide K super-steps (every row segment a lane group loads is 128
// contiguous bytes), two super-steps in flight per iteration (one with three jobs of 64 rows);
// the per-wave partial tiles are summed through LDS in wave order. Bound by the stream of X at
// many tokens; at few, by the workgroups that run: RT is the largest of 4, 2, 1 that still gives
// 256 of them (4096 tokens, K = 8960: 64 rows are 64 workgroups and 50 us = 1.5 TB/s, 16 rows
// 256 and 31 us; 16384 tokens, K = 10240, two jobs: 187 us = 3.6 TB/s with 64 rows).
// NJ = 1: blockIdx.y selects the job. NJ > 1: the NJ jobs share X (the q, k, v or gate, up
// down-projections of one normalised input), read once for all of them.
constexpr int LR_WAVES = 8;
template <class Op, int NJ, int RT>
__global__ __launch_bounds__(64 * LR_WAVES) void k_lora_rows(const LoraRowsArgs a) {
  constexpr int LR_ROWS = 16 * RT;
  __shared__ float red[LR_WAVES][LR_ROWS][17];
  const int jb0 = NJ > 1 ? 0 : blockIdx.y;
  const LoraRowsJob& jx = a.job[jb0];
  const u16* X = (const u16*)jx.X;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int m0 = blockIdx.x * LR_ROWS, M = a.M, K = jx.K, r = a.r;
  const int nsup = (K + 63) / 64;
  const int j = lane & 15;

  // Loads go through buffer resources: what lies past the rows, the reduction or the rank has an
  // offset past its resource and reads 0, without branches.
  const rsrc_t rX = make_rsrc(X + (size_t)m0 * jx.ldx, ((size_t)(min(LR_ROWS, M - m0) - 1) * jx.ldx + K) * 2);
  auto load_w = [&](const float* W, int k, uint4& bh, uint4& bl) {
    float f[8];
    const rsrc_t rW = make_rsrc(W, (size_t)r * K * 4);
    if (a.wt == 0) {
      const uint32_t o = (uint32_t)(j * K + k) * 4 | ((uint32_t)(K - 1 - k) & 0x80000000u);
      const uint4 p = bload128(rW, o), q = bload128(rW, o + 16);
      f[0] = __builtin_bit_cast(float, p.x); f[1] = __builtin_bit_cast(float, p.y);
      f[2] = __builtin_bit_cast(float, p.z); f[3] = __builtin_bit_cast(float, p.w);
      f[4] = __builtin_bit_cast(float, q.x); f[5] = __builtin_bit_cast(float, q.y);
      f[6] = __builtin_bit_cast(float, q.z); f[7] = __builtin_bit_cast(float, q.w);
    } else {
      const uint32_t bad = (uint32_t)(r - 1 - j) & 0x80000000u;
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = __builtin_bit_cast(float, bload32(rW, (uint32_t)((k + i) * r + j) * 4 | bad));
    }
    split_hi_lo<Op>(f, bh, bl);
  };
  // the super-step's two 32-wide halves of rows t*16 + lane%16 (K is a multiple of 8, so a
  // chunk is either wholly inside the row or wholly past it)
  const uint32_t xrow = (uint32_t)((lane & 15) * jx.ldx) * 2;
  auto load_x = [&](int k, uint4 (&xv)[2][RT]) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int kk = k + 32 * hh;
        xv[hh][t] = bload128s(rX, (xrow + 2 * kk) | ((uint32_t)(K - 1 - kk) & 0x80000000u), (uint32_t)(32 * t * jx.ldx));
      }
  };
  auto mma = [&](int k, const uint4 (&xv)[2][RT], f32x4 (&acc)[NJ][RT]) {
#pragma unroll
    for (int q = 0; q < NJ; ++q)
#pragma unroll
      for (int hh = 0; hh < 2; ++hh) {
        uint4 bh, bl;
        load_w(a.job[jb0 + q].W, k + 32 * hh, bh, bl);
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          acc[q][t] = mfma16_raw<Op>(xv[hh][t], bh, acc[q][t]);
          acc[q][t] = mfma16_raw<Op>(xv[hh][t], bl, acc[q][t]);
        }
      }
  };

  f32x4 acc[NJ][RT];
#pragma unroll
  for (int q = 0; q < NJ; ++q)
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int ko = 8 * (lane >> 4);
  if constexpr (NJ < 3 || RT < 4) {
    for (int ss = w; ss < nsup; ss += 2 * LR_WAVES) {
      const int k0 = ss * 64 + ko, k1 = (ss + LR_WAVES) * 64 + ko;
      uint4 x0[2][RT], x1[2][RT];
      load_x(k0, x0);
      load_x(k1, x1);
      mma(k0, x0, acc);
      mma(k1, x1, acc);
    }
  } else {
    // three jobs' accumulators leave registers for one super-step in flight
    for (int ss = w; ss < nsup; ss += LR_WAVES) {
      const int k0 = ss * 64 + ko;
      uint4 x0[2][RT];
      load_x(k0, x0);
      mma(k0, x0, acc);
    }
  }
  // lane holds rows t*16 + 4g + rr, column j; one job at a time through the LDS tile
#pragma unroll
  for (int q = 0; q < NJ; ++q) {
    if (q) __syncthreads();  // the previous job's sums have been read
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) red[w][t * 16 + 4 * (lane >> 4) + rr][j] = acc[q][t][rr];
    __syncthreads();
    float* out = a.job[jb0 + q].out;
    for (int o = tid; o < LR_ROWS * 16; o += 64 * LR_WAVES) {
      const int mm = o >> 4, jj = o & 15, m = m0 + mm;
      if (m < M && jj < r) {
        float v = 0.f;
#pragma unroll
        for (int ww = 0; ww < LR_WAVES; ++ww) v += red[ww][mm][jj];
        out[(size_t)m * r + jj] = a.s * v;
      }
    }
  }
}

// ------------------------------------------------------------------------- norm and rows
// A block's input RMSNorm with the down-projections that read it (the q, k, v or gate, up
// adapters), for the sizes whose row products take 16-row workgroups: y = fp16(x w rstd) and
// out_j = y A_j^T. Eight waves share 16 rows and split K as in k_lora_rows; a wave holds its
// NS super-steps of x in registers in the layout of the product's operand, so the normalised
// values go into it without another pass, and stores them on the way. The row statistics meet in
// LDS (one barrier). The adapters' and the norm's weights of PD super-steps are in flight ahead:
// the chain of a launch is one latency for x, one for the weights (512 tokens of 1152 with q, k,
// v and the table: 23 us as three launches, 14 here; 128 tokens of 896: 16.5 and 9.5; 4096 tokens
// of 1536: 27 and 20).
// Workgroups past the rows fill the RoPE table (as k_rope_table, in fp64), which is first read by
// the product behind this launch.
template <int NJ, int NS>
__global__ __launch_bounds__(64 * LR_WAVES) void k_norm_lora(const NormLoraArgs a) {
  __shared__ float red[LR_WAVES][16][17];
  __shared__ float sq[LR_WAVES][16];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  if ((int)blockIdx.x >= a.nrow) {
    rope_table_entry(((int)blockIdx.x - a.nrow) * 64 * LR_WAVES + tid, a.rope_T, a.rope_dh, a.rope_theta, a.rope_cs);
    return;
  }
  constexpr int PD = NS <= 5 ? 2 : 1;
  const int m0 = blockIdx.x * 16, M = a.M, K = a.K, r = a.r, j = lane & 15, ko = 8 * (lane >> 4);
  const rsrc_t rX = make_rsrc(a.x + (size_t)m0 * K, (size_t)min(16, M - m0) * K * 4);
  const rsrc_t rG = make_rsrc(a.w, (size_t)K * 4);
  auto f32x8 = [](rsrc_t rs, uint32_t o, float (&f)[8]) {
    const uint4 p = bload128(rs, o), q = bload128(rs, o + 16);
    f[0] = __builtin_bit_cast(float, p.x); f[1] = __builtin_bit_cast(float, p.y);
    f[2] = __builtin_bit_cast(float, p.z); f[3] = __builtin_bit_cast(float, p.w);
    f[4] = __builtin_bit_cast(float, q.x); f[5] = __builtin_bit_cast(float, q.y);
    f[6] = __builtin_bit_cast(float, q.z); f[7] = __builtin_bit_cast(float, q.w);
  };
  // chunk k of super-step s (K is a multiple of 8: wholly inside the row or wholly past it, where
  // the offset gets the sign bit and reads 0)
  auto kof = [&](int s, int hh) { return (w + LR_WAVES * s) * 64 + 32 * hh + ko; };
  auto past = [&](int k) { return (uint32_t)(K - 1 - k) & 0x80000000u; };
  float xv[NS][2][8], gv[PD][2][8], wv[PD][NJ][2][8];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) f32x8(rX, (uint32_t)(j * K + kof(s, hh)) * 4 | past(kof(s, hh)), xv[s][hh]);
  auto load_w = [&](int s, float (&g)[2][8], float (&wj)[NJ][2][8]) {
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int k = kof(s, hh);
      f32x8(rG, (uint32_t)k * 4 | past(k), g[hh]);
#pragma unroll
      for (int q = 0; q < NJ; ++q)
        f32x8(make_rsrc(a.W[q], (size_t)r * K * 4), (uint32_t)(j * K + k) * 4 | past(k), wj[q][hh]);
    }
  };
#pragma unroll
  for (int s = 0; s < PD; ++s) load_w(s, gv[s], wv[s]);
  float ss = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int i = 0; i < 8; ++i) ss += xv[s][hh][i] * xv[s][hh][i];
  ss += __shfl_xor(ss, 16, 64);
  ss += __shfl_xor(ss, 32, 64);
  if (lane < 16) sq[w][lane] = ss;
  __syncthreads();
  ss = 0.f;
#pragma unroll
  for (int ww = 0; ww < LR_WAVES; ++ww) ss += sq[ww][j];
  const float rs = 1.0f / sqrtf(ss / (float)K + a.eps);
  f32x4 acc[NJ];
#pragma unroll
  for (int q = 0; q < NJ; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    float (&g)[2][8] = gv[s % PD];
    float (&wj)[NJ][2][8] = wv[s % PD];
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int k = kof(s, hh);
      const float (&x)[8] = xv[s][hh];
      uint4 h;
      h.x = pack_f16x2(x[0] * rs * g[hh][0], x[1] * rs * g[hh][1]);
      h.y = pack_f16x2(x[2] * rs * g[hh][2], x[3] * rs * g[hh][3]);
      h.z = pack_f16x2(x[4] * rs * g[hh][4], x[5] * rs * g[hh][5]);
      h.w = pack_f16x2(x[6] * rs * g[hh][6], x[7] * rs * g[hh][7]);
      if (m0 + j < M && k < K) *(uint4*)(a.y + (size_t)(m0 + j) * K + k) = h;
#pragma unroll
      for (int q = 0; q < NJ; ++q) {
        uint4 bh, bl;
        split_hi_lo<OpF16>(wj[q][hh], bh, bl);
        acc[q] = mfma16_raw<OpF16>(h, bh, acc[q]);
        acc[q] = mfma16_raw<OpF16>(h, bl, acc[q]);
      }
    }
    if (s + PD < NS) load_w(s + PD, g, wj);
  }
  // lane holds rows 4 (lane / 16) + rr, column j; one job at a time through the LDS tile
#pragma unroll
  for (int q = 0; q < NJ; ++q) {
    if (q) __syncthreads();  // the previous job's sums have been read
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) red[w][4 * (lane >> 4) + rr][j] = acc[q][rr];
    __syncthreads();
    if (tid < 256) {
      const int mm = tid >> 4, jj = tid & 15, m = m0 + mm;
      if (m < M && jj < r) {
        float v = 0.f;
#pragma unroll
        for (int ww = 0; ww < LR_WAVES; ++ww) v += red[ww][mm][jj];
        a.out[q][(size_t)m * r + jj] = v;
      }
    }
  }
}

// The same norm where no adapter reads it, two rows per wave: lane 4 v + g of a row's 32 sums what
// wave v and lane group g sum above, and the sums meet in the same order, so that an adapter of
// zeros changes no bit (256 tokens of 896: 4 us; the kernel above without products 7).
template <int NS>
__global__ __launch_bounds__(256) void k_norm_plain(const NormLoraArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if ((int)blockIdx.x >= a.nrow) {
    rope_table_entry(((int)blockIdx.x - a.nrow) * 256 + tid, a.rope_T, a.rope_dh, a.rope_theta, a.rope_cs);
    return;
  }
  const int m = blockIdx.x * 8 + 2 * w + (lane >> 5), K = a.K, v = (lane >> 2) & 7, ko = 8 * (lane & 3);
  const bool ok = m < a.M;
  const rsrc_t rX = make_rsrc(a.x + (size_t)blockIdx.x * 8 * K, (size_t)min(8, a.M - (int)blockIdx.x * 8) * K * 4);
  const rsrc_t rG = make_rsrc(a.w, (size_t)K * 4);
  auto kof = [&](int s, int hh) { return (v + LR_WAVES * s) * 64 + 32 * hh + ko; };
  float4 x[NS][2][2], g[NS][2][2];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k = kof(s, hh);
        const uint32_t past = (uint32_t)(K - 1 - k) & 0x80000000u;
        x[s][hh][u] = __builtin_bit_cast(float4, bload128(rX, (uint32_t)((2 * w + (lane >> 5)) * K + k + 4 * u) * 4 | past));
        g[s][hh][u] = __builtin_bit_cast(float4, bload128(rG, (uint32_t)(k + 4 * u) * 4 | past));
      }
  float ss = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        ss += x[s][hh][u].x * x[s][hh][u].x;
        ss += x[s][hh][u].y * x[s][hh][u].y;
        ss += x[s][hh][u].z * x[s][hh][u].z;
        ss += x[s][hh][u].w * x[s][hh][u].w;
      }
  ss += __shfl_xor(ss, 1, 64);
  ss += __shfl_xor(ss, 2, 64);
  float t = 0.f;
#pragma unroll
  for (int ww = 0; ww < LR_WAVES; ++ww) t += __shfl(ss, (lane & 32) + 4 * ww, 64);
  const float rs = 1.0f / sqrtf(t / (float)K + a.eps);
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int k = kof(s, hh);
      const float4 x0 = x[s][hh][0], x1 = x[s][hh][1], g0 = g[s][hh][0], g1 = g[s][hh][1];
      if (ok && k < K)
        *(uint4*)(a.y + (size_t)m * K + k) =
            make_uint4(pack_f16x2(x0.x * rs * g0.x, x0.y * rs * g0.y), pack_f16x2(x0.z * rs * g0.z, x0.w * rs * g0.w),
                       pack_f16x2(x1.x * rs * g1.x, x1.y * rs * g1.y), pack_f16x2(x1.z * rs * g1.z, x1.w * rs * g1.w));
    }
}

// ----------------------------------------------------------------------------- outer
// R(c, j) = s * sum_m Mx[m][c] V[m][j] for every job of a stage in one launch (dB and dA; jobs
// that share Mx, such as dA of q, k, v, form a group that reads it once). A wave owns 64 columns
// and stages 64 tokens of them at a time transposed (c-major, token-contiguous) in LDS of its
// own; V^T goes beside them as hi / lo planes. The next step's tokens are loaded into registers
// meanwhile. Products run in bf16 (V may be a tiny gradient); an fp16 Mx is converted while
// staged. Two ways to share a launch out:
//  * TS, few tokens: the LO_W waves of a workgroup take interleaved token steps of the same 64
//    columns, with V planes of their own (no barrier in the loop), and their partial tiles are
//    summed in wave order through LDS. No reduce launch.
//  * else, many tokens: the waves stand side by side (64 LO_W columns) and share one double-
//    buffered V (a quarter of its loads and conversions each), one barrier per step; the tokens
//    are split over the grid (blockIdx.y, partial planes in a.part, summed in split order by the
//    reduce kernel).
// Bound by the stream of Mx, and at few tokens by the latency of one step: all of a step's loads
// are in flight at once. A layer's gradients, 999 tokens of 896 / 4864: 55 us in 4 launches (14
// launches and 120 us as single products with a token split and a reduction each).
constexpr int LO_C = 64, LO_M = 64, LO_LD = LO_M + 8, LO_W = 4, LO_V = 2 * 16 * LO_LD;
template <int NJ, bool TS>
__global__ __launch_bounds__(64 * LO_W) void k_lora_outer(const LoraOuterArgs a) {
  __shared__ __attribute__((aligned(16))) u16 smem[LO_W * LO_C * LO_LD + (TS ? LO_W : 2) * NJ * LO_V];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  int gi = 0;
  while (gi + 1 < a.ng && a.g[gi + 1].blk0 <= (int)blockIdx.x) ++gi;
  const LoraOuterGroup& gr = a.g[gi];
  const int C = gr.C, M = a.M, r = a.r, nj = min(gr.nj, NJ), ldm = gr.ldm;
  const int c0 = ((int)blockIdx.x - gr.blk0) * (TS ? LO_C : LO_C * LO_W) + (TS ? 0 : w * LO_C);
  const bool f16in = gr.f16in;
  // TS: wave-private tile and V planes; else private tile, two shared buffers of V planes
  u16* Mt = smem + w * LO_C * LO_LD;
  u16* Vall = smem + LO_W * LO_C * LO_LD;
  const int nsteps = (M + LO_M - 1) / LO_M, ms = blockIdx.y, MS = gridDim.y;
  const int sb = (int)((long long)nsteps * ms / MS), se = (int)((long long)nsteps * (ms + 1) / MS);
  const int rb = lane & 7, cb = lane >> 3;  // 8 x 8 block: tokens 8 rb .., columns 8 cb ..
  // V: output jv and NV tokens from NV tg on (TS: eight tokens each in two halves of 32)
  constexpr int NV = TS ? 8 : 64 / (4 * LO_W), NH = TS ? 2 : 1;
  const int jv = lane & 15, tg = TS ? lane >> 4 : tid >> 4;
  const uint32_t oc = c0 + 8 * cb < C ? (uint32_t)(8 * rb * ldm + c0 + 8 * cb) * 2 : 0x80000000u;
  // (an invalid output's offset gets the sign bit, past every resource: no branch per load, whose
  // waits would line the loads up one behind the other)
  const uint32_t vbad = (uint32_t)(r - 1 - jv) & 0x80000000u;
  uint4 in[8];
  float f[NJ][NH][NV];
  auto load = [&](int st) {
    const int mb = st * LO_M;
    const rsrc_t rT = make_rsrc((const u16*)gr.Mx + (size_t)mb * ldm, ((size_t)(min(LO_M, M - mb) - 1) * ldm + C) * 2);
#pragma unroll
    for (int i = 0; i < 8; ++i) in[i] = bload128s(rT, oc, (uint32_t)(i * ldm) * 2);
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
      if (q >= nj) break;
      const rsrc_t rV = make_rsrc(gr.V[q], (size_t)M * r * 4);
#pragma unroll
      for (int hh = 0; hh < NH; ++hh)
#pragma unroll
        for (int i = 0; i < NV; ++i)
          f[q][hh][i] = __builtin_bit_cast(
              float, bload32(rV, (uint32_t)((mb + 32 * hh + NV * tg + i) * r + jv) * 4 | vbad));
    }
  };
  auto store = [&](u16* Vp) {
    uint32_t x[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint4 v = f16in ? f16x8_to_bf16x8(in[i]) : in[i];
      x[i][0] = v.x; x[i][1] = v.y; x[i][2] = v.z; x[i][3] = v.w;
    }
#pragma unroll
    for (int jc = 0; jc < 8; ++jc) {
      const int d = jc >> 1;
      uint4 o;
      if (jc & 1)
        o = make_uint4(perm_hi16(x[0][d], x[1][d]), perm_hi16(x[2][d], x[3][d]), perm_hi16(x[4][d], x[5][d]),
                       perm_hi16(x[6][d], x[7][d]));
      else
        o = make_uint4(perm_lo16(x[0][d], x[1][d]), perm_lo16(x[2][d], x[3][d]), perm_lo16(x[4][d], x[5][d]),
                       perm_lo16(x[6][d], x[7][d]));
      *(uint4*)(Mt + (8 * cb + jc) * LO_LD + 8 * rb) = o;
    }
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
      if (q >= nj) break;
#pragma unroll
      for (int hh = 0; hh < NH; ++hh) {
        u16* ph = Vp + (2 * q * 16 + jv) * LO_LD + 32 * hh + NV * tg;
        u16* pl = ph + 16 * LO_LD;
        if constexpr (NV == 8) {
          uint4 hi, lo;
          split_hi_lo<OpBF16>(f[q][hh], hi, lo);
          *(uint4*)ph = hi;
          *(uint4*)pl = lo;
        } else {
          static_assert(NV == 4 || NV == 8, "tokens of V per lane");
          const float* v = f[q][hh];
          const uint32_t h0 = pack_bf16x2(v[0], v[1]), h1 = pack_bf16x2(v[2], v[3]);
          *(uint2*)ph = make_uint2(h0, h1);
          *(uint2*)pl = make_uint2(pack_bf16x2(v[0] - bf16_lo(h0), v[1] - bf16_hi(h0)),
                                   pack_bf16x2(v[2] - bf16_lo(h1), v[3] - bf16_hi(h1)));
        }
      }
    }
  };
  f32x4 acc[NJ][4];
#pragma unroll
  for (int q = 0; q < NJ; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[q][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // LDS accesses of one wave stay in order; the compiler must keep them so (other lanes' data)
  auto fence = [] {
    __builtin_amdgcn_wave_barrier();
    asm volatile("" ::: "memory");
  };
  const int s0 = TS ? sb + w : sb, ds = TS ? LO_W : 1;
  if (s0 < se) load(s0);
  for (int st = s0; st < se; st += ds) {
    u16* Vp = Vall + (TS ? w : (st - sb) & 1) * NJ * LO_V;
    fence();
    store(Vp);
    if constexpr (TS)
      fence();
    else
      __syncthreads();  // (the other buffer was read before the previous step's barrier)
    if (st + ds < se) load(st + ds);
#pragma unroll
    for (int kk = 0; kk < LO_M; kk += 32) {
      uint4 av[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) av[t] = *(const uint4*)(Mt + (16 * t + (lane & 15)) * LO_LD + kk + 8 * (lane >> 4));
#pragma unroll
      for (int q = 0; q < NJ; ++q) {
        if (q >= nj) break;
        const uint4 bh = *(const uint4*)(Vp + (2 * q * 16 + (lane & 15)) * LO_LD + kk + 8 * (lane >> 4));
        const uint4 bl = *(const uint4*)(Vp + ((2 * q + 1) * 16 + (lane & 15)) * LO_LD + kk + 8 * (lane >> 4));
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          acc[q][t] = mfma16_raw<OpBF16>(av[t], bh, acc[q][t]);
          acc[q][t] = mfma16_raw<OpBF16>(av[t], bl, acc[q][t]);
        }
      }
    }
  }
  auto put = [&](int q, int c, int j, float v) {
    const size_t at = gr.layout == 0 ? (size_t)c * r + j : (size_t)j * C + c;
    if (MS > 1)
      a.part[gr.part0 + ((size_t)q * MS + ms) * C * r + at] = v;
    else
      gr.out[q][at] = gr.s[q] * v;
  };
  // lane: column 16 t + 4 (lane / 16) + rr, output lane % 16
  if constexpr (!TS) {
#pragma unroll
    for (int q = 0; q < NJ; ++q) {
      if (q >= nj) break;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
          const int c = c0 + 16 * t + 4 * (lane >> 4) + rr, j = lane & 15;
          if (c < C && j < r) put(q, c, j, acc[q][t][rr]);
        }
    }
  } else {
    static_assert(!TS || LO_C * LO_LD * 2 >= LO_C * 16 * 4, "a job's partial tile fits the wave's staging tile");
    float* red = reinterpret_cast<float*>(Mt);
    for (int q = 0; q < nj; ++q) {
      // (every wave is done with its tile, or with the previous job's sums)
      __syncthreads();
#pragma unroll
      for (int qq = 0; qq < NJ; ++qq) {
        if (qq != q) continue;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) red[(16 * t + 4 * (lane >> 4) + rr) * 16 + (lane & 15)] = acc[qq][t][rr];
      }
      __syncthreads();
      for (int o = tid; o < LO_C * 16; o += 64 * LO_W) {
        // dA rows ([r][C]) are written column-fastest, dB rows ([C][r]) rank-fastest
        const int c = gr.layout == 0 ? o >> 4 : o & (LO_C - 1), j = gr.layout == 0 ? o & 15 : o / LO_C;
        if (c0 + c >= C || j >= r) continue;
        float v = 0.f;
#pragma unroll
        for (int ww = 0; ww < LO_W; ++ww)
          v += reinterpret_cast<const float*>(smem + ww * LO_C * LO_LD)[c * 16 + j];
        put(q, c0 + c, j, v);
      }
    }
  }
}

// sum the token-split partials of every job in split order; blockIdx.y counts the jobs
__global__ void k_lora_outer_reduce(const LoraOuterArgs a, int MS) {
  int gi = 0, q = blockIdx.y;
  while (q >= a.g[gi].nj) q -= a.g[gi++].nj;
  const LoraOuterGroup& gr = a.g[gi];
  const size_t n = (size_t)gr.C * a.r, i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float* p = a.part + gr.part0 + (size_t)q * MS * n + i;
  float acc = 0.f;
  for (int z = 0; z < MS; ++z) acc += p[(size_t)z * n];
  gr.out[q][i] = gr.s[q] * acc;
}

__global__ void k_fill_i32(int* p, int n, int v) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// token splits of an outer launch with `cols` columns over all groups. Up to 4096 tokens the
// waves split the tokens (TS), over the grid too from 2048 on (below, the reduce launch would
// cost as much as it saves); beyond, about 768 workgroups side by side, each with eight steps at
// least. Layer backward, side by side against TS (us): 2400 tokens 0.5B 620 and 593, 1.5B 1068 and
// 1043; 3300 0.5B 745 and 717, 1B 1044 and 1022; 4096 0.5B 839 and 814; then within 2 % either way
// up to 8192 (5200 0.5B 1095 and 1072, 1.5B 1789 and 1787, 6000 1B 1173 and 1156, 7200 4B 4124 and
// 4174); 16384 4B, the outer launches alone, 443 and 516.
constexpr int kOuterTsSteps = 64;
int outer_splits(int M, int cols) {
  const int steps = (M + LO_M - 1) / LO_M, ts = steps <= kOuterTsSteps, wide = ts ? LO_C : LO_C * LO_W;
  if (steps <= 32) return 1;
  const int cb = (cols + wide - 1) / wide;
  int s = ((ts ? 1024 : 768) + cb - 1) / cb;
  const int most = steps / (ts ? 4 * LO_W : 8);
  if (s > most) s = most;
  if (s > 64) s = 64;
  return s < 1 ? 1 : s;
}

// jobs that read the same input (pointer, leading dimension and width) run in one workgroup
template <class J>
bool same_input(const J* job, int n, const void* J::*x, int J::*ld, int J::*w) {
  for (int i = 1; i < n; ++i)
    if (job[i].*x != job[0].*x || job[i].*ld != job[0].*ld || job[i].*w != job[0].*w) return false;
  return n > 1;
}

}  // namespace

size_t lora_outer_part_floats(int M, int cols, int r) {
  const int s = outer_splits(M, cols);
  return s > 1 ? (size_t)s * cols * r : 0;
}

size_t lora_outer_group_floats(int M, int cols, int r, int jobs) {
  const int cb = (cols + 127) / 128, steps = (M + LO_M - 1) / LO_M;
  const int s = steps < 16 ? 1 : std::max(1, std::min({(512 + cb - 1) / cb, steps / 4, 64}));
  return s > 1 ? (size_t)jobs * s * cols * r : 0;
}

hipError_t launch_lora_rows(const LoraRowsArgs& a, int xbf16, hipStream_t st) {
  const bool shared = same_input(a.job, a.njobs, &LoraRowsJob::X, &LoraRowsJob::ldx, &LoraRowsJob::K);
  const int gy = shared ? 1 : a.njobs;
  const int rt = (a.M + 63) / 64 * gy >= 256 ? 4 : (a.M + 31) / 32 * gy >= 256 ? 2 : 1;
  const dim3 grid((a.M + 16 * rt - 1) / (16 * rt), gy);
  double flops = 0, bytes = 0;
  for (int i = 0; i < a.njobs; ++i) {
    flops += 2.0 * a.M * a.job[i].K * a.r;
    bytes += (i == 0 || !shared ? (double)a.M * a.job[i].K * 2 : 0.0) + (double)a.job[i].K * a.r * 4 +
             (double)a.M * a.r * 4;
  }
  const dim3 blk(64 * LR_WAVES);
#define LR_GO(OP, NJ)                                                                                                  \
  do {                                                                                                                 \
    if (rt == 4)                                                                                                       \
      MEBP_TIMED(st, "lora_rows", flops, bytes, hipLaunchKernelGGL((k_lora_rows<OP, NJ, 4>), grid, blk, 0, st, a));    \
    else if (rt == 2)                                                                                                  \
      MEBP_TIMED(st, "lora_rows", flops, bytes, hipLaunchKernelGGL((k_lora_rows<OP, NJ, 2>), grid, blk, 0, st, a));    \
    else                                                                                                               \
      MEBP_TIMED(st, "lora_rows", flops, bytes, hipLaunchKernelGGL((k_lora_rows<OP, NJ, 1>), grid, blk, 0, st, a));    \
  } while (0)
  const int nj = shared ? a.njobs : 1;
  if (xbf16) {
    if (nj == 3) LR_GO(OpBF16, 3); else if (nj == 2) LR_GO(OpBF16, 2); else LR_GO(OpBF16, 1);
  } else {
    if (nj == 3) LR_GO(OpF16, 3); else if (nj == 2) LR_GO(OpF16, 2); else LR_GO(OpF16, 1);
  }
#undef LR_GO
  return hipGetLastError();
}

bool norm_lora_ok(int M, int K) { return (M + 31) / 32 < 256 && (K & 7) == 0 && K <= 64 * LR_WAVES * 8; }

hipError_t launch_norm_lora(const NormLoraArgs& a0, hipStream_t st) {
  NormLoraArgs a = a0;
  if (!norm_lora_ok(a.M, a.K) || a.njobs < 0 || a.njobs > 3) return hipErrorInvalidValue;
  const int per = a.njobs ? 64 * LR_WAVES : 256;
  a.nrow = a.njobs ? (a.M + 15) / 16 : (a.M + 7) / 8;
  const int nrope = a.rope_cs ? (a.rope_T * (a.rope_dh / 2) + per - 1) / per : 0;
  const dim3 grid(a.nrow + nrope), blk(per);
  const double flops = 2.0 * a.M * a.K * a.r * a.njobs;
  const double bytes = (double)a.M * a.K * 6 + a.njobs * ((double)a.K * a.r * 4 + (double)a.M * a.r * 4);
  const int ns = (a.K + 64 * LR_WAVES - 1) / (64 * LR_WAVES);
#define NL_GO(NJ, NS) \
  MEBP_TIMED(st, "norm_lora", flops, bytes, hipLaunchKernelGGL((k_norm_lora<NJ, NS>), grid, blk, 0, st, a))
#define NL_NS(NJ)                \
  do {                           \
    if (ns <= 2) NL_GO(NJ, 2);   \
    else if (ns == 3) NL_GO(NJ, 3); \
    else if (ns <= 5) NL_GO(NJ, 5); \
    else NL_GO(NJ, 8);           \
  } while (0)
  if (a.njobs == 3) NL_NS(3); else if (a.njobs == 2) NL_NS(2); else if (a.njobs == 1) NL_NS(1);
  else {
#define NP_GO(NS) MEBP_TIMED(st, "rmsnorm_fwd", 0.0, bytes, hipLaunchKernelGGL(k_norm_plain<NS>, grid, blk, 0, st, a))
    if (ns <= 2) NP_GO(2); else if (ns == 3) NP_GO(3); else if (ns <= 5) NP_GO(5); else NP_GO(8);
#undef NP_GO
  }
#undef NL_NS
#undef NL_GO
  return hipGetLastError();
}

hipError_t launch_lora_outer(const LoraOuterArgs& a0, hipStream_t st) {
  LoraOuterArgs a = a0;
  double flops = 0, bytes = 0;
  int cols = 0, blocks = 0, njmax = 1, jobs = 0, cmax = 0;
  const bool ts = (a.M + LO_M - 1) / LO_M <= kOuterTsSteps;
  for (int i = 0; i < a.ng; ++i) {
    LoraOuterGroup& g = a.g[i];
    g.blk0 = blocks;
    blocks += ts ? (g.C + LO_C - 1) / LO_C : (g.C + LO_C * LO_W - 1) / (LO_C * LO_W);
    cols += g.C * g.nj;
    jobs += g.nj;
    njmax = g.nj > njmax ? g.nj : njmax;
    cmax = g.C > cmax ? g.C : cmax;
    flops += 2.0 * a.M * g.C * a.r * g.nj;
    bytes += (double)a.M * g.C * 2 + g.nj * ((double)a.M * a.r * 4 + (double)g.C * a.r * 4);
  }
  if (!blocks) return hipSuccess;
  int MS = outer_splits(a.M, cols);
  // (as many as the partials have room for)
  if (MS > 1) MS = (int)std::max<size_t>(1, std::min<size_t>(MS, a.part ? a.part_floats / ((size_t)cols * a.r) : 0));
  size_t p = 0;
  for (int i = 0; i < a.ng; ++i) {
    a.g[i].part0 = p;
    p += (size_t)a.g[i].nj * MS * a.g[i].C * a.r;
  }
  const dim3 grid(blocks, MS);
#define LO_GO(NJ)                                                                                                   \
  do {                                                                                                              \
    if (ts)                                                                                                         \
      MEBP_TIMED(st, "lora_outer", flops, bytes,                                                                    \
                 hipLaunchKernelGGL((k_lora_outer<NJ, true>), grid, dim3(64 * LO_W), 0, st, a));                    \
    else                                                                                                            \
      MEBP_TIMED(st, "lora_outer", flops, bytes,                                                                    \
                 hipLaunchKernelGGL((k_lora_outer<NJ, false>), grid, dim3(64 * LO_W), 0, st, a));                   \
  } while (0)
  if (njmax == 3) LO_GO(3); else if (njmax == 2) LO_GO(2); else LO_GO(1);
#undef LO_GO
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || MS == 1) return e;
  const dim3 rg((cmax * a.r + 255) / 256, jobs);
  MEBP_TIMED(st, "lora_outer_reduce", 0.0, 4.0 * MS * cols * a.r,
             hipLaunchKernelGGL(k_lora_outer_reduce, rg, dim3(256), 0, st, a, MS));
  return hipGetLastError();
}

hipError_t launch_fill_i32(int* p, int n, int v, hipStream_t st) {
  hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

}  // namespace mebp
