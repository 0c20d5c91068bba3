// Int4 group-dequant forward GEMMs whose reduction is a multiple of 64 (every configured
// shape), with every epilogue of the layer fused (LoRA up-projection, RoPE, act(gate) * up,
// residual, logits statistics): no partial plane and no finalize pass where the reduction is not
// split over the grid. Behind them the transposed products on bf16 weights in operand order.
//
// What bounded the kernels they replace: at few tokens the 128 x 128 tiles gave too few
// workgroups, so the reduction was split over workgroups and the fp32 planes went through
// memory (256 tokens: 40 MB per gate/up product); at many tokens the fetch of the weights. A
// lane's code and scale loads touch 32 weight rows at once, 32 bytes of codes and 2 of scales in
// each, and the 128-byte lines were evicted from the 32 KB vector cache between the K steps that
// use them: about 160 KB per K step and compute unit of line traffic against 64 bytes per clock.
// Loading two K steps' codes and four steps' scales at once took the 128 x 256 tile from 1706 to
// 1547 us at 16384 x 20480 x 2560 (fp32 out; without any weight load, in a timing copy, 31 % less
// time again) and halving the tile to 128 rows keeps two independent workgroups per compute
// unit, so that one's waits, first loads and epilogue run beside the other's MFMAs.
//
// Measured against the kernels that they replace (us, one product with its follow-up kernels):
// gate/up at 16384 tokens of the 2560-wide shape 1824 -> 1600 (1076 TFLOP/s), down 1000 -> 805,
// one 16384-column chunk of its logits 1613 -> 1298; at 4096 tokens of the 1536-wide shape qkv
// 57 -> 40, down 188 -> 159; at 999 tokens of the 896-wide shape gate/up 93 -> 35; at 256 tokens
// qkv 17 -> 7, logits 193 -> 105.
#include "device_common.h"
#include "mebp_internal.h"

namespace mebp {
namespace {

constexpr int BK = 64;
typedef uint16_t u16;

// v (8 fp32) in three bf16 parts, v = p[0] + p[1] + p[2] up to 2^-24: each part is the rounding of
// what the ones before leave
struct Split3 {
  uint4 p[3];
};
DEV Split3 split3_bf16(const float (&v)[8]) {
  float x[8];
  Split3 s;
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = v[e];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    float h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      h[e] = (float)(bf16)x[e];
      x[e] -= h[e];
    }
    s.p[q] = make_uint4(pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3]), pack_bf16x2(h[4], h[5]),
                        pack_bf16x2(h[6], h[7]));
  }
  return s;
}

// 16 bytes per lane from a buffer (per-lane and wave-uniform byte offsets) into LDS at
// dst + 16 lane, without passing through registers
DEV void load_lds16(rsrc_t r, lds_u8* dst, uint32_t voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, (int)voff, soff, 0, 0);
}

// c += u v^T of fp32 factors: the six products of parts that reach 2^-24 of the result, the
// smallest first; `two`: the three of two parts (2^-17: 4e-6 of the term instead of 1e-7)
DEV f32x16 mfma32_f32(const Split3& u, const Split3& v, f32x16 c, bool two) {
  if (!two) {
    c = mfma32<OpBF16>(u.p[2], v.p[0], c);
    c = mfma32<OpBF16>(u.p[1], v.p[1], c);
    c = mfma32<OpBF16>(u.p[0], v.p[2], c);
  }
  c = mfma32<OpBF16>(u.p[1], v.p[0], c);
  c = mfma32<OpBF16>(u.p[0], v.p[1], c);
  return mfma32<OpBF16>(u.p[0], v.p[0], c);
}

// One accumulator's LoRA term: acc[i][j] += s * U[m][:r] . V_j(lane)[:r]; u: 8 values of row
// 32 i + lane % 32, v: of column lane % 32 of block j, both for the ranks 8 (lane / 32) .. + 8
// (zero past r).
template <int MI, int NJ>
DEV void lora_acc(f32x16 (&acc)[MI][NJ], const float (&u)[MI][8], const float (&v)[NJ][8], bool two) {
  Split3 b[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) b[j] = split3_bf16(v[j]);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const Split3 a = split3_bf16(u[i]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = mfma32_f32(a, b[j], acc[i][j], two);
  }
}

// 8 consecutive floats at byte offset `off` of a resource (0 past its end), scaled; all zero
// when !keep
DEV void load8(rsrc_t r, uint32_t off, bool keep, float s, float (&o)[8]) {
  const uint4 a = bload128(r, keep ? off : 0x80000000u), b = bload128(r, keep ? off + 16 : 0x80000000u);
  o[0] = s * __builtin_bit_cast(float, a.x); o[1] = s * __builtin_bit_cast(float, a.y);
  o[2] = s * __builtin_bit_cast(float, a.z); o[3] = s * __builtin_bit_cast(float, a.w);
  o[4] = s * __builtin_bit_cast(float, b.x); o[5] = s * __builtin_bit_cast(float, b.y);
  o[6] = s * __builtin_bit_cast(float, b.z); o[7] = s * __builtin_bit_cast(float, b.w);
}

// Tile of this workgroup, numbered for the caches: every XCD gets a contiguous range (xcd_tile),
// walked in bands of eight row blocks, the rows of a band fastest. The 64 workgroups that an XCD
// runs at a time then cover 8 x 8 tiles, whose row and column operands are each fetched once
// into its L2 for eight users.
DEV TileId band_tile() {
  const TileId t = xcd_tile();
  const int gx = gridDim.x, gy = gridDim.y, lin = t.x + gx * t.y, band = lin / (8 * gx), r = lin - band * 8 * gx;
  const int hgt = min(8, gy - 8 * band), x = r / hgt;
  return TileId{x, 8 * band + r - x * hgt, t.z};
}

template <class T>
DEV T sel(bool c, T x, T y) {
  return c ? x : y;
}

// ------------------------------------------------------------------------------ forward
// C[m][n] = sum_k X[m][k] W[n][k], fp16 operands, on 32 MI x 64 WN output tiles: WN waves of
// 32 MI x 64 side by side, WK groups of them that split the reduction inside the workgroup.
//  * Activations go from global memory straight into a ring of two LDS stages of 32 MI x 64
//    (rows of 128 bytes, 16-byte chunk c at position c ^ ((row / 2) % 8): the 16 lanes of one
//    LDS read cycle hit 16 distinct bank groups), one ring per group.
//  * Each wave loads the int4 codes and scales of its own 64 columns into registers and
//    decompresses them there (nothing shared, nothing written to LDS).
//  * With WN = 1 a ring belongs to one wave: no barrier in the loop, only its own vmcnt.
//  * With WK > 1 the groups' accumulators meet in LDS (the idle rings) and are summed in group
//    order; each wave then finishes 1 / WK of the tile.
// The two 32-column blocks of a wave are chosen by the epilogue that pairs them in registers:
// the halves (e, e + dh/2) of a RoPE head, the gate and up columns of the same features, or
// simply 64 consecutive columns.
// MID_PLANES: raw fp32 tiles into plane blockIdx.z of `part` (grid-split reductions).
enum MidEpi { MID_F16 = 0, MID_F32 = 1, MID_LOGITS = 2, MID_GATED = 3, MID_PLANES = 4 };

// The waits of the loop count vector-memory instructions, so every load that it issues must
// have a use (the compiler drops the others): code rows (two steps' every two steps) and scales
// (four steps' every four) that step j loads, in the eight-step body and in the tail of up to seven
// steps behind it, which loads only what its own steps j + 2 .. 6 (codes) and 4 .. 6 (scales) use.
constexpr int code_rows(int j, bool tail) {
  if (j % 2) return 0;
  const int left = 7 - (j % 8 + 2);
  return !tail || left >= 2 ? 2 : left > 0 ? left : 0;
}
constexpr int scale_rows(int j, bool tail) { return j % 4 == 0 && (!tail || j % 8 == 0); }
constexpr int weight_loads(int j, bool tail) { return 2 * (code_rows(j, tail) + scale_rows(j, tail)); }

template <int MI, int WN, int WK, int EPI>
__global__ __launch_bounds__(64 * WN * WK, 2) void k_gemm_nt_mid(const NtArgs a) {
  constexpr int NJ = 2, BM = 32 * MI, NA = 4 * MI / WN, STB = BM * BK * 2;
  static_assert(WN == 1 || WK == 1, "a shared ring and a split reduction are not combined");
  static_assert(4 * MI % WN == 0, "the waves of a shared ring load equal parts of a stage");
  static_assert((4 * MI) % WK == 0, "waves finish whole row groups");
  __shared__ __attribute__((aligned(1024))) uint8_t lds0[WK * STB];
  __shared__ __attribute__((aligned(1024))) uint8_t lds1[WK * STB];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = WN > 1 ? wave : 0, wk = WK > 1 ? wave : 0, h = lane >> 5, l32 = lane & 31;
  auto stage = [&](auto S_) -> uint8_t* { return (decltype(S_)::value == 0 ? lds0 : lds1) + wk * STB; };
  // (plain order: every XCD keeps a few columns' weights; bands measured the same here)
  const int m0 = blockIdx.y * BM, K = a.K, Kh = K >> 1, kgroups = K >> 5;
  // this wave's two column blocks: weight rows c[j] .. c[j] + 32 of segment sj
  int s0 = 0, s1 = 0, c0, c1;
  if constexpr (EPI == MID_GATED) {
    c0 = c1 = 32 * ((int)blockIdx.x * WN + wn);
    s1 = 1;
  } else {
    const int nt = blockIdx.x;
    if (a.nseg > 1 && nt >= a.seg[1].tile0) s0 = 1;
    if (a.nseg > 2 && nt >= a.seg[2].tile0) s0 = 2;
    s1 = s0;
    const int ct = (nt - (s0 == 0 ? a.seg[0].tile0 : s0 == 1 ? a.seg[1].tile0 : a.seg[2].tile0)) * WN + wn;
    c0 = 64 * ct;
    c1 = c0 + 32;
    if (EPI == MID_F16 && (s0 == 0 ? a.seg[0].rope : s0 == 1 ? a.seg[1].rope : a.seg[2].rope)) {
      const int per = a.rope_dh >> 6, head = ct / per;
      c0 = head * a.rope_dh + 32 * (ct - head * per);
      c1 = c0 + (a.rope_dh >> 1);
    }
  }
#define SEG(s, f) ((s) == 0 ? a.seg[0].f : (s) == 1 ? a.seg[1].f : a.seg[2].f)
  const int Nn = SEG(s0, N);
  const int r0 = max(0, min(32, Nn - c0)), r1 = max(0, min(32, Nn - c1));
  const rsrc_t rA = make_rsrc((const u16*)a.X + (size_t)m0 * a.lda, (size_t)min(BM, a.M - m0) * a.lda * 2);
  const rsrc_t rB0 = make_rsrc(SEG(s0, q4) + (size_t)min(c0, Nn) * Kh, (size_t)r0 * Kh);
  const rsrc_t rB1 = make_rsrc(SEG(s1, q4) + (size_t)min(c1, Nn) * Kh, (size_t)r1 * Kh);
  const rsrc_t rS0 = make_rsrc(SEG(s0, scale) + (size_t)min(c0, Nn) * kgroups, (size_t)r0 * kgroups * 2);
  const rsrc_t rS1 = make_rsrc(SEG(s1, scale) + (size_t)min(c1, Nn) * kgroups, (size_t)r1 * kgroups * 2);
  // (ranges of a split reduction start on even steps: whole 64-byte pieces of the code rows)
  const int nk = K / BK, np = (nk + 1) >> 1;
  const int z = EPI == MID_PLANES ? (int)blockIdx.z * WK + wk : wk, Z = EPI == MID_PLANES ? (int)gridDim.z * WK : WK;
  const int kt_begin = 2 * (np * z / Z), kt_end = min(nk, 2 * (np * (z + 1) / Z));

  // activation loads: instruction i fills rows 8 (wn + WN i) .. + 8 of the group's stage
  uint32_t offA[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int row = 8 * (wn + WN * i) + (lane >> 3);
    offA[i] = (uint32_t)((row * a.lda + 8 * ((lane & 7) ^ ((row >> 1) & 7))) * 2);
  }
  const uint32_t offB = (uint32_t)(l32 * Kh + 16 * h), offS = (uint32_t)(l32 * kgroups * 2);
  const uint32_t ssel = h ? 0x03020302u : 0x01000100u;  // this half's scale, twice
  uint4 rb[2][2][NJ];   // codes of two steps, two buffers
  uint4 rsc[2][NJ];     // fp16 scales of four steps (eight groups), two buffers
  auto load_a = [&](auto S_, int kt) {
    lds_u8* dst = (lds_u8*)stage(S_);
#pragma unroll
    for (int i = 0; i < NA; ++i)
      load_lds16(rA, dst + 1024 * (wn + WN * i), offA[i], kt * (2 * BK));
    __builtin_amdgcn_sched_barrier(0);  // the waits count what follows as issued after the tile
  };
  // (steps past the end of the range or the row load bytes that are not used)
  auto load_codes = [&](auto B_, auto N_, int kt) {
    constexpr int bf = decltype(B_)::value;
#pragma unroll
    for (int t = 0; t < decltype(N_)::value; ++t) {
      rb[bf][t][0] = bload128s(rB0, offB, (kt + t) * (BK / 2));
      rb[bf][t][1] = bload128s(rB1, offB, (kt + t) * (BK / 2));
    }
  };
  auto load_scales = [&](auto B_, int kt) {
    constexpr int bf = decltype(B_)::value;
    rsc[bf][0] = bload128s(rS0, offS, kt * 4);
    rsc[bf][1] = bload128s(rS1, offS, kt * 4);
  };
  f32x16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  auto mma = [&](auto S_, const uint4 (&cw)[NJ], const uint32_t (&sw)[NJ]) {
    const uint8_t* As = stage(S_) + l32 * 128;
    f16x2 sc[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) sc[j] = __builtin_bit_cast(f16x2, __builtin_amdgcn_perm(0u, sw[j], ssel));
    auto rd = [&](int t, uint4 (&dst)[MI]) {
      const int pos = ((4 * h + t) ^ ((lane >> 1) & 7)) * 16;
#pragma unroll
      for (int i = 0; i < MI; ++i) dst[i] = *(const uint4*)(As + 4096 * i + pos);
    };
    auto dq = [&](int t, uint4 (&dst)[NJ]) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const uint32_t w = t == 0 ? cw[j].x : t == 1 ? cw[j].y : t == 2 ? cw[j].z : cw[j].w;
        dst[j] = dequant8_natural(w, sc[j]);
      }
    };
    // the fragments of substep t + 1 are read, and its weights decompressed, while the MFMAs
    // of substep t run
    uint4 af[2][MI], bq[2][NJ];
    rd(0, af[0]);
    dq(0, bq[0]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t < 3) rd(t + 1, af[(t + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      if (t < 3) dq(t + 1, bq[(t + 1) & 1]);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = mfma32<OpF16>(af[t & 1][i], bq[t & 1][j], acc[i][j]);
      if (t < 3) {
#pragma unroll
        for (int q = 0; q < MI * NJ; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 40 / (MI * NJ) + 1, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Step j (mod 8) of the loop issues the next activation tile, then (every two steps) the next two
  // steps' codes and (every four) the next four steps' scales, then multiplies. It ends when this
  // wave's loads of the next tile have landed (counting what was issued after them) and, with a
  // shared ring, so have the other waves'.
  auto sync = [&](auto J_, auto T_) {
    wait_vmcnt<weight_loads(decltype(J_)::value, decltype(T_)::value != 0)>();
    if constexpr (WN > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto step = [&](auto J_, auto T_, int k) {
    constexpr int j = decltype(J_)::value, cb = (j / 2) & 1, sb = (j / 4) & 1;
    constexpr bool tail = decltype(T_)::value != 0;
    load_a(IC<1 - j % 2>{}, min(k + 1, kt_end - 1));
    load_codes(IC<1 - cb>{}, IC<code_rows(j, tail)>{}, k + 2);
    if constexpr (scale_rows(j, tail) > 0) load_scales(IC<1 - sb>{}, k + 4);
    uint32_t sw[NJ];
#pragma unroll
    for (int q = 0; q < NJ; ++q)
      sw[q] = j % 4 == 0 ? rsc[sb][q].x : j % 4 == 1 ? rsc[sb][q].y : j % 4 == 2 ? rsc[sb][q].z : rsc[sb][q].w;
    mma(IC<j % 2>{}, rb[cb][j % 2], sw);
    sync(J_, T_);
  };
  if (kt_begin < kt_end) {
    // the LoRA term starts the accumulators while the first tiles are in flight (of a split
    // reduction: those of the last group, whose range is never empty)
    const bool lora0 = (WK == 1 || wk == WK - 1) && EPI != MID_LOGITS && EPI != MID_PLANES && SEG(s0, lora_B);
    const bool lora1 = EPI == MID_GATED ? (WK == 1 || wk == WK - 1) && a.seg[1].lora_B : lora0;
    load_codes(IC<0>{}, IC<2>{}, kt_begin);
    load_scales(IC<0>{}, kt_begin);
    load_a(IC<0>{}, kt_begin);
    if (lora0 || lora1) {
      const int q0 = 8 * h, r = a.r;
      const bool keep = q0 < r;
      float u[MI][8], v[NJ][8];
      const rsrc_t rV0 = make_rsrc(SEG(s0, lora_B), lora0 ? (size_t)Nn * r * 4 : 0);
      const rsrc_t rV1 = make_rsrc(SEG(s1, lora_B), lora1 ? (size_t)Nn * r * 4 : 0);
      load8(rV0, (uint32_t)(((c0 + l32) * r + q0) * 4), keep, 1.f, v[0]);
      load8(rV1, (uint32_t)(((c1 + l32) * r + q0) * 4), keep, 1.f, v[1]);
      const rsrc_t rU0 = make_rsrc(SEG(s0, lora_u), lora0 ? (size_t)a.M * r * 4 : 0);
#pragma unroll
      for (int i = 0; i < MI; ++i)
        load8(rU0, (uint32_t)(((m0 + 32 * i + l32) * r + q0) * 4), keep, a.lora_s, u[i]);
      if constexpr (EPI != MID_GATED) {
        lora_acc<MI, NJ>(acc, u, v, a.lora_two);
      } else {
        // gate and up have their own u
        const rsrc_t rU1 = make_rsrc(a.seg[1].lora_u, lora1 ? (size_t)a.M * r * 4 : 0);
        const Split3 b0 = split3_bf16(v[0]), b1 = split3_bf16(v[1]);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          float u1[8];
          load8(rU1, (uint32_t)(((m0 + 32 * i + l32) * r + q0) * 4), keep, a.lora_s, u1);
          acc[i][0] = mfma32_f32(split3_bf16(u[i]), b0, acc[i][0], a.lora_two);
          acc[i][1] = mfma32_f32(split3_bf16(u1), b1, acc[i][1], a.lora_two);
        }
      }
    }
    wait_vmcnt<0>();
    if constexpr (WN > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    int k = kt_begin;
    for (; k + 8 <= kt_end; k += 8) {
      step(IC<0>{}, IC<0>{}, k);
      step(IC<1>{}, IC<0>{}, k + 1);
      step(IC<2>{}, IC<0>{}, k + 2);
      step(IC<3>{}, IC<0>{}, k + 3);
      step(IC<4>{}, IC<0>{}, k + 4);
      step(IC<5>{}, IC<0>{}, k + 5);
      step(IC<6>{}, IC<0>{}, k + 6);
      step(IC<7>{}, IC<0>{}, k + 7);
    }
    if (k < kt_end) step(IC<0>{}, IC<1>{}, k);
    if (k + 1 < kt_end) step(IC<1>{}, IC<1>{}, k + 1);
    if (k + 2 < kt_end) step(IC<2>{}, IC<1>{}, k + 2);
    if (k + 3 < kt_end) step(IC<3>{}, IC<1>{}, k + 3);
    if (k + 4 < kt_end) step(IC<4>{}, IC<1>{}, k + 4);
    if (k + 5 < kt_end) step(IC<5>{}, IC<1>{}, k + 5);
    if (k + 6 < kt_end) step(IC<6>{}, IC<1>{}, k + 6);
  }
  // the rings are idle once the clamped loads of the last steps have landed
  wait_vmcnt<0>();

  if constexpr (EPI == MID_LOGITS) {
    static_assert(EPI != MID_LOGITS || WK == 1, "the logits product is not split");
    // per 16 rows through the wave's own 16 x 68 fp32 region: a lane holds 8 consecutive
    // columns of a row, so that the statistics of the row's 64-column tile reduce over 8 lanes
    // and its fp16 values leave as one 16-byte store. Per row and tile: max, sum of
    // exp(v - max), the values minus the max, and the fp32 logit of the target (vocabulary
    // columns are offset by vbase); the width is a multiple of 32, so an 8-column group is
    // wholly inside it or wholly past it.
    constexpr int LDE = 68;
    __syncthreads();
    static_assert(EPI != MID_LOGITS || (WN + 1) / 2 * (16 * LDE * 4) <= STB, "staging regions");
    float* ep = reinterpret_cast<float*>((wave & 1 ? lds1 : lds0) + (wave >> 1) * (16 * LDE * 4));
    const int rr = lane >> 3, ch = lane & 7, n = c0 + 8 * ch;
    const bool nok = n < Nn;
    _Float16* out = (_Float16*)a.seg[0].out;
#pragma unroll
    for (int ih = 0; ih < 2 * MI; ++ih) {
#pragma unroll
      for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          ep[(8 * (q >> 2) + 4 * h + (q & 3)) * LDE + 32 * j + l32] = acc[ih >> 1][j][8 * (ih & 1) + q];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int r = 8 * p + rr, m = m0 + 16 * ih + r;
        const float4 v0 = *(const float4*)(ep + r * LDE + 8 * ch), v1 = *(const float4*)(ep + r * LDE + 8 * ch + 4);
        const float v[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        float mx = -INFINITY, se = 0.f;
        if (nok) {
#pragma unroll
          for (int e = 0; e < 8; ++e) mx = fmaxf(mx, v[e]);
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        if (nok) {
#pragma unroll
          for (int e = 0; e < 8; ++e) se += __expf(v[e] - mx);
        }
#pragma unroll
        for (int o = 1; o < 8; o <<= 1) se += __shfl_xor(se, o, 64);
        if (m < a.M) {
          if (nok) {
            *(uint4*)(out + (size_t)m * a.seg[0].ldo + n) =
                make_uint4(pack_f16x2(v[0] - mx, v[1] - mx), pack_f16x2(v[2] - mx, v[3] - mx),
                           pack_f16x2(v[4] - mx, v[5] - mx), pack_f16x2(v[6] - mx, v[7] - mx));
            const int tg = a.tgt[m] - a.vbase - n;
            if (tg >= 0 && tg < 8) a.tgt_logit[m] = v[tg];
          }
          if (ch == 0 && c0 < Nn) a.stats[(size_t)m * a.ntiles + (c0 >> 6)] = make_float2(mx, se);
        }
      }
    }
    return;
  }
  // rows m0 + 32 i + 8 qg + 4 h + (0..3), column lane % 32 of both blocks. Outputs (and the
  // residual) go through buffer resources based at row m0: rows past M and columns past the
  // segment are dropped (or read 0) by the bounds check, without branches.
  const int n0 = c0 + l32, n1 = c1 + l32, rows = min(BM, a.M - m0);
  constexpr int ESZ = EPI == MID_F32 || EPI == MID_PLANES ? 4 : 2;
  const int ldo = EPI == MID_PLANES ? a.ldp : SEG(s0, ldo), rope = EPI == MID_F16 ? SEG(s0, rope) : 0;
  auto out_rsrc = [&](void* base, int ld) {
    return make_rsrc((char*)base + (size_t)m0 * ld * ESZ, ((size_t)(rows - 1) * ld + Nn) * ESZ);
  };
  const rsrc_t rO = out_rsrc(EPI == MID_PLANES ? (void*)(a.part + (size_t)blockIdx.z * a.M * a.ldp + SEG(s0, col0)) : SEG(s0, out), ldo);
  const uint32_t o0 = n0 < Nn ? (uint32_t)(4 * h * ldo + n0) * ESZ : 0x80000000u;
  const uint32_t o1 = n1 < Nn ? (uint32_t)(4 * h * ldo + n1) * ESZ : 0x80000000u;
  const rsrc_t rO1 = EPI == MID_GATED ? out_rsrc(a.seg[1].out, a.seg[1].ldo) : rO;
  const rsrc_t rZ = EPI == MID_GATED ? out_rsrc(a.z_out, Nn) : rO;
  const int ldr = a.seg[0].ldr;
  const rsrc_t rR = EPI == MID_F32 && a.seg[0].resid
                        ? make_rsrc(a.seg[0].resid + (size_t)m0 * ldr, ((size_t)(rows - 1) * ldr + Nn) * 4)
                        : make_rsrc(nullptr, 0);
  const int tb = EPI == MID_F16 && rope ? (m0 + 4 * h) % a.rope_T : 0;
  auto st16 = [&](rsrc_t r, uint32_t vo, int so, float v) {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, (f16)v), r, vo, so, 0);
  };
  // what the epilogue reads for the rows of one emit: the residual of both columns, or the RoPE
  // (cos, sin) of the rows' positions
  struct Extra {
    float x0[4], x1[4];
  };
  const rsrc_t rC = rope ? make_rsrc(a.rope_cs, (size_t)a.rope_T * a.rope_dh * 4) : make_rsrc(nullptr, 0);
  const uint32_t oC = (uint32_t)(n0 & ((a.rope_dh >> 1) - 1)) * 8;
  auto fetch = [&](int i, int qg, Extra& x) {
    const int row = 32 * i + 8 * qg;
    if constexpr (EPI == MID_F16) {
      if (rope) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int t = tb + row + r;
          if (a.rope_T >= BM)
            t = t >= a.rope_T ? t - a.rope_T : t;
          else
            t %= a.rope_T;
          const uint2 cs = bload64(rC, (uint32_t)(t * a.rope_dh) * 4 + oC);
          x.x0[r] = __builtin_bit_cast(float, cs.x);
          x.x1[r] = __builtin_bit_cast(float, cs.y);
        }
      }
    } else if constexpr (EPI == MID_F32) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t so = (uint32_t)((row + r + 4 * h) * ldr) * 4;
        x.x0[r] = __builtin_bit_cast(float, bload32(rR, n0 < Nn ? so + 4 * n0 : 0x80000000u));
        x.x1[r] = __builtin_bit_cast(float, bload32(rR, n1 < Nn ? so + 4 * n1 : 0x80000000u));
      }
    }
  };
  auto emit = [&](int i, int qg, const float (&v0)[4], const float (&v1)[4], const Extra& x) {
    const int row = 32 * i + 8 * qg;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int so = (row + r) * ldo * ESZ;
      if constexpr (EPI == MID_GATED) {
        // the activation sees the same fp16-rounded g and u that the backward reads
        const float g = (float)(f16)v0[r], u = (float)(f16)v1[r];
        if (a.store_gu) {
          st16(rO, o0, so, g);
          st16(rO1, o0, so, u);
        }
        st16(rZ, o0, so, act_f(g, a.act) * u);
      } else if constexpr (EPI == MID_F16) {
        if (rope) {  // heads divide the segment: both halves are inside it or past it
          st16(rO, o0, so, v0[r] * x.x0[r] - v1[r] * x.x1[r]);
          st16(rO, o1, so, v1[r] * x.x0[r] + v0[r] * x.x1[r]);
        } else {
          st16(rO, o0, so, v0[r]);
          st16(rO, o1, so, v1[r]);
        }
      } else {
        const float y0 = EPI == MID_F32 ? v0[r] + x.x0[r] : v0[r], y1 = EPI == MID_F32 ? v1[r] + x.x1[r] : v1[r];
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, y0), rO, o0, so, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, y1), rO, o1, so, 0);
      }
    }
  };
  if constexpr (WK == 1) {
    // (each 32-row block's reads are issued together, before its stores)
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      Extra x[4];
#pragma unroll
      for (int qg = 0; qg < 4; ++qg) fetch(i, qg, x[qg]);
#pragma unroll
      for (int qg = 0; qg < 4; ++qg) {
        const float v0[4] = {acc[i][0][4 * qg], acc[i][0][4 * qg + 1], acc[i][0][4 * qg + 2], acc[i][0][4 * qg + 3]};
        const float v1[4] = {acc[i][1][4 * qg], acc[i][1][4 * qg + 1], acc[i][1][4 * qg + 2], acc[i][1][4 * qg + 3]};
        emit(i, qg, v0, v1, x[qg]);
      }
    }
  } else {
    // block j of this wave's partial tile into its ring stage j: [i][q][lane]
    float* p0 = reinterpret_cast<float*>(lds0) + wk * (STB / 4) + lane;
    float* p1 = reinterpret_cast<float*>(lds1) + wk * (STB / 4) + lane;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        p0[(i * 16 + q) * 64] = acc[i][0][q];
        p1[(i * 16 + q) * 64] = acc[i][1][q];
      }
    constexpr int GPW = 4 * MI / WK;  // row groups per wave
    Extra x[GPW];
#pragma unroll
    for (int gi = 0; gi < GPW; ++gi) fetch((wk * GPW + gi) >> 2, (wk * GPW + gi) & 3, x[gi]);
    __syncthreads();
#pragma unroll
    for (int gi = 0; gi < GPW; ++gi) {
      const int g = wk * GPW + gi, i = g >> 2, qg = g & 3;
      const float* b0 = reinterpret_cast<const float*>(lds0) + (i * 16 + 4 * qg) * 64 + lane;
      const float* b1 = reinterpret_cast<const float*>(lds1) + (i * 16 + 4 * qg) * 64 + lane;
      float v0[4], v1[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v0[r] = b0[64 * r];
        v1[r] = b1[64 * r];
      }
#pragma unroll
      for (int z = 1; z < WK; ++z)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v0[r] += b0[z * (STB / 4) + 64 * r];
          v1[r] += b1[z * (STB / 4) + 64 * r];
        }
      emit(i, qg, v0, v1, x[gi]);
    }
  }
#undef SEG
}


// ---------------------------------------------------------------------------- transposed
// C[m][c] = sum_seg sum_n G_seg[m][n] W_seg[n][c], bf16 operands, on weights that a pass just
// before wrote as bf16 in the order in which the MFMA reads them: for every K step (64 rows n of
// a segment) and every 32 columns four 1 KiB blocks, block t holding for lane l the eight rows
// 32 (l / 32) + 8 t .. + 8 of column l % 32, as 16 bytes at 16 l. Rows past a segment and columns
// past Kout are zero. A wave's fragment is then one coalesced 1 KiB load straight into the
// registers of the MFMA: the weights pass through neither LDS nor a transpose, and LDS carries
// the gradient tile alone. What bounds the many-token products is the power-limited MFMA rate
// (1.0 .. 1.15 PFLOP/s; a large plain bf16 product of the library reaches 1.2), at few tokens the
// fetch of the weights by a few workgroups. Against the kernels they replace (us, conversion pass
// included, same GPU): activation backward of the 2560-wide shape at 16384 tokens 1258 + 17 ->
// 913 + 13, its gate/up input gradient 1963 + 33 -> 1679 + 25, its LM-head dH product per
// 16384-column chunk 1433 + 26 -> 1374 + 20; at 999 tokens of the 896-wide shape activation
// backward 85 -> 20 + 5, gate/up input gradient 107 -> 32 + 6; at 512 tokens of the 1152-wide one
// 94 -> 41 + 10. Converting a whole layer at once instead of product by product saves four
// launches.
constexpr int kFragBlock = 1024;

// bf16 of q * s (rounded to nearest even) in fragment order; one thread per 8 rows x 8 columns.
// Bound by its writes: 2 bytes per weight beside 0.56 read; a wave's 64 x 64 block is put in
// order in LDS, so that its stores are consecutive (52 million weights: 42 us with each lane
// storing its own 128 bytes, 25 us so, 5.5 TB/s).
__global__ __launch_bounds__(256) void k_frag_weights(const FragArgs a) {
  __shared__ uint4 buf[4][512];
  const int bid = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int s = 0;
  while (s + 1 < a.nseg && a.seg[s + 1].blk0 <= bid) ++s;
  const FragSeg sg = a.seg[s];
  // one wave per 64 rows x 64 columns; the four waves of a workgroup side by side
  const int nc = (sg.cols + 63) / 64, nr = (sg.N + BK - 1) / BK;
  const int tile = (bid - sg.blk0) * 4 + w, kt = tile / nc, cb = tile - kt * nc;
  if (kt >= nr) return;
  const int r8 = lane >> 3, c8 = lane & 7, n0 = BK * kt + 8 * r8, c0 = 64 * cb + 8 * c8;
  const int Kh = sg.cols >> 1, kg = (sg.cols + 31) >> 5;
  const rsrc_t rQ = make_rsrc(sg.q4, (size_t)sg.N * Kh), rS = make_rsrc(sg.scale, (size_t)sg.N * kg * 2);
  uint32_t q[8], sc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    // rows past N are past the resource and read 0; columns past the width are masked
    q[e] = bload32(rQ, c0 < sg.cols ? (uint32_t)((n0 + e) * Kh + (c0 >> 1)) : 0x80000000u);
    sc[e] = bload16(rS, c0 < sg.cols ? (uint32_t)((n0 + e) * kg + (c0 >> 5)) * 2 : 0x80000000u);
  }
  float v[8][8];
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int j = 0; j < 8; ++j) v[e][j] = (float)nib_s(q[e], j) * half_bits_to_f32((uint16_t)sc[e]);
  // 16-byte unit (column block c8 / 4, block t = r8 % 4, half r8 / 4, column 8 (c8 % 4) + j); the
  // low bits of j are XORed with c8, so that the eight lanes of one LDS cycle hit all banks
  const int u0 = (c8 >> 2) * 256 + (r8 & 3) * 64 + (r8 >> 2) * 32 + (c8 & 3) * 8;
#pragma unroll
  for (int j = 0; j < 8; ++j)
    buf[w][u0 + (j ^ c8)] = make_uint4(pack_bf16x2(v[0][j], v[1][j]), pack_bf16x2(v[2][j], v[3][j]),
                                       pack_bf16x2(v[4][j], v[5][j]), pack_bf16x2(v[6][j], v[7][j]));
  uint4* dst = (uint4*)sg.out + ((size_t)kt * nc + cb) * 512;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int u = 64 * i + lane, c = (i >> 2) * 4 + ((lane >> 3) & 3);
    dst[u] = buf[w][u ^ c];
  }
}

// Tiles of 32 MI x 64 WN with WK K ranges as in the forward kernel. NT epilogues of TnEpi; with
// WK = 1 the 16-bit ones go through LDS, 16 rows at a time, so that a lane moves 8 consecutive
// columns of a row (16-byte accesses instead of 2-byte ones in the MFMA layout).
template <int MI, int WN, int WK, int EPI>
__global__ __launch_bounds__(64 * WN * WK, 2) void k_gemm_tn_frag(const TnArgs a) {
  constexpr int NJ = 2, BM = 32 * MI, NA = 4 * MI / WN, STB = BM * BK * 2;
  constexpr bool RAW = EPI == TN_PARTIAL_F32 || EPI == TN_PLANES;  // fp32 tiles into planes
  static_assert(WN == 1 || WK == 1, "a shared ring and a split reduction are not combined");
  static_assert(4 * MI % WN == 0, "the waves of a shared ring load equal parts of a stage");
  static_assert((4 * MI) % WK == 0, "waves finish whole row groups");
  __shared__ __attribute__((aligned(1024))) uint8_t lds0[WK * STB];
  __shared__ __attribute__((aligned(1024))) uint8_t lds1[WK * STB];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = WN > 1 ? wave : 0, wk = WK > 1 ? wave : 0, h = lane >> 5, l32 = lane & 31;
  auto stage = [&](auto S_) -> uint8_t* { return (decltype(S_)::value == 0 ? lds0 : lds1) + wk * STB; };
  const TileId tl = band_tile();
  const int m0 = tl.y * BM, Kout = a.Kout, ct = tl.x * WN + wn, c0 = 64 * ct, rows = min(BM, a.M - m0);
  const int ncb = (Kout + 63) / 64 * 2;
  // K steps before the second, before the third segment and in all
  const int e0 = (a.seg[0].N + BK - 1) / BK, e1 = e0 + (a.nseg > 1 ? (a.seg[1].N + BK - 1) / BK : 0),
            total = e1 + (a.nseg > 2 ? (a.seg[2].N + BK - 1) / BK : 0);
  const int z = tl.z * WK + wk, Z = gridDim.z * WK;
  const int t_begin = (int)((long long)total * z / Z), t_end = (int)((long long)total * (z + 1) / Z);
  // (selected per step by value: a conditional on the variables themselves selects an address and
  // keeps them in scratch memory)
  const int ld0 = a.seg[0].ldg, ld1 = a.seg[1].ldg, ld2 = a.seg[2].ldg;
  const int N0 = a.seg[0].N, N1 = a.seg[1].N, N2 = a.seg[2].N;
  const u16* G0 = (const u16*)a.seg[0].G + (size_t)m0 * ld0;
  const u16* G1 = (const u16*)a.seg[1].G + (size_t)m0 * ld1;
  const u16* G2 = (const u16*)a.seg[2].G + (size_t)m0 * ld2;
  const rsrc_t rB = make_rsrc(a.w16, ct * 2 < ncb ? (size_t)total * ncb * 4 * kFragBlock : 0);
  const uint32_t offB = (uint32_t)(ct * 8 * kFragBlock + 16 * lane);
  uint4 rb[2][NJ][4];
  auto load_a = [&](auto S_, int t) {
    const bool i0 = t < e0, i1 = t < e1;
    const int ldg = sel(i0, ld0, sel(i1, ld1, ld2)), Ns = sel(i0, N0, sel(i1, N1, N2));
    const int n0 = (t - sel(i0, 0, sel(i1, e0, e1))) * BK;
    const rsrc_t ra = make_rsrc(sel(i0, G0, sel(i1, G1, G2)), (size_t)rows * ldg * 2);
    lds_u8* dst = (lds_u8*)stage(S_);
    // instruction i: rows row0 + 8 WN i .. + 8, whose chunk order depends on the parity of the
    // row block; columns past the segment read as zero (the sign bit puts the offset out of range)
    const int row0 = 8 * wn + (lane >> 3);
    uint32_t vo[2];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int n = n0 + 8 * ((lane & 7) ^ (((row0 + 8 * WN * p) >> 1) & 7));
      vo[p] = (uint32_t)(row0 * ldg + n) * 2 | ((uint32_t)(Ns - 1 - n) & 0x80000000u);
    }
#pragma unroll
    for (int i = 0; i < NA; ++i) load_lds16(ra, dst + 1024 * (wn + WN * i), vo[WN % 2 ? i & 1 : 0], 16 * WN * i * ldg);
    __builtin_amdgcn_sched_barrier(0);  // the waits count the weights as issued after the tile
  };
  auto load_b = [&](auto B_, int t) {
    constexpr int bf = decltype(B_)::value;
    const uint32_t so = (uint32_t)t * (uint32_t)ncb * (4 * kFragBlock);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) rb[bf][j][q] = bload128s(rB, offB + (4 * j + q) * kFragBlock, so);
  };
  f32x16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 16; ++q) acc[i][j][q] = 0.f;
  auto mma = [&](auto S_, const uint4 (&b)[NJ][4]) {
    const uint8_t* As = stage(S_) + l32 * 128;
    auto rd = [&](int t, uint4 (&dst)[MI]) {
      const int pos = ((4 * h + t) ^ ((lane >> 1) & 7)) * 16;
#pragma unroll
      for (int i = 0; i < MI; ++i) dst[i] = *(const uint4*)(As + 4096 * i + pos);
    };
    uint4 af[2][MI];
    rd(0, af[0]);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (t < 3) rd(t + 1, af[(t + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = mfma32<OpBF16>(af[t & 1][i], b[j][t], acc[i][j]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // step: the next tile's gradient rows and weights in flight during this one's MFMAs; ends when
  // this wave's (and, through a shared ring, every wave's) gradient rows have landed
  auto step = [&](auto I_, int t) {
    constexpr int I = decltype(I_)::value;
    const int tn = min(t + 1, t_end - 1);
    load_a(IC<1 - I>{}, tn);
    load_b(IC<1 - I>{}, tn);
    mma(IC<I>{}, rb[I]);
    wait_vmcnt<4 * NJ>();
    if constexpr (WN > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  if (t_begin < t_end) {
    load_a(IC<0>{}, t_begin);
    load_b(IC<0>{}, t_begin);
    // the LoRA term du A of every segment starts the accumulators (of the last K range)
    if (!RAW && z == Z - 1) {
      const int q0 = 8 * h, r = a.r;
      const bool keep = q0 < r;
      for (int s = 0; s < a.nseg; ++s) {
        const float* A = a.seg[s].lora_A;
        if (!A) continue;
        const rsrc_t rV = make_rsrc(A, (size_t)r * Kout * 4), rU = make_rsrc(a.seg[s].lora_du, (size_t)a.M * r * 4);
        float u[MI][8], v[NJ][8];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int c = c0 + 32 * j + l32;
#pragma unroll
          for (int e = 0; e < 8; ++e)
            v[j][e] = __builtin_bit_cast(
                float, bload32(rV, keep && c < Kout ? (uint32_t)((q0 + e) * Kout + c) * 4 : 0x80000000u));
        }
#pragma unroll
        for (int i = 0; i < MI; ++i) load8(rU, (uint32_t)(((m0 + 32 * i + l32) * r + q0) * 4), keep, 1.f, u[i]);
        lora_acc<MI, NJ>(acc, u, v, a.lora_two);
      }
    }
    wait_vmcnt<0>();
    if constexpr (WN > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    int t = t_begin;
    for (; t + 2 <= t_end; t += 2) {
      step(IC<0>{}, t);
      step(IC<1>{}, t + 1);
    }
    if (t < t_end) mma(IC<0>{}, rb[0]);
  }
  wait_vmcnt<0>();

  // fp32 outputs: column lane % 32 of both blocks, rows 32 i + 8 qg + 4 h + (0..3), through a
  // buffer resource based at row m0 (rows past M and columns past Kout are dropped)
  const int n0 = c0 + l32, n1 = n0 + 32;
  const int ldo = EPI == TN_ACT_BWD ? a.ldgu : a.ldo;
  const size_t osz = ((size_t)(rows - 1) * ldo + Kout);
  if constexpr (WK == 1 && (EPI == TN_ACT_BWD || EPI == TN_STORE_BF16)) {
    constexpr int LDE = (WN + 1) / 2 * (16 * 68 * 4) <= STB ? 68 : 64;
    __syncthreads();  // every wave is done with the ring
    static_assert((WN + 1) / 2 * (16 * LDE * 4) <= STB, "staging regions");
    float* ep = reinterpret_cast<float*>((wave & 1 ? lds1 : lds0) + (wave >> 1) * (16 * LDE * 4));
    const int rr = lane >> 3, ch = lane & 7, c = c0 + 8 * ch;
    const bool cok = c < Kout;  // (a multiple of 8: a lane's 8 columns are inside or past it)
    const rsrc_t r0 = make_rsrc((u16*)(EPI == TN_ACT_BWD ? a.g : a.outb) + (size_t)m0 * ldo, osz * 2);
    const rsrc_t r1 = make_rsrc(EPI == TN_ACT_BWD ? (u16*)a.u + (size_t)m0 * ldo : nullptr, EPI == TN_ACT_BWD ? osz * 2 : 0);
    auto off = [&](int row) { return cok ? (uint32_t)(row * ldo + c) * 2 : 0x80000000u; };
    auto put = [&](rsrc_t r, uint32_t o, uint4 v) {
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      const u32x4 x = {v.x, v.y, v.z, v.w};
      __builtin_amdgcn_raw_buffer_store_b128(x, r, (int)o, 0, 0);
    };
    auto run = [&](auto K_) {
      constexpr int KIND = decltype(K_)::value;
#pragma unroll
      for (int ih = 0; ih < 2 * MI; ++ih) {
        uint4 gw[2], uw[2];
        if constexpr (EPI == TN_ACT_BWD) {
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            gw[p] = bload128(r0, off(16 * ih + 8 * p + rr));
            uw[p] = bload128(r1, off(16 * ih + 8 * p + rr));
          }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            ep[(8 * (q >> 2) + 4 * h + (q & 3)) * LDE + 32 * j + l32] = acc[ih >> 1][j][8 * (ih & 1) + q];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int r = 8 * p + rr;
          const float4 v0 = *(const float4*)(ep + r * LDE + 8 * ch), v1 = *(const float4*)(ep + r * LDE + 8 * ch + 4);
          const float dz[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
          uint32_t o[4], ou[4];
          if constexpr (EPI == TN_ACT_BWD) {
            // dz -> dg = dz u act'(g), du = dz act(g), in place over g and u
            const uint32_t gq[4] = {gw[p].x, gw[p].y, gw[p].z, gw[p].w}, uq[4] = {uw[p].x, uw[p].y, uw[p].z, uw[p].w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              float a0, d0, a1, d1;
              act_and_grad<KIND>(f16_lo(gq[k]), a0, d0);
              act_and_grad<KIND>(f16_hi(gq[k]), a1, d1);
              o[k] = pack_bf16x2(dz[2 * k] * f16_lo(uq[k]) * d0, dz[2 * k + 1] * f16_hi(uq[k]) * d1);
              ou[k] = pack_bf16x2(dz[2 * k] * a0, dz[2 * k + 1] * a1);
            }
            put(r1, off(16 * ih + r), make_uint4(ou[0], ou[1], ou[2], ou[3]));
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) o[k] = pack_bf16x2(dz[2 * k], dz[2 * k + 1]);
          }
          put(r0, off(16 * ih + r), make_uint4(o[0], o[1], o[2], o[3]));
        }
      }
    };
    if (EPI == TN_ACT_BWD && a.act)
      run(IC<1>{});
    else
      run(IC<0>{});
    return;
  }
  const size_t plane = RAW ? (size_t)tl.z * a.M * ldo : 0;
  const rsrc_t rO = EPI == TN_ACT_BWD      ? make_rsrc((u16*)a.g + (size_t)m0 * ldo, osz * 2)
                    : EPI == TN_STORE_BF16 ? make_rsrc((u16*)a.outb + (size_t)m0 * ldo, osz * 2)
                                           : make_rsrc(a.out + plane + (size_t)m0 * ldo, osz * 4);
  const rsrc_t rU = EPI == TN_ACT_BWD ? make_rsrc((u16*)a.u + (size_t)m0 * ldo, osz * 2) : rO;
  constexpr int ESZ = RAW || EPI == TN_STORE_F32 ? 4 : 2;
  const uint32_t o0 = n0 < Kout ? (uint32_t)(4 * h * ldo + n0) * ESZ : 0x80000000u;
  const uint32_t o1 = n1 < Kout ? (uint32_t)(4 * h * ldo + n1) * ESZ : 0x80000000u;
  auto st16 = [&](rsrc_t r, uint32_t vo, int so, float v) {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, to_bf16(v)), r, vo, so, 0);
  };
  auto ld16 = [&](rsrc_t r, uint32_t vo, int so) {
    return (float)__builtin_bit_cast(f16, (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)vo, so, 0));
  };
  auto emit = [&](int i, int qg, const float (&v0)[4], const float (&v1)[4]) {
    const int row = 32 * i + 8 * qg;
    float g0[4], g1[4], u0[4], u1[4];
    if constexpr (EPI == TN_ACT_BWD) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int so = (row + r) * ldo * 2;
        g0[r] = ld16(rO, o0, so);
        g1[r] = ld16(rO, o1, so);
        u0[r] = ld16(rU, o0, so);
        u1[r] = ld16(rU, o1, so);
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int so = (row + r) * ldo * ESZ;
      if constexpr (EPI == TN_ACT_BWD) {
        st16(rO, o0, so, v0[r] * u0[r] * act_grad_f(g0[r], a.act));
        st16(rO, o1, so, v1[r] * u1[r] * act_grad_f(g1[r], a.act));
        st16(rU, o0, so, v0[r] * act_f(g0[r], a.act));
        st16(rU, o1, so, v1[r] * act_f(g1[r], a.act));
      } else if constexpr (EPI == TN_STORE_BF16) {
        st16(rO, o0, so, v0[r]);
        st16(rO, o1, so, v1[r]);
      } else {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v0[r]), rO, o0, so, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v1[r]), rO, o1, so, 0);
      }
    }
  };
  if constexpr (WK == 1) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int qg = 0; qg < 4; ++qg) {
        const float v0[4] = {acc[i][0][4 * qg], acc[i][0][4 * qg + 1], acc[i][0][4 * qg + 2], acc[i][0][4 * qg + 3]};
        const float v1[4] = {acc[i][1][4 * qg], acc[i][1][4 * qg + 1], acc[i][1][4 * qg + 2], acc[i][1][4 * qg + 3]};
        emit(i, qg, v0, v1);
      }
  } else {
    // the K ranges' partial tiles through the idle rings, summed in range order
    float* p0 = reinterpret_cast<float*>(lds0) + wk * (STB / 4) + lane;
    float* p1 = reinterpret_cast<float*>(lds1) + wk * (STB / 4) + lane;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        p0[(i * 16 + q) * 64] = acc[i][0][q];
        p1[(i * 16 + q) * 64] = acc[i][1][q];
      }
    __syncthreads();
    constexpr int GPW = 4 * MI / WK;
#pragma unroll
    for (int gi = 0; gi < GPW; ++gi) {
      const int g = wk * GPW + gi, i = g >> 2, qg = g & 3;
      const float* b0 = reinterpret_cast<const float*>(lds0) + (i * 16 + 4 * qg) * 64 + lane;
      const float* b1 = reinterpret_cast<const float*>(lds1) + (i * 16 + 4 * qg) * 64 + lane;
      float v0[4], v1[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        v0[r] = b0[64 * r];
        v1[r] = b1[64 * r];
      }
#pragma unroll
      for (int z2 = 1; z2 < WK; ++z2)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v0[r] += b0[z2 * (STB / 4) + 64 * r];
          v1[r] += b1[z2 * (STB / 4) + 64 * r];
        }
      emit(i, qg, v0, v1);
    }
  }
}

// Tile configurations and their cost model, in microseconds: `fix` of launch, first loads and
// epilogue, then per K step of a wave `lat` while a compute unit has one workgroup at most, or
// for each workgroup that it has `thr` per step and `wg` that no other one hides. Fitted to 27
// forward products of 128 .. 16384 tokens with reductions of 896 .. 10240 and 25 transposed ones
// with reductions of 688 .. 20480, each configuration timed on each: mostly within 15 % of the
// measured times, and the pick is the fastest configuration or one within 10 % of it. A
// reduction may also be split over the grid (S planes, summed by the finalize kernel that also
// applies the product's follow-up): a wave has 1 / S of the steps, at the cost of the planes'
// traffic at 3 TB/s and, where no follow-up kernel would have run anyway, of one more launch.
// (More K ranges inside a workgroup, 8 or 16 of 32 x 64, gain nothing: the compute unit's cache
// then bounds the tile.)
struct MidCfg {
  int mi, wn, wk;
  float fix, lat, thr, wg;
};
constexpr MidCfg kMidNt[] = {
    {4, 4, 1, 7.0f, 0.90f, 0.98f, 0.0f},  // 128 x 256: many tiles
    {4, 1, 4, 5.0f, 1.20f, 1.36f, 4.0f},  // 128 x 64, four K ranges: about 256 tiles
    {2, 1, 8, 6.0f, 1.40f, 1.70f, 0.0f},  // 64 x 64, eight K ranges: long reductions, few tiles
    {2, 1, 4, 5.0f, 0.80f, 0.85f, 0.0f},
    {2, 1, 2, 4.0f, 0.78f, 0.43f, 0.0f},
    {1, 1, 4, 3.5f, 0.50f, 0.53f, 0.0f},  // 32 x 64: the fewest tokens
};
constexpr MidCfg kMidTn[] = {
    {4, 4, 1, 7.0f, 0.86f, 1.04f, 0.0f}, {4, 1, 4, 5.0f, 1.10f, 1.40f, 2.0f},
    {2, 1, 8, 6.0f, 1.30f, 1.31f, 2.2f}, {2, 1, 4, 4.5f, 0.72f, 0.67f, 0.8f},
    {2, 1, 2, 4.0f, 0.65f, 0.37f, 0.7f}, {1, 1, 4, 3.5f, 0.50f, 0.52f, 0.0f},
    {2, 4, 1, 5.0f, 0.54f, 0.57f, 1.0f},  // 64 x 256
};
constexpr int kNtTiles = sizeof(kMidNt) / sizeof(MidCfg), kTnTiles = sizeof(kMidTn) / sizeof(MidCfg);
// row tiles of a launch (the y dimension of a grid takes 65535 workgroups): beyond 8 million tokens
// the 128-row tiles are too many, and the 256-row ones of the other kernels take over
constexpr int kMaxRowTiles = 65535;
struct MidPlan {
  int cfg, splits;
};

int mid_columns(const MidCfg& c, const int* Ns, int nseg, bool gated) {
  if (gated) return (Ns[0] + 32 * c.wn - 1) / (32 * c.wn);
  int t = 0;
  for (int s = 0; s < nseg; ++s) t += (Ns[s] + 64 * c.wn - 1) / (64 * c.wn);
  return t;
}

// columns(c): workgroup columns of configuration c; unit: K steps that a range is a multiple of;
// width: output columns (the planes); followup: a finalize kernel costs no extra launch
template <class F>
MidPlan mid_plan(const MidCfg* cfgs, int n, int M, int ksteps, int unit, int max_s, int width, bool followup, F columns) {
  MidPlan best{0, 1};
  float bt = 1e30f;
  for (int i = 0; i < n; ++i) {
    const MidCfg& c = cfgs[i];
    if ((M - 1) / (32 * c.mi) >= kMaxRowTiles) continue;
    const int base = columns(c) * ((M + 32 * c.mi - 1) / (32 * c.mi));
    for (int S = 1; S <= max_s; S = S < 4 ? S + 1 : S + S / 2) {
      if (S > 1 && S * c.wk * 2 > ksteps) break;  // two steps per wave at least
      const int units = (ksteps + unit - 1) / unit, steps = unit * ((units + c.wk * S - 1) / (c.wk * S));
      const long long tiles = (long long)base * S;
      const float per = (float)((tiles + 255) / 256), one = steps * c.lat, many = per * (steps * c.thr + c.wg);
      float t = c.fix + (per > 1.f && many > one ? many : one);
      if (S > 1) t += 1.5f + 8e-6f / 3.f * S * M * width + (followup ? 0.f : 4.5f);
      if (t < bt) {
        bt = t;
        best = MidPlan{i, S};
      }
    }
  }
  return best;
}

// Whether a product's LoRA terms take two bf16 parts of each factor instead of three. They have fp32
// bits wherever the sums of split planes or the 128 x 128 kernels give them those (in fp32
// instructions); from 160 tiles of 256 x 128 and 1024 tokens on, where the large tiles multiply two
// parts, a third would cost 1 .. 1.5 % of a layer (4 x 1024 tokens of 1536 forward: 564 -> 572 us,
// 8 x 2048 of 2560: 3473 -> 3518) below the fp16 and bf16 roundings of the product beside it.
bool mid_lora_two(int M, const int* Ns, int nseg) {
  long long t = 0;
  for (int s = 0; s < nseg; ++s) t += (Ns[s] + 127) / 128;
  return M >= 1024 && t * ((M + 255) / 256) >= 160;
}

MidPlan mid_plan_nt(int M, const int* Ns, int nseg, int K, bool gated, bool logits, bool followup) {
  int width = 0;
  for (int s = 0; s < nseg; ++s) width += Ns[s];
  // (the logits' statistics take whole rows of a wave: the widest tile)
  return mid_plan(kMidNt, logits ? 1 : kNtTiles, M, K / BK, 2, logits ? 1 : kMaxSplits, width,
                  followup, [&](const MidCfg& c) { return mid_columns(c, Ns, nseg, gated); });
}

MidPlan mid_plan_tn(int M, int Kout, const int* Ns, int nseg, int max_s, bool followup) {
  int kt = 0;
  for (int s = 0; s < nseg; ++s) kt += (Ns[s] + BK - 1) / BK;
  return mid_plan(kMidTn, kTnTiles, M, kt, 1, max_s, Kout, followup,
                  [&](const MidCfg& c) { return (Kout + 64 * c.wn - 1) / (64 * c.wn); });
}

}  // namespace

size_t frag_elems(int N, int cols) {
  return (size_t)((N + BK - 1) / BK * BK) * (size_t)((cols + 63) / 64 * 64);
}

hipError_t launch_frag_weights(FragArgs a, hipStream_t st) {
  long long blocks = 0;
  double bytes = 0;
  for (int s = 0; s < a.nseg; ++s) {
    FragSeg& g = a.seg[s];
    if (g.cols % 8) return hipErrorInvalidValue;
    g.blk0 = (int)blocks;
    const size_t n = frag_elems(g.N, g.cols);
    blocks += (long long)((n / 4096 + 3) / 4);
    bytes += 2.0 * n + (double)g.N * (g.cols / 2 + 2 * ((g.cols + 31) / 32));
  }
  if (!blocks) return hipSuccess;
  MEBP_TIMED(st, "frag_weights", 0.0, bytes,
             hipLaunchKernelGGL(k_frag_weights, dim3((unsigned)blocks), dim3(256), 0, st, a));
  return hipGetLastError();
}

bool gemm_mid_rows_ok(int M) { return (M - 1) / 128 < kMaxRowTiles; }

bool gemm_nt_mid_ok(int M, int K) { return K % BK == 0 && gemm_mid_rows_ok(M); }

bool gemm_nt_mid_aligned(const NtArgs& a) {
  bool ok = true;
  for (int s = 0; s < a.nseg; ++s) ok = ok && ((uintptr_t)a.seg[s].scale & 3) == 0;
  return ok;
}

int gemm_nt_mid_splits(int M, const int* Ns, int nseg, int K, bool gated, bool followup) {
  return mid_plan_nt(M, Ns, nseg, K, gated, false, followup).splits;
}

int gemm_tn_frag_splits(int M, int Kout, const int* Ns, int nseg, int max_s, bool followup) {
  return mid_plan_tn(M, Kout, Ns, nseg, max_s, followup).splits;
}

namespace {

int nt_planes_width(const NtArgs& a) {
  int w = 0;
  for (int s = 0; s < a.nseg; ++s) w += a.seg[s].N;
  return w;
}

// one forward product on tile configuration `cfg`, over S planes
hipError_t run_nt(NtArgs a, int cfg, MidEpi epi, int S, const char* name, double flops, double bytes, hipStream_t st) {
  const MidCfg& c = kMidNt[cfg];
  int Ns[3], t = 0;
  for (int s = 0; s < a.nseg; ++s) {
    Ns[s] = a.seg[s].N;
    a.seg[s].tile0 = t;
    t += (Ns[s] + 64 * c.wn - 1) / (64 * c.wn);
  }
  a.lora_two = mid_lora_two(a.M, Ns, a.nseg);
  const dim3 grid(mid_columns(c, Ns, a.nseg, epi == MID_GATED), (a.M + 32 * c.mi - 1) / (32 * c.mi), S);
#define MID_GO(MI, WN, WK, EPI)      \
  MEBP_TIMED(st, name, flops, bytes, \
             hipLaunchKernelGGL((k_gemm_nt_mid<MI, WN, WK, EPI>), grid, dim3(64 * WN * WK), 0, st, a))
#define MID_EPI(MI, WN, WK)                             \
  do {                                                  \
    switch (epi) {                                      \
      case MID_PLANES: MID_GO(MI, WN, WK, MID_PLANES); break; \
      case MID_GATED: MID_GO(MI, WN, WK, MID_GATED); break;   \
      case MID_F16: MID_GO(MI, WN, WK, MID_F16); break;       \
      case MID_F32: MID_GO(MI, WN, WK, MID_F32); break;       \
      default: return hipErrorInvalidValue;                   \
    }                                                         \
  } while (0)
  if (epi == MID_LOGITS) {
    if (cfg) return hipErrorInvalidValue;
    MID_GO(4, 4, 1, MID_LOGITS);
    return hipGetLastError();
  }
  switch (cfg) {
    case 0: MID_EPI(4, 4, 1); break;
    case 1: MID_EPI(4, 1, 4); break;
    case 2: MID_EPI(2, 1, 8); break;
    case 3: MID_EPI(2, 1, 4); break;
    case 4: MID_EPI(2, 1, 2); break;
    default: MID_EPI(1, 1, 4); break;
  }
#undef MID_EPI
#undef MID_GO
  return hipGetLastError();
}

// one transposed product on tile configuration `cfg`, over S planes
hipError_t run_tn(TnArgs a, int cfg, int epi, int S, const char* name, double flops, double bytes, hipStream_t st) {
  const MidCfg& c = kMidTn[cfg];
  a.lora_two = mid_lora_two(a.M, &a.Kout, 1);
  const dim3 grid((a.Kout + 64 * c.wn - 1) / (64 * c.wn), (a.M + 32 * c.mi - 1) / (32 * c.mi), S);
#define FRAG_GO(MI, WN, WK, EPI)     \
  MEBP_TIMED(st, name, flops, bytes, \
             hipLaunchKernelGGL((k_gemm_tn_frag<MI, WN, WK, EPI>), grid, dim3(64 * WN * WK), 0, st, a))
#define FRAG_EPI(MI, WN, WK)                                            \
  do {                                                                  \
    switch (epi) {                                                      \
      case TN_PARTIAL_F32: FRAG_GO(MI, WN, WK, TN_PARTIAL_F32); break;  \
      case TN_PLANES: FRAG_GO(MI, WN, WK, TN_PLANES); break;            \
      case TN_STORE_F32: FRAG_GO(MI, WN, WK, TN_STORE_F32); break;      \
      case TN_ACT_BWD: FRAG_GO(MI, WN, WK, TN_ACT_BWD); break;          \
      case TN_STORE_BF16: FRAG_GO(MI, WN, WK, TN_STORE_BF16); break;    \
      default: return hipErrorInvalidValue;                             \
    }                                                                   \
  } while (0)
  switch (cfg) {
    case 0: FRAG_EPI(4, 4, 1); break;
    case 1: FRAG_EPI(4, 1, 4); break;
    case 2: FRAG_EPI(2, 1, 8); break;
    case 3: FRAG_EPI(2, 1, 4); break;
    case 4: FRAG_EPI(2, 1, 2); break;
    case 5: FRAG_EPI(1, 1, 4); break;
    default: FRAG_EPI(2, 4, 1); break;
  }
#undef FRAG_EPI
#undef FRAG_GO
  return hipGetLastError();
}

MidPlan unsplit_nt(const NtArgs& a, const int* Ns, bool gated, bool logits) {
  return mid_plan(kMidNt, logits ? 1 : kNtTiles, a.M, a.K / BK, 2, 1, nt_planes_width(a), true,
                  [&](const MidCfg& c) { return mid_columns(c, Ns, a.nseg, gated); });
}

}  // namespace

hipError_t launch_gemm_nt_mid(const NtArgs& a, int epi, int S, double flops, double bytes, hipStream_t st) {
  if (!gemm_nt_mid_ok(a.M, a.K) || a.lda % 8 || ((uintptr_t)a.X & 15) || !gemm_nt_mid_aligned(a))
    return hipErrorInvalidValue;
  int Ns[3];
  for (int s = 0; s < a.nseg; ++s) Ns[s] = a.seg[s].N;
  const bool logits = epi == NT_LOGITS, gated = a.gated && S == 1;
  // the tile for S planes was planned with them; without (or after the caller dropped them) plan anew
  MidPlan p = mid_plan_nt(a.M, Ns, a.nseg, a.K, a.gated, logits, a.norm_w != nullptr);
  if (p.splits != S) p = unsplit_nt(a, Ns, gated, logits);
  const MidEpi e = logits ? MID_LOGITS : S > 1 ? MID_PLANES : gated ? MID_GATED : epi == NT_STORE_F16 ? MID_F16 : MID_F32;
  const char* name = logits ? "gemm_nt_logits" : S > 1 ? "gemm_nt_planes" : epi == NT_STORE_F16 ? "gemm_nt_f16out" : "gemm_nt_f32out";
  return run_nt(a, p.cfg, e, S, name, flops, bytes, st);
}

hipError_t launch_gemm_tn_frag(const TnArgs& a, int epi, int S, double flops, double bytes, hipStream_t st) {
  int Ns[3];
  for (int s = 0; s < a.nseg; ++s) {
    Ns[s] = a.seg[s].N;
    if (a.seg[s].N % 8 || a.seg[s].ldg % 8 || ((uintptr_t)a.seg[s].G & 15)) return hipErrorInvalidValue;
  }
  if (a.Kout % 8 || !a.w16 || !gemm_mid_rows_ok(a.M)) return hipErrorInvalidValue;
  // the tile from the plan that chose S planes; a plan of one plane where the caller dropped them
  MidPlan p = mid_plan_tn(a.M, a.Kout, Ns, a.nseg, epi == TN_PARTIAL_F32 ? kMaxHeadSplits : kMaxSplits,
                          epi == TN_PARTIAL_F32 || tn_followup(a, epi));
  if (p.splits != S) p = mid_plan_tn(a.M, a.Kout, Ns, a.nseg, S, true);
  TnArgs b = a;
  const bool planes = S > 1 && epi != TN_PARTIAL_F32;
  if (planes) {
    b.out = a.part;
    b.ldo = a.Kout;
  }
  const char* name = planes                 ? "gemm_tn_planes"
                     : epi == TN_PARTIAL_F32 ? "gemm_tn_probs_dh"
                     : epi == TN_STORE_F32  ? "gemm_tn_f32out"
                     : epi == TN_ACT_BWD    ? "gemm_tn_act_bwd"
                                            : "gemm_tn_bf16out";
  return run_tn(b, p.cfg, planes ? TN_PLANES : epi, S, name, flops, bytes, st);
}

hipError_t launch_gemm_nt_probe(int tile, const uint8_t* q4, const uint16_t* scale, int n_out, int n_in, const void* x,
                                int M, float* out, hipStream_t st) {
  NtArgs a{};
  a.X = x; a.lda = n_in; a.M = M; a.K = n_in; a.nseg = 1;
  a.seg[0].q4 = q4; a.seg[0].scale = scale; a.seg[0].N = n_out; a.seg[0].out = out; a.seg[0].ldo = n_out;
  if (a.K % BK || !gemm_nt_mid_aligned(a) || tile >= kNtTiles) return hipErrorInvalidValue;
  return run_nt(a, tile < 0 ? unsplit_nt(a, &n_out, false, false).cfg : tile, MID_F32, 1, "gemm_nt_f32out", 0.0, 0.0, st);
}

hipError_t launch_gemm_tn_probe(int tile, const uint8_t* q4, const uint16_t* scale, int n_out, int n_in, const void* g,
                                int M, float* out, uint16_t* frags, bool write, hipStream_t st) {
  if (tile >= kTnTiles) return hipErrorInvalidValue;
  if (write) {
    FragArgs f{};
    f.seg[f.nseg++] = FragSeg{q4, scale, n_out, n_in, frags, 0};
    const hipError_t e = launch_frag_weights(f, st);
    if (e != hipSuccess) return e;
  }
  TnArgs a{};
  a.M = M; a.Kout = n_in; a.nseg = 1; a.w16 = frags;
  a.seg[0].G = (const bf16*)g; a.seg[0].ldg = n_out; a.seg[0].N = n_out;
  a.out = out; a.ldo = n_in;
  return run_tn(a, tile < 0 ? mid_plan_tn(M, n_in, &n_out, 1, 1, true).cfg : tile, TN_STORE_F32, 1, "gemm_tn_f32out", 0.0,
                0.0, st);
}

}  // namespace mebp
