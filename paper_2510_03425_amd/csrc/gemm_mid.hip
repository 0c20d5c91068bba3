// Int4 group-dequant forward GEMMs whose reduction is a multiple of 64 (every configured
// shape), with every epilogue of the layer fused (LoRA up-projection, RoPE, act(gate) * up,
// residual, logits statistics): no partial plane and no finalize pass.
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
#include <stdlib.h>

#include "device_common.h"
#include "mebp_internal.h"

namespace mebp {
namespace {

constexpr int BK = 64;
typedef uint16_t u16;
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;

template <int N>
struct IC {
  static constexpr int value = N;
};

template <class Op>
DEV f32x16 mfma32(uint4 a, uint4 b, f32x16 c) {
  if constexpr (__is_same(Op, OpF16))
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                   0, 0);
}

// v (8 fp32) -> bf16 hi and lo parts with v ~ hi + lo
DEV void split_bf16(const float (&v)[8], uint4& hi, uint4& lo) {
  float h[8], l[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    h[e] = (float)(bf16)v[e];
    l[e] = v[e] - h[e];
  }
  hi = make_uint4(pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3]), pack_bf16x2(h[4], h[5]), pack_bf16x2(h[6], h[7]));
  lo = make_uint4(pack_bf16x2(l[0], l[1]), pack_bf16x2(l[2], l[3]), pack_bf16x2(l[4], l[5]), pack_bf16x2(l[6], l[7]));
}

// 8 int4 codes of a dword times scale into fp16 pairs (k0,k1),(k2,k3),(k4,k5),(k6,k7): the
// offset-binary nibbles (code ^ 8) of the even and odd elements as bytes, one of each placed
// in the two halves by a byte permute, 0x6400 | (q + 8) is the fp16 value 1024 + q + 8, so one
// packed subtraction of 1032 gives q exactly and one packed multiply rounds q * s to nearest.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
DEV uint4 dequant8_natural(uint32_t w, f16x2 s2) {
  const uint32_t x = w ^ 0x88888888u;
  const uint32_t ev = x & 0x0F0F0F0Fu, od = (x >> 4) & 0x0F0F0F0Fu;
  const f16x2 off = {(_Float16)1032.0f, (_Float16)1032.0f};
  uint32_t o[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    // byte 0 <- even byte j, byte 2 <- odd byte j, bytes 1 and 3 <- 0
    const uint32_t t = __builtin_amdgcn_perm(od, ev, (uint32_t)j | 0x0C00u | ((4u + j) << 16) | 0x0C000000u) | 0x64006400u;
    o[j] = __builtin_bit_cast(uint32_t, (__builtin_bit_cast(f16x2, t) - off) * s2);
  }
  return make_uint4(o[0], o[1], o[2], o[3]);
}

// 16 bytes per lane from a buffer (per-lane and wave-uniform byte offsets) into LDS at
// dst + 16 lane, without passing through registers
DEV void load_lds16(rsrc_t r, lds_u8* dst, uint32_t voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, dst, 16, (int)voff, soff, 0, 0);
}

template <int N>
DEV void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// One accumulator's LoRA term: acc[i][j] += s * U[m][:r] . V_j(lane)[:r] on three bf16 MFMAs
// (hi*hi + hi*lo + lo*hi); u: 8 values of row 32 i + lane % 32, v: of column lane % 32 of block
// j, both for the ranks 8 (lane / 32) .. + 8 (zero past r).
template <int MI, int NJ>
DEV void lora_acc(f32x16 (&acc)[MI][NJ], const float (&u)[MI][8], const float (&v)[NJ][8]) {
  uint4 bh[NJ], bl[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) split_bf16(v[j], bh[j], bl[j]);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    uint4 ah, al;
    split_bf16(u[i], ah, al);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      acc[i][j] = mfma32<OpBF16>(ah, bh[j], acc[i][j]);
      acc[i][j] = mfma32<OpBF16>(ah, bl[j], acc[i][j]);
      acc[i][j] = mfma32<OpBF16>(al, bh[j], acc[i][j]);
    }
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

// ------------------------------------------------------------------------------ forward
// C[m][n] = sum_k X[m][k] W[n][k], fp16 operands, on 32 MI x 64 WN output tiles: WN waves of
// 32 MI x 64 side by side, WK groups of them that split the reduction inside the workgroup.
//  * Activations go from global memory straight into a ring of ST LDS stages of 32 MI x 64
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
enum MidEpi { MID_F16 = 0, MID_F32 = 1, MID_LOGITS = 2, MID_GATED = 3 };

// The waits of the loop count vector-memory instructions, so every load that it issues must
// have a use (the compiler drops the others): code rows (of CS) and scales (0 or 1) that step j
// loads, in the eight-step body and in the tail of up to seven steps behind it, which loads
// only what its own steps 4 .. 6 (scales) and j + CS .. 6 (codes) use.
constexpr int code_rows(int j, int CS, bool tail) {
  if (j % CS) return 0;
  const int left = 7 - (j % 8 + CS);
  return !tail || left >= CS ? CS : left > 0 ? left : 0;
}
constexpr int scale_rows(int j, bool tail) { return j % 4 == 0 && (!tail || j % 8 == 0); }
constexpr int weight_loads(int j, int CS, bool tail) { return 2 * (code_rows(j, CS, tail) + scale_rows(j, tail)); }
// instructions issued after the activation tile of step j + 1 when step j ends (tiles are issued
// D steps ahead; the steps before a tail are the last ones of the body)
constexpr int after_tile(int j, int D, int NA, int CS, bool tail) {
  int n = 0;
  for (int t = j + 1 - D; t <= j; ++t)
    n += (t > j + 1 - D ? NA : 0) + weight_loads((t + 8) % 8, CS, tail && t >= 0);
  return n;
}

template <int MI, int WN, int WK, int ST, int CS, int EPI>
__global__ __launch_bounds__(64 * WN * WK, 2) void k_gemm_nt_mid(const NtArgs a) {
  constexpr int NJ = 2, BM = 32 * MI, NA = 4 * MI / WN, STB = BM * BK * 2;
  static_assert(ST == 2 || (ST == 4 && CS == 4), "ring stages");
  static_assert(CS == 2 || CS == 4, "K steps per load of the codes");
  static_assert(WN == 1 || WK == 1, "a shared ring and a split reduction are not combined");
  static_assert(4 * MI % WN == 0, "the waves of a shared ring load equal parts of a stage");
  static_assert(WK == 1 || (4 * MI) % WK == 0, "each wave finishes whole row groups");
  __shared__ __attribute__((aligned(1024))) uint8_t lds0[WK * STB];
  __shared__ __attribute__((aligned(1024))) uint8_t lds1[WK * STB];
  __shared__ __attribute__((aligned(1024))) uint8_t lds2[ST == 4 ? WK * STB : 16];
  __shared__ __attribute__((aligned(1024))) uint8_t lds3[ST == 4 ? WK * STB : 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wn = WN > 1 ? wave : 0, wk = WK > 1 ? wave : 0, h = lane >> 5, l32 = lane & 31;
  auto stage = [&](auto S_) -> uint8_t* {
    constexpr int st = decltype(S_)::value;
    return (st == 0 ? lds0 : st == 1 ? lds1 : st == 2 ? lds2 : lds3) + wk * STB;
  };
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
  const int kt_begin = 2 * (np * wk / WK), kt_end = min(nk, 2 * (np * (wk + 1) / WK));

  // activation loads: instruction i fills rows 8 (wn + WN i) .. + 8 of the group's stage
  uint32_t offA[NA];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int row = 8 * (wn + WN * i) + (lane >> 3);
    offA[i] = (uint32_t)((row * a.lda + 8 * ((lane & 7) ^ ((row >> 1) & 7))) * 2);
  }
  const uint32_t offB = (uint32_t)(l32 * Kh + 16 * h), offS = (uint32_t)(l32 * kgroups * 2);
  const uint32_t ssel = h ? 0x03020302u : 0x01000100u;  // this half's scale, twice
  uint4 rb[2][CS][NJ];  // codes of CS steps, two buffers
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
  // Step j (mod 8) of the loop issues the activation tile ST - 1 steps ahead, then (every CS
  // steps) the next CS steps' codes and (every four) the next four steps' scales, then
  // multiplies. It ends when this wave's loads of the next tile have landed (counting what was
  // issued after them) and, with a shared ring, so have the other waves'.
  constexpr int D = ST - 1;
  auto sync = [&](auto J_, auto T_) {
    wait_vmcnt<after_tile(decltype(J_)::value, D, NA, CS, decltype(T_)::value != 0)>();
    if constexpr (WN > 1) __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto step = [&](auto J_, auto T_, int k) {
    constexpr int j = decltype(J_)::value, cb = (j / CS) & 1, sb = (j / 4) & 1;
    constexpr bool tail = decltype(T_)::value != 0;
    load_a(IC<(j + D) % ST>{}, min(k + D, kt_end - 1));
    load_codes(IC<1 - cb>{}, IC<code_rows(j, CS, tail)>{}, k + CS);
    if constexpr (scale_rows(j, tail) > 0) load_scales(IC<1 - sb>{}, k + 4);
    uint32_t sw[NJ];
#pragma unroll
    for (int q = 0; q < NJ; ++q)
      sw[q] = j % 4 == 0 ? rsc[sb][q].x : j % 4 == 1 ? rsc[sb][q].y : j % 4 == 2 ? rsc[sb][q].z : rsc[sb][q].w;
    mma(IC<j % ST>{}, rb[cb][j % CS], sw);
    sync(J_, T_);
  };
  if (kt_begin < kt_end) {
    // the LoRA term starts the accumulators while the first tiles are in flight (of a split
    // reduction: those of the last group, whose range is never empty)
    const bool lora0 = (WK == 1 || wk == WK - 1) && EPI != MID_LOGITS && SEG(s0, lora_B);
    const bool lora1 = EPI == MID_GATED ? (WK == 1 || wk == WK - 1) && a.seg[1].lora_B : lora0;
    load_codes(IC<0>{}, IC<CS>{}, kt_begin);
    load_scales(IC<0>{}, kt_begin);
    load_a(IC<0>{}, kt_begin);
    if constexpr (ST == 4) {
      load_a(IC<1>{}, min(kt_begin + 1, kt_end - 1));
      load_a(IC<2>{}, min(kt_begin + 2, kt_end - 1));
    }
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
        lora_acc<MI, NJ>(acc, u, v);
      } else {
        // gate and up have their own u
        const rsrc_t rU1 = make_rsrc(a.seg[1].lora_u, lora1 ? (size_t)a.M * r * 4 : 0);
        uint4 bh[NJ], bl[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) split_bf16(v[j], bh[j], bl[j]);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          float u1[8];
          load8(rU1, (uint32_t)(((m0 + 32 * i + l32) * r + q0) * 4), keep, a.lora_s, u1);
          uint4 ah, al;
          split_bf16(u[i], ah, al);
          acc[i][0] = mfma32<OpBF16>(ah, bh[0], acc[i][0]);
          acc[i][0] = mfma32<OpBF16>(ah, bl[0], acc[i][0]);
          acc[i][0] = mfma32<OpBF16>(al, bh[0], acc[i][0]);
          split_bf16(u1, ah, al);
          acc[i][1] = mfma32<OpBF16>(ah, bh[1], acc[i][1]);
          acc[i][1] = mfma32<OpBF16>(ah, bl[1], acc[i][1]);
          acc[i][1] = mfma32<OpBF16>(al, bh[1], acc[i][1]);
        }
      }
    }
    wait_vmcnt<(D - 1) * NA>();
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
  constexpr int ESZ = EPI == MID_F32 ? 4 : 2;
  const int ldo = SEG(s0, ldo), rope = EPI == MID_F16 ? SEG(s0, rope) : 0;
  auto out_rsrc = [&](void* base, int ld) {
    return make_rsrc((char*)base + (size_t)m0 * ld * ESZ, ((size_t)(rows - 1) * ld + Nn) * ESZ);
  };
  const rsrc_t rO = out_rsrc(SEG(s0, out), ldo);
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
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v0[r] + x.x0[r]), rO, o0, so, 0);
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v1[r] + x.x1[r]), rO, o1, so, 0);
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


// Tile configurations and their cost model: `fix` microseconds of launch, first loads and
// epilogue, then per K step of a wave `lat` while a compute unit has one workgroup at most and
// `thr` per workgroup when it has several. Measured on 27 products of 128 .. 16384 tokens with
// reductions of 896 .. 10240 (each configuration timed on each): the estimate is within about
// 15 % and picks the fastest configuration or one within 6 % of it.
struct MidCfg {
  int mi, wn, wk;
  float fix, lat, thr;
};
constexpr MidCfg kMid[] = {
    {4, 4, 1, 7.0f, 0.90f, 0.98f},  // 128 x 256: many tiles
    {4, 1, 4, 5.0f, 1.20f, 1.56f},  // 128 x 64, four K ranges: about 256 tiles
    {2, 1, 8, 6.0f, 1.40f, 1.70f},  // 64 x 64, eight K ranges: long reductions, few tiles
    {2, 1, 4, 5.0f, 0.80f, 0.85f},
    {2, 1, 2, 4.0f, 0.78f, 0.43f},
    {1, 1, 4, 3.5f, 0.50f, 0.53f},  // 32 x 64: the fewest tokens
};
constexpr int kMidCount = sizeof(kMid) / sizeof(kMid[0]);

int mid_columns(const MidCfg& c, const int* Ns, int nseg, bool gated) {
  if (gated) return (Ns[0] + 32 * c.wn - 1) / (32 * c.wn);
  int t = 0;
  for (int s = 0; s < nseg; ++s) t += (Ns[s] + 64 * c.wn - 1) / (64 * c.wn);
  return t;
}

int mid_pick(int M, const int* Ns, int nseg, int K, bool gated, bool logits) {
  int best = 0;
  float bt = 1e30f;
  for (int i = 0; i < kMidCount; ++i) {
    const MidCfg& c = kMid[i];
    if (logits && i) break;  // (whose statistics take whole rows of a wave)
    const int tiles = mid_columns(c, Ns, nseg, gated) * ((M + 32 * c.mi - 1) / (32 * c.mi));
    const int pairs = (K / BK + 1) / 2, steps = 2 * ((pairs + c.wk - 1) / c.wk), per = (tiles + 255) / 256;
    const float t = c.fix + steps * (per <= 1 ? c.lat : per * c.thr);
    if (t < bt) {
      bt = t;
      best = i;
    }
  }
  return best;
}

}  // namespace

bool gemm_nt_mid_ok(int K) { return K % BK == 0; }

hipError_t launch_gemm_nt_mid(const NtArgs& a0, int epi, double flops, double bytes, hipStream_t st) {
  NtArgs a = a0;
  if (a.K % BK || a.lda % 8 || ((uintptr_t)a.X & 15)) return hipErrorInvalidValue;
  int Ns[3];
  for (int s = 0; s < a.nseg; ++s) Ns[s] = a.seg[s].N;
  const int pick = mid_pick(a.M, Ns, a.nseg, a.K, a.gated, epi == NT_LOGITS);
  const MidCfg& c = kMid[pick];
  int t = 0;
  for (int s = 0; s < a.nseg; ++s) {
    a.seg[s].tile0 = t;
    t += (a.seg[s].N + 64 * c.wn - 1) / (64 * c.wn);
  }
  const dim3 grid(mid_columns(c, Ns, a.nseg, a.gated), (a.M + 32 * c.mi - 1) / (32 * c.mi));
  const char* name = epi == NT_STORE_F16 ? "gemm_nt_f16out" : epi == NT_STORE_F32 ? "gemm_nt_f32out" : "gemm_nt_logits";
#define MID_GO(MI, WN, WK, EPI) \
  MEBP_TIMED(st, name, flops, bytes, \
             hipLaunchKernelGGL((k_gemm_nt_mid<MI, WN, WK, 2, 2, EPI>), grid, dim3(64 * WN * WK), 0, st, a))
#define MID_EPI(MI, WN, WK)              \
  do {                                   \
    if (a.gated)                         \
      MID_GO(MI, WN, WK, MID_GATED);     \
    else if (epi == NT_STORE_F16)        \
      MID_GO(MI, WN, WK, MID_F16);       \
    else                                 \
      MID_GO(MI, WN, WK, MID_F32);       \
  } while (0)
  if (epi == NT_LOGITS) {
    MID_GO(4, 4, 1, MID_LOGITS);
    return hipGetLastError();
  }
  switch (pick) {
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

}  // namespace mebp
