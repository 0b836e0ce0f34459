// Memory-bound (small M) kernels for both modes, wave-autonomous form.
//
// A workgroup of W wavefronts (8, or 4: namespace waves4) owns NT adjacent weight tiles (16 outputs each) over the whole
// of K and 16 TM token rows.  The K groups are dealt to the wavefronts; a wavefront loads the
// activations of its groups once and uses them against the NT weight tiles, which stream from
// HBM exactly once.  There is no barrier in the streaming loop: everything a wavefront stages
// sits in a part of LDS that is its own (LDS executes a wavefront's accesses in order).  The
// W fp32 sums of a tile are combined through LDS at the very end and stored as fp16.
//
// A launch takes its time on the chip plus 1.1 us, and never less than 1.7.  Of 3.0 us on the chip (4096 x 4096 at
// one token; a bare read 1.8) 0.5 are spent before the first loads are out and 0.45 after the last group, so
//  - what the first loads need comes first and from the host's arguments where it can; LDS addresses are worked
//    out while the loads are on the way;
//  - a wavefront lays its sums down 16 bytes per lane, all tiles at once, and the W sums of a tile are read
//    together;
//  - the loads of the next step are issued across the end of a chunk of scales as well.
// Together (us on eight wavefronts, one run): 4096 x 4096 at one token 4.4 -> 4.1, 12288 x 4096 7.1 -> 6.6, 22016 x 4096 at 32 tokens
// 11.9 -> 11.3, verify mode 14.5 -> 13.6; 27648 x 5120 at 64 tokens 27.1 -> 23.8.
//
// What bounds it is the read of the weights, and next to that the number of cache LINES its
// loads touch: the vector L1 looks up one 128-byte line per clock and quarter wavefront, so a
// load whose 16 lanes hit 16 rows costs 16 lookups however few bytes it brings.  Hence:
//  - activations are loaded with adjacent lanes on adjacent bytes of a row and turned into the
//    MFMA operand through LDS.  (Loaded in operand layout, with one token scale per row and
//    load, the draft mode at 64 tokens, 15360 x 5120, did 24200 lookups per compute unit
//    = 11.5 us of its 19; 14.9 with that alone.  5120 x 13824: 22.9 -> 17.7; 4096 x 11008 at 32 tokens:
//    10.8 -> 8.3.)
//  - the scales of up to 16 groups come in a few wide loads at the start and wait in LDS.
//  - neighbouring tile blocks run on the same XCD, whose L2 then serves the 128-byte lines of
//    weight scales that four tiles share (0.2 to 0.8 us of every call).
//  - no load is issued for work that does not exist, except in the last step of a wavefront
//    with an odd number of groups: loads past the end cost the same issue time as others
//    (a set of six: 0.35 us).
// A weight tile's registers are refilled, with the same tile of the next step, as soon as its
// codes are widened.  Two or three steps in flight are slower everywhere (22016 x 4096 at 32
// tokens 12.0 -> 13.4 us; the reads only queue up).
//
// MFMA roles: A = activations (row = token), B = weights (column = output feature); lane
// (r16 = lane % 16, kb = lane / 16) of D holds tokens 4 kb .. 4 kb + 3 of output r16.  So a lane
// needs ONE weight scale per tile and group.  Draft mode: the MFMA chain starts from the bit
// pattern of 1.5 * 2^23, the finished int32 register READ AS A FLOAT is 12582912 + 256 P exactly
// (|256 P| <= 2^21), t = fma(that, sw, -12582912 sw) is the correctly rounded 256 P sw, and
// acc = fma(t, sa 2^-8, acc), the four token scales from LDS in one read.  Verify mode: the operands are
// the exact integer codes, and the scale goes onto the fp32 group sum.
#pragma once
#include <type_traits>

#include "buffer.hpp"
#include "exchange.hpp"
#include "common.hpp"

namespace qspec {

struct StreamArgs {
  const uint4* codes;        // blob code tiles
  const uint16_t* scalesT;   // blob fp16 scales [G][N]
  const void* act;           // W4A4: qa bytes [M][K/2]; W4A16: x fp16 [M][K]
  const float* sa;           // W4A4: [M][G]
  uint16_t* y;               // fp16 [M][N]
  float* ws;                 // S > 1: fp32 partial sums [S][tile block][output tile of 256]
  unsigned* tickets;         // S > 1: one arrival counter per tile block, zero on entry and on exit
  int M, N, K, G;
  int S;                     // K-slices: tile block b / S, slice b % S
  int per_slice, more_slice; // G / S, G % S
  int ms;                    // token-row blocks (1 with K-slices)
  uint32_t ms_rcp;           // 2^32 / ms, rounded up
  int blocks;                // tile blocks
  uint32_t workgroups;
};

constexpr int kStreamWaves = 8;

template <bool W4A4, int TM, int NT>
struct StreamShape {
  // Groups per step.  Two adjacent ones where few tiles per step would leave too few bytes in
  // flight (4096 x 11008 at one token 8.8 -> 6.9 us); their activations fill whole cache lines.
  static constexpr int QS = NT <= 2 && TM <= 4 ? 2 : 1;
  static constexpr int CH = TM >= 4 ? 8 : 16;               // groups of a wavefront whose scales are in LDS at a time
  static constexpr int kActTile = W4A4 ? 1024 : 4096;       // bytes of 16 token rows of one group
  static constexpr int GPL = 64 / (2 * NT);                 // groups per weight-scale load
  static constexpr int kSwN = (CH + GPL - 1) / GPL;         // weight-scale loads of a full chunk
  static constexpr int kSaOff = QS * TM * kActTile;
  static constexpr int kSwOff = kSaOff + (W4A4 ? CH * 16 * TM * 4 : 0);
  static constexpr int kStage = kSwOff + kSwN * GPL * NT * 32;
  static constexpr int kRed = NT * TM * 1024;
  // LDS of one wavefront: activations of a step, scales; at the end its sums
  static constexpr int kRegion = ((kStage > kRed ? kStage : kRed) + 255) / 256 * 256;
};

// Four values of one column per lane (s.x .. s.w: rows 0 .. 3) -> fp16, and across each quad of lanes (four adjacent
// columns) to four columns of one row per lane: lane q of the quad gets row q.  Every lane of the quad must be active.
__device__ __forceinline__ uint2 quad_transpose(float4 s, int lane) {
  const uint32_t a = (uint32_t)float_to_half_bits(s.x) | ((uint32_t)float_to_half_bits(s.y) << 16);
  const uint32_t b = (uint32_t)float_to_half_bits(s.z) | ((uint32_t)float_to_half_bits(s.w) << 16);
  // rows 0, 1 of columns q, q + 2 to the lower two lanes, rows 2, 3 to the upper two
  const bool upper = lane & 2, odd = lane & 1;
  const uint32_t r = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(upper ? a : b), 0x4E, 0xF, 0xF, false);   // lane ^ 2
  const uint32_t u = upper ? r : a, v = upper ? b : r;
  // the low halves to the even lane, the high ones to the odd
  const uint32_t give = __builtin_amdgcn_perm(v, u, odd ? 0x05040100u : 0x07060302u);
  const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)give, 0xB1, 0xF, 0xF, false);           // lane ^ 1
  // even: (u.lo, got.lo), (v.lo, got.hi); odd: (got.lo, u.hi), (got.hi, v.hi)
  return uint2{__builtin_amdgcn_perm(got, u, odd ? 0x03020504u : 0x05040100u),
               __builtin_amdgcn_perm(got, v, odd ? 0x03020706u : 0x07060100u)};
}

// The first 14 dwords of the arguments arrive in scalar registers with the wavefront (build flag
// amdgpu-kernarg-preload-count; only arguments passed one by one do): what the first loads need.  The rest is read
// when it is needed.  (12288 x 4096 at 32 draft tokens 7.65 -> 7.35 us, 27648 x 5120 at 64: 24.2 -> 24.0.)
struct StreamRest {
  uint16_t* y;
  float* ws;
  unsigned* tickets;
  int S, per_slice, more_slice, blocks;
};

#define QSPEC_STREAM_PARAMS                                                                                               \
  const uint4 *codes, const uint16_t *scalesT, const void *act_rows, const float *sa, int M, int N, int K, uint32_t workgroups, \
      int ms, uint32_t ms_rcp, StreamRest rest

// workgroups: how many (each XCD gets an eighth of them, the first ones one more); ms == 0: K-slices.
template <bool W4A4, int TM, int NT, int W>
__device__ __forceinline__ void stream_product(QSPEC_STREAM_PARAMS) {
  using C = StreamShape<W4A4, TM, NT>;
  constexpr int QS = C::QS, CH = C::CH, T = NT * TM;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[W * C::kRegion];
  __shared__ unsigned ticket;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroups go to the eight XCDs in turn: each XCD gets a run of adjacent tile blocks, and of each of
  // them all token-row blocks one after the other, so that they find its weights in that XCD's L2.
  const int xcd = blockIdx.x & 7;
  const int bx = xcd * (int)(workgroups >> 3) + min(xcd, (int)(workgroups & 7)) + (int)(blockIdx.x >> 3);
  const int G = (int)((unsigned)K / kGroup);
  const bool sliced = ms == 0;
  int tb = bx, slice = 0, s0 = 0, s1 = G, m_base = 0;
  if (__builtin_expect(sliced, 0)) {
    tb = (int)((unsigned)bx / (unsigned)rest.S); slice = bx - tb * rest.S;
    s0 = slice * rest.per_slice + min(slice, rest.more_slice); s1 = s0 + rest.per_slice + (slice < rest.more_slice ? 1 : 0);
  } else if (ms > 1) {
    tb = (int)__umulhi((unsigned)bx, ms_rcp);    // bx / ms (exact below 2^28 workgroups), in the scalar unit
    m_base = (bx - tb * ms) * (16 * TM);
  }
  const int T0 = tb * NT;
  const int nt_valid = min(NT, (N >> 4) - T0);
  const int Mloc = M - m_base;
  if (Mloc <= 0) return;                           // (the whole workgroup: uniform)
  // group i of this wavefront, and how many it has: dealt round robin, QS adjacent ones at a time
  // (contiguous ranges per wavefront read the weights 10 to 20 % slower; workgroups that start at different
  // groups, so that they ask for different activations, are up to 10 % slower: the requests no longer meet)
  auto grp = [&](int i) -> int { return QS == 1 ? s0 + wave + W * i : s0 + QS * (wave + W * (i / QS)) + (i & (QS - 1)); };
  int n_g;
  {
    const int left = s1 - s0 - QS * wave, full = max(left, 0) / (QS * W);
    n_g = QS * full + min(max(left - full * (QS * W), 0), QS);
  }

  float facc[NT][TM][4];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int t = 0; t < TM; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) facc[j][t][r] = 0.0f;

  uint8_t* const mine = lds + wave * C::kRegion;
  if (n_g > 0) {
    const uint32_t codes_bytes = (uint32_t)(N >> 1) * (uint32_t)K;        // (all below 2^31)
    const uint32_t row_bytes = W4A4 ? (uint32_t)K >> 1 : (uint32_t)K * 2;
    const uint8_t* const act = static_cast<const uint8_t*>(act_rows) + (uint32_t)m_base * row_bytes;
    const rsrc_t r_act = make_rsrc(act, (uint32_t)Mloc * row_bytes);
    const rsrc_t r_scales = make_rsrc(scalesT, (uint32_t)N * (uint32_t)G * 2);
    const rsrc_t r_sa = make_rsrc(W4A4 ? (const void*)(sa + (uint32_t)m_base * (uint32_t)G) : (const void*)act, (uint32_t)Mloc * (uint32_t)G * 4);
    const uint32_t w_voff = lane * 16u;
    // activation loads of a step: kA of them, 1 KB each: 8 rows x 128 bytes (draft mode, two groups), 16 x 64
    // (draft mode, one group) or 4 x 256 (verify mode)
    constexpr int kA = W4A4 ? QS * TM : QS * TM * 4;
    constexpr int kLanesPerRow = W4A4 ? 4 * QS : 16, kRows = 64 / kLanesPerRow;
    const uint32_t a_voff = (uint32_t)(lane / kLanesPerRow) * row_bytes + (lane % kLanesPerRow) * 16u;
    // token scales: a load covers 16 tokens x 4 groups, four lines per quarter wavefront
    const int s_tok = 4 * (lane >> 4) + (lane & 3), s_grp = (lane >> 2) & 3;
    const uint32_t sa_voff = (uint32_t)s_tok * (uint32_t)G * 4u;
    const int z_grp = lane / (2 * NT), z_piece = lane - z_grp * (2 * NT);      // weight scales: 2 NT lanes per group
    const uint32_t sw_voff = (uint32_t)T0 * 32u + z_piece * 16u;
    const uint32_t z_gone = (uint32_t)((2 * nt_valid - 1 - z_piece) >> 31);

    uint4 w[QS][NT], ar[kA];
    const int n_s = (n_g + QS - 1) / QS;
    auto load_tile = [&](int s, int q, int j) __attribute__((always_inline)) {
      // (a tile past N or a group past the end: an empty buffer, zeros)
      const bool ok = (QS == 1 || s * QS + q < n_g) && j < nt_valid;
      const uint32_t soff = ((uint32_t)(T0 + j) * (uint32_t)G + (uint32_t)grp(s * QS + q)) * 1024u;
      typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
      const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(make_rsrc(codes, ok ? codes_bytes : 0u), w_voff, ok ? soff : 0u, 2);
      w[q][j] = uint4{v.x, v.y, v.z, v.w};
    };
    auto load_act = [&](int s) __attribute__((always_inline)) {
      if (W4A4) {
        const uint32_t gb = a_voff + (uint32_t)grp(s * QS) * 64u;
#pragma unroll
        for (int u = 0; u < kA; ++u) ar[u] = buf_load16(r_act, gb + (uint32_t)(kRows * u) * row_bytes);
      } else {
        const uint32_t gb = a_voff + (uint32_t)grp(s * QS) * 256u;
#pragma unroll
        for (int q = 0; q < QS; ++q)
#pragma unroll
          for (int u = 0; u < 4 * TM; ++u) ar[q * 4 * TM + u] = buf_load16(r_act, gb + q * 256u + (uint32_t)(4 * u) * row_bytes);
      }
    };
    // scales of CH groups from c0 on (zeros for groups and tiles that do not exist); token scales times 2^-8, exact
    constexpr int kSaN = CH / 4;
    float sar[W4A4 ? kSaN : 1][TM];
    uint4 swr[C::kSwN];
    auto load_scales = [&](int c0) __attribute__((always_inline)) {
      if (W4A4) {
#pragma unroll
        for (int k = 0; k < kSaN; ++k) {
          if (c0 + 4 * k >= n_g) break;
          const int i = c0 + 4 * k + s_grp;
          const uint32_t gone = (uint32_t)((n_g - 1 - i) >> 31) << 31;
#pragma unroll
          for (int t = 0; t < TM; ++t) sar[k][t] = buf_load_f32(r_sa, (sa_voff + (uint32_t)(16 * t * G + grp(i)) * 4u) | gone);
        }
      }
#pragma unroll
      for (int k = 0; k < C::kSwN; ++k) {
        if (c0 + C::GPL * k >= n_g) break;
        const int i = c0 + C::GPL * k + z_grp;
        const uint32_t gone = ((uint32_t)((n_g - 1 - i) >> 31) | z_gone) << 31;
        swr[k] = buf_load16(r_scales, ((uint32_t)grp(i) * (uint32_t)N * 2u + sw_voff) | gone);
      }
    };
    // (what takes the longest way first: with few rows the scales, whose lines nobody else has asked for; otherwise the
    // activations, which have to go through LDS.  15360 x 5120 at 64 tokens 13.6 us scales first, 13.2 activations
    // first, 4096 x 4096 at one token 4.1 and 4.2.  Weights before either cost 2 to 5 %.)
    if constexpr (TM == 1) {
      load_scales(0);
      load_act(0);
    } else {
      load_act(0);
      __builtin_amdgcn_sched_barrier(0);
      load_scales(0);
    }
#pragma unroll
    for (int q = 0; q < QS; ++q)
#pragma unroll
      for (int j = 0; j < NT; ++j) load_tile(0, q, j);
    __builtin_amdgcn_sched_barrier(0);
    // LDS addresses, from a copy of the lane number that does not exist before the first loads are out
    int lane2 = lane;
    asm volatile("" : "+v"(lane2));
    const int r16 = lane2 & 15, kb = lane2 >> 4;
    uint32_t st_off, rd_off[W4A4 ? QS : 4];
    if (W4A4) {
      if (QS == 2) {
        const int row = lane2 >> 3, sw = (r16 & 7) ^ (r16 >> 3);
        st_off = row * 128 + (((lane2 & 7) ^ row) << 4);     // rows 8 .. 15: the slot gets ^ 1
#pragma unroll
        for (int q = 0; q < QS; ++q) rd_off[q] = r16 * 128 + (((4 * q + kb) ^ sw) << 4);
      } else {
        const int row = lane2 >> 2;
        st_off = row * 64 + (((lane2 & 3) ^ ((row >> 1) & 3) ^ (row >> 3)) << 4);
        rd_off[0] = r16 * 64 + ((kb ^ ((r16 >> 1) & 3) ^ (r16 >> 3)) << 4);
      }
    } else {
      st_off = kb * 256 + ((r16 ^ kb) << 4);                 // rows 4u + kb: the slot gets ^ 4 (u % 4)
#pragma unroll
      for (int i = 0; i < 4; ++i) rd_off[i] = r16 * 256 + (((4 * i + kb) ^ r16) << 4);
    }
    uint32_t sa_wr = C::kSaOff + (s_grp * (16 * TM) + s_tok) * 4, sw_wr = C::kSwOff + z_grp * (NT * 32) + z_piece * 16;
    uint32_t sa_rd = C::kSaOff + kb * 16, sw_rd = C::kSwOff + r16 * 2;
    // (worked out before the first wait)
    asm volatile("" : "+v"(sa_wr), "+v"(sw_wr), "+v"(sa_rd), "+v"(sw_rd), "+v"(st_off));
#pragma unroll
    for (int i = 0; i < (W4A4 ? QS : 4); ++i) asm volatile("" : "+v"(rd_off[i]));
    auto put_scales = [&](int c0) __attribute__((always_inline)) {
      if (W4A4) {
#pragma unroll
        for (int k = 0; k < kSaN; ++k) {
          if (c0 + 4 * k >= n_g) break;
#pragma unroll
          for (int t = 0; t < TM; ++t) *reinterpret_cast<float*>(mine + sa_wr + k * (256 * TM) + t * 64) = sar[k][t] * 0.00390625f;
        }
      }
#pragma unroll
      for (int k = 0; k < C::kSwN; ++k) {
        if (c0 + C::GPL * k >= n_g) break;
        if (z_grp < C::GPL) *reinterpret_cast<uint4*>(mine + sw_wr + k * (C::GPL * NT * 32)) = swr[k];
      }
    };
    auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < kA; ++u) {
        uint32_t off = st_off;
        if (W4A4 && QS == 2 && (u & 1)) off ^= 16;
        if (!W4A4) off ^= (u & 3) << 6;
        *reinterpret_cast<uint4*>(mine + u * 1024 + off) = ar[u];
      }
    };
    constexpr int kSeed = 0x4B400000;                       // 12582912.0f
    v4i seed = {kSeed, kSeed, kSeed, kSeed};
    if (W4A4) asm volatile("" : "+v"(seed));
    auto rescale = [&](const v4i& acc, float sw, float swc, float4 S, float (&f)[4]) __attribute__((always_inline)) {
      const int b0 = acc[0], b1 = acc[1], b2 = acc[2], b3 = acc[3];
      f[0] = __builtin_fmaf(S.x, __builtin_fmaf(__builtin_bit_cast(float, b0), sw, swc), f[0]);
      f[1] = __builtin_fmaf(S.y, __builtin_fmaf(__builtin_bit_cast(float, b1), sw, swc), f[1]);
      f[2] = __builtin_fmaf(S.z, __builtin_fmaf(__builtin_bit_cast(float, b2), sw, swc), f[2]);
      f[3] = __builtin_fmaf(S.w, __builtin_fmaf(__builtin_bit_cast(float, b3), sw, swc), f[3]);
    };
    // one step: groups QS s .. QS s + QS - 1, whose scales sit in LDS from group c0 on.  (With an odd number of them the
    // draft mode multiplies the missing group's zeros, the verify mode skips it: zeros times an infinite activation.)
    auto step = [&](int s, int c0, auto refill_c) __attribute__((always_inline)) {
      constexpr bool kRefill = decltype(refill_c)::value;
      wave_lds_order();
      stage();
      if constexpr (kRefill) load_act(s + 1);                // (in between: a load goes out as soon as its registers are free)
      else __builtin_amdgcn_sched_barrier(0);                // (nothing that waits for weights in front of the stores)
      wave_lds_order();
      float swf[QS][NT];
      if constexpr (W4A4) {
        constexpr int D = 2;                              // an output tile is rescaled while the next D are in the matrix unit
        constexpr bool kTokenOuter = TM > NT;             // keep the fewer operands widened
        v4i acc[D + 1];
        float swc[QS][NT];
        float4 S[QS][TM];
        auto finish = [&](int e) __attribute__((always_inline)) {
          const int q = e / (NT * TM), j = kTokenOuter ? e % NT : e / TM % NT, t = kTokenOuter ? e / NT % TM : e % TM;
          rescale(acc[e % (D + 1)], swf[q][j], swc[q][j], S[q][t], facc[j][t]);
        };
#pragma unroll
        for (int q = 0; q < QS; ++q) {
          const int i = s * QS + q - c0;
#pragma unroll
          for (int t = 0; t < TM; ++t) S[q][t] = *reinterpret_cast<const float4*>(mine + sa_rd + i * (64 * TM) + t * 64);
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            swf[q][j] = half_bits_to_float(*reinterpret_cast<const uint16_t*>(mine + sw_rd + i * (NT * 32) + j * 32));
          }
          if constexpr (kTokenOuter) {
            I8Pair b[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) {
              b[j] = unpack_i8(w[q][j]);
              if constexpr (kRefill) load_tile(s + 1, q, j);
              swc[q][j] = swf[q][j] * -12582912.0f;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < TM; ++t) {
              const I8Pair a = unpack_i8(*reinterpret_cast<const uint4*>(mine + t * (QS * 1024) + rd_off[q]));
#pragma unroll
              for (int j = 0; j < NT; ++j) {
                const int e = (q * TM + t) * NT + j;
                acc[e % (D + 1)] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.lo, b[j].lo, seed, 0, 0, 0);
                acc[e % (D + 1)] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a.hi, b[j].hi, acc[e % (D + 1)], 0, 0, 0);
                if (e >= D) finish(e - D);
              }
            }
          } else {
            I8Pair a[TM];
#pragma unroll
            for (int t = 0; t < TM; ++t) a[t] = unpack_i8(*reinterpret_cast<const uint4*>(mine + t * (QS * 1024) + rd_off[q]));
            __builtin_amdgcn_sched_barrier(0);             // (no wait for weights before these are on the way)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
              const I8Pair b = unpack_i8(w[q][j]);
              if constexpr (kRefill) load_tile(s + 1, q, j);
              swc[q][j] = swf[q][j] * -12582912.0f;
              __builtin_amdgcn_sched_barrier(0);
#pragma unroll
              for (int t = 0; t < TM; ++t) {
                const int e = (q * NT + j) * TM + t;
                acc[e % (D + 1)] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[t].lo, b.lo, seed, 0, 0, 0);
                acc[e % (D + 1)] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[t].hi, b.hi, acc[e % (D + 1)], 0, 0, 0);
                if (e >= D) finish(e - D);
              }
            }
          }
        }
#pragma unroll
        for (int e = QS * NT * TM - D; e < QS * NT * TM; ++e) if (e >= 0) finish(e);
      } else {
        v4f acc[2][TM];
        auto finish = [&](int e) __attribute__((always_inline)) {
          const int q = e / NT, j = e % NT;
#pragma unroll
          for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) facc[j][t][r] = __builtin_fmaf(acc[e & 1][t][r], swf[q][j], facc[j][t][r]);
        };
#pragma unroll
        for (int q = 0; q < QS; ++q) {
          const int i = s * QS + q - c0;
          if (!kRefill && q > 0 && s * QS + q >= n_g) { finish(q * NT - 1); return; }
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            swf[q][j] = half_bits_to_float(*reinterpret_cast<const uint16_t*>(mine + sw_rd + i * (NT * 32) + j * 32));
          }
          v8h a[TM][4];
#pragma unroll
          for (int t = 0; t < TM; ++t)
#pragma unroll
            for (int k = 0; k < 4; ++k) a[t][k] = *reinterpret_cast<const v8h*>(mine + (q * TM + t) * 4096 + rd_off[k]);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            const int e = q * NT + j;
            const v8h b[4] = {dequant_word(w[q][j].x), dequant_word(w[q][j].y), dequant_word(w[q][j].z), dequant_word(w[q][j].w)};
            if constexpr (kRefill) load_tile(s + 1, q, j);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < TM; ++t) acc[e & 1][t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
              for (int t = 0; t < TM; ++t) acc[e & 1][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[t][k], b[k], acc[e & 1][t], 0, 0, 0);
            if (e > 0) finish(e - 1);
          }
        }
        finish(QS * NT - 1);
      }
    };
    put_scales(0);
    int s = 0;
    for (int c0 = 0;; c0 += CH) {
      const int stop = min(c0 / QS + CH / QS, n_s - 1);
      for (; s < stop; ++s) step(s, c0, std::integral_constant<bool, true>{});
      if (s == n_s - 1 && s < c0 / QS + CH / QS) {
        step(s, c0, std::integral_constant<bool, false>{});
        break;
      }
      load_scales(c0 + CH);                                  // (the loads of the next step are on the way meanwhile)
      wave_lds_order();                                      // (the scales of this chunk have been read)
      put_scales(c0 + CH);
    }
  }

  // ---- combine the W wavefronts through LDS: a wavefront lays its sums down 16 bytes per lane, as it holds
  // them (four tokens of one output), and adds up every W-th output tile; a 4 x 4 transposition among the lanes
  // of a quad then gives every lane four adjacent outputs of one token.  Rows past M take no part.  With
  // K-slices the sums go to the workspace first, and the workgroup that arrives last at the tile
  // block's counter adds the slices in slice order.
  const int kb = lane >> 4;
  uint16_t* const ytile = rest.y + (size_t)m_base * N + (size_t)T0 * 16 + (lane & 12);
  auto store_tile = [&](int o, float4 s) __attribute__((always_inline)) {
    const int j = o / TM, t = o - j * TM;
    const int m = 16 * t + 4 * kb + (lane & 3);
    const uint2 out = quad_transpose(s, lane);
    if (j < nt_valid && m < Mloc) *reinterpret_cast<uint2*>(ytile + (size_t)m * N + j * 16) = out;
  };
  // (overwrites only what this wavefront itself has read)
  wave_lds_order();
#pragma unroll
  for (int o = 0; o < T; ++o) {
    const float(&f)[4] = facc[o / TM][o % TM];
    if (16 * (o % TM) + 4 * kb < Mloc) *reinterpret_cast<float4*>(mine + o * 1024 + lane * 16) = float4{f[0], f[1], f[2], f[3]};
  }
  __syncthreads();
#pragma unroll
  for (int base = 0; base < T; base += W) {
    const int o = base + wave;
    if ((T % W == 0 || o < T) && 16 * (o % TM) + 4 * kb < Mloc) {
      float4 v[W];
#pragma unroll
      for (int u = 0; u < W; ++u) v[u] = *reinterpret_cast<const float4*>(lds + u * C::kRegion + o * 1024 + lane * 16);
      __builtin_amdgcn_sched_barrier(0);                     // (all of them on the way)
      float4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int u = 0; u < W; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
      if (__builtin_expect(sliced, 0)) {
        float* f = rest.ws + (((size_t)slice * rest.blocks + tb) * T + o) * 256 + lane * 4;
        store_shared_f2(f, s.x, s.y);
        store_shared_f2(f + 2, s.z, s.w);
      } else {
        store_tile(o, s);
      }
    }
  }
  if (!sliced) return;
  if (!last_arrival(rest.tickets, rest.S, (unsigned)tb, &ticket)) return;
  for (int o = wave; o < T; o += W) {
    if (16 * (o % TM) + 4 * kb >= Mloc) continue;
    float4 s = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int c = 0; c < rest.S; ++c) {            // fixed order: the result does not depend on who came last
      const float* f = rest.ws + (((size_t)c * rest.blocks + tb) * T + o) * 256 + lane * 4;
      const float2 a = load_shared_f2(f), b = load_shared_f2(f + 2);
      s.x += a.x; s.y += a.y; s.z += b.x; s.w += b.y;
    }
    store_tile(o, s);
  }
}

template <bool W4A4, int TM, int NT>
__global__ __launch_bounds__(kStreamWaves * 64, 2) void gemm_stream_kernel(QSPEC_STREAM_PARAMS) {
  stream_product<W4A4, TM, NT, kStreamWaves>(codes, scalesT, act_rows, sa, M, N, K, workgroups, ms, ms_rcp, rest);
}

// The same on four wavefronts, for plans of between one and two (from two token tiles on: three) rounds of
// workgroups.  The registers of eight wavefronts keep a second workgroup off a compute unit, so what comes before the
// first loads and after the last group of the one stands in front of the other; two workgroups of four wavefronts
// have it under each other's loops.  Measured against eight on the same plan: rule in qspec_api.hip.
namespace waves4 {
template <bool W4A4, int TM, int NT>
__global__ __launch_bounds__(256, 2) void gemm_stream_kernel(QSPEC_STREAM_PARAMS) {
  stream_product<W4A4, TM, NT, 4>(codes, scalesT, act_rows, sa, M, N, K, workgroups, ms, ms_rcp, rest);
}
}  // namespace waves4

}  // namespace qspec
