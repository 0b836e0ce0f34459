// Tiled verify-mode (W4A16) kernel for M > 32: in-register int4 -> fp16
// dequantisation feeding v_mfma_f32_32x32x16_f16 (paper Sec. 1 item (1): the
// 4-bit weights are dequantised to fp16 at run time; Sec. 4.1: groups of 128).
//
// A workgroup of WGN x WGM x WGK wavefronts owns BN x BM outputs (BN = 32*PN*WGN
// features, BM = 32*PM*WGM tokens) over a range of K groups; a wavefront owns
// PN x PM MFMA tiles of 32 x 32.  WGK > 1: the wavefronts are WGK sets that cover the
// same block, set wk takes every WGK-th group, and the sets' partial sums meet in LDS at
// the end.  That is how eight wavefronts work on a block of 128 x 64 or 64 x 64 where the
// problem has no more blocks than compute units: with four (one per SIMD) every wait of a
// wave idles its SIMD (128 x 64 blocks, 12288 x 4096 at 128 tokens, 192 blocks: 22.3 us on four
// wavefronts, 18.5 on eight; 5120 x 5120 at 384, 240 blocks: 27.6 and 24.3).
//   - Activations: the BM x 128 fp16 block of a group travels global -> LDS
//     with buffer loads that write LDS directly (no registers, no ds_write),
//     one group ahead, into two stages that are separate arrays (the compiler
//     then knows that a transfer into one never aliases a read of another
//     and inserts no wait between them).  A wave-wide transfer fills 1 KB of
//     LDS linearly (lane l -> bytes 16l..16l+15) = four token rows; the
//     16-byte slot s of row r holds k-chunk s ^ (r % 16), chosen on the
//     global-address side, so that the 16 rows a quarter-wave reads fall into
//     16 different bank groups.
//   - Weights: every wavefront fetches the code tiles of its own rows straight
//     into registers in MFMA operand layout through a ring of NW groups and
//     dequantises them itself.
//   - Order of issue inside a group is pinned with scheduling fences: the LDS
//     reads of a later k-step first, then the MFMAs of this k-step with the
//     dequantisation of the NEXT k-step cut into stages of independent operations
//     between them.  Left to itself the compiler puts every LDS read next to its first use.
//   - What bounds the loop where the power limit does not: issue slots.  Between the MFMAs (32
//     cycles each) two wavefronts of a SIMD fit six independent vector operations, one wavefront
//     alone four; every further one costs 4.9 cycles (a loop of MFMAs with n packed fp16
//     products behind each, ns per MFMA of a SIMD: 15.7 up to n = 3, 17 at 4 to 6, 18.9 at 7, 24.0
//     at 10; one wavefront: 34.5 cycles at n = 0, 38 at 4, 48 at 6, 62 at 10).  A 64-token wave tile
//     needs 6.5 for the dequantisation alone.  Hence no address arithmetic in the loop: what
//     moves with the group is a scalar offset of the load, LDS addresses differ from a lane's
//     fixed one by constant bits (vector operations per MFMA in the compiled loops: 7.5 -> 6.5 on
//     64-token wave tiles, 4.0 -> 3.3 on 128-token ones; on the same 128 x 128 blocks 57344 x 8192
//     at 512 tokens 455 -> 442 us, 11008 -> 4096 at 2050 238 -> 227).
//
// A operand (32 rows x 16 k): lane l supplies 8 consecutive k of row l % 32,
// lanes 0..31 the first 8 k of the step, lanes 32..63 the second 8.  In the blob
// the 16 bytes of tile lane (r, kb) are words i = 0..3 holding k-chunks (8 k each)
// 4i + kb.  So lane l = (h = l / 32, row = l % 32) fetches, from the 16-row tile
// that holds its row, the 16 bytes of tile lane (row % 16, h) ["lo"] and of tile
// lane (row % 16, h + 2) ["hi"]: word i of lo is chunk 4i + h, word i of hi is
// chunk 4i + 2 + h, and step s = 2i + e (e = 0: lo, 1: hi) covers the 16
// consecutive k = 32i + 16e .. +15.  The B operand of that step is, for lane
// (h, m = l % 32), chunk 4i + 2e + h of token row m.
// D: lane holds column m = l % 32 and rows 8a + 4h + r (a, r = 0..3) in
// register 4a + r: four runs of four consecutive output features.
#pragma once
#include "tile_common.hpp"

namespace qspec {

// s_waitcnt immediate for "at most n vector-memory operations outstanding",
// leaving the other counters alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14,
// expcnt 6:4, lgkmcnt 11:8).
constexpr int waitcnt_vm(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }
// the same with lgkmcnt(0): every LDS (and scalar-memory) operation of the wave has completed too
constexpr int waitcnt_vm_lgkm0(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4); }

template <int PN, int PM, int WGN, int WGM, int WGK, int NW, int OCC>
__global__ __launch_bounds__(64 * WGN * WGM * WGK, OCC) void gemm_tile16w_kernel(QSPEC_TILE_PARAMS) {
  const TileArgs p = QSPEC_TILE_ARGS;
  constexpr int kWaves = WGN * WGM * WGK;
  constexpr int kTileWaves = WGN * WGM;                // the waves that cover the output block once
  constexpr int BM = 32 * PM * WGM;
  constexpr int kStageBytes = BM * 256 * WGK;
  constexpr int U = BM * 256 / 1024 / kTileWaves;      // wave-wide transfers per wave and group
  static_assert(BM * 256 % (1024 * kTileWaves) == 0, "the stage divides evenly among the waves");
  static_assert(NW == 2 || NW == 4, "the stage of a group must follow from its ring slot");
  // two stages, each an array of its own (see the head of this file)
  __shared__ __attribute__((aligned(1024))) uint8_t xs0[kStageBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t xs1[kStageBytes];
  auto stage_ptr = [&](int i) -> uint8_t* { return i == 0 ? xs0 : xs1; };

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / kTileWaves, wt = wave % kTileWaves;
  const int wn = wt % WGN, wm = wt / WGN;
  const int m32 = lane & 31, h = lane >> 5;
  const int G = p.G;
  const TileCoord tc = tile_coord(p, total);
  const int g0 = tc.g0, g1 = tc.g1;
  const int n0 = (tc.nblk * (PN * WGN) + wn * PN) * 32;      // first output feature of this wave
  const int m0 = tc.mblk * BM;
  const int mw0 = wm * (PM * 32);

  // Every workgroup walks its K groups in the same order, trip q = 0 .. ng-1 -> group g0 + q:
  // the workgroups of an XCD then need the same narrow window of activation columns at
  // about the same time and find it in their L2.  (Starting each weight stripe at a
  // different group was measured: no faster, and 9x the algorithmic bytes fetched,
  // because the whole activation matrix then has to live in a 4 MB L2.)
  // (WGK > 1: trip q of the workgroup is the WGK groups g0 + q * WGK .., one for each set of waves;
  // a set that has no group in the last trip, nmine = ng - 1, sits that trip out)
  const int ng = (g1 - g0 + WGK - 1) / WGK;
  const int nmine = (g1 - g0 - wk + WGK - 1) / WGK;
  auto group_of = [&](int q) -> int { return g0 + q * WGK + wk; };
  // A lane's part of an address is fixed; what moves with the group is wave-uniform and goes into
  // the load's scalar offset, so that a group costs no vector address arithmetic.  Requests past
  // the end go through an empty buffer descriptor: zeros, no traffic, no branch.

  // ---- activations: global -> LDS.  Transfer u of this wave fills block q = wt +
  // u*kTileWaves of its set's stage (1 KB = rows 4q..4q+3).  Lane l writes slot l%16 of row 4q + l/16 and so
  // must fetch k-chunk (l%16) ^ (row%16).  Rows past M are out of range: no traffic, and
  // whatever the stage holds there reaches only outputs that are not stored.
  uint32_t x_voff[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int row = 4 * (wt + u * kTileWaves) + (lane >> 4);
    x_voff[u] = m0 + row < p.M ? (uint32_t)(m0 + row) * (uint32_t)p.K * 2u + (uint32_t)(((lane & 15) ^ (row & 15)) << 4) : kOutOfRange;
  }
  auto dma_x = [&](int q, uint8_t* stage) {
    const int g = group_of(q);
    const uint32_t bytes = g < g1 ? (uint32_t)((size_t)p.M * p.K * 2) : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u)
      buf_load16_lds(p.act, bytes, stage + wk * (BM * 256) + (wt + u * kTileWaves) * 1024, x_voff[u], (uint32_t)g * 256u);
  };

  // ---- weights: per 32-row pair two 16-byte pieces (lo, hi) and the row's scale (bit 31 of a
  // lane's offset: its row lies past N)
  uint4 wlo[NW][PN], whi[NW][PN];
  uint32_t sq[NW][PN];
  const int n_lane = n0 + m32;          // this lane's weight row in pair 0
  uint32_t w_voff[PN], s_voff[PN];
#pragma unroll
  for (int j = 0; j < PN; ++j) {
    const uint32_t none = n_lane + 32 * j >= p.N ? kOutOfRange : 0u;
    w_voff[j] = ((uint32_t)((n_lane >> 4) + 2 * j) * G * 1024u + (uint32_t)((n_lane & 15) + 16 * h) * 16u) | none;
    s_voff[j] = (uint32_t)(n_lane + 32 * j) * 2u | none;
  }
  auto load_w = [&](int d, int q) {
    const int g = group_of(q);
    const uint32_t cbytes = g < g1 ? (uint32_t)((size_t)p.N * p.K / 2) : 0u, sbytes = g < g1 ? (uint32_t)((size_t)p.N * G * 2) : 0u;
#pragma unroll
    for (int j = 0; j < PN; ++j) {
      wlo[d][j] = buf_load16(p.codes, cbytes, w_voff[j], (uint32_t)g * 1024u);
      whi[d][j] = buf_load16(p.codes, cbytes, w_voff[j] + 512u, (uint32_t)g * 1024u);
      sq[d][j] = buf_load_u16(p.scalesT, sbytes, s_voff[j], (uint32_t)g * (uint32_t)p.N * 2u);
    }
  };

  v16f acc[PN][PM];
#pragma unroll
  for (int j = 0; j < PN; ++j)
#pragma unroll
    for (int t = 0; t < PM; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][t][r] = 0.0f;

  dma_x(0, xs0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int d = 0; d < NW; ++d) load_w(d, d);
  __builtin_amdgcn_sched_barrier(0);

  v2h s2[PN], s2n[PN], wa0[PN][4];
#pragma unroll
  for (int j = 0; j < PN; ++j) {
    const _Float16 sc = __builtin_bit_cast(_Float16, (uint16_t)sq[0][j]);
    s2[j] = v2h{sc, sc};
    s2n[j] = s2[j];
#pragma unroll
    for (int hh = 0; hh < 4; ++hh) wa0[j][hh] = dequant_pair_scaled(wlo[0][j].x, hh, s2[j]);
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(3 * PN * NW));       // (the activations; of the weights the first group has been waited for)
  __builtin_amdgcn_s_barrier();

  constexpr int Q = PN * PM;                   // MFMAs per k-step (16 k), one LDS read feeds PN of them
  static_assert(PM >= 2, "the dequantisation of a word takes two stages at least");

  // LDS reads run XB-1 k-steps ahead of the MFMAs that consume them: a k-step of a
  // small wave tile is too short (PN*PM*32 cycles) to cover the LDS latency alone.
  // EARLY (wave tiles of four or more MFMAs per k-step, reads one step ahead): the barrier
  // that ends a group stands in front of its LAST k-step instead of behind it.  By then a
  // wave has issued every LDS read of the group, so the barrier certifies what the one at
  // the end did (everyone is done with this stage, everyone's transfers of the next stage
  // have landed), and the first operands of the next group are read under the last
  // k-step's MFMAs: no wave starts a group by waiting for LDS with nothing to issue.
  constexpr bool EARLY = PN * PM >= 4;
  constexpr int XB = EARLY ? 2 : 4;
  uint4 xb[XB][PM];
  // this lane's k-chunk of step s is 2 s + h: s only flips bits of a lane's address
  const int x_lane = wk * (BM * 256) + (mw0 + m32) * 256 + ((h ^ (m32 & 15)) << 4);
  auto read_step_from = [&](const uint8_t* xl, int s, uint4 (&dst)[PM]) {
#pragma unroll
    for (int t = 0; t < PM; ++t) dst[t] = *reinterpret_cast<const uint4*>(xl + (x_lane ^ (s << 5)) + t * 8192);
  };
  if constexpr (EARLY) read_step_from(xs0, 0, xb[0]);      // group 0, k-step 0

  // LEFT_OVER: one of the last groups, behind the loop.  Its ring slot is not refilled, so nothing is
  // younger than the next group's activations and the wait for them is for everything.  (A refill
  // that nobody reads would be removed by the compiler, and the counted wait with it be too lax.)
  auto group_body = [&](auto slot_c, int g, auto left_over_c) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_c)::value;
    constexpr bool LEFT_OVER = decltype(left_over_c)::value;
    constexpr int kYounger = LEFT_OVER ? 0 : 3 * PN;   // loads issued after those activations: the ring slot's
    constexpr int NEXT = (SLOT + 1) % NW;
    const uint8_t* xl = stage_ptr(SLOT % 2);
    uint8_t* xl_next = stage_ptr((SLOT + 1) % 2);      // last read in the group before this one
    auto read_step = [&](int s, uint4 (&dst)[PM]) { read_step_from(xl, s, dst); };
    auto word_of_step = [&](int d, int j, int s) -> uint32_t {
      const uint4& q = (s & 1) ? whi[d][j] : wlo[d][j];
      return word_of(q, s >> 1);
    };
    if constexpr (!EARLY) {
#pragma unroll
      for (int s = 0; s < XB - 1; ++s) read_step(s, xb[s]);
    }
    __builtin_amdgcn_sched_barrier(0);
    DequantWord dw;
    v2h wa[2][PN][4];                            // k-step s lives in wa[s & 1]
#pragma unroll
    for (int j = 0; j < PN; ++j)
#pragma unroll
      for (int hh = 0; hh < 4; ++hh) wa[0][j][hh] = wa0[j][hh];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      if (kWaves == 8 && s % 2 == 0) setprio_quarter(s / 2);
      if (s + XB - 1 < 8) read_step(s + XB - 1, xb[(s + XB - 1) % XB]);
      if constexpr (EARLY) {
        if (s == 7) {
          // (the count as at the end of the group: the ring refill of k-step 6 is the youngest
          // load; lgkmcnt(0): this wave's reads of the stage have completed, not only issued)
          __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(kYounger));
          __builtin_amdgcn_s_barrier();
          read_step_from(xl_next, 0, xb[0]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (s == 1) {
        // every wave has passed the barrier that ended the last group reading that
        // stage; issued here rather than at the top so that the first MFMAs of the
        // group do not queue behind the address computations
        dma_x(g + 1, xl_next);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int t = q / PN, j = q % PN;
        {
          const v8h av = v8h{wa[s & 1][j][0].x, wa[s & 1][j][0].y, wa[s & 1][j][1].x, wa[s & 1][j][1].y,
                             wa[s & 1][j][2].x, wa[s & 1][j][2].y, wa[s & 1][j][3].x, wa[s & 1][j][3].y};
          const v8h xv = __builtin_bit_cast(v8h, xb[s % XB][t]);
          acc[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, xv, acc[j][t], 0, 0, 0);
        }
        // the word of pair jj for the next k-step, in PM stages between the MFMAs (t counts within jj)
        {
          const int jj = q / PM, st = q % PM;
          const uint32_t word = s < 7 ? word_of_step(SLOT, jj, s + 1) : wlo[NEXT][jj].x;
          if (st == 0) dw.bits(word);
          if (st == (PM > 2 ? 1 : 0)) dw.codes_lo();
          if (st == 1) dw.codes_hi();
          if (st == (PM > 2 ? 2 : 1)) {
            if (s < 7) dw.scale(s2[jj], wa[(s + 1) & 1][jj]);
            else dw.scale(s2n[jj], wa0[jj]);
          }
        }
        if (s == 6 && q + 1 == Q) {
          // every word of this slot is in registers as fp16 now: refill it, and turn the
          // next slot's scales (fetched NW-1 groups ago) into fp16 pairs
          if constexpr (!LEFT_OVER) load_w(SLOT, g + NW);
#pragma unroll
          for (int jn = 0; jn < PN; ++jn) {
            const _Float16 sn = __builtin_bit_cast(_Float16, (uint16_t)sq[NEXT][jn]);
            s2n[jn] = v2h{sn, sn};
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int j = 0; j < PN; ++j) s2[j] = s2n[j];
    // The next group's activations were requested before the 3*PN loads that refill the ring
    // slot.  Loads complete in order: at most that many outstanding means those activations
    // have landed.  (No store may sit between them - stores complete out of order with
    // loads - so this kernel must compile without register spills in the loop.)
    if constexpr (!EARLY) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(kYounger));
      __builtin_amdgcn_s_barrier();
    }
  };

  // Whole turns of the weight ring, then the groups left over in copies of their own: no arithmetic
  // on zeros for a group past the end (an infinite activation would turn it into NaN), and no
  // exit inside the loop.  (One loop with an exit behind every group takes up to 56 registers
  // more and is slower on every shape: 12288 x 4096 at 128 tokens on 128 x 64 blocks in two sets
  // 21.9 us, 20.6 this way; 13824 -> 5120 at 384 on 128 x 128 in two sets 82.3 and 73.0; 57344 x
  // 8192 at 64 on 128 x 64, three per unit, 88.2 and 82.1.)
  std::false_type in_loop;
  std::true_type left_over;
  int q = 0;
  for (; q + NW <= nmine; q += NW) {
    group_body(std::integral_constant<int, 0>{}, q, in_loop);
    group_body(std::integral_constant<int, 1>{}, q + 1, in_loop);
    if constexpr (NW > 2) {
      group_body(std::integral_constant<int, 2 % NW>{}, q + 2, in_loop);
      group_body(std::integral_constant<int, 3 % NW>{}, q + 3, in_loop);
    }
  }
  if (q < nmine) group_body(std::integral_constant<int, 0>{}, q, left_over);
  if constexpr (NW > 2) {
    if (q + 1 < nmine) group_body(std::integral_constant<int, 1>{}, q + 1, left_over);
    if (q + 2 < nmine) group_body(std::integral_constant<int, 2 % NW>{}, q + 2, left_over);
  }
  // the barrier of the trip that this set sat out (a set reads only activations it fetched itself)
  if (WGK > 1 && nmine < ng) __builtin_amdgcn_s_barrier();

  if constexpr (WGK == 1) {
    // (every wave's reads of the stages are behind the last group's barrier; transfers past the end may still be under way)
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    static_assert(kWaves * 4096 * PN <= kStageBytes, "4096 PN bytes of a stage for each wave");
    tile_store32<PN, PM, 64 * kWaves>(p, tc, acc, n0, m0 + mw0, xs0 + wave * (4096 * PN));
  } else {
    // Each of the WGK waves of an output tile set finishes PN * PM / WGK of its tiles.  All partial
    // sums go through LDS (a wave's own too: which tiles it finishes is not known at compile
    // time); the stages are dead, the barrier that ended the last group is behind every read of
    // them, and requests past the end have landed.
    constexpr int kT = PN * PM, PF = kT / WGK;
    static_assert(kT % WGK == 0 && kT % 2 == 0 && PM % PF == 0, "whole tiles of one feature column to finish per wave");
    static_assert(kTileWaves * WGK * (kT / 2) * 4096 <= kStageBytes, "half the tiles fit a stage");
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    // partial src of tile t: floats 4a .. 4a+3 of lane l at a * 256 + 4 l
    auto slot = [&](int t, int src) -> float4* {
      const int i = ((t % (kT / 2)) * WGK + src) * kTileWaves + wt;
      return reinterpret_cast<float4*>(t < kT / 2 ? xs0 : xs1) + i * 256 + lane;
    };
#pragma unroll
    for (int t = 0; t < kT; ++t)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        const v16f& v = acc[t / PM][t % PM];
        slot(t, wk)[a * 64] = float4{v[4 * a], v[4 * a + 1], v[4 * a + 2], v[4 * a + 3]};
      }
    __syncthreads();
    float fin[1][PF][16];
#pragma unroll
    for (int f = 0; f < PF; ++f)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        float4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int src = 0; src < WGK; ++src) {
          const float4 v = slot(wk * PF + f, src)[a * 64];
          sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        fin[0][f][4 * a] = sum.x; fin[0][f][4 * a + 1] = sum.y; fin[0][f][4 * a + 2] = sum.z; fin[0][f][4 * a + 3] = sum.w;
      }
    // (only this wave reads the partial sums of its tiles: one of them is its scratch now)
    tile_store32<1, PF, 64 * kWaves>(p, tc, fin, n0 + 32 * (wk * PF / PM), m0 + mw0 + 32 * (wk * PF % PM),
                                     reinterpret_cast<uint8_t*>(slot(wk * PF, 0) - lane));
  }
}

}  // namespace qspec
