// Verify-mode (W4A16) kernel for large problems: 512 outputs x 128 tokens per workgroup of eight
// wavefronts, 64 x 128 per wavefront.  Same data layout, staging and dequantisation as
// gemm_tile16w_kernel (see there); no K-slices.
//
// What bounds it: the power limit.  The matrix loop of this part runs at 1.62 PFLOP/s on operands
// like these with nothing else in the loop, whatever the instruction rate would allow, and every
// vector operation and operand read beside it takes from that.  So the wave tile is chosen for
// energy, not for issue slots: with two 32-wide feature tiles per wavefront an activation operand
// is read from LDS once for two matrix instructions instead of for one (32 x 128 wave tiles), and
// 512 outputs per workgroup halve the activation bytes that enter a compute unit per output
// against 256.  Both need the registers of one workgroup per compute unit: 128 of 256 are
// accumulators.
// Measured at 57344 x 8192 and 512 tokens, one run: 442 us on 128 x 128 blocks, 445 on 256 x 128, 408
// with this kernel (381 on another machine, 1.26 PFLOP/s); 11008 -> 4096 at 2050 tokens 227, 247 and 216.
//
// Order inside a k-step: token tile by token tile, both feature tiles of it one after the other,
// then the operand register quad of that token tile is refilled for the next k-step (six matrix
// instructions ahead of its use).  The barrier that ends a group stands in the middle of its last
// k-step: by then the wave's reads of the stage have completed, and half a k-step of matrix
// instructions covers the first reads of the next stage.  The two waves of a SIMD take turns
// by progress (a wave's priority falls over a group): left to the hardware the older wave
// runs ahead to the barrier and the younger one then runs alone (384.7 us without the priorities,
// 380.8 with them; 11008 -> 4096 at 2050 tokens 191.1 and 185.6).
#pragma once
#include "gemm_tile16.hpp"

namespace qspec {

__global__ __launch_bounds__(512, 1) void gemm_tile16w2_kernel(QSPEC_TILE_PARAMS) {
  const TileArgs p = QSPEC_TILE_ARGS;
  constexpr int PN = 2, PM = 4, kWaves = 8;
  constexpr int BM = 32 * PM;
  constexpr int kStageBytes = BM * 256;
  constexpr int U = kStageBytes / 1024 / kWaves;
  __shared__ __attribute__((aligned(1024))) uint8_t xs0[kStageBytes];
  __shared__ __attribute__((aligned(1024))) uint8_t xs1[kStageBytes];
  auto stage_ptr = [&](int i) -> uint8_t* { return i == 0 ? xs0 : xs1; };

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m32 = lane & 31, h = lane >> 5;
  const int G = p.G;
  const TileCoord tc = tile_coord(p, total);
  const int n0 = (tc.nblk * kWaves + wave) * (PN * 32);
  const int m0 = tc.mblk * BM;

  uint32_t x_voff[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int row = 4 * (wave + u * kWaves) + (lane >> 4);
    x_voff[u] = m0 + row < p.M ? (uint32_t)(m0 + row) * (uint32_t)p.K * 2u + (uint32_t)(((lane & 15) ^ (row & 15)) << 4) : kOutOfRange;
  }
  auto dma_x = [&](int q, uint8_t* stage) {
    const uint32_t bytes = q < G ? (uint32_t)((size_t)p.M * p.K * 2) : 0u;
#pragma unroll
    for (int u = 0; u < U; ++u)
      buf_load16_lds(p.act, bytes, stage + (wave + u * kWaves) * 1024, x_voff[u], (uint32_t)q * 256u);
  };

  uint4 wlo[2][PN], whi[2][PN];
  uint32_t sq[2][PN];
  const int n_lane = n0 + m32;
  uint32_t w_voff[PN], s_voff[PN];
#pragma unroll
  for (int j = 0; j < PN; ++j) {
    const uint32_t none = n_lane + 32 * j >= p.N ? kOutOfRange : 0u;
    w_voff[j] = ((uint32_t)((n_lane >> 4) + 2 * j) * G * 1024u + (uint32_t)((n_lane & 15) + 16 * h) * 16u) | none;
    s_voff[j] = (uint32_t)(n_lane + 32 * j) * 2u | none;
  }
  auto load_w = [&](int d, int q) {
    const uint32_t cbytes = q < G ? (uint32_t)((size_t)p.N * p.K / 2) : 0u, sbytes = q < G ? (uint32_t)((size_t)p.N * G * 2) : 0u;
#pragma unroll
    for (int j = 0; j < PN; ++j) {
      wlo[d][j] = buf_load16(p.codes, cbytes, w_voff[j], (uint32_t)q * 1024u);
      whi[d][j] = buf_load16(p.codes, cbytes, w_voff[j] + 512u, (uint32_t)q * 1024u);
      sq[d][j] = buf_load_u16(p.scalesT, sbytes, s_voff[j], (uint32_t)q * (uint32_t)p.N * 2u);
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
  load_w(0, 0);
  load_w(1, 1);
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
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(3 * PN * 2));        // (the activations; of the weights the first group has been waited for)
  __builtin_amdgcn_s_barrier();
  const int x_lane = m32 * 256 + ((h ^ (m32 & 15)) << 4);
  v8h xb[PM];
  auto read_x = [&](const uint8_t* st, int s, int t) {
    xb[t] = *reinterpret_cast<const v8h*>(st + (x_lane ^ (s << 5)) + t * 8192);
  };
#pragma unroll
  for (int t = 0; t < PM; ++t) read_x(xs0, 0, t);

  auto group_body = [&](auto slot_c, int g) __attribute__((always_inline)) {
    constexpr int SLOT = decltype(slot_c)::value;
    constexpr int NEXT = SLOT ^ 1;
    const uint8_t* xl = stage_ptr(SLOT);
    uint8_t* xl_next = stage_ptr(NEXT);
    DequantWord dw;
    v2h wa[2][PN][4];
#pragma unroll
    for (int j = 0; j < PN; ++j)
#pragma unroll
      for (int hh = 0; hh < 4; ++hh) wa[0][j][hh] = wa0[j][hh];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      __builtin_amdgcn_sched_barrier(0);
      if (s % 2 == 0) setprio_quarter(s / 2);
      if (s == 0) {
        dma_x(g + 1, xl_next);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int t = 0; t < PM; ++t) {
#pragma unroll
        for (int j = 0; j < PN; ++j) {
          const v8h av = v8h{wa[s & 1][j][0].x, wa[s & 1][j][0].y, wa[s & 1][j][1].x, wa[s & 1][j][1].y,
                             wa[s & 1][j][2].x, wa[s & 1][j][2].y, wa[s & 1][j][3].x, wa[s & 1][j][3].y};
          acc[j][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, xb[t], acc[j][t], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          // the words of the next k-step, one per half of this one, in three stages
          const int pp = t * PN + j, jj = pp >> 2, st = pp & 3;
          const uint4& q = ((s + 1) & 1) ? whi[SLOT][jj] : wlo[SLOT][jj];
          if (st == 0) dw.bits(s < 7 ? word_of(q, (s + 1) >> 1) : wlo[NEXT][jj].x);
          if (st == 1) { dw.codes_lo(); dw.codes_hi(); }
          if (st == 2) {
            if (s < 7) dw.scale(s2[jj], wa[(s + 1) & 1][jj]);
            else dw.scale(s2n[jj], wa0[jj]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
        if (s < 7) {
          read_x(xl, s + 1, t);
        } else if (t == 1) {
          __builtin_amdgcn_s_waitcnt(waitcnt_vm_lgkm0(3 * PN));
          __builtin_amdgcn_s_barrier();
          read_x(xl_next, 0, 0);
          read_x(xl_next, 0, 1);
        } else if (t > 1) {
          read_x(xl_next, 0, t);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (s == 6) {
        load_w(SLOT, g + 2);
#pragma unroll
        for (int jn = 0; jn < PN; ++jn) {
          const _Float16 sn = __builtin_bit_cast(_Float16, (uint16_t)sq[NEXT][jn]);
          s2n[jn] = v2h{sn, sn};
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int j = 0; j < PN; ++j) s2[j] = s2n[j];
  };
  for (int q = 0; q + 1 < G; q += 2) {
    group_body(std::integral_constant<int, 0>{}, q);
    group_body(std::integral_constant<int, 1>{}, q + 1);
  }
  if (G & 1) group_body(std::integral_constant<int, 0>{}, G - 1);      // (no stage is read behind it: its counted wait guards nothing)
  // (every wave's reads of the stages are behind the last group's barrier; transfers past the end may still be under way)
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __syncthreads();
  static_assert(kWaves * 4096 * PN == 2 * kStageBytes, "4096 PN bytes of the stages for each wave");
  tile_write_rows<PN, PM>(p, acc, n0, m0, (wave < kWaves / 2 ? xs0 : xs1) + (wave % (kWaves / 2)) * (4096 * PN));
}

}  // namespace qspec
