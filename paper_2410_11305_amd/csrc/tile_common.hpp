// Shared pieces of the tiled (M > 32) kernels of both modes: launch arguments,
// the workgroup -> output block mapping, the int4 -> fp16 pair dequantiser, and
// the exchange of K-slice partial sums between workgroups.
//
// With S > 1 K-slices the S workgroups of one output block write their fp32
// accumulators to the workspace; the one that arrives last (an atomic ticket per
// output block) adds the S slices in slice order and stores fp16.  Nobody waits
// for anybody, so no workgroup needs another one to be resident.
#pragma once
#include "buffer.hpp"
#include "common.hpp"
#include "exchange.hpp"

#include <type_traits>

namespace qspec {

struct TileArgs {
  const uint4* codes;        // blob code tiles
  const uint16_t* scalesT;   // blob fp16 scales [G][N]
  const void* act;           // W4A4: qa bytes [M][K/2]; W4A16: x fp16 [M][K]
  const float* sa;           // W4A4: [M][G]
  uint16_t* y;               // fp16 [M][N]
  float* ws;                 // S > 1: fp32 partial sums, [S][output block][accumulator fragment]
  unsigned* tickets;         // S > 1: one counter per output block, zero on entry, zero on exit
  int M, N, K, G;
  int S;                     // K-slices
  int nb, mb;                // output blocks along N and along M
  uint32_t row_rcp;          // 2^32 / (mb S), rounded up; 0: not exact for these sizes, divide
};

// What a kernel needs late; the rest comes as arguments of its own, 13 dwords, in scalar registers when a wavefront
// starts (build flag amdgpu-kernarg-preload-count).
struct TileRest {
  uint16_t* y;
  float* ws;
  unsigned* tickets;
  int nb;
};
#define QSPEC_TILE_PARAMS \
  const uint4 *codes, const void *act, const float *sa, int M, int N, int K, int slices, int mb, uint32_t total, uint32_t row_rcp, TileRest rest
// (the scales follow the code tiles)
#define QSPEC_TILE_ARGS                                                                                                     \
  TileArgs {                                                                                                                \
    codes, reinterpret_cast<const uint16_t*>(reinterpret_cast<const uint8_t*>(codes) + (uint32_t)(N >> 1) * (uint32_t)K), act, sa, \
        rest.y, rest.ws, rest.tickets, M, N, K, (int)((unsigned)K / kGroup), slices, rest.nb, mb, row_rcp                        \
  }

// Which output block and K-slice a workgroup owns.  Workgroup ids are dealt
// round-robin to the 8 XCDs (each with its own L2): ids with the same id % 8 are
// renumbered to be neighbours, so that the blocks sharing a weight stripe (same
// n-block, all m-blocks and K-slices) run on one XCD and fetch it from HBM once.
struct TileCoord { int nblk, mblk, slice, g0, g1; };

__device__ __forceinline__ TileCoord tile_coord(const TileArgs& p, uint32_t total) {
  uint32_t logical = blockIdx.x;
  const uint32_t per = total >> 3;              // ids per XCD in the part that divides evenly
  if (blockIdx.x < per * 8) logical = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  TileCoord c;
  const uint32_t per_row = (uint32_t)(p.mb * p.S);
  // (five divisions in the vector unit took 0.3 us in front of the first load)
  uint32_t nblk = logical;
  if (p.row_rcp) nblk = __umulhi(logical, p.row_rcp);
  else if (per_row > 1) nblk = (uint32_t)__builtin_amdgcn_readfirstlane((int)(logical / per_row));
  c.nblk = (int)nblk;
  c.mblk = (int)(logical - nblk * per_row);
  c.slice = 0; c.g0 = 0; c.g1 = p.G;
  if (p.S > 1) {
    // (the divisions run in the vector unit; what depends on them, buffer descriptors among it,
    // has to be known to the compiler as wave-uniform)
    const unsigned rem = (unsigned)c.mblk, S = (unsigned)p.S;
    c.mblk = __builtin_amdgcn_readfirstlane((int)(rem / S));
    c.slice = (int)rem - c.mblk * p.S;
    c.g0 = __builtin_amdgcn_readfirstlane((int)((unsigned)(c.slice * p.G) / S));
    c.g1 = __builtin_amdgcn_readfirstlane((int)((unsigned)((c.slice + 1) * p.G) / S));
  }
  return c;
}

// Issue priority of the wave (q is a constant after unrolling): 3, 2, 1, 0 over the quarters of a group.
__device__ __forceinline__ void setprio_quarter(int q) {
  if (q == 0) __builtin_amdgcn_s_setprio(3);
  else if (q == 1) __builtin_amdgcn_s_setprio(2);
  else if (q == 2) __builtin_amdgcn_s_setprio(1);
  else __builtin_amdgcn_s_setprio(0);
}

// Pair h (0..3) of a word: codes (c_2h, c_2h+1) -> fp16 weights code*scale.
__device__ inline v2h dequant_pair_scaled(uint32_t w, int h, v2h s2) {
  const uint32_t v = h < 2 ? w : w >> 8;
  if ((h & 1) == 0) {
    const uint32_t b = (v & 0x000F000Fu) ^ 0x64086408u;           // 1024 + (code + 8)
    const v2h k1032 = {(_Float16)1032.0f, (_Float16)1032.0f};
    return (__builtin_bit_cast(v2h, b) - k1032) * s2;
  }
  const uint32_t b = (v & 0x00F000F0u) ^ 0x64806480u;             // 1024 + 16 * (code + 8)
  const v2h k72 = {(_Float16)72.0f, (_Float16)72.0f};
  const v2h k16th = {(_Float16)0.0625f, (_Float16)0.0625f};
  return (__builtin_bit_cast(v2h, b) * k16th - k72) * s2;
}

// The four pairs of a word together, cut into the stages a matrix loop places between its
// instructions: a stage holds only independent operations, so that a wave never waits for
// the vector unit's own latency (pair by pair, the three operations of a pair are a chain).
struct DequantWord {
  v2h b[4];
  __device__ __forceinline__ void bits(uint32_t w) {
    const uint32_t w8 = w >> 8;
    b[0] = __builtin_bit_cast(v2h, (w & 0x000F000Fu) ^ 0x64086408u);     // 1024 + (code + 8)
    b[1] = __builtin_bit_cast(v2h, (w & 0x00F000F0u) ^ 0x64806480u);     // 1024 + 16 * (code + 8)
    b[2] = __builtin_bit_cast(v2h, (w8 & 0x000F000Fu) ^ 0x64086408u);
    b[3] = __builtin_bit_cast(v2h, (w8 & 0x00F000F0u) ^ 0x64806480u);
  }
  __device__ __forceinline__ void codes_lo() {
    const v2h k1032 = {(_Float16)1032.0f, (_Float16)1032.0f};
    b[0] = b[0] - k1032;
    b[2] = b[2] - k1032;
  }
  __device__ __forceinline__ void codes_hi() {
    const v2h k72 = {(_Float16)72.0f, (_Float16)72.0f};
    const v2h k16th = {(_Float16)0.0625f, (_Float16)0.0625f};
    b[1] = b[1] * k16th - k72;
    b[3] = b[3] * k16th - k72;
  }
  __device__ __forceinline__ void scale(v2h s2, v2h (&out)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) out[i] = b[i] * s2;
  }
};

__device__ inline uint32_t word_of(const uint4& q, int i) {
  return i == 0 ? q.x : i == 1 ? q.y : i == 2 ? q.z : q.w;
}

// The partial sums of K-slice c of output block blk: the workgroup's accumulator
// registers in register-pair-major, thread-minor order (pair q of thread t at float
// 2*(q*threads + t)), so that every wave-wide store or load is one contiguous run
// of 512 bytes whatever the MFMA register layout is.
__device__ __forceinline__ float* slice_frag(const TileArgs& p, int c, unsigned blk, int floats_per_block) {
  return p.ws + ((size_t)c * (p.nb * p.mb) + blk) * (size_t)floats_per_block;
}
// fp16 store of a wave's PN x PM accumulator tiles of 32 x 32 (first output feature n0, first token row mrow0).  Two MFMA
// D layouts (h = lane / 32; a, r = 0..3; register 4a + r):
//   LANE_IS_TOKEN   lane holds token m = lane % 32 and features 8a + 4h + r;
//   !LANE_IS_TOKEN  lane holds feature n = lane % 32 and tokens 8a + 4h + r.
// LANE_IS_TOKEN: through LDS (`scratch`: 4096 PN bytes that belong to the wave), so that whole
// runs of 32 PN features of a token are stored 16 bytes per lane: a store in accumulator layout touches 32 lines with 16
// bytes each, 256 lines for a tile pair of 64 features where 32 hold it (512 x 128 blocks: 3.6 to 6.2 us between the last
// matrix instruction and the end of a workgroup).  The 16-byte slot s of row r sits at s ^ f(r), so that neither the
// 8-byte writes of 32 rows nor the reads meet in a bank.
template <int PN, int PM, typename Acc>
__device__ __forceinline__ void tile_write_rows(const TileArgs& p, const Acc (&acc)[PN][PM], int n0, int mrow0, uint8_t* scratch) {
  static_assert(PN <= 2, "slots of a row");
  constexpr int kRow = 64 * PN, kSlots = kRow / 16, kShift = PN == 1 ? 2 : 1;
  const int lane = threadIdx.x & 63;
  const int m32 = lane & 31, h = lane >> 5;
  const int wr = m32 * kRow + (((m32 >> kShift) & (kSlots - 1)) << 4) + 8 * h;
  const int row = lane / kSlots, slot = lane % kSlots;
  constexpr int kRows = 64 / kSlots;                       // token rows per store
  const int n = n0 + 8 * slot;
#pragma unroll
  for (int t = 0; t < PM; ++t) {
    uint8_t* const buf = scratch + (t & 1) * (32 * kRow);
    wave_lds_order();
#pragma unroll
    for (int j = 0; j < PN; ++j)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        uint2 out;
        out.x = (uint32_t)float_to_half_bits(acc[j][t][4 * a + 0]) | ((uint32_t)float_to_half_bits(acc[j][t][4 * a + 1]) << 16);
        out.y = (uint32_t)float_to_half_bits(acc[j][t][4 * a + 2]) | ((uint32_t)float_to_half_bits(acc[j][t][4 * a + 3]) << 16);
        *reinterpret_cast<uint2*>(buf + (wr ^ ((4 * j + a) << 4))) = out;
      }
    wave_lds_order();
#pragma unroll
    for (int i = 0; i < 32 / kRows; ++i) {
      const int r = i * kRows + row, m = mrow0 + 32 * t + r;
      const uint4 v = *reinterpret_cast<const uint4*>(buf + r * kRow + ((slot ^ ((r >> kShift) & (kSlots - 1))) << 4));
      if (m < p.M && n < p.N) *reinterpret_cast<uint4*>(p.y + (size_t)m * p.N + n) = v;
    }
  }
}

// The same for !LANE_IS_TOKEN tiles: a lane holds one feature of 16 tokens, so neighbouring lanes first trade halves (each
// gets two adjacent features of one token), and a row of 32 features is 64 bytes of LDS.
template <int PN, int PM, typename Acc>
__device__ __forceinline__ void tile_write_columns(const TileArgs& p, const Acc (&acc)[PN][PM], int n0, int mrow0, uint8_t* scratch) {
  const int lane = threadIdx.x & 63;
  const int l32 = lane & 31, h = lane >> 5, odd = lane & 1;
  const int row = lane >> 2, slot = lane & 3;
  // token 8a + 4h + r: its 16-byte slot is turned by bits 2 and 3 of the token
  const int wr = (4 * h + odd) * 64 + (l32 & ~1) * 2;
#pragma unroll
  for (int j = 0; j < PN; ++j)
#pragma unroll
    for (int t = 0; t < PM; ++t) {
      uint8_t* const buf = scratch + ((j * PM + t) & 1) * 2048;
      wave_lds_order();
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const uint32_t own = (uint32_t)float_to_half_bits(acc[j][t][4 * a + r]) | ((uint32_t)float_to_half_bits(acc[j][t][4 * a + r + 1]) << 16);
          const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0xB1, 0xF, 0xF, false);      // lane ^ 1
          // even lane: token r of features n, n + 1; odd lane: token r + 1 of features n - 1, n
          const uint32_t pair = __builtin_amdgcn_perm(other, own, odd ? 0x03020706u : 0x05040100u);
          const int turn = ((2 * a + h) & 3) << 4;            // bits 2 and 3 of the token
          *reinterpret_cast<uint32_t*>(buf + ((wr + (8 * a + r) * 64) ^ turn)) = pair;
        }
      wave_lds_order();
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int tok = 16 * i + row, m = mrow0 + 32 * t + tok, n = n0 + 32 * j + 8 * slot;
        const uint4 v = *reinterpret_cast<const uint4*>(buf + tok * 64 + ((slot ^ ((tok >> 2) & 3)) << 4));
        if (m < p.M && n < p.N) *reinterpret_cast<uint4*>(p.y + (size_t)m * p.N + n) = v;
      }
    }
}

// Add the K-slices of output block blk in the fixed order 0 .. S-1 whoever arrives last (its own
// slice is read back like the others, so the result does not depend on timing) and store fp16.
// The loads bypass the caches and each batch of them costs a trip to memory, so SB slices of
// two tiles go out at once (slices past S through an empty descriptor: zeros, no traffic).
// Against one slice at a time: 11008 -> 4096 at 128 draft tokens in four slices 19.3 -> 18.6 us,
// 13824 -> 5120 at 96 in four 27.7 -> 26.8; two slices take the narrow form (the empty loads of
// the wide one cost 1.2 us).
template <int PN, int PM, int kThreads, bool LANE_IS_TOKEN, int SB>
__device__ __forceinline__ void tile_sum_slices(const TileArgs& p, unsigned blk, int n0, int mrow0, uint8_t* scratch) {
  constexpr int kAcc = PN * PM * 16;
  constexpr int TB = PM % 2 == 0 ? 2 : 1;
#pragma unroll 1
  for (int q = 0; q < PN * PM; q += TB) {
    float sum[1][TB][16];
#pragma unroll
    for (int t = 0; t < TB; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[0][t][r] = 0.0f;
#pragma unroll 1
    for (int c0 = 0; c0 < p.S; c0 += SB) {
      float2 v[SB][TB][8];
#pragma unroll
      for (int c = 0; c < SB; ++c) {
        const float* f = slice_frag(p, min(c0 + c, p.S - 1), blk, kThreads * kAcc);
        const uint32_t bytes = c0 + c < p.S ? (uint32_t)(kThreads * kAcc * 4) : 0u;
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e)
            v[c][t][e] = buf_load_f32x2_shared(f, bytes, threadIdx.x * 8, (uint32_t)((q + t) * 64 * kThreads + e * 8 * kThreads));
      }
#pragma unroll
      for (int c = 0; c < SB; ++c)
#pragma unroll
        for (int t = 0; t < TB; ++t)
#pragma unroll
          for (int e = 0; e < 8; ++e) { sum[0][t][2 * e] += v[c][t][e].x; sum[0][t][2 * e + 1] += v[c][t][e].y; }
    }
    if constexpr (LANE_IS_TOKEN) tile_write_rows<1, TB>(p, sum, n0 + 32 * (q / PM), mrow0 + 32 * (q % PM), scratch);
    else tile_write_columns<1, TB>(p, sum, n0 + 32 * (q / PM), mrow0 + 32 * (q % PM), scratch);
  }
}

// Output of a wave's PN x PM tiles of 32 x 32.  S == 1: fp16 stores.  S > 1: see the
// head of this file.
template <int PN, int PM, int kThreads, bool LANE_IS_TOKEN = true, typename Acc>
__device__ __forceinline__ void tile_store32(const TileArgs& p, const TileCoord& tc, Acc (&acc)[PN][PM],
                                             int n0, int mrow0, uint8_t* scratch = nullptr) {
  const int tid = threadIdx.x;
  if (p.S == 1) {
    if constexpr (LANE_IS_TOKEN) tile_write_rows<PN, PM>(p, acc, n0, mrow0, scratch);
    else tile_write_columns<PN, PM>(p, acc, n0, mrow0, scratch);
    return;
  }
  const unsigned blk = (unsigned)(tc.nblk * p.mb + tc.mblk);
  constexpr int kAcc = PN * PM * 16;
  // (one running pointer: the steps between a thread's pairs lie beyond a store's immediate
  // offset, and an address of its own for each of them would take the registers of the tiles)
  float* mine = slice_frag(p, tc.slice, blk, kThreads * kAcc) + 2 * tid;
#pragma unroll
  for (int j = 0; j < PN; ++j)
#pragma unroll
    for (int t = 0; t < PM; ++t)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        store_shared_f2(mine, acc[j][t][2 * e], acc[j][t][2 * e + 1]);
        mine += 2 * kThreads;
        asm volatile("" : "+v"(mine));
      }
  __shared__ unsigned ticket32;
  if (!last_arrival(p.tickets, p.S, blk, &ticket32)) return;
  if (p.S == 2) tile_sum_slices<PN, PM, kThreads, LANE_IS_TOKEN, 2>(p, blk, n0, mrow0, scratch);
  else tile_sum_slices<PN, PM, kThreads, LANE_IS_TOKEN, 4>(p, blk, n0, mrow0, scratch);
}

}  // namespace qspec
