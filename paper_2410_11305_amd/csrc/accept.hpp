// The two steps that follow the verify pass (paper Sec. 3.1): the greedy
// acceptance policy and the KV-cache overwrite.
//
// Acceptance: the verify pass returns gamma + 1 rows of fp16 logits per sequence;
// a drafted token is accepted exactly when it equals the top-1 token of the
// verify distribution at its position, the first rejection discards the later
// drafts, and the token at that position (or, when every draft is accepted, one
// extra token) is the verify pass's own top-1.  Ties go to the lowest token id.
//
// Two launches, no atomics, no state: argmax_partial_kernel scans one chunk of
// one row per workgroup (every logit is read once, 16 bytes per lane) and leaves
// a 64-bit key per chunk in the workspace; accept_kernel (one workgroup per
// sequence, one wavefront per row) reduces the keys of its rows and finds the
// first rejected draft.  A key is (order-preserving image of the fp16 value) << 32
// | ~index, so that the unsigned maximum is the largest value and, among equals,
// the lowest index.
#pragma once
#include "buffer.hpp"
#include "common.hpp"

namespace qspec {

constexpr int kArgmaxThreads = 256;
constexpr int kArgmaxLoads = 2;             // 16-byte loads in flight per lane: 4096 logits per trip of a workgroup
constexpr int kArgmaxMaxChunks = 64;        // one lane of the second kernel per chunk

// fp16 bits -> 16-bit unsigned whose order is the order of the values
// (-0 and +0 compare equal, as they do as numbers; NaN is not handled).
__device__ inline uint32_t half_order_key(uint32_t bits) {
  bits &= 0xFFFFu;
  if (bits == 0x8000u) bits = 0u;
  return (bits & 0x8000u) ? (bits ^ 0xFFFFu) : (bits | 0x8000u);
}

// The same order as a signed 16-bit value, for both halves of a word at once (three
// operations for two logits): negative values count down from 0, -0 and +0 are 0.
typedef short v2s __attribute__((ext_vector_type(2)));
__device__ inline v2s half_order_pair(uint32_t w) {
  const v2s x = __builtin_bit_cast(v2s, w);
  const v2s neg = x >> (short)15;
  const uint32_t mag = (w & 0x7FFF7FFFu) ^ __builtin_bit_cast(uint32_t, neg);
  return __builtin_bit_cast(v2s, mag) - neg;
}
__device__ inline uint32_t half_order_of(int k) { return (uint32_t)(k + 0x8000); }   // the same order, unsigned (half_order_key's is one lower for negative values)

// Maximum over the 64 lanes (all active), wave-uniform.  DPP moves inside rows of 16 and
// across them: six vector operations where six ds_bpermute are six trips through LDS.
__device__ inline uint32_t wave_max_u32(uint32_t v) {
#define QSPEC_DPP_MAX(ctrl, rows) \
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, rows, 0xf, false))
  QSPEC_DPP_MAX(0x111, 0xf);      // row_shr 1, 2, 4, 8: lane 15 of a row holds the row's maximum
  QSPEC_DPP_MAX(0x112, 0xf);
  QSPEC_DPP_MAX(0x114, 0xf);
  QSPEC_DPP_MAX(0x118, 0xf);
  QSPEC_DPP_MAX(0x142, 0xa);      // row_bcast 15 into rows 1 and 3
  QSPEC_DPP_MAX(0x143, 0xc);      // row_bcast 31 into rows 2 and 3: lane 63 holds the maximum
#undef QSPEC_DPP_MAX
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
__device__ inline uint64_t wave_max_u64(uint64_t k) {
  const uint32_t hi = wave_max_u32((uint32_t)(k >> 32));
  const uint32_t lo = wave_max_u32((uint32_t)(k >> 32) == hi ? (uint32_t)k : 0u);
  return ((uint64_t)hi << 32) | lo;
}

struct ArgmaxArgs {
  const uint16_t* logits;   // fp16 [R][V]
  uint64_t* keys;           // [R][C]
  int V, C, chunk;          // chunk: elements per chunk (a multiple of 8 when VEC)
};

// grid (C, R).  VEC: V % 8 == 0, rows are 16-byte aligned, 8 logits per load.
// The scan costs two vector operations per logit (packed order, packed maximum); only the
// lanes that hold the wave's maximum then look for its lowest index.  (One comparison and
// two selects per logit, ten operations in all, took as long as the memory reads: 512 rows of
// 32000 logits, median of 31 traced launches 9.8 -> 8.4 us.)
template <bool VEC>
__global__ __launch_bounds__(kArgmaxThreads) void argmax_partial_kernel(ArgmaxArgs p) {
  constexpr int U = kArgmaxLoads;
  const int c = blockIdx.x, r = blockIdx.y;
  const int begin = c * p.chunk;
  const int end = min(p.V, begin + p.chunk);
  const uint16_t* row = p.logits + (size_t)r * p.V;
  uint64_t key = 0ull;                               // below every real key
  if (VEC) {
    for (int base = begin; base < end; base += U * kArgmaxThreads * 8) {
      // pieces past the end re-read the last one, under its own index
      uint4 q[U];
#pragma unroll
      for (int u = 0; u < U; ++u) q[u] = *reinterpret_cast<const uint4*>(row + min(base + (u * kArgmaxThreads + (int)threadIdx.x) * 8, end - 8));
      v2s k[U][4];
      v2s m2 = {(short)-0x8000, (short)-0x8000};
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t w[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          k[u][e] = half_order_pair(w[e]);
          m2 = __builtin_elementwise_max(m2, k[u][e]);
        }
      }
      const int m = max((int)m2.x, (int)m2.y);
      const uint32_t top = wave_max_u32(half_order_of(m));
      if (top <= (uint32_t)(key >> 32)) continue;    // (wave-uniform) equal values further on do not count
      uint32_t first = 0xFFFFFFFFu;
      if (half_order_of(m) == top) {
#pragma unroll
        for (int u = U - 1; u >= 0; --u) {
          const uint32_t i = (uint32_t)min(base + (u * kArgmaxThreads + (int)threadIdx.x) * 8, end - 8);
#pragma unroll
          for (int e = 3; e >= 0; --e) {
            if ((int)k[u][e].y == m) first = i + 2 * e + 1;
            if ((int)k[u][e].x == m) first = i + 2 * e;
          }
        }
      }
      key = ((uint64_t)top << 32) | wave_max_u32(~first);
    }
  } else {
    uint32_t best = 0u, best_i = 0xFFFFFFFFu;
    bool have = false;
    for (int i = begin + (int)threadIdx.x; i < end; i += kArgmaxThreads) {
      const uint32_t k = half_order_key(row[i]);
      // indices rise inside a thread: a strict comparison keeps the lowest index of equal values
      if (!have || k > best) { best = k; best_i = (uint32_t)i; have = true; }
    }
    key = wave_max_u64(have ? (((uint64_t)best << 32) | (uint64_t)(~best_i)) : 0ull);
  }
  __shared__ uint64_t part[kArgmaxThreads / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t k = part[0];
#pragma unroll
    for (int w = 1; w < kArgmaxThreads / 64; ++w) k = part[w] > k ? part[w] : k;
    p.keys[(size_t)r * p.C + c] = k;
  }
}

struct AcceptArgs {
  const uint64_t* keys;     // [B*(gamma+1)][C]
  const int32_t* draft;     // [B][gamma]
  int32_t* n_accept;        // [B]
  int32_t* out_tokens;      // [B][gamma+1]
  int gamma, C;
};

// One workgroup per sequence, one wavefront per row, kAcceptRows rows at a time (the loop of
// further rows is for longer drafts): the rows' keys arrive together.  (One wavefront walking the
// rows paid a trip to memory for each: the stores of the tokens keep the loads behind them.  Both
// launches over 1000 logits a row, where the walk is most of it, back to back in a graph: 128
// sequences of 4 rows 6.3 -> 4.9 us, of 17 rows 13.1 -> 6.9; with 32000 logits 12.1 -> 7.8 and the scan.)
constexpr int kAcceptRows = 16;
__global__ __launch_bounds__(64 * kAcceptRows) void accept_kernel(AcceptArgs p) {
  __shared__ int32_t tops[kAcceptRows];
  __shared__ int32_t same[kAcceptRows];
  const int b = blockIdx.x, lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), waves = blockDim.x >> 6;
  const int rows = p.gamma + 1;
  bool open = true;                       // no draft rejected so far
  for (int base = 0; base < rows; base += waves) {
    const int here = min(waves, rows - base);
    if (wave < here) {
      const int j = base + wave;
      const int32_t draft = p.draft[(size_t)b * p.gamma + min(j, p.gamma - 1)];
      const uint64_t k = wave_max_u64(lane < p.C ? p.keys[((size_t)b * rows + j) * p.C + lane] : 0ull);
      const int32_t top = (int32_t)(~(uint32_t)k);
      if (lane == 0) { tops[wave] = top; same[wave] = j < p.gamma && draft == top; }
    }
    __syncthreads();
    // the row where the drafts of this part end: the verify pass's own token (the correction, or the
    // extra one at row gamma) is the last that is emitted
    const uint64_t miss = __ballot(lane < here && same[lane < here ? lane : 0] == 0);
    const int stop = miss ? __builtin_ctzll(miss) : here;
    if (wave == 0) {
      if (lane < here) p.out_tokens[(size_t)b * rows + base + lane] = open && lane <= stop ? tops[lane] : -1;
      if (lane == 0 && open && miss) p.n_accept[b] = base + stop;
    }
    if (miss) open = false;
    __syncthreads();                      // tops and same are free for the next part
  }
}

struct KvArgs {
  const uint4* src;         // fp16 [B][gamma+1][D]
  uint4* cache;             // fp16 [B][S][D]
  const int32_t* n_accept;  // [B]
  const int32_t* pos;       // [B]
  int gamma, D8, S;         // D8 = D / 8 (16-byte pieces per row)
};

// grid B*(gamma+1): row j of sequence b goes to cache row pos[b] + j when j <= n_accept[b]
// (and the target lies inside the cache).
__global__ __launch_bounds__(256) void kv_overwrite_kernel(KvArgs p) {
  const int rows = p.gamma + 1;
  const int b = blockIdx.x / rows, j = blockIdx.x - b * rows;
  const int a = min(max(p.n_accept[b], 0), p.gamma);
  const long long s = (long long)p.pos[b] + j;
  if (j > a || s < 0 || s >= p.S) return;
  const uint4* src = p.src + ((size_t)b * rows + j) * p.D8;
  uint4* dst = p.cache + ((size_t)b * p.S + (size_t)s) * p.D8;
  for (int i = threadIdx.x; i < p.D8; i += 256) dst[i] = src[i];
}

}  // namespace qspec
