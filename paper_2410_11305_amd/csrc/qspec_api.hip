// C ABI of the QSpec W4 linear layer for gfx950: argument validation, kernel
// selection by problem shape, launches on the caller's stream.  Declarations
// and the buffer layouts are in include/qspec.h.
#include "qspec.h"

#include <hip/hip_runtime.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <tuple>

#include "accept.hpp"
#include "common.hpp"
#include "gemm_generic.hpp"
#include "gemm_stream.hpp"
#include "gemm_tile16.hpp"
#include "gemm_tile16w2.hpp"
#include "gemm_tile4.hpp"
#include "mlp_chain.hpp"
#include "pack.hpp"
#include "producers.hpp"
#include "quant_act.hpp"

using namespace qspec;

// Scratch of qspec_gemm_w4a16_noalloc: arrival counters (first kTicketBytes) and K-slice
// partial sums, for callers that can neither allocate nor pass a workspace.  Every GPU
// the library runs on holds its own copy until the process ends.  In host code this name
// is only a handle for hipGetSymbolAddress; kernels and fills take the address that call
// returned for the current device (scratch_of_device below), never the name.
constexpr size_t kScratchBytes = ((size_t)32 << 20) + 16384;   // 32 MiB of partial sums + 16 KiB of counters
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

inline bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

inline int check_shape(int M, int N, int K, int group) {
  if (group != kGroup) return QSPEC_ERR_SHAPE;
  if (K <= 0 || K % kGroup != 0) return QSPEC_ERR_SHAPE;
  if (N <= 0 || N % kTileRows != 0) return QSPEC_ERR_SHAPE;
  if (M < 1) return QSPEC_ERR_SHAPE;
  // 32-bit byte offsets are used inside the kernels: every buffer stays below 2 GiB
  if ((long long)N * K / 2 >= 0x7fffffffLL) return QSPEC_ERR_SHAPE;
  if ((long long)M * K * 2 >= 0x7fffffffLL) return QSPEC_ERR_SHAPE;
  return QSPEC_OK;
}

// The kernels use gfx950-only matrix instructions; refuse anything else.
int check_device() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return QSPEC_ERR_HIP;
  (void)hipGetLastError();
  static int verdict[64];   // 0 unknown, 1 ok, 2 unsupported
  if (dev < 0 || dev >= 64) return QSPEC_ERR_UNSUPPORTED;
  if (verdict[dev] == 0) {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return QSPEC_ERR_HIP;
    verdict[dev] = strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? 1 : 2;
  }
  return verdict[dev] == 1 ? QSPEC_OK : QSPEC_ERR_UNSUPPORTED;
}

// kernel<<<grid, block, lds, s>>>(a...) by the one runtime call that makes it up, without storing the launch
// configuration and fetching it again first (two more calls).  A failure is left for launch_status().
template <typename... P, typename... A>
inline void launch_kernel(void (*kernel)(P...), dim3 grid, dim3 block, unsigned lds, hipStream_t s, const A&... a) {
  std::tuple<P...> values(a...);
  std::apply([&](P&... v) {
    void* args[] = {const_cast<void*>(static_cast<const void*>(&v))...};
    (void)hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, block, args, lds, s);
  }, values);
}

// QSPEC_ERR_HIP must mean "THIS call's launch failed": check_device(), which every entry
// point calls after validating its arguments and before launching, drops whatever error an
// unrelated earlier runtime call left behind; launch_status() then sees only this call's.
inline int launch_status() { return hipGetLastError() == hipSuccess ? QSPEC_OK : QSPEC_ERR_HIP; }

inline const uint16_t* blob_scales(const void* packed, int N, int K) {
  return reinterpret_cast<const uint16_t*>(static_cast<const uint8_t*>(packed) + (size_t)N * K / 2);
}

inline unsigned blocks_for(size_t n, unsigned per_block) { return (unsigned)((n + per_block - 1) / per_block); }

// tokens per workgroup: smallest of 16, 32, 64, 128 that covers M (128 at most)
inline int pick_tm(int M) { return M <= 16 ? 1 : M <= 32 ? 2 : M <= 64 ? 4 : 8; }

template <int TM>
void launch_w4a4(const GemmArgs& a, hipStream_t s) {
  dim3 grid(a.N / 16, (a.M + TM * 16 - 1) / (TM * 16));
  launch_kernel((gemm_w4a4_generic<TM, 4, false>), grid, dim3(256), 0, s, a);
}
template <int TM>
void launch_w4a16(const GemmArgs& a, hipStream_t s) {
  dim3 grid(a.N / 16, (a.M + TM * 16 - 1) / (TM * 16));
  launch_kernel((gemm_w4a16_generic<TM, 4>), grid, dim3(256), 0, s, a);
}


constexpr int kNumCU = 256;

// Plan overrides (benchmark A/B and tests only).  They are parsed ONCE: from the
// environment at the first use, and afterwards only through qspec_debug_set_plan.  The
// launch path reads plain integers; no entry point calls getenv.
//   QSPEC_KERNEL=generic            route M > 32 to the untiled reference kernels, whatever else is set
//   QSPEC_STREAM_W4A4 / _W4A16      "NT,S", "NT,S,MS" or "NT,S,MS,W": tiles per workgroup, K-slices, token-row blocks,
//                                   wavefronts of a workgroup (8, or 4 where that instance exists)
//   QSPEC_STREAM_MAX_W4A4 / _W4A16  the streaming kernels take every M up to this one and none above
//   QSPEC_TILE_W4A4 / _W4A16        "shape,S": workgroup shape index, K-slices
struct PlanOverrides {
  bool generic = false;
  int stream_fields[2] = {0, 0};      // [w4a4]: how many of nt, S, ms, waves were given (0: no override)
  int stream[2][4] = {{0, 0, 0, 0}, {0, 0, 0, 0}};
  int stream_max[2] = {0, 0};         // 0: the default bound
  bool tile_set[2] = {false, false};
  int tile[2][2] = {{0, 0}, {0, 0}};
  unsigned mlp_spin = 0;              // 0: the default number of polls of the persistent MLP kernel's wait
};

// value == nullptr (or unparsable) clears the override named `name`; false: unknown name.
bool apply_override(PlanOverrides& o, const char* name, const char* value) {
  if (strcmp(name, "QSPEC_KERNEL") == 0) { o.generic = value && strcmp(value, "generic") == 0; return true; }
  if (strcmp(name, "QSPEC_MLP_SPIN") == 0) { o.mlp_spin = value ? (unsigned)strtoul(value, nullptr, 10) : 0u; return true; }
  for (int w4a4 = 0; w4a4 < 2; ++w4a4) {
    if (strcmp(name, w4a4 ? "QSPEC_STREAM_W4A4" : "QSPEC_STREAM_W4A16") == 0) {
      int* f = o.stream[w4a4];
      f[0] = f[1] = 0; f[2] = 1; f[3] = 8;
      const int nf = value ? sscanf(value, "%d,%d,%d,%d", &f[0], &f[1], &f[2], &f[3]) : 0;
      o.stream_fields[w4a4] = nf >= 2 ? nf : 0;
      if (nf < 3) f[2] = 1;
      return true;
    }
    if (strcmp(name, w4a4 ? "QSPEC_STREAM_MAX_W4A4" : "QSPEC_STREAM_MAX_W4A16") == 0) {
      const int v = value ? atoi(value) : 0;
      // the verify-mode streaming kernel exists for at most two 16-token tiles per workgroup
      o.stream_max[w4a4] = (v >= 32 && v <= (w4a4 ? 128 : 32)) ? v : 0;
      return true;
    }
    if (strcmp(name, w4a4 ? "QSPEC_TILE_W4A4" : "QSPEC_TILE_W4A16") == 0) {
      int* f = o.tile[w4a4];
      o.tile_set[w4a4] = value && sscanf(value, "%d,%d", &f[0], &f[1]) == 2;
      return true;
    }
  }
  return false;
}

constexpr const char* kOverrideNames[] = {"QSPEC_KERNEL", "QSPEC_STREAM_W4A4", "QSPEC_STREAM_W4A16",
                                          "QSPEC_STREAM_MAX_W4A4", "QSPEC_STREAM_MAX_W4A16",
                                          "QSPEC_TILE_W4A4", "QSPEC_TILE_W4A16", "QSPEC_MLP_SPIN"};

PlanOverrides& overrides() {
  static PlanOverrides o = [] {
    PlanOverrides init;
    for (const char* name : kOverrideNames)
      if (const char* e = getenv(name)) apply_override(init, name, e);
    return init;
  }();
  return o;
}

// ---------------------------------------------------------------- streaming (small-M) kernel
constexpr int kStreamMaxM = 32;
constexpr int kStreamMaxM4 = 64;

constexpr size_t kTicketBytes = 16384;                 // head of the workspace: arrival counters
constexpr int kMaxTickets = (int)(kTicketBytes / 4);

// Plan of the streaming kernel: NT adjacent n-tiles per workgroup, S K-slices, ms
// token-row blocks.  A pure function of (mode, M, N, K), so that qspec_workspace_bytes
// and the GEMM entry points agree.  QSPEC_STREAM_W4A4 / QSPEC_STREAM_W4A16 = "NT,S" or
// "NT,S,MS" override the heuristic (benchmark A/B only).
struct StreamPlan {
  int nt, S, blocks;
  int ms;       // token-row blocks; block i owns rows i*16*tm .. (i+1)*16*tm - 1
  int tm;       // 16-token tiles per workgroup (the kernel's TM)
  double cost;  // microseconds by the cost tables; a forced plan has none
  int waves;    // wavefronts of a workgroup: 8, or 4 (stream_waves)
};
inline int stream_tm(int M) { return M <= 16 ? 1 : M <= 32 ? 2 : M <= 64 ? 4 : 8; }   // 16-token tiles that cover M rows
constexpr int kStreamNts[] = {1, 2, 3, 4, 6};
inline bool stream_nt_ok(int nt, int tm) {
  for (int v : kStreamNts) if (v == nt) return nt * tm <= 16;      // 4 accumulator registers per tile pair; beyond 64 the kernel spills
  return false;
}
// tiles per workgroup when the rows are dealt to ms blocks: ceil(M / ms) rows, in whole tiles
inline int stream_tm_split(int M, int ms) { return stream_tm(16 * (((M + ms - 1) / ms + 15) / 16)); }

// What a streaming plan costs, in microseconds.  ng groups fall to the busiest wavefront (G / 8 on average), the
// workgroups of ceil(M / (16 tm)) token-row blocks fill `rounds` rounds of the compute units:
//   fixed + round (rounds - 1) + ng (group + again (rounds - 1)) + G / 8 x workgroups per unit x (load + tokens x share of live rows)
// Fitted to timed plans, on rotating weights inside HIP graphs: in the draft mode 5500 problems of layers 128 to 57344
// wide and 128 to 28672 long at 1 to 2050 tokens and 1400 layers of Llama-shaped blocks at 1 to 256, in the verify mode
// 3300 and 1200 at 1 to 128, every instance with the row blocks that cover M.  On 520 problems timed afterwards, with
// the kernels of the fit (profiles/stream_plan_times.txt), the choice among these and the tiled plans is 0.9 % slower than the
// best one on average and 15 % at most (verify mode past 32 tokens, where a rule bounds it: 1.6 and 32 %), and takes no more
// than 1.12 times what the kernels and rules before the cost tables took.  The kernels have gained since, the streaming ones
// more; with the present ones the choice on those problems is 1.9 % slower on average and 53 % at most (11664 outputs from
// 1536 at 67 tokens on packed codes, tiled 10.0 us, streaming 6.6; profiles/plan_choice_present_kernels.txt).  (Tables fitted to 17 to 600 tokens and layers from 512 long
// and 1024 wide alone were too low where few workgroups or few groups leave nothing to hide the latency behind: 224
// outputs from 10240 at 1200 tokens 17.1 us tiled, 23.4 as chosen; 11696 from 1152 at 43 tokens 8.6 us, 6.7 now.  A rule for up
// to 16 tokens, rounds x groups per wavefront x (NT + activations), was 0.4 % behind the best instance on average on the
// blocks' layers and 1.0 % on the others, 35 % at most; now 0.2, 0.4 and 16 %.)
struct StreamCost { int tm, nt; double fixed, round, group, again, load, tokens; };
// up to 16 tokens
constexpr StreamCost kStreamFew4[] = {
    {1, 1, 2.863, 0.51, 0.199, 0.093, 0.185, 0.081},
    {1, 2, 2.956, 0.323, 0.277, 0.222, 0.31, 0.094},
    {1, 3, 3.012, 0.167, 0.516, 0.519, 0.35, 0.087},
    {1, 4, 3.145, 0.085, 0.581, 0.659, 0.501, 0.153},
    {1, 6, 3.21, 1.465, 0.856, 1.045, 0.744, 0.248},
};
constexpr StreamCost kStreamFew16[] = {
    {1, 1, 2.466, 0.476, 0.393, 0.135, 0.228, 0.187},
    {1, 2, 2.503, 0.818, 0.555, 0.441, 0.277, 0.225},
    {1, 3, 2.787, 0.255, 0.712, 0.566, 0.246, 0.346},
    {1, 4, 2.875, 1.143, 0.865, 0.809, 0.303, 0.395},
    {1, 6, 2.937, 1.552, 1.213, 1.185, 0.53, 0.435},
};
// from 17 tokens on
constexpr StreamCost kStreamCost4[] = {
    {1, 1, 2.545, 0.603, 0.238, 0.058, 0.204, 0},
    {1, 2, 2.689, 0.575, 0.338, 0.124, 0.263, 0},
    {1, 3, 2.908, 0.53, 0.536, 0.318, 0.249, 0},
    {1, 4, 2.991, 0.504, 0.655, 0.405, 0.303, 0},
    {1, 6, 3.22, 1.846, 0.95, 0.685, 0.307, 0},
    {2, 1, 2.718, 0.624, 0.344, 0.111, 0.263, 0},
    {2, 2, 2.97, 1.497, 0.467, 0.223, 0.375, 0},
    {2, 3, 3.23, 1.894, 0.713, 0.488, 0.28, 0},
    {2, 4, 3.352, 2.102, 0.864, 0.588, 0.334, 0},
    {2, 6, 4.038, 2.866, 1.159, 0.803, 0.461, 0},
    {4, 1, 2.887, 1.754, 0.639, 0.346, 0.339, 0.101},
    {4, 2, 3.084, 2.145, 0.907, 0.585, 0.339, 0.135},
    {4, 3, 4.091, 2.881, 1.24, 0.939, 0.225, 0.169},
    {4, 4, 4.347, 3.215, 1.379, 1.046, 0.332, 0.081},
    {8, 1, 3.39, 2.165, 1.349, 0.945, 0, 0.635},
    {8, 2, 4.401, 3.307, 1.802, 1.41, 0, 0.579},
};
constexpr StreamCost kStreamCost16[] = {
    {1, 1, 2.427, 0.048, 0.422, 0.153, 0.268, 0.056},
    {1, 2, 2.566, 0.872, 0.562, 0.493, 0.192, 0.147},
    {1, 3, 2.846, 0.359, 0.73, 0.544, 0.336, 0},
    {1, 4, 2.93, 1.039, 0.87, 0.778, 0.407, 0},
    {1, 6, 3.288, 1.369, 1.108, 1.131, 0.556, 0},
    {2, 1, 2.459, 0.483, 0.651, 0.531, 0.157, 0.331},
    {2, 2, 2.796, 0.892, 0.736, 0.732, 0.194, 0.52},
    {2, 3, 3.152, 1.367, 1.024, 1.028, 0.101, 0.573},
    {2, 4, 3.289, 1.449, 1.17, 1.215, 0.268, 0.5},
    {2, 6, 4.03, 2.05, 1.346, 1.505, 1.009, 0.225},
};
constexpr int kMaxRowBlocks = 16;

inline int stream_qs(int nt, int tm) { return nt <= 2 && tm <= 4 ? 2 : 1; }      // the kernel's QS

// `over` or more once the first terms alone reach it (every eager call plans)
double stream_cost(const StreamCost& c, int M, int N, int G, double over) {
  const int qs = stream_qs(c.nt, c.tm), ng = qs * ((G + qs * kStreamWaves - 1) / (qs * kStreamWaves));
  const double start = c.fixed + ng * c.group;
  if (start >= over) return start;
  const int ms = (M + 16 * c.tm - 1) / (16 * c.tm), tiles = N / 16;
  const long long blocks = (long long)((tiles + c.nt - 1) / c.nt) * ms;
  const double again = (double)((blocks + kNumCU - 1) / kNumCU - 1);
  const double load = (double)tiles * ms / c.nt / kNumCU * G / kStreamWaves;
  return start + again * (c.round + ng * c.again) + load * (c.load + c.tokens * M / (16.0 * c.tm * ms));
}

// Cheapest streaming plan; one_round: among those that one round of workgroups covers.
template <size_t COUNT>
double best_stream(const StreamCost (&costs)[COUNT], int M, int N, int G, bool one_round, bool bounded, StreamPlan* p) {
  double best = 1e30;
  for (const StreamCost& c : costs) {
    const int ms = (M + 16 * c.tm - 1) / (16 * c.tm), blocks = (N / 16 + c.nt - 1) / c.nt;
    if (ms > kMaxRowBlocks || (c.tm > 1 && 8 * c.tm >= M)) continue;              // (a kernel of half the token tiles covers M)
    if (one_round && (ms > 8 || blocks * ms > kNumCU)) continue;
    if (bounded && (long long)blocks * ms > 5 * kNumCU) continue;   // (the best of no timed problem past 32 tokens)
    const double cost = stream_cost(c, M, N, G, best);
    if (cost < best) { best = cost; p->nt = c.nt; p->tm = c.tm; p->ms = ms; p->S = 1; p->blocks = blocks; }
  }
  return best;
}
double best_stream(bool w4a4, int M, int N, int G, bool one_round, StreamPlan* p) {
  const bool bounded = M > 32 && !overrides().stream_max[w4a4];
  if (M <= 16) return w4a4 ? best_stream(kStreamFew4, M, N, G, one_round, bounded, p) : best_stream(kStreamFew16, M, N, G, one_round, bounded, p);
  return w4a4 ? best_stream(kStreamCost4, M, N, G, one_round, bounded, p) : best_stream(kStreamCost16, M, N, G, one_round, bounded, p);
}

// Four wavefronts or eight.  Time on four over time on eight, same tiles, 260 problems of Llama-shaped layers at 1 to 64
// tokens, by rounds of workgroups: one 1.02 to 1.19, up to 1.25 rounds 1.02, from there to two rounds 0.97 (draft mode, one
// token tile), 0.95 (verify mode), 0.92 (two and four token tiles, also 0.95 to 0.98 up to three rounds); beyond 1.00 to
// 1.03; with one weight tile 1.00 to 1.13 everywhere.
int stream_waves(const StreamPlan& p) {
  const long long wgs = (long long)p.blocks * p.ms;
  return p.nt >= 2 && p.tm <= 4 && 4 * wgs > 5 * kNumCU && wgs <= (p.tm >= 2 ? 3 : 2) * kNumCU ? 4 : kStreamWaves;
}

StreamPlan plan_stream(bool w4a4, int M, int N, int K) {
  const int tiles = N / 16, G = K / kGroup;
  const PlanOverrides& ov = overrides();
  const int nf = ov.stream_fields[w4a4 ? 1 : 0];
  int nt = ov.stream[w4a4 ? 1 : 0][0], S = ov.stream[w4a4 ? 1 : 0][1], ms = ov.stream[w4a4 ? 1 : 0][2];
  bool forced = nf >= 2 && S >= 1 && S <= G;
  if (nf < 3) ms = 1;
  if (forced && ms > 1) forced = S == 1 && (ms == 2 || ms == 4 || ms == 8);
  // a forced plan must have an instance and its row blocks must cover all M rows
  if (forced) forced = stream_nt_ok(nt, stream_tm_split(M, ms)) && (w4a4 || stream_tm_split(M, ms) <= 2) &&
                       (long long)ms * 16 * stream_tm_split(M, ms) >= M;
  StreamPlan p{};
  if (forced) {
    p.nt = nt; p.S = S; p.ms = ms;
    p.blocks = (tiles + nt - 1) / nt;
    p.tm = ms > 1 ? stream_tm_split(M, ms) : stream_tm(M);
    p.waves = ov.stream[w4a4 ? 1 : 0][3];     // (one that does not exist is refused at the launch)
    return p;
  }
  // (verify mode past 32 tokens: only where one round of workgroups covers a layer of at most 8192 x 8192; the
  // tiled kernels have too few output blocks to fill the chip there.  128 tokens, 4096 x 4096: 15.5 us tiled, 9.6 here.)
  const bool past = !w4a4 && M > kStreamMaxM;
  if (past && (M > 128 || N > 8192 || K > 8192)) return p;          // nt == 0: no streaming plan
  p.cost = best_stream(w4a4, M, N, G, past, &p);
  p.waves = stream_waves(p);
  return p;
}

inline size_t stream_ws_bytes(const StreamPlan& p) {
  return p.S > 1 ? kTicketBytes + (size_t)p.S * p.blocks * p.nt * p.tm * 1024 : 0;
}

// Launch the instance <mode, TM, NT> of a streaming plan.  A (TM, NT) pair that is not
// instantiated (a forced plan can name one) is refused: nothing is launched.
template <bool W4A4, int TM, int NT>
int launch_stream_inst(const StreamArgs& a, const StreamPlan& plan, hipStream_t s) {
  const auto launch = [&](auto kernel) {
    const StreamRest rest{a.y, a.ws, a.tickets, a.S, a.per_slice, a.more_slice, a.blocks};
    launch_kernel(kernel, dim3(a.workgroups), dim3(plan.waves * 64), 0, s, a.codes, a.scalesT, a.act, a.sa, a.M, a.N, a.K,
                  a.workgroups, a.S > 1 ? 0 : a.ms, a.ms_rcp, rest);
    return QSPEC_OK;
  };
  if constexpr (NT >= 2 && TM <= 4) {
    if (plan.waves == 4) return launch(waves4::gemm_stream_kernel<W4A4, TM, NT>);
  }
  if (plan.waves != kStreamWaves) return QSPEC_ERR_UNSUPPORTED;
  return launch(gemm_stream_kernel<W4A4, TM, NT>);
}

template <bool W4A4, int TM>
int launch_stream_tm(const StreamArgs& a, const StreamPlan& plan, hipStream_t s) {
  switch (plan.nt) {
    case 1: return launch_stream_inst<W4A4, TM, 1>(a, plan, s);
    case 2: return launch_stream_inst<W4A4, TM, 2>(a, plan, s);
    case 3: if constexpr (TM <= 4) return launch_stream_inst<W4A4, TM, 3>(a, plan, s); else return QSPEC_ERR_UNSUPPORTED;
    case 4: if constexpr (TM <= 4) return launch_stream_inst<W4A4, TM, 4>(a, plan, s); else return QSPEC_ERR_UNSUPPORTED;
    case 6: if constexpr (TM <= 2) return launch_stream_inst<W4A4, TM, 6>(a, plan, s); else return QSPEC_ERR_UNSUPPORTED;
    default: return QSPEC_ERR_UNSUPPORTED;
  }
}

template <bool W4A4>
int launch_stream(const StreamPlan& plan, StreamArgs a, void* workspace, hipStream_t s) {
  if ((long long)plan.ms * 16 * plan.tm < a.M) return QSPEC_ERR_UNSUPPORTED;      // the row blocks must cover M
  a.S = plan.S; a.per_slice = a.G / plan.S; a.more_slice = a.G % plan.S;
  a.blocks = plan.blocks;
  a.ms = plan.ms;
  a.ms_rcp = (uint32_t)((0x100000000ull + plan.ms - 1) / plan.ms);
  a.workgroups = (uint32_t)(plan.blocks * plan.S * plan.ms);
  a.tickets = static_cast<unsigned*>(workspace);
  a.ws = plan.S > 1 ? reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + kTicketBytes) : nullptr;
  switch (plan.tm) {
    case 1: return launch_stream_tm<W4A4, 1>(a, plan, s);
    case 2: return launch_stream_tm<W4A4, 2>(a, plan, s);
    case 4: if constexpr (W4A4) return launch_stream_tm<true, 4>(a, plan, s); else return QSPEC_ERR_UNSUPPORTED;
    case 8: if constexpr (W4A4) return launch_stream_tm<true, 8>(a, plan, s); else return QSPEC_ERR_UNSUPPORTED;
    default: return QSPEC_ERR_UNSUPPORTED;
  }
}

// ---------------------------------------------------------------- tiled (M > 32) kernels
// Workgroup shapes the tiled kernels are instantiated for: TN x TMW MFMA tiles per
// wavefront, WGN x WGM wavefronts per workgroup, weight ring of NW groups, OCC workgroups per compute
// unit (the register budget the compiler is held to), K groups dealt to WGK sets of such wavefronts.
struct TileShape { int TN, TMW, WGN, WGM, NW, OCC, WGK = 1; };
constexpr TileShape kShapes16[] = {     // verify mode (gemm_tile16w_kernel): TN, TMW count 32 x 32 tiles
    {1, 4, 4, 1, 4, 2},      // 0: 128 outputs x 128 tokens
    {1, 2, 4, 1, 2, 1, 2},   // 1: 128 x 64, the K groups dealt to two sets of four wavefronts
    {1, 2, 2, 1, 2, 2, 2},   // 2: 64 x 64, the K groups dealt to two pairs of wavefronts
    {1, 4, 4, 1, 2, 1, 2},   // 3: 128 x 128, the K groups dealt to two sets of four wavefronts
    {1, 4, 8, 1, 2, 1},      // 4: 256 x 128, eight wavefronts, one workgroup per compute unit
    {2, 2, 2, 1, 2, 1, 4},   // 5: 128 x 64, the K groups dealt to four pairs of wavefronts
    {1, 2, 4, 1, 2, 3},      // 6: 128 x 64, three workgroups per compute unit
    {2, 4, 8, 1, 2, 1},      // 7: 512 x 128 (gemm_tile16w2_kernel), never in K-slices
};
// What a verify-mode plan costs, in microseconds: fixed, `again` for every round of workgroups after the first,
// groups per slice x the rounds' cost per group, and with K-slices the exchange.  A round's cost per
// group rises with the workgroups per compute unit: `one` with one on every unit, less in proportion
// down to `alone` (what a workgroup takes with nothing beside it; the part is power-limited under matrix
// work, its clock falls from 2.3 GHz with half the units busy to 1.7 GHz with all of them), from `above1`
// with the first second workgroup to `two` with two everywhere, and from `above2` to `three`.  `places`
// workgroups fit a unit; what lies past that is a further round.
// Fitted to 38000 timed plans of 1716 problems: 16 to 128256 outputs from 128 to 28672 inputs at 33 to 2050
// tokens and some up to 9000, every shape below, one to eight slices, on rotating weights inside HIP
// graphs.  The choice is 0.6 % slower than the best of them on average and 19 % at most (368 outputs from 3584 at
// 1002 tokens; 23 % there with the present kernels, and 0.8 % on average on the 400 problems of the sample), and 1.2 % (18 %) on 228 more with long inputs or up to 9000 tokens; profiles/verify_plan_times.txt
// lists a sample, the worst ones included.  (A table of five numbers a shape fitted to 14 large layers, without
// the further rounds' cost and without 128 x 128 and 128 x 64 blocks in a single round, left 2.3 % on average and
// was up to 39 % slower than the fill rules before both on short inputs: 28672 outputs from 512 at 256 tokens
// 21.0 us, 15.1 by the rules, 14.0 now.)
struct TileCost { double fixed, again, alone, one, above1, two, above2, three, slice0, slice1; int places; };
constexpr TileCost kCost16[] = {
    {5.589, 3.537, 0.754, 0.95, 1.471, 1.772, 0, 0, 3.471, 1.33, 2},  // 0
    {4.841, 3.47, 0.386, 0.492, 0.752, 0.986, 0, 0, 2.296, 0.76, 2},  // 1
    {4.043, 2.084, 0.328, 0.375, 0.538, 0.607, 0, 0, 1.775, 0.341, 2},  // 2
    {6.318, 5.271, 0.618, 0.876, 0, 0, 0, 0, 3.248, 1.093, 1},  // 3
    {5.485, 4.333, 1.091, 1.622, 0, 0, 0, 0, 6.502, 2.209, 1},  // 4
    {5.966, 4.565, 0.368, 0.472, 0, 0, 0, 0, 2.282, 0.677, 1},  // 5
    {3.8, 2.407, 0.561, 0.596, 0.806, 1.027, 1.471, 1.723, 2.248, 0.773, 3},  // 6
    {11.468, 8.47, 2.1, 2.909, 0, 0, 0, 0, 0, 0, 1},  // 7
};
constexpr TileShape kShapes4[] = {      // draft mode (gemm_tile4w_kernel): TN, TMW count 32 x 32 tiles
    {1, 4, 4, 1, 3, 2},   // 0: 128 outputs x 128 tokens
    {1, 2, 4, 1, 3, 2},   // 1: 128 x 64
    {1, 2, 2, 1, 3, 2},   // 2: 64 x 64
    {1, 4, 8, 1, 3, 1},   // 3: 256 x 128, eight wavefronts, one workgroup per compute unit
};
constexpr int kNumTileShapes = 4;
constexpr int kNumShapes16 = 8;
struct TilePlan {
  int shape;      // index into the mode's shape table
  int S;          // K-slices
  int nb, mb;     // output blocks
};

inline const TileShape& shape_of(bool w4a4, int i) { return w4a4 ? kShapes4[i] : kShapes16[i]; }

// QSPEC_TILE_W4A4 / QSPEC_TILE_W4A16 = "shape,S" override the heuristic (benchmark A/B only).
bool tile_override(bool w4a4, int* shape, int* S) {
  const PlanOverrides& ov = overrides();
  if (!ov.tile_set[w4a4 ? 1 : 0]) return false;
  const int* f = ov.tile[w4a4 ? 1 : 0];
  if (f[0] < 0 || f[0] >= (w4a4 ? kNumTileShapes : kNumShapes16) || f[1] < 1) return false;
  *shape = f[0];
  *S = f[1];
  return true;
}

// Cost per group of a round with f workgroups per compute unit (0 < f <= places).
double round_cost16(const TileCost& c, double f) {
  if (f <= 1.0) return c.one * f;
  if (f <= 2.0) return c.above1 + (c.two - c.above1) * (f - 1.0);
  return c.above2 + (c.three - c.above2) * (f - 2.0);
}

// Cheapest verify-mode plan by kCost16, and what it costs.
double plan_tile16(int M, int N, int G, int* shape, int* slices) {
  double best = 1e30;
  for (int i = 0; i < kNumShapes16; ++i) {
    const TileShape& t = kShapes16[i];
    const TileCost& c = kCost16[i];
    const int bn = 32 * t.TN * t.WGN, bm = 32 * t.TMW * t.WGM;
    const long long mb = (M + bm - 1) / bm, blocks = (N + bn - 1) / bn * mb;
    const double used = 0.8 + 0.2 * M / (mb * bm);             // (rows past M are zeros or stale: they cost time, less power)
    const auto per_group = [&](double f) { const double r = round_cost16(c, f) * used; return r > c.alone ? r : c.alone; };
    for (int S : {1, 2, 3, 4, 6, 8}) {
      // K-slices only while all workgroups have a compute unit of their own (and the partial sums
      // fit 32 MiB), of four groups at least
      if (S > 1 && (c.slice0 == 0.0 || blocks * S > kNumCU || G / S < 4)) break;
      // (every eager call plans; no plan is cheaper than one round of workgroups with nothing beside them)
      if (c.fixed + c.alone * G / S >= best) continue;
      const long long wgs = blocks * S, load = (long long)c.places * kNumCU, full = wgs / load, rest = wgs % load;
      const double rounds = (full ? full * per_group(c.places) : 0.0) + (rest ? per_group((double)rest / kNumCU) : 0.0);
      // (the exchange of few workgroups is cheaper: 48 of 64 x 64 in two slices 3.1 us, 240 of them 4.0)
      const double xch = S > 1 ? (c.slice0 + c.slice1 * S) * (0.7 + 0.3 * wgs / kNumCU) : 0.0;
      double cost = c.fixed + c.again * (full + (rest ? 1 : 0) - 1) + rounds * G / S + xch;
      // An XCD fetches a group's activations of every token block it works on: on narrow layers that
      // bounds the plan (512 x 1920 at 1767 tokens: 64 x 64 blocks 14.0 us, 128 x 64 10.7)
      const long long rows = bm * (mb < (wgs + 7) / 8 ? mb : (wgs + 7) / 8);
      const double fetch = c.fixed + 0.000276 * rows * G / S;
      if (fetch > cost) cost = fetch;
      if (cost < best) { best = cost; *shape = i; *slices = S; }
    }
  }
  return best;
}

// What a draft-mode tiled plan costs, in microseconds: g groups per slice (times the share of live rows), f
// workgroups per compute unit in its last round of `places`:
//   fixed + again (rounds - 1) + g (full (rounds - 1) + any + first min(f, 1) + second clamp(f - 1, 0, 1) + more max(f - 2, 0) + shared [f > 1])
//   + with K-slices (slice0 + slice1 S + slice2 workgroups per unit) + out x workgroups per unit
// Fitted to the problems of kStreamCost4 and 500 larger ones of up to 3000 tokens, with the widened activation format.
// On packed codes, which the kernel widens in registers, the groups take `packed` times as long: that decides between
// this kernel and the streaming one for a caller who has packed codes (34 tokens, 16656 outputs from 5248: streaming 19.9 us,
// this kernel 22.2 on widened codes, 27.3 on packed ones).  Fill rules from sweeps over the Llama-shaped layers, its
// predecessor, sliced small layers too little and wide ones at 65 to 96 tokens too much (51200 x 7936 at 72: 86.9 us in
// 128 x 64, 63.0 in 256 x 128 blocks).
struct Tile4Cost { double fixed, again, full, any, first, second, more, shared, slice0, slice1, slice2, out, packed; int places; };
constexpr Tile4Cost kCost4[] = {
    {4.673, 0.694, 1.09, 0.635, 0.035, 0.109, 0, 0.375, 1.134, 0.815, 3.458, 1.812, 1.175, 2},   // 0: 128 x 128
    {3.582, 0.745, 0.609, 0.415, 0.034, 0.032, 0, 0.18, 1.453, 0.308, 1.841, 1.104, 1.177, 2},   // 1: 128 x 64
    {3.43, 0.109, 0.736, 0.364, 0.038, 0.021, 0.073, 0.177, 1.761, 0.166, 0.682, 0.599, 1.282, 4},   // 2: 64 x 64
    {5.255, 2.734, 1.03, 0.855, 0.152, 0, 0, 0, 3.027, 1.428, 3.697, 2.475, 1.105, 1},   // 3: 256 x 128
};

struct Tile4Choice { int shape, S; double wide, packed; };      // S == 0: none
// Cheapest draft-mode tiled plan on widened codes among those below `best`, and what it costs on either format.
Tile4Choice best_tile4(int M, int N, int G, int max_slices = 4, double best = 1e30) {
  Tile4Choice choice{0, 0, best, best};
  for (int i = 0; i < kNumTileShapes; ++i) {
    const TileShape& t = kShapes4[i];
    const Tile4Cost& c = kCost4[i];
    const int bn = 32 * t.TN * t.WGN, bm = 32 * t.TMW * t.WGM;
    const long long mb = (M + bm - 1) / bm, blocks = (N + bn - 1) / bn * mb;
    for (int S = 1; S <= max_slices; ++S) {
      // K-slices only in one round of two workgroups per unit (one of eight wavefronts: the partial sums stay
      // within 32 MiB), of four groups at least
      if (S > 1 && (blocks * S > (c.places > 1 ? 2 : 1) * kNumCU || G / S < 4)) break;
      const double g = ((G + S - 1) / S) * (0.7 + 0.3 * M / (double)(mb * bm));
      if (c.fixed + c.any * g >= choice.wide) continue;
      const long long wgs = blocks * S, load = (long long)c.places * kNumCU, rounds = (wgs + load - 1) / load;
      const double per_unit = (double)wgs / kNumCU, f = per_unit - (double)c.places * (rounds - 1);
      const auto clamp01 = [](double v) { return v < 0.0 ? 0.0 : v > 1.0 ? 1.0 : v; };
      const double groups = g * (c.full * (rounds - 1) + c.any + c.first * clamp01(f) + c.second * clamp01(f - 1) +
                                 c.more * (f > 2 ? f - 2 : 0.0) + (f > 1 ? c.shared : 0.0));
      double cost = c.fixed + c.again * (rounds - 1) + c.out * per_unit + groups;
      if (S > 1) cost += c.slice0 + c.slice1 * S + c.slice2 * per_unit;
      if (cost < choice.wide) choice = Tile4Choice{i, S, cost, cost + (c.packed - 1.0) * groups};
    }
  }
  return choice;
}

TilePlan tile_plan(bool w4a4, int M, int N, int K, int shape, int S) {
  const TileShape& t = shape_of(w4a4, shape);
  const int edge = 32;                  // MFMA tile edge
  const int bn = edge * t.TN * t.WGN, bm = edge * t.TMW * t.WGM, G = K / kGroup;
  TilePlan p{};
  p.shape = shape;
  p.nb = (N + bn - 1) / bn;
  p.mb = (M + bm - 1) / bm;
  if (S > G) S = G;
  if (p.nb * p.mb > kMaxTickets || (!w4a4 && shape == 7)) S = 1;
  p.S = S;
  return p;
}

inline size_t plan_ws_bytes(bool w4a4, const TilePlan& p) {
  if (p.S <= 1) return 0;
  const TileShape& t = shape_of(w4a4, p.shape);
  const int edge = 32;
  const size_t block_floats = (size_t)(edge * t.TN * t.WGN) * (edge * t.TMW * t.WGM);   // whole blocks, ragged or not
  return kTicketBytes + (size_t)p.S * p.nb * p.mb * block_floats * 4;
}

// ---------------------------------------------------------------- the plan of a product
enum Product { kVerify, kDraft, kDraftWide };      // W4A16; W4A4 on packed codes; W4A4 on widened codes
enum class Kernel { none, stream, tile, generic };
struct Plan {
  Kernel kernel;      // none: not a size this product takes
  StreamPlan stream;
  TilePlan tile;
  size_t need;        // bytes of workspace
  bool optional;      // runs unsliced, so without any, where the workspace does not hold that
  double cost;        // verify mode: microseconds by the cost tables; a forced plan has none
};
// Tokens from which the draft mode may run on the tiled kernel (the streaming one is always the faster below) and
// the widened format is accepted
constexpr int kTileMinM4 = 25;

// What the streaming kernels take of what kStreamCost4 says, beside the tiled ones and kCost4, since the tables were fitted
// (loads sooner, sums combined in one pass, workgroups of four wavefronts; the tiled kernels gained less).  The medians
// on 260 products are 0.94 and, on four wavefronts, 0.87, but they spread: at 64 tokens 27648 outputs from 5120 (0.96 of
// the tiled cost by the tables) still take 24.0 us streaming and 23.4 on widened codes, 36864 from 6144 (0.99) 33.7 and
// 41.2.  So only what the tables call a tie goes over.  Past 64 tokens and on fewer than 16 groups they decide alone.
double stream_since(int M, int G) { return M <= 64 && G >= 16 ? 0.97 : 1.0; }

// A pure function of its arguments and the overrides, worked out once per call: the entry points launch what it
// says and ask for the workspace it needs, qspec_workspace_bytes gives the most that any product of the size needs.
Plan plan_product(Product product, int M, int N, int K) {
  const bool w4a4 = product != kVerify;
  const PlanOverrides& ov = overrides();
  const int G = K / kGroup;
  Plan p{};
  if (ov.generic && M > kStreamMaxM) {
    p.kernel = product == kDraftWide ? Kernel::none : Kernel::generic;
    return p;
  }
  // up to here the streaming kernels have it without a look at the tiled ones' shapes: 32 verify-mode tokens, 64
  // draft-mode tokens where the tiled kernel has no cheaper plan
  const bool within = M <= (w4a4 ? kStreamMaxM4 : kStreamMaxM);
  int shape = 0, S = 0;                            // S == 0: no tiled plan yet
  const bool forced_tile = tile_override(w4a4, &shape, &S);
  bool stream = true;
  if (ov.stream_max[w4a4]) stream = M <= ov.stream_max[w4a4];
  else if (within && (!w4a4 || M < kTileMinM4 || ov.stream_fields[1] != 0 || ov.generic)) stream = true;
  else if (!within && forced_tile) stream = false;
  else if (!w4a4 || ov.stream_fields[1] != 0) {
    p.stream = plan_stream(w4a4, M, N, K);
    stream = p.stream.nt > 0;
  } else {                                         // draft mode: the cheaper of the two kernels
    double streaming = best_stream(true, M, N, G, false, &p.stream);
    p.stream.waves = stream_waves(p.stream);
    streaming *= stream_since(M, G);
    const Tile4Choice tiled = best_tile4(M, N, G, 4, streaming);
    stream = tiled.S == 0 || (product == kDraft && tiled.packed >= streaming);
    if (!forced_tile) { shape = tiled.shape; S = tiled.S; }
  }
  if (stream && product != kDraftWide) {
    p.kernel = Kernel::stream;
    if (p.stream.nt == 0) p.stream = plan_stream(w4a4, M, N, K);
    p.need = stream_ws_bytes(p.stream);
    p.cost = p.stream.cost;
    return p;
  }
  if (stream) {
    // A caller that has quantised to the widened format before it knew the size is served by the tiled kernel, in
    // the slices it would have there (1024 outputs from 28672 at 300 tokens 32.1 us, unsliced 84.2).
    if (M < kTileMinM4 || ov.stream_fields[1] != 0 || ov.stream_max[1] != 0 || ov.generic) return p;
    p.optional = true;
  }
  if (S == 0 && w4a4) {
    const Tile4Choice tiled = best_tile4(M, N, G);
    shape = tiled.shape; S = tiled.S;
  } else if (S == 0) {
    p.cost = plan_tile16(M, N, G, &shape, &S);
  }
  p.kernel = Kernel::tile;
  p.tile = tile_plan(w4a4, M, N, K, shape, S);
  p.need = plan_ws_bytes(w4a4, p.tile);
  return p;
}

// A verify-mode product whose last block of 128 tokens is a short one can run as two launches: the whole blocks, and
// the rows that are left on what is cheapest for so few.  The short block costs a workgroup as much as a full one,
// and where it adds a round of workgroups or keeps a smaller shape from fitting one the rest is cheaper on its own, though
// it reads the weights a second time: 11008 -> 4096 at 2050 tokens 190.8 us on 136 blocks of 512 x 128, 166.9 on
// 256 of 256 x 128 and two rows on the streaming kernel; 21760 -> 7936 at 513 tokens 213 and 177.  The line lies at
// 0.9 of the cost of the one launch: on 90 ragged products of 129 to 2050 tokens the second launch measures 0.06 more of it
// than the tables say on average; of those below the line the slowest took 1.004 times the one launch, the mean 0.91.
// No product needs more workspace for it.
struct Split {
  int rows;           // of the first launch; 0: one launch
  Plan first, rest;
};
Split split_tokens(Product product, const Plan& whole, int M, int N, int K) {
  Split s{};
  const int rows = M / 128 * 128, left = M - rows;
  if (product != kVerify || whole.kernel != Kernel::tile || whole.cost == 0.0 || rows == 0 || left == 0) return s;
  s.first = plan_product(product, rows, N, K);
  if (s.first.cost == 0.0 || s.first.cost >= 0.9 * whole.cost || s.first.need > whole.need) return s;
  s.rest = plan_product(product, left, N, K);
  if (s.rest.cost > 0.0 && s.rest.need <= whole.need && s.first.cost + s.rest.cost < 0.9 * whole.cost) s.rows = rows;
  return s;
}

// Where qspec_workspace_bytes covers optional slices: sizes that ran on the tiled kernel before the streaming one took
// row blocks of every size, so that programs hold widened codes for them.  Not everywhere: a caller on packed
// codes would allocate 4 to 32 MiB for nothing (0.2 to 0.3 ms before the first call of two decoder blocks at 32 tokens).
// And where the tables alone, before the streaming kernels gained on them, advised that format.
bool covers_optional(int M, int N, int K) {
  StreamPlan stream{};
  if (best_tile4(M, N, K / kGroup, 4, best_stream(true, M, N, K / kGroup, false, &stream)).S != 0) return true;
  return M > 128 || (M > 64 && (N > 8192 || K > 8192)) || (M >= 48 && N >= 170 * 128);
}

template <typename Kernel>
int launch_tile_kernel(Kernel kernel, int threads, const TileArgs& a, hipStream_t s) {
  const uint32_t total = (uint32_t)(a.nb * a.mb * a.S);
  launch_kernel(kernel, dim3(total), dim3(threads), 0, s, a.codes, a.act, a.sa, a.M, a.N, a.K, a.S, a.mb, total, a.row_rcp,
                     TileRest{a.y, a.ws, a.tickets, a.nb});
  return QSPEC_OK;
}

template <int PN, int PM, int WGN, int WGM, int OCC>
int launch_tile4w_inst(const TileArgs& a, bool wide, hipStream_t s) {
  return wide ? launch_tile_kernel(gemm_tile4w_kernel<PN, PM, WGN, WGM, OCC, true>, 64 * WGN * WGM, a, s)
              : launch_tile_kernel(gemm_tile4w_kernel<PN, PM, WGN, WGM, OCC, false>, 64 * WGN * WGM, a, s);
}

template <int PN, int PM, int WGN, int WGM, int NW, int OCC, int WGK = 1>
int launch_tile16w_inst(const TileArgs& a, hipStream_t s) {
  return launch_tile_kernel(gemm_tile16w_kernel<PN, PM, WGN, WGM, WGK, NW, OCC>, 64 * WGN * WGM * WGK, a, s);
}

template <bool W4A4>
int launch_tile(const TilePlan& plan, TileArgs a, void* workspace, hipStream_t s, bool wide = false) {
  a.S = plan.S; a.nb = plan.nb; a.mb = plan.mb;
  // exact while total x (mb S) stays below 2^32
  const uint64_t per_row = (uint64_t)plan.mb * plan.S;
  a.row_rcp = per_row > 1 && per_row * per_row * plan.nb < 0x100000000ull ? (uint32_t)((0x100000000ull + per_row - 1) / per_row) : 0u;
  a.tickets = static_cast<unsigned*>(workspace);
  a.ws = plan.S > 1 ? reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + kTicketBytes) : nullptr;
  if (W4A4) {
    switch (plan.shape) {
      case 0: return launch_tile4w_inst<1, 4, 4, 1, 2>(a, wide, s);
      case 1: return launch_tile4w_inst<1, 2, 4, 1, 2>(a, wide, s);
      case 2: return launch_tile4w_inst<1, 2, 2, 1, 2>(a, wide, s);
      default: return launch_tile4w_inst<1, 4, 8, 1, 1>(a, wide, s);
    }
  }
  switch (plan.shape) {
    case 0: return launch_tile16w_inst<1, 4, 4, 1, 4, 2>(a, s);
    case 1: return launch_tile16w_inst<1, 2, 4, 1, 2, 1, 2>(a, s);
    case 2: return launch_tile16w_inst<1, 2, 2, 1, 2, 2, 2>(a, s);
    case 3: return launch_tile16w_inst<1, 4, 4, 1, 2, 1, 2>(a, s);
    case 4: return launch_tile16w_inst<1, 4, 8, 1, 2, 1>(a, s);
    case 5: return launch_tile16w_inst<2, 2, 2, 1, 2, 1, 4>(a, s);
    case 6: return launch_tile16w_inst<1, 2, 4, 1, 2, 3>(a, s);
    default:
      return launch_tile_kernel(gemm_tile16w2_kernel, 512, a, s);
  }
}

// ---------------------------------------------------------------- acceptance (after the verify pass)
// Chunks per logits row: about 4096 logits per workgroup, at most one chunk per lane
// of the second kernel.  A pure function of V.
struct ArgmaxPlan { int C, chunk; };
ArgmaxPlan plan_argmax(int V) {
  int C = (V + 4095) / 4096;
  if (C > kArgmaxMaxChunks) C = kArgmaxMaxChunks;
  if (C < 1) C = 1;
  int chunk = ((V + C - 1) / C + 7) & ~7;
  C = (V + chunk - 1) / chunk;
  return ArgmaxPlan{C, chunk};
}

// Device address of `scratch` on the current device, looked up once per device (with that
// device current) and kept.  nullptr: the lookup failed.
constexpr int kMaxDevices = 64;
void* scratch_of_device(int* status) {
  static void* ptr[kMaxDevices];
  static bool known[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { *status = QSPEC_ERR_HIP; return nullptr; }
  if (!known[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      *status = QSPEC_ERR_HIP;
      return nullptr;
    }
    ptr[dev] = p;
    known[dev] = true;
  }
  *status = QSPEC_OK;
  return ptr[dev];
}

// Zero the arrival counters at the head of a scratch area (a kernel, not a memset: the
// launch may be captured into a graph).
__global__ __launch_bounds__(256) void clear_tickets_kernel(unsigned* tickets, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) tickets[i] = 0u;
}

// ---------------------------------------------------------------- persistent draft-pass MLP
// Workgroups of the persistent launch: one per compute unit of the current device (looked up
// once per device).  0: the query failed.
int mlp_workgroups() {
  static int cus[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
  if (cus[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 0;
    cus[dev] = n;
  }
  return cus[dev];
}

constexpr size_t kMlpCounterBytes = 16384;
constexpr unsigned kMlpDefaultSpin = 200000;      // polls of about a microsecond each before a workgroup gives up

// Tiles per workgroup of the two projections for nwg workgroups; false: the shape does not fit the kernel.
bool mlp_plan(int M, int H, int I, int nwg, int* nt1, int* nt2) {
  if (M < 1 || M > 32 || nwg < 1) return false;
  const int tiles1 = 2 * I / 16, tiles2 = H / 16, G2 = I / kGroup;
  const int need1 = (tiles1 + nwg - 1) / nwg, need2 = (tiles2 + nwg - 1) / nwg;
  *nt1 = need1 <= 2 ? 2 : need1 <= 4 ? 4 : 6;
  *nt2 = need2 <= 1 ? 1 : 2;
  if (need1 > 6 || need2 > 2) return false;
  if (need2 * G2 > kMlpWBufTiles) return false;               // the down-projection tiles of a workgroup must fit LDS
  if ((size_t)(G2 + 2) * sizeof(unsigned) > kMlpCounterBytes) return false;
  return true;
}

template <int TM, int NT1>
int launch_mlp_nt2(const MlpArgs& a, int nt2, int nwg, hipStream_t s) {
  if (nt2 == 1) launch_kernel((mlp_draft_kernel<TM, NT1, 1>), dim3(nwg), dim3(kStreamWaves * 64), 0, s, a);
  else launch_kernel((mlp_draft_kernel<TM, NT1, 2>), dim3(nwg), dim3(kStreamWaves * 64), 0, s, a);
  return QSPEC_OK;
}
template <int TM>
int launch_mlp(const MlpArgs& a, int nt1, int nt2, int nwg, hipStream_t s) {
  switch (nt1) {
    case 2: return launch_mlp_nt2<TM, 2>(a, nt2, nwg, s);
    case 4: return launch_mlp_nt2<TM, 4>(a, nt2, nwg, s);
    case 6: return launch_mlp_nt2<TM, 6>(a, nt2, nwg, s);
    default: return QSPEC_ERR_UNSUPPORTED;
  }
}

inline bool misaligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) != 0; }

inline int check_accept_shape(int B, int gamma, int V) {
  if (B < 1 || gamma < 1 || V < 1) return QSPEC_ERR_SHAPE;
  if ((long long)B * (gamma + 1) > 65535) return QSPEC_ERR_SHAPE;        // one grid row per logits row
  return QSPEC_OK;
}

// ---------------------------------------------------------------- the three products
int check_gemm(const void* packed, const void* act, const float* sa, int M, int N, int K, int group, void* y_f16) {
  if (!packed || !act || !y_f16) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, N, K, group)) return st;
  if (misaligned(packed) || misaligned(act) || misaligned(sa) || misaligned(y_f16)) return QSPEC_ERR_ALIGN;
  return QSPEC_OK;
}

int launch_product(Product product, const Plan& plan, const void* packed, const void* act, const float* sa,
                   int M, int N, int K, void* y_f16, void* workspace, hipStream_t s) {
  const bool w4a4 = product != kVerify;
  const auto operands = [&](auto& a) {
    a.codes = static_cast<const uint4*>(packed);
    a.scalesT = blob_scales(packed, N, K);
    a.act = act;
    a.sa = sa;
    a.y = static_cast<uint16_t*>(y_f16);
    a.M = M; a.N = N; a.K = K; a.G = K / kGroup;
  };
  if (plan.kernel == Kernel::stream) {
    StreamArgs a{};
    operands(a);
    if (int st = w4a4 ? launch_stream<true>(plan.stream, a, workspace, s) : launch_stream<false>(plan.stream, a, workspace, s)) return st;
  } else if (plan.kernel == Kernel::tile) {
    TileArgs a{};
    operands(a);
    if (int st = w4a4 ? launch_tile<true>(plan.tile, a, workspace, s, product == kDraftWide)
                      : launch_tile<false>(plan.tile, a, workspace, s)) return st;
  } else {
    GemmArgs a{};
    operands(a);
    switch (pick_tm(M)) {
      case 1: w4a4 ? launch_w4a4<1>(a, s) : launch_w4a16<1>(a, s); break;
      case 2: w4a4 ? launch_w4a4<2>(a, s) : launch_w4a16<2>(a, s); break;
      case 4: w4a4 ? launch_w4a4<4>(a, s) : launch_w4a16<4>(a, s); break;
      default: w4a4 ? launch_w4a4<8>(a, s) : launch_w4a16<8>(a, s); break;
    }
  }
  return launch_status();
}

// One launch, or two (split_tokens).
int launch_whole_or_split(Product product, const Plan& plan, const void* packed, const void* act, const float* sa,
                          int M, int N, int K, void* y_f16, void* workspace, hipStream_t s) {
  const Split split = split_tokens(product, plan, M, N, K);
  if (split.rows == 0) return launch_product(product, plan, packed, act, sa, M, N, K, y_f16, workspace, s);
  if (int st = launch_product(product, split.first, packed, act, sa, split.rows, N, K, y_f16, workspace, s)) return st;
  return launch_product(product, split.rest, packed, static_cast<const uint8_t*>(act) + (size_t)split.rows * K * 2, sa,
                        M - split.rows, N, K, static_cast<uint8_t*>(y_f16) + (size_t)split.rows * N * 2, workspace, s);
}

int gemm(Product product, const void* packed, const void* act, const float* sa, int M, int N, int K, int group,
         void* y_f16, void* workspace, size_t workspace_bytes, void* stream) {
  if (int st = check_gemm(packed, act, sa, M, N, K, group, y_f16)) return st;
  Plan plan = plan_product(product, M, N, K);
  if (plan.kernel == Kernel::none) return QSPEC_ERR_UNSUPPORTED;   // too few tokens for the widened format
  if (plan.need > 0 && (!workspace || workspace_bytes < plan.need)) {
    if (!plan.optional) return QSPEC_ERR_WORKSPACE;
    plan.tile = tile_plan(true, M, N, K, best_tile4(M, N, K / kGroup, 1).shape, 1);
  }
  if (int st = check_device()) return st;
  return launch_whole_or_split(product, plan, packed, act, sa, M, N, K, y_f16, workspace, static_cast<hipStream_t>(stream));
}

}  // namespace

extern "C" {

const char* qspec_status_string(int status) {
  switch (status) {
    case QSPEC_OK: return "ok";
    case QSPEC_ERR_NULL: return "null pointer";
    case QSPEC_ERR_SHAPE: return "unsupported shape or argument value (need group == 128, K % 128 == 0, N % 16 == 0, M >= 1, every buffer below 2 GiB; see the entry point for its other arguments)";
    case QSPEC_ERR_ALIGN: return "pointer not 16-byte aligned";
    case QSPEC_ERR_WORKSPACE: return "workspace too small";
    case QSPEC_ERR_HIP: return "HIP runtime error";
    case QSPEC_ERR_UNSUPPORTED: return "device is not gfx950, a forced plan names a kernel instance that does not exist, or the shape lies outside what this variant entry point takes";
    default: return "unknown status";
  }
}

int qspec_version(void) { return 1000; }

size_t qspec_packed_weight_bytes(int N, int K, int group) {
  if (check_shape(1, N, K, group) != QSPEC_OK) return 0;
  return (size_t)N * K / 2 + (size_t)N * (K / kGroup) * 2;
}

size_t qspec_workspace_bytes(int M, int N, int K, int group) {
  if (check_shape(M, N, K, group) != QSPEC_OK) return 0;
  size_t most = 0;
  for (Product product : {kVerify, kDraft, kDraftWide}) {
    const Plan plan = plan_product(product, M, N, K);
    if (plan.optional && !covers_optional(M, N, K)) continue;
    if (plan.need > most) most = plan.need;
  }
  return most;
}

int qspec_pack_weights(const int8_t* codes, const void* scales_f16, int N, int K, int group,
                       void* packed, void* stream) {
  if (!codes || !scales_f16 || !packed) return QSPEC_ERR_NULL;
  if (int st = check_shape(1, N, K, group)) return st;
  if (misaligned(codes) || misaligned(scales_f16) || misaligned(packed)) return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int G = K / kGroup;
  const size_t n_words = (size_t)N * K / 8;
  launch_kernel(pack_codes_kernel, dim3(blocks_for(n_words, 256)), dim3(256), 0, s,
                     codes, static_cast<uint32_t*>(packed), N, K, G);
  uint16_t* sc_out = reinterpret_cast<uint16_t*>(static_cast<uint8_t*>(packed) + (size_t)N * K / 2);
  launch_kernel(transpose_scales_kernel, dim3(blocks_for((size_t)N * G, 256)), dim3(256), 0, s,
                     static_cast<const uint16_t*>(scales_f16), sc_out, N, G);
  return launch_status();
}

int qspec_unpack_weights(const void* packed, int N, int K, int group,
                         int8_t* codes, void* scales_f16, void* stream) {
  if (!codes || !scales_f16 || !packed) return QSPEC_ERR_NULL;
  if (int st = check_shape(1, N, K, group)) return st;
  if (misaligned(codes) || misaligned(scales_f16) || misaligned(packed)) return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int G = K / kGroup;
  const size_t n_words = (size_t)N * K / 8;
  launch_kernel(unpack_codes_kernel, dim3(blocks_for(n_words, 256)), dim3(256), 0, s,
                     static_cast<const uint32_t*>(packed), codes, N, K, G);
  // [G][N] -> [N][G] is the same transpose with the roles swapped
  launch_kernel(transpose_scales_kernel, dim3(blocks_for((size_t)N * G, 256)), dim3(256), 0, s,
                     blob_scales(packed, N, K), static_cast<uint16_t*>(scales_f16), G, N);
  return launch_status();
}

int qspec_quant_act(const void* x_f16, int M, int K, int group, uint8_t* qa, float* sa, void* stream) {
  if (!x_f16 || !qa || !sa) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, kTileRows, K, group)) return st;
  if (misaligned(x_f16) || misaligned(qa) || misaligned(sa)) return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  const size_t n_words = (size_t)M * K / 8;
  launch_kernel(quant_act_kernel, dim3(blocks_for(n_words, 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), QuantArgs{static_cast<const uint4*>(x_f16), reinterpret_cast<uint32_t*>(qa), sa, n_words});
  return launch_status();
}

int qspec_w4a4_takes_wide(int M, int N, int K, int group) {
  if (check_shape(M, N, K, group) != QSPEC_OK) return 0;
  const Plan plan = plan_product(kDraftWide, M, N, K);
  return plan.kernel == Kernel::tile && !plan.optional ? 1 : 0;
}

int qspec_quant_act_wide(const void* x_f16, int M, int K, int group, int8_t* qa8, float* sa, void* stream) {
  if (!x_f16 || !qa8 || !sa) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, kTileRows, K, group)) return st;
  if (misaligned(x_f16) || misaligned(qa8) || misaligned(sa)) return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  const size_t n_words = (size_t)M * K / 8;
  launch_kernel(quant_act_wide_kernel, dim3(blocks_for(n_words, 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), QuantArgs{static_cast<const uint4*>(x_f16), reinterpret_cast<uint32_t*>(qa8), sa, n_words});
  return launch_status();
}

int qspec_rmsnorm_quant(const void* x_f16, const void* weight_f16, float eps, int M, int K, int group,
                        int rotate, uint8_t* qa, float* sa, void* h_f16, void* stream) {
  if (!x_f16 || !weight_f16 || !qa || !sa) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, kTileRows, K, group)) return st;
  if (!(eps >= 0.0f) || !(eps <= 3.0e38f) || rotate < 0 || rotate > 3) return QSPEC_ERR_SHAPE;
  if (misaligned(x_f16) || misaligned(weight_f16) || misaligned(qa) || misaligned(sa) || misaligned(h_f16))
    return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  const uint4* x = static_cast<const uint4*>(x_f16);
  const uint4* w = static_cast<const uint4*>(weight_f16);
  uint32_t* words = reinterpret_cast<uint32_t*>(qa);
  uint4* h = static_cast<uint4*>(h_f16);
  // threads per row: one per 8 features up to 1024, whole wavefronts
  const int kw = K / 8;
  const int T = kw >= kRowMaxThreads ? kRowMaxThreads : (kw + 63) / 64 * 64;
  const int chunks = (kw + T - 1) / T;
  const double inv_K = 1.0 / (double)K;
  const dim3 grid(M), block(T);
  if (chunks <= 1) launch_kernel(rmsnorm_quant_kernel<1>, grid, block, 0, s, x, w, eps, K, inv_K, words, sa, h, rotate);
  else if (chunks <= 2) launch_kernel(rmsnorm_quant_kernel<2>, grid, block, 0, s, x, w, eps, K, inv_K, words, sa, h, rotate);
  else if (chunks <= 4) launch_kernel(rmsnorm_quant_kernel<4>, grid, block, 0, s, x, w, eps, K, inv_K, words, sa, h, rotate);
  else launch_kernel(rmsnorm_quant_kernel<0>, grid, block, 0, s, x, w, eps, K, inv_K, words, sa, h, rotate);
  return launch_status();
}

int qspec_silu_mul_quant(const void* gate_up_f16, int M, int I, int group,
                         int rotate, uint8_t* qa, float* sa, void* h_f16, void* stream) {
  if (!gate_up_f16 || !qa || !sa) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, kTileRows, I, group)) return st;
  if (rotate < 0 || rotate > 3) return QSPEC_ERR_SHAPE;
  if (misaligned(gate_up_f16) || misaligned(qa) || misaligned(sa) || misaligned(h_f16)) return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  launch_kernel(silu_mul_quant_kernel, dim3(blocks_for(I / 8, 256), M < 65535 ? M : 65535), dim3(256), 0,
                     static_cast<hipStream_t>(stream), static_cast<const uint4*>(gate_up_f16), I / 8, M, rotate,
                     reinterpret_cast<uint32_t*>(qa), sa, static_cast<uint4*>(h_f16));
  return launch_status();
}

int qspec_hadamard_quant(const void* x_f16, int M, int K, int group,
                         uint8_t* qa, float* sa, void* h_f16, void* stream) {
  if (!x_f16 || !qa || !sa) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, kTileRows, K, group)) return st;
  if (misaligned(x_f16) || misaligned(qa) || misaligned(sa) || misaligned(h_f16)) return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  const size_t n_words = (size_t)M * K / 8;
  launch_kernel(hadamard_quant_kernel, dim3(blocks_for(n_words, 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), static_cast<const uint4*>(x_f16),
                     reinterpret_cast<uint32_t*>(qa), sa, static_cast<uint4*>(h_f16), n_words);
  return launch_status();
}

int qspec_reorder_quant(const void* x_f16, const int32_t* perm, int M, int K, int group,
                        int n_outlier_groups, uint8_t* qa, float* sa, void* h_f16, void* stream) {
  if (!x_f16 || !perm || !qa || !sa) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, kTileRows, K, group)) return st;
  if (n_outlier_groups < 0 || n_outlier_groups > K / kGroup) return QSPEC_ERR_SHAPE;
  if (int st = check_shape(M, kTileRows, K + kGroup * n_outlier_groups, group)) return st;
  if (misaligned(x_f16) || misaligned(perm) || misaligned(qa) || misaligned(sa) || misaligned(h_f16))
    return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  const size_t n_words = (size_t)M * K / 8;
  launch_kernel(reorder_quant_kernel, dim3(blocks_for(n_words, 256)), dim3(256), 0,
                     static_cast<hipStream_t>(stream), static_cast<const uint16_t*>(x_f16), perm, K,
                     n_outlier_groups, reinterpret_cast<uint32_t*>(qa), sa, static_cast<uint4*>(h_f16), n_words);
  return launch_status();
}

int qspec_gemm_w4a4(const void* packed, const uint8_t* qa, const float* sa, int M, int N, int K, int group,
                    void* y_f16, void* workspace, size_t workspace_bytes, void* stream) {
  if (!sa) return QSPEC_ERR_NULL;
  return gemm(kDraft, packed, qa, sa, M, N, K, group, y_f16, workspace, workspace_bytes, stream);
}

int qspec_gemm_w4a4_wide(const void* packed, const int8_t* qa8, const float* sa, int M, int N, int K, int group,
                         void* y_f16, void* workspace, size_t workspace_bytes, void* stream) {
  if (!sa) return QSPEC_ERR_NULL;
  return gemm(kDraftWide, packed, qa8, sa, M, N, K, group, y_f16, workspace, workspace_bytes, stream);
}

int qspec_gemm_w4a16(const void* packed, const void* x_f16, int M, int N, int K, int group,
                     void* y_f16, void* workspace, size_t workspace_bytes, void* stream) {
  return gemm(kVerify, packed, x_f16, nullptr, M, N, K, group, y_f16, workspace, workspace_bytes, stream);
}

int qspec_gemm_w4a16_noalloc(const void* packed, const void* x_f16, int M, int N, int K, int group,
                             void* y_f16, void* stream) {
  if (int st = check_gemm(packed, x_f16, nullptr, M, N, K, group, y_f16)) return st;
  const Plan plan = plan_product(kVerify, M, N, K);
  if (plan.need > kScratchBytes) return QSPEC_ERR_WORKSPACE;       // beyond the built-in scratch: use qspec_gemm_w4a16
  if (int st = check_device()) return st;
  int st = QSPEC_OK;
  void* ws = scratch_of_device(&st);
  if (!ws) return st;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  if (plan.need > 0) {
    // the counters must start at zero whatever an earlier (possibly failed) call left
    launch_kernel(clear_tickets_kernel, dim3(kMaxTickets / 256), dim3(256), 0, s, static_cast<unsigned*>(ws), kMaxTickets);
  }
  return launch_whole_or_split(kVerify, plan, packed, x_f16, nullptr, M, N, K, y_f16, ws, s);
}

size_t qspec_mlp_draft_workspace_bytes(int M, int H, int I, int group) {
  if (check_shape(M, H, I, group) != QSPEC_OK || check_shape(M, 2 * I, H, group) != QSPEC_OK) return 0;
  return kMlpCounterBytes;
}

int qspec_mlp_draft(const void* packed_gate_up, const void* packed_down, const uint8_t* qa_h, const float* sa_h,
                    int M, int H, int I, int group, void* gate_up_f16, uint8_t* qa_i, float* sa_i, void* y_f16,
                    void* workspace, size_t workspace_bytes, int* status_word, void* stream) {
  if (!packed_gate_up || !packed_down || !qa_h || !sa_h || !gate_up_f16 || !qa_i || !sa_i || !y_f16 || !workspace || !status_word)
    return QSPEC_ERR_NULL;
  if (int st = check_shape(M, 2 * I, H, group)) return st;
  if (int st = check_shape(M, H, I, group)) return st;
  if (misaligned(packed_gate_up) || misaligned(packed_down) || misaligned(qa_h) || misaligned(sa_h) || misaligned(gate_up_f16) ||
      misaligned(qa_i) || misaligned(sa_i) || misaligned(y_f16) || misaligned(workspace) || misaligned4(status_word))
    return QSPEC_ERR_ALIGN;
  if (workspace_bytes < kMlpCounterBytes) return QSPEC_ERR_WORKSPACE;
  if (int st = check_device()) return st;
  const int nwg = mlp_workgroups();
  if (nwg <= 0) return QSPEC_ERR_HIP;
  int nt1 = 0, nt2 = 0;
  if (!mlp_plan(M, H, I, nwg, &nt1, &nt2)) return QSPEC_ERR_UNSUPPORTED;
  MlpArgs a{};
  a.codes1 = static_cast<const uint4*>(packed_gate_up);
  a.scales1T = blob_scales(packed_gate_up, 2 * I, H);
  a.qa_h = qa_h; a.sa_h = sa_h;
  a.y_gu = static_cast<uint16_t*>(gate_up_f16);
  a.qa_i = qa_i; a.sa_i = sa_i;
  a.codes2 = static_cast<const uint4*>(packed_down);
  a.scales2T = blob_scales(packed_down, H, I);
  a.y = static_cast<uint16_t*>(y_f16);
  a.counters = static_cast<unsigned*>(workspace);
  a.status = status_word;
  a.M = M; a.N1 = 2 * I; a.K1 = H; a.N2 = H; a.K2 = I;
  a.spin_limit = overrides().mlp_spin ? overrides().mlp_spin : kMlpDefaultSpin;   // QSPEC_MLP_SPIN: tests of the give-up path
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (int st = (M <= 16 ? launch_mlp<1>(a, nt1, nt2, nwg, s) : launch_mlp<2>(a, nt1, nt2, nwg, s))) return st;
  return launch_status();
}

int qspec_gemm_w4a4_partials(const void* packed, const uint8_t* qa, int M, int N, int K, int group,
                             int n0, int n_count, int32_t* partials, void* stream) {
  if (!packed || !qa || !partials) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, N, K, group)) return st;
  if (n0 < 0 || n_count <= 0 || n0 % 16 || n_count % 16 || (long long)n0 + n_count > N) return QSPEC_ERR_SHAPE;
  if (misaligned(packed) || misaligned(qa) || misaligned(partials)) return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  GemmArgs a{};
  a.codes = static_cast<const uint4*>(packed);
  a.scalesT = blob_scales(packed, N, K);
  a.act = qa;
  a.partials = partials;
  a.M = M; a.N = N; a.K = K; a.G = K / kGroup;
  a.n0 = n0; a.n_count = n_count;
  dim3 grid(n_count / 16, (M + 15) / 16);
  launch_kernel((gemm_w4a4_generic<1, 4, true>), grid, dim3(256), 0,
                     static_cast<hipStream_t>(stream), a);
  return launch_status();
}

size_t qspec_accept_workspace_bytes(int B, int gamma, int V) {
  if (check_accept_shape(B, gamma, V) != QSPEC_OK) return 0;
  return (size_t)B * (gamma + 1) * plan_argmax(V).C * sizeof(uint64_t);
}

int qspec_greedy_accept(const void* logits_f16, const int32_t* draft_tokens, int B, int gamma, int V,
                        int32_t* n_accept, int32_t* out_tokens,
                        void* workspace, size_t workspace_bytes, void* stream) {
  if (!logits_f16 || !draft_tokens || !n_accept || !out_tokens || !workspace) return QSPEC_ERR_NULL;
  if (int st = check_accept_shape(B, gamma, V)) return st;
  if (misaligned(logits_f16) || misaligned(workspace) || misaligned4(draft_tokens) || misaligned4(n_accept) ||
      misaligned4(out_tokens))
    return QSPEC_ERR_ALIGN;
  if (workspace_bytes < qspec_accept_workspace_bytes(B, gamma, V)) return QSPEC_ERR_WORKSPACE;
  if (int st = check_device()) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const ArgmaxPlan plan = plan_argmax(V);
  const int R = B * (gamma + 1);
  ArgmaxArgs a{static_cast<const uint16_t*>(logits_f16), static_cast<uint64_t*>(workspace), V, plan.C, plan.chunk};
  if (V % 8 == 0) launch_kernel((argmax_partial_kernel<true>), dim3(plan.C, R), dim3(kArgmaxThreads), 0, s, a);
  else launch_kernel((argmax_partial_kernel<false>), dim3(plan.C, R), dim3(kArgmaxThreads), 0, s, a);
  AcceptArgs f{static_cast<const uint64_t*>(workspace), draft_tokens, n_accept, out_tokens, gamma, plan.C};
  launch_kernel(accept_kernel, dim3(B), dim3(64 * (gamma + 1 < kAcceptRows ? gamma + 1 : kAcceptRows)), 0, s, f);
  return launch_status();
}

int qspec_kv_overwrite(const void* kv_verify_f16, const int32_t* n_accept, const int32_t* pos,
                       int B, int gamma, int D, int S, void* cache_f16, void* stream) {
  if (!kv_verify_f16 || !n_accept || !pos || !cache_f16) return QSPEC_ERR_NULL;
  if (B < 1 || gamma < 1 || S < 1 || D < 8 || D % 8 != 0) return QSPEC_ERR_SHAPE;
  if ((long long)B * (gamma + 1) > 0x7fffffffLL) return QSPEC_ERR_SHAPE;
  if (misaligned(kv_verify_f16) || misaligned(cache_f16) || misaligned4(n_accept) || misaligned4(pos))
    return QSPEC_ERR_ALIGN;
  if (int st = check_device()) return st;
  KvArgs a{static_cast<const uint4*>(kv_verify_f16), static_cast<uint4*>(cache_f16), n_accept, pos, gamma, D / 8, S};
  launch_kernel(kv_overwrite_kernel, dim3(B * (gamma + 1)), dim3(256), 0, static_cast<hipStream_t>(stream), a);
  return launch_status();
}

int qspec_debug_set_plan(const char* name, const char* value) {
  if (!name) return QSPEC_ERR_NULL;
  return apply_override(overrides(), name, value) ? QSPEC_OK : QSPEC_ERR_SHAPE;
}

int qspec_describe_kernel(int mode_w4a4, int M, int N, int K, int group, char* out, size_t cap) {
  if (!out || cap == 0) return QSPEC_ERR_NULL;
  if (int st = check_shape(M, N, K, group)) return st;
  const int launch = mode_w4a4 == 4 || mode_w4a4 == 5 ? mode_w4a4 - 3 : 0;      // of the verify mode's launches: 0 the plan of one
  if (launch) mode_w4a4 = 0;
  const char* b = mode_w4a4 ? "true" : "false";
  const bool wide = mode_w4a4 == 2;
  Plan plan = plan_product(wide ? kDraftWide : mode_w4a4 ? kDraft : kVerify, M, N, K);
  if (plan.kernel == Kernel::none) return QSPEC_ERR_UNSUPPORTED;
  if (launch) {
    const Split split = split_tokens(kVerify, plan, M, N, K);
    if (launch == 2 && split.rows == 0) { out[0] = 0; return QSPEC_OK; }
    if (split.rows) { plan = launch == 1 ? split.first : split.rest; M = launch == 1 ? split.rows : M - split.rows; }
  }
  if (plan.kernel == Kernel::stream) {
    snprintf(out, cap, "%sgemm_stream_kernel<%s, %d, %d>", plan.stream.waves == 4 ? "waves4::" : "", b, plan.stream.tm, plan.stream.nt);
  } else if (plan.kernel == Kernel::tile) {
    const TileShape& t = shape_of(mode_w4a4 != 0, plan.tile.shape);
    if (mode_w4a4) snprintf(out, cap, "gemm_tile4w_kernel<%d, %d, %d, %d, %d, %s>", t.TN, t.TMW, t.WGN, t.WGM, t.OCC, wide ? "true" : "false");
    else if (t.TN == 2 && t.TMW == 4) snprintf(out, cap, "gemm_tile16w2_kernel");
    else snprintf(out, cap, "gemm_tile16w_kernel<%d, %d, %d, %d, %d, %d, %d>", t.TN, t.TMW, t.WGN, t.WGM, t.WGK, t.NW, t.OCC);
  } else if (mode_w4a4) snprintf(out, cap, "gemm_w4a4_generic<%d, 4, false>", pick_tm(M));
  else snprintf(out, cap, "gemm_w4a16_generic<%d, 4>", pick_tm(M));
  return QSPEC_OK;
}

}  // extern "C"
