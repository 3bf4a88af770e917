// C ABI of the TreeSpark draft-tree step: argument checks, launch plans,
// the best-first wave builder and the verification drivers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <tuple>
#include <unordered_map>
#include <vector>

#include "launch.hpp"
#include "verify_fused.hpp"

// The scratch of ts_expand_noalloc, one copy per GPU.  In host code `scratch`
// names a host-side stand-in, not device memory: kernels get the device
// address that hipGetSymbolAddress returns, taken once per device with that
// device current (noalloc_scratch below).
static __device__ __align__(256) char scratch[TS_NOALLOC_SCRATCH_BYTES];

namespace ts {
namespace {

thread_local std::string g_last_error;

int32_t fail(int32_t code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return code;
}

#define TS_HIP(call)                                                                     \
  do {                                                                                   \
    hipError_t e_ = (call);                                                              \
    if (e_ != hipSuccess) return fail(TS_EHIP, "%s: %s", #call, hipGetErrorString(e_));  \
  } while (0)

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Armed once work is queued on a stream: an error return then waits for that
// work, so that no kernel or copy is still writing the caller's workspace or
// the staging buffer when the call returns.  Success paths disarm it.
struct DrainOnError {
  hipStream_t s;
  bool armed = true;
  ~DrainOnError() {
    if (armed) (void)hipStreamSynchronize(s);
  }
};

// Polls of one wait of a one-launch verification round before it gives up (a
// poll takes about a microsecond).
constexpr int kFusedSpinLimit = 1 << 16;

// Page-locked host staging for the small transfers of the host loops, so that
// they are true asynchronous DMA copies (kernels also read and write parts of
// it directly).  It belongs to the calling host thread, grows on demand and
// lives until ts_release_thread_state() frees it; every user synchronises its
// stream before it rewrites or grows the buffer.  There is deliberately no
// destructor: a thread-exit destructor of the main thread would run inside
// exit(), after the HIP runtime (and any profiler attached to it) may have
// been torn down.
struct ThreadState {
  char* stage = nullptr;
  size_t stage_bytes = 0;
  // T > 0 verification levels run in one launch, run again through the
  // per-stage launches after a wait ran out, and run per stage from the start
  int64_t fused_levels = 0, fused_fallbacks = 0, staged_levels = 0;
  int32_t verify_mode = TS_VERIFY_AUTO;
  int32_t wait_limit = kFusedSpinLimit;
};
ThreadState& thread_state() {
  thread_local ThreadState st;
  return st;
}

int32_t host_stage(size_t bytes, char** out) {
  ThreadState& st = thread_state();
  if (st.stage_bytes < bytes) {
    if (st.stage) TS_HIP(hipHostFree(st.stage));
    st.stage = nullptr;
    st.stage_bytes = 0;
    void* q = nullptr;
    // coherent: kernels read and write parts of it directly
    TS_HIP(hipHostMalloc(&q, bytes, hipHostMallocCoherent));
    st.stage = static_cast<char*>(q);
    st.stage_bytes = bytes;
  }
  *out = st.stage;
  return TS_OK;
}

// ---------------------------------------------------------------- checks

int32_t check_drafter(const ts_drafter* d) {
  if (!d) return fail(TS_EINVAL, "drafter is NULL");
  if (!d->U || !d->E || !d->W2) return fail(TS_EINVAL, "drafter tensor pointer is NULL");
  if (d->R <= 0 || d->D <= 0 || d->V <= 0 || d->r <= 0)
    return fail(TS_EINVAL, "drafter sizes must be positive (R=%d D=%d V=%d r=%d)", d->R, d->D, d->V, d->r);
  if (d->dtype != TS_F32 && d->dtype != TS_BF16) return fail(TS_EINVAL, "unknown dtype %d", d->dtype);
  if (((reinterpret_cast<uintptr_t>(d->U) | reinterpret_cast<uintptr_t>(d->E) |
        reinterpret_cast<uintptr_t>(d->W2)) & 15) != 0)
    return fail(TS_EINVAL, "U, E and W2 must start at 16-byte aligned addresses");
  if (d->D > TS_MAX_D) return fail(TS_EUNSUPPORTED, "D=%d exceeds %d (4-bit path digits)", d->D, TS_MAX_D);
  if (d->R >= TS_MAX_R) return fail(TS_EUNSUPPORTED, "R=%d exceeds %d", d->R, TS_MAX_R - 1);
  if (d->V > TS_MAX_V) return fail(TS_EUNSUPPORTED, "V=%d exceeds %d", d->V, TS_MAX_V);
  const bool ok = d->dtype == TS_BF16 ? (d->r == 32 || d->r == 64 || d->r == 128 || d->r == 256)
                                      : (d->r == 16 || d->r == 32 || d->r == 64);
  if (!ok) return fail(TS_EUNSUPPORTED, "rank r=%d not supported for dtype %d", d->r, d->dtype);
  return TS_OK;
}

int32_t check_k_T(const ts_drafter* d, int32_t k, float T) {
  if (k < 1 || k > TS_MAX_K) return fail(k < 1 ? TS_EINVAL : TS_EUNSUPPORTED, "k=%d outside [1, %d]", k, TS_MAX_K);
  if (k > d->V) return fail(TS_EINVAL, "k=%d exceeds V=%d", k, d->V);
  if (!(T >= 0.0f) || !std::isfinite(T)) return fail(TS_EINVAL, "T must be finite and >= 0");
  return TS_OK;
}

int32_t check_sampler(int32_t sampler) {
  if (sampler != TS_SAMPLER_GUMBEL && sampler != TS_SAMPLER_SEQUENTIAL)
    return fail(TS_EINVAL, "unknown sampler %d", sampler);
  return TS_OK;
}

PhiloxKeys philox_keys(uint64_t seed) {
  PhiloxKeys k;
  uint32_t a = (uint32_t)seed, b = (uint32_t)(seed >> 32);
  for (int r = 0; r < 10; ++r) {
    k.k0[r] = a;
    k.k1[r] = b;
    a += 0x9E3779B9u;
    b += 0xBB67AE85u;
  }
  return k;
}

// ---------------------------------------------------------------- expansion plan

struct Plan {
  int NB, S, n_pblocks, wpg, n_pgroups, S8;
  ChunkMap cm;
  int ks;
  int mode;     // kModeGreedy, kModeGumbel or kModeSeq (the kernels' mode)
  bool sample;  // T > 0: the merge takes lse of z/T and draws
  EvalPath path;  // LDS-staged bf16 streaming kernel (aligned or ragged rows) or the register one
  int nblk;     // 64-token blocks of the vocabulary
  int blk_ld;   // row stride of the block table (nblk rounded up to 16)
  size_t off_m, off_s0, off_sT, off_z[2], off_g[2], off_blk;
  size_t bytes;
};

// Compute units of the current device (256 when no device answers).
int device_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    cached[dev] = n;
  }
  return cached[dev];
}

// Resident blocks per CU of the streaming kernel for this plan (2 if unknown).
int eval_blocks_per_cu(int dtype, int ks, int nb, int mode, bool store_z, EvalPath path, int block) {
  static std::mutex mu;
  static std::map<std::tuple<int, int, int, int, bool, EvalPath, int>, int> cache;
  const auto key = std::make_tuple(dtype, ks, nb, mode, store_z, path, block);
  {
    std::lock_guard<std::mutex> lock(mu);
    const auto it = cache.find(key);
    if (it != cache.end()) return it->second;
  }
  int n = 0;
  if (dtype == TS_BF16) {
    switch (ks) {
      case 1: n = eval_blocks_per_cu_t<uint16_t, 1>(nb, mode, store_z, path, block); break;
      case 2: n = eval_blocks_per_cu_t<uint16_t, 2>(nb, mode, store_z, path, block); break;
      case 4: n = eval_blocks_per_cu_t<uint16_t, 4>(nb, mode, store_z, path, block); break;
      default: n = eval_blocks_per_cu_t<uint16_t, 8>(nb, mode, store_z, path, block); break;
    }
  } else {
    switch (ks) {
      case 4: n = eval_blocks_per_cu_t<float, 4>(nb, mode, store_z, path, block); break;
      case 8: n = eval_blocks_per_cu_t<float, 8>(nb, mode, store_z, path, block); break;
      default: n = eval_blocks_per_cu_t<float, 16>(nb, mode, store_z, path, block); break;
    }
  }
  if (n <= 0) n = 2;
  std::lock_guard<std::mutex> lock(mu);
  cache[key] = n;
  return n;
}

// Launch plan of one expansion.  store_z: the verification recompute, which
// writes the logits, runs one parent block per wave and makes no draws.
// sizing_only: the workspace size, which must not depend on the device or the
// sampler, so it assumes the largest chunk count and room for both samplers.
static_assert(TS_MAX_V <= kMaxChunks * 4096, "the merge holds kMaxChunks chunks of <= 4096 tokens");

// max_chunks: the most chunks the vocabulary allows (the plan of a launch
// whose parent count is only bounded on the host: parallelism comes from the
// chunks, and workgroups beyond the parents the device holds exit at once).
// even_chunks: the fewer chunks that one rounded-up length takes, for scratch
// that the plan with more of them does not fit.
Plan make_plan(const ts_drafter* d, int P, float T, int sampler, bool store_z = false,
               bool sizing_only = false, bool max_chunks = false, bool even_chunks = false) {
  Plan pl{};
  pl.sample = T > 0.0f && !store_z;
  pl.mode = !pl.sample ? kModeGreedy : sampler == TS_SAMPLER_SEQUENTIAL ? kModeSeq : kModeGumbel;
  // the streaming kernel's mode: with the separate z / T sum when T != 1
  const int eval_mode = pl.mode | (pl.sample && T != 1.0f ? kModeNeedT : 0);
  pl.nblk = (d->V + kBlkTokens - 1) / kBlkTokens;
  pl.blk_ld = ((pl.nblk + 15) / 16) * 16;
  pl.ks = d->dtype == TS_BF16 ? d->r / 32 : d->r / 4;
  // two parent blocks per wave pay off only when the parents fill them; a
  // bound on a device-held count (max_chunks) usually overstates them
  pl.NB = (P >= 512 && !max_chunks) ? 2 : 1;
  if (store_z) pl.NB = 1;
  // the LDS kernel reads U and W2 as raw buffers: byte offsets under 2^31
  // (and the stored logits as one under 2^32)
  const bool lds = d->dtype == TS_BF16 && ((uint64_t)d->R * d->D + 1) * d->V * 2 + 64 < (1ull << 31) &&
                   (uint64_t)d->V * d->r * 2 < (1ull << 31) &&
                   (!store_z || (uint64_t)P * d->V * 4 + 256 < (1ull << 32));
  pl.path = !lds ? EvalPath::kRegisters : d->V % 8 == 0 ? EvalPath::kLds : EvalPath::kLdsRagged;
  pl.n_pblocks = (P + 16 * pl.NB - 1) / (16 * pl.NB);
  // waves per workgroup (each workgroup loads every W2 tile of its chunk
  // once): eight for the greedy LDS kernel with two blocks per wave at rank
  // <= 64 (that kernel fits four waves per SIMD; with the ragged rows' extra
  // pieces its LDS would leave one workgroup per CU), else four
  pl.wpg = lds ? 4 : std::min(4, std::max(1, pl.n_pblocks));
  if (pl.path == EvalPath::kLds && pl.NB == 2 && pl.ks <= 2 && pl.mode == kModeGreedy) pl.wpg = 8;
  pl.n_pgroups = (pl.n_pblocks + pl.wpg - 1) / pl.wpg;
  // Chunks: as many workgroups as fit the chip at the kernel's occupancy, in
  // whole rounds (a few more would take a round of their own), chunks of
  // 256..4096 tokens, at most kMaxChunks per parent, their lengths within
  // one unit of each other (ChunkMap).  Units of 256 tokens keep the quads of
  // steps that sequential draws sum block masses over whole.
  const int unit = lds && pl.mode == kModeSeq ? 256 : 64;
  const int units = (d->V + unit - 1) / unit;
  const int s_min = (units * unit + 4095) / 4096;
  // the logit recompute leaves no partials: its chunks are not limited
  const int s_max = std::max(1, std::min((d->V + 255) / 256, store_z && !sizing_only ? INT_MAX : kMaxChunks));
  int S = s_max;
  if (!sizing_only && !max_chunks) {
    // At most four workgroups per CU: the kernels with one parent block per
    // wave fit five, but filling them all leaves no slack to even out the
    // chunks and more prologues.  ts_expand, V = 128256, r = 64, planned for five
    // and for four: 400 greedy parents 51.2 and 42.5 us, 320 38.1 and 34.4;
    // sequential draws T = 0.7, 384 parents 56.2 and 46.5, 450 63.8 and 52.5.
    // Where scratch is short, rows at any address plan for two workgroups per CU
    // (three fit): ts_expand_noalloc's array then takes 3072 parents at V = 151937
    // with sequential draws, 2816 with the chunks that three take.
    const bool ragged_even = even_chunks && pl.path == EvalPath::kLdsRagged;
    const int fit = ragged_even ? 2 : eval_blocks_per_cu(d->dtype, pl.ks, pl.NB, eval_mode, store_z, pl.path, 64 * pl.wpg);
    const int concurrent = device_cus() * (store_z ? fit : std::min(fit, 4));
    const int rounds = std::max(1, (pl.n_pgroups * s_min + concurrent - 1) / concurrent);
    S = std::max(1, rounds * concurrent / pl.n_pgroups);
    // Chunks are dealt to the 8 XCDs in turn, all parent groups of one to the
    // same XCD: with S no multiple of 8 some XCDs get one chunk more and, when
    // the groups do not divide their share, more workgroups than fit them (600
    // greedy parents: 170 chunks x 3 groups put 66 on two XCDs that hold 64;
    // ts_expand 56.9 us, with 168 chunks 49.9).
    if (S > 8 && !even_chunks && S < s_max) S &= ~7;
    if (even_chunks) {
      // chunks of one rounded-up length: fewer of them
      const int quantum = pl.path == EvalPath::kLds ? 256 : 64;
      int vc = std::max((d->V + S - 1) / S, (d->V + kMaxChunks - 1) / kMaxChunks);
      vc = std::min(std::max((vc + quantum - 1) / quantum * quantum, 256), 4096);
      S = (d->V + vc - 1) / vc;
    }
  }
  pl.S = std::min(std::max(S, s_min), std::max(s_max, s_min));
  // Where every workgroup has a CU to itself the longest chunk counts, and with
  // units of 256 tokens as many chunks as their limit allows often leave it no
  // shorter than fewer would: V = 151936 is 82 chunks of three units and 174 of
  // two, or 198 of three.  The fewer cost less in the merge and the draws, unless
  // they are so few that they leave much of the chip idle (ts_expand, the most and
  // the fewest chunks: T = 0.7, r = 64, 1 parent 25.6 and 25.2 us, 16 parents 26.4 and
  // 25.9, 4 parents at V = 160000 24.5 and 23.8, at V = 110000 (215 of 256), r = 128
  // 27.2 and 26.9, 17 parents at V = 140000 (183), K = 16 38.8 and 38.2; T = 1, 2 parents
  // at V = 75200 (147), r = 256, K = 16 52.6 and 55.0, at V = 66000 (129) 21.1 and
  // 21.4).  Units of 64 tokens keep the most: f32, 2 parents, V = 150000 50.0 and 50.9.
  if (!sizing_only && !max_chunks && unit == 256 && (long long)pl.S * pl.n_pgroups <= device_cus()) {
    const int longest = (units + pl.S - 1) / pl.S, fewest = (units + longest - 1) / longest;
    if (fewest * 10 >= pl.S * 7) pl.S = fewest;
  }
  pl.S8 = ((pl.S + 7) / 8) * 8;
  pl.cm = ChunkMap{unit, units / pl.S, units % pl.S};
#ifdef TS_DEBUG_RUNS
  if (!sizing_only)
    fprintf(stderr, "[plan] P=%d NB=%d path=%d wpg=%d n_pgroups=%d S=%d grid=%d bpc=%d cus=%d\n", P,
            pl.NB, (int)pl.path, pl.wpg, pl.n_pgroups, pl.S, pl.S8 * pl.n_pgroups,
            eval_blocks_per_cu(d->dtype, pl.ks, pl.NB, eval_mode, store_z, pl.path, 64 * pl.wpg), device_cus());
#endif
  const size_t a = align256((size_t)std::max(P, 1) * pl.S * 4);
  const size_t a4 = align256((size_t)std::max(P, 1) * pl.S * 4 * kTopRuns);
  size_t o = 0;
  pl.off_m = o; o += a;
  pl.off_s0 = o; o += a;
  pl.off_z[0] = o; o += a4;
  pl.off_z[1] = o; o += a;
  if (pl.sample || (sizing_only && T > 0.0f && !store_z)) {
    pl.off_sT = o; o += a;
    if (pl.mode == kModeGumbel || sizing_only) {
      pl.off_g[0] = o; o += a4;
      pl.off_g[1] = o; o += a;
    }
    if (pl.mode == kModeSeq || sizing_only) {
      pl.off_blk = o; o += align256((size_t)std::max(P, 1) * pl.blk_ld * 4);
    }
  }
  pl.bytes = o;
  return pl;
}

RunSummaryPtr summary_ptr(char* ws, const size_t (&off)[2]) {
  RunSummaryPtr r;
  r.m = reinterpret_cast<float*>(ws + off[0]);
  r.rest = reinterpret_cast<float*>(ws + off[1]);
  return r;
}

size_t expand_ws_max(const ts_drafter* d, int Pmax, float T) {
  return make_plan(d, std::max(Pmax, 1), T, TS_SAMPLER_GUMBEL, false, true).bytes;
}

void launch_eval(const ts_drafter* d, const ExpandParams& p, const Plan& pl, hipStream_t s) {
  const dim3 grid(pl.S8 * pl.n_pgroups), block(64 * pl.wpg);
  const bool z = p.z_out != nullptr;
  const int mode = pl.mode | (p.need_T && pl.mode != kModeGreedy ? kModeNeedT : 0);
  if (d->dtype == TS_BF16) {
    switch (pl.ks) {
      case 1: launch_eval_t<uint16_t, 1>(p, pl.NB, mode, z, pl.path, grid, block, s); break;
      case 2: launch_eval_t<uint16_t, 2>(p, pl.NB, mode, z, pl.path, grid, block, s); break;
      case 4: launch_eval_t<uint16_t, 4>(p, pl.NB, mode, z, pl.path, grid, block, s); break;
      default: launch_eval_t<uint16_t, 8>(p, pl.NB, mode, z, pl.path, grid, block, s); break;
    }
  } else {
    switch (pl.ks) {
      case 4: launch_eval_t<float, 4>(p, pl.NB, mode, z, pl.path, grid, block, s); break;
      case 8: launch_eval_t<float, 8>(p, pl.NB, mode, z, pl.path, grid, block, s); break;
      default: launch_eval_t<float, 16>(p, pl.NB, mode, z, pl.path, grid, block, s); break;
    }
  }
}

void launch_merge(const ts_drafter* d, const MergeParams& p, const Plan& pl, hipStream_t s) {
  // sequential draws: one parent per workgroup of two waves.  Otherwise one
  // parent per wave, or per workgroup of kCoopWaves for few parents; where
  // the device holds the count that kernel takes either form by it, and the
  // grid covers both.
  const bool seq = pl.mode == kModeSeq;
  const bool coop = !seq && (p.P_dev || p.P <= coop_parents(pl.mode));
  const int waves = seq ? 2 : coop ? kCoopWaves : 4;
  const int groups = seq ? p.P : std::max((p.P + waves - 1) / waves, coop ? std::min(p.P, coop_parents(pl.mode)) : 0);
  const dim3 grid(groups), block(64 * waves);
  if (d->dtype == TS_BF16) {
    switch (pl.ks) {
      case 1: launch_merge_t<uint16_t, 1>(p, pl.mode, coop, grid, block, s); break;
      case 2: launch_merge_t<uint16_t, 2>(p, pl.mode, coop, grid, block, s); break;
      case 4: launch_merge_t<uint16_t, 4>(p, pl.mode, coop, grid, block, s); break;
      default: launch_merge_t<uint16_t, 8>(p, pl.mode, coop, grid, block, s); break;
    }
  } else {
    switch (pl.ks) {
      case 4: launch_merge_t<float, 4>(p, pl.mode, coop, grid, block, s); break;
      case 8: launch_merge_t<float, 8>(p, pl.mode, coop, grid, block, s); break;
      default: launch_merge_t<float, 16>(p, pl.mode, coop, grid, block, s); break;
    }
  }
}

// z_out: the logits are stored there and nothing is kept in ws (null).
ExpandParams eval_params(const ts_drafter* d, const ts_parent* parents, int P, float T, uint64_t seed,
                         const Plan& pl, char* ws, float* z_out) {
  ExpandParams p{};
  p.U = d->U; p.E = d->E; p.W2 = d->W2;
  p.R = d->R; p.D = d->D; p.V = d->V; p.r = d->r;
  p.parents = parents;
  p.P = P;
  p.cm = pl.cm; p.S = pl.S;
  p.n_pblocks = pl.n_pblocks; p.wpg = pl.wpg; p.n_pgroups = pl.n_pgroups;
  p.cT = T > 0.0f ? kLog2e / T : 0.0f;
  p.need_T = (T > 0.0f && T != 1.0f) ? 1 : 0;
  p.hr = 60.0f / std::max(kLog2e, p.cT);
  p.keys = philox_keys(seed);
  p.z_out = z_out;
  if (z_out) return p;
  p.part_m = reinterpret_cast<float*>(ws + pl.off_m);
  p.part_s0 = reinterpret_cast<float*>(ws + pl.off_s0);
  p.part_sT = pl.sample ? reinterpret_cast<float*>(ws + pl.off_sT) : nullptr;
  p.zs = summary_ptr(ws, pl.off_z);
  if (pl.mode == kModeGumbel) p.gs = summary_ptr(ws, pl.off_g);
  p.nblk = pl.nblk;
  p.blk_ld = pl.blk_ld;
  if (pl.mode == kModeSeq) p.blk = reinterpret_cast<float*>(ws + pl.off_blk);
  return p;
}

// Both passes of one expansion; all arguments already checked.
// P_dev (optional): the device holds the parent count (<= P); P then sizes
// the grids, and the plan takes the most chunks unless P is close to the count
// (tight).
int32_t run_expand(const ts_drafter* d, const ts_parent* parents, int P, ts_calib calib, int k,
                   float T, uint64_t seed, int sampler, const ts_expand_out* out, char* ws,
                   hipStream_t s, const int* P_dev = nullptr, bool even_chunks = false, bool tight = false) {
  if (P == 0) return TS_OK;
  const Plan pl = make_plan(d, P, T, sampler, false, false, P_dev && !tight, even_chunks);
  ExpandParams ep = eval_params(d, parents, P, T, seed, pl, ws, nullptr);
  ep.P_dev = P_dev;
  hipEvent_t* ev = reinterpret_cast<hipEvent_t*>(out->events);
  if (ev) TS_HIP(hipEventRecord(ev[0], s));
  launch_eval(d, ep, pl, s);
  TS_HIP(hipGetLastError());
  if (ev) TS_HIP(hipEventRecord(ev[1], s));
  MergeParams mp{};
  mp.U = d->U; mp.E = d->E; mp.W2 = d->W2;
  mp.R = d->R; mp.D = d->D; mp.V = d->V; mp.r = d->r;
  mp.parents = parents;
  mp.P = P;
  mp.cm = pl.cm; mp.S = pl.S;
  mp.K = k;
  mp.T = T; mp.cT = ep.cT; mp.need_T = ep.need_T;
  mp.calib_a = calib.a; mp.calib_b = calib.b;
  mp.keys = ep.keys;
  mp.part_m = ep.part_m; mp.part_s0 = ep.part_s0; mp.part_sT = ep.part_sT;
  mp.zs = ep.zs;
  mp.gs = ep.gs;
  mp.blk = ep.blk;
  mp.nblk = ep.nblk;
  mp.blk_ld = ep.blk_ld;
  mp.out = *out;
  mp.P_dev = P_dev;
  launch_merge(d, mp, pl, s);
  TS_HIP(hipGetLastError());
  if (ev) TS_HIP(hipEventRecord(ev[2], s));
  return TS_OK;
}

// ---------------------------------------------------------------- tree building

struct Slot {
  float key;
  int depth;       // depth of the child this slot creates
  uint64_t path;   // path id of that child
  int token;
  float log_surv, log_q0, log_qT;
  bool evaluated;  // the child has been evaluated (its own slots are known)
};

// (key desc, child depth asc, child path asc): the pop order of Algorithm 1.
inline bool slot_before(const Slot& a, const Slot& b) {
  if (a.key != b.key) return a.key > b.key;
  if (a.depth != b.depth) return a.depth < b.depth;
  return a.path < b.path;
}

// A slot in the global order of a budget shared by all requests:
// (key desc, request asc, child depth asc, child path asc).
struct GlobalRef {
  float key;
  int q;
  int depth;
  uint64_t path;
};
inline bool global_before(const GlobalRef& a, const GlobalRef& b) {
  if (a.key != b.key) return a.key > b.key;
  if (a.q != b.q) return a.q < b.q;
  if (a.depth != b.depth) return a.depth < b.depth;
  return a.path < b.path;
}

// A tree in the ts_tree layout packed into one block (device staging and
// its host copy): n [R], evals [R], err, then token, parent, depth, rank
// [R][cap] int32, path [R][cap] uint64, log_surv, log_q0, log_qT, key
// [R][cap] float.
struct TreeBlock {
  size_t n, evals, err, token, parent, depth, rank, path, log_surv, log_q0, log_qT, key, bytes;
};

TreeBlock tree_block(int R, int cap) {
  TreeBlock t{};
  const size_t rc = (size_t)R * cap;
  size_t o = 0;
  t.n = o; o += align256((size_t)R * 4);
  t.evals = o; o += align256((size_t)R * 4);
  t.err = o; o += 256;
  t.token = o; o += align256(rc * 4);
  t.parent = o; o += align256(rc * 4);
  t.depth = o; o += align256(rc * 4);
  t.rank = o; o += align256(rc * 4);
  t.path = o; o += align256(rc * 8);
  t.log_surv = o; o += align256(rc * 4);
  t.log_q0 = o; o += align256(rc * 4);
  t.log_qT = o; o += align256(rc * 4);
  t.key = o; o += align256(rc * 4);
  t.bytes = o;
  return t;
}

struct BuildLayout {
  size_t off_par, off_out, off_exp;
  // device-resident waves
  size_t off_par2, off_list, off_lsize, off_evals, off_pcount, off_span, off_anchor, off_ltheta;
  size_t bytes;
  int Pmax;
};

BuildLayout build_layout(const ts_drafter* d, int N, int K, float T) {
  BuildLayout b{};
  const int R = d->R;
  b.Pmax = R * std::max(N, 1);
  const size_t pk = align256((size_t)b.Pmax * K * 4);
  size_t o = 0;
  b.off_par = o; o += align256((size_t)b.Pmax * sizeof(ts_parent));
  b.off_out = o; o += 5 * pk;  // child token, log q0, log qT, log S, key: [P][K] each, packed
  b.off_exp = o; o += expand_ws_max(d, b.Pmax, T);
  b.off_par2 = o; o += align256((size_t)b.Pmax * sizeof(ts_parent));
  b.off_list = o; o += align256((size_t)R * std::max(N, 1) * sizeof(WaveSlot));
  b.off_lsize = o; o += align256((size_t)R * 4);
  b.off_evals = o; o += align256((size_t)R * 4);
  b.off_pcount = o; o += align256((size_t)(d->D + 2) * 8);
  b.off_span = o; o += 2 * align256((size_t)R * sizeof(WaveSpan));
  b.off_anchor = o; o += align256((size_t)R * 4);
  b.off_ltheta = o; o += align256((size_t)R * 4);
  b.bytes = o;
  return b;
}

// The waves run on the device when the per-request lists fit the control
// kernel and no budget is shared across requests.
bool device_waves(int N, int K, int budget) {
  return N >= 1 && budget <= 0 && N <= kWaveMaxN && std::max(1, N - 1) * K <= kWaveMaxNew;
}

WaveTreeOut tree_out_of(const ts_tree* t) {
  WaveTreeOut o{};
  o.cap = t->cap;
  o.n = t->n; o.token = t->token; o.parent = t->parent; o.depth = t->depth; o.rank = t->rank;
  o.path = t->path; o.log_surv = t->log_surv; o.log_q0 = t->log_q0; o.log_qT = t->log_qT;
  o.key = t->key; o.evals = t->evals;
  return o;
}

// ts_build_tree with the waves on the device (no budget; N, K within the
// control kernel's limits).  Wave w + 1 is queued before the host learns
// its size (its kernels read the size the control step wrote), so the GPU
// never waits for the host between waves; the host reads each wave's size
// from the pinned word the control step writes and stops queueing at the
// first empty wave.
int32_t build_tree_device(const ts_drafter* d, const int32_t* anchor, const std::vector<float>& log_theta,
                          int N, int K, ts_calib calib, float T, uint64_t seed, int sampler, ts_tree* out,
                          const ts_tree* device_out, char* ws, const BuildLayout& bl, hipStream_t s) {
  const int R = d->R, D = d->D, cap = out->cap;
  const TreeBlock tb = tree_block(R, cap);
  char* hs = nullptr;
  const size_t hs_up = align256((size_t)R * 8), hs_cnt = align256((size_t)(D + 2) * 4);
  int32_t rc = host_stage(hs_up + hs_cnt + tb.bytes, &hs);
  if (rc != TS_OK) return rc;
  // roots and thresholds stay in the pinned buffer: the init kernel reads them
  std::memcpy(hs, anchor, (size_t)R * 4);
  std::memcpy(hs + (size_t)R * 4, log_theta.data(), (size_t)R * 4);
  volatile int32_t* hcnt = reinterpret_cast<volatile int32_t*>(hs + hs_up);
  char* htree = hs + hs_up + hs_cnt;

  WaveParams wp{};
  wp.R = R; wp.N = N; wp.K = K; wp.D = D;
  wp.anchor = reinterpret_cast<const int32_t*>(ws + bl.off_anchor);
  wp.log_theta = reinterpret_cast<const float*>(ws + bl.off_ltheta);
  wp.anchor_host = reinterpret_cast<const int32_t*>(hs);
  wp.log_theta_host = reinterpret_cast<const float*>(hs + (size_t)R * 4);
  wp.anchor_w = reinterpret_cast<int32_t*>(ws + bl.off_anchor);
  wp.log_theta_w = reinterpret_cast<float*>(ws + bl.off_ltheta);
  wp.host_count = hcnt;
  wp.list = reinterpret_cast<WaveSlot*>(ws + bl.off_list);
  wp.lsize = reinterpret_cast<int*>(ws + bl.off_lsize);
  wp.evals = reinterpret_cast<int*>(ws + bl.off_evals);
  wp.pcount = reinterpret_cast<uint64_t*>(ws + bl.off_pcount);
  wp.par[0] = reinterpret_cast<ts_parent*>(ws + bl.off_par);
  wp.par[1] = reinterpret_cast<ts_parent*>(ws + bl.off_par2);
  wp.span[0] = reinterpret_cast<WaveSpan*>(ws + bl.off_span);
  wp.span[1] = reinterpret_cast<WaveSpan*>(ws + bl.off_span + align256((size_t)R * sizeof(WaveSpan)));
  const size_t nk = (size_t)bl.Pmax * K;
  char* dout = ws + bl.off_out;
  ts_expand_out eo{};
  eo.child_token = reinterpret_cast<int32_t*>(dout);
  eo.child_log_q0 = reinterpret_cast<float*>(dout + align256(nk * 4));
  eo.child_log_qT = reinterpret_cast<float*>(dout + 2 * align256(nk * 4));
  eo.child_log_surv = reinterpret_cast<float*>(dout + 3 * align256(nk * 4));
  eo.slot_key = reinterpret_cast<float*>(dout + 4 * align256(nk * 4));
  wp.child_token = eo.child_token;
  wp.child_log_q0 = eo.child_log_q0;
  wp.child_log_qT = eo.child_log_qT;
  wp.child_log_surv = eo.child_log_surv;
  wp.slot_key = eo.slot_key;
  DrainOnError drain{s};
  launch_wave_init(wp, s);
  TS_HIP(hipGetLastError());

  // A chain (K = 1) has as many parents as the wave before until a price stops
  // it: its waves take the plan of that count.  With the most chunks, 256 requests
  // at V = 151936, r = 128 made 1024 workgroups where 768 fit the chip (16 waves of
  // sequential draws, T = 1: 1064 us, so 918; 198 chunks of rounded-up length 1061),
  // 600 at V = 64000, r = 64 1027 and 873.
  const bool tight = K == 1;
  // queue wave w: expansion of par[w & 1] (at most Pub parents; the device
  // holds the count) and the control step, which also writes the next
  // wave's size into hcnt[w + 1] (pinned, -1 until then).  The host polls
  // that word: an event recorded between the waves' kernels would hold the
  // next kernel back by about 6 us on the device.
  for (int i = 0; i < D + 2; ++i) hcnt[i] = -1;
  auto queue_wave = [&](int w, int Pub) -> int32_t {
    int32_t r = run_expand(d, wp.par[w & 1], Pub, calib, K, T, seed, sampler, &eo, ws + bl.off_exp, s,
                           reinterpret_cast<const int*>(wp.pcount + w), false, tight);
    if (r != TS_OK) return r;
    launch_wave_control(wp, w, s);
    TS_HIP(hipGetLastError());
    return TS_OK;
  };
  // the size of wave i from its word.  After 20 ms the wait also asks the
  // stream (a stream query enqueues a marker, which would hold the next
  // kernel back like an event): one that has drained or failed without
  // writing the word ends it
  auto wave_size = [&](int i, int* out_n) -> int32_t {
    const auto t0 = std::chrono::steady_clock::now();
    for (unsigned n = 1;; ++n) {
      const int v = hcnt[i];
      if (v >= 0) {
        *out_n = v;
        return TS_OK;
      }
      if ((n & 4095) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(20)) {
        const hipError_t q = hipStreamQuery(s);
        if (q != hipSuccess && q != hipErrorNotReady) return fail(TS_EHIP, "HIP error %d while waiting for wave %d", (int)q, i);
        if (q == hipSuccess && hcnt[i] < 0) return fail(TS_EINTERNAL, "wave %d ended without its size", i);
      }
    }
  };
  const int per_req = std::max(0, N - 1);  // children a request can send to the next wave
  int Pw = R;                              // size of wave w, known
  if ((rc = queue_wave(0, R)) != TS_OK) return rc;
  for (int w = 0;; ++w) {
    const long long ub = std::min<long long>((long long)Pw * K, (long long)R * per_req);
    if (w + 1 < D && ub > 0)
      if ((rc = queue_wave(w + 1, (int)ub)) != TS_OK) return rc;
    int Pn = 0;
    if ((rc = wave_size(w + 1, &Pn)) != TS_OK) return rc;
    if (Pn <= 0 || w + 1 >= D || ub == 0) break;
    if (Pn > ub) return fail(TS_EINTERNAL, "wave %d has %d parents, more than the bound %lld", w + 1, Pn, ub);
    Pw = Pn;
  }

  // the trees: written straight into the pinned block, and into the caller's
  // device arrays
  char* dt = htree;
  *reinterpret_cast<volatile int32_t*>(htree + tb.err) = 0;
  ts_tree st{};
  st.R = R; st.cap = cap;
  st.n = reinterpret_cast<int32_t*>(dt + tb.n);
  st.evals = reinterpret_cast<int32_t*>(dt + tb.evals);
  st.token = reinterpret_cast<int32_t*>(dt + tb.token);
  st.parent = reinterpret_cast<int32_t*>(dt + tb.parent);
  st.depth = reinterpret_cast<int32_t*>(dt + tb.depth);
  st.rank = reinterpret_cast<int32_t*>(dt + tb.rank);
  st.path = reinterpret_cast<uint64_t*>(dt + tb.path);
  st.log_surv = reinterpret_cast<float*>(dt + tb.log_surv);
  st.log_q0 = reinterpret_cast<float*>(dt + tb.log_q0);
  st.log_qT = reinterpret_cast<float*>(dt + tb.log_qT);
  st.key = reinterpret_cast<float*>(dt + tb.key);
  WaveTreeOut ho = tree_out_of(&st);
  ho.err = reinterpret_cast<int32_t*>(htree + tb.err);
  // one launch writes the host's copy and, when given, the device copy
  launch_wave_tree(wp, ho, device_out ? tree_out_of(device_out) : WaveTreeOut{}, s);
  TS_HIP(hipGetLastError());
  TS_HIP(hipStreamSynchronize(s));
  if (*reinterpret_cast<const volatile int32_t*>(htree + tb.err) != 0)
    return fail(TS_EINTERNAL, "a tree slot has no materialised parent");
  const size_t rcn = (size_t)R * cap;
  std::memcpy(out->n, htree + tb.n, (size_t)R * 4);
  if (out->evals) std::memcpy(out->evals, htree + tb.evals, (size_t)R * 4);
  std::memcpy(out->token, htree + tb.token, rcn * 4);
  std::memcpy(out->parent, htree + tb.parent, rcn * 4);
  std::memcpy(out->depth, htree + tb.depth, rcn * 4);
  std::memcpy(out->rank, htree + tb.rank, rcn * 4);
  std::memcpy(out->path, htree + tb.path, rcn * 8);
  std::memcpy(out->log_surv, htree + tb.log_surv, rcn * 4);
  std::memcpy(out->log_q0, htree + tb.log_q0, rcn * 4);
  std::memcpy(out->log_qT, htree + tb.log_qT, rcn * 4);
  std::memcpy(out->key, htree + tb.key, rcn * 4);
  drain.armed = false;
  return TS_OK;
}

// The children of every tree node, in creation order, as flat per-request
// lists: node p of request q has count(q, p) children starting at
// first(q, p).  The arrays are kept per thread and reused, so indexing a
// tree allocates nothing once they have grown to its size.
struct KidIndex {
  std::vector<int> off;   // [R][cap + 1]: start of node p's children in list
  std::vector<int> list;  // [R][cap]: child ids, grouped by parent
  int cap = 0;
  const int* first(int q, int p) const { return list.data() + (size_t)q * cap + off[(size_t)q * (cap + 1) + p]; }
  int count(int q, int p) const {
    const size_t o = (size_t)q * (cap + 1) + p;
    return off[o + 1] - off[o];
  }
};

// Builds the index of a tree whose parents were checked (0 <= parent[i] < i).
const KidIndex& kid_index(const ts_tree* t) {
  thread_local KidIndex k;
  const int R = t->R, cap = t->cap;
  k.cap = cap;
  k.off.resize((size_t)R * (cap + 1));
  k.list.resize((size_t)R * cap);
  for (int q = 0; q < R; ++q) {
    const int n = t->n[q];
    int* off = k.off.data() + (size_t)q * (cap + 1);  // only entries 0 .. n + 1 are ever read
    std::fill(off, off + n + 2, 0);
    const int32_t* par = t->parent + (size_t)q * cap;
    for (int i = 1; i <= n; ++i) ++off[par[i] + 1];
    for (int p = 0; p <= n; ++p) off[p + 1] += off[p];
    // fill in increasing id order, which is creation order; off[p] ends at
    // the start of node p + 1 and is moved back afterwards
    int* list = k.list.data() + (size_t)q * cap;
    for (int i = 1; i <= n; ++i) list[off[par[i]]++] = i;
    for (int p = n + 1; p > 0; --p) off[p] = off[p - 1];
    off[0] = 0;
  }
  return k;
}

// Where the nodes of a round are among its items (kNextHost: not there), by
// request * cap + node.  The array is kept per thread: a verification sets and
// clears the few that it uses.
class NodeMarks {
 public:
  explicit NodeMarks(size_t n) : at_(array()) {
    if (at_.size() < n) at_.resize(n, kNextHost);
  }
  ~NodeMarks() { clear(); }
  int operator[](size_t o) const { return at_[o]; }
  void set(size_t o, int v) {
    set_.push_back(o);
    at_[o] = v;
  }
  void clear() {
    for (size_t o : set_) at_[o] = kNextHost;
    set_.clear();
  }

 private:
  static std::vector<int>& array() {
    thread_local std::vector<int> at;
    return at;
  }
  std::vector<int>& at_;
  std::vector<size_t> set_;
};

struct VerifyLayout {
  size_t off_pa, off_zp, off_bp, off_cst, off_rec, off_sync;
  // the logit rows of a round's nodes, the parents they are recomputed from
  // and the nodes' items and children (last: their count follows the workspace)
  size_t off_z, off_par, off_items;
  int zrows, nodes;
  size_t bytes;
  int max_chunks;
};

// Vocabulary chunks per item for the T > 0 passes: about 2048 workgroups in
// all, chunks a multiple of kVChunkQuantum tokens.
void verify_chunks(int V, int nitems, int* nchunks, int* chunk) {
  const int max_chunks = (V + kVChunkQuantum - 1) / kVChunkQuantum;
  int nc = std::min(max_chunks, std::max(1, (2048 + nitems - 1) / std::max(nitems, 1)));
  int len = (V + nc - 1) / nc;
  len = ((len + kVChunkQuantum - 1) / kVChunkQuantum) * kVChunkQuantum;
  *chunk = len;
  *nchunks = (V + len - 1) / len;
}

// Launch shape of a level in one launch (register-resident chunks), or ok =
// false when the level's chunks would not all be resident at once.  Chunks
// are at least kVChunkQuantum tokens long (the partial arrays hold that many
// per item) and at most what a workgroup holds.
struct FusedPlan {
  bool ok;
  int cpi, chunk;
};
// Workgroups of a one-launch level that the device holds at once, the most
// such a launch has (its slots beyond them are never used, nor cleared).
long long fused_capacity(bool bf16) { return (long long)std::max(verify_fused_blocks_per_cu(bf16), 0) * device_cus(); }
FusedPlan fused_plan(int V, int nitems, bool bf16) {
  FusedPlan fp{false, 0, 0};
  const long long capacity = fused_capacity(bf16);
  if (nitems < 1 || capacity < 1) return fp;
  const int per_wg = verify_fused_quads(bf16) * kVChunkQuantum;
  const int cpi_min = (V + per_wg - 1) / per_wg;
  if (cpi_min > kFusedMaxCpi || (long long)nitems * cpi_min > std::min<long long>(capacity, kFusedMaxGrid)) return fp;
  const int max_chunks = (V + kVChunkQuantum - 1) / kVChunkQuantum;
  int cpi = (int)std::min<long long>(std::min<long long>(capacity, kFusedMaxGrid) / nitems,
                                     std::min(max_chunks, kFusedMaxChunks));
  cpi = std::max(cpi, cpi_min);
  int chunk = (V + cpi - 1) / cpi;
  chunk = (chunk + 3) / 4 * 4;
  fp.ok = true;
  fp.chunk = chunk;
  fp.cpi = (V + chunk - 1) / chunk;
  return fp;
}

// Slot words of the one-launch levels: kSlotWords per workgroup, for the
// most workgroups a launch over R items can have.
size_t fused_slot_words(int R) {
  return (size_t)kSlotWords * (size_t)std::min<long long>((long long)R * kFusedMaxCpi, kFusedMaxGrid);
}

// Logit rows a round of the T > 0 walk recomputes at most: those of the nodes
// where the walks stand (at most R) and, with them, of nodes below that the
// walks may reach, which a launch then goes on to by itself.  A row costs its
// U row and the logits written, 6 V bytes (bf16), a round more about 35 us
// (a recompute, a launch, the host's turn around), in which the chip moves
// some 150 MB.
constexpr size_t kAheadBytes = 144u << 20;
constexpr int kAheadRows = 4096;
// The first round, after which walks often end, looks ahead only to all the
// nodes with children below the roots together, and only where their bytes are
// few or worth the chance that a walk gets past its root: kRoundBytes stand for
// the round then saved.  ts_verify with the roots alone and with all nodes: 4
// requests of 64 nodes, V = 128256 (some 90 MB, 5 us), walks that end at the root
// 70.0 and 71.6 us, that go on 117.3 and 93.1; 1 request of 64 nodes, V = 151936,
// r = 256 (20 MB) 79.0 and 77.9, 92.3 and 68.7; 64 requests of 64 nodes, V = 65536,
// as many rows as kAheadBytes hold, 103.4 and 140.6, 153.2 and 188.0.
constexpr size_t kRoundBytes = 112u << 20, kFewBytes = 24u << 20;
// Nodes that take the host some 35 us to index.
constexpr size_t kManyNodes = 8192;
int verify_rows(const ts_drafter* d, int cap) {
  const long long nodes = (long long)d->R * std::max(cap - 1, 1);
  const long long ahead = std::min<long long>(kAheadRows, (long long)(kAheadBytes / ((size_t)d->V * 6)));
  return (int)std::max<long long>(d->R, std::min(nodes, ahead));
}

// zrows: logit rows (at least R); a workspace that holds fewer than
// verify_rows takes as many as fit.
VerifyLayout verify_layout(const ts_drafter* d, float T, int zrows) {
  VerifyLayout v{};
  size_t o = 0;
  if (T == 0.0f) {
    o = 256;  // the greedy walk works in the pinned staging buffer; 0 would mean an error
  } else {
    v.max_chunks = (d->V + kVChunkQuantum - 1) / kVChunkQuantum;
    const size_t ic = (size_t)d->R * v.max_chunks;
    v.off_pa = o; o += align256(ic * sizeof(VPartA));
    v.off_zp = o; o += align256(ic * TS_MAX_K * sizeof(double));
    v.off_bp = o; o += align256(ic * sizeof(VBonusPart));
    v.off_cst = o; o += align256((size_t)d->R * sizeof(VConst));
    v.off_rec = o; o += align256((size_t)d->R * TS_MAX_K * sizeof(VRec));
    v.off_sync = o; o += align256(fused_slot_words(d->R) * 8 + 16);
    v.zrows = zrows;
    v.nodes = zrows + d->R;  // and the walks that stand at nodes without children
    v.off_z = o; o += align256((size_t)zrows * d->V * 4);
    v.off_par = o; o += align256((size_t)zrows * sizeof(ts_parent));
    v.off_items = o; o += align256((size_t)v.nodes * (sizeof(VerifyItem) + sizeof(VerifyNext)));
  }
  v.bytes = o;
  return v;
}
VerifyLayout verify_layout_for(const ts_drafter* d, int cap, float T, size_t have) {
  int lo = d->R, hi = verify_rows(d, cap);  // the most rows that fit, at least R
  VerifyLayout v = verify_layout(d, T, hi);
  if (v.bytes <= have || T == 0.0f) return v;
  while (lo < hi) {
    const int mid = lo + (hi - lo + 1) / 2;
    if (verify_layout(d, T, mid).bytes <= have) lo = mid; else hi = mid - 1;
  }
  return verify_layout(d, T, lo);
}

// Waits until every item of a one-launch round has its result words in pinned
// memory.  poll: a round may follow, and polling the words spares it the
// runtime's report of the launch's end (64 requests, V = 100003: 157 us against
// 148).  A last round goes through the runtime at once: the end of the stream
// has to be waited for anyway, and asked for only after the words have arrived
// its report comes on top of the launch (11 requests of one node, V = 6976: 43.8
// us polled, 41.1 so).  *failed: a wait between the launch's workgroups ran out;
// the stream is then idle.  Polling gives up after 20 ms (the work that the
// caller had queued on the stream before counts among them), and the runtime
// then reports a failed launch.
int32_t wait_round(const uint64_t* done, int words, uint32_t epoch, const volatile int32_t* herr, bool poll,
                   hipStream_t s, bool* failed) {
  const auto t0 = std::chrono::steady_clock::now();
  bool slow = !poll;
  int i = 0;
  for (unsigned n = 1; i < words && *herr == 0 && !slow; ++n) {
    const uint64_t w = __atomic_load_n(done + i, __ATOMIC_ACQUIRE);
    if ((uint32_t)(w >> 32) == epoch) {
      ++i;
      continue;
    }
    slow = (n & 1023) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(20);
  }
  *failed = false;
  if (i == words) return TS_OK;
  TS_HIP(hipStreamSynchronize(s));
  *failed = *herr != 0;
  for (; i < words && !*failed; ++i)
    if ((uint32_t)(done[i] >> 32) != epoch) return fail(TS_EINTERNAL, "verification word %d has no result", i);
  return TS_OK;
}

// Host checks shared by ts_expand and ts_expand_noalloc.
int32_t check_expand_args(const ts_drafter* d, const ts_parent* parents, int P, ts_calib calib, int k, float T,
                          int sampler, const ts_expand_out* out) {
  int32_t rc = check_drafter(d);
  if (rc != TS_OK) return rc;
  if ((rc = check_k_T(d, k, T)) != TS_OK) return rc;
  if ((rc = check_sampler(sampler)) != TS_OK) return rc;
  if (P < 0) return fail(TS_EINVAL, "P=%d is negative", P);
  if (P == 0) return TS_OK;
  if (!parents) return fail(TS_EINVAL, "parents is NULL");
  if (!out || !out->child_token || !out->child_log_q0 || !out->child_log_surv || !out->slot_key)
    return fail(TS_EINVAL, "a required output pointer is NULL");
  if (!std::isfinite(calib.a) || !std::isfinite(calib.b)) return fail(TS_EINVAL, "calibration must be finite");
  return TS_OK;
}

int32_t noalloc_scratch(char** out) {
  static std::mutex mu;
  static void* addr[64] = {nullptr};
  int dev = 0;
  TS_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= 64) return fail(TS_EUNSUPPORTED, "device %d beyond the 64 the library tracks", dev);
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    TS_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(TS_EHIP, "hipGetSymbolAddress returned no address for the scratch array");
    addr[dev] = p;
  }
  *out = static_cast<char*>(addr[dev]);
  return TS_OK;
}

}  // namespace
}  // namespace ts

using namespace ts;

extern "C" {

const char* ts_last_error(void) { return g_last_error.c_str(); }

const char* ts_version(void) { return "treespark-mi355x 0.2 (gfx950)"; }

int32_t ts_verify_set_mode(int32_t mode) {
  g_last_error.clear();
  if (mode != TS_VERIFY_AUTO && mode != TS_VERIFY_STAGED) return fail(TS_EINVAL, "unknown verify mode %d", mode);
  thread_state().verify_mode = mode;
  return TS_OK;
}

// Not part of the ABI: the calling thread's limit on the polls of one wait
// between the workgroups of a verification round, for the tests of the way
// back to the per-stage launches (0: every wait gives up at once; negative:
// the default).  Every kernel still runs to its end.
void ts_internal_verify_wait_limit(int32_t polls) { thread_state().wait_limit = polls < 0 ? kFusedSpinLimit : polls; }

int32_t ts_verify_level_counts(int64_t* fused, int64_t* fallbacks, int64_t* staged) {
  g_last_error.clear();
  if (!fused || !fallbacks || !staged) return fail(TS_EINVAL, "an output is NULL");
  const ThreadState& st = thread_state();
  *fused = st.fused_levels;
  *fallbacks = st.fused_fallbacks;
  *staged = st.staged_levels;
  return TS_OK;
}

int32_t ts_release_thread_state(void) {
  g_last_error.clear();
  ThreadState& st = thread_state();
  if (!st.stage) return TS_OK;
  // every stream that used them has been synchronised by its call, but a
  // caller's later work may still reference the staging buffer's contents:
  // wait for the device before freeing anything
  TS_HIP(hipDeviceSynchronize());
  if (st.stage) TS_HIP(hipHostFree(st.stage));
  st.stage = nullptr;
  st.stage_bytes = 0;
  return TS_OK;
}

size_t ts_expand_workspace_size(const ts_drafter* d, int32_t P, int32_t k, float T) {
  (void)k;
  if (check_drafter(d) != TS_OK || P <= 0) return 0;
  return make_plan(d, P, T, TS_SAMPLER_GUMBEL, false, true).bytes;
}

int32_t ts_expand(const ts_drafter* d, const ts_parent* parents, int32_t P, ts_calib calib,
                  int32_t k, float T, uint64_t seed, int32_t sampler, const ts_expand_out* out,
                  void* workspace, size_t workspace_bytes, void* stream) {
  g_last_error.clear();
  int32_t rc = check_expand_args(d, parents, P, calib, k, T, sampler, out);
  if (rc != TS_OK || P == 0) return rc;
  const size_t need = make_plan(d, P, T, TS_SAMPLER_GUMBEL, false, true).bytes;
  if (!workspace || workspace_bytes < need)
    return fail(TS_ENOSPACE, "workspace %zu bytes < %zu needed", workspace_bytes, need);
  return run_expand(d, parents, P, calib, k, T, seed, sampler, out, static_cast<char*>(workspace),
                    static_cast<hipStream_t>(stream));
}

int32_t ts_expand_noalloc(const ts_drafter* d, const ts_parent* parents, int32_t P, ts_calib calib,
                          int32_t k, float T, uint64_t seed, int32_t sampler, const ts_expand_out* out,
                          void* stream) {
  g_last_error.clear();
  int32_t rc = check_expand_args(d, parents, P, calib, k, T, sampler, out);
  if (rc != TS_OK || P == 0) return rc;
  const size_t need = make_plan(d, P, T, sampler, false, false, false, true).bytes;
  if (need > (size_t)TS_NOALLOC_SCRATCH_BYTES)
    return fail(TS_EUNSUPPORTED, "this launch needs %zu bytes of scratch, more than the %u of ts_expand_noalloc",
                need, TS_NOALLOC_SCRATCH_BYTES);
  char* scratch = nullptr;
  if ((rc = noalloc_scratch(&scratch)) != TS_OK) return rc;
  const bool even = make_plan(d, P, T, sampler).bytes > (size_t)TS_NOALLOC_SCRATCH_BYTES;
  return run_expand(d, parents, P, calib, k, T, seed, sampler, out, scratch, static_cast<hipStream_t>(stream), nullptr,
                    even);
}

size_t ts_build_tree_workspace_size(const ts_drafter* d, int32_t N, int32_t K, float T) {
  if (check_drafter(d) != TS_OK || N < 0 || K < 1 || K > TS_MAX_K) return 0;
  return build_layout(d, N, K, T).bytes;
}

int32_t ts_build_tree(const ts_drafter* d, const int32_t* anchor, const float* theta, int32_t N,
                      int32_t budget, int32_t K, ts_calib calib, float T, uint64_t seed,
                      int32_t sampler, ts_tree* out, const ts_tree* device_out, void* workspace,
                      size_t workspace_bytes, void* stream) {
  g_last_error.clear();
  int32_t rc = check_drafter(d);
  if (rc != TS_OK) return rc;
  if ((rc = check_k_T(d, K, T)) != TS_OK) return rc;
  if ((rc = check_sampler(sampler)) != TS_OK) return rc;
  if (N < 0) return fail(TS_EINVAL, "N=%d is negative", N);
  if (!anchor || !theta || !out) return fail(TS_EINVAL, "anchor, theta or out is NULL");
  if (!out->n || !out->token || !out->parent || !out->depth || !out->rank || !out->path ||
      !out->log_surv || !out->log_q0 || !out->log_qT || !out->key)
    return fail(TS_EINVAL, "a tree array is NULL");
  if (out->R != d->R || out->cap < N + 1) return fail(TS_EINVAL, "tree has R=%d cap=%d, need R=%d cap>=%d", out->R, out->cap, d->R, N + 1);
  if (device_out && (device_out->R != out->R || device_out->cap != out->cap || !device_out->n ||
                     !device_out->token || !device_out->parent || !device_out->depth || !device_out->rank ||
                     !device_out->path || !device_out->log_surv || !device_out->log_q0 ||
                     !device_out->log_qT || !device_out->key))
    return fail(TS_EINVAL, "device_out must have the R and cap of out and no NULL array");
  if (!std::isfinite(calib.a) || !std::isfinite(calib.b)) return fail(TS_EINVAL, "calibration must be finite");
  const int R = d->R;
  for (int q = 0; q < R; ++q) {
    if (anchor[q] < 0 || anchor[q] >= d->V) return fail(TS_EINVAL, "anchor[%d]=%d outside [0, V)", q, anchor[q]);
    if (!(theta[q] >= 0.0f) || !std::isfinite(theta[q])) return fail(TS_EINVAL, "theta[%d] must be finite and >= 0", q);
  }
  const BuildLayout bl = build_layout(d, N, K, T);
  if (!workspace || workspace_bytes < bl.bytes)
    return fail(TS_ENOSPACE, "workspace %zu bytes < %zu needed", workspace_bytes, bl.bytes);
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  ts_parent* dpar = reinterpret_cast<ts_parent*>(ws + bl.off_par);
  ts_expand_out eo{};
  char* hs = nullptr;
  const size_t hs_par = align256((size_t)bl.Pmax * sizeof(ts_parent));
  if ((rc = host_stage(hs_par + (size_t)5 * bl.Pmax * K * 4, &hs)) != TS_OK) return rc;

  std::vector<float> log_theta(R);
  for (int q = 0; q < R; ++q) log_theta[q] = theta[q] > 0.0f ? logf(theta[q]) : -INFINITY;
  if (device_waves(N, K, budget))
    return build_tree_device(d, anchor, log_theta, N, K, calib, T, seed, sampler, out, device_out, ws, bl, s);
  DrainOnError drain{s};
  std::vector<std::vector<Slot>> known(R);
  std::vector<ts_parent> frontier;
  std::vector<int32_t> evals(R, 0);
  if (N > 0)
    for (int q = 0; q < R; ++q) frontier.push_back(ts_parent{anchor[q], 0, q, 0.0f, 0});
  while (!frontier.empty()) {
    const int P = (int)frontier.size();
    const size_t nk = (size_t)P * K;
    // this wave's five outputs, packed, so that one copy brings them back
    char* dout = ws + bl.off_out;
    eo.child_token = reinterpret_cast<int32_t*>(dout);
    eo.child_log_q0 = reinterpret_cast<float*>(dout + nk * 4);
    eo.child_log_qT = reinterpret_cast<float*>(dout + nk * 8);
    eo.child_log_surv = reinterpret_cast<float*>(dout + nk * 12);
    eo.slot_key = reinterpret_cast<float*>(dout + nk * 16);
    std::memcpy(hs, frontier.data(), P * sizeof(ts_parent));
    TS_HIP(hipMemcpyAsync(dpar, hs, P * sizeof(ts_parent), hipMemcpyHostToDevice, s));
    rc = run_expand(d, dpar, P, calib, K, T, seed, sampler, &eo, ws + bl.off_exp, s);
    if (rc != TS_OK) return rc;
    char* hout = hs + hs_par;
    TS_HIP(hipMemcpyAsync(hout, dout, nk * 20, hipMemcpyDeviceToHost, s));
    const int32_t* h_tok = reinterpret_cast<const int32_t*>(hout);
    const float* h_q0 = reinterpret_cast<const float*>(hout + nk * 4);
    const float* h_qT = reinterpret_cast<const float*>(hout + nk * 8);
    const float* h_ls = reinterpret_cast<const float*>(hout + nk * 12);
    const float* h_key = reinterpret_cast<const float*>(hout + nk * 16);
    TS_HIP(hipStreamSynchronize(s));
    for (int i = 0; i < P; ++i) {
      const ts_parent& par = frontier[i];
      ++evals[par.request];
      for (int j = 0; j < K; ++j) {
        const size_t o = (size_t)i * K + j;
        Slot sl;
        sl.key = h_key[o];
        sl.depth = par.depth + 1;
        sl.path = par.path | ((uint64_t)j << (4 * par.depth));
        sl.token = h_tok[o];
        sl.log_surv = h_ls[o];
        sl.log_q0 = h_q0[o];
        sl.log_qT = h_qT[o];
        sl.evaluated = false;
        known[par.request].push_back(sl);
      }
    }
    // Next wave: children of the slots that can still be among the tree's
    // nodes: key >= log(theta_q), strictly above the request's N-th such slot
    // and, under a global budget B, strictly above the B-th best of all
    // requests' top-N slots in the global order (key desc, request asc,
    // depth asc, path asc).  Any node of the final trees descends from such
    // a child, because a slot's key never exceeds the key of the slot whose
    // pop created it.
    frontier.clear();
    std::vector<Slot> nth(R);
    std::vector<char> have_n(R, 0);
    std::vector<GlobalRef> pool;
    for (int q = 0; q < R; ++q) {
      std::vector<Slot> el;
      for (const Slot& sl : known[q])
        if (sl.key >= log_theta[q]) el.push_back(sl);
      if (N > 0 && (int)el.size() >= N) {
        std::nth_element(el.begin(), el.begin() + (N - 1), el.end(), slot_before);
        nth[q] = el[N - 1];
        have_n[q] = 1;
      }
      if (budget > 0) {
        const int take = std::min<int>(N, (int)el.size());
        if (take < (int)el.size()) el.resize(take);  // nth_element left the top N first
        for (const Slot& sl : el) pool.push_back(GlobalRef{sl.key, q, sl.depth, sl.path});
      }
    }
    bool have_g = false;
    GlobalRef gth{};
    if (budget > 0 && (int)pool.size() >= budget) {
      std::nth_element(pool.begin(), pool.begin() + (budget - 1), pool.end(), global_before);
      gth = pool[budget - 1];
      have_g = true;
    }
    for (int q = 0; q < R; ++q) {
      const size_t first = frontier.size();
      for (Slot& sl : known[q]) {
        if (sl.evaluated || sl.depth >= d->D || sl.key < log_theta[q]) continue;
        if (have_n[q] && !slot_before(sl, nth[q])) continue;
        if (have_g && !global_before(GlobalRef{sl.key, q, sl.depth, sl.path}, gth)) continue;
        sl.evaluated = true;
        frontier.push_back(ts_parent{sl.token, sl.depth, q, sl.log_surv, sl.path});
      }
      std::sort(frontier.begin() + first, frontier.end(),
                [](const ts_parent& a, const ts_parent& b) { return a.depth < b.depth; });
    }
  }
  // The trees: each request's slots in pop order, at most N, stopping below
  // log(theta_q); under a global budget, the best B of those in the global order.
  std::vector<int> take(R, 0);
  {
    std::vector<GlobalRef> pool;
    for (int q = 0; q < R; ++q) {
      std::vector<Slot>& ks = known[q];
      std::sort(ks.begin(), ks.end(), slot_before);
      int t = 0;
      while (t < (int)ks.size() && t < N && ks[t].key >= log_theta[q]) ++t;
      take[q] = t;
      if (budget > 0)
        for (int i = 0; i < t; ++i) pool.push_back(GlobalRef{ks[i].key, q, ks[i].depth, ks[i].path});
    }
    if (budget > 0 && (int)pool.size() > budget) {
      std::nth_element(pool.begin(), pool.begin() + budget, pool.end(), global_before);
      std::fill(take.begin(), take.end(), 0);
      for (int i = 0; i < budget; ++i) ++take[pool[i].q];  // a prefix of each request's order
    }
  }
  const int cap = out->cap;
  for (int q = 0; q < R; ++q) {
    std::vector<Slot>& ks = known[q];
    const size_t b = (size_t)q * cap;
    out->token[b] = anchor[q];
    out->parent[b] = -1;
    out->depth[b] = 0;
    out->rank[b] = 0;
    out->path[b] = 0;
    out->log_surv[b] = 0.0f;
    out->log_q0[b] = 0.0f;
    out->log_qT[b] = NAN;
    out->key[b] = 0.0f;
    std::unordered_map<uint64_t, int> node_of[TS_MAX_D + 1];
    node_of[0][0] = 0;
    int n = 0;
    for (const Slot& sl : ks) {
      if (n >= take[q]) break;
      const int pd = sl.depth - 1;
      const uint64_t ppath = sl.path & ((pd == 0) ? 0ull : ((1ull << (4 * pd)) - 1ull));
      const auto it = node_of[pd].find(ppath);
      if (it == node_of[pd].end()) return fail(TS_EINTERNAL, "request %d: slot without a materialised parent", q);
      const int c = ++n;
      out->token[b + c] = sl.token;
      out->parent[b + c] = it->second;
      out->depth[b + c] = sl.depth;
      out->rank[b + c] = (int)((sl.path >> (4 * pd)) & 15ull) + 1;
      out->path[b + c] = sl.path;
      out->log_surv[b + c] = sl.log_surv;
      out->log_q0[b + c] = sl.log_q0;
      out->log_qT[b + c] = sl.log_qT;
      out->key[b + c] = sl.key;
      node_of[sl.depth][sl.path] = c;
    }
    out->n[q] = n;
    if (out->evals) out->evals[q] = evals[q];
    for (int c = n + 1; c < cap; ++c) {  // rows past the tree, as the device waves leave them
      out->token[b + c] = -1;
      out->parent[b + c] = -1;
      out->depth[b + c] = 0;
      out->rank[b + c] = 0;
      out->path[b + c] = 0;
      out->log_surv[b + c] = NAN;
      out->log_q0[b + c] = NAN;
      out->log_qT[b + c] = NAN;
      out->key[b + c] = NAN;
    }
  }
  if (device_out) {
    const size_t rcn = (size_t)R * cap;
    const hipMemcpyKind h2d = hipMemcpyHostToDevice;
    TS_HIP(hipMemcpyAsync(device_out->n, out->n, (size_t)R * 4, h2d, s));
    if (device_out->evals && out->evals) TS_HIP(hipMemcpyAsync(device_out->evals, out->evals, (size_t)R * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->token, out->token, rcn * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->parent, out->parent, rcn * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->depth, out->depth, rcn * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->rank, out->rank, rcn * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->path, out->path, rcn * 8, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->log_surv, out->log_surv, rcn * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->log_q0, out->log_q0, rcn * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->log_qT, out->log_qT, rcn * 4, h2d, s));
    TS_HIP(hipMemcpyAsync(device_out->key, out->key, rcn * 4, h2d, s));
    TS_HIP(hipStreamSynchronize(s));
  }
  drain.armed = false;
  return TS_OK;
}

size_t ts_verify_workspace_size(const ts_drafter* d, int32_t cap, float T) {
  if (check_drafter(d) != TS_OK || cap < 1 || !(T >= 0.0f)) return 0;
  return verify_layout(d, T, verify_rows(d, cap)).bytes;
}

int32_t ts_verify(const ts_drafter* d, const ts_tree* tree, const void* target, int32_t target_dtype,
                  float T, uint64_t seed, int32_t* path_nodes, int32_t* path_len, int32_t* bonus,
                  void* workspace, size_t workspace_bytes, void* stream) {
  g_last_error.clear();
  int32_t rc = check_drafter(d);
  if (rc != TS_OK) return rc;
  if (!tree || !target || !path_nodes || !path_len || !bonus)
    return fail(TS_EINVAL, "tree, target or an output is NULL");
  if (!tree->n || !tree->token || !tree->parent || !tree->depth || !tree->path)
    return fail(TS_EINVAL, "a tree array is NULL");
  if (tree->R != d->R || tree->cap < 1) return fail(TS_EINVAL, "tree R=%d cap=%d does not match R=%d", tree->R, tree->cap, d->R);
  if (target_dtype != TS_F32 && target_dtype != TS_BF16) return fail(TS_EINVAL, "unknown target dtype %d", target_dtype);
  if (!(T >= 0.0f) || !std::isfinite(T)) return fail(TS_EINVAL, "T must be finite and >= 0");
  const int R = d->R, cap = tree->cap, V = d->V;
  size_t tree_nodes = 0;
  for (int q = 0; q < R; ++q) {
    const int n = tree->n[q];
    if (n < 0 || n >= cap) return fail(TS_EINVAL, "tree n[%d]=%d outside [0, cap)", q, n);
    tree_nodes += n;
    for (int i = 1; i <= n; ++i) {
      const size_t o = (size_t)q * cap + i;
      const int pa = tree->parent[o];
      if (pa < 0 || pa >= i || tree->token[o] < 0 || tree->token[o] >= V ||
          tree->depth[o] != tree->depth[(size_t)q * cap + pa] + 1 || tree->depth[o] > d->D)
        return fail(TS_EINVAL, "tree of request %d is malformed at node %d", q, i);
    }
    if (tree->token[(size_t)q * cap] < 0 || tree->token[(size_t)q * cap] >= V)
      return fail(TS_EINVAL, "root token of request %d outside [0, V)", q);
  }
  const VerifyLayout vl = verify_layout_for(d, cap, T, workspace ? workspace_bytes : 0);
  if (!workspace || workspace_bytes < vl.bytes)
    return fail(TS_ENOSPACE, "workspace %zu bytes < %zu needed", workspace_bytes, vl.bytes);
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);

  DrainOnError drain{s};
  for (int q = 0; q < R; ++q) path_len[q] = 0;

  if (T == 0.0f) {
    // Rounds of one argmax launch each: the rows where the walks stand, and
    // the levels of their descendants that have at most kGreedyBytes each (the
    // walks then go on without another launch).  A launch and its
    // synchronisation cost about 15 us, in which the GPU reads some 70 MB of
    // rows: reading a level of which only some rows are visited is cheaper than
    // a round more up to about that size, reading every row of a large batch is
    // not (64 trees of 64 nodes, V = 151936: 1.3 GB).  64 trees of up to 10
    // nodes, V = 151936 bf16 and V = 100001 f32: with 96 MB for a round's levels
    // together 56.7 and 55.4 us, with 72 MB for each 44.3 and 49.7.
    constexpr size_t kGreedyBytes = 72u << 20, kGreedyRows = 1u << 20;
    const bool bf16 = target_dtype == TS_BF16;
    const size_t row_bytes = (size_t)V * (bf16 ? 2 : 4);
    // All rows of trees that have no more than two levels' bytes are one round's,
    // listed as they stand, and the trees are indexed while the launch runs: many
    // short rows cost the host more than the chip (V = 1024, bf16, 64 trees of 64
    // nodes gathered level by level 51.6 us, so 36.1; 256 of 200 331 and 169).
    const size_t all = tree_nodes + R;
    const bool every = all * row_bytes <= 2 * kGreedyBytes && all <= kGreedyRows;
    const KidIndex* kids_at = every ? nullptr : &kid_index(tree);  // children of every node in creation order
    std::vector<int> cur(R, 0), active(R), rows, known(every ? 0 : (size_t)R * cap, -1), start(every ? R : 0);
    rows.reserve(every ? all : 0);
    for (int q = 0; q < R; ++q) active[q] = q;
    while (!active.empty()) {
      rows.clear();
      for (int q = 0; every && q < R; ++q) {
        start[q] = (int)rows.size();
        for (int i = 0; i <= tree->n[q]; ++i) rows.push_back(q * cap + i);
      }
      for (size_t i = 0; !every && i < active.size(); ++i) rows.push_back(active[i] * cap + cur[active[i]]);
      for (size_t level = 0; !every;) {
        const KidIndex& kids = *kids_at;
        const size_t end = rows.size();
        size_t more = 0;
        for (size_t i = level; i < end; ++i) more += kids.count(rows[i] / cap, rows[i] % cap);
        if (more == 0 || more * row_bytes > kGreedyBytes || end + more > kGreedyRows) break;
        for (size_t i = level; i < end; ++i) {
          const int q = rows[i] / cap, p = rows[i] % cap;
          const int* ch = kids.first(q, p);
          for (int j = 0, m = kids.count(q, p); j < m; ++j) rows.push_back(q * cap + ch[j]);
        }
        level = end;
      }
      const int nrows = (int)rows.size();
      const int nc = verify_argmax_chunks(V, nrows, bf16, 64);
      const size_t hs_rows = align256((size_t)nrows * 4);
      char* hs = nullptr;
      if ((rc = host_stage(hs_rows + (size_t)nrows * nc * sizeof(ArgmaxPart), &hs)) != TS_OK) return rc;
      std::memcpy(hs, rows.data(), (size_t)nrows * 4);
      // the kernel reads the row list from the pinned buffer and writes its parts there
      const ArgmaxPart* part = reinterpret_cast<const ArgmaxPart*>(hs + hs_rows);
      launch_verify_argmax(target, bf16, V, reinterpret_cast<const int*>(hs), nrows, nc,
                           reinterpret_cast<ArgmaxPart*>(hs + hs_rows), s);
      TS_HIP(hipGetLastError());
      for (int i = 0; !every && i < nrows; ++i) known[rows[i]] = i;
      if (!kids_at) kids_at = &kid_index(tree);
      const KidIndex& kids = *kids_at;
      TS_HIP(hipStreamSynchronize(s));
      size_t left = 0;
      for (int q : active) {
        bool done = false;
        for (int i; !done && (i = every ? start[q] + cur[q] : known[(size_t)q * cap + cur[q]]) >= 0;) {
          const ArgmaxPart* pi = part + (size_t)i * nc;
          ArgmaxPart best = pi[0];
          for (int c = 1; c < nc; ++c)
            if (argmax_better(pi[c], best)) best = pi[c];
          const int gtok = best.id;
          int next = -1;
          const int* ch = kids.first(q, cur[q]);
          for (int j = 0, m = kids.count(q, cur[q]); j < m; ++j)
            if (tree->token[(size_t)q * cap + ch[j]] == gtok) { next = ch[j]; break; }
          if (next < 0 || path_len[q] >= TS_MAX_D) {
            bonus[q] = gtok;
            done = true;
          } else {
            path_nodes[(size_t)q * TS_MAX_D + path_len[q]++] = next;
            cur[q] = next;
          }
        }
        if (!done) active[left++] = q;
      }
      active.resize(left);
      for (int i = 0; !every && i < nrows; ++i) known[rows[i]] = -1;  // the parts go with the next round's
    }
    drain.armed = false;
    return TS_OK;
  }

  // T > 0: rounds over the requests still walking.  A round recomputes the
  // logits of the nodes with children where the walks stand, and of as many
  // such nodes below them as fit; then one launch walks every request from
  // node to node until it ends or reaches a node without logits.  (Per-stage
  // launches take one level a round.)  The host goes on as soon as it has seen
  // every item's result in pinned memory.
  float* zbuf = reinterpret_cast<float*>(ws + vl.off_z);
  const PhiloxKeys keys = philox_keys(seed);
  const bool bf16 = target_dtype == TS_BF16;
  std::vector<int> cur(R, 0), active(R);
  for (int q = 0; q < R; ++q) active[q] = q;
  char* hs = nullptr;
  const size_t hs_par = align256((size_t)vl.zrows * sizeof(ts_parent));
  const size_t hs_nodes = align256((size_t)vl.nodes * (sizeof(VerifyItem) + sizeof(VerifyNext)));
  const size_t hs_res = align256((size_t)R * sizeof(VerifyResult));
  const size_t hs_done = align256((size_t)R * kDoneWords * 8);
  if ((rc = host_stage(hs_par + hs_nodes + hs_res + hs_done + 256, &hs)) != TS_OK) return rc;
  ts_parent* hpar = reinterpret_cast<ts_parent*>(hs);
  VerifyItem* hitem = reinterpret_cast<VerifyItem*>(hs + hs_par);  // a round's children records follow its items
  VerifyResult* res = reinterpret_cast<VerifyResult*>(hs + hs_par + hs_nodes);
  uint64_t* done = reinterpret_cast<uint64_t*>(hs + hs_par + hs_nodes + hs_res);
  volatile int32_t* herr = reinterpret_cast<volatile int32_t*>(hs + hs_par + hs_nodes + hs_res + hs_done);
  // the one-launch levels' slots and flag start the call at zero; each
  // level of a launch tags its slot words with an epoch of its own
  uint64_t* dslots = reinterpret_cast<uint64_t*>(ws + vl.off_sync);
  const size_t nslots = std::min<size_t>(fused_slot_words(R), 2 * kSlotWords * fused_capacity(bf16));
  int* derr = reinterpret_cast<int*>(dslots + nslots);
  // cleared before the first launch; before the others the flag alone: a wait
  // can run out beside a walk that still completes, and a flag left over would
  // end the next launch's waits with nothing to tell the host
  void* clear_at = dslots;
  size_t clear = nslots * 8 + 4;
  uint32_t epoch = 1;
  // the rows in hpar and, with them, b bytes of the pinned buffer at h to the
  // device, what has to be cleared, and the rows' logits
  auto queue_rows = [&](int nz, const void* h, void* to, size_t b) -> int32_t {
    launch_verify_stage_in(hpar, ws + vl.off_par, nz * sizeof(ts_parent), clear_at, clear, s, h, to, b);
    TS_HIP(hipGetLastError());
    clear_at = derr;
    clear = 4;
    if (nz == 0) return TS_OK;
    const Plan pl = make_plan(d, nz, T, TS_SAMPLER_GUMBEL, true);
    launch_eval(d, eval_params(d, reinterpret_cast<const ts_parent*>(ws + vl.off_par), nz, T, seed, pl, nullptr, zbuf), pl,
                s);
    TS_HIP(hipGetLastError());
    return TS_OK;
  };
  // Of trees so large that their rows (one for every fourth node, at the least
  // to be expected) are more than a round is worth, or that indexing them takes the
  // host a round's time, the first recompute is queued before that: its rows are
  // the roots of the trees with children (n > 0), in request order.
  const bool roots_first = tree_nodes / 4 * V * 6 > kRoundBytes || tree_nodes > kManyNodes;
  if (roots_first) {
    int nz = 0;
    for (int q = 0; q < R; ++q) {
      const size_t o = (size_t)q * cap;
      if (tree->n[q] > 0) hpar[nz++] = ts_parent{tree->token[o], tree->depth[o], q, 0.0f, tree->path[o]};
    }
    if ((rc = queue_rows(nz, nullptr, nullptr, 0)) != TS_OK) return rc;
  }
  // children of every node in creation order (= draw order)
  const KidIndex& kids = kid_index(tree);
  bool first = true;
  std::vector<int> next;
  std::vector<size_t> nodes;  // request * cap + node
  NodeMarks node_at((size_t)R * cap);
  bool idle = false;  // the stream has been waited for since the last launch
  while (!active.empty()) {
    const int ni = (int)active.size();
    const FusedPlan fp = thread_state().verify_mode == TS_VERIFY_STAGED ? FusedPlan{false, 0, 0}
                                                                          : fused_plan(V, ni, bf16);
    // a launch that goes on to further nodes needs both halves of its slots
    const bool ahead = fp.ok && (size_t)2 * ni * fp.cpi * kSlotWords <= nslots;
    // the round's nodes: where the walks stand, then those below with
    // children, breadth first; the rows of those with children in that order
    nodes.clear();
    int nz = 0;
    const bool queued = first && roots_first;  // (the rows of its nodes)
    auto add_node = [&](int q, int node) {
      const size_t o = (size_t)q * cap + node;
      node_at.set(o, (int)nodes.size());
      nodes.push_back(o);
      if (kids.count(q, node) == 0) return;
      if (!queued) hpar[nz] = ts_parent{tree->token[o], tree->depth[o], q, 0.0f, tree->path[o]};
      ++nz;
    };
    for (int q : active) add_node(q, cur[q]);
    int most = ahead ? vl.zrows : 0;  // rows
    if (queued) {
      most = 0;
    } else if (first && most > 0) {
      // the nodes with children below the roots, and the chance that every walk
      // ends at its root or at a leaf below it, from the draft's estimate of each
      // child's survival (one half where the tree carries none)
      size_t below = 0;
      float stay = 1.0f;
      for (int q = 0; q < R; ++q)
        for (int i = 1; i <= tree->n[q]; ++i) {
          if (kids.count(q, i) == 0) continue;
          ++below;
          const size_t o = (size_t)q * cap + i;
          if (tree->parent[o] != 0) continue;
          const float ls = tree->log_surv ? tree->log_surv[o] : NAN;
          stay *= 1.0f - (ls <= 0.0f ? expf(ls) : 0.5f);
        }
      const double worth = std::max((1.0 - stay) * kRoundBytes, (double)kFewBytes);
      if ((double)below * V * 6 > worth || nz + below > (size_t)most) most = 0;
    }
    for (size_t i = 0; i < nodes.size() && nz < most; ++i) {
      const int q = (int)(nodes[i] / cap), p = (int)(nodes[i] % cap);
      const int* ch = kids.first(q, p);
      for (int j = 0, m = std::min(kids.count(q, p), TS_MAX_K); j < m && nz < most; ++j)
        if (kids.count(q, ch[j]) > 0) add_node(q, ch[j]);
    }
    const int nn = (int)nodes.size();
    // the nodes' items and, after them, their children's records
    int mmax = 0;
    bool open = false;  // a walk can reach a node with children that is not among them
    auto build_items = [&] {
      VerifyNext* hnext = reinterpret_cast<VerifyNext*>(hitem + nn);
      for (int i = 0, z = 0; i < nn; ++i) {
        const int q = (int)(nodes[i] / cap);
        const size_t row = (size_t)q * cap, o = nodes[i];
        VerifyItem it{};
        VerifyNext nx{};
        it.request = q;
        it.node = (int)(nodes[i] % cap);
        it.depth = tree->depth[o];
        it.path = tree->path[o];
        const int* ch = kids.first(q, it.node);
        it.m = std::min(kids.count(q, it.node), TS_MAX_K);
        for (int j = 0; j < it.m; ++j) {
          it.child_tok[j] = tree->token[row + ch[j]];
          nx.child_node[j] = ch[j];
          nx.child_path[j] = tree->path[row + ch[j]];
          nx.child_item[j] = kids.count(q, ch[j]) == 0 ? kNextLeaf : node_at[row + ch[j]];
          open = open || nx.child_item[j] == kNextHost;
        }
        it.zrow = it.m > 0 ? z++ : -1;
        mmax = std::max(mmax, it.m);
        hitem[i] = it;
        hnext[i] = nx;
      }
      node_at.clear();
    };
    VerifyItem* ditems = reinterpret_cast<VerifyItem*>(ws + vl.off_items);
    VerifyNext* dnext = reinterpret_cast<VerifyNext*>(ditems + nn);
    static_assert(sizeof(VerifyItem) % 8 == 0 && sizeof(VerifyNext) % 8 == 0, "aligned one after the other");
    const size_t items_bytes = nn * (sizeof(VerifyItem) + sizeof(VerifyNext));
    // Every workgroup of the recompute reads all of its rows' parents: they
    // are copied to the device first, with the clearing (594 workgroups x 64
    // parents out of pinned memory took it from 22 to 31 us).  The items go with
    // them, a launch less between the recompute and the walk (one request of 5
    // nodes, V = 6000: 47.6 us apart, 44.5 together; 64 requests whose trees have
    // 148 nodes in all, V = 151936: 87.5 and 84.4), unless they are so many that the
    // recompute would wait for the host.
    const bool together = !queued && nn <= 256;
    first = false;
    if (together) build_items();
    if (!queued && (rc = queue_rows(nz, hitem, ditems, together ? items_bytes : 0)) != TS_OK) return rc;
    if (!together) {
      build_items();
      launch_verify_stage_in(hitem, ditems, items_bytes, nullptr, 0, s);
      TS_HIP(hipGetLastError());
    }
    VerifyPass vp{};
    vp.target = target;
    vp.cap = cap;
    vp.V = V;
    vp.items = ditems;
    vp.nitems = ni;
    vp.zbuf = zbuf;
    vp.c = kLog2e / T;
    vp.keys = keys;
    verify_chunks(V, ni, &vp.nchunks, &vp.chunk);
    vp.pa = reinterpret_cast<VPartA*>(ws + vl.off_pa);
    vp.zp = reinterpret_cast<double*>(ws + vl.off_zp);
    vp.bp = reinterpret_cast<VBonusPart*>(ws + vl.off_bp);
    vp.consts = reinterpret_cast<VConst*>(ws + vl.off_cst);
    vp.recs = reinterpret_cast<VRec*>(ws + vl.off_rec);
    vp.results = res;  // pinned: the resolve kernel writes it
    bool staged = !fp.ok;
    if (fp.ok) {
      // one launch for the round; a wait that ran out (some workgroup was
      // not resident) sends its first level through the per-stage launches
      VerifyPass fvp = vp;
      fvp.nchunks = fp.cpi;
      fvp.chunk = fp.chunk;
      VFused f{};
      f.cpi = fp.cpi;
      f.chunk = fp.chunk;
      f.slots = dslots;
      f.epoch = epoch;
      f.err = derr;
      f.herr = const_cast<int32_t*>(herr);
      f.spin_limit = thread_state().wait_limit;
      f.next = dnext;
      f.done = done;
      std::fill(done, done + (size_t)ni * kDoneWords, 0ull);
      *herr = 0;
      launch_verify_fused(fvp, f, bf16, s);
      TS_HIP(hipGetLastError());
      bool failed = false;
      idle = !open;
      if ((rc = wait_round(done, ni * kDoneWords, epoch, herr, open, s, &failed)) != TS_OK) return rc;
      epoch += TS_MAX_D + 1;  // a walk's levels, and the leaf it ends at
      if (failed) {
        ++thread_state().fused_levels;
        ++thread_state().fused_fallbacks;
        staged = true;
      }
    } else {
      ++thread_state().staged_levels;
    }
    if (staged) {
      launch_verify_level(vp, bf16, mmax, s);
      TS_HIP(hipGetLastError());
      TS_HIP(hipStreamSynchronize(s));
      idle = true;
    }
    next.clear();
    int levels = 0;
    for (int i = 0; i < ni; ++i) {
      const int q = active[i];
      int accepted, b;
      uint64_t digits = 0;
      bool ended;
      if (staged) {
        accepted = res[i].accepted > 0 ? 1 : 0;
        digits = (uint64_t)(accepted ? res[i].accepted - 1 : 0);
        b = res[i].bonus;
        ended = !accepted;
      } else {
        const uint64_t* w = done + (size_t)i * kDoneWords;
        const uint32_t state = (uint32_t)w[kDoneState];
        accepted = (int)(state & 255u);
        ended = (state & kDoneEnded) != 0;
        digits = (uint64_t)(uint32_t)w[kDonePath] | ((uint64_t)(uint32_t)w[kDonePath + 1] << 32);
        b = (int32_t)(uint32_t)w[kDoneBonus];
        // the accepted children's levels and that of the node whose children were all rejected
        levels = std::max(levels, std::max(accepted + (ended && !(state & kDoneLeaf) ? 1 : 0), 1));
      }
      for (int l = 0; l < accepted; ++l) {
        if (path_len[q] >= TS_MAX_D) {
          ended = true;
          break;
        }
        const int c = kids.first(q, cur[q])[(digits >> (4 * l)) & 15];
        path_nodes[(size_t)q * TS_MAX_D + path_len[q]++] = c;
        cur[q] = c;
      }
      bonus[q] = b;
      if (!ended) next.push_back(q);
    }
    if (!staged) thread_state().fused_levels += levels;
    active.swap(next);
  }
  if (!idle) TS_HIP(hipStreamSynchronize(s));
  drain.armed = false;
  return TS_OK;
}

int32_t ts_ladder_lookup(const ts_ladder_rung* rungs, int32_t n, int32_t bs, float T, int32_t K,
                         int32_t N, int32_t block_len, ts_round_policy* out) {
  g_last_error.clear();
  if (!rungs || !out) return fail(TS_EINVAL, "rungs or out is NULL");
  if (n < 1) return fail(TS_EINVAL, "the ladder has no rungs");
  if (bs < 1) return fail(TS_EINVAL, "batch size %d < 1", bs);
  if (!(T >= 0.0f) || !std::isfinite(T)) return fail(TS_EINVAL, "T must be finite and >= 0");
  if (K < 1 || K > TS_MAX_K) return fail(TS_EINVAL, "K=%d outside [1, %d]", K, TS_MAX_K);
  if (N < 0) return fail(TS_EINVAL, "N=%d is negative", N);
  if (block_len < 1 || block_len > TS_MAX_D) return fail(TS_EINVAL, "block length %d outside [1, %d]", block_len, TS_MAX_D);
  // nearest tabulated temperature, ties to the lower one
  float best_T = rungs[0].T;
  for (int i = 1; i < n; ++i) {
    const float d = std::fabs(rungs[i].T - T), db = std::fabs(best_T - T);
    if (d < db || (d == db && rungs[i].T < best_T)) best_T = rungs[i].T;
  }
  int pick = -1, widest = -1;
  for (int i = 0; i < n; ++i) {
    if (rungs[i].T != best_T) continue;
    if (widest < 0 || rungs[i].bs_max > rungs[widest].bs_max) widest = i;
    if (rungs[i].bs_max >= bs && (pick < 0 || rungs[i].bs_max < rungs[pick].bs_max)) pick = i;
  }
  if (pick < 0) pick = widest;
  if (rungs[pick].theta < 0.0f) {
    *out = ts_round_policy{0.0f, 1, block_len, 1};
  } else {
    *out = ts_round_policy{rungs[pick].theta, K, N, 0};
  }
  return TS_OK;
}

int32_t ts_ladder_default(ts_ladder_rung* rungs, int32_t cap) {
  static const ts_ladder_rung kLadder[] = {
      {4, 0.0f, 0.02f}, {8, 0.0f, 0.05f}, {INT32_MAX, 0.0f, 0.15f},
      {8, 0.5f, 0.05f}, {INT32_MAX, 0.5f, -1.0f},
      {8, 1.0f, 0.05f}, {INT32_MAX, 1.0f, -1.0f}};
  const int32_t count = (int32_t)(sizeof(kLadder) / sizeof(kLadder[0]));
  for (int32_t i = 0; rungs && i < cap && i < count; ++i) rungs[i] = kLadder[i];
  return count;
}

// ---------------------------------------------------------------- calibration

namespace {
// pieces a target row is cut into for its argmax: the parts go through the
// workspace, whose size does not know V
constexpr int kCalibChunks = 8;
struct CalibLayout {
  size_t parent, token, log_q0, n, rows, off, upload, greedy, part, bytes;
};
CalibLayout calib_layout(int R, int cap) {
  CalibLayout c{};
  const size_t rc = (size_t)R * cap;
  size_t o = 0;
  c.parent = o; o += align256(rc * 4);
  c.token = o; o += align256(rc * 4);
  c.log_q0 = o; o += align256(rc * 4);
  c.n = o; o += align256((size_t)R * 4);
  c.rows = o; o += align256(rc * 4);
  c.off = o; o += align256((size_t)R * 4);
  c.upload = o;  // everything above is one host-to-device copy
  c.greedy = o; o += align256(rc * 4);
  c.part = o; o += align256(rc * kCalibChunks * sizeof(ArgmaxPart));
  c.bytes = o;
  return c;
}
}  // namespace

size_t ts_calib_labels_workspace_size(int32_t R, int32_t cap) {
  if (R < 1 || cap < 1) return 0;
  return calib_layout(R, cap).bytes;
}

int32_t ts_calib_labels(const ts_tree* tree, const void* target, int32_t target_dtype, int32_t V, float* x,
                        int32_t* y, int32_t* sel, void* workspace, size_t workspace_bytes, void* stream) {
  g_last_error.clear();
  if (!tree || !target || !x || !y || !sel) return fail(TS_EINVAL, "tree, target or an output is NULL");
  if (!tree->n || !tree->token || !tree->parent || !tree->log_q0) return fail(TS_EINVAL, "a tree array is NULL");
  if (tree->R < 1 || tree->cap < 1) return fail(TS_EINVAL, "tree R=%d cap=%d", tree->R, tree->cap);
  if (V < 1) return fail(TS_EINVAL, "V=%d", V);
  if (target_dtype != TS_F32 && target_dtype != TS_BF16) return fail(TS_EINVAL, "unknown target dtype %d", target_dtype);
  const int R = tree->R, cap = tree->cap;
  for (int q = 0; q < R; ++q) {
    const int nq = tree->n[q];
    if (nq < 0 || nq >= cap) return fail(TS_EINVAL, "tree n[%d]=%d outside [0, cap)", q, nq);
    for (int i = 1; i <= nq; ++i) {
      const size_t o = (size_t)q * cap + i;
      if (tree->parent[o] < 0 || tree->parent[o] >= i || tree->token[o] < 0 || tree->token[o] >= V)
        return fail(TS_EINVAL, "tree of request %d is malformed at node %d", q, i);
    }
  }
  const CalibLayout cl = calib_layout(R, cap);
  if (!workspace || workspace_bytes < cl.bytes)
    return fail(TS_ENOSPACE, "workspace %zu bytes < %zu needed", workspace_bytes, cl.bytes);
  char* hs = nullptr;
  int32_t rc = host_stage(cl.upload, &hs);
  if (rc != TS_OK) return rc;
  const size_t rcn = (size_t)R * cap;
  std::memcpy(hs + cl.parent, tree->parent, rcn * 4);
  std::memcpy(hs + cl.token, tree->token, rcn * 4);
  std::memcpy(hs + cl.log_q0, tree->log_q0, rcn * 4);
  std::memcpy(hs + cl.n, tree->n, (size_t)R * 4);
  int32_t* rows = reinterpret_cast<int32_t*>(hs + cl.rows);
  int32_t* off = reinterpret_cast<int32_t*>(hs + cl.off);
  int nrows = 0;
  for (int q = 0; q < R; ++q) {
    off[q] = nrows;
    for (int i = 0; i <= tree->n[q]; ++i) rows[nrows++] = q * cap + i;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  DrainOnError drain{s};
  TS_HIP(hipMemcpyAsync(ws, hs, cl.upload, hipMemcpyHostToDevice, s));
  int32_t* greedy = reinterpret_cast<int32_t*>(ws + cl.greedy);
  const int nc = verify_argmax_chunks(V, nrows, target_dtype == TS_BF16, kCalibChunks);
  ArgmaxPart* part = reinterpret_cast<ArgmaxPart*>(ws + cl.part);
  launch_verify_argmax(target, target_dtype == TS_BF16, V, reinterpret_cast<const int*>(ws + cl.rows), nrows, nc, part,
                       s);
  TS_HIP(hipGetLastError());
  launch_calib_labels(reinterpret_cast<const int32_t*>(ws + cl.parent), reinterpret_cast<const int32_t*>(ws + cl.token),
                      reinterpret_cast<const float*>(ws + cl.log_q0), reinterpret_cast<const int32_t*>(ws + cl.n), R,
                      cap, part, nc, greedy, reinterpret_cast<const int32_t*>(ws + cl.off), x, y, sel, s);
  TS_HIP(hipGetLastError());
  TS_HIP(hipStreamSynchronize(s));
  drain.armed = false;
  return TS_OK;
}

int32_t ts_calib_fit(const float* x, const int32_t* y, const int32_t* sel, int32_t n, int32_t max_iter,
                     double tol, float* out, void* stream) {
  g_last_error.clear();
  if (!x || !y || !sel || !out) return fail(TS_EINVAL, "an array is NULL");
  if (n < 0 || max_iter < 1 || !(tol > 0.0)) return fail(TS_EINVAL, "n=%d max_iter=%d tol=%g", n, max_iter, tol);
  launch_calib_fit(x, y, sel, n, max_iter, tol, out, static_cast<hipStream_t>(stream));
  TS_HIP(hipGetLastError());
  return TS_OK;
}

int32_t ts_tree_mask_words(int32_t cap) { return cap < 1 ? 0 : (cap + 31) / 32; }

int32_t ts_tree_mask(const int32_t* parent, const int32_t* n, int32_t R, int32_t cap,
                     const int32_t* pos_offset, uint32_t* mask, int32_t* pos, void* stream) {
  g_last_error.clear();
  if (R < 0) return fail(TS_EINVAL, "R=%d is negative", R);
  if (cap < 1 || cap > TS_MAX_CAP) return fail(TS_EINVAL, "cap=%d outside [1, %d]", cap, TS_MAX_CAP);
  if (R == 0) return TS_OK;
  if (!parent || !n || !mask || !pos) return fail(TS_EINVAL, "parent, n, mask or pos is NULL");
  hipStream_t s = static_cast<hipStream_t>(stream);
  launch_tree_mask(parent, n, R, cap, pos_offset, mask, pos, s);
  TS_HIP(hipGetLastError());
  return TS_OK;
}

}  // extern "C"
