// One launch for the levels of the T > 0 walk (§3.3, Proposition 1) with the
// rows held in registers.
//
// The per-stage launches read an item's target and draft rows once for pass A
// and again for every rejected child, so a node whose children are all
// rejected costs 1 + m sweeps of both rows.  Here each workgroup (item,
// chunk) loads its chunk of the two rows into registers once and keeps it for
// the whole walk at that node: pass A, the Z_j reductions of every rejected
// stage and the bonus keys all read registers.
//
// The chunks of an item meet between the walk's steps through tagged slots
// in global memory: a workgroup stores its partial result for a step as
// 64-bit words holding the value and the launch's epoch, with agent-scope
// relaxed stores (coherent across the XCDs' L2 caches); wave 0 of every
// workgroup that needs the step's total polls the item's slots of that step
// with agent-scope loads until every chunk's words carry the epoch, and reduces
// them in the same fixed order, so all workgroups take the same decisions.
// The slots are cleared once per ts_verify call and each level of each launch of
// the call has its own epoch, so no stale word matches.
//
// An accepted child whose logits were recomputed for the same launch is the
// item's next node: its workgroups go on there without the host.  Items walk
// independently, and a level taken this way costs the loads and pass A
// (about 10 us) instead of a recompute, a launch and the host's turn around
// (about 35 us).  With a launch per level and with this, 64 requests with trees of
// up to 8 nodes (V = 151936, bf16, T = 0.7) take 187 and 110 us, one request with
// 64 nodes (V = 128256) 148 and 78.  Consecutive levels use the two halves of the
// item's slots in turn: a workgroup can be one level ahead of another (which still
// reads the level's words), never two.
//
// The host sizes the grid to
// what the device holds at once, so every workgroup is resident and every wait
// ends; each wait is also bounded, and one that runs out sets a flag (device
// and pinned host copies) that ends the other waits early: the host then runs
// the level again through the per-stage launches.
#pragma once

#include "verify_kernels.hpp"

namespace ts {

// Quads of four tokens each thread holds: 40 tokens of a bf16 target (20 KB
// of LDS per workgroup for the target, 40 VGPRs for the draft), 24 of a
// float target (24 KB of LDS).
constexpr int kFusedQuadsBf16 = 10;
constexpr int kFusedQuadsF32 = 6;
// Most chunks an item is split into (more only when the chunk would not fit).
constexpr int kFusedMaxChunks = 32;

// Words of an item's slots, each [cpi] long: pass A (maxima and sums of
// both rows), the Z_j partial of each stage, the best bonus key and its token.
constexpr int kSlotPA = 0, kSlotZ = 4, kSlotB = 4 + TS_MAX_K, kSlotWords = 6 + TS_MAX_K;
// Most chunks of an item in one launch (one polling lane per chunk), and
// most workgroups of one launch (the slots are sized for that many).
constexpr int kFusedMaxCpi = 64;
constexpr int kFusedMaxGrid = 4096;

struct VFused {
  int cpi;           // chunks per item (<= kFusedMaxCpi)
  int chunk;         // tokens per chunk, a multiple of 4
  uint64_t* slots;   // [2][nitems][kSlotWords][cpi]: value bits | epoch << 32 (one half when no node goes on)
  uint32_t epoch;    // the first level's tag, the next levels count on (slots start the call at zero)
  int* err;          // device flag: a wait ran out
  int32_t* herr;     // the flag's pinned host copy
  int spin_limit;    // polls before a wait gives up (0: no wait is begun)
  const VerifyNext* next;  // of the launch's nodes, as vp.items
  uint64_t* done;    // [nitems][kDoneWords], pinned host memory: the items' results, zero before the launch
};

// The kernel's only argument.
struct VFusedArgs {
  VerifyPass vp;
  VFused f;
};
typedef const __attribute__((address_space(4))) VFusedArgs* FusedArgPtr;
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
#ifdef __HIP_DEVICE_COMPILE__
  __builtin_assume(!__builtin_amdgcn_is_shared((const void*)p) && !__builtin_amdgcn_is_private((const void*)p));
#endif
  return p;
}

// An item's result: 32-bit words, each stored with the launch's epoch above
// it (one 64-bit store), so that the host can go on as soon as it has seen
// every item's words instead of waiting for the launch to end and the stream
// to report it.
enum : int {
  kDoneBonus = 0,   // the bonus token
  kDonePath = 1,    // and 2: the accepted children's places in draw order, 4 bits a level
  kDoneState = 3,   // accepted children | kDoneEnded | kDoneLeaf
  kDoneWords = 4
};
constexpr uint32_t kDoneEnded = 256;  // the walk has ended (the bonus counts)
constexpr uint32_t kDoneLeaf = 512;   // at a node without children (no level of its own)
static_assert(TS_MAX_K <= 16 && TS_MAX_D <= 16, "a level takes 4 bits of two words");

// Quad of target values as loaded: four bf16 in two words, or four floats.
template <typename TT>
struct TQuad;
template <>
struct TQuad<uint16_t> {
  using type = uint2;
};
template <>
struct TQuad<float> {
  using type = f32x4;
};
__device__ __forceinline__ float tquad_at(const uint2& w, int e) {
  const uint32_t x = (e < 2) ? w.x : w.y;
  return __uint_as_float((e & 1) ? (x & 0xFFFF0000u) : (x << 16));
}
__device__ __forceinline__ float tquad_at(const f32x4& v, int e) { return v[e]; }

// Tokens b .. b+3 of both rows (z only when zrow is set); tokens at or past
// y1 read as -inf, which no maximum, sum or key takes up.  Quad loads when
// the rows hold a multiple of 4 tokens (every quad of a chunk, a multiple of
// 4 long, then lies wholly inside or outside it); otherwise loads of any
// alignment for whole quads, token loads for the one the row's end cuts.
template <typename TT>
__device__ __forceinline__ void load_quad_vec(const TT* trow, const float* zrow, int b, int y1,
                                              typename TQuad<TT>::type& t, f32x4& z) {
  if (b < y1) {
    if constexpr (sizeof(TT) == 2)
      t = *reinterpret_cast<const uint2*>(trow + b);
    else
      t = *reinterpret_cast<const f32x4*>(trow + b);
    if (zrow) z = *reinterpret_cast<const f32x4*>(zrow + b);
    else z = f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
  } else {
    if constexpr (sizeof(TT) == 2)
      t = uint2{0xFF80FF80u, 0xFF80FF80u};
    else
      t = f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
    z = f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
  }
}
template <typename TT>
__device__ __forceinline__ void load_quad_tok(const TT* trow, const float* zrow, int b, int y1,
                                              typename TQuad<TT>::type& t, f32x4& z) {
  if (b + 4 <= y1) {
    t = quad_words(trow + b);
    z = zrow ? quad_words(zrow + b) : f32x4{kNegInf, kNegInf, kNegInf, kNegInf};
    return;
  }
  uint32_t tw[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int y = b + e;
    if constexpr (sizeof(TT) == 2)
      tw[e] = y < y1 ? (uint32_t)trow[y] : 0xFF80u;
    else
      tw[e] = y < y1 ? __float_as_uint(trow[y]) : 0xFF800000u;
    z[e] = (zrow && y < y1) ? zrow[y] : kNegInf;
  }
  if constexpr (sizeof(TT) == 2)
    t = uint2{tw[0] | (tw[1] << 16), tw[2] | (tw[3] << 16)};
  else
    t = f32x4{__uint_as_float(tw[0]), __uint_as_float(tw[1]), __uint_as_float(tw[2]), __uint_as_float(tw[3])};
}

// Agent-scope relaxed accesses of 64-bit words.
__device__ __forceinline__ void st_agent(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t ld_agent(const uint64_t* p) {
  return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t pack_f32x2(float lo, float hi) {
  return (uint64_t)__float_as_uint(lo) | ((uint64_t)__float_as_uint(hi) << 32);
}
__device__ __forceinline__ float lo_f32(uint64_t w) { return __uint_as_float((uint32_t)w); }
__device__ __forceinline__ float hi_f32(uint64_t w) { return __uint_as_float((uint32_t)(w >> 32)); }

// Thread 0: the workgroup's word w of a step, tagged with the launch's epoch.
__device__ __forceinline__ void put_slot(const VFused& f, int it, int ck, int w, uint32_t bits) {
  st_agent(f.slots + ((size_t)it * kSlotWords + w) * f.cpi + ck, ((uint64_t)f.epoch << 32) | bits);
}

// Wave 0: lane k < cpi waits until words w0 .. w0 + NW - 1 of chunk k carry
// the launch's epoch and returns their values in out.  False when the wait
// ran out (the flag is then set) or another wait did.
template <int NW>
__device__ __forceinline__ bool poll_slots(const VFused& f, int it, int w0, uint32_t (&out)[NW]) {
  const int lane = threadIdx.x & 63;
  const bool mine = lane < f.cpi;
  const uint64_t* base = f.slots + ((size_t)it * kSlotWords + w0) * f.cpi + (mine ? lane : 0);
  bool ready = !mine;
#pragma unroll
  for (int i = 0; i < NW; ++i) out[i] = 0u;
  for (int n = 0;; ++n) {
    if (n >= f.spin_limit) {
      if (lane == 0) {
        __hip_atomic_store(f.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(f.herr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      }
      return false;
    }
    if (!ready) {
      uint64_t v[NW];
#pragma unroll
      for (int i = 0; i < NW; ++i) v[i] = ld_agent(base + (size_t)i * f.cpi);
      bool ok = true;
#pragma unroll
      for (int i = 0; i < NW; ++i) ok = ok && (uint32_t)(v[i] >> 32) == f.epoch;
      if (ok) {
#pragma unroll
        for (int i = 0; i < NW; ++i) out[i] = (uint32_t)v[i];
        ready = true;
      }
    }
    if (__all(ready)) return true;
    if ((n & 63) == 63 && __hip_atomic_load(f.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
    __builtin_amdgcn_s_sleep(1);
  }
}

// Best bonus key and its token (smallest on ties).
struct BonusBest {
  float best = kNegInf;
  int idx = 0x7FFFFFFF;
  __device__ __forceinline__ void add(float key, int y) {
    if (key > best) { best = key; idx = y; }
  }
};
// The workgroup's best key into the chunk's bonus words.
__device__ __forceinline__ void put_bonus(const BonusBest& bt, const VFused& f, int it, int ck, float* redv, int* redi) {
  float vb = bt.best;
  int id = bt.idx;
  block_argmax(vb, id, redv, redi);
  if (threadIdx.x == 0) {
    put_slot(f, it, ck, kSlotB, __float_as_uint(vb));
    put_slot(f, it, ck, kSlotB + 1, (uint32_t)id);
  }
}

// One level of the workgroup's walk; true if the walk goes on to another.
template <typename TT, int NQ>
__device__ __forceinline__ bool fused_level(FusedArgPtr apv, int levelv) {
  using Q = typename TQuad<TT>::type;
  static_assert(4 * NQ <= 64, "a thread's tokens fit the 64-bit child mask");
  __shared__ Q tl[NQ * kVerifyThreads];  // each thread's target quads, [q][thread]
  __shared__ VerifyItem sitem;
  __shared__ VerifyNext snext;
  __shared__ VConst sC;
  __shared__ VRec shr;
  __shared__ float redv[4];
  __shared__ int redi[4];
  __shared__ double redd[4];
  __shared__ int loc[TS_MAX_K];   // children inside the chunk: token
  __shared__ int locj[TS_MAX_K];  // and its place in the draw order (1-based)
  __shared__ int sh_n, sh_ok;
  // the walk: the node it stands at (an index into vp.items), the children
  // accepted so far (4 bits a level), its level in this launch
  __shared__ int sh_node;
  __shared__ uint64_t sh_digits;
  const int tid = threadIdx.x;
  constexpr int kItemWords = (int)(sizeof(VerifyItem) / 4);
  constexpr int kNextWords = (int)(sizeof(VerifyNext) / 4);
  static_assert(kItemWords + kNextWords <= kVerifyThreads, "item and next words");
  // function arguments arrive in vector registers
  const int level = __builtin_amdgcn_readfirstlane(levelv);
  const uint64_t apb = (uint64_t)apv;
  const FusedArgPtr ap = (FusedArgPtr)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(apb >> 32)) << 32) |
                                       (uint32_t)__builtin_amdgcn_readfirstlane((int)apb));
  // read through the constant address space: scalar loads
  uint32_t aw[sizeof(VFusedArgs) / 4];
#pragma unroll
  for (unsigned i = 0; i < sizeof(VFusedArgs) / 4; ++i)
    aw[i] = reinterpret_cast<const __attribute__((address_space(4))) uint32_t*>(ap)[i];
  VFusedArgs A;
  __builtin_memcpy(&A, aw, sizeof(A));
  // all of them point to global memory (else: flat loads)
  A.vp.target = as_global(ap->vp.target);
  A.vp.items = as_global(ap->vp.items);
  A.vp.zbuf = as_global(ap->vp.zbuf);
  A.f.slots = as_global(ap->f.slots);
  A.f.err = as_global(ap->f.err);
  A.f.herr = as_global(ap->f.herr);
  A.f.next = as_global(ap->f.next);
  A.f.done = as_global(ap->f.done);
  const VerifyPass& vp = A.vp;
  VFused& f = A.f;
  const uint32_t epoch0 = f.epoch;
  const int it = __builtin_amdgcn_readfirstlane((int)blockIdx.x / f.cpi);
  const int ck = __builtin_amdgcn_readfirstlane((int)blockIdx.x % f.cpi);
  if (it >= vp.nitems) return false;  // never: the grid is nitems * cpi
  if (level == 0 && tid == 0) {
    sh_node = it;
    sh_digits = 0;
  }
  f.epoch += (uint32_t)level;
  __syncthreads();  // the walk's place is set, the previous level's readers of the shared records are done
  const int at_node = __builtin_amdgcn_readfirstlane(sh_node);
  // every lane's own copy: at the walk's end wave 0 reports the path from it
  uint64_t digits = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)sh_digits) |
                    ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(sh_digits >> 32)) << 32);
  if (at_node < 0)  // an accepted leaf: its item is in place
    ;
  else if (tid < kItemWords)
    reinterpret_cast<int32_t*>(&sitem)[tid] = reinterpret_cast<const int32_t*>(vp.items + at_node)[tid];
  else if (tid < kItemWords + kNextWords)
    reinterpret_cast<int32_t*>(&snext)[tid - kItemWords] =
        reinterpret_cast<const int32_t*>(f.next + at_node)[tid - kItemWords];
  __syncthreads();
  const int m = __builtin_amdgcn_readfirstlane(sitem.m);
  // a leaf uses the bonus words only, which its walk has not used before
  if (m > 0) f.slots += (size_t)(level & 1) * vp.nitems * kSlotWords * f.cpi;
  const int y0 = ck * f.chunk, y1 = min(vp.V, y0 + f.chunk);
  const TT* trow = static_cast<const TT*>(vp.target) + ((size_t)sitem.request * vp.cap + sitem.node) * vp.V;
  const float* zrow = m > 0 ? vp.zbuf + (size_t)sitem.zrow * vp.V : nullptr;
  if (tid == 0) {
    int k = 0;
    for (int s = 0; s < m; ++s) {
      const int x = sitem.child_tok[s];
      if (x >= y0 && x < y1) {
        loc[k] = x;
        locj[k] = s + 1;
        ++k;
      }
    }
    sh_n = k;
  }
  // thread t holds the quads y0 + 4 t + 1024 q, q < NQ
  int b0 = y0 + 4 * tid;
  asm volatile("" : "+v"(b0));
  Q tq[NQ];
  f32x4 zq[NQ];
  if (vector_rows<TT>(vp)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) load_quad_vec<TT>(trow, zrow, b0 + 1024 * q, y1, tq[q], zq[q]);
  } else {
#pragma unroll
    for (int q = 0; q < NQ; ++q) load_quad_tok<TT>(trow, zrow, b0 + 1024 * q, y1, tq[q], zq[q]);
  }
  __syncthreads();
  const int nloc = __builtin_amdgcn_readfirstlane(sh_n);
  const float c = vp.c;
  const uint32_t pc1 = (uint32_t)sitem.path, pc2 = (uint32_t)(sitem.path >> 32);
  const uint32_t c3 = counter_word3(sitem.request, sitem.depth, 3u);
  bool alive = true;
  bool bonus = false;  // the walk ended without an accepted child: chunk 0 draws the bonus
  VRec rec;
  rec.status = kExhausted;  // a leaf: the bonus comes from the target itself
  rec.stage = 1;
  rec.alpha = 1.0f; rec.beta = 0.0f; rec.betap = 1.0f;
  rec.margin = __builtin_huge_valf();

  if (m == 0) {
    // leaf: bonus keys from the target row
    // (r = 2^(t c - const): the draw comes from the target itself), one quad
    // of the thread at a time out of LDS
#pragma unroll
    for (int q = 0; q < NQ; ++q) tl[q * kVerifyThreads + tid] = tq[q];
    BonusBest bt;
#pragma unroll 1
    for (int q = 0; q < NQ; ++q) {
      const int bq = b0 + 1024 * q;
      if (bq >= y1) break;
      const Q t = tl[q * kVerifyThreads + tid];
      uint32_t w[4];
      bonus_words(w, bq, pc1, pc2, c3, vp.keys);
#pragma unroll
      for (int e = 0; e < 4; ++e) bt.add(tquad_at(t, e) * c + gumbel_neg(w[e]), bq + e);
    }
    put_bonus(bt, f, it, ck, redv, redi);
    bonus = true;
  } else {
    // an item with children holds the level's longest chain of steps: its
    // waves go first when leaves' bonus keys share the SIMDs
    __builtin_amdgcn_s_setprio(2);
    // the children's values, for the constants, on their way during pass A
    VChildVals cv{0.0f, 0.0f};
    if (tid < 64) cv = load_child_vals<TT>(vp, sitem);
    // pass A: the chunk's maxima, then its sums relative to them; the draft
    // sum leaves every child out.  The target quads then move to LDS.
    float mt = kNegInf, mz = kNegInf;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        mt = fmaxf(mt, tquad_at(tq[q], e) * c);
        mz = fmaxf(mz, zq[q][e] * c);
      }
    mt = block_max(mt, redv);
    mz = block_max(mz, redv);
    const float mts = mt > kNegInf ? mt : 0.0f, mzs = mz > kNegInf ? mz : 0.0f;
    float st = 0.0f, snc = 0.0f;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
      for (int e = 0; e < 4; ++e) st += exp2_fast(tquad_at(tq[q], e) * c - mts);
      tl[q * kVerifyThreads + tid] = tq[q];
    }
    if (nloc == 0) {
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) snc += exp2_fast(zq[q][e] * c - mzs);
    } else {
      // bit 4 q + e: the thread's token (q, e) is a child, left out of the sum
      uint64_t cmask = 0;
      for (int k = 0; k < nloc; ++k) {
        const int at = loc[k] - b0;
        if (at >= 0 && at < 1024 * NQ && (at & 1023) < 4) cmask |= 1ull << (4 * (at >> 10) + (at & 3));
      }
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = exp2_fast(zq[q][e] * c - mzs);
          snc += ((cmask >> (4 * q + e)) & 1) ? 0.0f : x;
        }
    }
    const double dst = block_sum_f64((double)st, redd);
    const double dsnc = block_sum_f64((double)snc, redd);
    if (tid == 0) {
      put_slot(f, it, ck, kSlotPA, __float_as_uint(mt));
      put_slot(f, it, ck, kSlotPA + 1, __float_as_uint(mz));
      put_slot(f, it, ck, kSlotPA + 2, __float_as_uint((float)dst));
      put_slot(f, it, ck, kSlotPA + 3, __float_as_uint((float)dsnc));
    }
    // every workgroup: the item's constants and the test of child 1
    if (tid < 64) {
      const int lane = tid;
      uint32_t w[4];
      const bool ok = poll_slots<4>(f, it, kSlotPA, w);
      if (ok) {
        const VConstLane C = verify_consts_lane<TT>(vp, sitem, f.cpi, [&](int) {
          VPartA a;
          a.mt = __uint_as_float(w[0]);
          a.mz = __uint_as_float(w[1]);
          a.st = (double)__uint_as_float(w[2]);
          a.snc = (double)__uint_as_float(w[3]);
          return a;
        }, cv);
        if (lane < m) {
          sC.lp[lane] = C.lp;
          sC.lq[lane] = C.lq;
          sC.lR[lane] = C.lR;
          sC.invR[lane] = C.invR;
          sC.lu[lane] = C.lu;
        }
        if (lane == 0) {
          sC.Lt = C.Lt;
          sC.Lz = C.Lz;
          shr = stage_test(C.lp, C.lq, C.lR, C.invR, C.lu, 1, 1.0f, 0.0f, __builtin_huge_valf());
        }
      }
      if (lane == 0) sh_ok = ok ? 1 : 0;
    }
    __syncthreads();
    alive = __builtin_amdgcn_readfirstlane(sh_ok) != 0;
    if (alive) {
      rec = shr;
      const float Lt = sC.Lt, Lz = sC.Lz;
      // the draft quads become q = 2^(z c - Lz) (zero outside the chunk); p =
      // 2^(t c - Lt) is taken from the LDS quads in each sweep
#pragma unroll
      for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) zq[q][e] = exp2_fast(zq[q][e] * c - Lz);
      // stage j rejected: Z_j over the tokens not drawn up to j; at the last
      // child the same residual also gives the bonus keys
      for (int j = 1; __builtin_amdgcn_readfirstlane(rec.status) == kRejected; ++j) {
        if (nloc) {
          for (int k = 0; k < nloc; ++k) {
            if (locj[k] != j) continue;
            // the drawn child leaves the sums: q = 0 and t = -inf
            const int at = loc[k] - b0;
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (1024 * q + e == at) {
                  zq[q][e] = 0.0f;
                  Q t = tl[q * kVerifyThreads + tid];
                  if constexpr (sizeof(TT) == 2) {
                    uint32_t& x = (e < 2) ? t.x : t.y;
                    x = (e & 1) ? ((x & 0xFFFFu) | 0xFF800000u) : ((x & 0xFFFF0000u) | 0xFF80u);
                  } else {
                    t[e] = kNegInf;
                  }
                  tl[q * kVerifyThreads + tid] = t;
                }
          }
        }
        const float a = rec.alpha, bb = rec.betap;
        if (j == m) {
          BonusBest bt;
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            if (b0 + 1024 * q >= y1) break;
            const Q t = tl[q * kVerifyThreads + tid];
            int bq = b0 + 1024 * q;
            asm volatile("" : "+v"(bq) : "v"(bt.best));
            uint32_t w[4];
            bonus_words(w, bq, pc1, pc2, c3, vp.keys);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float r = a * exp2_fast(tquad_at(t, e) * c - Lt) - bb * zq[q][e];
              if (r > 0.0f) bt.add(__builtin_amdgcn_logf(r) + gumbel_neg(w[e]), b0 + 1024 * q + e);
            }
          }
          put_bonus(bt, f, it, ck, redv, redi);
          rec.status = kExhausted;
          rec.stage = j + 1;
          bonus = true;
          break;
        }
        float acc = 0.0f;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const Q t = tl[q * kVerifyThreads + tid];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc += fmaxf(a * exp2_fast(tquad_at(t, e) * c - Lt) - bb * zq[q][e], 0.0f);
        }
        const double z = block_sum_f64((double)acc, redd);
        if (tid == 0) put_slot(f, it, ck, kSlotZ + j - 1, __float_as_uint((float)z));
        if (tid < 64) {
          uint32_t w[1];
          const bool ok = poll_slots<1>(f, it, kSlotZ + j - 1, w);
          if (ok) {
            const double Z = wave_sum_f64(tid < f.cpi ? (double)__uint_as_float(w[0]) : 0.0);
            const VRec nr = verify_advance(rec, Z, child_consts(sC, j), m, j + 1);
            if (tid == 0) shr = nr;
          }
          if (tid == 0) sh_ok = ok ? 1 : 0;
        }
        __syncthreads();
        alive = __builtin_amdgcn_readfirstlane(sh_ok) != 0;
        if (!alive) break;
        rec = shr;
      }
    }
  }
  const bool ended = bonus;
  const bool took = alive && m > 0 && __builtin_amdgcn_readfirstlane(rec.status) == kAccepted;
  if (took) {
    const int s = __builtin_amdgcn_readfirstlane(rec.stage) - 1;
    const int ci = __builtin_amdgcn_readfirstlane(snext.child_item[s]);
    digits |= (uint64_t)s << (4 * level);
    if (tid == 0) {
      sh_digits = digits;
      sh_node = ci;  // >= 0, or set below
    }
    // the accepted child's logits are there: the walk goes on at it (a walk
    // has at most TS_MAX_D levels; the path's digits have room for no more)
    if (ci >= 0 && level + 1 < TS_MAX_D) return true;
    if (ci == kNextLeaf) {
      // a child without children: the next level draws the bonus from its target row
      if (tid == 0) {
        sitem.m = 0;
        sitem.node = snext.child_node[s];
        sitem.path = snext.child_path[s];
        sitem.depth += 1;
        sh_node = -1;
      }
      return true;
    }
  }
  // chunk 0 hands the item's walk to the host: the accepted children, and the
  // bonus token from the chunks' best keys if it has ended
  if (ck == 0 && alive && tid < 64) {
    uint32_t w[2] = {0u, 0u};
    const bool ok = ended ? poll_slots<2>(f, it, kSlotB, w) : true;
    if (ok) {
      float vb = tid < f.cpi ? __uint_as_float(w[0]) : kNegInf;
      int id = tid < f.cpi ? (int)w[1] : 0x7FFFFFFF;
#pragma unroll
      for (int o = 32; o >= 1; o >>= 1) {
        const float ov = __shfl_xor(vb, o, 64);
        const int oi = __shfl_xor(id, o, 64);
        if (ov > vb || (ov == vb && oi < id)) { vb = ov; id = oi; }
      }
      const int accepted = level + (took ? 1 : 0);
      if (tid < kDoneWords) {
        const uint32_t v = tid == kDoneBonus ? (uint32_t)id
                           : tid == kDoneState ? (uint32_t)accepted | (ended ? kDoneEnded : 0u) | (m == 0 ? kDoneLeaf : 0u)
                                               : (uint32_t)(digits >> (32 * (tid - kDonePath)));
        __hip_atomic_store(f.done + (size_t)it * kDoneWords + tid, ((uint64_t)epoch0 << 32) | v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
      }
    }
  }
  return false;
}

// The levels after the first are calls of a function: as the body of a loop over
// the levels, the compiler carried addresses, bounds and masks over them and
// spilled 79 to 151 registers in the middle of the work (64 requests, T = 0.7:
// 178 us).  A call saves some 50 registers per lane at its entry, 50 MB of scratch
// written and read back for 1024 workgroups, so the first level, at which many
// walks end, is the kernel's own body (that measurement's case 125 us with every
// level a call, 115 so; 64 requests whose trees have 148 nodes 96 and 89).
template <typename TT, int NQ>
__device__ __attribute__((noinline)) bool fused_next_level(FusedArgPtr ap, int level) {
  return fused_level<TT, NQ>(ap, level);
}

template <typename TT, int NQ>
__global__ __launch_bounds__(kVerifyThreads) __attribute__((amdgpu_waves_per_eu(4))) void verify_fused_kernel(
    const VFusedArgs) {
  const FusedArgPtr ap = (FusedArgPtr)__builtin_amdgcn_kernarg_segment_ptr();
  if (!fused_level<TT, NQ>(ap, 0)) return;
  for (int level = 1; fused_next_level<TT, NQ>(ap, level); ++level) {
  }
}

}  // namespace ts
