// HIP kernels of the LightBeam gfx950 decoder (wave64, CDNA4).
//
// A decode call is one launch of k_decode on the caller's stream: one
// workgroup per stream runs Alg. 1 over the call's frames with the stream's
// beam resident in LDS (fan-out, recombination, theta / top-K pruning, trie
// advance, Eq. (1) with the hashed 4-gram LM, Eq. (2) with the synthetic
// scorer).  The output -- each stream's hypotheses ranked, their word ids and
// scores written (after the final fusion at the end of an utterance) -- is
// written by the call's last k_decode launch, or by k_output when the call
// ends without one.  k_fuse_select,
// k_fuse_export and k_fuse_apply carry the round trip to an external fusion
// scorer; k_build_order fills the n-gram hash tables; k_begin resets streams.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <mutex>

#include "lb_device.h"
#include "lb_launch.h"

namespace lb {

namespace {

constexpr double kNegInf = -HUGE_VAL;
constexpr int kBoundaryCap = 256;   // candidates resolved exactly inside the boundary bin
constexpr int kMaxLevels = 16;      // refinement levels of the top-K selection
constexpr uint32_t kGroupHeavy = 0x80000000u;  // query group scored through its explicit homophones

// ------------------------------------------------------------------ block helpers

// Workgroup barrier that orders LDS only: it waits for the wave's LDS
// operations, not for its outstanding global loads and stores (those are
// waited for where their registers are used, and by a full __syncthreads
// where global memory is handed between threads).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders LDS accesses among the lanes of a wavefront (the hardware runs them in
// order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Cross-lane moves inside rows of 16 lanes (DPP): lane i reads lane i^1
// (quad_perm [1,0,3,2]), lane i^2 (quad_perm [2,3,0,1]), the mirror lane in
// its half-row (7-i) and in its row (15-i).  Applying an associative,
// commutative operation after each of the four leaves every lane with the
// result over its row; the four rows are then combined through readlane.  A
// lane whose source lane is inactive receives `ident` (the operation's
// identity).
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int CTRL>
__device__ __forceinline__ int dpp_i32(int x, int ident) {
  return __builtin_amdgcn_update_dpp(ident, x, CTRL, 0xF, 0xF, false);
}

// The value of lane L of the lane's quad.
template <int L>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t x) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), L * 0x55, 0xF, 0xF, true));
}

template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x, double ident) {
  return __hiloint2double(dpp_i32<CTRL>(__double2hiint(x), __double2hiint(ident)),
                          dpp_i32<CTRL>(__double2loint(x), __double2loint(ident)));
}

__device__ __forceinline__ double readlane_f64(double x, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                          __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// Wavefront maximum of *mx and minimum of *mn, in every lane.
__device__ __forceinline__ void wave_minmax(double* mx, double* mn) {
  double a = *mx, c = *mn;
#define LB_MM_STEP(C)                    \
  a = fmax(a, dpp_f64<C>(a, -HUGE_VAL)); \
  c = fmin(c, dpp_f64<C>(c, HUGE_VAL));
  LB_MM_STEP(kDppXor1)
  LB_MM_STEP(kDppXor2)
  LB_MM_STEP(kDppHalfMirror)
  LB_MM_STEP(kDppMirror)
#undef LB_MM_STEP
  *mx = fmax(fmax(readlane_f64(a, 0), readlane_f64(a, 16)), fmax(readlane_f64(a, 32), readlane_f64(a, 48)));
  *mn = fmin(fmin(readlane_f64(c, 0), readlane_f64(c, 16)), fmin(readlane_f64(c, 32), readlane_f64(c, 48)));
}

// Wavefront maximum of x, in every lane.
__device__ __forceinline__ double wave_max(double x) {
  x = fmax(x, dpp_f64<kDppXor1>(x, -HUGE_VAL));
  x = fmax(x, dpp_f64<kDppXor2>(x, -HUGE_VAL));
  x = fmax(x, dpp_f64<kDppHalfMirror>(x, -HUGE_VAL));
  x = fmax(x, dpp_f64<kDppMirror>(x, -HUGE_VAL));
  return fmax(fmax(readlane_f64(x, 0), readlane_f64(x, 16)), fmax(readlane_f64(x, 32), readlane_f64(x, 48)));
}

// Wavefront sum of x, in every lane.
__device__ __forceinline__ double wave_sum(double x) {
  x += dpp_f64<kDppXor1>(x, 0.0);
  x += dpp_f64<kDppXor2>(x, 0.0);
  x += dpp_f64<kDppHalfMirror>(x, 0.0);
  x += dpp_f64<kDppMirror>(x, 0.0);
  return (readlane_f64(x, 0) + readlane_f64(x, 16)) + (readlane_f64(x, 32) + readlane_f64(x, 48));
}

// One DPP step of the wavefront arg-max of (L desc, q asc).
template <int CTRL>
__device__ __forceinline__ void argmax_step(double* L, int* q) {
  const double oL = dpp_f64<CTRL>(*L, -HUGE_VAL);
  const int oq = dpp_i32<CTRL>(*q, 0x7FFFFFFF);
  const bool take = oL > *L || (oL == *L && oq < *q);
  *L = take ? oL : *L;
  *q = take ? oq : *q;
}

// Wavefront arg-max of (L desc, q asc), in every lane.
__device__ __forceinline__ void wave_argmax(double* L, int* q) {
  argmax_step<kDppXor1>(L, q);
  argmax_step<kDppXor2>(L, q);
  argmax_step<kDppHalfMirror>(L, q);
  argmax_step<kDppMirror>(L, q);
  double bL = readlane_f64(*L, 0);
  int bq = __builtin_amdgcn_readlane(*q, 0);
#pragma unroll
  for (int r = 16; r < 64; r += 16) {
    const double oL = readlane_f64(*L, r);
    const int oq = __builtin_amdgcn_readlane(*q, r);
    if (oL > bL || (oL == bL && oq < bq)) {
      bL = oL;
      bq = oq;
    }
  }
  *L = bL;
  *q = bq;
}

// Block-wide maximum of `mx` and minimum of `mn` in one reduction (SYNC as in
// block_scan).
template <int BLOCK, bool SYNC = true>
__device__ inline void block_minmax(double mx, double mn, double* red, double* out_max, double* out_min) {
  wave_minmax(&mx, &mn);
  constexpr int NW = BLOCK / 64;
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = mx;
    red[NW + (threadIdx.x >> 6)] = mn;
  }
  lds_barrier();
  double a = red[0], c = red[NW];
#pragma unroll
  for (int k = 1; k < NW; ++k) {
    a = fmax(a, red[k]);
    c = fmin(c, red[NW + k]);
  }
  if (SYNC) lds_barrier();
  *out_max = a;
  *out_min = c;
}

// Inclusive prefix sum over the wavefront: shifts by 1, 2, 4, 8 inside each
// row of 16 lanes (lanes shifted in from outside the row add 0), then rows 1
// and 3 add the last lane of the row before them, and rows 2 and 3 add lane 31.
__device__ __forceinline__ int wave_scan_incl(int v) {
  int x = v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
  return x;
}

// Exclusive prefix sum over the block; *total receives the block sum.  With
// SYNC = false the trailing barrier is left out: `red` must then not be
// written again before the next barrier.
template <int BLOCK, bool SYNC = true>
__device__ inline int block_scan(int v, int* red, int* total) {
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const int x = wave_scan_incl(v);
  if (lane == 63) red[w] = x;
  lds_barrier();
  int base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < BLOCK / 64; ++k) {
    const int t = red[k];
    base += (k < w) ? t : 0;
    tot += t;
  }
  if (SYNC) lds_barrier();
  *total = tot;
  return base + x - v;
}

// (score desc, key asc)
__device__ inline bool ranks_before(double sa, uint64_t ka, double sb, uint64_t kb) {
  return sa > sb || (sa == sb && ka < kb);
}

// In-place bitonic sort of N entries (N a power of two, at most the block
// size) by (score desc, key asc); every thread of the block calls it.
template <int N>
__device__ inline void bitonic_sort(double* sc, uint64_t* ky, uint32_t* val) {
  const int i = threadIdx.x;
  for (int k = 2; k <= N; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int ixj = i ^ j;
      if (i < N && ixj > i) {
        const bool up = (i & k) == 0;
        const bool swap = up ? ranks_before(sc[ixj], ky[ixj], sc[i], ky[i])
                             : ranks_before(sc[i], ky[i], sc[ixj], ky[ixj]);
        if (swap) {
          const double s = sc[i];
          sc[i] = sc[ixj];
          sc[ixj] = s;
          const uint64_t kk = ky[i];
          ky[i] = ky[ixj];
          ky[ixj] = kk;
          const uint32_t vv = val[i];
          val[i] = val[ixj];
          val[ixj] = vv;
        }
      }
      lds_barrier();
    }
  }
}

// Two unsigned 16-bit halves at once: bit 0 of each half of the result: the half
// of x is below the half of y.  (A saturating difference cut to 1; as C++ the
// compiler turns it into two compares and two selects.)
__device__ __forceinline__ uint32_t pk_below(uint32_t x, uint32_t y) {
  uint32_t d, r;
  asm("v_pk_sub_u16 %0, %1, %2 clamp" : "=v"(d) : "v"(y), "v"(x));
  asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(d), "v"(0x00010001));
  return r;
}

// ------------------------------------------------------------------ n-gram tables

// Looks `key` up; `lines` counts the 64-B bucket lines read.
__device__ inline bool probe(const NgramTable& t, uint64_t key, uint32_t* slot, float* lp, float* bo,
                             uint32_t* lines) {
  if (t.nbuckets == 0) return false;
  uint64_t bk = bucket_of(key, t.nbuckets);
  for (uint64_t it = 0; it < t.nbuckets; ++it) {
    ++*lines;
    const uint4* line = reinterpret_cast<const uint4*>(t.slots + bk * 4);
    uint4 q[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) q[s] = line[s];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const uint64_t k = static_cast<uint64_t>(q[s].x) | (static_cast<uint64_t>(q[s].y) << 32);
      if (k == key) {
        *slot = static_cast<uint32_t>(bk * 4 + s);
        *lp = __uint_as_float(q[s].z);
        *bo = __uint_as_float(q[s].w);
        return true;
      }
      if (k == kEmptyKey) return false;
    }
    bk = (bk + 1 == t.nbuckets) ? 0 : bk + 1;
  }
  return false;
}

// 0 = inserted, 1 = duplicate key, 2 = table full
__device__ inline int insert(const NgramTable& t, uint64_t key, float lp, float bo) {
  uint64_t bk = bucket_of(key, t.nbuckets);
  for (uint64_t it = 0; it < t.nbuckets; ++it) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      Slot* sl = t.slots + bk * 4 + s;
      const unsigned long long prev =
          atomicCAS(reinterpret_cast<unsigned long long*>(&sl->key), kEmptyKey, key);
      if (prev == kEmptyKey) {
        sl->logp = lp;
        sl->bo = bo;
        return 0;
      }
      if (prev == key) return 1;
    }
    bk = (bk + 1 == t.nbuckets) ? 0 : bk + 1;
  }
  return 2;
}

// Inserts a chunk of order-`order` n-grams; each n-gram's context id (the word
// id for order 2, the slot of its context n-gram for orders 3 and 4) goes to
// ctx_out[e] when ctx_out is given (kNone on error).
__global__ void k_build_order(int order, const int32_t* __restrict__ ids, const float* __restrict__ lp,
                              const float* __restrict__ bo, int64_t count, int32_t vocab, NgramTable t2,
                              NgramTable t3, NgramTable dst, uint32_t* flags, uint32_t* ctx_out) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  for (int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < count; e += stride) {
    const int32_t* r = ids + e * order;
    if (ctx_out) ctx_out[e] = kNone;
    bool ok = true;
    for (int k = 0; k < order; ++k) ok = ok && r[k] >= 0 && r[k] < vocab;
    if (!ok) {
      atomicOr(flags, kFlagBuildRange);
      continue;
    }
    uint64_t ctx = static_cast<uint32_t>(r[0]);
    if (order >= 3) {
      uint32_t s2, nl = 0;
      float a, c;
      if (!probe(t2, (static_cast<uint64_t>(r[0]) << 32) | static_cast<uint32_t>(r[1]), &s2, &a, &c, &nl)) {
        atomicOr(flags, kFlagBuildContext);
        continue;
      }
      ctx = s2;
      if (order == 4) {
        uint32_t s3;
        if (!probe(t3, (static_cast<uint64_t>(s2) << 32) | static_cast<uint32_t>(r[2]), &s3, &a, &c, &nl)) {
          atomicOr(flags, kFlagBuildContext);
          continue;
        }
        ctx = s3;
      }
    }
    const uint64_t key = (ctx << 32) | static_cast<uint32_t>(r[order - 1]);
    if (ctx_out) ctx_out[e] = static_cast<uint32_t>(ctx);
    const int st = insert(dst, key, lp[e], bo ? bo[e] : 0.0f);
    if (st == 1) atomicOr(flags, kFlagBuildDup);
    if (st == 2) atomicOr(flags, kFlagBuildFull);
  }
}

// ------------------------------------------------------------------ stream reset

__global__ void k_begin(DevParams P, DevState S, int32_t B) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  const size_t i = static_cast<size_t>(b) * P.K;
  S.nbeam[b] = 1;
  S.key[i] = 0;
  S.pkey[i] = kNoParent;
  S.ab[i] = 0.0;
  S.anb[i] = kNegInf;
  S.pt[i] = lse2(0.0, kNegInf);
  S.node[i] = kRootNode;
  S.meta[i] = 1u << 8;  // no last symbol, one sub-beam
  S.Lw[i * P.O] = 0.0;
  S.hist[i * P.O] = kRootHist;
  S.t0[b] = 0;
  S.arena_n[b] = 0;
}

// ------------------------------------------------------------------ n-gram lookup

// One 64-B bucket: four 16-B slots {key lo, key hi, log10 p, backoff}.
struct Bucket {
  uint4 s0, s1, s2, s3;
};

// (NgramTable and PresTable share the bucket layout: 16-B slots {u64 key, u32, u32})
template <typename Table>
__device__ __forceinline__ Bucket load_bucket(const Table& t, uint64_t bk) {
  // (tables are in global memory: a table pointer kept in LDS loses that, and
  // flat loads would also wait for LDS)
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  const u4 __attribute__((address_space(1)))* line =
      (const u4 __attribute__((address_space(1)))*)reinterpret_cast<uintptr_t>(t.slots + bk * 4);
  Bucket q;
  q.s0 = __builtin_bit_cast(uint4, line[0]);
  q.s1 = __builtin_bit_cast(uint4, line[1]);
  q.s2 = __builtin_bit_cast(uint4, line[2]);
  q.s3 = __builtin_bit_cast(uint4, line[3]);
  return q;
}

__device__ __forceinline__ uint64_t slot_key(const uint4& v) {
  return static_cast<uint64_t>(v.x) | (static_cast<uint64_t>(v.y) << 32);
}

// Scans a bucket for `key`: 1 found (slot index and the slot's two values set),
// 0 absent, -1 bucket full.
__device__ __forceinline__ int scan_bucket(const Bucket& q, uint64_t key, uint64_t bk, uint32_t* slot, uint32_t* z,
                                           uint32_t* w) {
#define LB_SCAN_SLOT(V, K)                              \
  {                                                     \
    const uint64_t kk = slot_key(V);                    \
    if (kk == key) {                                    \
      *slot = static_cast<uint32_t>(bk * 4 + (K));      \
      *z = (V).z;                                       \
      *w = (V).w;                                       \
      return 1;                                         \
    }                                                   \
    if (kk == kEmptyKey) return 0;                      \
  }
  LB_SCAN_SLOT(q.s0, 0)
  LB_SCAN_SLOT(q.s1, 1)
  LB_SCAN_SLOT(q.s2, 2)
  LB_SCAN_SLOT(q.s3, 3)
#undef LB_SCAN_SLOT
  return -1;
}

// Resolves a lookup whose first bucket `bk` is already loaded; linear probing
// continues bucket by bucket while buckets are full.
template <typename Table>
__device__ __forceinline__ bool resolve(const Table& t, uint64_t key, uint64_t bk, const Bucket& first,
                                        uint32_t* slot, uint32_t* z, uint32_t* w, uint32_t* lines) {
  int r = scan_bucket(first, key, bk, slot, z, w);
  for (uint64_t it = 1; r < 0 && it < t.nbuckets; ++it) {
    bk = (bk + 1 == t.nbuckets) ? 0 : bk + 1;
    ++*lines;
    r = scan_bucket(load_bucket(t, bk), key, bk, slot, z, w);
  }
  return r == 1;
}

// log10 P(w | the last three words of history ctx) by Katz backoff over the
// hashed tables (Eq. (1), App. E.3), and the n-gram state after w.
struct LmResult {
  double lp;
  QState st;
};

// The n-gram context of a history node: its last word, the slots of its 2- and
// 3-word contexts and the three backoffs.
struct Ctx {
  int32_t word;
  uint32_t c2, c3;
  float bo1, bo2, bo3;
};

__device__ __forceinline__ Ctx ctx_of(const HistNode& h) {
  Ctx c;
  c.word = h.word;
  c.c2 = h.c2;
  c.c3 = h.c3;
  c.bo1 = h.bo1;
  c.bo2 = h.bo2;
  c.bo3 = h.bo3;
  return c;
}

// Result of one probe: the slot index and the slot's two values (kNone, 0 and 0
// where the key is absent).
struct Hit {
  uint32_t slot, z, y;
};

// log10 P(w | ctx) and the state after w from the probes of orders 2, 3 and 4.
__device__ __forceinline__ LmResult lm_result(const Hit& h2, const Hit& h3, const Hit& h4, float bo1, float bo2,
                                              float bo3, int32_t w, float logp, float bo) {
  const bool f2 = h2.slot != kNone, f3 = h3.slot != kNone, f4 = h4.slot != kNone;
  // log10 P(w | context) by backoff, innermost order first
  double lp;
  if (f4) {
    lp = static_cast<double>(__uint_as_float(h4.z));
  } else {
    double l3;
    if (f3) {
      l3 = static_cast<double>(__uint_as_float(h3.z));
    } else {
      const double l2 = f2 ? static_cast<double>(__uint_as_float(h2.z)) : static_cast<double>(bo1) + static_cast<double>(logp);
      l3 = static_cast<double>(bo2) + l2;
    }
    lp = static_cast<double>(bo3) + l3;
  }
  LmResult r;
  r.lp = lp;
  r.st.c2 = h2.slot;
  r.st.c3 = h3.slot;
  r.st.bo2 = f2 ? __uint_as_float(h2.y) : 0.0f;
  r.st.bo3 = f3 ? __uint_as_float(h3.y) : 0.0f;
  r.st.w = w;
  r.st.bo1 = bo;
  return r;
}

// Identity of an n-gram query group: the context of a history node (its 3-word
// context slot if the LM has that trigram, else its 2-word context slot, else
// its last word; the backoff weights are functions of these) and the trie
// node of the completed word (by its first word offset, < 2^30).
__device__ __forceinline__ unsigned long long group_key(const Ctx& ctx, uint32_t woff) {
  const uint64_t tag = ctx.c3 != kNone ? 2u : (ctx.c2 != kNone ? 1u : 0u);
  const uint64_t id = ctx.c3 != kNone ? ctx.c3 : (ctx.c2 != kNone ? ctx.c2 : static_cast<uint32_t>(ctx.word));
  return (tag << 62) | (id << 30) | woff;
}

// ------------------------------------------------------------------ decoding loop

// A wavefront that scores completed words: words and lookups per turn, lookup
// results kept in LDS (further ones go to the stream's scratch), homophones up
// to which a fully looked-up group is ranked by one lane.
constexpr int kWaveWords = 64 / kMaxSub;
constexpr int kWaveTasks = 16;
constexpr uint32_t kTopWords = 4;  // of a heavy word, read ahead in unigram order (o + 1 decide it, o <= 3)
constexpr int kLmRes = 64;
constexpr uint32_t kLaneMaxH = 16;
constexpr int kNoCandidate = 0x7FFFFFFF;  // an empty place of a ranked list (after every sub-beam << 16 | homophone)
struct LmWave {
  double lp[kLmRes];
  QState st[kLmRes];
  uint8_t owner[kWaveTasks];  // the group (its first lane) of each task
};
static_assert(sizeof(LmWave) % 8 == 0, "wavefront scratch alignment");

// A stream's hypotheses in LDS (structure of arrays); the fields of each
// hypothesis' trie node travel with it.
template <int KMAX>
struct BeamLds {
  uint64_t key[KMAX];
  uint64_t pkey[KMAX];
  uint64_t tmask[KMAX];  // trie child mask, separator bit, word count << 48
  double ab[KMAX];
  double anb[KMAX];
  double pt[KMAX];  // log-sum-exp(ab, anb)
  double Lw[KMAX * kMaxSub];
  uint32_t hist[KMAX * kMaxSub];
  uint32_t node[KMAX];
  uint32_t meta[KMAX];   // last symbol | number of sub-beams << 8
  uint32_t first[KMAX];  // the trie node's first child
  uint32_t woff[KMAX];   // the trie node's first word in trie_words
};

template <int NT, int N>
__device__ __forceinline__ void write_output(const DevParams& P, const DevState& S, int b, const int32_t* lengths,
                                             int32_t Tc, int32_t fin, int32_t* out_hyps, float* out_scores, int n,
                                             bool root, double total, uint64_t key, uint32_t hist, double* sc,
                                             uint64_t* ky, uint32_t* ix, uint32_t* hh, int32_t* sScan);
template <int NT, int N>
__device__ __forceinline__ void emit_output(const DevParams& P, const DevState& S, int b, const int32_t* lengths,
                                            int32_t Tc, int32_t fin, int32_t* out_hyps, float* out_scores, double* sc,
                                            uint64_t* ky, uint32_t* ix, uint32_t* hh, int32_t* sScan);

// The best end-of-sentence mark after `word` by the synthetic scorer (the
// first of equal scores), or -1 without marks.
__device__ inline int32_t best_eos(const DevParams& P, int32_t word, double* score) {
  int32_t best = -1;
  double bs = kNegInf;
  for (int k = 0; k < P.eos_count; ++k) {
    const double v = bigram_score(P, word, P.eos_ids[k]);
    if (v > bs) {
      bs = v;
      best = P.eos_ids[k];
    }
  }
  *score = bs;
  return best;
}

// The synthetic fusion score of a history at the end of an utterance: its best
// end-of-sentence mark, where there are marks, counts with it.
__device__ inline double final_score(const DevParams& P, const HistNode& hn) {
  double f = hn.sfus;
  if (P.eos_count > 0) {
    double e;
    (void)best_eos(P, hn.word, &e);
    f += e;
  }
  return f;
}

// Stable sort of nsub sub-beams, the best score first.
__device__ __forceinline__ void rank_subs(int nsub, double* L, uint32_t* h) {
#pragma unroll
  for (int pass = 0; pass < kMaxSub - 1; ++pass) {
#pragma unroll
    for (int j = 0; j + 1 < kMaxSub; ++j) {
      if (j + 1 < nsub && L[j] < L[j + 1]) {
        const double tL = L[j];
        L[j] = L[j + 1];
        L[j + 1] = tL;
        const uint32_t th = h[j];
        h[j] = h[j + 1];
        h[j + 1] = th;
      }
    }
  }
}

// Frames [tau0, min(tau1, length)) of Alg. 1 for every stream: one workgroup
// per stream, which keeps the stream's beam in LDS from frame to frame.  Each
// frame:
//   * fan-out of every hypothesis by blank, repeat and each lexicon-valid
//     symbol (trie child mask), token / word bonuses, recombination of equal
//     prefixes by log-sum-exp, theta pruning, top-K selection (16-bit scores
//     in bins, exact rank around the boundary bin), beam update, trie-state
//     advance; hypothesis i is owned by LPB consecutive lanes: lane s of it
//     handles the extensions v = 1 + NC s .. NC (s + 1) and lane 0 also the
//     merged stay;
//   * Eq. (1) for the hypotheses that completed a word, by wavefronts of their
//     own (score_words): the (word, sub-beam) pairs are grouped by (n-gram
//     context, trie node); each group is looked up once per homophone, or, for
//     a node with many homophones, only for those the explicit-continuation
//     index lists (the others back off to their unigrams); each word's top-o
//     (four lanes per word, or a wavefront for a word with a large fully
//     looked-up group) survive lambda pruning and receive word-history nodes.
//     Meanwhile the wavefronts that hold the hypotheses recombine the next
//     frame's (one thread per hypothesis), which needs no word-level score.
//     Before, the whole workgroup went through Eq. (1) in six barrier-separated
//     steps and then through the recombination: 512 x 500 frames at K = 256
//     9.05 -> 7.39 ms, 256 x 500 at K = 64 5.21 -> 4.17, 64 x 200 at K = 32
//     2.02 -> 1.60, 100 x 333 at K = 100 with four sub-beams 4.15 -> 3.01;
//   * Eq. (2) with the synthetic scorer on fusion frames.
// After the last frame the beam goes back to global memory, and, when out_hyps
// is given, the workgroup also writes the stream's output (emit_output; out_fin:
// the end of the utterance).
// Barriers per frame: the histogram, the boundary's list, the selection, the new
// hypotheses (two when in place), and the one that joins Eq. (1) and the next
// recombination (the exact selection, where it is needed, has more).
// WPE: wavefronts per SIMD the register allocation aims for (four workgroups
// of 256 threads per CU need 4).  DB: the hypotheses are double-buffered in
// LDS; otherwise one buffer is rewritten in place (every source entry is read
// before any new entry is written), which lets two K = 256 workgroups share a
// CU.  HSF: LDS hash slots per hypothesis for the prefix keys (more slots,
// shorter linear probe chains, more LDS).  The decoder's parameters and state
// (P, S) are read from their device copy A_ in constant memory.  opts bit 0
// (kOptPhaseTimers): one thread adds the clock cycles of each phase of the
// frame to the stream's phase counters (kCntPhase0 + kPh*).  scratch: when
// given, the n-gram lookup scratch of the call's streams (scratch_layout)
// instead of the decoder's own buffers.
template <int KMAX, int LPB, int WPE, bool DB, int HSF>
__global__ __launch_bounds__(KMAX * LPB) __attribute__((amdgpu_waves_per_eu(WPE))) void k_decode(
    const KArgs LB_CONST* A_, const float* __restrict__ logits, const int32_t* __restrict__ lengths, int32_t Tc,
    int32_t tau0, int32_t tau1, int32_t out_fin, int32_t* __restrict__ out_hyps, float* __restrict__ out_scores,
    uint32_t opts, unsigned char* __restrict__ scratch) {
  // P and S are read through a pointer that is made opaque in every frame, so
  // that each field is loaded (scalar, from the constant cache) where it is
  // used instead of staying live in scalar registers across the whole loop
  const KArgs LB_CONST* A = A_;
#define P (*(const DevParams*)(&A->P))
#define S (*(const DevState*)(&A->S))

  constexpr int BLOCK = KMAX * LPB;
  // LDS hash slots for the current prefix keys: a load of at most 1/4 keeps the
  // linear probe chains short (at 1/2, a parent that is not in the beam took
  // ~2.5 probes, and the whole frame 6 % longer)
  constexpr int HS = HSF * KMAX;
  static_assert(HSF >= 4 && (HSF & (HSF - 1)) == 0, "hash slots: a power of two, load at most 1/4");
  constexpr int kIdxBits = 9;  // (never all ones: no slot equals kEmptyKey)
  static_assert(KMAX < (1 << kIdxBits) - 1, "a hash slot holds its hypothesis in kIdxBits bits");
  constexpr int NW = BLOCK / 64;
  constexpr int NC = (kSep + LPB - 1) / LPB;  // extension slots per lane
  static_assert(LPB * NC >= kSep && NC + 2 <= 32, "a lane's candidates (its slots, the stay and the repeat) fit a 32-bit set");
  // slots in pairs (p, p + NH), 16-bit scores in the halves of a register
  constexpr int NH = (NC + 1) / 2;
  static_assert(NH + 1 <= 16, "the pairs' sets: 16 bits a half");
  // the wavefronts that hold the hypotheses (one thread each), and those that
  // score completed words meanwhile: the others, as many as a beam can fill
  constexpr int RW = (KMAX + 63) / 64;
  constexpr int kWordWaves = (KMAX + kWaveWords - 1) / kWaveWords;
  // (a block of one wavefront scores them before the recombination)
  constexpr int LM0 = NW > RW ? RW : 0;
  constexpr int LMW = NW - LM0 < kWordWaves ? NW - LM0 : kWordWaves;
  // score bins of the top-K selection: 512 from K = 128 on; 256 for the smaller
  // beams' fewer candidates (512 x 500 frames at K = 256: 5.39 ms with 512, 5.54
  // with 256; 256 x 500 at K = 64: 3.21 with 256, 3.25 with 512)
  constexpr int kBinBits = KMAX >= 128 ? 9 : 8;
  constexpr int kBins = 1 << kBinBits;
  constexpr int kBinShift = 16 - kBinBits;  // of a 16-bit score
  constexpr int SEL_BYTES = kBoundaryCap * 20;
  constexpr int LM_BYTES = LMW * static_cast<int>(sizeof(LmWave));
  // K >= 128: the top F
  constexpr int FUSE_BYTES = KMAX >= 128 ? 4 * kBins + 24 * KMAX : 20 * KMAX;
  constexpr int MAX1 = SEL_BYTES > LM_BYTES ? SEL_BYTES : LM_BYTES;
  constexpr int UNI_BYTES = MAX1 > FUSE_BYTES ? MAX1 : FUSE_BYTES;
  static_assert(24 * KMAX <= UNI_BYTES, "output sort scratch");
  const int b = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int len = lengths[b];
  const int tend = len < tau1 ? len : tau1;

  __shared__ __align__(16) BeamLds<KMAX> sBeam[DB ? 2 : 1];
  // this frame's row and the next one's: classes 0..40; 41..63 are zero (slots past the separator)
  __shared__ double sD[2][64];
  // the row for the 16-bit scores: Dtop, the largest of D + bonus over symbols
  // 1..40, and every symbol's distance from it in units, 65535 at most, in the
  // order in which the lanes own them (word ln * NH + p: slots p and p + NH)
  __shared__ double sDtop[2];
  __shared__ double sQ[2];  // units per nat, nats per unit
  // the bonus of a class (beta, gamma for the separator; 0 past it): a select
  // between two parameters would be a load from global memory in every lane
  __shared__ double sBonus[64];
  __shared__ uint32_t sDq[2][LPB * NH];
  __shared__ double sAb2[KMAX], sAnb2[KMAX], sPt2[KMAX];
  __shared__ uint64_t sCut[KMAX];  // symbols whose extension went to a live hypothesis' stay
  // the prefix keys of the frame's hypotheses: inserted when the hypotheses
  // are written (in the previous frame, or when the beam is loaded), cleared
  // once this frame's parent lookups are done (the frame's later barriers
  // separate the clear from the next inserts)
  // (a slot: the key's bits from kIdxBits on, and the hypothesis below them, so
  // that one read finds both; a full match is checked against the hypothesis)
  __shared__ unsigned long long sHKey[HS];
  // top-K selection scratch; the LM step, the fusion and the output reuse it
  __shared__ __align__(16) unsigned char sSel[UNI_BYTES];
  __shared__ __align__(16) uint32_t sHisto[kBins];  // zero at the start of a frame
  __shared__ double sLvHi[kMaxLevels], sLvInv[kMaxLevels];
  __shared__ int32_t sLvBeta[kMaxLevels], sLvShift[kMaxLevels];
  __shared__ uint32_t sSelSrc[KMAX];
  // hypotheses that completed a word this frame: those of wavefront w from 64 w on
  __shared__ uint4 sEv[KMAX];
  __shared__ int32_t sEvCnt[RW];
  __shared__ double sRed[2 * NW], sRedB[2 * NW];
  __shared__ int32_t sScan[NW], sScanB[NW], sScanD[NW];
  __shared__ int32_t sBucket, sAbove, sBCount, sAthr;
  __shared__ int32_t sWild;  // the last frame (tau + 1) whose scores the 16-bit ones do not describe
  // counters: probed lines, completed words, LM queries, index lines (summed over
  // the threads at the end), expansions, fused hypotheses, lookups (added by
  // thread 0 as they occur: kept here, not in every thread's registers)
  __shared__ unsigned long long sCnt[7];
  // phase cycles of one thread (kPh*), and the last timestamp
  __shared__ unsigned long long sPhase[kPhases + 1];
  // tables of orders 2..4 and of the continuation index
  __shared__ NgramTable sTab[6];
  // the log-sum-exp's series coefficients (log1p_unit), read from LDS
  __shared__ double sAtanh[kAtanhTerms];
  const bool timing = (opts & kOptPhaseTimers) != 0;
  // closes the current phase as phase k, by a thread of the first wavefront that
  // scores words (taken after the barrier that ends the phase, or, inside Eq.
  // (1), where that wavefront is done with it)
  auto mark = [&](int k) {
    if (timing && threadIdx.x == 64 * LM0) {
      const unsigned long long now = __builtin_amdgcn_s_memtime();
      sPhase[k] += now - sPhase[kPhases];
      sPhase[kPhases] = now;
    }
  };

  double* const sBScore = reinterpret_cast<double*>(sSel);
  uint64_t* const sBKey = reinterpret_cast<uint64_t*>(sSel + kBoundaryCap * 8);
  uint32_t* const sBSrc = reinterpret_cast<uint32_t*>(sSel + kBoundaryCap * 16);
  LmWave* const sLm = reinterpret_cast<LmWave*>(sSel);
  if (tau0 >= tend) {  // no frames of this stream in the launch
    if (out_hyps)
      emit_output<BLOCK, KMAX>(P, S, b, lengths, Tc, out_fin, out_hyps, out_scores, reinterpret_cast<double*>(sSel),
                               reinterpret_cast<uint64_t*>(sSel + 8 * KMAX), reinterpret_cast<uint32_t*>(sSel + 16 * KMAX),
                               reinterpret_cast<uint32_t*>(sSel + 20 * KMAX), sScan);
    return;
  }

  const size_t gb = static_cast<size_t>(b) * P.K;
  const int O = P.O;
  const bool synth = P.fusion_source == 1;
  // parameters that every frame waits for, in scalar registers (spilled ones cost
  // a lane read, a load from the constant cache a hundred cycles and more)
  const int K = P.K;
  const double theta = P.theta;
  const bool merge_max = P.merge_max != 0;
  const TrieNode* const trie = S.trie;
  HistNode* const arena = S.arena;
  const WordRank* const wrank = S.wrank;
  const int32_t* const trie_words = S.trie_words;
  const Unigram* const uni = S.uni;
  const uint32_t heavy_min = P.heavy_min;
  const double comega = P.comega, lam = P.lam;
  const uint64_t arena_cap = S.arena_cap;
  const uint32_t word_scratch = static_cast<uint32_t>(S.scap) / static_cast<uint32_t>(P.K);  // lookup results of a word
  const bool fuse_frames = synth && P.fusion_interval > 0;
  const int64_t t0 = S.t0[b];
  const uint32_t arena0 = 1u + static_cast<uint32_t>(static_cast<uint64_t>(b) * S.arena_cap);

  // ---- the stream's beam into LDS
  // (every entry's fields with the number of entries, in one round of reads;
  // those past it are left)
  int n = S.nbeam[b];
  {
    BeamLds<KMAX>& B0 = sBeam[0];
    const size_t g = gb + tid;
    uint64_t key = 0, pkey = 0;
    double ab = 0.0, anb = 0.0, pt = 0.0, Lw[kMaxSub] = {};
    uint32_t node = 0, meta = 0, hist[kMaxSub] = {};
    if (tid < K) {
      key = S.key[g];
      pkey = S.pkey[g];
      ab = S.ab[g];
      anb = S.anb[g];
      pt = S.pt[g];
      node = S.node[g];
      meta = S.meta[g];
#pragma unroll
      for (int j = 0; j < kMaxSub; ++j) {
        if (j < O) {
          Lw[j] = S.Lw[g * O + j];
          hist[j] = S.hist[g * O + j];
        }
      }
    }
    if (tid < n) {
      const TrieNode tn = trie[node];
      B0.key[tid] = key;
      B0.pkey[tid] = pkey;
      B0.ab[tid] = ab;
      B0.anb[tid] = anb;
      B0.pt[tid] = pt;
      B0.node[tid] = node;
      B0.meta[tid] = meta;
#pragma unroll
      for (int j = 0; j < kMaxSub; ++j) {
        B0.Lw[tid * kMaxSub + j] = Lw[j];
        B0.hist[tid * kMaxSub + j] = hist[j];
      }
      B0.tmask[tid] = tn.mask;
      B0.first[tid] = tn.first_child;
      B0.woff[tid] = tn.word_off;
    }
  }
  if (tid < 7) sCnt[tid] = 0;
  if (tid < 6) {
    // (one layout for both kinds of table)
    const NgramTable& t = tid == 0 ? S.t2 : (tid == 1 ? S.t3 : S.t4);
    const PresTable& p = tid == 3 ? S.p2 : (tid == 4 ? S.p3 : S.p4);
    sTab[tid].slots = tid < 3 ? t.slots : reinterpret_cast<Slot*>(p.slots);
    sTab[tid].nbuckets = tid < 3 ? t.nbuckets : p.nbuckets;
  }
  if (tid < kAtanhTerms) sAtanh[tid] = 1.0 / (2 * tid + 3);
  if (timing && tid == 0) {
    for (int k = 0; k < kPhases; ++k) sPhase[k] = 0;
    sPhase[kPhases] = __builtin_amdgcn_s_memtime();
  }
  uint32_t arena_n = S.arena_n[b];
  int cur = 0;  // the current buffer (DB)
  for (int q = tid; q < HS; q += BLOCK) sHKey[q] = kEmptyKey;
  for (int d = tid; d < kBins; d += BLOCK) sHisto[d] = 0;
  for (int d = tid; d < 2 * LPB * NH; d += BLOCK) sDq[d / (LPB * NH)][d % (LPB * NH)] = 0xFFFFFFFFu;
  if (tid == 0) {
    sBCount = 0;
    sWild = 0;
  }
  // a new hypothesis' prefix key into the hash table, with its index r
  auto insert_key = [&](uint64_t key, int r) {
    uint32_t s = static_cast<uint32_t>(key) & (HS - 1);
    const unsigned long long entry = ((key >> kIdxBits) << kIdxBits) | static_cast<unsigned long long>(r);
    while (atomicCAS(&sHKey[s], kEmptyKey, entry) != kEmptyKey) s = (s + 1) & (HS - 1);
  };
  uint32_t lines = 0, plines = 0, c_words = 0, c_look = 0;  // per thread
  uint64_t c_queries = 0;
  const ScratchLayout slay = scratch_layout(gridDim.x, S.scap, P.K);
  double* const scrL = (scratch ? reinterpret_cast<double*>(scratch) : S.scrL) + static_cast<size_t>(b) * S.scap;
  QState* const scrS =
      (scratch ? reinterpret_cast<QState*>(scratch + slay.off_state) : S.scrS) + static_cast<size_t>(b) * S.scap;
  uint32_t* const scrE = (scratch ? reinterpret_cast<uint32_t*>(scratch + slay.off_explicit) : S.scrE) +
                         static_cast<size_t>(b) * P.K * kMaxSub * kMaxExplicit;
  if (tid < 64) sBonus[tid] = tid >= 1 && tid < kSep ? P.beta : (tid == kSep ? P.gamma : 0.0);
  if (tid == 0) {
    sQ[0] = P.qscale;
    sQ[1] = P.qunit;
  }
  // D = alpha * log-probs of a frame into row q of sD, by one wavefront (every
  // lane): raw scores are first normalised by a log-softmax over the 41 classes
  auto set_row = [&](const DevParams& Pr, int q, float xin, int lane) {
    double x = lane < kClasses ? static_cast<double>(xin) : kNegInf;
    if (Pr.raw_input) {
      double m = x, unused = x;
      wave_minmax(&m, &unused);
      const double sum = wave_sum(lane < kClasses ? exp(x - m) : 0.0);
      x = (x - m) - log(sum);
    }
    const double dv = lane < kClasses ? Pr.alpha * x : 0.0;
    sD[q][lane] = dv;
    const bool sym = lane >= 1 && lane < kClasses;
    const double db = dv + sBonus[lane];
    const double top = wave_max(sym ? db : kNegInf);
    if (lane == 0) sDtop[q] = top;
    if (sym) {
      const double u = (top - db) * sQ[0];
      const int ln = (lane - 1) / NC, k = (lane - 1) % NC;
      const int h = 2 * (ln * NH + (k < NH ? k : k - NH)) + (k < NH ? 0 : 1);
      reinterpret_cast<uint16_t*>(&sDq[q][0])[h] = u < 65535.0 ? static_cast<uint16_t>(u) : uint16_t{65535};  // (also of NaN)
    }
  };
  // the first two frames' rows now; in each frame the last wavefront loads the
  // row after the next one's early, and sets it where this frame's was, beside
  // the word scoring
  int row = 0;
  auto load_row = [&](int t, int lane) -> float {
    return lane < kClasses && t < tend ? logits[(static_cast<size_t>(b) * Tc + t) * kClasses + lane] : 0.0f;
  };
  lds_barrier();
  if (wave == 0) set_row(P, 0, load_row(tau0, lane), lane);
  if (wave == NW - 1) set_row(P, 1, load_row(tau0 + 1, lane), lane);
  float dnext = 0.0f;
  lds_barrier();
  // the loaded hypotheses' keys for the first frame, and their best total
  if (tid < n) {
    insert_key(sBeam[0].key[tid], tid);
    sCut[tid] = 0;
  }
  auto best_total = [&](const BeamLds<KMAX>& H, int nh, int tid) -> double {
    const double m = wave_max(tid < nh ? H.pt[tid] + H.Lw[tid * kMaxSub] : kNegInf);
    if ((tid & 63) == 0) sRed[tid >> 6] = m;
    lds_barrier();
    double r = sRed[0];
#pragma unroll
    for (int w = 1; w < RW; ++w) r = fmax(r, sRed[w]);
    return r;
  };
  // an upper bound of the hypotheses' totals (but for those that a word raised),
  // and whether the next selection starts with the 16-bit scores (a full beam)
  double btotal = best_total(sBeam[0], n, tid);
  bool coarse = n == P.K;
  mark(kPhOther);

  // ---- recombination of a frame's hypotheses (buffer H, log-probs D): a
  // hypothesis whose parent prefix is also live receives the parent's extension
  // by its last symbol; that extension is removed from the parent's fan-out
  // (sCut).  Stay candidates: blank-stay, repeat-stay, merged parent extension.
  // Reads nothing that Eq. (1) writes (it adds the word-level scores later), so
  // the wavefronts that hold the hypotheses run it while the others score the
  // words that the frame before completed.
  auto recombine = [&](BeamLds<KMAX>& H, const double* D, int tid, uint64_t pkey, uint32_t meta, double pt, double anb) {
    {
      const int last = meta & 0xFF;
      const double ab2 = pt + D[0];
      const double dl = D[last], bl = sBonus[last];
      const double rep = last ? anb + dl : kNegInf;
      double ext = kNegInf;
      if (pkey != kNoParent) {
        uint32_t s = static_cast<uint32_t>(pkey) & (HS - 1);
        for (int probes = 0; probes < HS; ++probes) {
          const unsigned long long e = sHKey[s];
          if (e == kEmptyKey) break;
          if (((e ^ pkey) >> kIdxBits) == 0) {
            const int par = static_cast<int>(e & ((1u << kIdxBits) - 1u));
            const uint64_t pk = H.key[par];
            const int plast = H.meta[par] & 0xFF;
            const double pab = H.ab[par], ppt = H.pt[par];
            if (pk == pkey) {
              atomicOr(reinterpret_cast<unsigned long long*>(&sCut[par]), 1ull << last);
              ext = ((last == plast ? pab : ppt) + dl) + bl;
              break;
            }
          }
          s = (s + 1) & (HS - 1);
        }
      }
      // anb2 = merge(rep, ext), then pt2 = merge(ab2, anb2); merge is
      // log-sum-exp, or max for the best-alignment recombination
      double x = rep, y = ext, anb2 = 0.0;
#pragma unroll 1
      for (int pass = 0; pass < 2; ++pass) {
        const double l = merge_max ? fmax(x, y) : lse2(x, y, [&](int k) { return sAtanh[k]; });
        if (pass == 0) {
          anb2 = l;
          x = ab2;
          y = l;
        } else {
          y = l;
        }
      }
      sAb2[tid] = ab2;
      sAnb2[tid] = anb2;
      sPt2[tid] = y;
    }
  };

  // (where the registers allow: read ahead what the ranking may need)
  constexpr bool kAhead = WPE < 4;
  // ---- Eq. (1) for the words that a frame completed (events 0..nev-1 of buffer
  // H), by one wavefront for 4 to kWaveWords words at a time: lane 4 el + j holds
  // sub-beam j of word el.  No barrier: each of the nw wavefronts that score
  // takes its own words.
  //   * a word's sub-beams of equal n-gram context share the lookups of the
  //     first of them;
  //   * round 1: the lookups of the groups with few homophones, and one task
  //     per heavy group for the continuation index; round 2: the heavy groups'
  //     listed homophones (or all, if the list is long).  A task takes four
  //     lanes, one per order and one for the unigram, so that a lane holds one
  //     64-B bucket (three of them would not fit the registers);
  //   * each lane ranks its sub-beam's candidates, the four lanes of a word
  //     merge their top-o, and lane k of them writes the k-th history node.
  // Bound by the latency of its dependent reads (history node, hash-table
  // lines, unigram order), each made by all lanes at once.
  auto score_words = [&](const DevParams& Pr, const DevState& Sr, BeamLds<KMAX>& H, int nev, int wv, int nw, int lane) {
    LmWave& W = sLm[wv];
    // words per turn: up to 4 words share a wavefront's lookups, more are spread
    int per = (nev + nw - 1) / nw;
    per = per < 4 ? 4 : (per > kWaveWords ? kWaveWords : per);
#pragma unroll 1
    for (int e0 = wv * per; e0 < nev; e0 += nw * per) {
      const int j = lane & (kMaxSub - 1);
      const int el = lane / kMaxSub;
      const int e = e0 + el;
      const bool word = el < per && e < nev;
      uint32_t rr = 0, woff = 0, Hn = 0, ph = 0;
      int nsub = 0;
      double Lw = kNegInf;
      HistNode par{};      // the pair's history node
      uint4 top0{}, top1{}, top2{}, top3{};  // a heavy word's first homophones in unigram order (WordRank)
      int32_t w0 = 0, w1 = 0;
      if (word) {
        int k = e;
#pragma unroll
        for (int w = 0, left = e; w < RW; ++w) {
          if (left >= 0 && left < sEvCnt[w]) k = 64 * w + left;
          left -= sEvCnt[w];
        }
        const uint4 ev = sEv[k];
        rr = ev.x;
        nsub = static_cast<int>(ev.y);
        woff = ev.z;
        Hn = ev.w;
      }
      const bool pair = word && j < nsub;
      const bool heavy = Hn >= heavy_min;
      if (pair) {
        ph = H.hist[rr * kMaxSub + j];
        Lw = H.Lw[rr * kMaxSub + j];
        par = arena[ph];
        w0 = trie_words[woff];
        if (Hn > 1) w1 = trie_words[woff + 1];
      }
      // (in every lane of the word: the k-th winner's node is written by lane k,
      // which may hold no sub-beam)
      if (kAhead && word && heavy) {
        const uint4* const wr = reinterpret_cast<const uint4*>(wrank + woff);
        top0 = wr[0];
        if (Hn > 1) top1 = wr[1];
        if (Hn > 2) top2 = wr[2];
        if (Hn > 3) top3 = wr[3];
      }
      const Ctx ctx = ctx_of(par);
      // the groups: the first of the word's sub-beams with the same context
      int lead = lane;
      {
        const uint64_t key = pair ? group_key(ctx, woff) : ~static_cast<uint64_t>(lane);
        const uint32_t klo = static_cast<uint32_t>(key), khi = static_cast<uint32_t>(key >> 32);
        const int q0 = lane & ~(kMaxSub - 1);
        // (every lane takes part in each move: a source lane that is masked off gives 0)
        const uint32_t l2 = quad_bcast<2>(klo), h2 = quad_bcast<2>(khi), l1 = quad_bcast<1>(klo), h1 = quad_bcast<1>(khi),
                       l0 = quad_bcast<0>(klo), h0 = quad_bcast<0>(khi);
        if (l2 == klo && h2 == khi && j > 2) lead = q0 + 2;
        if (l1 == klo && h1 == khi && j > 1) lead = q0 + 1;
        if (l0 == klo && h0 == khi && j > 0) lead = q0;
      }
      const bool leader = pair && lead == lane;
      const uint64_t below = (1ull << lane) - 1ull;
      // round 1's tasks and results (a heavy group's task has no result of its own)
      int cnt = leader ? (heavy ? 1 : static_cast<int>(Hn)) : 0;
      int incl = wave_scan_incl(cnt);
      int pos = incl - cnt;
      int U = __builtin_amdgcn_readlane(incl, 63);
      const uint64_t hleads = __ballot(leader && heavy);
      int roff = pos - __popcll(hleads & below);
      int R = U - __popcll(hleads);
      uint32_t gcnt = heavy ? kGroupHeavy : Hn;  // (leaders) lookups | kGroupHeavy
      uint64_t gmask = 0;  // (leaders) heavy: bit h mod 64 of every listed homophone h
      // a batch's results past those that LDS holds: the stream's scratch, from
      // the words before it on
      const size_t gbase = static_cast<size_t>(e0) * word_scratch;
      mark(kPhGroup);
#pragma unroll 1
      for (int round = 0; round < 2; ++round) {
#pragma unroll 1
        for (int c0 = 0; c0 < U; c0 += kWaveTasks) {
          if (leader)
            for (int q = pos > c0 ? pos : c0; q < pos + cnt && q < c0 + kWaveTasks; ++q)
              W.owner[q - c0] = static_cast<uint8_t>(lane);
          wave_sync();
          const int o = lane & 3;  // this lane's part of the task: order o + 2, or the unigram
          const bool task = c0 + lane / 4 < U;
          const int own = task ? W.owner[lane / 4] : lane;
          wave_sync();
          const uint32_t k = static_cast<uint32_t>(c0 + lane / 4 - __shfl(pos, own, 64));
          const uint32_t x1 = static_cast<uint32_t>(__shfl(ctx.word, own, 64));
          const uint32_t x2 = static_cast<uint32_t>(__shfl(static_cast<int>(ctx.c2), own, 64));
          const uint32_t x3 = static_cast<uint32_t>(__shfl(static_cast<int>(ctx.c3), own, 64));
          const uint32_t gw = static_cast<uint32_t>(__shfl(static_cast<int>(woff), own, 64));
          const uint32_t gH = static_cast<uint32_t>(__shfl(static_cast<int>(Hn), own, 64));
          const uint32_t gc = static_cast<uint32_t>(__shfl(static_cast<int>(gcnt), own, 64));
          const int a0 = __shfl(w0, own, 64), a1 = __shfl(w1, own, 64);
          uint32_t* const E = scrE + static_cast<size_t>(e0 * kMaxSub + own) * kMaxExplicit;
          const bool index = round == 0 && gH >= heavy_min;
          uint32_t id = gw;
          if (task && !index) {
            uint32_t h = k;
            if (round == 1 && (gc & kGroupHeavy)) h = E[k];
            id = static_cast<uint32_t>(h == 0 ? a0 : (h == 1 ? a1 : trie_words[gw + h]));
          }
          Unigram un{0.0f, 0.0f};
          if (task && !index && o == 3) un = uni[id];
          Hit hit{kNone, 0, 0};
          const uint32_t cid = o == 0 ? x1 : (o == 1 ? x2 : x3);
          if (task && o < 3 && (o == 0 || cid != kNone)) {
            const NgramTable tb = sTab[(index ? 3 : 0) + o];
            const uint64_t pk = (static_cast<uint64_t>(cid) << 32) | id;
            const uint64_t bk = bucket_of(pk, tb.nbuckets);
            uint32_t nl = 1;
            (void)resolve(tb, pk, bk, load_bucket(tb, bk), &hit.slot, &hit.z, &hit.y, &nl);
            lines += index ? 0u : nl;
            plines += index ? nl : 0u;
          }
          // the quad's findings in each of its lanes
          const Hit h2{quad_bcast<0>(hit.slot), quad_bcast<0>(hit.z), quad_bcast<0>(hit.y)};
          const Hit h3{quad_bcast<1>(hit.slot), quad_bcast<1>(hit.z), quad_bcast<1>(hit.y)};
          const Hit h4{quad_bcast<2>(hit.slot), quad_bcast<2>(hit.z), quad_bcast<2>(hit.y)};
          const float ulp = __uint_as_float(quad_bcast<3>(__float_as_uint(un.logp)));
          const float ubo = __uint_as_float(quad_bcast<3>(__float_as_uint(un.bo)));
          const float b1 = __shfl(ctx.bo1, own, 64), b2 = __shfl(ctx.bo2, own, 64), b3 = __shfl(ctx.bo3, own, 64);
          const int gr = __shfl(roff, own, 64);
          uint32_t tcnt = 0;
          uint64_t tmask = 0;
          if (task && o == 0) {
            if (index) {
              const uint32_t ne = h2.y + h3.y + h4.y;
              tcnt = gH;
              if (ne <= static_cast<uint32_t>(kMaxExplicit)) {
                uint32_t nd = 0;
                // each homophone once (it can be listed for several context
                // orders); the list is read back only when its mask bit is set
                auto add = [&](uint32_t x) {
                  const uint64_t bit = 1ull << (x & 63u);
                  bool seen = false;
                  if (tmask & bit)
                    for (uint32_t m = 0; m < nd; ++m) seen |= E[m] == x;
                  if (!seen) {
                    E[nd++] = x;
                    tmask |= bit;
                  }
                };
                auto add_list = [&](const Hit& h, const uint32_t* lists) {
                  if (h.y == 1) {
                    add(h.z);
                  } else {
                    for (uint32_t m = 0; m < h.y; ++m) add(lists[h.z + m]);
                  }
                };
                add_list(h2, Sr.p2.lists);
                add_list(h3, Sr.p3.lists);
                add_list(h4, Sr.p4.lists);
                tcnt = nd | kGroupHeavy;
              }
            } else {
              const LmResult res = lm_result(h2, h3, h4, b1, b2, b3, static_cast<int32_t>(id), ulp, ubo);
              const int u = gr + static_cast<int>(k);
              if (u < kLmRes) {
                W.lp[u] = res.lp;
                W.st[u] = res.st;
              } else {
                scrL[gbase + u] = res.lp;
                scrS[gbase + u] = res.st;
              }
            }
          }
          if (round == 0) {
            // the index's findings back to the groups' leaders
            const int at = pos - c0;
            const bool mine = leader && heavy && at >= 0 && at < kWaveTasks;
            const int src = (4 * at) & 63;
            const uint32_t fc = static_cast<uint32_t>(__shfl(static_cast<int>(tcnt), src, 64));
            const uint32_t fl = static_cast<uint32_t>(__shfl(static_cast<int>(tmask), src, 64));
            const uint32_t fh = static_cast<uint32_t>(__shfl(static_cast<int>(tmask >> 32), src, 64));
            if (mine) {
              gcnt = fc;
              gmask = fl | (static_cast<uint64_t>(fh) << 32);
            }
          }
        }
        if (lane == 0) c_look += static_cast<uint32_t>(round == 0 ? R : U);
        if (round == 0) {
          // round 2: the heavy groups' lookups
          cnt = (leader && heavy) ? static_cast<int>(gcnt & ~kGroupHeavy) : 0;
          incl = wave_scan_incl(cnt);
          pos = incl - cnt;
          U = __builtin_amdgcn_readlane(incl, 63);
          if (leader && heavy) roff = R + pos;
          if (U > 0) {  // the lists (global memory) are read by other lanes
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
          }
        }
      }
      R += U;
      if (R > kLmRes) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      }
      wave_sync();
      mark(kPhLookup);
      auto res_lp = [&](int u) -> double { return u < kLmRes ? W.lp[u] : scrL[gbase + u]; };
      // the pair's group: result offset, lookups, mask of the listed homophones
      const int off = __shfl(roff, lead, 64);
      const uint32_t gc = static_cast<uint32_t>(__shfl(static_cast<int>(gcnt), lead, 64));
      const uint64_t gm = static_cast<uint32_t>(__shfl(static_cast<int>(gmask), lead, 64)) |
                          (static_cast<uint64_t>(static_cast<uint32_t>(__shfl(static_cast<int>(gmask >> 32), lead, 64))) << 32);
      const uint32_t* const E = scrE + static_cast<size_t>(e0 * kMaxSub + lead) * kMaxExplicit;
      const bool full = pair && !(gc & kGroupHeavy);
      const bool walk = pair && (gc & kGroupHeavy);
      // a word with a group looked up in full over many homophones is ranked by
      // the whole wavefront below, any other by its four lanes
      const uint64_t manyb = __ballot(full && Hn > kLaneMaxH);
      const bool many = ((manyb >> (lane & ~(kMaxSub - 1))) & ((1ull << kMaxSub) - 1ull)) != 0;
      // this lane's best o: score, j << 16 | h (the order of equal scores), and
      // the source: its lookup result (>= 0), or, for a homophone that backs off
      // to its unigram in a heavy group, -1 - its rank in unigram order
      double tL[kMaxSub];
      int tq[kMaxSub], ts[kMaxSub];
#pragma unroll
      for (int k = 0; k < kMaxSub; ++k) {
        tL[k] = kNegInf;
        tq[k] = kNoCandidate;
        ts[k] = 0;
      }
      auto insert = [&](double L, int qq, int ss) {
#pragma unroll
        for (int k = 0; k < kMaxSub; ++k) {
          if (k < O && (L > tL[k] || (L == tL[k] && qq < tq[k]))) {
            const double t = tL[k];
            const int u = tq[k], v = ts[k];
            tL[k] = L;
            tq[k] = qq;
            ts[k] = ss;
            L = t;
            qq = u;
            ss = v;
          }
        }
      };
      // Katz backoff to the unigram
      auto unigram_score = [&](const Ctx& c, double lw, float logp) -> double {
        const double lp = static_cast<double>(c.bo3) +
                          (static_cast<double>(c.bo2) + (static_cast<double>(c.bo1) + static_cast<double>(logp)));
        return lw + comega * lp;
      };
      // A candidate put at an empty list's head without a comparison: a score that
      // is no number (omega = 0 times a log10 P of -inf) counts as -inf there, as no
      // comparison would ever move it.  (insert leaves such a candidate out.)
      auto head = [&](double L) -> double { return fmax(L, kNegInf); };
      // the word's k-th homophone in unigram order
      auto ranked = [&](uint32_t k) -> WordRank {
        auto pick = [&](uint32_t a, uint32_t b, uint32_t c, uint32_t d) -> uint32_t {
          return k < 2 ? (k == 0 ? a : b) : (k == 2 ? c : d);
        };
        uint4 v = {pick(top0.x, top1.x, top2.x, top3.x), pick(top0.y, top1.y, top2.y, top3.y),
                   pick(top0.z, top1.z, top2.z, top3.z), pick(top0.w, top1.w, top2.w, top3.w)};
        if (!kAhead || k >= kTopWords) v = reinterpret_cast<const uint4*>(wrank + woff)[k];
        return __builtin_bit_cast(WordRank, v);
      };
      if (!many && pair) {
        const int nl = static_cast<int>(gc & ~kGroupHeavy);
        // (the first candidate of an empty list is put there)
        if (nl > 0) {
          tL[0] = head(Lw + comega * res_lp(off));
          tq[0] = (j << 16) | static_cast<int>(walk ? E[0] : 0u);
          ts[0] = off;
        }
#pragma unroll 1
        for (int m = 1; m < nl; ++m)
          insert(Lw + comega * res_lp(off + m), (j << 16) | static_cast<int>(walk ? E[m] : static_cast<uint32_t>(m)), off + m);
        if (walk) {
          // the heavy group's other homophones in unigram order (scores
          // non-increasing), until its o-th such candidate scores strictly
          // above the next word's
          int got = 0;
          double Lth = HUGE_VAL;
          uint32_t k = 0;
          if (nl == 0) {
            const WordRank wr = ranked(0);
            tL[0] = head(unigram_score(ctx, Lw, wr.logp));
            tq[0] = (j << 16) | static_cast<int>(wr.h);
            ts[0] = -1;
            got = 1;
            if (O == 1) Lth = tL[0];
            k = 1;
          }
#pragma unroll 1
          for (; k < Hn; ++k) {
            const WordRank wr = ranked(k);
            const double L = unigram_score(ctx, Lw, wr.logp);
            if (got >= O && Lth > L) break;
            bool member = false;
            if ((gm >> (wr.h & 63u)) & 1ull)
              for (int m = 0; m < nl; ++m) member |= E[m] == wr.h;
            if (!member) {
              insert(L, (j << 16) | static_cast<int>(wr.h), -1 - static_cast<int>(k));
              got += 1;
              if (got == O) Lth = L;
            }
          }
        }
      }
      // o rounds of an arg-max over the word's four lanes; lane k keeps the k-th
      // winner; lambda is relative to the best.  A word whose every reading scores
      // -inf keeps them: its hypothesis is never a candidate again, unless a fusion
      // scores it anew, but it has sub-beams and their histories, as every one has
      double myL = kNegInf, bestL = kNegInf;
      int myq = 0, mys = 0, kept = 0;
      bool open = true;
#pragma unroll
      for (int k = 0; k < kMaxSub; ++k) {
        if (k < O) {
          // the best head; of equal ones the first in (sub-beam, homophone) order
          double m4 = fmax(tL[0], dpp_f64<kDppXor1>(tL[0], kNegInf));
          m4 = fmax(m4, dpp_f64<kDppXor2>(m4, kNegInf));
          int q4 = tL[0] == m4 ? tq[0] : kNoCandidate;
          q4 = min(q4, dpp_i32<kDppXor1>(q4, kNoCandidate));
          q4 = min(q4, dpp_i32<kDppXor2>(q4, kNoCandidate));
          const bool win = tL[0] == m4 && tq[0] == q4;
          int s4 = win ? ts[0] : 0;
          s4 |= dpp_i32<kDppXor1>(s4, 0);
          s4 |= dpp_i32<kDppXor2>(s4, 0);
          if (k == 0) bestL = m4;
          open = open && q4 != kNoCandidate && !(m4 < bestL - lam);
          if (open) {
            if (j == k) {
              myL = m4;
              myq = q4;
              mys = s4;
            }
            kept = k + 1;
          }
          if (win) {
#pragma unroll
            for (int m = 0; m + 1 < kMaxSub; ++m) {
              tL[m] = tL[m + 1];
              tq[m] = tq[m + 1];
              ts[m] = ts[m + 1];
            }
            tL[kMaxSub - 1] = kNegInf;
            tq[kMaxSub - 1] = kNoCandidate;
          }
        }
      }
      // words ranked by the whole wavefront: lane h reads homophone h
#pragma unroll 1
      for (uint64_t left = manyb; left;) {
        const int l0 = __builtin_ctzll(left) & ~(kMaxSub - 1);  // the word's first lane
        left &= ~(((1ull << kMaxSub) - 1ull) << l0);
        const int xn = __builtin_amdgcn_readlane(nsub, l0);
        const int xH = __builtin_amdgcn_readlane(static_cast<int>(Hn), l0);
        const uint32_t xw = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(woff), l0));
        double sL[kMaxSub];
        int sq[kMaxSub], ss[kMaxSub];
#pragma unroll
        for (int k = 0; k < kMaxSub; ++k) {
          sL[k] = kNegInf;
          sq[k] = kNoCandidate;
          ss[k] = 0;
        }
        auto put = [&](double L, int qq, int sr) {
#pragma unroll
          for (int k = 0; k < kMaxSub; ++k) {
            if (k < O && (L > sL[k] || (L == sL[k] && qq < sq[k]))) {
              const double t = sL[k];
              const int u = sq[k], v = ss[k];
              sL[k] = L;
              sq[k] = qq;
              ss[k] = sr;
              L = t;
              qq = u;
              sr = v;
            }
          }
        };
#pragma unroll 1
        for (int jj = 0; jj < xn; ++jj) {
          const double lw = readlane_f64(Lw, l0 + jj);
          const uint32_t xc = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(gc), l0 + jj));
          const int xo = __builtin_amdgcn_readlane(off, l0 + jj);
          if (!(xc & kGroupHeavy)) {
            for (int h = lane; h < xH; h += 64) put(head(lw + comega * res_lp(xo + h)), (jj << 16) | h, xo + h);
          } else {
            // lane m holds the m-th listed homophone, a candidate with its
            // looked-up score; the others in unigram order, 64 at a time, until
            // the sub-beam has o candidates strictly above all that remain
            const int xl = __builtin_amdgcn_readlane(lead, l0 + jj);
            const int ne = static_cast<int>(xc & ~kGroupHeavy);
            uint32_t eh = kNone;
            if (lane < ne) {
              eh = scrE[static_cast<size_t>(e0 * kMaxSub + xl) * kMaxExplicit + lane];
              put(head(lw + comega * res_lp(xo + lane)), (jj << 16) | static_cast<int>(eh), xo + lane);
            }
            Ctx cx{};
            cx.bo1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(ctx.bo1), l0 + jj));
            cx.bo2 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(ctx.bo2), l0 + jj));
            cx.bo3 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(ctx.bo3), l0 + jj));
            int cum = 0;
#pragma unroll 1
            for (int c0 = 0; c0 < xH; c0 += 64) {
              const int k = c0 + lane;
              const bool valid = k < xH;
              WordRank wr = WordRank{0, 0.0f, 0.0f, kNone};
              if (valid) wr = wrank[xw + k];
              const int last = (xH - 1 - c0) < 63 ? xH - 1 - c0 : 63;
              bool member = false;
              for (int m = 0; m < ne; ++m)
                member |= static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(eh), m)) == wr.h;
              const double L = unigram_score(cx, lw, wr.logp);
              const bool cand = valid && !member;
              if (cand) put(head(L), (jj << 16) | static_cast<int>(wr.h), -1 - k);
              const double lastL = readlane_f64(L, last);
              cum += __popcll(__ballot(cand && L > lastL));
              if (cum >= O) break;
            }
          }
        }
        // o rounds of wavefront arg-max; lane l0 + k keeps the k-th winner
        double xbest = kNegInf;
        int xkept = 0;
#pragma unroll 1
        for (int k = 0; k < O; ++k) {
          double bL = sL[0];
          int bq = sq[0];
          wave_argmax(&bL, &bq);
          if (bq == kNoCandidate) break;
          if (k == 0) xbest = bL;
          if (bL < xbest - lam) break;
          const bool holder = sL[0] == bL && sq[0] == bq;  // one lane: queries are distinct
          const int hl = __builtin_ctzll(__ballot(holder));
          const int bs = __builtin_amdgcn_readlane(ss[0], hl);
          if (lane == l0 + k) {
            myL = bL;
            myq = bq;
            mys = bs;
          }
          if (holder) {
#pragma unroll
            for (int m = 0; m + 1 < kMaxSub; ++m) {
              sL[m] = sL[m + 1];
              sq[m] = sq[m + 1];
              ss[m] = ss[m + 1];
            }
            sL[kMaxSub - 1] = kNegInf;
            sq[kMaxSub - 1] = kNoCandidate;
          }
          xkept = k + 1;
        }
        if ((lane & ~(kMaxSub - 1)) == l0) kept = xkept;
      }
      // history nodes (o reserved per word, in order), one lane per kept sub-beam
      const bool room = static_cast<uint64_t>(arena_n) + static_cast<uint64_t>(e + 1) * O <= arena_cap;
      // (the parent: the history node of the winner's sub-beam, in that lane)
      const int pl = (lane & ~(kMaxSub - 1)) + ((myq >> 16) & (kMaxSub - 1));
      const uint32_t pn = static_cast<uint32_t>(__shfl(static_cast<int>(ph), pl, 64));
      HistNode pr;
      if constexpr (kAhead) {
        pr.blk = static_cast<uint32_t>(__shfl(static_cast<int>(par.blk), pl, 64));
        pr.depth = static_cast<uint32_t>(__shfl(static_cast<int>(par.depth), pl, 64));
        pr.word = __shfl(par.word, pl, 64);
        pr.sfus = __shfl(par.sfus, pl, 64);
#pragma unroll
        for (int i = 0; i < kHistBlock - 2; ++i) pr.w[i] = __shfl(par.w[i], pl, 64);
      } else if (word && room && j < kept) {
        pr = arena[pn];
      }
      if (word && room && j < kept) {
        QState st;
        if (mys >= 0) {
          st = mys < kLmRes ? W.st[mys] : scrS[gbase + mys];
        } else {
          const WordRank wr = ranked(static_cast<uint32_t>(-1 - mys));
          st.c2 = kNone;
          st.c3 = kNone;
          st.bo2 = 0.0f;
          st.bo3 = 0.0f;
          st.w = wr.w;
          st.bo1 = wr.bo;
        }
        HistNode hn;
        hn.word = st.w;
        hn.c2 = st.c2;
        hn.c3 = st.c3;
        hn.bo1 = st.bo1;
        hn.bo2 = st.bo2;
        hn.bo3 = st.bo3;
        hn.depth = pr.depth + 1;
        hn.sfus = synth ? pr.sfus + bigram_score(Pr, pr.word, st.w) : 0.0;
        // a parent that ends a block (the root included) starts a new one
        const bool starts = pr.depth % kHistBlock == 0;
        hn.blk = starts ? pn : pr.blk;
        hn.w[0] = starts ? -1 : pr.word;
#pragma unroll
        for (int i = 1; i < kHistBlock - 1; ++i) hn.w[i] = starts ? -1 : pr.w[i - 1];
        const uint32_t node = arena0 + arena_n + static_cast<uint32_t>(e * O + j);
        arena[node] = hn;
        H.Lw[rr * kMaxSub + j] = myL;
        H.hist[rr * kMaxSub + j] = node;
      }
      if (word && j == 0) {
        if (room)
          H.meta[rr] = (H.meta[rr] & 0xFFu) | (static_cast<uint32_t>(kept) << 8);
        else
          atomicOr(Sr.flags, kFlagArena);
        c_words += 1;
        c_queries += static_cast<uint64_t>(nsub) * Hn;
      }
      wave_sync();
      mark(kPhRank);
    }
  };

  // the first frame's hypotheses
  if (tid < n) recombine(sBeam[0], sD[0], tid, sBeam[0].pkey[tid], sBeam[0].meta[tid], sBeam[0].pt[tid], sBeam[0].anb[tid]);
  lds_barrier();
  mark(kPhRecomb);
  // frames until the next fusion frame (t > 0, a multiple of the interval); counted
  // down, as a 64-bit remainder in every frame took hundreds of cycles
  const int fuse_every = fuse_frames ? P.fusion_interval : 0x7FFFFFFF;
  int fuse_in = 0x7FFFFFFF;
  if (fuse_frames) {
    const int64_t t = t0 + tau0;
    const int past = static_cast<int>(t % fuse_every);
    fuse_in = t > 0 && past == 0 ? 0 : fuse_every - past;
  }

  for (int tau = tau0; tau < tend; ++tau) {
    // the thread index is made opaque to the optimizer in every frame so that
    // values derived from it are not hoisted out of the loop (they would stay
    // live in registers across all frames)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    asm volatile("" : "+s"(A));
    const int lane = tid & 63;
    const int wave = tid >> 6;
    BeamLds<KMAX>& C = sBeam[DB ? cur : 0];        // the frame's hypotheses (recombined)
    BeamLds<KMAX>& N = sBeam[DB ? (cur ^ 1) : 0];  // the new ones (the same buffer when !DB)
    const double* const Dc = sD[row];              // the frame's scaled log-probs
    const bool more = tau + 1 < tend;
    const bool fuses = fuse_in == 0;
    fuse_in = fuses ? fuse_every - 1 : fuse_in - 1;

    if (wave == NW - 1) dnext = load_row(tau + 2, lane);
    for (int s = tid; s < HS; s += BLOCK) sHKey[s] = kEmptyKey;  // for the new hypotheses' keys
    // Workgroups that share a CU: the CU's arbitration favours the older
    // wavefronts, so the workgroup dispatched second (the later half of the
    // grid, when workgroups are dispatched to the CUs in order) falls behind
    // and the launch waits for it.  It gets the higher issue priority in 3
    // frames of 4, the first one in the 4th (512 x 500 frames at K = 256: 5.21
    // ms against 5.46 without; 5.16 against 5.26 with turns 1:1; 1024 streams in
    // ten calls at K = 64 the same within 0.2 %).  This holds up to the word
    // scoring: its wavefronts then go to 2 and stay there until their next
    // frame starts, through a fusion and, in the instance of one wavefront,
    // through the recombination.
    if ((blockIdx.x >= gridDim.x / 2) ? (tau & 3) != 0 : (tau & 3) == 0)
      __builtin_amdgcn_s_setprio(1);
    else
      __builtin_amdgcn_s_setprio(0);


    // ---- this lane's candidates: slot k is the extension by v = 1 + NC * ln + k,
    // plus the merged stay on lane 0 and the repeat extension (the hypothesis'
    // last symbol again, from its blank-ending part) on the lane of its symbol,
    // whose slot is then left out of the slots, which all start from pt.  Exact
    // scores are computed where they are needed, from LDS (same operations, same
    // result): kept in registers across the barriers they would spill in the
    // 128-register instances.  (A lane past the last hypothesis reads what is
    // there and has no candidates: one round of reads, no branch.)
    const int hi_ = tid / LPB;
    const int ln = tid - hi_ * LPB;
    const bool live = hi_ < n;
    const int last_ = static_cast<int>(C.meta[hi_] & 0x3F);  // (a class; in range also of what lies past the last hypothesis)
    // bit k: slot k is an extension (the trie mask is cut to bits 1..40, its
    // bits 48..63 hold the node's word count)
    uint32_t c_val = static_cast<uint32_t>((C.tmask[hi_] & ~sCut[hi_] & ((2ull << kSep) - 1ull)) >> (1 + NC * ln)) & ((1u << NC) - 1u);
    c_val = live ? c_val : 0u;
    const int rk = last_ - 1 - NC * ln;
    const uint32_t rbit = static_cast<unsigned>(rk) < static_cast<unsigned>(NC) ? 1u << (rk & 31) : 0u;
    const bool stays = live && ln == 0, reps = (c_val & rbit) != 0;
    c_val &= ~rbit;
    // position k of the lane: slot k (k < NC), the stay (NC), the repeat (NC + 1)
    auto pos_v = [&](int k) -> int {
      const int v = k == NC + 1 ? last_ : 1 + NC * ln + k;
      return k == NC ? 0 : v;
    };
    auto pos_score = [&](int k) -> double {
      const double* const b = k == NC ? sPt2 : (k == NC + 1 ? C.ab : C.pt);
      const int x = k == NC ? kClasses : pos_v(k);  // (class 41: nothing added, no bonus)
      return ((b[hi_] + Dc[x]) + sBonus[x]) + C.Lw[hi_ * kMaxSub];
    };
    auto key_of = [&](int v) -> uint64_t {
      const uint64_t k = C.key[hi_];
      return v == 0 ? k : prefix_step(k, v);
    };
    // The bin that holds the need-th candidate of sHisto, the candidates above
    // and in it (bin kBins: fewer than need candidates), and a bin that no
    // candidate lies above.  Every wavefront scans the bins, kBins / 64 per
    // lane, and has the result in scalar registers: one scan and a barrier for
    // its result took twice as long.
    struct Found {
      int bin, above, count, top;
    };
    auto find_bin = [&](int need_in) -> Found {
      constexpr int PERW = kBins / 64;
      static_assert(PERW % 4 == 0, "bins per lane in 16-B loads");
      int h[PERW];
      const uint4* hp = reinterpret_cast<const uint4*>(sHisto + lane * PERW);
#pragma unroll
      for (int q = 0; q < PERW / 4; ++q) {
        const uint4 x4 = hp[q];
        h[4 * q] = static_cast<int>(x4.x);
        h[4 * q + 1] = static_cast<int>(x4.y);
        h[4 * q + 2] = static_cast<int>(x4.z);
        h[4 * q + 3] = static_cast<int>(x4.w);
      }
      int local = 0;
#pragma unroll
      for (int q = 0; q < PERW; ++q) local += h[q];
      const int incl = wave_scan_incl(local);
      const int before = incl - local;
      const uint64_t some = __ballot(local > 0);
      const uint64_t hit = __ballot(before < need_in && incl >= need_in);
      // this lane's bin, were it the one: the first q whose sum reaches need_in
      int bin = 0, above = before, count = h[0];
#pragma unroll
      for (int q = 1, acc = before; q < PERW; ++q) {
        acc += h[q - 1];
        const bool past = acc < need_in;
        bin = past ? q : bin;
        above = past ? acc : above;
        count = past ? h[q] : count;
      }
      Found f{kBins, 0, 0, some ? static_cast<int>(__builtin_ctzll(some)) * PERW : 0};
      if (hit) {
        const int l = __builtin_ctzll(hit);
        f.bin = l * PERW + __builtin_amdgcn_readlane(bin, l);
        f.above = __builtin_amdgcn_readlane(above, l);
        f.count = __builtin_amdgcn_readlane(count, l);
      }
      return f;
    };
    int nsel = 0;
    bool done = false;

    // ---- top-K by 16-bit scores: a candidate's distance below a reference, in
    // units of sQ[1] nats, as the sum of its hypothesis' and its symbol's,
    // both rounded down -- two slots in one saturating packed addition, where
    // the 64-bit score and its bin took a dozen instructions per slot and first
    // needed the range of the scores, a reduction over the workgroup.  (With
    // it, and everything read from LDS without branches, the frame's top-K went
    // from 14.7 k to 10.5 k cycles at K = 256, 7.6 k to 6.2 k at K = 32; 512 x
    // 500 frames at K = 256 7.39 -> 5.86 ms, 256 x 500 at K = 64 4.17 -> 3.62.)
    // The distance is at
    // most 2 units above the 16-bit score (and less than one more for the
    // rounding of the 64-bit sums, all below 1e9 here: a lower word-level score,
    // or one of -inf, puts its candidates past the 16 bits).  So with the K-th
    // candidate in bin b of 2^kBinShift units, every candidate 3 units before
    // the bin is selected, none 3 units past it is, and those between, ranked
    // exactly by (score desc, key asc), fill the rest.
    // The reference bounds every candidate from above: the beam's best total
    // plus the best that this frame can add (its blank, or its best symbol with
    // its bonus, and log 3 for the paths that a stay sums).  Where it does not
    // (a word raised a hypothesis; scores or bonuses of 1e9), where fewer than K candidates
    // are within the 16 bits, where theta may cut or the bin is crowded, the
    // exact selection below takes the frame.
    double ref = 0.0;
    if (coarse) {
      ref = btotal + (fmax(sDtop[row], Dc[0]) + 1.2);
      done = fabs(ref) < 1e9;
    }
    if (done) {
      typedef unsigned short us2 __attribute__((ext_vector_type(2)));
      constexpr int NP = NH + 1;  // the pairs of slots, and (stay, repeat)
      const double qscale = sQ[0];
      const double p = C.pt[hi_], lw = C.Lw[hi_ * kMaxSub], dtop = sDtop[row];
      const double sc_s = sPt2[hi_] + lw;
      const double sc_r = ((C.ab[hi_] + Dc[last_]) + sBonus[last_]) + lw;
      const double base = (p + lw) + dtop;
      us2 q2[NP];
#pragma unroll
      for (int w = 0; w < NH; ++w) q2[w] = __builtin_bit_cast(us2, sDq[row][ln * NH + w]);
      auto units = [&](double sc) -> uint32_t { return static_cast<uint32_t>(fmin(fmax((ref - sc) * qscale, 0.0), 65535.0)); };
      const uint32_t bq = units(base), qs = units(sc_s), qr = units(sc_r);
      const bool wild = !(fabs(p) < 1e9 && lw < 1e9 && base <= ref) || (stays && !(sc_s <= ref)) || (reps && !(sc_r <= ref));
      if (live && wild) sWild = tau + 1;
      const us2 b2 = __builtin_bit_cast(us2, bq | (bq << 16));
#pragma unroll
      for (int w = 0; w < NH; ++w) q2[w] = __builtin_elementwise_add_sat(b2, q2[w]);
      q2[NH] = __builtin_bit_cast(us2, qs | (qr << 16));
      // the candidates as bits in the pairs' order: slot w at bit w, slot w + NH
      // at bit 16 + w, the stay at bit NH, the repeat at bit 16 + NH
      const uint32_t vbits = (c_val & ((1u << NH) - 1u)) | ((c_val >> NH) << 16) | (stays ? 1u << NH : 0u) |
                             (reps ? 1u << (16 + NH) : 0u);
      // (what lies past the 16 bits counts in the last bin, which is never used)
#pragma unroll
      for (int w = 0; w < NP; ++w) {
        const uint32_t x = __builtin_bit_cast(uint32_t, q2[w]);
        if (vbits & (1u << w)) atomicAdd(&sHisto[(x & 0xFFFFu) >> kBinShift], 1u);
        if (w == NH || w + NH < NC) {
          if (vbits & (1u << (16 + w))) atomicAdd(&sHisto[x >> (16 + kBinShift)], 1u);
        }
      }
      lds_barrier();
      const double qunit = sQ[1];
      const Found f = find_bin(K);
      const int bk = f.bin;
      // no candidate scores above top, the K-th at least low
      const double top = ref - static_cast<double>(f.top << kBinShift) * qunit;
      const double low = ref - static_cast<double>(((bk + 1) << kBinShift) + 4) * qunit;
      done = bk < kBins - 1 && sWild != tau + 1 && low >= top - theta;
      if (done) {
        const int ta = (bk << kBinShift) - 3;         // selected: below ta
        const int tb = ((bk + 1) << kBinShift) + 3;   // not selected: tb and above
        const uint32_t ua = static_cast<uint32_t>(ta < 0 ? 0 : ta), ub = static_cast<uint32_t>(tb);
        const uint32_t a2 = ua | (ua << 16), c2 = ub | (ub << 16);
        uint32_t sel = 0, amb = 0;
#pragma unroll
        for (int w = 0; w < NP; ++w) {
          sel |= pk_below(__builtin_bit_cast(uint32_t, q2[w]), a2) << w;
          amb |= pk_below(__builtin_bit_cast(uint32_t, q2[w]), c2) << w;
        }
        sel &= vbits;
        amb &= vbits & ~sel;
        // set bit -> position of the lane
        auto pos_of = [&](int bit) -> int {
          const int w = bit & 15, h = bit >> 4;
          return w == NH ? NC + h : w + h * NH;
        };
        const int cnt = __popc(sel);
        const int incl = wave_scan_incl(cnt);
        if (lane == 63) sScanB[wave] = incl;
#pragma unroll 1
        for (uint32_t m = amb; m; m &= m - 1) {
          const int k = pos_of(__ffs(m) - 1);
          const int v = pos_v(k);
          const int slot = atomicAdd(&sBCount, 1);
          const double sc = pos_score(k);
          const uint64_t key = key_of(v);
          if (slot < kBoundaryCap) {
            sBScore[slot] = sc;
            sBKey[slot] = key;
            sBSrc[slot] = static_cast<uint32_t>(hi_) | (static_cast<uint32_t>(v) << 16);
          }
        }
        lds_barrier();
        int wpos = incl - cnt, nsure = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const int c = sScanB[w];
          wpos += w < wave ? c : 0;
          nsure += c;
        }
        const int nbc = sBCount;
        const int need = K - nsure;
        done = nbc <= kBoundaryCap && need >= 0 && need <= nbc;
        if (done) {
#pragma unroll 1
          for (uint32_t m = sel; m; m &= m - 1) {
            const uint32_t v = static_cast<uint32_t>(pos_v(pos_of(__ffs(m) - 1)));
            sSelSrc[wpos++] = static_cast<uint32_t>(hi_) | (v << 16);
          }
          // eight lanes per candidate of the list share the count of those that
          // rank before it
          for (int m = tid >> 3; m < nbc; m += BLOCK / 8) {
            const double sc = sBScore[m];
            const uint64_t key = sBKey[m];
            int rank = 0;
            for (int u = tid & 7; u < nbc; u += 8) {
              const double su = sBScore[u];
              const uint64_t ku = sBKey[u];
              rank += (su > sc || (su == sc && ku < key)) ? 1 : 0;
            }
            rank += dpp_i32<kDppXor1>(rank, 0);
            rank += dpp_i32<kDppXor2>(rank, 0);
            rank += dpp_i32<kDppHalfMirror>(rank, 0);
            if ((tid & 7) == 0 && rank < need) sSelSrc[nsure + rank] = sBSrc[m];
          }
          nsel = K;
          btotal = top;
        }
      }
    }
    if (!done) {
    // ---- top-K and the theta cut, exactly.  A first pass finds the best and the
    // lowest candidate; level 0 bins the candidates within theta of the best by
    // (best - score) into kBins; the map is monotone, so bins above the one
    // holding the K-th candidate are taken whole.  That bin is resolved exactly
    // by rank on (score desc, key asc) when it holds at most kBoundaryCap
    // candidates; otherwise it is re-binned over its own score range (deeper
    // levels), and when its scores are all equal, by the bits of the key
    // (smaller key first).
    lds_barrier();  // the coarse selection's reads are done
    for (int d = tid; d < kBins; d += BLOCK) sHisto[d] = 0;
    if (tid == 0) sBCount = 0;
    double best;
    double c_p = kNegInf, c_L = 0.0, c_stay = kNegInf, c_rps = kNegInf;
    if (live) {
      c_p = C.pt[hi_];
      c_L = C.Lw[hi_ * kMaxSub];
      if (stays) c_stay = pos_score(NC);
      if (reps) c_rps = pos_score(NC + 1);
    }
    // the separator can only be slot (kSep - 1) % NC of lane (kSep - 1) / NC
    const double bon_ph = P.beta, bon_sep = P.gamma;
    auto score_now = [&](int k) -> double {
      const bool sep = k == (kSep - 1) % NC && ln == (kSep - 1) / NC;
      const double sc = ((c_p + Dc[1 + NC * ln + k]) + (sep ? bon_sep : bon_ph)) + c_L;
      return ((c_val >> k) & 1u) ? sc : kNegInf;
    };
    double mx = fmax(c_stay, c_rps);
    double mn = fmin(c_stay != kNegInf ? c_stay : HUGE_VAL, c_rps != kNegInf ? c_rps : HUGE_VAL);
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const double sc = score_now(k);
      mx = fmax(mx, sc);
      mn = fmin(mn, sc != kNegInf ? sc : HUGE_VAL);
    }
    double lowest;
    block_minmax<BLOCK, false>(mx, mn, sRed, &best, &lowest);
    const double U = best, L0 = fmax(best - theta, lowest);
    const double inv0 = U > L0 ? static_cast<double>(kBins) / (U - L0) : 0.0;
    const int shift0 = U > L0 ? -1 : 64 - kBinBits;
    auto bin_score = [&](double hi, double inv, double s) -> int {
      const double x = (hi - s) * inv;
      return x >= static_cast<double>(kBins - 1) ? kBins - 1 : static_cast<int>(x);
    };
    // level 0: (U - s) * inv0 as one fused multiply-add of s, clamped to the
    // bins; each step rounds monotonically, so a higher score never takes a
    // higher bin
    const double ninv0 = -inv0, uinv0 = U * inv0;
    auto bin_lv0 = [&](double s) -> int {
      return static_cast<int>(fmax(fmin(fma(s, ninv0, uinv0), static_cast<double>(kBins - 1)), 0.0));
    };
    auto bin0 = [&](int v, double s) -> int {
      return shift0 < 0 ? bin_lv0(s) : static_cast<int>((key_of(v) >> shift0) & (kBins - 1));
    };
    // deeper levels (rare): parameters in LDS
    auto bin_at = [&](int l, int v, double s) -> int {
      const int sh = sLvShift[l];
      if (sh >= 0) return static_cast<int>((key_of(v) >> sh) & (kBins - 1));
      return bin_score(sLvHi[l], sLvInv[l], s);
    };
    // level-0 bin of each of the lane's candidates, kept packed 16 bits per slot
    // (0xFFFF: no candidate); exact scores are recomputed only inside the boundary bin
    uint32_t binp[(NC + 1) / 2];
    uint32_t bin_stay = 0xFFFFu, bin_rep = 0xFFFFu;
    if (c_stay >= L0) bin_stay = static_cast<uint32_t>(bin0(0, c_stay));  // (-inf: no stay)
    if (c_rps >= L0) bin_rep = static_cast<uint32_t>(bin0(pos_v(NC + 1), c_rps));
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const double sc = score_now(k);
      const uint32_t bn = sc >= L0 ? static_cast<uint32_t>(bin0(1 + NC * ln + k, sc)) : 0xFFFFu;
      if (k & 1)
        binp[k >> 1] |= bn << 16;
      else
        binp[k >> 1] = bn;
    }
    if (bin_stay != 0xFFFFu) atomicAdd(&sHisto[bin_stay], 1u);
    if (bin_rep != 0xFFFFu) atomicAdd(&sHisto[bin_rep], 1u);
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const uint32_t bn = (binp[k >> 1] >> ((k & 1) * 16)) & 0xFFFFu;
      if (bn != 0xFFFFu) atomicAdd(&sHisto[bn], 1u);
    }
    lds_barrier();
    const Found f0 = find_bin(K);
    // the K-th candidate's bin is resolved, or every binned candidate is selected
    int beta0 = kBins, nlev = 1, need = 0, nbc = 0, cntb = 0;
    bool all_bin = false;
    const bool resolve = f0.bin < kBins;
    if (resolve) {
      beta0 = f0.bin;
      need = K - f0.above;
      cntb = f0.count;
    }
    // level 0 decides every candidate outside the boundary bin: above it taken,
    // below it dropped; bnd marks this lane's candidates inside it
    uint32_t sel_bits = 0, bnd = 0;  // bit k: position k
    auto classify = [&](uint32_t bn, int bit) {
      sel_bits |= static_cast<uint32_t>(static_cast<int>(bn) < beta0) << bit;
      bnd |= static_cast<uint32_t>(static_cast<int>(bn) == beta0) << bit;
    };
    classify(bin_stay, NC);
    classify(bin_rep, NC + 1);
#pragma unroll
    for (int k = 0; k < NC; ++k) classify((binp[k >> 1] >> ((k & 1) * 16)) & 0xFFFFu, k);
    // the lane's boundary-bin candidates (v, exact score) that also lie in the
    // boundary bins of levels 1..L-1
    auto for_bnd = [&](int L, auto&& f) {
#pragma unroll 1
      for (uint32_t m = bnd; m; m &= m - 1) {
        const int k = __ffs(m) - 1;
        const int v = pos_v(k);
        const double sc = pos_score(k);
        bool in = true;
        for (int l = 1; l < L && in; ++l) in = bin_at(l, v, sc) == sLvBeta[l];
        if (in) f(k, v, sc);
      }
    };
    if (resolve) {
      int key_shift = shift0 >= 0 ? shift0 - kBinBits : 64 - kBinBits;
      bool key_level = shift0 >= 0;
      int last_shift = shift0;  // shift of the deepest level (-1: score bins)
      while (cntb != need && cntb > kBoundaryCap && !(key_level && last_shift == 0) && nlev < kMaxLevels) {
        // refine: score range of the boundary bin's members, or key bits when it is flat
        const int L = nlev;
        double bmx = kNegInf, bmn = HUGE_VAL;
        for_bnd(L, [&](int, int, double sc) {
          bmx = fmax(bmx, sc);
          bmn = fmin(bmn, sc);
        });
        double lv_hi, lv_lo;
        block_minmax<BLOCK>(bmx, bmn, sRedB, &lv_hi, &lv_lo);
        if (tid == 0) {
          sLvHi[L] = lv_hi;
          sLvInv[L] = lv_hi > lv_lo ? static_cast<double>(kBins) / (lv_hi - lv_lo) : 0.0;
          sLvShift[L] = lv_hi > lv_lo ? -1 : (key_shift > 0 ? key_shift : 0);
        }
        // (block_minmax's barrier follows every wavefront's scan of the bins)
        for (int d = tid; d < kBins; d += BLOCK) sHisto[d] = 0;
        lds_barrier();
        last_shift = sLvShift[L];
        key_level = last_shift >= 0;
        if (key_level) key_shift -= kBinBits;
        for_bnd(L, [&](int, int v, double sc) { atomicAdd(&sHisto[bin_at(L, v, sc)], 1u); });
        lds_barrier();
        const Found f = find_bin(need);
        if (tid == 0) sLvBeta[L] = f.bin;
        need -= f.above;
        cntb = f.count;
        nlev = L + 1;
        lds_barrier();
      }
      if (cntb == need) {
        all_bin = true;
      } else {
        // exact rank inside the boundary bin (a flat key level of shift 0 holds one key)
        for_bnd(nlev, [&](int, int v, double sc) {
          const int slot = atomicAdd(&sBCount, 1);
          if (slot < kBoundaryCap) {
            sBScore[slot] = sc;
            sBKey[slot] = key_of(v);
          }
        });
        lds_barrier();
        nbc = sBCount < kBoundaryCap ? sBCount : kBoundaryCap;
        if (sBCount > kBoundaryCap && tid == 0) atomicOr(S.flags, kFlagSelect);
      }
    }
    // the boundary bin's candidates: the deeper levels, then the exact rank on
    // (score desc, key asc)
#pragma unroll 1
    for (uint32_t m = bnd; m; m &= m - 1) {
      const int k = __ffs(m) - 1;
      const int v = pos_v(k);
      const double sc = pos_score(k);
      bool take = true;
      bool decided = false;
      for (int l = 1; l < nlev && !decided; ++l) {
        const int bl = bin_at(l, v, sc);
        if (bl != sLvBeta[l]) {
          take = bl < sLvBeta[l];
          decided = true;
        }
      }
      if (!decided && !all_bin) {
        const uint64_t key = key_of(v);
        int rank = 0;
        for (int u = 0; u < nbc; ++u) rank += ranks_before(sBScore[u], sBKey[u], sc, key);
        take = rank < need;
      }
      if (take) sel_bits |= 1u << k;
    }
    int wpos = block_scan<BLOCK, false>(__popc(sel_bits), sScanD, &nsel);
    if (nsel > K) {  // cannot happen when the selection is exact; never write past K entries
      nsel = K;
      if (tid == 0) atomicOr(S.flags, kFlagSelect);
    }
#pragma unroll 1
    for (uint32_t m = sel_bits; m && wpos < nsel; m &= m - 1) {
      const uint32_t v = static_cast<uint32_t>(pos_v(__ffs(m) - 1));
      sSelSrc[wpos++] = static_cast<uint32_t>(hi_) | (v << 16);
    }
    btotal = best;
    coarse = nsel == K;
    }
    lds_barrier();
    mark(kPhTopK);

    // ---- the new hypotheses; an extension's trie node is fetched now and
    // stored after the next frame's recombination.  (The next selection's bins
    // are cleared meanwhile.)
    for (int d = tid; d < kBins; d += BLOCK) sHisto[d] = 0;
    if (tid == 0) sBCount = 0;
    // Every field of an entry comes from its source in one round of reads, for
    // a stay and an extension alike.
    const int r = tid;
    const bool mine = r < nsel;
    bool tn_load = false;
    TrieNode tn{};
    uint64_t w_key = 0, w_pkey = 0, w_tmask = 0;
    double w_ab = 0.0, w_anb = 0.0, w_pt = 0.0;
    uint32_t w_node = 0, w_meta = 0, w_first = 0, w_woff = 0;
    uint4 w_L01{}, w_L23{}, w_hist{};  // the sub-beams: four word-level scores, four history nodes
    bool is_event = false;
    if (mine) {
      const uint32_t src = sSelSrc[r];
      const int i = src & 0xFFFF;
      const int v = src >> 16;
      const uint32_t meta_i = C.meta[i];
      const uint64_t key_i = C.key[i], pkey_i = C.pkey[i];
      const double ab_i = C.ab[i], pt_i = C.pt[i], ab2 = sAb2[i], anb2 = sAnb2[i], pt2 = sPt2[i];
      const double dv = Dc[v], bv = sBonus[v];
      const uint32_t node_i = C.node[i];
      w_tmask = C.tmask[i];
      w_first = C.first[i];
      w_woff = C.woff[i];
      w_L01 = reinterpret_cast<const uint4*>(&C.Lw[i * kMaxSub])[0];
      w_L23 = reinterpret_cast<const uint4*>(&C.Lw[i * kMaxSub])[1];
      w_hist = reinterpret_cast<const uint4*>(&C.hist[i * kMaxSub])[0];
      tn_load = v != 0;
      is_event = v == kSep;
      const double base = v == static_cast<int>(meta_i & 0xFF) ? ab_i : pt_i;
      const double ext = (base + dv) + bv;
      const uint32_t child = is_event ? kRootNode : w_first + __popcll(w_tmask & ((1ull << v) - 1ull));
      if (tn_load) tn = trie[child];
      w_key = tn_load ? prefix_step(key_i, v) : key_i;
      w_pkey = tn_load ? key_i : pkey_i;
      w_ab = tn_load ? kNegInf : ab2;
      w_anb = tn_load ? ext : anb2;
      w_pt = tn_load ? ext : pt2;  // log-sum-exp(-inf, ext)
      w_node = tn_load ? child : node_i;
      w_meta = tn_load ? (static_cast<uint32_t>(v) | (meta_i & 0xFF00u)) : meta_i;
    }
    if constexpr (!DB) lds_barrier();  // every source entry has been read
    if (mine) {
      insert_key(w_key, r);  // for the next frame's parent lookups
      sCut[r] = 0;
      N.key[r] = w_key;
      N.pkey[r] = w_pkey;
      N.ab[r] = w_ab;
      N.anb[r] = w_anb;
      N.pt[r] = w_pt;
      N.node[r] = w_node;
      N.meta[r] = w_meta;
      if (!tn_load) {
        N.tmask[r] = w_tmask;
        N.first[r] = w_first;
        N.woff[r] = w_woff;
      }
      reinterpret_cast<uint4*>(&N.Lw[r * kMaxSub])[0] = w_L01;
      reinterpret_cast<uint4*>(&N.Lw[r * kMaxSub])[1] = w_L23;
      reinterpret_cast<uint4*>(&N.hist[r * kMaxSub])[0] = w_hist;
    }
    // the memory that a completed word's scoring reads first, touched here: its
    // wavefronts then find it in the CU's cache
    uint32_t t0_ = 0, t1_ = 0, t2_ = 0, t3_ = 0, t4_ = 0, t5_ = 0;
    if (kAhead && is_event) {
      const int nsub = (w_meta >> 8) & 0xFF;
      t0_ = arena[w_hist.x].blk;
      if (nsub > 1) t1_ = arena[w_hist.y].blk;
      if (nsub > 2) t2_ = arena[w_hist.z].blk;
      if (nsub > 3) t3_ = arena[w_hist.w].blk;
      t4_ = static_cast<uint32_t>(trie_words[w_woff]);
      t5_ = wrank[w_woff].h;
    }
    if (wave < RW) {
      const uint64_t evs = __ballot(is_event);
      if (is_event)  // the hypothesis, its sub-beams, the completed word's node
        sEv[64 * wave + __popcll(evs & ((1ull << lane) - 1ull))] =
            uint4{static_cast<uint32_t>(r), (w_meta >> 8) & 0xFFu, w_woff, static_cast<uint32_t>(w_tmask >> kWordCountShift)};
      if (lane == 0) sEvCnt[wave] = __popcll(evs);
    }
    if (wave >= LM0) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");  // (the frame before's history nodes)
    lds_barrier();  // the new hypotheses, their keys and the completed words are in place
    mark(kPhNewBeam);
    int nev = 0;
#pragma unroll
    for (int w = 0; w < RW; ++w) nev += sEvCnt[w];

    // ---- Eq. (1) for the completed words, and, on the wavefronts that hold the
    // hypotheses, the next frame's recombination, which needs none of its
    // results: neither waits for the other.  The row after the next one's is set
    // by the last wavefront, or, if that one may have words to score, by the
    // first one after its recombination.
    const bool last_busy = LMW == NW - LM0 && nev > 4 * (LMW - 1);
    if (wave == NW - 1 && !last_busy && tau + 2 < tend) set_row(P, row, dnext, lane);
    if (wave >= LM0 && wave < LM0 + LMW) {
      // (a chain of dependent reads that the others wait for at the next barrier:
      // it issues first.  512 x 500 frames at K = 256 5.30 -> 5.15 ms, 1024
      // streams in ten calls at K = 64 1.72 -> 1.69, fewer per CU unchanged.)
      __builtin_amdgcn_s_setprio(2);
      score_words(P, S, N, nev, wave - LM0, LMW, lane);
      // the history nodes (global memory) are read by the fusion, if this frame
      // fuses, else by the next frame's scoring: then they are waited for at
      // the end of its selection
      if (fuses || !more) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    }
    if (wave < RW) {
      if (more && mine) recombine(N, sD[row ^ 1], tid, w_pkey, w_meta, w_pt, w_anb);
      if (tn_load) {
        N.tmask[r] = tn.mask;
        N.first[r] = tn.first_child;
        N.woff[r] = tn.word_off;
      }
      if (wave == 0 && last_busy && tau + 2 < tend) set_row(P, row, load_row(tau + 2, lane), lane);
      asm volatile("" ::"v"(t0_), "v"(t1_), "v"(t2_), "v"(t3_), "v"(t4_), "v"(t5_));
    }
    {
      // nodes reserved this frame; past the capacity the count stays at cap + 1
      // (every later word event then sees no room and raises the flag)
      const uint64_t an = static_cast<uint64_t>(arena_n) + static_cast<uint64_t>(nev * O);
      arena_n = static_cast<uint32_t>(an <= arena_cap ? an : arena_cap + 1);
    }
    if (tid == 0) sCnt[4] += static_cast<unsigned long long>(n) * kClasses;
    n = nsel;
    row ^= 1;
    lds_barrier();
    mark(kPhRecomb);

    // ---- Eq. (2) on fusion frames: the top-F hypotheses by (total desc, key
    // asc); each sub-beam's score becomes phi * its synthetic fusion score and
    // the sub-beams are re-ranked (stable)
    if (fuses) {
      double* sc = reinterpret_cast<double*>(sSel);
      uint64_t* ky = reinterpret_cast<uint64_t*>(sSel + 8 * KMAX);
      uint32_t* ix = reinterpret_cast<uint32_t*>(sSel + 16 * KMAX);
      const int F = (P.fusion_top_f <= 0 || P.fusion_top_f >= n) ? n : P.fusion_top_f;
      const uint32_t* sel = ix;  // the selected hypotheses (any order: each is fused on its own)
      if (F < n) {
        if constexpr (KMAX >= 128) {
          // the top F as a set, from a histogram of the totals (a sort of K =
          // 256 totals takes 36 barrier-separated stages): bins of (hi -
          // total) over [lo, hi], monotone; the bin holding the F-th found by
          // one wavefront; the bins above it taken whole, and its members
          // ranked exactly among themselves by (total desc, key asc; the
          // index for exact ties, which distinct prefixes do not have)
          uint32_t* const fH = reinterpret_cast<uint32_t*>(sSel);
          double* const fT = reinterpret_cast<double*>(sSel + 4 * kBins);
          uint64_t* const fK = reinterpret_cast<uint64_t*>(sSel + 4 * kBins + 8 * KMAX);
          uint32_t* const fI = reinterpret_cast<uint32_t*>(sSel + 4 * kBins + 16 * KMAX);
          uint32_t* const fSel = fI + KMAX;
          static_assert(4 * kBins + 24 * KMAX <= UNI_BYTES, "top-F scratch");
          for (int d = tid; d < kBins; d += BLOCK) fH[d] = 0;
          if (tid == 0) {
            sBCount = 0;
            sAthr = 0;
          }
          const bool own = tid < n;
          double tot = kNegInf;
          uint64_t key = ~0ull;
          if (own) {
            tot = N.pt[tid] + N.Lw[tid * kMaxSub];
            key = N.key[tid];
          }
          double hi, lo;
          block_minmax<BLOCK>(own ? tot : kNegInf, own ? tot : HUGE_VAL, sRed, &hi, &lo);
          const double inv = hi > lo ? static_cast<double>(kBins) / (hi - lo) : 0.0;
          int bin = -1;
          if (own) {
            const double x = (hi - tot) * inv;
            bin = x < static_cast<double>(kBins - 1) ? static_cast<int>(x) : kBins - 1;  // NaN: a total of -inf
            atomicAdd(&fH[bin], 1u);
          }
          lds_barrier();
          if (wave == 0) {
            constexpr int PERW = kBins / 64;
            int h[PERW];
            const uint4* hp = reinterpret_cast<const uint4*>(fH + lane * PERW);
#pragma unroll
            for (int q = 0; q < PERW / 4; ++q) {
              const uint4 x4 = hp[q];
              h[4 * q] = static_cast<int>(x4.x);
              h[4 * q + 1] = static_cast<int>(x4.y);
              h[4 * q + 2] = static_cast<int>(x4.z);
              h[4 * q + 3] = static_cast<int>(x4.w);
            }
            int local = 0;
#pragma unroll
            for (int q = 0; q < PERW; ++q) local += h[q];
            const int incl = wave_scan_incl(local);
            const int before = incl - local;
            if (before < F && incl >= F) {
              int acc = before;
              bool found = false;
#pragma unroll
              for (int q = 0; q < PERW; ++q) {
                if (!found && acc + h[q] >= F) {
                  sBucket = lane * PERW + q;
                  sAbove = acc;
                  found = true;
                }
                acc += h[q];
              }
            }
          }
          lds_barrier();
          const int fb = sBucket, fa = sAbove;
          if (own && bin < fb) fSel[atomicAdd(&sAthr, 1)] = static_cast<uint32_t>(tid);  // positions 0..fa-1
          if (own && bin == fb) {
            const int m = atomicAdd(&sBCount, 1);
            fT[m] = tot;
            fK[m] = key;
            fI[m] = static_cast<uint32_t>(tid);
          }
          lds_barrier();
          const int nbm = sBCount;
          for (int m = tid; m < nbm; m += BLOCK) {
            const double tm = fT[m];
            const uint64_t km = fK[m];
            const uint32_t im = fI[m];
            int r = 0;
            for (int u = 0; u < nbm; ++u) {
              const double tu = fT[u];
              const uint64_t ku = fK[u];
              r += (tu > tm || (tu == tm && (ku < km || (ku == km && fI[u] < im)))) ? 1 : 0;
            }
            if (r < F - fa) fSel[fa + r] = im;
          }
          lds_barrier();
          sel = fSel;
        } else if constexpr (WPE == 1) {
          // the top F as a set by rank counting: the LPB lanes of each
          // hypothesis count, a share each, the hypotheses ranking before it
          // (total desc, key asc; the keys are distinct), and one lane places
          // it; one barrier (in the instances with registers to spare: in the
          // 128-register ones it costs a spill)
          const int hf = tid / LPB, lf = tid - hf * LPB;
          int cnt = 0;
          if (hf < n) {
            const double ti = N.pt[hf] + N.Lw[hf * kMaxSub];
            const uint64_t ki = N.key[hf];
            for (int j = lf; j < n; j += LPB) cnt += ranks_before(N.pt[j] + N.Lw[j * kMaxSub], N.key[j], ti, ki) ? 1 : 0;
          }
#pragma unroll
          for (int o = 1; o < LPB; o <<= 1) cnt += __shfl_xor(cnt, o, 64);
          if (hf < n && lf == 0 && cnt < F) ix[cnt] = static_cast<uint32_t>(hf);
          lds_barrier();
        } else {
          if (tid < KMAX) {
            sc[tid] = tid < n ? N.pt[tid] + N.Lw[tid * kMaxSub] : kNegInf;
            ky[tid] = tid < n ? N.key[tid] : ~0ull;
            ix[tid] = tid < n ? static_cast<uint32_t>(tid) : 0u;
          }
          lds_barrier();
          bitonic_sort<KMAX>(sc, ky, ix);
        }
      }
      if (tid < F) {
        const int i = F < n ? static_cast<int>(sel[tid]) : tid;
        const int nsub = (N.meta[i] >> 8) & 0xFF;
        double L[kMaxSub];
        uint32_t h[kMaxSub];
#pragma unroll
        for (int j = 0; j < kMaxSub; ++j) {
          if (j < nsub) {
            h[j] = N.hist[i * kMaxSub + j];
            L[j] = P.phi * S.arena[h[j]].sfus;
          } else {
            L[j] = kNegInf;
            h[j] = 0;
          }
        }
        rank_subs(nsub, L, h);
#pragma unroll
        for (int j = 0; j < kMaxSub; ++j) {
          if (j < nsub) {
            N.Lw[i * kMaxSub + j] = L[j];
            N.hist[i * kMaxSub + j] = h[j];
          }
        }
      }
      if (tid == 0) {
        sCnt[5] += static_cast<unsigned long long>(F);
        sBCount = 0;
      }
      lds_barrier();
      btotal = best_total(N, n, tid);
      mark(kPhFusion);
    }
    if constexpr (DB) cur ^= 1;
  }

  // (the thread index opaque again: addresses of the load above are not kept
  // through the frames for the write-back)
  {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const size_t gb = static_cast<size_t>(b) * K;
  // ---- the end of an utterance: the final fusion of every hypothesis
  BeamLds<KMAX>& E = sBeam[DB ? cur : 0];
  if (out_hyps && out_fin && fuse_frames) {
    if (tid < n) {
      const int nsub = (E.meta[tid] >> 8) & 0xFF;
      double L[kMaxSub];
      uint32_t h[kMaxSub];
#pragma unroll
      for (int j = 0; j < kMaxSub; ++j) {
        L[j] = kNegInf;
        h[j] = 0;
        if (j < nsub) {
          h[j] = E.hist[tid * kMaxSub + j];
          L[j] = P.phi * final_score(P, arena[h[j]]);
        }
      }
      rank_subs(nsub, L, h);
#pragma unroll
      for (int j = 0; j < kMaxSub; ++j) {
        if (j < nsub) {
          E.Lw[tid * kMaxSub + j] = L[j];
          E.hist[tid * kMaxSub + j] = h[j];
        }
      }
    }
    if (tid == 0) sCnt[5] += static_cast<unsigned long long>(n);
  }

  // ---- the beam back to HBM (each thread the entry that it fused)
  bool o_root = false;
  double o_total = kNegInf;
  uint64_t o_key = ~0ull;
  uint32_t o_hist = 0;
  if (tid < n) {
    const size_t g = gb + tid;
    o_key = E.key[tid];
    o_root = E.node[tid] == kRootNode;
    o_total = E.pt[tid] + E.Lw[tid * kMaxSub];
    o_hist = E.hist[tid * kMaxSub];
    S.key[g] = o_key;
    S.pkey[g] = E.pkey[tid];
    S.ab[g] = E.ab[tid];
    S.anb[g] = E.anb[tid];
    S.pt[g] = E.pt[tid];
    S.node[g] = E.node[tid];
    const uint32_t meta = E.meta[tid];
    S.meta[g] = meta;
    const int nsub = (meta >> 8) & 0xFF;
#pragma unroll
    for (int j = 0; j < kMaxSub; ++j) {
      if (j < nsub) {
        S.Lw[g * O + j] = E.Lw[tid * kMaxSub + j];
        S.hist[g * O + j] = E.hist[tid * kMaxSub + j];
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lines += __shfl_xor(lines, o, 64);
    plines += __shfl_xor(plines, o, 64);
    c_words += __shfl_xor(c_words, o, 64);
    c_queries += __shfl_xor(c_queries, o, 64);
  }
  if (lane == 0) {
    atomicAdd(&sCnt[6], static_cast<unsigned long long>(c_look));
    atomicAdd(&sCnt[0], static_cast<unsigned long long>(lines));
    atomicAdd(&sCnt[1], static_cast<unsigned long long>(c_words));
    atomicAdd(&sCnt[2], static_cast<unsigned long long>(c_queries));
    atomicAdd(&sCnt[3], static_cast<unsigned long long>(plines));
  }
  lds_barrier();
  if (tid == 0) {
    S.nbeam[b] = n;
    S.arena_n[b] = arena_n;
    // (this workgroup's own counters: the additions are atomic so that nothing waits for their old values)
    unsigned long long* cn = S.counters + static_cast<size_t>(b) * kNumCounters;
    atomicAdd(&cn[kCntExpansions], sCnt[4]);
    atomicAdd(&cn[kCntFrames], static_cast<unsigned long long>(tend - tau0));
    atomicAdd(&cn[kCntWordEvents], sCnt[1]);
    atomicAdd(&cn[kCntLmQueries], sCnt[2]);
    atomicAdd(&cn[kCntFused], sCnt[5]);
    atomicAdd(&cn[kCntProbeLines], sCnt[0] + sCnt[3]);
    atomicAdd(&cn[kCntPresLines], sCnt[3]);
    atomicAdd(&cn[kCntLookups], sCnt[6]);
  }
  if (out_hyps)
    write_output<BLOCK, KMAX>(P, S, b, lengths, Tc, out_fin, out_hyps, out_scores, n, o_root, o_total, o_key, o_hist,
                              reinterpret_cast<double*>(sSel), reinterpret_cast<uint64_t*>(sSel + 8 * KMAX),
                              reinterpret_cast<uint32_t*>(sSel + 16 * KMAX), reinterpret_cast<uint32_t*>(sSel + 20 * KMAX),
                              sScan);
  }
  if (timing) {
    __syncthreads();
    mark(kPhOther);
    if (threadIdx.x == 64 * LM0) {  // (the thread that marks: it alone knows the last interval)
      unsigned long long* cn = S.counters + static_cast<size_t>(b) * kNumCounters;
      for (int k = 0; k < kPhases; ++k) cn[kCntPhase0 + k] += sPhase[k];
    }
  }
}

// ------------------------------------------------------------------ delayed fusion

// Selects the top-F hypotheses of stream b by (total desc, key asc) into
// S.fsel[b][0..F) and S.fsel_n[b] (F = all hypotheses when top_f <= 0); the
// sort covers BLOCK >= K entries (the workgroup may be larger).
#undef P
#undef S

template <int BLOCK>
__device__ __forceinline__ void select_fused(const DevParams& P, const DevState& S, int b, int top_f, double* sc, uint64_t* ky,
                             uint32_t* ix) {
  const int tid = threadIdx.x;
  const int n = S.nbeam[b];
  const size_t gb = static_cast<size_t>(b) * P.K;
  const int F = (top_f <= 0 || top_f >= n) ? n : top_f;
  if (F < n) {
    if (tid < n) {
      sc[tid] = S.pt[gb + tid] + S.Lw[(gb + tid) * P.O];
      ky[tid] = S.key[gb + tid];
      ix[tid] = tid;
    } else if (tid < BLOCK) {
      sc[tid] = kNegInf;
      ky[tid] = ~0ull;
      ix[tid] = 0;
    }
    __syncthreads();
    bitonic_sort<BLOCK>(sc, ky, ix);
  }
  if (tid < F) S.fsel[gb + tid] = (F < n) ? static_cast<int32_t>(ix[tid]) : tid;
  if (tid == 0) S.fsel_n[b] = F;
  __syncthreads();
}

// Delayed fusion on the selected hypotheses of stream b (Eq. (2)): each
// sub-beam's word-level score becomes phi * its fusion score -- the caller's
// ext[b][rank][j], or the synthetic score at the end of an utterance -- and the
// sub-beams are re-ranked (stable).
template <int BLOCK>
__device__ __forceinline__ void apply_fused(const DevParams& P, const DevState& S, int b, const float* ext) {
  const int tid = threadIdx.x;
  const size_t gb = static_cast<size_t>(b) * P.K;
  const int F = S.fsel_n[b];
  if (tid < F) {
    const size_t bi = gb + S.fsel[gb + tid];
    const uint32_t meta = S.meta[bi];
    const int nsub = (meta >> 8) & 0xFF;
    double L[kMaxSub];
    uint32_t h[kMaxSub];
#pragma unroll
    for (int j = 0; j < kMaxSub; ++j) {
      if (j < nsub) {
        h[j] = S.hist[bi * P.O + j];
        double f;
        if (ext) {
          f = static_cast<double>(ext[(gb + tid) * P.O + j]);
        } else {
          f = final_score(P, S.arena[h[j]]);
        }
        L[j] = P.phi * f;
      } else {
        L[j] = kNegInf;
        h[j] = 0;
      }
    }
    rank_subs(nsub, L, h);
#pragma unroll
    for (int j = 0; j < kMaxSub; ++j) {
      if (j < nsub) {
        S.Lw[bi * P.O + j] = L[j];
        S.hist[bi * P.O + j] = h[j];
      }
    }
  }
  if (tid == 0) {
    unsigned long long* cn = S.counters + static_cast<size_t>(b) * kNumCounters;
    cn[kCntFused] += static_cast<unsigned long long>(F);
  }
  __syncthreads();
}

// External scorer, step 1: per stream, the hypotheses to fuse (flag 1: a
// fusion frame, top-F; flag 2: end of utterance, all; 0: none).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_fuse_select(const DevParams P, const DevState S,
                                                       const int32_t* __restrict__ flag) {
  const int b = blockIdx.x;
  __shared__ double sc[BLOCK];
  __shared__ uint64_t ky[BLOCK];
  __shared__ uint32_t ix[BLOCK];
  if (flag[b] == 0) {
    if (threadIdx.x == 0) S.fsel_n[b] = 0;
    return;
  }
  select_fused<BLOCK>(P, S, b, flag[b] == 1 ? P.fusion_top_f : 0, sc, ky, ix);
}

// External scorer, step 2: word sequences of every sub-beam of the selected
// hypotheses, words [B][K][O][W] (-1 padded) and n_words [B][K][O] (-1 where
// nothing is to be scored).
// Writes -1 past each row's words: rows [nrows][W] with len[r] words in row r;
// the whole block on consecutive addresses, 16 B per store when W allows.
typedef int v4i __attribute__((ext_vector_type(4)));
template <int BLOCK>
__device__ inline void pad_rows(int32_t* rows, int nrows, int W, const int32_t* len) {
  if ((W & 3) == 0 && (reinterpret_cast<uintptr_t>(rows) & 15) == 0 && W > 0) {
    // thread t writes the 16-B column t % per of rows t / per, t / per + rstep,
    // ... (per = min(W / 4, BLOCK) columns of a row per pass, rstep rows)
    const int W4 = W >> 2;
    const int per = W4 < BLOCK ? W4 : BLOCK;  // columns per pass of a row
    const int rstep = BLOCK / per;            // rows per pass
    const int tid = threadIdx.x;
    if (tid < rstep * per) {
      for (int r = tid / per; r < nrows; r += rstep) {
        int4* row = reinterpret_cast<int4*>(rows + static_cast<size_t>(r) * W);
        const int n = len[r];
        for (int c = tid % per; c < W4; c += per) {
          const int c0 = 4 * c;
          if (c0 >= n) {
            // streamed past the caches: the rows are read by the caller, not here
            const v4i m1 = {-1, -1, -1, -1};
            __builtin_nontemporal_store(m1, reinterpret_cast<v4i*>(row + c));
          } else if (c0 + 3 >= n) {
            int32_t* e = rows + static_cast<size_t>(r) * W + c0;
            for (int q = n - c0; q < 4; ++q) e[q] = -1;
          }
        }
      }
    }
  } else {
    for (int r = 0; r < nrows; ++r) {
      int32_t* row = rows + static_cast<size_t>(r) * W;
      for (int c = len[r] + static_cast<int>(threadIdx.x); c < W; c += BLOCK) row[c] = -1;
    }
  }
}

// Writes the `depth` words of history h into row[0..min(depth, W)), one node
// read per block of kHistBlock words (the node's word and the earlier words of
// its block, then the node that ends the previous block).
__device__ inline void trace_words(const DevState& S, uint32_t h, int depth, int32_t* row, int W) {
  int d = depth;
  while (d >= 1) {
    const HistNode x = S.arena[h];
    const int nb = (d - 1) % kHistBlock;  // earlier words of the block
    if (d - 1 < W) row[d - 1] = x.word;
#pragma unroll
    for (int i = 0; i < kHistBlock - 1; ++i)
      if (i < nb && d - 2 - i < W) row[d - 2 - i] = x.w[i];
    d -= nb + 1;
    h = x.blk;
  }
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_fuse_export(const DevParams P, const DevState S,
                                                       int32_t* __restrict__ words, int32_t* __restrict__ n_words) {
  const int b = blockIdx.x;
  const size_t gb = static_cast<size_t>(b) * P.K;
  const int F = S.fsel_n[b];
  __shared__ int32_t sLen[BLOCK * kMaxSub];  // words written per request row (BLOCK >= K)
  for (int idx = threadIdx.x; idx < P.K * P.O; idx += BLOCK) {
    const int r = idx / P.O;
    const int j = idx - r * P.O;
    const size_t slot = (gb + r) * P.O + j;
    int32_t* row = words + slot * P.W;
    int len = -1;
    if (r < F) {
      const size_t bi = gb + S.fsel[gb + r];
      const int nsub = (S.meta[bi] >> 8) & 0xFF;
      if (j < nsub) {
        const uint32_t h = S.hist[bi * P.O + j];
        len = static_cast<int>(S.arena[h].depth);
        if (len > P.W) atomicOr(S.flags, kFlagWords);
        trace_words(S, h, len, row, P.W);
        if (len > P.W) len = P.W;
      }
    }
    sLen[idx] = len < 0 ? 0 : len;
    n_words[slot] = len;
  }
  __syncthreads();
  pad_rows<BLOCK>(words + gb * P.O * P.W, P.K * P.O, P.W, sLen);
}

// External scorer, step 3: apply the caller's scores [B][K][O] to the selection.
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_fuse_apply(const DevParams P, const DevState S,
                                                      const float* __restrict__ scores) {
  apply_fused<BLOCK>(P, S, blockIdx.x, scores);
}

// ------------------------------------------------------------------ output

// One stream's output: at the end of an utterance the mid-word filter (when some
// hypothesis ends at a word boundary); then the hypotheses ranked by (total
// desc, key asc), each one's words traced back from its best sub-beam, rows
// padded with -1.  Run by a whole workgroup of NT threads; thread i < n holds
// hypothesis i (root: it ends at a word boundary; hist: its best sub-beam's
// history).  The sort covers N >= K entries (N a power of two, N <= NT) in sc /
// ky / ix; hh holds N histories, sScan NT / 64 entries.
template <int NT, int N>
__device__ __forceinline__ void write_output(const DevParams& P, const DevState& S, int b, const int32_t* lengths,
                                             int32_t Tc, int32_t fin, int32_t* out_hyps, float* out_scores, int n,
                                             bool root, double total, uint64_t key, uint32_t hist, double* sc,
                                             uint64_t* ky, uint32_t* ix, uint32_t* hh, int32_t* sScan) {
  const int tid = threadIdx.x;
  // at the end of an utterance, hypotheses inside a word are dropped when at
  // least one hypothesis ends at a word boundary; otherwise all are ranked
  int nroot = 0;
  if (fin) (void)block_scan<NT>(tid < n && root ? 1 : 0, sScan, &nroot);
  bool ok = false;
  if (tid < n) {
    ok = !fin || root || nroot == 0;
    sc[tid] = ok ? total : kNegInf;
    ky[tid] = ok ? key : ~0ull;
    ix[tid] = tid;
    hh[tid] = hist;
  } else if (tid < N) {
    sc[tid] = kNegInf;
    ky[tid] = ~0ull;
    ix[tid] = 0;
  }
  int m = 0;
  (void)block_scan<NT>(ok ? 1 : 0, sScan, &m);
  // lanes per entry: the position of an entry is the number of those before it in
  // (score desc, key asc, index asc), counted by NT / N lanes, a share each (two
  // barriers; a sort of 256 entries takes 36 barrier-separated stages, and one
  // lane per entry took 3 us for 64); without lanes to share, from 128 entries
  // on, a sort
  constexpr int LANES = NT / N;
  if constexpr (LANES > 1 || N <= 64) {
    static_assert(LANES <= 16 && (LANES & (LANES - 1)) == 0, "an entry's lanes are neighbours in a wavefront");
    const int i = tid / LANES, part = tid % LANES;  // (NT == N * LANES)
    const double si = sc[i];
    const uint64_t ki = ky[i];
    int rk = 0;
#pragma unroll 8
    for (int j = part; j < N; j += LANES) {
      const double sj = sc[j];
      const uint64_t kj = ky[j];
      rk += (ranks_before(sj, kj, si, ki) || (sj == si && kj == ki && j < i)) ? 1 : 0;
    }
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1) rk += __shfl_xor(rk, o, 64);
    __syncthreads();
    if (part == 0) {
      sc[rk] = si;
      ky[rk] = ki;
      ix[rk] = static_cast<uint32_t>(i);
    }
  } else {
    bitonic_sort<N>(sc, ky, ix);
  }
  if (tid == 0) {
    // the stream's frame counter advances by the frames decoded in this call:
    // a length outside 0..Tc is clamped (the decode did the same) and flagged
    const int32_t len = lengths[b];
    const int32_t adv = len < 0 ? 0 : (len > Tc ? Tc : len);
    if (adv != len) atomicOr(S.flags, kFlagLength);
    atomicAdd(reinterpret_cast<unsigned long long*>(&S.t0[b]), static_cast<unsigned long long>(adv));
  }
  int32_t* const sLen = reinterpret_cast<int32_t*>(ky);  // words written per rank (the keys are read)
  __syncthreads();
  for (int r = tid; r < P.K; r += NT) {
    int32_t* row = out_hyps + (static_cast<size_t>(b) * P.K + r) * P.W;
    int n = 0;
    if (r < m) {
      out_scores[static_cast<size_t>(b) * P.K + r] = static_cast<float>(sc[r]);
      const uint32_t h = hh[ix[r]];
      const HistNode top = S.arena[h];
      const int len = static_cast<int>(top.depth);
      // at the end of an utterance with end-of-sentence marks, the best mark follows the words
      int32_t mark = -1;
      if (fin && P.fusion_source == 1 && P.fusion_interval > 0 && P.eos_count > 0) {
        double e;
        mark = best_eos(P, top.word, &e);
      }
      n = len + (mark >= 0 ? 1 : 0);
      if (n > P.W) atomicOr(S.flags, kFlagWords);
      trace_words(S, h, len, row, P.W);
      if (mark >= 0 && len < P.W) row[len] = mark;
    } else {
      out_scores[static_cast<size_t>(b) * P.K + r] = kNegInf;
    }
    sLen[r] = n < P.W ? n : P.W;
  }
  __syncthreads();
  pad_rows<NT>(out_hyps + static_cast<size_t>(b) * P.K * P.W, P.K, P.W, sLen);
}

// The output of a stream's beam in global memory, at the end of an utterance
// after the final synthetic fusion over all hypotheses.
template <int NT, int N>
__device__ __forceinline__ void emit_output(const DevParams& P, const DevState& S, int b, const int32_t* lengths,
                                            int32_t Tc, int32_t fin, int32_t* out_hyps, float* out_scores, double* sc,
                                            uint64_t* ky, uint32_t* ix, uint32_t* hh, int32_t* sScan) {
  const int tid = threadIdx.x;
  if (fin && P.fusion_source == 1 && P.fusion_interval > 0) {
    select_fused<N>(P, S, b, 0, sc, ky, ix);
    apply_fused<N>(P, S, b, nullptr);
  }
  const int n = S.nbeam[b];
  const size_t i = static_cast<size_t>(b) * P.K + tid;
  bool root = false;
  double total = kNegInf;
  uint64_t key = ~0ull;
  uint32_t hist = 0;
  if (tid < n) {
    root = S.node[i] == kRootNode;
    total = S.pt[i] + S.Lw[i * P.O];
    key = S.key[i];
    hist = S.hist[i * P.O];
  }
  write_output<NT, N>(P, S, b, lengths, Tc, fin, out_hyps, out_scores, n, root, total, key, hist, sc, ky, ix, hh, sScan);
}

// The output as a launch of its own (when the call's last decode launch did
// not write it).
template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_output(const DevParams P, const DevState S,
                                                  const int32_t* __restrict__ lengths, int32_t Tc, int32_t fin,
                                                  int32_t* __restrict__ out_hyps,
                                                  float* __restrict__ out_scores) {
  __shared__ double sc[BLOCK];
  __shared__ uint64_t ky[BLOCK];
  __shared__ uint32_t ix[BLOCK], hh[BLOCK];
  __shared__ int32_t sScan[BLOCK / 64];
  emit_output<BLOCK, BLOCK>(P, S, blockIdx.x, lengths, Tc, fin, out_hyps, out_scores, sc, ky, ix, hh, sScan);
}

// ------------------------------------------------------------------ gather ceiling

// Reads kGatherPerThread random 64-B lines of a table per thread (line index:
// the multiply-high of splitmix64(seed + i) and the line count, i the global
// gather number), all loads issued before any is used, and writes each thread's
// XOR of what it read so that no load is optimised away: the access pattern of
// the n-gram probes, one 64-B bucket line per probe, as independent threads.
constexpr int kGatherPerThread = 8;
__global__ __launch_bounds__(256) void k_gather_probe(const uint4* __restrict__ table, uint64_t lines, uint64_t n,
                                                      uint64_t seed, uint32_t* __restrict__ out) {
  const uint64_t t = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  uint4 v[kGatherPerThread][4];
#pragma unroll
  for (int g = 0; g < kGatherPerThread; ++g) {
    const uint64_t i = t * kGatherPerThread + g;
    const uint64_t line = i < n ? __umul64hi(splitmix64(seed + i), lines) : 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) v[g][q] = i < n ? table[line * 4 + q] : make_uint4(0, 0, 0, 0);
  }
  uint32_t x = 0;
#pragma unroll
  for (int g = 0; g < kGatherPerThread; ++g)
#pragma unroll
    for (int q = 0; q < 4; ++q) x ^= v[g][q].x ^ v[g][q].y ^ v[g][q].z ^ v[g][q].w;
  if (t * kGatherPerThread < n) out[t] = x;
}

}  // namespace

// ------------------------------------------------------------------ launchers

// Optional start/stop events for the next decode-kernel launch.  They go into
// the kernel's own dispatch (hipExtLaunchKernel), so their elapsed time is the
// kernel's execution without the gaps around it.
namespace {
thread_local hipEvent_t g_ev_start = nullptr;
thread_local hipEvent_t g_ev_stop = nullptr;
}  // namespace

void set_launch_events(hipEvent_t start, hipEvent_t stop) {
  g_ev_start = start;
  g_ev_stop = stop;
}

#define LB_LAUNCH(KERNEL, GRID, BLOCK, ST, ...)                                                  \
  do {                                                                                         \
    hipExtLaunchKernelGGL(KERNEL, GRID, BLOCK, 0, ST, g_ev_start, g_ev_stop, 0, __VA_ARGS__);  \
    g_ev_start = g_ev_stop = nullptr;                                                          \
  } while (0)

hipError_t launch_build_order(int order, const int32_t* ids, const float* lp, const float* bo, int64_t count,
                              int32_t vocab, NgramTable t2, NgramTable t3, NgramTable dst, uint32_t* flags,
                              uint32_t* ctx_out, hipStream_t st) {
  if (count <= 0) return hipSuccess;
  const int64_t blocks = (count + 255) / 256;
  const int grid = static_cast<int>(blocks < 65536 ? blocks : 65536);
  hipLaunchKernelGGL(k_build_order, dim3(grid), dim3(256), 0, st, order, ids, lp, bo, count, vocab, t2, t3,
                     dst, flags, ctx_out);
  return hipGetLastError();
}

uint64_t gather_probe_threads(uint64_t n) { return (n + kGatherPerThread - 1) / kGatherPerThread; }

hipError_t launch_gather_probe(const void* table, uint64_t lines, uint64_t n, uint64_t seed, uint32_t* out,
                               hipStream_t st) {
  const uint64_t threads = gather_probe_threads(n);
  const uint64_t blocks = (threads + 255) / 256;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFFull) return hipErrorInvalidValue;
  LB_LAUNCH(k_gather_probe, dim3(static_cast<unsigned>(blocks)), dim3(256), st, static_cast<const uint4*>(table), lines,
            n, seed, out);
  return hipGetLastError();
}

hipError_t launch_begin(const DevParams& P, const DevState& S, int32_t B, hipStream_t st) {
  LB_LAUNCH(k_begin, dim3((B + 255) / 256), dim3(256), st, P, S, B);
  return hipGetLastError();
}

#define LB_DISPATCH_BLOCK(BLK, KERNEL, GRID, ...)                                           \
  do {                                                                                      \
    if ((BLK) == 64)                                                                        \
      LB_LAUNCH(KERNEL<64>, dim3(GRID), dim3(64), st, __VA_ARGS__);                         \
    else if ((BLK) == 128)                                                                  \
      LB_LAUNCH(KERNEL<128>, dim3(GRID), dim3(128), st, __VA_ARGS__);                       \
    else                                                                                    \
      LB_LAUNCH(KERNEL<256>, dim3(GRID), dim3(256), st, __VA_ARGS__);                       \
  } while (0)

// Decode-kernel shapes: (hypotheses per workgroup, lanes per hypothesis).
// Compute units of the current device (queried once).
int cu_count() {
  static int n = 0;
  if (n <= 0) {
    int dev = 0, c = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && c > 0)
      n = c;
    else
      n = 256;
  }
  return n;
}

hipError_t launch_decode(int K, const KArgs* args, const float* logits, const int32_t* lengths, int32_t B,
                         int32_t Tc, int32_t tau0, int32_t tau1, int32_t fin, int32_t* out_hyps, float* out_scores,
                         uint32_t opts, void* scratch, hipStream_t st) {
  unsigned char* const scr = static_cast<unsigned char*>(scratch);
  const KArgs LB_CONST* A = (const KArgs LB_CONST*)args;
  // One workgroup per stream; a frame is a chain of latencies, so the instances
  // trade lanes and registers per stream against workgroups per CU.
  // - A batch that leaves CUs to spare: 256 or 512 threads per stream (four times
  //   as many lanes per hypothesis at K <= 32, twice at K = 64, as many wavefronts
  //   for the words as a beam can fill), registers without a limit.
  // - More streams than CUs: the instances that fit more workgroups per CU.
  //   K <= 16: 128 threads, 6 per CU; past that one wavefront per stream in 128
  //   registers, 12 to 13 per CU.
  //   K <= 32: 128 threads, 6 per CU, past that in two rounds.
  //   K <= 64: 256 threads, 3 per CU; past that 4 in 128 registers with the beam
  //   in place.
  //   K <= 128 and K <= 256: 512 threads, 2 per CU in 128 registers with the beam
  //   in place.
  // Both instances at each line, 60 frames, 125k words and 10 M n-grams, us of a
  // call with 256 streams (256 CUs: the first instance is taken) and with 320 (the
  // second):
  //   K <=  16: 256 threads 540, 435; 128 threads 536, 433 (equal)
  //   K <=  32: 512 threads 627, 785; 128 threads 885, 583
  //   K <=  64: 512 threads 571, 866; 256 threads 670, 565
  //   K <= 128: one per CU  621, 1003; two        611, 615
  //   K <= 256: one per CU  825, 1320; two        828, 851
  // and past the first one:
  //   K <= 64, 768 / 800 / 1024 streams: 3 per CU 784, 882, 992; 4 786, 663, 652
  //   K <= 16, 1536 / 1600 / 2000: 128 threads 621, 696, 918; one wavefront 722,
  //   771, 804 (60 frames of 20k words, 1536 / 2000 / 3072: 451, 752, 1014 and
  //   537, 534, 571)
  //   K <= 32, 1536 / 1600 / 2000: 128 threads 803, 1006, 1143; one wavefront of
  //   two lanes per hypothesis (no instance of its own) 885, 1089, 1071
  const int cus = cu_count();
  const bool spare = B <= cus;
  // (hash slots per hypothesis: 16 with one workgroup per CU and K <= 64, 8 at
  // K = 256; where workgroups share a CU, 4 with two tables, 8 or 16 with one,
  // as their LDS allows)
#define LB_DECODE(KM, LP, WP, DBUF, HSLOTS, THREADS)                                                         \
  LB_LAUNCH((k_decode<KM, LP, WP, DBUF, HSLOTS>), dim3(B), dim3(THREADS), st, A, logits, lengths, Tc, tau0, tau1, \
            fin, out_hyps, out_scores, opts, scr)
  if (K <= 16 && spare)
    LB_DECODE(16, 16, 1, true, 16, 256);
  else if (K <= 16 && B > 6 * cus)
    LB_DECODE(16, 4, 4, false, 4, 64);
  else if (K <= 16)
    LB_DECODE(16, 8, 1, true, 8, 128);
  else if (K <= 32 && spare)
    LB_DECODE(32, 16, 1, true, 16, 512);
  else if (K <= 32)
    LB_DECODE(32, 4, 1, true, 4, 128);
  else if (K <= 64 && spare)
    LB_DECODE(64, 8, 1, true, 16, 512);
  else if (K <= 64 && B > 3 * cus)
    LB_DECODE(64, 4, 4, false, 16, 256);
  else if (K <= 64)
    LB_DECODE(64, 4, 3, true, 4, 256);
  else if (K <= 128 && !spare)
    LB_DECODE(128, 4, 4, false, 8, 512);
  else if (K <= 128)
    LB_DECODE(128, 4, 1, true, 4, 512);
  else if (spare)
    LB_DECODE(256, 2, 1, true, 8, 512);
  else
    LB_DECODE(256, 2, 4, false, 8, 512);
#undef LB_DECODE
  return hipGetLastError();
}

hipError_t launch_fuse_select(int block, const DevParams& P, const DevState& S, const int32_t* flag, int32_t B,
                              hipStream_t st) {
  LB_DISPATCH_BLOCK(block, k_fuse_select, B, P, S, flag);
  return hipGetLastError();
}

hipError_t launch_fuse_export(int block, const DevParams& P, const DevState& S, int32_t* words, int32_t* n_words,
                              int32_t B, hipStream_t st) {
  LB_DISPATCH_BLOCK(block, k_fuse_export, B, P, S, words, n_words);
  return hipGetLastError();
}

hipError_t launch_fuse_apply(int block, const DevParams& P, const DevState& S, const float* scores, int32_t B,
                             hipStream_t st) {
  LB_DISPATCH_BLOCK(block, k_fuse_apply, B, P, S, scores);
  return hipGetLastError();
}

hipError_t launch_output(int block, const DevParams& P, const DevState& S, const int32_t* lengths, int32_t B,
                         int32_t Tc, int32_t fin, int32_t* out_hyps, float* out_scores, hipStream_t st) {
  LB_DISPATCH_BLOCK(block, k_output, B, P, S, lengths, Tc, fin, out_hyps, out_scores);
  return hipGetLastError();
}

// ------------------------------------------------------------------ static lookup scratch

// The n-gram lookup scratch of the decode calls that allocate nothing
// (lb_decode_batch_noalloc): one array per device, held until the process
// ends, shared by every such call on that device.  Host code never uses the
// name itself as an address (on the host it stands for the symbol, not for the
// device memory): static_scratch_address() returns the device address, found
// with hipGetSymbolAddress once per device, with that device current.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

static std::mutex g_scratch_mu;
static void* g_scratch_addr[kMaxDevices] = {};

hipError_t static_scratch_address(void** out) {
  *out = nullptr;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_addr[dev] = p;
  }
  *out = g_scratch_addr[dev];
  return hipSuccess;
}

}  // namespace lb
