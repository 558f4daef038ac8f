// Decode attention over the mixed INT8 / FP16 cache with the attention-mass EMA fused in
// (paper: "Tiled attention and mixed precision" -- blockwise read, running max and
// normaliser, dequantisation fused into the read; "Budget and ranker" -- EMA of attention
// mass; Algorithm 1 -- append in FP16, update EMA metadata).
//
// One launch per layer, grid (splits, kv-heads, sequences) -- or (kv-heads, splits, sequences)
// when the number of kv-heads is a multiple of eight, which puts all splits of a unit on one
// XCD -- of 512 threads.  The `splits` workgroups of a unit (b, kv-head) each stream a
// contiguous, byte-balanced slice of the unit's slots once and serve all G query heads of
// the group from that single read:
//
//   stream   running (max, normaliser, output) per head (online softmax); the raw scores
//            s[h][i] of the slice stay in LDS
//   publish  the workgroup's (m, l) per head go out first, then its merged output partial;
//            every published 8-byte word carries the launch's tag (its number since the last
//            commit plus a base kept on the device), so nothing waits for stores to land, no
//            counter is shared, and a recorded launch can be replayed
//   mass     gather the (m, l) words of every split of the unit (a bounded poll on their
//            tags: they all publish at about the same time), form the exact global (M, L),
//            then per slot A_i = sum_h e^{s[h][i]-M[h]} / L[h] and
//            ema_i <- lambda ema_i + (1-lambda) A_i; every split also normalises its share of
//            the unit's output row from the splits' tagged output partials.
//
// Every K/V byte is read once; the scores never leave the chip.  The wait is between
// workgroups of one launch, so the host only launches grids that are co-resident
// (splits * units <= occupancy * CUs) and the wait itself is bounded.
//
// Two streaming bodies share the prologue and the epilogue:
//   * vector-ALU body (any G, any D): lane c of a group of D/16 lanes owns channels
//     [16c, 16c+16) of a slot row, so a wavefront load covers whole rows, contiguous in
//     memory; each lane-group keeps its own running softmax state.
//   * matrix-core body (2 <= G <= 8, D = 128) for the INT8 slots: the G query heads against a
//     32-slot tile are two small contractions (scores: [G x 128] x [128 x 32]; output, transposed:
//     [128 x 32] x [32 x G]) issued as v_mfma_f32_16x16x32_f16 with the head dimension
//     padded to 16.  The vector ALU then only converts int8 -> fp16 and keeps the softmax
//     state, which is what lets the kernel stay memory-bound for grouped-query shapes.
//     FP16 slots go through the same contractions in 16-slot tiles, no conversion needed.
//     The same body with all 16 tile rows as query rows serves calls that carry several
//     tokens per sequence (conf_kv_attend_chunk), and a variant of it folds per-channel INT8
//     scales into the query and the output.
// When the splits of a unit cannot all be resident, or a slice's scores do not fit LDS, the
// launch is replaced by two (stream + publish with the scores in device scratch; merge + mass),
// which need no wait inside a kernel.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <map>
#include <set>
#include <mutex>
#include <tuple>
#include <type_traits>

#include "confkv_dev.h"
#include "launch.h"

namespace confkv {

constexpr int kAttThreads = 512;
constexpr int kAttWaves = 8;

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

// q-th dword of a 128-bit register quad (q is a compile-time constant after unrolling)
__device__ __forceinline__ unsigned dword_of(const int4 &v, int q) {
  return (unsigned)(q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w);
}

// Optional in-kernel phase trace (build with -DCONFKV_TRACE): lane 0 of every wavefront
// notes the 100 MHz wall clock at numbered points, 32 slots per wavefront, in 2 KB of LDS behind
// the kernel's own dynamic LDS (so a time stamp costs no trip to memory and no address
// translation while the kernel runs); the workgroup copies them to the debug buffer as its last
// act.  Compiled out otherwise.
#ifdef CONFKV_TRACE
#define TS_SLOT(k) ts_lds_[a.trace_off / 8 + (threadIdx.x >> 6) * 32 + (k)]
#define TS_INIT()                                                              \
  do {                                                                         \
    extern __shared__ unsigned long long ts_lds_[];                            \
    if (a.dbg && (threadIdx.x & 63) < 32) TS_SLOT(threadIdx.x & 63) = 0ull;     \
  } while (0)
#define TS(k)                                                                  \
  do {                                                                         \
    extern __shared__ unsigned long long ts_lds_[];                            \
    if (a.dbg && (threadIdx.x & 63) == 0) TS_SLOT(k) = wall_clock64();         \
  } while (0)
#define TS_DUMP()                                                              \
  do {                                                                         \
    extern __shared__ unsigned long long ts_lds_[];                            \
    __syncthreads();                                                           \
    if (a.dbg && threadIdx.x < kAttWaves * 32)                                 \
      a.dbg[(size_t)(unit_in_layer(cv, a) * ns + split_index(a)) * kAttWaves * 32 + threadIdx.x] = \
          ts_lds_[a.trace_off / 8 + threadIdx.x];                              \
  } while (0)
#else
#define TS_INIT() do { } while (0)
#define TS(k) do { } while (0)
#define TS_DUMP() do { } while (0)
#endif

// Partials travel between workgroups (possibly on different XCDs, whose L2s are not
// coherent for ordinary accesses) through agent-scope relaxed atomics: such loads and
// stores are coherent across the device by themselves, so no cache-wide release/acquire
// fence (an L2 write-back plus invalidate on this hardware) is ever issued.  No ordering
// between different words is needed either: every published word carries the tag of the
// launch that wrote it, so a reader can tell on its own whether the word it got is current.

// The host passes a launch's number since the last commit and the device completes it: the
// tag base and the position of the next appended token live in cv.ctl, where the commit at the
// end of conf_kv_evict_compact advances them.  A recorded sequence of launches can therefore be
// replayed: nothing that changes from step to step is a launch argument.
// The two words are only requested here: the first instruction that needs one of them (the
// append, the publish at the end of the stream) is where the kernel waits, long after the tile
// requests have gone out.
__device__ __forceinline__ AttendLaunch resolve_launch(const CacheView &cv, AttendLaunch a) {
  a.tag_base = cv.ctl[kCtlTag];
  a.pos_new = (int)cv.ctl[kCtlPos + a.layer];
  return a;
}
__device__ __forceinline__ unsigned tag_of(const AttendLaunch &a) { return a.tag_base + a.epoch; }

// A float that travels with the tag of the launch that wrote it: one 8-byte word, so a
// reader sees value and tag together or neither.
__device__ __forceinline__ void st_tagged(unsigned long long *p, unsigned epoch, float v) {
  __hip_atomic_store(p, ((unsigned long long)epoch << 32) | (unsigned long long)__float_as_uint(v),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_tagged(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// LDS traffic between lanes of one wavefront: LDS operations of a wavefront execute in
// program order, so a compiler-level barrier is all that is needed between a write phase
// and the read phase that consumes other lanes' data.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Workgroup barrier that orders LDS traffic only: global loads and stores issued before it
// stay in flight across it (__syncthreads waits for them as well).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ void unpack_i8x16(const int4 &r, float (&f)[16]) {
  const int wds[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int e = 0; e < 4; ++e) f[4 * k + e] = (float)((wds[k] << (24 - 8 * e)) >> 24);
  }
}

__device__ __forceinline__ void unpack_h16x16(const int4 &r0, const int4 &r1, float (&f)[16]) {
  half8_t a = __builtin_bit_cast(half8_t, r0), b = __builtin_bit_cast(half8_t, r1);
#pragma unroll
  for (int e = 0; e < 8; ++e) { f[e] = (float)a[e]; f[8 + e] = (float)b[e]; }
}

// ---------------------------------------------------------------------------------------
// Slice bookkeeping shared by both bodies
// ---------------------------------------------------------------------------------------
struct Slice {
  int u, ul, b, g, j;          // unit, unit within the layer, batch, kv-head, split
  int n, n8, h16, n16;         // length with the append, INT8 slots, FP16 ring head, FP16 slots
  int h8;                      // head of the rings anchored at the oldest slot (EMA, position, INT8 rows)
  int lo8, hi8;                // INT8 slots of this split
  int lo16, hi16;              // FP16 slots of this split (slot numbers, >= n8)
  int cnt8, ntok;              // hi8 - lo8, and cnt8 + (hi16 - lo16)
  const int32_t *tab;          // paged layout: the unit's block table (device memory, or a copy in LDS)
  // stash index t in [0, ntok) <-> slot
  __device__ __forceinline__ int slot_of(int t) const { return t < cnt8 ? lo8 + t : lo16 + (t - cnt8); }
};

// x / ns for any slot number, by the launch's multiplier and shift (0: a single split).  Scalar arithmetic throughout:
// nothing of a slice depends on the lane.
__device__ __forceinline__ unsigned div_splits(const AttendLaunch &a, unsigned x) {
  return a.ns_magic ? __umulhi(x, a.ns_magic) >> a.ns_shift : x;
}
// floor(x * j / ns) for x = q * ns + r
__device__ __forceinline__ int share_cut(const AttendLaunch &a, unsigned q, unsigned r, int j) {
  return (int)(q * (unsigned)j + div_splits(a, r * (unsigned)j));
}
// The launch grid is (splits, kv-heads, sequences), or (kv-heads, splits, sequences) when
// a.kv_major is set: workgroups go to the XCDs round-robin in linear order, so with eight
// kv-heads (or a multiple) in front all splits of a unit then run on one XCD.
__device__ __forceinline__ int kv_head_index(const AttendLaunch &a) { return a.kv_major ? blockIdx.x : blockIdx.y; }
__device__ __forceinline__ int split_index(const AttendLaunch &a) { return a.kv_major ? blockIdx.y : blockIdx.x; }
__device__ __forceinline__ int unit_in_layer(const CacheView &cv, const AttendLaunch &a) {
  return blockIdx.z * cv.Hkv + kv_head_index(a);
}

// Every split takes an equal share of the INT8 slots (cut at multiples of 32, the tile of
// the matrix-core body) and an equal share of the FP16 slots, so all splits of a unit carry
// the same mix of work and reach the arrival point together.
// words: the unit's counters when the kernel has requested them already (see unit_words), else null.
__device__ __forceinline__ Slice make_slice(const CacheView &cv, const AttendLaunch &a, int ns, int S,
                                            const int *words = nullptr) {
  Slice s;
  s.g = kv_head_index(a);
  s.b = blockIdx.z;
  s.ul = unit_in_layer(cv, a);
  s.j = split_index(a);
  s.u = a.layer * cv.B * cv.Hkv + s.ul;
  s.tab = cv.pt + (size_t)s.u * cv.npages;
  // The unit's four counters in ONE round trip: lanes 0..3 of every wavefront read one array
  // each with a single load instruction (four scalar loads get spread over the prologue by the
  // compiler, each waiting for the one before).
  const int k4 = threadIdx.x & 3;
  const int32_t *arr = k4 == 0 ? cv.len : k4 == 1 ? cv.n8 : k4 == 2 ? cv.head16 : cv.head8;
  const int mv = words ? *words : arr[s.u];
  const int len = __builtin_amdgcn_readlane(mv, 0), n8 = __builtin_amdgcn_readlane(mv, 1);
  s.h16 = __builtin_amdgcn_readlane(mv, 2);
  s.h8 = __builtin_amdgcn_readlane(mv, 3);
  // an observation call sees the unit as it was when its last query was the newest token
  s.n = (a.observe_first >= 0 ? a.observe_first : len) + a.tq;     // the appended tokens included
  s.n8 = min(n8, s.n);                                             // n8 <= len outside observation calls
  s.n16 = s.n - s.n8;
  const unsigned q8 = div_splits(a, s.n8), r8 = (unsigned)s.n8 - q8 * (unsigned)ns;
  const unsigned q16 = div_splits(a, s.n16), r16 = (unsigned)s.n16 - q16 * (unsigned)ns;
  s.lo8 = share_cut(a, q8, r8, s.j) & ~31;
  s.hi8 = s.j == ns - 1 ? s.n8 : share_cut(a, q8, r8, s.j + 1) & ~31;
  // outside observation calls the tail split's FP16 share is never empty (n16 >= 1), so its
  // owner holds slot n-1
  s.lo16 = s.n8 + share_cut(a, q16, r16, s.j);
  s.hi16 = s.n8 + share_cut(a, q16, r16, s.j + 1);
  s.cnt8 = s.hi8 - s.lo8;
  s.ntok = s.cnt8 + (s.hi16 - s.lo16);
  if (s.ntok > S) {                       // cannot happen when the host plan is right
    if (threadIdx.x == 0) atomicAdd(&cv.stats[kStatDeviceErr], 1ull);
    s.hi8 = s.lo8; s.cnt8 = 0;
    s.hi16 = min(s.hi16, s.lo16 + S);
    s.ntok = s.hi16 - s.lo16;
  }
  return s;
}

// Row of slot i in the EMA and position planes.  kPaged is the layout, known at compile time: the look-up in the block
// table costs branches and registers wherever a row is addressed.
template <bool kPaged>
__device__ __forceinline__ int slot_plane_row(const CacheView &cv, const Slice &s, int i) {
  return kPaged ? slot_row(cv, s.tab, s.h8, s.n8, s.h16, i) : ring_row_u(s.h8, i, cv.cap);
}

// The workgroup that owns the tail writes the new token into the FP16 ring.
// Nobody reads the appended row back in this launch (the new token is taken from the call's
// arguments), so nothing waits for the stores.
// (tq: a.tq, as a constant where the call has one token.)
template <int D, bool kPaged = false>
__device__ __forceinline__ void append_new_token(const CacheView &cv, const AttendLaunch &a,
                                                 const Slice &s, int ns, int tq) {
  if (s.j != ns - 1 || a.observe_first >= 0) return;
  const int tid = threadIdx.x;
  constexpr int PPR = D / 8;                        // 16-byte pieces per row
  // token t of the call: K/V rows [B][tq][Hkv][D] -> FP16 ring row of slot n - tq + t
  for (int i = tid; i < 2 * tq * PPR; i += kAttThreads) {
    const int which = i >= tq * PPR, r = i - which * tq * PPR, t = r / PPR, c = r % PPR;
    const int row = ring_row(s.h16, s.n16 - tq + t, cv.cap16);
    const __half *src = (which ? a.vnew : a.knew) + (((size_t)s.b * tq + t) * cv.Hkv + s.g) * D;
    __half *dst = (which ? cv.v16 : cv.k16) + ((size_t)s.u * cv.cap16 + row) * D;
    ((int4 *)dst)[c] = ((const int4 *)src)[c];
  }
  if (tid < tq)
    cv.pos[(size_t)s.u * cv.cap + slot_plane_row<kPaged>(cv, s, s.n - tq + tid)] = a.pos_new + tid;
}

// max / sum over the 16 lanes of a DPP row; every lane of the row gets the result
#define CONFKV_DPP(v, ctrl) \
  __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), ctrl, 0xf, 0xf, true))
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, CONFKV_DPP(v, 0xB1));    // quad_perm [1,0,3,2]
  v = fmaxf(v, CONFKV_DPP(v, 0x4E));    // quad_perm [2,3,0,1]
  v = fmaxf(v, CONFKV_DPP(v, 0x141));   // row_half_mirror
  v = fmaxf(v, CONFKV_DPP(v, 0x140));   // row_mirror
  return v;
}
__device__ __forceinline__ float row16_sum(float v) {
  v += CONFKV_DPP(v, 0xB1);
  v += CONFKV_DPP(v, 0x4E);
  v += CONFKV_DPP(v, 0x141);
  v += CONFKV_DPP(v, 0x140);
  return v;
}

// The same over aligned groups of gs lanes (a power of two, uniform); all 64 lanes must be active.
// Lane moves inside a row cost a few cycles, an exchange through LDS (__shfl_xor) some hundred.
__device__ __forceinline__ float group_max(float v, int gs) {
  if (gs >= 2) v = fmaxf(v, CONFKV_DPP(v, 0xB1));
  if (gs >= 4) v = fmaxf(v, CONFKV_DPP(v, 0x4E));
  if (gs >= 8) v = fmaxf(v, CONFKV_DPP(v, 0x141));
  if (gs >= 16) v = fmaxf(v, CONFKV_DPP(v, 0x140));
  if (gs >= 32) v = fmaxf(v, __shfl_xor(v, 16, kWave));
  if (gs >= 64) v = fmaxf(v, __shfl_xor(v, 32, kWave));
  return v;
}
__device__ __forceinline__ float group_sum(float v, int gs) {
  if (gs >= 2) v += CONFKV_DPP(v, 0xB1);
  if (gs >= 4) v += CONFKV_DPP(v, 0x4E);
  if (gs >= 8) v += CONFKV_DPP(v, 0x141);
  if (gs >= 16) v += CONFKV_DPP(v, 0x140);
  if (gs >= 32) v += __shfl_xor(v, 16, kWave);
  if (gs >= 64) v += __shfl_xor(v, 32, kWave);
  return v;
}
// Sums over the lanes of a wavefront that agree modulo LPT (4 or 8).  Halves: of two values the
// lower rows keep the first one's sum over a pair of rows, the upper rows the second one's.
__device__ __forceinline__ float swap_halves32(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float((unsigned)r[0]) + __uint_as_float((unsigned)r[1]);
}
__device__ __forceinline__ float swap_halves16(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float((unsigned)r[0]) + __uint_as_float((unsigned)r[1]);
}
// over the lanes of a row of 16
template <int LPT>
__device__ __forceinline__ float row_stride_sum(float v) {
  if (LPT <= 4) v += CONFKV_DPP(v, 0x124);    // row_ror:4
  return v + CONFKV_DPP(v, 0x128);            // row_ror:8
}
#undef CONFKV_DPP
#define CONFKV_DPP(v, ctrl)                                                                                   \
  __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true),                         \
                   __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true))
__device__ __forceinline__ double group_sum(double v, int gs) {
  if (gs >= 2) v += CONFKV_DPP(v, 0xB1);
  if (gs >= 4) v += CONFKV_DPP(v, 0x4E);
  if (gs >= 8) v += CONFKV_DPP(v, 0x141);
  if (gs >= 16) v += CONFKV_DPP(v, 0x140);
  if (gs >= 32) v += __shfl_xor(v, 16, kWave);
  if (gs >= 64) v += __shfl_xor(v, 32, kWave);
  return v;
}
#undef CONFKV_DPP

// ---------------------------------------------------------------------------------------
// Vector-ALU streaming body
// ---------------------------------------------------------------------------------------

// Running softmax state of one slot lane-group: per head the maximum so far, the
// normaliser and this lane's 16 channels of the un-normalised output.
template <int G>
struct Stream {
  float m[G], l[G], acc[G][16];
  __device__ __forceinline__ void reset() {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m[h] = -INFINITY;
      l[h] = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[h][e] = 0.f;
    }
  }
};

// Fold a batch of R slots into the running state.  s[r][h] are the slots' scores,
// value(r, vf) unpacks the value channels of slot r owned by this lane, vsc[r] is the value
// scale, ok[r] validity; the first nr slots exist (uniform over the workgroup).
template <int G, int R, typename Value>
__device__ __forceinline__ void fold_batch(Stream<G> &st, const float (&s)[R][G], Value value,
                                           const float (&vsc)[R], const bool (&ok)[R], int nr) {
  const float NEG = -INFINITY;
  float p[R][G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float bm = NEG;
#pragma unroll
    for (int r = 0; r < R; ++r) bm = ok[r] ? fmaxf(bm, s[r][h]) : bm;
    const float mn = fmaxf(st.m[h], bm);
    const float corr = (mn == NEG) ? 1.f : __expf(st.m[h] - mn);
    st.m[h] = mn;
    float lsum = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      p[r][h] = ok[r] ? __expf(s[r][h] - mn) : 0.f;
      lsum += p[r][h];
      p[r][h] *= vsc[r];
    }
    st.l[h] = fmaf(st.l[h], corr, lsum);
#pragma unroll
    for (int e = 0; e < 16; ++e) st.acc[h][e] *= corr;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r >= nr) break;
    float vf[16];
    value(r, vf);
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < 16; ++e) st.acc[h][e] = fmaf(p[r][h], vf[e], st.acc[h][e]);
  }
}

template <int D, int G>
__device__ __forceinline__ void load_q_slices(const CacheView &cv, const AttendLaunch &a,
                                              const Slice &sl, float (&qf)[G][16]) {
  constexpr int LPT = D / 16;
  const int c = (threadIdx.x & 63) % LPT;
  const int Hq = cv.Hkv * G;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const int4 *qp = (const int4 *)(a.q + ((size_t)(sl.b * Hq + sl.g * G + h)) * D + c * 16);
    unpack_h16x16(qp[0], qp[1], qf[h]);
  }
}

// INT8 slots [lo, hi8) on the vector ALU.
template <int D, int G>
__device__ __forceinline__ void stream_int8_valu(const CacheView &cv, const Slice &sl, float sm,
                                                 const float (&qf)[G][16], Stream<G> &st,
                                                 float *stash, int S) {
  constexpr int LPT = D / 16, TW = kWave / LPT, TB = kAttWaves * TW, R8 = 4;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = lane % LPT, ts = lane / LPT;
  const int8_t *K8 = cv.k8 + (size_t)sl.u * cv.cap8 * D;
  const int8_t *V8 = cv.v8 + (size_t)sl.u * cv.cap8 * D;
  // per-channel scales: the caller folded the K scales into qf and applies the V scales to the
  // accumulator afterwards; every slot then has the factors (sm, 1).  The per-token loads stay
  // branch-free on element 0 of the unit's scale plane.
  const bool chan = cv.chan != 0;
  const __half *KS = cv.ks + (size_t)sl.u * (chan ? D : cv.cap8);
  const __half *VS = cv.vs + (size_t)sl.u * (chan ? D : cv.cap8);
  if (sl.lo8 >= sl.hi8) return;
  int4 kr[R8], vr[R8];
  unsigned short ksh[R8], vsh[R8];
  // branch-free loads (rows past the slice re-read its last row and are masked below); a trip's
  // keys are requested as soon as the previous trip's have become scores, its values behind
  // the previous trip's sums
  auto row_of = [&](int base, int r) { return ring_row_u(sl.h8, min(base + r * TB + w * TW + ts, sl.hi8 - 1), cv.cap8); };
  auto load_k = [&](int base) {
#pragma unroll
    for (int r = 0; r < R8; ++r) {
      const int ic = row_of(base, r);
      kr[r] = *(const int4 *)(K8 + (size_t)ic * D + c * 16);
      ksh[r] = ((const unsigned short *)KS)[chan ? 0 : ic];
    }
  };
  auto load_v = [&](int base) {
#pragma unroll
    for (int r = 0; r < R8; ++r) {
      const int ic = row_of(base, r);
      vr[r] = *(const int4 *)(V8 + (size_t)ic * D + c * 16);
      vsh[r] = ((const unsigned short *)VS)[chan ? 0 : ic];
    }
  };
  load_k(sl.lo8);
  load_v(sl.lo8);
  for (int base = sl.lo8; base < sl.hi8; base += TB * R8) {
    float s[R8][G], vsc[R8];
    bool ok[R8];
    const int nr = (sl.hi8 - base + TB - 1) / TB;
#pragma unroll
    for (int r = 0; r < R8; ++r) {
      if (r >= nr) {
#pragma unroll
        for (int h = 0; h < G; ++h) s[r][h] = 0.f;
        continue;
      }
      float kf[16];
      unpack_i8x16(kr[r], kf);
      const float f = chan ? sm : __half2float(__ushort_as_half(ksh[r])) * sm;
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc = fmaf(qf[h][e], kf[e], acc);
        s[r][h] = group_sum(acc, LPT) * f;
      }
    }
    const bool more = base + TB * R8 < sl.hi8;
    if (more) load_k(base + TB * R8);
#pragma unroll
    for (int r = 0; r < R8; ++r) {
      const int i = base + r * TB + w * TW + ts;
      ok[r] = i < sl.hi8;
      vsc[r] = chan ? 1.f : __half2float(__ushort_as_half(vsh[r]));
#pragma unroll
      for (int h = 0; h < G; ++h)
        if (ok[r] && c == 0) stash[h * S + (i - sl.lo8)] = s[r][h];
    }
    fold_batch<G, R8>(st, s, [&](int r, float (&vf)[16]) { unpack_i8x16(vr[r], vf); }, vsc, ok, nr);
    if (more) load_v(base + TB * R8);
  }
}

// FP16 ring slots [lo16, hi) on the vector ALU.
// The new token (slot n - 1) is taken from the call's arguments, not read back from the ring.  A
// trip covers four slots per lane-group of a single head (two where a group of heads fills the
// registers; eight take all of them and with that the second workgroup of a CU: 12 heads, 8
// sequences 1.2 times slower).  The next trip is requested while this one is summed up, and the
// slots a last trip does not have cost no arithmetic.  12 heads of 64 channels, 513 slots: 8.8 us
// per launch with trips of two slots and nothing ahead, 8.1 like this.
template <int D, int G>
__device__ __forceinline__ void stream_fp16_valu(const CacheView &cv, const AttendLaunch &a, const Slice &sl, float sm,
                                                 const float (&qf)[G][16], Stream<G> &st,
                                                 float *stash, int S) {
  constexpr int LPT = D / 16, TW = kWave / LPT, TB = kAttWaves * TW, R16 = G == 1 ? 4 : 2;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int c = lane % LPT, ts = lane / LPT;
  const __half *K16 = cv.k16 + (size_t)sl.u * cv.cap16 * D + c * 16;
  const __half *V16 = cv.v16 + (size_t)sl.u * cv.cap16 * D + c * 16;
  const size_t call_row = ((size_t)sl.b * cv.Hkv + sl.g) * D + c * 16;
  if (sl.lo16 >= sl.hi16) return;
  int4 kr[R16][2], vr[R16][2];
  auto load = [&](int base, const __half *ring, const __half *call, int4 (&x)[R16][2]) {
#pragma unroll
    for (int r = 0; r < R16; ++r) {
      const int i = min(base + r * TB + w * TW + ts, sl.hi16 - 1);
      const int4 *p = (const int4 *)(i == sl.n - 1 ? call + call_row : ring + (size_t)ring_row(sl.h16, i - sl.n8, cv.cap16) * D);
      x[r][0] = p[0];
      x[r][1] = p[1];
    }
  };
  load(sl.lo16, K16, a.knew, kr);
  load(sl.lo16, V16, a.vnew, vr);
  for (int base = sl.lo16; base < sl.hi16; base += TB * R16) {
    float s[R16][G], vsc[R16];
    bool ok[R16];
    const int nr = (sl.hi16 - base + TB - 1) / TB;
#pragma unroll
    for (int r = 0; r < R16; ++r) {
      if (r >= nr) {
#pragma unroll
        for (int h = 0; h < G; ++h) s[r][h] = 0.f;
        continue;
      }
      float kf[16];
      unpack_h16x16(kr[r][0], kr[r][1], kf);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc = fmaf(qf[h][e], kf[e], acc);
        s[r][h] = group_sum(acc, LPT) * sm;
      }
    }
    const bool more = base + TB * R16 < sl.hi16;
    if (more) load(base + TB * R16, K16, a.knew, kr);
#pragma unroll
    for (int r = 0; r < R16; ++r) {
      const int i = base + r * TB + w * TW + ts;
      ok[r] = i < sl.hi16;
      vsc[r] = 1.f;
#pragma unroll
      for (int h = 0; h < G; ++h)
        if (ok[r] && c == 0) stash[h * S + sl.cnt8 + (i - sl.lo16)] = s[r][h];
    }
    fold_batch<G, R16>(st, s, [&](int r, float (&vf)[16]) { unpack_h16x16(vr[r][0], vr[r][1], vf); }, vsc, ok, nr);
    if (more) load(base + TB * R16, V16, a.vnew, vr);
  }
}

// Merge the slot lane-groups of a wavefront and store the wavefront's partial
// (m, l, o[G][D]) as entry `pidx` of the workgroup's LDS partial arrays.
template <int D, int G>
__device__ __forceinline__ void store_stream_partial(Stream<G> &st, int pidx, float *wm, float *wl,
                                                     float *wo_p) {
  constexpr int LPT = D / 16;
  const int lane = threadIdx.x & 63;
  const int c = lane % LPT;
  const float NEG = -INFINITY;
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float mw = wave_max(st.m[h]);
    const float f = (st.m[h] == NEG) ? 0.f : __expf(st.m[h] - mw);
    const float lf = st.l[h] * f;
    const float l = row_stride_sum<LPT>(swap_halves16(swap_halves32(lf, lf), swap_halves32(lf, lf)));
    // sixteen channel sums over the lane-groups: every exchange between rows halves the values a
    // lane carries (12 exchanges instead of 32), so row r of 16 lanes ends up with channels
    // [4 r, 4 r + 4) of every lane-group's sixteen
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float lo = swap_halves32(st.acc[h][e] * f, st.acc[h][8 + e] * f);
      const float hi = swap_halves32(st.acc[h][4 + e] * f, st.acc[h][12 + e] * f);
      o[e] = row_stride_sum<LPT>(swap_halves16(lo, hi));
    }
    if (lane == 0) { wm[h * kAttWaves + pidx] = mw; wl[h * kAttWaves + pidx] = l; }
    if ((lane & 15) < LPT) *(float4 *)&wo_p[h * D + c * 16 + 4 * (lane >> 4)] = make_float4(o[0], o[1], o[2], o[3]);
  }
}

// e^x for x <= 0 (-inf included, which gives 0) to about one ulp: the hardware exponential of the
// rounded product p = x log2 e, times e^d of what the rounding lost, d = x - p ln 2 (ln 2 in two
// floats; |d| < 1e-5, so 1 + d is exact enough).
// No range checks: the result cannot overflow, and below 2^-126 it may flush to zero.
__device__ __forceinline__ float exp_nonpos(float x) {
  x = fmaxf(x, -100.0f);
  const float p = x * 1.44269502e+00f;
  const float d = fmaf(-p, -1.90465430e-09f, fmaf(-p, 6.93147182e-01f, x));
  const float r = __builtin_amdgcn_exp2f(p);
  return fmaf(r, d, r);
}
// The same to the bit down to -100, where a NaN must show and -inf must weigh nothing (probabilities of an output, whose sum nothing
// else carries a NaN into).  Not the argument is bounded, whose maximum would take a NaN for -100, but the correction, which
// is no number where the argument is infinite.
__device__ __forceinline__ float exp_nonpos_or_nan(float x) {
  const float p = x * 1.44269502e+00f;
  const float d = fmaxf(fmaf(-p, -1.90465430e-09f, fmaf(-p, 6.93147182e-01f, x)), -1e-4f);
  const float r = __builtin_amdgcn_exp2f(p);
  return fmaf(r, d, r);
}
// 1 / x for a positive, finite double to about 1e-15 relative: the fp32 reciprocal estimate and two
// Newton steps (a correctly rounded division costs ten times the instructions and nothing
// downstream is that exact).
__device__ __forceinline__ double recip_pos(double x) {
  double r = (double)__builtin_amdgcn_rcpf((float)x);
  r = r * (2.0 - x * r);
  return r * (2.0 - x * r);
}

// The fp16 number nearest to x, rounded once.  The fp32 number in between is rounded to odd (towards zero, the last bit
// set where x is none): with thirteen bits more than fp16 it then never lies on a tie that x does not, eight instructions
// against the forty of the compiler's conversion.
__device__ __forceinline__ __half half_of_double(double x) {
  const float f = (float)x;
  const unsigned toward_zero = __float_as_uint(f) - (fabs((double)f) > fabs(x) ? 1u : 0u);
  return __float2half_rn(__uint_as_float(toward_zero | ((double)f != x ? 1u : 0u)));
}

// lambda^k
__device__ __forceinline__ double pow_count(double x, unsigned k) {
  double r = 1.0;
  for (; k; k >>= 1) {
    if (k & 1u) r *= x;
    x *= x;
  }
  return r;
}
// r / gq for a row r < 16 (gq_mul = 65536 / gq + 1)
__device__ __forceinline__ int token_of_row(const AttendLaunch &a, int r) { return (int)((unsigned)(r * a.gq_mul) >> 16); }
// Weight of row r's mass in the importance update of a call with tq tokens:
// lambda^(tq - 1 - token), 0 for padding rows; for a single token (G rows, one per head) exactly 1.
template <int G>
__device__ __forceinline__ double row_weight(const AttendLaunch &a, int r) {
  if constexpr (G <= 8) return 1.0;
  const int left = a.tq - 1 - token_of_row(a, r);
  return left < 0 ? 0.0 : pow_count((double)a.ema_decay, (unsigned)left);
}

// Query row r of a unit is (token r / gq of the call, head r % gq of the group); rows past
// tq * gq are padding.  Element e = r * D + d of the unit's [rows][D] output lives at
// out[b][token][g * gq + head][d].
template <bool kRows>
__device__ __forceinline__ size_t out_index(const CacheView &cv, const AttendLaunch &a, const Slice &sl, int tq, int gq,
                                            int e, int D) {
  // (32-bit arithmetic: the output of one call stays far below 2^31 elements)
  const unsigned r = (unsigned)e / (unsigned)D, d = (unsigned)e - r * (unsigned)D;
  const unsigned t = kRows ? (unsigned)token_of_row(a, (int)r) : 0u, hq = r - t * (unsigned)gq;   // (r < gq of a single token)
  return (size_t)(((((unsigned)sl.b * (unsigned)tq + t) * (unsigned)cv.Hkv + (unsigned)sl.g) * (unsigned)gq + hq) * (unsigned)D + d);
}

constexpr int kEmaAhead = 4;                         // slots per thread whose EMA is requested ahead
// The EMA values a thread will update, requested behind the first rows and used behind the exchange.
template <bool kPaged>
__device__ __forceinline__ void request_ema(const CacheView &cv, const Slice &sl, float (&ema_old)[kEmaAhead]) {
  const float *EMA = cv.ema + (size_t)sl.u * cv.cap;
#pragma unroll
  for (int k = 0; k < kEmaAhead; ++k) {
    // no branch per lane (a slot past the slice re-reads its last one; the appended token's slot
    // holds a stale value): the uses mask both cases
    ema_old[k] = 0.f;
    const int t = threadIdx.x + k * kAttThreads;
    if (k * kAttThreads < sl.ntok) ema_old[k] = EMA[slot_plane_row<kPaged>(cv, sl, sl.slot_of(min(t, sl.ntok - 1)))];
  }
}

// ---------------------------------------------------------------------------------------
// Epilogue shared by both bodies.  On entry wm/wl/wo hold NP per-wavefront partials
// (after a workgroup barrier): partial k is [G][D] floats, rows DS apart, at
// wo + (k % kAttWaves) * WSTR + (k / kAttWaves) * G * DS; stash holds the slice's raw scores.
// kPhase 0: the whole epilogue in one kernel (merge, publish, wait for the unit's other splits,
// gather, EMA, output).  kPhase 1: merge and publish only; kPhase 2: gather, EMA and output in a
// later launch, which needs no wait (wm/wl are unused and wo holds the [G][gs] weights) --
// the pair serves shapes whose splits cannot all be resident at once.
// ---------------------------------------------------------------------------------------
template <int D, int G, int NP, int WSTR, int kPhase = 0, int DR = D, int DS = D, bool kPaged = false>
__device__ __forceinline__ void attend_epilogue(const CacheView &cv, const AttendLaunch &a,
                                                const Slice &sl, int ns, int S, float *stash,
                                                float *wm, float *wl, float *wo, float *gm,
                                                double *ginv, float (&ema_old)[kEmaAhead]) {
  const int tid = threadIdx.x;
  const float NEG = -INFINITY;
  // more than 8 rows only occur in multi-token calls; otherwise rows are the heads of one token
  const int tq = G > 8 ? a.tq : 1, gq = G > 8 ? a.gq : G;
  unsigned long long *ml = a.part_ml + ((size_t)sl.ul * a.max_splits + sl.j) * G * 2;
  unsigned long long *po = a.part_o + ((size_t)sl.ul * a.max_splits + sl.j) * G * D;
  constexpr int kPre = kPhase == 0 ? kEmaAhead : 0;
  const bool exchange = kPhase != 0 || ns > 1;       // partials go through device memory
  float *EMA = cv.ema + (size_t)sl.u * cv.cap;
  auto ema_row = [&](int t) { return slot_plane_row<kPaged>(cv, sl, sl.slot_of(t)); };
  // The EMA values requested at the start are taken here: loads and stores share one in-order counter, so that a wait for
  // them further down would be one for the published words and the gathered partials too.
#pragma unroll
  for (int k = 0; k < kPre; ++k) asm volatile("" : "+v"(ema_old[k]));
  // Weights of the workgroup merge: a wavefront's output elements all belong to one row, so a row's NP statistics lie in
  // eight neighbouring lanes (lane k of group r: wavefront k's part of row 8 b + r) and three lane moves merge them; the
  // weights reach the merge as scalars.  (Every thread formed the eight weights of its row for itself before, behind a thread
  // per row that did the same for the statistics: 16 splits 1218 -> 1176 us per step of 64 launches, with the lane arithmetic
  // of the EMA rows below.)
  constexpr int HB = (G + 7) / 8;
  static_assert(kPhase == 2 || NP == 8, "one group of eight lanes per row");
  const int lane8 = tid & 63;
  float row_m[HB], row_l[HB], part_w[HB];              // of row 8 b + lane / 8: maximum, normaliser, weight of partial lane % 8
  if (kPhase != 2) {
#pragma unroll
    for (int b = 0; b < HB; ++b) {
      const int at = min(64 * b + lane8, G * NP - 1);  // (lanes past the last row repeat its last partial; nothing reads them)
      const float mk = wm[at], lk = wl[at];
      row_m[b] = group_max(mk, 8);
      const bool live = mk > NEG;                      // an empty partial may hold anything and weighs nothing
      part_w[b] = live ? __expf(mk - row_m[b]) : 0.f;
      row_l[b] = group_sum(live ? lk * part_w[b] : 0.f, 8);
    }
    // the statistics go out first: their trip to the unit's other splits runs behind the output merge
    if (exchange && tid < kWave && (!a.withhold || sl.j != 0)) {   // (test hook: split 0 keeps its words to itself)
#pragma unroll
      for (int b = 0; b < HB; ++b) {
        const int h = 8 * b + (lane8 >> 3);
        if ((lane8 & 7) == 0 && h < G) {
          st_tagged(&ml[h * 2], tag_of(a), row_m[b]);
          st_tagged(&ml[h * 2 + 1], tag_of(a), row_l[b]);
        }
      }
    }
  }
  // A unit with a single split is complete here: global statistics per row, uniform over the workgroup.
  float g_m[G];
  double g_w[G];                                       // the row's mass weight over its normaliser
  double row_inv[HB], row_w[HB];
  if (kPhase == 0 && !exchange) {
#pragma unroll
    for (int b = 0; b < HB; ++b) {
      row_inv[b] = recip_pos((double)row_l[b]);
      row_w[b] = row_inv[b] * row_weight<G>(a, 8 * b + (lane8 >> 3));
    }
  }
  auto lane_f = [](float v, int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l)); };
  auto lane_d = [](double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
  };
  // workgroup merge of the per-wavefront output partials: kEPT channels per thread, each
  // published as a word that carries the launch's epoch, so that nobody has to wait for the
  // stores to land before announcing them
  constexpr int kEPT = G * D > kAttThreads ? 2 : 1;
  constexpr int kMerge = (G * D + kEPT * kAttThreads - 1) / (kEPT * kAttThreads);
  static_assert(D % (kEPT * kWave) == 0, "a wavefront's elements belong to one row");
  if (kPhase != 2) {
#pragma unroll
    for (int p = 0; p < kMerge; ++p) {
      const int idx = kEPT * (tid + p * kAttThreads);
      const int h = __builtin_amdgcn_readfirstlane(idx / D);
      if (h >= G) break;
      // row 8 b + r: one pass of two channels per thread covers exactly eight rows, other shapes have one pass
      const int b = p, r8 = (h - 8 * b) * 8;
      float ok2[NP][kEPT];
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        // partial k belongs to wavefront k % kAttWaves
        const float *src = &wo[(k % kAttWaves) * WSTR + (k / kAttWaves) * G * DS + h * DS + (idx - h * D)];
        if constexpr (kEPT == 2) {
          const float2 t2 = *(const float2 *)src;
          ok2[k][0] = t2.x;
          ok2[k][kEPT - 1] = t2.y;
        } else {
          ok2[k][0] = *src;
        }
      }
      float o[kEPT] = {};
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const float f = lane_f(part_w[b], r8 + k);
#pragma unroll
        for (int e = 0; e < kEPT; ++e) o[e] = __float_as_int(f) != 0 ? fmaf(ok2[k][e], f, o[e]) : o[e];
      }
      if (!exchange) {
        // same arithmetic as the general merge below (weight e^0 = 1), without the trip through device memory
        const double inv = lane_d(row_inv[b], r8);
#pragma unroll
        for (int e = 0; e < kEPT; ++e) {
          // (DR < D: the matrix-core body pads a 64-channel head to its 128-channel tiles)
          if (h < tq * gq && a.out && idx + e - h * D < DR)
            a.out[out_index<(G > 8)>(cv, a, sl, tq, gq, h * DR + (idx + e - h * D), DR)] = half_of_double((double)o[e] * inv);
        }
      } else {
#pragma unroll
        for (int e = 0; e < kEPT; ++e) st_tagged(&po[idx + e], tag_of(a), o[e]);
      }
    }
  }
  TS(19);
  if (kPhase == 1) return;
  // The unit's global softmax statistics.  A wavefront takes one (row, split) per lane, so the gs
  // lanes (gs = ns rounded up to a power of two) that share a row reduce to the row's (M, L) with
  // lane moves; a unit of up to 64 (row, split) pairs is one wavefront's work.  (All wavefronts
  // polling for themselves saves the barrier behind it and is slower: the polls then crowd out the
  // stores they wait for -- 12.6 against 10.6 us per launch with 16 splits.)
  const unsigned long long *words = a.part_ml + (size_t)sl.ul * a.max_splits * G * 2;
  const unsigned long long *pou = a.part_o + (size_t)sl.ul * a.max_splits * G * D;
  float *pml = wo;                                   // [G][gs] weights of the splits' partials, reuses the merge buffer
  const int lg = ns > 1 ? 32 - __builtin_clz(ns - 1) : 0;   // <= 6: groups never straddle a wavefront
  const int gs = 1 << lg;
  // This split normalises `per` elements of the unit's [G][D] output.  A lane takes kOut of an element's ns partial values
  // (split sub + q * lanes), the `lanes` that share an element are neighbours: the words a thread needs are requested
  // together, and an element's address, sum and store come once (16 rows, four splits: 0.9 us from the request to the
  // store; a pass per kOut-th element with a lane per split took 1.8).
  constexpr int kOutLg = G > 8 ? 2 : G > 4 ? 1 : 0, kOut = 1 << kOutLg;
  const int per = (int)div_splits(a, G * D + ns - 1);
  const int lgl = max(lg - kOutLg, 0);               // log2(lanes)
  const int epp = kAttThreads >> lgl;                // output elements per pass over the workgroup
  const int sub = tid & ((1 << lgl) - 1), oe = tid >> lgl;   // this thread's first split and element within a pass
  unsigned long long opre[kOut];
  auto out_word = [&](int p, int q) {                // of pass p: the q-th word, or the unit's first where there is none
    const int os = sub + (q << lgl), i = p * epp + oe, e = sl.j * per + i;
    return &pou[os < ns && i < per && e < G * D ? (size_t)os * G * D + e : 0];
  };
  const unsigned tag = tag_of(a);
  __shared__ int s_ok;
  if (exchange) {
    const int lane = tid & 63, hpr = kWave >> lg;    // rows per round
    const int os = lane & (gs - 1);
    if (tid == 0) s_ok = 1;
    if (kPhase == 0) lds_barrier();                  // the merge has read the buffer the weights land in
    else __syncthreads();
    TS(20);
    for (int h0 = (tid >> 6) * hpr; h0 < G; h0 += kAttWaves * hpr) {
      const int h = h0 + (lane >> lg);
      const bool mine = h < G && os < ns;
      const unsigned long long *src = words + (mine ? (size_t)os * G + h : 0) * 2;
      unsigned long long wvm, wvl;
      bool here;
      // the wait is bounded; in a second launch every word is there
      for (int spins = 0;; ++spins) {
        wvm = ld_tagged(src);
        wvl = ld_tagged(src + 1);
        here = !mine || ((unsigned)(wvm >> 32) == tag && (unsigned)(wvl >> 32) == tag);
        if (__builtin_amdgcn_ballot_w64(!here) == 0ull || spins > a.spin_limit) break;
        __builtin_amdgcn_s_sleep(1);
      }
      if (!here) s_ok = 0;
      const float ms = mine ? __uint_as_float((unsigned)wvm) : NEG;
      const float ls = mine ? __uint_as_float((unsigned)wvl) : 0.f;
      const float M = group_max(ms, gs);
      const float es = ms > NEG ? exp_nonpos(ms - M) : 0.f;          // an empty partial weighs nothing
      const double inv = recip_pos(group_sum((double)es * (double)ls, gs));
      if (mine) {
        if (os == 0) { gm[h] = M; ginv[h] = inv; ginv[G + h] = inv * row_weight<G>(a, h); }
        // what split os's output partial of this row is multiplied by
        pml[(h << lg) + os] = es * (float)inv;
      }
    }
    lds_barrier();
    TS(21);
    if (s_ok == 0) {                                 // the wait expired
      if (tid == 0) atomicAdd(&cv.stats[kStatDeviceErr], 1ull);
      return;
    }
    // the output partials are requested now and used behind the importance arithmetic
#pragma unroll
    for (int q = 0; q < kOut; ++q) opre[q] = ld_tagged(out_word(0, q));
#pragma unroll
    for (int h = 0; h < G; ++h) { g_m[h] = gm[h]; g_w[h] = ginv[G + h]; }
  } else {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      g_m[h] = lane_f(row_m[h / 8], 8 * (h & 7));
      g_w[h] = lane_d(row_w[h / 8], 8 * (h & 7));
    }
  }
  TS(22);
  // ---- this split normalises its share of the unit's output (online-softmax merge) ----
  auto finish_output = [&]() {
    for (int p = 0; p * epp < per; ++p) {
      const int i = p * epp + oe, e = sl.j * per + i;                // element of the [G][D] output
      const bool mine = i < per && e < G * D;
      if (p > 0) {
#pragma unroll
        for (int q = 0; q < kOut; ++q) opre[q] = ld_tagged(out_word(p, q));
      }
      // a word that is not this launch's yet is asked for again (bounded)
      auto all_here = [&]() {
        bool here = true;
#pragma unroll
        for (int q = 0; q < kOut; ++q) here &= !mine || sub + (q << lgl) >= ns || (unsigned)(opre[q] >> 32) == tag;
        return here;
      };
      bool here = all_here();
      for (int spins = 0; __builtin_amdgcn_ballot_w64(!here) != 0ull; ++spins) {
        if (spins > a.spin_limit) break;
        __builtin_amdgcn_s_sleep(1);
        if (!here) {
#pragma unroll
          for (int q = 0; q < kOut; ++q) opre[q] = ld_tagged(out_word(p, q));
          here = all_here();
        }
      }
      const unsigned long long missing = __builtin_amdgcn_ballot_w64(!here);
      if (missing) {                                                 // the wait expired: no output from this wavefront
        if ((tid & 63) == __builtin_ctzll(missing)) atomicAdd(&cv.stats[kStatDeviceErr], 1ull);
        continue;
      }
      const int h = mine ? e / D : 0;
      float c = 0.f;
#pragma unroll
      for (int q = 0; q < kOut; ++q) {
        const int os = sub + (q << lgl);
        const float wgt = mine && os < ns ? pml[(h << lg) + os] : 0.f;   // e^{m_s - M} / L of that split and row
        c += wgt > 0.f ? __uint_as_float((unsigned)opre[q]) * wgt : 0.f;   // (an empty partial may hold anything)
      }
      c = group_sum(c, 1 << lgl);
      if (mine && sub == 0 && h < tq * gq && a.out && e - h * D < DR)
        a.out[out_index<(G > 8)>(cv, a, sl, tq, gq, h * DR + (e - h * D), DR)] = __float2half_rn(c);
    }
  };
  // ---- mass + EMA of the slice ----
  // a <- lambda^tq a + gain * sum over the rows of lambda^(tq-1-token) p; ginv[G + h] holds
  // row h's weight over its normaliser.  Slots appended by this call start at 0.
  const double lam = pow_count((double)a.ema_decay, (unsigned)tq);
  const double oml = a.mass_gain;
  const int first_new = sl.n - tq;
  // The new values of the first kPre slots per thread stay in registers until the output is
  // out: a store between the request of the output partials and their use would make that use
  // wait for the store's acknowledgement as well (loads and stores share one in-order counter).
  float ema_new[kPre + 1];
#pragma unroll
  for (int k = 0; k < kPre; ++k) {
    const int t = tid + k * kAttThreads;
    if (t < sl.ntok) {
      double A = 0.0;
#pragma unroll
      for (int h = 0; h < G; ++h) A += (double)exp_nonpos(stash[h * S + t] - g_m[h]) * g_w[h];
      const double old = (sl.slot_of(t) >= first_new) ? 0.0 : (double)ema_old[k];   // a new token starts at 0
      ema_new[k] = (float)(lam * old + oml * A);
      if (!exchange) EMA[ema_row(t)] = ema_new[k];
    }
  }
  TS(30);
  if (exchange) {
    finish_output();
    TS(23);
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
      const int t = tid + k * kAttThreads;
      if (t < sl.ntok) EMA[ema_row(t)] = ema_new[k];
    }
  }
  // the rest of the slice in batches of kBatch slots per thread: branch-free loads first (a
  // slot past the slice re-reads its last one), so a long slice costs one round trip per
  // batch, not one per slot
  constexpr int kBatch = 4;
  for (int t0 = tid + kPre * kAttThreads; t0 < sl.ntok; t0 += kBatch * kAttThreads) {
    float old[kBatch];
    int row[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      row[k] = ema_row(min(t0 + k * kAttThreads, sl.ntok - 1));
      old[k] = EMA[row[k]];
    }
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int t = t0 + k * kAttThreads;
      if (t < sl.ntok) {
        double A = 0.0;
#pragma unroll
        for (int h = 0; h < G; ++h) A += (double)exp_nonpos(stash[h * S + t] - g_m[h]) * g_w[h];
        const double prev = (sl.slot_of(t) >= first_new) ? 0.0 : (double)old[k];   // a new token starts at 0
        EMA[row[k]] = (float)(lam * prev + oml * A);
      }
    }
  }
  TS(31);
}

// ---------------------------------------------------------------------------------------
// Kernel 1: vector-ALU body for every slot
// ---------------------------------------------------------------------------------------
// kSpill: the first launch of the two-launch form -- the slice's raw scores go to device
// scratch instead of LDS and the kernel ends after publishing its partial.
template <int D, int G, bool kSpill = false>
__global__ __launch_bounds__(kAttThreads) void attend_kernel(const int32_t *w_len, const int32_t *w_n8, const int32_t *w_h16, const int32_t *w_h8, int w_unit0, int w_hkv, int w_kvm, CacheView cv, AttendLaunch a_in, int ns,
                                                             int S) {
  // (the unit's counters are requested first, from arguments that arrive in registers: see attend_mfma_kernel)
  const int w_words = (((threadIdx.x & 3) == 0 ? w_len : (threadIdx.x & 3) == 1 ? w_n8 : (threadIdx.x & 3) == 2 ? w_h16 : w_h8))
      [w_unit0 + blockIdx.z * w_hkv + (w_kvm ? blockIdx.x : blockIdx.y)];
  const AttendLaunch a = resolve_launch(cv, a_in);
  constexpr int NP = kAttWaves;
  extern __shared__ __align__(16) float smem[];
  float *stash = kSpill ? a.spill + ((size_t)unit_in_layer(cv, a) * ns + split_index(a)) * G * S
                        : smem;                 // [G][S] raw scores of the slice
  float *wo = smem + (kSpill ? 0 : (size_t)G * S);   // [NP][G][D] per-wave un-normalised output
  float *wm = wo + NP * G * D;                  // [G][NP] per-wave maximum
  float *wl = wm + NP * G;                      // [G][NP] per-wave normaliser
  float *gm = wl + NP * G;                      // [G] global maximum
  double *ginv = (double *)(gm + G + (G & 1));  // [2 G]: 1 / global normaliser, the same times the row's mass weight

  // the queries with them: their place does not depend on the counters
  constexpr int LPT = D / 16;
  const int c = (threadIdx.x & 63) % LPT;
  int4 qraw[G][2];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const int4 *qp = (const int4 *)(a.q + ((size_t)(blockIdx.z * cv.Hkv + kv_head_index(a)) * G + h) * D + c * 16);
    qraw[h][0] = qp[0];
    qraw[h][1] = qp[1];
  }
  const Slice sl = make_slice(cv, a, ns, S, &w_words);
  append_new_token<D>(cv, a, sl, ns, 1);
  float ema_old[kEmaAhead];
  if (!kSpill) request_ema<false>(cv, sl, ema_old);

  Stream<G> st;
  st.reset();
  float qf[G][16];
#pragma unroll
  for (int h = 0; h < G; ++h) unpack_h16x16(qraw[h][0], qraw[h][1], qf[h]);
  if (cv.chan) {
    // per-channel scales: fold the K scales of this lane's 16 channels into the query for the
    // INT8 slots, scale the accumulated INT8 output by the V scales, reload the plain query
    float sc[16];
    const int4 *kp = (const int4 *)(cv.ks + (size_t)sl.u * D + c * 16);
    unpack_h16x16(kp[0], kp[1], sc);
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < 16; ++e) qf[h][e] *= sc[e];
    stream_int8_valu<D, G>(cv, sl, a.sm_scale, qf, st, stash, S);
    const int4 *vp = (const int4 *)(cv.vs + (size_t)sl.u * D + c * 16);
    unpack_h16x16(vp[0], vp[1], sc);
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < 16; ++e) st.acc[h][e] *= sc[e];
    load_q_slices<D, G>(cv, a, sl, qf);
  } else {
    stream_int8_valu<D, G>(cv, sl, a.sm_scale, qf, st, stash, S);
  }
  stream_fp16_valu<D, G>(cv, a, sl, a.sm_scale, qf, st, stash, S);
  store_stream_partial<D, G>(st, threadIdx.x >> 6, wm, wl, wo + (threadIdx.x >> 6) * G * D);
  __syncthreads();
  attend_epilogue<D, G, NP, G * D, kSpill ? 1 : 0>(cv, a, sl, ns, S, stash, wm, wl, wo, gm, ginv, ema_old);
}

// Second launch of the two-launch form: same grid; merges the published partials of the unit,
// updates the EMA of its slice from the spilled scores and normalises its share of the output.
template <int D, int G, int DR = D>
__global__ __launch_bounds__(kAttThreads) void attend_finish_kernel(const int32_t *w_len, const int32_t *w_n8, const int32_t *w_h16, const int32_t *w_h8, int w_unit0, int w_hkv, int w_kvm, CacheView cv, AttendLaunch a_in, int ns,
                                                                    int S) {
  const AttendLaunch a = resolve_launch(cv, a_in);
  extern __shared__ __align__(16) float smem[];
  float *pml = smem;                            // [G][gs], gs = ns rounded up to a power of two (below 2 ns)
  float *gm = pml + (size_t)ns * G * 2;         // [G]
  double *ginv = (double *)(gm + G + (G & 1));  // [2 G]
  const Slice sl = make_slice(cv, a, ns, S);
  float *stash = a.spill + ((size_t)unit_in_layer(cv, a) * ns + split_index(a)) * G * S;
  float unused[kEmaAhead];
  attend_epilogue<D, G, 1, 0, 2, DR>(cv, a, sl, ns, S, stash, nullptr, nullptr, pml, gm, ginv, unused);
}

// ---------------------------------------------------------------------------------------
// Kernel 2: matrix-core body (D = 128, or D = 64 padded to the same tiles)
// ---------------------------------------------------------------------------------------
constexpr int kTile = 32;              // slots per wavefront tile
constexpr int kKRow = 128 + 16;        // LDS row stride of the INT8 K tile (bytes)
constexpr int kKRow16 = 256 + 16;      // LDS row stride of the 16-slot FP16 K tile (bytes)
constexpr int kVRow16 = 256 + 32;      // and of the FP16 V tile: the transposing read takes eight-lane pieces of four
                                       // rows, which this stride puts on different banks
constexpr int kPRow = 32 + 8;          // LDS row stride of the probability tile (halfs)
constexpr int kPartRow = 128 + 4;      // LDS row stride of a wavefront's output partial (floats): a 16-byte store of
                                       // sixteen rows meets different banks
constexpr int kStashPad = 4;           // the same for the raw scores of sixteen rows
// per wavefront: K, V and the scales, and for single tokens the probabilities of up to eight heads
constexpr int kRowsTileBytes = 2 * kTile * kKRow + 2 * kTile * 4;
constexpr int kHeadTileBytes = kRowsTileBytes + 8 * kPRow * 2;
static_assert(16 * kKRow16 <= kTile * kKRow && 16 * kVRow16 <= kTile * kKRow, "an FP16 tile takes the room of an INT8 one");

// Transposing LDS reads, per group of sixteen lanes.  tr8: lane l reads 8 bytes of row l / 2, columns 8 (l & 1) + [0, 8),
// and gets byte l of each of the eight rows.  tr16: lane l reads four halfs of row l / 4, columns 4 (l & 3) + [0, 4),
// and gets half l of each of the four rows.  p is the lane's own piece.
typedef int confkv_i2 __attribute__((ext_vector_type(2)));
typedef short confkv_s4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 lds_read_tr8(const uint8_t *p) {
  const confkv_i2 v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) confkv_i2 *)p);
  return make_uint2((unsigned)v.x, (unsigned)v.y);
}
__device__ __forceinline__ half4_t lds_read_tr16(const uint8_t *p) {
  return __builtin_bit_cast(half4_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) confkv_s4 *)p));
}

// 4 int8 (one dword) -> 4 fp16 (two dwords), exact: c ^ 0x80 is c + 128 as an unsigned byte,
// 0x6400 | byte is the fp16 number 1024 + byte, and subtracting 1152 leaves c.
__device__ __forceinline__ void cvt_i8x4_f16x4(unsigned w, half2_t &lo, half2_t &hi) {
  const unsigned x = w ^ 0x80808080u;
  const unsigned a = __builtin_amdgcn_perm(x, 0x64646464u, 0x00050004u);
  const unsigned b = __builtin_amdgcn_perm(x, 0x64646464u, 0x00070006u);
  const half2_t bias = {(_Float16)1152.0f, (_Float16)1152.0f};
  lo = __builtin_bit_cast(half2_t, a) - bias;
  hi = __builtin_bit_cast(half2_t, b) - bias;
}

// Same without the subtraction: the fp16 numbers c + 1152.  Used for the value operand, where
// the constant is taken out again after the contraction (sum_i p_i (v_i + 1152) =
// sum_i p_i v_i + 1152 sum_i p_i) at a cost of one accumulated sum per head.
constexpr float kCodeBias = 1152.0f;
__device__ __forceinline__ half8_t cvt_i8x8_f16x8_biased(unsigned w0, unsigned w1) {
  const unsigned x0 = w0 ^ 0x80808080u, x1 = w1 ^ 0x80808080u;
  uint4 r;
  r.x = __builtin_amdgcn_perm(x0, 0x64646464u, 0x00050004u);
  r.y = __builtin_amdgcn_perm(x0, 0x64646464u, 0x00070006u);
  r.z = __builtin_amdgcn_perm(x1, 0x64646464u, 0x00050004u);
  r.w = __builtin_amdgcn_perm(x1, 0x64646464u, 0x00070006u);
  return __builtin_bit_cast(half8_t, r);
}

__device__ __forceinline__ half8_t cvt_i8x8_f16x8(unsigned w0, unsigned w1) {
  half2_t p0, p1, p2, p3;
  cvt_i8x4_f16x4(w0, p0, p1);
  cvt_i8x4_f16x4(w1, p2, p3);
  half8_t r;
  r[0] = p0[0]; r[1] = p0[1]; r[2] = p1[0]; r[3] = p1[1];
  r[4] = p2[0]; r[5] = p2[1]; r[6] = p3[0]; r[7] = p3[1];
  return r;
}

// A 16x16 score tile leaves the matrix core with head 4 * (lane / 16) + i in element i, so at
// G <= 4 only the first 16 lanes hold real rows and every softmax instruction would work on
// three quarters of padding.  Two lane-row swaps regroup the real rows over the whole wavefront:
//   G <= 4: one value per lane; lane row r = lane / 16 holds head r
//   G  > 4: two values per lane; value j of lane row r holds head 2j + (r >> 1) + 4 (r & 1)
// The slot (tile column lane % 16) stays where it is.
template <int G>
struct RowMap {
  static constexpr int NV = G <= 4 ? 1 : 2;
  static __device__ __forceinline__ int head(int j, int r) { return G <= 4 ? r : 2 * j + (r >> 1) + 4 * (r & 1); }
};
// rows (a0, b0, a2, b2) of the two operands
__device__ __forceinline__ float swap16_even(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, a),
                                                   __builtin_bit_cast(unsigned, b), false, false);
  return __builtin_bit_cast(float, r[0]);
}
// rows (a0, a1, b0, b1) of the two operands
__device__ __forceinline__ float swap32_low(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a),
                                                   __builtin_bit_cast(unsigned, b), false, false);
  return __builtin_bit_cast(float, r[0]);
}
template <int G>
__device__ __forceinline__ void regroup_rows(const floatx4_t &acc, float (&z)[RowMap<G>::NV]) {
  if constexpr (G <= 4) {
    z[0] = swap32_low(swap16_even(acc[0], acc[1]), swap16_even(acc[2], acc[3]));
  } else {
    z[0] = swap32_low(acc[0], acc[1]);
    z[1] = swap32_low(acc[2], acc[3]);
  }
}
// A quantity that is uniform over each lane row of the regrouped layout, for the lanes of the transposed output: the
// value of head t16 = lane % 16 (lanes past the heads get anything).  The 16-row form holds it there already.
template <int G, int NV>
__device__ __forceinline__ float head_of_column(const float (&x)[NV], int t16) {
  if constexpr (G > 8) {
    return x[0];
  } else if constexpr (G <= 4) {
    // (all four read before the choice: a read inside it becomes a branch)
    float row[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) row[r] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x[0]), 16 * r));
    const float lo = (t16 & 1) ? row[1] : row[0], hi = (t16 & 1) ? row[3] : row[2];
    return (t16 & 2) ? hi : lo;
  } else {
    const int from = 32 * (t16 & 1) + 16 * ((t16 >> 2) & 1);
    const float v0 = __shfl(x[0], from, kWave), v1 = __shfl(x[1], from, kWave);
    return (t16 & 2) ? v1 : v0;
  }
}
// maximum and sum over the four lanes that share lane % 16
__device__ __forceinline__ float rows4_max(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float((unsigned)a[0]), __uint_as_float((unsigned)a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float((unsigned)b[0]), __uint_as_float((unsigned)b[1]));
}
__device__ __forceinline__ float rows4_sum(float v) {
  v = swap_halves32(v, v);
  return swap_halves16(v, v);
}

// ---------------------------------------------------------------------------------------
// Requests for a slice's rows, shared by the single-tile and the many-rows kernel: item it of a slice is its it-th 32-slot
// INT8 tile, or behind those a 16-slot FP16 tile; a wavefront takes either as 8 KB of rows, four 1 KB pieces of K and four of V.
// ---------------------------------------------------------------------------------------
// One item in flight: lane (piece, row) of piece q holds 16 bytes of row r8 + 8 q (INT8, r8 = lane / 8) or r4 + 4 q (FP16,
// r4 = lane / 16), and of INT8 slots one raw scale: lanes 0..31 the K scales of the tile's slots, 32..63 the V scales.
struct TileRegs {
  int4 k0, k1, k2, k3, v0, v1, v2, v3;
  unsigned short sc;
};
struct TileSource {
  const int8_t *k8, *v8, *k16, *v16;     // the unit's planes
  const unsigned short *ks, *vs;
  const int8_t *kn, *vn;                 // calls of several tokens: their rows of this kv-head, tok bytes apart
  unsigned tok;
  int cap8, cap16, ntiles, first_new;    // first_new: first slot whose row comes from the call (0x3fffffff: none)
};
template <int DR, bool kRows>
__device__ __forceinline__ TileSource tile_source(const CacheView &cv, const AttendLaunch &a, const Slice &sl, const int8_t *k8,
                                                  const int8_t *v8, const __half *k16, const __half *v16, const __half *ks,
                                                  const __half *vs, int ntiles, int tq, int first_new) {
  TileSource t = {k8, v8, (const int8_t *)k16, (const int8_t *)v16, (const unsigned short *)ks, (const unsigned short *)vs,
                  nullptr, nullptr, 0u, cv.cap8, cv.cap16, ntiles, first_new};
  if constexpr (kRows) {
    t.kn = (const int8_t *)(a.knew + ((size_t)sl.b * tq * cv.Hkv + sl.g) * DR);
    t.vn = (const int8_t *)(a.vnew + ((size_t)sl.b * tq * cv.Hkv + sl.g) * DR);
    t.tok = (unsigned)(cv.Hkv * DR * 2);
  }
  // (held in registers: a choice between two kernel arguments would become a load from the chosen one's address)
  asm("" : "+s"(t.cap8), "+s"(t.cap16));
  return t;
}
// A branch only chooses bases and offsets; all kinds of items share the load instructions.  (Loads in the branches
// themselves cost the overlap: where two of them meet, the compiler waits for the data to move registers.)
// An item whose rows are one run of the ring -- 1 KB of INT8 or of FP16 rows per piece either way -- takes its
// place from the scalar base; others give every lane its rows; rows past the slice re-read its last one (their scores
// are masked and their probabilities are zero).  Single tokens (kRows false) leave out the call's token: its row is put in
// its place in LDS, and what the ring holds there is not used.
template <int DR, bool kRows, bool kPaged, bool kScales, typename Fp16>
__device__ __forceinline__ void load_item_rows(const CacheView &cv, const TileSource &t, const Slice &sl, int lane, int it,
                                               Fp16 known_fp16, TileRegs &tr) {
  const bool fp16 = known_fp16 || it >= t.ntiles;
  const int base = fp16 ? sl.lo16 + 16 * (it - t.ntiles) : sl.lo8 + it * kTile, end = fp16 ? sl.hi16 : sl.hi8;
  const int head = fp16 ? sl.h16 - sl.n8 : sl.h8, cap = fp16 ? t.cap16 : t.cap8;
  const unsigned row_bytes = fp16 ? 2 * DR : DR;
  const int slots = fp16 ? 16 : kTile;
  const unsigned row0 = (unsigned)ring_row_u(head, base, cap);
  const bool run = !(kPaged && !fp16) && base + slots <= (kRows && fp16 ? min(end, t.first_new) : end) && row0 + slots <= (unsigned)cap;
  const int8_t *kb = fp16 ? t.k16 : t.k8, *vb = fp16 ? t.v16 : t.v8;
  // row of INT8 slot i in the INT8 planes
  auto row8 = [&](int i) -> unsigned {
    if constexpr (kPaged) return (unsigned)((sl.tab[i >> cv.page_lg] << cv.page_lg) | (i & ((1 << cv.page_lg) - 1)));
    else return (unsigned)ring_row_u(sl.h8, i, t.cap8);
  };
  // offsets of the lane's four rows from the (wavefront-uniform) bases, in bytes (see reload_far_item), kRows in pieces of
  // sixteen bytes, which reach everywhere; the rows of call tokens apart
  constexpr unsigned U = kRows ? 16 : 1;
  const unsigned r = DR == 128 && run ? 0u : (unsigned)lane >> (fp16 ? 4 : 3);
  const unsigned col = (unsigned)(lane & (fp16 ? DR / 8 - 1 : DR / 16 - 1)) * (16u / U);
  unsigned o[4], so = row0 + (unsigned)(lane & 31);
  int fresh[kRows ? 4 : 1];
  if (run) {
    kb += (size_t)row0 * row_bytes;
    vb += (size_t)row0 * row_bytes;
#pragma unroll
    for (int q = 0; q < 4; ++q) o[q] = (DR == 128 ? (unsigned)lane * (16u / U) : r * (row_bytes / U) + col) + q * (8 * DR / U);
#pragma unroll
    for (int q = 0; q < (kRows ? 4 : 1); ++q) fresh[q] = -1;
  } else {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int slot = min(base + (int)r + q * (slots / 4), end - 1);
      unsigned row;
      if (kPaged && !fp16) row = row8(slot);
      else row = (unsigned)ring_row_u(head, slot, cap);
      o[q] = row * (row_bytes / U) + col;
      if constexpr (kRows) fresh[q] = fp16 ? slot - t.first_new : -1;
    }
    if (!fp16) so = row8(min(base + (lane & 31), end - 1));
  }
  if constexpr (kRows) {
    const int8_t *pk[4], *pv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const size_t off = (size_t)(fresh[q] >= 0 ? (unsigned)fresh[q] * (t.tok / U) + col : o[q]) * U;
      pk[q] = (fresh[q] >= 0 ? t.kn : kb) + off;
      pv[q] = (fresh[q] >= 0 ? t.vn : vb) + off;
    }
    tr.k0 = ld_stream16(pk[0]); tr.v0 = ld_stream16(pv[0]);
    tr.k1 = ld_stream16(pk[1]); tr.v1 = ld_stream16(pv[1]);
    tr.k2 = ld_stream16(pk[2]); tr.v2 = ld_stream16(pv[2]);
    tr.k3 = ld_stream16(pk[3]); tr.v3 = ld_stream16(pv[3]);
  } else {
    tr.k0 = ld_stream16(kb + o[0]); tr.v0 = ld_stream16(vb + o[0]);
    tr.k1 = ld_stream16(kb + o[1]); tr.v1 = ld_stream16(vb + o[1]);
    tr.k2 = ld_stream16(kb + o[2]); tr.v2 = ld_stream16(vb + o[2]);
    tr.k3 = ld_stream16(kb + o[3]); tr.v3 = ld_stream16(vb + o[3]);
  }
  // (an FP16 tile has no scales: its lanes read anything, the tile's own first bytes)
  if (kScales && !known_fp16)
    tr.sc = ld_stream(fp16 ? (const unsigned short *)kb + lane : (lane < 32 ? t.ks : t.vs) + so);
}

// Rows of an FP16 ring of more than 4 GiB are out of reach of 32-bit offsets from the plane: there an item that is no run of
// the ring (all others count from their own first row) is requested again, by full addresses, where it is used.  (INT8 rows
// take half the room.)
template <int DR>
__device__ __forceinline__ void reload_far_item(const TileSource &t, const Slice &sl, int lane, int it, TileRegs &tr) {
  if (__builtin_expect((unsigned)t.cap16 <= 0x80000000u / DR, 1)) return;
  const int base = sl.lo16 + 16 * (it - t.ntiles), head = sl.h16 - sl.n8;
  if (base + 16 <= sl.hi16 && ring_row_u(head, base, t.cap16) + 16 <= t.cap16) return;
  size_t o[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    o[q] = (size_t)ring_row_u(head, min(base + (lane >> 4) + 4 * q, sl.hi16 - 1), t.cap16) * (2 * DR) + (lane & (DR / 8 - 1)) * 16;
  tr.k0 = ld_stream16(t.k16 + o[0]); tr.v0 = ld_stream16(t.v16 + o[0]);
  tr.k1 = ld_stream16(t.k16 + o[1]); tr.v1 = ld_stream16(t.v16 + o[1]);
  tr.k2 = ld_stream16(t.k16 + o[2]); tr.v2 = ld_stream16(t.v16 + o[2]);
  tr.k3 = ld_stream16(t.k16 + o[3]); tr.v3 = ld_stream16(t.v16 + o[3]);
  // (awaited here: with these loads last in line the others would wait for all that was requested after their rows)
  __builtin_amdgcn_s_waitcnt(0x0f70);
}

// kChan: the INT8 scales are per (unit, channel).  The K scales are folded into the query (a
// second query operand, split into an fp16 head and tail so the fold costs no accuracy), the V
// scales multiply the output once, after the last INT8 tile; the FP16 slots then come last.
// G is the number of query rows per unit: the group size for single-token calls (row = head),
// or kChunkRows for multi-token calls, where row r is (token r / gq, head r % gq), padding rows
// carry a zero query, and a row sees the call's own tokens causally.
// kSpill: the first launch of the two-launch form (raw scores to device scratch, ends after
// publishing its partial).
// kPaged: the INT8 slots live in pages (cv.page_lg), at compile time: see slot_plane_row.
//
// What bounds it: launches of a few MB are a chain (counters, first rows, a tile or two, merge, exchange), and every
// instruction of that chain counts; launches of tens of MB are bound by the vector ALU (two wavefronts per SIMD) about as
// much as by memory.  So a tile costs as few instructions as it can:
//  - a tile that neither wraps nor ends early is loaded from one scalar base and one lane offset;
//  - rows of K and of V go to LDS as they are; the transposing LDS read hands the output contraction its V operand (a
//    register transpose before took 32 byte permutes and 16 stores per INT8 tile);
//  - the output is formed transposed, [channel][row], so a lane holds four neighbouring channels of one row and a
//    wavefront's partial leaves in eight 16-byte stores.
template <int G, bool kChan = false, bool kSpill = false, int DR = 128, bool kPaged = false>
__global__ __launch_bounds__(kAttThreads)
__attribute__((amdgpu_waves_per_eu(2, 2)))
void attend_mfma_kernel(const int32_t *w_len, const int32_t *w_n8, const int32_t *w_h16, const int32_t *w_h8, int w_unit0, int w_hkv, int w_kvm, CacheView cv, AttendLaunch a_in, int ns, int S) {
  // The unit's counters are requested before anything else, from leading scalar kernel arguments
  // (the four arrays, the layer's first unit, the kv-head count, the grid order): the hardware
  // can hand those over in registers when the wavefront starts, so this request does not wait
  // for the fetch of the argument block as everything else does.
  const int w_words = (((threadIdx.x & 3) == 0 ? w_len : (threadIdx.x & 3) == 1 ? w_n8 : (threadIdx.x & 3) == 2 ? w_h16 : w_h8))
      [w_unit0 + blockIdx.z * w_hkv + (w_kvm ? blockIdx.x : blockIdx.y)];
  const AttendLaunch a = resolve_launch(cv, a_in);
  // D: channels of the tiles and partials on chip.  DR: the head dimension in memory; a 64-channel
  // head runs on the same tiles with channels 64..127 holding a second copy of its rows, which the
  // contractions leave out (two k-steps over the real channels for the scores, four channel
  // groups for the output; the other channels of the partial are never written out).
  constexpr int D = 128;
  constexpr bool kRows = G > 8;                 // the 16-row form: scores come out transposed, a lane holds slots of one row
  constexpr int kSteps = DR / 32;               // k-steps of 32 channels in the score contraction
  constexpr int kTileBytes = kRows ? kRowsTileBytes : kHeadTileBytes;
  static_assert(DR == 64 || DR == 128, "head dimension");
  static_assert(!(kChan && DR != 128), "per-channel scales need 128 channels");
  static_assert(!(kPaged && (kChan || kSpill || kRows)), "paged: single tokens, per-token scales, one launch");
  static_assert(G * kPartRow * 4 <= kTileBytes, "a wavefront's output partial must fit its tile buffer");
  constexpr int NP = kAttWaves;                 // one partial per wavefront
  constexpr int kTileFloats = kAttWaves * kTileBytes / 4;
  extern __shared__ __align__(16) float smem[];
  float *tiles = smem;                          // per-wave tile buffers, later [NP][G][kPartRow] partials
  // [G] rows of raw scores; sixteen rows of LDS lie four floats further apart, on different banks
  const int SS = S + (kRows && !kSpill ? kStashPad : 0);
  float *stash = kSpill ? a.spill + ((size_t)unit_in_layer(cv, a) * ns + split_index(a)) * G * S
                        : smem + kTileFloats;
  float *gm = smem + kTileFloats + (kSpill ? 0 : (size_t)G * SS);   // [G]
  double *ginv = (double *)(gm + G + (-G & 3)); // [2 G]
  float *wm = (float *)(ginv + 2 * G);          // [G][NP], on a 16-byte boundary
  float *wl = wm + NP * G;                      // [G][NP]
  float *wo = tiles;

  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tq = kRows ? a.tq : 1, gq = kRows ? a.gq : G;   // tokens of the call, heads per token
  TS_INIT();
  TS(0);
  // every kernel argument the streaming prologue needs, fetched now (one round trip) rather
  // than piecemeal between the dependent loads below
  asm volatile("" ::"s"(cv.k8), "s"(cv.v8), "s"(cv.ks), "s"(cv.vs), "s"(cv.k16), "s"(cv.v16), "s"(cv.len),
               "s"(cv.n8), "s"(cv.head16), "s"(cv.head8), "s"(cv.cap8), "s"(cv.cap16), "s"(cv.Hkv), "s"(cv.B),
               "s"(a.layer), "s"(a.tq), "s"(a.observe_first), "s"(a.q), "s"(a.knew), "s"(a.vnew), "s"(a.ns_magic), "s"(a.ns_shift), "s"(ns));
  const int t16 = lane & 15, g4 = lane >> 4;    // MFMA operand coordinates of this lane
  // Query operand of the score contraction; k-step s covers channels g4*32 + 8s + [0,8), matching
  // the K bytes this lane reads from the tile below.  Rows past the heads of a group repeat the
  // last one: a row of the contraction only reaches its own scores, and nothing reads theirs.  (Requested with the
  // counters: the queries' place does not depend on them.)
  half8_t qa[4];
  {
    // row t16 = (token, head) of the call's [B][tq][Hq][D] queries
    const int row = kRows ? t16 : min(t16, G - 1);
    const int q_tok = kRows ? token_of_row(a, row) : 0, q_head = row - q_tok * gq;
    const bool real = !kRows || q_tok < tq;
    const __half *qrow = a.q + ((((size_t)blockIdx.z * tq + (real ? q_tok : 0)) * cv.Hkv + kv_head_index(a)) * gq + q_head) * DR;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      // (a 64-channel head: two k-steps, step s of lane group g4 covers channels 16 g4 + 8 s + [0, 8))
      int4 raw = make_int4(0, 0, 0, 0);
      if (s < kSteps) raw = *(const int4 *)(qrow + g4 * (8 * kSteps) + 8 * s);
      if (!real) raw = make_int4(0, 0, 0, 0);
      qa[s] = __builtin_bit_cast(half8_t, raw);
    }
  }
  // Paged layout: the unit's block table comes into LDS (requested before the counters, so both
  // trips overlap); every INT8 row address below goes through it.
  int32_t *tab = (int32_t *)((char *)smem + a.tab_off);
  if constexpr (kPaged) {
    const int32_t *gt = cv.pt + (size_t)(a.layer * cv.B * cv.Hkv + unit_in_layer(cv, a)) * cv.npages;
    for (int i = tid; i < cv.npages; i += kAttThreads) tab[i] = gt[i];
  }
  Slice sl = make_slice(cv, a, ns, S, &w_words);
  if constexpr (kPaged) {
    sl.tab = tab;
    __syncthreads();
  }
  TS(2);
  const int c8 = lane & 7, r8 = lane >> 3;      // load coordinates of INT8 rows: 16-byte piece, row
  const int c16 = lane & 15, r4 = lane >> 4;    // and of FP16 rows
  const int8_t *K8 = cv.k8 + (size_t)sl.u * cv.cap8 * DR;
  const int8_t *V8 = cv.v8 + (size_t)sl.u * cv.cap8 * DR;
  const __half *KS = cv.ks + (size_t)sl.u * (kChan ? D : cv.cap8);
  const __half *VS = cv.vs + (size_t)sl.u * (kChan ? D : cv.cap8);
  const __half *K16 = cv.k16 + (size_t)sl.u * cv.cap16 * DR;
  const __half *V16 = cv.v16 + (size_t)sl.u * cv.cap16 * DR;

  // ---------------- the slice as a list of work items ----------------
  // Items 0 .. ntiles-1 are the 32-slot INT8 tiles, the rest the 16-slot FP16 tiles (the same
  // 8 KB of rows each).  Wavefront w takes items w, w + 8, ..; the rows of its next item are
  // requested as soon as the current ones have left the registers for LDS, so one item per
  // wavefront is always in flight.
  const int ntiles = (sl.cnt8 + kTile - 1) / kTile;            // 0 when the split has no INT8 slot
  const int nitems = ntiles + (sl.hi16 - sl.lo16 + 15) / 16;
  // the call's own tokens (slots n - tq .. n - 1, at the end of the unit's last split) are
  // taken from the call's arguments, not read back from the ring: no wait on the append's stores
  // (an observation call appends nothing: every row comes from the ring)
  const int first_new = a.observe_first >= 0 ? 0x3fffffff : sl.n - tq;
  const TileSource ts = tile_source<DR, kRows>(cv, a, sl, K8, V8, K16, V16, KS, VS, ntiles, tq, first_new);
  TileRegs tr;
  auto load_item = [&](int it, auto known_fp16) { load_item_rows<DR, kRows, kPaged, !kChan>(cv, ts, sl, lane, it, known_fp16, tr); };
  // the first item is requested before anything else: its latency covers the append and
  // the query loads
  if (w < nitems) load_item(w, std::false_type{});
  // Single tokens: the new token, slot n - 1, is the last row of the unit's last item.  Lanes 0..15 hold the pieces of
  // its K row, each sixteen of the others those of its V row.
  const bool owns_new = !kRows && sl.hi16 == sl.n && nitems > 0 && ((nitems - 1) & (kAttWaves - 1)) == w;
  int4 new_piece;
  if (owns_new)
    new_piece = *(const int4 *)((r4 ? a.vnew : a.knew) + ((size_t)sl.b * cv.Hkv + sl.g) * DR + (c16 & (DR / 8 - 1)) * 8);
  float ema_old[kEmaAhead];
  if (!kSpill) request_ema<kPaged>(cv, sl, ema_old);
  TS(3);
  append_new_token<DR, kPaged>(cv, a, sl, ns, tq);
  const float NEG = -INFINITY;
  const float sm = a.sm_scale;
  TS(1);

  uint8_t *Kt = (uint8_t *)tiles + (size_t)w * kTileBytes;   // [32][kKRow], or [16][kKRow16] of FP16 slots
  uint8_t *Vt = Kt + kTile * kKRow;                           // [32][kKRow], or [16][kVRow16]
  float *Sc = (float *)(Vt + kTile * kKRow);                  // [32] K scales times sm, [32] V scales
  _Float16 *Pb = (_Float16 *)(Sc + 2 * kTile);                // [kPb][kPRow] (not in the 16-row form)
  constexpr int kPb = G <= 4 ? 4 : 8;

  // Per-channel scales: query operand of the INT8 scores = q * s_k * 2^8 as head + tail in fp16
  // (the power of two keeps the tail of every term that matters a normal number; it is taken
  // back in the score factor), and the V scales of this lane's channels 16 nt + 4 g4 + [0, 4).
  constexpr float kFoldUp = 256.0f;
  half8_t qh[kChan ? 4 : 1], ql[kChan ? 4 : 1];
  half4_t vch[kChan ? 8 : 1];
  if constexpr (kChan) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const half8_t ksv = __builtin_bit_cast(half8_t, *(const int4 *)(KS + g4 * 32 + 8 * s));
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float prod = (float)qa[s][e] * (float)ksv[e] * kFoldUp;
        const _Float16 hi = (_Float16)prod;
        qh[s][e] = hi;
        ql[s][e] = (_Float16)(prod - (float)hi);
      }
    }
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) vch[nt] = *(const half4_t *)(VS + 16 * nt + 4 * g4);
  }
  // Transposed output: element i of group nt is channel 16 nt + 4 g4 + i of row t16.
  floatx4_t O[8];
#pragma unroll
  for (int nt = 0; nt < 8; ++nt) O[nt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  // running softmax state (heads: the regrouped layout; 16 rows: row t16, the same in the four
  // lanes of a row): reference, normaliser (per-lane partial sum) and the sum of the fp16
  // probabilities that met biased INT8 values
  constexpr int NV = kRows ? 1 : RowMap<G>::NV;
  float mrun[NV], lrun[NV], pbias[NV];
  int hd[NV];                                    // head of value j of this lane
#pragma unroll
  for (int j = 0; j < NV; ++j) { mrun[j] = NEG; lrun[j] = 0.f; pbias[j] = 0.f; hd[j] = kRows ? t16 : RowMap<G>::head(j, g4); }
  // causal order inside the call: row t16's token sees slots below this
  const int seen = kRows ? sl.n - tq + token_of_row(a, t16) + 1 : 0;
  float *stash_row = kRows ? stash + (size_t)t16 * SS : stash;

  // A raw score goes to its place in the stash; where there is none, to the wavefront's own scales, which are used up (no
  // branch between the score and the softmax).
  auto keep_score = [&](bool real, int head, int t, float v) {
    if constexpr (kSpill) {
      if (real) stash[(size_t)head * S + t] = v;
    } else {
      smem[real ? kTileFloats + head * SS + t : (int)(Sc - smem) + lane] = v;
    }
  };
  auto rescale = [&](const float (&corr)[NV]) {
    const float c = head_of_column<G>(corr, t16);
#pragma unroll
    for (int nt = 0; nt < DR / 16; ++nt) O[nt] *= c;
  };
  // A wavefront with a single item has no earlier output to rescale (8 splits of a 1000-slot unit: 8.1 -> 7.85 us per
  // launch).  Leaving the first of several items out as well cost units of two items per wavefront 1 %.
  const bool several = nitems > kAttWaves;
  // A loop per kind of item (one loop over both kinds keeps two sets of output registers and copies them in every turn).
  int item = w;
  [[maybe_unused]] int tix = 0;
  for (; item < ntiles; item += kAttWaves) {
    if (tix < 6) TS(4 + 2 * tix);
    // ---- an INT8 tile: registers -> LDS, rows as they are ----
    *(int4 *)(Kt + (r8)*kKRow + c8 * 16) = tr.k0;
    *(int4 *)(Kt + (8 + r8) * kKRow + c8 * 16) = tr.k1;
    *(int4 *)(Kt + (16 + r8) * kKRow + c8 * 16) = tr.k2;
    *(int4 *)(Kt + (24 + r8) * kKRow + c8 * 16) = tr.k3;
    *(int4 *)(Vt + (r8)*kKRow + c8 * 16) = tr.v0;
    *(int4 *)(Vt + (8 + r8) * kKRow + c8 * 16) = tr.v1;
    *(int4 *)(Vt + (16 + r8) * kKRow + c8 * 16) = tr.v2;
    *(int4 *)(Vt + (24 + r8) * kKRow + c8 * 16) = tr.v3;
    if constexpr (!kChan) Sc[lane] = __half2float(__ushort_as_half(tr.sc)) * (lane < 32 ? sm : 1.0f);
    wave_lds_sync();
    if (tix < 6) TS(5 + 2 * tix);
    ++tix;
    // the registers are free again: fetch this wavefront's next item while computing
    if (item + kAttWaves < nitems) load_item(item + kAttWaves, std::false_type{});

    const int base = sl.lo8 + item * kTile;
    // ---- scores of its two 16-slot halves ----
    // heads: sc[sb][j] is slot 16 sb + t16; 16 rows: sc[sb][i] is slot 8 g4 + 4 sb + i of row t16, so that the lane's
    // eight probabilities are the operand of the output contraction as they stand
    constexpr int NS = kRows ? 4 : NV;
    float sc[2][NS], vs[2][kRows ? 4 : 1], ks[2][kRows ? 4 : 1];
    floatx4_t acc[2];
    half8_t kb[2][4];
#pragma unroll
    for (int sb = 0; sb < 2; ++sb) {
      const int krow_of = kRows ? 8 * (t16 >> 2) + 4 * sb + (t16 & 3) : 16 * sb + t16;
      const uint8_t *krow = Kt + krow_of * kKRow + g4 * (8 * kSteps);
      const int4 b0 = *(const int4 *)(krow);
      int4 b1 = b0;
      if constexpr (kSteps == 4) b1 = *(const int4 *)(krow + 16);
      kb[sb][0] = cvt_i8x8_f16x8(b0.x, b0.y);
      kb[sb][1] = cvt_i8x8_f16x8(b0.z, b0.w);
      kb[sb][2] = cvt_i8x8_f16x8(b1.x, b1.y);
      kb[sb][3] = cvt_i8x8_f16x8(b1.z, b1.w);
      acc[sb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
      if constexpr (kChan) {
#pragma unroll
        for (int i = 0; i < (kRows ? 4 : 1); ++i) { ks[sb][i] = sm * (1.0f / kFoldUp); vs[sb][i] = 1.0f; }
      } else if constexpr (kRows) {
        const float4 k4 = *(const float4 *)(Sc + 8 * g4 + 4 * sb), v4 = *(const float4 *)(Sc + kTile + 8 * g4 + 4 * sb);
        ks[sb][0] = k4.x; ks[sb][1] = k4.y; ks[sb][2] = k4.z; ks[sb][3] = k4.w;
        vs[sb][0] = v4.x; vs[sb][1] = v4.y; vs[sb][2] = v4.z; vs[sb][3] = v4.w;
      } else {
        ks[sb][0] = Sc[16 * sb + t16];
        vs[sb][0] = Sc[kTile + 16 * sb + t16];
      }
    }
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        auto contract = [&](const half8_t &q) {
          acc[sb] = kRows ? __builtin_amdgcn_mfma_f32_16x16x32_f16(kb[sb][s], q, acc[sb], 0, 0, 0)
                          : __builtin_amdgcn_mfma_f32_16x16x32_f16(q, kb[sb][s], acc[sb], 0, 0, 0);
        };
        if constexpr (kChan) {
          contract(ql[s]);
          contract(qh[s]);
        } else {
          contract(qa[s]);
        }
      }
    if constexpr (kRows) {
      // an INT8 slot is ahead of a query only in an observation call (appended tokens are FP16)
      const bool plain = base + kTile <= min(sl.hi8, sl.n - tq + 1);
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const int slot = base + 8 * g4 + 4 * sb;
        if (plain) {
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[sb][i] = acc[sb][i] * ks[sb][i];
          *(float4 *)(stash_row + (slot - sl.lo8)) = make_float4(sc[sb][0], sc[sb][1], sc[sb][2], sc[sb][3]);
        } else {
          const int lim = min(seen, sl.hi8);
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            sc[sb][i] = slot + i < lim ? acc[sb][i] * ks[sb][i] : NEG;
            if (slot + i < sl.hi8) stash_row[slot + i - sl.lo8] = sc[sb][i];
          }
        }
      }
    } else {
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const bool valid = base + 16 * sb + t16 < sl.hi8;
        float z[NV];
        regroup_rows<G>(acc[sb], z);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
          const bool real = valid && hd[j] < G;
          sc[sb][j] = real ? z[j] * ks[sb][0] : NEG;
          keep_score(real, hd[j], base + 16 * sb + t16 - sl.lo8, sc[sb][j]);
        }
      }
    }
    if (tix <= 2) TS(24 + (tix - 1) * 3);
    // ---- online softmax ----
    // The running reference m only has to stay within a few units of the true maximum (the
    // merge is exact for any reference), so the row reduction and the rescale of O run only
    // when some score of the tile exceeds the reference by more than kSlack; e^kSlack times
    // the largest fp16 value scale still fits fp16.
    constexpr float kSlack = 4.0f;
    float lm[NV];
    bool grow = false;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      lm[j] = fmaxf(sc[0][j], sc[1][j]);
      if constexpr (kRows) {
#pragma unroll
        for (int i = 1; i < 4; ++i) lm[0] = fmaxf(lm[0], fmaxf(sc[0][i], sc[1][i]));
      }
      grow |= lm[j] > mrun[j] + kSlack;             // also true on the first tile (m = -inf)
    }
    if (__builtin_amdgcn_ballot_w64(grow)) {
      float corr[NV];
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const float mn = fmaxf(mrun[j], kRows ? rows4_max(lm[j]) : row16_max(lm[j]));
        corr[j] = (mn == NEG) ? 1.f : __expf(mrun[j] - mn);
        mrun[j] = mn;
        lrun[j] *= corr[j];
        pbias[j] *= corr[j];
      }
      if (__builtin_expect(several, 0)) rescale(corr);
    }
    half8_t pa;
    if constexpr (kRows) {
#pragma unroll
      for (int sb = 0; sb < 2; ++sb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = (sc[sb][i] == NEG) ? 0.f : __expf(sc[sb][i] - mrun[0]);
          lrun[0] += p;
          const _Float16 ph = (_Float16)(p * vs[sb][i]);
          pbias[0] += (float)ph;                             // exactly what the matrix core will see
          pa[4 * sb + i] = ph;
        }
    } else {
#pragma unroll
      for (int j = 0; j < NV; ++j) {
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
          const float p = (sc[sb][j] == NEG) ? 0.f : __expf(sc[sb][j] - mrun[j]);
          lrun[j] += p;
          const _Float16 ph = (_Float16)(p * vs[sb][0]);
          pbias[j] += (float)ph;                             // exactly what the matrix core will see
          Pb[hd[j] * kPRow + 16 * sb + t16] = ph;            // (rows past the heads of the group: zeros)
        }
      }
      wave_lds_sync();
      // (columns past the heads of the group repeat others; a column only reaches its own output)
      pa = *(const half8_t *)(Pb + (t16 & (kPb - 1)) * kPRow + 8 * g4);
    }
    if (tix <= 2) TS(25 + (tix - 1) * 3);
    // ---- output: O[channel][row] += V[slot][channel] P[slot][row] ----
    // lane t16 of a group of sixteen reads eight channels of row 8 g4 + t16 / 2 and gets the eight slots of channel t16
    const uint8_t *vrow = Vt + (8 * g4 + (t16 >> 1)) * kKRow + 8 * (t16 & 1);
#pragma unroll
    for (int nt = 0; nt < DR / 16; ++nt) {
      const uint2 v = lds_read_tr8(vrow + 16 * nt);
      O[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(cvt_i8x8_f16x8_biased(v.x, v.y), pa, O[nt], 0, 0, 0);
    }
    wave_lds_sync();
  }
  if constexpr (kChan) {
    // The accumulator leaves code units behind the wavefront's last INT8 item: the code bias goes out and the V scales come in.
    float pb[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      pb[j] = (kRows ? rows4_sum(pbias[j]) : row16_sum(pbias[j])) * kCodeBias;
      pbias[j] = 0.f;
    }
    const float bias = head_of_column<G>(pb, t16);
#pragma unroll
    for (int nt = 0; nt < 8; ++nt)
#pragma unroll
      for (int i = 0; i < 4; ++i) O[nt][i] = (O[nt][i] - bias) * (float)vch[nt][i];
  }
  // (everything requested so far, the queries among it, is awaited here: later waits would take the next rows in)
  if constexpr (!kChan) asm volatile("" ::"v"(tr.sc));
  for (; item < nitems; item += kAttWaves) {
    // ---- an FP16 tile: 16 slots ----
    if constexpr (!kRows) reload_far_item<DR>(ts, sl, lane, item, tr);
    *(int4 *)(Kt + (r4)*kKRow16 + c16 * 16) = tr.k0;
    *(int4 *)(Kt + (4 + r4) * kKRow16 + c16 * 16) = tr.k1;
    *(int4 *)(Kt + (8 + r4) * kKRow16 + c16 * 16) = tr.k2;
    *(int4 *)(Kt + (12 + r4) * kKRow16 + c16 * 16) = tr.k3;
    *(int4 *)(Vt + (r4)*kVRow16 + c16 * 16) = tr.v0;
    *(int4 *)(Vt + (4 + r4) * kVRow16 + c16 * 16) = tr.v1;
    *(int4 *)(Vt + (8 + r4) * kVRow16 + c16 * 16) = tr.v2;
    *(int4 *)(Vt + (12 + r4) * kVRow16 + c16 * 16) = tr.v3;
    if (owns_new && item == nitems - 1) {
      // behind the rows above: LDS keeps a wavefront's order.  Its V row takes the rows past the slice too: those hold
      // what the ring had there, and a zero probability does not silence a NaN.
      const int row = sl.n - 1 - (sl.lo16 + 16 * (item - ntiles));
      if (r4 == 0) *(int4 *)(Kt + row * kKRow16 + c16 * 16) = new_piece;
      else
        for (int r = row + r4 - 1; r < 16; r += 3) *(int4 *)(Vt + r * kVRow16 + c16 * 16) = new_piece;
    }
    wave_lds_sync();
    if (item + kAttWaves < nitems) load_item(item + kAttWaves, std::true_type{});

    const int base = sl.lo16 + 16 * (item - ntiles);
    const uint8_t *krow = Kt + t16 * kKRow16 + g4 * (16 * kSteps);
    floatx4_t acc = {0.f, 0.f, 0.f, 0.f};
    half4_t pa;
    bool changed = false;
    float corr[NV];
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
      const half8_t k = *(const half8_t *)(krow + 16 * s);
      acc = kRows ? __builtin_amdgcn_mfma_f32_16x16x32_f16(k, qa[s], acc, 0, 0, 0)
                  : __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], k, acc, 0, 0, 0);
    }
    if constexpr (kRows) {
      // element i: slot base + 4 g4 + i of row t16
      const int slot = base + 4 * g4, lim = min(seen, sl.hi16);
      float sv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sv[i] = slot + i < lim ? acc[i] * sm : NEG;
        if (slot + i < sl.hi16) stash_row[sl.cnt8 + (slot + i - sl.lo16)] = sv[i];
      }
      const float mn = fmaxf(mrun[0], rows4_max(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]))));
      corr[0] = (mn == NEG) ? 1.f : __expf(mrun[0] - mn);
      changed = mn != mrun[0];
      mrun[0] = mn;
      lrun[0] *= corr[0];
      pbias[0] *= corr[0];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float p = sv[i] == NEG ? 0.f : __expf(sv[i] - mn);
        lrun[0] += p;
        pa[i] = (_Float16)p;
      }
    } else {
      const bool valid = base + t16 < sl.hi16;
      float z[NV];
      regroup_rows<G>(acc, z);
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const bool real = valid && hd[j] < G;
        const float sv = real ? z[j] * sm : NEG;
        keep_score(real, hd[j], sl.cnt8 + (base + t16 - sl.lo16), sv);
        const float mn = fmaxf(mrun[j], row16_max(sv));
        corr[j] = (mn == NEG) ? 1.f : __expf(mrun[j] - mn);
        changed |= (mn != mrun[j]);
        mrun[j] = mn;
        const float p = real ? __expf(sv - mn) : 0.f;
        Pb[hd[j] * kPRow + t16] = (_Float16)p;
        lrun[j] = fmaf(lrun[j], corr[j], p);
        pbias[j] *= corr[j];
      }
    }
    if (several && __builtin_amdgcn_ballot_w64(changed)) rescale(corr);
    if constexpr (!kRows) {
      wave_lds_sync();
      pa = *(const half4_t *)(Pb + (t16 & (kPb - 1)) * kPRow + 4 * g4);
    }
    // lane t16 of a group of sixteen reads four channels of row 4 g4 + t16 / 4 and gets the four slots of channel t16
    // (a 64-channel head has four real channel groups: the copies in groups 4..7 are not multiplied)
    const uint8_t *vrow = Vt + (4 * g4 + (t16 >> 2)) * kVRow16 + 8 * (t16 & 3);
#pragma unroll
    for (int nt = 0; nt < DR / 16; ++nt)
      O[nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(lds_read_tr16(vrow + 32 * nt), pa, O[nt], 0, 0, 0);
    wave_lds_sync();
  }
  TS(16);
  // Everything requested has arrived -- which the compiler cannot know of the rows: without this it waits further down, where
  // their registers are used anew, for the published words as well (16 rows: 0.8 us).
  __builtin_amdgcn_s_waitcnt(0x0f70);                  // vmcnt(0)
  // the wavefront's partial goes into its own (now idle) tile buffer
  float *wo_w = tiles + w * (kTileBytes / 4);
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    lrun[j] = kRows ? rows4_sum(lrun[j]) : row16_sum(lrun[j]);
    pbias[j] = (kRows ? rows4_sum(pbias[j]) : row16_sum(pbias[j])) * kCodeBias;   // what the biased INT8 values added per channel
    if ((kRows ? g4 == 0 : t16 == 0) && hd[j] < G) { wm[hd[j] * NP + w] = mrun[j]; wl[hd[j] * NP + w] = lrun[j]; }
  }
  const float bias = head_of_column<G>(pbias, t16);
  if (t16 < G) {
#pragma unroll
    for (int nt = 0; nt < 8; ++nt)
      *(float4 *)(wo_w + t16 * kPartRow + 16 * nt + 4 * g4) =
          make_float4(O[nt][0] - bias, O[nt][1] - bias, O[nt][2] - bias, O[nt][3] - bias);
  }

  TS(17);
  __syncthreads();
  TS(18);
  attend_epilogue<D, G, NP, kTileBytes / 4, kSpill ? 1 : 0, DR, kPartRow, kPaged>(cv, a, sl, ns, SS, stash, wm, wl, wo, gm, ginv, ema_old);
  TS_DUMP();
}

#include "attend_wide.h"
#include "attend_rows.h"
#include "attend_observe.h"

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------

typedef void (*AttendFn)(const int32_t *, const int32_t *, const int32_t *, const int32_t *, int, int, int, CacheView,
                         AttendLaunch, int, int);

static std::atomic<bool> g_use_mfma{true};

static AttendFn attend_fn_valu(int D, int G) {
#define CONFKV_CASE(d, g) \
  if (D == d && G == g) return attend_kernel<d, g>;
  CONFKV_CASE(64, 1) CONFKV_CASE(64, 2) CONFKV_CASE(64, 3) CONFKV_CASE(64, 4) CONFKV_CASE(64, 5)
  CONFKV_CASE(64, 6) CONFKV_CASE(64, 7) CONFKV_CASE(64, 8)
  CONFKV_CASE(128, 1) CONFKV_CASE(128, 2) CONFKV_CASE(128, 3) CONFKV_CASE(128, 4) CONFKV_CASE(128, 5)
  CONFKV_CASE(128, 6) CONFKV_CASE(128, 7) CONFKV_CASE(128, 8)
#undef CONFKV_CASE
  return nullptr;
}

static AttendFn attend_fn_spill(int D, int G, bool finish) {
#define CONFKV_CASE(d, g) \
  if (D == d && G == g) return finish ? (AttendFn)attend_finish_kernel<d, g> : (AttendFn)attend_kernel<d, g, true>;
  CONFKV_CASE(64, 1) CONFKV_CASE(64, 2) CONFKV_CASE(64, 3) CONFKV_CASE(64, 4) CONFKV_CASE(64, 5)
  CONFKV_CASE(64, 6) CONFKV_CASE(64, 7) CONFKV_CASE(64, 8)
  CONFKV_CASE(128, 1) CONFKV_CASE(128, 2) CONFKV_CASE(128, 3) CONFKV_CASE(128, 4) CONFKV_CASE(128, 5)
  CONFKV_CASE(128, 6) CONFKV_CASE(128, 7) CONFKV_CASE(128, 8)
#undef CONFKV_CASE
  // multi-token calls: only the second launch exists for 16 rows (the first is the matrix-core body)
  if (D == 128 && G == kChunkRows && finish) return (AttendFn)attend_finish_kernel<128, kChunkRows>;
  return nullptr;
}

// Second launch behind the matrix-core body at D = 64: the partials are 128 channels wide.
static AttendFn attend_fn_finish_padded(int G) {
#define CONFKV_CASE(g) \
  case g: return (AttendFn)attend_finish_kernel<128, g, 64>;
  switch (G) {
    CONFKV_CASE(2) CONFKV_CASE(3) CONFKV_CASE(4) CONFKV_CASE(5) CONFKV_CASE(6) CONFKV_CASE(7) CONFKV_CASE(8)
    default: return nullptr;
  }
#undef CONFKV_CASE
}

static AttendFn attend_fn_mfma(int D, int G, bool chan) {
  if (D == 64 && !chan) {
#define CONFKV_CASE(g) \
  case g: return (AttendFn)attend_mfma_kernel<g, false, false, 64>;
    switch (G) {
      CONFKV_CASE(2) CONFKV_CASE(3) CONFKV_CASE(4) CONFKV_CASE(5) CONFKV_CASE(6) CONFKV_CASE(7) CONFKV_CASE(8)
      default: return nullptr;
    }
#undef CONFKV_CASE
  }
  if (D != 128) return nullptr;
#define CONFKV_CASE(g) \
  case g: return chan ? (AttendFn)attend_mfma_kernel<g, true> : (AttendFn)attend_mfma_kernel<g, false>;
  switch (G) {
    CONFKV_CASE(2) CONFKV_CASE(3) CONFKV_CASE(4) CONFKV_CASE(5) CONFKV_CASE(6) CONFKV_CASE(7) CONFKV_CASE(8)
    CONFKV_CASE(kChunkRows)
    default: return nullptr;
  }
#undef CONFKV_CASE
}

// The same of the paged layout (single tokens, per-token scales).
static AttendFn attend_fn_paged(int D, int G) {
#define CONFKV_CASE(g) \
  case g: return D == 64 ? (AttendFn)attend_mfma_kernel<g, false, false, 64, true> : (AttendFn)attend_mfma_kernel<g, false, false, 128, true>;
  if (D != 64 && D != 128) return nullptr;
  switch (G) {
    CONFKV_CASE(2) CONFKV_CASE(3) CONFKV_CASE(4) CONFKV_CASE(5) CONFKV_CASE(6) CONFKV_CASE(7) CONFKV_CASE(8)
    default: return nullptr;
  }
#undef CONFKV_CASE
}

static AttendFn attend_fn_mfma_spill(int D, int G, bool chan) {
  if (D == 64 && !chan) {
#define CONFKV_CASE(g) \
  case g: return (AttendFn)attend_mfma_kernel<g, false, true, 64>;
    switch (G) {
      CONFKV_CASE(2) CONFKV_CASE(3) CONFKV_CASE(4) CONFKV_CASE(5) CONFKV_CASE(6) CONFKV_CASE(7) CONFKV_CASE(8)
      default: return nullptr;
    }
#undef CONFKV_CASE
  }
  if (D != 128) return nullptr;
#define CONFKV_CASE(g) \
  case g: return chan ? (AttendFn)attend_mfma_kernel<g, true, true> : (AttendFn)attend_mfma_kernel<g, false, true>;
  switch (G) {
    CONFKV_CASE(2) CONFKV_CASE(3) CONFKV_CASE(4) CONFKV_CASE(5) CONFKV_CASE(6) CONFKV_CASE(7) CONFKV_CASE(8)
    CONFKV_CASE(kChunkRows)
    default: return nullptr;
  }
#undef CONFKV_CASE
}

// The matrix-core kernel serves every grouped-query shape, FP16-only caches included (at G >= 4
// the vector-ALU body runs out of registers); at D = 64 it pads the head to its 128-channel tiles.
static bool wants_mfma(int D, int G, bool /*has_int8*/) {
  return g_use_mfma && attend_fn_mfma(D, G, false) != nullptr;
}

// Groups of 9 to 16 query heads run as a one-token call of the 16-row matrix-core kernel (D = 128).
bool attend_supported(int D, int G) {
  return attend_fn_valu(D, G) != nullptr || (D == 128 && G > 8 && G <= kChunkRows);
}

static size_t attend_lds_bytes(int D, int G, int S, bool mfma) {
  if (mfma) {
    const int NP = kAttWaves;
    size_t floats = (size_t)G * (S + (G > 8 ? kStashPad : 0)) + G + 2 + 2 * NP * G;
    size_t tiles = (size_t)kAttWaves * (G > 8 ? kRowsTileBytes : kHeadTileBytes);
    return (floats * sizeof(float) + (size_t)2 * G * sizeof(double) + tiles + 32 + 15) / 16 * 16;
  }
  size_t floats = (size_t)G * S + (size_t)kAttWaves * G * D + 2 * kAttWaves * G + G + 2;
  return floats * sizeof(float) + (size_t)2 * G * sizeof(double) + 16;
}

struct DeviceLimits {
  int cus = 0;
  size_t max_lds = 0;
  bool ok = false;
};

// The two caches below are shared by every handle of the process; handles may live on
// different host threads, so both are guarded.
static std::mutex g_plan_mutex;

static const DeviceLimits &device_limits() {
  static DeviceLimits lim;
  std::lock_guard<std::mutex> lock(g_plan_mutex);
  if (!lim.ok) {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess) {
      lim.cus = prop.multiProcessorCount;
      lim.max_lds = prop.sharedMemPerBlockOptin ? prop.sharedMemPerBlockOptin
                                                : prop.sharedMemPerBlock;
      if (lim.max_lds > 160 * 1024) lim.max_lds = 160 * 1024;
      lim.ok = lim.cus > 0;
      if (const char *e = getenv("CONF_KV_NO_MFMA")) g_use_mfma = atoi(e) == 0;
    }
  }
  return lim;
}
static int device_cus() { return device_limits().cus; }

// Resident workgroups per CU of a kernel with `lds` bytes of dynamic LDS.
static int attend_occupancy(AttendFn fn, size_t lds) {
  static std::map<std::tuple<const void *, size_t>, int> cache;
  std::lock_guard<std::mutex> lock(g_plan_mutex);
  auto key = std::make_tuple((const void *)fn, lds);
  auto it = cache.find(key);
  if (it != cache.end()) return it->second;
  int nb = 0;
  // The dynamic-LDS ceiling of a kernel is raised once, to the most any plan can ask for: a
  // ceiling set per plan would be lowered again by a later, smaller plan of the same kernel.
  static std::set<const void *> raised;
  if (lds > 64 * 1024 && raised.insert((const void *)fn).second) {
    hipFuncAttributes fa;
    size_t fixed = 0;                            // LDS the kernel declares itself counts against the same limit
    if (hipFuncGetAttributes(&fa, (const void *)fn) == hipSuccess) fixed = fa.sharedSizeBytes;
    (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)(160 * 1024 - std::min<size_t>(fixed, 64 * 1024)));
  }
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void *)fn, kAttThreads, lds) !=
      hipSuccess)
    nb = 0;
  cache[key] = nb;
  return nb;
}

bool attend_plan(int D, int G, bool chan, bool paged, bool chunk, int units_per_layer, int n_ub, int n16_ub, int forced_splits,
                 bool force_two_launch, size_t extra_lds, AttendPlan *plan) {
  const DeviceLimits &lim = device_limits();
  if (!lim.ok) return false;
  if (chunk ? attend_fn_mfma(D, G, chan) == nullptr : attend_fn_valu(D, G) == nullptr) return false;
  const bool mfma = chunk || wants_mfma(D, G, n16_ub < n_ub);
  AttendFn fn = mfma ? (paged ? attend_fn_paged(D, G) : attend_fn_mfma(D, G, chan)) : attend_fn_valu(D, G);
  if (!fn) return false;
  const long long nv = (long long)n_ub + n16_ub;
  // One workgroup per CU measured best: the exchange between the splits of a unit (statistics
  // and partial gather) gets slower with more participants, and a grid that is not a
  // whole number of waves over the CUs leaves a straggler round.  That holds above half of the
  // CUs too: 136 to 256 units of 700 to 9000 slots take 1.03 to 1.38 times as long on two
  // workgroups each as on one (one head, 128 channels, 192 units of 2000 slots, FP16: 41.4 against
  // 46.8 us; 64-slot window: 27.4 against 31.0).
  int want = lim.cus / units_per_layer;
  if (want < 1) want = 1;
  // Measured on 8- and 12-unit layers of 500 to 32768 slots: a unit below about 192 KB is
  // fastest on one workgroup (no exchange at all); above, splits down to about 32 KB each
  // (one 32-slot tile per wavefront) still pay.
  const long long unit_bytes = (long long)(n_ub - n16_ub) * (2 * D + 4) + (long long)n16_ub * 4 * D;
  want = unit_bytes <= 192 * 1024 ? 1 : (int)std::min<long long>(want, unit_bytes / (32 * 1024));
  if (forced_splits > 0) want = std::min<long long>(forced_splits, std::max<long long>(1, nv / 128));
  want = std::max(1, std::min(want, kAttendMaxSplits));
  // preference order: want, want-1, .., 1 (fewer, always co-resident), then want+1, .. (more
  // splits shrink the LDS stash when a long unit does not fit otherwise)
  plan->two_launch = false;
  plan->wide_groups = 0;
  for (int k = 0; k < kAttendMaxSplits && !force_two_launch; ++k) {
    const int ns = k < want ? want - k : k + 1;
    // LDS is sized in steps of 256 slots so the occupancy query is cached across calls
    const int need = (n_ub + ns - 1) / ns + (n16_ub + ns - 1) / ns + 34;
    int S = (need + 255) / 256 * 256;
    size_t lds = attend_lds_bytes(D, G, S, mfma) + extra_lds;
    if (lds > lim.max_lds) {                    // a tight fit: give the rounding up
      S = (need + 31) / 32 * 32;
      lds = attend_lds_bytes(D, G, S, mfma) + extra_lds;
    }
    if (lds > lim.max_lds) continue;
    if (ns > 1) {
      int occ = attend_occupancy(fn, lds);
      if ((long long)occ * lim.cus < (long long)ns * units_per_layer) continue;
    } else if (lds > 64 * 1024) {
      (void)attend_occupancy(fn, lds);          // raises the dynamic-LDS limit
    }
    plan->splits = ns;
    plan->stash_tokens = S;
    plan->lds_bytes = lds;
    plan->mfma = mfma;
    return true;
  }
  // No single-kernel plan: the splits of a unit cannot all be resident (many long units), or
  // the slice's scores do not fit LDS.  Two launches then: the first streams and publishes
  // partials, keeping the raw scores in device scratch; the second merges and updates the EMA.
  // Nothing waits inside a kernel, so any split count works.
  {
    // same split count as the single-kernel plan would like (measured on 64 units of 4096
    // slots: 4 splits 40 us, 16 splits 80 us -- the second launch grows with the split count)
    const int ns = want;
    int S = (n_ub + ns - 1) / ns + (n16_ub + ns - 1) / ns + 34;
    S = (S + 255) / 256 * 256;
    const size_t lds = attend_lds_bytes(D, G, 0, mfma) + extra_lds;
    if (lds > lim.max_lds) return false;
    if (lds > 64 * 1024) (void)attend_occupancy(attend_fn_mfma_spill(D, G, chan), lds);   // raises the dynamic-LDS limit
    plan->splits = ns;
    plan->stash_tokens = S;
    plan->lds_bytes = lds;
    plan->mfma = mfma;
    plan->two_launch = true;
    return true;
  }
}

// Splits of a unit in the many-rows kernel, whose workgroups have a CU each and wait for the unit's other splits: two
// launches on two streams that together need more CUs than there are can each hold some that the other's splits wait for, until the
// polls expire.  256 slots a split, up to eight, are taken while the grid fits the chip.  Beyond that twice the splits pay while a
// split keeps 96 slots, 160 from eight to sixteen, and are taken where two such launches cannot stop each other: a grid of at
// most half of the CUs, or eight kv-heads or a multiple in the kv-head-first grid (major_kv; 0: the other grid).  An XCD then gets
// the splits of kv/8 units in order, so that of a launch that is not all there at most kv/8 * (splits - 1) workgroups per XCD
// wait -- all earlier units are complete and end -- and two launches leave a CU free if that is less than half of its CUs.
// us per launch, eight kv-heads with four heads, 16 tokens: 64 units of 500 slots in 1, 2, 4 splits 31, 24.8, 20.2, of 1000
// in 2, 4 32.1, 26.5; 32 of 1200 in 4, 8 25.8, 22.8; 16 of 5000 in 8, 16 37.3, 33.8, of 9000 52.0, 42.8; 8 of 2000 26.8, 28.3, of
// 3000 30.7, 29.8; of 300 slots, 8 tokens in 1, 2, 4 19.2, 16.8, 16.4; of 600 in 2, 4, 8 20.1, 17.6, 18.5.
int attend_wide_splits(int units_per_layer, int major_kv, int n_ub, int most, int cus) {
  int ns = 1;
  while (ns * 2 <= std::min(most, 8) && ns * 2 * units_per_layer <= cus && n_ub / (ns * 2) >= 256) ns *= 2;
  auto beside = [&](int n) {
    return 2 * n * units_per_layer <= cus ||
           (n * units_per_layer <= cus && major_kv > 0 && major_kv % 8 == 0 && 2 * (major_kv / 8) * (n - 1) < cus / 8);
  };
  while (ns * 2 <= most && beside(ns * 2) && n_ub / (ns * 2) >= (ns * 2 > 8 ? 160 : 96)) ns *= 2;
  return ns;
}

// Calls with more than 16 query rows per unit: row groups (a power of two) and split count.  The
// splits of a unit exchange partials inside the launch, so with more than one split the whole grid
// must be resident (one workgroup per CU: the tile buffers take most of the LDS).
static AttendFn attend_fn_wide(int rg, bool kept) {
  if (kept) return rg == 1 ? (AttendFn)attend_rows_kernel<1> : (AttendFn)attend_rows_kernel<2>;
  return rg == 1 ? (AttendFn)attend_wide_kernel<1> : rg == 2 ? (AttendFn)attend_wide_kernel<2> : (AttendFn)attend_wide_kernel<4>;
}
bool attend_wide_plan(int rows, int units_per_layer, int major_kv, int n_ub, int n16_least, int n16_ub, int forced_splits, AttendPlan *plan) {
  const DeviceLimits &lim = device_limits();
  if (!lim.ok || rows <= kChunkRows || rows > kWideMaxRows) return false;
  int rg = 1;
  while (rg * kWideRows < rows) rg *= 2;
  int ns = attend_wide_splits(units_per_layer, major_kv, n_ub, wide_max_splits(rg * kWideRows), lim.cus);
  if (forced_splits > 0) {
    ns = 1;
    while (ns * 2 <= std::min(forced_splits, wide_max_splits(rg * kWideRows)) && ns * 2 * units_per_layer <= lim.cus && n_ub / (ns * 2) >= 64) ns *= 2;
  }
  // (wherever they fit: 1.00 to 1.15 times as fast over 23 shapes, of one tile to all 48 / rg)
  plan->wide_kept = rg <= 2 && rows_tiles(n_ub, n16_least, n16_ub, ns) <= rows_rounds(rg) * kAttWaves;
  const size_t lds = plan->wide_kept ? attend_rows_lds_bytes(rg, ns) : attend_wide_lds_bytes(rg * kWideRows, ns);
  if (lds > lim.max_lds || attend_occupancy(attend_fn_wide(rg, plan->wide_kept), lds) < 1) return false;
  plan->splits = ns;
  plan->stash_tokens = 0;
  plan->lds_bytes = lds;
  plan->mfma = true;
  plan->two_launch = false;
  plan->wide_groups = rg;
  return true;
}

size_t attend_spill_floats(int units_per_layer, int G, int cap) {
  // splits * S <= n + n16 + splits * (2 + 34 + 255) with n, n16 <= cap
  return (size_t)units_per_layer * G * (2 * (size_t)cap + (size_t)kAttendMaxSplits * 291);
}

// With k = ceil(log2 ns) and the multiplier (2^(31 + k) + e) / ns, e < ns <= 2^k, the quotient before rounding down is x / ns plus
// x e / (ns 2^(31 + k)), which is below 1 / ns for x < 2^31.
unsigned split_divisor(int ns, int *shift) {
  int k = 1;
  while ((1 << k) < ns) ++k;
  *shift = k - 1;
  return (unsigned)((((unsigned long long)1 << (31 + k)) + ns - 1) / ns);
}

hipError_t launch_attend(const CacheView &cv, const AttendLaunch &a_in, const AttendPlan &plan,
                         hipStream_t stream) {
  AttendLaunch a = a_in;
  a.gq_mul = 65536 / std::max(1, a.gq) + 1;
  a.ns_magic = plan.splits > 1 ? split_divisor(plan.splits, &a.ns_shift) : 0u;
  if (plan.two_launch || !plan.mfma) a.dbg = nullptr;      // only the single matrix-core kernel is traced
  const dim3 grid = a.kv_major ? dim3(cv.Hkv, plan.splits, cv.B) : dim3(plan.splits, cv.Hkv, cv.B);
  if (plan.two_launch) {
    const bool rows16 = a.tq > 1 || a.observe_first >= 0 || cv.G > 8;
    const int rows2 = rows16 ? kChunkRows : cv.G;                   // query rows per unit
    if (rows16 && !plan.mfma) return hipErrorInvalidValue;
    AttendFn first = plan.mfma ? attend_fn_mfma_spill(cv.D, rows2, cv.chan != 0) : attend_fn_spill(cv.D, cv.G, false);
    AttendFn second = plan.mfma && cv.D == 64 ? attend_fn_finish_padded(rows2) : attend_fn_spill(cv.D, rows2, true);
    if (!first || !second || !a.spill) return hipErrorInvalidValue;
    hipLaunchKernelGGL(first, grid, dim3(kAttThreads), plan.lds_bytes, stream, cv.len, cv.n8, cv.head16, cv.head8, a.layer * cv.B * cv.Hkv, cv.Hkv, a.kv_major, cv, a, plan.splits,
                       plan.stash_tokens);
    const size_t lds2 = ((size_t)plan.splits * rows2 * 2 + rows2 + 2) * sizeof(float) + 2 * rows2 * sizeof(double);
    hipLaunchKernelGGL(second, grid, dim3(kAttThreads), lds2, stream, cv.len, cv.n8, cv.head16, cv.head8, a.layer * cv.B * cv.Hkv, cv.Hkv, a.kv_major, cv, a, plan.splits,
                       plan.stash_tokens);
    return hipGetLastError();
  }
  if (plan.wide_groups) {
    a.dbg = nullptr;
    a.max_splits = wide_max_splits(plan.wide_groups * kWideRows);
    hipLaunchKernelGGL(attend_fn_wide(plan.wide_groups, plan.wide_kept), grid, dim3(kAttThreads), plan.lds_bytes, stream, cv.len, cv.n8, cv.head16, cv.head8, a.layer * cv.B * cv.Hkv, cv.Hkv, a.kv_major, cv, a, plan.splits, 0);
    return hipGetLastError();
  }
  const bool rows16 = a.tq > 1 || a.observe_first >= 0 || cv.G > 8;
  const int rows = rows16 ? kChunkRows : cv.G;
  if (rows16 && !plan.mfma) return hipErrorInvalidValue;
  AttendFn fn = plan.mfma ? (cv.page_lg ? attend_fn_paged(cv.D, rows) : attend_fn_mfma(cv.D, rows, cv.chan != 0))
                          : attend_fn_valu(cv.D, cv.G);
  if (!fn) return hipErrorInvalidValue;
#ifdef CONFKV_TRACE
  if (a.dbg && plan.mfma) {             // time stamps live in LDS behind the kernel's own
    AttendLaunch at = a;
    at.trace_off = (int)((plan.lds_bytes + 15) / 16 * 16);
    const size_t lds = at.trace_off + kAttWaves * 32 * 8;
    (void)hipFuncSetAttribute((const void *)fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(fn, grid, dim3(kAttThreads), lds, stream, cv.len, cv.n8, cv.head16, cv.head8, a.layer * cv.B * cv.Hkv, cv.Hkv, a.kv_major, cv, at, plan.splits, plan.stash_tokens);
    return hipGetLastError();
  }
#endif
  hipLaunchKernelGGL(fn, grid, dim3(kAttThreads), plan.lds_bytes, stream, cv.len, cv.n8, cv.head16, cv.head8, a.layer * cv.B * cv.Hkv, cv.Hkv, a.kv_major, cv, a, plan.splits,
                     plan.stash_tokens);
  return hipGetLastError();
}

}  // namespace confkv
