// Decode attention for calls that carry more query rows per kv-head than one matrix-core tile
// holds (conf_kv_attend_chunk / conf_kv_observe with tq * G > 16: chunks of a prompt, draft
// tokens under verification; paper: "Compatibility with serving systems").  Included by
// attend.hip, inside namespace confkv, after the helpers of the single-tile kernels.
//
// The call is DEFINED as tq single-token steps (see conf_kv_attend_chunk).  Rows r = token * G +
// head are cut into RG groups of 32; a workgroup of eight wavefronts is RG row groups times
// NS = 8 / RG tile streams.  The slice's K/V tiles (32 INT8 slots or 16 FP16 slots each) are
// brought into LDS eight at a time, one per wavefront -- every K/V byte is read from memory
// once per pass whatever the number of rows, and INT8 codes become fp16 once, exactly, when the tile
// is stored -- and each wavefront then runs ITS rows against the tiles of its stream.  Both
// contractions are formed transposed: scores [slot][row], so that a lane holds slots of one query --
// one reference and one sum per lane and 16 rows, and its probabilities are the operand of the output
// contraction [channel][row] as they stand, with no trip through LDS.  No score is stashed (R x slots
// floats would not fit anywhere): after the splits have exchanged their (m, l, o) per row, a second
// pass gives every wavefront 32 slots at a time and all rows: it recomputes the same scores (the same
// products in the same order), turns them into exact probabilities with the global (M, L), sums each
// slot's column over the rows (weights lambda^(tq-1-token)) in its own registers and updates the
// EMA: no barrier, no LDS but the rows' statistics.  Key bytes are therefore read twice, value bytes once.
//
// Calls of up to 64 rows whose splits have at most 48 / RG tiles go to the kernel in attend_rows.h; this one serves the rest.
// 64 rows against 64 units of 4112 slots in four splits (16 tokens of 4 heads): 54 us per launch in the kernel trace; one sequence of
// 30 000 slots 79 us.  Of 35.3 against 2064 slots, which it served before: 17 for the first pass -- 5 until the first tiles are in
// LDS, then a round of eight in 3.5 to 5 -- 4.5 for the merge and publishing, 4.5 for the exchange and 8 for the second pass.  It uses all 256 registers, and
// what must outlive the first pass is formed anew behind it: with 7 to 10 of them spilled that launch was 40 us.  With sixteen
// rows per wavefront, the scores the other way round, value codes converted by every reader and the second pass through
// the same tiles and barriers it was 50 us (and 203).  Slower too: the second pass's keys requested ahead of the exchange, whose
// polls then wait for them, and three splits' partials at once, 1.08 each.
#pragma once

// A tile in LDS: K as fp16 rows, in an order that makes the four slots a lane's transposed V words hold
// adjacent: row 4 * (slot % 8) + slot / 8 of an INT8 tile, 4 * (slot % 4) + slot / 4 of an FP16 tile.
// V transposed, 64 bytes per channel in that order (its 16-byte pieces xor-ed with the channel, groups of 16
// channels 64 bytes further apart: neither stores nor reads then pile up on few banks); per row the
// factor of the raw score and the value scale.
constexpr int kWideRows = 32;                          // query rows per wavefront
constexpr int kWideVGroup = 16 * 64 + 64;
constexpr int kWideKBytes = kTile * kKRow16;
constexpr int kWideCoreBytes = kWideKBytes + 8 * kWideVGroup;
constexpr int kWideTileBytes = kWideCoreBytes + 2 * kTile * 4;
constexpr int kWidePartRow = 128 + 4;                  // floats per row of a wavefront's output partial
static_assert(kWideRows * kWidePartRow * 4 <= kWideTileBytes, "a partial fits the wavefront's tile buffer");
constexpr int kWideMaxRows = 128;
// (the exchange arrays hold 1024 rows of partials per unit)
__host__ __device__ constexpr int wide_max_splits(int R) { return R <= 64 ? 16 : 8; }

// rows, and behind the tiles: per wavefront and row (m, l); per stream and row a weight; five words per row; the splits' (m, l)
__host__ __device__ constexpr size_t attend_wide_lds_bytes(int R, int ns) {
  return (size_t)kAttWaves * kWideTileBytes + ((size_t)kAttWaves * kWideRows * 3 + 5 * R + (size_t)ns * R * 2) * 4 + 16;
}

// A tile's registers into its LDS buffer; factors of the raw scores and value scales go where the kernel keeps them.
__device__ __forceinline__ void store_wide_tile(uint8_t *Kt, float *factor, float *value, bool is8, int lane, float sm, const TileRegs &tr) {
  const int c8 = lane & 7, r8 = lane >> 3, c16 = lane & 15, r4 = lane >> 4;
  uint8_t *Vt = Kt + kWideKBytes;
  if (is8) {
    // sixteen codes of a row per lane -> sixteen fp16 values (exact)
    auto put_k = [&](int row, const int4 &k) {
      half8_t *dst = (half8_t *)(Kt + row * kKRow16 + c8 * 32);
      dst[0] = cvt_i8x8_f16x8((unsigned)k.x, (unsigned)k.y);
      dst[1] = cvt_i8x8_f16x8((unsigned)k.z, (unsigned)k.w);
    };
    put_k(4 * r8, tr.k0);
    put_k(4 * r8 + 1, tr.k1);
    put_k(4 * r8 + 2, tr.k2);
    put_k(4 * r8 + 3, tr.k3);
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const unsigned x0 = dword_of(tr.v0, q4), x1 = dword_of(tr.v1, q4);
      const unsigned x2 = dword_of(tr.v2, q4), x3 = dword_of(tr.v3, q4);
      const unsigned t0 = __builtin_amdgcn_perm(x1, x0, 0x05010400u), t1 = __builtin_amdgcn_perm(x1, x0, 0x07030602u);
      const unsigned t2 = __builtin_amdgcn_perm(x3, x2, 0x05010400u), t3 = __builtin_amdgcn_perm(x3, x2, 0x07030602u);
      // byte r of o[e] is slot 8r + r8 at channel 16*c8 + 4*q4 + e: K rows 4*r8 .. 4*r8 + 3
      const unsigned o[4] = {__builtin_amdgcn_perm(t2, t0, 0x05040100u), __builtin_amdgcn_perm(t2, t0, 0x07060302u),
                             __builtin_amdgcn_perm(t3, t1, 0x05040100u), __builtin_amdgcn_perm(t3, t1, 0x07060302u)};
      // K rows 16 sb + 4 g + i are piece g, half sb of the channel's 64 bytes; r8 = 4 sb + g
      uint8_t *dst = Vt + c8 * kWideVGroup + 4 * q4 * 64 + (((r8 & 3) ^ q4) * 16) + (r8 >> 2) * 8;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        half2_t lo, hi;
        cvt_i8x4_f16x4(o[e], lo, hi);
        *(uint2 *)(dst + 64 * e) = make_uint2(__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi));
      }
    }
    // row 4 * (slot % 8) + slot / 8 of slot lane % 32
    (lane < 32 ? factor : value)[4 * (lane & 7) + ((lane >> 3) & 3)] = __half2float(__ushort_as_half(tr.sc)) * (lane < 32 ? sm : 1.0f);
  } else {
    *(int4 *)(Kt + (4 * r4) * kKRow16 + c16 * 16) = tr.k0;
    *(int4 *)(Kt + (4 * r4 + 1) * kKRow16 + c16 * 16) = tr.k1;
    *(int4 *)(Kt + (4 * r4 + 2) * kKRow16 + c16 * 16) = tr.k2;
    *(int4 *)(Kt + (4 * r4 + 3) * kKRow16 + c16 * 16) = tr.k3;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const unsigned x0 = dword_of(tr.v0, q4), x1 = dword_of(tr.v1, q4);
      const unsigned x2 = dword_of(tr.v2, q4), x3 = dword_of(tr.v3, q4);
      // half r of a channel's word is slot 4r + r4: K rows 4*r4 .. 4*r4 + 3, piece r4 of eight bytes
      uint8_t *dst = Vt + (c16 >> 1) * kWideVGroup + (8 * (c16 & 1) + 2 * q4) * 64 + r4 * 8;
      *(uint2 *)dst = make_uint2(__builtin_amdgcn_perm(x1, x0, 0x05040100u), __builtin_amdgcn_perm(x3, x2, 0x05040100u));
      *(uint2 *)(dst + 64) = make_uint2(__builtin_amdgcn_perm(x1, x0, 0x07060302u), __builtin_amdgcn_perm(x3, x2, 0x07060302u));
    }
  }
}

// Polls of the unit's ns * R * 2 statistics words (bounded).
__device__ __forceinline__ void gather_statistics(const AttendLaunch &a, const Slice &sl, int ns, int R, unsigned tag, int tid, float *pml, int *s_ok) {
  // every thread gathers some of the ns * R * 2 statistics words of the unit (bounded poll)
  const unsigned long long *words = a.part_ml + (size_t)sl.ul * a.max_splits * R * 2;
  for (int base = 0; base < ns * R * 2; base += kAttThreads) {
    const int idx = base + tid;
    bool here = idx >= ns * R * 2;
    for (int spins = 0;; ++spins) {
      if (!here) {
        const unsigned long long wv = ld_tagged(&words[idx]);
        if ((unsigned)(wv >> 32) == tag) {
          pml[idx] = __uint_as_float((unsigned)wv);
          here = true;
        }
      }
      if (__builtin_amdgcn_ballot_w64(!here) == 0ull) break;
      __builtin_amdgcn_s_sleep(1);
      if (spins > a.spin_limit) {
        if (!here) *s_ok = 0;
        break;
      }
    }
  }
}
// The unit's (M, L) of a row; the statistics of (split, row) become the weight of that split's output partial.  A padding row weighs
// nothing and has the reference `padding`.
template <typename Weight>
__device__ __forceinline__ void finish_statistics(const AttendLaunch &a, int ns, int R, int row, int gq, int tq, float padding, float *pml,
                                                  float *Mrow, float *Irow, Weight *Frow) {
  constexpr float kNothing = -1e30f;
  float M = kNothing;
  for (int s = 0; s < ns; ++s) M = fmaxf(M, pml[(s * R + row) * 2]);
  double L = 0.0;
  for (int s = 0; s < ns; ++s) {
    const float es = exp_nonpos(pml[(s * R + row) * 2] - M);
    L += (double)es * (double)pml[(s * R + row) * 2 + 1];
    pml[(s * R + row) * 2] = es;
  }
  const double inv = recip_pos(L);
  Mrow[row] = row / gq < tq ? M : padding;
  Irow[row] = (float)inv;
  Frow[row] = row / gq < tq ? (Weight)(inv * pow_count((double)a.ema_decay, (unsigned)(tq - 1 - row / gq))) : (Weight)0;
}
// The output rows [own0, own1) from the unit's partials; own(row) is this split's, at the thread's channel.
template <typename Own>
__device__ __forceinline__ void gather_output(const CacheView &cv, const AttendLaunch &a, const Slice &sl, int ns, int R, unsigned tag, int tid, int own0,
                                              int own1, const float *pml, const int *Orow, const float *Irow, Own own) {
  constexpr int D = 128, kRows = kAttThreads / D, kPass = 4;
  const int ch = tid & (D - 1), lane = tid & 63, first = __builtin_amdgcn_readfirstlane(tid >> 6) / (D / kWave);   // (uniform)
  // four rows of a thread at a time, one split after the other (the words of several splits requested together are
  // asked for again as long as one of them is missing: 16 tokens of 4 heads on 64 units 40 against 38 us)
  for (int r0 = own0 + first; r0 < own1; r0 += kRows * kPass) {
    float o[kPass];
#pragma unroll
    for (int k = 0; k < kPass; ++k) {
      const int row = min(r0 + k * kRows, own1 - 1);
      o[k] = own(row) * pml[(sl.j * R + row) * 2];
    }
    for (int s = 0; s < ns; ++s) {
      if (s == sl.j) continue;
      const unsigned long long *src = a.part_o + ((size_t)sl.ul * a.max_splits + s) * R * D + ch;
      unsigned long long wv[kPass];
      auto request = [&]() {
#pragma unroll
        for (int k = 0; k < kPass; ++k) wv[k] = ld_tagged(src + (size_t)min(r0 + k * kRows, own1 - 1) * D);
      };
      auto ready = [&]() {
        bool ok = true;
#pragma unroll
        for (int k = 0; k < kPass; ++k) ok &= (unsigned)(wv[k] >> 32) == tag;
        return ok;
      };
      request();
      bool here = ready();
      for (int spins = 0; __builtin_amdgcn_ballot_w64(!here) != 0ull && spins <= a.spin_limit; ++spins) {   // (bounded)
        __builtin_amdgcn_s_sleep(1);
        request();
        here = ready();
      }
      const unsigned long long missing = __builtin_amdgcn_ballot_w64(!here);
      if (missing && lane == __builtin_ctzll(missing)) atomicAdd(&cv.stats[kStatDeviceErr], 1ull);
#pragma unroll
      for (int k = 0; k < kPass; ++k) {
        const float wgt = pml[(s * R + min(r0 + k * kRows, own1 - 1)) * 2];
        o[k] = fmaf(wgt > 0.f ? __uint_as_float((unsigned)wv[k]) : 0.f, wgt, o[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < kPass; ++k) {
      const int row = r0 + k * kRows;
      const int to = __builtin_amdgcn_readfirstlane(Orow[min(row, own1 - 1)]);
      if (row < own1 && to >= 0) a.out[(size_t)to * D + ch] = __float2half_rn(o[k] * Irow[row]);
    }
  }
}

template <int RG>
__global__ __launch_bounds__(kAttThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attend_wide_kernel(const int32_t *w_len, const int32_t *w_n8, const int32_t *w_h16, const int32_t *w_h8, int w_unit0, int w_hkv, int w_kvm, CacheView cv, AttendLaunch a_in, int ns, int /*unused*/) {
  // (the unit's counters are requested first, from arguments that arrive in registers: see attend_mfma_kernel)
  const int w_words = (((threadIdx.x & 3) == 0 ? w_len : (threadIdx.x & 3) == 1 ? w_n8 : (threadIdx.x & 3) == 2 ? w_h16 : w_h8))
      [w_unit0 + blockIdx.z * w_hkv + (w_kvm ? blockIdx.x : blockIdx.y)];
  const AttendLaunch a = resolve_launch(cv, a_in);
  constexpr int D = 128, NS = kAttWaves / RG, R = RG * kWideRows, RB = R / 16;
  extern __shared__ __align__(16) float smem[];
  uint8_t *tiles = (uint8_t *)smem;
  float *stat_m = (float *)(tiles + kAttWaves * kWideTileBytes);   // [wavefront][32] reference of a row in a stream
  float *stat_l = stat_m + kAttWaves * kWideRows;                  // [wavefront][32] sum of its exponentials
  float *weight = stat_l + kAttWaves * kWideRows;                  // [wavefront][32] what its partial is multiplied by
  float *Mrow = weight + kAttWaves * kWideRows;                    // [R] maximum of a row: the split's, then the unit's
  float *Irow = Mrow + R;                                          // [R] 1 / normaliser
  float *Frow = Irow + R;                                          // [R] the same times the row's mass weight
  int *Srow = (int *)(Frow + R);                                   // [R] slots the row sees (padding rows: 0x7fffffff)
  int *Orow = Srow + R;                                            // [R] its row of the output (padding rows: -1)
  float *pml = (float *)(Orow + R);                                // [ns][R][2] gathered statistics
  __shared__ int s_ok;
  constexpr float kNothing = -1e30f;                               // reference of a row that has seen no slot

  int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = w % RG, st = w / RG;
  const int tq = a.tq;
  int gq = a.gq;
  const float sm = a.sm_scale;
  int t16 = lane & 15, g4 = lane >> 4;
  // Query rows as a matrix-core operand: lane (row t16, channels 32 g4 + 8 s + [0, 8)).  Requested with the counters, which
  // their place does not depend on.  Padding rows repeat the last token's: nothing reads what comes of them.
  half8_t qa[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int row = (2 * rg + r) * 16 + t16, tok = row / gq, head = row - tok * gq;
    const __half *src = a.q + ((((size_t)blockIdx.z * tq + min(tok, tq - 1)) * cv.Hkv + kv_head_index(a)) * gq + head) * D + g4 * 32;
#pragma unroll
    for (int s = 0; s < 4; ++s) qa[r][s] = __builtin_bit_cast(half8_t, *(const confkv_v4i *)(src + 8 * s));
  }
  const Slice sl = make_slice(cv, a, ns, 0x7fffffff, &w_words);

  // a lane's rows: query t16 of each of the wavefront's two blocks.  The row of token t sees slots below
  // n - tq + t + 1; padding rows see everything and weigh nothing.
  int seen[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int tok = (rg * kWideRows + 16 * r + t16) / gq;
    seen[r] = tok < tq ? sl.n - tq + tok + 1 : 0x7fffffff;
  }
  const int see_all = sl.n - tq + 1;                               // slots below this are seen by every row

  const int8_t *K8 = cv.k8 + (size_t)sl.u * cv.cap8 * D;
  const int8_t *V8 = cv.v8 + (size_t)sl.u * cv.cap8 * D;
  const __half *KS = cv.ks + (size_t)sl.u * cv.cap8;
  const __half *VS = cv.vs + (size_t)sl.u * cv.cap8;
  const __half *K16 = cv.k16 + (size_t)sl.u * cv.cap16 * D;
  const __half *V16 = cv.v16 + (size_t)sl.u * cv.cap16 * D;
  const int ntiles = (sl.cnt8 + kTile - 1) / kTile;
  const int ntiles16 = (sl.hi16 - sl.lo16 + 15) / 16;
  const int nitems = ntiles + ntiles16;
  const int nsup = (nitems + kAttWaves - 1) / kAttWaves;

  // the call's own tokens come from the call's arguments, not from the ring
  const TileSource ts = tile_source<D, true>(cv, a, sl, K8, V8, K16, V16, KS, VS, ntiles, tq,
                                             a.observe_first >= 0 ? 0x3fffffff : sl.n - tq);
  // registers -> this wavefront's LDS buffer
  auto store_item = [&](int it, const TileRegs &tr) {
    uint8_t *Kt = tiles + (size_t)w * kWideTileBytes;
    float *sc = (float *)(Kt + kWideCoreBytes);
    store_wide_tile(Kt, sc, sc + kTile, it < ntiles, lane, sm, tr);
  };

  // ---------------- pass 1: online softmax and output per row ----------------
  TileRegs tr;
  auto load_item = [&](int it) { load_item_rows<D, true, false, true>(cv, ts, sl, lane, it, std::false_type{}, tr); };
  if (w < nitems) load_item(w);
  floatx4_t O[2][8];                                       // [block][channel group]: channels 16 nt + 4 g4 + [0, 4) of query t16
  float m[2], l[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    m[r] = kNothing;
    l[r] = 0.f;
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) O[r][nt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  // One 16-slot half of a tile is N = 4 scores per lane and block; an INT8 tile is two of them.  slot(sb, i) is the
  // slot of score i of half sb; the raw scores come in acc, factors and value scales in f and vs.  Leaves the probabilities
  // times the value scales, rounded to fp16, in p.
  auto soften = [&](auto halves, const floatx4_t (&acc)[2][2], const float (&f)[2][4], const float (&vs)[2][4], int lim, bool edge,
                    auto slot, half8_t (&p)[2]) {
    constexpr int H = decltype(halves)::value;
    auto above = [&](int r, int sb, int i, float ref) { return fmaf(acc[r][sb][i], f[sb][i], -ref); };
    float x[2][H][4], top = -INFINITY;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int sb = 0; sb < H; ++sb)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[r][sb][i] = above(r, sb, i, m[r]);
    auto mask = [&]() {
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int sb = 0; sb < H; ++sb)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (slot(sb, i) >= min(lim, seen[r])) x[r][sb][i] = -INFINITY;
    };
    if (edge) mask();
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int sb = 0; sb < H; ++sb)
#pragma unroll
        for (int i = 0; i < 4; ++i) top = fmaxf(top, x[r][sb][i]);
    // INT8 tiles, lazy reference: rescale only when a score of the tile exceeds it by more than this (e^4 times the
    // largest fp16 value scale still fits fp16).  FP16 tiles rescale at every new maximum: their largest probability is
    // then 1, which fp16 holds exactly, where e^3 carries a rounding that the normaliser does not share (FP16-only caches of
    // 100 to 2000 slots 5 to 14 % further from float64).
    if (__builtin_amdgcn_ballot_w64(top > (H == 2 ? 4.0f : 0.0f))) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        float mn = -INFINITY;
#pragma unroll
        for (int sb = 0; sb < H; ++sb)
#pragma unroll
          for (int i = 0; i < 4; ++i) mn = fmaxf(mn, edge && slot(sb, i) >= min(lim, seen[r]) ? -INFINITY : above(r, sb, i, 0.f));
        mn = fmaxf(mn, __shfl_xor(mn, 16, kWave));
        mn = fmaxf(m[r], fmaxf(mn, __shfl_xor(mn, 32, kWave)));
        const float corr = __expf(m[r] - mn);
        m[r] = mn;
        l[r] *= corr;
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) O[r][nt] *= corr;
#pragma unroll
        for (int sb = 0; sb < H; ++sb)
#pragma unroll
          for (int i = 0; i < 4; ++i) x[r][sb][i] = above(r, sb, i, mn);
      }
      if (edge) mask();
    }
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int sb = 0; sb < H; ++sb) {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          e[i] = __expf(x[r][sb][i]);
          p[r][4 * sb + i] = (_Float16)(e[i] * vs[sb][i]);
        }
        l[r] += (e[0] + e[1]) + (e[2] + e[3]);
      }
  };

  __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0): queries and first rows, so that no wait for them is in the loop
  for (int sup = 0; sup < nsup; ++sup) {
    const int mine = sup * kAttWaves + w;
    if (sup > 0) __syncthreads();                      // everybody has left the previous eight tiles
    if (mine < nitems) store_item(mine, tr);
    __syncthreads();
    if (mine + kAttWaves < nitems) load_item(mine + kAttWaves);
#pragma unroll 1
    for (int j = st; j < kAttWaves; j += NS) {
      const int it = sup * kAttWaves + j;
      if (it >= nitems) break;
      const uint8_t *Kt = tiles + (size_t)j * kWideTileBytes;
      const uint8_t *Vt = Kt + kWideKBytes;
      const float *sc = (const float *)(Kt + kWideCoreBytes);
      const uint8_t *krow = Kt + t16 * kKRow16 + g4 * 64;
      floatx4_t acc[2][2];                             // [block][half]
      half8_t p[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) acc[r][0] = acc[r][1] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const half8_t kf = *(const half8_t *)(krow + 16 * s);
#pragma unroll
        for (int r = 0; r < 2; ++r) acc[r][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qa[r][s], acc[r][0], 0, 0, 0);
      }
      if (it < ntiles) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const half8_t kf = *(const half8_t *)(krow + 16 * kKRow16 + 16 * s);
#pragma unroll
          for (int r = 0; r < 2; ++r) acc[r][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qa[r][s], acc[r][1], 0, 0, 0);
        }
        const int base = sl.lo8 + it * kTile;
        const float4 f0 = *(const float4 *)(sc + 4 * g4), f1 = *(const float4 *)(sc + 16 + 4 * g4);
        const float4 v0 = *(const float4 *)(sc + kTile + 4 * g4), v1 = *(const float4 *)(sc + kTile + 16 + 4 * g4);
        const float f[2][4] = {{f0.x, f0.y, f0.z, f0.w}, {f1.x, f1.y, f1.z, f1.w}};
        const float vs[2][4] = {{v0.x, v0.y, v0.z, v0.w}, {v1.x, v1.y, v1.z, v1.w}};
        soften(std::integral_constant<int, 2>{}, acc, f, vs, sl.hi8, base + kTile > min(sl.hi8, see_all),
               [&](int sb, int i) { return base + 8 * i + 4 * sb + g4; }, p);
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
          const half8_t vf = *(const half8_t *)(Vt + nt * kWideVGroup + t16 * 64 + ((g4 ^ (t16 >> 2)) * 16));
#pragma unroll
          for (int r = 0; r < 2; ++r) O[r][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf, p[r], O[r][nt], 0, 0, 0);
        }
      } else {
        const int base = sl.lo16 + 16 * (it - ntiles);
        const float f[2][4] = {{sm, sm, sm, sm}, {sm, sm, sm, sm}}, vs[2][4] = {{1.f, 1.f, 1.f, 1.f}, {1.f, 1.f, 1.f, 1.f}};
        soften(std::integral_constant<int, 1>{}, acc, f, vs, sl.hi16, base + 16 > min(sl.hi16, see_all),
               [&](int, int i) { return base + 4 * i + g4; }, p);
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
          const half4_t vf = *(const half4_t *)(Vt + nt * kWideVGroup + t16 * 64 + g4 * 8);
#pragma unroll
          for (int r = 0; r < 2; ++r)
            O[r][nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf, half4_t{p[r][0], p[r][1], p[r][2], p[r][3]}, O[r][nt], 0, 0, 0);
        }
      }
    }
  }

  // (the lane's indices and the reciprocal of gq anew: kept through the first pass they would spill)
  asm("" : "+v"(tid));
  asm("" : "+s"(gq));
  lane = tid & 63;
  t16 = lane & 15;
  g4 = lane >> 4;
  __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0): nothing is outstanding, which the compiler cannot know
  append_new_token<D>(cv, a, sl, ns, a.tq);                    // (nobody reads the appended rows back in this launch)

  // ---------------- the tile streams of a row merge in LDS ----------------
  if (tid == 0) s_ok = 1;
  __syncthreads();                                       // the tile buffers are free
  {
    float *part = (float *)(tiles + (size_t)w * kWideTileBytes);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      l[r] += __shfl_xor(l[r], 16, kWave);
      l[r] += __shfl_xor(l[r], 32, kWave);
      if (g4 == 0) {
        stat_m[w * kWideRows + 16 * r + t16] = m[r];
        stat_l[w * kWideRows + 16 * r + t16] = l[r];
      }
#pragma unroll
      for (int nt = 0; nt < 8; ++nt) *(floatx4_t *)&part[(16 * r + t16) * kWidePartRow + 16 * nt + 4 * g4] = O[r][nt];
    }
  }
  __syncthreads();
  const size_t row0 = ((size_t)sl.ul * a.max_splits + sl.j) * R;      // this split's first row in the exchange arrays
  const unsigned tag = tag_of(a);
  if (tid < R) {
    const int at = (tid / kWideRows) * kWideRows + tid % kWideRows;   // wavefront (stream s, group): s * RG + tid / 32
    float M = kNothing, L = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) M = fmaxf(M, stat_m[s * R + at]);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const float e = __expf(stat_m[s * R + at] - M);
      weight[s * R + at] = e;
      L = fmaf(stat_l[s * R + at], e, L);
    }
    const int tok = tid / gq;
    Srow[tid] = tok < tq ? sl.n - tq + tok + 1 : 0x7fffffff;
    Orow[tid] = tok < tq ? ((sl.b * tq + tok) * cv.Hkv + sl.g) * gq + tid - tok * gq : -1;
    if (ns > 1) {
      st_tagged(&a.part_ml[(row0 + tid) * 2], tag, M);
      st_tagged(&a.part_ml[(row0 + tid) * 2 + 1], tag, L);
    } else {
      const double inv = recip_pos((double)L);
      Mrow[tid] = tok < tq ? M : 0.f;                      // (the second pass has zero queries in padding rows)
      Irow[tid] = (float)inv;
      Frow[tid] = tok < tq ? (float)(inv * pow_count((double)a.ema_decay, (unsigned)(tq - 1 - tid / gq))) : 0.f;
    }
  }
  __syncthreads();
  // the query rows as the second pass reads them, on their way to LDS
  constexpr int kQ = R * 16 / kAttThreads;               // 16-byte pieces per thread: 1, 2 or 4
  confkv_v4i qreg[kQ];
#pragma unroll
  for (int k = 0; k < kQ; ++k) {                         // (a query's row is its output's)
    const int from = Orow[k * (kAttThreads / 16) + (tid >> 4)];
    const confkv_v4i v = *(const confkv_v4i *)(a.q + (size_t)max(from, 0) * D + (tid & 15) * 8);
    qreg[k] = from >= 0 ? v : confkv_v4i{0, 0, 0, 0};
  }
  // The sum over the streams, complete with one split: four channels of a row per thread and pass, a row's place in the
  // output divided out once.  Otherwise split j finishes the rows [j R / ns, (j + 1) R / ns), whose sum replaces the
  // first stream's partial, and publishes the others: a channel per thread, consecutive lanes on consecutive words (four
  // words of a row per lane took 5.4 us where this takes 2.1), four rows' reads before their writes.  (Read, divided and
  // written one after the other, the 32 rows of a thread took 6 of the 19 us of a call of 128 rows on an empty cache.)
  constexpr int kRows = kAttThreads / D, kPass = 4;
  const int row_w = w / (D / kWave);                     // (uniform)
  const int ch = tid & (D - 1), own0 = sl.j * (R / ns), own1 = own0 + R / ns;
  auto partial = [&](int wave, int row) { return (float *)(tiles + (size_t)wave * kWideTileBytes) + (row % kWideRows) * kWidePartRow + ch; };
  if (a.out && ns == 1) {
    const int c4 = 4 * (tid & 31);
#pragma unroll
    for (int k = 0; k < R / 16; ++k) {
      const int row = 16 * k + (tid >> 5);
      floatx4_t o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const int wave = s * RG + row / kWideRows;
        const floatx4_t v = *(const floatx4_t *)((const float *)(tiles + (size_t)wave * kWideTileBytes) + (row % kWideRows) * kWidePartRow + c4);
        const float wgt = weight[wave * kWideRows + row % kWideRows];
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = fmaf(v[i], wgt, o[i]);
      }
      const int to = Orow[row];
      const half4_t h = {(_Float16)(o[0] * Irow[row]), (_Float16)(o[1] * Irow[row]), (_Float16)(o[2] * Irow[row]), (_Float16)(o[3] * Irow[row])};
      if (to >= 0) *(half4_t *)(a.out + (size_t)to * D + c4) = h;
    }
  } else if (a.out) {
#pragma unroll 1
    for (int k0 = 0; k0 < R / kRows; k0 += kPass) {
      float o[kPass];
#pragma unroll
      for (int k = 0; k < kPass; ++k) {
        const int row = row_w + (k0 + k) * kRows;
        o[k] = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int wave = s * RG + row / kWideRows;
          o[k] = fmaf(*partial(wave, row), weight[wave * kWideRows + row % kWideRows], o[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < kPass; ++k) {
        const int row = row_w + (k0 + k) * kRows;
        if (row >= own0 && row < own1) *partial(row / kWideRows, row) = o[k];
        else st_tagged(&a.part_o[(row0 + row) * D + ch], tag, o[k]);
      }
    }
  }
  uint8_t *Qs = tiles + (size_t)RG * kWideTileBytes;     // (behind the partials that hold the own rows)
  static_assert(R * kKRow16 <= (kAttWaves - RG) * kWideTileBytes, "the query rows fit the idle tile buffers");

  // ---------------- exchange between the splits of the unit ----------------
  if (ns > 1) {
    gather_statistics(a, sl, ns, R, tag, tid, pml, &s_ok);
    __syncthreads();
    if (s_ok == 0) {
      if (tid == 0) atomicAdd(&cv.stats[kStatDeviceErr], 1ull);
      return;
    }
    if (tid < R) finish_statistics(a, ns, R, tid, gq, tq, 0.f, pml, Mrow, Irow, Frow);
  }
  if (ns == 1) __syncthreads();                          // (the partials have been read)
#pragma unroll
  for (int k = 0; k < kQ; ++k) *(confkv_v4i *)(Qs + (k * (kAttThreads / 16) + (tid >> 4)) * kKRow16 + (tid & 15) * 16) = qreg[k];
  __syncthreads();
  if (ns > 1 && a.out) {
    gather_output(cv, a, sl, ns, R, tag, tid, own0, own1, pml, Orow, Irow, [&](int row) { return *partial(row / kWideRows, row); });
  }

  // ---------------- pass 2: exact mass per slot, EMA ----------------
  const double lam = pow_count((double)a.ema_decay, (unsigned)tq);
  const int first_new = sl.n - tq;                       // a token of the call starts at 0
  float *EMA = cv.ema + (size_t)sl.u * cv.cap;
  const int subs8 = (sl.cnt8 + 31) / 32, subs = subs8 + (sl.hi16 - sl.lo16 + 31) / 32;
  // Eight subtiles at a time, one per wavefront; of those left over (all, where there are fewer than eight) several
  // wavefronts share a subtile's rows, and their sums meet in LDS.  (One wavefront took 3 us for the 128 rows of 8 slots, and
  // the seventeenth of 17 subtiles cost a third round.)
  const int whole = subs & ~(kAttWaves - 1), rest = subs - whole;
  int across = 1;
  while (across < rest) across *= 2;
  const int rest_shares = rest ? min(kAttWaves / across, RB) : 1;
  double *red = (double *)stat_m;                        // [wavefront][32]: the streams' statistics are done with
  static_assert(kAttWaves * 32 * sizeof(double) <= (size_t)kAttWaves * kWideRows * 2 * sizeof(float), "the shares' sums fit");
  for (int first = 0; first < subs; first += kAttWaves) {
    const bool split_rows = first == whole;
    const int shares = split_rows ? rest_shares : 1, share = split_rows ? w / across : 0;
    const int t = first + (split_rows ? w % across : w);
    const bool live = share < shares && t < subs;
    int slot_e = 0, row_e = 0;
    bool writes = false;
    float old = 0.f;
    double sum[2] = {0.0, 0.0};
    if (live) {
      const bool is8 = t < subs8;
      const int base = is8 ? sl.lo8 + 32 * t : sl.lo16 + 32 * (t - subs8), lim = is8 ? sl.hi8 : sl.hi16;
      half8_t kb[2][4];
      float f[2];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const int slot = min(base + 16 * sb + t16, lim - 1);
        if (is8) {
          const unsigned row = (unsigned)ring_row_u(sl.h8, slot, cv.cap8);
          const confkv_v4i c0 = *(const confkv_v4i *)(K8 + row * D + g4 * 32), c1 = *(const confkv_v4i *)(K8 + row * D + g4 * 32 + 16);
          kb[sb][0] = cvt_i8x8_f16x8((unsigned)c0[0], (unsigned)c0[1]);
          kb[sb][1] = cvt_i8x8_f16x8((unsigned)c0[2], (unsigned)c0[3]);
          kb[sb][2] = cvt_i8x8_f16x8((unsigned)c1[0], (unsigned)c1[1]);
          kb[sb][3] = cvt_i8x8_f16x8((unsigned)c1[2], (unsigned)c1[3]);
          f[sb] = __half2float(KS[row]) * sm;
        } else {
          // the call's own tokens come from the call's arguments, not from the ring
          const int fresh = a.observe_first >= 0 ? -1 : slot - first_new;
          const __half *src = fresh >= 0 ? a.knew + (((size_t)sl.b * tq + fresh) * cv.Hkv + sl.g) * D
                                         : K16 + (size_t)ring_row(sl.h16, slot - sl.n8, cv.cap16) * D;
#pragma unroll
          for (int s = 0; s < 4; ++s) kb[sb][s] = __builtin_bit_cast(half8_t, *(const confkv_v4i *)(src + g4 * 32 + 8 * s));
          f[sb] = sm;
        }
      }
      // lanes of row g4 = 0 and 1 update the slots of half g4
      slot_e = base + 16 * (g4 & 1) + t16;
      writes = g4 < 2 && slot_e < lim;
      row_e = slot_row(cv, sl.tab, sl.h8, sl.n8, sl.h16, min(slot_e, lim - 1));
      old = EMA[row_e];
      const bool edge = base + 32 > see_all;
#pragma unroll 1
      for (int rb = share; rb < RB; rb += shares) {
        half8_t qf[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[s] = *(const half8_t *)(Qs + (16 * rb + t16) * kKRow16 + g4 * 64 + 16 * s);
        const float4 M4 = *(const float4 *)&Mrow[16 * rb + 4 * g4], F4 = *(const float4 *)&Frow[16 * rb + 4 * g4];
        const int4 S4 = *(const int4 *)&Srow[16 * rb + 4 * g4];
        const float Mi[4] = {M4.x, M4.y, M4.z, M4.w}, Fi[4] = {F4.x, F4.y, F4.z, F4.w};
        const int Si[4] = {S4.x, S4.y, S4.z, S4.w};
        floatx4_t acc[2] = {floatx4_t{0.f, 0.f, 0.f, 0.f}, floatx4_t{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int sb = 0; sb < 2; ++sb) acc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qf[s], kb[sb][s], acc[sb], 0, 0, 0);
#pragma unroll
        for (int sb = 0; sb < 2; ++sb) {
          float c = 0.f;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float e = exp_nonpos(fmaf(acc[sb][i], f[sb], -Mi[i]));
            c = fmaf(edge && base + 16 * sb + t16 >= Si[i] ? 0.f : e, Fi[i], c);
          }
          sum[sb] += (double)c;
        }
      }
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        sum[sb] += __shfl_xor(sum[sb], 16, kWave);
        sum[sb] += __shfl_xor(sum[sb], 32, kWave);
      }
    }
    double mass = g4 == 0 ? sum[0] : sum[1];
    if (shares > 1) {                                    // (the last turn: every wavefront takes it)
      if (live && g4 < 2) red[w * 32 + 16 * g4 + t16] = mass;
      __syncthreads();
      if (share == 0 && writes)
        for (int k = 1; k < shares; ++k) mass += red[(w + k * across) * 32 + 16 * g4 + t16];
    }
    if (share == 0 && writes) EMA[row_e] = (float)(lam * (slot_e >= first_new ? 0.0 : (double)old) + a.mass_gain * mass);
  }
}
