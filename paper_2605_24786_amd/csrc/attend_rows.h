// Decode attention for calls of 17 to 64 query rows per kv-head whose slices are short enough that a wavefront's probabilities stay
// in registers: up to 48 / RG tiles of a split.  Included by attend.hip, inside namespace confkv, behind the general
// many-rows kernel (attend_wide.h), whose tiles and exchange it shares.
//
// That kernel gives every wavefront rows and a stream of tiles, so eight output partials meet in LDS, and a score is formed twice,
// since no place holds rows x slots of them through the exchange: its second pass (keys read again, products again) is 8 us of
// 35 for 64 rows against 64 units of 2064 slots in four splits.  Here a wavefront scores the tiles of its stream for its 32 rows,
// but the output it sums is 16 RG channels of those rows over ALL tiles: the probabilities of a round of eight tiles go
// through LDS (over the keys, which have been used by then) against a reference that the streams share.  The output
// takes 8 RG registers instead of 64, the probabilities 96 in their place, and nothing is merged at the end.  The importance
// needs neither keys nor products again, nor exponentials: a round's probabilities are multiplied by e^(its reference less the
// unit's maximum), one number per row and round, formed in 64 bits.  (Kept as scores, with the exponentials anew,
// the last part took 8.6 us, now 2.)
//
// The launch above: 35.3 -> 33.5 us (medians of kernel traces; 33.0 without the look at infinite values).  By leaving parts out: 12 for its bytes in three rounds, 5 for scores and
// probabilities, 5 for the output (3 with the probabilities rounded to fp16, see there), 4 for publishing, 4 for the exchange, 2 for the importance.  Rounds are vector instructions
// (conversions, exponentials), LDS and matrix instructions in turn, since four barriers keep the wavefronts in step.  Whole steps of
// eight layers, 23 shapes of 17 to 64 rows, 1 to 192 units of 64 to 9000 slots: 1.00 to 1.15 times as fast (1.00 to 1.16 without that look).  Scores and probabilities of a round were
// written out for each kind of tile at first: 240 KB of code, against 50.
#pragma once

constexpr int kRowsRounds = 6;                         // rounds of eight tiles, times RG: 96 registers
__host__ __device__ constexpr int rows_rounds(int RG) { return kRowsRounds / RG; }
constexpr int kRowsPartRow = 128 + 4;                  // floats per row of the split's output

// tiles; their factors; per wavefront and row a maximum and a sum; six words per row; per round and row a reference, then a weight;
// the splits' (m, l)
__host__ __device__ constexpr size_t attend_rows_lds_bytes(int RG, int ns) {
  return (size_t)kAttWaves * kWideTileBytes +
         ((size_t)rows_rounds(RG) * kAttWaves * kTile + 2 * kAttWaves * kWideRows + (5 + rows_rounds(RG)) * RG * kWideRows + (size_t)ns * RG * kWideRows * 2) * 4 + 16;
}
// The most tiles that a split of a unit of at most n slots, least16 to n16 of them FP16, may have (make_slice: INT8 slots cut at
// multiples of 32, FP16 slots evenly).  Fewer FP16 slots than n16 -- an eviction took some, an import brought few, an observation
// ends ahead of the last ones -- are more INT8 slots: a tile more, as long as the FP16 share still fills t16.  So the INT8 slots
// counted are those beside the fewest FP16 slots that do.  (Every FP16 tile less makes room for half an INT8 tile.)
int rows_tiles(int n, int least16, int n16, int ns) {
  const int t16 = ((n16 + ns - 1) / ns + 15) / 16;
  const int n8 = n - std::min(n16, std::max(least16, 16 * ns * (t16 - 1) + 1));
  return (least16 < n ? ((n8 + ns - 1) / ns + 31 + kTile - 1) / kTile : 0) + t16;
}

// Sum over the sixteen lanes of a row of eight values, each of which ends in a pair of lanes: value 4 (t16 / 8) + (t16 / 2) % 4.
// Partners mirror a row, its half and a quad, so the lanes that differ in a bit exchange the halves it chooses between.
// (two rows by the caller and two lanes in fp32, the rest in 64 bits)
__device__ __forceinline__ double row16_scatter_sum(const float (&v)[8], int t16) {
#define CONFKV_DPP(v, ctrl)                                                                                   \
  __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(v), ctrl, 0xf, 0xf, true),                         \
                   __builtin_amdgcn_mov_dpp(__double2loint(v), ctrl, 0xf, 0xf, true))
  double a[4], b[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float keep = t16 & 8 ? v[4 + i] : v[i], send = t16 & 8 ? v[i] : v[4 + i];
    a[i] = (double)(keep + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, send), 0x140, 0xf, 0xf, true)));   // row_mirror
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double keep = t16 & 4 ? a[2 + i] : a[i], send = t16 & 4 ? a[i] : a[2 + i];
    b[i] = keep + CONFKV_DPP(send, 0x141);              // row_half_mirror
  }
  const double keep = t16 & 2 ? b[1] : b[0], send = t16 & 2 ? b[0] : b[1];
  const double c = keep + CONFKV_DPP(send, 0x1B);       // quad_perm [3,2,1,0]
  return c + CONFKV_DPP(c, 0xB1);                       // quad_perm [1,0,3,2]
#undef CONFKV_DPP
}
// Maximum over the lanes that agree modulo 16.
__device__ __forceinline__ float column_max(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float((unsigned)r[0]), __uint_as_float((unsigned)r[1]));
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float((unsigned)s[0]), __uint_as_float((unsigned)s[1]));
}

// Whether a tile holds a value or a value scale that is not finite (of any lane, to all).
__device__ __forceinline__ bool odd_values(const TileRegs &tr, bool is8, int lane) {
  bool odd;
  if (is8) {
    odd = lane >= 32 && (tr.sc & 0x7c00) == 0x7c00;
  } else {
    half2_t sum = {0, 0};                                // finite values times 0
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const unsigned x[4] = {dword_of(tr.v0, q4), dword_of(tr.v1, q4), dword_of(tr.v2, q4), dword_of(tr.v3, q4)};
#pragma unroll
      for (int r = 0; r < 4; ++r) sum = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, x[r]), half2_t{0, 0}, sum);
    }
    odd = !(sum[0] == 0 && sum[1] == 0);
  }
  return __builtin_amdgcn_ballot_w64(odd) != 0ull;
}

template <int RG>
__global__ __launch_bounds__(kAttThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attend_rows_kernel(const int32_t *w_len, const int32_t *w_n8, const int32_t *w_h16, const int32_t *w_h8, int w_unit0, int w_hkv, int w_kvm, CacheView cv, AttendLaunch a_in, int ns, int /*unused*/) {
  // (the unit's counters are requested first, from arguments that arrive in registers: see attend_mfma_kernel)
  const int w_words = (((threadIdx.x & 3) == 0 ? w_len : (threadIdx.x & 3) == 1 ? w_n8 : (threadIdx.x & 3) == 2 ? w_h16 : w_h8))
      [w_unit0 + blockIdx.z * w_hkv + (w_kvm ? blockIdx.x : blockIdx.y)];
  const AttendLaunch a = resolve_launch(cv, a_in);
  constexpr int D = 128, NS = kAttWaves / RG, R = RG * kWideRows, kRounds = rows_rounds(RG);
  extern __shared__ __align__(16) float smem[];
  uint8_t *tiles = (uint8_t *)smem;
  float *factor = (float *)(tiles + kAttWaves * kWideTileBytes);   // [tile][32] factors of the raw scores
  float *stat_m = factor + kRounds * kAttWaves * kTile;            // [wavefront][32] maximum of a row in a round
  float *stat_l = stat_m + kAttWaves * kWideRows;                  // [wavefront][32] sum of a row's exponentials
  double *Frow = (double *)(stat_l + kAttWaves * kWideRows);       // [R] a row's mass weight over its normaliser
  float *Mrow = (float *)(Frow + R);                               // [R] its maximum over the unit
  float *Irow = Mrow + R;                                          // [R] 1 / normaliser
  int *Orow = (int *)(Irow + R);                                   // [R] its row of the output (padding rows: -1)
  float *refs = (float *)(Orow + R);                               // [round][R] its reference in a round, then what its probabilities weigh
  float *pml = refs + kRounds * R;                                 // [ns][R][2] gathered statistics
  __shared__ int s_ok, s_odd[kAttWaves];                           // [tile] some value of it is not finite
  constexpr float kNothing = -1e30f, kPadding = 1e30f;             // references: of a row that has seen no slot; of a padding row in the importance

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int rg = w % RG, st = w / RG;
  const int tq = a.tq, gq = a.gq;
  const float sm = a.sm_scale;
  const int t16 = lane & 15, g4 = lane >> 4;
  // queries as a matrix-core operand: lane (row t16, channels 32 g4 + 8 s + [0, 8)); padding rows repeat the last token's
  half8_t qa[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int row = (2 * rg + r) * 16 + t16, tok = row / gq, head = row - tok * gq;
    const __half *src = a.q + ((((size_t)blockIdx.z * tq + min(tok, tq - 1)) * cv.Hkv + kv_head_index(a)) * gq + head) * D + g4 * 32;
#pragma unroll
    for (int s = 0; s < 4; ++s) qa[r][s] = __builtin_bit_cast(half8_t, *(const confkv_v4i *)(src + 8 * s));
  }
  const Slice sl = make_slice(cv, a, ns, 0x7fffffff, &w_words);
  int seen[2];                                                     // the row of token t sees slots below n - tq + t + 1
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int tok = (rg * kWideRows + 16 * r + t16) / gq;
    seen[r] = tok < tq ? sl.n - tq + tok + 1 : 0x7fffffff;
  }
  const int first_new = sl.n - tq, see_all = first_new + 1;        // slots below see_all are seen by every row

  const int ntiles = (sl.cnt8 + kTile - 1) / kTile;
  int nitems = ntiles + (sl.hi16 - sl.lo16 + 15) / 16;
  if (nitems > kRounds * kAttWaves) {                              // cannot happen when the host plan is right
    if (tid == 0) atomicAdd(&cv.stats[kStatDeviceErr], 1ull);
    nitems = kRounds * kAttWaves;
  }
  const TileSource ts = tile_source<D, true>(cv, a, sl, cv.k8 + (size_t)sl.u * cv.cap8 * D, cv.v8 + (size_t)sl.u * cv.cap8 * D,
                                             cv.k16 + (size_t)sl.u * cv.cap16 * D, cv.v16 + (size_t)sl.u * cv.cap16 * D,
                                             cv.ks + (size_t)sl.u * cv.cap8, cv.vs + (size_t)sl.u * cv.cap8, ntiles, tq,
                                             a.observe_first >= 0 ? 0x3fffffff : first_new);
  TileRegs tr;
  auto load_item = [&](int it) { load_item_rows<D, true, false, true>(cv, ts, sl, lane, it, std::false_type{}, tr); };
  if (w < nitems) load_item(w);

  auto tile_at = [&](int j) { return tiles + (size_t)j * kWideTileBytes; };
  // slot of score i of half sb of an item, the end of its kind's slots, and whether some row must not see some slot
  auto slot_of = [&](int it, int sb, int i) {
    return it < ntiles ? sl.lo8 + it * kTile + 8 * i + 4 * sb + g4 : sl.lo16 + 16 * (it - ntiles) + 4 * i + g4;
  };
  auto end_of = [&](int it) { return it < ntiles ? sl.hi8 : sl.hi16; };
  auto is_edge = [&](int it) {
    return (it < ntiles ? sl.lo8 + it * kTile + kTile : sl.lo16 + 16 * (it - ntiles) + 16) > min(end_of(it), see_all);
  };
  // the four factors of a half of an item's slots
  auto factors = [&](int it, int sb) { return *(const floatx4_t *)&factor[it * kTile + 16 * sb + 4 * g4]; };

  floatx4_t S[kRounds][RG][2][2];                        // scores, then probabilities: [round][tile of the stream][block][half]
  floatx4_t O[2][RG];                                    // [block][channel group]: channels 16 (st RG + nt) + 4 g4 + [0, 4) of query t16
  float m[2], l[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    m[r] = kNothing;
    l[r] = 0.f;
#pragma unroll
    for (int nt = 0; nt < RG; ++nt) O[r][nt] = floatx4_t{0.f, 0.f, 0.f, 0.f};
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0): queries and first rows, so that no wait for them is in the rounds
#pragma unroll
  for (int sup = 0; sup < kRounds; ++sup) {
    const int it0 = sup * kAttWaves;
    if (it0 >= nitems) break;
    if (sup > 0) lds_barrier();                          // everybody has left the previous eight tiles
    if (it0 + w < nitems) {
      uint8_t *Kt = tile_at(w);
      float *sc = (float *)(Kt + kWideCoreBytes);
      store_wide_tile(Kt, factor + (it0 + w) * kTile, sc, it0 + w < ntiles, lane, sm, tr);
      s_odd[w] = odd_values(tr, it0 + w < ntiles, lane);
      if (it0 + w >= ntiles && lane < 16) {
        factor[(it0 + w) * kTile + lane] = sm;
        sc[lane] = 1.0f;
      }
    }
    if (it0 + kAttWaves + w < nitems) load_item(it0 + kAttWaves + w);
    lds_barrier();
    const int odd_tile = s_odd[lane & 7];
    // scores and the rows' maxima
    float top[2] = {kNothing, kNothing};
#pragma unroll
    for (int k = 0; k < RG; ++k) {
      const int j = st + k * NS, it = it0 + j;
      if (it >= nitems) continue;
      const uint8_t *krow = tile_at(j) + t16 * kKRow16 + g4 * 64;
#pragma unroll
      for (int r = 0; r < 2; ++r) S[sup][k][r][0] = S[sup][k][r][1] = floatx4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const half8_t kf = *(const half8_t *)(krow + 16 * s);
#pragma unroll
        for (int r = 0; r < 2; ++r) S[sup][k][r][0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qa[r][s], S[sup][k][r][0], 0, 0, 0);
      }
      if (it < ntiles) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const half8_t kf = *(const half8_t *)(krow + 16 * kKRow16 + 16 * s);
#pragma unroll
          for (int r = 0; r < 2; ++r) S[sup][k][r][1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qa[r][s], S[sup][k][r][1], 0, 0, 0);
        }
      }
      const int lim = end_of(it);
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        if (sb > 0 && it >= ntiles) break;
        const floatx4_t f = factors(it, sb);
        floatx4_t v[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) v[r] = S[sup][k][r][sb] * f;
        if (is_edge(it)) {
#pragma unroll
          for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (slot_of(it, sb, i) >= min(lim, seen[r])) v[r][i] = kNothing;
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) top[r] = fmaxf(fmaxf(fmaxf(top[r], v[r][0]), fmaxf(v[r][1], v[r][2])), v[r][3]);
      }
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      top[r] = column_max(top[r]);
      if (g4 == 0) stat_m[w * kWideRows + 16 * r + t16] = top[r];
    }
    lds_barrier();                                       // the maxima are there, the keys have been used
    float mn[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      mn[r] = m[r];
#pragma unroll
      for (int s = 0; s < NS; ++s) mn[r] = fmaxf(mn[r], stat_m[s * R + rg * kWideRows + 16 * r + t16]);
      const float corr = __expf(m[r] - mn[r]);
      m[r] = mn[r];
      if (st == 0 && g4 == 0) refs[sup * R + rg * kWideRows + 16 * r + t16] = mn[r];
      l[r] *= corr;
#pragma unroll
      for (int nt = 0; nt < RG; ++nt) O[r][nt] *= corr;
    }
    // probabilities times value scales over the tile's keys as fp16 head and tail, [head, tail][row group][block][lane].  (Rounded to
    // fp16 alone, only the largest of a row is exact, where a reference of its own for every stream has one exact in each: outputs of
    // 16 tokens of 4 heads on 500 slots 2.69e-4 from float64, against 2.48e-4 in the other kernel.)
#pragma unroll
    for (int k = 0; k < RG; ++k) {
      const int j = st + k * NS, it = it0 + j;
      if (it >= nitems) continue;
      const float *sc = (const float *)(tile_at(j) + kWideCoreBytes);
      const int lim = end_of(it);
      half8_t p[2] = {}, tail[2] = {};
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        if (sb > 0 && it >= ntiles) break;
        const floatx4_t f = factors(it, sb), vs = *(const floatx4_t *)(sc + 16 * sb + 4 * g4);
        floatx4_t x[2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
          for (int i = 0; i < 4; ++i) x[r][i] = fmaf(S[sup][k][r][sb][i], f[i], -mn[r]);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          floatx4_t e;
#pragma unroll
          for (int i = 0; i < 4; ++i) e[i] = exp_nonpos_or_nan(x[r][i]);
          if (is_edge(it)) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (slot_of(it, sb, i) >= min(lim, seen[r])) e[i] = 0.f;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = e[i] * vs[i];
            p[r][4 * sb + i] = (_Float16)v;
            tail[r][4 * sb + i] = (_Float16)(v - (float)p[r][4 * sb + i]);
          }
          l[r] += (e[0] + e[1]) + (e[2] + e[3]);
          S[sup][k][r][sb] = e;
        }
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        *(half8_t *)(tile_at(j) + (2 * rg + r) * 1024 + lane * 16) = p[r];
        *(half8_t *)(tile_at(j) + (2 * (RG + rg) + r) * 1024 + lane * 16) = tail[r];
      }
    }
    lds_barrier();
    // the wavefront's channels of all tiles.  Beside a value that is infinite the heads alone: the tails, of any sign and 0 among them,
    // have no sum with it, and the heads' is what the other kernels return.
    const unsigned odd = (unsigned)__builtin_amdgcn_ballot_w64(odd_tile != 0) & 0xffu;   // (bits past the last tile are not looked at)
    auto contract = [&](int j, bool is8, bool tails) {
      const uint8_t *Kt = tile_at(j), *Vt = Kt + kWideKBytes + st * RG * kWideVGroup + t16 * 64;
      static_assert(4 * RG * 1024 <= kWideKBytes, "probabilities fit the tile's keys");
      half8_t p[2], tail[2];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        p[r] = *(const half8_t *)(Kt + (2 * rg + r) * 1024 + lane * 16);
        tail[r] = *(const half8_t *)(Kt + (2 * (RG + rg) + r) * 1024 + lane * 16);
      }
#pragma unroll
      for (int nt = 0; nt < RG; ++nt) {
        if (is8) {
          const half8_t vf = *(const half8_t *)(Vt + nt * kWideVGroup + ((g4 ^ (t16 >> 2)) * 16));
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            if (tails) O[r][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf, tail[r], O[r][nt], 0, 0, 0);
            O[r][nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf, p[r], O[r][nt], 0, 0, 0);
          }
        } else {
          const half4_t vf = *(const half4_t *)(Vt + nt * kWideVGroup + g4 * 8);
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            if (tails) O[r][nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf, half4_t{tail[r][0], tail[r][1], tail[r][2], tail[r][3]}, O[r][nt], 0, 0, 0);
            O[r][nt] = __builtin_amdgcn_mfma_f32_16x16x16f16(vf, half4_t{p[r][0], p[r][1], p[r][2], p[r][3]}, O[r][nt], 0, 0, 0);
          }
        }
      }
    };
    if (!a.out) continue;
    if (it0 + kAttWaves <= ntiles && odd == 0u) {
#pragma unroll
      for (int j = 0; j < kAttWaves; ++j) contract(j, true, true);
    } else {
#pragma unroll 1
      for (int j = 0; j < kAttWaves && it0 + j < nitems; ++j) {
        if (odd >> j & 1u) contract(j, it0 + j < ntiles, false);
        else if (it0 + j < ntiles) contract(j, true, true);
        else contract(j, false, true);
      }
    }
  }

  // ---------------- the split's statistics and output ----------------
  append_new_token<D>(cv, a, sl, ns, tq);                // (nobody reads the appended rows back in this launch)
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    l[r] += __shfl_xor(l[r], 16, kWave);
    l[r] += __shfl_xor(l[r], 32, kWave);
    if (g4 == 0) stat_l[w * kWideRows + 16 * r + t16] = l[r];
  }
  lds_barrier();                                         // the tile buffers are free, and the last round's maxima have been read
#pragma unroll
  for (int r = 0; r < 2; ++r)
    if (st == 0 && g4 == 0) stat_m[w * kWideRows + 16 * r + t16] = m[r];   // (the streams agree)
  if (tid == 0) s_ok = 1;
  float *part = (float *)tiles;                          // [R][kRowsPartRow]
  if (a.out) {
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int nt = 0; nt < RG; ++nt)
        *(floatx4_t *)&part[(rg * kWideRows + 16 * r + t16) * kRowsPartRow + 16 * (st * RG + nt) + 4 * g4] = O[r][nt];
  }
  lds_barrier();
  const size_t row0 = ((size_t)sl.ul * a.max_splits + sl.j) * R;      // this split's first row in the exchange arrays
  const unsigned tag = tag_of(a);
  if (tid < R) {
    const float M = stat_m[tid];
    float L = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) L += stat_l[s * R + tid];
    const int tok = tid / gq;
    Orow[tid] = tok < tq ? ((sl.b * tq + tok) * cv.Hkv + sl.g) * gq + tid - tok * gq : -1;
    if (ns > 1) {
      st_tagged(&a.part_ml[(row0 + tid) * 2], tag, M);
      st_tagged(&a.part_ml[(row0 + tid) * 2 + 1], tag, L);
    } else {
      const double inv = recip_pos((double)L);
      Mrow[tid] = tok < tq ? M : kPadding;
      Irow[tid] = (float)inv;
      Frow[tid] = tok < tq ? inv * pow_count((double)a.ema_decay, (unsigned)(tq - 1 - tok)) : 0.0;
    }
  }
  float *EMA = cv.ema + (size_t)sl.u * cv.cap;
  // which of a lane's eight scores its row sums up, and its slot's row of the plane
  const int sb_e = t16 >> 3, i_e = (t16 >> 1) & 3;
  auto finishes = [&](int it) { return (t16 & 1) == 0 && (it < ntiles || sb_e == 0) && slot_of(it, sb_e, i_e) < end_of(it); };
  auto row_of = [&](int it) { return slot_row(cv, sl.tab, sl.h8, sl.n8, sl.h16, min(slot_of(it, sb_e, i_e), end_of(it) - 1)); };
  float old[kRounds][RG];
  auto request_old = [&]() {
#pragma unroll
    for (int sup = 0; sup < kRounds; ++sup)
#pragma unroll
      for (int k = 0; k < RG; ++k) {
        const int it = sup * kAttWaves + st + k * NS;
        old[sup][k] = 0.f;
        if (rg == 0 && it < nitems) old[sup][k] = EMA[row_of(it)];
      }
  };
  // what a row's probabilities of a round weigh: its weight times e^(the round's reference less the unit's maximum)
  auto weigh_rounds = [&]() {
    for (int k = tid; k < kRounds * R; k += kAttThreads) {
      const int row = k % R;
      if (k / R * kAttWaves < nitems) refs[k] = (float)(exp((double)refs[k] - (double)Mrow[row]) * Frow[row]);
    }
  };
  // split j finishes the rows [j R / ns, (j + 1) R / ns) and publishes the others, consecutive lanes on consecutive words
  const int own0 = sl.j * (R / ns), own1 = own0 + R / ns, ch = tid & (D - 1);
  if (ns == 1) {
    request_old();
    lds_barrier();
    weigh_rounds();
    if (a.out) {
      const int c4 = 4 * (tid & 31);
#pragma unroll
      for (int k = 0; k < R / 16; ++k) {
        const int row = 16 * k + (tid >> 5), to = Orow[row];
        const floatx4_t o = *(const floatx4_t *)&part[row * kRowsPartRow + c4];
        const half4_t h = {(_Float16)(o[0] * Irow[row]), (_Float16)(o[1] * Irow[row]), (_Float16)(o[2] * Irow[row]), (_Float16)(o[3] * Irow[row])};
        if (to >= 0) *(half4_t *)(a.out + (size_t)to * D + c4) = h;
      }
    }
  } else {
    if (a.out) {
#pragma unroll 4
      for (int k = 0; k < R / (kAttThreads / D); ++k) {
        const int row = w / (D / kWave) + k * (kAttThreads / D);
        if (row < own0 || row >= own1) st_tagged(&a.part_o[(row0 + row) * D + ch], tag, part[row * kRowsPartRow + ch]);
      }
    }
    gather_statistics(a, sl, ns, R, tag, tid, pml, &s_ok);
    request_old();                                       // (behind the polls, which would wait for it)
    lds_barrier();
    if (s_ok == 0) {
      if (tid == 0) atomicAdd(&cv.stats[kStatDeviceErr], 1ull);
      return;
    }
    if (tid < R) finish_statistics(a, ns, R, tid, gq, tq, kPadding, pml, Mrow, Irow, Frow);
    lds_barrier();
    weigh_rounds();
    if (a.out) gather_output(cv, a, sl, ns, R, tag, tid, own0, own1, pml, Orow, Irow, [&](int row) { return part[row * kRowsPartRow + ch]; });
  }

  // ---------------- exact mass per slot from the kept probabilities, EMA ----------------
  lds_barrier();
  const double lam = pow_count((double)a.ema_decay, (unsigned)tq);
  double *shared_sum = (double *)(tiles + 4 * kWideTileBytes);   // [tile][32] sums over the second row group
  static_assert(RG <= 2 && R * kRowsPartRow * 4 <= 4 * kWideTileBytes && kRounds * kAttWaves * 32 * 8 <= 4 * kWideTileBytes, "behind the split's output");
  double mass[kRounds][RG];
#pragma unroll
  for (int sup = 0; sup < kRounds; ++sup) {
    float F[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) F[r] = refs[sup * R + rg * kWideRows + 16 * r + t16];
#pragma unroll
    for (int k = 0; k < RG; ++k) {
      const int it = sup * kAttWaves + st + k * NS;
      if (it >= nitems) continue;
      float v[8] = {};
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        if (sb > 0 && it >= ntiles) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * sb + i] = fmaf(S[sup][k][1][sb][i], F[1], S[sup][k][0][sb][i] * F[0]);
      }
      mass[sup][k] = row16_scatter_sum(v, t16);
      if (RG > 1 && rg > 0 && (t16 & 1) == 0) shared_sum[it * 32 + (lane >> 1)] = mass[sup][k];
    }
  }
  if (RG > 1) {
    lds_barrier();
    if (rg > 0) return;
  }
#pragma unroll
  for (int sup = 0; sup < kRounds; ++sup)
#pragma unroll
    for (int k = 0; k < RG; ++k) {
      const int it = sup * kAttWaves + st + k * NS;
      if (it >= nitems || !finishes(it)) continue;
      const double A = RG > 1 ? mass[sup][k] + shared_sum[it * 32 + (lane >> 1)] : mass[sup][k];
      EMA[row_of(it)] = (float)(lam * (slot_of(it, sb_e, i_e) >= first_new ? 0.0 : (double)old[sup][k]) + a.mass_gain * A);
    }
}
