// Prompt-phase importance (conf_kv_observe_prompt): every prompt query attends causally to the
// stored prompt and adds its mass to the slots it sees.  Included by attend.hip, inside namespace
// confkv, after the helpers of the attention kernels.
//
// As consecutive observation windows a prompt of 3001 tokens was 94 launches of 64 workgroups that
// each re-read the whole cache: 4.1 ms per layer.  But the stored cache does not change while its
// prompt observes it, and the windows' updates telescope to
//   a_i = gain * sum_{t >= i} lambda^(T-1-t) sum_h p_{t,h,i},
// so two launches over all queries do: the first finds every row's softmax statistics, the second
// every slot's weighted column sum.  Both recompute the scores on the matrix cores (nothing of
// size T x T is stored).  A layer of that prompt with 32 query heads: 4060 -> 239 us (121 + 118).
#pragma once

constexpr int kObsThreads = 256, kObsWaves = kObsThreads / kWave;
constexpr int kMassThreads = 512, kMassWaves = kMassThreads / kWave, kMassTile = 64;   // slots per workgroup of the second
constexpr int kObsTileBytes = kTile * kKRow16;         // 32 slots as fp16 rows

// Softmax statistics of a prompt query: 1 / (sum of the exponentials) in 64 bits, then for all
// rows the reference the exponentials are taken against; both [unit in layer][head of the
// group][token, padded to 16].
__host__ __device__ constexpr int observe_stride(int T) { return (T + 15) / 16 * 16; }
struct ObserveStats {
  double *inv;
  float *ref;
};
size_t observe_scratch_floats(int units_per_layer, int G, int cap) {
  return (size_t)units_per_layer * G * observe_stride(cap) * 3;
}

// Causal work falls along the list of work items, so a workgroup takes two, one from either end:
// item y and item n - 1 - y (the middle one of an odd list alone).
// Both grids are (kv-heads times items, 1, sequences), kv-head fastest: the y dimension ends at
// 65536, which the row statistics of half a million tokens with 16 heads pass.

// The slots of a unit in tiles of 32: first the INT8 ones, then the FP16 ones.
struct ObserveUnit {
  const int8_t *K8;
  const __half *KS, *K16;
  int n8, h8, h16, cap8, cap16;
};
__device__ __forceinline__ ObserveUnit observe_unit(const CacheView &cv, int u, int T) {
  ObserveUnit s;
  s.K8 = cv.k8 + (size_t)u * cv.cap8 * 128;
  s.K16 = cv.k16 + (size_t)u * cv.cap16 * 128;
  s.KS = cv.ks + (size_t)u * (cv.chan ? 128 : cv.cap8);
  s.n8 = min(cv.n8[u], T);
  s.h8 = cv.head8[u];
  s.h16 = cv.head16[u];
  s.cap8 = cv.cap8;
  s.cap16 = cv.cap16;
  return s;
}

// Eight codes with their channels' scales as fp16 head + tail: the product has 19 significant
// bits and its last one is at least 2^-24, so the pair is exact.  (A channel that reaches 65504 has
// the scale 516, and 127 * 516 rounds to infinity: the head stops at 65504, the tail holds the rest.)
__device__ __forceinline__ void scale_codes(const uint2 &raw, const __half *scales, half8_t &hi, half8_t &lo) {
  const half8_t c = cvt_i8x8_f16x8(raw.x, raw.y);
  const half8_t s = __builtin_bit_cast(half8_t, *(const int4 *)scales);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float v = (float)c[e] * (float)s[e];
    const _Float16 h = (_Float16)fminf(fmaxf(v, -65504.0f), 65504.0f);
    hi[e] = h;
    lo[e] = (_Float16)(v - (float)h);
  }
}

// Row statistics.  Items are groups of four blocks of rows: a wavefront owns a block, 16 consecutive
// tokens of one head, and the workgroup walks the slots its last token sees in tiles of 32, staged
// once for its four blocks as fp16 in two alternating LDS buffers (one barrier per tile).  Every
// lane keeps a running reference and sum of its own columns, so no reduction runs inside the loop;
// the sum goes over to 64 bits every eight tiles.  A score costs a multiply-add, a product with
// log2 e, one hardware exponential and one addition.  (log2 e folded into the slots' factors would
// save the product, but rounds the factor once more: an error of the score, and so of a
// probability, that grows with it.)
template <bool kChan>
__global__ __launch_bounds__(kObsThreads) void observe_stats_kernel(CacheView cv, int layer, const __half *__restrict__ q,
                                                                    int T, float sm, ObserveStats stats) {
  constexpr int D = 128, kBuf = kObsTileBytes * (kChan ? 2 : 1);
  __shared__ __align__(16) uint8_t tiles[2][kBuf];
  __shared__ float factor[2][kTile];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int t16 = lane & 15, g4 = lane >> 4;
  const int g = blockIdx.x % cv.Hkv, y = blockIdx.x / cv.Hkv, b = blockIdx.z, G = cv.G;
  const int ul = b * cv.Hkv + g;
  const ObserveUnit un = observe_unit(cv, layer * cv.B * cv.Hkv + ul, T);
  constexpr float kNothing = -1e30f;                    // reference of a lane that has seen no slot

  const int nblocks = (T + 15) / 16 * G, nitems = (nblocks + kObsWaves - 1) / kObsWaves;   // blocks are (token block, head)
  for (int end = 0; end < 2; ++end) {
    const int item = end == 0 ? nitems - 1 - y : y;
    if (end == 1) {
      if (item == nitems - 1 - item) break;
      __syncthreads();                                  // the tile buffers are free
    }
    const int last_block = min((item + 1) * kObsWaves, nblocks) - 1;
    const int slots = min(T, last_block / G * 16 + 16);                // what the workgroup's last token sees
    const int nt8 = (min(un.n8, slots) + kTile - 1) / kTile;
    const int ntiles = nt8 + (max(0, slots - un.n8) + kTile - 1) / kTile;

    const int block = item * kObsWaves + w;
    const bool live = block < nblocks;
    const int tok0 = (live ? block : 0) / G * 16, head = (live ? block : 0) % G;
    half8_t qa[4];
    {
      const __half *row = q + (((size_t)b * T + min(tok0 + t16, T - 1)) * cv.Hkv * G + (size_t)g * G + head) * D + g4 * 8;
#pragma unroll
      for (int s = 0; s < 4; ++s) qa[s] = __builtin_bit_cast(half8_t, *(const int4 *)(row + 32 * s));
    }

    // thread (row, piece): sixteen channels of one slot
    const int lrow = tid >> 3, lc = tid & 7;
    int4 r0 = {}, r1 = {};
    unsigned short rs = 0;
    auto load = [&](int it) {
      if (it < nt8) {
        const unsigned row = (unsigned)ring_row_u(un.h8, min(it * kTile + lrow, un.n8 - 1), un.cap8);
        r0 = *(const int4 *)(un.K8 + (size_t)row * D + lc * 16);
        if (!kChan) rs = ((const unsigned short *)un.KS)[row];
      } else {
        const int slot = min(un.n8 + (it - nt8) * kTile + lrow, T - 1);
        const int4 *src = (const int4 *)(un.K16 + (size_t)ring_row(un.h16, slot - un.n8, un.cap16) * D + lc * 16);
        r0 = src[0];
        r1 = src[1];
      }
    };
    auto store = [&](int it) {
      half8_t *dst = (half8_t *)(tiles[it & 1] + lrow * kKRow16 + lc * 32);
      half8_t *low = (half8_t *)(tiles[it & 1] + (kChan ? kObsTileBytes : 0) + lrow * kKRow16 + lc * 32);
      if (it < nt8) {
        if constexpr (kChan) {
          scale_codes(make_uint2((unsigned)r0.x, (unsigned)r0.y), un.KS + lc * 16, dst[0], low[0]);
          scale_codes(make_uint2((unsigned)r0.z, (unsigned)r0.w), un.KS + lc * 16 + 8, dst[1], low[1]);
        } else {
          dst[0] = cvt_i8x8_f16x8((unsigned)r0.x, (unsigned)r0.y);
          dst[1] = cvt_i8x8_f16x8((unsigned)r0.z, (unsigned)r0.w);
        }
        if (lc == 0) factor[it & 1][lrow] = kChan ? sm : __half2float(__ushort_as_half(rs)) * sm;
      } else {
        dst[0] = __builtin_bit_cast(half8_t, r0);
        dst[1] = __builtin_bit_cast(half8_t, r1);
        if (lc == 0) factor[it & 1][lrow] = sm;
      }
    };

    float m[4], l[4];
    double ld[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) { m[i] = kNothing; l[i] = 0.f; ld[i] = 0.0; }

    load(0);
    store(0);
    if (ntiles > 1) load(1);
    for (int it = 0; it < ntiles; ++it) {
      __syncthreads();                                  // tile `it` is there; the buffer of tile it - 1 is free
      const bool is8 = it < nt8;
      const int base = is8 ? it * kTile : un.n8 + (it - nt8) * kTile, lim = is8 ? un.n8 : T;
      const uint8_t *Kt = tiles[it & 1];
      floatx4_t acc[2];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        acc[sb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        const uint8_t *krow = Kt + (16 * sb + t16) * kKRow16 + g4 * 16;
        if (kChan && is8) {
#pragma unroll
          for (int s = 0; s < 4; ++s)
            acc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], *(const half8_t *)(krow + kObsTileBytes + 64 * s), acc[sb], 0, 0, 0);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
          acc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], *(const half8_t *)(krow + 64 * s), acc[sb], 0, 0, 0);
      }
      const float f[2] = {factor[it & 1][t16], factor[it & 1][16 + t16]};
      // edge: the diagonal, or a partial tile; a masked score is -inf
      auto fold = [&](auto edge) {
        // the score less a reference, in one rounding here and in the second kernel: what a dominating
        // slot's score loses must be the same in its probability and in the normaliser
        auto above = [&](int sb, int i, float ref) {
          const float v = fmaf(acc[sb][i], f[sb], -ref);
          return edge && base + 16 * sb + t16 >= min(lim, tok0 + 4 * g4 + i + 1) ? -INFINITY : v;
        };
        float x[2][4], top = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
          for (int sb = 0; sb < 2; ++sb) x[sb][i] = above(sb, i, m[i]);
          top = fmaxf(top, fmaxf(x[0][i], x[1][i]));
        }
        // a lane's reference only has to stay within a few units of its columns' maximum
        if (__builtin_amdgcn_ballot_w64(top > 5.0f)) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float mn = fmaxf(m[i], fmaxf(above(0, i, 0.f), above(1, i, 0.f)));
            const float corr = __expf(m[i] - mn);
            m[i] = mn;
            l[i] *= corr;
            ld[i] *= (double)corr;
#pragma unroll
            for (int sb = 0; sb < 2; ++sb) x[sb][i] = above(sb, i, mn);
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) l[i] += __expf(x[0][i]) + __expf(x[1][i]);
      };
      if (live && base <= tok0 + 15) {                  // (uniform over the wavefront) a row of the block sees the tile
        if (base + kTile - 1 > tok0 || base + kTile > lim) fold(std::true_type{});
        else fold(std::false_type{});
      }
      if ((it & 7) == 7) {
#pragma unroll
        for (int i = 0; i < 4; ++i) { ld[i] += (double)l[i]; l[i] = 0.f; }
      }
      if (it + 1 < ntiles) store(it + 1);
      if (it + 2 < ntiles) load(it + 2);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float M = row16_max(m[i]);
      const float es = exp_nonpos(m[i] - M);
      const double L = group_sum((ld[i] + (double)l[i]) * (double)es, 16);
      const int tok = tok0 + 4 * g4 + i;
      if (live && t16 == 0 && tok < T) {
        const size_t row = ((size_t)ul * G + head) * observe_stride(T) + tok;
        stats.ref[row] = M;
        stats.inv[row] = recip_pos(L);
      }
    }
  }
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

// Column sums.  Items are tiles of slots: a workgroup keeps its 64 slots' keys in registers, so that
// every query read serves 64 slots (32 took 1.6 times as long; 64: 118 us per layer of 3001
// tokens); its wavefronts take every eighth block of 16 tokens from the prompt's end back to the
// tile, all heads of a block in turn (the queries of the unit stay in its XCD's L2: with eight
// kv-heads one XCD serves one of them).  A token's weight gain * lambda^(T-1-t) is a running product
// in 64 bits; every probability goes into the column sum in 64 bits by itself.
template <bool kChan>
__global__ __launch_bounds__(kMassThreads) void observe_mass_kernel(CacheView cv, int layer, const __half *__restrict__ q, int T,
                                                                   float sm, double decay, double gain,
                                                                   ObserveStats stats) {
  constexpr int D = 128, kSb = kMassTile / 16;
  __shared__ double red[kMassWaves][kMassTile];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int t16 = lane & 15, g4 = lane >> 4;
  const int g = blockIdx.x % cv.Hkv, tile = blockIdx.x / cv.Hkv, b = blockIdx.z, G = cv.G;
  const int ul = b * cv.Hkv + g, u = layer * cv.B * cv.Hkv + ul;
  const ObserveUnit un = observe_unit(cv, u, T);
  const int ntiles8 = (un.n8 + kMassTile - 1) / kMassTile;
  const bool is8 = tile < ntiles8;
  const int base = is8 ? tile * kMassTile : un.n8 + (tile - ntiles8) * kMassTile, lim = is8 ? un.n8 : T;
  if (base >= lim) return;                              // (the grid is sized for the worst rounding)

  half8_t kb[kSb][4], kl[kChan ? kSb : 1][4];
  float f[kSb];
#pragma unroll
  for (int sb = 0; sb < kSb; ++sb) {
    const int slot = min(base + 16 * sb + t16, lim - 1);
    if (is8) {
      const unsigned row = (unsigned)ring_row_u(un.h8, slot, un.cap8);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint2 c = *(const uint2 *)(un.K8 + (size_t)row * D + s * 32 + g4 * 8);
        if constexpr (kChan) scale_codes(c, un.KS + s * 32 + g4 * 8, kb[sb][s], kl[sb][s]);
        else kb[sb][s] = cvt_i8x8_f16x8(c.x, c.y);
      }
      f[sb] = kChan ? sm : __half2float(un.KS[row]) * sm;
    } else {
      const __half *src = un.K16 + (size_t)ring_row(un.h16, slot - un.n8, un.cap16) * D + g4 * 8;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        kb[sb][s] = __builtin_bit_cast(half8_t, *(const int4 *)(src + 32 * s));
        if constexpr (kChan) kl[sb][s] = half8_t{};
      }
      f[sb] = sm;
    }
  }

  const int ntb = (T + 15) / 16, tb_first = base / 16, stride = observe_stride(T);
  double wt[4], sum[kSb] = {};
  const double step = pow_count(decay, 16 * kMassWaves);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int tok = (ntb - 1 - w) * 16 + 4 * g4 + i;
    wt[i] = tok < T && tok >= 0 ? gain * pow_count(decay, (unsigned)(T - 1 - tok)) : 0.0;
  }
  half8_t qa[4];
  float4 ref = {};
  double2 inv0 = {}, inv1 = {};
  const int row_step = cv.Hkv * G * D;                  // elements from a token's queries to the next token's
  const __half *q_lane = q + ((size_t)b * T * cv.Hkv + g) * G * D + g4 * 8;
  const size_t s_lane = (size_t)ul * G * stride + 4 * g4;
  // queries and statistics of (token block, head), requested one step ahead
  auto load = [&](int tb, int h) {
    const __half *row = q_lane + (size_t)min(tb * 16 + t16, T - 1) * row_step + h * D;
#pragma unroll
    for (int s = 0; s < 4; ++s) qa[s] = __builtin_bit_cast(half8_t, *(const int4 *)(row + 32 * s));
    const size_t at = s_lane + (size_t)h * stride + tb * 16;
    ref = *(const float4 *)(stats.ref + at);
    inv0 = *(const double2 *)(stats.inv + at);
    inv1 = *(const double2 *)(stats.inv + at + 2);
  };
  int tb = ntb - 1 - w;
  if (tb >= tb_first) load(tb, 0);
  for (bool first = true; tb >= tb_first; tb -= kMassWaves, first = false) {
    if (!first) {
      // (the first block may have held tokens past the end, whose weight is 0: start those over)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int tok = tb * 16 + 4 * g4 + i;
        wt[i] = tok + 16 * kMassWaves >= T ? gain * pow_count(decay, (unsigned)(T - 1 - tok)) : wt[i] * step;
      }
    }
    auto heads = [&](auto edge) {
      for (int h = 0; h < G; ++h) {
        floatx4_t acc[kSb];
#pragma unroll
        for (int sb = 0; sb < kSb; ++sb) {
          acc[sb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
          if constexpr (kChan) {
            if (is8) {
#pragma unroll
              for (int s = 0; s < 4; ++s) acc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], kl[sb][s], acc[sb], 0, 0, 0);
            }
          }
#pragma unroll
          for (int s = 0; s < 4; ++s) acc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], kb[sb][s], acc[sb], 0, 0, 0);
        }
        const float M[4] = {ref.x, ref.y, ref.z, ref.w};
        const double wi[4] = {wt[0] * inv0.x, wt[1] * inv0.y, wt[2] * inv1.x, wt[3] * inv1.y};
        if (h + 1 < G) load(tb, h + 1);
        else if (tb - kMassWaves >= tb_first) load(tb - kMassWaves, 0);
#pragma unroll
        for (int sb = 0; sb < kSb; ++sb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float e = exp_nonpos(fmaf(acc[sb][i], f[sb], -M[i]));   // (a reference may lie up to 5 below a score)
            const int tok = tb * 16 + 4 * g4 + i;
            // (rows past the end have no statistics)
            const double term = (double)e * wi[i];
            sum[sb] += edge && (tok >= T || base + 16 * sb + t16 > tok) ? 0.0 : term;
          }
      }
    };
    if (tb * 16 < base + kMassTile - 1 || tb == ntb - 1) heads(std::true_type{});
    else heads(std::false_type{});
  }
#pragma unroll
  for (int sb = 0; sb < kSb; ++sb) {
    sum[sb] += __shfl_xor(sum[sb], 16, kWave);
    sum[sb] += __shfl_xor(sum[sb], 32, kWave);
    if (g4 == 0) red[w][16 * sb + t16] = sum[sb];
  }
  __syncthreads();
  if (tid < kMassTile && base + tid < lim) {
    double A = 0.0;
#pragma unroll
    for (int k = 0; k < kMassWaves; ++k) A += red[k][tid];
    cv.ema[(size_t)u * cv.cap + slot_row(cv, cv.pt, un.h8, un.n8, un.h16, base + tid)] = (float)A;
  }
}

hipError_t launch_observe_prompt(const CacheView &cv, int layer, const __half *q, int T, float sm, double decay, double gain,
                                 float *scratch, hipStream_t stream) {
  if (cv.D != 128 || cv.page_lg || T < 1) return hipErrorInvalidValue;
  const int nblocks = (T + 15) / 16 * cv.G;
  const dim3 rows(cv.Hkv * (((nblocks + kObsWaves - 1) / kObsWaves + 1) / 2), 1, cv.B);
  const dim3 slots(cv.Hkv * ((T + kMassTile - 1) / kMassTile + 1), 1, cv.B);
  const size_t n_rows = (size_t)cv.B * cv.Hkv * cv.G * observe_stride(T);
  const ObserveStats stats = {(double *)scratch, scratch + 2 * n_rows};
  if (cv.chan) {
    hipLaunchKernelGGL(observe_stats_kernel<true>, rows, dim3(kObsThreads), 0, stream, cv, layer, q, T, sm, stats);
    hipLaunchKernelGGL(observe_mass_kernel<true>, slots, dim3(kMassThreads), 0, stream, cv, layer, q, T, sm, decay, gain, stats);
  } else {
    hipLaunchKernelGGL(observe_stats_kernel<false>, rows, dim3(kObsThreads), 0, stream, cv, layer, q, T, sm, stats);
    hipLaunchKernelGGL(observe_mass_kernel<false>, slots, dim3(kMassThreads), 0, stream, cv, layer, q, T, sm, decay, gain, stats);
  }
  return hipGetLastError();
}
