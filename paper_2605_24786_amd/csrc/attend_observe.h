// Prompt-phase importance (conf_kv_observe_prompt): every prompt query attends causally to the
// stored prompt and adds its mass to the slots it sees.  Included by attend.hip, inside namespace
// confkv, after the helpers of the attention kernels.
//
// As consecutive observation windows a prompt of 3001 tokens was 94 launches of 64 workgroups that
// each re-read the whole cache: 4.1 ms per layer.  But the stored cache does not change while its
// prompt observes it, and the windows' updates telescope to
//   a_i = gain * sum_{t >= i} lambda^(T-1-t) sum_h p_{t,h,i},
// so launches over all queries whose weight an fp32 sum can show (observe_first_block) do: the first finds every row's softmax statistics,
// the second every slot's weighted column sum, both in parts where one piece of work per rows or slots would leave the
// chip idle, which two small kernels join.  Both recompute the scores on the matrix cores (nothing of
// size T x T is stored).  A layer of that prompt with 32 query heads: 254 us in two launches of 16 rows per
// wavefront and of 64 slots per workgroup, 170 to 175 us in these four with all rows; with those that count
// 113, and 5 for the fifth launch, which looks at the other rows' queries (observe_odd_kernel).
#pragma once

constexpr int kObsThreads = 256, kObsWaves = kObsThreads / kWave;
constexpr int kObsItem = 2 * kObsWaves;                // blocks of 16 rows per workgroup of the first kernel: two per wavefront, or
constexpr int kObsShortItem = kObsWaves, kObsShort = 512;   // one, up to so many tokens
constexpr int kMassWave = 64, kMassTile = kObsWaves * kMassWave;   // slots per wavefront and workgroup of the second
constexpr int kMassSb = kMassWave / 16;
constexpr int kMassShortThreads = 512, kMassShortWaves = kMassShortThreads / kWave;   // of its form for short prompts
constexpr int kMassStep = 4;                           // blocks of 16 rows it stages at a time
constexpr int kMassPartsMax = 32, kMassGroups = 1536, kMassStart = 3, kMassSum = 5;

// Per prompt query (row): the reference its exponentials are taken against, and in 64 bits
// gain * lambda^(T-1-t) over the sum of the exponentials; both [unit in layer][head of the
// group][token, padded to 16] (padding: a reference no score reaches, weight 0).
__host__ __device__ constexpr int observe_stride(int T) { return (T + 15) / 16 * 16; }
struct ObserveStats {
  double *weight;
  float *ref;
  double *partial;                                     // [unit in layer][part][token, padded to 16] column sums
  double *row_sum;                                     // the first kernel's parts: [part][rows] sums of exponentials
  float *row_ref;                                      // and references
};
// Parts the slots that the first kernel's rows see are cut into (a small kernel joins them): the count whose workgroups -- one
// per item of blocks and part not wholly behind the diagonal -- take the least time.  In us: a tile 0.6 and 0.65 for
// every workgroup that shares the CU, three at most, the join 6.5 with its launch.  Measured over 77 runs of 20 to 3001 tokens,
// 1 to 16 heads and 1 to 256 units in 1 to 16 parts, the choice takes 1.012 times the best count's time at the mean and 1.14 at
// most.  (At least eight tiles a part, and no price for the join: 500 tokens, 1 head and 8 kv-heads in a part of eight tiles and one
// of one 20.1 us, in six parts 10.7; 64 units of 500 tokens, 2 heads 29.1, uncut 20.3.)  before: tiles ahead of the first row.
constexpr int kObsPartsMax = 16;
static int observe_row_parts(long long items, int before, int tiles, int most, bool chan, int cus) {
  const double scale = chan ? 0.55 : 1.0, work = 0.5 * items * (before + tiles + 1);
  double cost[kObsPartsMax + 1], best = INFINITY;
  most = std::max(1, std::min(most, kObsPartsMax));
  for (int n = 1; n <= most; ++n) {
    const int len = (tiles + n - 1) / n;
    const double groups = 0.5 * items * (before / len + n + 1), per_cu = groups / cus;
    cost[n] = scale * (per_cu <= 3.0 ? len * (0.6 + 0.65 * per_cu) : 0.77 * ((work + groups) / cus + 1.8 * len)) + (n > 1 ? 6.5 : 0.0);
    if ((tiles + len - 1) / len != n) cost[n] = INFINITY;
    best = std::min(best, cost[n]);
  }
  int n = 1;                                           // (the fewest within 3 %)
  while (cost[n] > 1.03 * best) ++n;
  return n;
}
// Parts the rows of the second kernel are cut into, by a cost that was fitted and does not describe the chip (768 workgroups
// are resident, 512 with per-channel scales; a workgroup alone on its CU takes 5 us to begin and 3 per step, the sum 5):
// groups -- the pairs of a slot tile and a part that are not wholly behind the diagonal -- in rounds of kMassGroups, each
// as long as a part's steps and kMassStart.  Measured over 40 shapes of 100 to 3001 tokens in up to twelve part counts of 1 to 32,
// the choice takes 1.02 times the best of those at the mean; 1.2 for 64 units of 3001 tokens, 4 heads (eight parts 515 us, the
// three that kMassGroups allows 630) and 256 of 500 tokens, 2 heads (79, uncut 67), 1.16 with per-channel scales (1000 tokens).
static int observe_mass_parts(int units_per_layer, int G, int T, int b0, int most) {
  const long long tiles = (T + kMassTile - 1) / kMassTile, nb = (T + 15) / 16 * G - b0, steps = (nb + kMassStep - 1) / kMassStep;
  long long best = 0;
  int parts = 1;
  for (int p = 1; p == 1 || (p <= most && 2 * p <= steps + 1); ++p) {
    const long long len = (steps + p - 1) / p;
    long long groups = 0;
    for (long long t = 0; t < tiles && groups <= 4 * kMassGroups; ++t)
      groups += p - std::min<long long>(p, std::max<long long>(0, t * (kMassTile / 16) * G - b0) / (len * kMassStep));
    groups *= units_per_layer;
    if (p > 1 && groups > 4 * kMassGroups) break;
    const long long cost = (groups + kMassGroups - 1) / kMassGroups * (len + kMassStart) + (p > 1 ? kMassSum : 0);
    if (p == 1 || cost < best) { best = cost; parts = p; }
  }
  return parts;
}
// The first block of rows that counts, 0 for most prompts: a row's weight falls with lambda^(T-1-t), and the rows before it add
// less than 2^-150 to any slot all together, half of the smallest number that fp32 holds, so the importance is the same to the
// bit without them (a tie within 2^-150 of a rounding apart).  1000 tokens of 4 heads at lambda = 0.9, 10 500 at 0.99, all at 1.  A layer of
// 3001 tokens, 32 query heads, 8 kv-heads: statistics 79 -> 48 us, columns 90 -> 56.
int observe_first_block(int G, int T, double decay, double gain) {
  if (!(decay < 1.0)) return 0;
  double reach = 1.0;                                   // rows (tokens) that count
  if (decay > 0.0 && gain > 0.0) reach = std::ceil((150.0 * M_LN2 + std::log(gain * G / (1.0 - decay))) / -std::log(decay));
  return reach < T ? (T - std::max(1, (int)reach)) / 16 * G : 0;
}
// The final statistics of `cap` tokens.  Parts take what the launch is given beyond those of its own tokens.
size_t observe_scratch_floats(int units_per_layer, int G, int cap) {
  return (size_t)units_per_layer * G * observe_stride(cap) * 3;
}
// What a launch over T tokens runs, with at most `have` floats of scratch: the rows' final statistics and behind them
// the parts of one kernel at a time (the first kernel's are done with before the second's are written).
// (A reservation for the most parts that any T could take was 0.1 to 1.6 GB larger than a launch could use on long caches.)
struct ObservePlan {
  int b0;                                              // the first block of rows that counts
  int item, tile, per_part, row_parts;                 // first kernel: blocks per workgroup, slots per tile, tiles per part, parts
  bool short_form;                                     // second: the kernel of short prompts, or
  int subtiles, width, parts;                          // subtiles of a unit, per workgroup, parts
  size_t n_rows, stat_floats, floats;
};
static ObservePlan observe_plan(int units_per_layer, int G, int T, int b0, int n8, bool chan, size_t have, int cus) {
  ObservePlan p;
  const int nblocks = (T + 15) / 16 * G - b0;
  p.b0 = b0;
  p.n_rows = (size_t)units_per_layer * G * observe_stride(T);
  p.stat_floats = 3 * p.n_rows;                         // (even: rows come in sixteens)
  const size_t room = have > p.stat_floats ? have - p.stat_floats : 0;
  p.tile = chan ? 32 : 64;
  // First kernel.  With one block per wavefront a tile takes 0.8 us instead of 1.2 and a half as long as the chip has room for
  // twice the workgroups: 100 tokens of 4 heads and 8 kv-heads 7.2 -> 5.5 us, 256 10.3 -> 7.8, 500 17 -> 13; 64 units of 150 tokens, 4 heads
  // (640 workgroups) 10.9 -> 8.8, but of 500 tokens, 2 heads (1024) 20.7 -> 22.8.  Parts and their join gain nothing on it.
  const int tiles = (n8 + p.tile - 1) / p.tile + (T - n8 + p.tile - 1) / p.tile;
  const bool one = T <= kObsShort && (long long)units_per_layer * ((nblocks + kObsShortItem - 1) / kObsShortItem) <= 2 * cus;
  p.item = one ? kObsShortItem : kObsItem;
  p.row_parts = one ? 1 : observe_row_parts((long long)units_per_layer * ((nblocks + kObsItem - 1) / kObsItem), b0 / G * 16 / p.tile, tiles,
                                            (int)std::min<size_t>(kObsPartsMax, room / (3 * p.n_rows)), chan, cus);
  p.per_part = (tiles + p.row_parts - 1) / p.row_parts;
  // Second kernel.  More than eight blocks per wavefront of the form for short prompts are cut into parts where parts find idle
  // CUs.  Otherwise that form, up to a round of workgroups, two of long ones (one of its workgroups fills a CU), and for short prompts
  // of many units a subtile per workgroup of the other form, whose wavefronts share the rows.  Measured (us, with the sum): 8 units of
  // 256 tokens, 8 heads 23.6 in the short form, 13.9 in 16 parts; 64 such units 24.5 and 44; 8 units of 300 tokens, 4 heads (76 blocks)
  // 17.4 and 17.6, 2 heads (38) 13.0 and 15.8; 128 units of 200 tokens, 4 heads (two rounds) 26.6, a subtile per workgroup 32.6, parts
  // 35.5; 256 units of 65 tokens, 4 heads 21.7 and 15.8, of 40 tokens, 1 head (a round, three blocks) 12.4 and 8.2.
  p.subtiles = (n8 + kMassWave - 1) / kMassWave + (T - n8 + kMassWave - 1) / kMassWave;
  const long long subtiles = (long long)units_per_layer * p.subtiles;
  const bool tile = T <= kMassTile, cut = nblocks > 8 * kMassShortWaves && (!tile || 2 * subtiles <= cus);
  const long long rounds2 = !tile || nblocks > 4 * kMassShortWaves ? 4 : nblocks > kMassShortWaves ? 2 : 1;   // half rounds
  p.short_form = !cut && 2 * subtiles <= rounds2 * cus;
  p.width = !p.short_form && !cut && tile ? 1 : kObsWaves;
  const size_t column = 2 * (size_t)units_per_layer * observe_stride(T);
  p.parts = p.short_form || p.width == 1 ? 1 : observe_mass_parts(units_per_layer, G, T, b0, (int)std::min<size_t>(kMassPartsMax, room / column));
  p.floats = p.stat_floats + std::max(p.row_parts > 1 ? 3 * p.row_parts * p.n_rows : 0, p.parts > 1 ? column * p.parts : 0);
  return p;
}
size_t observe_plan_floats(int units_per_layer, int G, int T, int b0, int n8, int chan, size_t have, int cus) {
  return observe_plan(units_per_layer, G, T, b0, n8, chan != 0, have, cus).floats;
}
static int device_cus();                                // (below, with the attention plans)

// The slots of a unit come in tiles: first the INT8 ones, then the FP16 ones.
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

__device__ __forceinline__ void finish_row(const ObserveStats &stats, size_t row, int tok, int T, float M, double L, double decay,
                                           double gain) {
  stats.ref[row] = tok < T ? M : 1e30f;
  stats.weight[row] = tok < T ? gain * pow_count(decay, (unsigned)(T - 1 - tok)) * recip_pos(L) : 0.0;
}

// Row statistics.  A block of rows is 16 consecutive tokens of one head; a wavefront owns two (one of short prompts), so
// that a key fragment read from LDS serves 32 rows (with 16 the reads alone took 47 of 120 us per
// layer of 3001 tokens and 32 heads, and the conversion of the keys five of fourteen vector
// instructions per score), and the workgroup walks the slots its last token sees in tiles that
// are staged once for its eight blocks as fp16 in two alternating LDS buffers (one barrier per tile).
// Scores come transposed, a lane's rows being slots of one query: one running reference and sum
// per lane and block, no reduction inside the loop; the sum goes over to 64 bits with every tile.
// 120 -> 79 us per layer of 3001 tokens and 32 heads with all rows, 48 with those that count; while a CU is busy, vector ALU and matrix
// cores are at work in turn 88 % of the time.
// Causal work falls along the list of items: long ones are cut into parts of their slots.
// A score costs a multiply-add, a product with log2 e, one hardware exponential and one addition.
// (log2 e folded into the slots' factors would save the product, but rounds the factor once more: an
// error of the score, and so of a probability, that grows with it.)
// The grid is (kv-heads times items, 1, sequences), kv-head fastest: the y dimension ends at 65536,
// which the row blocks of half a million tokens with 16 heads pass.
template <bool kChan, int kObsBlocks>
__global__ __launch_bounds__(kObsThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
void observe_stats_kernel(CacheView cv, int layer, const __half *__restrict__ q, int T,
                                                                    float sm, double decay, double gain, int b0, int per_part, ObserveStats stats) {
  constexpr int D = 128, TS = kChan ? 32 : 64, kItem = kObsWaves * kObsBlocks;   // slots per tile, blocks per workgroup
  constexpr int kTileB = TS * kKRow16, kBuf = kTileB * (kChan ? 2 : 1);
  __shared__ __align__(16) uint8_t tiles[2][kBuf];
  __shared__ __align__(16) float factor[2][TS];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t16 = lane & 15, g4 = lane >> 4;
  const int g = blockIdx.x % cv.Hkv, b = blockIdx.z, G = cv.G;
  const int ul = b * cv.Hkv + g;
  const ObserveUnit un = observe_unit(cv, layer * cv.B * cv.Hkv + ul, T);
  constexpr float kNothing = -1e30f;                    // reference of a lane that has seen no slot

  const int nblocks = (T + 15) / 16 * G, nitems = (nblocks - b0 + kItem - 1) / kItem;   // blocks are (token block, head)
  const int item = nitems - 1 - (int)(blockIdx.x / cv.Hkv) % nitems, part = (int)(blockIdx.x / cv.Hkv) / nitems;
  const int last_block = min(b0 + (item + 1) * kItem, nblocks) - 1;
  const int slots = min(T, last_block / G * 16 + 16);                // what the workgroup's last token sees
  const int nt8 = (min(un.n8, slots) + TS - 1) / TS;
  const int ntiles = nt8 + (max(0, slots - un.n8) + TS - 1) / TS;
  const int first = part * per_part, last = min(ntiles, first + per_part);   // this workgroup's tiles
  if (first >= last) return;

  int tok0[kObsBlocks], head[kObsBlocks];
  bool live[kObsBlocks];
  half8_t qa[kObsBlocks][4];
#pragma unroll
  for (int r = 0; r < kObsBlocks; ++r) {
    const int block = b0 + item * kItem + w * kObsBlocks + r;
    live[r] = block < nblocks;
    tok0[r] = (live[r] ? block : last_block) / G * 16;
    head[r] = (live[r] ? block : last_block) % G;
    const __half *row = q + (((size_t)b * T + min(tok0[r] + t16, T - 1)) * cv.Hkv * G + (size_t)g * G + head[r]) * D + g4 * 8;
#pragma unroll
    for (int s = 0; s < 4; ++s) qa[r][s] = __builtin_bit_cast(half8_t, *(const int4 *)(row + 32 * s));
  }
  const int see = __builtin_amdgcn_readfirstlane(tok0[kObsBlocks - 1] + 16);   // slots the wavefront's rows see at most
  const int all = __builtin_amdgcn_readfirstlane(tok0[0] + 1);                 // and what every row of it sees

  // thread (row, piece): sixteen channels of one slot out of every 32
  const int lrow = tid >> 3, lc = tid & 7;
  struct Piece {
    confkv_v4i a, b;                                    // sixteen codes (twice), or sixteen fp16 values
    unsigned short scale;
  };
  // (no branch around the loads: they would be waited for where its sides meet)
  auto load = [&](int it, int k) -> Piece {
    const bool is8 = it < nt8;
    const int i = is8 ? min(it * TS + 32 * k + lrow, un.n8 - 1) : min((it - nt8) * TS + 32 * k + lrow, T - 1 - un.n8);
    const unsigned row = is8 ? (unsigned)ring_row_u(un.h8, i, un.cap8) : (unsigned)ring_row(un.h16, i, un.cap16);
    const char *p = (is8 ? (const char *)un.K8 : (const char *)un.K16) + (size_t)row * (is8 ? D : 2 * D) + lc * (is8 ? 16 : 32);
    Piece r;
    r.a = *(const confkv_v4i *)p;
    r.b = *(const confkv_v4i *)(is8 ? p : p + 16);
    r.scale = *(is8 && !kChan ? (const unsigned short *)un.KS + row : (const unsigned short *)q);
    return r;
  };
  auto store = [&](int it, int k, const Piece &r) {
    uint8_t *at = tiles[it & 1] + (32 * k + lrow) * kKRow16 + lc * 32;
    half8_t *dst = (half8_t *)at, *low = (half8_t *)(at + (kChan ? kTileB : 0));
    if (it < nt8) {
      if constexpr (kChan) {
        scale_codes(make_uint2((unsigned)r.a[0], (unsigned)r.a[1]), un.KS + lc * 16, dst[0], low[0]);
        scale_codes(make_uint2((unsigned)r.a[2], (unsigned)r.a[3]), un.KS + lc * 16 + 8, dst[1], low[1]);
      } else {
        dst[0] = cvt_i8x8_f16x8((unsigned)r.a[0], (unsigned)r.a[1]);
        dst[1] = cvt_i8x8_f16x8((unsigned)r.a[2], (unsigned)r.a[3]);
      }
      if (lc == 0) factor[it & 1][32 * k + lrow] = kChan ? sm : __half2float(__ushort_as_half(r.scale)) * sm;
    } else {
      dst[0] = __builtin_bit_cast(half8_t, r.a);
      dst[1] = __builtin_bit_cast(half8_t, r.b);
      if (lc == 0) factor[it & 1][32 * k + lrow] = sm;
    }
  };

  float m[kObsBlocks], l[kObsBlocks];
  double ld[kObsBlocks];
#pragma unroll
  for (int r = 0; r < kObsBlocks; ++r) { m[r] = kNothing; l[r] = 0.f; ld[r] = 0.0; }

  Piece p0 = load(first, 0), p1 = TS > 32 ? load(first, 1) : p0;
  for (int it = first; it < last; ++it) {
    store(it, 0, p0);
    if (TS > 32) store(it, 1, p1);
    __syncthreads();                                    // tile `it` is there, and nobody reads tile it - 1 any more
    p0 = load(min(it + 1, last - 1), 0);
    if (TS > 32) p1 = load(min(it + 1, last - 1), 1);
    const bool is8 = it < nt8;
    const int tile0 = is8 ? it * TS : un.n8 + (it - nt8) * TS, lim = is8 ? un.n8 : T;
#pragma unroll 1
    for (int half = 0; half < TS / 32; ++half) {
      const int base = tile0 + 32 * half;
      if (base >= min(see, lim)) continue;              // (uniform over the wavefront) no row of it sees the slots
      floatx4_t acc[kObsBlocks][2];
#pragma unroll
      for (int sb = 0; sb < 2; ++sb) {
        const uint8_t *krow = tiles[it & 1] + (32 * half + 16 * sb + t16) * kKRow16 + g4 * 16;
#pragma unroll
        for (int r = 0; r < kObsBlocks; ++r) acc[r][sb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        if (kChan && is8) {
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const half8_t kf = *(const half8_t *)(krow + kTileB + 64 * s);
#pragma unroll
            for (int r = 0; r < kObsBlocks; ++r) acc[r][sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qa[r][s], acc[r][sb], 0, 0, 0);
          }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const half8_t kf = *(const half8_t *)(krow + 64 * s);
#pragma unroll
          for (int r = 0; r < kObsBlocks; ++r) acc[r][sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qa[r][s], acc[r][sb], 0, 0, 0);
        }
      }
      const float4 f4[2] = {*(const float4 *)&factor[it & 1][32 * half + 4 * g4], *(const float4 *)&factor[it & 1][32 * half + 16 + 4 * g4]};
      const float f[2][4] = {{f4[0].x, f4[0].y, f4[0].z, f4[0].w}, {f4[1].x, f4[1].y, f4[1].z, f4[1].w}};
      // edge: the diagonal, or a partial tile; a masked score is -inf
      auto fold = [&](auto edge) {
        // the score less a reference, in one rounding here and in the second kernel: what a dominating
        // slot's score loses must be the same in its probability and in the normaliser
        auto above = [&](int r, int sb, int i, float ref) {
          const float v = fmaf(acc[r][sb][i], f[sb][i], -ref);
          return edge && base + 16 * sb + 4 * g4 + i >= min(lim, tok0[r] + t16 + 1) ? -INFINITY : v;
        };
        float x[kObsBlocks][2][4], top[kObsBlocks];
#pragma unroll
        for (int r = 0; r < kObsBlocks; ++r) {
#pragma unroll
          for (int sb = 0; sb < 2; ++sb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              x[r][sb][i] = above(r, sb, i, m[r]);
              top[r] = sb + i == 0 ? x[r][sb][i] : fmaxf(top[r], x[r][sb][i]);
            }
        }
        auto sum = [&]() {
#pragma unroll
          for (int r = 0; r < kObsBlocks; ++r)
#pragma unroll
            for (int sb = 0; sb < 2; ++sb)
              l[r] += (__expf(x[r][sb][0]) + __expf(x[r][sb][1])) + (__expf(x[r][sb][2]) + __expf(x[r][sb][3]));
        };
        // a lane's reference only has to stay within a few units of its slots' maximum
        if (__builtin_amdgcn_ballot_w64(fmaxf(top[0], top[kObsBlocks - 1]) > 5.0f)) {
#pragma unroll
          for (int r = 0; r < kObsBlocks; ++r) {
            float mn = m[r];
#pragma unroll
            for (int sb = 0; sb < 2; ++sb)
#pragma unroll
              for (int i = 0; i < 4; ++i) mn = fmaxf(mn, above(r, sb, i, 0.f));
            const float corr = __expf(m[r] - mn);
            m[r] = mn;
            l[r] *= corr;
            ld[r] *= (double)corr;
#pragma unroll
            for (int sb = 0; sb < 2; ++sb)
#pragma unroll
              for (int i = 0; i < 4; ++i) x[r][sb][i] = above(r, sb, i, mn);
          }
          sum();
        } else {
          sum();                                        // (a copy of its own: joining the two would move every score)
        }
      };
      if (base + 32 > min(all, lim)) fold(std::true_type{});
      else fold(std::false_type{});
    }
#pragma unroll
    for (int r = 0; r < kObsBlocks; ++r) { ld[r] += (double)l[r]; l[r] = 0.f; }
  }
#pragma unroll
  for (int r = 0; r < kObsBlocks; ++r) {
    float M = fmaxf(m[r], __shfl_xor(m[r], 16, kWave));
    M = fmaxf(M, __shfl_xor(M, 32, kWave));
    double L = ld[r] * (double)exp_nonpos(m[r] - M);
    L += __shfl_xor(L, 16, kWave);
    L += __shfl_xor(L, 32, kWave);
    const int tok = tok0[r] + t16;
    if (live[r] && g4 == 0) {
      const size_t row = ((size_t)ul * G + head[r]) * observe_stride(T) + tok;
      if (stats.row_sum) {
        const size_t at = (size_t)part * cv.B * cv.Hkv * G * observe_stride(T) + row;
        stats.row_ref[at] = M;
        stats.row_sum[at] = L;
      } else {
        finish_row(stats, row, tok, T, M, L, decay, gain);
      }
    }
  }
}

// The parts of the rows joined, in order.  (TS: slots per tile of the kernel above.)
__global__ __launch_bounds__(kObsThreads) void observe_join_kernel(CacheView cv, int layer, int T, int TS, double decay, double gain,
                                                                   int b0, int per_part, ObserveStats stats) {
  const int stride = observe_stride(T), G = cv.G;
  const size_t n_rows = (size_t)cv.B * cv.Hkv * G * stride, row = (size_t)blockIdx.x * kObsThreads + threadIdx.x;
  if (row >= n_rows) return;
  const int tok = (int)(row % stride), uh = (int)(row / stride), ul = uh / G;
  const int block = tok / 16 * G + uh % G;
  if (block < b0) return;
  const int n8 = min(cv.n8[layer * cv.B * cv.Hkv + ul], T);
  const int nblocks = stride / 16 * G, item = (block - b0) / kObsItem;
  const int slots = min(T, (min(b0 + (item + 1) * kObsItem, nblocks) - 1) / G * 16 + 16);
  const int ntiles = (min(n8, slots) + TS - 1) / TS + (max(0, slots - n8) + TS - 1) / TS;
  float M = -1e30f;
  double L = 0.0;
  for (int p = 0; p * per_part < ntiles; ++p) {
    const float m = stats.row_ref[p * n_rows + row];
    const double l = stats.row_sum[p * n_rows + row];
    const float top = fmaxf(M, m);
    L = L * (double)exp_nonpos(M - top) + l * (double)exp_nonpos(m - top);
    M = top;
  }
  finish_row(stats, row, tok, T, M, L, decay, gain);
}

// Column sums.  A wavefront keeps 64 slots' keys in registers, its workgroup 256 slots'; the blocks of
// 16 rows -- (token block, head), from the first that sees one of the slots, or a part of them --
// come through LDS four at a time, staged once for the four wavefronts.  Each wavefront reading the
// queries for itself asked 622 MB of L2 per layer of 3001 tokens and 32 heads, 5.2 TB/s, and 384 workgroups of
// falling work ended late: 118 us, 90 with all rows and 56 with those that count, of which the vector ALU (ten instructions a score) works 70 %.
// Every probability goes into its column's sum in 64 bits by itself.
struct MassTile {
  int base, lim;                                       // slots [base, min(base + kMassWave, lim)) of subtile `at`
  bool is8;
};
__device__ __forceinline__ MassTile mass_subtile(const ObserveUnit &un, int at, int T) {
  const int nt8 = (un.n8 + kMassWave - 1) / kMassWave;
  MassTile t;
  t.is8 = at < nt8;
  t.base = t.is8 ? at * kMassWave : un.n8 + (at - nt8) * kMassWave;
  t.lim = t.is8 ? un.n8 : T;
  return t;
}
// Blocks per part, from block b0 on, and the first block that sees a slot of a subtile.
__device__ __forceinline__ int mass_part_blocks(int parts, int G, int T, int b0) {
  const int steps = ((T + 15) / 16 * G - b0 + kMassStep - 1) / kMassStep;
  return (steps + parts - 1) / parts * kMassStep;
}
__device__ __forceinline__ int mass_first_block(const ObserveUnit &un, int sub, int G, int T, int b0) {
  return max(b0, mass_subtile(un, sub, T).base / 16 * G);
}

// The keys of a subtile as a matrix-core operand, lane (slot t16 of each sixteen, channels 32 s + 8 g4 + [0, 8)), and the
// slots' factors.
template <bool kChan>
__device__ __forceinline__ void mass_keys(const ObserveUnit &un, const MassTile &mt, float sm, int t16, int g4, half8_t (&kb)[kMassSb][4],
                                          half8_t (&kl)[kChan ? kMassSb : 1][4], float (&f)[kMassSb]) {
#pragma unroll
  for (int sb = 0; sb < kMassSb; ++sb) {
    const int slot = min(mt.base + 16 * sb + t16, mt.lim - 1);
    if (mt.is8) {
      const unsigned row = (unsigned)ring_row_u(un.h8, slot, un.cap8);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint2 c = *(const uint2 *)(un.K8 + (size_t)row * 128 + s * 32 + g4 * 8);
        if constexpr (kChan) scale_codes(c, un.KS + s * 32 + g4 * 8, kb[sb][s], kl[sb][s]);
        else kb[sb][s] = cvt_i8x8_f16x8(c.x, c.y);
      }
      f[sb] = kChan ? sm : __half2float(un.KS[row]) * sm;
    } else {
      const __half *src = un.K16 + (size_t)(mt.base < mt.lim ? ring_row(un.h16, slot - un.n8, un.cap16) : 0) * 128 + g4 * 8;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        kb[sb][s] = __builtin_bit_cast(half8_t, *(const int4 *)(src + 32 * s));
        if constexpr (kChan) kl[sb][s] = half8_t{};
      }
      f[sb] = sm;
    }
  }
}
// What a block of sixteen rows (queries qa of tokens tok0 .., references and weights of rows 4 g4 + [0, 4)) adds to the
// subtile's columns.
template <bool kChan>
__device__ __forceinline__ void mass_block(const MassTile &mt, const half8_t (&qa)[4], const half8_t (&kb)[kMassSb][4],
                                           const half8_t (&kl)[kChan ? kMassSb : 1][4], const float (&f)[kMassSb], const float4 &ref,
                                           const double2 &w0, const double2 &w1, int tok0, int t16, int g4, double (&sum)[kMassSb]) {
  const float M[4] = {ref.x, ref.y, ref.z, ref.w};
  const double wi[4] = {w0.x, w0.y, w1.x, w1.y};
  floatx4_t acc[kMassSb];
#pragma unroll
  for (int sb = 0; sb < kMassSb; ++sb) {
    acc[sb] = floatx4_t{0.f, 0.f, 0.f, 0.f};
    if constexpr (kChan) {
      if (mt.is8) {
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], kl[sb][s], acc[sb], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int sb = 0; sb < kMassSb; ++sb) acc[sb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], kb[sb][s], acc[sb], 0, 0, 0);
  auto add = [&](auto edge) {
#pragma unroll
    for (int sb = 0; sb < kMassSb; ++sb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float e = exp_nonpos(fmaf(acc[sb][i], f[sb], -M[i]));   // (a reference may lie up to 5 below a score)
        const double term = (double)e * wi[i];
        sum[sb] += edge && mt.base + 16 * sb + t16 > tok0 + 4 * g4 + i ? 0.0 : term;
      }
  };
  if (tok0 < mt.base + kMassWave - 1) add(std::true_type{});
  else add(std::false_type{});
}

// Short prompts: a workgroup of eight wavefronts per 64 slots, its wavefronts taking the blocks of rows in turn, each reading
// its queries for itself, so that nobody waits for anybody before the sums meet.  In the kernel below the few steps of such
// a prompt are latency: 100 tokens of 4 heads and 8 kv-heads 18.7 us there (13.8 in four parts with their sum), 9.4 here.
template <bool kChan>
__global__ __launch_bounds__(kMassShortThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void observe_mass_short_kernel(CacheView cv, int layer, const __half *__restrict__ q, int T, float sm, int b0, ObserveStats stats) {
  constexpr int D = 128;
  __shared__ double red[kMassShortWaves][kMassWave];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t16 = lane & 15, g4 = lane >> 4;
  const int g = blockIdx.x % cv.Hkv, b = blockIdx.z, G = cv.G;
  const int ul = b * cv.Hkv + g, u = layer * cv.B * cv.Hkv + ul;
  const ObserveUnit un = observe_unit(cv, u, T);
  const MassTile mt = mass_subtile(un, blockIdx.x / cv.Hkv, T);
  if (mt.base >= mt.lim) return;
  const int first = max(b0, mt.base / 16 * G), last = (T + 15) / 16 * G, stride = observe_stride(T);
  struct Rows {
    confkv_v4i q[4];
    float4 ref;
    double2 w0, w1;
  };
  auto load = [&](int block) -> Rows {
    const int at = min(block, last - 1), tb = at / G, h = at - tb * G;
    const __half *src = q + (((size_t)b * T + min(tb * 16 + t16, T - 1)) * cv.Hkv * G + (size_t)g * G + h) * D + g4 * 8;
    const size_t row = ((size_t)ul * G + h) * stride + tb * 16 + 4 * g4;
    Rows r;
#pragma unroll
    for (int s = 0; s < 4; ++s) r.q[s] = *(const confkv_v4i *)(src + 32 * s);
    r.ref = *(const float4 *)&stats.ref[row];
    r.w0 = *(const double2 *)&stats.weight[row];
    r.w1 = *(const double2 *)&stats.weight[row + 2];
    return r;
  };
  Rows next = load(first + w);
  half8_t kb[kMassSb][4], kl[kChan ? kMassSb : 1][4];
  float f[kMassSb];
  mass_keys<kChan>(un, mt, sm, t16, g4, kb, kl, f);
  double sum[kMassSb] = {};
  for (int block = first + w; block < last; block += kMassShortWaves) {
    const Rows r = next;
    next = load(block + kMassShortWaves);
    half8_t qa[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) qa[s] = __builtin_bit_cast(half8_t, r.q[s]);
    mass_block<kChan>(mt, qa, kb, kl, f, r.ref, r.w0, r.w1, block / G * 16, t16, g4, sum);
  }
#pragma unroll
  for (int sb = 0; sb < kMassSb; ++sb) {
    sum[sb] += __shfl_xor(sum[sb], 16, kWave);
    sum[sb] += __shfl_xor(sum[sb], 32, kWave);
    if (g4 == 0) red[w][16 * sb + t16] = sum[sb];
  }
  __syncthreads();
  const int slot = mt.base + lane;
  if (w > 0 || slot >= mt.lim) return;
  double A = 0.0;
#pragma unroll
  for (int k = 0; k < kMassShortWaves; ++k) A += red[k][lane];
  cv.ema[(size_t)u * cv.cap + slot_row(cv, cv.pt, un.h8, un.n8, un.h16, slot)] = (float)A;
}

template <bool kChan>
__global__ __launch_bounds__(kObsThreads) __attribute__((amdgpu_waves_per_eu(kChan ? 2 : 3, kChan ? 2 : 3)))
void observe_mass_kernel(CacheView cv, int layer, const __half *__restrict__ q, int T, float sm, int ntiles, int width /* subtiles per workgroup */,
                         int b0, int parts, ObserveStats stats) {
  constexpr int D = 128, kSb = kMassSb, kRows = 16 * kMassStep;
  __shared__ __align__(16) uint8_t rows[2][kRows * kKRow16];
  __shared__ __align__(16) float s_ref[2][kRows];
  __shared__ __align__(16) double s_weight[2][kRows];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t16 = lane & 15, g4 = lane >> 4;
  const int g = blockIdx.x % cv.Hkv, y = blockIdx.x / cv.Hkv, tile = y % ntiles, part = y / ntiles, b = blockIdx.z, G = cv.G;
  const int ul = b * cv.Hkv + g, u = layer * cv.B * cv.Hkv + ul;
  const ObserveUnit un = observe_unit(cv, u, T);
  const int len = mass_part_blocks(parts, G, T, b0);
  const int first = max(b0 + part * len, mass_first_block(un, tile * width, G, T, b0)), last = min(b0 + (part + 1) * len, (T + 15) / 16 * G);
  if (first >= last || mass_subtile(un, tile * width, T).base >= T) return;
  // (a tile of one or two subtiles: its wavefronts share the rows of a step, and their sums meet in LDS)
  const int subs = min(width, (un.n8 + kMassWave - 1) / kMassWave + (T - un.n8 + kMassWave - 1) / kMassWave - tile * width);
  const int across = subs >= 3 ? 4 : subs, shares = kObsWaves / across, share = w / across;
  const MassTile mt = mass_subtile(un, tile * width + w % across, T);
  const int base = mt.base, lim = mt.lim;
  const bool mine = base < lim;

  // rows of step `at`: thread (token, piece) takes sixteen bytes of each of its blocks' rows
  const int ltok = tid >> 4, lc = tid & 15, stride = observe_stride(T);
  static_assert(kMassStep == 4 && kRows == kWave, "four blocks of sixteen rows");
  int4 raw0, raw1, raw2, raw3;                         // (an array would go through memory)
  float rref = 0.f;
  double rweight = 0.0;
  int tb = first / G, h = first - tb * G;              // of the next block to request
  int tbc = tb, hc = h;                                // of the next block to work on
  const __half *q_lane = q + (size_t)g * G * D + lc * 8;
  auto load = [&](int at) {
    int my_tb = tb, my_h = h;
    auto block = [&](int k) {
      const int4 v = *(const int4 *)(q_lane + (((size_t)b * T + min(tb * 16 + ltok, T - 1)) * cv.Hkv * G + h) * D);
      if (at + k + 1 < last) {                          // (a step's last blocks may not exist: the last one again, with weight 0)
        const bool wrap = h + 1 == G;
        h = wrap ? 0 : h + 1;
        tb += wrap;
      }
      my_tb = tid >> 4 > k ? tb : my_tb;
      my_h = tid >> 4 > k ? h : my_h;
      return v;
    };
    raw0 = block(0);
    raw1 = block(1);
    raw2 = block(2);
    raw3 = block(3);
    if (w == 0) {
      const size_t row = ((size_t)ul * G + my_h) * stride + my_tb * 16 + (tid & 15);
      const bool there = at + (tid >> 4) < last;
      const float r = stats.ref[row];
      const double v = stats.weight[row];
      rref = there ? r : 1e30f;
      rweight = there ? v : 0.0;
    }
  };
  load(first);

  half8_t kb[kSb][4], kl[kChan ? kSb : 1][4];
  float f[kSb];
  mass_keys<kChan>(un, mt, sm, t16, g4, kb, kl, f);

  double sum[kSb] = {};
  for (int at = first, buf = 0; at < last; at += kMassStep, buf ^= 1) {
    uint8_t *at_lane = rows[buf] + ltok * kKRow16 + lc * 16;
    *(int4 *)at_lane = raw0;
    *(int4 *)(at_lane + 16 * kKRow16) = raw1;
    *(int4 *)(at_lane + 32 * kKRow16) = raw2;
    *(int4 *)(at_lane + 48 * kKRow16) = raw3;
    if (w == 0) { s_ref[buf][tid] = rref; s_weight[buf][tid] = rweight; }
    __syncthreads();                                    // the step is there, and nobody reads the one before any more
    if (at + kMassStep < last) load(at + kMassStep);
    if (!mine) continue;
    const int here = min(kMassStep, last - at);
    // (one copy of the body: a cold instruction cache costs more than the loop)
#pragma unroll 1
    for (int k = 0; k < here; ++k) {
      const int tok0 = tbc * 16;
      if (++hc == G) {
        hc = 0;
        ++tbc;
      }
      if (tok0 + 15 < base || k % shares != share) continue;   // (uniform over the wavefront)
      half8_t qa[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) qa[s] = *(const half8_t *)(rows[buf] + (16 * k + t16) * kKRow16 + s * 64 + g4 * 16);
      const float4 ref = *(const float4 *)&s_ref[buf][16 * k + 4 * g4];
      const double2 w0 = *(const double2 *)&s_weight[buf][16 * k + 4 * g4], w1 = *(const double2 *)&s_weight[buf][16 * k + 4 * g4 + 2];
      mass_block<kChan>(mt, qa, kb, kl, f, ref, w0, w1, tok0, t16, g4, sum);
    }
  }
#pragma unroll
  for (int sb = 0; sb < kSb; ++sb) {
    sum[sb] += __shfl_xor(sum[sb], 16, kWave);
    sum[sb] += __shfl_xor(sum[sb], 32, kWave);
  }
  if (shares > 1) {
    double *red = (double *)rows;                       // [wavefront][slot]
    __syncthreads();
#pragma unroll
    for (int sb = 0; sb < kSb; ++sb)
      if (g4 == 0) red[w * kMassWave + 16 * sb + t16] = sum[sb];
    __syncthreads();
    if (share > 0) return;
#pragma unroll
    for (int sb = 0; sb < kSb; ++sb)
      for (int k = 1; k < shares; ++k) sum[sb] += red[(w + k * across) * kMassWave + 16 * sb + t16];
  }
  if (!mine) return;
#pragma unroll
  for (int sb = 0; sb < kSb; ++sb) {
    const int slot = base + 16 * sb + t16;
    if (g4 == 0 && slot < lim) {
      if (parts > 1) stats.partial[((size_t)ul * parts + part) * stride + slot] = sum[sb];
      else cv.ema[(size_t)u * cv.cap + slot_row(cv, cv.pt, un.h8, un.n8, un.h16, slot)] = (float)sum[sb];
    }
  }
}

// The parts' column sums, in order.
__global__ __launch_bounds__(kObsThreads) void observe_sum_kernel(CacheView cv, int layer, int T, int b0, int parts, ObserveStats stats) {
  const int g = blockIdx.x % cv.Hkv, slot = blockIdx.x / cv.Hkv * kObsThreads + threadIdx.x, b = blockIdx.z;
  const int ul = b * cv.Hkv + g, u = layer * cv.B * cv.Hkv + ul;
  if (slot >= T) return;
  const ObserveUnit un = observe_unit(cv, u, T);
  const int nt8 = (un.n8 + kMassWave - 1) / kMassWave;
  const int sub = slot < un.n8 ? slot / kMassWave : nt8 + (slot - un.n8) / kMassWave;
  const int len = mass_part_blocks(parts, cv.G, T, b0), from = (mass_first_block(un, sub / kObsWaves * kObsWaves, cv.G, T, b0) - b0) / len;
  const int to = ((T + 15) / 16 * cv.G - b0 + len - 1) / len;               // (the last parts may be empty)
  const double *src = stats.partial + (size_t)ul * parts * observe_stride(T) + slot;
  double A = 0.0;
#pragma unroll 8
  for (int p = from; p < to; ++p) A += src[(size_t)p * observe_stride(T)];
  cv.ema[(size_t)u * cv.cap + slot_row(cv, cv.pt, un.h8, un.n8, un.h16, slot)] = (float)A;
}

// The rows ahead of the first that counts (observe_first_block) weigh nothing, unless they are no numbers: a query that is NaN or
// infinite leaves no number in any slot that its token sees, as in the kernels above.  Reads the queries of those tokens once, a
// workgroup kOddTokens of a kv-head (2000 of 3001 tokens with 32 heads, 16 MB: 4.7 us); nearly always that is all.
constexpr int kOddTokens = 32, kOddBatch = 8;
__global__ __launch_bounds__(kObsThreads) void observe_odd_kernel(CacheView cv, int layer, const __half *__restrict__ q, int T, int tokens) {
  constexpr int D = 128, kPieces = D / 8;
  __shared__ int s_last;
  const int tid = threadIdx.x, g = blockIdx.x % cv.Hkv, tok0 = (int)(blockIdx.x / cv.Hkv) * kOddTokens, b = blockIdx.z, G = cv.G;
  const int pieces = (min(tok0 + kOddTokens, tokens) - tok0) * G * kPieces;
  if (tid == 0) s_last = -1;
  __syncthreads();
  int last = -1;
  for (int base = tid; base < pieces; base += kOddBatch * kObsThreads) {
    confkv_v4i x[kOddBatch];
    int tok[kOddBatch];
#pragma unroll
    for (int k = 0; k < kOddBatch; ++k) {
      const int p = min(base + k * kObsThreads, pieces - 1), row = p / kPieces, head = row % G;
      tok[k] = tok0 + row / G;
      x[k] = *(const confkv_v4i *)(q + ((((size_t)b * T + tok[k]) * cv.Hkv + g) * G + head) * D + p % kPieces * 8);
    }
#pragma unroll
    for (int k = 0; k < kOddBatch; ++k) {
      half2_t sum = {0, 0};                              // finite numbers times 0
#pragma unroll
      for (int i = 0; i < 4; ++i) sum = __builtin_elementwise_fma(__builtin_bit_cast(half2_t, (int)x[k][i]), half2_t{0, 0}, sum);
      if (!(sum[0] == 0 && sum[1] == 0)) last = tok[k];  // (tokens rise)
    }
  }
  if (last >= 0) atomicMax(&s_last, last);
  __syncthreads();
  if (s_last < 0) return;
  const int u = (layer * cv.B + b) * cv.Hkv + g;
  const ObserveUnit un = observe_unit(cv, u, T);
  for (int slot = tid; slot <= s_last; slot += kObsThreads)
    cv.ema[(size_t)u * cv.cap + slot_row(cv, cv.pt, un.h8, un.n8, un.h16, slot)] = NAN;
}

hipError_t launch_observe_prompt(const CacheView &cv, int layer, const __half *q, int T, float sm, double decay, double gain,
                                 float *scratch, size_t scratch_floats, hipStream_t stream) {
  if (cv.D != 128 || cv.page_lg || T < 1) return hipErrorInvalidValue;
  const int units = cv.B * cv.Hkv, b0 = observe_first_block(cv.G, T, decay, gain), nblocks = (T + 15) / 16 * cv.G - b0;
  const int n8 = cv.W < 0 ? 0 : std::max(0, T - cv.W);    // (as the prompt was loaded)
  const ObservePlan plan = observe_plan(units, cv.G, T, b0, n8, cv.chan != 0, scratch_floats, device_cus());
  if (plan.floats > scratch_floats) return hipErrorInvalidValue;
  const int tile = plan.tile, per_part = plan.per_part, row_parts = plan.row_parts, width = plan.width, parts = plan.parts;
  // (an odd count: a unit's workgroups follow one another on its XCD, and with an even one the tiles of most rows always fall to
  // the same shader engines: 64 units of 300 tokens, 8 heads 80 us with two tiles, 65 with three; of 700 tokens, 2 heads 88 with four)
  const int ntiles = (plan.subtiles + width - 1) / width | 1;
  const int nitems = (nblocks + plan.item - 1) / plan.item;
  const dim3 rows(cv.Hkv * nitems * row_parts, 1, cv.B), slots(cv.Hkv * ntiles * parts, 1, cv.B);
  const size_t n_rows = plan.n_rows;
  // final statistics, then the partial ones of the rows, and over them those of the columns
  ObserveStats stats{};
  stats.weight = (double *)scratch;
  stats.ref = scratch + 2 * n_rows;
  stats.partial = (double *)(scratch + plan.stat_floats);
  if (row_parts > 1) {
    stats.row_sum = stats.partial;
    stats.row_ref = (float *)(stats.row_sum + row_parts * n_rows);
  }
  const auto first = cv.chan ? plan.item == kObsShortItem ? observe_stats_kernel<true, 1> : observe_stats_kernel<true, 2>
                             : plan.item == kObsShortItem ? observe_stats_kernel<false, 1> : observe_stats_kernel<false, 2>;
  hipLaunchKernelGGL(first, rows, dim3(kObsThreads), 0, stream, cv, layer, q, T, sm, decay, gain, b0, per_part, stats);
  if (row_parts > 1)
    hipLaunchKernelGGL(observe_join_kernel, dim3((unsigned)((n_rows + kObsThreads - 1) / kObsThreads)), dim3(kObsThreads), 0, stream, cv, layer, T, tile, decay, gain, b0, per_part, stats);
  if (plan.short_form) {
    const dim3 grid(cv.Hkv * plan.subtiles, 1, cv.B);
    if (cv.chan) hipLaunchKernelGGL(observe_mass_short_kernel<true>, grid, dim3(kMassShortThreads), 0, stream, cv, layer, q, T, sm, b0, stats);
    else hipLaunchKernelGGL(observe_mass_short_kernel<false>, grid, dim3(kMassShortThreads), 0, stream, cv, layer, q, T, sm, b0, stats);
  } else {
    if (cv.chan) hipLaunchKernelGGL(observe_mass_kernel<true>, slots, dim3(kObsThreads), 0, stream, cv, layer, q, T, sm, ntiles, width, b0, parts, stats);
    else hipLaunchKernelGGL(observe_mass_kernel<false>, slots, dim3(kObsThreads), 0, stream, cv, layer, q, T, sm, ntiles, width, b0, parts, stats);
    if (parts > 1)
      hipLaunchKernelGGL(observe_sum_kernel, dim3(cv.Hkv * ((T + kObsThreads - 1) / kObsThreads), 1, cv.B), dim3(kObsThreads), 0, stream, cv, layer, T, b0, parts, stats);
  }
  if (const int tokens = b0 / cv.G * 16)
    hipLaunchKernelGGL(observe_odd_kernel, dim3(cv.Hkv * ((tokens + kOddTokens - 1) / kOddTokens), 1, cv.B), dim3(kObsThreads), 0, stream, cv, layer, q, T, tokens);
  return hipGetLastError();
}
