// Outlier CHANNELS (Section 3.2, Eq. 1): the activation is a row-major matrix of `tokens` rows and
// `hidden` channels; S_h = sum over the tokens of |x|, Z_h = (S_h - mu) / sigma over the channels,
// channels with Z_h above the threshold are kept whole, zeroed in the activation, and the rest is
// group-quantised (Eq. 2 / Eq. 3) by the same encoder as a tensor without outliers.
//
// The selection is an integer decision taken by floating-point sums, so the order of the sums is
// fixed: chunks of 64 tokens added one after the other in binary32; the chunk sums added one after
// the other in binary64; sums over channels in 512 binary64 accumulators, an octet of channels at a time, folded by halves.
#pragma once

#include "adacc_common.hpp"
#include "adacc_compress.hpp"
#include "adacc_decompress.hpp"

namespace adacc {
namespace ADACC_DT_NS {

constexpr int kSelectThreads = 512;     // accumulators of the sums over channels

// ---- step 1: binary32 sums of |x| over chunks of 64 tokens, partial[chunk][hidden].  A workgroup
// takes one chunk of a strip of 512 channels: a lane owns 8 adjacent channels (one 16-byte load per
// token, rows fully coalesced), each wavefront a run of the chunk's tokens, all its loads in flight
// at once; the wavefronts' sums meet in LDS and are added in token order, a thread per channel (by one wavefront, 8 channels a
// lane, a pass of [8192, 4096] both ways took 54.2 us, 53.9 now).  Short-lived workgroups in
// the hardware's order walk through the tensor as a window, which reads faster than a grid that is
// resident as a whole and covers the tensor all the time.
template <bool STREAM>
__global__ __launch_bounds__(kPartialWaves * kWave) void channel_partial_kernel(const uint16_t* __restrict__ x,
                                                                               uint32_t tokens, uint32_t hidden,
                                                                               float* __restrict__ partial,
                                                                               uint32_t strips) {
  // [wavefront][element of the octet][lane], 8 lanes' room behind 64: the threads of a sum read 8 elements of 8 lanes from banks of their own
  constexpr uint32_t kRoom = kWave + 8;
  __shared__ float meet[kPartialWaves][kOct * kRoom];
  const uint32_t wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint32_t chunk = blockIdx.x / strips;
  const uint32_t strip = blockIdx.x - chunk * strips;
  const uint32_t oct = strip * kWave + lane;
  const bool live = oct < hidden / kOct;
  const uint32_t t0 = chunk * kChunkTokens + wave * kPartialRows;
  const uint32_t rows = t0 >= tokens ? 0u : (tokens - t0 < kPartialRows ? tokens - t0 : kPartialRows);
  const uint16_t* p = x + (size_t)t0 * hidden + (size_t)oct * kOct;
  uint4 v[kPartialRows];
#pragma unroll
  for (uint32_t i = 0; i < kPartialRows; ++i) {
    v[i] = make_uint4(0u, 0u, 0u, 0u);  // a token that is not there adds +0
    if (live && i < rows) v[i] = load_stats16<STREAM>(p + (size_t)i * hidden);
  }
  float acc[kOct];
#pragma unroll
  for (int e = 0; e < kOct; ++e) acc[e] = 0.0f;
#pragma unroll
  for (uint32_t i = 0; i < kPartialRows; ++i) {
    const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      acc[2 * k] = acc[2 * k] + fabsf(widen_lo(w[k]));
      acc[2 * k + 1] = acc[2 * k + 1] + fabsf(widen_hi(w[k]));
    }
  }
#pragma unroll
  for (uint32_t e = 0; e < (uint32_t)kOct; ++e) meet[wave][e * kRoom + lane] = acc[e];
  __syncthreads();
  const uint32_t col = threadIdx.x;  // of the strip
  if (col < (uint32_t)kRow && strip * (uint32_t)kRow + col < hidden) {
    const uint32_t at = (col % (uint32_t)kOct) * kRoom + col / (uint32_t)kOct;
    float sum = meet[0][at];
#pragma unroll
    for (uint32_t w = 1; w < kPartialWaves; ++w) sum = sum + meet[w][at];
    partial[(size_t)chunk * hidden + strip * (uint32_t)kRow + col] = sum;
  }
}

// ---- step 2: S_h = binary64 sum of the chunk sums, in chunk order.  The additions of one channel
// form a chain, so the kernel is bound by latency, not by bytes: a workgroup takes 32 channels, all
// its threads fetch a block of 256 chunk sums per channel into LDS at once, then one lane per channel
// adds them up in order.
constexpr int kScoreChannels = 32;
constexpr int kScoreChunks = 256;
__global__ __launch_bounds__(kThreads) void channel_score_kernel(const float* __restrict__ partial, uint32_t n_chunks,
                                                                 uint32_t hidden, double* __restrict__ S) {
  __shared__ __attribute__((aligned(16))) float stage[kScoreChunks][kScoreChannels];
  const uint32_t h0 = blockIdx.x * kScoreChannels;
  const uint32_t quad = threadIdx.x % (kScoreChannels / 4);   // which 4 channels of the 32
  const uint32_t row = threadIdx.x / (kScoreChannels / 4);    // 0..31
  constexpr uint32_t kRowsPerPass = kThreads / (kScoreChannels / 4);
  const bool col_ok = h0 + quad * 4u < hidden;                // hidden is a multiple of 8
  constexpr uint32_t kPasses = kScoreChunks / kRowsPerPass;
  float4 v[kPasses];
  auto fetch = [&](uint32_t c0) {
    const uint32_t rows = n_chunks - c0 < (uint32_t)kScoreChunks ? n_chunks - c0 : (uint32_t)kScoreChunks;
#pragma unroll
    for (uint32_t i = 0; i < kPasses; ++i) {
      const uint32_t r = row + i * kRowsPerPass;
      v[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if (col_ok && r < rows)
        v[i] = *reinterpret_cast<const float4*>(partial + (size_t)(c0 + r) * hidden + h0 + quad * 4u);
    }
  };
  double s = 0.0;
  fetch(0u);
  for (uint32_t c0 = 0; c0 < n_chunks; c0 += kScoreChunks) {
    const uint32_t rows = n_chunks - c0 < (uint32_t)kScoreChunks ? n_chunks - c0 : (uint32_t)kScoreChunks;
#pragma unroll
    for (uint32_t i = 0; i < kPasses; ++i)
      *reinterpret_cast<float4*>(&stage[row + i * kRowsPerPass][quad * 4u]) = v[i];
    __syncthreads();
    if (c0 + kScoreChunks < n_chunks) fetch(c0 + kScoreChunks);  // in flight while this block is added up
    if (threadIdx.x < (uint32_t)kScoreChannels) {
      constexpr uint32_t kBatch = 32;  // LDS reads in flight ahead of the chain of additions
      uint32_t r = 0;
      for (; r + kBatch <= rows; r += kBatch) {
        float w[kBatch];
#pragma unroll
        for (uint32_t i = 0; i < kBatch; ++i) w[i] = stage[r + i][threadIdx.x];
#pragma unroll
        for (uint32_t i = 0; i < kBatch; ++i) s = __dadd_rn(s, (double)w[i]);
      }
      for (; r < rows; ++r) s = __dadd_rn(s, (double)stage[r][threadIdx.x]);
    }
    __syncthreads();
  }
  if (threadIdx.x < (uint32_t)kScoreChannels && h0 + threadIdx.x < hidden) S[h0 + threadIdx.x] = s;
}

__device__ __forceinline__ bool finite_f64(double v) {
  return ((uint64_t)__double_as_longlong(v) & 0x7FF0000000000000ull) != 0x7FF0000000000000ull;
}

// The sum of all threads' accumulators, in a fixed order: the butterfly inside a wavefront (both partners add the same two
// numbers, so every lane ends with the same bits), then the wavefronts' sums through LDS, added in wavefront order by every
// thread.  One barrier; `a` (LDS, one per wavefront) is used for one sum only.
constexpr int kSelectWaves = kSelectThreads / kWave;
__device__ __forceinline__ double meet_accumulators(double mine, double* a) {
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) mine = __dadd_rn(mine, __shfl_xor(mine, o, kWave));
  if (threadIdx.x % kWave == 0) a[threadIdx.x / kWave] = mine;
  __syncthreads();
  double total = a[0];
#pragma unroll
  for (int w = 1; w < kSelectWaves; ++w) total = __dadd_rn(total, a[w]);
  return total;
}
// what the wavefronts counted, in all; before: in the wavefronts before this one (a barrier lies between the writes to cnt and this)
__device__ __forceinline__ uint32_t sum_counts(const uint32_t* cnt, uint32_t* before) {
  const uint32_t wave = threadIdx.x / kWave;
  uint32_t total = 0u;
  *before = 0u;
#pragma unroll
  for (int w = 0; w < kSelectWaves; ++w) {
    if ((uint32_t)w < wave) *before += cnt[w];
    total += cnt[w];
  }
  return total;
}

// ---- step 3 (Eq. 1): mu, sigma, Z, the channel mask, the list of outlier channels.  One workgroup; thread j takes the octets j,
// j + 512, .. of channels, one mask byte each, and keeps the first two octets' sums in registers over the three passes (mean,
// variance, selection): up to 8192 channels S is read once.  Bound by the chain of its steps: three reductions, a square root and two
// divisions.  Z > z_thresh is decided by a product where rounding cannot matter, S - mu further from z_thresh * sigma than 2^-40 of
// it; a division of every channel was half the time.  (1024 threads, S read three times, two barriers a reduction: 7.9
// us for 4096 channels, 9.0 for 8192; 4.8 and 5.8 now.)
constexpr uint32_t kSelectKept = 2;
// FEW: of at most kFewChunks chunks, where no channel is read twice, the kernel adds the chunk sums up itself, the same additions in the same
// order as step 2's, which is left out.
template <bool FEW>
__global__ __launch_bounds__(kSelectThreads) void channel_select_kernel(const double* __restrict__ S, ChannelDesc c, const float* __restrict__ partial,
                                                                         uint32_t n_chunks) {
  __shared__ double a[2][kSelectWaves];
  __shared__ uint32_t cnt[2][kSelectWaves];
  const uint32_t j = threadIdx.x, wave = j / kWave;
  const uint32_t n_bytes = c.hidden / 8u;
  const double skip = __longlong_as_double(0x7FF0000000000000ll);  // a channel that is not there reads as a sum that is not finite
  double kept[kSelectKept][8];
  auto load = [&](uint32_t b, double (&v)[8]) {
    if constexpr (FEW) {
      const float* p = partial + (size_t)(b < n_bytes ? b : 0u) * 8u;
#pragma unroll
      for (uint32_t e = 0; e < 8u; ++e) v[e] = 0.0;
      float4 t[kFewChunks][2];
#pragma unroll
      for (uint32_t i = 0; i < kFewChunks; ++i) {  // chunks past the end re-read the last one
        const float* q = p + (size_t)(i < n_chunks ? i : n_chunks - 1u) * c.hidden;
        t[i][0] = reinterpret_cast<const float4*>(q)[0];
        t[i][1] = reinterpret_cast<const float4*>(q)[1];
      }
#pragma unroll
      for (uint32_t i = 0; i < kFewChunks; ++i) {
        const float w[8] = {t[i][0].x, t[i][0].y, t[i][0].z, t[i][0].w, t[i][1].x, t[i][1].y, t[i][1].z, t[i][1].w};
#pragma unroll
        for (uint32_t e = 0; e < 8u; ++e) v[e] = i < n_chunks ? __dadd_rn(v[e], (double)w[e]) : v[e];
      }
#pragma unroll
      for (uint32_t e = 0; e < 8u; ++e) v[e] = b < n_bytes ? v[e] : skip;
    } else {
      const double2* p = reinterpret_cast<const double2*>(S + (size_t)(b < n_bytes ? b : 0u) * 8u);
#pragma unroll
      for (uint32_t e = 0; e < 4u; ++e) {
        const double2 t = p[e];
        v[2u * e] = b < n_bytes ? t.x : skip;
        v[2u * e + 1u] = b < n_bytes ? t.y : skip;
      }
    }
  };
#pragma unroll
  for (uint32_t k = 0; k < kSelectKept; ++k) load(j + k * kSelectThreads, kept[k]);
  // use(b, values) for every octet of this thread
  auto each = [&](auto use) {
#pragma unroll
    for (uint32_t k = 0; k < kSelectKept; ++k) use(j + k * kSelectThreads, kept[k]);
    for (uint32_t b = j + kSelectKept * kSelectThreads; b < n_bytes; b += kSelectThreads) {
      double v[8];
      load(b, v);
      use(b, v);
    }
  };

  double acc = 0.0;
  uint32_t n = 0u;
  each([&](uint32_t, const double (&v)[8]) {
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e)
      if (finite_f64(v[e])) { acc = __dadd_rn(acc, v[e]); ++n; }
  });
  n = wave_sum_u32(n);
  if (j % kWave == 0u) cnt[0][wave] = n;  // (behind the barrier of the sum)
  const double total = meet_accumulators(acc, a[0]);
  uint32_t unused;
  const double finite = (double)sum_counts(cnt[0], &unused);
  const double mu = __ddiv_rn(total, finite);

  acc = 0.0;
  each([&](uint32_t, const double (&v)[8]) {
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) {
      const double d = __dsub_rn(v[e], mu);
      if (finite_f64(v[e])) acc = __fma_rn(d, d, acc);
    }
  });
  const double sigma = __dsqrt_rn(__ddiv_rn(meet_accumulators(acc, a[1]), finite));
  const double zt = (double)c.z_thresh;
  const double bar = zt * sigma, margin = fabs(bar) * 0x1p-40;
  const bool plain = fabs(bar) > 0x1p-900 && fabs(bar) < 0x1p900;  // uniform; not: sigma or the threshold zero, sigma not finite

  // a round of octets (512 bytes of the mask) after the other, so that the channels stay in order
  uint32_t running = 0u;  // outlier channels of the rounds before
  uint32_t round = 0u;
  auto select = [&](uint32_t b, const double (&v)[8]) {
    uint32_t m = 0u, close = 0u;
#pragma unroll
    for (uint32_t e = 0; e < 8u; ++e) {
      const double d = __dsub_rn(v[e], mu);
      if (!finite_f64(v[e]) || d > bar) m |= 1u << e;
      if (finite_f64(v[e]) && !(plain && fabs(d - bar) > margin)) close |= 1u << e;
    }
    if (close != 0u) {  // few lanes, if any: the definition itself
#pragma unroll
      for (uint32_t e = 0; e < 8u; ++e) {
        const double z = __ddiv_rn(__dsub_rn(v[e], mu), sigma);
        if ((close >> e) & 1u) m = z > zt ? m | (1u << e) : m & ~(1u << e);  // a NaN z selects nothing
      }
    }
    if (b >= n_bytes) m = 0u;
    // where this thread's channels go in the list: behind the outlier channels of the threads before it
    uint32_t mine;
    const uint32_t below = count_below((uint32_t)__builtin_popcount(m), mine);
    if (j % kWave == 0u) cnt[round & 1u][wave] = mine;
    __syncthreads();  // (the other set of words was read before the barrier of this round)
    uint32_t before;
    const uint32_t all = sum_counts(cnt[round & 1u], &before);
    ++round;
    uint32_t at = running + before + below;
    running += all;
    if (b < n_bytes) {
      c.mask[b] = (uint8_t)m;
      c.base[b] = at;
      while (m != 0u) {
        const uint32_t e = (uint32_t)__builtin_ctz(m);
        m &= m - 1u;
        if (at < c.max_channels) c.ch_idx[at] = (int32_t)(b * 8u + e);
        ++at;
      }
    }
  };
  // every thread goes through every round (the barriers)
  const uint32_t rounds = (n_bytes + (uint32_t)kSelectThreads - 1u) / (uint32_t)kSelectThreads;
  round = 1u;  // (the finite counts lie in set 0, and are read before the barrier of the variance)
#pragma unroll
  for (uint32_t k = 0; k < kSelectKept; ++k)
    if (k < rounds) select(j + k * kSelectThreads, kept[k]);  // uniform
  for (uint32_t k = kSelectKept; k < rounds; ++k) {
    double v[8];
    load(j + k * kSelectThreads, v);
    select(j + k * kSelectThreads, v);
  }
  if (j == 0) {
    c.status[0] = running;
    c.status[1] = running > c.max_channels ? 1u : 0u;
    c.status[2] = 0u;
    c.status[3] = 0u;
  }
}

// element e (0..7) of an octet held as 4 words
__device__ __forceinline__ uint32_t octet_half(const uint32_t (&w)[4], uint32_t e) {
  const uint32_t lo = (e & 4u) ? w[2] : w[0];
  const uint32_t hi = (e & 4u) ? w[3] : w[1];
  const uint32_t word = (e & 2u) ? hi : lo;
  return (e & 1u) ? word >> 16 : word & 0xFFFFu;
}

// where the tile's rows lie in the matrix
struct ChannelGeo {
  uint32_t row0, col0;  // uniform: token and channel of the tile's first element
};
__device__ __forceinline__ ChannelGeo channel_geo(uint32_t tile, uint32_t hidden) {
  const uint32_t base = tile * (uint32_t)(4 * kRow);  // numel < 2^32 in this mode
  ChannelGeo g;
  g.row0 = base / hidden;
  g.col0 = base - g.row0 * hidden;
  return g;
}

// off = q * hidden + col for off < hidden + 2048 <= 2^24 / 8: the quotient through a binary32 reciprocal
// that the host rounded down, so the estimate is the true quotient or one less.
__device__ __forceinline__ void split_offset(uint32_t off, uint32_t hidden, float inv_hidden, uint32_t& q,
                                             uint32_t& col) {
  q = (uint32_t)((float)off * inv_hidden);
  col = off - __umul24(q, hidden);
  if (col >= hidden) { col -= hidden; ++q; }
}

// ---- step 4: the outlier channels of one tile are stored and zeroed, then the tile is encoded
// like one of a tensor without outliers.  A wavefront takes one tile of consecutive elements; which of the channels of a lane's octets
// are outlier channels, and where their values go in a token's record, is asked for together with the values and the status, one
// round trip to memory.  (With copies of mask and ranks in LDS for workgroups that looped over tiles, and the octets in scratch memory
// because the loop over rows was not unrolled, us both ways: [17840, 768] int8 asymmetric 45.9, [8000, 3000] int4 58.8, [4000, 11008] 89.8,
// [600, 3000] 22.2; 41.3, 49.5, 73.9 and 20.7 so.)
template <int BITS, bool ASYM, bool ROWWISE, bool COMPLETE>
__device__ __forceinline__ void channel_compress_tile(const TensorDesc& d, const ChannelDesc& c, uint32_t tile) {
  constexpr int E = 4;
  const uint32_t found = c.status[0], over = c.status[1];
  uint32_t raw[E][4];
  load_tile<E, COMPLETE>(d, tile, raw);
  const TileGeo<E> g = tile_geo<E, COMPLETE>(d, tile);
  const ChannelGeo cg = channel_geo(tile, c.hidden);
  uint32_t m[E], first[E], row[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const uint32_t in_tile = g.lane_off + (uint32_t)(j * kRow);
    uint32_t q, col;
    split_offset(cg.col0 + in_tile, c.hidden, c.inv_hidden, q, col);
    row[j] = cg.row0 + q;
    m[j] = c.mask[col >> 3];
    first[j] = c.base[col >> 3];
    if (!COMPLETE && in_tile >= g.rem) m[j] = 0u;
  }
  asm volatile("" ::: "memory");  // (the loads stay ahead of the return)
  if (__builtin_amdgcn_readfirstlane(over) != 0u) return;  // more outlier channels than the blob holds: nothing else is produced
  const uint32_t n_ch = __builtin_amdgcn_readfirstlane(found);
  if constexpr (!COMPLETE) blank_tail<E>(g, raw);
  static_for<E>([&](auto Jc) {  // the data-dependent loop inside must not keep this one rolled
    constexpr int j = decltype(Jc)::value;
    if (m[j] != 0u) {
      uint16_t* dst = c.ch_val + (size_t)row[j] * n_ch + first[j];
      // the values go out first (one round per outlier channel of the octet: mostly one), then they are cleared
      uint32_t todo = m[j], r = 0u;
      while (todo != 0u) {
        const uint32_t e = (uint32_t)__builtin_ctz(todo);
        todo &= todo - 1u;
        dst[r++] = (uint16_t)octet_half(raw[j], e);
      }
      clear_elements(raw[j], m[j]);
    }
  });
  encode_tile<kModeNone, BITS, ASYM, E, ROWWISE, false, true>(d, g, raw, tile, NullSink{}, 0u, 0u);
}

template <int BITS, bool ASYM, bool ROWWISE>
__global__ __launch_bounds__(kThreads) void channel_compress_kernel(TensorDesc d, ChannelDesc c) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t t = blockIdx.x * kWavesPerWg + wave;
  if (t >= d.n_tiles) return;
  if (t + 1u < d.n_tiles) channel_compress_tile<BITS, ASYM, ROWWISE, true>(d, c, t);
  else channel_compress_tile<BITS, ASYM, ROWWISE, false>(d, c, t);
}

// ---- step 4 for matrices whose rows are whole multiples of 512 channels, groups inside 512 channels:
// a wavefront takes a strip of 512 adjacent channels (8 per lane) over kChannelStripRows consecutive
// tokens.  Which of a lane's 8 channels are outlier channels, and where their values go in a token's
// record, is the same for every token: looked up once, no table in LDS and no division per octet.  All
// loads of the strip are issued first; its rows are then encoded four at a time like a tile's.
// (Eight tokens to a wavefront, two times four: [8192, 4096] int4 18.9 us, restored in 20.0; four: 16.7 and 18.1;
// [2192, 5120] asymmetric, restored: 10.9 -> 8.6.)
// The values are asked for together with the status, the mask and the ranks, in both directions, one round trip to memory instead of
// three in a row; a wavefront lives for little more.  ([8192, 4096] int4, compressed and restored: 56.2 -> 54.9 us.)
constexpr uint32_t kChannelStripRows = 4;

template <int BITS, bool ASYM>
__global__ __launch_bounds__(kThreads) void channel_compress_strip_kernel(TensorDesc d, ChannelDesc c) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t found = c.status[0], over = c.status[1];
  const uint32_t strips = c.hidden / (uint32_t)kRow;
  const uint32_t unit = blockIdx.x * kWavesPerWg + wave;
  const uint32_t block = unit / strips;
  const uint32_t row0 = block * kChannelStripRows;
  if (row0 >= c.tokens) return;  // uniform
  const uint32_t col0 = (unit - block * strips) * (uint32_t)kRow;
  const uint32_t rows = c.tokens - row0 < kChannelStripRows ? c.tokens - row0 : kChannelStripRows;
  const uint32_t lane_off = (uint32_t)lane_id() * kOct;

  // everything that is read is asked for at once: the status decides what is done with it, not whether it is read
  const uint32_t m = c.mask[(col0 + lane_off) >> 3], first = c.base[(col0 + lane_off) >> 3];
  const uint64_t base = (uint64_t)row0 * c.hidden + col0;  // uniform
  const uint16_t* sp = d.src + base;
  uint32_t raw[kChannelStripRows][4];
#pragma unroll
  for (uint32_t i = 0; i < kChannelStripRows; ++i) {  // rows past the end re-read the last one
    const uint32_t row = i < rows ? i : rows - 1u;
    const uint4 v = ADACC_LOAD16(sp + (row * c.hidden + lane_off));
    raw[i][0] = v.x; raw[i][1] = v.y; raw[i][2] = v.z; raw[i][3] = v.w;
  }
  asm volatile("" ::: "memory");  // (the loads stay ahead of the return)
  if (__builtin_amdgcn_readfirstlane(over) != 0u) return;  // more outlier channels than the blob holds: nothing else is produced
  const uint32_t n_ch = __builtin_amdgcn_readfirstlane(found);
  if (m != 0u) {  // the kept channels go out first, then they are cleared
    uint16_t* dst = c.ch_val + (size_t)row0 * n_ch + first;
    static_for<(int)kChannelStripRows>([&](auto Ic) {  // the data-dependent loop inside must not keep this one rolled
      constexpr uint32_t i = (uint32_t)decltype(Ic)::value;
      if (i < rows) {
        uint32_t todo = m, r = 0u;
        while (todo != 0u) {
          const uint32_t e = (uint32_t)__builtin_ctz(todo);
          todo &= todo - 1u;
          dst[(size_t)i * n_ch + r++] = (uint16_t)octet_half(raw[i], e);
        }
      }
      clear_elements(raw[i], m);
    });
  }
  if (rows == kChannelStripRows) {  // uniform
    TileGeo<(int)kChannelStripRows, true> g;
    g.base = base;
    g.rem = kChannelStripRows * (uint32_t)kRow;
    g.lane_off = lane_off;
    g.full = true;
    g.stride = c.hidden;
    encode_tile_rowwise<kModeNone, BITS, ASYM, (int)kChannelStripRows, true>(d, g, raw, 0u, NullSink{}, 0u, 0u);
  } else {
    static_for<(int)kChannelStripRows>([&](auto Ic) {  // the last tokens of the matrix, one row at a time
      constexpr uint32_t i = (uint32_t)decltype(Ic)::value;
      if (i < rows) {
        TileGeo<1, true> g;
        g.base = base + (uint64_t)i * c.hidden;
        g.rem = (uint32_t)kRow;
        g.lane_off = lane_off;
        g.full = true;
        g.stride = c.hidden;
        const uint32_t one[1][4] = {{raw[i][0], raw[i][1], raw[i][2], raw[i][3]}};
        encode_tile_rowwise<kModeNone, BITS, ASYM, 1, true>(d, g, one, 0u, NullSink{}, 0u, 0u);
      }
    });
  }
}

// ---- decompression: dequantise, put the outlier channels back, store.
// A wavefront takes a strip of 512 adjacent channels (8 per lane; binary32: 256, 4 per lane, see chunk_elems) over
// kChannelStripRows consecutive tokens: which of a lane's channels are outlier channels, and where their values start in a token's record, is
// the same for every token, so it is looked up once (no table in LDS, no division per octet).  The loads of
// four tokens (codes, scale, offset, the first kept value of the octet) are issued before their first store;
// a second outlier channel in the same octet is rare and fetched when it is needed.
template <int BITS, bool ASYM, bool F32>
__global__ __launch_bounds__(kThreads) void channel_decompress_kernel(TensorDesc d, ChannelDesc c) {
  constexpr int V = chunk_elems<F32>();
  constexpr uint32_t W = (uint32_t)(kWave * V);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t found = c.status[0], over = c.status[1];
  const uint32_t strips = (c.hidden + W - 1u) / W;
  const uint32_t unit = blockIdx.x * kWavesPerWg + wave;
  const uint32_t block = unit / strips;
  const uint32_t row0 = block * kChannelStripRows;
  const uint32_t col = (unit - block * strips) * W + (uint32_t)(lane_id() * V);
  if (row0 >= c.tokens || col >= c.hidden) return;
  const uint32_t rows = c.tokens - row0 < kChannelStripRows ? c.tokens - row0 : kChannelStripRows;

  // Everything but the kept values is asked for at once: the status decides what is done with it, not whether it is read.
  // The lane's channels: which are outlier channels, and the rank of the first of them.
  uint32_t m = c.mask[col >> 3], first = c.base[col >> 3];
  uint32_t cw[kChannelStripRows][V * BITS > 32 ? 2 : 1];
  float sc[kChannelStripRows], zp[kChannelStripRows];
#pragma unroll
  for (uint32_t i = 0; i < kChannelStripRows; ++i) {  // rows past the end re-read the last one
    const uint32_t row = row0 + (i < rows ? i : rows - 1u);
    const uint64_t e0 = (uint64_t)row * c.hidden + col;
    const uint8_t* p = d.codes + e0 * BITS / 8;
    if constexpr (V * BITS == 64) {
      const uint2 w = *reinterpret_cast<const uint2*>(p);
      cw[i][0] = w.x; cw[i][1] = w.y;
    } else if constexpr (V * BITS == 32) {
      cw[i][0] = *reinterpret_cast<const uint32_t*>(p);
    } else {
      cw[i][0] = *reinterpret_cast<const uint16_t*>(p);
    }
    const uint64_t grp = e0 >> d.lgq;
    sc[i] = d.scales[grp];
    zp[i] = 0.0f;
    if constexpr (ASYM) zp[i] = d.zp[grp];
  }
  asm volatile("" ::: "memory");  // (the loads stay ahead of the return)
  if (__builtin_amdgcn_readfirstlane(over) != 0u) return;  // not a usable blob
  uint32_t n_ch = __builtin_amdgcn_readfirstlane(found);
  if (n_ch > c.max_channels) n_ch = c.max_channels;  // a damaged blob must not make the reads leave it
  if constexpr (V == 4) {  // the octet's lower or upper half
    first += (col & 4u) ? (uint32_t)__popc(m & 0xFu) : 0u;
    m = (col & 4u) ? m >> 4 : m & 0xFu;
  }
  if (first >= n_ch) m = 0u;  // no outlier channels, or a damaged blob, which must not be read past its end
  const uint32_t lowest = m & (0u - m);
  const uint32_t rest = m ^ lowest;
  uint32_t pre[kChannelStripRows];
  const uint16_t* src[kChannelStripRows];
#pragma unroll
  for (uint32_t i = 0; i < kChannelStripRows; ++i) {
    src[i] = c.ch_val + (size_t)(row0 + (i < rows ? i : rows - 1u)) * n_ch + first;
    pre[i] = m != 0u ? (uint32_t)src[i][0] : 0u;
  }
#pragma unroll
  for (uint32_t i = 0; i < kChannelStripRows; ++i) {
    if (i >= rows) break;
    const uint64_t e0 = (uint64_t)(row0 + i) * c.hidden + col;
    int code[V];
    unpack_codes<BITS, V>(cw[i], code);
    float v[V];
#pragma unroll
    for (int e = 0; e < V; ++e) v[e] = ASYM ? __fmaf_rn((float)code[e], sc[i], zp[i]) : (float)code[e] * sc[i];

    // the kept channels of this octet, as their stored 16-bit patterns (hold[e] valid where keep has bit e)
    uint32_t keep = lowest, hold[V];
#pragma unroll
    for (int e = 0; e < V; ++e) hold[e] = lowest == (1u << e) ? pre[i] : 0u;
    if (rest != 0u) {
#pragma unroll
      for (int e = 1; e < V; ++e)
        if (rest & (1u << e)) {
          const uint32_t rank = (uint32_t)__popc(m & ((1u << e) - 1u));
          if (rank < n_ch - first) { hold[e] = src[i][rank]; keep |= 1u << e; }
        }
    }

    if constexpr (F32) {
      if (keep != 0u) {
#pragma unroll
        for (int e = 0; e < V; ++e) v[e] = (keep & (1u << e)) ? widen_lo(hold[e]) : v[e];
      }
      float* p = reinterpret_cast<float*>(d.dst) + e0;
      ADACC_STORE16(p, make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])));
    } else {
      uint32_t w[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = narrow_pair(v[2 * k], v[2 * k + 1]);
      if (keep != 0u) {  // the kept values go in as they were stored, bit for bit (no conversion touches a NaN)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (keep & (1u << (2 * k))) w[k] = (w[k] & 0xFFFF0000u) | hold[2 * k];
          if (keep & (2u << (2 * k))) w[k] = (w[k] & 0x0000FFFFu) | (hold[2 * k + 1] << 16);
        }
      }
      ADACC_STORE16(reinterpret_cast<uint16_t*>(d.dst) + e0, make_uint4(w[0], w[1], w[2], w[3]));
    }
  }
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
