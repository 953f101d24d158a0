// Compression with outliers of a short tensor in one launch.
//
// The order of the outlier stream needs the number of outliers in all tiles before a tile's own.  For a tensor of up to
// kShortWorkgroups workgroups those do not wait for a second kernel: every workgroup encodes its four tiles, keeps their
// outliers in LDS, publishes their number in a word of the workspace, and looks at the words of the workgroups before it
// until they are there.  A word carries the number of the launch, of all such launches of the process, above the count (short_tag) and
// says everything by itself, so nothing has to be cleared, and no other memory has to be ordered; what other calls may have
// left in its place does not read as one.
//
// No wait is without an end, whatever order workgroups are started in: a wavefront whose patience is at an end counts the
// outliers of the missing tiles itself, from the source.  Workgroups are started in the order of their numbers on every XCD and nobody
// waits for a later one, so one such launch alone always goes on; two at a time could fill an XCD each with workgroups that wait for
// some the other keeps out, and there the patience, some 0.5 ms where a wait as a rule takes a few microseconds, ends it.
#pragma once

#include "adacc_compress.hpp"
#include "adacc_tail.hpp"

namespace adacc {
namespace ADACC_DT_NS {

struct ShortShared {
  uint32_t record[kWavesPerWg][kSlot];  // a tile's outliers: number in the tile << 16 | value
  uint32_t count[kWavesPerWg];          // a tile's outliers, how many
  uint32_t part[kWavesPerWg];           // of the sum over the words
  uint32_t arrived;                     // tiles whose outliers are found << 24 | those of them
};

// The wavefront's record.  The last wavefront of a workgroup to know its outliers publishes their number, ahead of the codes (all_found):
// the word is on its way while they are formed.  That is why methods whose groups lie inside a row go through the general encoder
// here too, and not through the one by rows, which knows its outliers at the end.  ([rows, 1024] STD over 1024, both ways: 1024 rows
// 10.3 us with the word behind the codes, 8.6 so; [3000, 2051] STD over 512 15.1, 13.3; by rows / so: softmax, ABS, [1200, 512] 11.0, 9.5, GELU
// at 3 sigma over 64, [1200, 3072] 17.2, 14.9.)
struct ShortSink : SlotSink {
  uint32_t* arrived;
  uint32_t tiles;  // of the workgroup
  unsigned long long tag;
  unsigned long long* word;
  __device__ __forceinline__ void tell(uint32_t found) const {
    if (lane_id() == 0) {
      const uint32_t before = atomicAdd(arrived, 1u << 24 | found);
      if ((before >> 24) + 1u == tiles)
        __hip_atomic_store(word, tag | ((before & 0xFFFFFFu) + found), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
};
__device__ __forceinline__ void all_found(const ShortSink& sink, uint32_t found) { sink.tell(found); }

// Which of a tile's elements are outliers, once more from the source: how many, and those below `limit` to the stream.
template <int MODE, int E, bool WHOLE>
__device__ __forceinline__ uint32_t select_tile(const TensorDesc& d, uint32_t tile, uint32_t pos, uint32_t limit) {
  uint32_t raw[E][4];
  load_tile<E, false>(d, tile, raw);
  const TileGeo<E> g = tile_geo<E, false>(d, tile);
  blank_tail<E>(g, raw);
  return encode_tile<MODE, 8, false, E, false, WHOLE, false>(d, g, raw, tile, StreamSink{d.idx, d.val}, pos, limit);
}

// a1 .. a8 of a tile, its outliers to the wavefront's record
template <int MODE, int BITS, bool ASYM, int E, bool WHOLE>
__device__ __forceinline__ uint32_t short_tile(const TensorDesc& d, uint32_t tile, const ShortSink& sink) {
  uint32_t raw[E][4];
  load_tile<E, WHOLE>(d, tile, raw);
  const TileGeo<E> g = tile_geo<E, WHOLE>(d, tile);
  if constexpr (!WHOLE) blank_tail<E>(g, raw);
  return encode_tile<MODE, BITS, ASYM, E, false, WHOLE, true>(d, g, raw, tile, sink, 0u, (uint32_t)kSlot);
}

// What workgroup `i` has published of this launch: true, and the count, or false.
__device__ __forceinline__ bool look(const unsigned long long* words, uint32_t i, unsigned long long tag, uint32_t& count) {
  const unsigned long long w = __hip_atomic_load(words + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  count = (uint32_t)(w - tag);
  return w >> kShortCountBits == tag >> kShortCountBits;
}

// The outliers in the tiles of the first `n` workgroups, to every thread.  The patience is that of a wavefront for the whole wait; when it is at
// an end, all words are looked at once more, and what is missing is counted here and published for all: it is the number that
// the workgroup itself will publish.  Waiting workgroups begin at different words, so that they share the missing ones among them.
template <int MODE, int E, bool WHOLE>
__device__ __forceinline__ uint32_t outliers_of_others(const TensorDesc& d, uint32_t n, unsigned long long tag, uint32_t patience,
                                                       unsigned long long* words, uint32_t (&part)[kWavesPerWg]) {
  uint32_t sum = 0u, looks = 0u;
  for (uint32_t i0 = 0u; i0 < n; i0 += (uint32_t)kThreads) {  // uniform
    const uint32_t i = i0 + threadIdx.x;
    bool open = i < n;
    uint64_t left = __builtin_amdgcn_ballot_w64(open);
    for (bool first = true; left != 0ull && (first || looks < patience); first = false, ++looks) {  // uniform
      if (!first) __builtin_amdgcn_s_sleep(1);
      uint32_t count;
      if (open && look(words, i, tag, count)) {
        sum += count;
        open = false;
      }
      left = __builtin_amdgcn_ballot_w64(open);
    }
    while (__builtin_expect(left != 0ull, 0)) {  // uniform
      const uint32_t begin = blockIdx.x % (uint32_t)kWave;
      const uint64_t behind = left >> begin << begin;
      const uint32_t lane = (uint32_t)__builtin_ctzll(behind != 0ull ? behind : left);
      left &= ~(1ull << lane);
      const uint32_t g = (uint32_t)__builtin_amdgcn_readlane((int)i, (int)lane);
      uint32_t found;
      if (__builtin_amdgcn_ballot_w64(!look(words, g, tag, found)) != 0ull) {  // uniform
        found = 0u;
        for (uint32_t t = g * (uint32_t)kWavesPerWg; t < (g + 1u) * (uint32_t)kWavesPerWg && t < d.n_tiles; ++t)
          found += select_tile<MODE, E, WHOLE>(d, t, 0u, 0u);
        if (lane_id() == 0) __hip_atomic_store(words + g, tag | found, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if ((uint32_t)lane_id() == lane) sum += found;
    }
  }
  return block_sum_u32<kWavesPerWg>(sum, part);
}

// The fallback's registers are what bounds it; a short tensor does not fill the device anyway.
template <int MODE, int E, bool WHOLE>
__global__ __launch_bounds__(kThreads, 4) void compress_short_kernel(TensorDesc d, unsigned long long tag, unsigned long long* words, uint32_t patience) {
  __shared__ union {
    ShortShared tiles;
    struct {
      uint32_t part[kWavesPerWg];
      __attribute__((aligned(16))) unsigned char rest[kTailLdsBytes];
    } tail;
  } lds;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t tile = blockIdx.x * kWavesPerWg + wave;
  const uint32_t workgroups = (d.n_tiles + (uint32_t)kWavesPerWg - 1u) / (uint32_t)kWavesPerWg;
  if (blockIdx.x == workgroups) {  // the end that the groups do not divide
    compress_tail<false>(d, [&] {
      return outliers_of_others<MODE, E, WHOLE>(d, workgroups, tag, patience, words, lds.tail.part);
    }, lds.tail.rest);
    return;
  }
  if (threadIdx.x == 0u) lds.tiles.arrived = 0u;
  __syncthreads();
  uint32_t found = 0u;
  if (tile < d.n_tiles) {  // uniform
    const uint32_t tiles = d.n_tiles - blockIdx.x * (uint32_t)kWavesPerWg;
    const ShortSink record{{lds.tiles.record[wave], tile * (uint32_t)(E * kRow)}, &lds.tiles.arrived,
                           tiles < (uint32_t)kWavesPerWg ? tiles : (uint32_t)kWavesPerWg, tag, words + blockIdx.x};
    if constexpr (!WHOLE) {  // (the codes' form is looked at behind the selection)
      found = short_tile<MODE, kBitsAny, false, E, false>(d, tile, record);
    } else {
      switch (d.variant & 6u) {
        case 0: found = short_tile<MODE, 4, false, E, WHOLE>(d, tile, record); break;
        case 2: found = short_tile<MODE, 4, true, E, WHOLE>(d, tile, record); break;
        case 4: found = short_tile<MODE, 8, false, E, WHOLE>(d, tile, record); break;
        default: found = short_tile<MODE, 8, true, E, WHOLE>(d, tile, record); break;
      }
    }
  }
  if (lane == 0u) lds.tiles.count[wave] = found;
  __syncthreads();
  uint32_t before = 0u;
#pragma unroll
  for (uint32_t w = 0; w < (uint32_t)kWavesPerWg; ++w) before += w < wave ? lds.tiles.count[w] : 0u;
  const uint32_t pos = before + outliers_of_others<MODE, E, WHOLE>(d, blockIdx.x, tag, patience, words, lds.tiles.part);
  if (tile >= d.n_tiles) return;
  if (lane == 0u) {
    d.tile_ptr[tile] = pos;
    if (tile + 1u == d.n_tiles) {  // the blob's last tile closes it, unless elements behind it still have to be added
      const uint32_t n_out = pos + found;
      if (d.n_tiles_all > d.n_tiles || d.tail == 0u) d.tile_ptr[d.n_tiles] = n_out;
      if (d.tail == 0u) { d.status[0] = n_out; d.status[1] = n_out > d.cap ? 1u : 0u; d.status[2] = 0u; d.status[3] = 0u; }
    }
  }
  if (found <= (uint32_t)kSlot) {  // uniform
    if (lane < found && pos + lane < d.cap) {
      const uint32_t r = lds.tiles.record[wave][lane];
      d.idx[pos + lane] = (int32_t)(tile * (uint32_t)(E * kRow) + (r >> 16));
      d.val[pos + lane] = (uint16_t)r;
    }
  } else {
    const uint32_t end = pos + found;
    select_tile<MODE, E, WHOLE>(d, tile, pos, end < d.cap ? end : d.cap);
  }
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
