// The kernels that place the outliers in the stream (single tensor and batch): a workgroup per kPlaceTiles (kSumTiles) tiles
// of one tensor, whatever the method (the choice of the selection code for tiles that have to be looked at again is a uniform
// switch), and one more for the end of a tensor that its groups do not divide.
#include "adacc_kernels.hpp"
#include "adacc_tail.hpp"

namespace adacc {
namespace ADACC_DT_NS {

template <int WAVES, bool LIST>
union PlaceLds {  // a workgroup places tiles or does the tensor's end
  typedef typename std::conditional<LIST, PlaceListShared, PlaceShared<WAVES>>::type Place;
  Place place;
  __attribute__((aligned(16))) unsigned char tail[(sizeof(PlaceShared<WAVES>) + 15) / 16 * 16 + kTailLdsBytes];
};

// block: of kPlaceTiles tiles (kSumTiles of a long tensor), or the one behind the last: the tensor's end
// WAVES: of the workgroup.  WIDE: blocks of kSumTiles tiles too.  TOPK: tensors of that mode too
template <int WAVES, bool WIDE, bool TOPK>
__device__ __forceinline__ void place_dispatch(const TensorDesc& d, uint32_t block, uint32_t epoch, PlaceLds<WAVES, WIDE>& lds) {
  const bool from_sums = d.from_sums != 0u;
  const bool topk = TOPK && d.mode == kModeTopk;
  // TOPK: regular counts everywhere (the usual case): the compression kernel has placed everything already
  const bool regular = topk && __hip_atomic_load(d.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch;
  const bool wide = WIDE && d.place_per == (uint32_t)kSumTiles;
  const uint32_t per = wide ? (uint32_t)kSumTiles : (uint32_t)kPlaceTiles;
  const uint32_t blocks = (d.n_tiles + per - 1u) / per;
  if (block >= blocks) {
    if (d.tail == 0u || block != blocks) return;
    // the counts of all tiles are asked for together with the elements, by every wavefront (their sums go through the words before lds.tail's)
    compress_tail<true>(d, [&] {
      return regular ? d.topk * (uint32_t)(d.numel >> d.lgs) : outliers_before<WAVES>(d, d.n_tiles, from_sums, lds.place);
    }, lds.tail + (sizeof(PlaceShared<WAVES>) + 15) / 16 * 16);
    return;
  }
  if (regular) return;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  PlacedTiles p;
  if constexpr (WIDE) {
    p = wide ? place_tiles<kSumTiles, WAVES>(d, block * per, per, false, 0u, from_sums, !topk, lds.place)
             : place_tiles<kPlaceTiles, WAVES>(d, block * per, per, false, 0u, false, !topk, lds.place);
  } else {
    p = place_tiles<kPlaceTiles, WAVES>(d, block * per, per, false, 0u, false, !topk, lds.place);
  }
  const uint32_t room = topk ? 0u : (uint32_t)kSlot;
  if (__builtin_amdgcn_ballot_w64(p.count > room) == 0ull) return;  // the usual case: every tile is in its slot
  const uint32_t j = wide ? 0u : wave, step = wide ? 1u : (uint32_t)WAVES;
  const bool e8 = (d.variant & 1u) != 0u;
  switch (d.variant >> 3) {
    case kModeAbs:
      if (d.rowwise) reselect_tiles<kModeAbs, 4, true, false>(d, p, room, j, step);
      else if (e8) reselect_tiles<kModeAbs, 8, false, false>(d, p, room, j, step);
      else reselect_tiles<kModeAbs, 4, false, false>(d, p, room, j, step);
      break;
    case kModeStd:
      if (d.rowwise) reselect_tiles<kModeStd, 4, true, false>(d, p, room, j, step);
      else if (e8) reselect_tiles<kModeStd, 8, false, false>(d, p, room, j, step);
      else reselect_tiles<kModeStd, 4, false, false>(d, p, room, j, step);
      break;
    case kModeTopk:
      if constexpr (TOPK) {
        if (topk_whole(d)) {
          if (e8) reselect_tiles<kModeTopk, 8, false, true>(d, p, room, j, step);
          else reselect_tiles<kModeTopk, 4, false, true>(d, p, room, j, step);
        } else {
          if (e8) reselect_tiles<kModeTopk, 8, false, false>(d, p, room, j, step);
          else reselect_tiles<kModeTopk, 4, false, false>(d, p, room, j, step);
        }
      }
      break;
    default: break;
  }
}

// single tensor: blockIdx.x is the block of tiles
__global__ __launch_bounds__(kPlaceThreads) void place_sum_kernel(TensorDesc d) {
  __shared__ PlaceShared<kPlaceThreads / kWave> sh;
  place_sum_block(d, blockIdx.x, sh);
}

// The selection code for tiles that have to be looked at again would take 173 registers and leave room
// for two wavefronts per SIMD; the kernel is a chain of dependent memory round trips, so it is held to 128.
__global__ __launch_bounds__(kPlaceThreads, 4) void place_kernel(TensorDesc d, uint32_t epoch) {
  constexpr int WAVES = kPlaceThreads / kWave;
  __shared__ PlaceLds<WAVES, true> lds;
  place_dispatch<WAVES, true, true>(d, blockIdx.x, epoch, lds);
}
// ABS and STD up to kPlaceManyTiles tiles: sixteen wavefronts to a workgroup's 64 tiles, so that those whose slot is too
// small are selected again four after the other and not sixteen, each of them a load from memory and some 600 instructions
// by a wavefront alone.  ([8192, 4096] int8, the placement: STD at 3 sigma over groups of 64 of GELU values, every tile with more
// than 64 outliers, 50.4 -> 25.4 us; over 512 of SiLU values 41.8 -> 20.8.  Where no tile has that many, both ways: [16000, 1024] STD at 6
// sigma over 1024 26.4 -> 25.6, [14000, 2051] at 4 sigma over 512 40.7 -> 40.3.)  Where this launch as a rule finds nothing to do, TOPK among
// others, the smaller workgroups stay (place_many).
__global__ __launch_bounds__(kPlaceManyThreads) void place_many_kernel(TensorDesc d, uint32_t epoch) {
  constexpr int WAVES = kPlaceManyThreads / kWave;
  __shared__ PlaceLds<WAVES, false> lds;
  place_dispatch<WAVES, false, false>(d, blockIdx.x, epoch, lds);
}

// a group of tensors of a table: blockIdx.y picks the tensor, blockIdx.x its block of tiles
__global__ __launch_bounds__(kPlaceThreads) void place_sum_batch_kernel(const TensorDesc* table, const uint32_t* members) {
  __shared__ PlaceShared<kPlaceThreads / kWave> sh;
  const TensorDesc d = table[members[blockIdx.y]];
  if (blockIdx.x < (d.n_tiles + (uint32_t)kSumTiles - 1u) / (uint32_t)kSumTiles) place_sum_block(d, blockIdx.x, sh);
}

__global__ __launch_bounds__(kPlaceThreads, 4) void place_batch_kernel(const TensorDesc* table, const uint32_t* members,
                                                                    uint32_t epoch) {
  constexpr int WAVES = kPlaceThreads / kWave;
  __shared__ PlaceLds<WAVES, true> lds;
  const TensorDesc d = table[members[blockIdx.y]];
  place_dispatch<WAVES, true, true>(d, blockIdx.x, epoch, lds);
}

PlaceSumFn place_sum_fn() { return place_sum_kernel; }
PlaceFn place_fn(bool many) { return many ? place_many_kernel : place_kernel; }
PlaceSumBatchFn place_sum_batch_fn() { return place_sum_batch_kernel; }
PlaceBatchFn place_batch_fn() { return place_batch_kernel; }

}  // namespace ADACC_DT_NS
}  // namespace adacc
