// Kernel templates of libadacc.  Included by the translation units that instantiate them
// (one per outlier mode, one for decompression, one per batch kernel), so that the library builds
// in parallel; the host code reaches the instantiations through the getters of adacc_fn.hpp.
#pragma once

#include "adacc_common.hpp"
#include "adacc_compress.hpp"
#include "adacc_decompress.hpp"
#include "adacc_fn.hpp"

namespace adacc {
namespace ADACC_DT_NS {

// ---- single tensor, compress: tiles are independent, one tile per wavefront, workgroups in the
// hardware's own order (which walks through memory front to back).
// Wavefronts per SIMD the register allocation of a variant is held to, as many as do without a spill (the compiler would
// otherwise spend registers on overlapping the rows of a tile, which pays less than another resident wavefront).
template <int MODE, bool ASYM, int E, bool WHOLE>
constexpr int compress_min_waves() {
  if (E == 4) return 8;
  if (WHOLE) return 6;
  return (ASYM ? 4 : 5) - (MODE == (int)kModeTopk ? 1 : 0);
}
template <int MODE, int BITS, bool ASYM, int E, bool ROWWISE, bool WHOLE = false>
__global__ __launch_bounds__(kThreads, (compress_min_waves<MODE, ASYM, E, WHOLE>())) void compress_kernel(TensorDesc d, uint32_t epoch) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform, and the compiler shall know it
  // one tile per wavefront and no loop: inside a loop over tiles the compiler would prepare, ahead of
  // the loop, the lane's addresses for every group size the encoders can be asked for
  const uint32_t t = blockIdx.x * kWavesPerWg + wave;
  if (t >= d.n_tiles) {
    if constexpr (MODE == kModeNone) {
      if (t == d.n_tiles && d.tail != 0u) compress_plain_tail<BITS, ASYM>(d);
    }
    return;
  }
  if constexpr (MODE == kModeNone) compress_tile_plain<BITS, ASYM, E, ROWWISE>(d, t);
  else compress_tile_outliers<MODE, BITS, ASYM, E, ROWWISE, WHOLE>(d, t, epoch);
}

// TOPK whose statistics group is the whole tile, with quantisation groups inside a row, has an encoder of its own
__device__ __forceinline__ bool topk_whole(const TensorDesc& d) { return d.lgs == d.lgt && d.lgq <= 9u; }

// d.n_tiles counts pieces here
template <int BITS, bool ASYM, bool F32, bool GENERIC, int ROWS>
__global__ __launch_bounds__(piece_waves(ROWS) * kWave) void decompress_kernel(TensorDesc d, uint32_t has_outliers) {
  constexpr int WAVES = piece_waves(ROWS);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform, and the compiler shall know it
  __shared__ DecompressShared<F32, ROWS, WAVES> shared;
  const uint32_t piece = blockIdx.x * (uint32_t)WAVES + wave;  // (no loop over pieces: it would cost 20 registers)
  // what the first loads need is asked for together with n_tiles, one round trip to the kernel's arguments instead of two
  // (2^25 values of int8 codes: 15.3 -> 15.1 us from a blob in the caches, 15.7 -> 15.5 from memory)
  asm volatile("" ::"s"(d.codes), "s"(d.scales), "s"(d.zp), "s"(d.dst), "s"(d.numel), "s"(d.lgq));
  if (piece < d.n_tiles) decompress_piece<BITS, ASYM, F32, GENERIC, ROWS, WAVES>(d, piece, has_outliers != 0u, shared);
}

// ---- batch
// One launch for a group of tensors of a table: blockIdx.y picks the tensor, blockIdx.x its tiles, four per workgroup; workgroups past the end of a
// shorter tensor leave at once.  The host groups the tensors by kernel and by size (tile counts
// within a factor of two), so few workgroups are empty; within a launch the hardware goes through
// the tensors one after the other, front to back.
// A kernel holds as many wavefronts per SIMD as its heaviest variant allows, so the variants come
// in five kernels by weight:
//   kBatchRows4   tiles of 4 rows, all groups inside a row (TOPK: over the quantisation groups)   lightest
//   kBatchAny4    tiles of 4 rows, any other grouping
//   kBatchTopk4   tiles of 4 rows, TOPK over the whole tile, quantisation groups inside a row
//   kBatchAny8    tiles of 8 rows, general encoder                                   heaviest
//   kBatchTopk8   tiles of 8 rows, TOPK over the whole tile, quantisation groups inside a row

template <int MODE, int E, bool ROWWISE, bool WHOLE>
__device__ __forceinline__ void compress_dispatch(const TensorDesc& d, uint32_t tile, uint32_t epoch) {
  if constexpr (!ROWWISE && !WHOLE) {  // (the codes' form is looked at behind the selection)
    if constexpr (MODE == kModeNone) compress_tile_plain<kBitsAny, false, E, false>(d, tile);
    else compress_tile_outliers<MODE, kBitsAny, false, E, false>(d, tile, epoch);
  } else if constexpr (MODE == kModeNone) {
    switch (d.variant & 6u) {
      case 0: compress_tile_plain<4, false, E, ROWWISE>(d, tile); break;
      case 2: compress_tile_plain<4, true, E, ROWWISE>(d, tile); break;
      case 4: compress_tile_plain<8, false, E, ROWWISE>(d, tile); break;
      default: compress_tile_plain<8, true, E, ROWWISE>(d, tile); break;
    }
  } else {
    switch (d.variant & 6u) {
      case 0: compress_tile_outliers<MODE, 4, false, E, ROWWISE, WHOLE>(d, tile, epoch); break;
      case 2: compress_tile_outliers<MODE, 4, true, E, ROWWISE, WHOLE>(d, tile, epoch); break;
      case 4: compress_tile_outliers<MODE, 8, false, E, ROWWISE, WHOLE>(d, tile, epoch); break;
      default: compress_tile_outliers<MODE, 8, true, E, ROWWISE, WHOLE>(d, tile, epoch); break;
    }
  }
}

template <int KIND>
constexpr int batch_min_waves() {
  return KIND == kBatchAny8 ? 3 : KIND == kBatchTopk8 ? 6 : KIND == kBatchTopk4 ? 8 : 7;
}

template <int KIND>
__global__ __launch_bounds__(kThreads, (batch_min_waves<KIND>())) void compress_batch_kernel(const TensorDesc* table, uint32_t epoch) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform, and the compiler shall know it
  // the group's entries are table[0 .. gridDim.y) themselves (the host lays the table out in the order of these
  // launches): no list of members to look up before the wavefront's first load
  const TensorDesc d = table[blockIdx.y];
  const uint32_t tile = blockIdx.x * kWavesPerWg + wave;
  if (tile >= d.n_tiles) {
    if (tile == d.n_tiles && d.tail != 0u && d.variant >> 3 == kModeNone) {  // the end of a tensor without outliers
      switch (d.variant & 6u) {
        case 0: compress_plain_tail<4, false>(d); break;
        case 2: compress_plain_tail<4, true>(d); break;
        case 4: compress_plain_tail<8, false>(d); break;
        default: compress_plain_tail<8, true>(d); break;
      }
    }
    return;
  }
  constexpr int E = (KIND == kBatchAny8 || KIND == kBatchTopk8) ? 8 : 4;
  if constexpr (KIND == kBatchTopk4 || KIND == kBatchTopk8) {
    compress_dispatch<kModeTopk, E, false, true>(d, tile, epoch);
  } else {
    constexpr bool ROWWISE = KIND == kBatchRows4;
    switch (d.variant >> 3) {
      case kModeNone: compress_dispatch<kModeNone, E, ROWWISE, false>(d, tile, epoch); break;
      case kModeAbs: compress_dispatch<kModeAbs, E, ROWWISE, false>(d, tile, epoch); break;
      case kModeStd: compress_dispatch<kModeStd, E, ROWWISE, false>(d, tile, epoch); break;
      default: compress_dispatch<kModeTopk, E, ROWWISE, false>(d, tile, epoch); break;
    }
  }
}

// Batch decompression: the same grouping, over the 2048-element pieces of the tensors.
// The group's entries are table[0 .. gridDim.y) themselves here too.
template <bool F32>
__global__ __launch_bounds__(kThreads) void decompress_batch_kernel(const TensorDesc* table) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform, and the compiler shall know it
  const TensorDesc d = table[blockIdx.y];
  const uint32_t piece = blockIdx.x * kWavesPerWg + wave;
  // all of the descriptor that a piece needs is asked for together with n_tiles: one round trip to memory ahead of the
  // first load of the codes, where a wait for n_tiles alone would make it two
  asm volatile("" ::"s"(d.codes), "s"(d.scales), "s"(d.zp), "s"(d.dst), "s"(d.numel), "s"(d.lgq), "s"(d.variant), "s"(d.tile_ptr),
               "s"(d.idx), "s"(d.val), "s"(d.cap), "s"(d.per_tile), "s"(d.mode), "s"(d.ptr_shift));
  if (piece >= d.n_tiles) return;
  const bool ho = (d.variant >> 3) != kModeNone;
  constexpr int ROWS = (int)full_piece_rows(F32);
  __shared__ DecompressShared<F32, ROWS, kWavesPerWg> shared;
  switch (d.variant & 6u) {
    case 0: decompress_piece<4, false, F32, false, ROWS, kWavesPerWg>(d, piece, ho, shared); break;
    case 2: decompress_piece<4, true, F32, false, ROWS, kWavesPerWg>(d, piece, ho, shared); break;
    case 4: decompress_piece<8, false, F32, false, ROWS, kWavesPerWg>(d, piece, ho, shared); break;
    default: decompress_piece<8, true, F32, false, ROWS, kWavesPerWg>(d, piece, ho, shared); break;
  }
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
