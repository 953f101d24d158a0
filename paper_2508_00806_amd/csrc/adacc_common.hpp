// Shared device/host definitions of libadacc (gfx950 only).
//
// Work decomposition used by every kernel here:
//   - a lane owns one "octet": 8 consecutive bf16 elements = one 16-byte load;
//   - a wavefront (64 lanes) covers one "row" of 512 consecutive elements per load
//     instruction, fully coalesced (1 KiB);
//   - a tile is E rows (E = 4 or 8, i.e. 2048 or 4096 elements) and belongs to ONE
//     wavefront; every statistics / quantisation group lies inside one tile, so all
//     reductions are wavefront-local, and a workgroup is just 4 independent wavefronts.
// (The tile and piece kernels; the placement, the fallback kernels and the statistics passes of the channel schemes
// share work over a workgroup, with barriers.)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace adacc {

constexpr int kWave = 64;
constexpr int kOct = 8;               // elements per lane per row
constexpr int kRow = kWave * kOct;    // 512 elements
constexpr int kWavesPerWg = 4;
constexpr int kThreads = kWave * kWavesPerWg;

// Streaming accesses: data that is read or written once and not again by the same launch.  The
// non-temporal hint keeps such lines from being retained by the caches on their way; on this part a
// pure read stream runs about a third faster with it.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 load_stream16(const void* p) {
  const u32x4_t t = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(p));
  return make_uint4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void store_stream16(void* p, uint4 v) {
  u32x4_t t = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(t, reinterpret_cast<u32x4_t*>(p));
}
__device__ __forceinline__ void store_stream8(void* p, uint2 v) {
  u32x2_t t = {v.x, v.y};
  __builtin_nontemporal_store(t, reinterpret_cast<u32x2_t*>(p));
}
__device__ __forceinline__ void store_stream4(void* p, uint32_t v) {
  __builtin_nontemporal_store(v, reinterpret_cast<uint32_t*>(p));
}

// The tensor streams of the compression / decompression kernels go through these (ADACC_NO_STREAM_HINT
// builds the plain accesses, for comparison).  The codes a decompression reads stay plain loads: on a
// blob that was written shortly before they are served by the caches, and the hint made that slower.
#ifndef ADACC_NO_STREAM_HINT
#define ADACC_LOAD16(p) load_stream16(p)
#define ADACC_STORE16(p, v) store_stream16((p), (v))
#define ADACC_STORE8(p, v) store_stream8((p), (v))
#define ADACC_STORE4(p, v) store_stream4((p), (v))
#else
#define ADACC_LOAD16(p) (*reinterpret_cast<const uint4*>(p))
#define ADACC_STORE16(p, v) (*reinterpret_cast<uint4*>(p) = (v))
#define ADACC_STORE8(p, v) (*reinterpret_cast<uint2*>(p) = (v))
#define ADACC_STORE4(p, v) (*reinterpret_cast<uint32_t*>(p) = (v))
#endif

// The statistics pass of the two-pass schemes reads what the second pass reads again: for a tensor that the
// Infinity Cache can hold a good part of, it leaves the lines to the caches (plain loads); for a larger one
// nothing would survive until the second pass, and it streams like every other pass (STREAM).
constexpr uint64_t kStatsKeepBytes = 128ull << 20;
template <bool STREAM>
__device__ __forceinline__ uint4 load_stats16(const void* p) {
  if constexpr (STREAM) return load_stream16(p);
  else return *reinterpret_cast<const uint4*>(p);
}

enum : uint32_t { kModeNone = 0, kModeAbs = 1, kModeStd = 2, kModeTopk = 3 };

// One tensor as the kernels see it.  Passed by value for single-tensor launches
// and read from a device table for batch launches.
struct TensorDesc {
  const uint16_t* src;  // compress: bf16 input
  void* dst;            // decompress: output
  uint8_t* codes;
  float* scales;
  float* zp;
  uint32_t* tile_ptr;
  int32_t* idx;
  uint16_t* val;
  uint32_t* status;
  uint32_t* cnt;            // compress, workspace: outliers found in every tile
  uint32_t* block_sum;      // compress, workspace (ABS / STD): outliers in every block of kSumTiles tiles
  uint32_t* slot;           // compress, workspace (ABS / STD): kSlot records (number in the tile << 16 | value) per
                            //   tile, the tile's outliers until the placement kernel has moved them to the stream
  uint32_t* flag;           // compress, workspace (TOPK): set to the epoch by a tile whose count is not the regular one
  uint64_t numel;           // compress: elements the tile kernels take, the whole groups of the larger kind; decompress: all
  uint64_t magic_q, magic_t;  // decompress, fallback: ceil(2^64 / n) for the octets of a quantisation group resp. a tile (0: n = 1)
  float recip_q;            // decompress, fallback: 1 / octets of a quantisation group, moved up (see group_of)
  uint32_t per_tile;        // decompress, TOPK: outliers of a regular tile
  uint32_t tail;            // compress: elements after numel (fewer than the larger group): one short group
  uint32_t n_tiles;         // tiles of the first numel elements (decompress: pieces of 2048 of them)
  uint32_t n_tiles_all;     // tiles of the whole tensor, tail included: tile_ptr has one entry more
  uint32_t bits, asym, mode;  // the method, for kernels that do not get it as template arguments
  uint32_t gq, gs;          // group sizes as numbers (the fallback kernels take groups that are no powers of two)
  uint32_t tile_elems;      // elements per tile of the blob
  uint32_t generic;         // 1: the method goes through the fallback kernels
  uint32_t from_sums;       // compress: 1 = the placement starts from block_sum (a kernel of its own forms them)
  uint32_t place_per;       // compress: tiles (fallback: segments) that a workgroup of the placement takes
  uint32_t lgt;             // log2(elements per tile): 11 or 12
  uint32_t lgq;         // log2(quant group)
  uint32_t lgs;         // log2(stat group) (STD / TOPK)
  uint32_t cap;         // capacity of idx / val
  uint32_t topk;
  float param;          // ABS: tau.  STD: k*k
  float divisor;        // D of Eq. 2 resp. Eq. 3 (2^(b-1), 2^b, or one less)
  float inv_divisor;    // 1/D when D is a power of two (the paper's rule), else 0
  uint32_t pow2_divisor;  // 1 when D is a power of two
  uint32_t rowwise;     // compress: 1 = every group lies inside a row (row-at-a-time encoder)
  uint32_t variant;     // index into the instantiation table
  uint32_t ptr_shift;   // decompress: works on pieces of 2048 elements or fewer; piece u belongs to tile u >> ptr_shift
};

// Outlier channels (Section 3.2, Eq. 1): what those kernels need beside the TensorDesc of the quantised part.
constexpr uint32_t kChunkTokens = 64;  // tokens per binary32 partial sum of the channel statistics
constexpr uint32_t kPartialWaves = 16;  // wavefronts that share a chunk in the statistics pass (one workgroup)
constexpr uint32_t kPartialRows = kChunkTokens / kPartialWaves;  // tokens per wavefront there
// Up to this many chunks and channels the selection adds the chunk sums up itself and their kernel is left out: one workgroup takes
// that on where it costs less than a launch.  (us both ways with that kernel / without, int4, 128, 256 and 512 tokens: 1024 channels 16.6 /
// 15.4, 16.8 / 15.9, 16.8 / 17.4; 4096 channels 17.6 / 16.4, 17.7 / 16.8, 18.4 / 19.1; 8192 19.3 / 17.9, 19.8 / 18.8, 21.9 / 23.0.)
constexpr uint32_t kFewChunks = 4, kFewHidden = 8192;
struct ChannelDesc {
  uint8_t* mask;        // hidden/8 bytes: bit (h & 7) of byte h >> 3 is set for an outlier channel
  uint32_t* base;       // hidden/8 words: number of outlier channels below channel 8 * (h >> 3)
  int32_t* ch_idx;      // the outlier channels, ascending
  uint16_t* ch_val;     // [tokens][n_ch] bf16 bit patterns
  uint32_t* status;     // [0] n_ch, [1] 1 if n_ch > max_channels
  uint32_t hidden;
  uint32_t tokens;
  uint32_t max_channels;
  float z_thresh;
  float inv_hidden;     // 1 / hidden rounded towards zero twice: never above the true reciprocal
};

// Channel-wise symmetric quantisation (Section 3.2, the Query / Key / Value scheme): one scale per channel.
struct ChannelwiseDesc {
  const uint16_t* src;  // compress: bf16 input [tokens][hidden]
  void* dst;            // decompress: output
  uint8_t* codes;
  float* scales;        // [hidden], S_h of Eq. 2
  float* inv;           // workspace [hidden]: D / max_h
  uint16_t* partial;    // workspace [n_chunks][hidden]: chunk maxima of the finite magnitudes
  uint64_t numel;
  uint32_t tokens, hidden, n_chunks;
  uint32_t strip_rows;   // decompress: tokens a wavefront takes
  float divisor, inv_divisor;  // D of Eq. 2 and, when D is a power of two, 1/D (else 0)
};

// The piece of a tensor that a wavefront restores: rows of 64 chunks of 8 elements (of 4 where the output is binary32), 2048 elements
// as a rule.  Fewer in long tensors, where what all wavefronts write at a time lies closer together; a wavefront of a
// piece looks through all outliers of its tile.  (us of a pass both ways.  Binary32, with outliers, 8 rows / 4 / 2: STD over 4096 at 4
// sigma, 2^25 values 56.8 / 56.4 / 60.6, 2^27 189 / 177 / 201; the 4 largest of 4096, 2^27, 164 / 158 / 172; two in a hundred outliers, 2^27,
// 338 / 329 / 350; below 2^25 equal or slower, 2^24 31.5 / 32.1 / 34.5.  Binary32 without, 2^25 int8 47.8 / 47.5 / 46.0, 2^27 177 / 182 / 168,
// int4 160 / 166 / 155; 2^24 25.6 / 26.2 / 26.0.  16 bits without outliers, 4 rows / 2: 2^25 int8 36.2 / 36.6, 2^26 int4 58.4 / 57.2, 2^28 222 / 218
// and int8 256 / 254; with ABS or STD: 2^27 142.6 / 141.3 and, two in a hundred outliers, 285 / 288, 2^28 270 / 265 and 444 / 447, 2^29 533 /
// 517; TOPK equal.)
constexpr uint32_t full_piece_rows(bool f32) { return f32 ? 8u : 4u; }
// wavefronts of a workgroup (two rows: with four, 2^28 values int8 256.1 where two take 253.2)
constexpr int piece_waves(int rows) { return rows == 2 ? 2 : kWavesPerWg; }

// The mask kernels: 16-byte pieces of the byte format that a lane has in flight, one after the other 4 KiB apart.  (us both ways with
// 8 / 6 / 4 / 2: 268 M elements 99.1 / 98.2 / 92.2 / 95.7, 134 M 50.9 / 51.1 / 49.4 / 50.7, 64 M 23.8 / 24.0 / 23.7 / 23.6, 34 M 13.6 /
// 13.8 / 13.0 / 13.4: with more in flight a wavefront writes further apart from its neighbours.)
constexpr int kMaskAhead = 4;

// Outliers of a tile that travel through the tile's slot in the workspace (ABS / STD); a tile with
// more is selected a second time by the placement kernel.
constexpr int kSlot = 64;
// The placement kernels: a workgroup of kPlaceThreads threads takes kPlaceTiles consecutive tiles, one of kPlaceManyThreads where
// its wavefronts have something to share (ABS / STD, adacc_k_place.hip).
constexpr int kPlaceThreads = 256;
constexpr int kPlaceManyThreads = 1024;
constexpr int kPlaceTiles = 64;
// Of the fallback kernels' segments, which the whole workgroup selects again where a slot does not do, one after the
// other, it takes 1, 2, 4, .. kPlaceSegments: the fewest with which kPlaceWorkgroups workgroups, as many as the device
// holds at once, are enough.  (Always 16, at half the wavefronts: 128 rows of 11008 values with some 94 outliers each
// 113 us, 1024 of them 126 and 8192 of them 201; 19, 27 and 146 us like this.)  TOPK, where only values that are not
// finite make the placement do anything, and then all segments go through it: four times the workgroups for short
// segments, of which a CU holds twice as many and which leave at once in every other call (0.6 us for 4096 of them);
// and several times 16 segments rather than more workgroups, because it has no block sums: every workgroup adds up all
// counts before its own.  (67 M values in groups of 24, one of them with 33 infinities: 619 us, 427 us like this.)
constexpr int kPlaceSegments = 16;
constexpr uint32_t kPlaceWorkgroups = 1024;
// In a tensor of more tiles than this a workgroup of the placement takes kSumTiles of them, and the counts are added up in
// blocks of that many first, in a kernel of its own (ABS / STD: TOPK, whose placement does nothing in ordinary calls, has
// none).  Below, and for TOPK, every workgroup adds up all counts before its own: at most four rounds of eight loads of
// 16 bytes per thread up to this many tiles, about as long as that launch (4.5 us).  (Blocks of 64 tiles behind the sums:
// 524288 tiles with an outlier each take 24.6 us, 8192 workgroups of which a CU holds four; blocks of 256 10.8 us, where a
// thread per record and a bisection took 14.1.  TOPK of 1000000 tiles, one of them irregular, with 64 to a workgroup: 2.53
// ms, most of it counts that 15625 workgroups add up; with 256 1.80.)
constexpr int kSumTiles = 256;
constexpr uint32_t kPlaceDirectTiles = 32768;
// Up to this many tiles by sixteen wavefronts to a workgroup (adacc_k_place.hip).  (us both ways by four / sixteen: [16000, 4096], 16000 tiles,
// 71.1 / 69.9; [79977, 512] of softmax values, 19995 tiles of 13 outliers, 57.9 / 58.7.)
constexpr uint32_t kPlaceManyTiles = 16384;
// The workspace's launch counter ("epoch", kept on the host in adacc_workspace) marks what a launch
// wrote: a word that holds an older epoch reads as not set, so nothing has to be cleared per call.
constexpr uint32_t kEpochMax = 0x3FFFFFFFu;
// Tensors of at most this many workgroups of tiles (and one for the end) are compressed in one launch (adacc_short.hpp), a word of
// 8 bytes for each at the end of a workspace that has the room: with an end that the groups do not divide, without, methods that have
// the encoder by rows in two launches, TOPK.  The lines lie where the wait for the other workgroups begins to cost as much as the
// second launch.  (us both ways, two launches / one.  [rows, 1024] STD at 6 sigma over 1024: 20 rows 9.8 / 7.9, 128 10.3 / 8.2, 1024 11.0 /
// 8.6, 4096 13.4 / 11.1, 8000 16.9 / 15.6, 12000 20.5 / 19.8, 16000 24.9 / 25.4.  [rows, 2051] at 4 sigma over 512: 3000 16.8 / 13.3, 7000
// 24.1 / 22.7, 8191 35.3 / 32.8 (binary32), 12000 37.3 / 37.5; over 4096, [4000, 2255] 22.6 / 18.9, [12000, 2255] 41.0 / 38.4.  Where there is
// an encoder by rows: STD at 8 sigma over 64, [300, 3072] 10.0 / 7.5, [2000, 3072] 12.4 / 11.4, [4000, 3072] 18.9 / 19.1; softmax, ABS, [1200,
// 512] 12.1 / 9.5, [20000, 512] 21.2 / 20.1, [40000, 512] 35.0 / 36.4; with more outliers a tile than a slot holds, STD at 3 sigma over 64, [1200,
// 3072] 33.3 / 14.9, [4000, 3072] 42.6 / 28.4.  TOPK, whose second launch finds nothing to do: [20, 1024] 10.0 / 7.9, [300, 4096] 10.1 / 9.5,
// [1000, 4096] 11.4 / 11.2, [2000, 4096] 14.1 / 14.2.)
constexpr uint32_t kShortWorkgroups = 2560, kShortWorkgroupsEven = 1792, kShortWorkgroupsRows = 1280, kShortWorkgroupsTopk = 256;
constexpr uint64_t kShortBytes = 8ull * kShortWorkgroups;
constexpr uint32_t kShortCountBits = 16;  // of a word; a workgroup's tiles have at most 16384 elements
// A word: a one and 31 bits of the launch's number, a one and its other 15 bits, the count.  Nothing else that a call writes to a workspace looks like
// one, so what other calls leave in its place, whatever struct they went through, does not read as a word.  Counts, their sums, launch counters
// and a slot's records are below 2^31 and written 4 bytes at a time: either half of a word that they replace has lost its top bit.  The
// table of a batch covers words whole, and its upper halves (sizes, upper halves of addresses, floats that are not negative) are below
// 2^31 too, but for a capacity, which would have to be the number itself, more than any tensor's length; numbers begin at an arbitrary one.
// (Counted from 1 in 48 bits, element number L of a slot's record beside an empty record read as a word of launch L, and under any upper half
// that an earlier word had left there still did.)
constexpr unsigned long long kShortFirstLaunch = 0x95A793E1ull << 15;
constexpr unsigned long long short_tag(unsigned long long launch) {
  return launch >> 15 << 32 | 1ull << 31 | (launch & 0x7FFFull) << kShortCountBits;
}
static_assert(short_tag(kShortFirstLaunch) == 0x95A793E180000000ull && short_tag(kShortFirstLaunch + 0x8001) == 0x95A793E280010000ull, "both halves");

// the batch compression kernels, by the weight of the variants they hold (adacc_kernels.hpp)
enum : int { kBatchRows4 = 0, kBatchAny4 = 1, kBatchTopk4 = 2, kBatchAny8 = 3, kBatchTopk8 = 4, kBatchKinds = 5 };

// variant index: ((mode*2 + (bits==8)) * 2 + asym) * 2 + (E==8)
__host__ __device__ inline uint32_t variant_index(uint32_t mode, uint32_t bits, uint32_t asym, uint32_t e8) {
  return ((mode * 2 + (bits == 8 ? 1u : 0u)) * 2 + asym) * 2 + e8;
}

}  // namespace adacc
