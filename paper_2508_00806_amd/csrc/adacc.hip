// libadacc: kernels and C ABI (see include/adacc.h).  gfx950 only.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <atomic>
#include <mutex>
#include <vector>

#include "adacc.h"
#include "adacc_common.hpp"
#include "adacc_fn.hpp"

namespace adacc {

// ===================================================================== kernels

// ---- utilities
// The table of a batch and the member lists behind it reach the device as kernel arguments, a slice per launch: the
// runtime copies kernel arguments when the launch is enqueued, so the host buffer may go away at once
// and the host never waits for the stream (a copy from pageable memory would).
// The slices come in sizes: the host writes all of a launch's arguments, word by word, across the bus to the device, and a launch
// whose 4 KiB are mostly padding costs more than the kernels behind it.
constexpr uint32_t kWordsPerUpload = 992;
template <uint32_t N>
struct WordSlice { uint32_t w[N]; };
static_assert(sizeof(WordSlice<kWordsPerUpload>) <= 3968, "kernel arguments are limited to 4 KiB");
static_assert(sizeof(TensorDesc) % 4 == 0, "copied as 32-bit words");
template <uint32_t N>
__global__ __launch_bounds__(kThreads) void words_upload_kernel(WordSlice<N> slice, uint32_t* dst, uint32_t count) {
  for (uint32_t i = threadIdx.x; i < count; i += kThreads) dst[i] = slice.w[i];
}

// clears a workspace (a kernel rather than a memset node, so that callers may capture it in a graph)
__global__ __launch_bounds__(kThreads) void workspace_clear_kernel(uint4* p, uint64_t n16) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = make_uint4(0, 0, 0, 0);
}

// Streams of known size in the shape the tensor kernels use (one piece of 4 KiB per wavefront per
// operand, full grid in the hardware's order, non-temporal accesses): what a kernel that only moves
// bytes reaches on this part for a given mix of reads and writes.
//   MIX 0: read a          1: write dst          2: dst = a (copy)          3: dst = a ^ b (two reads, one write)
template <int MIX>
__global__ __launch_bounds__(kThreads) void hbm_stream_kernel(uint4* __restrict__ dst, const uint4* __restrict__ a,
                                                              const uint4* __restrict__ b, uint64_t n16,
                                                              uint32_t* sink) {
  const uint64_t piece = ((uint64_t)blockIdx.x * kWavesPerWg + threadIdx.x / kWave) * 256u + (threadIdx.x % kWave);
  uint4 acc = make_uint4(0u, 0u, 0u, 0u);
  uint4 v[4], w[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint64_t i = piece + (uint64_t)j * 64u;
    const uint64_t ic = i < n16 ? i : n16 - 1u;
    if constexpr (MIX != 1) v[j] = load_stream16(a + ic);
    if constexpr (MIX == 3) w[j] = load_stream16(b + ic);
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint64_t i = piece + (uint64_t)j * 64u;
    if constexpr (MIX == 0) { acc.x ^= v[j].x; acc.y ^= v[j].y; acc.z ^= v[j].z; acc.w ^= v[j].w; }
    if constexpr (MIX == 1) { if (i < n16) store_stream16(dst + i, make_uint4((uint32_t)i, 1u, 2u, 3u)); }
    if constexpr (MIX == 2) { if (i < n16) store_stream16(dst + i, v[j]); }
    if constexpr (MIX == 3) { if (i < n16) store_stream16(dst + i, make_uint4(v[j].x ^ w[j].x, v[j].y ^ w[j].y, v[j].z ^ w[j].z, v[j].w ^ w[j].w)); }
  }
  if constexpr (MIX == 0) {
    // keeps the loads alive; practically never true, so nothing is written
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9E3779B9u && sink) *sink = acc.x;
  }
}

// ===================================================================== host side

static thread_local char g_hip_err[256] = "no HIP error recorded";

static int hip_fail(hipError_t e, const char* what) {
  std::snprintf(g_hip_err, sizeof g_hip_err, "%s: %s", what, hipGetErrorString(e));
  return ADACC_EHIP;
}

static int env_int(const char* name, int dflt) {
  const char* s = std::getenv(name);
  if (!s || !*s) return dflt;
  const long v = std::strtol(s, nullptr, 10);
  return v > 0 ? (int)v : dflt;
}

// Run-time knobs for measurements, read from the environment once per process.
struct Knobs {
  int mask_wgs_per_cu;  // ADACC_MASK_WGS_PER_CU: grid of the mask kernels
  int short_polls;      // ADACC_SHORT_POLLS: a wavefront's looks at the words before it counts missing tiles itself (adacc_short.hpp)
};
static const Knobs& knobs() {
  static const Knobs k = {env_int("ADACC_MASK_WGS_PER_CU", 256), env_int("ADACC_SHORT_POLLS", 512)};
  return k;
}

static int device_cus(int* cus) {
  static int cached[64];
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev >= 0 && dev < 64 && cached[dev] > 0) { *cus = cached[dev]; return ADACC_OK; }
  int n = 0;
  e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
  if (dev >= 0 && dev < 64) cached[dev] = n;
  *cus = n;
  return ADACC_OK;
}

static bool is_pow2(uint64_t v) { return v && !(v & (v - 1)); }
static uint32_t ilog2(uint64_t v) { uint32_t l = 0; while ((1ull << l) < v) ++l; return l; }
static uint64_t align256(uint64_t v) { return (v + 255ull) & ~255ull; }

struct Plan {  // everything derived from (method, numel)
  bool noop;
  bool outliers;
  uint32_t tile_elems, lgq, lgs, variant;
  uint64_t numel_main;   // the whole groups of the larger kind: what the tile kernels take
  uint32_t tail;         // elements after those: one short group, an extra wavefront's or workgroup's share of a launch
  uint32_t n_tiles;      // tiles of the main part
  uint32_t n_tiles_all;  // tiles of the whole tensor (what the layout reports)
  bool rowwise;  // every group lies inside a 512-element row and both kinds of group coincide
  bool half;     // the tensor is binary16 (else bf16)
  bool generic;  // group sizes the tile kernels do not take: the fallback kernels do the whole tensor
  bool wave_groups;  // generic: a wavefront per group instead of a workgroup
  float param, divisor;
};

// Groups from which on a wavefront for each is faster than a workgroup whatever their length, three for every SIMD of the device.
// (STD, int8, over SiLU rows of 2200 / 5160 / 8000 / 11008 at 8 sigma, us by workgroups and by wavefronts: 1024 rows 9.3 8.5 / 11.3 10.9 /
// 12.0 12.6 / 14.2 15.6; 2048 rows 11.7 9.8 / 14.3 13.1 / 15.6 16.0 / 22.1 20.4; 3072 rows 14.8 10.9 / 18.4 15.2 / 20.5 19.3 / 27.9 25.6.
// The 8 largest of values in quarters, int4: 1024 rows 10.1 9.2 / 11.6 12.0 / 12.7 14.2 / 14.9 18.0; 3072 rows 17.5 11.7 / 19.9 16.3 / 21.9 20.4 /
// 29.2 26.4.)
constexpr uint64_t kLongGroups = 3072;
static CompressFn long_fn(const adacc_method* m, const Plan& p) {
  return ADACC_PICK(p.half, compress_long_fn(p.tile_elems, m->outlier_mode, m->topk, m->bits, m->asym));
}

constexpr uint32_t kGenericMaxGroup = 16384;  // the longest segment of the fallback kernels

static int make_plan(const adacc_method* m, uint64_t numel, Plan* p) {
  std::memset(p, 0, sizeof *p);
  if (m->kind == ADACC_KIND_NOOP) { p->noop = true; return ADACC_OK; }
  if (m->kind != ADACC_KIND_QUANT) return ADACC_EINVAL;
  if (m->bits != 4 && m->bits != 8) return ADACC_EINVAL;
  if (m->asym > 1 || m->scale_rule > 1 || m->outlier_mode > ADACC_OUTLIER_TOPK) return ADACC_EINVAL;
  if (m->dtype > ADACC_DTYPE_F16) return ADACC_EINVAL;
  p->half = m->dtype == ADACC_DTYPE_F16;
  if (m->quant_group < 8 || m->quant_group % 8 != 0 || m->quant_group > kGenericMaxGroup) return ADACC_EINVAL;
  uint32_t gs = m->quant_group;
  const bool stat = m->outlier_mode == ADACC_OUTLIER_STD || m->outlier_mode == ADACC_OUTLIER_TOPK;
  if (stat) {
    if (m->stat_group < m->quant_group || m->stat_group % m->quant_group != 0 || m->stat_group > kGenericMaxGroup)
      return ADACC_EINVAL;
    gs = m->stat_group;
  }
  // the tile kernels take powers of two up to 4096; everything else goes through the fallback kernels
  p->generic = !is_pow2(m->quant_group) || !is_pow2(gs) || gs > 4096;
  if (m->outlier_mode == ADACC_OUTLIER_TOPK && (m->topk < 1 || m->topk > 32 || m->topk > gs)) return ADACC_EINVAL;
  if (m->outlier_mode == ADACC_OUTLIER_ABS || m->outlier_mode == ADACC_OUTLIER_STD) {
    if (!(m->thresh >= 0.0f) || std::isinf(m->thresh)) return ADACC_EINVAL;
  }
  p->outliers = m->outlier_mode != ADACC_OUTLIER_NONE;
  if (p->outliers && numel >= (1ull << 31)) return ADACC_EINVAL;  // 32-bit signed flat indices
  if (numel >= (1ull << 42)) return ADACC_EINVAL;
  if (p->generic) {
    // a segment: as many whole groups of the larger kind as fit 4096 elements (one, if it is larger);
    // the last segment and its last groups may be short, so there is no tail
    p->tile_elems = gs >= 4096 ? gs : gs * (4096u / gs);
    p->numel_main = numel;
    p->tail = 0;
    const uint64_t segs = (numel + p->tile_elems - 1) / p->tile_elems;
    if (segs >= (1ull << 31)) return ADACC_EINVAL;
    p->n_tiles = p->n_tiles_all = (uint32_t)segs;
    // One group to a segment, quantisation groups that are the segment or line up with its 512-element rows, whole octets,
    // and groups enough: a wavefront per group (adacc_long.hpp) does the compression, if it can hold the group.
    p->lgq = is_pow2(m->quant_group) ? ilog2(m->quant_group) : 0;
    p->wave_groups = gs > 2048 && segs >= kLongGroups && numel % 8 == 0 &&
                     (m->quant_group == gs || (is_pow2(m->quant_group) && m->quant_group <= 512)) && long_fn(m, *p) != nullptr;
  } else {
    p->tile_elems = gs > 2048 ? 4096u : 2048u;
    p->numel_main = numel - numel % gs;
    p->tail = (uint32_t)(numel % gs);
    p->n_tiles = (uint32_t)((p->numel_main + p->tile_elems - 1) / p->tile_elems);
    p->n_tiles_all = (uint32_t)((numel + p->tile_elems - 1) / p->tile_elems);
    p->lgq = ilog2(m->quant_group);
    p->lgs = ilog2(gs);
  }
  p->variant = variant_index(m->outlier_mode, m->bits, m->asym, p->tile_elems == 4096 ? 1u : 0u);
  p->rowwise = !p->generic && m->outlier_mode != ADACC_OUTLIER_TOPK && m->quant_group <= 512 &&
               (m->outlier_mode != ADACC_OUTLIER_STD || m->stat_group == m->quant_group);
  const float q = (float)(1u << (m->bits - 1));
  if (m->asym) p->divisor = m->scale_rule == ADACC_SCALE_PAPER ? 2.0f * q : 2.0f * q - 1.0f;
  else p->divisor = m->scale_rule == ADACC_SCALE_PAPER ? q : q - 1.0f;
  if (m->outlier_mode == ADACC_OUTLIER_ABS) p->param = m->thresh;
  if (m->outlier_mode == ADACC_OUTLIER_STD) p->param = m->thresh * m->thresh;
  return ADACC_OK;
}

static void fill_layout(const adacc_method* m, uint64_t numel, const Plan& p, adacc_layout* L) {
  std::memset(L, 0, sizeof *L);
  if (p.noop) return;
  const uint64_t groups = (numel + m->quant_group - 1) / m->quant_group;  // the last one may be short
  uint64_t off = 0;
  L->codes_off = off;   off = align256(off + (numel * m->bits + 7) / 8);
  L->scales_off = off;  off = align256(off + 4 * groups);
  L->zp_off = off;      off = align256(off + (m->asym ? 4 * groups : 0));
  L->tile_ptr_off = off; off = align256(off + (p.outliers ? 4ull * ((uint64_t)p.n_tiles_all + 1) : 0));
  L->idx_off = off;     off = align256(off + (p.outliers ? 4ull * m->max_outliers : 0));
  L->val_off = off;     off = align256(off + (p.outliers ? 2ull * m->max_outliers : 0));
  L->status_off = off;  off = align256(off + 16);
  L->total_bytes = off;
  L->tile_elems = p.tile_elems;
  L->n_tiles = p.n_tiles_all;
}

// TOPK whose statistics group is the tile, with every quantisation group inside a 512-element row, has kernels of its own
static bool topk_whole_tile(const adacc_method* m, const Plan& p) {
  return m->outlier_mode == ADACC_OUTLIER_TOPK && m->stat_group == p.tile_elems && m->quant_group <= 512;
}
// TOPK over groups that are the quantisation groups and lie inside a 512-element row: the row-at-a-time encoder
static bool topk_in_rows(const adacc_method* m, const Plan& p) {
  return !p.generic && m->outlier_mode == ADACC_OUTLIER_TOPK && m->stat_group == m->quant_group && m->quant_group <= 512;
}
static int batch_kind(const adacc_method* m, const Plan& p) {
  const bool whole = topk_whole_tile(m, p);
  if (p.tile_elems == 4096) return whole ? kBatchTopk8 : kBatchAny8;
  return (p.rowwise || topk_in_rows(m, p)) ? kBatchRows4 : (whole ? kBatchTopk4 : kBatchAny4);
}

static uint32_t decompress_pieces(uint64_t numel) { return (uint32_t)((numel + 2047ull) / 2048ull); }
// ceil(2^64 / n); 0 for n = 1, which the kernels know
static uint64_t reciprocal64(uint32_t n) { return n > 1u ? ~0ull / n + 1ull : 0ull; }
// 1 / n moved up by three units in the last place: the binary32 product with an integer below 4096 then lies at or
// above the quotient where that is an integer, and below the next integer everywhere else (n <= 2048)
static float reciprocal_up(uint32_t n) {
  const float r = 1.0f / (float)n;
  uint32_t bits;
  std::memcpy(&bits, &r, sizeof bits);
  bits += 3u;
  float up;
  std::memcpy(&up, &bits, sizeof up);
  return up;
}

// Workspace of one tensor that keeps outliers: [cnt: one word per tile][flag][block_sum][slots],
// block sums and slots for ABS / STD only.  Offsets relative to the tensor's region.
struct WsPlan { uint64_t cnt_off, flag_off, block_sum_off, slot_off, bytes; };
static uint32_t blocks_of(uint32_t n, int per) { return (n + (uint32_t)per - 1u) / (uint32_t)per; }
static WsPlan ws_plan(const adacc_method* m, const Plan& p) {
  WsPlan w;
  std::memset(&w, 0, sizeof w);
  if (p.noop || !p.outliers) return w;
  uint64_t off = 0;
  w.cnt_off = off;  off = align256(off + 4ull * p.n_tiles);
  w.flag_off = off; off += 256;
  if (m->outlier_mode != ADACC_OUTLIER_TOPK) {
    w.block_sum_off = off; off = align256(off + 4ull * blocks_of(p.n_tiles, kSumTiles));
    w.slot_off = off; off = align256(off + 4ull * kSlot * p.n_tiles);
  }
  w.bytes = off;
  return w;
}
// does the placement of this tensor start from per-block sums (a kernel of its own computes them)?
static bool needs_block_sums(const adacc_method* m, const Plan& p) {
  return p.outliers && m->outlier_mode != ADACC_OUTLIER_TOPK && p.n_tiles > kPlaceDirectTiles;
}
// tiles (segments) that a workgroup of the placement takes, and its workgroups: one more for the end that the groups do
// not divide
static uint32_t place_per(const adacc_method* m, const Plan& p) {
  if (!p.generic) return p.n_tiles > kPlaceDirectTiles ? (uint32_t)kSumTiles : (uint32_t)kPlaceTiles;
  const bool topk = m->outlier_mode == ADACC_OUTLIER_TOPK;
  const uint32_t workgroups = topk && p.tile_elems <= 4096 ? 4u * kPlaceWorkgroups : kPlaceWorkgroups;
  uint32_t per = 1;
  while (per < (uint32_t)kPlaceSegments && per * workgroups < p.n_tiles) per *= 2;
  if (topk && per * workgroups < p.n_tiles) per *= blocks_of(p.n_tiles, (int)(per * workgroups));
  return per;
}
static uint32_t place_grid(const adacc_method* m, const Plan& p) {
  if (!p.outliers) return 0u;
  return blocks_of(p.n_tiles, (int)place_per(m, p)) + (!p.generic && p.tail != 0 ? 1u : 0u);
}
// wavefronts of the tile launch: one per tile, one more for the end of a tensor without outliers
static uint32_t tile_waves(const Plan& p) { return p.n_tiles + (!p.outliers && p.tail != 0 ? 1u : 0u); }

static void fill_desc(const adacc_method* m, uint64_t numel, const Plan& p, const adacc_layout& L, const void* src,
                      void* blob, void* dst, void* ws_region, TensorDesc* d) {
  std::memset(d, 0, sizeof *d);
  unsigned char* b = static_cast<unsigned char*>(blob);
  d->src = static_cast<const uint16_t*>(src);
  d->dst = dst;
  d->codes = b + L.codes_off;
  d->scales = reinterpret_cast<float*>(b + L.scales_off);
  d->zp = reinterpret_cast<float*>(b + L.zp_off);
  d->tile_ptr = reinterpret_cast<uint32_t*>(b + L.tile_ptr_off);
  d->idx = reinterpret_cast<int32_t*>(b + L.idx_off);
  d->val = reinterpret_cast<uint16_t*>(b + L.val_off);
  d->status = reinterpret_cast<uint32_t*>(b + L.status_off);
  if (ws_region && p.outliers) {
    const WsPlan w = ws_plan(m, p);
    unsigned char* r = static_cast<unsigned char*>(ws_region);
    d->cnt = reinterpret_cast<uint32_t*>(r + w.cnt_off);
    d->flag = reinterpret_cast<uint32_t*>(r + w.flag_off);
    d->block_sum = reinterpret_cast<uint32_t*>(r + w.block_sum_off);
    d->slot = reinterpret_cast<uint32_t*>(r + w.slot_off);
  }
  d->numel = p.numel_main;
  d->tail = p.tail;
  d->n_tiles = p.n_tiles;
  d->n_tiles_all = p.n_tiles_all;
  d->bits = m->bits;
  d->asym = m->asym;
  d->mode = m->outlier_mode;
  d->gq = m->quant_group;
  d->gs = (m->outlier_mode == ADACC_OUTLIER_STD || m->outlier_mode == ADACC_OUTLIER_TOPK) ? m->stat_group : m->quant_group;
  d->tile_elems = p.tile_elems;
  d->generic = p.generic ? 1u : 0u;
  d->from_sums = needs_block_sums(m, p) ? 1u : 0u;
  d->place_per = p.outliers ? place_per(m, p) : 0u;
  d->lgt = p.tile_elems == 4096 ? 12u : 11u;
  if (dst) {  // decompression counts pieces of the whole tensor, 2048 elements as a rule (launch_decompress)
    d->numel = numel;
    d->tail = 0;
    d->n_tiles = decompress_pieces(numel);
    d->ptr_shift = p.tile_elems == 4096 ? 1u : 0u;
    d->per_tile = m->outlier_mode == ADACC_OUTLIER_TOPK ? m->topk * (p.tile_elems / d->gs) : 0u;
    if (p.generic) {
      d->magic_q = reciprocal64(m->quant_group / 8u);
      d->magic_t = reciprocal64(p.tile_elems / 8u);
      d->recip_q = reciprocal_up(m->quant_group / 8u);
    }
  }
  d->lgq = p.lgq;
  d->lgs = p.lgs;
  d->cap = m->max_outliers;
  d->topk = m->topk;
  d->param = p.param;
  d->divisor = p.divisor;
  {
    int ex = 0;
    d->inv_divisor = (std::frexp(p.divisor, &ex) == 0.5f) ? 1.0f / p.divisor : 0.0f;  // exact for a power of two
    d->pow2_divisor = d->inv_divisor != 0.0f ? 1u : 0u;
  }
  d->variant = p.variant;
  d->rowwise = p.rowwise ? 1u : 0u;
}

static bool misaligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

static BatchCompressFn compress_batch_fn(bool half, int kind) {
  return kind >= kBatchAny8 ? ADACC_PICK(half, compress_batch_fn8(kind)) : ADACC_PICK(half, compress_batch_fn4(kind));
}

// `whole` (TOPK only): the statistics group is the whole tile; that case has kernels of its own.
// `rowwise`: for TOPK, statistics group = quantisation group inside a row (topk_in_rows)
static CompressFn compress_fn(const adacc_method* m, bool e8, bool rowwise, bool whole) {
  const bool half = m->dtype == ADACC_DTYPE_F16;
  switch (m->outlier_mode) {
    case ADACC_OUTLIER_NONE: return ADACC_PICK(half, compress_fn_none(m->bits, m->asym, e8, rowwise));
    case ADACC_OUTLIER_ABS: return ADACC_PICK(half, compress_fn_abs(m->bits, m->asym, e8, rowwise));
    case ADACC_OUTLIER_STD: return ADACC_PICK(half, compress_fn_std(m->bits, m->asym, e8, rowwise));
    default: return ADACC_PICK(half, compress_fn_topk(m->bits, m->asym, e8, whole, rowwise));
  }
}

static int clear_device(void* mem, uint64_t bytes, hipStream_t s);

// The words of the one-launch compression lie at the end of a workspace, each with the number of its launch, which is one of all such
// launches of the process and has no like among what other calls write (short_tag): a word that names a launch was written by it,
// whatever is left in the buffer by calls through other structs, replayed graphs or an earlier use.  The host struct says whether all
// other calls through it have kept in front of the words so far; one that needed their place ends the short way of this struct, whose
// buffer has no room to spare.
constexpr uint32_t kShortWordsOurs = 1;
static_assert(kShortBytes == ADACC_SHORT_BYTES, "adacc.h says how much room that is");
static uint64_t short_words_off(const adacc_workspace* ws) { return (ws->bytes - kShortBytes) & ~255ull; }
static void use_workspace(adacc_workspace* ws, uint64_t bytes) {
  if (ws->reserved == kShortWordsOurs && bytes > short_words_off(ws)) ws->reserved = 0;
}
// A launch that is being captured would be replayed with the same number.
static bool captured(hipStream_t s) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return true;
}

// Next epoch of a workspace; clears the buffer first when the counter is about to wrap.
static int next_epoch(adacc_workspace* ws, hipStream_t s, uint32_t* epoch) {
  if (ws->epoch >= kEpochMax) {
    const int rc = clear_device(ws->device_mem, ws->bytes, s);
    if (rc != ADACC_OK) return rc;
    ws->epoch = 0;
  }
  ws->epoch += 1;
  *epoch = ws->epoch;
  return ADACC_OK;
}

static int launch_check(const char* what) {
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? ADACC_OK : hip_fail(e, what);
}

// The table to the start of the batch workspace and the member lists to their place behind it (two launches for each of
// a batch of two layers, 4.5 us apiece, before they went up together).
template <uint32_t N>
static int upload_words(const uint32_t* words, uint32_t count, uint32_t* dst, hipStream_t s) {
  WordSlice<N> slice;
  std::memcpy(slice.w, words, count * sizeof(uint32_t));
  hipLaunchKernelGGL(words_upload_kernel<N>, dim3(1), dim3(kThreads), 0, s, slice, dst, count);
  return launch_check("words_upload_kernel");
}
static int upload_batch(const std::vector<TensorDesc>& table, const std::vector<uint32_t>& members, uint64_t members_off,
                        void* device_mem, hipStream_t s) {
  const size_t table_words = table.size() * sizeof(TensorDesc) / 4;
  std::vector<uint32_t> words(members.empty() ? table_words : members_off / 4 + members.size(), 0u);
  std::memcpy(words.data(), table.data(), table.size() * sizeof(TensorDesc));
  if (!members.empty()) std::memcpy(words.data() + members_off / 4, members.data(), members.size() * 4);
  for (size_t i = 0; i < words.size(); i += kWordsPerUpload) {
    const uint32_t count = (uint32_t)std::min<size_t>(kWordsPerUpload, words.size() - i);
    uint32_t* dst = static_cast<uint32_t*>(device_mem) + i;
    const uint32_t* from = words.data() + i;
    const int rc = count <= 128u ? upload_words<128>(from, count, dst, s) : count <= 256u ? upload_words<256>(from, count, dst, s)
                   : count <= 512u ? upload_words<512>(from, count, dst, s) : upload_words<kWordsPerUpload>(from, count, dst, s);
    if (rc != ADACC_OK) return rc;
  }
  return ADACC_OK;
}

static int clear_device(void* mem, uint64_t bytes, hipStream_t s) {
  const uint64_t n16 = bytes / 16;
  uint32_t grid = (uint32_t)((n16 + kThreads - 1) / kThreads);
  if (grid > 4096) grid = 4096;
  if (grid == 0) return ADACC_OK;
  hipLaunchKernelGGL(workspace_clear_kernel, dim3(grid), dim3(kThreads), 0, s, static_cast<uint4*>(mem), n16);
  return launch_check("workspace_clear_kernel");
}

// batch workspace: [table: n descriptors][member lists of the launches: 4 n words][the tensors' regions]
struct BatchPlan {
  uint64_t members_off, regions_off, bytes;
};
static BatchPlan batch_plan(uint32_t n_active, uint64_t region_bytes) {
  BatchPlan b;
  const uint64_t n = n_active ? n_active : 1;
  b.members_off = align256(n * sizeof(TensorDesc));
  b.regions_off = b.members_off + align256(4ull * 4ull * n);
  b.bytes = b.regions_off + region_bytes;
  return b;
}

// The block sums and the placement of a batch are one launch each up to this many workgroups, two tensors of 44032 tiles
// next to four of 8192 for instance: a workgroup without tiles leaves at once, at about 2 ns, a launch takes 4.5 us.
constexpr uint64_t kPlaceTogether = 8192;
// Tiles and pieces of tensors of unequal sizes go in one launch up to this many wavefronts, 2048 workgroups of which as a rule fewer
// than half have nothing to do: 1 to 2 us, where a launch takes 3.5 us of the host's time.
constexpr uint64_t kTilesTogether = 8192;

// A launch over a group of table entries: grid.y = the group's entries, grid.x covers the largest.
struct GroupLaunch {
  uint32_t first_member, n_members, max_units;
  int kind;  // what the caller makes of it (register class, kernel)
};
// Groups the entries for which units[i] > 0 by kind[i] and by size (unit counts within a factor of
// two of each other, at most 65535 entries per launch) and appends their member lists to `members`.
// `together` > 0: whatever their size, as long as the grid of a kind has at most that many units - for kernels
// whose empty workgroups cost less than another launch.
static void group_launches(const std::vector<uint32_t>& units, const std::vector<int>& kind,
                           std::vector<uint32_t>* members, std::vector<GroupLaunch>* launches, uint64_t together = 0) {
  for (int k = 0; k < 2 * kBatchKinds; ++k) {  // kinds of the second half: the same for binary16 tensors
    uint64_t most = 0, n = 0;
    for (uint32_t i = 0; i < units.size(); ++i)
      if (units[i] != 0 && kind[i] == k) { most = std::max<uint64_t>(most, units[i]); ++n; }
    if (n == 0) continue;
    const bool one = most * n <= together;
    for (uint32_t bucket = 0; bucket <= (one ? 0u : 32u); ++bucket) {
      GroupLaunch g = {(uint32_t)members->size(), 0u, 0u, k};
      for (uint32_t i = 0; i < units.size(); ++i) {
        if (units[i] == 0 || kind[i] != k || (!one && ilog2(units[i]) != bucket)) continue;
        if (g.n_members == 65535u) {
          launches->push_back(g);
          g = GroupLaunch{(uint32_t)members->size(), 0u, 0u, k};
        }
        members->push_back(i);
        g.n_members += 1;
        g.max_units = std::max(g.max_units, units[i]);
      }
      if (g.n_members) launches->push_back(g);
    }
  }
}

// one wavefront per strip of `width` channels (512, or 256 for a binary32 output) and `rows` tokens, four per workgroup
static uint32_t strip_grid(uint64_t tokens, uint32_t hidden, uint32_t rows, uint32_t width = 512u) {
  const uint64_t units = ((tokens + rows - 1) / rows) * ((hidden + width - 1u) / width);
  return (uint32_t)((units + kWavesPerWg - 1) / kWavesPerWg);  // tokens * hidden < 2^32: far below 2^31
}
static uint32_t strip_width(int dst_dtype) { return dst_dtype == ADACC_DST_F32 ? 256u : 512u; }

// ---- outlier channels (Section 3.2, Eq. 1)
struct ChannelPlan {
  adacc_method quant;  // the quantisation of the rest: the same method without outliers
  Plan plan;
  adacc_layout quant_layout;
  uint64_t numel;
  uint32_t n_chunks;
};

static int make_channel_plan(const adacc_channel_method* m, uint64_t tokens, uint32_t hidden, ChannelPlan* cp) {
  std::memset(cp, 0, sizeof *cp);
  if (hidden < 8 || hidden > 65536 || hidden % 8 != 0) return ADACC_EINVAL;
  if (tokens > 0xFFFFFFFFull / hidden) return ADACC_EINVAL;  // tokens * hidden < 2^32
  if (m->quant_group > 2048) return ADACC_EINVAL;
  if (m->max_channels < 1 || m->max_channels > hidden) return ADACC_EINVAL;
  if (!std::isfinite(m->z_thresh)) return ADACC_EINVAL;
  cp->quant.kind = ADACC_KIND_QUANT;
  cp->quant.bits = m->bits;
  cp->quant.quant_group = m->quant_group;
  cp->quant.asym = m->asym;
  cp->quant.scale_rule = m->scale_rule;
  cp->quant.outlier_mode = ADACC_OUTLIER_NONE;
  cp->quant.dtype = m->dtype;
  cp->numel = tokens * hidden;
  const int rc = make_plan(&cp->quant, cp->numel, &cp->plan);
  if (rc != ADACC_OK) return rc;
  if (cp->plan.tail != 0 || cp->plan.generic) return ADACC_EINVAL;  // here: a power of two that divides the tensor
  fill_layout(&cp->quant, cp->numel, cp->plan, &cp->quant_layout);
  cp->n_chunks = (uint32_t)((tokens + kChunkTokens - 1) / kChunkTokens);
  return ADACC_OK;
}

static void fill_channel_layout(const adacc_channel_method* m, uint64_t tokens, uint32_t hidden, const ChannelPlan& cp,
                                adacc_channel_layout* L) {
  std::memset(L, 0, sizeof *L);
  L->codes_off = cp.quant_layout.codes_off;
  L->scales_off = cp.quant_layout.scales_off;
  L->zp_off = cp.quant_layout.zp_off;
  uint64_t off = cp.quant_layout.status_off;  // the sections of this mode start where the plain blob's status would be
  L->ch_mask_off = off;  off = align256(off + hidden / 8);
  L->ch_base_off = off;  off = align256(off + 4ull * (hidden / 8));
  L->ch_idx_off = off;   off = align256(off + 4ull * m->max_channels);
  L->ch_val_off = off;   off = align256(off + 2ull * tokens * m->max_channels);
  L->status_off = off;   off = align256(off + 16);
  L->total_bytes = off;
}

static uint64_t channel_partial_bytes(uint32_t n_chunks, uint32_t hidden) { return align256(4ull * n_chunks * hidden); }

static void fill_channel_desc(const adacc_channel_method* m, uint64_t tokens, uint32_t hidden,
                              const adacc_channel_layout& L, void* blob, ChannelDesc* c) {
  unsigned char* b = static_cast<unsigned char*>(blob);
  c->mask = b + L.ch_mask_off;
  c->base = reinterpret_cast<uint32_t*>(b + L.ch_base_off);
  c->ch_idx = reinterpret_cast<int32_t*>(b + L.ch_idx_off);
  c->ch_val = reinterpret_cast<uint16_t*>(b + L.ch_val_off);
  c->status = reinterpret_cast<uint32_t*>(b + L.status_off);
  c->hidden = hidden;
  c->tokens = (uint32_t)tokens;
  c->max_channels = m->max_channels;
  c->z_thresh = m->z_thresh;
  c->inv_hidden = std::nextafter(std::nextafter(1.0f / (float)hidden, 0.0f), 0.0f);
}

}  // namespace adacc

using namespace adacc;

// ===================================================================== C ABI

extern "C" {

const char* adacc_version(void) { return "0.1"; }

const char* adacc_strerror(int code) {
  switch (code) {
    case ADACC_OK: return "ok";
    case ADACC_EINVAL: return "invalid method or size";
    case ADACC_ENULL: return "null pointer";
    case ADACC_ESIZE: return "blob or workspace too small";
    case ADACC_EALIGN: return "device pointer not aligned";
    case ADACC_EHIP: return g_hip_err;
    case ADACC_ELIMIT: return "size beyond the limit of this entry point";
    default: return "unknown error code";
  }
}

int adacc_layout_of(const adacc_method* method, uint64_t numel, adacc_layout* out) {
  if (!method || !out) return ADACC_ENULL;
  Plan p;
  const int rc = make_plan(method, numel, &p);
  if (rc != ADACC_OK) return rc;
  fill_layout(method, numel, p, out);
  return ADACC_OK;
}

uint64_t adacc_workspace_bytes(const adacc_method* method, uint64_t numel) {
  if (!method) return 0;
  Plan p;
  if (make_plan(method, numel, &p) != ADACC_OK) return 0;
  return ws_plan(method, p).bytes;
}

int adacc_workspace_init(adacc_workspace* ws, void* device_mem, uint64_t bytes, void* hip_stream) {
  if (!ws || !device_mem) return ADACC_ENULL;
  if (bytes < 256 || bytes % 16 != 0) return ADACC_ESIZE;
  if (misaligned(device_mem, 256)) return ADACC_EALIGN;
  const int rc = clear_device(device_mem, bytes, static_cast<hipStream_t>(hip_stream));
  if (rc != ADACC_OK) return rc;
  ws->device_mem = device_mem;
  ws->bytes = bytes;
  ws->epoch = 0;
  ws->reserved = bytes >= kShortBytes ? kShortWordsOurs : 0;
  return ADACC_OK;
}

// The tiles' counts in blocks, where the placement starts from those.
static int launch_block_sums(const adacc_method* method, const Plan& p, const TensorDesc& d, hipStream_t s) {
  if (!needs_block_sums(method, p)) return ADACC_OK;
  hipLaunchKernelGGL(ADACC_PICK(p.half, place_sum_fn()), dim3(blocks_of(p.n_tiles, kSumTiles)), dim3(kPlaceThreads), 0, s, d);
  return launch_check("place_sum_kernel");
}

// The fallback kernels for one tensor: everything but the places of the outliers, then those.
static int launch_generic_compress(const adacc_method* method, const Plan& p, const TensorDesc& d, uint32_t epoch,
                                   hipStream_t s) {
  const bool topk = method->outlier_mode == ADACC_OUTLIER_TOPK;
  const uint32_t lds = ADACC_PICK(p.half, generic_lds_bytes(p.tile_elems, method->quant_group, topk && d.gs < p.tile_elems));
  const uint32_t threads = ADACC_PICK(p.half, generic_threads());
  if (p.wave_groups) {
    hipLaunchKernelGGL(long_fn(method, p), dim3(blocks_of(p.n_tiles, kWavesPerWg)), dim3(kThreads), 0, s, d, epoch);
  } else {
    hipLaunchKernelGGL(ADACC_PICK(p.half, compress_generic_fn(p.tile_elems, method->outlier_mode, d.gs)), dim3(p.n_tiles), dim3(threads), lds, s, d, epoch);
  }
  int rc = launch_check("compression of the fallback methods");
  if (rc != ADACC_OK || !p.outliers) return rc;
  rc = launch_block_sums(method, p, d, s);
  if (rc != ADACC_OK) return rc;
  hipLaunchKernelGGL(ADACC_PICK(p.half, place_generic_fn(p.tile_elems, method->outlier_mode, d.gs)), dim3(place_grid(method, p)), dim3(threads), lds, s, d, epoch);
  return launch_check("place_generic_kernel");
}

// LDS that the general encoder of tiles of 4 rows does not use but that bounds the workgroups of a CU to six, where its registers
// (41 to 60) allow eight: from three rounds of the device on, a stream reads and writes a little faster with fewer wavefronts on its way
// at once.  ([262144, 2048], int8, us with eight / six / five and, before, with the registers' 5 to 8: without outliers in groups of
// 1024 asymmetric 270 / 262 / 258 and 267; STD over 2048 at 6 sigma 266 / 260 / 257 and 260; softmax values, ABS, asymmetric, 268 /
// 261 / 262 and 260.  Where a tile has many outliers issue counts for more: SiLU, ABS at 3, asymmetric, 300 / 312 / 325 and 334.
// [28000, 2048], the same: 29.3 / 29.0 / 28.9 and 29.3; 36.2 / 36.2 / 35.8 and 36.8; 37.7 / 37.1 / 37.7 and 37.6; 42.1 / 42.9 / 44.6 and 45.9.)
constexpr uint32_t kStreamTiles = 24576;
static uint32_t residency_lds(const adacc_method* m, const Plan& p) {
  const bool general = !p.rowwise && p.tile_elems == 2048 && m->outlier_mode != ADACC_OUTLIER_TOPK;
  return general && p.n_tiles >= kStreamTiles ? 24320u : 0u;  // (19 of the 128 pieces of 1280 bytes)
}

// Many wavefronts for the placement (adacc_k_place.hip), but where there is as a rule nothing to place: STD over groups of so few that
// no finite value lies that far from the mean (z <= sqrt(n - 1); [2886, 16384] at 8 sigma over 64: 47.3 us both ways, 47.9 by many).
static bool place_many(const adacc_method* m, const Plan& p) {
  if (m->outlier_mode == ADACC_OUTLIER_TOPK || p.n_tiles > kPlaceManyTiles) return false;
  return m->outlier_mode != ADACC_OUTLIER_STD || p.param < (float)(m->stat_group - 1u);
}

static CompressShortFn compress_short_fn(const adacc_method* m, const Plan& p) {
  const bool e8 = p.tile_elems == 4096;
  switch (m->outlier_mode) {
    case ADACC_OUTLIER_ABS: return ADACC_PICK(p.half, compress_short_fn_abs(e8));
    case ADACC_OUTLIER_STD: return ADACC_PICK(p.half, compress_short_fn_std(e8));
    default: return ADACC_PICK(p.half, compress_short_fn_topk(e8, topk_whole_tile(m, p)));
  }
}
static bool in_one_launch(const adacc_method* m, const Plan& p) {
  if (p.generic) return false;
  const uint32_t workgroups = blocks_of(p.n_tiles, kWavesPerWg);
  // TOPK of more outliers a tile than its record holds would be selected twice
  if (m->outlier_mode == ADACC_OUTLIER_TOPK) return workgroups <= kShortWorkgroupsTopk && m->topk * (p.tile_elems / m->stat_group) <= (uint32_t)kSlot;
  return workgroups <= (p.rowwise ? kShortWorkgroupsRows : p.tail != 0 ? kShortWorkgroups : kShortWorkgroupsEven);
}

static int compress_one(const adacc_method* method, const void* src, uint64_t numel, void* blob, uint64_t blob_bytes,
                        adacc_workspace* ws, void* hip_stream) {
  if (!method) return ADACC_ENULL;
  Plan p;
  int rc = make_plan(method, numel, &p);
  if (rc != ADACC_OK) return rc;
  if (p.noop || numel == 0) return ADACC_OK;
  if (!src || !blob) return ADACC_ENULL;
  adacc_layout L;
  fill_layout(method, numel, p, &L);
  if (blob_bytes < L.total_bytes) return ADACC_ESIZE;
  if (misaligned(src, 16) || misaligned(blob, 256)) return ADACC_EALIGN;
  if (p.outliers) {
    if (!ws || !ws->device_mem) return ADACC_ENULL;
    if (ws->bytes < ws_plan(method, p).bytes) return ADACC_ESIZE;
    if (misaligned(ws->device_mem, 256)) return ADACC_EALIGN;
  }
  int cus = 0;
  rc = device_cus(&cus);  // also: fail here, before any state changes, when there is no device
  if (rc != ADACC_OK) return rc;
  if (p.outliers) use_workspace(ws, ws_plan(method, p).bytes);
  TensorDesc d;
  fill_desc(method, numel, p, L, src, blob, nullptr, p.outliers ? ws->device_mem : nullptr, &d);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (p.generic) {
    uint32_t epoch = 0;
    if (p.outliers) {
      rc = next_epoch(ws, s, &epoch);
      if (rc != ADACC_OK) return rc;
    }
    return launch_generic_compress(method, p, d, epoch, s);
  }
  if (p.outliers && ws->reserved == kShortWordsOurs && in_one_launch(method, p) && !captured(s)) {
    uint32_t epoch = 0;
    rc = next_epoch(ws, s, &epoch);  // counts this launch too
    if (rc != ADACC_OK) return rc;
    static std::atomic<unsigned long long> launches{kShortFirstLaunch};
    const unsigned long long tag = short_tag(launches.fetch_add(1));
    unsigned long long* words = reinterpret_cast<unsigned long long*>(static_cast<unsigned char*>(ws->device_mem) + short_words_off(ws));
    hipLaunchKernelGGL(compress_short_fn(method, p), dim3(blocks_of(p.n_tiles, kWavesPerWg) + (p.tail != 0 ? 1u : 0u)), dim3(kThreads), 0, s, d,
                       tag, words, (uint32_t)knobs().short_polls);
    return launch_check("compress_short_kernel");
  }
  CompressFn fn = compress_fn(method, p.tile_elems == 4096, p.rowwise || topk_in_rows(method, p), topk_whole_tile(method, p));
  const uint32_t grid = blocks_of(tile_waves(p), kWavesPerWg);  // one tile per wavefront
  uint32_t epoch = 0;
  if (p.outliers) {
    rc = next_epoch(ws, s, &epoch);
    if (rc != ADACC_OK) return rc;
  }
  if (grid != 0) {
    hipLaunchKernelGGL(fn, dim3(grid), dim3(kThreads), residency_lds(method, p), s, d, epoch);
    rc = launch_check("compress_kernel");
    if (rc != ADACC_OK) return rc;
  }
  if (p.outliers) {
    rc = launch_block_sums(method, p, d, s);
    if (rc != ADACC_OK) return rc;
    const bool many = place_many(method, p);
    hipLaunchKernelGGL(ADACC_PICK(p.half, place_fn(many)), dim3(place_grid(method, p)), dim3(many ? kPlaceManyThreads : kPlaceThreads), 0, s, d, epoch);
    rc = launch_check("place_kernel");
  }
  return rc;
}

int adacc_compress(const adacc_method* method, const void* src, uint64_t numel, void* blob, uint64_t blob_bytes,
                   adacc_workspace* ws, void* hip_stream) {
  return compress_one(method, src, numel, blob, blob_bytes, ws, hip_stream);
}

// ---- the same for callers that cannot allocate: the workspace is a device array of the library
constexpr uint64_t kNoallocScratchBytes = 24ull << 20;
static __device__ __align__(256) unsigned char scratch[kNoallocScratchBytes + kShortBytes];

int adacc_compress_noalloc(const adacc_method* method, const void* src, uint64_t numel, void* blob,
                           uint64_t blob_bytes, void* hip_stream) {
  if (!method) return ADACC_ENULL;
  Plan p;
  int rc = make_plan(method, numel, &p);
  if (rc != ADACC_OK) return rc;
  if (p.noop || numel == 0 || !p.outliers) return compress_one(method, src, numel, blob, blob_bytes, nullptr, hip_stream);
  if (ws_plan(method, p).bytes > kNoallocScratchBytes) return ADACC_ELIMIT;
  // Every device has its own copy of the array at its own address: looked up once per device, with
  // that device current, and kept together with the launch counter of the words in it.
  static adacc_workspace per_device[64];
  static std::mutex lock;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= 64) return ADACC_EINVAL;
  std::lock_guard<std::mutex> hold(lock);  // calls that share the array are serialised on the host; on the GPU they must not overlap
  adacc_workspace* ws = &per_device[dev];
  if (!ws->device_mem) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    // the flag word of a tensor must not hold a value that a later launch counter takes: cleared by a
    // kernel on the caller's stream before the first use
    rc = clear_device(ptr, sizeof scratch, static_cast<hipStream_t>(hip_stream));
    if (rc != ADACC_OK) return rc;
    ws->device_mem = ptr;
    ws->bytes = sizeof scratch;
    ws->epoch = 0;
    ws->reserved = kShortWordsOurs;
  }
  return compress_one(method, src, numel, blob, blob_bytes, ws, hip_stream);
}

// rows of a piece, see full_piece_rows; at most 2^34 elements in small pieces: a grid has fewer than 2^32 threads
static uint32_t piece_rows(const adacc_method* m, const Plan& p, uint64_t numel, bool f32) {
  const uint32_t full = full_piece_rows(f32);
  if (numel > (1ull << 34)) return full;
  if (f32) return numel < (1ull << 25) ? full : p.outliers ? 4u : 2u;
  if (p.generic) return full;
  if (!p.outliers) return numel < (1ull << 26) ? full : 2u;
  return m->outlier_mode != ADACC_OUTLIER_TOPK && numel >= (1ull << 28) ? 2u : full;
}
static int launch_decompress(const adacc_method* m, const Plan& p, const TensorDesc& d, int dst_dtype, hipStream_t s) {
  const bool f32 = dst_dtype == ADACC_DST_F32;
  const uint32_t rows = piece_rows(m, p, d.numel, f32), waves = (uint32_t)piece_waves((int)rows);
  TensorDesc own = d;
  if (rows != full_piece_rows(f32)) {
    const uint32_t piece = rows * (uint32_t)kWave * (f32 ? 4u : 8u);
    own.n_tiles = (uint32_t)((d.numel + piece - 1u) / piece);
    own.ptr_shift += ilog2(2048u / piece);  // (the fallback kernels' tiles are found by division)
  }
  DecompressFn fn = ADACC_PICK(p.half, decompress_fn(m->bits, m->asym, f32, p.generic, rows));
  hipLaunchKernelGGL(fn, dim3((own.n_tiles + waves - 1u) / waves), dim3(waves * (uint32_t)kWave), 0, s, own, p.outliers ? 1u : 0u);  // one piece per wavefront
  return launch_check("decompress_kernel");
}

int adacc_decompress(const adacc_method* method, const void* blob, uint64_t blob_bytes, uint64_t numel, void* dst,
                     int dst_dtype, void* hip_stream) {
  if (!method) return ADACC_ENULL;
  if (dst_dtype != ADACC_DST_16 && dst_dtype != ADACC_DST_F32) return ADACC_EINVAL;
  Plan p;
  int rc = make_plan(method, numel, &p);
  if (rc != ADACC_OK) return rc;
  if (p.noop || numel == 0) return ADACC_OK;
  if (!blob || !dst) return ADACC_ENULL;
  adacc_layout L;
  fill_layout(method, numel, p, &L);
  if (blob_bytes < L.total_bytes) return ADACC_ESIZE;
  if (misaligned(dst, 16) || misaligned(blob, 256)) return ADACC_EALIGN;
  TensorDesc d;
  fill_desc(method, numel, p, L, nullptr, const_cast<void*>(blob), dst, nullptr, &d);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  return launch_decompress(method, p, d, dst_dtype, s);
}

static int batch_prepare(uint32_t n, const adacc_method* methods, const uint64_t* numels, std::vector<Plan>* plans,
                         uint32_t* total_tiles, uint32_t* n_active, uint64_t* region_bytes) {
  plans->resize(n);
  uint64_t tiles = 0, regions = 0;
  uint32_t act = 0;
  for (uint32_t i = 0; i < n; ++i) {
    const int rc = make_plan(&methods[i], numels[i], &(*plans)[i]);
    if (rc != ADACC_OK) return rc;
    if ((*plans)[i].noop || numels[i] == 0) { (*plans)[i].noop = true; continue; }
    tiles += (*plans)[i].n_tiles;
    regions += ws_plan(&methods[i], (*plans)[i]).bytes;
    ++act;
  }
  if (tiles >= (1ull << 32)) return ADACC_EINVAL;
  *total_tiles = (uint32_t)tiles;
  *n_active = act;
  *region_bytes = regions;
  return ADACC_OK;
}

uint64_t adacc_batch_workspace_bytes(uint32_t n, const adacc_method* methods, const uint64_t* numels) {
  if (n && (!methods || !numels)) return 0;
  std::vector<Plan> plans;
  uint32_t total = 0, act = 0;
  uint64_t regions = 0;
  if (batch_prepare(n, methods, numels, &plans, &total, &act, &regions) != ADACC_OK) return 0;
  return batch_plan(act, regions).bytes;
}

// Descriptors of the active tensors of a batch.
static int batch_table(uint32_t n, const adacc_method* methods, const std::vector<Plan>& plans, const uint64_t* numels,
                       const void* const* srcs, void* const* blobs, const uint64_t* blob_bytes, void* const* dsts,
                       bool compress, unsigned char* regions, std::vector<TensorDesc>* descs,
                       std::vector<uint32_t>* origin) {
  uint64_t region_off = 0;
  for (uint32_t i = 0; i < n; ++i) {
    if (plans[i].noop) continue;
    if (!blobs[i]) return ADACC_ENULL;
    if (compress ? !srcs[i] : !dsts[i]) return ADACC_ENULL;
    adacc_layout L;
    fill_layout(&methods[i], numels[i], plans[i], &L);
    if (blob_bytes[i] < L.total_bytes) return ADACC_ESIZE;
    if (misaligned(blobs[i], 256)) return ADACC_EALIGN;
    if (compress ? misaligned(srcs[i], 16) : misaligned(dsts[i], 16)) return ADACC_EALIGN;
    TensorDesc d;
    fill_desc(&methods[i], numels[i], plans[i], L, compress ? srcs[i] : nullptr, blobs[i], compress ? nullptr : dsts[i],
              compress ? regions + region_off : nullptr, &d);
    descs->push_back(d);
    origin->push_back(i);
    if (compress) region_off += ws_plan(&methods[i], plans[i]).bytes;
  }
  return ADACC_OK;
}

int adacc_compress_batch(uint32_t n, const adacc_method* methods, const void* const* srcs, const uint64_t* numels,
                         void* const* blobs, const uint64_t* blob_bytes, adacc_workspace* ws, void* hip_stream) {
  if (n == 0) return ADACC_OK;
  if (!methods || !srcs || !numels || !blobs || !blob_bytes) return ADACC_ENULL;
  std::vector<Plan> plans;
  uint32_t total = 0, act = 0;
  uint64_t region_bytes = 0;
  int rc = batch_prepare(n, methods, numels, &plans, &total, &act, &region_bytes);
  if (rc != ADACC_OK) return rc;
  if (act == 0) return ADACC_OK;
  if (!ws || !ws->device_mem) return ADACC_ENULL;
  const BatchPlan bp = batch_plan(act, region_bytes);
  if (ws->bytes < bp.bytes) return ADACC_ESIZE;
  if (misaligned(ws->device_mem, 256)) return ADACC_EALIGN;
  unsigned char* mem = static_cast<unsigned char*>(ws->device_mem);
  std::vector<TensorDesc> descs;
  std::vector<uint32_t> origin;
  rc = batch_table(n, methods, plans, numels, srcs, blobs, blob_bytes, nullptr, true, mem + bp.regions_off, &descs,
                   &origin);
  if (rc != ADACC_OK) return rc;  // every argument is checked before the device is touched
  int cus = 0;
  rc = device_cus(&cus);
  if (rc != ADACC_OK) return rc;
  // the launches: tiles (by register class), block sums, placement
  const uint32_t nt = (uint32_t)descs.size();
  std::vector<uint32_t> units(nt), members;
  std::vector<int> kind(nt);
  std::vector<GroupLaunch> tiles, sums, places;
  // (tensors that go through the fallback kernels are launched one by one, after the others)
  for (uint32_t i = 0; i < nt; ++i) {
    units[i] = descs[i].generic ? 0u : tile_waves(plans[origin[i]]);
    kind[i] = batch_kind(&methods[origin[i]], plans[origin[i]]) + (plans[origin[i]].half ? kBatchKinds : 0);
  }
  group_launches(units, kind, &members, &tiles, kTilesTogether);
  // The table goes up in the order of the tile launches' member lists, so that the tile kernels find the entry
  // of blockIdx.y at table + first_member without looking a number up first; the other kernels keep their lists.
  const uint32_t n_listed = (uint32_t)members.size();
  std::vector<uint32_t> place(nt, 0xFFFFFFFFu);
  std::vector<TensorDesc> ordered;
  ordered.reserve(nt);
  for (uint32_t j = 0; j < n_listed; ++j) { place[members[j]] = j; ordered.push_back(descs[members[j]]); }
  for (uint32_t i = 0; i < nt; ++i)
    if (place[i] == 0xFFFFFFFFu) { place[i] = (uint32_t)ordered.size(); ordered.push_back(descs[i]); }
  for (uint32_t i = 0; i < nt; ++i) {
    units[i] = (!descs[i].generic && needs_block_sums(&methods[origin[i]], plans[origin[i]])) ? blocks_of(descs[i].n_tiles, kSumTiles) : 0u;
    kind[i] = plans[origin[i]].half ? kBatchKinds : 0;
  }
  group_launches(units, kind, &members, &sums, kPlaceTogether);
  for (uint32_t i = 0; i < nt; ++i) units[i] = descs[i].generic ? 0u : place_grid(&methods[origin[i]], plans[origin[i]]);
  group_launches(units, kind, &members, &places, kPlaceTogether);
  for (uint32_t j = n_listed; j < (uint32_t)members.size(); ++j) members[j] = place[members[j]];
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  use_workspace(ws, bp.bytes);
  uint32_t epoch = 0;
  rc = next_epoch(ws, s, &epoch);
  if (rc != ADACC_OK) return rc;
  TensorDesc* dt = reinterpret_cast<TensorDesc*>(mem);
  uint32_t* dm = reinterpret_cast<uint32_t*>(mem + bp.members_off);
  rc = upload_batch(ordered, members.size() > n_listed ? members : std::vector<uint32_t>(), bp.members_off, mem, s);
  if (rc != ADACC_OK) return rc;
  for (const GroupLaunch& g : tiles)
    hipLaunchKernelGGL(compress_batch_fn(g.kind >= kBatchKinds, g.kind % kBatchKinds),
                       dim3((g.max_units + kWavesPerWg - 1) / kWavesPerWg, g.n_members),
                       dim3(kThreads), 0, s, dt + g.first_member, epoch);
  rc = launch_check("compress_batch_kernel");
  if (rc != ADACC_OK) return rc;
  for (const GroupLaunch& g : sums)
    hipLaunchKernelGGL(ADACC_PICK(g.kind >= kBatchKinds, place_sum_batch_fn()), dim3(g.max_units, g.n_members), dim3(kPlaceThreads), 0, s, dt,
                       dm + g.first_member);
  for (const GroupLaunch& g : places)
    hipLaunchKernelGGL(ADACC_PICK(g.kind >= kBatchKinds, place_batch_fn()), dim3(g.max_units, g.n_members), dim3(kPlaceThreads), 0, s, dt,
                       dm + g.first_member, epoch);
  rc = launch_check("place_batch_kernel");
  if (rc != ADACC_OK) return rc;
  for (uint32_t i = 0; i < nt && rc == ADACC_OK; ++i)
    if (descs[i].generic) rc = launch_generic_compress(&methods[origin[i]], plans[origin[i]], descs[i], epoch, s);
  return rc;
}

int adacc_decompress_batch(uint32_t n, const adacc_method* methods, const void* const* blobs, const uint64_t* blob_bytes,
                           const uint64_t* numels, void* const* dsts, int dst_dtype, adacc_workspace* ws,
                           void* hip_stream) {
  if (n == 0) return ADACC_OK;
  if (!methods || !blobs || !numels || !dsts || !blob_bytes) return ADACC_ENULL;
  if (dst_dtype != ADACC_DST_16 && dst_dtype != ADACC_DST_F32) return ADACC_EINVAL;
  std::vector<Plan> plans;
  uint32_t total = 0, act = 0;
  uint64_t region_bytes = 0;
  int rc = batch_prepare(n, methods, numels, &plans, &total, &act, &region_bytes);
  if (rc != ADACC_OK) return rc;
  if (act == 0) return ADACC_OK;
  if (!ws || !ws->device_mem) return ADACC_ENULL;
  const BatchPlan bp = batch_plan(act, region_bytes);
  if (ws->bytes < bp.bytes) return ADACC_ESIZE;
  if (misaligned(ws->device_mem, 256)) return ADACC_EALIGN;
  std::vector<TensorDesc> descs;
  std::vector<uint32_t> origin;
  rc = batch_table(n, methods, plans, numels, nullptr, const_cast<void* const*>(blobs), blob_bytes, dsts,
                   false, nullptr, &descs, &origin);
  if (rc != ADACC_OK) return rc;
  int cus = 0;
  rc = device_cus(&cus);
  if (rc != ADACC_OK) return rc;
  const uint32_t nt = (uint32_t)descs.size();
  std::vector<uint32_t> units(nt), members;
  std::vector<int> kind(nt, 0);
  std::vector<GroupLaunch> launches;
  for (uint32_t i = 0; i < nt; ++i) {
    units[i] = descs[i].generic ? 0u : descs[i].n_tiles;  // pieces of 2048 elements
    kind[i] = plans[origin[i]].half ? kBatchKinds : 0;
  }
  group_launches(units, kind, &members, &launches, kTilesTogether);
  // The table goes up in the order of the launches, so that the kernels find the entry of blockIdx.y at table +
  // first_member without looking a number up first.  (Tensors with groups that the batch kernel does not take are
  // launched one by one.)
  std::vector<TensorDesc> ordered;
  ordered.reserve(members.size());
  for (const uint32_t i : members) ordered.push_back(descs[i]);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  use_workspace(ws, bp.bytes);
  TensorDesc* dt = static_cast<TensorDesc*>(ws->device_mem);
  rc = upload_batch(ordered, std::vector<uint32_t>(), 0, dt, s);
  if (rc != ADACC_OK) return rc;
  for (const GroupLaunch& g : launches)
    hipLaunchKernelGGL(ADACC_PICK(g.kind >= kBatchKinds, decompress_batch_fn(dst_dtype == ADACC_DST_F32)),
                       dim3((g.max_units + kWavesPerWg - 1) / kWavesPerWg, g.n_members), dim3(kThreads), 0, s,
                       dt + g.first_member);
  rc = launch_check("decompress_batch_kernel");
  for (uint32_t i = 0; i < nt && rc == ADACC_OK; ++i)
    if (descs[i].generic) rc = launch_decompress(&methods[origin[i]], plans[origin[i]], descs[i], dst_dtype, s);
  return rc;
}

int adacc_read_status(const void* blob, const adacc_layout* layout, void* hip_stream, uint32_t status_out[4]) {
  if (!blob || !layout || !status_out) return ADACC_ENULL;
  if (layout->total_bytes == 0) { status_out[0] = status_out[1] = status_out[2] = status_out[3] = 0; return ADACC_OK; }
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  hipError_t e = hipMemcpyAsync(status_out, static_cast<const unsigned char*>(blob) + layout->status_off, 16,
                                hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(status)");
  e = hipStreamSynchronize(s);
  return e == hipSuccess ? ADACC_OK : hip_fail(e, "hipStreamSynchronize");
}

int adacc_channel_layout_of(const adacc_channel_method* method, uint64_t tokens, uint32_t hidden,
                            adacc_channel_layout* out) {
  if (!method || !out) return ADACC_ENULL;
  ChannelPlan cp;
  const int rc = make_channel_plan(method, tokens, hidden, &cp);
  if (rc != ADACC_OK) return rc;
  fill_channel_layout(method, tokens, hidden, cp, out);
  return ADACC_OK;
}

uint64_t adacc_channel_workspace_bytes(uint64_t tokens, uint32_t hidden) {
  if (hidden < 8 || hidden > 65536 || hidden % 8 != 0 || tokens > 0xFFFFFFFFull / hidden) return 0;
  const uint32_t n_chunks = (uint32_t)((tokens + kChunkTokens - 1) / kChunkTokens);
  return channel_partial_bytes(n_chunks, hidden) + align256(8ull * hidden);
}

int adacc_channel_compress(const adacc_channel_method* method, const void* src, uint64_t tokens, uint32_t hidden,
                           void* blob, uint64_t blob_bytes, void* workspace, uint64_t workspace_bytes,
                           void* hip_stream) {
  if (!method) return ADACC_ENULL;
  ChannelPlan cp;
  int rc = make_channel_plan(method, tokens, hidden, &cp);
  if (rc != ADACC_OK) return rc;
  if (tokens == 0) return ADACC_OK;
  if (!src || !blob || !workspace) return ADACC_ENULL;
  adacc_channel_layout L;
  fill_channel_layout(method, tokens, hidden, cp, &L);
  if (blob_bytes < L.total_bytes) return ADACC_ESIZE;
  if (workspace_bytes < adacc_channel_workspace_bytes(tokens, hidden)) return ADACC_ESIZE;
  if (misaligned(src, 16) || misaligned(blob, 256) || misaligned(workspace, 256)) return ADACC_EALIGN;
  TensorDesc d;
  fill_desc(&cp.quant, cp.numel, cp.plan, cp.quant_layout, src, blob, nullptr, nullptr, &d);
  ChannelDesc c;
  fill_channel_desc(method, tokens, hidden, L, blob, &c);
  d.status = c.status;  // (octets behind the matrix's end go to the unused part of this block; the plain blob's has the channel mask in its place)
  float* partial = static_cast<float*>(workspace);
  double* S = reinterpret_cast<double*>(static_cast<unsigned char*>(workspace) + channel_partial_bytes(cp.n_chunks, hidden));
  const bool half = cp.plan.half;
  // strips of 512 channels where the matrix and the groups allow them, else tiles of 2048 consecutive elements
  const bool by_strips = cp.plan.rowwise && hidden % 512u == 0;
  ChannelFn fn = by_strips ? ADACC_PICK(half, channel_compress_strip_fn(method->bits, method->asym))
                           : ADACC_PICK(half, channel_compress_fn(method->bits, method->asym, cp.plan.rowwise));
  const uint32_t grid = by_strips ? strip_grid(tokens, hidden, ADACC_PICK(half, channel_strip_rows())) : blocks_of(cp.plan.n_tiles, kWavesPerWg);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  const uint32_t strips = (hidden / 8 + kWave - 1) / kWave;  // a workgroup: one chunk of a strip of 512 channels
  hipLaunchKernelGGL(ADACC_PICK(half, channel_partial_fn(2ull * cp.numel > kStatsKeepBytes)), dim3(cp.n_chunks * strips),
                     dim3(ADACC_PICK(half, channel_partial_threads())), 0, s, static_cast<const uint16_t*>(src), (uint32_t)tokens,
                     hidden, partial, strips);
  rc = launch_check("channel_partial_kernel");
  if (rc != ADACC_OK) return rc;
  const bool few = cp.n_chunks <= kFewChunks && hidden <= kFewHidden;
  if (!few) {
    const uint32_t per_wg = ADACC_PICK(half, channel_score_channels());
    hipLaunchKernelGGL(ADACC_PICK(half, channel_score_fn()), dim3((hidden + per_wg - 1) / per_wg), dim3(kThreads), 0, s,
                       static_cast<const float*>(partial), cp.n_chunks, hidden, S);
    rc = launch_check("channel_score_kernel");
    if (rc != ADACC_OK) return rc;
  }
  hipLaunchKernelGGL(ADACC_PICK(half, channel_select_fn(few)), dim3(1), dim3(ADACC_PICK(half, channel_select_threads())), 0, s,
                     static_cast<const double*>(S), c, static_cast<const float*>(partial), cp.n_chunks);
  rc = launch_check("channel_select_kernel");
  if (rc != ADACC_OK) return rc;
  hipLaunchKernelGGL(fn, dim3(grid), dim3(kThreads), 0, s, d, c);
  return launch_check("channel_compress_kernel");
}

int adacc_channel_decompress(const adacc_channel_method* method, const void* blob, uint64_t blob_bytes,
                             uint64_t tokens, uint32_t hidden, void* dst, int dst_dtype, void* hip_stream) {
  if (!method) return ADACC_ENULL;
  if (dst_dtype != ADACC_DST_16 && dst_dtype != ADACC_DST_F32) return ADACC_EINVAL;
  ChannelPlan cp;
  int rc = make_channel_plan(method, tokens, hidden, &cp);
  if (rc != ADACC_OK) return rc;
  if (tokens == 0) return ADACC_OK;
  if (!blob || !dst) return ADACC_ENULL;
  adacc_channel_layout L;
  fill_channel_layout(method, tokens, hidden, cp, &L);
  if (blob_bytes < L.total_bytes) return ADACC_ESIZE;
  if (misaligned(dst, 16) || misaligned(blob, 256)) return ADACC_EALIGN;
  TensorDesc d;
  fill_desc(&cp.quant, cp.numel, cp.plan, cp.quant_layout, nullptr, const_cast<void*>(blob), dst, nullptr, &d);
  ChannelDesc c;
  fill_channel_desc(method, tokens, hidden, L, const_cast<void*>(blob), &c);
  ChannelFn fn = ADACC_PICK(cp.plan.half, channel_decompress_fn(method->bits, method->asym, dst_dtype == ADACC_DST_F32));
  const uint32_t grid = strip_grid(tokens, hidden, ADACC_PICK(cp.plan.half, channel_strip_rows()), strip_width(dst_dtype));
  hipLaunchKernelGGL(fn, dim3(grid), dim3(kThreads), 0, static_cast<hipStream_t>(hip_stream), d, c);
  return launch_check("channel_decompress_kernel");
}

int adacc_channel_read_status(const void* blob, const adacc_channel_layout* layout, void* hip_stream,
                              uint32_t status_out[4]) {
  if (!blob || !layout || !status_out) return ADACC_ENULL;
  if (layout->total_bytes == 0) return ADACC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  hipError_t e = hipMemcpyAsync(status_out, static_cast<const unsigned char*>(blob) + layout->status_off, 16,
                                hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync(status)");
  e = hipStreamSynchronize(s);
  return e == hipSuccess ? ADACC_OK : hip_fail(e, "hipStreamSynchronize");
}

// ---- channel-wise symmetric quantisation (Section 3.2, Query / Key / Value)
static bool channelwise_sizes_ok(uint32_t bits, uint64_t tokens, uint32_t hidden) {
  if (bits != 4 && bits != 8) return false;
  if (hidden < 8 || hidden > 65536 || hidden % 8 != 0) return false;
  return tokens <= 0xFFFFFFFFull / hidden;
}

static void channelwise_layout(uint32_t bits, uint64_t tokens, uint32_t hidden, adacc_channelwise_layout* L) {
  L->codes_off = 0;
  L->scales_off = align256(tokens * hidden * bits / 8);
  L->total_bytes = L->scales_off + align256(4ull * hidden);
}

static uint64_t channelwise_partial_bytes(uint64_t tokens, uint32_t hidden) {
  return align256(2ull * ((tokens + kChunkTokens - 1) / kChunkTokens) * hidden);
}

int adacc_channelwise_layout_of(uint32_t bits, uint64_t tokens, uint32_t hidden, adacc_channelwise_layout* out) {
  if (!out) return ADACC_ENULL;
  if (!channelwise_sizes_ok(bits, tokens, hidden)) return ADACC_EINVAL;
  channelwise_layout(bits, tokens, hidden, out);
  return ADACC_OK;
}

uint64_t adacc_channelwise_workspace_bytes(uint64_t tokens, uint32_t hidden) {
  if (!channelwise_sizes_ok(8, tokens, hidden)) return 0;
  return channelwise_partial_bytes(tokens, hidden) + align256(4ull * hidden);
}

static void channelwise_desc(uint32_t bits, uint32_t scale_rule, uint64_t tokens, uint32_t hidden,
                             const adacc_channelwise_layout& L, void* blob, ChannelwiseDesc* c) {
  std::memset(c, 0, sizeof *c);
  unsigned char* b = static_cast<unsigned char*>(blob);
  c->codes = b + L.codes_off;
  c->scales = reinterpret_cast<float*>(b + L.scales_off);
  c->numel = tokens * hidden;
  c->tokens = (uint32_t)tokens;
  c->hidden = hidden;
  c->n_chunks = (uint32_t)((tokens + kChunkTokens - 1) / kChunkTokens);
  const float q = (float)(1u << (bits - 1));
  c->divisor = scale_rule == ADACC_SCALE_PAPER ? q : q - 1.0f;
  c->inv_divisor = scale_rule == ADACC_SCALE_PAPER ? 1.0f / q : 0.0f;  // exact for a power of two
}

int adacc_channelwise_compress(uint32_t bits, uint32_t scale_rule, uint32_t dtype, const void* src, uint64_t tokens,
                               uint32_t hidden, void* blob, uint64_t blob_bytes, void* workspace,
                               uint64_t workspace_bytes, void* hip_stream) {
  if (!channelwise_sizes_ok(bits, tokens, hidden) || scale_rule > 1 || dtype > ADACC_DTYPE_F16) return ADACC_EINVAL;
  const bool half = dtype == ADACC_DTYPE_F16;
  if (tokens == 0) return ADACC_OK;
  if (!src || !blob || !workspace) return ADACC_ENULL;
  adacc_channelwise_layout L;
  channelwise_layout(bits, tokens, hidden, &L);
  if (blob_bytes < L.total_bytes) return ADACC_ESIZE;
  if (workspace_bytes < adacc_channelwise_workspace_bytes(tokens, hidden)) return ADACC_ESIZE;
  if (misaligned(src, 16) || misaligned(blob, 256) || misaligned(workspace, 256)) return ADACC_EALIGN;
  ChannelwiseDesc c;
  channelwise_desc(bits, scale_rule, tokens, hidden, L, blob, &c);
  c.src = static_cast<const uint16_t*>(src);
  c.partial = static_cast<uint16_t*>(workspace);
  c.inv = reinterpret_cast<float*>(static_cast<unsigned char*>(workspace) + channelwise_partial_bytes(tokens, hidden));
  ChannelwiseFn quant = ADACC_PICK(half, channelwise_quantise_fn(bits));
  const uint32_t grid = strip_grid(tokens, hidden, ADACC_PICK(half, channelwise_strip_rows(false, c.numel)));
  int rc = ADACC_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const uint32_t strips = (hidden / 8 + kWave - 1) / kWave;  // a workgroup: one chunk of a strip of 512 channels
  hipLaunchKernelGGL(ADACC_PICK(half, channelwise_partial_fn(2ull * c.numel > kStatsKeepBytes)), dim3(c.n_chunks * strips),
                     dim3(ADACC_PICK(half, channelwise_partial_threads())), 0, s, c, strips);
  rc = launch_check("channelwise_partial_kernel");
  if (rc != ADACC_OK) return rc;
  const uint32_t per_wg = ADACC_PICK(half, channelwise_fold_octets());
  hipLaunchKernelGGL(ADACC_PICK(half, channelwise_fold_fn()), dim3((hidden / 8 + per_wg - 1) / per_wg), dim3(kThreads), 0, s, c);
  rc = launch_check("channelwise_fold_kernel");
  if (rc != ADACC_OK) return rc;
  hipLaunchKernelGGL(quant, dim3(grid), dim3(kThreads), 0, s, c);
  return launch_check("channelwise_quantise_kernel");
}

int adacc_channelwise_decompress(uint32_t bits, uint32_t dtype, const void* blob, uint64_t blob_bytes, uint64_t tokens,
                                 uint32_t hidden, void* dst, int dst_dtype, void* hip_stream) {
  if (dst_dtype != ADACC_DST_16 && dst_dtype != ADACC_DST_F32) return ADACC_EINVAL;
  if (dtype > ADACC_DTYPE_F16) return ADACC_EINVAL;
  if (!channelwise_sizes_ok(bits, tokens, hidden)) return ADACC_EINVAL;
  if (tokens == 0) return ADACC_OK;
  if (!blob || !dst) return ADACC_ENULL;
  adacc_channelwise_layout L;
  channelwise_layout(bits, tokens, hidden, &L);
  if (blob_bytes < L.total_bytes) return ADACC_ESIZE;
  if (misaligned(dst, 16) || misaligned(blob, 256)) return ADACC_EALIGN;
  ChannelwiseDesc c;
  channelwise_desc(bits, 0, tokens, hidden, L, const_cast<void*>(blob), &c);
  c.dst = dst;
  ChannelwiseFn fn = ADACC_PICK(dtype == ADACC_DTYPE_F16, channelwise_dequantise_fn(bits, dst_dtype == ADACC_DST_F32));
  c.strip_rows = ADACC_PICK(dtype == ADACC_DTYPE_F16, channelwise_strip_rows(true, c.numel));
  const uint32_t grid = strip_grid(tokens, hidden, c.strip_rows, strip_width(dst_dtype));
  hipLaunchKernelGGL(fn, dim3(grid), dim3(kThreads), 0, static_cast<hipStream_t>(hip_stream), c);
  return launch_check("channelwise_dequantise_kernel");
}

uint64_t adacc_mask_packed_bytes(uint64_t n) { return (n + 7u) / 8u; }

static int mask_launch(MaskFn fn, const void* in, uint64_t n, void* out, void* hip_stream, const char* what) {
  if (n == 0) return ADACC_OK;
  if (!in || !out) return ADACC_ENULL;
  if (misaligned(in, 16) || misaligned(out, 16)) return ADACC_EALIGN;
  int cus = 0;
  const int rc = device_cus(&cus);
  if (rc != ADACC_OK) return rc;
  const uint64_t pieces = n / 16u;  // one lane turns over 16 elements at a time, kMaskAhead times per round
  constexpr uint64_t per = (uint64_t)kMaskAhead * kThreads;
  uint64_t grid = (pieces + per - 1) / per;
  const uint64_t cap = (uint64_t)cus * (uint64_t)knobs().mask_wgs_per_cu;
  if (grid > cap) grid = cap;
  if (grid == 0) grid = 1;
  hipLaunchKernelGGL(fn, dim3((uint32_t)grid), dim3(kThreads), 0, static_cast<hipStream_t>(hip_stream),
                     static_cast<const uint8_t*>(in), n, static_cast<uint8_t*>(out));
  return launch_check(what);
}

int adacc_mask_pack(const void* mask, uint64_t n, void* bits, void* hip_stream) {
  return mask_launch(mask_pack_fn(), mask, n, bits, hip_stream, "mask_pack_kernel");
}

int adacc_mask_unpack(const void* bits, uint64_t n, void* mask, void* hip_stream) {
  return mask_launch(mask_unpack_fn(), bits, n, mask, hip_stream, "mask_unpack_kernel");
}

uint64_t adacc_compressed_bytes(const adacc_method* method, uint64_t numel, uint64_t n_outliers) {
  if (!method) return 0;
  Plan p;
  if (make_plan(method, numel, &p) != ADACC_OK) return 0;
  if (p.noop) return 2ull * numel;
  const uint64_t groups = (numel + method->quant_group - 1) / method->quant_group;
  uint64_t bytes = (numel * method->bits + 7) / 8 + 4ull * groups * (method->asym ? 2u : 1u);
  if (p.outliers) bytes += 6ull * n_outliers + 4ull * ((uint64_t)p.n_tiles_all + 1u);
  return bytes;
}

uint64_t adacc_channel_compressed_bytes(const adacc_channel_method* method, uint64_t tokens, uint32_t hidden,
                                        uint64_t n_channels) {
  if (!method) return 0;
  ChannelPlan cp;
  if (make_channel_plan(method, tokens, hidden, &cp) != ADACC_OK) return 0;
  const uint64_t numel = tokens * hidden;
  const uint64_t groups = numel / method->quant_group;
  return numel * method->bits / 8 + 4ull * groups * (method->asym ? 2u : 1u) + n_channels * (2ull * tokens + 4u);
}

int adacc_hbm_stream(int mix, void* dst, const void* src_a, const void* src_b, uint64_t bytes, void* hip_stream) {
  if (mix < ADACC_STREAM_READ || mix > ADACC_STREAM_READ2_WRITE) return ADACC_EINVAL;
  const bool wr = mix != ADACC_STREAM_READ, rd = mix != ADACC_STREAM_WRITE, rd2 = mix == ADACC_STREAM_READ2_WRITE;
  if ((wr && !dst) || (rd && !src_a) || (rd2 && !src_b)) return ADACC_ENULL;
  if (bytes % 16 != 0) return ADACC_EINVAL;
  if ((wr && misaligned(dst, 16)) || (rd && misaligned(src_a, 16)) || (rd2 && misaligned(src_b, 16))) return ADACC_EALIGN;
  if (bytes == 0) return ADACC_OK;
  const uint64_t n16 = bytes / 16;
  const uint64_t grid = (n16 + 1023u) / 1024u;  // a workgroup moves 4 x 4 KiB per operand
  if (grid >= (1ull << 31)) return ADACC_EINVAL;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  uint4* d = static_cast<uint4*>(dst);
  const uint4* a = static_cast<const uint4*>(src_a);
  const uint4* b = static_cast<const uint4*>(src_b);
  switch (mix) {
    case ADACC_STREAM_READ: hipLaunchKernelGGL(hbm_stream_kernel<0>, dim3((uint32_t)grid), dim3(kThreads), 0, s, d, a, b, n16, static_cast<uint32_t*>(dst)); break;
    case ADACC_STREAM_WRITE: hipLaunchKernelGGL(hbm_stream_kernel<1>, dim3((uint32_t)grid), dim3(kThreads), 0, s, d, a, b, n16, nullptr); break;
    case ADACC_STREAM_COPY: hipLaunchKernelGGL(hbm_stream_kernel<2>, dim3((uint32_t)grid), dim3(kThreads), 0, s, d, a, b, n16, nullptr); break;
    default: hipLaunchKernelGGL(hbm_stream_kernel<3>, dim3((uint32_t)grid), dim3(kThreads), 0, s, d, a, b, n16, nullptr); break;
  }
  return launch_check("hbm_stream_kernel");
}

int adacc_hbm_copy(void* dst, const void* src, uint64_t bytes, void* hip_stream) {
  return adacc_hbm_stream(ADACC_STREAM_COPY, dst, src, nullptr, bytes, hip_stream);
}

}  // extern "C"
