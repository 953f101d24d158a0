// Compression of one tile by one wavefront (Section 3.2, Fig. 3(c) compression workflow):
// load -> statistics -> outlier mask -> zero the outliers -> group scale (Eq. 2 / Eq. 3)
// -> quantise, pack, store -> ordered append of the outliers to the (index, value) stream.
//
// The kernel is bound by vector-ALU issue as much as by HBM (about 20 lane-operations per
// element are affordable at 70 % of peak bandwidth), so the common case - a row of 512
// elements without any outlier - is kept to the operations that can not be avoided, and
// everything that only matters when outliers are present sits behind wavefront-uniform
// branches.
#pragma once

#include <type_traits>

#include "adacc_common.hpp"
#include "adacc_dtype.hpp"

namespace adacc {
namespace ADACC_DT_NS {

// ------------------------------------------------------------------ small helpers
__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// element e (0..7) of an octet held in 4 dwords
#define ADACC_ELEM_F32(oct, e) (((e)&1) ? widen_hi((oct)[(e) >> 1]) : widen_lo((oct)[(e) >> 1]))
#define ADACC_ELEM_MAG(oct, e) ((((e)&1) ? ((oct)[(e) >> 1] >> 16) : (oct)[(e) >> 1]) & 0x7FFFu)

// compile-time loop: body(std::integral_constant<int, J>) for J = 0..N-1.  Used where a
// data-dependent inner loop would otherwise keep the compiler from unrolling, which would
// turn the per-row register arrays into scratch memory.
template <int N, int J = 0, class F>
__device__ __forceinline__ void static_for(F&& body) {
  if constexpr (J < N) {
    body(std::integral_constant<int, J>());
    static_for<N, J + 1>(body);
  }
}

struct OpAdd { __device__ __forceinline__ float operator()(float a, float b) const { return a + b; } };
struct OpMax { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct OpMin { __device__ __forceinline__ float operator()(float a, float b) const { return fminf(a, b); } };
struct OpUMax { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a > b ? a : b; } };
struct OpIMax { __device__ __forceinline__ int32_t operator()(int32_t a, int32_t b) const { return a > b ? a : b; } };
struct OpIMin { __device__ __forceinline__ int32_t operator()(int32_t a, int32_t b) const { return a < b ? a : b; } };

// Order-preserving map between finite floats and signed integers (and back: it is its own
// inverse).  Cross-lane max / min run on these integers: the integer instructions take the
// DPP lane permute as an operand, while a float max would first have to quiet a possible NaN.
__device__ __forceinline__ int32_t float_key(float f) {
  const int32_t u = (int32_t)__float_as_uint(f);
  return u ^ ((u >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float key_float(int32_t k) {
  return __uint_as_float((uint32_t)(k ^ ((k >> 31) & 0x7FFFFFFF)));
}

// value of the partner lane of one xor-butterfly step over 1, 2, 4 or 8 lanes: DPP lane permutes (they fuse into the
// arithmetic instruction).
// row_half_mirror / row_mirror stand in for xor 4 / xor 8: after the lower steps every
// value is uniform within its 4 resp. 8 lanes, so reversing the order is the same exchange.
template <int CTRL, class T>
__device__ __forceinline__ T dpp_move(T v) {
  const int i = __builtin_bit_cast(int, v);
  return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xF, 0xF, true));
}
// The steps over 16 and 32 lanes: STEP lanes of `a` change places with STEP lanes of `b`, so that an operation on the two
// then takes in every lane's partner: with a = b a step of the butterfly, with two different values a step of two
// butterflies at once, whose results lie STEP lanes apart (a: the groups of STEP lanes with an even number, b: odd).
// (gfx950 swaps lanes between registers; through the LDS crossbar each step was a round trip of some 60 clocks.)
template <int STEP, class T>
__device__ __forceinline__ void exchange(T& a, T& b) {
  static_assert(STEP == 16 || STEP == 32, "lanes of one row or one half");
  const uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
  if constexpr (STEP == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    a = __builtin_bit_cast(T, (uint32_t)r[0]); b = __builtin_bit_cast(T, (uint32_t)r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    a = __builtin_bit_cast(T, (uint32_t)r[0]); b = __builtin_bit_cast(T, (uint32_t)r[1]);
  }
}
template <int STEP, class T, class Op>
__device__ __forceinline__ T meet(T a, T b, Op op) {
  exchange<STEP>(a, b);
  return op(a, b);
}

// all-reduce over LANES adjacent lanes (power of two; every lane is active) by xor butterfly, masks 1, 2, 4, ...
// For sums the association is the balanced binary tree over lane order, which is what makes
// the variance a function of the input bits alone.
template <int LANES, class T, class Op>
__device__ __forceinline__ T lanes_reduce(T v, Op op) {
  if constexpr (LANES > 1) v = op(v, dpp_move<0xB1>(v));   // quad_perm [1,0,3,2]
  if constexpr (LANES > 2) v = op(v, dpp_move<0x4E>(v));   // quad_perm [2,3,0,1]
  if constexpr (LANES > 4) v = op(v, dpp_move<0x141>(v));  // row_half_mirror
  if constexpr (LANES > 8) v = op(v, dpp_move<0x140>(v));  // row_mirror
  if constexpr (LANES == 32) v = meet<16>(v, v, op);
  if constexpr (LANES == 64) {
    // The whole wavefront: rows 1 and 3 meet the row before them, row 3 meets row 1, and lane 63 goes to a scalar register: the same
    // sums in three instructions, where two exchanges take two moves each besides.  (The 32 largest of groups of 512, 2^25 values:
    // 121 us through the LDS crossbar, 131 by exchanges, 123 like this; STD over 512, asymmetric, 4 sigma 35.3 -> 32.9.)
    v = op(v, dpp_move<0x142>(v));  // row_bcast:15
    v = op(v, dpp_move<0x143>(v));  // row_bcast:31
    v = __builtin_bit_cast(T, (uint32_t)__builtin_amdgcn_readlane(__builtin_bit_cast(int, v), kWave - 1));
  }
  return v;
}

// Per-row, per-lane values -> those of groups of 2^lg elements, in every lane of the group.  lg <= 9: the group is
// 2^(lg-3) adjacent lanes of one row; sums are formed in the order of the balanced tree over lanes.  lg > 9: the group is
// 2^(lg-9) whole rows, combined in the lane first (for operations that any order suits).
// The group size is a run-time value of the method; one switch selects straight-line code for it, so that the
// butterflies themselves carry no branches.
template <int E, int LANES, class T, class Op>
__device__ __forceinline__ void each_row_reduce(T (&s)[E], Op op) {
#pragma unroll
  for (int j = 0; j < E; ++j) s[j] = lanes_reduce<LANES>(s[j], op);
}
template <int E, int R, class T, class Op>
__device__ __forceinline__ void row_groups_reduce(T (&s)[E], Op op) {
  if constexpr (R <= E) {
#pragma unroll
    for (int j = 0; j < E; j += R) {
#pragma unroll
      for (int i = 1; i < R; ++i) s[j] = op(s[j], s[j + i]);
      s[j] = lanes_reduce<kWave>(s[j], op);
#pragma unroll
      for (int i = 1; i < R; ++i) s[j + i] = s[j];
    }
  }
}
template <int E, class T, class Op>
__device__ __forceinline__ void groups_reduce(T (&s)[E], uint32_t lg, Op op) {
  switch (lg) {
    case 3: break;
    case 4: each_row_reduce<E, 2>(s, op); break;
    case 5: each_row_reduce<E, 4>(s, op); break;
    case 6: each_row_reduce<E, 8>(s, op); break;
    case 7: each_row_reduce<E, 16>(s, op); break;
    case 8: each_row_reduce<E, 32>(s, op); break;
    case 9: each_row_reduce<E, 64>(s, op); break;
    case 10: row_groups_reduce<E, 2>(s, op); break;
    default: row_groups_reduce<E, 4>(s, op); break;
  }
}
// one value, groups inside a row: LANES = 2^lg adjacent lanes, lg a run-time (uniform) value
template <class T, class Op>
__device__ __forceinline__ T lanes_reduce_lg(T v, uint32_t lg, Op op) {
  switch (lg) {
    case 0: break;
    case 1: v = lanes_reduce<2>(v, op); break;
    case 2: v = lanes_reduce<4>(v, op); break;
    case 3: v = lanes_reduce<8>(v, op); break;
    case 4: v = lanes_reduce<16>(v, op); break;
    case 5: v = lanes_reduce<32>(v, op); break;
    default: v = lanes_reduce<64>(v, op); break;
  }
  return v;
}
// The sums of four rows over all their lanes, row j's in the lanes 16 j .. 16 j + 15: the balanced tree over lane order, two
// rows sharing a step over 16 lanes and all four the one over 32.
template <class T, class Op>
__device__ __forceinline__ T four_rows_reduce(T r0, T r1, T r2, T r3, Op op) {
  const T r01 = meet<16>(lanes_reduce<16>(r0, op), lanes_reduce<16>(r1, op), op);
  const T r23 = meet<16>(lanes_reduce<16>(r2, op), lanes_reduce<16>(r3, op), op);
  return meet<32>(r01, r23, op);
}

// maximum over the whole wavefront, returned in a scalar register: four butterfly steps inside
// the rows of 16 lanes, two row broadcasts (lane 15 of rows 0 and 2 into rows 1 and 3, then
// lane 31 into rows 2 and 3), and lane 63 holds the result
__device__ __forceinline__ uint32_t wave_max_u32_scalar(uint32_t v) {
  v = lanes_reduce<16>(v, OpUMax());
  // rows that receive nothing read 0, the identity of the maximum, so each step is one instruction
  int t = __builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v = OpUMax()(v, (uint32_t)t);
  t = __builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);      // row_bcast:31
  v = OpUMax()(v, (uint32_t)t);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The largest t < 2^15 with count(t) >= k (0 if there is none), count falling in t: bit by bit, uniform.
template <class Count>
__device__ __forceinline__ uint32_t kth_by_halving(uint32_t k, Count count) {
  uint32_t t = 0u;
#pragma unroll
  for (int bit = 14; bit >= 0; --bit) {
    const uint32_t c = t | (1u << bit);
    t = count(c) >= k ? c : t;
  }
  return t;
}
// lanes for which v holds
__device__ __forceinline__ uint32_t lanes_where(bool v) { return (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(v)); }
// LDS takes a wavefront's accesses in order; this keeps the compiler from moving any of them across.
__device__ __forceinline__ void lds_in_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// number of set bits of a wavefront mask in the lanes below this one
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// ------------------------------------------------------------------ rounding and packing of codes
// code = clip(nearest integer of the binary32 product y * inv) (Eq. 2 / Eq. 3).  The product is
// rounded to binary32 by the multiplication (never fused with what follows: the library is built
// with contraction off); adding 1.5 * 2^23 then rounds it to the nearest integer (ties to even)
// and leaves that integer, in two's complement, in the low mantissa bits; the clip is a median
// with the two bounds shifted the same way ("values greater than 7 are capped at 7"); a NaN
// lands on the lower bound.
// Symmetric codes need the upper bound only (pack_codes): |y| <= max and inv = RN(D / max) (or less, when that was
// cut to the largest finite value) give |y * inv| <= D * (1 + 2^-24), which rounds to at most D <= Q in
// magnitude, -Q is a code, and neither factor can be a NaN or infinite.  (Asymmetric codes keep both
// bounds: a group of huge values can make O infinite and the product a NaN.)
constexpr float kMagic = 12582912.0f;
template <int Q>
__device__ __forceinline__ uint32_t code_bits(float p) {
  return __float_as_uint(fminf(fmaxf(__fadd_rn(p, kMagic), kMagic - (float)Q), kMagic + (float)(Q - 1)));
}

typedef short i16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_min_i16(uint32_t a, int16_t bound) {
  const i16x2_t q = {bound, bound};
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(i16x2_t, a), q));
}
// The codes of an octet from its products y * inv, packed: 8 bytes in w[0], w[1], or 8 nibbles in w[0] (element e in nibble e).  Two codes meet
// in the halves of a word first, e and e + 2 resp. e and e + 4; symmetric codes are clipped there, two at a time
// (|code| <= D before the clip: 16 bits hold it), asymmetric ones before (their products know no bound).
template <int BITS, bool ASYM>
__device__ __forceinline__ void pack_codes(const float (&p)[kOct], uint32_t (&w)[2]) {
  constexpr int Q = 1 << (BITS - 1);
  uint32_t c[kOct];
#pragma unroll
  for (int e = 0; e < kOct; ++e) c[e] = ASYM ? code_bits<Q>(p[e]) : __float_as_uint(__fadd_rn(p[e], kMagic));
  constexpr int STEP = BITS == 8 ? 2 : 4;
  uint32_t h[4];  // BITS 8: (0,2) (1,3) (4,6) (5,7); BITS 4: (0,4) (1,5) (2,6) (3,7)
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = BITS == 8 ? (i >> 1) * 4 + (i & 1) : i;
    h[i] = __builtin_amdgcn_perm(c[e + STEP], c[e], 0x05040100u);  // the low halves
    if constexpr (!ASYM) h[i] = pk_min_i16(h[i], (int16_t)(Q - 1));
  }
  if constexpr (BITS == 8) {
    w[0] = __builtin_amdgcn_perm(h[1], h[0], 0x06020400u);
    w[1] = __builtin_amdgcn_perm(h[3], h[2], 0x06020400u);
  } else {
    const uint32_t t01 = (h[0] & 0x000F000Fu) | ((h[1] << 4) & ~0x000F000Fu);
    const uint32_t t23 = (h[2] & 0x000F000Fu) | ((h[3] << 4) & ~0x000F000Fu);
    w[0] = (t01 & 0x00FF00FFu) | ((t23 << 8) & ~0x00FF00FFu);
    w[1] = 0u;
  }
}

// ------------------------------------------------------------------ tile geometry, loads and stores
// A tile is addressed as a wavefront-uniform base (kept in scalar registers) plus a 32-bit
// lane offset, so that address arithmetic costs no vector instructions.
// STRIP: the E rows of 512 elements are not adjacent in memory but `stride` elements apart (rows of a
// matrix: a strip of 512 columns); such a tile is always complete, and base, stride are multiples of 512.
template <int E, bool STRIP = false>
struct TileGeo {
  uint64_t base;      // uniform: index of the tile's first element
  uint32_t rem;       // uniform: elements of the tensor from `base` on, at most E*512 (a multiple of 8, > 0)
  uint32_t lane_off;  // lane * 8
  bool full;          // known to the compiler: rem is E*512 (else it may be less)
  uint32_t stride;    // uniform, STRIP only: elements from one row to the next
  __device__ __forceinline__ uint32_t row_offset(int j) const {
    if constexpr (STRIP) return (uint32_t)j * stride;
    else return (uint32_t)(j * kRow);
  }
};
// COMPLETE: the caller knows that every tile of the tensor is complete (the tile is a statistics
// group, and group sizes divide the tensor), so nothing about short tiles is computed or tested.
template <int E, bool COMPLETE = false>
__device__ __forceinline__ TileGeo<E> tile_geo(const TensorDesc& d, uint32_t tile) {
  TileGeo<E> g;
  g.base = (uint64_t)tile * (uint64_t)(E * kRow);
  g.lane_off = (uint32_t)lane_id() * kOct;
  g.stride = (uint32_t)kRow;
  if constexpr (COMPLETE) {
    g.rem = (uint32_t)(E * kRow);
    g.full = true;
  } else {
    const uint64_t left = d.numel - g.base;
    g.rem = left < (uint64_t)(E * kRow) ? (uint32_t)left : (uint32_t)(E * kRow);
    g.full = false;  // (known here, so that the code for the last tile holds no copy of that for the others)
  }
  return g;
}

// ---- a1: load (16 bytes per lane per row).  The loads are issued unconditionally (octets past
// the end of the tensor re-read its last octet and are blanked afterwards): a load under a
// branch would make the number of loads in flight unknown to the compiler's wait-count
// bookkeeping, which then waits for the prefetched tile together with the current one.
template <int E, bool COMPLETE = false>
__device__ __forceinline__ void load_tile(const TensorDesc& d, uint32_t tile, uint32_t (&raw)[E][4]) {
  const TileGeo<E> g = tile_geo<E, COMPLETE>(d, tile);
  const uint16_t* sp = d.src + g.base;
  const uint32_t last = g.rem - kOct;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    uint32_t off = g.lane_off + (uint32_t)(j * kRow);
    if constexpr (!COMPLETE) off = off < last ? off : last;
    const uint4 v = ADACC_LOAD16(sp + off);
    raw[j][0] = v.x; raw[j][1] = v.y; raw[j][2] = v.z; raw[j][3] = v.w;
  }
}
// blank the octets of a tile that lie past the end of the tensor (only a tensor's last tile can have any)
template <int E>
__device__ __forceinline__ void blank_tail(const TileGeo<E>& g, uint32_t (&raw)[E][4]) {
  if (g.full) return;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    if (g.lane_off + (uint32_t)(j * kRow) >= g.rem) raw[j][0] = raw[j][1] = raw[j][2] = raw[j][3] = 0u;
  }
}

// Makes the compiler forget everything it derived from the raw octets (their values do not
// change).  Between two phases that both widen the octets this keeps the 8 widened values per
// row from staying in registers all the way: forming them again costs one instruction each,
// keeping them costs a quarter of the wavefronts a SIMD can hold.
template <int E>
__device__ __forceinline__ void forget_derived(const uint32_t (&raw)[E][4]) {
  uint32_t(&r)[E][4] = const_cast<uint32_t(&)[E][4]>(raw);
#pragma unroll
  for (int j = 0; j < E; ++j) {
    asm volatile("" : "+v"(r[j][0]), "+v"(r[j][1]), "+v"(r[j][2]), "+v"(r[j][3]));
  }
}

// 16-bit format -> binary32 (exact)
__device__ __forceinline__ void widen_row(const uint32_t (&oct)[4], float (&x)[kOct]) {
#pragma unroll
  for (int e = 0; e < kOct; ++e) x[e] = ADACC_ELEM_F32(oct, e);
}

// ---- a8: store the codes of one octet and the scale (offset) of its group.  Every lane stores,
// always: a store under a branch would make the number of stores in flight unknown to the
// compiler's wait-count bookkeeping, and the wait for the prefetched tile would then also wait
// for these stores.  In a tensor's last tile, octets past the end go to a scrap area in the
// unused part of the blob's status block; all lanes of a group store their (identical) scale.
// y: the values to be quantised (asymmetric: less the offset)
template <int BITS, bool ASYM, int E, bool STRIP>
__device__ __forceinline__ void store_row(const TensorDesc& d, const TileGeo<E, STRIP>& g, int j,
                                          const float (&y)[kOct], float scl, float inv, float off) {
  // What differs from row to row is uniform: the lanes' offsets are the same two registers for all rows.  (Groups are
  // powers of two and rows multiples of 512, so that row and lane add up to the group's number separately.)
  const uint32_t ro = g.row_offset(j);  // uniform
  unsigned char* cp = d.codes + (g.base + ro) * BITS / 8;                       // uniform
  float* sp = d.scales + ((g.base >> d.lgq) + (uint64_t)(ro >> d.lgq));        // uniform
  float* zp = d.zp + ((g.base >> d.lgq) + (uint64_t)(ro >> d.lgq));
  const uint32_t co = g.lane_off * (uint32_t)BITS / 8u;
  const uint32_t gl = g.lane_off >> d.lgq;
  float p[kOct];
#pragma unroll
  for (int e = 0; e < kOct; ++e) p[e] = __fmul_rn(y[e], inv);
  uint32_t w[2];
  pack_codes<BITS, ASYM>(p, w);
  const uint2 w8 = make_uint2(w[0], w[1]);
  const uint32_t w4 = w[0];
  if (g.full) {
    if constexpr (BITS == 8) ADACC_STORE8(cp + co, w8);
    else ADACC_STORE4(cp + co, w4);
    sp[gl] = scl;
    if constexpr (ASYM) zp[gl] = off;
  } else {
    const bool valid = ro + g.lane_off < g.rem;
    unsigned char* scrap = reinterpret_cast<unsigned char*>(d.status) + 64;
    if constexpr (BITS == 8) ADACC_STORE8(valid ? cp + co : scrap, w8);
    else ADACC_STORE4(valid ? cp + co : scrap, w4);
    *(valid ? sp + gl : reinterpret_cast<float*>(scrap + 16)) = scl;
    if constexpr (ASYM) *(valid ? zp + gl : reinterpret_cast<float*>(scrap + 32)) = off;
  }
}

// ------------------------------------------------------------------ per-row pieces shared by both tile encoders
constexpr float kFltMax = 3.402823466e+38f;

// STD: limit = k^2 * var from the group's sums (population variance about the mean).
__device__ __forceinline__ float std_limit(float s1, float s2, float inv_gs, float k2) {
  const float mean = s1 * inv_gs;
  float var = __fmaf_rn(-mean, mean, s2 * inv_gs);
  var = (var < 0.0f) ? 0.0f : var;  // a NaN stays a NaN: then nothing passes the test
  return k2 * var;
}

// Bookkeeping of one row from the ballots of its 8 outlier tests: per-lane mask, number of the
// row's outliers in lower lanes, row count.  Only rows that have outliers do the work, and the
// usual such row - a few outliers, no two in one lane - does it mostly in scalar registers:
// the ballots live there, and a lane reads its own bit back as a select condition.
__device__ __forceinline__ void row_bookkeeping(const uint64_t (&b)[kOct], uint32_t& mask, uint32_t& lane_excl,
                                                uint32_t& row_cnt, bool& any_out, bool& sparse) {
  uint64_t any = 0ull;
#pragma unroll
  for (int e = 0; e < kOct; ++e) any |= b[e];
  any_out = any != 0ull;
  sparse = true;
  if (any_out) {
    uint32_t cnt = 0u;
#pragma unroll
    for (int e = 0; e < kOct; ++e) cnt += (uint32_t)__popcll(b[e]);
    row_cnt = cnt;
    sparse = cnt == (uint32_t)__popcll(any);
    uint32_t m = 0u;
    if (sparse) {
      lane_excl = lanes_below(any);
#pragma unroll
      for (int e = 0; e < kOct; ++e) m = __builtin_amdgcn_inverse_ballot_w64(b[e]) ? (1u << e) : m;  // at most one bit per lane
    } else {
      uint32_t below = 0u;
#pragma unroll
      for (int e = 0; e < kOct; ++e) {
        m |= __builtin_amdgcn_inverse_ballot_w64(b[e]) ? (1u << e) : 0u;
        below += lanes_below(b[e]);
      }
      lane_excl = below;
    }
    mask = m;
  } else {
    mask = 0u; lane_excl = 0u; row_cnt = 0u;
  }
}
// extremes of the inlier view of one octet: symmetric ext0 = max |y|; asymmetric ext0 = max y, ext1 = min y
template <bool ASYM>
__device__ __forceinline__ void row_extremes(const float (&y)[kOct], float& ext0, float& ext1) {
  float mx = ASYM ? y[0] : fabsf(y[0]), mn = y[0];
#pragma unroll
  for (int e = 1; e < kOct; ++e) {
    if constexpr (ASYM) { mx = fmaxf(mx, y[e]); mn = fminf(mn, y[e]); }
    else mx = fmaxf(mx, fabsf(y[e]));
  }
  ext0 = mx; ext1 = mn;
}

// ---- a6: scale, reciprocal and offset of a group from its reduced extremes (Eq. 2 / Eq. 3)
template <bool ASYM>
__device__ __forceinline__ void group_scale(const TensorDesc& d, uint32_t r0, int32_t k0, int32_t k1, float& scl,
                                            float& inv, float& off) {
  if constexpr (!ASYM) {
    const float am = __uint_as_float(r0);
    // Eq. 2: S = max|X| / D.  For a power-of-two D the division is a multiplication by 1/D, same bits
    scl = d.inv_divisor != 0.0f ? am * d.inv_divisor : am / d.divisor;
    inv = (am != 0.0f) ? fminf(d.divisor / am, kFltMax) : 0.0f;  // one division per group
    off = 0.0f;
  } else {
    // a zero extreme is +0 whatever signs the zeros had
    const float h = key_float(k0) + 0.0f, l = key_float(k1) + 0.0f;
    off = (h + l) * 0.5f;  // Eq. 3: O = (max+min)/2
    const float r = h - l;
    scl = d.inv_divisor != 0.0f ? r * d.inv_divisor : r / d.divisor;  // Eq. 3: S = (max-min) / D2
    inv = (r != 0.0f) ? fminf(d.divisor / r, kFltMax) : 0.0f;
  }
}

__device__ __forceinline__ bool is_nonfinite(float x) { return (__float_as_uint(x) & 0x7FFFFFFFu) >= 0x7F800000u; }

// ---- a4: where the outliers of a tile go.  Entry `pos` of the stream of the blob (two arrays) ...
struct StreamSink {
  int32_t* idx;
  uint16_t* val;
  __device__ __forceinline__ void operator()(uint32_t pos, uint32_t index, uint32_t bits) const {
    idx[pos] = (int32_t)index;
    val[pos] = (uint16_t)bits;
  }
};
// ... or of a tile's slot in the workspace (one word per entry: the element's number in the tile, its pattern) ...
struct SlotSink {
  uint32_t* rec;
  uint32_t first;  // index of the tile's first element
  __device__ __forceinline__ void operator()(uint32_t pos, uint32_t index, uint32_t bits) const {
    rec[pos] = ((index - first) << 16) | bits;
  }
};
// ... or nowhere (tiles without outliers)
struct NullSink {
  __device__ __forceinline__ void operator()(uint32_t, uint32_t, uint32_t) const {}
};

// What a sink is told when all outliers of a tile are found, where codes are still to be formed
template <class Sink>
__device__ __forceinline__ void all_found(const Sink&, uint32_t) {}

// The outliers of one row, in ascending index order, to positions pos_row, pos_row + 1, ... of the
// sink (entries at or past `limit` are dropped).  mask: this lane's outliers among its 8 elements;
// lane_excl: the row's outliers in lower lanes; sparse (uniform): no lane holds more than one;
// i0: flat index of the lane's first element of the row.
template <class Sink>
__device__ __forceinline__ void emit_row(const uint32_t (&oct)[4], uint32_t mask, uint32_t lane_excl, bool sparse,
                                         uint32_t i0, const Sink& sink, uint32_t pos_row, uint32_t limit) {
  uint32_t pos = pos_row + lane_excl;
  if (sparse) {
    if (mask != 0u && pos < limit) {
      const uint32_t e = (uint32_t)__builtin_ctz(mask);
      const uint64_t lo = ((uint64_t)oct[1] << 32) | oct[0], hi = ((uint64_t)oct[3] << 32) | oct[2];
      const uint64_t half = (e & 4u) ? hi : lo;
      sink(pos, i0 + e, (uint32_t)(half >> ((e & 3u) * 16u)) & 0xFFFFu);
    }
  } else {
    static_for<kOct>([&](auto Ec) {
      constexpr int e = decltype(Ec)::value;
      if ((mask >> e) & 1u) {
        if (pos < limit) sink(pos, i0 + (uint32_t)e, (e & 1) ? (oct[e >> 1] >> 16) : (oct[e >> 1] & 0xFFFFu));
        ++pos;
      }
    });
  }
}

// ------------------------------------------------------------------ rows without outliers
typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t,
                            __builtin_elementwise_max(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}

// zero the elements of an octet that `mask` names (bit e: element e)
__device__ __forceinline__ void clear_elements(uint32_t (&oct)[4], uint32_t mask) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe((int)mask, 2 * k, 1);  // 0 or all ones
    const uint32_t hi = (uint32_t)__builtin_amdgcn_sbfe((int)mask, 2 * k + 1, 1);
    oct[k] &= ~((lo & 0x0000FFFFu) | (hi & 0xFFFF0000u));
  }
}

// largest magnitude (15 low bits of the patterns) among the 8 elements of an octet
__device__ __forceinline__ uint32_t octet_magnitude(const uint32_t (&oct)[4]) {
  constexpr uint32_t kMag2 = 0x7FFF7FFFu;
  const uint32_t m = pk_max_u16(pk_max_u16(oct[0] & kMag2, oct[1] & kMag2), pk_max_u16(oct[2] & kMag2, oct[3] & kMag2));
  const uint32_t hi = m >> 16, lo = m & 0xFFFFu;
  return hi > lo ? hi : lo;
}

// ------------------------------------------------------------------ outliers by a threshold on the magnitude
// ABS and STD select what exceeds a limit that depends on the group alone, and both tests are monotonic in the magnitude:
// the limit becomes a pattern once per group, the largest 15-bit magnitude that does not pass, and the tests are packed
// 16-bit integer operations on the raw octets, two elements at a time.  Inf and NaN lie above every such pattern, so the
// values that are always outliers need no test of their own.

// m, m + 1 or m - 1: the largest magnitude t with f(t) <= limit, f monotonic, where m is that close
template <class F>
__device__ __forceinline__ uint32_t settle_magnitude(uint32_t m, float limit, F f) {
  const float above = f(__uint_as_float(mag_bits32(m + 1u))), at = f(__uint_as_float(mag_bits32(m)));
  return above <= limit ? m + 1u : (at <= limit ? m : m - 1u);
}
__device__ __forceinline__ uint32_t narrow_magnitude(float v) { return narrow_pair(v, 0.0f) & 0x7FFFu; }
// ABS: the largest magnitude not above tau (>= 0, finite)
__device__ __forceinline__ uint32_t magnitude_limit(float tau) {
  const float t = fabsf(tau);  // (-0 is accepted for 0)
  const uint32_t m = narrow_magnitude(t);  // rounds, perhaps to infinity; the largest finite one is above a tau beyond the format
  const uint32_t least = m < kNonfiniteMag ? m : kNonfiniteMag - 1u;
  return __uint_as_float(mag_bits32(least)) <= t ? least : least - 1u;
}
// STD: the largest magnitude whose square, in binary32, is not above `limit` (never negative); every finite one for a limit that is
// infinite or NaN.  The hardware's square root is within a unit in the last place of binary32, its rounding to the format
// within one of the format, so that three candidates decide; squares below 2^-100 may be subnormal or zero, where equal
// squares belong to many magnitudes: there, bit by bit.
__device__ __forceinline__ uint32_t magnitude_limit_squared(float limit) {
  auto square = [](float v) { return v * v; };
  uint32_t t = settle_magnitude(narrow_magnitude(__builtin_amdgcn_sqrtf(limit)), limit, square);
  if constexpr (ADACC_F16 == 0) {  // (binary16 has no square below 2^-48)
    if (__builtin_amdgcn_ballot_w64(limit < 0x1p-100f) != 0ull) {  // uniform, rare
      uint32_t s = 0u;
      for (int bit = 14; bit >= 0; --bit) {
        const uint32_t c = s | (1u << bit);
        s = square(__uint_as_float(mag_bits32(c))) <= limit ? c : s;
      }
      t = limit < 0x1p-100f ? s : t;
    }
  }
  return limit < __builtin_inff() ? t : kNonfiniteMag - 1u;
}
__device__ __forceinline__ uint32_t both_halves(uint32_t m) { return m | m << 16; }

// What the lanes hold (at most 8 each) below this lane, and in all (uniform)
__device__ __forceinline__ uint32_t count_below(uint32_t n, uint32_t& all) {
  uint32_t below = 0u;
  all = 0u;
#pragma unroll
  for (int b = 0; b < 4; ++b) {  // the bits of the lanes' numbers
    const uint64_t m = __builtin_amdgcn_ballot_w64((n >> b & 1u) != 0u);
    all += (uint32_t)__builtin_popcountll(m) << b;
    below += lanes_below(m) << b;
  }
  return below;
}

// The elements of a row whose magnitude exceeds the threshold (t2: in both halves) are cleared; with a sink they go
// there first, in index order, to positions pos, pos + 1, .. (entries at or past `limit` are dropped).  i0: index of the lane's first
// element.  Returns their number (uniform).
template <class Sink>
__device__ __forceinline__ uint32_t take_above(uint32_t (&oct)[4], uint32_t t2, uint32_t i0, const Sink& sink, uint32_t pos, uint32_t limit) {
  // All ones in the halves that exceed it: the sign of (threshold - magnitude).  (The threshold goes through an empty asm:
  // where the compiler knows its range it makes compares and selects of this, half by half.)
  asm("" : "+v"(t2));
  uint32_t over[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const u16x2_t left = __builtin_bit_cast(u16x2_t, t2) - __builtin_bit_cast(u16x2_t, oct[k] & 0x7FFF7FFFu);
    over[k] = __builtin_bit_cast(uint32_t, (i16x2_t)(__builtin_bit_cast(i16x2_t, left) >> 15));
  }
  uint32_t count = 0u;
  if constexpr (!std::is_same_v<Sink, NullSink>) {
    // bit e: element e (the low halves are the even elements)
    const uint32_t two = (over[0] & 0x00020001u) | (over[1] & 0x00080004u) | (over[2] & 0x00200010u) | (over[3] & 0x00800040u);
    uint32_t todo = (two | two >> 16) & 0xFFu;
    uint64_t any = __builtin_amdgcn_ballot_w64(todo != 0u);
    uint32_t at = pos;
    if (__builtin_amdgcn_ballot_w64((todo & (todo - 1u)) != 0u) == 0ull) {  // uniform: no two in one octet
      count = (uint32_t)__builtin_popcountll(any);
      at += lanes_below(any);
    } else {
      at += count_below((uint32_t)__builtin_popcount(todo), count);
    }
    while (any != 0ull) {  // uniform: mostly once; an octet's first, then its second, ..
      if (todo != 0u && at < limit) {
        const uint32_t e = (uint32_t)__builtin_ctz(todo);
        const uint32_t lo = (e & 4u) ? oct[2] : oct[0], hi = (e & 4u) ? oct[3] : oct[1];
        const uint32_t word = (e & 2u) ? hi : lo;
        sink(at, i0 + e, (e & 1u) ? word >> 16 : word & 0xFFFFu);
      }
      ++at;
      todo &= todo - 1u;
      any = __builtin_amdgcn_ballot_w64(todo != 0u);
    }
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) oct[k] &= ~over[k];
  return count;
}

// a6, symmetric, for a row free of outliers and of values that are not finite: S and D / max from
// the group's largest magnitude (`am_bits`: its binary32 bits; it has at most 11 significant bits).
// For the paper's divisor, a power of two, D / max needs no division sequence: the hardware
// reciprocal is within one unit in the last place, and for an operand of 11 significant bits one
// Newton step then gives the correctly rounded 1 / max (verified for every significand and every
// such starting value); the factor D is exact.  Outside 2^-100 .. 2^100 (where the reciprocal, or
// D / max, leaves the normal range) and for other divisors the division is carried out.
__device__ __forceinline__ void scale_sym_clean(const TensorDesc& d, uint32_t am_bits, float& scl, float& inv) {
  const float am = __uint_as_float(am_bits);
  const bool mid = am_bits - 0x0D800000u <= 0x71800000u - 0x0D800000u;  // 2^-100 <= max <= 2^100
  const bool hard = !mid && am_bits != 0u;
  if ((d.pow2_divisor != 0u) & (__builtin_amdgcn_ballot_w64(hard) == 0ull)) {  // uniform
    scl = am * d.inv_divisor;
    float r = __builtin_amdgcn_rcpf(am);
    const float e = __fmaf_rn(-am, r, 1.0f);
    r = __fmaf_rn(r, e, r);
    inv = am_bits != 0u ? r * d.divisor : 0.0f;
  } else {
    float off;
    group_scale<false>(d, am_bits, 0, 0, scl, inv, off);
  }
}

// a6 .. a8 for one row of a tile without outliers and values that are not finite (they are zero in `x`).
// top: symmetric, the lane's largest magnitude of the row as binary32 bits.
template <int BITS, bool ASYM, int E, int LANES, bool STRIP>
__device__ __forceinline__ void encode_clean_values(const TensorDesc& d, const TileGeo<E, STRIP>& g, int j,
                                                    float (&x)[kOct], uint32_t top) {
  float scl, inv, off = 0.0f;
  if constexpr (!ASYM) {
    scale_sym_clean(d, lanes_reduce<LANES>(top, OpUMax()), scl, inv);
  } else {
    float ext0, ext1;
    row_extremes<true>(x, ext0, ext1);
    const int32_t k0 = lanes_reduce<LANES>(float_key(ext0), OpIMax());
    const int32_t k1 = lanes_reduce<LANES>(float_key(ext1), OpIMin());
    group_scale<true>(d, 0u, k0, k1, scl, inv, off);
  }
  if constexpr (ASYM) {
#pragma unroll
    for (int e = 0; e < kOct; ++e) x[e] = x[e] - off;
  }
  store_row<BITS, ASYM, E>(d, g, j, x, scl, inv, off);
}
template <int BITS, bool ASYM, int E, int LANES, bool STRIP>
__device__ __forceinline__ void encode_clean_row(const TensorDesc& d, const TileGeo<E, STRIP>& g, int j,
                                                 const uint32_t (&oct)[4], uint32_t top) {
  float x[kOct];
  widen_row(oct, x);
  encode_clean_values<BITS, ASYM, E, LANES>(d, g, j, x, top);
}

// ------------------------------------------------------------------ TOPK over groups inside a row
// The k largest of every group of LANES lanes (8 * LANES elements of one row) by (magnitude, lower index),
// as the 8 ballots of the row: k rounds of a maximum over keys (magnitude in the high bits, the reversed
// position in the group below it, plus one so that no live key is zero); the winner's key is unique in its
// group, its owner sets it to zero.  Every value that is not finite is an outlier besides.
template <int LANES>
__device__ __forceinline__ void topk_row_ballots(const TensorDesc& d, const uint32_t (&oct)[4], uint64_t (&b)[kOct]) {
  const uint32_t last = (uint32_t)(LANES * kOct) - 1u - ((uint32_t)lane_id() & (uint32_t)(LANES - 1)) * kOct;  // reversed position of element 0
  uint32_t key[kOct];
  bool nonfinite[kOct];
#pragma unroll
  for (int e = 0; e < kOct; ++e) {
    const uint32_t word = oct[e >> 1];
    const uint32_t mag = (e & 1) ? (word >> 16) & 0x7FFFu : word & 0x7FFFu;
    nonfinite[e] = mag >= kNonfiniteMag;
    key[e] = ((mag << 9) | (last - (uint32_t)e)) + 1u;
  }
  for (uint32_t r = 0; r < d.topk; ++r) {  // uniform
    uint32_t best = key[0];
#pragma unroll
    for (int e = 1; e < kOct; ++e) best = key[e] > best ? key[e] : best;
    const uint32_t win = lanes_reduce<LANES>(best, OpUMax());
#pragma unroll
    for (int e = 0; e < kOct; ++e) key[e] = key[e] == win ? 0u : key[e];
  }
#pragma unroll
  for (int e = 0; e < kOct; ++e) b[e] = __builtin_amdgcn_ballot_w64(key[e] == 0u || nonfinite[e]);
}

// ------------------------------------------------------------------ tile encoder for groups inside a row
// Used when every group (statistics and quantisation) lies inside one 512-element row and both
// kinds have the same size: each row is taken from the raw octets to its stored codes in one
// go, so nothing but the raw octets lives across rows.  LANES = lanes per group.
template <int MODE, int BITS, bool ASYM, int E, int LANES, bool STORE, class Sink, bool STRIP>
__device__ __forceinline__ uint32_t encode_rows(const TensorDesc& d, const TileGeo<E, STRIP>& g,
                                                const uint32_t (&raw)[E][4], uint32_t tile, const Sink& sink,
                                                uint32_t pos0, uint32_t limit) {
  static_assert(!STRIP || MODE == kModeNone, "element indices of outliers are formed for adjacent rows only");
  const float inv_gs = __uint_as_float((127u - d.lgs) << 23);  // 2^-lgs, exact
  const uint32_t lane_first = tile * (uint32_t)(E * kRow) + (uint32_t)lane_id() * kOct;
  uint32_t total = 0u;  // uniform: outliers of the rows so far
#pragma unroll
  for (int j = 0; j < E; ++j) {
    __builtin_amdgcn_sched_barrier(0);  // one row after the other
    float x[kOct];
    widen_row(raw[j], x);
    // First a test per lane that is cheap and errs on the safe side: can this lane's octet hold an
    // outlier (or, without outliers, a value that is not finite)?  If no lane says yes - nearly
    // every row - the row is quantised as it is.  am_bits: the lane's largest |x| (ABS, NONE).
    float limit_sq = 0.0f;
    uint32_t am_bits = 0u;
    bool suspect;
    uint64_t b[kOct];  // STD, TOPK
    float q[kOct];     // STD
    if constexpr (MODE == kModeTopk) {
      suspect = true;  // every group has outliers: its k largest
      topk_row_ballots<LANES>(d, raw[j], b);
      if (!g.full) {  // uniform; the tensor's last tile: groups past its end (blanked) have no outliers
        const uint64_t valid = __builtin_amdgcn_ballot_w64(g.lane_off + g.row_offset(j) < g.rem);
#pragma unroll
        for (int e = 0; e < kOct; ++e) b[e] &= valid;
      }
    } else if constexpr (MODE == kModeStd) {
#pragma unroll
      for (int e = 0; e < kOct; ++e) q[e] = x[e] * x[e];  // exact: two significands of at most 11 bits
      float s1 = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
      float s2 = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
      s1 = lanes_reduce<LANES>(s1, OpAdd());
      s2 = lanes_reduce<LANES>(s2, OpAdd());
      limit_sq = std_limit(s1, s2, inv_gs, d.param);
      const float qm = fmaxf(fmaxf(fmaxf(q[0], q[1]), fmaxf(q[2], q[3])), fmaxf(fmaxf(q[4], q[5]), fmaxf(q[6], q[7])));
      // an Inf or NaN anywhere in a group makes its limit NaN
      suspect = !(qm <= limit_sq);
    } else {
      am_bits = mag_bits32(octet_magnitude(raw[j]));  // Inf / NaN show as a value of 0x7F800000 or more
      if constexpr (MODE == kModeAbs) suspect = am_bits > __float_as_uint(d.param);  // tau >= 0, finite
      else suspect = am_bits >= 0x7F800000u;
    }
    const uint32_t i0 = lane_first + (uint32_t)(j * kRow);
    if constexpr (MODE == kModeTopk || (MODE == kModeStd && STORE)) {
      if (MODE == kModeTopk || __builtin_amdgcn_ballot_w64(suspect) != 0ull) {  // uniform
        // The tests as wavefront ballots (scalar registers); the widened values are cleared as they are, and rows with and without
        // outliers share one copy of what follows.  (Through the threshold on the magnitude, widened again behind it: 2^25 values, STD
        // over 512, int8, at 4 sigma 30.5 us symmetric and 35.3 asymmetric, 27.5 and 28.7 like this; at 8 sigma 24.1 and 27.4, 24.0
        // and 25.0; the largest of every 128 27.2 and 25.5.  With a second copy for rows with outliers: 29.0, 30.5; 25.1, 26.5; 25.2.)
        if constexpr (MODE == kModeStd) {
#pragma unroll
          for (int e = 0; e < kOct; ++e) b[e] = __builtin_amdgcn_ballot_w64(q[e] > limit_sq);
          if (__builtin_amdgcn_ballot_w64(limit_sq != limit_sq) != 0ull) {  // then every element is tested for Inf / NaN
#pragma unroll
            for (int e = 0; e < kOct; ++e) b[e] |= __builtin_amdgcn_ballot_w64(is_nonfinite(x[e]));
          }
        }
        uint32_t mask, lane_excl, row_cnt;
        bool any, sparse;
        row_bookkeeping(b, mask, lane_excl, row_cnt, any, sparse);
        if (any) {  // uniform: the row's outliers leave at once, nothing about them is kept
          emit_row(raw[j], mask, lane_excl, sparse, i0, sink, pos0 + total, limit);
          total += row_cnt;
        }
        if constexpr (STORE) {
#pragma unroll
          for (int e = 0; e < kOct; ++e) x[e] = __builtin_amdgcn_inverse_ballot_w64(b[e]) ? 0.0f : x[e];
        }
      }
      if constexpr (STORE) {
        float most = 0.0f, unused;
        if constexpr (!ASYM) row_extremes<false>(x, most, unused);
        encode_clean_values<BITS, ASYM, E, LANES>(d, g, j, x, __float_as_uint(most));
      }
    } else {
      if (__builtin_amdgcn_ballot_w64(suspect) == 0ull) {  // uniform
        if constexpr (STORE) encode_clean_row<BITS, ASYM, E, LANES>(d, g, j, raw[j], am_bits);
        continue;
      }
      // by a threshold on the magnitude, in a copy of the octets
      uint32_t oct[4] = {raw[j][0], raw[j][1], raw[j][2], raw[j][3]};
      uint32_t most = kNonfiniteMag - 1u;  // NONE: what is not finite is zeroed, and reported nowhere
      if constexpr (MODE == kModeStd) most = magnitude_limit_squared(limit_sq);
      if constexpr (MODE == kModeAbs) most = magnitude_limit(d.param);
      total += take_above(oct, both_halves(most), i0, sink, pos0 + total, limit);
      if constexpr (STORE) encode_clean_row<BITS, ASYM, E, LANES>(d, g, j, oct, mag_bits32(octet_magnitude(oct)));
    }
  }
  return total;
}

template <int MODE, int BITS, bool ASYM, int E, bool STORE, class Sink, bool STRIP>
__device__ __forceinline__ uint32_t encode_tile_rowwise(const TensorDesc& d, const TileGeo<E, STRIP>& g,
                                                        const uint32_t (&raw)[E][4], uint32_t tile, const Sink& sink,
                                                        uint32_t pos0, uint32_t limit) {
  switch (d.lgq) {  // one switch per tile selects straight-line code for the group size
    case 3: return encode_rows<MODE, BITS, ASYM, E, 1, STORE>(d, g, raw, tile, sink, pos0, limit);
    case 4: return encode_rows<MODE, BITS, ASYM, E, 2, STORE>(d, g, raw, tile, sink, pos0, limit);
    case 5: return encode_rows<MODE, BITS, ASYM, E, 4, STORE>(d, g, raw, tile, sink, pos0, limit);
    case 6: return encode_rows<MODE, BITS, ASYM, E, 8, STORE>(d, g, raw, tile, sink, pos0, limit);
    case 7: return encode_rows<MODE, BITS, ASYM, E, 16, STORE>(d, g, raw, tile, sink, pos0, limit);
    case 8: return encode_rows<MODE, BITS, ASYM, E, 32, STORE>(d, g, raw, tile, sink, pos0, limit);
    default: return encode_rows<MODE, BITS, ASYM, E, 64, STORE>(d, g, raw, tile, sink, pos0, limit);
  }
}

// ------------------------------------------------------------------ TOPK selection
// Magnitudes are the 15 low bits of the patterns.  The largest magnitude of a lane's 8 elements in every row, two
// rows to a word (row 2i in the low half of pm[i], row 2i + 1 in the high half): half the registers, and
// the maxima of a lane's rows come two at a time.  An Inf or NaN shows as a value >= kNonfiniteMag.
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t,
                            __builtin_elementwise_min(__builtin_bit_cast(u16x2_t, a), __builtin_bit_cast(u16x2_t, b)));
}
template <int E>
struct RowMags {
  uint32_t pm[E / 2];
  __device__ __forceinline__ uint32_t at(int j) const { return (j & 1) ? pm[j >> 1] >> 16 : pm[j >> 1] & 0xFFFFu; }
  __device__ __forceinline__ void set(int j, uint32_t m) {
    pm[j >> 1] = (j & 1) ? (pm[j >> 1] & 0x0000FFFFu) | (m << 16) : (pm[j >> 1] & 0xFFFF0000u) | m;
  }
  __device__ __forceinline__ void of(const uint32_t (&raw)[E][4]) {
    constexpr uint32_t kMag2 = 0x7FFF7FFFu;
#pragma unroll
    for (int j = 0; j < E; j += 2) {
      uint32_t m[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        m[i] = pk_max_u16(pk_max_u16(raw[j + i][0] & kMag2, raw[j + i][1] & kMag2),
                          pk_max_u16(raw[j + i][2] & kMag2, raw[j + i][3] & kMag2));
      pm[j / 2] = pk_max_u16(__builtin_amdgcn_perm(m[1], m[0], 0x05040100u), __builtin_amdgcn_perm(m[1], m[0], 0x07060302u));
    }
  }
};

// One group per tile, in straight-line code: t16 <- the k-th largest of the candidates the lanes offer, as
// a 15-bit magnitude.  Returns (uniform) false when the tile holds an Inf or NaN.
// Every lane offers its two largest row maxima: the threshold then fails to cut off exactly k
// elements only when a lane holds three of the k largest, or two of them in one octet, or on a tie.
template <int E>
__device__ __forceinline__ bool topk_whole_threshold(uint32_t k, const RowMags<E>& rowmag, uint32_t& t16) {
  uint32_t p1 = rowmag.pm[0], p2 = 0u;  // the two largest of the even and of the odd rows
#pragma unroll
  for (int i = 1; i < E / 2; ++i) {
    p2 = pk_max_u16(p2, pk_min_u16(p1, rowmag.pm[i]));
    p1 = pk_max_u16(p1, rowmag.pm[i]);
  }
  const uint32_t a1 = p1 & 0xFFFFu, b1 = p1 >> 16, a2 = p2 & 0xFFFFu, b2 = p2 >> 16;
  const uint32_t m1 = a1 > b1 ? a1 : b1;
  uint32_t m2 = a1 > b1 ? b1 : a1;
  m2 = m2 > a2 ? m2 : a2;
  m2 = m2 > b2 ? m2 : b2;
  const bool finite = __builtin_amdgcn_ballot_w64(m1 >= kNonfiniteMag) == 0ull;
  // The k-th largest of the 128.  Two rounds of a maximum over the wavefront take 22 vector instructions, more of them 11
  // each; halving takes 30 comparisons whatever k is, and scalar work.  ([32768, 2048], k = 2: 31.1 us by rounds, 31.7 by
  // halving; [8192, 4096], k = 4, is faster by halving.)
  if (k <= 2u) {  // uniform
    const uint32_t lane = (uint32_t)lane_id();
    uint32_t cur = (m1 << 6) | lane;  // unique per lane: equal maxima are taken one after the other
    uint32_t win = wave_max_u32_scalar(cur);
    if (k == 2u) {
      cur = cur == win ? (m2 << 6) | lane : cur;
      win = wave_max_u32_scalar(cur);
    }
    t16 = win >> 6;
  } else {
    t16 = kth_by_halving(k, [&](uint32_t t) { return lanes_where(m1 >= t) + lanes_where(m2 >= t); });
  }
  return finite;
}

// Rounds over a tile that is one statistics group: the k-th largest key, uniform.  Returns whether
// it belongs to an Inf / NaN (then there may be more than k outliers).
template <int E>
__device__ __forceinline__ bool topk_select_rounds_whole(uint32_t k, const uint32_t (&raw)[E][4], uint32_t& kth_out,
                                                         uint32_t lane_pos) {
  uint32_t kth = 0xFFFFFFFFu;
  for (uint32_t r = 0; r < k; ++r) {
    forget_derived<E>(raw);  // the keys are formed again in every round ...
    asm volatile("" : "+v"(lane_pos));  // ... and so are the position codes: 8 per row would sit in registers otherwise
    uint32_t m = 0u;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" : "+v"(lane_pos));
      const uint32_t row_pos = ((uint32_t)j << 9) | lane_pos;
#pragma unroll
      for (int e = 0; e < kOct; ++e) {
        const uint32_t key = (ADACC_ELEM_MAG(raw[j], e) << 16) | (0xFFFFu - (row_pos | (uint32_t)e));
        const uint32_t cand = (key < kth) ? key : 0u;
        m = (cand > m) ? cand : m;
      }
    }
    kth = wave_max_u32_scalar(m);
  }
  kth_out = kth;
  return (kth >> 16) >= kNonfiniteMag;
}

// ------------------------------------------------------------------ TOPK over a tile, or over a part of one of whole rows
// The E rows are one statistics group (so they are complete: group sizes divide what the tile kernels take).  The paper's
// order, literally: the outliers are found, handed to the sink, and set to zero in the registers that hold the rows; what is left
// is quantised row by row with no thought of outliers.  first: the index of the group's first element.

// Extraction by keys (any tile): the k largest keys (magnitude above, inverted position below), and
// every value that is not finite when those are more than k.  Returns the number of outliers.
template <int E, class Sink>
__device__ __forceinline__ uint32_t topk_extract_by_keys(uint32_t k, uint32_t (&raw)[E][4], uint32_t first,
                                                        const Sink& sink, uint32_t pos0, uint32_t limit) {
  uint32_t lane_pos = (uint32_t)lane_id() << 3;
  uint32_t kth;
  const bool poisoned = topk_select_rounds_whole<E>(k, raw, kth, lane_pos);
  const uint32_t lane_first = first + (uint32_t)lane_id() * kOct;
  uint32_t total = 0u;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    __builtin_amdgcn_sched_barrier(0);  // row after row, and the position codes of a row formed when its turn comes
    asm volatile("" : "+v"(lane_pos));
    const uint32_t row_pos = ((uint32_t)j << 9) | lane_pos;
    uint64_t b[kOct];
#pragma unroll
    for (int e = 0; e < kOct; ++e) {
      const uint32_t mag = ADACC_ELEM_MAG(raw[j], e);
      const uint32_t key = (mag << 16) | (0xFFFFu - (row_pos | (uint32_t)e));
      b[e] = __builtin_amdgcn_ballot_w64(key >= kth || (poisoned && mag >= kNonfiniteMag));
    }
    uint32_t mask, lane_excl, row_cnt;
    bool any, sparse;
    row_bookkeeping(b, mask, lane_excl, row_cnt, any, sparse);
    if (any) {
      emit_row(raw[j], mask, lane_excl, sparse, lane_first + (uint32_t)(j * kRow), sink, pos0 + total, limit);
      total += row_cnt;
      clear_elements(raw[j], mask);
    }
  }
  return total;
}

// The extraction: finds the k largest, hands them to the sink, clears them in `raw`.  rowmag: the
// lane's largest magnitude per row of what is left.  Returns the number of outliers (uniform).
//
// Only octets whose largest magnitude reaches the threshold of the lanes' maxima can hold any of the k: as a rule k of
// them.  Up to 16 go to a list of the wavefront in LDS, in index order, all octets of a row at once; then a lane takes
// an element (two beyond 8 octets) and the selection is two ballots: all that reach the threshold, if those are k, else
// (equals at the k-th place, two of the largest in one octet) the k-th largest by halving and the lowest of its equals.
// The outliers leave with one store, are zeroed in the list, and the octets' owners read them back.  (Before, octets
// were taken one by one through scalar registers, and a tile with equals at the k-th place - one in 70 of bf16
// rows - was read and decided again by keys, which took so long that a launch of 8192 tiles waited for the last of
// them: 26 us, 21 us now.)
struct TopkList {
  uint4 oct[16];
  uint32_t where[16];  // the octet's first element, in the tile
};
// The selection from the list of a wavefront: the k outliers leave for entries pos0 .. of the sink, and are zeroed in the list
// (CLEAR).  CHECK: false (uniform), nothing done, where the k-th is not finite, since there may be more of those.
template <bool CLEAR, bool CHECK, class Sink>
__device__ __forceinline__ bool topk_take_from_list(TopkList& list, uint32_t octets, uint32_t k, uint32_t t16, uint32_t first,
                                                    const Sink& sink, uint32_t pos0, uint32_t limit) {
  const uint32_t lane = (uint32_t)lane_id();
  uint16_t* elem = reinterpret_cast<uint16_t*>(list.oct);
  // elements `lane` and 64 + `lane` of the list (-1: not there)
  const uint32_t pa = elem[lane], pb = elem[kWave + lane];
  const int32_t ma = lane < octets * kOct ? (int32_t)(pa & 0x7FFFu) : -1;
  const int32_t mb = lane + kWave < octets * kOct ? (int32_t)(pb & 0x7FFFu) : -1;
  uint64_t hit_a = __builtin_amdgcn_ballot_w64(ma >= (int32_t)t16), hit_b = __builtin_amdgcn_ballot_w64(mb >= (int32_t)t16);
  if ((uint32_t)(__builtin_popcountll(hit_a) + __builtin_popcountll(hit_b)) != k) {  // uniform
    const int32_t t = (int32_t)kth_by_halving(k, [&](uint32_t c) { return lanes_where(ma >= (int32_t)c) + lanes_where(mb >= (int32_t)c); });
    if constexpr (CHECK) {
      if (t >= (int32_t)kNonfiniteMag) return false;  // uniform
    }
    hit_a = __builtin_amdgcn_ballot_w64(ma > t);
    hit_b = __builtin_amdgcn_ballot_w64(mb > t);
    uint64_t eq_a = __builtin_amdgcn_ballot_w64(ma == t), eq_b = __builtin_amdgcn_ballot_w64(mb == t);
    for (uint32_t n = (uint32_t)(__builtin_popcountll(hit_a) + __builtin_popcountll(hit_b)); n < k; ++n) {  // k <= 8 rounds
      if (eq_a != 0ull) { hit_a |= eq_a & (0ull - eq_a); eq_a &= eq_a - 1ull; }
      else { hit_b |= eq_b & (0ull - eq_b); eq_b &= eq_b - 1ull; }
    }
  }
  if (__builtin_amdgcn_inverse_ballot_w64(hit_a)) {
    const uint32_t pos = pos0 + lanes_below(hit_a);
    if (pos < limit) sink(pos, first + list.where[lane >> 3] + (lane & 7u), pa);
    if constexpr (CLEAR) elem[lane] = 0;
  }
  if (hit_b != 0ull) {  // uniform
    if (__builtin_amdgcn_inverse_ballot_w64(hit_b)) {
      const uint32_t pos = pos0 + (uint32_t)__builtin_popcountll(hit_a) + lanes_below(hit_b);
      if (pos < limit) sink(pos, first + list.where[8u + (lane >> 3)] + (lane & 7u), pb);
      if constexpr (CLEAR) elem[kWave + lane] = 0;
    }
  }
  return true;
}
template <int E, bool STORE, class Sink>
__device__ __forceinline__ uint32_t topk_extract(uint32_t k, uint32_t (&raw)[E][4], RowMags<E>& rowmag,
                                                 uint32_t first, const Sink& sink, uint32_t pos0, uint32_t limit) {
  __shared__ TopkList lists[kWavesPerWg];
  rowmag.of(raw);
  const uint32_t lane = (uint32_t)lane_id();
  uint32_t t16;
  if (k <= 8u && topk_whole_threshold<E>(k, rowmag, t16)) {  // false if the tile holds an Inf or a NaN
    uint64_t cand[E];
    uint32_t octets = 0u;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      cand[j] = __builtin_amdgcn_ballot_w64(rowmag.at(j) >= t16);
      octets += (uint32_t)__builtin_popcountll(cand[j]);
    }
    if (octets <= 16u) {  // uniform (a constant tile, where every octet passes, is done by keys)
      TopkList& list = lists[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)];
      uint32_t before = 0u;  // uniform
#pragma unroll
      for (int j = 0; j < E; ++j) {
        if (cand[j] == 0ull) continue;  // uniform
        if (__builtin_amdgcn_inverse_ballot_w64(cand[j])) {
          const uint32_t c = before + lanes_below(cand[j]);
          list.oct[c] = make_uint4(raw[j][0], raw[j][1], raw[j][2], raw[j][3]);
          list.where[c] = (uint32_t)(j * kRow) + lane * kOct;
        }
        before += (uint32_t)__builtin_popcountll(cand[j]);
      }
      lds_in_order();
      topk_take_from_list<STORE, false>(list, octets, k, t16, first, sink, pos0, limit);
      if constexpr (STORE) {
        lds_in_order();
        before = 0u;
#pragma unroll
        for (int j = 0; j < E; ++j) {
          if (cand[j] == 0ull) continue;  // uniform
          if (__builtin_amdgcn_inverse_ballot_w64(cand[j])) {
            const uint4 v = list.oct[before + lanes_below(cand[j])];
            raw[j][0] = v.x; raw[j][1] = v.y; raw[j][2] = v.z; raw[j][3] = v.w;
            rowmag.set(j, octet_magnitude(raw[j]));
          }
          before += (uint32_t)__builtin_popcountll(cand[j]);
        }
      }
      return k;
    }
  }
  const uint32_t total = topk_extract_by_keys<E>(k, raw, first, sink, pos0, limit);
  if constexpr (STORE) rowmag.of(raw);
  return total;
}

// ------------------------------------------------------------------ a6 for a few rows without outliers
// From the extremes of the rows' groups of 2^lg elements (symmetric: t, the largest magnitudes; asymmetric: the keys hi and lo),
// which every lane of a group holds.  Four rows at a time lane l of every quad forms the scale of row l, where every lane of
// the group would form the same one, and the quad's lanes pass them around.
template <bool ASYM, int B>
__device__ __forceinline__ void scales_of(const TensorDesc& d, uint32_t lg, const uint32_t (&t)[B], const int32_t (&hi)[B], const int32_t (&lo)[B],
                                          float (&scl)[B], float (&inv)[B], float (&off)[B]) {
  auto scale = [&](uint32_t tt, int32_t h, int32_t l, float& s, float& v, float& o) {
    o = 0.0f;
    if constexpr (!ASYM) scale_sym_clean(d, mag_bits32(tt), s, v);
    else group_scale<true>(d, 0u, h, l, s, v, o);
  };
  if constexpr (B == 4) {
    if (lg >= 5u) {  // uniform: a group has four lanes at least
      auto pick = [&](auto a, auto b, auto c, auto e) {  // lane l of a quad: argument l
        const bool second = __builtin_amdgcn_inverse_ballot_w64(0x2222222222222222ull);
        const bool third = __builtin_amdgcn_inverse_ballot_w64(0x4444444444444444ull);
        const bool fourth = __builtin_amdgcn_inverse_ballot_w64(0x8888888888888888ull);
        auto v = second ? b : a;
        v = third ? c : v;
        return fourth ? e : v;
      };
      float s, v, o;
      if constexpr (!ASYM) scale(pick(t[0], t[1], t[2], t[3]), 0, 0, s, v, o);
      else scale(0u, pick(hi[0], hi[1], hi[2], hi[3]), pick(lo[0], lo[1], lo[2], lo[3]), s, v, o);
      scl[0] = dpp_move<0x00>(s); scl[1] = dpp_move<0x55>(s); scl[2] = dpp_move<0xAA>(s); scl[3] = dpp_move<0xFF>(s);
      inv[0] = dpp_move<0x00>(v); inv[1] = dpp_move<0x55>(v); inv[2] = dpp_move<0xAA>(v); inv[3] = dpp_move<0xFF>(v);
      off[0] = dpp_move<0x00>(o); off[1] = dpp_move<0x55>(o); off[2] = dpp_move<0xAA>(o); off[3] = dpp_move<0xFF>(o);
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < B; ++i) {
    if constexpr (!ASYM) scale(t[i], 0, 0, scl[i], inv[i], off[i]);
    else scale(0u, hi[i], lo[i], scl[i], inv[i], off[i]);
  }
}

// ------------------------------------------------------------------ a6 .. a8 for a tile without outliers
// (none left, and nothing that is not finite), quantisation groups of any size.  top: symmetric, the lane's largest magnitude
// of every row.  Four rows at a time: their extremes meet group by group, the one step that depends on the size of the groups;
// then the scales, then the codes.  ROWS: no group is longer than a row, and the compiler shall know it (with the code for a group of 4096
// beside it the batch kernel for binary16 TOPK over 4096 kept 28 registers in scratch memory).
template <int BITS, bool ASYM, int E, bool ROWS>
__device__ __forceinline__ void quantise_tile(const TensorDesc& d, const TileGeo<E>& g, const uint32_t (&raw)[E][4], const uint32_t (&top)[E]) {
  constexpr int B = E < 4 ? E : 4;
  static_assert(E % B == 0 && (B == 4 || B == 1), "rows in fours");
  // a group of 4096 takes both fours: its extremes in the lane first
  const bool all = !ROWS && E == 8 && d.lgq == 12u;  // uniform
  const uint32_t lg = all ? 11u : d.lgq;
  uint32_t top_all = 0u;
  int32_t hi_all = 0, lo_all = 0;
  if (all) {
    float hi = 0.0f, lo = 0.0f;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      if constexpr (!ASYM) {
        top_all = OpUMax()(top_all, top[j]);
      } else {
        __builtin_amdgcn_sched_barrier(0);
        float x[kOct], h, l;
        widen_row(raw[j], x);
        row_extremes<true>(x, h, l);
        hi = j == 0 ? h : fmaxf(hi, h);
        lo = j == 0 ? l : fminf(lo, l);
      }
    }
    hi_all = float_key(hi);
    lo_all = float_key(lo);
  }
  static_for<E / B>([&](auto Fc) {
    constexpr int first = decltype(Fc)::value * B;
    uint32_t t[B];
    int32_t hi[B], lo[B];
    if constexpr (!ASYM) {
#pragma unroll
      for (int i = 0; i < B; ++i) t[i] = all ? top_all : top[first + i];
      groups_reduce<B>(t, lg, OpUMax());
    } else {
#pragma unroll
      for (int i = 0; i < B; ++i) {
        __builtin_amdgcn_sched_barrier(0);
        if (all) {
          hi[i] = hi_all;
          lo[i] = lo_all;
        } else {
          float x[kOct], h, l;
          widen_row(raw[first + i], x);
          row_extremes<true>(x, h, l);
          hi[i] = float_key(h);
          lo[i] = float_key(l);
        }
      }
      groups_reduce<B>(hi, lg, OpIMax());
      groups_reduce<B>(lo, lg, OpIMin());
      forget_derived<E>(raw);  // nothing widened for the extremes is kept for the codes
    }
    float scl[B], inv[B], off[B];
    scales_of<ASYM, B>(d, lg, t, hi, lo, scl, inv, off);
#pragma unroll
    for (int i = 0; i < B; ++i) {
      // one row after the other: the compiler shall not start on the next rows to hide this row's
      // latencies (other wavefronts do that), it would pay for it with the registers of a wavefront
      __builtin_amdgcn_sched_barrier(0);
      float x[kOct];
      widen_row(raw[first + i], x);
      if constexpr (ASYM) {
#pragma unroll
        for (int e = 0; e < kOct; ++e) x[e] = x[e] - off[i];
      }
      store_row<BITS, ASYM, E>(d, g, first + i, x, scl[i], inv[i], off[i]);
    }
  });
}

// BITS = kBitsAny: as the descriptor says (the batch kernels: the selection before it is the same code for all)
constexpr int kBitsAny = 0;
template <int BITS, bool ASYM, int E, bool ROWS>
__device__ __forceinline__ void quantise_tile_as(const TensorDesc& d, const TileGeo<E>& g, const uint32_t (&raw)[E][4], uint32_t (&top)[E]) {
  if constexpr (BITS != kBitsAny) {
    quantise_tile<BITS, ASYM, E, ROWS>(d, g, raw, top);
  } else {
    switch (d.variant & 6u) {
      case 0: quantise_tile<4, false, E, ROWS>(d, g, raw, top); break;
      case 2: quantise_tile<4, true, E, ROWS>(d, g, raw, top); break;
      case 4: quantise_tile<8, false, E, ROWS>(d, g, raw, top); break;
      default: quantise_tile<8, true, E, ROWS>(d, g, raw, top); break;
    }
  }
}

template <int BITS, bool ASYM, int E, bool STORE, class Sink>
__device__ __forceinline__ uint32_t encode_tile_topk_whole(const TensorDesc& d, const TileGeo<E>& g,
                                                           uint32_t (&raw)[E][4], uint32_t tile, const Sink& sink,
                                                           uint32_t pos0, uint32_t limit) {
  RowMags<E> rowmag;
  const uint32_t total = topk_extract<E, STORE>(d.topk, raw, rowmag, tile * (uint32_t)(E * kRow), sink, pos0, limit);
  if constexpr (STORE) {
    all_found(sink, total);
    uint32_t top[E];
#pragma unroll
    for (int j = 0; j < E; ++j) top[j] = rowmag.at(j);
    quantise_tile_as<BITS, ASYM, E, true>(d, g, raw, top);
  }
  return total;
}

// ------------------------------------------------------------------ general tile encoder
// Groups of any supported size (up to the whole tile), the two kinds of any sizes.  Two steps with nothing but the raw
// octets and the lane's largest magnitude per row between them: the outliers are found, leave for the sink and are cleared in
// the octets, group by group; what is left is quantised by the code of tiles without outliers.
// Bound by instruction issue beside memory.  (Tests on widened values with ballots, masks and counts of all rows kept
// for an emission behind the codes, and widened values masked anew for them, at 2 to 7 wavefronts per SIMD: STD over 512
// with int8 groups of 64 and some 20 outliers a tile, 824 vector + 287 scalar instructions, 664 + 109 like this; [8191,
// 2051] 16.0 -> 13.4 us.  STD over 4096, [726, 4096]: 10.5 -> 8.0 us; over 1024, [4346, 1024]: 9.4 -> 7.5 us; the four
// largest of 1024, [9968, 1024]: 16.1 -> 11.4 us.)

// STD: the thresholds of the rows, in both halves of a word
template <int E>
__device__ __forceinline__ void std_thresholds(const TensorDesc& d, const uint32_t (&raw)[E][4], uint32_t (&t2)[E]) {
  float s1[E], s2[E];
#pragma unroll
  for (int j = 0; j < E; ++j) {
    float x[kOct];
    widen_row(raw[j], x);
    s1[j] = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
    // squares of 16-bit values (at most 11 significant bits) are exact in binary32
    s2[j] = ((x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3])) +
            ((x[4] * x[4] + x[5] * x[5]) + (x[6] * x[6] + x[7] * x[7]));
  }
  const float inv_gs = __uint_as_float((127u - d.lgs) << 23);  // 2^-lgs, exact
  if (E == 8 || d.lgs >= 9u) {  // groups of whole rows: one threshold for four rows, a quarter of the lanes each
    // the canonical tree: every row over its lanes, then rows two by two
    float a1 = four_rows_reduce(s1[0], s1[1], s1[2], s1[3], OpAdd()), a2 = four_rows_reduce(s2[0], s2[1], s2[2], s2[3], OpAdd());
    if (E == 8 || d.lgs >= 10u) { a1 = meet<16>(a1, a1, OpAdd()); a2 = meet<16>(a2, a2, OpAdd()); }
    if (E == 8 || d.lgs >= 11u) { a1 = meet<32>(a1, a1, OpAdd()); a2 = meet<32>(a2, a2, OpAdd()); }
    if constexpr (E == 8) {  // one group of 4096
      float b1 = four_rows_reduce(s1[4], s1[5], s1[6], s1[7], OpAdd()), b2 = four_rows_reduce(s2[4], s2[5], s2[6], s2[7], OpAdd());
      b1 = meet<16>(b1, b1, OpAdd()); b2 = meet<16>(b2, b2, OpAdd());
      b1 = meet<32>(b1, b1, OpAdd()); b2 = meet<32>(b2, b2, OpAdd());
      a1 = a1 + b1;
      a2 = a2 + b2;
    }
    const uint32_t t = both_halves(magnitude_limit_squared(std_limit(a1, a2, inv_gs, d.param)));
#pragma unroll
    for (int j = 0; j < E; ++j) t2[j] = (uint32_t)__builtin_amdgcn_readlane((int)t, 16 * (j & 3));
  } else {
    groups_reduce<E>(s1, d.lgs, OpAdd());
    groups_reduce<E>(s2, d.lgs, OpAdd());
#pragma unroll
    for (int j = 0; j < E; ++j) t2[j] = both_halves(magnitude_limit_squared(std_limit(s1[j], s2[j], inv_gs, d.param)));
  }
  forget_derived<E>(raw);  // nothing widened for the sums is kept for the codes
}

// TOPK over groups inside a row that are longer than the quantisation groups: by ballots, row by row
template <int E, int LANES, class Sink>
__device__ __forceinline__ uint32_t topk_rows_extract(const TensorDesc& d, const TileGeo<E>& g, uint32_t (&raw)[E][4], uint32_t tile,
                                                      const Sink& sink, uint32_t pos0, uint32_t limit) {
  const uint32_t lane_first = tile * (uint32_t)(E * kRow) + g.lane_off;
  uint32_t total = 0u;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    uint64_t b[kOct];
    topk_row_ballots<LANES>(d, raw[j], b);
    if (!g.full) {  // uniform; groups past the end of the tensor (blanked) have no outliers
      const uint64_t valid = __builtin_amdgcn_ballot_w64(g.lane_off + g.row_offset(j) < g.rem);
#pragma unroll
      for (int e = 0; e < kOct; ++e) b[e] &= valid;
    }
    uint32_t mask, lane_excl, row_cnt;
    bool any, sparse;
    row_bookkeeping(b, mask, lane_excl, row_cnt, any, sparse);
    if (any) {  // uniform
      emit_row(raw[j], mask, lane_excl, sparse, lane_first + (uint32_t)(j * kRow), sink, pos0 + total, limit);
      total += row_cnt;
      clear_elements(raw[j], mask);
    }
  }
  return total;
}
// TOPK over groups of R whole rows, one after the other
template <int E, int R, bool STORE, class Sink>
__device__ __forceinline__ uint32_t topk_spans_extract(const TensorDesc& d, const TileGeo<E>& g, uint32_t (&raw)[E][4], uint32_t tile,
                                                       const Sink& sink, uint32_t pos0, uint32_t limit) {
  uint32_t total = 0u;
  static_for<E / R>([&](auto Sc) {
    constexpr int first = decltype(Sc)::value * R;
    if (first == 0 || g.full || g.rem > (uint32_t)(first * kRow)) {  // uniform; groups past the end of the tensor have no outliers
      uint32_t rows[R][4];
#pragma unroll
      for (int j = 0; j < R; ++j) {
#pragma unroll
        for (int k = 0; k < 4; ++k) rows[j][k] = raw[first + j][k];
      }
      RowMags<R> mags;
      total += topk_extract<R, STORE>(d.topk, rows, mags, tile * (uint32_t)(E * kRow) + (uint32_t)(first * kRow), sink, pos0 + total, limit);
      lds_in_order();  // the next group uses the same list
#pragma unroll
      for (int j = 0; j < R; ++j) {
#pragma unroll
        for (int k = 0; k < 4; ++k) raw[first + j][k] = rows[j][k];
      }
    }
  });
  return total;
}

template <int MODE, int BITS, bool ASYM, int E, bool STORE, class Sink>
__device__ __forceinline__ uint32_t encode_tile_general(const TensorDesc& d, const TileGeo<E>& g, uint32_t (&raw)[E][4], uint32_t tile,
                                                        const Sink& sink, uint32_t pos0, uint32_t limit) {
  uint32_t top[E];  // the lane's largest magnitude of every row of what is left
  uint32_t total = 0u;
  if constexpr (MODE == kModeTopk) {
    if constexpr (E == 8) {  // one group of 4096 (with quantisation groups longer than a row)
      total = topk_spans_extract<E, 8, STORE>(d, g, raw, tile, sink, pos0, limit);
    } else {
      switch (d.lgs) {
        case 4: total = topk_rows_extract<E, 2>(d, g, raw, tile, sink, pos0, limit); break;
        case 5: total = topk_rows_extract<E, 4>(d, g, raw, tile, sink, pos0, limit); break;
        case 6: total = topk_rows_extract<E, 8>(d, g, raw, tile, sink, pos0, limit); break;
        case 7: total = topk_rows_extract<E, 16>(d, g, raw, tile, sink, pos0, limit); break;
        case 8: total = topk_rows_extract<E, 32>(d, g, raw, tile, sink, pos0, limit); break;
        case 9: total = topk_rows_extract<E, 64>(d, g, raw, tile, sink, pos0, limit); break;
        case 10: total = topk_spans_extract<E, 2, STORE>(d, g, raw, tile, sink, pos0, limit); break;
        default: total = topk_spans_extract<E, 4, STORE>(d, g, raw, tile, sink, pos0, limit); break;
      }
    }
    if constexpr (STORE) {
#pragma unroll
      for (int j = 0; j < E; ++j) top[j] = octet_magnitude(raw[j]);
    }
  } else {
    uint32_t t2[E];
    if constexpr (MODE == kModeStd) {
      std_thresholds<E>(d, raw, t2);
    } else {
      // NONE: what is not finite is zeroed, and reported nowhere
      const uint32_t t = both_halves(MODE == kModeAbs ? magnitude_limit(d.param) : kNonfiniteMag - 1u);
#pragma unroll
      for (int j = 0; j < E; ++j) t2[j] = t;
    }
    const uint32_t lane_first = tile * (uint32_t)(E * kRow) + g.lane_off;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      top[j] = octet_magnitude(raw[j]);
      if (__builtin_amdgcn_ballot_w64(top[j] > (t2[j] & 0xFFFFu)) != 0ull) {  // uniform
        total += take_above(raw[j], t2[j], lane_first + (uint32_t)(j * kRow), sink, pos0 + total, limit);
        top[j] = octet_magnitude(raw[j]);
      }
    }
  }
  if constexpr (STORE) {
    all_found(sink, total);
    quantise_tile_as<BITS, ASYM, E, false>(d, g, raw, top);
  }
  return total;
}

// ------------------------------------------------------------------ one tile, whatever the encoder
// Encodes the tile (a2 .. a8) and hands its outliers, in ascending index order, to `sink` from
// position pos0 on (entries at or past `limit` are dropped).  Returns the number of outliers of the
// tile (uniform).
// ROWWISE: all groups lie inside a row and statistics and quantisation groups coincide.
// WHOLE (TOPK): the statistics group is the whole tile and every quantisation group lies inside a row.
// STORE = false: only the outliers are found (nothing is quantised or stored).
template <int MODE, int BITS, bool ASYM, int E, bool ROWWISE, bool WHOLE, bool STORE, class Sink>
__device__ __forceinline__ uint32_t encode_tile(const TensorDesc& d, const TileGeo<E>& g, uint32_t (&raw)[E][4],
                                                uint32_t tile, const Sink& sink, uint32_t pos0, uint32_t limit) {
  static_assert(!WHOLE || (MODE == kModeTopk && !ROWWISE), "WHOLE is a TOPK encoder");
  if constexpr (ROWWISE) {
    return encode_tile_rowwise<MODE, BITS, ASYM, E, STORE>(d, g, raw, tile, sink, pos0, limit);
  } else if constexpr (WHOLE) {
    return encode_tile_topk_whole<BITS, ASYM, E, STORE>(d, g, raw, tile, sink, pos0, limit);
  } else {
    return encode_tile_general<MODE, BITS, ASYM, E, STORE>(d, g, raw, tile, sink, pos0, limit);
  }
}

// ------------------------------------------------------------------ one tile with outliers (ABS / STD / TOPK)
// Tiles are independent: a wavefront compresses one tile and never waits for another.  What the
// ordered outlier stream needs from all tiles together - the offset of every tile - is settled
// afterwards by place_tiles (below), from the per-tile counts written here.
//
// ABS / STD: the tile's outliers (ascending) go to the tile's own slot of kSlot records in the
// workspace; the placement kernel moves them to their final position.  A tile with more than
// kSlot outliers leaves the rest out; the placement kernel then selects that tile's outliers from
// the source once more.
// TOPK: every statistics group has exactly topk outliers unless it holds more than topk values that
// are not finite, so the offsets are known in advance: group g starts at topk * g.  The outliers
// are written to their final position at once, and a tile that finds another count raises the
// tensor's flag (the current epoch of the workspace); only then does the placement kernel do
// anything, and it then does everything again from the source.
template <int MODE, int BITS, bool ASYM, int E, bool ROWWISE, bool WHOLE = false>
__device__ __forceinline__ void compress_tile_outliers(const TensorDesc& d, uint32_t tile, uint32_t epoch) {
  static_assert(MODE != kModeNone, "tiles without outliers have compress_tile_plain");
  const bool last = tile + 1u == d.n_tiles;
  const bool lane0 = lane_id() == 0;
  uint32_t raw[E][4];
  if constexpr (MODE == kModeTopk) {
    const uint32_t per_tile = d.topk << (d.lgt - d.lgs);  // outliers of a complete, regular tile
    const uint32_t pos0 = per_tile * tile;
    uint32_t expected = per_tile;
    if (last) expected = d.topk * (uint32_t)((d.numel - (uint64_t)tile * (uint64_t)(E * kRow)) >> d.lgs);
    const uint32_t end = pos0 + expected;
    const StreamSink sink{d.idx, d.val};
    const uint32_t limit = end < d.cap ? end : d.cap;
    uint32_t total;
    if (WHOLE || !last) {  // only the last tile can be short: the copy for the others knows nothing of it
      load_tile<E, true>(d, tile, raw);
      total = encode_tile<MODE, BITS, ASYM, E, ROWWISE, WHOLE, true>(d, tile_geo<E, true>(d, tile), raw, tile, sink, pos0, limit);
    } else {
      load_tile<E, false>(d, tile, raw);
      const TileGeo<E> g = tile_geo<E, false>(d, tile);
      blank_tail<E>(g, raw);
      total = encode_tile<MODE, BITS, ASYM, E, ROWWISE, WHOLE, true>(d, g, raw, tile, sink, pos0, limit);
    }
    if (lane0) {
      d.tile_ptr[tile] = pos0;
      d.cnt[tile] = total;
      if (total != expected) *d.flag = epoch;
      if (last) {
        d.tile_ptr[d.n_tiles] = end;
        d.status[0] = end; d.status[1] = end > d.cap ? 1u : 0u; d.status[2] = 0u; d.status[3] = 0u;
      }
    }
  } else {
    const SlotSink sink{d.slot + (uint64_t)tile * (uint64_t)kSlot, tile * (uint32_t)(E * kRow)};
    uint32_t total;
    if (!last) {
      load_tile<E, true>(d, tile, raw);
      total = encode_tile<MODE, BITS, ASYM, E, ROWWISE, false, true>(d, tile_geo<E, true>(d, tile), raw, tile, sink, 0u, (uint32_t)kSlot);
    } else {
      load_tile<E, false>(d, tile, raw);
      const TileGeo<E> g = tile_geo<E, false>(d, tile);
      blank_tail<E>(g, raw);
      total = encode_tile<MODE, BITS, ASYM, E, ROWWISE, false, true>(d, g, raw, tile, sink, 0u, (uint32_t)kSlot);
    }
    if (lane0) d.cnt[tile] = total;
  }
}

// ------------------------------------------------------------------ placement of the outliers (a4)
// One workgroup of kPlaceThreads threads takes kPlaceTiles consecutive tiles (kPlaceSegments of the fallback kernels'
// segments; kSumTiles tiles of a long tensor).  It needs the number of outliers in all tiles before them: a workgroup
// adds up the counts itself, or, for a long tensor, the sums of blocks of kSumTiles counts that a kernel in between has
// formed.  Nobody waits for anybody.  Every wavefront then scans counts, a lane per tile, and moves the outliers of its
// share of the tiles from the slots to their final positions, a lane per record.  Tiles that hold more outliers than a
// slot takes (TOPK: all tiles) are selected again from the source (reselect_tiles), one wavefront per tile, and written
// straight to the stream.
// (Bound by round trips to memory and by how few workgroups there are: with 256 tiles to a workgroup, a thread per
// output position found by bisection and slots of 32 records, 8203 tiles of 20 outliers took 17.8 us on 33
// workgroups, and 4.5 us for the sums, 6.5 us now; the two-byte index in the tile makes a record one word, so that a slot of 256 bytes
// holds 64: 37 tiles of 4096 values with 35 outliers each were all selected again, 25.6 us, 5.5 us now.)
template <int WAVES>
struct PlaceShared {
  uint32_t part[WAVES];
  uint32_t window[WAVES];
};
struct PlaceListShared : PlaceShared<kPlaceThreads / kWave> {
  uint16_t list[kPlaceThreads / kWave][kWave * kSlot];  // 8 KiB per wavefront: every slot of a window full
};

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  struct OpUAdd { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a + b; } };
  v = lanes_reduce<16>(v, OpUAdd());
  int t = __builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += (uint32_t)t;
  t = __builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);      // row_bcast:31
  v += (uint32_t)t;
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// sum over the workgroup (WAVES wavefronts), returned to every thread
template <int WAVES>
__device__ __forceinline__ uint32_t block_sum_u32(uint32_t v, uint32_t (&part)[WAVES]) {
  const uint32_t w = wave_sum_u32(v);
  const uint32_t wave = threadIdx.x / kWave;
  __syncthreads();  // earlier readers of part[] are done
  if (lane_id() == 0) part[wave] = w;
  __syncthreads();
  uint32_t s = 0u;
#pragma unroll
  for (int i = 0; i < WAVES; ++i) s += part[i];
  return s;
}

// this thread's share of the sum of n 32-bit words (16-byte aligned); eight loads of 16 bytes per thread are in flight
// at a time
template <int WAVES>
__device__ __forceinline__ uint32_t sum_share(const uint32_t* words, uint32_t n) {
  constexpr uint32_t kStep = (uint32_t)(WAVES * kWave);
  const uint4* w4 = reinterpret_cast<const uint4*>(words);
  const uint32_t n4 = n / 4u;
  uint32_t acc = 0u;
  for (uint32_t i0 = 0u; i0 < n4; i0 += 8u * kStep) {
    uint4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const uint32_t i = i0 + (uint32_t)k * kStep + threadIdx.x;
      v[k] = i < n4 ? w4[i] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) acc += (v[k].x + v[k].y) + (v[k].z + v[k].w);
  }
  if (threadIdx.x < (n & 3u)) acc += words[4u * n4 + threadIdx.x];
  return acc;
}

// outliers in the first `tiles` tiles, to every thread of the workgroup
template <int WAVES>
__device__ __forceinline__ uint32_t outliers_before(const TensorDesc& d, uint32_t tiles, bool from_sums, PlaceShared<WAVES>& sh) {
  uint32_t acc;
  if (from_sums) {  // uniform
    const uint32_t blocks = tiles / (uint32_t)kSumTiles;
    const uint32_t t = blocks * (uint32_t)kSumTiles + threadIdx.x;  // kSumTiles = kPlaceThreads
    static_assert(WAVES * kWave >= kSumTiles, "a thread per tile of the last block");
    acc = sum_share<WAVES>(d.block_sum, blocks) + (t < tiles ? d.cnt[t] : 0u);
  } else {
    acc = sum_share<WAVES>(d.cnt, tiles);
  }
  return block_sum_u32(acc, sh.part);
}

// block_sum[block] = outliers in the block's tiles
__device__ __forceinline__ void place_sum_block(const TensorDesc& d, uint32_t block, PlaceShared<kPlaceThreads / kWave>& sh) {
  static_assert(kSumTiles == kPlaceThreads, "a thread per tile");
  const uint32_t t = block * (uint32_t)kSumTiles + threadIdx.x;
  const uint32_t s = block_sum_u32(t < d.n_tiles ? d.cnt[t] : 0u, sh.part);
  if (threadIdx.x == 0) d.block_sum[block] = s;
}

// select the outliers of one tile again and write them to the stream, into the tile's own `count`
// entries from position `pos` (an attempt of the selection that has to be given up must not reach
// into a neighbour's entries)
template <int MODE, int E, bool ROWWISE, bool WHOLE>
__device__ __forceinline__ void reselect_tile(const TensorDesc& d, uint32_t tile, uint32_t pos, uint32_t count) {
  uint32_t raw[E][4];
  load_tile<E, false>(d, tile, raw);
  const TileGeo<E> g = tile_geo<E, false>(d, tile);
  blank_tail<E>(g, raw);
  const uint32_t end = pos + count;
  encode_tile<MODE, 8, false, E, ROWWISE, WHOLE, false>(d, g, raw, tile, StreamSink{d.idx, d.val}, pos, end < d.cap ? end : d.cap);
}

// What a wavefront of the placement knows of a window of up to 64 tiles (lane j: tile first + j)
struct PlacedTiles {
  uint32_t first, n_here;  // uniform
  uint32_t base;           // uniform: outliers of all tiles before the window
  uint32_t after;          // uniform: and with those of the window (a window of the whole workgroup only)
  uint32_t count, excl;    // outliers of the lane's tile, and of the window's tiles before it
};

// The offsets of TILES tiles from the counts: tile_ptr, and by the workgroup that holds the last tile the total and the
// overflow flag (unless elements behind the last tile still have to be added, then those do it).  `move`: the records
// of tiles that fit their slot go to the stream.  TILES <= 64: the window of all wavefronts is the workgroup's tiles,
// each moves its share; TILES = 256: a window per wavefront.  first: the first tile, `most`: at most that many of the
// TILES; before: the outliers of all tiles before them, where the caller knows (`known`).
template <int TILES, int WAVES, class Shared>
__device__ __forceinline__ PlacedTiles place_tiles(const TensorDesc& d, uint32_t first, uint32_t most, bool known, uint32_t before,
                                                   bool from_sums, bool move, Shared& sh) {
  constexpr bool OWN = TILES > kWave;  // a window per wavefront
  constexpr int WINDOW = OWN ? kWave : TILES;
  constexpr int PER = OWN ? 0 : TILES / WAVES;  // tiles whose records a wavefront moves
  static_assert(!OWN || TILES == WAVES * kWave, "a lane per tile");
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  PlacedTiles p;
  p.first = first + (OWN ? wave * (uint32_t)kWave : 0u);
  const uint32_t left = p.first < d.n_tiles ? d.n_tiles - p.first : 0u;
  p.n_here = left < (uint32_t)WINDOW ? left : (uint32_t)WINDOW;
  if constexpr (!OWN) p.n_here = p.n_here < most ? p.n_here : most;
  p.count = lane < p.n_here ? d.cnt[p.first + lane] : 0u;  // (asked for ahead of the sums)
  if constexpr (OWN) {
    const uint32_t mine = wave_sum_u32(p.count);
    if (lane == 0u) sh.window[wave] = mine;  // (read behind the barriers of outliers_before)
  }
  p.base = known ? before : outliers_before<WAVES>(d, first, from_sums, sh);  // uniform
  if constexpr (OWN) {
#pragma unroll
    for (int w = 0; w < WAVES - 1; ++w) p.base += (uint32_t)w < wave ? sh.window[w] : 0u;
  }
  uint32_t incl = p.count;
#pragma unroll
  for (int off = 1; off < WINDOW; off <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)incl, off);
    if (lane >= (uint32_t)off) incl += up;
  }
  p.excl = incl - p.count;
  p.after = p.base + (uint32_t)__builtin_amdgcn_readlane((int)incl, WINDOW - 1);
  if ((OWN || wave == 0u) && p.n_here != 0u) {  // uniform
    if (lane < p.n_here) d.tile_ptr[p.first + lane] = p.base + p.excl;
    if (p.first + p.n_here == d.n_tiles && lane == p.n_here - 1u) {  // the blob's last tile closes it
      const uint32_t n_out = p.base + incl;
      if (d.n_tiles_all > d.n_tiles || d.tail == 0u) d.tile_ptr[d.n_tiles] = n_out;
      if (d.tail == 0u) { d.status[0] = n_out; d.status[1] = n_out > d.cap ? 1u : 0u; d.status[2] = 0u; d.status[3] = 0u; }
    }
  }
  if (move && __builtin_amdgcn_ballot_w64(p.count != 0u) != 0ull) {  // uniform
    if constexpr (OWN) {
      // Long tensors, where few tiles may have any: a list of the window's records in LDS (tile and number in its
      // slot), written by the lanes of the tiles, then a lane per record.
      const uint32_t in_slot = p.count <= (uint32_t)kSlot ? p.count : 0u;
      uint32_t at = p.excl, total = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
      if (__builtin_amdgcn_ballot_w64(p.count > (uint32_t)kSlot) != 0ull) {  // rare: the records' numbers without such tiles
        uint32_t sum = in_slot;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
          const uint32_t up = (uint32_t)__shfl_up((int)sum, off);
          if (lane >= (uint32_t)off) sum += up;
        }
        at = sum - in_slot;
        total = (uint32_t)__builtin_amdgcn_readlane((int)sum, kWave - 1);
      }
      uint16_t* list = sh.list[wave];
      for (uint32_t k = 0; __builtin_amdgcn_ballot_w64(k < in_slot) != 0ull; ++k)  // at most kSlot rounds
        if (k < in_slot) list[at + k] = (uint16_t)(lane << 8 | k);
      lds_in_order();
      for (uint32_t r0 = 0u; r0 < total; r0 += 4u * (uint32_t)kWave) {  // uniform
        uint32_t rec[4], pos[4], tile[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t r = r0 + (uint32_t)(i * kWave) + lane;
          const uint32_t e = r < total ? list[r] : 0u;
          tile[i] = e >> 8;
          pos[i] = p.base + (uint32_t)__shfl((int)p.excl, (int)tile[i]) + (e & 0xFFu);
          rec[i] = d.slot[(uint64_t)(p.first + tile[i]) * (uint64_t)kSlot + (e & 0xFFu)];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (r0 + (uint32_t)(i * kWave) + lane < total && pos[i] < d.cap) {
            d.idx[pos[i]] = (int32_t)((p.first + tile[i]) * d.tile_elems + (rec[i] >> 16));
            d.val[pos[i]] = (uint16_t)rec[i];
          }
        }
      }
    } else {
      // a lane per record, the loads of all tiles of this wavefront in flight at once
      uint32_t rec[PER];
      const uint32_t j0 = wave * (uint32_t)PER;
#pragma unroll
      for (int i = 0; i < PER; ++i) {  // a lane without a record reads a tile's first word
        const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)p.count, (int)j0 + i);
        const uint32_t t = j0 + (uint32_t)i < p.n_here ? p.first + j0 + (uint32_t)i : p.first;
        rec[i] = d.slot[(uint64_t)t * (uint64_t)kSlot + (lane < n ? lane : 0u)];
      }
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)p.count, (int)j0 + i);
        const uint32_t pos = p.base + (uint32_t)__builtin_amdgcn_readlane((int)p.excl, (int)j0 + i) + lane;
        if (n <= (uint32_t)kSlot && lane < n && pos < d.cap) {
          d.idx[pos] = (int32_t)((p.first + j0 + (uint32_t)i) * d.tile_elems + (rec[i] >> 16));
          d.val[pos] = (uint16_t)rec[i];
        }
      }
    }
  }
  return p;
}

// the tiles of the window whose outliers are not (all) in a slot: once more from the source, by this wavefront those
// from `j` on in steps of `step`
template <int MODE, int E, bool ROWWISE, bool WHOLE>
__device__ __forceinline__ void reselect_tiles(const TensorDesc& d, const PlacedTiles& p, uint32_t room, uint32_t j, uint32_t step) {
  for (; j < p.n_here; j += step) {
    const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)p.count, (int)j);
    if (n > room)
      reselect_tile<MODE, E, ROWWISE, WHOLE>(d, p.first + j, p.base + (uint32_t)__builtin_amdgcn_readlane((int)p.excl, (int)j), n);
  }
}

// ------------------------------------------------------------------ one tile without outliers (NONE)
template <int BITS, bool ASYM, int E, bool ROWWISE>
__device__ __forceinline__ void compress_tile_plain(const TensorDesc& d, uint32_t tile) {
  uint32_t raw[E][4];
  if (tile + 1u < d.n_tiles) {  // only the last tile can be short: the copy for the others knows nothing of it
    load_tile<E, true>(d, tile, raw);
    encode_tile<kModeNone, BITS, ASYM, E, ROWWISE, false, true>(d, tile_geo<E, true>(d, tile), raw, tile, NullSink{}, 0u, 0u);
  } else {
    load_tile<E, false>(d, tile, raw);
    const TileGeo<E> g = tile_geo<E, false>(d, tile);
    blank_tail<E>(g, raw);
    encode_tile<kModeNone, BITS, ASYM, E, ROWWISE, false, true>(d, g, raw, tile, NullSink{}, 0u, 0u);
  }
  if (tile == 0 && lane_id() == 0) {
    d.status[0] = 0u; d.status[1] = 0u; d.status[2] = 0u; d.status[3] = 0u;
  }
}

// The end of a tensor without outliers that its groups do not divide: d.tail elements behind d.numel, one short group,
// by one wavefront of the same launch.  (A launch of its own behind the tiles': 4.5 us.)
template <int BITS, bool ASYM>
__device__ __forceinline__ void compress_plain_tail(const TensorDesc& d) {
  constexpr int Q = 1 << (BITS - 1);
  constexpr uint32_t kRound = 4u * (uint32_t)kRow;  // four octets per lane at a time, at most two rounds
  const uint32_t lane = (uint32_t)lane_id();
  const uint16_t* sp = d.src + d.numel;
  uint32_t raw[4][4];
  auto load = [&](uint32_t i0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = i0 + (uint32_t)(j * kRow) + lane * kOct;
      uint4 v = make_uint4(0u, 0u, 0u, 0u);
      if (i + kOct <= d.tail) v = *reinterpret_cast<const uint4*>(sp + i);
      raw[j][0] = v.x; raw[j][1] = v.y; raw[j][2] = v.z; raw[j][3] = v.w;
      if (i < d.tail && i + kOct > d.tail) {  // the ragged end, element by element
#pragma unroll
        for (int e = 0; e < kOct - 1; ++e)
          if (i + (uint32_t)e < d.tail) raw[j][e >> 1] |= (uint32_t)sp[i + (uint32_t)e] << (16 * (e & 1));
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {  // what is not finite counts as zero
        if ((raw[j][k] & 0x7FFFu) >= kNonfiniteMag) raw[j][k] &= 0xFFFF0000u;
        if (((raw[j][k] >> 16) & 0x7FFFu) >= kNonfiniteMag) raw[j][k] &= 0x0000FFFFu;
      }
    }
  };
  uint32_t am = 0u;
  int32_t hi = (int32_t)0x80000000, lo = (int32_t)0x7FFFFFFF;
#pragma nounroll
  for (uint32_t i0 = 0; i0 < d.tail; i0 += kRound) {
    load(i0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (!ASYM) {
        am = OpUMax()(am, mag_bits32(octet_magnitude(raw[j])));
      } else {
        const uint32_t i = i0 + (uint32_t)(j * kRow) + lane * kOct;
#pragma unroll
        for (int e = 0; e < kOct; ++e) {
          const int32_t k = float_key(ADACC_ELEM_F32(raw[j], e));
          hi = (i + (uint32_t)e < d.tail && k > hi) ? k : hi;
          lo = (i + (uint32_t)e < d.tail && k < lo) ? k : lo;
        }
      }
    }
  }
  float scl, inv, off;
  if constexpr (!ASYM) group_scale<false>(d, lanes_reduce<kWave>(am, OpUMax()), 0, 0, scl, inv, off);
  else group_scale<true>(d, 0u, lanes_reduce<kWave>(hi, OpIMax()), lanes_reduce<kWave>(lo, OpIMin()), scl, inv, off);
  const uint64_t grp = d.numel >> d.lgq;
  if (lane == 0u) {
    d.scales[grp] = scl;
    if constexpr (ASYM) d.zp[grp] = off;
  }
  uint8_t* out = d.codes + d.numel * BITS / 8;  // behind the codes of the tiles, which end on a multiple of 8 elements
#pragma nounroll
  for (uint32_t i0 = 0; i0 < d.tail; i0 += kRound) {
    if (d.tail > kRound) load(i0);  // uniform
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = i0 + (uint32_t)(j * kRow) + lane * kOct;
      uint32_t c[kOct];
#pragma unroll
      for (int e = 0; e < kOct; ++e) {
        const float y = ADACC_ELEM_F32(raw[j], e);
        c[e] = code_bits<Q>(__fmul_rn(ASYM ? y - off : y, inv)) & (uint32_t)(2 * Q - 1);
        c[e] = i + (uint32_t)e < d.tail ? c[e] : 0u;  // an odd end: the high nibble is 0
      }
#pragma unroll
      for (int k = 0; k < BITS; ++k) {  // byte by byte: a few hundred bytes in all
        uint32_t byte = c[k * 8 / BITS];
        if constexpr (BITS == 4) byte |= c[2 * k + 1] << 4;
        if (i + (uint32_t)(k * 8 / BITS) < d.tail) out[(i * BITS) / 8 + (uint32_t)k] = (uint8_t)byte;
      }
    }
  }
  if (d.n_tiles == 0u && lane == 0u) { d.status[0] = 0u; d.status[1] = 0u; d.status[2] = 0u; d.status[3] = 0u; }
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
