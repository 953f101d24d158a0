// Compression of long groups: statistics groups of more than half a segment of the fallback kernels (2049 elements and more: a
// whole row of 2200 or 11008 values as one group), with quantisation groups that are the statistics group or a power of two up to
// a 512-element row.
//
// A wavefront takes a group, all of it in registers: row j, octet of lane l, as a tile of up to 22 rows.  Every step is the
// tile kernels': sums over lanes, then rows two by two; thresholds on the 16-bit magnitude; the k largest by lane maxima,
// halving and a list in LDS; four scales at a time.  No barrier, and no octet that exists only to fill a workgroup's
// slices.  (A workgroup per group, adacc_generic.hpp: in us, groups of one row each, int8, workgroup -> wavefront
//   STD   [26000, 2200] 82.5 -> 48.4   [16000, 4104] 68.6 -> 47.9   [12000, 5160] 56.8 -> 44.3   [8192, 11008] 76.7 -> 62.2
//   TOPK  [26000, 2200] 83.0 -> 42.7   NONE  39.4 -> 31.3   ABS  62.1 -> 40.7
// and TOPK-8, int4 in groups of 128: [8192, 4104] 36.7 -> 22.3  [8192, 6144] 39.3 -> 28.5  [8192, 8192] 42.5 -> 37.0
//   [8192, 11008] 62.9 -> 49.1, of which 36 are what its 227 MB take at 6.3 TB/s.)
// Where the workgroup is the better one, it stays: more than 8 of the largest, longer groups without outliers ([8192, 11008]: NONE 44.8
// us by workgroups, 50.0 by wavefronts), tensors of few groups (a wavefront each leaves the device empty), quantisation groups
// whose lanes do not line up with a row, and more than 22 rows, which four wavefronts per SIMD would not hold without a spill.
// The blob, its tiles and the workspace are those of adacc_generic.hpp, whose placement kernel follows here too.
#pragma once

#include "adacc_common.hpp"
#include "adacc_compress.hpp"
#include "adacc_dtype.hpp"

namespace adacc {
namespace ADACC_DT_NS {

struct LongGeo {
  uint64_t first;     // uniform: index of the group's first element
  uint32_t cnt;       // uniform: its elements, a multiple of 8 (the tensor's last group may be short)
  // elements of row j (uniform): 512, fewer in the last one, 0 behind it
  __device__ __forceinline__ uint32_t row_elems(int j) const {
    const uint32_t at = (uint32_t)(j * kRow);
    return cnt <= at ? 0u : (cnt - at < (uint32_t)kRow ? cnt - at : (uint32_t)kRow);
  }
};
// lane * 8, formed anew where it is called: offsets and comparisons of all rows would otherwise be kept from the loads to the
// stores, a register each
__device__ __forceinline__ uint32_t lane_offset() {
  uint32_t v = (uint32_t)lane_id() * kOct;
  asm volatile("" : "+v"(v));
  return v;
}

// What does not exist reads as +0.  The loads are issued without a branch between them (an octet that does not exist
// reads its row's last one again, a row that does not exist the first one).
template <int E>
__device__ __forceinline__ void load_long(const TensorDesc& d, const LongGeo& g, uint32_t (&raw)[E][4]) {
  const uint16_t* sp = d.src + g.first;
  const uint32_t lane_off = lane_offset();
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const uint32_t n = g.row_elems(j), last = n != 0u ? n - (uint32_t)kOct : 0u;
    const uint4 v = ADACC_LOAD16(sp + (n != 0u ? j * kRow : 0) + (lane_off < last ? lane_off : last));
    raw[j][0] = v.x; raw[j][1] = v.y; raw[j][2] = v.z; raw[j][3] = v.w;
  }
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const uint32_t n = g.row_elems(j);
    if (n != (uint32_t)kRow) {  // uniform
      const bool there = lane_offset() < n;
#pragma unroll
      for (int k = 0; k < 4; ++k) raw[j][k] = there ? raw[j][k] : 0u;
    }
  }
}

// STD: the sums of the group as the balanced tree over octets padded with +0 to a power of two (an octet's part is its own tree,
// then the lanes of a row, then rows two by two), four rows at a time, so that no row's part is kept; then the threshold.
template <int E>
__device__ __forceinline__ uint32_t long_std_threshold(const TensorDesc& d, const LongGeo& g, const uint32_t (&raw)[E][4]) {
  constexpr int Q = (E + 3) / 4;
  float b1[Q], b2[Q];
  static_for<Q>([&](auto Qc) {
    constexpr int q = decltype(Qc)::value;
    float s1[4], s2[4];
    static_for<4>([&](auto Ic) {
      constexpr int i = decltype(Ic)::value, j = 4 * q + i;
      s1[i] = 0.0f;
      s2[i] = 0.0f;
      if constexpr (j < E) {
        __builtin_amdgcn_sched_barrier(0);
        float x[kOct];
        widen_row(raw[j], x);
        s1[i] = ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
        s2[i] = ((x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3])) +
                ((x[4] * x[4] + x[5] * x[5]) + (x[6] * x[6] + x[7] * x[7]));
      }
    });
    b1[q] = four_rows_reduce(s1[0], s1[1], s1[2], s1[3], OpAdd());
    b2[q] = four_rows_reduce(s2[0], s2[1], s2[2], s2[3], OpAdd());
    b1[q] = meet<16>(b1[q], b1[q], OpAdd());
    b2[q] = meet<16>(b2[q], b2[q], OpAdd());
    b1[q] = meet<32>(b1[q], b1[q], OpAdd());
    b2[q] = meet<32>(b2[q], b2[q], OpAdd());
  });
#pragma unroll
  for (int w = 1; w < Q; w <<= 1) {
#pragma unroll
    for (int q = 0; q + w < Q; q += 2 * w) {
      b1[q] = b1[q] + b1[q + w];
      b2[q] = b2[q] + b2[q + w];
    }
  }
  const float n = (float)g.cnt;
  const float m = __fdiv_rn(b1[0], n);
  float var = __fmaf_rn(-m, m, __fdiv_rn(b2[0], n));
  var = (var < 0.0f) ? 0.0f : var;  // a NaN stays a NaN: then nothing passes the test
  forget_derived<E>(raw);           // nothing widened for the sums is kept for the codes
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)magnitude_limit_squared(d.param * var));  // param = k * k
}

template <int E>
__device__ __forceinline__ void forget_unpacked(RowMags<E>& mags) {  // as forget_derived: at(j) of all rows is not kept
#pragma unroll
  for (int i = 0; i < E / 2; ++i) asm volatile("" : "+v"(mags.pm[i]));
}

// TOPK, k <= 8: which octets the list has to take when more than its 16 reach the bound t16, which coarse values, clipped ones,
// constant and empty rows do.  t16 goes up, by halving over the octets' largest magnitudes, until at most 16 octets
// reach it and k still do, and those are the list as they would be.  If there is no such magnitude, t16 is the largest that k octets reach,
// fewer than k are larger, and equals of t16 are chosen by index: the first 8 octets among those whose largest is t16 hold all that can be
// chosen.  Then mags is 1 where an octet goes to the list and 0 elsewhere.  Returns the number of octets (uniform); marked: mags is
// that.  No value is looked at but in the list, and nothing is read again.  (us, k = 8, int4 in groups of 128, by workgroups, by a
// wavefront that found the k-th magnitude by halving over all elements, read again for it, and like this: values rounded to
// quarters [3072, 8192] 22.3 / 37.9 / 22.3, [8192, 11008] 65.6 / 75.4 / 52.5; three bits of significand [8192, 11008] 67.5 / 108 / 56.2;
// clipped [8192, 2560] 45.2 / 68.7 / 19.5.)
template <int E>
__device__ __forceinline__ uint32_t long_topk_narrow(uint32_t k, uint32_t octets, RowMags<E>& mags, uint32_t& t16, bool& marked) {
  uint32_t most = 0u;
#pragma unroll
  for (int j = 0; j < E; ++j) most = mags.at(j) > most ? mags.at(j) : most;
  uint32_t beyond = wave_max_u32_scalar(most) + 1u;
#pragma unroll 1
  while (octets > 16u && beyond - t16 > 1u) {  // uniform
    const uint32_t c = t16 + (beyond - t16) / 2u;
    uint32_t n = 0u;
    forget_unpacked(mags);
#pragma unroll
    for (int j = 0; j < E; ++j) n += lanes_where(mags.at(j) >= c);
    if (n >= k) {
      t16 = c;
      octets = n;
    } else {
      beyond = c;
    }
  }
  marked = octets > 16u;
  if (!marked) return octets;
  octets = 0u;
  uint32_t equals = 0u;
  forget_unpacked(mags);
#pragma unroll
  for (int j = 0; j < E; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    const uint64_t same = __builtin_amdgcn_ballot_w64(mags.at(j) == t16);
    const bool take = mags.at(j) > t16 || (mags.at(j) == t16 && equals + lanes_below(same) < 8u);
    equals += (uint32_t)__builtin_popcountll(same);
    octets += lanes_where(take);
    mags.set(j, take ? 1u : 0u);
  }
  return octets;
}

// TOPK, k <= 8: topk_extract's way over the list, for any group; what that keeps for every row (the candidates' ballots) is
// formed again where it is used.  Returns false (uniform), raw and mags as they were, if k values are not finite, or more.
template <int E, class Sink>
__device__ __forceinline__ bool long_topk_by_list(uint32_t k, uint32_t (&raw)[E][4], RowMags<E>& mags, uint32_t first,
                                                  const Sink& sink, uint32_t pos0, uint32_t limit) {
  __shared__ TopkList lists[kWavesPerWg];
  mags.of(raw);
  uint32_t t16;
  topk_whole_threshold<E>(k, mags, t16);  // a bound: k octets reach it
  uint32_t octets = 0u;
#pragma unroll
  for (int j = 0; j < E; ++j) octets += lanes_where(mags.at(j) >= t16);
  bool marked = false;
  // (uniform, as every rare way here; told to the compiler, so that the usual groups do not pay for what it parks in lanes of vector
  // registers: [8192, 11008], k = 8, 2081 -> 2027 vector instructions a group, 48.8 -> 48.3 us)
  if (__builtin_expect(octets > 16u, 0)) octets = long_topk_narrow<E>(k, octets, mags, t16, marked);
  const uint32_t reach = marked ? 1u : t16;
  TopkList& list = lists[__builtin_amdgcn_readfirstlane(threadIdx.x / kWave)];
  uint32_t before = 0u;  // uniform
  forget_unpacked(mags);
#pragma unroll
  for (int j = 0; j < E; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    const uint64_t cand = __builtin_amdgcn_ballot_w64(mags.at(j) >= reach);
    if (cand == 0ull) continue;  // uniform
    if (__builtin_amdgcn_inverse_ballot_w64(cand)) {
      const uint32_t c = before + lanes_below(cand);
      list.oct[c] = make_uint4(raw[j][0], raw[j][1], raw[j][2], raw[j][3]);
      list.where[c] = (uint32_t)(j * kRow) + lane_offset();
    }
    before += (uint32_t)__builtin_popcountll(cand);
  }
  lds_in_order();
  const bool taken = topk_take_from_list<true, true>(list, octets, k, t16, first, sink, pos0, limit);
  if (taken) {  // uniform
    lds_in_order();
    forget_unpacked(mags);
    before = 0u;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      const uint64_t cand = __builtin_amdgcn_ballot_w64(mags.at(j) >= reach);
      if (cand == 0ull) continue;  // uniform
      if (__builtin_amdgcn_inverse_ballot_w64(cand)) {
        const uint4 v = list.oct[before + lanes_below(cand)];
        raw[j][0] = v.x; raw[j][1] = v.y; raw[j][2] = v.z; raw[j][3] = v.w;
        mags.set(j, octet_magnitude(raw[j]));
      }
      before += (uint32_t)__builtin_popcountll(cand);
    }
  }
  if (__builtin_expect(marked, 0)) mags.of(raw);  // uniform
  return taken;
}

// What exceeds a threshold (t, uniform) leaves, row by row, and is cleared; mags follows.  Returns the number (uniform).
template <int E, class Sink>
__device__ __forceinline__ uint32_t long_take_above(uint32_t t, uint32_t (&raw)[E][4], RowMags<E>& mags, uint32_t first,
                                                    const Sink& sink, uint32_t pos0, uint32_t limit) {
  const uint32_t t2 = both_halves(t);
  uint32_t total = 0u;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    __builtin_amdgcn_sched_barrier(0);
    if (__builtin_amdgcn_ballot_w64(mags.at(j) > t) == 0ull) continue;  // uniform
    total += take_above(raw[j], t2, first + lane_offset() + (uint32_t)(j * kRow), sink, pos0 + total, limit);
    mags.set(j, octet_magnitude(raw[j]));
  }
  return total;
}

// a6 .. a8, outliers and what is not finite gone.  top(j): the lane's largest magnitude of row j.
template <int BITS, bool ASYM, int E, class Top>
__device__ __forceinline__ void quantise_long(const TensorDesc& d, const LongGeo& g, uint32_t seg, const uint32_t (&raw)[E][4], const Top& top) {
  const bool single = d.gq >= d.tile_elems;  // uniform: one scale for the whole group
  const uint32_t lg = single ? 9u : d.lgq;
  uint8_t* codes = d.codes + g.first * BITS / 8;
  float* scales = d.scales + (single ? (uint64_t)seg : g.first >> d.lgq);
  float* zp = d.zp + (single ? (uint64_t)seg : g.first >> d.lgq);
  auto scale_of = [&](uint32_t t, int32_t h, int32_t l, float& s, float& v, float& o) {
    o = 0.0f;
    if constexpr (!ASYM) scale_sym_clean(d, mag_bits32(t), s, v);
    else group_scale<true>(d, 0u, h, l, s, v, o);
  };
  auto extremes = [&](int j, int32_t& h, int32_t& l) {  // a lane without an octet brings the identity
    float x[kOct], hi, lo;
    widen_row(raw[j], x);
    row_extremes<true>(x, hi, lo);
    const bool there = lane_offset() < g.row_elems(j);
    h = there ? float_key(hi) : (int32_t)0x80000000;
    l = there ? float_key(lo) : (int32_t)0x7FFFFFFF;
  };
  float one_s = 0.0f, one_v = 0.0f, one_o = 0.0f;
  if (single) {
    uint32_t t = 0u;
    int32_t h = (int32_t)0x80000000, l = (int32_t)0x7FFFFFFF;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      if constexpr (!ASYM) {
        t = OpUMax()(t, top(j));
      } else {
        __builtin_amdgcn_sched_barrier(0);
        int32_t hj, lj;
        extremes(j, hj, lj);
        h = OpIMax()(h, hj);
        l = OpIMin()(l, lj);
      }
    }
    if constexpr (!ASYM) t = lanes_reduce<kWave>(t, OpUMax());
    else { h = lanes_reduce<kWave>(h, OpIMax()); l = lanes_reduce<kWave>(l, OpIMin()); }
    scale_of(t, h, l, one_s, one_v, one_o);
    if (lane_id() == 0) {
      scales[0] = one_s;
      if constexpr (ASYM) zp[0] = one_o;
    }
    if constexpr (ASYM) forget_derived<E>(raw);
  }
  static_for<(E + 3) / 4>([&](auto Fc) {
    constexpr int first = decltype(Fc)::value * 4;
    if ((uint32_t)(first * kRow) >= g.cnt) return;  // uniform
    float scl[4], inv[4], off[4];
    if (single) {
#pragma unroll
      for (int i = 0; i < 4; ++i) { scl[i] = one_s; inv[i] = one_v; off[i] = one_o; }
    } else {
      uint32_t t[4];
      int32_t h[4], l[4];
      static_for<4>([&](auto Ic) {
        constexpr int i = decltype(Ic)::value;
        t[i] = 0u; h[i] = (int32_t)0x80000000; l[i] = (int32_t)0x7FFFFFFF;
        if constexpr (first + i < E) {
          if constexpr (!ASYM) t[i] = top(first + i);
          else extremes(first + i, h[i], l[i]);
        }
      });
      if constexpr (!ASYM) {
        groups_reduce<4>(t, lg, OpUMax());
      } else {
        groups_reduce<4>(h, lg, OpIMax());
        groups_reduce<4>(l, lg, OpIMin());
        forget_derived<E>(raw);
      }
      scales_of<ASYM, 4>(d, lg, t, h, l, scl, inv, off);
    }
    static_for<4>([&](auto Ic) {
      constexpr int i = decltype(Ic)::value, j = first + i;
      if constexpr (j < E) {
        __builtin_amdgcn_sched_barrier(0);  // one row after the other
        const uint32_t n = g.row_elems(j);
        if (n == 0u) return;  // uniform
        float x[kOct];
        widen_row(raw[j], x);
#pragma unroll
        for (int e = 0; e < kOct; ++e) x[e] = __fmul_rn(ASYM ? x[e] - off[i] : x[e], inv[i]);
        uint32_t w[2];
        pack_codes<BITS, ASYM>(x, w);
        const uint32_t lane_off = lane_offset();
        if (lane_off < n) {
          uint8_t* cp = codes + j * kRow * BITS / 8;
          if constexpr (BITS == 8) ADACC_STORE8(cp + lane_off, make_uint2(w[0], w[1]));
          else ADACC_STORE4(cp + lane_off / 2u, w[0]);
          if (!single) {  // uniform; all lanes of a group store the same
            const uint32_t row_grp = (uint32_t)(j * kRow) >> lg, grp = lane_off >> lg;
            scales[row_grp + grp] = scl[i];
            if constexpr (ASYM) zp[row_grp + grp] = off[i];
          }
        }
      }
    });
  });
}

template <int E, bool TOPK, int BITS, bool ASYM>
__device__ __forceinline__ void compress_long(const TensorDesc& d, uint32_t seg, uint32_t epoch) {
  LongGeo g;
  g.first = (uint64_t)seg * d.tile_elems;
  const uint64_t left = d.numel - g.first;
  g.cnt = left < (uint64_t)d.tile_elems ? (uint32_t)left : d.tile_elems;
  const bool lane0 = lane_id() == 0, last = seg + 1u == d.n_tiles;
  uint32_t raw[E][4];
  load_long<E>(d, g, raw);
  RowMags<E> mags;
  if constexpr (TOPK) {
    const uint32_t pos0 = seg * d.topk;
    const uint32_t expected = d.topk < g.cnt ? d.topk : g.cnt;
    const uint32_t end = pos0 + expected;
    const uint32_t limit = end < d.cap ? end : d.cap;
    const StreamSink sink{d.idx, d.val};
    uint32_t total = expected;
    // (k values that are not finite, or more: all of those leave.  Nine Inf in every row, k = 8, with the placement that writes all of it
    // again, [8192, 11008]: 144 us by workgroups, 166 by a second read, 107 like this)
    if (__builtin_expect(!long_topk_by_list<E>(expected, raw, mags, (uint32_t)g.first, sink, pos0, limit), 0))
      total = long_take_above<E>(kNonfiniteMag - 1u, raw, mags, (uint32_t)g.first, sink, pos0, limit);
    if (lane0) {
      d.tile_ptr[seg] = pos0;
      d.cnt[seg] = total;
      if (total != expected) *d.flag = epoch;
      if (last) {
        d.tile_ptr[d.n_tiles] = end;
        d.status[0] = end; d.status[1] = end > d.cap ? 1u : 0u; d.status[2] = 0u; d.status[3] = 0u;
      }
    }
  } else {
    uint32_t most = kNonfiniteMag - 1u;  // NONE: what is not finite is zeroed, and reported nowhere
    if (d.mode == kModeStd) most = long_std_threshold<E>(d, g, raw);
    if (d.mode == kModeAbs) most = magnitude_limit(d.param);
    mags.of(raw);
    const uint32_t t2 = both_halves(most);
    uint32_t total = 0u;
    const SlotSink sink{d.slot + (uint64_t)seg * (uint64_t)kSlot, (uint32_t)g.first};
#pragma unroll
    for (int j = 0; j < E; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      if (__builtin_amdgcn_ballot_w64(mags.at(j) > most) == 0ull) continue;  // uniform
      if (d.mode == kModeNone) take_above(raw[j], t2, 0u, NullSink{}, 0u, 0u);
      else total += take_above(raw[j], t2, (uint32_t)g.first + lane_offset() + (uint32_t)(j * kRow), sink, total, (uint32_t)kSlot);
      mags.set(j, octet_magnitude(raw[j]));
    }
    if (lane0) {
      if (d.mode != kModeNone) d.cnt[seg] = total;
      else if (seg == 0u) { d.status[0] = 0u; d.status[1] = 0u; d.status[2] = 0u; d.status[3] = 0u; }
    }
  }
  quantise_long<BITS, ASYM, E>(d, g, seg, raw, [&](int j) { return mags.at(j); });
}

// Wavefronts per SIMD the registers are held to, as many as do without a spill: four registers a row for the values, and some forty
// beside them.  (STD symmetric over 13 to 16 rows at 5, with 21 values spilled, and at 4: int4 at 8 sigma [8192, 8000] 42.0 and 36.2
// us, at 4 sigma 99.2 and 93.6; int8 46.8 and 41.2, 100.3 and 95.2.)
template <int E, bool TOPK, bool ASYM>
constexpr int long_min_waves() {
  if (E <= 8) return TOPK ? 7 : 8;
  if (E <= 12) return TOPK && ASYM ? 5 : 6;
  return E <= 16 && ASYM != TOPK ? 5 : 4;
}
template <int E, bool TOPK, int BITS, bool ASYM>
__global__ __launch_bounds__(kThreads, (long_min_waves<E, TOPK, ASYM>())) void compress_long_kernel(TensorDesc d, uint32_t epoch) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // uniform, and the compiler shall know it
  const uint32_t seg = blockIdx.x * kWavesPerWg + wave;
  if (seg < d.n_tiles) compress_long<E, TOPK, BITS, ASYM>(d, seg, epoch);
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
