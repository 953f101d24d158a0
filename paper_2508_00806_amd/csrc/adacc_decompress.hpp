// Decompression of one piece by one wavefront (Section 3.2: X^ = code * S, resp. code * S + O,
// then the outliers are written back; Fig. 3(c) decompression workflow).
#pragma once

#include "adacc_common.hpp"
#include "adacc_compress.hpp"
#include "adacc_dtype.hpp"

namespace adacc {
namespace ADACC_DT_NS {

// Decompression works on pieces of the flat tensor, 2048 elements or, in long tensors, fewer (full_piece_rows), one per wavefront,
// whatever the tile of the blob and whatever the group sizes: a piece looks through the outliers of the tiles it touches and
// takes those that fall inside it.
//
// A complete piece takes its outliers into the output words in registers before they are stored, so nothing is
// written twice and nothing waits for a store:
//   - at most 64 entries, no two of them in the same chunk (every piece of a TOPK tensor with few, nearly all others):
//     the lanes that hold the entries drop them into a mailbox of the wavefront in LDS (one word per chunk of the
//     piece), every lane picks up the words of its own chunks;
//   - otherwise the entries go, 64 at a time, to a picture of the piece in LDS (the 16-bit pattern at the element's
//     place, and a bit per element that says so); every lane merges its chunks with it.  The picture is not
//     cleared, only its bits are.  (Before, such a piece was stored, waited for its own stores and wrote the
//     outliers over them, 2 or 4 bytes each: 16.8 M values of 2051-element rows with 1 % outliers restored as
//     binary32 took 31 + 4.5 us with the launch for the short end, 18 us now with the chunks below.)
// The last piece of a tensor, when it is not complete, is stored first; the wavefront waits until those stores have
// reached the L2 (its store counter at zero), and then stores the outliers of the piece to their positions.
//
// GENERIC: methods whose groups are no powers of two or exceed 4096.  Group and tile numbers of the piece's first
// octet come from a multiplication by the 64-bit reciprocal that the host prepared, those of a lane's octets from
// the binary32 one (exact below 4096 octets).  The entries of the piece are found by a 64-way search where the
// tile holds more than a wavefront looks at once.  (A workgroup per tile, as the compression has it, went through
// a row of 11008 values in 5.4 rounds with a barrier before the outliers: [8192, 11008], int4, 70 us; 43 us now.)
// What a lane takes at a time ("chunk"): as many consecutive elements as one 16-byte store holds, V = 8 of a 16-bit
// output and V = 4 of a binary32 one, so that every store instruction of a wavefront covers 1 KiB without gaps.  A row
// is the 64 chunks of one such instruction; a piece has 4 resp. 8 rows, or fewer.  (With octets for both, a lane wrote its 32
// bytes of binary32 in two stores 32 bytes apart from its neighbour's: 49.5 M values of int8 codes took 68 .. 74 us,
// 3.4 TB/s; 46 us now, 5.3 TB/s.)
template <bool F32>
constexpr int chunk_elems() { return F32 ? 4 : 8; }
template <bool F32, int ROWS>
constexpr int piece_elems() { return ROWS * kWave * chunk_elems<F32>(); }

template <int BITS, int V>
struct RowCodes {
  uint32_t w[V * BITS > 32 ? 2 : 1];
  float s, o;
};

// p: the codes of the lane's chunk, grp: its quantisation group
template <int BITS, int V, bool ASYM>
__device__ __forceinline__ void load_row_codes(const TensorDesc& d, const uint8_t* p, uint64_t grp, RowCodes<BITS, V>& r) {
  if constexpr (V * BITS == 64) {
    const uint2 w = *reinterpret_cast<const uint2*>(p);
    r.w[0] = w.x; r.w[1] = w.y;
  } else if constexpr (V * BITS == 32) {
    r.w[0] = *reinterpret_cast<const uint32_t*>(p);
  } else {
    r.w[0] = *reinterpret_cast<const uint16_t*>(p);
  }
  r.s = d.scales[grp];
  r.o = 0.0f;
  if constexpr (ASYM) r.o = d.zp[grp];
}

// the codes of a chunk, sign-extended
template <int BITS, int V>
__device__ __forceinline__ void unpack_codes(const uint32_t (&w)[V * BITS > 32 ? 2 : 1], int (&c)[V]) {
#pragma unroll
  for (int e = 0; e < V; ++e) {
    if constexpr (BITS == 8) c[e] = (int)(int8_t)((w[e >> 2] >> (8 * (e & 3))) & 0xFFu);
    else c[e] = ((int)(w[0] << (28 - 4 * e))) >> 28;
  }
}

// What goes over the dequantised values of a row before they are stored.
struct NoPatch {
  __device__ __forceinline__ void words(uint32_t (&)[4]) const {}
};
// What a lane finds in the mailbox for one of its chunks: 0, or bit 31 set, the element (0 .. V - 1) in bits 16..18
// and the outlier's 16-bit pattern in the low half.
constexpr uint32_t kMailFull = 0x80000000u;
template <bool F32>
struct MailPatch {
  uint32_t mail;
  __device__ __forceinline__ void words(uint32_t (&w)[4]) const {
    const bool mine = mail != 0u;
    const uint32_t e = (mail >> 16) & 7u;
    const uint32_t pat = mail & 0xFFFFu;
    if constexpr (F32) {
      const uint32_t bits = __float_as_uint(widen_lo(pat));
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = (mine && e == (uint32_t)k) ? bits : w[k];
    } else {
      const uint32_t keep = (e & 1u) ? 0x0000FFFFu : 0xFFFF0000u;
      const uint32_t put = (e & 1u) ? pat << 16 : pat;
#pragma unroll
      for (int k = 0; k < 4; ++k) w[k] = (mine && (e >> 1) == (uint32_t)k) ? ((w[k] & keep) | put) : w[k];
    }
  }
};
// The chunk of the picture in LDS (16-bit patterns, two per word) and its V bits
template <bool F32>
struct PicturePatch {
  uint32_t bits;
  uint32_t pat[F32 ? 2 : 4];
  __device__ __forceinline__ void words(uint32_t (&w)[4]) const {
#pragma unroll
    for (int k = 0; k < (F32 ? 2 : 4); ++k) {
      const uint32_t lo = (uint32_t)__builtin_amdgcn_sbfe((int)bits, 2 * k, 1);      // 0 or all ones
      const uint32_t hi = (uint32_t)__builtin_amdgcn_sbfe((int)bits, 2 * k + 1, 1);
      if constexpr (F32) {
        w[2 * k] = lo != 0u ? __float_as_uint(widen_lo(pat[k])) : w[2 * k];
        w[2 * k + 1] = hi != 0u ? __float_as_uint(widen_hi(pat[k])) : w[2 * k + 1];
      } else {
        const uint32_t take = (lo & 0x0000FFFFu) | (hi & 0xFFFF0000u);
        w[k] = (w[k] & ~take) | (pat[k] & take);
      }
    }
  }
};

// a9 for one row: unpack, dequantise, [patch outliers in,] store
template <int BITS, bool ASYM, bool F32, class Patch>
__device__ __forceinline__ void store_row_values(const TensorDesc& d, uint64_t e0, const RowCodes<BITS, chunk_elems<F32>()>& r,
                                                 const Patch& patch) {
  constexpr int V = chunk_elems<F32>();
  int c[V];
  unpack_codes<BITS, V>(r.w, c);
  float v[V];
#pragma unroll
  for (int e = 0; e < V; ++e) v[e] = ASYM ? __fmaf_rn((float)c[e], r.s, r.o) : (float)c[e] * r.s;
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if constexpr (F32) w[k] = __float_as_uint(v[k]);
    else w[k] = narrow_pair(v[2 * k], v[2 * k + 1]);
  }
  patch.words(w);
  if constexpr (F32) ADACC_STORE16(reinterpret_cast<float*>(d.dst) + e0, make_uint4(w[0], w[1], w[2], w[3]));
  else ADACC_STORE16(reinterpret_cast<uint16_t*>(d.dst) + e0, make_uint4(w[0], w[1], w[2], w[3]));
}

// What the kernels that call decompress_piece keep in LDS for every wavefront of the workgroup (17 KiB in all: eight
// workgroups of a CU, as many as its wavefronts allow, fit).
template <bool F32, int ROWS, int WAVES>
struct DecompressShared {
  uint4 picture[WAVES][piece_elems<F32, ROWS>() / 8];  // 16-bit patterns of the piece; its first words serve as the mailbox
  uint32_t bits[WAVES][kWave];                         // V bits per row: elements of lane l's chunk in that row that the picture holds
};

// floor(x / n) for x < 2^39 with the host's m = ceil(2^64 / n), 1 < n <= 2^11; m = 0 stands for n = 1
__device__ __forceinline__ uint64_t div_by_magic(uint64_t x, uint64_t m) { return m == 0ull ? x : __umul64hi(x, m); }

// The range [p0, p1) of the stream narrowed to the entries whose index lies in [first, end), or a little more: 64
// probes at a time.  Ends with at most 64 entries, or when a step no longer takes away a quarter.
__device__ __forceinline__ void narrow_entries(const TensorDesc& d, uint64_t first, uint64_t end, uint32_t& p0, uint32_t& p1) {
  const uint32_t lane = (uint32_t)__lane_id();
  while (p1 - p0 > (uint32_t)kWave) {  // uniform
    const uint32_t n = p1 - p0, step = (n + (uint32_t)kWave - 1u) / (uint32_t)kWave;
    const bool probes = lane * step < n;
    const uint64_t v = probes ? (uint32_t)d.idx[p0 + lane * step] : 0u;
    // probes ascend: those below `first` and those below `end` are the lowest lanes
    const uint32_t below = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(probes && v < first));
    const uint32_t upto = (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(probes && v < end));
    const uint32_t q0 = below != 0u ? p0 + (below - 1u) * step : p0;
    const uint32_t q1 = upto * step < n ? p0 + upto * step : p1;
    p0 = q0;
    p1 = q1 > q0 ? q1 : q0;
    if (p1 - p0 > n - n / 4u) break;
  }
}

template <int BITS, bool ASYM, bool F32, bool GENERIC, int ROWS, int WAVES>
__device__ __forceinline__ void decompress_piece(const TensorDesc& d, uint32_t piece, bool has_outliers, DecompressShared<F32, ROWS, WAVES>& shared) {
  constexpr int V = chunk_elems<F32>(), E = ROWS, W = kWave * V, kPiece = piece_elems<F32, ROWS>();  // W: elements of a row
  const int lane = (int)__lane_id();
  const uint64_t base = (uint64_t)piece * (uint64_t)kPiece;
  const uint64_t lane_base = base + (uint64_t)(lane * V);
  const bool complete = base + (uint64_t)kPiece <= d.numel;  // uniform; only a tensor's last piece can be short

  // group of a lane's chunk in row j
  const uint64_t first_oct = (uint64_t)piece * (uint64_t)(kPiece / kOct);
  uint64_t first_grp = 0ull;    // GENERIC: group of the piece's first octet ...
  uint32_t oct_in_grp = 0u;     // ... and that octet's number in it
  if constexpr (GENERIC) {
    first_grp = div_by_magic(first_oct, d.magic_q);
    oct_in_grp = (uint32_t)(first_oct - first_grp * (uint64_t)(d.gq >> 3));
  }
  auto group = [&](int j) -> uint64_t {
    if constexpr (GENERIC)
      return first_grp + (uint64_t)(uint32_t)((float)(oct_in_grp + ((uint32_t)(lane * V + j * W) >> 3)) * d.recip_q);
    else return (lane_base + (uint64_t)(j * W)) >> d.lgq;
  };

  // All loads of the piece are issued before anything waits for one of them: a complete piece
  // (every piece but possibly the last) has no branch between them.  The codes' address is formed once, the rows are
  // constant offsets from it.  (Formed from each row's element number, e0 * BITS / 8, whose product the compiler has to
  // take for one that may wrap, the addresses held the loads back: 12 tensors of 90 M int8 codes without outliers in a
  // batch took 568 us, 559 us like this.)
  const uint8_t* codes = d.codes + (BITS == 8 ? lane_base : lane_base >> 1);
  RowCodes<BITS, V> rc[E];
  if (complete) {
#pragma unroll
    for (int j = 0; j < E; ++j) load_row_codes<BITS, V, ASYM>(d, codes + j * W * BITS / 8, group(j), rc[j]);
  } else {
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const uint64_t e0 = lane_base + (uint64_t)(j * W);
      if (e0 + V <= d.numel) load_row_codes<BITS, V, ASYM>(d, codes + j * W * BITS / 8, group(j), rc[j]);
    }
  }

  // The slice of the outlier stream that belongs to the tiles of this piece, and its first 64 entries.  The entries
  // can only be asked for when the slice is known, a second round trip to memory behind the first - except for TOPK,
  // where every tile has k entries per group unless some group held more than k values that are not finite: there
  // the entries of that slice are asked for at once, together with the tiles' offsets, and are used if the offsets
  // turn out to be those.
  uint32_t t0 = 0u, t1 = 0u;  // uniform: tile_ptr[t0] .. tile_ptr[t1]
  if (has_outliers) {
    if constexpr (GENERIC) {
      t0 = (uint32_t)div_by_magic(first_oct, d.magic_t);
      t1 = (uint32_t)div_by_magic(first_oct + (uint64_t)(kPiece / kOct) - 1u, d.magic_t) + 1u;
      t1 = t1 < d.n_tiles_all ? t1 : d.n_tiles_all;
    } else {
      t0 = piece >> d.ptr_shift;  // (a short last group lies inside the last tile)
      t1 = t0 + 1u;
    }
  }
  const bool guess = has_outliers && d.mode == kModeTopk;  // uniform
  uint32_t g0 = 0u, g1 = 0u, o_idx = 0u, o_val = 0u;
  if (guess) {
    g0 = d.per_tile * t0;
    g1 = d.per_tile * t1;
    g0 = g0 < d.cap ? g0 : d.cap;
    g1 = g1 < d.cap ? g1 : d.cap;
    if (g0 + (uint32_t)lane < g1) {
      o_idx = (uint32_t)d.idx[g0 + (uint32_t)lane];
      o_val = d.val[g0 + (uint32_t)lane];
    }
  }
  uint32_t p0 = 0u, p1 = 0u;
  if (has_outliers) {
    // One address for the whole wavefront, so the scalar unit asks for it: the branches on the range below are then
    // branches (held per lane, the range made each of them a region under an execution mask), and the range does not
    // wait in line behind the codes.  With it the 12 tensors above took 552 us instead of 559.
    typedef const __attribute__((address_space(4))) uint32_t* ScalarWords;
    const ScalarWords ptr = (ScalarWords)(uintptr_t)d.tile_ptr;
    p0 = ptr[t0];
    p1 = ptr[t1];
    p0 = p0 < d.cap ? p0 : d.cap;
    p1 = p1 < d.cap ? p1 : d.cap;
    if (p1 < p0) p1 = p0;
  }
  bool fetched = guess && p0 == g0 && p1 == g1;  // uniform
  if constexpr (GENERIC) {
    if (p1 - p0 > (uint32_t)kWave) {  // uniform
      narrow_entries(d, base, base + (uint64_t)kPiece, p0, p1);
      fetched = false;
    }
  }
  const bool patch = p1 > p0;  // uniform over the wavefront
  if (patch && !fetched) {     // uniform
    o_idx = 0u; o_val = 0u;
    if (p0 + (uint32_t)lane < p1) {
      o_idx = (uint32_t)d.idx[p0 + (uint32_t)lane];
      o_val = d.val[p0 + (uint32_t)lane];
    }
  }

  // ---- a9 / a10: unpack, dequantise, take the outliers in, store
  if (complete && patch) {
    const uint32_t w = threadIdx.x / kWave;
    uint32_t rel = o_idx - (uint32_t)base;  // a tensor that keeps outliers has fewer than 2^31 elements
    bool valid = (uint32_t)lane < p1 - p0 && rel < (uint32_t)kPiece;  // also: not in the tile's other pieces
    // the stream is ascending, so two entries of one chunk are neighbours in it
    const uint32_t prev = (uint32_t)__shfl_up((int)(rel / V), 1, kWave);
    if (p1 - p0 <= (uint32_t)kWave && __builtin_amdgcn_ballot_w64(valid && lane != 0 && rel / V == prev) == 0ull) {  // uniform
      uint32_t(*box)[E] = reinterpret_cast<uint32_t(*)[E]>(shared.picture[w]);
#pragma unroll
      for (int j = 0; j < E; ++j) box[lane][j] = 0u;
      lds_in_order();
      if (valid) box[(rel / V) & 63u][rel / W] = kMailFull | ((rel % V) << 16) | (o_val & 0xFFFFu);
      lds_in_order();
      uint32_t m[E];
#pragma unroll
      for (int j = 0; j < E; ++j) m[j] = box[lane][j];
      lds_in_order();  // the next piece of this wavefront clears the mailbox only after this
#pragma unroll
      for (int j = 0; j < E; ++j)
        store_row_values<BITS, ASYM, F32>(d, lane_base + (uint64_t)(j * W), rc[j], MailPatch<F32>{m[j]});
      return;
    }
    uint16_t* picture = reinterpret_cast<uint16_t*>(shared.picture[w]);
    shared.bits[w][lane] = 0u;
    lds_in_order();
    for (uint32_t c = p0;;) {  // uniform
      if (valid) {
        picture[rel] = (uint16_t)o_val;
        atomicOr(&shared.bits[w][(rel / V) & 63u], 1u << (rel / W * V + rel % V));
      }
      c += (uint32_t)kWave;
      if (c >= p1) break;
      valid = c + (uint32_t)lane < p1;
      if (valid) {
        rel = (uint32_t)d.idx[c + (uint32_t)lane] - (uint32_t)base;
        o_val = d.val[c + (uint32_t)lane];
        valid = rel < (uint32_t)kPiece;
      }
    }
    lds_in_order();
    const uint32_t mine = shared.bits[w][lane];
#pragma unroll
    for (int j = 0; j < E; ++j) {
      const uint64_t e0 = lane_base + (uint64_t)(j * W);
      PicturePatch<F32> pic;
      pic.bits = (mine >> (V * j)) & ((1u << V) - 1u);
      if (__builtin_amdgcn_ballot_w64(pic.bits != 0u) != 0ull) {  // uniform
        // (what no entry was written to is not used)
        if constexpr (F32) {
          const uint2 v = reinterpret_cast<const uint2*>(shared.picture[w])[j * kWave + lane];
          pic.pat[0] = v.x; pic.pat[1] = v.y;
        } else {
          const uint4 v = shared.picture[w][j * kWave + lane];
          pic.pat[0] = v.x; pic.pat[1] = v.y; pic.pat[2] = v.z; pic.pat[3] = v.w;
        }
        store_row_values<BITS, ASYM, F32>(d, e0, rc[j], pic);
      } else {
        store_row_values<BITS, ASYM, F32>(d, e0, rc[j], NoPatch{});
      }
    }
    lds_in_order();
    return;
  }
  if (complete) {
#pragma unroll
    for (int j = 0; j < E; ++j) store_row_values<BITS, ASYM, F32>(d, lane_base + (uint64_t)(j * W), rc[j], NoPatch{});
    return;
  }

  // the tensor's last piece, not complete: whole chunks, then what is left of a ragged one, element by element
#pragma unroll
  for (int j = 0; j < E; ++j) {
    const uint64_t e0 = lane_base + (uint64_t)(j * W);
    if (e0 + V <= d.numel) {
      store_row_values<BITS, ASYM, F32>(d, e0, rc[j], NoPatch{});
    } else if (e0 < d.numel) {
      const uint64_t grp = group(j);
      const float s = d.scales[grp];
      for (uint64_t i = e0; i < d.numel; ++i) {
        int code;
        if constexpr (BITS == 8) code = (int)(int8_t)d.codes[i];
        else code = ((int)((uint32_t)d.codes[i >> 1] << (28u - 4u * (uint32_t)(i & 1ull)))) >> 28;
        float v = (float)code * s;
        if constexpr (ASYM) v = __fmaf_rn((float)code, s, d.zp[grp]);
        if constexpr (F32) reinterpret_cast<float*>(d.dst)[i] = v;
        else reinterpret_cast<uint16_t*>(d.dst)[i] = (uint16_t)narrow_pair(v, 0.0f);
      }
    }
  }
  // its outliers overwrite their positions
  if (patch) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the stores above are complete
    for (uint32_t cpos = p0 + (uint32_t)lane; cpos < p1; cpos += kWave) {
      if (cpos >= p0 + (uint32_t)kWave) {  // past the entries fetched at the start
        o_idx = (uint32_t)d.idx[cpos];
        o_val = d.val[cpos];
      }
      const uint64_t i = o_idx;
      if (i >= base && i < d.numel) {  // a damaged stream must not write outside the piece
        if constexpr (F32) reinterpret_cast<float*>(d.dst)[i] = widen_lo(o_val);
        else reinterpret_cast<uint16_t*>(d.dst)[i] = (uint16_t)o_val;
      }
    }
  }
}

}  // namespace ADACC_DT_NS
}  // namespace adacc
