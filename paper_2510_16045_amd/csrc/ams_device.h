// Device code that the Linear kernels share: the packed formats' lane records, their bit-level
// restoration to fp16 MFMA operands (Sec. 3.2, Sec. 3.3 stages 2-3), the kernels' arguments, and
// what the host's launch plans need to know of the kernels built in other files.
#ifndef AMS_DEVICE_H_
#define AMS_DEVICE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/ams.h"
#include "ams_layout.h"

namespace ams_dev {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u3 __attribute__((ext_vector_type(3)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
typedef unsigned short us4 __attribute__((ext_vector_type(4)));

constexpr int FMT_FP533 = AMS_FMT_FP533_E2M3;
constexpr int FMT_FP425 = AMS_FMT_FP425_E2M2;
constexpr int FMT_FP45 = AMS_FMT_FP45_E2M2;
constexpr int FMT_FP433 = AMS_FMT_FP433_E2M2;
constexpr int FMT_FP6 = AMS_FMT_FP6_E2M3;
constexpr int FMT_FP5 = AMS_FMT_FP5_E2M2;
constexpr int FMT_FP4 = AMS_FMT_FP4_E2M1;
constexpr int FMT_FP16 = 100;  // internal: unquantized row-major fp16 weights (baseline)
static_assert(FMT_FP533 == ams::kFmtFp533 && FMT_FP425 == ams::kFmtFp425 && FMT_FP45 == ams::kFmtFp45 &&
              FMT_FP433 == ams::kFmtFp433 && FMT_FP6 == ams::kFmtFp6 && FMT_FP5 == ams::kFmtFp5 && FMT_FP4 == ams::kFmtFp4, "format numbers");

constexpr float kTwo14 = 16384.0f;  // restored patterns are value * 2^-14

__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

__device__ __forceinline__ uint32_t pk_mul_u16(uint32_t a, uint32_t c) {
  us2 x = __builtin_bit_cast(us2, a), y = __builtin_bit_cast(us2, c);
  return __builtin_bit_cast(uint32_t, (us2)(x * y));
}

// e2m2 formats (Sec. 3.2): one 32-bit word = two half-words of four 4-bit remainders.
// sh[t] holds the last mantissa bits of pair t already placed at bits 8 and 24.
// Produces the four fp16 pairs (A_t low, B_t high) as bit patterns of value * 2^-14:
// sign -> bit 15, e1 e0 m1 -> bits 11..9, last bit m0 -> bit 8.
__device__ __forceinline__ void restore_e2m2(uint32_t s, const uint32_t sh[4], uint32_t out[4]) {
  constexpr uint32_t M = 0x8E008E00u;
  out[0] = bfi(M, s, sh[0]);
  out[1] = bfi(M, s << 3, sh[1]);
  // members 2 and 3: sign and magnitude need different shifts; a packed 16-bit
  // multiply by (2^a + 2^b) makes both shifted copies at once
  out[2] = bfi(M, pk_mul_u16(s & 0x40384038u, 0x00420042u), sh[2]);
  out[3] = bfi(M, pk_mul_u16(s & 0x20072007u, 0x02040204u), sh[3]);
}
// FP4.25: the four members of a half-word are one group, one pair of shared bits per word
__device__ __forceinline__ void restore_fp425(uint32_t s, uint32_t sh, uint32_t out[4]) {
  const uint32_t same[4] = {sh, sh, sh, sh};
  restore_e2m2(s, same, out);
}

// Last bits kept in a side byte: bit t belongs to pair t's A half, bit 4+t to its B half.
__device__ __forceinline__ uint32_t spread_side_byte(uint32_t byte) { return byte | (byte << 12); }
__device__ __forceinline__ uint32_t pair_bits_e2m2(uint32_t spread, int t) { return (spread << (8 - t)) & 0x01000100u; }

// e2m3 formats (Sec. 3.3 item 1): one 32-bit word = two half-words of three 5-bit
// remainders; sh0..sh2 hold the last bits of the three pairs at bits 7 and 23.
// Produces three fp16 pairs (A_i low, B_i high): sign -> bit 15, e1 e0 m2 m1 ->
// bits 11..8, last bit m0 -> bit 7.
__device__ __forceinline__ void restore_e2m3(uint32_t s, uint32_t sh0, uint32_t sh1, uint32_t sh2, uint32_t out[3]) {
  constexpr uint32_t M = 0x8F008F00u;
  out[0] = bfi(M, s, sh0);
  {
    // member 1: magnitude and sign need different shifts; the first half is spelled out (left to itself the compiler
    // makes two ands and a three-way or: one operation more).  The second half must stay the compiler's: an MFMA may
    // read a VALU result only two instructions later, which it sees to for its own instructions and not for assembly.
    uint32_t t;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(t) : "v"(s << 4), "s"(0x0F000F00u), "v"(sh1));
    out[1] = bfi(0x80008000u, s << 1, t);
  }
  out[2] = bfi(M, pk_mul_u16(s & 0x200F200Fu, 0x01040104u), sh2);
}
// FP5.33: each half-word is a whole group, its shared bit sits at bit 12
__device__ __forceinline__ void restore_fp533(uint32_t s, uint32_t out[3]) {
  const uint32_t sh = (s >> 5) & 0x00800080u;
  restore_e2m3(s, sh, sh, sh, out);
}

template <int FMT>
struct Fmt {
  static constexpr int REC_K = ams::kFormats[FMT].rec_k, REC_BYTES = ams::kFormats[FMT].rec_bytes,
                       CHUNK = ams::kFormats[FMT].chunk_bytes, SIDE = ams::kFormats[FMT].side_bytes,
                       PB = ams::kFormats[FMT].perm_block, N_MFMA = REC_K / 32,
                       SG = ams::side_group(ams::kFormats[FMT]),       // records per unit (a power of two)
                       CB = ams::chunk_block_bytes(ams::kFormats[FMT]),  // bytes of one record's lane chunks
                       UNIT = ams::unit_bytes(ams::kFormats[FMT]);
};
template <>
struct Fmt<FMT_FP16> {
  static constexpr int REC_K = 128, REC_BYTES = 0, CHUNK = 0, SIDE = 0, PB = 8, N_MFMA = 4, SG = 1, CB = 0, UNIT = 0;
};

// Input channel (inside its permutation block) of every operand slot of the block.
template <int FMT>
struct SlotChannel {
  int v[Fmt<FMT>::PB];
  constexpr SlotChannel() : v{} {
    for (int i = 0; i < Fmt<FMT>::PB; i++) v[i] = FMT == FMT_FP16 ? i : ams::slot_channel(FMT == FMT_FP16 ? 0 : FMT, i);
  }
};
template <int FMT>
__device__ constexpr int slot_channel(int s) {
  constexpr SlotChannel<FMT> tab{};
  return tab.v[s];
}

// The inverse: operand slot (inside its permutation block) of every input channel of the block.
template <int FMT>
__device__ constexpr int channel_slot(int j) {
  int s = 0;
  for (int i = 0; i < Fmt<FMT>::PB; i++)
    if (slot_channel<FMT>(i) == j) s = i;
  return s;
}

// What one lane holds of one record: the words of its chunk and, for formats with side bits,
// the lane's side dword of the record's unit (the record's own byte(s) are picked where it is restored).
template <int SIDE>
struct SideBits {
  uint32_t t;
};
template <>
struct SideBits<0> {};
template <int FMT>
struct LaneRec : SideBits<Fmt<FMT>::SIDE> {
  uint32_t w[Fmt<FMT>::CHUNK / 4];
};
template <>
struct LaneRec<FMT_FP16> {
  u4 w[4];
};

struct LinearArgs {
  const uint8_t* W;        // packed records, or row-major fp16 for the baseline
  const uint16_t* scales;  // [N] fp16, unused by the baseline
  const uint16_t* X;       // [M, K] fp16
  uint16_t* Y;             // [M, N] fp16
  int M, N, K;
  int n_rec;     // records per strip
  int x_stride;  // halfs between activation rows inside a wave's LDS region
  int x_region;  // halfs of one wave's LDS region
  int x_shift;   // log2 of the staging units per activation row, rounded up to a power of two
  int n_strips;  // strips of 16 output channels
  int spw;       // stream kernel: strips per workgroup
  int red_slots; // stream kernel: partial tiles a wave may park in LDS (strips its piece can touch)
  int piece_q, piece_r;  // stream kernel: pairs per wave in a full workgroup: quotient, remainder
  int rc;                // stream kernel: records per strip in one phase of K
  int n_sg, sg_shift;    // scales per run of input channels: runs per row, log2(records per run)
  // split of K over gk workgroups per strip (sweep kernel with a workspace): workgroups along N,
  // slices of K, per-slice partial tiles [gk][strip][MT][64] f4, per-strip arrival counters
  int gn, gk;
  int row_tiles, tile_rows;  // slice kernel: workgroups that share the rows of X, rows each of them takes (the last what is left)
  int wps;  // wavefronts that share a strip (sweep kernel: the workgroup works on S / wps strips at a time)
  int wpa;  // column kernel: how many of a strip's wps wavefronts take records (the others idle: a count that divides the work evenly)
  f4* ws_tiles;
  unsigned* ws_count;
};

// One lane's part of a record: its chunk at `chunks` (one dwordx4, or three dwords that the
// compiler merges) and its dword of the unit's side block at `side`.
template <int FMT, bool NT, bool WITH_SIDE = true>
__device__ __forceinline__ void load_lane_rec(LaneRec<FMT>& r, const uint8_t* chunks, const uint8_t* side, int lane) {
  constexpr int CHUNK = Fmt<FMT>::CHUNK, SIDE = Fmt<FMT>::SIDE;
  auto ld = [](auto* p) { return NT ? __builtin_nontemporal_load(p) : *p; };
  if constexpr (CHUNK == 16) {
    const u4 v = ld((const u4*)(chunks + lane * 16));
    r.w[0] = v[0], r.w[1] = v[1], r.w[2] = v[2], r.w[3] = v[3];
  } else {
    const uint32_t* p = (const uint32_t*)(chunks + lane * CHUNK);
#pragma unroll
    for (int d = 0; d < CHUNK / 4; d++) r.w[d] = ld(p + d);
  }
  // WITH_SIDE = false: the caller keeps the group's side dword elsewhere
  if constexpr (SIDE != 0 && WITH_SIDE) r.t = ld((const uint32_t*)side + lane);
}

// The MFMA A operands of one record as packed fp16 pairs: o[4u + t] = elements 2t, 2t+1
// of the lane's row in MFMA u (bit patterns of value * 2^-14).
// side_shift: first bit of this record's side bits inside the unit's side dword (wave-uniform).
template <int FMT>
__device__ __forceinline__ void restore_rec(const LaneRec<FMT>& r, int side_shift, uint32_t (&o)[4 * Fmt<FMT>::N_MFMA]) {
  if constexpr (FMT == FMT_FP533) {
#pragma unroll
    for (int d = 0; d < 4; d++) restore_fp533(r.w[d], &o[3 * d]);
  } else if constexpr (FMT == FMT_FP6) {
    // side bits: bit 2d + (i-1) = member i of half A of word d, the same + 8 for half B
    const uint32_t t = r.t >> side_shift;
    const uint32_t spread = (t & 0xFFu) | ((t & 0xFF00u) << 8);
#pragma unroll
    for (int d = 0; d < 4; d++)
      restore_e2m3(r.w[d], (r.w[d] >> 5) & 0x00800080u, (spread << (7 - 2 * d)) & 0x00800080u, (spread << (6 - 2 * d)) & 0x00800080u,
                   &o[3 * d]);
  } else if constexpr (FMT == FMT_FP425) {
    const uint32_t spread = spread_side_byte(__builtin_amdgcn_ubfe(r.t, (uint32_t)side_shift, 8u));
#pragma unroll
    for (int d = 0; d < 4; d++) restore_fp425(r.w[d], pair_bits_e2m2(spread, d), &o[4 * d]);
  } else if constexpr (FMT == FMT_FP4) {
    // an e2m1 code is an e2m2 remainder whose last bit is 0
    const uint32_t none[4] = {0, 0, 0, 0};
#pragma unroll
    for (int d = 0; d < 4; d++) restore_e2m2(r.w[d], none, &o[4 * d]);
  } else {
    // FP4.33: one side byte for all words; FP4.5: one per two words; FP5: one per word
    constexpr int WORDS_PER_BYTE = FMT == FMT_FP433 ? 3 : (FMT == FMT_FP45 ? 2 : 1);
    const uint32_t t = Fmt<FMT>::SIDE == 4 ? r.t : __builtin_amdgcn_ubfe(r.t, (uint32_t)side_shift, (uint32_t)(8 * Fmt<FMT>::SIDE));
    uint32_t sh[4];
#pragma unroll
    for (int d = 0; d < Fmt<FMT>::CHUNK / 4; d++) {
      if (d % WORDS_PER_BYTE == 0) {
        const uint32_t spread = spread_side_byte(Fmt<FMT>::SIDE == 1 ? t : (t >> (8 * (d / WORDS_PER_BYTE))) & 0xFFu);
#pragma unroll
        for (int i = 0; i < 4; i++) sh[i] = pair_bits_e2m2(spread, i);
      }
      restore_e2m2(r.w[d], sh, &o[4 * d]);
    }
  }
}

// Unconditional loads of one record (rec must be a valid record of the strip).  NT: packed
// records bypass the caches' retention (they are read once per call, and a model's other
// layers pass through the caches before the next call); only tiny matrices use ordinary loads.
template <int FMT, bool NT = true>
__device__ __forceinline__ void load_rec(LaneRec<FMT>& r, const LinearArgs& a, int strip, int rec, int lane) {
  if constexpr (FMT == FMT_FP16) {
    // rows beyond N and K-chunks beyond K are redirected to the matrix's first 16 bytes
    // and zeroed afterwards: keeps the loads free of control flow
    const int row = strip * 16 + (lane & 15);
    const int kq = lane >> 4;
#pragma unroll
    for (int d = 0; d < 4; d++) {
      const int k = rec * 128 + 32 * d + 8 * kq;
      const bool ok = row < a.N && k < a.K;  // K is a multiple of 8
      const size_t off = ok ? ((size_t)row * a.K + k) * 2 : 0;
      const u4 v = *(const u4*)(a.W + off);  // cached: the two halves of a 128-byte line come from two loads
      const uint32_t keep = ok ? 0xFFFFFFFFu : 0u;
      r.w[d] = u4{v[0] & keep, v[1] & keep, v[2] & keep, v[3] & keep};
    }
  } else {
    // unit (rec / SG, strip) of the K-major packed matrix, record rec % SG inside it
    constexpr int SG = Fmt<FMT>::SG;
    const uint8_t* unit = a.W + ((size_t)((unsigned)rec / SG) * (unsigned)a.n_strips + (unsigned)strip) * Fmt<FMT>::UNIT;
    load_lane_rec<FMT, NT>(r, unit + ((unsigned)rec % SG) * Fmt<FMT>::CB, unit + SG * Fmt<FMT>::CB, lane);
  }
}

// Multiply one record (16 rows x REC_K) into the accumulators.  x0 / x1 point at this
// lane's activation row(s) in LDS at the first operand slot of its K-quarter of the record.
// side_shift: see restore_rec (8 * SIDE * (rec % SG); 0 for formats without side bits).
template <int FMT, int MT>
__device__ __forceinline__ void mac_rec(const LaneRec<FMT>& r, const _Float16* x0, const _Float16* x1, f4 acc[MT], int side_shift = 0) {
  h8 a[Fmt<FMT>::N_MFMA];
  if constexpr (FMT == FMT_FP16) {
#pragma unroll
    for (int d = 0; d < 4; d++) a[d] = __builtin_bit_cast(h8, r.w[d]);
  } else {
    uint32_t o[4 * Fmt<FMT>::N_MFMA];
    restore_rec<FMT>(r, side_shift, o);
#pragma unroll
    for (int u = 0; u < Fmt<FMT>::N_MFMA; u++) a[u] = __builtin_bit_cast(h8, u4{o[4 * u], o[4 * u + 1], o[4 * u + 2], o[4 * u + 3]});
  }
#pragma unroll
  for (int u = 0; u < Fmt<FMT>::N_MFMA; u++) {
    // FP16 records interleave the K-quarters per MFMA (32 consecutive k each)
    const int off = FMT == FMT_FP16 ? 32 * u : 8 * u;
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u], *(const h8*)(x0 + off), acc[0], 0, 0, 0);
    if constexpr (MT == 2) acc[1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[u], *(const h8*)(x1 + off), acc[1], 0, 0, 0);
  }
}

// Operand slot of activation k (relative to its record) in LDS.
template <int FMT>
__device__ __forceinline__ int x_slot(int kk) {
  if constexpr (FMT == FMT_FP16) {
    return kk;
  } else {
    constexpr int PB = Fmt<FMT>::PB;
    const int blk = kk / PB, j = kk - blk * PB;
    int slot = 0;
    for (int s = 0; s < PB; s++)
      if (slot_channel<FMT>(s) == j) slot = s;
    return blk * PB + slot;
  }
}

// dword made of half `ia` (low) and half `ib` (high) of an array of packed half pairs
__device__ __forceinline__ uint32_t pick2(const uint32_t* in, int ia, int ib) {
  const uint32_t sel = (uint32_t)(2 * (ia & 1)) | (uint32_t)(2 * (ia & 1) + 1) << 8 | (uint32_t)(4 + 2 * (ib & 1)) << 16 |
                       (uint32_t)(5 + 2 * (ib & 1)) << 24;
  return __builtin_amdgcn_perm(in[ib >> 1], in[ia >> 1], sel);
}

// One permutation block of activations from input-channel order into operand order
// (packed pairs in, packed pairs out).
template <int FMT>
__device__ __forceinline__ void permute_unit(const uint32_t (&in)[Fmt<FMT>::PB / 2], uint32_t (&out)[Fmt<FMT>::PB / 2]) {
#pragma unroll
  for (int m = 0; m < Fmt<FMT>::PB / 2; m++) {
    if constexpr (FMT == FMT_FP16)
      out[m] = in[m];
    else
      out[m] = pick2(in, slot_channel<FMT>(2 * m), slot_channel<FMT>(2 * m + 1));
  }
}

// Eight halfs (packed pairs) moved down by n places with zeros behind (n <= 0: as they are; n >= 8 does not matter,
// such a chunk lies beyond K and is zero already).
__device__ __forceinline__ void shift_tail(uint32_t* v, int n) {
  n = max(n, 0);
  if (n & 4) v[0] = v[2], v[1] = v[3], v[2] = 0, v[3] = 0;
  if (n & 2) v[0] = v[1], v[1] = v[2], v[2] = v[3], v[3] = 0;
  if (n & 1) {
    v[0] = v[0] >> 16 | v[1] << 16, v[1] = v[1] >> 16 | v[2] << 16;
    v[2] = v[2] >> 16 | v[3] << 16, v[3] = v[3] >> 16;
  }
}

constexpr int kLdsMaxBytes = 160 * 1024;  // LDS of a gfx950 compute unit
constexpr int kOutOfRange = 0x7FFE0000;   // an offset beyond the range of every buffer: such a lane's load reads no memory and gives 0
constexpr int kDeviceScope = 16;          // cache policy (sc1) of a buffer load or store that the whole device sees
constexpr int kMaxSlices = 8;             // slices of K that workgroups may share

// ---- slice_kernel (ams_slice.hip): what its launch needs ------------------------------------------
// Variants: one scale per row of W; one per run of input channels; rows of X that are not 16-byte aligned; one scale per row, or per
// run, and more asked for ahead.
constexpr int kSlicePlain = 0, kSliceRunScales = 1, kSliceRagged = 2, kSliceDeep = 3, kSliceDeepRuns = 4, kSliceVariants = 5;
constexpr int kSliceRaggedMaxStrips = 4, kSliceRaggedMaxRows = 8;  // of kSliceRagged
// Whether there is a kernel of the last two for `rows` staged rows and `strips` strips (where they are taken: more_ahead_is_faster).
constexpr bool slice_has_deep(int fmt, int variant, int rows, int strips) {
  const bool rec96 = ams::kFormats[fmt].rec_k == 96;
  if (strips != 1) return false;
  return variant == kSliceDeepRuns ? rows == 16 && !rec96 : (rows == 4 && ams::side_group(ams::kFormats[fmt]) == 1) || rows == 16;
}
constexpr int kSliceMaxStrips = 8;  // strips per workgroup it is built for
constexpr int slice_rows(int M) { return M <= 4 ? 4 : M <= 8 ? 8 : M <= 16 ? 16 : 32; }  // staged activation rows
// Wavefronts of a workgroup and what each of them asks for ahead of its work.  A compute unit keeps about 32 KiB of
// requests in flight, in order: what is asked for beyond that does not come sooner, it only stands before another
// wavefront's next record, activations before weights and the other way round.  So a wavefront asks for little: one record of
// activations ahead (not two), and weights one to three (record, strip) pairs ahead.  us, two records of activations and two or
// three pairs of weights ahead (before) / here: 4096 x 14336 FP4.25 M = 4 8.9 / 8.0, M = 16 12.7 / 11.5, M = 32 15.8 / 14.5; 8192 x
// 28672 FP5.33 M = 8 29.4 / 28.4, M = 16 37.2 / 34.9; 6144 x 4096 FP4.25 M = 8 5.9 / 5.4; 28672 x 4096 FP4.25 M = 32 17.0 /
// 15.9; four records of activations ahead instead of two 0.93-1.0 x, six pairs of weights 0.89-1.02 x.
struct SliceAsk {
  int waves;    // wavefronts of the workgroup
  int streams;  // of them, those that take records; the others help with the sum at the end
  int weights;  // (record, strip) pairs of weights asked for ahead
  int acts;     // records of activations asked for ahead
  int behind;   // strips of a record whose weights are asked for before the next record's activations
};
constexpr SliceAsk slice_ask(int fmt, int R, int NS, int variant) {
  const bool rec96 = ams::kFormats[fmt].rec_k == 96, runs = variant == kSliceRunScales, loads2 = ams::kFormats[fmt].side_bytes != 0 || runs;
  // Unaligned rows come through registers, one record ahead and one pair of weights on one strip.  Against two records and two pairs,
  // seven formats: 5 to 8 rows 1.18 x on one strip, 1.12 on two, 1.08 on three and four (11003 x 4099 FP5.33 M = 5 8.8 / 8.1 us, 4096 x 14339
  // M = 8 14.9 / 12.7); up to four rows 1.07, 1.03, 1.02, 1.01 (twelve streams of 96-weight records 0.94-0.97 x on two strips).
  if (variant == kSliceRagged) return {16, R == 4 && NS == 2 && loads2 && !rec96 ? 12 : 16, NS == 1 ? 1 : 2, 1, 0};
  if (variant >= kSliceDeep) return R == 4 ? SliceAsk{16, 16, 2, 2, 0} : SliceAsk{8, 8, rec96 ? 2 : 1, 2, 0};
  if (NS == 1) {
    // One strip: many wavefronts that each wait for one record (4096 x 9728 FP4.25 M = 1, sixteen with two records ahead / with
    // one / twelve / eight with two: 1.00 / 1.10 / 1.02 / 1.03 x; two of both only as kSliceDeep).  Up to eight rows eight stay, two ahead of both (one ahead
    // 0.88-1.0 x of it); up to sixteen rows twelve stream (FP4.25 1.05-1.16 x, FP5.33 M = 9 to 15 1.02-1.07 x but for
    // kSliceDeep's 16 to 36 records), but for 96-weight records with a scale per run (11 to 28 records 1.01-1.08 x, twelve 0.96-1.01 x;
    // those of 128 as kSliceDeepRuns).
    if (R == 4) return {16, 16, 1, 1, 0};
    if (R == 8) return {8, 8, 2, 2, 0};
    if (R == 16) return rec96 && runs ? SliceAsk{8, 8, 1, 2, 0} : SliceAsk{16, 12, 1, 1, 0};
    return {8, 8, 1, 1, 0};
  }
  // Two strips: the next record's.  At M <= 4 sixteen wavefronts, of which twelve stream where a record takes more than one load
  // (its side dword, its scales): 6144 x 4096 FP4.25 M = 1 eight / twelve / sixteen 1.02 / 1.09 / 1.04 x the time before, 8192 x
  // 28672 FP5.33 M = 1 0.98 (twelve) / 1.03 x (sixteen), 6144 x 4096 1.05 / 1.05.
  if (NS == 2) return R == 4 ? SliceAsk{16, loads2 ? 12 : 16, 2, 1, 0} : SliceAsk{8, 8, 2, 1, 0};
  // More strips keep a wavefront busy for longer than a trip to the L2: the next activations are asked for shortly before the
  // record ends (28672 x 4096 M = 32 FP4.25 at its start / before the last strip but one: 15.9 / 15.5; 20480 x 4096 M = 16 1.04 /
  // 1.07 x).  Up to eight rows earlier: at the end of a short stream the last request is one for nothing and waited for (K = 1024
  // and less, M <= 8: 0.99 x before the last strip but one, 1.02 x behind the first).
  return {8, 8, 3, 1, R > 8 ? NS - 2 : NS >= 5 ? 1 : 0};
}
// 1 KiB loads that bring one record's activations
constexpr int slice_x_loads(int fmt, int R) {
  const int rb = R > 16 ? 16 : R, pieces = (ams::kFormats[fmt].rec_k / 8 + 3) / 4 * 4;
  return (rb * pieces + 63) / 64 * (R > 16 ? 2 : 1);
}
// floats between the rows of a partial tile in LDS: 20 keeps a column's float4s in different banks, where it fits
constexpr int slice_tile_row(int S, int R, int NS) { return S * NS * R * 20 * 4 <= 150 * 1024 ? 20 : 16; }
// Floats between the tiles of neighbouring strips.  The final sum reads four strips at a time, 64 bytes of each: from 16 rows on
// they would all lie in the same banks (28672 x 4096 FP5.33 M = 32 19.2 -> 18.9 us; up to eight rows two at a time, no gain).
constexpr int slice_tile_strip(int S, int R, int NS) { return R * slice_tile_row(S, R, NS) + (NS > 1 && R >= 16 ? 16 : 0); }
// LDS of one wavefront: its records of activations and, when its stream has ended, its partial tiles in the same place.  It
// leaves them as soon as it is done itself, without a barrier (28672 x 4096 FP4.25 M = 16 14.0 -> 13.7, M = 32 17.8 -> 17.5).
constexpr int slice_wave_lds(int fmt, int R, int NS, int variant) {
  const SliceAsk a = slice_ask(fmt, R, NS, variant);
  const int staged = a.acts * slice_x_loads(fmt, R) * 1024, tiles = NS * slice_tile_strip(a.streams, R, NS) * 4;
  return staged > tiles ? staged : tiles;
}
constexpr int slice_lds(int fmt, int R, int NS, int variant) { return slice_ask(fmt, R, NS, variant).streams * slice_wave_lds(fmt, R, NS, variant) + NS * 64 + NS * 4; }
// Whether two workgroups of `strips` strips fit on a compute unit at M <= 4 with one scale per run of input channels: at
// most 128 registers (as the compiler reports them; the formats of 96 weights per record take 125 at most, FP4.25, FP4.5
// and FP5 124 with six strips and 136 with seven, FP4 128 with seven and 131 with eight).
constexpr bool slice_two_fit(int fmt, int strips) {
  return ams::kFormats[fmt].rec_k == 96 || strips <= (fmt == FMT_FP4 ? 7 : 6);
}
// Its arguments but for those that are needed before the first request: those are 14 plain dwords, which the build has
// preloaded into scalar registers (with the address of one struct instead, every wavefront of a launch starts with a trip
// to memory: 4096 x 4096 at M = 12 5.84 us, preloaded 5.69; 256 x 768 2.84, 2.78).  Four vector parameters rather than eleven
// scalars and pointers: the host pays for every parameter of a launch.
struct SliceArgs {
  uint16_t* Y;
  f4* ws_tiles;
  unsigned* ws_count;
  int n_sg, sg_shift;
  int row_tiles;  // = gridDim.y, which would bring the runtime's hidden arguments into every launch
};
// The kernel for `rows` staged rows and `strips` strips per workgroup (nullptr: there is none).
template <int FMT, int VARIANT>
const void* slice_kernel_of(int rows, int strips);

}  // namespace ams_dev
#endif
